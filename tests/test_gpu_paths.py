"""GPU tests of single kernels and dispatch branches at the sizes where they can go wrong
(edges of tiles, remainders, both sides of a rule), against the oracle or plain torch."""
import numpy as np
import pytest
import torch

from _gpu import Pair, gpu_step, host_weights, oracle_step
from oracle import Oracle, group_by_route
from paper_2606_09514_amd import lib as blib
from paper_2606_09514_amd import synth
from perf import cases
from test_gpu_parity import check_prefill, gpu_prefill, gqa_shape, one_step_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", ["hd128-32", "hd128-33", "hd64-32", "hd64-33", "hd128-G1-70"])
def test_chunk_merge_widths(case):
    """The chunk merge on both sides of its wide launch (32 and 33 chunks; 128-row chunks for
    head_dim 128, 256-row ones for head_dim 64), with as many thread groups as the head
    dimension leaves, and a last chunk of a single row (the odd chunk counts)."""
    hd64, n = case.startswith("hd64"), int(case.split("-")[-1])
    per = 256 if hd64 else 128
    T = per * 32 if n == 32 else per * (n - 1) + 1
    shape = dict(synth.SHAPES["tiny"], n_layers=4) if hd64 else gqa_shape(1 if "G1" in case else 4)
    P = Pair(shape, "bf16", T, 1, seed=200 + n, omega=0.1)
    g = torch.Generator().manual_seed(201)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    x = synth.hidden_inputs(1, P.cfg["d_model"], seed=202).numpy()
    print(case, one_step_all(P, hk, hv, [T - 1], [1], x))


@pytest.mark.parametrize("B,n", [(63, 64), (64, 65), (255, 128), (256, 129), (257, 64), (511, 65), (1000, 255)])
def test_group_widths(B, n):
    """Path grouping at the edges of its word counts (64 blocks a word), of a wavefront's and
    of the one-workgroup launch's sequences; starts past the last group stay untouched."""
    rng = np.random.default_rng(B + n)
    m = rng.integers(0, 2, size=(max(1, B // 3), n)).astype(np.uint8)[rng.integers(0, max(1, B // 3), size=B)]
    m[B // 2:, : n - 1] = m[0, : n - 1]   # long runs of routes that differ in the last block only
    m = np.ascontiguousarray(m * 200)
    perm = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    starts = torch.full((B + 1,), -7, dtype=torch.int32, device="cuda")
    ng = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    blib.group_by_route(torch.from_numpy(m).cuda(), perm, starts, ng)
    ref_perm, ref_starts = group_by_route(m)
    g = int(ng.item())
    assert g == len(ref_starts) - 1
    assert np.array_equal(perm.cpu().numpy(), ref_perm)
    assert np.array_equal(starts.cpu().numpy(), np.concatenate([ref_starts, np.full(B - g, -7)]))


@pytest.mark.parametrize("B", [3, 4])
def test_small_batch_rule(B):
    """Both sides of the rule that takes batches of two to four sequences to the MFMA path
    (rows x weight bytes of a block: 159 MB here, 478 and 637 MB), blocks routed by one to
    all sequences.  Both keep fp32 activations: the same bound."""
    shape = dict(n_layers=5, d_model=2048, n_heads=16, n_kv_heads=4, head_dim=128, d_ffn=11264,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    T = 200
    P = Pair(shape, "bf16", T, B, seed=220, omega=0.1)
    g = torch.Generator().manual_seed(221)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    x = synth.hidden_inputs(B, 2048, seed=222).numpy()
    rep = one_step_all(P, hk, hv, [T - 1, 150, 60, 199][:B], [1, 3, 2, 0][:B], x)
    print(B, rep)
    assert rep["max_hidden_err"] < 1e-5


@pytest.mark.parametrize("B", [5, 6, 8, 9])
def test_packed_activation_parts(B):
    """The batches at the edges of the activation layouts: three parts (24 bits) packed up to
    5 sequences, two packed up to 8, split tiles beyond; K-split O and down projections,
    deferred sums, rows that a block does not route.  A misplaced part leaves bf16's 8 bits
    (errors of 1e-3); with 24 bits the hidden state is 1e-7 to 2e-7 off, with 16 about 5e-7:
    ten times that is allowed."""
    shape = dict(n_layers=6, d_model=256, n_heads=4, n_kv_heads=1, head_dim=128, d_ffn=1024,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    T = 600
    P = Pair(shape, "bf16", T, B, seed=210, omega=0.1)
    g = torch.Generator().manual_seed(211 + B)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    pos = [T - 1 - 37 * b for b in range(B)]
    ks = [b % (P.L_mid + 1) for b in range(B)]
    x = synth.hidden_inputs(B, 256, seed=212).numpy()
    rep = one_step_all(P, hk, hv, pos, ks, x)
    print(B, rep)
    assert rep["max_hidden_err"] < (2e-6 if B <= 5 else 5e-6)


@pytest.mark.parametrize("B,f", [(2, 11264), (5, 1024), (5, 1152), (5, 640), (8, 1152)])
def test_infinite_weights_small_batches(B, f):
    """Infinite weights in small batches, whose activations enter the MFMA in two or three parts: a
    part of 0 times infinity must not turn the sum into NaN.  One infinite weight in every row of
    the last down projection gives plus or minus infinity, as the oracle's sums do (K of whole and
    half rounds of k-steps; 2 sequences past the rule that takes them to the MFMA)."""
    d = 4096 if B == 2 else 256
    shape = dict(n_layers=3, d_model=d, n_heads=d // 128, n_kv_heads=1 if d == 256 else 8, head_dim=128, d_ffn=f,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    T = 40
    P = Pair(shape, "bf16", T, B, seed=270, omega=0.1, device_gen=d > 256)
    rows = torch.arange(d, device="cuda")
    P.Wd["layers"][-1]["wdown"][rows, rows * 7 % f] = float("inf")
    P.orc = Oracle(P.cfg, *host_weights(P.Wd))
    g = torch.Generator().manual_seed(271)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    x = synth.hidden_inputs(B, d, seed=272).numpy()
    dk, dv = P.upload(hk.copy()), P.upload(hv.copy())
    got, mask, _ = gpu_step(P, dk, dv, x, [T - 1] * B, [1] * B)
    for b in range(B):
        ref = np.asarray(oracle_step(P, hk, hv, b, T - 1, 1, x[b], route=mask[b])[0])
        assert np.all(np.isinf(ref))
        assert np.array_equal(got[b], ref.astype(np.float32)), (b, int(np.isnan(got[b]).sum()))


@pytest.mark.parametrize("B", [1, 2, 17])
def test_infinite_router_weights(B):
    """An infinite weight of the router's first layer: infinite scores, as the oracle's.  The
    hidden value it meets has no remainder beyond bf16, whose product with infinity is NaN."""
    shape = dict(n_layers=6, d_model=96, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=128,
                 dm_hidden=40, dm_act="gelu", rope_theta=1e4, rms_eps=1e-5)
    T = 30
    P = Pair(shape, "bf16", T, B, seed=280, omega=0.1)
    P.Wd["dm"]["w1"][33, -5] = float("inf")
    P.orc = Oracle(P.cfg, *host_weights(P.Wd))
    g = torch.Generator().manual_seed(281)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    h = synth.hidden_inputs(B, 96, seed=282)
    h[:, -5] = 1.5
    scores = torch.zeros((B, P.L_mid), device="cuda")
    P.gpu.pool_route(P.upload(hk), P.upload(hv), [T - 1] * B, h.cuda(), scores)
    got = scores.cpu().numpy()
    for b in range(B):
        ref = np.asarray(P.orc.dm_scores(P.orc.context(hk[0, b], hv[0, b], T - 1, h[b].numpy())))
        assert np.all(np.isinf(ref))
        assert np.array_equal(got[b], ref.astype(np.float32)), (b, got[b], ref)


@pytest.mark.parametrize("B,H,ctx,d,T", [(2, 8, "kv", 96, 40), (2, 136, "k+v", 96, 3000), (16, 128, "k", 3936, 70),
                                         (17, 264, "v", 608, 500), (33, 4096, "kv", 352, 90), (3, 4104, "kv", 352, 90),
                                         (3, 64, "kv", 232, 90), (1, 64, "kv", 96, 90)])
def test_router_first_layer(B, H, ctx, d, T):
    """The Decision Module's first layer on the MFMA at the edges of its tiles (units, sequences,
    K slices and k-steps that do not divide, one to 24 pool splits per row), and the sizes that stay on
    the GEMV: hidden widths past the router kernel's LDS, inputs that are not whole k-steps, one
    sequence.  fp32 context on both: the scores' 1e-5; the entry point without a handle gives
    the same bits."""
    shape = dict(n_layers=6, d_model=d, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=128,
                 dm_hidden=H, dm_act="gelu", rope_theta=1e4, rms_eps=1e-5, router_ctx=ctx)
    P = Pair(shape, "bf16", T, B, seed=230, omega=0.1)
    g = torch.Generator().manual_seed(231)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    dk, dv = P.upload(hk), P.upload(hv)
    h = synth.hidden_inputs(B, d, seed=232)
    pos = [(T - 1 - 13 * b) % T for b in range(B)]
    scores, again = (torch.zeros((B, P.L_mid), device="cuda") for _ in range(2))
    P.gpu.pool_route(dk, dv, pos, h.cuda(), scores)
    blib.pool_route_noalloc(P.cfg, P.Wd["dm"], B, dk, dv, pos, h.cuda(), again)
    got = scores.cpu().numpy()
    assert np.array_equal(got, again.cpu().numpy())
    for b in range(B):
        ref = P.orc.dm_scores(P.orc.context(hk[0, b], hv[0, b], pos[b], h[b].numpy()))
        assert np.max(np.abs(got[b] - ref)) <= 1e-5 * max(1.0, float(np.max(np.abs(ref)))), b


@pytest.mark.parametrize("lens", [[64], [127], [129], [200, 57], [300, 215], [900, 90]])
def test_prefill_short_prompts(lens):
    """The tiled GEMM's automatic choices for short prompts: 128 x 128, 128 x 256 and
    256 x 256 tiles with K split up to eight ways for every kind of projection (rotary and
    cache append, SwiGLU, residual add behind the split sums), ragged last tiles, blocks run
    by one prompt only.  Against the oracle, and against the unsplit 128 x 128 tile: the same
    products summed in another order, each then rounded to bf16 for the next projection
    (2^-9 a rounding; 1e-2 of the largest output allowed)."""
    shape = dict(n_layers=4, d_model=1024, n_heads=8, n_kv_heads=2, head_dim=128, d_ffn=2304,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    T = max(lens)
    P = Pair(shape, "bf16", T, len(lens), seed=240, omega=0.1)
    ks = [1, 2][:len(lens)]
    if T <= 300:
        check_prefill(P, lens, ks, T, seed=241)
    auto = gpu_prefill(P, lens, ks, T, seed=241)
    P.gpu.set_gemm_tile(blib.GEMM_TILE_128)
    plain = gpu_prefill(P, lens, ks, T, seed=241)
    assert np.array_equal(auto[1], plain[1])
    for b, n in enumerate(lens):
        a, p = auto[0][b, :n], plain[0][b, :n]
        assert np.max(np.abs(a - p)) <= 1e-2 * np.max(np.abs(p))


def test_prefill_split_and_tail_columns():
    """A down projection of 257 to 384 tiles of 256 x 256 (16 x 17 here) over a deep K: the
    automatic choice splits K, and the tile's last, partly filled round must then stay with the
    first launch, for the split sums of every weight row are added behind it.  An earlier prefill of
    the handle, split without a tail, has left its sums in the partial buffer.  Every hidden column
    against the unsplit 128 x 128 tile: the sums differ in their order only, and what the next
    projections read is rounded to bf16 (2^-9 a value): 1e-2 of a column's norm is allowed, sums
    added twice or out of an older call are of the column's own size."""
    n = 4100
    shape = dict(n_layers=3, d_model=4096, n_heads=8, n_kv_heads=2, head_dim=128, d_ffn=14336,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    cfg = synth.model_config(shape, "bf16", n)
    model = blib.Model(cfg, synth.model_weights(cfg, 250, "cuda", omega=0.1), max_batch=1)
    k, v = synth.kv_cache(cfg, 1, 0, 251, "cuda")
    gen = torch.Generator(device="cuda").manual_seed(252)
    x, other = (torch.randn((1, n, 4096), generator=gen, device="cuda") for _ in range(2))

    def prefill(inp, tile):
        model.set_gemm_tile(tile)
        hidden = inp.clone()
        model.prefill(k, v, hidden, [n], [1])
        return hidden[0].double()

    plain = prefill(x, blib.GEMM_TILE_128)
    for tile in (blib.GEMM_TILE_AUTO, blib.GEMM_TILE_256_SPLIT):
        prefill(other, blib.GEMM_TILE_256_SPLIT)
        err = (prefill(x, tile) - plain).norm(dim=0) / plain.norm(dim=0)
        print(tile, float(err.max()), flush=True)
        assert float(err.max()) < 1e-2, (tile, int(err.argmax()))


def test_prefill_same_bits_after_a_longer_prompt():
    """The K splits of a prompt's projections follow from its own tokens: the partial buffer that
    an earlier, longer prompt left on the handle must not allow more of them (gate/up of 150
    tokens at this width would be split in two there, which its own buffer has no room for)."""
    n, long = 150, 1100
    shape = dict(n_layers=3, d_model=4096, n_heads=8, n_kv_heads=2, head_dim=128, d_ffn=14336,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    cfg = synth.model_config(shape, "bf16", long)
    model = blib.Model(cfg, synth.model_weights(cfg, 260, "cuda", omega=0.1), max_batch=1)
    k, v = synth.kv_cache(cfg, 1, 0, 261, "cuda")
    gen = torch.Generator(device="cuda").manual_seed(262)
    x, other = (torch.randn((1, t, 4096), generator=gen, device="cuda") for t in (n, long))

    def prefill(inp):
        hidden = inp.clone()
        model.prefill(k, v, hidden, [inp.shape[1]], [1])
        return [hidden] + [c[:, :, :, :n].clone() for c in (k, v)]

    fresh = prefill(x)
    prefill(other)
    assert all(torch.equal(a, b) for a, b in zip(fresh, prefill(x)))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_prefill_workspace_follows_the_model(dtype):
    """The prefill workspace of a small model: 512 prompt rows of a few hundred values.  Its split
    sums are those its projections can use (none in fp32, two splits of the residual adds in
    bf16), not a wide model's 49152 floats a row (100 MB)."""
    n = 512
    cfg = synth.model_config("tiny", dtype, n)
    model = blib.Model(cfg, synth.model_weights(cfg, 290, "cuda", omega=0.1), max_batch=1)
    k, v = synth.kv_cache(cfg, 1, 0, 291, "cuda")
    hidden = torch.randn((1, n, cfg["d_model"]), device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    model.prefill(k, v, hidden, [n], [1])
    grown = free - torch.cuda.mem_get_info()[0]
    row = 4 * (2 * cfg["n_heads"] * cfg["head_dim"] + 3 * cfg["d_ffn"] + 4 * cfg["d_model"])
    print(dtype, grown, n * row)
    assert grown <= 4 * n * row + (8 << 20)


@pytest.mark.parametrize("G,nkv,pos", [(4, 8, [6599, 40, 0, 900, 130, 6000]), (1, 16, [5200, 5, 700, 5199]),
                                       (2, 30, [3000, 64, 63, 128, 500, 1, 999]), (4, 12, [3299, 3290, 3280, 3150])])
def test_uneven_lengths(G, nkv, pos):
    """Decode over lengths on both sides of the rule for uneven ones (the mean under 9/10 of the
    longest: 13, 10 and 5 chunks where even lengths have 10, 8 and 2; the short sequences have rows
    in the first only)."""
    T = max(pos) + 1
    P = Pair(dict(gqa_shape(G), d_model=512, n_heads=G * nkv, n_kv_heads=nkv), "bf16", T, len(pos), seed=300, omega=0.1)
    g = torch.Generator().manual_seed(301)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    x = synth.hidden_inputs(len(pos), P.cfg["d_model"], seed=302).numpy()
    print(pos, one_step_all(P, hk, hv, pos, [b % (P.L_mid + 1) for b in range(len(pos))], x))


def attention_us(model, layer, k, v, hidden, pos):
    """Time of a block's attention score kernel in steps with a budget of 1, microseconds."""
    hip = blib.HipEvents()
    st, sp = hip.create(12), hip.create(12)
    model.set_timing_events(blib.KERNEL_ATTENTION, layer, st, sp)
    for _ in range(12):
        model.decode_step(k, v, hidden[:len(pos)].clone(), pos, [1] * len(pos))
    torch.cuda.synchronize()
    us = sorted(1e3 * hip.elapsed_ms(a, b) for a, b in zip(st, sp))
    hip.destroy(st + sp)
    return us[3]


def test_one_long_sequence_in_a_batch():
    """One sequence of 16000 rows beside 23 of 100: the attention kernel may take a few times what
    it takes for the long one alone (shared out in 32 chunks, here in 11).  With the two chunks that
    24 such sequences of equal length have, it takes about nine times as long."""
    B, T = 24, 16001
    shape = dict(n_layers=3, d_model=1024, n_heads=32, n_kv_heads=8, head_dim=128, d_ffn=512,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    cfg = synth.model_config(shape, "bf16", T)
    model = blib.Model(cfg, synth.model_weights(cfg, 310, "cuda", omega=0.1), max_batch=B)
    k, v = (torch.zeros((3, B, 8, T, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    hidden = torch.randn((B, 1024), device="cuda")
    alone = attention_us(model, 2, k, v, hidden, [T - 1])
    uneven = attention_us(model, 2, k, v, hidden, [T - 1] + [100] * (B - 1))
    print("alone", alone, "beside short ones", uneven)
    assert uneven < 5 * alone


def test_block_that_few_sequences_run():
    """A device-routed block that few of 24 sequences of 8000 rows run (each runs one of six): its
    attention may take a few times what one sequence alone takes in 32 chunks; with the two chunks
    that suit 24 running sequences it takes five times as long."""
    B, T = 24, 8001
    shape = dict(n_layers=8, d_model=1024, n_heads=32, n_kv_heads=8, head_dim=128, d_ffn=512,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    cfg = synth.model_config(shape, "bf16", T)
    model = blib.Model(cfg, synth.model_weights(cfg, 320, "cuda"), max_batch=B)
    k, v = (torch.zeros((8, B, 8, T, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    gen = torch.Generator(device="cuda").manual_seed(321)
    hidden = torch.randn((B, 1024), generator=gen, device="cuda")
    mask = torch.zeros((B, 6), dtype=torch.uint8, device="cuda")
    model.decode_step(k, v, hidden.clone(), [T - 1] * B, [1] * B, mask_out=mask)
    runs = mask.sum(0).tolist()
    block = min((n, i) for i, n in enumerate(runs) if n > 0)[1]
    alone = attention_us(model, 7, k, v, hidden, [T - 1])
    few = attention_us(model, 1 + block, k, v, hidden, [T - 1] * B)
    print("runs", runs, "alone", alone, "few", few)
    assert runs[block] <= 4 and few < 3.5 * alone


def test_split_tile_of_any_k():
    """GEMM_TILE_256_SPLIT splits K of the residual adds wherever the tiled GEMM runs: with K of an odd
    number of 64s (576 and 2240 here) too, on the 128 x 128 tile.  Other bits than the unsplit tile, from
    the order of the sums alone (1e-2 of the largest output, as for the short prompts)."""
    n, f = 200, 2240
    shape = dict(n_layers=3, d_model=576, n_heads=9, n_kv_heads=3, head_dim=64, d_ffn=f,
                 dm_hidden=64, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    P = Pair(shape, "bf16", n, 1, seed=330, omega=0.1)
    out = {}
    for tile in (blib.GEMM_TILE_128, blib.GEMM_TILE_256, blib.GEMM_TILE_256_SPLIT, blib.GEMM_TILE_AUTO):
        P.gpu.set_gemm_tile(tile)
        out[tile] = gpu_prefill(P, [n], [1], n, seed=331)[0][0, :n]
    plain, split = out[blib.GEMM_TILE_128], out[blib.GEMM_TILE_256_SPLIT]
    assert np.array_equal(plain, out[blib.GEMM_TILE_256])
    assert not np.array_equal(plain, split)
    for a in (split, out[blib.GEMM_TILE_AUTO]):
        assert np.max(np.abs(a - plain)) <= 1e-2 * np.max(np.abs(plain))


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_router_context(bad):
    """A value that is not finite in one sequence's router context, whose remainders beyond bf16 do
    not exist: that sequence's scores are the oracle's (infinite or NaN), and the others', in the
    same MFMA tile, are as accurate as without it."""
    B, T = 6, 30
    shape = dict(n_layers=6, d_model=96, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=128,
                 dm_hidden=40, dm_act="silu", rope_theta=1e4, rms_eps=1e-5)
    P = Pair(shape, "bf16", T, B, seed=340, omega=0.1)
    g = torch.Generator().manual_seed(341)
    hk = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    hv = synth.storage_numpy(torch.randn(P.shape5, generator=g).to(P.tdt))
    h = synth.hidden_inputs(B, 96, seed=342)
    h[2, 7] = bad
    scores = torch.zeros((B, P.L_mid), device="cuda")
    P.gpu.pool_route(P.upload(hk), P.upload(hv), [T - 1] * B, h.cuda(), scores)
    got = scores.cpu().numpy()
    for b in range(B):
        ref = np.asarray(P.orc.dm_scores(P.orc.context(hk[0, b], hv[0, b], T - 1, h[b].numpy())))
        if b == 2:
            assert not np.any(np.isfinite(ref))
            assert np.array_equal(got[b], ref.astype(np.float32), equal_nan=True), (got[b], ref)
        else:
            assert np.max(np.abs(got[b] - ref)) <= 1e-5 * max(1.0, float(np.max(np.abs(ref)))), b


def test_router_scores_error():
    """Scores of 16 sequences at the Llama-8B router's width (48 K slices) against float64: no further
    off than one sequence at a time, whose GEMV adds 64 lanes' sums as a tree (rms of the scores,
    ten seeds of other inputs each: 1.38e-7 there; 1.64e-7 with the slices added one by one in
    fp32, 1.15e-7 in fp64)."""
    B, n, nkv, hd, d, H, Lm = 16, 21, 8, 128, 4096, 512, 30
    cfg = synth.model_config(dict(synth.SHAPES["llama3_8b"]), "bf16", 64)
    err = {B: [], 1: []}
    for seed in range(10):
        g = torch.Generator(device="cuda").manual_seed(350 + seed)
        rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
        k, v = (rnd(1, B, nkv, 64, hd).bfloat16() for _ in range(2))
        w1, w2 = (0.02 * rnd(H, 2 * nkv * hd + d)).bfloat16(), (0.02 * rnd(Lm, H)).bfloat16()
        b1, b2 = (0.02 * rnd(H)).bfloat16(), (0.02 * rnd(Lm)).bfloat16()
        h = rnd(B, d)
        dm = dict(w1=w1, b1=b1, w2=w2, b2=b2, omega=0.0, prior=None)
        z = torch.cat([t[0, :, :, :n].double().mean(2).reshape(B, -1) for t in (k, v)] + [h.double()], 1)
        ref = torch.nn.functional.silu(z @ w1.double().T.contiguous() + b1.double()) @ w2.double().T.contiguous() + b2.double()
        out = torch.zeros((B, Lm), device="cuda")
        for step in err:
            for b in range(0, B, step):
                # the cache layout's batch capacity is that of the slice passed
                blib.pool_route_noalloc(cfg, dm, step, k[:, b:b + step].contiguous(), v[:, b:b + step].contiguous(),
                                        [n - 1] * step, h[b:b + step].contiguous(), out[b:b + step])
            err[step].append(float((out.double() - ref).norm() / ref.norm()))
    batch, one = np.mean(err[B]), np.mean(err[1])
    print("batch", batch, "one at a time", one)
    assert batch <= one


@pytest.mark.parametrize("shape,B,gemv", [("llama3_8b", 2, 4.18e-7), ("llama3_8b", 4, 4.13e-7), ("qwen2_7b", 3, 4.15e-7)])
def test_packed_activations_error(shape, B, gemv):
    """Hidden states of two to four sequences (packed activations on the MFMA) against float64 at
    the real widths: no further off than the fp32 GEMV had them (gemv: rms over 30 seeds; 3.98e-7,
    3.97e-7 and 3.75e-7 here, 4.84e-7 to 5.0e-7 with a wavefront's k-steps in two chains).  Many
    cached rows, so that single K/V rounding flips do not decide it; eight seeds spread by 1 %."""
    case = dict({c["name"]: c for c in cases.listed()}["decode_8b_long"], shape=shape, batch=B, ctx=9000,
                layers=3, share=1.0)
    err = []
    for seed in range(8):
        state = cases.prepare(case, 360 + seed)
        hidden = cases.run(state)["hidden"].double()
        state["model"].close()
        ref = cases.exact(case, 360 + seed)["hidden"]
        err.append(float((hidden - ref).norm() / ref.norm()))
    rms = float(np.sqrt(np.mean(np.square(err))))
    print(shape, B, rms)
    assert rms <= gemv


def test_pooled_scores_error_of_a_long_context():
    """Scores of one decode step over 30000 cached rows against float64 means of the same cache, the
    hidden state left out of the context (its columns of the first layer are 0): the pool sums come
    from the attention's chunks, and longer chunks sum less accurately (geometric mean over 60 seeds
    2.0e-7 with 64 chunks, 2.8e-7 with 32; the seeds' spread puts 9 % on it)."""
    case = dict({c["name"]: c for c in cases.listed()}["decode_8b_long"], ctx=30000, layers=3, share=1.0)
    err = []
    for seed in range(1, 61):
        s = cases.prepare(case, seed)
        d = s["cfg"]["d_model"]
        s["W"]["dm"]["w1"][:, -d:] = 0
        s["W"]["dm"]["w1"] *= 50
        s["W"]["dm"].update(prior=None, omega=0.0)
        s["model"].close()
        s["model"] = blib.Model(s["cfg"], s["W"], max_batch=1)
        got = cases.run(s)["scores"].double()
        zero = torch.zeros((1, d), device="cuda", dtype=torch.float64)
        ref = cases._scores(s, zero, s["lens"])[1]
        err.append(float((got - ref).norm() / ref.norm()))
        s["model"].close()
    mean = float(np.exp(np.mean(np.log(err))))
    print(mean)
    assert mean < 2.4e-7
