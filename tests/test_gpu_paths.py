"""GPU tests of single kernels and dispatch branches at the sizes where they can go wrong
(edges of tiles, remainders, both sides of a rule), against the oracle or plain torch."""
import numpy as np
import pytest
import torch

from _gpu import Pair
from paper_2606_09514_amd import synth
from test_gpu_parity import gqa_shape, one_step_all

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
