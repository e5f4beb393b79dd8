"""GPU: top-k of rows of any length, from group maxima and by the row scan.

The logits are planted (one input is 1, so they are a weight column, exact in
every form), with ties, rows of one value and rows of -inf; ids and values are
compared exactly with the oracle's.
"""

import numpy as np
import pytest

import oracle
from paper_2506_01986_amd import synth
from tests.gpu_time import graph_us

from tests.test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


class Rows:
    """Planted rows [head][vocab] as the weights of one sequence's heads."""

    def __init__(self, torch, rows, dtype, packed, B=1):
        from paper_2506_01986_amd import specmemo as sm
        from paper_2506_01986_amd.runner import to_device
        self.torch, self.sm, (self.nh, self.V) = torch, sm, rows.shape
        self.dt = sm.FP32 if dtype == "fp32" else sm.BF16
        store = (lambda x: x.astype(np.float32)) if dtype == "fp32" else \
            (lambda x: synth.to_bf16_bits(x.astype(np.float32)).reshape(x.shape))
        w, h = np.zeros((self.nh, self.V, 8)), np.zeros((B, 8))
        w[:, :, 3], h[:, 3] = rows, 1.0
        self.h, self.w = to_device(store(h), dtype, "cuda"), to_device(store(w), dtype, "cuda")
        self.layout = sm.HEADS_ROWMAJOR
        if packed:
            p = torch.empty(sm.packed_heads_bytes(self.dt, self.nh, self.V, 8), dtype=torch.uint8, device="cuda")
            sm.pack_heads(self.dt, self.nh, self.V, 8, self.w, p)
            self.w, self.layout = p, sm.HEADS_PACKED
        zero = np.zeros(B, np.int32)
        self.tr = sm.Trees(np.arange(B + 1), np.full(B, -1), zero, zero, device="cuda")   # single-node trees
        self.tok = torch.zeros(B, dtype=torch.int32, device="cuda")
        self.z = torch.empty((B, self.nh, self.V), device="cuda")
        self.nb = sm.workspace_bytes(sm.WS_TOPK, self.dt, self.tr, None, self.nh, self.V)
        self.ws = torch.empty(self.nb, dtype=torch.uint8, device="cuda")
        self.B = B

    def call(self, k, maxima):
        """maxima: with a workspace that holds the group maxima (bf16); else the rows are scanned."""
        ids = self.torch.full((self.B, self.nh, k), -7, dtype=self.torch.int32, device="cuda")
        vals = self.torch.full((self.B, self.nh, k), float("nan"), device="cuda")

        def run():
            self.sm.medusa_topk(self.dt, self.tr, 8, self.V, self.nh, [k] * self.nh, self.h, self.w, self.tok, ids,
                                self.tok, logits_out=self.z, topk_vals=vals, ws=self.ws if maxima else None,
                                ws_bytes=self.nb if maxima else 0, head_layout=self.layout)
        return run, ids, vals


@pytest.mark.parametrize("form", ["bf16", "bf16_packed", "fp32"])
@pytest.mark.parametrize("V", [1, 31, 32, 33, 64, 100, 127, 128, 257, 639, 1280, 1281, 2047, 2052, 4096, 9217, 40001])
def test_planted_rows(torch_cuda, V, form):  # noqa: F811
    rng = np.random.default_rng(V)
    rows = rng.normal(size=(6, V))
    rows[1] = rng.integers(0, 4, V)                              # ties everywhere
    rows[2] = 2.5                                                # one value
    rows[3] = -np.inf
    rows[3, rng.choice(V, min(V, 3), replace=False)] = [1.0, -2.0, 1.0][:min(V, 3)]
    rows[4] = np.where(rng.random(V) < 0.9, -3e38, rows[4])      # few values above the lowest
    rows = rows.astype(np.float32).astype(np.float64)            # as stored
    if form != "fp32":
        rows = synth.storage_to_f64(synth.to_bf16_bits(rows.astype(np.float32)).reshape(rows.shape), "bf16")
    r = Rows(torch_cuda, rows, form[:4], form == "bf16_packed")
    for k in sorted({1, min(V, 10), min(V, 32)}):
        want, wv = oracle.topk(rows, k)
        for maxima in (True, False):
            run, ids, vals = r.call(k, maxima)
            run()
            assert np.array_equal(ids.cpu().numpy()[0], want), (k, maxima)
            assert np.array_equal(vals.double().cpu().numpy()[0], wv)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("V,k", [(700, 10), (2000, 10), (2000, 32), (9216, 10), (24000, 32)])
def test_group_maxima_are_no_slower(torch_cuda, V, k, packed):  # noqa: F811
    """Few groups: threshold sets left empty made the call with maxima 2 to 50 times the scan's."""
    r = Rows(torch_cuda, np.random.default_rng(V).normal(size=(4, V)), "bf16", packed, B=10)
    with_maxima, scan = (graph_us(torch_cuda, r.call(k, m)[0]) for m in (True, False))
    assert with_maxima <= 1.4 * scan, (with_maxima, scan)
