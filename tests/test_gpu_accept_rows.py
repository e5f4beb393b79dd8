"""GPU: the row passes of the acceptance on rows of any length and alignment.

Rows are read in 16-byte chunks at aligned addresses and up to 14 single values
around them, rows of up to 512 values as single values alone; they stay in
registers up to 4096 chunks, in forms of 1, 2, 4 and 8 chunks a thread.  48 rows of an odd
vocabulary meet every alignment.  Arg-best tokens are exact; lse and entropy are
fp32 sums of positive terms over a row (tree-wise below 100 terms in sequence,
2^-24 each, on values of about 12, and the exponentials' few ulp): within 2e-5.
"""

import numpy as np
import pytest

import oracle
from paper_2506_01986_amd import synth
from tests.gpu_time import graph_us

from tests.test_gpu_parity import _argbest_rows, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("vocab", [7, 9, 30, 511, 512, 513, 520, 1001, 2049, 2060, 4094, 4097, 4110, 8197, 16384, 16393, 32003, 32761, 32783, 40009])
def test_ragged_rows(torch_cuda, vocab, dtype):  # noqa: F811
    import torch
    from paper_2506_01986_amd import specmemo as sm
    from paper_2506_01986_amd.runner import to_device
    rng = np.random.default_rng(vocab)
    B, T = 48, 0.7
    node_off, root, zeros = np.arange(B + 1, dtype=np.int32), np.full(B, -1, np.int32), np.zeros(B, np.int32)
    tr = sm.Trees(node_off, root, zeros, zeros, device="cuda")      # single-node trees
    raw = _argbest_rows(rng, vocab, B)
    lg = raw if dtype == "fp32" else synth.to_bf16_bits(raw)
    dlg = to_device(lg, dtype, "cuda")
    dt = sm.FP32 if dtype == "fp32" else sm.BF16
    tok = torch.zeros(B, dtype=torch.int32, device="cuda")
    _, _, want = oracle.accept_greedy(lg, zeros, node_off, root, zeros, 1)
    for mode in (sm.GREEDY, sm.TYPICAL):
        acc, nxt = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        path = torch.full((B, 1), -7, dtype=torch.int32, device="cuda")
        ws = torch.empty(sm.workspace_bytes(sm.WS_ACCEPT, dt, tr, None, mode), dtype=torch.uint8, device="cuda")
        sm.accept(dt, tr, vocab, mode, dlg, tok, acc, path, 1, nxt, temperature=T, ws=ws, ws_bytes=ws.numel())
        assert np.array_equal(nxt.cpu().numpy(), want)
    stats = ws[:8 * B].view(torch.float32).cpu().numpy().reshape(B, 2).astype(np.float64)
    finite = np.arange(B) % 8 != 6                                  # the rows that are not all -inf
    lse, H = oracle.softmax_stats(lg[finite], T)
    assert np.abs(stats[finite, 0] - lse).max() <= 2e-5 * max(1.0, 50 / T / 12)    # rows with a value of 50: lse 71
    assert np.abs(stats[finite, 1] - H).max() <= 2e-5


@pytest.mark.parametrize("mode,at_most", [("greedy", 0.35), ("typical", 0.42)])
def test_short_rows_skip_the_long_rows_work(torch_cuda, mode, at_most):  # noqa: F811
    """Rows of 50 values against rows of 32000: no work for chunks that a short row lacks."""
    import torch
    from paper_2506_01986_amd import specmemo as sm
    B, us = 40, []
    t = synth.t64()
    tr = sm.Trees(np.arange(B + 1) * t.n, *(np.tile(x, B) for x in (t.parent, t.depth, t.rank)), device="cuda")
    m = sm.TYPICAL if mode == "typical" else sm.GREEDY
    tok, acc, nxt = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in (B * t.n, B, B))
    stride = tr.max_depth + 1
    path = torch.zeros((B, stride), dtype=torch.int32, device="cuda")
    ws = torch.empty(sm.workspace_bytes(sm.WS_ACCEPT, sm.BF16, tr, None, m), dtype=torch.uint8, device="cuda")
    for vocab in (50, 32000):
        lg = torch.empty((B * t.n, vocab), dtype=torch.bfloat16, device="cuda").normal_()
        us.append(graph_us(torch, lambda: sm.accept(sm.BF16, tr, vocab, m, lg, tok, acc, path, stride, nxt,
                                                    temperature=0.7, ws=ws, ws_bytes=ws.numel())))
    assert us[0] <= at_most * us[1], us
