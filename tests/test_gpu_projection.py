"""GPU: the projection kernels at the edges of their forms.

Packed weights: the launch picks the batch tiles of a block (1, 2, 4, 6 or 8 of 16 states) from
the batch, and the row groups and k ranges of a block from the number of row
groups; the k steps divide into pipelined groups, the ranges' rests and a last
partial step.  Sizes sit on both sides of every such line, and a second list
(test_projection_forms.py) reaches every form with several pipelined groups.
References are fp64;
|error| <= (hidden + 8) 2^-24 sum |w h| (fp32 summation in any order), and for
the residual blocks half a bf16 step more (of eight significant bits: 2^-8 of
the value).
"""

import numpy as np
import pytest

import oracle
from paper_2506_01986_amd import synth
from tests.gpu_time import graph_us
from tests.test_projection_forms import FORM_CASES, packed_form

pytestmark = pytest.mark.gpu

# heads, batch, vocabulary, hidden: 64-row groups x heads against 256 blocks of 1, 2, 4 and 8 groups
HEADS = [
    (3, 1, 64, 40), (4, 16, 4096, 136), (4, 33, 4090, 264), (2, 129, 700, 1000), (4, 97, 4096, 520),    # one group
    (4, 5, 4160, 1000), (4, 17, 8192, 264), (4, 64, 5001, 136), (4, 96, 8190, 72), (2, 128, 10000, 392),  # two
    (4, 16, 8256, 264), (4, 32, 16384, 40), (4, 65, 9001, 328), (4, 113, 16380, 136),                    # four
    (4, 10, 16448, 136), (4, 40, 28000, 72), (4, 96, 20001, 40), (4, 128, 32760, 264),                   # eight
    (4, 3, 32760, 520), (4, 16, 31000, 264), (4, 12, 37000, 136), (4, 18, 37003, 72), (4, 200, 36992, 40),
]


def bits(rng, shape, std):
    return synth.to_bf16_bits((std * rng.standard_normal(shape)).astype(np.float32)).reshape(shape)


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2506_01986_amd import runner, specmemo as sm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    sm.load()
    return torch, sm, lambda x: runner.to_device(x, "bf16", "cuda")


def pack(torch, sm, w):
    n, rows, hidden = w.shape
    out = torch.empty(sm.packed_heads_bytes(sm.BF16, n, rows, hidden), dtype=torch.uint8, device="cuda")
    sm.pack_heads(sm.BF16, n, rows, hidden, w, out)
    return out


# row-major: 128-row blocks, 128-column chunks (rings of 2, 3 and 4), 1 to 8 batch tiles
ROWS = [(3, 1, 1, 8), (2, 16, 128, 128), (4, 5, 129, 392), (4, 16, 4003, 1000), (4, 17, 1000, 256), (3, 32, 255, 520),
        (4, 33, 2001, 640), (2, 64, 130, 1160), (2, 65, 700, 136), (4, 120, 1001, 384), (1, 200, 300, 904)]


@pytest.mark.parametrize("packed,n_heads,B,vocab,hidden", [(True, *c) for c in HEADS] + [(False, *c) for c in ROWS])
def test_heads_forms(gpu, packed, n_heads, B, vocab, hidden):
    torch, sm, dev = gpu
    rng = np.random.default_rng(B + vocab + hidden)
    h, w = bits(rng, (B, hidden), 1.0), bits(rng, (n_heads, vocab, hidden), 0.05)
    hd, wd = dev(h), dev(w)
    wp = pack(torch, sm, wd) if packed else wd
    z = torch.full((B, n_heads, vocab), float("nan"), device="cuda")
    k = min(10, vocab)
    ids = torch.empty((B, n_heads, k), dtype=torch.int32, device="cuda")
    zero = np.zeros(B, np.int32)
    tr = sm.Trees(np.arange(B + 1), np.full(B, -1), zero, zero, device="cuda")       # single-node trees
    tok, root = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
    nb = sm.workspace_bytes(sm.WS_TOPK, sm.BF16, tr, None, n_heads, vocab)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    sm.medusa_topk(sm.BF16, tr, hidden, vocab, n_heads, [k] * n_heads, hd, wp, root, ids, tok, logits_out=z, ws=ws,
                   ws_bytes=nb, head_layout=sm.HEADS_PACKED if packed else sm.HEADS_ROWMAJOR)
    for i in range(n_heads):
        w64 = wd[i].double().t()
        ref, size = hd.double() @ w64, hd.double().abs() @ w64.abs()
        err = (z[:, i].double() - ref).abs() - (hidden + 8) * 2.0 ** -24 * size
        assert float(err.max()) <= 0 and bool(torch.isfinite(z[:, i]).all())
    if B * vocab <= 400_000:      # the group maxima lead to the same ids as the logits themselves
        want, _ = oracle.topk(z.cpu().numpy().astype(np.float64).reshape(B * n_heads, vocab), k)
        assert np.array_equal(ids.cpu().numpy().reshape(B * n_heads, k), want)


@pytest.mark.parametrize("n_heads,B,hidden", [(2, 1, 8), (4, 16, 520), (3, 34, 1000), (5, 70, 392), (2, 120, 4104),
                                              (4, 33, 4160), (4, 130, 136)])
def test_resblock_forms(gpu, n_heads, B, hidden):
    torch, sm, dev = gpu
    rng = np.random.default_rng(B + hidden)
    h, w, b = bits(rng, (B, hidden), 1.0), bits(rng, (n_heads, hidden, hidden), 0.05), bits(rng, (n_heads, hidden), 0.5)
    hd, wd, bd = dev(h), dev(w), dev(b)
    out = torch.full((n_heads, B, hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
    sm.medusa_resblock(sm.BF16, B, hidden, n_heads, hd, pack(torch, sm, wd), bd, out)
    for i in range(n_heads):
        y = hd.double() @ wd[i].double().t() + bd[i].double()
        ref = hd.double() + y * torch.sigmoid(y)
        size = hd.double().abs() @ wd[i].double().abs().t() + bd[i].double().abs()
        # |SiLU'| <= 1.1; the activation itself adds a few ulp of y
        bound = 1.1 * (hidden + 8) * 2.0 ** -24 * size + 2.0 ** -20 * (1 + y.abs()) + 2.0 ** -8 * ref.abs()
        assert float(((out[i].double() - ref).abs() - bound).max()) <= 0


def device_normal(torch, shape, std, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)


def check_heads(torch, sm, n_heads, B, vocab, hidden, packed):
    h, w = device_normal(torch, (B, hidden), 1.0, 1), device_normal(torch, (n_heads, vocab, hidden), 0.05, 2)
    k = 10
    z = torch.full((B, n_heads, vocab), float("nan"), device="cuda")
    ids = torch.full((B, n_heads, k), -1, dtype=torch.int32, device="cuda")
    vals = torch.empty((B, n_heads, k), device="cuda")
    zero = np.zeros(B, np.int32)
    tr = sm.Trees(np.arange(B + 1), np.full(B, -1), zero, zero, device="cuda")       # single-node trees
    tok, root = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
    nb = sm.workspace_bytes(sm.WS_TOPK, sm.BF16, tr, None, n_heads, vocab)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    sm.medusa_topk(sm.BF16, tr, hidden, vocab, n_heads, [k] * n_heads, h, pack(torch, sm, w) if packed else w, root,
                   ids, tok, logits_out=z, topk_vals=vals, ws=ws, ws_bytes=nb,
                   head_layout=sm.HEADS_PACKED if packed else sm.HEADS_ROWMAJOR)
    hd = h.double()
    for i in range(n_heads):
        w64 = w[i].double().t()
        err = (z[:, i].double() - hd @ w64).abs() - (hidden + 8) * 2.0 ** -24 * (hd.abs() @ w64.abs())
        assert float(err.max()) <= 0 and bool(torch.isfinite(z[:, i]).all())
    # the group maxima lead to the largest of these logits
    assert torch.equal(vals, torch.topk(z, k, dim=2).values)
    assert torch.equal(z.gather(2, ids.long()), vals)


@pytest.mark.parametrize("n_heads,B,vocab,hidden", FORM_CASES)
def test_every_packed_form(gpu, n_heads, B, vocab, hidden):
    torch, sm, dev = gpu
    check_heads(torch, sm, n_heads, B, vocab, hidden, True)


# row-major: 256 blocks of 128 rows, so that 17, 33 and 65 states make 2, 4 and 8 tiles; chunks that go round
# the rings of 4, 3, 3 and 2, and a rest; then few rows, the batch over several blocks
@pytest.mark.parametrize("n_heads,B,vocab,hidden", [
    (4, 16, 8101, 1160), (4, 20, 8101, 904), (4, 33, 8101, 1160), (4, 64, 8192, 904), (4, 65, 8101, 648),
    (4, 128, 8130, 1160), (4, 200, 8101, 136), (2, 100, 4003, 648), (1, 129, 300, 904)])
def test_every_rowmajor_form(gpu, n_heads, B, vocab, hidden):
    torch, sm, dev = gpu
    check_heads(torch, sm, n_heads, B, vocab, hidden, False)


@pytest.mark.parametrize("B", [1, 16])
def test_heads_of_four_groups_sum_two_ranges(gpu, B):
    """513 to 1024 row groups: columns in two ranges, whose sums lie nearer to 64 bits than one chain's.

    The error of a chain of random terms grows with the root of its length: 256 k steps in one chain measured 5.8e-7,
    two chains of 128 steps 4.0e-7, 1.4 times less.  The line lies between."""
    torch, sm, dev = gpu
    n_heads, vocab, hidden = 4, 9000, 8192
    h, w = device_normal(torch, (B, hidden), 1.0, 1), device_normal(torch, (n_heads, vocab, hidden), 0.02, 2)
    z = torch.empty((B, n_heads, vocab), device="cuda")
    sm.head_logits(sm.BF16, B, hidden, vocab, n_heads, h, pack(torch, sm, w), z, sm.HEADS_PACKED)
    ref = torch.stack([h.double() @ w[i].double().t() for i in range(n_heads)], 1)
    assert float((z.double() - ref).norm() / ref.norm()) <= 4.8e-7


@pytest.mark.parametrize("n_heads,hidden", [(4, 2104), (10, 2104), (15, 3208)])
@pytest.mark.parametrize("B", [10, 20, 40, 70, 100])
def test_residual_block_forms_in_groups(gpu, n_heads, hidden, B):
    """One, two and four row groups a block, 1 to 8 batch tiles, several pipelined groups."""
    torch, sm, dev = gpu
    assert packed_form(B, n_heads, hidden, hidden, residual=True)[1] >= 3
    h, w, b = (device_normal(torch, s, std, i) for i, (s, std) in enumerate(
        [((B, hidden), 1.0), ((n_heads, hidden, hidden), 0.05), ((n_heads, hidden), 0.5)]))
    out = torch.full((n_heads, B, hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
    sm.medusa_resblock(sm.BF16, B, hidden, n_heads, h, pack(torch, sm, w), b, out)
    hd = h.double()
    for i in range(n_heads):
        w64 = w[i].double().t()
        y = hd @ w64 + b[i].double()
        ref = hd + y * torch.sigmoid(y)
        bound = 1.1 * (hidden + 8) * 2.0 ** -24 * (hd.abs() @ w64.abs() + b[i].double().abs()) + \
            2.0 ** -20 * (1 + y.abs()) + 2.0 ** -8 * ref.abs()
        assert float(((out[i].double() - ref).abs() - bound).max()) <= 0


@pytest.mark.parametrize("hidden", [40, 264, 640, 648, 1000, 1032])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 32])
def test_fp32_forms(gpu, B, hidden):
    """fp32 heads and residual blocks: one, two and four states a wave, short rows and several strides, row counts
    that are no multiple of a wave's four or a block's sixteen."""
    torch, sm, dev = gpu
    g = torch.Generator(device="cuda")
    g.manual_seed(B * hidden)

    def normal(*shape):
        return torch.empty(shape, device="cuda").normal_(generator=g)
    h, hs = normal(B, hidden), (2 * hidden + 40) * 2.0 ** -24
    hd = h.double()
    for vocab in (1, 50, 333):
        w = normal(3, vocab, hidden)
        z = torch.full((B, 3, vocab), float("nan"), device="cuda")
        sm.head_logits(sm.FP32, B, hidden, vocab, 3, h, w, z)
        for i in range(3):
            w64 = w[i].double().t()
            assert float(((z[:, i].double() - hd @ w64).abs() - hs * (hd.abs() @ w64.abs())).max()) <= 0
    w, b = normal(2, hidden, hidden), normal(2, hidden)
    out = torch.full((2, B, hidden), float("nan"), device="cuda")
    sm.medusa_resblock(sm.FP32, B, hidden, 2, h, w, b, out, w1_layout=sm.HEADS_ROWMAJOR)
    for i in range(2):
        w64 = w[i].double().t()
        y = hd @ w64 + b[i].double()
        ref = hd + y * torch.sigmoid(y)
        bound = 1.1 * hs * (hd.abs() @ w64.abs() + b[i].double().abs()) + 2.0 ** -20 * (1 + y.abs() + ref.abs())
        assert float(((out[i].double() - ref).abs() - bound).max()) <= 0


@pytest.mark.parametrize("n_heads,hidden,few,many,at_most", [(2, 512, 16, 128, 2.0), (2, 4096, 64, 128, 1.6)])
def test_residual_blocks_spread_the_batch(gpu, n_heads, hidden, few, many, at_most):
    """Few row groups: more states go to more blocks, not to more work of one wave each."""
    torch, sm, dev = gpu
    us = []
    for B in (few, many):
        h, b = (torch.zeros(n, hidden, dtype=torch.bfloat16, device="cuda") for n in (B, n_heads))
        w = torch.zeros(sm.packed_heads_bytes(sm.BF16, n_heads, hidden, hidden), dtype=torch.uint8, device="cuda")
        out = torch.empty(n_heads, B, hidden, dtype=torch.bfloat16, device="cuda")
        us.append(graph_us(torch, lambda: sm.medusa_resblock(sm.BF16, B, hidden, n_heads, h, w, b, out)))
    assert us[1] <= at_most * us[0], us


@pytest.mark.parametrize("layout", ["packed", "rowmajor"])
def test_small_heads_spread_the_batch(gpu, layout):
    torch, sm, dev = gpu
    n_heads, vocab, hidden, us = 2, 50, 1000, []
    nb = sm.packed_heads_bytes(sm.BF16, n_heads, vocab, hidden)        # more than the row-major heads
    w = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    for B in (16, 128):
        h, z = torch.zeros(B, hidden, dtype=torch.bfloat16, device="cuda"), torch.empty(B, n_heads, vocab, device="cuda")
        us.append(graph_us(torch, lambda: sm.head_logits(sm.BF16, B, hidden, vocab, n_heads, h, w, z,
                                                         sm.HEADS_PACKED if layout == "packed" else sm.HEADS_ROWMAJOR)))
    assert us[1] <= 2.0 * us[0], us
