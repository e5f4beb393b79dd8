"""GPU: attention of batches whose descriptors travel packed in the kernel
arguments (33 to 120 sequences, KV heads a multiple of eight), and items with
waves that hold no query row.  Both sides of the limits, against the oracle.
"""

import numpy as np
import pytest

import oracle
from paper_2506_01986_amd import runner, synth
from tests.gpu_time import graph_us

from tests.test_gpu_padded import padded_workload, run_padded_parity
from tests.test_gpu_parity import close, edge_cfg, run_parity, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def lens(n, hi, *first):
    return [*first, *(int(x) for x in np.random.default_rng(n).integers(0, hi, n - len(first)))]


# sequences, query heads, KV heads, most tree nodes, committed lengths
BATCHES = {
    "b33_mha_few_rows": (33, 8, 8, 20, lens(33, 200)),           # 64-row items, second wave group often empty
    "b64_split": (64, 8, 8, 64, lens(64, 300, 6000, 2500, 0)),   # some sequences in several chunks, one empty
    "b65_gqa": (65, 32, 8, 40, lens(65, 150, 3000)),             # 128-row items, row blocks with one to four waves
    "b120_kv16": (120, 16, 16, 6, lens(120, 90, 700)),           # the most sequences in the arguments
    "b121": (121, 8, 8, 6, lens(121, 90, 700)),                  # one more: the workspace table
    "b40_kv12": (40, 12, 12, 10, lens(40, 200, 900)),            # KV heads not a multiple of eight: the table
}


@pytest.mark.parametrize("name", list(BATCHES))
def test_batches(torch_cuda, name):  # noqa: F811
    B, n_q, n_kv, nodes, L = BATCHES[name]
    rng = np.random.default_rng(B)
    trees = [synth.random_tree(rng, int(rng.integers(1, nodes + 1))) for _ in range(B)]
    cfg = edge_cfg(B=B, n_q=n_q, n_kv=n_kv, hidden=32, vocab=256)
    run_parity(torch_cuda, synth.make(cfg, trees=trees, lens=L), label=name)


# sequences, query heads, KV heads, most tree nodes, tokens held, runs of pads (whole chunks of the first sequences)
PADDED = {
    "b40_mha_few_rows": (40, 8, 8, 20, lens(40, 200, 40), {}),              # 64-row items, waves without rows
    "b36_mha_split": (36, 16, 16, 12, lens(36, 120, 4000), {0: (900, 2200)}),
    "b34_gqa_split": (34, 32, 8, 40, lens(34, 150, 5000, 60), {0: (1500, 3600), 1: (3, 10 ** 6)}),   # 128-row items
    "b120": (120, 8, 8, 6, lens(120, 60, 500), {}),
    "b121": (121, 8, 8, 6, lens(121, 60, 500), {}),                         # one more: the workspace table
}


@pytest.mark.parametrize("name", list(PADDED))
def test_padded_batches(torch_cuda, name):  # noqa: F811
    """The pad mask's words are found from the packed 32-bit bases, which are no multiples of 32 here."""
    B, n_q, n_kv, nodes, held, runs = PADDED[name]
    rng = np.random.default_rng(B)
    cfg = edge_cfg(B=B, n_q=n_q, n_kv=n_kv, hidden=32, vocab=256)
    trees = [synth.random_tree(rng, int(rng.integers(1, nodes + 1)), max_depth=4) for _ in range(B)]
    wl, flags = padded_workload(cfg, trees, [x + 45 for x in held], 8, seed=B, pad_runs=runs)
    assert len({int(x) % 32 for x in wl.seq_base}) > 8
    run_padded_parity(torch_cuda, wl, flags, label=name)


@pytest.mark.parametrize("head_dim", [32, 64, 128])
def test_fp32_overflowed_scores(torch_cuda, head_dim):  # noqa: F811
    """Keys whose score overflows to -inf get weight 0, also where a key slot of the kernel holds no other."""
    cfg = edge_cfg(dtype="fp32", B=2, n_q=4, n_kv=2, head_dim=head_dim, hidden=32, vocab=256)
    wl = synth.make(cfg, trees=[synth.chain_tree(1), synth.t16()], lens=[13, 60])
    wl.q = (np.abs(wl.q) + 1).astype(np.float32)
    for b in range(2):
        wl.pool_k[:, int(wl.seq_base[b]):int(wl.seq_base[b]) + 13] = -3e38
    step = runner.VerifyStep(wl)
    step.tree_attn()
    torch_cuda.cuda.synchronize()
    got = step.out.double().cpu().numpy()
    ref = oracle.tree_attn(wl.q, wl.pool_k, wl.pool_v, wl.node_off, wl.parent, wl.lens, wl.seq_base, cfg.n_kv)
    assert close(got.reshape(ref.shape), ref, "fp32") <= 0


@pytest.mark.parametrize("longest", [0, 8, 9, 16, 17, 65])
@pytest.mark.parametrize("head_dim", [4, 32, 36, 64, 96, 128])
def test_fp32_short_contexts(torch_cuda, head_dim, longest):  # noqa: F811
    """One wave a block up to 16 committed keys (two past 8 of more than 64 columns), four beyond; root paths of up to
    16 nodes."""
    cfg = edge_cfg(dtype="fp32", B=4, n_q=6, n_kv=2, head_dim=head_dim, hidden=32, vocab=256, n_heads=15, topk=(2,) * 15)
    rng = np.random.default_rng(head_dim)
    trees = [synth.chain_tree(16), synth.random_tree(rng, 128), synth.chain_tree(1), synth.t16()]
    wl = synth.make(cfg, trees=trees, lens=[longest, longest // 2, max(longest - 1, 0), min(longest, 1)])
    step = runner.VerifyStep(wl)
    step.tree_attn()
    torch_cuda.cuda.synchronize()
    ref = oracle.tree_attn(wl.q, wl.pool_k, wl.pool_v, wl.node_off, wl.parent, wl.lens, wl.seq_base, cfg.n_kv)
    assert close(step.out.double().cpu().numpy().reshape(ref.shape), ref, "fp32") <= 0


def test_fp32_short_contexts_cost_less(torch_cuda):  # noqa: F811
    """4 committed keys against 64: waves that would only wait are not launched."""
    us = []
    for L in (4, 64):
        cfg = edge_cfg(dtype="fp32", B=8, n_q=32, n_kv=8, hidden=32, vocab=256)
        step = runner.VerifyStep(synth.make(cfg, trees=[synth.t64()] * 8, lens=[L] * 8))
        us.append(graph_us(torch_cuda, step.tree_attn))
    assert us[0] <= 0.4 * us[1], us
