"""Which kernel form the packed projection's launch rule takes, read a second
time, and the cases of the GPU tests that reach every form in several pipelined
groups of k steps (a group that refills its registers, more than once).
"""

CUS, PRE = 256, 4     # compute units; k steps of a pipelined group (8 where the weights come in bursts)


def packed_form(B, n_heads, rows, hidden, residual=False):
    """((waves, batch tiles, k ranges, steps per chunk of states, bursts), pipelined groups) of the launch."""
    def cdiv(a, b):
        return -(-a // b)
    nG, nF = cdiv(rows, 64), hidden // 32
    nb = next(n for n in (1, 2, 4, 6, 8) if B <= 16 * n or n == 8)
    if nG * n_heads <= CUS:
        nb = next((n for n in (1, 2, 4) if n < nb and nG * n_heads * cdiv(B, 16 * n) <= CUS), nb)
        if nb > 4 and hidden <= 2048:
            nb = 4
    blocks = {g: cdiv(nG, g) * n_heads for g in (1, 2, 4, 8)}
    rounds = cdiv(blocks[8], CUS)
    full = blocks[8] * 100 >= rounds * CUS * 97
    wide = rounds == 1 or blocks[8] * 10 >= rounds * CUS * 9
    if blocks[1] <= CUS:
        f = (4, nb, 4, 2 if nb <= 4 else 1, False)
    elif blocks[2] <= CUS:
        f = (8, nb, 4, 2 if nb == 6 else 1, False) if nb >= 6 else (4, nb, 2, 4, False)
    elif blocks[4] <= CUS:
        f = (4, 1, 1, 4, False) if nb == 1 and residual else (8, nb, 2, 2 if nb >= 6 else 4, False)
    elif (blocks[8] * 8 <= CUS * 7 if nb == 1 else wide and not (full and nb == 2 and hidden <= 4096)):
        f = (8, nb, 1, 4, False)
    else:
        f = (4, nb, 1, 4, nb == 1 and full and hidden >= 1024)
    pre = 8 if f[4] else PRE
    return f, max(0, nF - (f[2] - 1) * cdiv(nF, f[2])) // pre


# heads, vocabulary, hidden of each group of forms, and the batches that give 1, 2, 4, 6 and 8 tiles
FORMS = [
    (3, 3190, 2104, (7, 20, 40, 70, 100)),          # one row group a block, four ranges
    (4, 6370, 2104, (16, 17, 64, 96, 128)),         # two
    (4, 12790, 1064, (16, 31, 33, 65, 97)),         # four
    (4, 19150, 520, (3, 32, 64, 90, 120)),          # eight
    (4, 33250, 424, (16, 20, 50, 81, 113)),         # eight would leave a short last round
    (4, 32000, 1032, (10, 24)),                     # a full round: bursts, 4-wave blocks
    (4, 32000, 424, (10,)),                         # the same of short columns: no bursts
    (4, 29650, 424, (10, 24)),                      # nearly full
    (2, 650, 2104, (40, 100, 200)),                 # few groups: the batch over several blocks
    (5, 1000, 2040, (64, 200)),
]
FORM_CASES = [(n, B, V, H) for n, V, H, Bs in FORMS for B in Bs]


def test_form_cases_reach_every_form():
    want = {(4, nb, 4, 2 if nb <= 4 else 1, False) for nb in (1, 2, 4, 6, 8)} | \
           {(4, 1, 2, 4, False), (4, 2, 2, 4, False), (4, 4, 2, 4, False), (8, 6, 4, 2, False), (8, 8, 4, 1, False)} | \
           {(8, nb, 2, 2 if nb >= 6 else 4, False) for nb in (1, 2, 4, 6, 8)} | \
           {(w, nb, 1, 4, False) for w in (4, 8) for nb in (1, 2, 4, 6, 8)} | {(4, 1, 1, 4, True)}
    got = [packed_form(B, n, V, H) for n, B, V, H in FORM_CASES]
    assert {f for f, _ in got} == want
    for f, groups in got:
        assert groups >= 3, f                       # the refilling loop runs, and more than once
    assert all(H % 32 for _, _, _, H in FORM_CASES)  # and a rest follows
