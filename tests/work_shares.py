"""How many diagonal blocks each XCD group's share of a ragged symmetric batch leaves to the
half-block launch: the rule of csrc/mpm_work.h in plain Python, so that a GPU test can say
that its batch reaches that launch. test_work_order.py compares it with the header."""


def place(i, B):
    """The image at place i of the batch's order."""
    run = max(1, B // 8)
    k = i // run
    return k + 8 * (i - k * run) if k < 8 else i


def deferred(ns, rows=256, groups=8, slots=32, lone=False):
    """Deferred diagonal blocks per group for images of ns tokens in blocks of `rows`."""
    B = len(ns)
    diag = []  # whether item p of the order is a diagonal block
    for i in range(B):
        nb = -(-ns[place(i, B)] // rows)
        for q in range(nb):
            diag += [True] + [False] * (nb - q - 1)
    lone = lone and 2 * -(-len(diag) // groups) <= slots
    out = []
    for g in range(groups):
        lo, hi = len(diag) * g // groups, len(diag) * (g + 1) // groups
        cnt, m = hi - lo, (hi - lo) % slots
        defers = (lone or cnt > slots) and 0 < 2 * m <= slots and sum(diag[lo:hi]) >= m
        out.append(m if defers else 0)
    return out
