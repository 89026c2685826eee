"""polyspec_issued_flops counts the tiles that the contraction kernels multiply, those that fill
up a slot or a group without holding a tuple among them."""
import pytest

pytestmark = pytest.mark.gpu


def _issued_tiles(N, order, nb, precision, batch=1):
    import paper_1904_11055_amd as ps
    plan = ps.Plan(N, order, nb, 0.25, precision=precision, batch=batch, device="cuda:0")
    flops = ps.polyspec_issued_flops(plan.handle, "contract")
    candidates = plan.candidates()[0] - 1
    plan.close()
    return flops / (512.0 * (1 if precision == 0 else 3) * batch * N ** 3), candidates


def _pair_tiles(candidates):
    """(A block, B block) of the pair products of order 4, pairs (i <= j) numbered by j, then i."""
    i, j, k, l = candidates.T.astype(int)
    return {(a, b) for a, b in zip((j * (j + 1) // 2 + i) // 16, (l * (l + 1) // 2 + k) // 16)}


@pytest.mark.parametrize("nb,batch", [(12, 2), (24, 1), (28, 1), (31, 1), (40, 1)])
def test_order4_fp16(gpu, nb, batch):
    """Slots of two aligned A blocks up to 28 pair blocks (always multiplied together), of four
    above (multiplied by twos): either way the twos that hold a tile."""
    got, candidates = _issued_tiles(64, 4, nb, 2, batch)
    assert got == 2 * len({(a // 2, b) for a, b in _pair_tiles(candidates)})


@pytest.mark.parametrize("precision", [0, 1])
def test_order4_other_precisions(gpu, precision):
    got, candidates = _issued_tiles(64, 4, 24, precision)
    assert got == len(_pair_tiles(candidates))


def _aligned_operands(candidates):
    """Product operand -> shell blocks of its tiles, with the operands as the order-3 kernel lays
    them out: (kind, wave), a candidate's middle shell j deciding the kind."""
    used = {}
    for i, j, k in candidates.astype(int):
        ib, jb, kb, jl = i // 16, j // 16, k // 16, j % 16
        if jb == 1 and ib == 0:
            key, column = ("low", j), kb
        elif jb == 2 and kb == 3:
            key, column = ("high", j), ib
        else:
            a = jl if jb <= 1 else 15 - jl       # rows i <= j, or k >= j mirrored
            column = kb if jb <= 1 else ib
            # two shells whose rows add up to 16 share an operand; the half-full ones of two
            # blocks share one whose tiles go to two waves
            key = ("shared", jb // 2, column // 2) if a == 7 else ("diag", jb, min(a, 14 - a) if a < 15 else 15)
        used.setdefault(key, set()).add(column)
    return used


@pytest.mark.parametrize("precision,nb", [(0, 14), (1, 14), (2, 9), (2, 24), (2, 40), (2, 53), (2, 64)])
def test_order3_aligned(gpu, precision, nb):
    """Which column blocks one product operand takes together: blocks 0 and 1, or 1 to 3, or all,
    by its kind.  64 shells use every operand."""
    got, candidates = _issued_tiles(64, 3, nb, precision)
    n_blk = (nb + 15) // 16
    want = 0
    for key, columns in _aligned_operands(candidates).items():
        if key[0] == "low":
            group = {1, 2}
        elif key[0] == "high":
            group = {0, 1, 2}
        elif key[0] == "shared":
            group = {2 * key[2], 2 * key[2] + 1}
        else:
            group = [{0, 1}, {1, 2, 3}, {0, 1, 2}, {0, 1, 2, 3}][key[1]]
        group = {c for c in group if c < n_blk}
        alone = columns - group                  # the corner tiles
        want += len(alone) + (len(group) if columns & group else 0)
    assert got == want


@pytest.mark.parametrize("order,nb,precision", [(2, 20, 0), (3, 24, 0), (3, 24, 1)])
def test_pair_tiles(gpu, order, nb, precision):
    got, candidates = _issued_tiles(64, order, nb, precision)
    c = candidates.astype(int)
    a = c[:, 0] // 16 if order == 2 else (c[:, 1] * (c[:, 1] + 1) // 2 + c[:, 0]) // 16
    assert got == len(set(zip(a, c[:, -1] // 16)))
