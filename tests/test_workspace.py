"""Workspace of cells-only systems: second positions only where steps use them (small
systems without reorder; not with bonded terms, not in batches, which integrate
in a pass of their own).  Host-only calls."""
import pytest

from paper_2003_14061_amd import inputs, md


def params(n, **kw):
    return md.Params(n, md.MD_LJ_SHIFTED, inputs.box_length(n, 0.8), 1.0, 1.0, 1.0, 2 ** (1 / 6),
                     0.3, 0.005, md.MD_FP64, kw.get("mode", md.MD_CELLS_ONLY), 0, 0,
                     kw.get("reorder", 0), 256, kw.get("pipeline", 0))


def size(n, bonded=False, **kw):
    ctx = md.md_init(params(n, **kw))
    try:
        if bonded:
            md.md_set_bonded(ctx, chain_length=10)
        return md.md_workspace_bytes(ctx)
    finally:
        md.md_destroy(ctx)


def batch_size(n, **kw):
    b = md.md_batch_init([params(n, **kw)] * 3, 3)
    try:
        return int(md.lib().md_batch_workspace_bytes(b))
    finally:
        md.lib().md_batch_destroy(b)


def up(nbytes):
    return (nbytes + 255) // 256 * 256


def permuted(n):
    """What reorder adds: nine double arrays and two of int32."""
    return 9 * up(8 * n) + 2 * up(4 * n)


@pytest.mark.parametrize("n", [500, 65530, 65540, 300000])
def test_second_positions_of_one_system(n):
    second = 3 * up(8 * n) if n <= 65536 else 0
    assert size(n, reorder=1) - size(n) == permuted(n) - second


@pytest.mark.parametrize("n", [500, 4000, 300000])
def test_none_with_bonded_terms(n):
    assert size(n, reorder=1, bonded=True) - size(n, bonded=True) == permuted(n)


@pytest.mark.parametrize("n", [500, 4000, 300000])
def test_none_in_a_batch(n):
    assert batch_size(n, reorder=1) - batch_size(n) == 3 * permuted(n)


def test_bonds_removed_again():
    ctx = md.md_init(params(4000))
    before = md.md_workspace_bytes(ctx)
    md.md_set_bonded(ctx, chain_length=10)
    md.md_set_bonded(ctx, None)
    assert md.md_workspace_bytes(ctx) == before
    md.md_destroy(ctx)
