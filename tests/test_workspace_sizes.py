"""The workspaces that the eigensolver, the Jacobi filter and the multilevel
eigensolver ask for: what the calls carve from them, in 256-byte steps, and
not much more."""
import os

import pytest

MIB = 1 << 20
BLOCK = 64          # widest block of columns
LEVELS = 32         # of a hierarchy at most


def _G():
    from paper_1812_08942_amd import build, graphreduce

    if not os.path.exists(graphreduce.LIB_PATH):
        build.build(force=False)
    return graphreduce


def _carved(*sizes):
    return sum((s + 255) // 256 * 256 for s in sizes)


def _operator(n):
    # degrees and inverses; long rows; their flags and places, the scan's tiles
    return _carved(8 * (n + 1), 8 * (n + 1), 4 * (n + 1), 4 * n, 4 * (n + 1),
                   4 * (n // 2048 + 1), 4 * (n // 2048 + 1))


def _eig(n):
    return _operator(n) + _carved(
        *[8 * (n * BLOCK + 1)] * 4, 8 * 128 * BLOCK * BLOCK, *[8 * BLOCK * BLOCK] * 2,
        *[8 * BLOCK] * 3, 8 * 8, 4 * 4, 8 * (n + 1), 8 * (n + 1), 8 * 8)


def _jacobi(n, k):
    return _operator(n) + _carved(8 * (n * k + 1), 8 * k)


SIZES = [2, 255, 20000, 1000003, 16777216]


@pytest.mark.parametrize("n", SIZES)
def test_eigensolver(n):
    need, got = _eig(n), _G().gr_eig_workspace(n, 32)
    assert need <= got <= 1.1 * need + 2 * MIB


@pytest.mark.parametrize("k", [1, 10, 64])
@pytest.mark.parametrize("n", SIZES)
def test_jacobi_filter(n, k):
    need, got = _jacobi(n, k), _G().gr_jacobi_workspace(n, k)
    assert need <= got <= 1.1 * need + 2 * MIB


@pytest.mark.parametrize("k", [1, 32])
@pytest.mark.parametrize("n", SIZES)
def test_multilevel(n, k):
    # B of every level, however slowly they shrink, the two vector blocks,
    # degrees; then one phase after another
    held = _carved(*[8 * (n + 1)] * (LEVELS + 2), *[8 * (n * k + 1)] * 2)
    need, got = held + max(_eig(n), _jacobi(n, k)), _G().gr_multilevel_workspace(n, 6 * n, k)
    assert need <= got <= 1.2 * need + 4 * MIB
