"""GPU parity of the rank 64, 128 and 256 kernels (split bf16 operands) at the edges of their tiles:
rows and columns on both sides of the 32-index blocks, of the 64- and 128-index tiles, of the
1024-column decompress tiles and of a Q-step row chunk, row lengths that are not a multiple of four,
values of very different sizes, and the error against 64 bits beside that of plain fp32 products."""

import numpy as np
import pytest
import torch

import synthgrad as sg
from tests import parity_util as PU
from tests.test_gpu_powersgd import run_psgd_parity
from tests.test_gpu_state import _grouped_vs_per_bucket

pytestmark = pytest.mark.gpu


def _shapes(rank):
    """Sides of at least twice the rank (a factor close to square is ill-conditioned)."""
    lo = 2 * rank
    return [(lo, lo + 1), (lo + 31, lo + 32), (5,), (lo + 33, lo + 63), (lo + 65, lo + 127), (lo + 129, lo + 2),
            (3,), (lo + 96, 1023), (lo, 1025), (2049 + (512 if rank == 64 else 1), lo + 3)]


@pytest.mark.parametrize("rank", [64, 128, 256])
@pytest.mark.parametrize("ef", [True, False])
def test_tile_edges(rank, ef):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    shapes = _shapes(rank)
    params = [sg.Param(f"t{i}", s) for i, s in enumerate(shapes)]
    wl = sg.Workload("edges", params, rank, 4, lambda p: 0.05, seed=8, cap_bytes=1 << 20)
    rep = PU.run_parity(wl, "fresh", 4, range(1, 5), list(range(len(shapes))), ef=ef, free=2, grouped=not ef)
    assert not rep.failures, "\n".join(rep.failures[:20])


def test_powersgd_tile_edges():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    shapes = _shapes(64)
    wl = sg.Workload("edges", [sg.Param(f"t{i}", s) for i, s in enumerate(shapes)], 64, 3, lambda p: 0.05, seed=9,
                     cap_bytes=1 << 20)
    rep = run_psgd_parity(wl, 3, list(range(len(shapes))), free=2)
    assert not rep.failures, "\n".join(rep.failures[:20])


@pytest.mark.parametrize("rank", [64, 256])
@pytest.mark.parametrize("scale,spread", [(1.0, 3), (1e-12, 3), (1e12, 3), (1e-30, 3), (1e33, 3), (1e-33, 0)])
def test_error_is_that_of_fp32(rank, scale, spread):
    """One P-step and its decompress on a matrix whose entries span six orders of magnitude (or one, at
    a scale where the lowest parts of the split values are bf16 subnormals): the split products are as
    close to 64 bits as fp32 products (CPU, fp32 accumulation) of the same operands, within a factor
    of 1.5 for the order of the sums."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    n, m = 600, 1100
    rng = np.random.default_rng(4)
    g = (scale * rng.standard_normal((n, m)) * 10.0 ** rng.uniform(-spread, spread, (n, m))).astype(np.float32)
    run = PU.Runner([(n, m)], rank)
    run.step(1, run.pack({0: g}))
    torch.cuda.synchronize()
    p, hat, q = run.factor_slice(1, 0).reshape(n, rank), run.out_slice(0).reshape(n, m), run.ortho(1, 0).reshape(m, rank)
    for x, a, b in ((p, g, q), (hat, p, np.ascontiguousarray(q.T))):
        exact = a.astype(np.float64) @ b.astype(np.float64)
        plain = np.zeros(exact.shape, np.float32)
        for k in range(a.shape[1]):  # one rounding per term, as a chain of fp32 multiply-adds has
            plain += a[:, k:k + 1] * b[k:k + 1, :]
        assert PU.rel_err(x, exact) <= 1.5 * PU.rel_err(plain, exact)
    # the decompress adds all small products first: r / 16 roundings of the large sum, each at most
    # 2^-24 of it and of either sign, stay below two of them together
    assert PU.rel_err(hat, p.astype(np.float64) @ q.astype(np.float64).T) <= 2.0 ** -23


@pytest.mark.parametrize("rank", [64, 128, 256])
def test_largest_values(rank):
    """Values between the largest bf16 and the largest fp32 stay finite; an infinity or NaN makes its
    own row of P not finite and no other."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    n, m = 600, 700
    rng = np.random.default_rng(6)
    g = (1e30 * rng.standard_normal((n, m))).astype(np.float32)
    g[rng.integers(0, n, 40), rng.integers(0, m, 40)] = np.float32(3.4e38)
    g[rng.integers(0, n, 40), rng.integers(0, m, 40)] = np.float32(-3.395e38)

    def p_of(grad):
        run = PU.Runner([(n, m)], rank)
        run.step(1, run.pack({0: grad}))
        torch.cuda.synchronize()
        return (run.factor_slice(1, 0).reshape(n, rank), run.out_slice(0).reshape(n, m),
                run.ortho(1, 0).reshape(m, rank))

    p, hat, q = p_of(g)
    # fp32 sums of at most 700 products: 1e-5 is far above their error, far below a lost part's
    assert PU.rel_err(p / 1e38, (g.astype(np.float64) / 1e38) @ q.astype(np.float64)) < 1e-5
    assert PU.rel_err(hat / 1e38, (p.astype(np.float64) / 1e38) @ q.astype(np.float64).T) < 1e-5
    bad = g.copy()
    bad[17, 3], bad[130, 699] = np.inf, np.nan
    pb = p_of(bad)[0]
    rows = np.isfinite(pb).all(axis=1)
    assert np.flatnonzero(~rows).tolist() == [17, 130] and not np.isfinite(pb[~rows]).any()
    assert np.array_equal(pb[rows], p[rows])


def sums_shapes(rank):
    """Enough of them that all-bucket launches fill the GPU (see test_plan_host.py)."""
    return [(12000, 600), (77,), (600, 12000)] * (12 if rank == 64 else 6)


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128, 256])
def test_split_sums_agree_between_calls(rank):
    """Per-bucket calls, whose launches are too small to fill the GPU and split every sum into
    parts, against all-bucket calls over enough buckets that they do not (at rank 256 both take a
    tile per part): the same bits."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    shapes = sums_shapes(rank)
    rng = np.random.default_rng(2)
    base = {i: (0.02 * rng.standard_normal(s)).astype(np.float32) for i, s in enumerate(shapes[:3])}

    def grads_of(t):
        return {i: np.roll(base[i % 3], 7 * t + i).reshape(s) for i, s in enumerate(shapes)}

    _grouped_vs_per_bucket(shapes, rank, grads_of, 4)
