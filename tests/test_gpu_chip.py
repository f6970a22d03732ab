"""Krylov runs on chip (one launch per run, the vectors in registers and LDS)
against the CPU oracle and against the two-kernel iteration (PF_CHIP=0).

Both sides stop at a true relative residual of 1e-12 (mixed: 1e-10), so their
solutions differ by the operator's amplification of that residual; the bars are
the ones of the parity tests, 1e-9 (FP64) and 1e-8 (mixed).
"""
import os

import numpy as np
import pytest

import oracle
from paper_1711_04060_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

D, NM = oracle.DIRICHLET, oracle.NEUMANN


def _pf():
    from paper_1711_04060_amd import pf
    pf.load()
    return pf


def dev(a):
    return None if a is None else torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _blocks(nx, ny, nz, bc, values=2, seed=5, h=0.37):
    """Piecewise-constant dielectric of `values` values in random blocks, a few
    FIXED nodes, random right-hand side, and the three kinds of shift."""
    rng = np.random.default_rng(seed)
    N = nx * ny * nz
    pal = np.array([2.0, 78.45, 20.0, 5.0])[:values]
    kz, ky, kx = (np.arange(n) // max(2, n // 4) for n in (nz, ny, nx))
    blk = rng.integers(0, values, size=(kz.max() + 1, ky.max() + 1, kx.max() + 1))
    which = blk[kz[:, None, None], ky[None, :, None], kx[None, None, :]].reshape(-1)
    typ = np.where(which == 0, oracle.SOLUTE, 0).astype(np.uint8)
    typ[rng.choice(N, 5, replace=False)] = oracle.FIXED
    p = inputs.Problem(name="blocks", nx=nx, ny=ny, nz=nz, h=h, origin=(0, 0, 0), eps=pal[which], node_type=typ,
                       fixed_charge=np.zeros(N), bc_phi=tuple(bc), bc_value=(0.5, -1, 2, 0, 1.5, -0.25),
                       fixed_value=rng.normal(size=N))
    sigma = {"none": None, "class": np.where(which == 1, 3.0, 0.0), "node": np.where(which == 1, rng.uniform(0, 9, N), 0.0)}
    return p, sigma, rng.normal(size=N) * 50


def _solve(pf, g, sigma, b, mixed, chip=True):
    x = torch.zeros_like(b)
    opts = pf.pf_lin_opts_default(rel_tol=1e-10 if mixed else 1e-12, precision=pf.PF_MIXED if mixed else pf.PF_FP64)
    if not chip:
        os.environ["PF_CHIP"] = "0"
    try:
        info = pf.pf_linear_solve(g, sigma, b, x, opts)
    finally:
        os.environ.pop("PF_CHIP", None)
    assert info["status"] == 0
    return x.cpu().numpy()


# the smallest grids, one unknown thick, tiles of every number of planes (4, 8,
# 16: the last only without a shift per node), ragged edges, columns of tiles
# along one axis, mirror faces on every side
SMALL = [(3, 3, 3, (D,) * 6), (5, 4, 3, (NM,) * 5 + (D,)), (4, 29, 31, (D, D, NM, NM, D, D)),
         (37, 23, 19, (NM, NM, D, D, D, NM)), (130, 5, 9, (D,) * 6), (7, 131, 6, (NM, D, NM, D, NM, D)),
         (6, 7, 133, (NM, NM, NM, NM, D, D))]


@pytest.mark.parametrize("sigma", ["none", "class", "node"])
@pytest.mark.parametrize("shape", SMALL, ids=lambda s: f"{s[0]}x{s[1]}x{s[2]}")
def test_on_chip_solve_matches_oracle(shape, sigma):
    pf = _pf()
    nx, ny, nz, bc = shape
    for values in (2, 4):
        p, sig, b = _blocks(nx, ny, nz, bc, values)
        print(p.nx, p.ny, p.nz, sigma, values, flush=True)
        ref, _ = oracle.linear_solve(p, sig[sigma], b, tol=1e-13)
        g = pf.grid_from_problem(p)
        assert _rel(_solve(pf, g, dev(sig[sigma]), dev(b), False), ref) <= 1e-9
        assert _rel(_solve(pf, g, dev(sig[sigma]), dev(b), True), ref) <= 1e-8


# sizes about the switches of the tiles' planes, and the largest grids that fit
LARGE = [(49, 50, 47, "node", 2), (66, 63, 65, "class", 3), (73, 89, 57, "node", 2), (97, 97, 97, "node", 4),
         (99, 101, 97, "none", 2), (113, 105, 121, "class", 2), (129, 129, 129, "class", 2), (129, 130, 131, "none", 2)]


@pytest.mark.parametrize("case", LARGE, ids=lambda c: "%dx%dx%d-%s-%d" % c)
def test_on_chip_solve_matches_two_kernel_iteration(case):
    pf = _pf()
    nx, ny, nz, sigma, values = case
    bc = (NM, NM, NM, NM, D, D) if sigma == "node" else (D,) * 6
    p, sig, b = _blocks(nx, ny, nz, bc, values)
    g = pf.grid_from_problem(p)
    for mixed, bar in ((False, 1e-9), (True, 1e-8)):
        print(case, mixed, flush=True)
        got = _solve(pf, g, dev(sig[sigma]), dev(b), mixed)
        assert _rel(got, _solve(pf, g, dev(sig[sigma]), dev(b), mixed, chip=False)) <= bar


def test_on_chip_batch_matches_single_solves():
    """Members of different sizes, shifts and numbers of planes per tile in one
    batch, one that does not fit (a field of many values), and batches whose
    exchange buffers serve several runs."""
    pf = _pf()
    shapes = [(17, 19, 23), (33, 33, 33), (65, 40, 51), (97, 97, 97), (113, 113, 113), (49, 49, 49)]
    kinds = ["none", "class", "node", "class", "class", "node"]
    made = [_blocks(*s, (D,) * 6, 2, seed=i) for i, s in enumerate(shapes)]
    probs = [m[0] for m in made]
    probs[5].eps = probs[5].eps * np.linspace(1.0, 1.1, probs[5].N)
    grids = [pf.grid_from_problem(p) for p in probs]
    sig = [dev(m[1][k]) for m, k in zip(made, kinds)]
    bs = [dev(m[2]) for m in made]
    for mixed, bar in ((False, 1e-9), (True, 1e-8), (False, 1e-9)):
        print("batch", mixed, flush=True)
        xs = [torch.zeros_like(b) for b in bs]
        opts = pf.pf_lin_opts_default(rel_tol=1e-10 if mixed else 1e-12, precision=pf.PF_MIXED if mixed else pf.PF_FP64)
        infos = pf.pf_linear_solve_batch(grids, sig, bs, xs, opts)
        for i, (g, s, b, x) in enumerate(zip(grids, sig, bs, xs)):
            assert infos[i]["status"] == 0
            assert _rel(x.cpu().numpy(), _solve(pf, g, s, b, mixed, chip=False)) <= bar, shapes[i]


def test_on_chip_runs_are_the_ones_that_run(capfd):
    pf = _pf()
    os.environ["PF_LOG"] = "1"
    try:
        p, sig, b = _blocks(33, 33, 33, (D,) * 6)
        _solve(pf, pf.grid_from_problem(p), None, dev(b), False)
        assert "on-chip runs of 33x33x33" in capfd.readouterr().err
        q, _, b = _blocks(161, 161, 161, (D,) * 6)   # more unknowns than the tiles hold
        _solve(pf, pf.grid_from_problem(q), None, dev(b), False)
        assert "on-chip runs of 161x161x161" not in capfd.readouterr().err
    finally:
        os.environ.pop("PF_LOG", None)


def test_on_chip_iteration_limit_and_non_finite_input():
    """A run that stops at its iteration limit returns the iterate so far; a
    non-finite right-hand side ends with its own error, as before."""
    pf = _pf()
    p, sig, b = _blocks(33, 35, 37, (D,) * 6)
    g = pf.grid_from_problem(p)
    x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
    with pytest.raises(pf.PfError) as e:
        pf.pf_linear_solve(g, None, dev(b), x, pf.pf_lin_opts_default(rel_tol=1e-12, max_iter=7))
    assert e.value.code == pf.PF_ERR_NOCONV
    assert torch.isfinite(x).all() and float(x.abs().max()) > 0
    b2 = dev(b)
    b2[p.N // 2] = float("nan")
    with pytest.raises(pf.PfError) as e:
        pf.pf_linear_solve(g, None, b2, x)
    assert e.value.code == pf.PF_ERR_NONFINITE
    assert _rel(_solve(pf, g, None, dev(b), False), _solve(pf, g, None, dev(b), False, chip=False)) <= 1e-9
