"""The first call of a kind on a grid shape, which times launch shapes before it
does its work: refused input stays refused, results are those of later calls.
(Sizes that no other test uses: the shapes are kept per size.)"""
import numpy as np
import pytest

import oracle
from test_gpu_chip import D, _blocks, _pf, _rel, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _field_of_many_values(nx, ny, nz):
    """No palette, so the two-kernel iteration, whose launch shapes are timed."""
    p, sig, b = _blocks(nx, ny, nz, (D,) * 6)
    p.eps = p.eps * np.linspace(1.0, 1.1, p.N)
    return p, sig, b


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
def test_negative_shift_is_refused_on_first_use(mixed, batch):
    pf = _pf()
    p, sig, b = _field_of_many_values(27 + mixed, 22 + batch, 25)
    s = sig["node"].copy()
    inner = [i for i in range(p.N // 2, p.N) if p.node_type[i] != oracle.FIXED and 0 < i % p.nx < p.nx - 1
             and 0 < i // p.nx % p.ny < p.ny - 1]
    s[inner[0]] = -1e-3     # one free row
    g = pf.grid_from_problem(p)
    opts = pf.pf_lin_opts_default(max_iter=50, precision=pf.PF_MIXED if mixed else pf.PF_FP64)
    x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
    for use in range(2):
        print("use", use, flush=True)
        if batch:
            info = pf.pf_linear_solve_batch([g], [dev(s)], [dev(b)], [x], opts, check=False)
            assert info[0]["status"] == pf.PF_ERR_ARG
        else:
            with pytest.raises(pf.PfError) as e:
                pf.pf_linear_solve(g, dev(s), dev(b), x, opts)
            assert e.value.code == pf.PF_ERR_ARG
    # and the same shift without the sign solves
    ref, _ = oracle.linear_solve(p, np.abs(s), b, tol=1e-13)
    x.zero_()
    pf.pf_linear_solve(g, dev(np.abs(s)), dev(b), x, pf.pf_lin_opts_default(rel_tol=1e-12))
    assert _rel(x.cpu().numpy(), ref) <= 1e-9
