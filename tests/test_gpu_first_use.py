"""The first call of a kind on a grid shape, which times launch shapes before it
does its work: refused input stays refused, results are those of later calls.
(Sizes that no other test uses: the shapes are kept per size.)"""
import threading

import numpy as np
import pytest

import oracle
from test_gpu_chip import D, _blocks, _pf, _rel, _solve, dev

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


@pytest.mark.parametrize("kind", ["none", "class", "node"])
def test_on_chip_solve_is_the_same_whatever_was_timed_before(kind):
    """The same on-chip solve before and after calls that time launch shapes on
    its grid (residual, products, a solve by the two-kernel iteration): bit for
    bit, iterations included."""
    pf = _pf()
    p, sig, b = _blocks(38, 43, 52 + len(kind), (D,) * 6)
    s, b = dev(sig[kind]), dev(b)
    g = pf.grid_from_problem(p)
    opts = pf.pf_lin_opts_default(rel_tol=1e-12)
    out = []
    for k in range(4):
        x = torch.zeros_like(b)
        print(kind, k, flush=True)
        info = pf.pf_linear_solve(g, s, b, x, opts)
        out.append((x.cpu().numpy().tobytes(), info["iters"], info["rel_res"]))
        r, y = torch.empty_like(b), torch.empty_like(b)
        if k == 0:
            rel = pf.pf_residual(g, s, b, x, r)
            assert rel == pytest.approx(info["rel_res"], rel=1e-6)
            rn = torch.empty_like(b)
            assert pf.pf_residual_noalloc(g, s, b, x, rn) == rel and torch.equal(r, rn)
        elif k == 1:
            pf.pf_spmv(g, s, x, y, 0)
            pf.pf_spmv(g, s, x, y, 1)
        else:
            _solve(pf, g, s, b, False, chip=False)
    assert all(o == out[0] for o in out)


@pytest.mark.parametrize("mixed", [False, True])
def test_solve_that_turns_out_not_to_fit_the_chip_repeats(mixed):
    """A shift per node on a grid that would fit with one per class: the
    two-kernel iteration after all, its shapes timed in the middle of the first
    solve, which equals the second bit for bit."""
    pf = _pf()
    p, sig, b = _blocks(111, 107, 109 + mixed, (D,) * 6)
    s, b = dev(sig["node"]), dev(b)
    g = pf.grid_from_problem(p)
    out = []
    for k in range(2):
        x = torch.zeros_like(b)
        print(mixed, k, flush=True)
        info = pf.pf_linear_solve(g, s, b, x, pf.pf_lin_opts_default(
            rel_tol=1e-9, precision=pf.PF_MIXED if mixed else pf.PF_FP64))
        out.append((x.cpu().numpy().tobytes(), info["iters"], info["rel_res"]))
        assert pf.pf_residual(g, s, b, x) <= 1e-9
    assert out[0] == out[1]


def test_first_calls_of_several_threads():
    """Each thread times the launch shapes of its own grid's size; the maps that
    keep them are the process's.  (Nothing else runs in the threads: work on the
    default stream beside a solve that captures its graph is an error.)"""
    pf = _pf()
    jobs = []
    for i in range(6):
        p, sig, b = _field_of_many_values(30 + i, 21, 23)
        x = dev(np.random.default_rng(i).normal(size=p.N))
        jobs.append((pf.grid_from_problem(p), dev(sig["node"]), dev(b), x, *(torch.empty_like(x) for _ in range(3))))
    rel = [None] * len(jobs)

    def work(i):
        g, s, b, x, r, y, z = jobs[i]
        rel[i] = pf.pf_residual(g, s, b, x, r)
        pf.pf_spmv(g, s, x, y, 0)
        pf.pf_spmv(g, s, x, z, 1)

    torch.cuda.synchronize()
    print("threads", flush=True)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, (g, s, b, x, r, y, z) in enumerate(jobs):
        again = [torch.empty_like(x) for _ in range(3)]
        assert pf.pf_residual(g, s, b, x, again[0]) == rel[i]
        pf.pf_spmv(g, s, x, again[1], 0)
        pf.pf_spmv(g, s, x, again[2], 1)
        assert all(torch.equal(u, v) for u, v in zip((r, y, z), again))
