"""Limits of the on-chip Krylov runs: what an instance of the kernel holds,
and what happens when a run cannot have the chip, its memory or its time.

Bars as in the parity tests: 1e-9 (FP64, stop 1e-12), 1e-8 (mixed, 1e-10).
"""
import os
import re
import threading
import time

import pytest

from test_gpu_chip import D, _blocks, _pf, _rel, _solve, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _opts(pf, mixed, **kw):
    return pf.pf_lin_opts_default(rel_tol=1e-10 if mixed else 1e-12,
                                  precision=pf.PF_MIXED if mixed else pf.PF_FP64, **kw)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("kind", ["none", "class"])
def test_batch_of_fields_with_different_numbers_of_values(kind, mixed):
    """A two-valued member of 16 planes per tile beside members of three and
    four values, whose classes do not fit that instance: each iterates on its
    own operator, so it takes the iterations and refinements it takes alone, but
    for rounding (another partition adds up in another order: a few iterations,
    or one restart from a true residual just above the stop)."""
    pf = _pf()
    made = [_blocks(*s, (D,) * 6, v, seed=9 + v) for s, v in
            (((113, 113, 113), 2), ((33, 35, 37), 4), ((49, 50, 47), 3), ((41, 33, 29), 2))]
    grids = [pf.grid_from_problem(m[0]) for m in made]
    sig = [dev(m[1][kind]) for m in made]
    bs = [dev(m[2]) for m in made]
    xs = [torch.zeros_like(b) for b in bs]
    print("batch", kind, mixed, flush=True)
    infos = pf.pf_linear_solve_batch(grids, sig, bs, xs, _opts(pf, mixed, max_iter=4000))
    for m, s, b, x, info in zip(made, sig, bs, xs, infos):
        g = pf.grid_from_problem(m[0])
        one = pf.pf_linear_solve(g, s, b, torch.zeros_like(b), _opts(pf, mixed, max_iter=4000))
        assert info["status"] == 0 and info["fp64_fallback"] == one["fp64_fallback"]
        assert info["iters"] <= 1.5 * one["iters"] and info["refinements"] <= one["refinements"] + 1
        assert _rel(x.cpu().numpy(), _solve(pf, g, s, b, mixed, chip=False)) <= (1e-8 if mixed else 1e-9)


# polls of a wait: 0 gives up before the run, the others at a late neighbour
# somewhere in it, not necessarily in every tile
@pytest.mark.parametrize("spin", [0, 1, 2, 4, 12])
@pytest.mark.parametrize("mixed", [False, True])
def test_run_that_gives_up_waiting_is_done_again(spin, mixed, monkeypatch, capfd):
    """Tiles of 4 planes, of 8 with sums in two levels, and of 16, alone and as
    a batch: with few polls allowed, tiles leave the run (every kernel ends by
    itself), and the solve gives the same solution by the two-kernel
    iteration, whatever part of x was written."""
    pf = _pf()
    made = [_blocks(*s, (D,) * 6, 2, seed=3 + i) for i, s in enumerate([(33, 35, 37), (97, 95, 97), (113, 105, 113)])]
    bs = [dev(m[2]) for m in made]
    refs = [_solve(pf, pf.grid_from_problem(m[0]), None, b, mixed, chip=False) for m, b in zip(made, bs)]
    monkeypatch.setenv("PF_LOG", "1")
    monkeypatch.setenv("PF_CHIP_SPIN", str(spin))
    bar = 1e-8 if mixed else 1e-9
    for m, b, ref in zip(made, bs, refs):
        monkeypatch.setenv("PF_CHIP", "1")   # no pause after a give-up
        print("alone", m[0].nx, spin, mixed, flush=True)
        assert _rel(_solve(pf, pf.grid_from_problem(m[0]), None, b, mixed), ref) <= bar
    print("batch", spin, mixed, flush=True)
    monkeypatch.setenv("PF_CHIP", "1")
    xs = [torch.zeros_like(b) for b in bs]
    infos = pf.pf_linear_solve_batch([pf.grid_from_problem(m[0]) for m in made], [None] * 3, bs, xs, _opts(pf, mixed))
    for x, ref, info in zip(xs, refs, infos):
        assert info["status"] == 0 and _rel(x.cpu().numpy(), ref) <= bar
    if spin == 0:
        assert capfd.readouterr().err.count("gave up waiting") >= 6   # every run, restarts included


def test_runs_fit_the_compute_units_there_are(monkeypatch, capfd):
    """A device (or partition) of 32 compute units holds at most 32 tiles that
    can wait for each other: small grids take fewer tiles, larger ones the
    two-kernel iteration; a batch with more tiles than the device runs them in
    turn."""
    pf = _pf()
    made = [_blocks(*s, (D,) * 6, 2, seed=i) for i, s in enumerate([(33, 35, 37), (17, 19, 23), (97, 97, 97), (41, 40, 39)])]
    bs = [dev(m[2]) for m in made]
    refs = [_solve(pf, pf.grid_from_problem(m[0]), None, b, False, chip=False) for m, b in zip(made, bs)]
    monkeypatch.setenv("PF_LOG", "1")
    monkeypatch.setenv("PF_CHIP_CUS", "32")
    capfd.readouterr()
    for m, b, ref in zip(made, bs, refs):
        print(m[0].nx, flush=True)
        assert _rel(_solve(pf, pf.grid_from_problem(m[0]), None, b, False), ref) <= 1e-9
    grids = [pf.grid_from_problem(m[0]) for m in made] + [pf.grid_from_problem(made[0][0]) for _ in range(3)]
    xs = [torch.zeros_like(b) for b in bs + [bs[0]] * 3]
    infos = pf.pf_linear_solve_batch(grids, [None] * 7, bs + [bs[0]] * 3, xs, _opts(pf, False))
    for x, ref, info in zip(xs, refs + [refs[0]] * 3, infos):
        assert info["status"] == 0 and _rel(x.cpu().numpy(), ref) <= 1e-9
    err = capfd.readouterr().err
    tiles = re.findall(r"on-chip runs of (\S+): (\d+) x (\d+) x (\d+) tiles", err)
    assert {t[0] for t in tiles} == {"33x35x37", "17x19x23", "41x40x39"} and "gave up" not in err
    assert all(int(a) * int(b) * int(c) <= 32 for _, a, b, c in tiles)


def test_device_pauses_after_a_run_that_gave_up(monkeypatch):
    """Whatever kept the tiles waiting, later runs (of any grid) do not pay for
    it again at once: 64 of them take the two-kernel iteration, then the chip
    is tried again."""
    pf = _pf()
    p, _, b = _blocks(33, 35, 37, (D,) * 6)
    b = dev(b)
    g = pf.grid_from_problem(p)

    def same(a, b):
        return a.tobytes() == b.tobytes()

    _solve(pf, g, None, b, False, chip=False)       # the launch shapes of the two-kernel iteration
    two = _solve(pf, g, None, b, False, chip=False)
    chip = _solve(pf, g, None, b, False)
    assert same(two, _solve(pf, g, None, b, False, chip=False)) and not same(two, chip)
    monkeypatch.setenv("PF_CHIP_SPIN", "0")
    _solve(pf, pf.grid_from_problem(p), None, b, False)
    monkeypatch.delenv("PF_CHIP_SPIN")
    took = 0
    while same(_solve(pf, g, None, b, False), two):
        took += 1
        assert took <= 64
    assert took >= 32       # (a solve is one run or a few)
    assert same(chip, _solve(pf, g, None, b, False))


@pytest.mark.parametrize("most", [0, 400_000])
def test_runs_without_exchange_memory_take_the_two_kernel_iteration(most, monkeypatch, capfd):
    """Where the exchange memory of a run cannot be had, the solve goes on
    without it, alone and in a batch (whose other members stay on chip)."""
    pf = _pf()
    made = [_blocks(*s, (D,) * 6, 2, seed=20 + i) for i, s in enumerate([(65, 60, 63), (9, 9, 9), (113, 105, 113)])]
    bs = [dev(m[2]) for m in made]
    monkeypatch.setenv("PF_LOG", "1")
    for mixed, bar in ((False, 1e-9), (True, 1e-8)):
        refs = [_solve(pf, pf.grid_from_problem(m[0]), None, b, mixed, chip=False) for m, b in zip(made, bs)]
        monkeypatch.setenv("PF_CHIP_MEM", str(most))
        capfd.readouterr()
        for m, b, ref in zip(made, bs, refs):
            print("alone", m[0].nx, most, mixed, flush=True)
            assert _rel(_solve(pf, pf.grid_from_problem(m[0]), None, b, mixed), ref) <= bar
        print("batch", most, mixed, flush=True)
        xs = [torch.zeros_like(b) for b in bs]
        infos = pf.pf_linear_solve_batch([pf.grid_from_problem(m[0]) for m in made], [None] * 3, bs, xs, _opts(pf, mixed))
        for x, ref, info in zip(xs, refs, infos):
            assert info["status"] == 0 and _rel(x.cpu().numpy(), ref) <= bar
        err = capfd.readouterr().err
        assert "run of 113x105x113 has no exchange memory" in err and "run of 65x60x63 has no exchange memory" in err
        assert ("run of 9x9x9 has no exchange memory" in err) == (most == 0)
        monkeypatch.delenv("PF_CHIP_MEM")


def test_grown_exchange_memory_replaces_the_old():
    """FP64 runs take twice the exchange memory of FP32 runs (97^3: about 5 and
    10 MB).  In whichever order a grid first needs them, it ends with the same
    memory."""
    pf = _pf()
    p, _, b = _blocks(97, 97, 97, (D,) * 6)
    b = dev(b)
    x = torch.zeros_like(b)
    opts = {m: pf.pf_lin_opts_default(rel_tol=1e-3, precision=pf.PF_MIXED if m else pf.PF_FP64) for m in (False, True)}

    def used(order):
        g = pf.grid_from_problem(p)
        for m in (True, False):     # workspaces of both precisions, without the chip
            os.environ["PF_CHIP"] = "0"
            try:
                pf.pf_linear_solve(g, None, b, x.zero_(), opts[m])
            finally:
                os.environ.pop("PF_CHIP")
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        for m in order:
            pf.pf_linear_solve(g, None, b, x.zero_(), opts[m])
        torch.cuda.synchronize()
        return before - torch.cuda.mem_get_info()[0]

    used((False, True))             # what the first use of the kernels themselves takes
    large_first, small_first = used((False, True)), used((True, False))
    print("exchange memory", large_first, small_first, flush=True)
    assert 0 < large_first and small_first <= large_first + (2 << 20)


def test_threads_share_the_chip():
    """Solves of several threads, each with its own grid: small runs side by
    side (33x35x37 takes 90 of 256 tiles, so two fit), large ones in their turn,
    every solution bit for bit the one of the solve by itself."""
    pf = _pf()
    shapes = [(33, 35, 37), (33, 35, 37), (17, 19, 23), (97, 97, 97), (41, 40, 39), (113, 105, 113)]
    made = [_blocks(*s, (D,) * 6, 2, seed=i) for i, s in enumerate(shapes)]
    grids = [pf.grid_from_problem(m[0]) for m in made]
    bs = [dev(m[2]) for m in made]
    refs = [_solve(pf, g, None, b, False) for g, b in zip(grids, bs)]
    bad = []

    def work(i):
        x = torch.zeros_like(bs[i])
        for _ in range(6):
            x.zero_()
            torch.cuda.current_stream().synchronize()
            pf.pf_linear_solve(grids[i], None, bs[i], x, _opts(pf, False))
            if x.cpu().numpy().tobytes() != refs[i].tobytes():
                bad.append(shapes[i])

    def run(jobs):
        ts = [threading.Thread(target=f, args=a) for f, a in jobs]
        t = time.perf_counter()
        for th in ts:
            th.start()
        for th in ts:
            th.join()
        return time.perf_counter() - t

    print("threads", flush=True)
    run([(work, (i,)) for i in range(len(shapes))])
    assert not bad

    neg = [-b for b in bs[:2]]      # (no work on the default stream between the solves)

    def many(i, x):
        for _ in range(40):
            pf.pf_linear_solve(grids[i], None, bs[i], x, _opts(pf, False, max_iter=100), check=False)
            pf.pf_linear_solve(grids[i], None, neg[i], x, _opts(pf, False, max_iter=100), check=False)

    x0, x1 = torch.zeros_like(bs[0]), torch.zeros_like(bs[1])
    ratio = []
    for _ in range(3):
        one = run([(many, (0, x0))]) + run([(many, (1, x1))])
        ratio.append(run([(many, (0, x0)), (many, (1, x1))]) / one)
    print("two threads / one after the other", ratio, flush=True)
    assert sorted(ratio)[1] <= 0.75       # 0.5 where they overlap in full, about 0.9 in turn


@pytest.mark.parametrize("mixed", [False, True])
def test_run_cut_at_the_iterations_of_a_launch_goes_on(mixed, monkeypatch):
    """A launch ends after a number of iterations.  The solve goes on from the
    true residual as often as it takes, to the caller's limit of iterations:
    not counted as restarts, refinements or stalled runs, of which a few end a
    solve."""
    pf = _pf()
    p, _, b = _blocks(33, 35, 37, (D,) * 6)
    b = dev(b)
    ref = _solve(pf, pf.grid_from_problem(p), None, b, mixed, chip=False)
    monkeypatch.setenv("PF_CHIP_RUN", "24")
    g = pf.grid_from_problem(p)
    for batch in (False, True):
        x = torch.zeros_like(b)
        opts = _opts(pf, mixed, max_iter=20000)
        print("batch", batch, mixed, flush=True)
        if batch:
            info = pf.pf_linear_solve_batch([g], [None], [b], [x], opts)[0]
        else:
            info = pf.pf_linear_solve(g, None, b, x, opts)
        assert info["status"] == 0 and info["restarts"] <= 2 and info["refinements"] <= 6 and not info["fp64_fallback"]
        assert _rel(x.cpu().numpy(), ref) <= (1e-8 if mixed else 1e-9)
    # a few iterations a launch make next to no progress: the limit ends it, nothing else
    monkeypatch.setenv("PF_CHIP_RUN", "2")
    with pytest.raises(pf.PfError) as e:
        pf.pf_linear_solve(g, None, b, torch.zeros_like(b), _opts(pf, False, max_iter=60))
    assert e.value.code == pf.PF_ERR_NOCONV and "after 60 iterations" in str(e.value)
