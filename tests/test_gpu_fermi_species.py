"""The steric root and the Fermi update for every number of species the kernel
has an instance for (2, 3, 4) and those of its general loop, against the
oracle's bisection: the root to 1e-12 (its own rounding at potentials of
+-2000), concentrations to 1e-12 (1 + |z phi|), the bars of the parity test."""
import numpy as np
import pytest

import oracle
from paper_1711_04060_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

Z = [1.0, -1.0, 0.0, 2.0, -2.0, 1.0]
R = [0.95, 1.81, 1.4, 0.99, 2.6, 3.4]          # volumes from 0.02 to 2.3 of their mean
BATH = [0.1, 0.102, 55.5, 1e-3, 0.5, 0.2]


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6])
def test_fermi_species_counts_match_oracle(n):
    from paper_1711_04060_amd import pf
    pf.load()
    m, N = 11, 11 ** 3
    rng = np.random.default_rng(n)
    phi = np.concatenate([rng.normal(0, 3, N // 2), rng.uniform(-2000, 2000, N - N // 2 - 5), [0.0, 1e-3, -1e-3, 2e3, -2e3]])
    p = inputs.Problem("f", m, m, m, 1.0, (0, 0, 0), np.full(N, 2.0), np.zeros(N, np.uint8), np.zeros(N))
    g = pf.grid_from_problem(p)
    rho, sig, S = (torch.empty(N, dtype=torch.float64, device="cuda") for _ in range(3))
    conc = torch.empty(n * N, dtype=torch.float64, device="cuda")
    pf.pf_fermi(g, pf.Params(Z[:n], R[:n], BATH[:n]), torch.as_tensor(phi, device="cuda"), rho, sig, conc, S)
    sp = oracle.species_from_molar(Z[:n], R[:n], BATH[:n])
    orho, osig, oconc, oS = oracle.fermi(phi, sp, np.zeros(N, np.uint8))
    np.testing.assert_allclose(S.cpu().numpy(), oS, rtol=1e-12, atol=1e-12)
    z = np.abs(np.asarray(Z[:n]))[:, None]
    c = conc.cpu().numpy().reshape(n, N)
    assert np.all(np.abs(c - oconc) <= 1e-12 * (1 + z * np.abs(phi)[None, :]) * np.abs(oconc) + 1e-300)
    scale = 4e-12 * (1 + 2 * np.abs(phi)) * (np.abs(osig) + 1e-300)
    assert np.all(np.abs(sig.cpu().numpy() - osig) <= scale)
    assert np.all(np.abs(rho.cpu().numpy() - orho) <= scale)
