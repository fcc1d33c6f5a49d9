"""GPU tests of the energy that amh_grad returns: the digits it keeps."""
import math

import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

import gpu_util as gu  # noqa: E402  (an import error fails the run)


def _flat_energy(L, y0, yn, B=1):
    """V by amh_grad of a compact conformation whose pairs all lie below the first knot, where
    pair r has the energy y0[r] (yn[r] beyond the last knot), and the table's y0."""
    w = sy.CFG1.replace(L=L, n_chains=1, protein_seed=L, noise_seed=L + 1)
    s_ref = sy.reference_torsions(L, L)
    P = L * (L - 1) // 2
    y = np.zeros((P, w.n_bins), dtype=np.float32)
    y[:, :-1] = np.asarray(y0, dtype=np.float32)[:, None]
    y[:, -1] = yn
    ctx = gu.context(w, y, d_min=1e5)
    V, g = ctx.grad(torch.from_numpy(np.tile(s_ref, (B, 1))).to(gu.DEV))
    V, g = V.cpu().numpy(), g.cpu().numpy()
    ctx.poll()
    ctx.close()
    assert np.all(g == 0.0) and np.all(V == V[0])
    return V[0], y[:, 0].astype(np.float64)


@pytest.mark.parametrize("L", [2, 3, 9, 65, 130])
@pytest.mark.parametrize("scale", [1e-6, 1.0, 1e3])
def test_gradient_energies_keep_every_digit(L, scale):
    """Energies of pairs far smaller and far larger than their no-contact values: the sum is the
    exact one (math.fsum) rounded once.  Terms are held to multiples of 2^-70, 2^-71 each at
    most, and the last sum is rounded to half an ulp."""
    gu.say("energies of the gradient, L", L, "scale", scale)
    rng = np.random.Generator(np.random.PCG64(L))
    P = L * (L - 1) // 2
    V, e = _flat_energy(L, scale * rng.random(P), 3.0 + rng.random(P))
    exact = math.fsum(e)
    assert abs(V - exact) <= np.spacing(abs(exact)) + P * 2.0**-71


@pytest.mark.parametrize("L", [2, 9, 65, 130])
@pytest.mark.parametrize("scale", [7e4, 1e10, 1e17, 1e30])
def test_gradient_energies_of_any_size(L, scale):
    """Finite energies far beyond those of a probability (walls), some pairs' and all: no numeric
    error, the sum of Neumaier's compensated order (an ulp) and the same for every launch."""
    gu.say("large energies of the gradient, L", L, "scale", scale)
    rng = np.random.Generator(np.random.PCG64(L))
    P = L * (L - 1) // 2
    for share in (0.1, 1.0):
        y0 = np.where(rng.random(P) < share, scale, 1.0) * (1.0 + rng.random(P))
        y0[0] = scale
        for B in (1, 600):
            V, e = _flat_energy(L, y0, 3.0 + rng.random(P), B)
            exact = math.fsum(e)
            assert abs(V - exact) <= 2 * np.spacing(exact)
