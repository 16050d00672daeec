"""How far a float V-cycle is from the exact one, against other float arithmetic of the same cycle.

The error of a float cycle is the rounding of its sums: how a kernel groups the
neighbours of a node, and which residuals it forms, decide it.  Each test
compares the error of every mode with that of the row-phase
kernels on the same input.  One mode's
ratio is chance; the mean logarithm over the modes must not lie above zero by more than
twice its own standard error.
"""

import ctypes

import numpy as np
import pytest
import torch

from gpu_util import note

pytestmark = pytest.mark.gpu


def _errors(u, exact):
    return ((u.double() - exact).norm(dim=0) / exact.norm(dim=0)).cpu().numpy()


def _no_further(err, ref):
    d = np.log(err / ref)
    mean, spread = d.mean(), d.std() / np.sqrt(d.size)
    note(f"error ratio {np.exp(mean):.4f}, standard error of its logarithm {spread:.4f}, {d.size} modes")
    assert mean <= 2 * spread


def _inputs(N, width, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((N, width), generator=gen, dtype=torch.float32, device="cuda") * 2 - 1


@pytest.mark.parametrize("disc", ["q1", "p1"])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1)])
def test_streaming_cycle_is_no_further_off_than_row_phases(disc, nu1, nu2):
    """A row stride past what the legs address takes the row-phase kernels."""
    import paper_1304_1755_amd as sgbt
    lib = sgbt.load_library()
    n, width = 256, 210
    note(f"float accuracy n={n} {disc} nu={nu1},{nu2}")
    g = sgbt.Problem(n, 6, 4, 0.1 if disc == "p1" else 0.3, corr_len=1.0 if disc == "p1" else 0.5, nu1=nu1, nu2=nu2,
                     coarsest=8, disc=disc)
    ld = 2 ** 32 // (80 * 4 * (n - 1)) + 1
    wide = torch.empty(((g.N - 1) * ld + width,), dtype=torch.float32, device="cuda")  # 14 GB, a few columns of it used
    rows = torch.as_strided(wide, (g.N, width), (ld, 1))
    err, ref = [], []
    for seed in (1, 2):
        f = _inputs(g.N, width, seed)
        exact = g.vcycle(f.double())
        err.append(_errors(g.vcycle(f, prec=sgbt.SG_F32), exact))
        code = lib.sg_vcycle(g._ctx, ctypes.c_void_p(f.data_ptr()), width, ctypes.c_void_p(wide.data_ptr()), ld, width,
                             sgbt.SG_F32)
        assert code == sgbt.SG_OK
        ref.append(_errors(rows, exact))
    g.close()
    _no_further(np.concatenate(err), np.concatenate(ref))
