"""How far a float V-cycle is from the exact one, against other float arithmetic of the same cycle.

The error of a float cycle is the rounding of its sums: how a kernel groups the
neighbours of a node, and which residuals it forms, decide it.  Each test
compares the error of every mode with that of a reference in float (the
row-phase kernels, or a replay of the sweeps on the CPU) on the same input.  One mode's
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


def _fma(a, b, c):
    """fl(a b + c) in float: the product of two floats is exact in double."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def _replay_lex(tables, f, n, nu1, nu2):
    """A lexicographic P1 V-cycle in float on two levels and an exact coarsest one, plain sums: a relaxation
    subtracts the neighbours below and to the west from f, adds up the others, and multiplies by 1 / diagonal."""
    stens = [tables["fine"].astype(np.float32), tables["l1"].astype(np.float32)]
    offsets = [(dy, dx) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]

    def at(v, y, x, e):
        return v[y + 1 + offsets[e][0], x + 1 + offsets[e][1]]

    def sweep(s9, v, f, nx, reverse):
        order = [(y, x) for y in range(nx) for x in range(nx)]
        for y, x in order[::-1] if reverse else order:
            s = s9[y * nx + x]
            lo = f[y, x]
            for e in (0, 1, 2, 3):
                lo = _fma(-s[e], at(v, y, x, e), lo)
            hi = s[6] * at(v, y, x, 6)
            for e in (7, 8, 5):
                hi = _fma(s[e], at(v, y, x, e), hi)
            v[y + 1, x + 1] = (lo - hi) * (np.float32(1) / s[4])

    def cycle(f, level, nx):
        if level == len(stens):
            u = (tables["cinv"] @ f.reshape(nx * nx, -1).astype(np.float64)).astype(np.float32)
            return np.pad(u.reshape(f.shape), ((1, 1), (1, 1), (0, 0)))
        s9 = stens[level]
        v = np.zeros((nx + 2, nx + 2, f.shape[2]), dtype=np.float32)
        for _ in range(nu1):
            sweep(s9, v, f, nx, False)
        s = s9.reshape(nx, nx, 9)[..., None]
        r = f
        for e, (dy, dx) in enumerate(offsets):
            r = _fma(-s[:, :, e], v[1 + dy:1 + dy + nx, 1 + dx:1 + dx + nx], r)
        nc = (nx - 1) // 2
        fc = np.zeros((nc, nc, f.shape[2]), dtype=np.float32)
        half = np.float32(0.5)
        for dy, dx, w in ((-1, -1, half), (-1, 0, half), (0, -1, half), (0, 0, np.float32(1)), (0, 1, half), (1, 0, half),
                          (1, 1, half)):
            fc = _fma(w, r[1 + dy:nx - 1 + dy + 1:2, 1 + dx:nx - 1 + dx + 1:2], fc)
        e = cycle(fc, level + 1, nc)  # with a border of zeros
        p = np.zeros_like(f)
        p[1::2, 1::2] = e[1:-1, 1:-1]
        p[1::2, 0::2] = half * (e[1:-1, :-1] + e[1:-1, 1:])
        p[0::2, 1::2] = half * (e[:-1, 1:-1] + e[1:, 1:-1])
        p[0::2, 0::2] = half * (e[:-1, :-1] + e[1:, 1:])
        v[1:-1, 1:-1] += p
        for _ in range(nu2):
            sweep(s9, v, f, nx, True)
        return v

    nx = n - 1
    return cycle(f.reshape(nx, nx, -1), 0, nx)[1:-1, 1:-1].reshape(nx * nx, -1)


@pytest.mark.parametrize("n,coarsest", [(16, 4), (24, 6), (32, 8)])
@pytest.mark.parametrize("nu", [1, 2])
def test_lexicographic_cycle_is_no_further_off_than_plain_sums(n, coarsest, nu):
    """K_0 of the triangulation and its coarse operators are exact in float for a0 = 1: what is left is the
    order of the sums.  Grids of 15, 23 (a hierarchy that is not 2^k - 1) and 31 nodes a side."""
    import paper_1304_1755_amd as sgbt
    note(f"lexicographic float accuracy n={n} nu={nu}")
    tables = sgbt.setup_host(n, 1, 1, 0.1, corr_len=1.0, coarsest=coarsest, disc="p1")
    g = sgbt.Problem(n, 6, 4, 0.1, corr_len=1.0, nu1=nu, nu2=nu, coarsest=coarsest, colour="lex", disc="p1")
    err, ref = [], []
    for seed in (1, 2, 3, 4):
        f = _inputs(g.N, g.P, seed)
        exact = g.vcycle(f.double())
        err.append(_errors(g.vcycle(f, prec=sgbt.SG_F32), exact))
        ref.append(_errors(torch.from_numpy(_replay_lex(tables, f.cpu().numpy(), n, nu, nu)).cuda(), exact))
    g.close()
    _no_further(np.concatenate(err), np.concatenate(ref))
