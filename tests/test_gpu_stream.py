"""Streaming V-cycle legs against the oracle's cycle, at the sizes where their split can go wrong.

Strips hold 128 columns of which 112 are kept (120 at a domain edge), segments
two to thirty-two coarse rows, lanes one, two or four modes; a level's last
panel repeats modes when the width is no multiple of that.  Tolerances: the
cycle is compared with one in another rounding order, 1e-11 relative in double
and 2e-5 in float, as for the other V-cycle forms.
"""

import functools

import numpy as np
import pytest
import torch

from gpu_util import note, rel_max, to_dev, to_host

pytestmark = pytest.mark.gpu

# (cells, coarsest): 71 and 35 nodes a side; 127 (one strip); 135 and 67 (two strips, one); 239 and 247
# (the most two strips hold, three strips); 255
GRIDS = [(72, 9), (128, 8), (136, 17), (240, 15), (248, 31), (256, 8)]


@functools.lru_cache(maxsize=4)
def _oracle(n, coarsest, nu1, nu2, disc):
    from oracle import mg, paper_mode, system
    o = paper_mode.build_problem_paper(n, 1, 1, 0.2) if disc == "p1" else system.build_problem(n, 1, 1, 0.3, 0.5)
    return mg.Hierarchy(o.K[0], n, coarsest=coarsest, nu1=nu1, nu2=nu2, transfer="p1" if disc == "p1" else "bilinear")


def _check(n, coarsest, width, prec, nu1, nu2, disc):
    import sg_inputs
    import paper_1304_1755_amd as sgbt
    note(f"stream n={n} coarsest={coarsest} width={width} prec={prec} nu={nu1},{nu2} {disc}")
    H = _oracle(n, coarsest, nu1, nu2, disc)
    g = sgbt.Problem(n, 4, 4 if width > 35 else 3, 0.2 if disc == "p1" else 0.3, corr_len=1.0 if disc == "p1" else 0.5, coarsest=coarsest,
                     nu1=nu1, nu2=nu2, disc=disc)
    f = sg_inputs.uniform_block(g.N, width, seed=n + width)
    dt = torch.float32 if prec == "f32" else torch.float64
    fd = to_dev(f, dt)
    guard = torch.full((g.N + 2, width), 7.0, dtype=dt, device="cuda")  # rows before and after the result
    u = guard[1:-1]
    g.vcycle(fd, u, prec=sgbt.SG_F32 if prec == "f32" else sgbt.SG_F64)
    ref = H.vcycle(to_host(fd))
    assert rel_max(to_host(u), ref) < (2e-5 if prec == "f32" else 1e-11)
    assert bool((guard[0] == 7.0).all()) and bool((guard[-1] == 7.0).all())
    again = torch.empty_like(fd)
    g.vcycle(fd, again, prec=sgbt.SG_F32 if prec == "f32" else sgbt.SG_F64)
    assert torch.equal(again, u)
    g.close()


@pytest.mark.parametrize("width,prec", [(1, "f32"), (3, "f32"), (7, "f32"), (21, "f32"), (34, "f32"), (1, "f64"),
                                        (3, "f64"), (8, "f64"), (35, "f64"), (40, "f32"), (47, "f32")])
@pytest.mark.parametrize("n,coarsest", GRIDS)
def test_stream_cycle_matches_oracle(n, coarsest, width, prec):
    _check(n, coarsest, width, prec, 2, 2, "q1")


@pytest.mark.parametrize("nu1,nu2", [(1, 1), (2, 1), (1, 2)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_stream_cycle_sweep_counts(nu1, nu2, prec):
    _check(136, 17, 17, prec, nu1, nu2, "q1")


@pytest.mark.parametrize("width,prec", [(2, "f32"), (18, "f32"), (5, "f64")])
def test_stream_cycle_p1(width, prec):
    _check(144, 9, width, prec, 2, 2, "p1")


def test_stream_cycle_infinity_stays_in_its_mode():
    """Modes do not mix: an infinite right-hand side spoils its own mode only."""
    import paper_1304_1755_amd as sgbt
    g = sgbt.Problem(136, 4, 3, 0.3, coarsest=17)
    gen = torch.Generator(device="cuda").manual_seed(3)
    f = torch.rand((g.N, 19), generator=gen, dtype=torch.float64, device="cuda")
    want = g.vcycle(f).clone()
    f[g.N // 2, 17] = float("inf")
    got = g.vcycle(f)
    keep = [i for i in range(19) if i != 17]
    assert torch.equal(got[:, keep], want[:, keep])
    assert not bool(torch.isfinite(got[:, 17]).all())
    g.close()


def test_preconditioners_at_odd_level_widths():
    """B_T and B_S at level widths no panel divides (1, 5 and 15 modes; 1, 4, 10 and 20) against the oracle."""
    import sg_inputs
    import paper_1304_1755_amd as sgbt
    from oracle import mg, precond, system
    note("odd levels n=72 m=5 p=2, m=4 p=3")
    for m, p in ((5, 2), (4, 3)):
        o = system.build_problem(72, m, p, 0.2, 0.5)
        H = mg.Hierarchy(o.K[0], 72, coarsest=9)
        g = sgbt.Problem(72, m, p, 0.2, coarsest=9)
        r = sg_inputs.uniform_block(g.N, g.P, seed=11)
        for kind, fn in (("tri", precond.precond_tri), ("sym", precond.precond_sym)):
            ref = fn(o, np.ascontiguousarray(r.T), H.vcycle).T
            assert rel_max(to_host(g.precond(to_dev(r), kind=kind)), ref) < 1e-11
            assert rel_max(to_host(g.precond(to_dev(r), kind=kind, prec=sgbt.SG_MIXED)), ref) < 5e-5
        g.close()


@pytest.mark.parametrize("n,coarsest", [(64, 4), (48, 3), (60, 15), (128, 8)])
@pytest.mark.parametrize("width,prec", [(1, "f64"), (5, "f64"), (3, "f32")])
def test_lexicographic_sweeps(n, coarsest, width, prec):
    """The lexicographic cycle by fronts: 63 rows (every lane but one), 47 and 23 (a hierarchy that is not
    2^k - 1), 59 and 29, and 127 (more rows than lanes: the barrier form above the fronts)."""
    import sg_inputs
    import paper_1304_1755_amd as sgbt
    from oracle import mg, system
    note(f"lex n={n} coarsest={coarsest} width={width} {prec}")
    o = system.build_problem(n, 1, 1, 0.3, 0.5)
    H = mg.Hierarchy(o.K[0], n, coarsest=coarsest, colour_mode="lex")
    g = sgbt.Problem(n, 2, 2, 0.3, coarsest=coarsest, colour="lex")
    f = to_dev(sg_inputs.uniform_block(g.N, width, seed=n), torch.float32 if prec == "f32" else torch.float64)
    u = g.vcycle(f, prec=sgbt.SG_F32 if prec == "f32" else sgbt.SG_F64)
    assert rel_max(to_host(u), H.vcycle(to_host(f))) < (2e-5 if prec == "f32" else 1e-11)
    g.close()


def test_longest_segments():
    """511 nodes a side and 53 (float) or 105 (double) panels: segments of thirty-two coarse rows."""
    from test_gpu_cycle_forms import _check as check_strided
    check_strided(512, 8, (210,), 2, 2, "q1")
