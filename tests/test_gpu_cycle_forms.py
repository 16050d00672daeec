"""V-cycle kernels that a call reaches only by its sizes, sweep counts or strides, against the oracle's cycle.

Streaming legs: stencils loaded by every wavefront (launches of one or two
panels and more than a workgroup per CU), one sweep and P1 transfers at every
number of modes a lane, the coarsest solve in panels.
Row phases and tiles: no sweeps on one side, three sweeps, and row strides past what
the legs address.  Tolerances as for the other cycles: 1e-11 relative in
double and 2e-5 in float.
"""

import ctypes
import functools

import numpy as np
import pytest
import torch

from gpu_util import note, rel_max, to_dev, to_host

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=2)
def _hierarchy(n, coarsest, nu1, nu2, disc, colour="four"):
    from oracle import mg, paper_mode, system
    o = paper_mode.build_problem_paper(n, 1, 1, 0.1) if disc == "p1" else system.build_problem(n, 1, 1, 0.3, 0.5)
    return mg.Hierarchy(o.K[0], n, coarsest=coarsest, colour_mode=colour, nu1=nu1, nu2=nu2,
                        transfer="p1" if disc == "p1" else "bilinear")


def _check(n, coarsest, widths, nu1, nu2, disc, precs=("f64", "f32"), ld=None, colour="four"):
    """ld(size): row stride of the result by the size of its elements (None: the width)."""
    import sg_inputs
    import paper_1304_1755_amd as sgbt
    lib = sgbt.load_library()
    H = _hierarchy(n, coarsest, nu1, nu2, disc, colour)
    # at most 252 modes: m = 5, p = 5, or 70: m = 4, p = 4
    m, p = (5, 5) if max(widths) > 70 else (4, 4)
    g = sgbt.Problem(n, m, p, 0.1 if disc == "p1" else 0.3, corr_len=1.0 if disc == "p1" else 0.5, coarsest=coarsest,
                     nu1=nu1, nu2=nu2, disc=disc, colour=colour)
    for width in widths:
        f = sg_inputs.uniform_block(g.N, width, seed=n + width)
        pick = np.unique(np.linspace(0, width - 1, min(width, 12)).astype(int))  # modes do not mix
        ref = H.vcycle(f[:, pick])
        for prec in precs:
            note(f"cycle n={n} coarsest={coarsest} width={width} {prec} nu={nu1},{nu2} {disc} {colour}")
            dt = torch.float32 if prec == "f32" else torch.float64
            fd = to_dev(f, dt)
            stride = ld(4 if prec == "f32" else 8) if ld else width
            out = torch.empty(((g.N - 1) * stride + width,), dtype=dt, device="cuda")
            code = lib.sg_vcycle(g._ctx, ctypes.c_void_p(fd.data_ptr()), width, ctypes.c_void_p(out.data_ptr()), stride,
                                 width, sgbt.SG_F32 if prec == "f32" else sgbt.SG_F64)
            assert code == sgbt.SG_OK
            u = to_host(torch.as_strided(out, (g.N, width), (stride, 1))[:, torch.from_numpy(pick).cuda()])
            assert rel_max(u, ref) < (2e-5 if prec == "f32" else 1e-11)
    g.close()


# one and two panels on a grid whose launches have more than 256 workgroups of one panel: 383 nodes a side, four
# strips, 96 segments
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1)])
@pytest.mark.parametrize("disc", ["q1", "p1"])
def test_stencils_loaded_by_every_wavefront(nu1, nu2, disc):
    _check(384, 12, (1, 2, 3, 4), nu1, nu2, disc)


@pytest.mark.parametrize("nu1,nu2", [(1, 1), (2, 1), (1, 2)])
@pytest.mark.parametrize("disc", ["q1", "p1"])
def test_sweep_counts_at_every_panel_width(nu1, nu2, disc):
    _check(136, 17, (1, 2, 43), nu1, nu2, disc)


def test_p1_transfers_at_every_panel_width():
    _check(144, 9, (1, 39, 40, 47), 2, 2, "p1")


@pytest.mark.parametrize("disc", ["q1", "p1"])
def test_coarsest_solve_in_panels(disc):
    """A coarsest grid of 33 nodes a side does not fit the LDS cycle in double; 1, 2 and 5 modes (a panel that
    repeats one) and 40."""
    _check(68, 34, (1, 2, 5, 40), 2, 2, disc, precs=("f64",))


# tiles (at most 8 modes, or 32 on grids up to 127), a row-phase level over tiled ones (255 over 127), row phases
# below and from 32 modes
@pytest.mark.parametrize("nu1,nu2", [(0, 2), (2, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("disc", ["q1", "p1"])
@pytest.mark.parametrize("n,coarsest", [(136, 17), (256, 8)])
def test_no_sweeps_on_one_side(n, coarsest, disc, nu1, nu2):
    _check(n, coarsest, (1, 6, 21, 35, 126), nu1, nu2, disc)


# row phases alone: one node a thread below 16 modes, walks from 16, wavefronts of modes from 32
@pytest.mark.parametrize("nu1,nu2", [(3, 3), (1, 3), (4, 2)])
@pytest.mark.parametrize("disc", ["q1", "p1"])
def test_three_sweeps(disc, nu1, nu2):
    _check(136, 17, (1, 6, 21, 35, 126), nu1, nu2, disc)


@pytest.mark.parametrize("n,widths", [(128, (1, 6, 21, 35)), (256, (21, 126))])
@pytest.mark.parametrize("disc", ["q1", "p1"])
def test_strides_the_legs_do_not_address(n, widths, disc):
    _check(n, 8, widths, 2, 2, disc, ld=lambda size: 2 ** 32 // (80 * size * (n - 1)) + 1)


def test_lexicographic_strides_past_two_gigabytes():
    _check(64, 8, (1, 5), 2, 2, "q1", precs=("f64",), ld=lambda size: 2 ** 31 // (size * 63 * 63) + 1, colour="lex")


def test_values_of_the_modes_a_panel_repeats_are_dropped():
    """Where the last panel repeats modes of the one before, the coarse kernels write only their first copy, and the
    legs compute with whatever the second holds: it must not reach a result, whatever it is."""
    import paper_1304_1755_amd as sgbt
    for n, coarsest, prec, dt in ((136, 17, sgbt.SG_F32, torch.float32), (136, 17, sgbt.SG_F64, torch.float64),
                                  (68, 34, sgbt.SG_F64, torch.float64)):
        note(f"repeated modes n={n} coarsest={coarsest} {dt}")
        g = sgbt.Problem(n, 4, 4, 0.3, coarsest=coarsest)
        gen = torch.Generator(device="cuda").manual_seed(5)
        for width in (3, 41, 43, 47):
            f = torch.rand((g.N, width), generator=gen, dtype=dt, device="cuda")
            want = g.vcycle(f, prec=prec).clone()
            # buffers full of NaN at the widest panels of both kinds
            for w in (70, 39, 2):
                g.vcycle(torch.full((g.N, w), float("nan"), dtype=dt, device="cuda"), prec=prec)
            assert torch.equal(g.vcycle(f, prec=prec), want)
        g.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_cycle_buffers_of_one_mode(prec):
    """The first cycle allocates three vectors of the finest level, four of the coarser ones (a third of its nodes
    together) and one staging vector in double; a few granules of the allocator may come on top."""
    import paper_1304_1755_amd as sgbt
    note(f"cycle buffers P=1 {prec}")
    g = sgbt.Problem(1024, 0, 0, 0.3)
    f = torch.ones((g.N, 1), dtype=torch.float32 if prec == "f32" else torch.float64, device="cuda")
    u = torch.empty_like(f)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    g.vcycle(f, u, prec=sgbt.SG_F32 if prec == "f32" else sgbt.SG_F64)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    assert held <= g.N * (f.element_size() * (3 + 4 / 3) + 8) + 30 * 2 ** 21
    g.close()


def test_cycle_after_a_failed_allocation():
    """With memory for one of the finest level's three buffers the first cycle reports SG_ENOMEM; the next one, with
    memory again, completes the buffers and gives the usual result."""
    import paper_1304_1755_amd as sgbt
    note("cycle after a failed allocation")
    g = sgbt.Problem(512, 6, 4, 0.3)
    want = g.vcycle(torch.ones((g.N, 1), dtype=torch.float64, device="cuda")).clone()
    g.close()
    g = sgbt.Problem(512, 6, 4, 0.3)
    f = torch.ones((g.N, 1), dtype=torch.float64, device="cuda")
    u = torch.zeros_like(f)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    buffer = 8 * g.N * g.P
    rest = torch.empty((torch.cuda.mem_get_info()[0] - 3 * buffer // 2,), dtype=torch.uint8, device="cuda")
    with pytest.raises(sgbt.SGError) as e:
        g.vcycle(f, u)
    assert e.value.code == sgbt.SG_ENOMEM
    del rest
    torch.cuda.empty_cache()
    assert torch.equal(g.vcycle(f, u), want)
    g.close()
