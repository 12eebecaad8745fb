"""GPU: which kernel a Dslash shape entry launches, and the shapes on ragged
lattices.  The extents are used by no other test: table entries last as long as
the process."""
import numpy as np
import pytest

import oracle as O
from tests import synth
from tests.test_gpu_links import u3_field
from tests.test_gpu_parity import get_spinor, put_gauge, put_spinor, rel
from tests.test_gpu_service import run_manual, to_canon

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# as for the split shapes: FP64 eight hops of ~30 rounded operations each, the
# storages at their own rounding times the eight hops
BOUND = {0: 1e-14, 1: 1e-6, 2: 3e-3, 3: 2e-2}
# half-lattice sites 320 and 2520: a ragged last block of 64 and of 216 sites for
# the one-site shape, none and a ragged one of 24 for the others
RAGGED_L = [(4, 8, 2, 10), (6, 14, 10, 6)]


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1212_0785_amd import hmc
    hmc.lib()
    return hmc


def load(H, tmp_path, lines):
    table = tmp_path / "t.txt"
    table.write_text("".join(line + "\n" for line in lines))
    assert H.hmc_tune_load(str(table)) == len(lines)


def test_shape_entries_reach_the_launch_below_one_block(H, tmp_path):
    """160 half-lattice sites.  The kernels differ in how they round an FP16
    projection (scaled while it is summed, or before), so their outputs tell
    them apart: 2 is not run as 4, and 1, which does not fill a block, is."""
    L = (4, 2, 4, 10)
    F = H.Fields(L, 5.6, 0.13, flags=H.FIELDS_LOWPREC)
    put_gauge(H, F, synth.gauge_field(91, L, eps=0.4))
    src = put_spinor(H, F, synth.spinor(92, L), 1, prec=H.F16)
    got = {}
    for shape in (1, 2, 4):
        load(H, tmp_path, [f"dslash 4 2 4 10 2 {shape} 0"])
        assert H.hmc_tune_query(L, H.TUNE_DSLASH, H.F16) == (shape, True)
        out = F.spinor(prec=H.F16)
        H.hmc_wilson_dslash(F, out, src, 0, 0, H.F16)
        got[shape] = get_spinor(H, F, out, 0, prec=H.F16)
    assert np.array_equal(got[1], got[4])
    assert not np.array_equal(got[2], got[4])


@pytest.mark.parametrize("L", [(2, 6, 4, 4), (2, 6, 8, 8)])
def test_staple_force_reads_the_reported_form(H, L):
    """96 and 384 half-lattice sites: the bytes of the launch are those of the
    form that the query reports."""
    F = H.Fields(L, 5.6, 0.13)
    put_gauge(H, F, synth.gauge_field(93, L, eps=0.4))
    assert H.hmc_links_two_row(F)
    H.hmc_timing_reset()
    H.hmc_timing_enable(1)
    H.hmc_gauge_force(F, 0.1)
    torch.cuda.synchronize()
    t = H.hmc_timing_read()["gauge_force"]
    H.hmc_timing_enable(0)
    H.hmc_timing_reset()
    form, tuned = H.hmc_tune_query(L, H.TUNE_GAUGE_FORCE_LINKS)
    assert not tuned and t["launches"] == 1
    # per site four links of `form` reals, eight momenta a link read and written
    assert t["bytes_moved"] == np.prod(L) * 4 * (8 * form + 2 * 64)


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("shape", [1, 2, 4])
@pytest.mark.parametrize("L", RAGGED_L)
def test_shapes_on_ragged_lattices(H, tmp_path, L, shape, su3):
    """Both hops, Mhat and the epilogues of a CG against the oracle, on SU(3)
    links in both compact forms and on U(3) links (all entries read)."""
    k = 0.13
    ext = " ".join(map(str, L))
    U = synth.gauge_field(94, L, eps=0.4) if su3 else u3_field(95, L)
    psi = synth.spinor(96, L)
    for form in (12, 10) if su3 else (12,):
        load(H, tmp_path, [f"dslash {ext} {p} {shape} 0" for p in range(4)] +
             [f"dslash_links {ext} {p} {form} 0" for p in range(4)])
        F = H.Fields(L, 5.6, k, flags=H.FIELDS_LOWPREC)
        put_gauge(H, F, U)
        assert bool(H.hmc_links_two_row(F)) == su3
        for prec in range(4):
            for par in (0, 1):
                for dag in (0, 1):
                    out = F.spinor(prec=prec)
                    H.hmc_wilson_dslash(F, out, put_spinor(H, F, psi, 1 - par, prec=prec), par, dag, prec)
                    assert rel(get_spinor(H, F, out, par, prec=prec), O.dslash(L, U, psi, par, dag)) < BOUND[prec]
            out = F.spinor(prec=prec)
            H.hmc_mhat(F, out, put_spinor(H, F, psi, 0, prec=prec), 0, prec)
            assert rel(get_spinor(H, F, out, 0, prec=prec), O.mhat(L, U, k, psi, 0)) < BOUND[prec]
        b = put_spinor(H, F, psi, 0)
        x = F.spinor()
        H.hmc_cg_solve(F, x, b, H.cg_params(fixed_iters=5))
        want, _ = O.cg_mhat(L, U, k, get_spinor(H, F, b, 0), fixed_iters=5)
        assert rel(get_spinor(H, F, x, 0), want) < 1e-12


# 320 half-lattice sites, and 35672 (ragged too), where the batches of shape 4
# split by direction
@pytest.mark.parametrize("prec", range(4))
@pytest.mark.parametrize("L,shape", [(RAGGED_L[0], 1), (RAGGED_L[0], 2), (RAGGED_L[0], 4), ((14, 14, 14, 26), 4)])
def test_batched_shapes_on_a_ragged_lattice(H, tmp_path, L, shape, prec):
    """Two requests of one volume in one batch: each is what it is alone, bit
    for bit, and solves its system (the oracle's solution to 1e-8: both meet
    |b - M x| <= 1e-10 |b|)."""
    ext = " ".join(map(str, L))
    load(H, tmp_path, [f"dslash {ext} {p} {shape} 0" for p in range(4)])
    reqs = [(L, 0.150, 97, 0.3, 1, 3), (L, 0.154, 98, 0.4, 0, 5)]
    arena = 2 * H.hmc_request_bytes(H.solve_request(*reqs[0]), prec) + (4 << 20)  # two requests and the header
    res, outs = run_manual(H, reqs, prec, arena=arena)
    assert all(r["status"] == 0 and r["true_rel_res"] <= 1e-10 and r["max_group"] == 2 for r in res)
    for (lat, k, gs, eps, kind, ss), out in zip(reqs, outs):
        _, alone = run_manual(H, [(lat, k, gs, eps, kind, ss)], prec, arena=arena)
        assert torch.equal(alone[0], out)
        want, _ = O.wilson_solve(lat, O.weak_field(lat, gs, eps), k, O.source(lat, kind, ss, 0), tol=1e-12)
        assert rel(to_canon(H, lat, out), want) < 1e-8


def test_hops_add_up_in_fp32_as_precisely_as_directions(H, tmp_path):
    """FP32 hop of one wavefront per hop against the direction split's: no larger
    error (1% room: 850,000 numbers leave the ratio uncertain by 0.2%)."""
    L = (14, 14, 14, 26)
    U = synth.gauge_field(99, L, eps=0.4)
    psi = synth.spinor(100, L)
    want = O.dslash(L, U, psi, 0, 0)
    F = H.Fields(L, 5.6, 0.13, flags=H.FIELDS_LOWPREC)
    put_gauge(H, F, U)
    src = put_spinor(H, F, psi, 1, prec=H.F32)
    err = {}
    for shape in (2, 4):
        load(H, tmp_path, [f"dslash 14 14 14 26 1 {shape} 0"])
        out = F.spinor(prec=H.F32)
        H.hmc_wilson_dslash(F, out, src, 0, 0, H.F32)
        err[shape] = rel(get_spinor(H, F, out, 0, prec=H.F32), want)
    assert err[4] < 1.01 * err[2], err
