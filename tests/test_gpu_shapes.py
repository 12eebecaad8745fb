"""GPU: which kernel a Dslash shape entry launches, and the shapes on ragged
lattices.  The extents are used by no other test: table entries last as long as
the process."""
import numpy as np
import pytest

from tests import synth
from tests.test_gpu_parity import get_spinor, put_gauge, put_spinor

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


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
