"""GPU: the split Dslash shapes (two wavefronts per 64 sites, and one wavefront
per hop) at the sizes where they can go wrong: fewer sites than a wavefront,
ragged last blocks, extents of two and extents that are no powers of two.

Bounds: FP64 1e-14 of the field (eight hops of ~30 rounded operations each),
the storages at their own rounding times the eight hops (as for the one-site
shape)."""
import numpy as np
import pytest

import oracle as O
from tests import synth
from tests.test_gpu_parity import get_spinor, put_gauge, put_spinor, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {0: 1e-14, 1: 1e-6, 2: 3e-3, 3: 2e-2}
# half-lattice sites 8, 48, 96 and 128 (Mhat in one launch), 192 (below one
# block), 320 and 1260 (ragged)
HOP_L = [(2, 2, 2, 2), (2, 4, 6, 2), (6, 2, 4, 4), (4, 4, 4, 4), (4, 4, 4, 6), (8, 4, 2, 10), (10, 6, 14, 6)]


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1212_0785_amd import hmc
    hmc.lib()
    return hmc


@pytest.mark.parametrize("shape", [2, 4])
@pytest.mark.parametrize("L", HOP_L)
def test_split_shapes(H, tmp_path, L, shape):
    k = 0.13
    ext = " ".join(map(str, L))
    table = tmp_path / "t.txt"
    U = synth.gauge_field(71, L, eps=0.4)
    psi = synth.spinor(72, L)
    for form in (12, 10):
        table.write_text("".join(f"dslash {ext} {p} {shape} 0\ndslash_links {ext} {p} {form} 0\n" for p in range(4)))
        H.hmc_tune_load(str(table))
        F = H.Fields(L, 5.6, k, flags=H.FIELDS_LOWPREC)
        put_gauge(H, F, U)
        for prec in range(4):
            for par in (0, 1):
                for dag in (0, 1):
                    out = F.spinor(prec=prec)
                    H.hmc_wilson_dslash(F, out, put_spinor(H, F, psi, 1 - par, prec=prec), par, dag, prec)
                    got = get_spinor(H, F, out, par, prec=prec)
                    assert rel(got, O.dslash(L, U, psi, par, dag)) < BOUND[prec], (form, prec, par, dag)
            for dag in (0, 1):
                out = F.spinor(prec=prec)
                H.hmc_mhat(F, out, put_spinor(H, F, psi, 0, prec=prec), dag, prec)
                got = get_spinor(H, F, out, 0, prec=prec)
                assert rel(got, O.mhat(L, U, k, psi, dag)) < BOUND[prec], (form, prec, dag)
        # the norm and residual epilogues
        b = put_spinor(H, F, psi, 0)
        x = F.spinor()
        H.hmc_cg_solve(F, x, b, H.cg_params(fixed_iters=5))
        want, _ = O.cg_mhat(L, U, k, get_spinor(H, F, b, 0), fixed_iters=5)
        assert rel(get_spinor(H, F, x, 0), want) < 1e-12
