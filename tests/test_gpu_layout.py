"""GPU: the tiled layout conversions and the per-subset sums at the edges of
their tiles: fewer sites than a tile, ragged last tiles, one parity or both,
subset ids in runs, shuffled and out of range.  All exact: conversions move
bits, and the sums run over small integers."""
import numpy as np
import pytest

from tests import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# 16, 96, 384, 640 and 5040 sites: below, between and above tiles of 64
LAYOUT_L = [(2, 2, 2, 2), (2, 4, 6, 2), (4, 4, 4, 6), (8, 4, 2, 10), (10, 6, 14, 6)]


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1212_0785_amd import hmc
    hmc.lib()
    return hmc


def parities(L):
    c = np.indices(L[::-1])
    return (c.sum(0) % 2).reshape(-1)


@pytest.mark.parametrize("L", LAYOUT_L)
def test_conversions_move_every_entry(H, L):
    V = int(np.prod(L))
    par = parities(L)
    F = H.Fields(L, 5.6, 0.13)
    U = synth.gauge_field(81, L, eps=0.4)
    H.hmc_import_gauge(F, H.to_device_c128(U))
    assert H.hmc_links_two_row(F)
    back = H.canon_gauge_zeros(L)
    H.hmc_export_gauge(F, back)
    assert np.array_equal(back.cpu().numpy(), U)
    off = F.pointer(H.FIELD_GAUGE) - F.arena.data_ptr()
    dev = F.arena[off:off + V * 576].view(torch.float64).cpu().numpy().view(np.complex128).reshape(4, 2, 9, V // 2)
    for p in (0, 1):
        assert np.array_equal(dev[:, p], U[par == p].reshape(V // 2, 4, 9).transpose(1, 2, 0))
    # one entry off in the last link of the lattice is seen by the import
    bad = U.copy()
    bad[-1, 3, 2, 2] += 1e-12
    H.hmc_import_gauge(F, H.to_device_c128(bad))
    assert not H.hmc_links_two_row(F)
    psi = synth.spinor(82, L)
    for which in (-1, 0, 1):
        buf = F.spinor(full=which < 0)
        H.hmc_import_spinor(F, buf, H.to_device_c128(psi), which)
        halves = buf.view(torch.float64).cpu().numpy().view(np.complex128).reshape(-1, 12, V // 2)
        for h, p in zip(halves, (0, 1) if which < 0 else (which,)):
            assert np.array_equal(h, psi[par == p].reshape(V // 2, 12).T)
        out = torch.full((V, 4, 3), float("nan"), dtype=torch.complex128, device="cuda")
        H.hmc_export_spinor(F, out, buf, which)
        want = psi if which < 0 else np.where((par == which)[:, None, None], psi, 0)
        assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("nsub", [1, 3, 130, 1024])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 6), (10, 6, 14, 6)])
def test_subset_sums(H, L, nsub):
    V = int(np.prod(L))
    F = H.Fields(L, 5.6, 0.13)
    rng = np.random.default_rng(83)
    x = rng.integers(-3, 4, size=(2, 12, V // 2, 2)).astype(np.float64)
    per_site = (x ** 2).sum((1, 3)).reshape(-1)
    dev = torch.from_numpy(x).to("cuda")
    runs = np.minimum(np.arange(V) * nsub // V, nsub - 1)
    for ids in (runs, rng.integers(0, nsub, V), rng.integers(-2, nsub + 2, V), np.full(V, -1)):
        sub = torch.from_numpy(ids.astype(np.int32)).to("cuda")
        for halves in (1, 2):
            n = halves * V // 2
            want = [per_site[:n][ids[:n] == k].sum() for k in range(nsub)]
            assert H.hmc_sum_multi(F, dev, halves, sub, nsub) == want
