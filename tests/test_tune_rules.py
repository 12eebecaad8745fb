"""Built-in launch rules on both sides of their thresholds, on lattices with no
table entry (host side of libhmc; no GPU needed)."""
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1212_0785_amd", "libhmc.so")
pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="libhmc.so not built"),
              pytest.mark.skipif(any(k.startswith(("HMC_DSLASH_", "HMC_LINK_", "HMC_GFORCE_", "HMC_TUNE_"))
                                     for k in os.environ), reason="environment overrides the rules")]

# half-lattice sites 2^16 + 4096, 2^20 - 32768, 2^20 + 65536
AT_2_16, BELOW_2_20, FROM_2_20 = (16, 16, 16, 34), (32, 32, 32, 62), (32, 32, 34, 64)


@pytest.fixture(scope="module")
def H():
    from paper_1212_0785_amd import hmc
    hmc.lib()
    return hmc


def test_links_keep_two_rows_below_2_20_sites(H):
    """Two rows rebuild a reunitarised link exactly, row 0 and column 2 do not."""
    for prec in range(4):
        for L in (AT_2_16, BELOW_2_20):
            assert H.hmc_tune_query(L, H.TUNE_DSLASH_LINKS, prec) == (H.LINK_ROWS2, False), (L, prec)
        assert H.hmc_tune_query(FROM_2_20, H.TUNE_DSLASH_LINKS, prec) == (H.LINK_ROWCOL, False)


@pytest.mark.parametrize("prec", [2, 3])
def test_shipped_table_keeps_two_rows_for_the_halves_of_24c48(H, prec):
    assert H.hmc_tune_query((24, 24, 24, 48), H.TUNE_DSLASH_LINKS, prec) == (H.LINK_ROWS2, True)


def test_tiled_order_only_where_one_site_per_work_item_runs(H, tmp_path):
    """The order belongs to the one-site shape: no other shape walks in it."""
    q = lambda L: (H.hmc_tune_query(L, H.TUNE_DSLASH, H.F64)[0], H.hmc_tune_query(L, H.TUNE_DSLASH_ORDER, H.F64)[0])
    assert q((32, 32, 32, 64)) == (4, 0)    # 2^20 half-lattice sites
    assert q((32, 32, 32, 88)) == (4, 0)    # 3 * 2^19 - 131072
    assert q((32, 32, 32, 96)) == (1, 1)    # 3 * 2^19
    assert q((32, 32, 32, 100)) == (1, 0)   # not a multiple of eight time slices
    src = tmp_path / "t.txt"
    src.write_text("dslash 32 32 32 104 0 4 1.0\n")
    assert H.hmc_tune_load(str(src)) == 1
    assert q((32, 32, 32, 104)) == (4, 0)
