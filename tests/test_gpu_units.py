"""Packed units of the attention kernels: 32 consecutive (token, head of the group) rows of a KV head.  Group sizes whose
multiples meet the 32-row unit everywhere but at its edges, groups wider than a unit, chunks that leave wavefronts of
the last workgroup without rows, and pieces of the key range shorter than the ring of tiles; every row against the oracle."""
import pytest

from paper_2605_12471_amd import inputs as I
from test_gpu_parity_small import H, _run_case  # noqa: F401  (H: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("G,Hkv", [(1, 2), (3, 2), (5, 1), (31, 1), (32, 1), (33, 1), (40, 1), (100, 1)])
def test_group_sizes_around_the_unit(H, oracle, dtype, G, Hkv):
    cfg = I.FoldConfig("units_group", 60, 1, G * Hkv, Hkv, 64, 70, 0, dtype)
    _run_case(H, oracle, cfg, [70, 1, 13, 64, 2])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upw", [1, 2])
@pytest.mark.parametrize("chunks", [[1, 300, 1, 8, 9], [7, 64, 65, 33, 130], [64, 64, 64, 63, 1], [320, 17, 40]])
@pytest.mark.parametrize("splits", [1, 2, 5])
def test_pieces_and_wavefronts_without_rows(H, oracle, d, upw, chunks, splits):
    """Prefix pieces of one to a few tiles (the main loop runs over them alone), pieces that straddle the old cache's
    end or reach a last tile that is not full, and one to eight units for the workgroup's wavefronts."""
    cfg = I.FoldConfig("units_pieces", 61, 1, 8, 2, d, max(chunks), 0, "bf16")
    _run_case(H, oracle, cfg, chunks, splits=splits, upw=upw)


@pytest.mark.parametrize("upw,pair", [(1, 0), (2, 1), (2, 2)])
def test_long_prefix_pieces(H, oracle, upw, pair):
    """Cache lengths on and off the tile grid with pieces long enough for every loop of the kernel."""
    cfg = I.FoldConfig("units_long", 62, 1, 4, 1, 128, 700, 0, "bf16")
    _run_case(H, oracle, cfg, [700, 580, 131, 389, 20], splits=2, upw=upw, pair=pair)
    _run_case(H, oracle, cfg, [700, 580, 131, 389, 20], splits=1, upw=upw, pair=pair)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("splits", [1, 3])
def test_grids_of_one_and_of_two_workgroups_a_cu(H, oracle, d, splits):
    """The one-unit kernel's ring has a slot more where no CU gets a second workgroup: 130 heads, as many workgroups and three times as
    many, one unit a workgroup and four; pieces of one tile to the ring's length and over, on and off the tile grid."""
    cfg = I.FoldConfig("units_rings", 63, 1, 130, 130, d, 128, 0, "bf16")
    _run_case(H, oracle, cfg, [128, 33, 64, 95, 1 + 32], splits=splits, upw=1)
    cfg = I.FoldConfig("units_ring_alone", 64, 1, 5, 5, d, 300, 0, "bf16")
    _run_case(H, oracle, cfg, [300, 33, 300, 60, 40], splits=splits, upw=1)
