"""Tags that the tile kernel folds from several queue entries, and the owner check's batches of labels, against the
oracle.  Segments of one to six 2 MiB tiles, cut into pieces or whole, whose sums meet in the wave that completes the
segment; one rejected and one tampered.  Row counts at the edges of what a wave (64 threads) or a workgroup (256) reads
in one batch of eight labels per thread, the only foreign label at the first, the last or some other row."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from gpu_helpers import dev_u32, host  # noqa: E402
from paper_2608_25431_amd import gift  # noqa: E402
from test_tile_teams import check, table_of, users  # noqa: E402,F401

TILE = 131072  # blocks


@pytest.mark.parametrize("blocks", [
    (TILE, TILE + 1, 33 * 1024, 70, 2 * TILE),            # cut into pieces of a few rows, one or two tiles
    (4 * TILE, 4 * TILE + 1, 6 * TILE - 1023, 1025, 70),  # up to four tiles and more: both ways to fold
])
@pytest.mark.parametrize("row_bytes", [16, 12])
def test_several_entries_per_segment(users, blocks, row_bytes):
    rows = [b * 16 // row_bytes for b in blocks]
    check(users, *table_of(rows, range(len(rows))), row_bytes, 21, reject=1, flips=2)


def test_more_tiles_than_compute_units(users):
    # one segment of 70 tiles (more than a wave's lanes) among whole and cut tiles
    n = torch.cuda.get_device_properties(0).multi_processor_count
    blocks = [70 * TILE] + [2048] * n + [TILE + 5] * 3
    check(users, *table_of(blocks, [i % 40 for i in range(len(blocks))]), 16, 22, reject=2, flips=2)


@pytest.mark.parametrize("counts", [
    (1, 63, 64, 65, 7 * 64, 8 * 64 - 1, 8 * 64, 8 * 64 + 1, 16 * 64 + 1),  # long and short: a workgroup per segment
    (8 * 256 - 1, 8 * 256, 8 * 256 + 1, 17 * 256 + 3),
    tuple([1, 2] * 40 + [511, 512, 513]),                                  # few rows on average: a wave per segment
])
@pytest.mark.parametrize("where", ["first", "last", "some"])
def test_one_foreign_label(counts, where):
    r = np.random.default_rng(len(counts))
    table, n_rows = table_of(counts, range(len(counts)))
    labels = np.repeat(np.arange(len(counts), dtype=np.uint32), counts)
    bad = r.random(len(counts)) < 0.5
    for i in np.flatnonzero(bad):
        at = {"first": 0, "last": counts[i] - 1, "some": int(r.integers(0, counts[i]))}[where]
        labels[table[i][0] + at] ^= 0x80
    ver = torch.full((len(counts),), -1, dtype=torch.int32, device="cuda")
    gift.check_owner(table, dev_u32(labels), n_rows, ver)
    assert (host(ver) == np.where(bad, gift.SEG_OWNER_MIXED, gift.SEG_OK)).all()
