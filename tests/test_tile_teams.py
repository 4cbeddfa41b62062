"""The per-block kernel's two forms against the oracle, every byte, tag and verdict: one team of 16 waves per
workgroup (long tiles, or no more tiles than CUs) and two teams of 8 (more, short tiles), where a wave can be a tile
ahead of another and the last one to arrive finishes the tile.  Segment lengths at the edges of a wave (64 blocks), of
a team's row (512, 1024) and of a tile's first, partial row; several tiles per team; rejected and tampered segments
between good ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from gpu_helpers import dev_u8, dev_u32, host, open_, oracle_segments, seal  # noqa: E402
from paper_2608_25431_amd import gift  # noqa: E402

EDGES = (65, 127, 511, 512, 513, 1023, 1024, 1025, 1535, 1537, 2049)


@pytest.fixture(scope="module")
def users():
    r = np.random.default_rng(11)
    keys = r.integers(0, 256, (40, 32), dtype=np.uint8)
    nb = r.integers(0, 256, (40, 12), dtype=np.uint8)
    return keys, nb, gift.KeyTable(keys)


def table_of(row_counts, users_of):
    row, t = 0, []
    for i, n in enumerate(row_counts):
        t.append((row, int(n), int(users_of[i]), 100 + i))
        row += int(n)
    return t, row


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def check(users, table, n_rows, rb, seed, reject=3, flips=4):
    """Seal with some segments relabelled, then open with some ciphertext and tag bits flipped."""
    keys, nb, kt = users
    r = np.random.default_rng(seed)
    n = len(table)
    segs = oracle.as_segments(table)
    data = r.integers(0, 256, n_rows * rb, dtype=np.uint8)
    labels = np.repeat(segs["user"], segs["row_count"].astype(np.int64)).astype(np.uint32)
    bad = [int(i) for i in r.choice(n, reject, replace=False)]
    for i in bad:
        labels[int(segs[i]["row_begin"]) + int(r.integers(0, segs[i]["row_count"]))] += 1
    cut = [slice(int(s["row_begin"]) * rb, int(s["row_begin"] + s["row_count"]) * rb) for s in segs]
    ref = oracle_segments(keys, nb, segs, rb, lambda i: data[cut[i]].tobytes())
    ct, tags, ver = seal(dev_u8(data), n_rows, rb, table, kt, nb, labels_dev=dev_u32(labels))
    ct_h, tg_h, ver_h = host(ct), host(tags).reshape(n, 16), host(ver)
    for i in range(n):
        want_c, want_t = (bytes(len(ref[i][0])), bytes(16)) if i in bad else ref[i]
        assert ct_h[cut[i]].tobytes() == want_c and tg_h[i].tobytes() == want_t, i
        assert ver_h[i] == (gift.SEG_OWNER_MIXED if i in bad else gift.SEG_OK), i
    # open the whole tensor as the oracle sealed it, with some bits flipped
    for i in bad:
        ct_h[cut[i]] = np.frombuffer(ref[i][0], np.uint8)
        tg_h[i] = np.frombuffer(ref[i][1], np.uint8)
    hit = [int(i) for i in r.choice(n, flips, replace=False)]
    for j, i in enumerate(hit):
        if j % 2:
            tg_h[i][int(r.integers(0, 16))] ^= 4
        else:
            ct_h[cut[i].start + int(r.integers(0, cut[i].stop - cut[i].start))] ^= 32
    back, ver = open_(dev_u8(ct_h), n_rows, rb, table, kt, nb, dev_u8(tg_h))
    back_h, ver_h = host(back), host(ver)
    for i in range(n):
        want = bytes(cut[i].stop - cut[i].start) if i in hit else data[cut[i]].tobytes()
        assert back_h[cut[i]].tobytes() == want, i
        assert ver_h[i] == (gift.SEG_AUTH_FAIL if i in hit else gift.SEG_OK), i


@pytest.mark.parametrize("row_bytes", [16, 20])
def test_two_teams_many_short_tiles(users, row_bytes):
    # more tiles than two per team, 20-byte rows unaligned with a ragged last block
    r = np.random.default_rng(1)
    n = 5 * cus()
    rows = r.choice(EDGES, n) * 16 // row_bytes + (0 if row_bytes == 16 else r.integers(0, 3, n))
    check(users, *table_of(rows, r.integers(0, 40, n)), row_bytes, 2)


def test_two_teams_with_a_cut_tail(users):
    # mostly short tiles, some longer than a 32-row piece: those are cut into pieces
    r = np.random.default_rng(3)
    n = 3 * cus()
    blocks = r.choice(EDGES, n)
    blocks[r.choice(n, 8, replace=False)] = r.integers(33 * 1024, 40 * 1024, 8)
    check(users, *table_of(blocks, r.integers(0, 40, n)), 16, 4)


@pytest.mark.parametrize("long_rows", [1, 20, 40])
def test_two_teams_reuse_their_slots(users, long_rows):
    # about eight tiles per team, of which four can be under way at once: records and sums are used again.  Some longer
    # tiles: whose next record is fetched after their rows (from 3 rows on), or cut into pieces (from 33)
    r = np.random.default_rng(13)
    n = 16 * cus()
    blocks = r.integers(65, 1026, n)
    blocks[r.choice(n, 40, replace=False)] = r.integers((long_rows - 1) * 1024 + 65, long_rows * 1024 + 2, 40)
    check(users, *table_of(blocks, r.integers(0, 40, n)), 16, 14, reject=9, flips=40)


def test_one_team_several_tiles(users):
    # tiles of 17 rows and a bit: one team, two tiles on some CUs, users change between tiles
    r = np.random.default_rng(5)
    n = cus() + 20
    check(users, *table_of(17 * 1024 + r.integers(-70, 70, n), r.integers(0, 40, n)), 16, 6)


def test_one_team_fewer_tiles_than_cus(users):
    r = np.random.default_rng(7)
    n = 60
    check(users, *table_of(r.choice(EDGES, n), r.integers(0, 40, n)), 16, 8)


@pytest.mark.parametrize("row_bytes", [16, 20])
def test_failed_tiles_are_zeroed_to_the_byte(users, row_bytes):
    # uncut one-tile segments, two thirds of them tampered, between good ones: one wave zeroes each, 512 whole blocks
    # at a time, then 64, then the bytes of a ragged end
    blocks = [b + d for b in (128, 512, 576, 1024, 1536, 2048, 2560) for d in (-1, 0, 1)]
    rows = [b * 16 // row_bytes + d for b in blocks for d in ((0,) if row_bytes == 16 else (0, 1, 2))]
    check(users, *table_of(rows, [i % 40 for i in range(len(rows))]), row_bytes, 10, reject=1, flips=len(rows) * 2 // 3)


def test_paged_two_teams(users):
    from test_gpu_parity import paged_case, paged_geom
    keys, nb, kt = users
    n = 2 * cus() + 30
    g = paged_geom("lbp", 3, 2, n + 5, 2048)
    r = np.random.default_rng(9)
    ids = r.permutation(n + 5)[:n].astype(np.uint32)
    reqs = [(ids[i:i + 1], int(r.integers(0, 40)), i) for i in range(n)]
    ver, ver2 = paged_case(keys, nb, kt, g, reqs)
    assert (np.asarray(ver) == 0).all() and (np.asarray(ver2) == 0).all()
    labels = np.full(n + 5, 0xFFFFFFFF, np.uint32)
    for b, u, _ in reqs:
        labels[b] = u
    labels[reqs[7][0]] += 1
    labels[reqs[n - 1][0]] += 1
    paged_case(keys, nb, kt, g, reqs, labels=labels)


def test_paged_two_teams_reuse_their_slots(users):
    from test_gpu_parity import paged_case, paged_geom
    keys, nb, kt = users
    r = np.random.default_rng(15)
    sizes = r.integers(1, 5, 12 * cus())
    at = np.concatenate([[0], np.cumsum(sizes)])
    g = paged_geom("lbp", 1, 1, int(at[-1]) + 3, 2048)
    ids = r.permutation(int(at[-1]) + 3).astype(np.uint32)
    reqs = [(ids[at[i]:at[i + 1]], int(r.integers(0, 40)), i) for i in range(len(sizes))]
    labels = np.full(int(at[-1]) + 3, 0xFFFFFFFF, np.uint32)
    for b, u, _ in reqs:
        labels[b] = u
    for i in r.choice(len(reqs), 9, replace=False):
        labels[reqs[int(i)][0][-1]] += 1
    paged_case(keys, nb, kt, g, reqs, labels=labels, tamper=int(at[700]) * 2048 + 5)
