"""Per-token encryption at the edges of its work records, every block, token and nonce against the oracle: the most
records that the kernel reads from the staging ring itself and one more (those are copied to the device first), and
enough tokens that workgroups of 64 tokens share a record, the last of them without tokens or with a few."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2608_25431_amd import gift  # noqa: E402
from test_gpu_parity import token_case  # noqa: E402


@pytest.mark.parametrize("counts", [
    [1] * 4096,
    [1] * 4095 + [65],
    [64 * 2048],
    [64 * 2048 + 1],
    [64 * 9 - 3] * 300,
    [64, 63, 65, 64 * 16384 - 200, 129, 1],
], ids=["direct", "copied", "unshared", "shared", "idle", "long"])
def test_token_runs(counts):
    r = np.random.default_rng(len(counts))
    keys = r.integers(0, 256, (5, 32), dtype=np.uint8)
    kt = gift.KeyTable(keys)
    segs, at = [], 3  # the first tokens and two between segments are nobody's
    for i, c in enumerate(counts):
        segs.append((at, c, int(r.integers(0, 5)), 0))
        at += c + (2 if i == len(counts) // 2 else 0)
    tok = r.integers(0, 1 << 62, at + 1).astype(np.uint64)
    tok[r.integers(0, at, 10)] = 7
    token_case(keys, kt, segs, tok, r.integers(0, 1 << 62, at + 1).astype(np.uint64), 7)
