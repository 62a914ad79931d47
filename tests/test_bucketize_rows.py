"""hstu_time_bucketize at the edges of its row grouping: the three row counts
per workgroup (16, 32 and 64, chosen by the batch's tokens), sequences that
begin and end inside a workgroup's rows, every alignment of a row's first
byte, rows past one slab of 8192 columns, both timestamp widths and the
clamped bucket counts.  Exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(ts, nb):
    d = np.abs(ts[:, None] - ts[None, :])
    return np.minimum(np.frexp(np.maximum(d, 1).astype(np.float64))[1] - 1, nb - 1)


SHORT = [
    tuple(range(1, 70)),                       # 2415 tokens: 16 rows
    tuple([7, 0, 129, 1000, 2049] * 3),        # 9555 tokens: 32 rows
    tuple([63, 64, 65, 1023, 0, 17] * 14),     # 17248 tokens: 64 rows
]
LONG = [(8191, 8193, 3)]
CASES = [(n, nb, 600) for n in SHORT + LONG for nb in (128, 32, 9, 1)]
CASES += [(n, 64, 1 << 34) for n in SHORT]     # 64-bit differences


@pytest.mark.parametrize("lengths,nb,gap", CASES)
def test_bucketize_row_groups(lengths, nb, gap):
    from paper_2402_17152_amd import hstu
    rng = np.random.default_rng(len(lengths) + nb)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    ts = np.concatenate([1_700_000_000 + np.cumsum(rng.integers(0, gap, n)) for n in lengths])
    ts = ts.astype(np.int64)
    dev = lambda a: torch.from_numpy(a).cuda()
    got = hstu.hstu_time_bucketize(dev(offs), dev(ts), nb).cpu().numpy()
    o = 0
    for b, n in enumerate(lengths):
        ref = _reference(ts[offs[b]:offs[b + 1]], nb)
        assert np.array_equal(got[o:o + n * n].reshape(n, n), ref), f"sequence {b} of {n} tokens"
        o += n * n
    assert o == got.size


@pytest.mark.parametrize("lengths", [tuple(range(60, 84)) * 2, (1,) * 700 + (2,) * 300 + (64,) * 9])
@pytest.mark.parametrize("nb,gap", [(128, 600), (9, 600), (64, 1 << 34)])
def test_bucketize_short_sequences(lengths, nb, gap):
    """Both sides of the 64 tokens up to which a sequence goes unstaged, at
    every alignment, and workgroups that meet many short sequences."""
    test_bucketize_row_groups(lengths, nb, gap)
