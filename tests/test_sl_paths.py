"""Stochastic Length and the row gather at the edges of their dispatch:
histories at and past the 8192 tokens whose keys stay in registers, lengths
around multiples of the 1024 threads, more sequences than one workgroup adds
up by itself (4096), ties that cross threads, and gathered rows of every word
size, width and alignment.  All exact."""
import numpy as np
import pytest
import torch

from paper_2402_17152_amd import inputs
from tests import test_sl as ts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ts.MODES)
@pytest.mark.parametrize("dup", [False, True])
def test_sl_long_histories(oracle_mod, mode, dup):
    lengths = [1023, 1024, 1025, 8191, 8192, 8193, 20000, 9000]
    nt = np.array([0, 0, 3, 0, 0, 0, 100, 808])
    offs, t = ts._batch(lengths, 3, dup_ts=dup)
    u, e = inputs.make_sl_draws(len(lengths), offs[-1], seed=11)
    u[:] = 0.999
    if dup:
        e[:] = np.floor(e * 4.0)  # few distinct keys: long runs of ties
    ts._check(ts._hs(), oracle_mod, offs, t, nt, 700, 1000.0, mode, u, e)


@pytest.mark.parametrize("count", [4096, 4097, 5000])
def test_sl_many_sequences(oracle_mod, count):
    lengths = np.random.default_rng(count).integers(0, 40, count)
    offs, t = ts._batch(lengths, 5)
    u, e = inputs.make_sl_draws(count, offs[-1], seed=5)
    ts._check(ts._hs(), oracle_mod, offs, t, None, 12, 12.0 ** 2.1, 1, u, e)


@pytest.mark.parametrize("row_bytes,shift", [(4, 0), (12, 4), (8, 0), (24, 8), (16, 0), (48, 16),
                                             (1024, 0), (1040, 16), (1032, 8), (1028, 4),
                                             (4096, 0)])
@pytest.mark.parametrize("rows", [1, 63, 1000, 40000])
def test_gather_row_widths(row_bytes, shift, rows):
    """Rows at a byte offset of `shift` (the widest word that still fits is
    used); nothing past the count is written."""
    hs = ts._hs()
    g = torch.Generator(device="cuda").manual_seed(row_bytes + rows)
    n = rows + rows // 2
    words = (n * row_bytes + shift) // 4
    flat = torch.randint(-2**31, 2**31 - 1, (words,), generator=g, device="cuda",
                         dtype=torch.int32)
    src = flat[shift // 4:].view(n, row_bytes // 4)
    idx = torch.randperm(n, generator=g, device="cuda")[:rows].sort().values
    cnt = torch.tensor([rows], dtype=torch.int64, device="cuda")
    full = torch.cat([idx, idx.new_zeros(7)])
    dst = torch.full((rows + 7, row_bytes // 4), 5, dtype=torch.int32, device="cuda")
    hs.hstu_gather_rows(src, full, cnt, dst=dst)
    torch.cuda.synchronize()
    assert torch.equal(dst[:rows], src[idx])
    assert (dst[rows:] == 5).all()


@pytest.mark.parametrize("rows,row_bytes", [(1, 1 << 20), (3, 65536 + 8), (17, 4096 + 4),
                                            (70, 16384), (16, 1040), (5, 2080), (9, 4112)])
def test_gather_wide_rows(rows, row_bytes):
    """Rows of more words than a wave: up to the whole workgroup shares one,
    longer ones are spread over workgroups, with words left over or not."""
    test_gather_row_widths(row_bytes, 0, rows)


@pytest.mark.parametrize("mode", ts.MODES)
@pytest.mark.parametrize("count", [1024, 1025, 1027, 4096, 4097])
def test_sl_sequences_per_workgroup(oracle_mod, mode, count):
    """Batches on both sides of the sizes where a workgroup takes 1, 4 and 16
    sequences, of which some stay whole and some are shortened, long ones and
    empty ones among them, the last group partly filled."""
    rng = np.random.default_rng(count)
    lengths = rng.integers(0, 60, count)
    lengths[[3, 100, 101, 255, count - 1]] = (1025, 4097, 0, 9000, 2000)
    nt = np.minimum(lengths, rng.integers(0, 30, count))
    offs, t = ts._batch(lengths, 9, dup_ts=True)
    u, e = inputs.make_sl_draws(count, offs[-1], seed=count)
    e[:] = np.floor(e * 8.0)  # few distinct keys: ties across threads
    ts._check(ts._hs(), oracle_mod, offs, t, nt, 20, 20.0 ** 2.1, mode, u, e)
