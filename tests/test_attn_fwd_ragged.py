"""The bf16 forward where waves hold rows past the end of their sequence
(those tiles take the full-tile paths): lengths around the 32-row waves and
128-row blocks, with and without candidates, on both timestamp paths, and the
cached pass with candidate counts that leave waves ragged or empty.  Bars as
in the other parity tests; what lies behind a sequence must not reach it."""
import numpy as np
import pytest
import torch

from paper_2402_17152_amd import inputs
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hs():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2402_17152_amd import hstu
    return hstu


@pytest.mark.parametrize("dqk,dv", [(32, 32), (64, 64), (128, 128), (32, 128)])
@pytest.mark.parametrize("targets", [0, 1, 31, 40])
@pytest.mark.parametrize("wide", [False, True])
def test_ragged_lengths(hs, oracle_mod, dqk, dv, targets, wide):
    lengths = (95, 96, 97, 127, 128, 129, 159, 161, 225, 255, 257, 1, 33, 383)
    ts = None
    if wide:  # steps of about 2^31 s: the 64-bit path
        ts = np.concatenate([np.arange(n, dtype=np.int64) * ((1 << 31) + 77) + 5 for n in lengths])
    batch = inputs.make_batch(3, seed=dqk + dv + targets, lengths=lengths, num_heads=2, d_qk=dqk,
                              d_v=dv, max_seq_len=400, dtype="bf16", timestamps=ts,
                              num_targets=tuple(min(targets, n) for n in lengths))
    d = gu.dev_inputs(batch)
    gu.assert_close("O", gu.to_f64(gu.gpu_fwd(hs, d, batch)), gu.oracle_fwd(oracle_mod, batch),
                    gu.tol(batch), "bf16")


def test_rows_behind_a_sequence_do_not_reach_it(hs):
    """A sequence's output does not change with its neighbour's values."""
    batch = inputs.make_batch(3, seed=5, lengths=(333, 120), num_heads=2, d_qk=64, d_v=64,
                              max_seq_len=400, dtype="bf16")
    d = gu.dev_inputs(batch)
    ref = gu.gpu_fwd(hs, d, batch)[:333].clone()
    for name in ("q", "k", "v"):
        d[name] = d[name].clone()
        d[name][333:] = float("nan")
    d["timestamps"][333:] += 1 << 40
    assert torch.equal(gu.gpu_fwd(hs, d, batch)[:333], ref)


@pytest.mark.parametrize("count", [1, 31, 33, 50, 97, 130])
def test_ragged_candidates(hs, oracle_mod, count):
    """Cached pass against the uncached target-aware forward (bf16 bar)."""
    lengths = (700 + count, 90 + count)
    batch = inputs.make_batch(4, seed=count, lengths=lengths, num_heads=2, d_qk=128, d_v=128,
                              max_seq_len=900, dtype="bf16", num_targets=(count, count))
    d = gu.dev_inputs(batch)
    ref = gu.oracle_fwd(oracle_mod, batch)
    hist = np.concatenate([np.arange(0, 700), np.arange(lengths[0], lengths[0] + 90)])
    cand = np.concatenate([np.arange(700, lengths[0]), np.arange(lengths[0] + 90, sum(lengths))])
    h, c = torch.from_numpy(hist).cuda(), torch.from_numpy(cand).cuda()
    offs = lambda *n: torch.tensor([0, n[0], n[0] + n[1]], dtype=torch.int64, device="cuda")
    out = hs.hstu_attn_fwd_cached(
        *(d[n][c].contiguous() for n in ("q", "k", "v")), offs(count, count), d["timestamps"][c],
        d["k"][h].contiguous(), d["v"][h].contiguous(), offs(700, 90), d["timestamps"][h],
        d["rab_pos"], d["rab_time"], 900)
    gu.assert_close("O", gu.to_f64(out), ref[cand], gu.tol(batch), "bf16")
