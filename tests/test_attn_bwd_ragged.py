"""The bf16 backward where the last 128-key block of a sequence holds few keys,
so that most of its lanes stand for keys past the end (they read the position
window from its first entry): attention (two-role kernel) and layer backward at
every head size, with and without candidates, on both timestamp paths."""
import numpy as np
import pytest

from paper_2402_17152_amd import inputs
from tests import test_parity as tp

pytestmark = pytest.mark.gpu

LENGTHS = (1, 2, 31, 33, 127, 129, 130, 160, 161, 255, 257, 385)


@pytest.fixture(scope="module")
def hs():
    from paper_2402_17152_amd import hstu
    return hstu


@pytest.mark.parametrize("dqk,dv", [(32, 32), (64, 64), (128, 128), (32, 128)])
@pytest.mark.parametrize("targets", [None, 1, 40])
@pytest.mark.parametrize("wide", [False, True])
def test_ragged_key_blocks(hs, oracle_mod, dqk, dv, targets, wide):
    ts = None
    if wide:  # steps of about 2^31 s: the 64-bit path
        ts = np.concatenate([np.arange(n, dtype=np.int64) * ((1 << 31) + 77) + 5 for n in LENGTHS])
    nt = None if targets is None else tuple(min(targets, n) for n in LENGTHS)
    batch = inputs.make_batch(3, seed=dqk + dv + (targets or 0), lengths=LENGTHS, num_heads=2,
                              d_qk=dqk, d_v=dv, max_seq_len=400, dtype="bf16", timestamps=ts,
                              num_targets=nt)
    tp._check_bwd(hs, oracle_mod, batch)
    tp._layer_bwd_check(hs, oracle_mod, batch)
