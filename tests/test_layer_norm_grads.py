"""hstu_layer_fwd / hstu_layer_bwd over the layer norm's dispatch: each
number of lanes per row and chunks per lane (h d_v from 32 to 4096), token
counts below and above one workgroup's rows, affine parameters that are only
4-byte aligned, and the space-bound partial sums of d_ln_weight / d_ln_bias
(d_qk = 32, d_v = 128).  Bars as in the other layer tests."""
import pytest
import torch

from paper_2402_17152_amd import inputs
from tests import test_parity as tp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hs():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2402_17152_amd import hstu
    return hstu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads,dqk,dv,lengths", [
    (1, 32, 32, (1,)), (1, 32, 32, (70, 61)), (3, 32, 32, (45,)), (3, 64, 64, (37, 0, 90)),
    (1, 32, 128, (3, 8)), (7, 64, 64, (33, 20)), (10, 32, 64, (41,)), (5, 32, 128, (39,)),
    (32, 32, 128, (9, 14))])
def test_layer_norm_widths(hs, oracle_mod, dtype, heads, dqk, dv, lengths):
    batch = inputs.make_batch(2, seed=900 + heads * dv + len(lengths), lengths=lengths,
                              num_heads=heads, d_qk=dqk, d_v=dv, max_seq_len=96, dtype=dtype)
    tp._layer_bwd_check(hs, oracle_mod, batch)


def test_layer_norm_parameters_need_no_alignment(hs):
    """Parameters at a 4-byte offset give the bits of aligned ones, and two
    runs the same parameter gradients bit for bit (fixed summation order)."""
    batch = inputs.make_batch(2, seed=77, lengths=(300, 129), num_heads=4, d_qk=64, d_v=64,
                              max_seq_len=300, dtype="bf16")
    d = inputs.to_device(batch)
    D, N = 256, 300
    w, b = (torch.from_numpy(x).cuda() for x in tp._ln_params(D, 5))
    dy = d["do"].reshape(-1, D)

    def step(w, b):
        args = (d["seq_offsets"], d["timestamps"], d["rab_pos"], d["rab_time"], N)
        ao, y, mu, rs = hs.hstu_layer_fwd(d["q"], d["k"], d["v"], d["u"], *args, ln_weight=w,
                                          ln_bias=b)
        g = hs.hstu_layer_bwd(d["q"], d["k"], d["v"], d["u"], ao, mu, rs, dy, *args, ln_weight=w,
                              ln_bias=b)
        torch.cuda.synchronize()
        return [y, *g[:6]]

    def shifted(x):
        return torch.cat([x.new_zeros(1), x])[1:]

    ref = step(w, b)
    for x, y in zip(ref, step(shifted(w), shifted(b))):
        assert torch.equal(x, y)
