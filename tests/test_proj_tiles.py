"""The linear maps over the product kernels' tile sizes and ring depths: token
counts around the 128- and 256-row tiles, widths off the tiles, contractions
of 2, 4, 6 and more 32-wide steps, batches that take 256 x 128 and 256 x 256
tiles, outputs past half of the last-level cache (stores that bypass it), and
token splits that end inside a step; against torch in fp64 on the same
values.  The bound is the storage rounding plus 1e-3 of the result's RMS for
bf16 outputs (dx, whose dpre is rounded to bf16 first: 2e-2), 1e-4 for the fp32
weight gradients (dw1, from the rounded dpre: 2e-2) and 1e-5 for the bias
gradients."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [
    # T, d_model, heads, d_qk, d_v
    (127, 64, 1, 32, 64), (128, 64, 1, 64, 64), (129, 128, 2, 32, 32), (255, 192, 1, 64, 64),
    (257, 320, 3, 64, 64), (1000, 64, 5, 64, 64),
    (33, 576, 9, 64, 64),
    (20011, 448, 8, 64, 64),    # 256 x 128 tiles of f_1
    (57500, 64, 1, 64, 64),     # 256 x 256 tiles, two contraction steps
    (57345, 96 * 2, 3, 64, 64),
    (34001, 64, 8, 128, 128),   # f_1's output past half of the last-level cache
]


def _close(name, got, ref, tau):
    got, ref = got.double(), ref.double()
    u = 2.0 ** -8 if tau[1] else 0.0
    rms = ref.pow(2).mean().sqrt()
    err = ((got - ref).abs() - u * ref.abs()).clamp(min=0).max() / rms
    assert err <= tau[0], f"{name}: {err.item():.2e} of the RMS"


@pytest.mark.parametrize("T,D,h,dqk,dv", SHAPES)
def test_proj_tiles(T, D, h, dqk, dv):
    from paper_2402_17152_amd import hstu
    g = torch.Generator(device="cuda").manual_seed(T + D)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(torch.bfloat16)

    hv, hq = h * dv, h * dqk
    F = 2 * hv + 2 * hq
    x, w1, b1 = rand(T, D), rand(F, D, std=D ** -0.5), rand(F).float()
    gg, w2, b2, dy = rand(T, hv), rand(D, hv, std=hv ** -0.5), rand(D).float(), rand(T, D)
    z, z_pre = hstu.hstu_proj_in_fwd(x, w1, b1, h, dqk, dv)
    pre = x.double() @ w1.double().t() + b1.double()
    _close("z_pre", z_pre, pre, (1e-3, True))
    _close("z", z, torch.nn.functional.silu(pre), (1e-3, True))
    y = hstu.hstu_proj_out_fwd(gg, w2, b2, x, h, dqk, dv)
    _close("y", y, gg.double() @ w2.double().t() + b2.double() + x.double(), (1e-3, True))
    dg, dw2, db2 = hstu.hstu_proj_out_bwd(gg, w2, dy, h, dqk, dv)
    _close("dg", dg, dy.double() @ w2.double(), (1e-3, True))
    _close("dw2", dw2, dy.double().t() @ gg.double(), (1e-4, False))
    _close("db2", db2, dy.double().sum(0), (1e-5, False))
    dz = [rand(T, h, d) for d in (dv, dv, dqk, dqk)]
    dx, dw1, db1 = hstu.hstu_proj_in_bwd(x, w1, z_pre, *dz, h, dqk, dv, dx_add=dy)
    p = z_pre.double()
    sg = torch.sigmoid(p)
    dpre = torch.cat([t.flatten(1) for t in dz], 1).double() * sg * (1 + p * (1 - sg))
    _close("dx", dx, dpre @ w1.double() + dy.double(), (2e-2, True))
    _close("dw1", dw1, dpre.t() @ x.double(), (2e-2, False))
    _close("db1", db1, dpre.sum(0), (1e-5, False))


@pytest.mark.parametrize("T,D,h,dqk,dv", [(70001, 1024, 1, 32, 64), (70001, 64, 16, 32, 64)])
def test_proj_streamed_sums(T, D, h, dqk, dv):
    """y (with its residual) and dx (with dx_add), then dg, past half of the
    last-level cache, with a ragged last tile: the stores of the products
    without a SiLU that bypass the cache."""
    test_proj_tiles(T, D, h, dqk, dv)
