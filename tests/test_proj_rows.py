"""A row of the linear maps' outputs has the same bits wherever it lies in a
batch and whatever batch it lies in: rows projected alone, in another order,
and in batches that take 128 x 128, 256 x 128 and 256 x 256 tiles."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# T of the batch, d_model, heads, d_qk, d_v
SHAPES = [(1500, 64, 1, 64, 64), (1031, 512, 8, 64, 64),
          (20011, 448, 8, 64, 64),   # 256 x 128 tiles of f_1
          (57500, 256, 4, 64, 64)]   # 256 x 256 tiles of f_2 and the gradients


@pytest.mark.parametrize("T,D,h,dqk,dv", SHAPES)
def test_rows_do_not_depend_on_their_place(T, D, h, dqk, dv):
    from paper_2402_17152_amd import hstu
    g = torch.Generator(device="cuda").manual_seed(T)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(torch.bfloat16)

    hv, hq = h * dv, h * dqk
    F = 2 * hv + 2 * hq
    w1, b1, w2, b2 = rand(F, D, std=D ** -0.5), rand(F).float(), rand(D, hv, std=hv ** -0.5), \
        rand(D).float()
    x, gg, dy = rand(T, D), rand(T, hv), rand(T, D)
    dz = [rand(T, h, d) for d in (dv, dv, dqk, dqk)]

    def maps(rows):
        xr, gr, yr = x[rows], gg[rows], dy[rows]
        z, z_pre = hstu.hstu_proj_in_fwd(xr, w1, b1, h, dqk, dv)
        y = hstu.hstu_proj_out_fwd(gr, w2, b2, xr, h, dqk, dv)
        dg = hstu.hstu_proj_out_bwd(gr, w2, yr, h, dqk, dv)[0]
        dx = hstu.hstu_proj_in_bwd(xr, w1, z_pre, *[t[rows] for t in dz], h, dqk, dv, dx_add=yr)[0]
        return dict(z=z, z_pre=z_pre, y=y, dg=dg, dx=dx)

    every = torch.arange(T, device="cuda")
    ref = maps(every)
    torch.cuda.synchronize()
    for rows in (torch.roll(every, 777), every[T // 3:T // 3 + 300], every[T - 1:]):
        for name, got in maps(rows).items():
            assert torch.equal(got, ref[name][rows]), name
