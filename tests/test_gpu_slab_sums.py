"""Column sums of the slab batch-normalisation kernels (kernels_batchnorm.hip), whose lanes meet through LDS and then within a
wave: every unit of a workgroup, rows that leave lanes without one, and both slab widths, against fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,C", [(1, 8), (15, 8), (65, 24), (1000, 40), (1024, 64), (1025, 16), (1500, 48), (2048, 128), (2047, 24)])
def test_slab_batchnorm_sums(rows, C):
    """A value passes at most 4 additions in its lane, 16 next to its neighbours and 6 across the wave, and a normalised one 8
    roundings before that and twice the error of a mean of the same kind: 64 roundings of 2^-24 of the sum of magnitudes.  A
    value left out or added twice is off by 1 / rows of it at least."""
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows + C)
    n = 2
    x = torch.from_numpy(rng.uniform(0.5, 1.5, (n, rows * C)) * rng.choice([-1, 1], (n, rows * C))).to(torch.bfloat16)
    dy = torch.from_numpy(rng.uniform(0.5, 1.5, (n, rows * C)) * rng.choice([-1, 1], (n, rows * C))).to(torch.bfloat16)
    st = GpuStage([("bn", C, rows, "none")], [np.ones(C, np.float32), np.zeros(C, np.float32)], dtype="bf16", mb=1, n=n,
                  stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    ys = [st.forward(0, i, x[i:i + 1].cuda())[0].double().cpu().numpy().reshape(rows, C) for i in range(n)]
    st.backward(0, dy.cuda())
    gg, gb = st.unpack(st.grad.cpu().numpy())
    st.close()
    x64, d64 = x.double().numpy().reshape(n, rows, C), dy.double().numpy().reshape(n, rows, C)
    rstd = 1 / np.sqrt(x64.var(1, keepdims=True) + 1e-5)
    xh = (x64 - x64.mean(1, keepdims=True)) * rstd
    if rows > 1:
        assert np.all(np.abs(np.stack(ys) - xh) <= 2.0 ** -8 * np.abs(xh) + 64 * 2.0 ** -24 * rstd)
    off = 64 * 2.0 ** -24
    mean_off = off * np.abs(x64).mean(1, keepdims=True) * rstd
    assert np.all(np.abs(gb - d64.sum((0, 1))) <= off * np.abs(d64).sum((0, 1)))
    assert np.all(np.abs(gg - (d64 * xh).sum((0, 1))) <= (np.abs(d64) * (off * np.abs(xh) + mean_off)).sum((0, 1)))
