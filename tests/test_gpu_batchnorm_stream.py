"""The streaming batch-normalisation kernels (kernels_batchnorm.hip) at the edges of their row chunks, unit lanes and
rows in flight: output, input gradient and both parameter gradients of two micro-batches against fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# fp32: an output passes at most 8 roundings of 2^-24; the variance is a difference of sums up to 10 times its size (the
# shift by a channel's first value is up to three standard deviations), each behind a chain of at most 128 additions
# (chunk / row lanes + row lanes + chunks / 16), whose roundings add up as their root.
TOL = 2.0 ** -24 * (8 + 10 * np.sqrt(128.0))
TOL_BF16 = 2.0 ** -8      # what a bf16 output is rounded by


def _rel(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("dtype,rows,C", [
    ("f32", 3, 4), ("f32", 17, 16), ("f32", 257, 20), ("f32", 1000, 36), ("f32", 5001, 64), ("f32", 4099, 132),
    ("f32", 2100, 6),                                                       # no whole 16-byte units
    ("bf16", 2049, 8), ("bf16", 2500, 32), ("bf16", 2600, 40), ("bf16", 5001, 64), ("bf16", 4100, 72), ("bf16", 70001, 136),
    ("bf16", 2051, 12),                                                     # no whole 16-byte units
])
def test_stream_batchnorm(dtype, rows, C):
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows + C)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gamma = (1 + 0.2 * rng.standard_normal(C)).astype(np.float32)
    beta = rng.standard_normal(C).astype(np.float32)
    mu = rng.standard_normal(C)
    x = [torch.from_numpy(rng.standard_normal((1, rows, C)) + mu).reshape(1, rows * C).to(td) for _ in range(2)]
    dy = torch.from_numpy(rng.standard_normal((2, rows * C))).to(td)
    st = GpuStage([("bn", C, rows, "none")], [gamma, beta], dtype=dtype, mb=1, n=2, stage_index=1, num_stages=2,
                  policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    ys = [st.forward(0, i, x[i].cuda())[0].float().cpu().numpy().reshape(rows, C) for i in range(2)]
    dx, _ = st.backward(0, dy.cuda())
    dx = dx.float().cpu().numpy().reshape(2, rows, C)
    gg, gb = st.unpack(st.grad.cpu().numpy())
    st.close()
    rg, rb = np.zeros(C), np.zeros(C)
    out = TOL if dtype == "f32" else TOL_BF16
    for i in range(2):
        x64, d64 = x[i].double().numpy().reshape(rows, C), dy[i].double().numpy().reshape(rows, C)
        rstd = 1.0 / np.sqrt(x64.var(0) + 1e-5)
        xh = (x64 - x64.mean(0)) * rstd
        assert _rel(ys[i], xh * gamma + beta) <= out
        assert _rel(dx[i], gamma * rstd * (d64 - d64.mean(0) - xh * (d64 * xh).mean(0))) <= out
        rg += (d64 * xh).sum(0)
        rb += d64.sum(0)
    assert _rel(gg, rg) <= TOL and _rel(gb, rb) <= TOL


def test_row_lanes_are_added_by_pairs_in_fp32():
    """Shift gradient of 64 rows.  A rounding of a partial sum s is off by 0.39 * 2^-24 |s| (root mean square over a binade).
    Sixteen row lanes by pairs: four levels, each off by one such rounding of the whole; the four chunks one after the
    other: partial sums of 2, 3 and 4 quarters.  A quarter is allowed for; sixteen lanes in a chain are 1.3 times off."""
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    rows, C = 64, 1024
    rng = np.random.default_rng(5)
    dy = rng.standard_normal((1, rows * C)).astype(np.float32)
    st = GpuStage([("bn", C, rows, "none")], [np.ones(C, np.float32), np.zeros(C, np.float32)], dtype="f32", mb=1, n=1,
                  stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    st.forward(0, 0, torch.from_numpy(rng.standard_normal((1, rows * C)).astype(np.float32)).cuda())
    st.backward(0, torch.from_numpy(dy).cuda())
    _, gb = st.unpack(st.grad.cpu().numpy())
    st.close()
    off = _rel(gb, dy.reshape(rows, C).astype(np.float64).sum(0))
    assert off <= 1.25 * 0.39 * 2.0 ** -24 * np.sqrt(4 + (2 + 3 + 4) / 4), off


@pytest.mark.parametrize("dtype,rows,C,n", [
    ("bf16", 2049, 64, 1), ("bf16", 5001, 256, 3), ("bf16", 2500, 2048, 2),   # units of a row: 8, 32, all lanes of a workgroup
    ("bf16", 70000, 8, 4), ("bf16", 2500, 2064, 1), ("bf16", 4000, 24, 2),    # one; more than lanes, three: a pass of their own
    ("f32", 100, 16, 3), ("f32", 3001, 1024, 2), ("f32", 65, 6, 2),           # 4, all lanes; values one by one
])
def test_bias_gradient_in_front_of_a_normalisation(dtype, rows, C, n):
    """The bias gradient of the dense layer in front is the column sum of the dx the normalisation stores; so is the
    weight gradient at an input that is 1 everywhere.  Both are fp32 sums of the same rows * n values: an error of a sum of N
    values of size r stays below N 2^-24 r, while a part left out would be missed by its values' size."""
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows + C)
    W = rng.standard_normal((C, 8)).astype(np.float32)
    st = GpuStage([(8, C, "none", rows), ("bn", C, rows, "none")],
                  [W, np.zeros(C, np.float32), np.ones(C, np.float32), np.zeros(C, np.float32)], dtype=dtype, mb=1, n=n,
                  stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = torch.randn(n, rows, 8, generator=g, device="cuda").to(st.tdtype)
    x[..., 0] = 1
    dy = torch.randn(n, rows, C, generator=g, device="cuda").to(st.tdtype)
    for ub in range(n):
        st.forward(0, ub, x[ub].reshape(1, -1))
    st.backward(0, dy.reshape(n, -1))
    gw, gb = st.unpack(st.grad.cpu().numpy())[:2]
    st.close()
    z = x.double() @ torch.from_numpy(W).cuda().double().T
    d = dy.double()
    rstd = 1 / torch.sqrt(z.var(1, unbiased=False, keepdim=True) + 1e-5)
    zh = (z - z.mean(1, keepdim=True)) * rstd
    dx = rstd * (d - d.mean(1, keepdim=True) - zh * (d * zh).mean(1, keepdim=True))
    size = dx.pow(2).mean((0, 1)).sqrt().cpu().numpy()
    assert np.all(np.abs(gb.astype(np.float64) - gw[:, 0]) <= 2 * rows * n * 2.0 ** -24 * size)
