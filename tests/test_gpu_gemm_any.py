"""The matrix-core kernels for shapes that fill no tile (kernels_gemm_any.hip, kernels_gemm_mfma.hip), at the edges of
their tiles: one layer's forward, input gradient and weight gradient against fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rel(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref))


def _sum_tol(terms):
    """fp32 sum of `terms` products in one chain: every step rounds a partial sum by at most 2^-24 of it; with random
    signs that is below 2^-24 sqrt(terms / 3) of the result, and the bound used is twice that (at least 4 ulp)."""
    return max(2.0 ** -22, 2.0 * 2.0 ** -24 * np.sqrt(terms / 3.0))


def _stage(layer, params, rows, dtype):
    from paper_2509_23241_amd.runner import GpuStage
    return GpuStage([layer], params, dtype=dtype, mb=rows, n=1, stage_index=1, num_stages=2, policy="latest", lam=0.1,
                    lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)


def _run(st, x, dy):
    import torch
    y, _ = st.forward(0, 0, torch.from_numpy(x).cuda().to(st.tdtype))
    dx, _ = st.backward(0, torch.from_numpy(dy).cuda().to(st.tdtype))
    out = y.float().cpu().numpy(), dx.float().cpu().numpy(), st.unpack(st.grad.cpu().numpy())
    st.close()
    return out


@pytest.mark.parametrize("rows,fin,fout", [
    # tiles of the forward product, the input gradient and the weight gradient (and its row ranges); 16-byte rows / words
    (1, 1, 1), (31, 33, 35), (32, 32, 32), (33, 36, 100),     # 32: less than one, one, one and a bit
    (1030, 1028, 1000),                                       # 32, 32, 128 over 3 ranges; 16 bytes
    (1023, 1021, 1027),                                       # 32, 64, 128 over 3 ranges; words
    (1024, 1024, 1024), (1500, 1504, 1500), (1499, 1501, 1503),   # 64, 64, 128 over 4 ranges | 64 in all three, both ways
    (2050, 2052, 2048), (2049, 2047, 2051),                   # 64 in all three, both ways
    (2048, 2044, 2040), (2047, 2045, 2043),                   # 128 in all three, both ways
    (4090, 1020, 1024),                                       # 128, 128, 128 over 4 ranges
    (2100, 40, 36), (2100, 41, 39),                           # 32, 32, 32 over 8 ranges, with a remainder
])
def test_dense_fp32(rows, fin, fout):
    rng = np.random.default_rng(rows + fin)
    W = (rng.standard_normal((fout, fin)) / np.sqrt(fin)).astype(np.float32)
    b = rng.standard_normal(fout).astype(np.float32)
    x = rng.standard_normal((rows, fin)).astype(np.float32)
    dy = rng.standard_normal((rows, fout)).astype(np.float32)
    y, dx, (gw, gb) = _run(_stage((fin, fout, "none"), [W, b], rows, "f32"), x, dy)
    x64, W64, dy64 = x.astype(np.float64), W.astype(np.float64), dy.astype(np.float64)
    assert _rel(y, x64 @ W64.T + b) <= _sum_tol(fin)
    assert _rel(dx, dy64 @ W64) <= _sum_tol(fout)
    assert _rel(gw, dy64.T @ x64) <= _sum_tol(rows)
    assert _rel(gb, dy64.sum(0)) <= _sum_tol(rows)


@pytest.mark.parametrize("rows,fin,fout", [
    (1, 1, 1), (3, 7, 9), (63, 65, 66), (129, 70, 10),        # values copied one by one at the edges, 64 x 64 tiles
    (1001, 1003, 1002),                                       # the same, 128 x 64 tiles
    (3001, 41, 39), (3001, 39, 40),                           # ... weight gradient over several row ranges
    (1, 8, 8), (130, 56, 16), (100, 200, 104),                # 16-byte chunks, 64 x 64 tiles: less than one k tile, a remainder
    (70, 72, 10),                                             # chunks forward, single values backward
    (3000, 40, 72),                                           # weight gradient over several row ranges, the last one shorter
    (1000, 136, 2040), (2040, 136, 2040), (2040, 136, 4088), (4000, 136, 4088),   # 128 x 64, 128 x 128, 256 x 128, 256 x 256
    (2040, 64, 4088), (2040, 128, 4088), (4000, 64, 4088), (4000, 128, 4088),     # fewer k tiles than the last two have stages
    (72, 2048, 6144), (72, 6144, 2048),                       # weight gradients on 384 x 128 and 128 x 384 tiles
    (6400, 768, 776), (6401, 520, 1032),                      # ... over 6 and 5 row ranges on 128 x 128 tiles
    (16384, 1024, 1024), (16389, 1032, 1032),                 # ... over 4 and 3; input gradients on 256 x 256 and 128 x 128
    (32769, 1024, 1024),                                      # ... over 16 ranges on 256 x 256 tiles, one row in the last k tile
])
@pytest.mark.parametrize("shift", [0, 1])                     # 1: the input starts at an odd element (rows of chunks: its copy is used)
def test_dense_bf16(rows, fin, fout, shift):
    import torch
    from synth_inputs import round_bf16
    if shift and rows > 1001:
        pytest.skip("alignment decides the kernel, which the smaller shapes run")
    rng = np.random.default_rng(rows + fin)
    cast = lambda t: round_bf16(t).astype(np.float32)
    W = cast(rng.standard_normal((fout, fin)) / np.sqrt(fin))
    b = rng.standard_normal(fout).astype(np.float32)
    x, dy = cast(rng.standard_normal((rows, fin))), cast(rng.standard_normal((rows, fout)))
    st = _stage((fin, fout, "none"), [W, b], rows, "bf16")
    xs = torch.zeros(rows * fin + shift, dtype=torch.bfloat16, device="cuda")
    ys = torch.zeros(rows * fout + shift, dtype=torch.bfloat16, device="cuda")
    xt, yt = xs[shift:].view(rows, fin), ys[shift:].view(rows, fout)
    xt.copy_(torch.from_numpy(x))
    st.forward(0, 0, xt, yt)
    dx, _ = st.backward(0, torch.from_numpy(dy).cuda().to(st.tdtype))
    gw, gb = st.unpack(st.grad.cpu().numpy())
    x64, W64, dy64 = x.astype(np.float64), W.astype(np.float64), dy.astype(np.float64)
    store = 2.0 ** -9                                         # the stored result is rounded once
    assert _rel(yt.float().cpu().numpy(), x64 @ W64.T + b) <= _sum_tol(fin) + store
    assert _rel(dx.float().cpu().numpy(), dy64 @ W64) <= _sum_tol(fout) + store
    assert _rel(gw, dy64.T @ x64) <= _sum_tol(rows)
    assert _rel(gb, dy64.sum(0)) <= _sum_tol(rows)
    st.close()


def test_operands_of_more_than_2_gib():
    """Byte offsets of an operand beyond 31 bits: rows at both ends, the input gradient and the weight gradient."""
    import torch
    rows, fin, fout = 1050000, 1024, 64                      # an input of 2.15 GB
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.empty(rows, fin, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    dy = torch.empty(rows, fout, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    W = (torch.randn(fout, fin, generator=g, device="cuda") / 32).to(torch.bfloat16).float()
    st = _stage((fin, fout, "none"), [W.cpu().numpy(), np.zeros(fout, np.float32)], rows, "bf16")
    y, _ = st.forward(0, 0, x)
    dx, _ = st.backward(0, dy)
    gw = torch.from_numpy(np.ascontiguousarray(st.unpack(st.grad.cpu().numpy())[0])).cuda().double()
    st.close()
    store = 2.0 ** -9
    for part in (slice(0, 1000), slice(524000, 525000), slice(rows - 1000, rows)):
        a, d = x[part].double(), dy[part].double()
        ry, rdx = a @ W.double().T, d @ W.double()
        assert float((y[part].double() - ry).norm() / ry.norm()) <= _sum_tol(fin) + store
        assert float((dx[part].double() - rdx).norm() / rdx.norm()) <= _sum_tol(fout) + store
    want = sum(dy[i:i + 150000].double().T @ x[i:i + 150000].double() for i in range(0, rows, 150000))
    assert float((gw - want).norm() / want.norm()) <= _sum_tol(rows)


@pytest.mark.parametrize("rows,fin,fout,act", [(256, 128, 256, "none"), (2048, 64, 4096, "gelu"), (128, 4096, 256, "gelu")])
@pytest.mark.parametrize("offset", [1, 2, 4])                 # elements: 2, 4 and 8 bytes
def test_outputs_at_any_address(rows, fin, fout, act, offset):
    """Whole tiles from aligned operands into a y and a dx that are not 16-byte aligned: the bits of the aligned ones."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    W = (torch.randn(fout, fin, generator=g, device="cuda") / fin ** 0.5).cpu().numpy()
    x = torch.randn(rows, fin, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(rows, fout, generator=g, device="cuda").to(torch.bfloat16)
    got = []
    for at in (0, offset):
        st = _stage((fin, fout, act), [W, np.zeros(fout, np.float32)], rows, "bf16")
        ys = torch.full((rows * fout + 16,), 3.0, dtype=torch.bfloat16, device="cuda")
        dxs = torch.full((rows * fin + 16,), 3.0, dtype=torch.bfloat16, device="cuda")
        st.forward(0, 0, x, ys[at:at + rows * fout].view(rows, fout))
        st.backward(0, dy, dxs[at:at + rows * fin].view(rows, fin))
        for t, n in ((ys, rows * fout), (dxs, rows * fin)):
            assert bool((t[:at] == 3).all()) and bool((t[at + n:] == 3).all())   # and nothing beside them
            got.append(t[at:at + n].clone())
        st.close()
    assert torch.equal(got[0], got[2]) and torch.equal(got[1], got[3])


def test_gelu_of_odd_widths_is_the_erf_form():
    """The bias alone as pre-activation, z in -4 .. -2: an fp32 error e of 0.5 z (1 + erf(z / sqrt 2)) makes the stored bf16
    value another one than fp64 gives with probability |e| / (spacing of bf16 there).  erf near -1, rounded correctly, is off
    by 2^-26 on average: 0.5 |z| 2^-26 over the spacing, 0.53 % on average over the range.  Twice that is allowed; the
    polynomial form, off by up to 1.5e-7, has 2 %."""
    import math
    import torch
    n = 100001
    z = np.linspace(-4.0, -2.0, n).astype(np.float32)
    st = _stage((1, n, "gelu"), [np.ones((n, 1), np.float32), z], 1, "bf16")
    y, _ = st.forward(0, 0, torch.zeros(1, 1, dtype=torch.bfloat16, device="cuda"))
    z64 = torch.from_numpy(z.astype(np.float64))
    want = (0.5 * z64 * torch.erfc(-z64 / math.sqrt(2.0))).float().to(torch.bfloat16)
    differ = float((y.cpu()[0] != want).double().mean())
    print(differ)
    st.close()
    assert differ <= 2 * 0.0053


def test_dense_bf16_keeps_nonfinite_values_in_their_row():
    """Remainders of a k tile are zeros in both operands: an infinity reaches its own row only."""
    import torch
    rows, fin, fout = 70, 72, 80
    st = _stage((fin, fout, "none"), [np.ones((fout, fin), np.float32), np.zeros(fout, np.float32)], rows, "bf16")
    x = torch.ones(rows, fin, dtype=torch.bfloat16, device="cuda")
    x[5, fin - 1] = float("inf")
    y, _ = st.forward(0, 0, x)
    want = torch.full((rows, fout), float(fin), device="cuda")
    want[5] = float("inf")
    assert torch.equal(y.float(), want)
    st.close()


def _conv_reference(x, W, b, dy, stride):
    """fp64 convolution and its gradients (torch on the CPU); NHWC tensors."""
    import torch
    xt = torch.from_numpy(x.astype(np.float64)).permute(0, 3, 1, 2).requires_grad_(True)
    Wt = torch.from_numpy(W.astype(np.float64)).permute(0, 3, 1, 2).requires_grad_(True)
    y = torch.nn.functional.conv2d(xt, Wt, torch.from_numpy(b.astype(np.float64)), stride=stride, padding=(W.shape[1] - 1) // 2)
    y.backward(torch.from_numpy(dy.astype(np.float64)).permute(0, 3, 1, 2))
    back = lambda t: t.detach().permute(0, 2, 3, 1).numpy()
    return back(y), back(xt.grad), back(Wt.grad)


@pytest.mark.parametrize("dtype,imgs,H,W,cin,cout,k,stride", [
    ("f32", 2, 5, 7, 3, 6, 3, 1),         # words, 32 x 32 tiles, every border
    ("f32", 3, 6, 10, 4, 12, 5, 2),       # 16-byte chunks that straddle taps inside a k tile, stride 2
    ("f32", 1, 4, 4, 20, 8, 1, 1),        # 1x1: the division by a kernel edge of one
    # tiles of forward product, input gradient and weight gradient (over its pixel ranges)
    ("f32", 40, 24, 24, 68, 64, 3, 1),    # 64, 64, 64 over 25
    ("f32", 150, 16, 16, 128, 132, 3, 1), # 64, 64, 128 over 14
    ("f32", 128, 16, 16, 128, 128, 3, 1), # 128, 128, 128 over 28
    ("f32", 128, 16, 16, 124, 128, 1, 1), # 128, 128, 64 over 64; a last tile of channels that is not whole
    ("f32", 127, 16, 16, 127, 125, 1, 1), # the same word by word
    ("bf16", 2, 6, 5, 8, 16, 3, 1),       # 32 in all three, image sizes that are no powers of two
    ("bf16", 3, 12, 20, 24, 40, 7, 2),
    ("bf16", 40, 24, 24, 64, 72, 3, 1),   # 32, 32, 128 over 45
    ("bf16", 90, 28, 28, 48, 56, 3, 1),   # 64, 64, 64 over 36
    ("bf16", 180, 20, 20, 96, 128, 5, 1), # 64, 32, 128 over 13
])
def test_convolution(dtype, imgs, H, W, cin, cout, k, stride):
    from synth_inputs import round_bf16
    rng = np.random.default_rng(imgs * H + k)
    cast = round_bf16 if dtype == "bf16" else (lambda t: t.astype(np.float32))
    wgt = cast(rng.standard_normal((cout, k, k, cin)) / np.sqrt(k * k * cin)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    x = cast(rng.standard_normal((imgs, H, W, cin))).astype(np.float32)
    dy = cast(rng.standard_normal((imgs, H // stride, W // stride, cout))).astype(np.float32)
    y, dx, (gw, gb) = _run(_stage(("conv", cin, cout, H, W, "none", stride, k), [wgt, b], imgs, dtype),
                           x.reshape(imgs, -1), dy.reshape(imgs, -1))
    ry, rdx, rgw = _conv_reference(x, wgt, b, dy, stride)
    # bf16: products of bf16 values are exact in fp32, the sums are fp32, the stored result is rounded once (2^-9 of it)
    store = 2.0 ** -9 if dtype == "bf16" else 0.0
    pixels = imgs * (H // stride) * (W // stride)
    assert _rel(y.reshape(ry.shape), ry) <= _sum_tol(k * k * cin) + store
    assert _rel(dx.reshape(rdx.shape), rdx) <= _sum_tol(k * k * cout) + store
    assert _rel(gw, rgw) <= _sum_tol(pixels)
    assert _rel(gb, dy.astype(np.float64).sum((0, 1, 2))) <= _sum_tol(pixels)


@pytest.mark.parametrize("dtype,imgs,size,cin,cout,k,stride", [
    ("f32", 16, 32, 64, 64, 3, 1), ("f32", 16, 16, 128, 128, 3, 1),   # ranges longer than a part, 64 x 64 and 128 x 128 tiles
    ("f32", 9, 20, 3, 12, 5, 2),                                      # the last part not whole, words
    ("bf16", 16, 20, 96, 128, 3, 1), ("bf16", 8, 64, 48, 48, 3, 1),
])
def test_convolution_weight_gradient_is_summed_in_parts(dtype, imgs, size, cin, cout, k, stride):
    """Products of 256 pixels are added up apart.  A rounding of a partial sum s is off by 0.39 * 2^-24 |s| (root mean square over
    a binade); the squares of n partial sums of random terms add up to n / 2 times that of the last one, so a sum of P
    products in parts of n roundings each is off by 0.39 * 2^-24 * sqrt(n / 2 + P / 512): n = 256 in fp32, 8 in bf16, where
    a matrix instruction adds 32 products.  One chain over a range of 512 would exceed it by 1.4; 15 % are allowed for."""
    from synth_inputs import round_bf16
    rng = np.random.default_rng(imgs * size + k)
    cast = round_bf16 if dtype == "bf16" else (lambda t: t.astype(np.float32))
    wgt = cast(rng.standard_normal((cout, k, k, cin))).astype(np.float32)
    x = cast(rng.standard_normal((imgs, size, size, cin))).astype(np.float32)
    dy = cast(rng.standard_normal((imgs, size // stride, size // stride, cout))).astype(np.float32)
    b = np.zeros(cout, np.float32)
    _, _, (gw, _) = _run(_stage(("conv", cin, cout, size, size, "none", stride, k), [wgt, b], imgs, dtype),
                         x.reshape(imgs, -1), dy.reshape(imgs, -1))
    off = _rel(gw, _conv_reference(x, wgt, b, dy, stride)[2])
    pixels = imgs * (size // stride) ** 2
    roundings = min(pixels, 256) / (32 if dtype == "bf16" else 1)
    bound = 1.15 * 0.39 * 2.0 ** -24 * np.sqrt(roundings / 2 + pixels / 512)
    print(off, bound)
    assert off <= bound


def _chain(a, b):
    """out[m][n] = fma(a[m][k], b[n][k], .) over ascending k in fp32: product and sum of two fp32 values have at most 48 + 24
    bits, the 64 of a long double round them a second time in fewer than 1 of 2^38 steps."""
    acc = np.zeros((a.shape[0], b.shape[0]), np.float32)
    for k in range(a.shape[1]):
        acc = (a[:, k, None].astype(np.longdouble) * b[None, :, k].astype(np.longdouble) + acc).astype(np.float32)
    return acc


def test_fp32_products_are_one_chain_of_fused_multiply_adds():
    rng = np.random.default_rng(2)
    for rows, fin, fout in ((33, 70, 45), (40, 64, 72)):                       # words, 16-byte rows
        W, x, dy = [rng.standard_normal(shape).astype(np.float32) for shape in ((fout, fin), (rows, fin), (rows, fout))]
        y, dx, _ = _run(_stage((fin, fout, "none"), [W, np.zeros(fout, np.float32)], rows, "f32"), x, dy)
        assert np.array_equal(y, _chain(x, W)) and np.array_equal(dx, _chain(dy, W.T))


@pytest.mark.parametrize("dtype,cin,cout,stride", [("f32", 3, 10, 1), ("f32", 12, 8, 2), ("bf16", 8, 16, 1)])
def test_convolutions_are_one_chain_of_fused_multiply_adds(dtype, cin, cout, stride):
    from synth_inputs import round_bf16
    rng = np.random.default_rng(cin)
    cast = round_bf16 if dtype == "bf16" else (lambda t: t.astype(np.float32))
    imgs, H, W_, k = 2, 6, 10, 3
    wgt, x, dy = [cast(rng.standard_normal(shape)).astype(np.float32)
                  for shape in ((cout, k, k, cin), (imgs, H, W_, cin), (imgs, H // stride, W_ // stride, cout))]
    y, dx, _ = _run(_stage(("conv", cin, cout, H, W_, "none", stride, k), [wgt, np.zeros(cout, np.float32)], imgs, dtype),
                    x.reshape(imgs, -1), dy.reshape(imgs, -1))
    # the operand rows as the kernels gather them: (tap, channel) ascending, zeros outside the image
    ho, wo = H // stride, W_ // stride
    pad = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    fwd = np.stack([pad[:, kh:kh + stride * ho:stride, kw:kw + stride * wo:stride] for kh in range(k) for kw in range(k)], 3)
    spread = np.zeros((imgs, H + 2, W_ + 2, cout), np.float32)                  # dz at the positions of its input pixels
    spread[:, 1:1 + stride * ho:stride, 1:1 + stride * wo:stride] = dy
    back = np.stack([spread[:, 2 - kh:2 - kh + H, 2 - kw:2 - kw + W_] for kh in range(k) for kw in range(k)], 3)
    ry = _chain(fwd.reshape(-1, k * k * cin), wgt.reshape(cout, -1))
    rdx = _chain(back.reshape(-1, k * k * cout), wgt.transpose(3, 1, 2, 0).reshape(cin, -1))
    assert np.array_equal(y.reshape(ry.shape), cast(ry)) and np.array_equal(dx.reshape(rdx.shape), cast(rdx))


def test_fp32_products_have_the_same_bits_on_every_tile():
    """The rows of a small call inside larger ones: 32, 64 and 128 tiles, rows copied in 16-byte units and word by word."""
    import torch
    fin = fout = 1020                                        # 128 rows: tiles of 32, 1024: 64, 4096: 128
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    W = torch.randn(fout, fin, generator=g, device="cuda").cpu().numpy()
    x, dy = [torch.randn(4096, 1020, generator=g, device="cuda") for _ in range(2)]
    first = None
    for rows in (128, 1024, 4096):
        for shift in (0, 1):                                 # 1: operands that are not 16-byte aligned
            room = [torch.empty(rows * 1020 + shift, device="cuda")[shift:].view(rows, 1020).copy_(t[:rows]) for t in (x, dy)]
            st = _stage((fin, fout, "none"), [W, np.zeros(fout, np.float32)], rows, "f32")
            y, _ = st.forward(0, 0, room[0])
            dx, _ = st.backward(0, room[1])
            got = y[:128].clone(), dx[:128].clone()
            st.close()
            first = first or got
            assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1]), (rows, shift)


@pytest.mark.parametrize("rows,widths", [
    # k tiles of 32 in the contractions of two layers, both ways: 1, 2 | 6, 7 | 7, 8 | 8, 9 | 15, 16, 17 of eight stages
    (1, (32, 64, 4)), (17, (192, 224, 64)), (33, (256, 224, 288)), (16, (288, 256, 36)), (50, (480, 512, 544)),
    (40, (64, 32, 10)),                                      # output columns that are no whole unit of four
])
def test_fp32_layers_of_few_tiles_are_chains(rows, widths):
    """One wave per 16 x 16 outputs, with what the epilogues read: bias and ReLU forward, the ReLU's mask backward."""
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows)
    fin, mid, fout = widths
    W1, W2, x, dy = [rng.standard_normal(s).astype(np.float32) for s in ((mid, fin), (fout, mid), (rows, fin), (rows, fout))]
    b1, b2 = [rng.standard_normal(n).astype(np.float32) for n in (mid, fout)]
    st = GpuStage([(fin, mid, "relu"), (mid, fout, "none")], [W1, b1, W2, b2], dtype="f32", mb=rows, n=1, stage_index=1,
                  num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    y, dx, _ = _run(st, x, dy)
    a1 = np.maximum(_chain(x, W1) + b1, np.float32(0))
    assert np.array_equal(y, _chain(a1, W2) + b2)
    dz1 = np.where(a1 > 0, _chain(dy, W2.T), np.float32(0))
    assert np.array_equal(dx, _chain(dz1, W1.T))


@pytest.mark.parametrize("rows,fin,fout", [(256, 1024, 1024), (257, 1024, 1024), (1024, 256, 256)])
def test_fp32_layers_at_the_line_between_waves_and_tiles(rows, fin, fout):
    """1024 tiles of 16 x 16 and one row of them more: the bits of operands at odd addresses, which the tiles of 32 take."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    W = torch.randn(fout, fin, generator=g, device="cuda").cpu().numpy()
    x, dy = torch.randn(rows, fin, generator=g, device="cuda"), torch.randn(rows, fout, generator=g, device="cuda")
    got = []
    for shift in (0, 1):
        xs, ds = [torch.empty(t.numel() + shift, device="cuda")[shift:].view(t.shape).copy_(t) for t in (x, dy)]
        st = _stage((fin, fout, "none"), [W, np.zeros(fout, np.float32)], rows, "f32")
        y, _ = st.forward(0, 0, xs)
        dx, _ = st.backward(0, ds)
        got.append((y.clone(), dx.clone()))
        st.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
