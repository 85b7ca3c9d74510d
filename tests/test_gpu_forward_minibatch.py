"""stage_forward_minibatch against one stage_forward per micro-batch: outputs, saved inputs and the gradients that follow from them
are the same bits, but where a bf16 stage of dense layers alone has few tiles by micro-batch and more in the whole."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DENSE = [(40, 72, "gelu"), (72, 24, "relu"), (24, 130, "none")]
BLOCK = [("res", 64, 5, "begin"), ("ln", 64, 5), (64, 64, "gelu", 5), ("res", 64, 5, "add"), (64, 32, "none", 5)]
CONV = [("conv", 3, 16, 8, 8, "relu"), ("pool", 16, 8, 8)]
NORM = [(16, 24, "none", 6), ("bn", 24, 6, "relu")]          # statistics of a micro-batch


@pytest.mark.parametrize("layers,dtype,streams", [
    (DENSE, "f32", 0), (DENSE, "bf16", 0), (DENSE, "bf16", 2), (BLOCK, "bf16", 0), (BLOCK, "f32", 0), (CONV, "f32", 0), (NORM, "bf16", 0),
])
@pytest.mark.parametrize("mb,n", [(1, 3), (33, 4), (64, 1)])
def test_whole_minibatch(layers, dtype, streams, mb, n):
    import torch
    from paper_2509_23241_amd import binding as B
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(mb)
    params = [(rng.standard_normal(s) / np.sqrt(np.prod(s[1:]) if len(s) > 1 else 4)).astype(np.float32) for l in layers
              for s in B.layer_param_shapes(l)]
    seen = []
    for whole in (False, True):
        st = GpuStage(layers, params, dtype=dtype, mb=mb, n=n, stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0,
                      momentum=0.0, ring_capacity=1, max_in_flight=2, forward_stream=streams)
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        x = torch.randn(mb * n, st.in_elems, generator=g, device="cuda").to(st.tdtype)
        dy = torch.randn(mb * n, st.out_elems, generator=g, device="cuda").to(st.tdtype)
        y = torch.empty(mb * n, st.out_elems, dtype=st.tdtype, device="cuda")
        if whole:
            _, v = st.forward_minibatch(0, x, y)
            assert v == 0 and st.query().in_flight_forwards[0] == n
            with pytest.raises(RuntimeError):
                st.forward_minibatch(0, x, y)            # the mini-batch has its forwards
        else:
            for ub in range(n):
                st.forward(0, ub, x[ub * mb:(ub + 1) * mb], y[ub * mb:(ub + 1) * mb])
        saved = [st.saved_input(0, ub, len(layers) - 1).clone() for ub in range(n)]
        dx, _ = st.backward(0, dy)
        seen.append([y, dx, st.grad.clone()] + saved)
        st.close()
    for a, b in zip(*seen):
        assert torch.equal(a, b)


@pytest.mark.parametrize("layer,dtype,mb,n,bits", [
    ((264, 520, "gelu"), "bf16", 33, 20, False),    # 34 tiles of 32 x 32 per micro-batch, 357 per mini-batch: in four parts up to 256
    ((2000, 1000, "relu"), "bf16", 100, 4, False),  # 128 and 416
    ((72, 512, "none"), "bf16", 64, 8, True),       # 32 and 256: parts in both
    ((72, 520, "none"), "bf16", 500, 2, True),      # 272: in neither
    ((64, 64, "gelu", 5), "bf16", 50, 20, True),    # several positions per sample: chains, 16 and 314
    ((64, 512, "gelu"), "f32", 33, 20, True),       # 96 and 1344 tiles of 16 x 16: one wave per SIMD up to 1024
])
def test_where_the_number_of_rows_moves_a_product_to_another_kernel(layer, dtype, mb, n, bits):
    """By micro-batches and whole, without and with forward streams.  Two fp32 sums of the same fin products differ by 2 fin roundings of
    2^-24 of the sum of magnitudes at most (and GELU by 1.13 times that), before each is rounded to bf16."""
    import torch
    from paper_2509_23241_amd import binding as B
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(n)
    params = [(rng.standard_normal(s) / np.sqrt(s[1] if len(s) > 1 else 4)).astype(np.float32) for s in B.layer_param_shapes(layer)]
    g = torch.Generator(device="cuda")
    g.manual_seed(mb)
    x, seen = None, {}
    for whole, streams in [(False, 0), (False, 2), (True, 2), (True, 0)]:
        st = GpuStage([layer], params, dtype=dtype, mb=mb, n=n, stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0,
                      momentum=0.0, ring_capacity=1, max_in_flight=2, forward_stream=streams)
        if x is None:
            x = torch.randn(mb * n, st.in_elems, generator=g, device="cuda").to(st.tdtype)
            torch.cuda.synchronize()
        y = torch.empty(mb * n, st.out_elems, dtype=st.tdtype, device="cuda")
        if whole:
            st.forward_minibatch(0, x, y)
        else:
            for ub in range(n):
                st.forward(0, ub, x[ub * mb:(ub + 1) * mb], y[ub * mb:(ub + 1) * mb])
        st.forward_join()
        seen[whole, streams] = y.clone()
        st.close()
    one = seen[False, 0]
    assert torch.equal(seen[False, 2], one) and torch.equal(seen[True, 2], one)
    if bits:
        assert torch.equal(seen[True, 0], one)
        return
    W = torch.from_numpy(params[0]).cuda().to(torch.bfloat16).double()
    off = 1.13 * 2 * layer[0] * 2.0 ** -24 * (x.double().abs() @ W.abs().T)
    a, b = seen[True, 0].double(), one.double()
    assert bool(((a - b).abs() <= off + 2.0 ** -8 * (a.abs() + b.abs())).all())
    assert float((a != b).double().mean()) <= 0.01         # most round alike
