"""stage_forward_minibatch against one stage_forward per micro-batch: outputs, saved inputs and the gradients that follow from them.
At these sizes the products add in one order whatever the number of rows, so the results are the same bits."""
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
