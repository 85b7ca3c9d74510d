"""bf16 forward products of few output tiles (gemm_bf16_skinny_kernel in kernels_gemm_mfma.hip) at the edges of tiles, k tiles and
rounds of four k tiles: in four parts against fp64, in chains against the 64 x 64 tiles, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8, 8), (31, 64, 40), (32, 72, 32), (33, 128, 72), (100, 192, 64), (64, 256, 96), (7, 264, 200), (96, 320, 33), (50, 520, 130),
          (65, 832, 520), (256, 40, 1024), (257, 40, 1024), (8, 2056, 8), (40, 512, 4096)]


def _layer(rows, fin, fout, act, layers, streams, mb=None, n=1):
    import torch
    from paper_2509_23241_amd import binding as B
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows + fin)
    params = [(rng.standard_normal(s) / np.sqrt(s[1] if len(s) > 1 else 4)).astype(np.float32) for l in layers
              for s in B.layer_param_shapes(l)]
    st = GpuStage(layers, params, dtype="bf16", mb=mb or rows, n=n, stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0,
                  momentum=0.0, ring_capacity=1, max_in_flight=2, forward_stream=streams)
    g = torch.Generator(device="cuda")
    g.manual_seed(fout)
    x = torch.randn(st.mb, st.in_elems, generator=g, device="cuda").to(torch.bfloat16)
    y, _ = st.forward(0, 0, x)
    st.forward_join()
    kept = st.saved_input(0, 0, 0)
    assert torch.equal(kept.reshape(-1), x.reshape(-1))
    out = y.clone(), params, x.float().cpu().numpy()
    st.close()
    return out


@pytest.mark.parametrize("rows,fin,fout", SHAPES)
@pytest.mark.parametrize("act", ["none", "gelu"])
def test_in_four_parts(rows, fin, fout, act):
    from scipy.special import erf
    from synth_inputs import round_bf16
    y, (W, b), x = _layer(rows, fin, fout, act, [(fin, fout, act)], 2)
    z = x.astype(np.float64) @ round_bf16(W).astype(np.float64).T + b
    want = 0.5 * z * (1 + erf(z / np.sqrt(2))) if act == "gelu" else z
    got = y.float().cpu().numpy().reshape(want.shape)
    # the sum: fin / 16 steps of 2^-24 each at most of a partial sum; the stored result is rounded once
    tol = max(2.0 ** -22, 2.0 ** -23 * np.sqrt(fin / 3)) + 2.0 ** -9
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
    assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -20 * fin)


@pytest.mark.parametrize("rows,fin,fout", SHAPES)
def test_in_chains(rows, fin, fout):
    """Two tokens per sample: the order of the sums is kept.  With a forward stream the product runs on the larger tiles."""
    import torch
    layers = [(fin, fout, "gelu", 2)]
    small, _, _ = _layer(rows, fin, fout, "gelu", layers, 0)
    large, _, _ = _layer(rows, fin, fout, "gelu", layers, 1)
    assert torch.equal(small, large)


@pytest.mark.parametrize("rows,width", [(3, 8), (31, 72), (64, 264), (33, 520)])
def test_in_chains_with_an_addend(rows, width):
    import torch
    layers = [("res", width, 3, "begin"), (width, width, "gelu", 3), ("res", width, 3, "add")]
    small, _, _ = _layer(rows, width, width, "gelu", layers, 0)
    large, _, _ = _layer(rows, width, width, "gelu", layers, 1)
    assert torch.equal(small, large)
