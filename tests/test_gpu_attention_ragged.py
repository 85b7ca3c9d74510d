"""The fused attention kernels on sequences that are not whole blocks of 64 tokens, against the fp64 oracle."""
import pytest

from stage_parity import run_stage
from synth_inputs import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,heads,dh,mb", [
    (1, 2, 64, 3), (31, 1, 128, 2), (65, 2, 64, 2),      # less than a block, a block and one token (four waves)
    (129, 1, 128, 2), (200, 2, 64, 2), (287, 1, 128, 1), # several workgroups per head, the last one partly filled
    (130, 16, 64, 16), (191, 16, 128, 16),               # enough heads for eight waves per workgroup
])
def test_ragged_attention_bf16(tokens, heads, dh, mb):
    d = heads * dh
    specs = (W.Dense(32, 3 * d, "none", tokens=tokens), W.Attention(d, heads, tokens), W.Dense(d, 32, "none", tokens=tokens))
    print(tokens, heads, dh, run_stage(specs, f"attn_ragged_{tokens}_{heads}_{dh}", "bf16", mb=mb, n=2, minibatches=2))


def _attention_stage(tokens, heads, dh, mb):
    """Attention behind which a dense layer passes everything on unchanged (unit matrix: bf16 values times one)."""
    import numpy as np
    from paper_2509_23241_amd.runner import GpuStage
    d = heads * dh
    return GpuStage([("attn", d, heads, tokens), (d, d, "none", tokens)], [np.eye(d, dtype=np.float32), np.zeros(d, np.float32)],
                    dtype="bf16", mb=mb, n=1, stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0,
                    ring_capacity=1, max_in_flight=1)


def _run_attention(qkv, dy, heads):
    """Outputs of one pass: y [mb][tokens][d] and the gradients of q, k, v."""
    mb, tokens, d3 = qkv.shape
    st = _attention_stage(tokens, heads, d3 // 3 // heads, mb)
    y, _ = st.forward(0, 0, qkv.reshape(mb, -1))
    dx, _ = st.backward(0, dy.reshape(mb, -1))
    st.close()
    return (y.reshape(mb, tokens, d3 // 3),) + dx.reshape(mb, tokens, d3).split(d3 // 3, -1)


def _attention64(qkv, dy, heads, stored=None):
    """The same in fp64; `stored`: the output the backward pass forms delta = rowsum(dO . O) from (its own, rounded)."""
    import torch
    mb, S, d3 = qkv.shape
    dh = d3 // 3 // heads
    rows = lambda t: t.double().reshape(mb, S, heads, dh).permute(0, 2, 1, 3).contiguous()
    flat = lambda t: t.permute(0, 2, 1, 3).reshape(mb, S, heads * dh)
    turned = lambda t: t.transpose(-1, -2).contiguous()
    q, k, v = [rows(t) for t in qkv.split(d3 // 3, -1)]
    do = rows(dy)
    s = torch.matmul(q, turned(k)) / dh ** 0.5
    p = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device=s.device).triu(1), -float("inf")).softmax(-1)
    o = torch.matmul(p, v)
    delta = (do * (o if stored is None else rows(stored))).sum(-1, keepdim=True)
    ds = p * (torch.matmul(do, turned(v)) - delta) / dh ** 0.5
    return flat(o), flat(torch.matmul(ds, k)), flat(torch.matmul(turned(ds), q)), flat(torch.matmul(turned(p), do))


@pytest.mark.parametrize("tokens,heads,dh,mb", [
    (2, 8, 128, 4), (3, 8, 64, 4), (4, 8, 64, 4),      # the shortest sequences the fused kernels take, and one they do not
    (17, 8, 64, 4), (31, 4, 128, 4), (65, 8, 64, 4), (100, 4, 128, 2), (287, 4, 128, 2),   # four waves
    (200, 8, 64, 32), (191, 16, 128, 16),                                                                 # eight waves
])
def test_probabilities_and_their_gradients_keep_32_bits(tokens, heads, dh, mb):
    """Only the rounding of a stored result separates it from fp64: probabilities or dS held in bf16 would add errors of
    2^-9 each to the sums, 1.2 to 1.4 times the rounding alone in the norm (fp32 sums: 1e-6, nothing next to 1.6e-3)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    d = heads * dh
    qkv = torch.randn(mb, tokens, 3 * d, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(mb, tokens, d, generator=g, device="cuda").to(torch.bfloat16)
    got = _run_attention(qkv, dy, heads)
    for name, a, ref in zip(("y", "dq", "dk", "dv"), got, _attention64(qkv, dy, heads, got[0])):
        off = float((a.double() - ref).norm() / ref.norm())
        rounding = float((ref.to(torch.bfloat16).double() - ref).norm() / ref.norm())
        print(name, off / rounding)
        assert off <= 1.05 * rounding, name


@pytest.mark.parametrize("tokens,heads,dh,mb", [(40, 2, 64, 2), (70, 2, 128, 2), (130, 2, 64, 1),     # four waves
                                                (150, 16, 64, 16), (150, 16, 128, 16)])                # eight waves
def test_non_finite_values_stay_in_the_rows_that_see_them(tokens, heads, dh, mb):
    """An infinity in a token's value, key or upstream gradient: rows that do not depend on it are what they are without
    (up to the order of the sums: one rounding of the stored result)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    d = heads * dh
    qkv = torch.randn(mb, tokens, 3 * d, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(mb, tokens, d, generator=g, device="cuda").to(torch.bfloat16)
    clean = dict(zip(("y", "dq", "dk", "dv"), _run_attention(qkv, dy, heads)))
    assert all(bool(torch.isfinite(t.float()).all()) for t in clean.values())

    def check(got, rows):
        for name, sel in rows.items():
            a, b = got[name][:, sel].double(), clean[name][:, sel].double()
            assert bool(torch.isfinite(a).all()), name
            assert float((a - b).norm()) <= 2.0 ** -8 * float(b.norm()), name

    t = tokens // 2 + 3
    before, after, others = slice(0, t), slice(t + 1, None), [i for i in range(tokens) if i != t]
    for where, unaffected in (
            ("v", {"y": before, "dq": before, "dv": slice(None)}),     # dV holds no value
            ("k", {"y": before, "dq": before}),
            ("dy", {"y": slice(None), "dq": others, "dk": after, "dv": after})):
        x, u = qkv.clone(), dy.clone()
        part = {"k": x[:, t, d:2 * d], "v": x[:, t, 2 * d:], "dy": u[:, t]}[where]
        part[:, ::3] = float("inf")
        got = dict(zip(("y", "dq", "dk", "dv"), _run_attention(x, u, heads)))
        check(got, unaffected)
        assert not bool(torch.isfinite(got["dq" if where == "dy" else "y"][:, t].float()).all())   # and it does arrive


@pytest.mark.parametrize("tokens", [40, 130])
def test_input_gradient_at_any_address(tokens):
    """Attention as first layer writes its gradients to the caller's tensor, which may start at an odd element."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    heads, dh, mb = 2, 64, 2
    d = heads * dh
    qkv = torch.randn(mb, tokens * 3 * d, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(mb, tokens * d, generator=g, device="cuda").to(torch.bfloat16)
    got = []
    for at in (0, 1):
        st = _attention_stage(tokens, heads, dh, mb)
        st.forward(0, 0, qkv)
        room = torch.full((qkv.numel() + 16,), 3.0, dtype=torch.bfloat16, device="cuda")
        st.backward(0, dy, room[at:at + qkv.numel()].view_as(qkv))
        assert bool((room[:at] == 3).all()) and bool((room[at + qkv.numel():] == 3).all())
        got.append(room[at:at + qkv.numel()].double())
        st.close()
    assert float((got[0] - got[1]).norm()) <= 2.0 ** -8 * float(got[0].norm())   # each rounded once
