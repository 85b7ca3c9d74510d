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
