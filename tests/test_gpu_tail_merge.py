"""Merge of a cut tile's key ranges for every number of ranges (one query tile is cut in up to 16)."""
import pytest

from synth import gen_qkv
from tests.util import assert_close, tail_plan, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("ranges", range(2, 17))
def test_every_number_of_ranges(ranges, d):
    import torch
    import paper_2511_12056_amd as pda
    from oracle import attention
    Sq, n_v = 201, 512 * ranges + 511
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n_cu >= 16:
        assert tail_plan(1, Sq, n_v, d, n_cu)["split"] == ranges
    qb, kb, vb = gen_qkv(500 + ranges, 1, 1, Sq, n_v, d, unit_rms=True)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    ro, rl = attention(qb, kb, vb, d ** -0.5)
    out = torch.full((1, 1, Sq, d), float("nan"), device="cuda")
    lse = torch.full((1, 1, Sq), float("nan"), device="cuda")
    pda.attn_fwd(q, k, v, out, lse, d ** -0.5)
    assert_close(out.cpu().numpy(), lse.cpu().numpy(), ro, rl, f"{ranges} ranges, d={d}")
    out16, lse16 = torch.full_like(out, float("nan"), dtype=torch.bfloat16), torch.full_like(lse, float("nan"))
    pda.attn_fwd_bf16out(q, k, v, out16, lse16, d ** -0.5)
    assert torch.equal(out16, out.to(torch.bfloat16)) and torch.equal(lse16, lse)
