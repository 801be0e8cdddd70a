"""Every way a sweep over the keys is put together from its first, main, tail and last iterations: 1 to 15
key tiles with a full or ragged last one, workgroups of eight and of four wavefronts, both sweeps."""
import pytest

from synth import gen_qkv
from tests.util import assert_close, to_dev_bf16, wavefronts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("tiles", range(1, 16))
def test_sweeps_of_few_tiles(tiles, d):
    import torch
    import paper_2511_12056_amd as pda
    from oracle import attention
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    base, Sq, scale = 3, 200, d ** -0.5
    for n_v in (64 * tiles, 64 * tiles - 63, 64 * tiles - 17):
        qb, kb, vb = gen_qkv(70 + n_v, 1, base, Sq, n_v, d, unit_rms=True)
        q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
        ro, rl = attention(qb, kb, vb, scale)
        got = []
        for H in (n_cu // 2 + 2, base):                  # eight wavefronts, four wavefronts; no tile is cut
            assert wavefronts(H, Sq, n_v, d, n_cu) == (8 if H > base else 4)
            idx = torch.arange(H, device="cuda") % base
            for variant in (0, 3):                       # 3: every row is swept a second time
                out = torch.full((1, H, Sq, d), float("nan"), device="cuda")
                lse = torch.full((1, H, Sq), float("nan"), device="cuda")
                pda.attn_fwd_variant(q[:, idx].contiguous(), k[:, idx].contiguous(), v[:, idx].contiguous(), out, lse, scale, variant=variant)
                torch.cuda.synchronize()
                assert torch.equal(out, out[:, idx]) and torch.equal(lse, lse[:, idx])
                assert_close(out[:, :base].cpu().numpy(), lse[:, :base].cpu().numpy(), ro, rl, f"{n_v} {d} {H} {variant}")
                got.append((out[:, :base], lse[:, :base]))
        for a, b in ((0, 2), (1, 3)):
            assert torch.equal(got[a][0], got[b][0]) and torch.equal(got[a][1], got[b][1])
