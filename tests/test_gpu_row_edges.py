"""Query counts around the pieces in which the attention kernel loads Q and stores its results (16 and 32
rows of a wavefront, 128 and 256 of a workgroup): every row is right and nothing beyond it is written."""
import numpy as np
import pytest

from synth import gen_qkv
from tests.util import LSE_REL, REL_L2, assert_close, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("Sq", [1, 15, 16, 17, 31, 32, 33, 48, 127, 129, 255, 257])
def test_rows_at_the_edges(Sq, d, bf16):
    import torch
    import paper_2511_12056_amd as pda
    from oracle import attention
    H, n_v, pad = 2, 600, 40
    qb, kb, vb = gen_qkv(900 + Sq, 1, H, Sq, n_v, d, unit_rms=True)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    ro, rl = attention(qb, kb, vb, d ** -0.5)
    # results inside larger buffers: what lies behind the last row stays as it is
    if bf16:
        big = torch.full((H * Sq * d + pad * d,), 7.0, device="cuda", dtype=torch.bfloat16)
        big_l = torch.full((H * Sq + pad,), 7.0, device="cuda")
        out, lse = big[:H * Sq * d].view(1, H, Sq, d), big_l[:H * Sq].view(1, H, Sq)
        pda.attn_fwd_bf16out(q, k, v, out, lse, d ** -0.5)
        assert (big[H * Sq * d:] == 7.0).all() and (big_l[H * Sq:] == 7.0).all()
        o = out.float().cpu().numpy()
        assert np.isfinite(o).all()
        assert np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= REL_L2 + 2.0 ** -9 / np.sqrt(3.0)
        assert (np.abs(lse.cpu().numpy() - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL
    else:
        big = torch.full((1, H, Sq + pad, d), 7.0, device="cuda")
        big_l = torch.full((1, H, Sq + pad), 7.0, device="cuda")
        out, lse = big[:, :, :Sq], big_l[:, :, :Sq]
        pda.attn_fwd_strided(q, k, v, out, lse, d ** -0.5)
        assert (big[:, :, Sq:] == 7.0).all() and (big_l[:, :, Sq:] == 7.0).all()
        assert_close(out.cpu().numpy(), lse.cpu().numpy(), ro, rl, f"Sq={Sq} d={d}")
