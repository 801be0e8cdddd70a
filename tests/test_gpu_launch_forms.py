"""The forms an attention launch takes, by the number of its work items: workgroups of four or of eight
wavefronts, each with one item (`direct`) or several one after the other (`chained`), whole tiles and
tiles cut into key ranges, fp32 and bf16 results, scores with a scale and as exponents of 2, items that
need the running-max sweep between items that do not.

Launches of many heads repeat a few generated ones; a repeated head must give the bits of that head
launched with few others (rows of tiles that both launches sweep in one pass), and those are compared
with the fp64 oracle.  Each case says which form it reaches on 256 compute units."""
import math

import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits, gen_qkv
from tests.util import REL_L2, LSE_REL, assert_close, cut_row_mask, tail_plan, to_dev_bf16, wavefronts

pytestmark = pytest.mark.gpu


def _n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _form(H, Sq, n_v, d):
    """(wavefronts per workgroup, items in a chain?, number of cut tiles) on this device."""
    n_cu = _n_cu()
    nw = wavefronts(H, Sq, n_v, d, n_cu)
    plan = tail_plan(H, Sq, n_v, d, n_cu)
    items = plan["n_tiles"] + plan["n_cut"] * (plan["split"] - 1)
    return nw, items > n_cu, plan["n_cut"]           # one workgroup per item and CU, or two of half an item


def _expect(form, H, Sq, n_v, d):
    if _n_cu() == 256:
        assert _form(H, Sq, n_v, d) == form, (_form(H, Sq, n_v, d), form)


def _launch(entry, q, k, v, scale):
    """entry: "fp32", "bf16", "base2" or "redo" (fp32, every row swept a second time)."""
    import torch
    import paper_2511_12056_amd as pda
    B, H, Sq, d = q.shape
    out = torch.full((B, H, Sq, d), float("nan"), device="cuda", dtype=torch.bfloat16 if entry == "bf16" else torch.float32)
    lse = torch.full((B, H, Sq), float("nan"), device="cuda")
    if entry == "fp32":
        pda.attn_fwd(q, k, v, out, lse, scale)
    elif entry == "bf16":
        pda.attn_fwd_bf16out(q, k, v, out, lse, scale)
    elif entry == "base2":
        pda.attn_fwd_base2(q, k, v, out, lse)
    else:
        pda.attn_fwd_variant(q, k, v, out, lse, scale, variant=3)
    torch.cuda.synchronize()
    return out, lse


def _scaled(qb, entry, d):
    """Q bits and the scale of the call and of the oracle: for base 2 the scale is folded into Q."""
    if entry != "base2":
        return qb, d ** -0.5
    return f32_to_bf16_bits(bf16_bits_to_f32(qb) * np.float32(d ** -0.5 * math.log2(math.e))), math.log(2.0)


def _repeat(t, H):
    import torch
    return t[:, torch.arange(H, device="cuda") % t.shape[1]].contiguous()


def _check(o, l, ro, rl, entry, what):
    """fp32 gates; a bf16 result adds its own rounding (half a step, 2^-9 relative, per element)."""
    o = o.float().cpu().numpy()
    if entry == "bf16":
        assert np.isfinite(o).all()
        assert np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= REL_L2 + 2.0 ** -9 / np.sqrt(3.0), what
        assert (np.abs(l.cpu().numpy() - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL, what
    else:
        assert_close(o, l.cpu().numpy(), ro, rl, what)


@pytest.mark.parametrize("d,n_v", [(128, n) for n in (1, 63, 64, 65, 128, 191, 256, 300, 321, 449)] +
                                  [(64, n) for n in (449, 511, 512, 513, 577, 640, 705)])
def test_chain_of_four_wavefront_items(d, n_v):
    """193 heads x 1 900 rows = six rounds and 8 tiles: workgroups of four wavefronts take several half
    tiles each (the last half of a head holds no row); every exit of the unrolled key loop."""
    import torch
    from oracle import attention
    base, H, Sq = 5, 193, 1900
    _expect((4, True, 0), H, Sq, n_v, d)
    qb, kb, vb = gen_qkv(51 + n_v, 1, base, Sq, n_v, d, unit_rms=True)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    ro, rl = attention(qb, kb, vb, d ** -0.5)
    for entry in ("fp32", "redo"):
        out, lse = _launch(entry, _repeat(q, H), _repeat(k, H), _repeat(v, H), d ** -0.5)
        o, l = _launch(entry, q, k, v, d ** -0.5)           # 40 tiles, none cut: one item per workgroup
        assert torch.equal(out, _repeat(o, H)) and torch.equal(lse, _repeat(l, H)), entry
        assert_close(o.cpu().numpy(), l.cpu().numpy(), ro, rl, f"{entry} d={d} n_v={n_v}")


@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2", "redo"])
@pytest.mark.parametrize("H,Sq,n_v,d,form", [
    (130, 2000, 1100, 128, (4, True, 16)),       # four rounds and 16 tiles, those cut in two
    (130, 2000, 1536, 128, (4, True, 16)),       # ... in three
    (130, 2000, 1100, 64, (4, True, 16)),
    (130, 2000, 1500, 64, (4, True, 16)),
    (24, 3000, 1800, 128, (8, True, 32)),        # one round and 32 tiles, those cut in three
    (24, 3000, 1800, 64, (8, True, 32)),
    (24, 700, 12850, 128, (8, False, 72)),       # 72 tiles, every one cut in three: 216 items
    (24, 700, 12850, 64, (8, False, 72)),
    (400, 300, 500, 128, (8, True, 0)),          # three rounds and 32 tiles, none cut
    (400, 300, 500, 64, (8, True, 0)),
])
def test_forms_against_the_oracle(H, Sq, n_v, d, form, entry):
    import torch
    from oracle import attention_head
    base = 6
    _expect(form, H, Sq, n_v, d)
    qb, kb, vb = gen_qkv(1300 + n_v, 1, base, Sq, n_v, d, unit_rms=True)
    qb, scale = _scaled(qb, entry, d)
    q, k, v = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    out, lse = _launch(entry, _repeat(q, H), _repeat(k, H), _repeat(v, H), scale)
    cut = cut_row_mask(1, H, Sq, n_v, d, _n_cu())[0]
    rng = np.random.default_rng(n_v)
    rows = np.unique(np.concatenate([[0, 127, 128, 255, 256, Sq - 1], rng.choice(Sq, size=40, replace=False)]))
    dr = torch.from_numpy(rows).cuda()
    want = [attention_head(qb[0, i], kb[0, i], vb[0, i], scale, n_v, rows=rows) for i in range(base)]
    first = {}
    for h in range(H):
        # every head against the oracle on sampled rows (tile edges among them), and against the first head
        # of the same content, bit for bit, on the rows that lie in whole tiles of both
        _check(out[0, h][dr], lse[0, h][dr], *want[h % base], entry, f"{(H, Sq, n_v, d)} {entry} head {h}")
        whole = torch.from_numpy(~cut[h]).cuda()
        o, l, w = first.setdefault(h % base, (out[0, h], lse[0, h], whole))
        both = whole & w
        assert torch.equal(out[0, h][both], o[both]) and torch.equal(lse[0, h][both], l[both]), h


@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2"])
@pytest.mark.parametrize("H,Sq,d,form", [(300, 300, 128, (8, True, 0)), (300, 300, 64, (8, True, 0)),
                                         (193, 1900, 128, (4, True, 0)), (193, 1900, 64, (4, True, 0))])
def test_second_sweep_inside_a_chain(H, Sq, d, form, entry):
    """Items that sweep a second time, for one row of the last wavefront or for all rows, between items
    that do not: the item after such a one, and the rows beside such a row, are what they are alone."""
    import torch
    from oracle import attention
    base, n_v = 5, 700
    _expect(form, H, Sq, n_v, d)
    rng = np.random.default_rng(4096 + d)
    q = rng.standard_normal((1, base, Sq, d)).astype(np.float32)
    k = (rng.standard_normal((1, base, n_v, d)) * 0.05).astype(np.float32)
    v = rng.standard_normal((1, base, n_v, d)).astype(np.float32)
    k[0, 1, 400] = q[0, 1, 250] * np.float32(1.5 * 128 / d)       # > 64 log2 units above the first tile, row 250
    k[0, 1, 500] = q[0, 1, 290] * np.float32(1.5 * 128 / d)       # and row 290, in the second tile
    k[0, 2, 600] = q[0, 2, 100] * np.float32(0.45 * 128 / d)      # ~50 log2 units, times values of 2^90
    v[0, 2] *= np.float32(2.0 ** 90)
    k[0, 4, 300:] *= np.float32(600.0)                            # every row, every tile
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    scale, oracle_scale = 1.0, 1.0
    if entry == "base2":
        qb = f32_to_bf16_bits(q * np.float32(math.log2(math.e)))
        oracle_scale = math.log(2.0)
    dq, dk, dv = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    out, lse = _launch(entry, _repeat(dq, H), _repeat(dk, H), _repeat(dv, H), scale)
    o, l = _launch(entry, dq, dk, dv, scale)
    assert torch.equal(out, _repeat(o, H)) and torch.equal(lse, _repeat(l, H))
    s = bf16_bits_to_f32(kb[0, 1]).astype(np.float64) @ bf16_bits_to_f32(qb[0, 1, 250]).astype(np.float64) * oracle_scale
    assert s[64:].max() - s[:64].max() > 64 * math.log(2.0)       # the inputs do what they are meant to
    ro, rl = attention(qb, kb, vb, oracle_scale)
    o, l = o.float().cpu().numpy().astype(np.float64), l.cpu().numpy()
    assert np.isfinite(o).all() and np.isfinite(l).all()
    for h in range(base):                                         # relative gates: head 2 spans 2^90
        tol = REL_L2 + (2.0 ** -9 / np.sqrt(3.0) if entry == "bf16" else 0.0)
        assert np.sqrt(((o[0, h] - ro[0, h]) ** 2).sum() / (ro[0, h] ** 2).sum()) <= tol, h
    assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL
