"""Pairs of tiles in which a few wavefronts' rows need the second sweep: the others only fetch their share of the tiles for it."""
import math

import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits
from tests.test_gpu_launch_forms import _launch, _repeat
from tests.test_gpu_wide_items import _n_cu, wide_plan
from tests.util import LSE_REL, REL_L2, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2"])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n_v", [224, 256, 257, 320, 321, 449, 512, 577, 640])
def test_few_rows_of_a_tile(n_v, d, entry):
    """Four key tiles and more, whole and ragged, every length of the loop's end; one row, one in either tile, one in each half of a
    tile, and every second wavefront.  Bits of a launch of few heads, which has no pairs, and the oracle's values."""
    import torch
    from oracle import attention
    base, H, Sq = 5, 140, 1000
    if _n_cu() == 256:
        assert wide_plan(H, Sq, n_v, 256)[0] > 0 and wide_plan(base, Sq, n_v, 256)[0] == 0
    rows = {0: [7], 1: [200, 300], 2: [3, 255], 3: list(range(40, 1000, 64)), 4: []}
    rng = np.random.default_rng(n_v + d)
    q = rng.standard_normal((1, base, Sq, d)).astype(np.float32)
    k = (rng.standard_normal((1, base, n_v, d)) * 0.02).astype(np.float32)
    v = rng.standard_normal((1, base, n_v, d)).astype(np.float32)
    for h, which in rows.items():
        for i, row in enumerate(which):
            k[0, h, 70 + 5 * i] = q[0, h, row] * np.float32(70.0 / np.square(q[0, h, row]).sum())      # beyond the 64 keys of the reference
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    oracle_scale = 1.0
    if entry == "base2":
        qb, oracle_scale = f32_to_bf16_bits(q * np.float32(math.log2(math.e))), math.log(2.0)
    for h, which in rows.items():                                  # those rows, and hardly any other, leave the safe range
        s = bf16_bits_to_f32(qb[0, h]).astype(np.float64) @ bf16_bits_to_f32(kb[0, h]).astype(np.float64).T * oracle_scale
        far = set(np.nonzero(s[:, 64:].max(1) - s[:, :64].max(1) > 64 * math.log(2.0))[0])
        assert far >= set(which) and len(far) <= len(which) + 2
    dq, dk, dv = to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb)
    o, l = _launch(entry, dq, dk, dv, 1.0)
    out, lse = _launch(entry, _repeat(dq, H), _repeat(dk, H), _repeat(dv, H), 1.0)
    assert torch.equal(out, _repeat(o, H)) and torch.equal(lse, _repeat(l, H))
    ro, rl = attention(qb, kb, vb, oracle_scale)
    o, l = o.double().cpu().numpy(), l.double().cpu().numpy()
    tol = REL_L2 + (2.0 ** -9 / np.sqrt(3.0) if entry == "bf16" else 0.0)
    assert np.isfinite(o).all() and np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= tol
    assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL
