"""Scores and values at the ends of their range in launches of few query rows: what one workgroup's wavefronts get of a
row's keys must not change what becomes of it."""
import numpy as np
import pytest

from synth import bf16_bits_to_f32, f32_to_bf16_bits
from tests.test_gpu_rows_form import _launch, _n_cu, rows_form
from tests.util import LSE_REL, REL_L2, to_dev_bf16

pytestmark = pytest.mark.gpu


def _reference(qb, kb, vb, scale):
    """fp64 softmax attention in which a score of -inf weighs 0, values scaled to one (they may lie near the largest float)."""
    q, k, v = (bf16_bits_to_f32(x).astype(np.float64) for x in (qb, kb, vb))
    with np.errstate(invalid="ignore"):
        s = np.einsum("bhqd,bhkd->bhqk", q, k) * scale
    m = s.max(-1, keepdims=True)
    w = np.exp(s - m)
    return np.matmul(w / w.sum(-1, keepdims=True), v), m[..., 0] + np.log(w.sum(-1))


def _check(o, l, ro, rl):
    o, l = o.double().cpu().numpy(), l.double().cpu().numpy()
    assert np.isfinite(o).all() and np.isfinite(l).all()
    assert np.sqrt(((o - ro) ** 2).sum() / (ro ** 2).sum()) <= REL_L2
    assert (np.abs(l - rl) / np.maximum(np.abs(rl), 1.0)).max() <= LSE_REL


@pytest.mark.parametrize("low", [-np.inf, -3.0e38])
@pytest.mark.parametrize("entry", ["fp32", "base2"])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("H,Sq,n_v,hidden", [(1, 70, 1024, (128, 160)),      # the first tile of a wavefront's share
                                             (1, 70, 1024, (128, 256)),      # a whole share
                                             (1, 33, 1500, (160, 1100)),     # several, and parts of two
                                             (2, 1024, 3072, (384, 420)),    # a long share, whose reference follows the max at first
                                             (13, 1000, 1100, (256, 300))])  # two row blocks a workgroup
def test_keys_that_score_minus_infinity(H, Sq, n_v, hidden, d, entry, low):
    """K entries of -inf, or products beyond fp32, in keys that are the first of a wavefront's share."""
    if _n_cu() == 256:
        assert rows_form(H, Sq, n_v, d, 256)
    rng = np.random.default_rng(n_v + d)
    q, k, v = (rng.standard_normal((1, H, s, d)).astype(np.float32) for s in (Sq, n_v, n_v))
    q[..., 0] = np.abs(q[..., 0]) + 2.0
    k[:, :, hidden[0]:hidden[1], 0] = low
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    scale = d ** -0.5 if entry == "fp32" else np.log(2.0)
    kb64 = bf16_bits_to_f32(kb).copy()
    kb64[:, :, hidden[0]:hidden[1], 0] = -np.inf                    # what the scores come to in fp32
    ro, rl = _reference(qb, f32_to_bf16_bits(kb64), vb, scale)
    o, l = _launch(entry, to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), scale, n_v)
    _check(o, l, ro, rl)


@pytest.mark.parametrize("entry", ["fp32", "bf16", "base2"])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("H,Sq,n_v", [(1, 70, 1024), (13, 1000, 1100)])
def test_values_near_the_largest_float(H, Sq, n_v, d, entry):
    """Values of 5e35: 512 of them, the keys of a range of the cut form, add up inside fp32, 1 024 of them do not."""
    if _n_cu() == 256:
        assert rows_form(H, Sq, n_v, d, 256)
    rng = np.random.default_rng(n_v - d)
    q, k, v = (rng.standard_normal((1, H, s, d)).astype(np.float32) for s in (Sq, n_v, n_v))
    q *= np.float32(2.0 ** -6)                                      # nearly equal weights
    v = np.float32(5e35) * (1 + v * np.float32(0.01))
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    scale = np.log(2.0) if entry == "base2" else 1.0
    ro, rl = _reference(qb, kb, vb, scale)
    o, l = _launch(entry, to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), scale, n_v)
    _check(o, l, ro, rl)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("H,Sq,n_v", [(1, 70, 1024), (2, 1024, 3072), (13, 1000, 1100)])
def test_scale_zero(H, Sq, n_v, d):
    """All weights are equal: the mean of V, whatever the scores, and ln n_v."""
    if _n_cu() == 256:
        assert rows_form(H, Sq, n_v, d, 256)
    rng = np.random.default_rng(n_v + 2 * d)
    qb, kb, vb = (f32_to_bf16_bits(rng.standard_normal((1, H, s, d)).astype(np.float32)) for s in (Sq, n_v, n_v))
    o, l = _launch("fp32", to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), 0.0, n_v)
    mean = bf16_bits_to_f32(vb).astype(np.float64).mean(2, keepdims=True)
    _check(o, l, np.broadcast_to(mean, (1, H, Sq, d)), np.full((1, H, Sq), np.log(n_v)))
