"""Rounding error of launches of few query rows against 64 bits, beside that of the cut form of the same launch (variant 3)."""
import math

import pytest

from tests.test_gpu_rows_form import _n_cu, rows_form

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Sq,n_v,d", [(2, 1024, 1024, 64), (4, 1024, 4096, 64), (3, 1024, 6144, 64), (1, 2048, 2048, 128), (2, 2048, 3500, 128), (4, 1024, 5120, 128)])
def test_error_is_not_larger_than_that_of_the_cut_form(H, Sq, n_v, d):
    """What differs is how often a row's largest weight is the reference and so needs no rounding.  The mean over six draws of
    2 048 rows and more scatters by 0.1 %; a reference from 32 keys of a share of 16 tiles and more is 0.9 to 1.4 % off."""
    import torch
    import paper_2511_12056_amd as pda
    if _n_cu() == 256:
        assert rows_form(H, Sq, n_v, d, 256)
    gen = torch.Generator(device="cuda").manual_seed(n_v + d)
    sums = [0.0, 0.0]
    for _ in range(6):
        q, k, v = (torch.randn(1, H, s, d, generator=gen, device="cuda") for s in (Sq, n_v, n_v))
        q, k, v = ((t * t.square().mean(-1, keepdim=True).rsqrt()).to(torch.bfloat16) for t in (q, k, v))
        outs = []
        for variant in (0, 3):
            o, l = torch.empty(1, H, Sq, d, device="cuda"), torch.empty(1, H, Sq, device="cuda")
            pda.attn_fwd_variant(q, k, v, o, l, d ** -0.5, variant=variant)
            outs.append(o)
        diff, norm = [0.0, 0.0], 0.0
        for h in range(H):
            s = torch.mm(q[0, h].double() * d ** -0.5, k[0, h].double().t().contiguous())
            ref = torch.mm(torch.softmax(s, -1), v[0, h].double())
            norm += float(ref.square().sum())
            for i, o in enumerate(outs):
                diff[i] += float((o[0, h] - ref).square().sum())
        for i in range(2):
            sums[i] += math.sqrt(diff[i] / norm)
    assert sums[0] <= 1.004 * sums[1], sums
