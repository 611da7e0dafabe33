"""GPU parity of the region sums that carry the softmax normaliser along
(region_grad_sums) against the fp64 oracle with its own exact normalisers:
one item per workgroup, equal shares whose rows are merged from several
chunks, re-bases of the running maximum, sections of every kind, both head
dimensions, groups of 1 to 8."""
import math
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2507_21526_amd import binding as B
from paper_2507_21526_amd.inputs import draw_dout, draw_qkv
from tests.parity import log

pytestmark = pytest.mark.gpu

# |GPU - oracle| <= REL_ABS * (sum of |A_ij <dO_i, V_j>| over the section): as
# for the probe with a given LSE (fp32 products, 32 of them summed in fp32, then
# fp64), and the row sum's own relative error of about 1e-6.  The oracle takes
# its LSE in fp32, |LSE| < 64 here: up to 2^-19 = 2e-6 relative on its side.
REL_ABS = 5e-5


def _sums(q, k, v, dout, cu, tile, S, W, L, scale, plan=None):
    hq, hkv, d = q.shape[1], k.shape[1], q.shape[2]
    plan = plan or B.Plan("causal", cu, 0, 1, 0, tile, hq, d)
    nbytes = B.ta_region_grad_workspace_bytes(plan.info, hq, hkv)
    ws = torch.full((max(nbytes, 1),), 0xFF, dtype=torch.uint8, device=q.device)
    sums = torch.full((hq, 3), float("nan"), dtype=torch.float64, device=q.device)
    B.region_grad_sums(q, k, v, dout, plan.sched, plan.info, scale, S, W, L, sums,
                       ws if nbytes else None)
    torch.cuda.synchronize()
    return sums.cpu().numpy()


def _check(cu, hq, hkv, d, tile, S, W, L, seed, grow=0.0, few_pairs=False):
    log(f"case region sums cu={cu} hq={hq} hkv={hkv} d={d} T={tile} S={S} W={W} L={L}")
    q, k, v = draw_qkv(cu, hq, hkv, d, seed)
    if grow:  # keys that grow along the sequence: row maxima keep rising
        f = 1 + grow * torch.arange(cu[-1]).float()[:, None, None] / cu[-1]
        k = (k.float() * f).bfloat16()
    dout = draw_dout(cu, hq, d, seed + 1)
    scale = 1.0 / math.sqrt(d)
    _, lse64 = oracle.attn_full(q, k, v, cu, "causal", 0, 1, 0, scale)
    want, absw = oracle.region_grad(q, k, v, dout, lse64.astype(np.float32), cu, S, W, L, scale)
    got = _sums(*(t.cuda() for t in (q, k, v, dout)), cu, tile, S, W, L, scale)
    assert np.all(np.isfinite(got))
    err = np.abs(got - want)
    log(f"  worst |err| / sum|term| = {float((err / np.maximum(absw, 1e-300)).max()):.2e}")
    bound = REL_ABS * absw + 1e-12
    if few_pairs:
        # a section of one or two pairs does not average out the rounding of
        # <dO_i, V_j> itself: d products summed in fp32, off by at most
        # d u sum_c |dO_ic V_jc|, u = 2^-24
        va = v.float().abs().repeat_interleave(hq // hkv, 1)
        dots = sum((dout[i].float().abs() * va[j]).sum(-1)
                   for b in range(len(cu) - 1) for i in range(cu[b], cu[b + 1])
                   for j in range(cu[b], i + 1))
        bound = bound + d * 2.0 ** -24 * dots.double().numpy()[:, None]
    assert np.all(err <= bound)
    return got


CASES = [
    # cu, hq, hkv, d, tile, S, W, L, slots, growth of the keys
    ([0, 1], 1, 1, 128, 128, 0, 1, 0, None, 0),
    ([0, 700], 8, 2, 128, 128, 16, 100, 50, None, 0),
    ([0, 0, 333, 900, 901], 28, 4, 128, 64, 4, 40, 30, 3, 0),
    ([0, 513], 6, 2, 64, 128, 0, 1, 0, 16, 20.0),
    ([0, 300], 5, 1, 128, 64, 300, 10, 300, 512, 0),
    ([0, 777], 4, 4, 128, 128, 8, 200, 128, 1, 20.0),
    ([0, 640], 2, 2, 64, 64, 5, 0, 10, 7, 0),
    ([0, 1500, 1900], 16, 2, 128, 128, 8, 512, 128, None, 20.0),
]


@pytest.mark.parametrize("cu,hq,hkv,d,tile,S,W,L,slots,grow", CASES)
def test_region_sums_parity(cu, hq, hkv, d, tile, S, W, L, slots, grow):
    try:
        if slots:
            os.environ["TRIATTN_PROBE_SLOTS"] = str(slots)
        _check(cu, hq, hkv, d, tile, S, W, L, 3 * hq + d, grow)
    finally:
        os.environ.pop("TRIATTN_PROBE_SLOTS", None)


def test_region_sums_per_item_equal_shares():
    """128 packed sequences run one item per workgroup; equal shares of the
    same batch give the same sums but for the summation order (a step's
    products are taken against another reference, so fp32 rounding too)."""
    cu = [300 * i for i in range(129)]
    q, k, v = (t.cuda() for t in draw_qkv(cu, 8, 8, 64, 5))
    dout = draw_dout(cu, 8, 64, 6).cuda()
    plan = B.Plan("causal", cu, 0, 1, 0, 128, 8, 64)
    assert plan.info.max_item_tiles * 64 * 2 <= plan.info.kept_tiles_per_qhead
    one = _sums(q, k, v, dout, cu, 128, 8, 64, 32, 0.125, plan)
    again = _sums(q, k, v, dout, cu, 128, 8, 64, 32, 0.125, plan)
    assert np.array_equal(one, again)
    os.environ["TRIATTN_PROBE_SLOTS"] = "40"
    try:
        shares = _sums(q, k, v, dout, cu, 128, 8, 64, 32, 0.125, plan)
    finally:
        del os.environ["TRIATTN_PROBE_SLOTS"]
    assert np.allclose(one, shares, rtol=1e-4, atol=1e-3)


@pytest.mark.parametrize("hq,hkv,d,tile,S,W,L", [(32, 8, 128, 128, 8, 64, 32),
                                                 (28, 4, 64, 64, 0, 40, 10)])
def test_region_sums_per_item_parity(hq, hkv, d, tile, S, W, L):
    """Short packed sequences, enough for one item per workgroup (as a long
    sequence runs): the rows' normalisers are divided out in that workgroup."""
    cu = [0] + [int(x) for x in np.cumsum([260, 131, 64, 199] * 20)]
    plan = B.Plan("causal", cu, 0, 1, 0, tile, hq, d)
    # no row states: the workspace is one partial per (item, 32 rows, head, section)
    partials = plan.info.n_items * (tile // 32) * hq * 3 * 8
    assert B.ta_region_grad_workspace_bytes(plan.info, hq, hkv) < partials + 512
    _check(cu, hq, hkv, d, tile, S, W, L, 40 + hq, 20.0)


def test_region_sums_many_heads():
    """More heads than a second grid dimension may count."""
    _check([0, 3], 65544, 8193, 64, 128, 0, 1, 1, 3, few_pairs=True)


def test_region_sums_masked_infinity_and_bad_schedule():
    """A key no earlier row may see does not reach their sums, infinite or
    not; a device schedule that does not match gives NaN."""
    cu, hq, hkv, d = [0, 400], 4, 1, 128
    q, k, v = draw_qkv(cu, hq, hkv, d, 9)
    dout = draw_dout(cu, hq, d, 10)
    v2 = v.clone()
    v2[399] = math.inf
    args = [t.cuda() for t in (q, k, v, dout)]
    # only row 399 sees key 399, and it is the one Last row: the middle
    # section holds no infinity
    base = _sums(*args, cu, 128, 16, 64, 1, 0.1)
    got = _sums(args[0], args[1], v2.cuda(), args[3], cu, 128, 16, 64, 1, 0.1)
    assert np.all(np.isfinite(base)) and not np.isfinite(got[:, 0]).any()
    assert np.array_equal(got[:, 1], base[:, 1])
    plan = B.Plan("causal", cu, 0, 1, 0, 128, hq, d)
    good = plan.sched.clone()
    item = B.HDR_WORDS + B.ITEM_WORDS * (plan.info.n_items - 1)
    for word, value in ((0, int(good[0]) ^ 1), (item + 10, int(good[item + 10]) + 1),
                        (item + 5, 1 << 20), (item + 3, 1 << 20)):
        plan.sched.copy_(good)
        plan.sched[word] = value
        assert np.isnan(_sums(*args, cu, 128, 16, 64, 0, 0.1, plan)).any(), word
    plan.sched.copy_(good)
    with pytest.raises(B.TriAttnError):
        B.region_grad_sums(*args, plan.sched, plan.info, 0.1, 16, 64, 0,
                           torch.empty((hq, 3), dtype=torch.float64, device="cuda"), None)
