"""GPU tests of where an infinite value may reach.  A row that keeps the key
of an infinite V element gets that infinity.  Of the rows that do not, those
that share a group of R rows (R of 128, 64 and 32 the largest whose row blocks
of all heads fit eight waves) with a row that keeps a key of the same 64-key
step multiply a zero probability by it: they are not looked at here.  All
others stay bit for bit, whatever rows their workgroup serves."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2507_21526_amd import binding as B
from paper_2507_21526_amd.inputs import draw_dout, draw_qkv
from tests.parity import log, run_pass

pytestmark = pytest.mark.gpu

STEP = 64

CASES = [
    # kind, n, hq, hkv, d, S, W, L, T, keys of the infinite elements
    ("causal", 192, 1, 1, 128, 0, 1, 0, 128, (0, 150, 191)),     # three steps
    ("causal", 330, 5, 1, 128, 0, 1, 0, 128, (70, 200)),    # 7, 7 and 6 row blocks
    ("causal", 330, 6, 1, 128, 0, 1, 0, 128, (70, 200, 300)),    # 8 of each 24
    ("causal", 330, 8, 1, 128, 0, 1, 0, 128, (70, 200)),
    ("causal", 330, 3, 1, 128, 0, 1, 0, 64, (70, 200)),
    ("causal", 330, 1, 1, 64, 0, 1, 0, 128, (70, 100, 200)),     # 128 rows of a head
    ("causal", 330, 2, 1, 64, 0, 1, 0, 128, (70, 100, 200)),
    ("causal", 330, 7, 1, 64, 0, 1, 0, 128, (70, 200)),
    ("lists", 330, 5, 1, 128, 0, 1, 0, 128, (70, 200)),
    ("lists", 330, 7, 1, 64, 0, 1, 0, 128, (70, 200)),
    ("triangle", 700, 5, 1, 128, 0, 130, 0, 128, (60, 200, 430)),     # no sink: late first step
    ("triangle", 700, 6, 1, 128, 8, 200, 40, 128, (3, 130, 320, 690)),
    ("triangle", 700, 4, 1, 64, 8, 130, 40, 128, (3, 130, 320, 690)),
    ("triangle", 700, 2, 1, 64, 8, 100, 40, 128, (3, 130, 320, 690)),
    ("triangle", 700, 1, 1, 64, 70, 65, 0, 128, (3, 130, 320)),
    ("triangle", 700, 7, 1, 64, 4, 200, 64, 64, (3, 320, 650)),
    # launches of more than one round, whose workgroups straddle groups of rows
    ("causal", 1250, 40, 8, 128, 0, 1, 0, 128, (70, 1000)),
    ("causal", 1250, 48, 8, 128, 0, 1, 0, 128, (70, 1000)),
    ("lists", 1250, 40, 8, 128, 0, 1, 0, 128, (70, 1000)),
    ("triangle", 1250, 40, 8, 128, 0, 130, 0, 128, (60, 200, 830)),
    ("triangle", 1250, 48, 8, 128, 8, 200, 40, 128, (3, 830, 1240)),
    ("causal", 700, 56, 8, 64, 0, 1, 0, 128, (70, 430)),
    ("lists", 700, 56, 8, 64, 0, 1, 0, 128, (70, 430)),
    ("triangle", 3300, 24, 8, 64, 8, 130, 40, 128, (3, 1700, 3290)),
    ("triangle", 800, 40, 8, 64, 4, 200, 64, 64, (3, 320, 750)),
]


def _run(kind, q, k, v, S, W, L, T, dtype=torch.float32):
    n, hq, d = q.shape
    if kind != "lists":
        o, lse, _ = run_pass(kind, q, k, v, [0, n], S, W, L, T, out_dtype=dtype, poison=True)
        return o, lse
    # block-sparse lists that hold every k-tile of the causal mask
    ptr, idx = [0], []
    for t in range(-(-n // T)):
        idx += range(t + 1)
        ptr.append(len(idx))
    plan = B.Plan("blocksparse", [0, n], 0, 1, 0, T, hq, d, blocks=(ptr, idx))
    o = torch.full(q.shape, math.nan, device="cuda", dtype=dtype)
    lse = torch.full((hq, n), math.nan, device="cuda")
    plan.run(q, k, v, o, lse)
    return o, lse


def _row_groups(n, group, L, T):
    """Row ranges of R rows: of the q-tiles, then of the Last q-tiles."""
    R = next(r for r in (128, 64, 32) if r <= T and group * r // 32 <= 8)
    ends = [min(t + T, n - L) for t in range(0, n - L, T)]
    tiles = list(zip(range(0, n - L, T), ends))
    tiles += [(t, min(t + T, n)) for t in range(n - L, n, T)]
    return [(r, min(r + R, b)) for a, b in tiles for r in range(a, b, R)]


@pytest.mark.parametrize("kind,n,hq,hkv,d,S,W,L,T,keys", CASES)
def test_infinite_value_reaches_its_rows_only(kind, n, hq, hkv, d, S, W, L, T, keys):
    log(f"case infinite value {kind} n={n} hq={hq} hkv={hkv} d={d} S={S} W={W} L={L} T={T}")
    cu = [0, n]
    q, k, v = (t.cuda() for t in draw_qkv(cu, hq, hkv, d, seed=hq + d))
    base, base_lse = _run(kind, q, k, v, S, W, L, T)
    mask = "causal" if kind == "lists" else kind
    kept = np.asarray(oracle.mask_matrix(mask, n, S, W, L)).astype(bool)
    for key in keys:
        v2 = v.clone()
        v2[key] = math.inf
        for dtype in (torch.float32, torch.bfloat16):
            o, lse = _run(kind, q, k, v2, S, W, L, T, dtype)
            sees = torch.from_numpy(kept[:, key]).cuda()
            assert bool((o[sees] == math.inf).all()), (key, dtype)
            assert torch.equal(lse, base_lse), key
            s0 = key // STEP * STEP
            away = [(a, b) for a, b in _row_groups(n, hq // hkv, 0 if mask == "causal" else L, T)
                    if not kept[a:b, s0:s0 + STEP].any()]
            for a, b in away:
                assert torch.equal(o[a:b], base[a:b].to(dtype)), (key, dtype, a)


@pytest.mark.parametrize("hq,hkv,d,n,L,slots", [
    (4, 1, 128, 400, 0, None),   # equal shares, eight waves
    (4, 1, 128, 400, 50, None),
    (1, 1, 64, 400, 0, None),    # four waves
    (28, 4, 64, 390, 0, 1),      # one share, seven waves
])
def test_infinite_value_stays_in_its_section(hq, hkv, d, n, L, slots, monkeypatch):
    """Row pairs of a key in the last window are all of the streaming section,
    in steps that hold no other: the sums of the other sections stay bit for bit."""
    log(f"case infinite value region sums hq={hq} hkv={hkv} d={d} n={n} L={L}")
    if slots:
        monkeypatch.setenv("TRIATTN_PROBE_SLOTS", str(slots))
    cu, S, W = [0, n], 16, 100
    q, k, v = draw_qkv(cu, hq, hkv, d, 9)
    dout = draw_dout(cu, hq, d, 10)
    args = [t.cuda() for t in (q, k, v, dout)]
    _, base = B.region_grad(*args, cu, S, W, L)
    for key in (n - 1, n - 6):
        v2 = v.clone()
        v2[key, :, 0] = math.inf
        _, got = B.region_grad(args[0], args[1], v2.cuda(), args[3], cu, S, W, L)
        assert not np.isfinite(got[:, 0]).any(), key
        assert np.array_equal(got[:, 1:], base[:, 1:]), key
