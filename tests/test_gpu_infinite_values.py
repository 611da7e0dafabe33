"""GPU tests of where an infinite value may reach.  A row that keeps the key
of an infinite V element gets that infinity.  A 32-row block that visits none
of the key's 64-key step keeps its rows bit for bit, whatever other rows its
workgroup serves.  (Rows of a block that visits the step without keeping the
key multiply a zero probability by it: not looked at here.)"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2507_21526_amd.inputs import draw_qkv
from tests.parity import log, run_pass

pytestmark = pytest.mark.gpu

STEP, BLOCK = 64, 32

CASES = [
    # kind, n, hq, hkv, d, S, W, L, T, keys of the infinite elements
    ("causal", 192, 1, 1, 128, 0, 1, 0, 128, (0, 150, 191)),     # three steps
]


@pytest.mark.parametrize("kind,n,hq,hkv,d,S,W,L,T,keys", CASES)
def test_infinite_value_reaches_its_rows_only(kind, n, hq, hkv, d, S, W, L, T, keys):
    log(f"case infinite value {kind} n={n} hq={hq} hkv={hkv} d={d} S={S} W={W} L={L} T={T}")
    cu = [0, n]
    q, k, v = (t.cuda() for t in draw_qkv(cu, hq, hkv, d, seed=hq + d))
    base, base_lse, _ = run_pass(kind, q, k, v, cu, S, W, L, T)
    kept = np.asarray(oracle.mask_matrix(kind, n, S, W, L)).astype(bool)
    for key in keys:
        v2 = v.clone()
        v2[key] = math.inf
        for dtype in (torch.float32, torch.bfloat16):
            o, lse, _ = run_pass(kind, q, k, v2, cu, S, W, L, T, out_dtype=dtype, poison=True)
            sees = torch.from_numpy(kept[:, key]).cuda()
            assert bool((o[sees] == math.inf).all()), (key, dtype)
            assert torch.equal(lse, base_lse), key
            s0 = key // STEP * STEP
            away = [b for b in range(0, n, BLOCK) if not kept[b:b + BLOCK, s0:s0 + STEP].any()]
            for b in away:
                assert torch.equal(o[b:b + BLOCK], base[b:b + BLOCK].to(dtype)), (key, dtype, b)
