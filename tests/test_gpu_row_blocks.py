"""GPU tests of the tile kernel's workgroups at the sizes where they can go
wrong: one step, an odd number of steps, row blocks of several heads with a
remainder in the last workgroup, tiles of 64 rows whose workgroups are not
full, ragged last tiles, tiles past the end of the sequence, list items, split
items, both head dimensions and both output types; and of the passes whose
Last q-tiles have one split each, which run without a merge."""
import math
import os

import numpy as np
import pytest
import torch

from paper_2507_21526_amd import binding
from paper_2507_21526_amd.inputs import draw_qkv
from tests.parity import compare, kernels_of, log, run_pass

pytestmark = pytest.mark.gpu

ENV = "TRIATTN_UNITS_PER_WG"

CASES = [
    # kind, cu, hq, hkv, d, S, W, L, T, splits
    ("causal", [0, 33], 1, 1, 128, 0, 1, 0, 128, 0),              # one step, one row block
    ("causal", [0, 65], 4, 1, 64, 0, 1, 0, 64, 0),                # second step of one key
    ("causal", [0, 191, 192, 449], 5, 1, 128, 0, 1, 0, 128, 0),   # G 5: 20 row blocks
    ("causal", [0, 700], 6, 2, 64, 0, 1, 0, 64, 0),               # G 3, T 64: six blocks
    ("causal", [0, 1000], 7, 1, 128, 0, 1, 0, 64, 0),             # G 7, T 64: 14 blocks
    ("triangle", [0, 1537], 8, 8, 128, 8, 130, 40, 128, 0),       # G 1: 128 rows of a head
    ("triangle", [0, 64, 900], 4, 2, 64, 130, 65, 129, 128, 3),   # sink not aligned, splits
    ("triangle", [0, 1000], 8, 1, 128, 16, 1, 200, 128, 8),       # splits without steps
    ("triangle", [0, 2000], 6, 1, 128, 0, 320, 0, 128, 0),        # no Last rows, no sink
    ("triangle", [0, 930], 12, 2, 64, 8, 300, 70, 128, 0),        # G 6: 24 row blocks
    ("causal", [0, 300, 397], 10, 2, 128, 0, 1, 0, 64, 0),        # G 5, T 64: 10 blocks
    # d 64: four-wave workgroups of dealt row blocks
    ("causal", [0, 300, 397], 10, 2, 64, 0, 1, 0, 64, 0),         # 4, 4 and 2 blocks
    ("triangle", [0, 933], 7, 1, 64, 8, 130, 70, 64, 0),          # G 7: 4, 4, 4 and 2 blocks
    ("triangle", [0, 33, 1201], 7, 1, 64, 8, 130, 150, 128, 3),   # G 7, T 128: 28 blocks
    ("triangle", [0, 700], 3, 3, 64, 0, 65, 40, 128, 0),          # G 1: 128 rows of a head
]

# launches of more than one round, whose workgroups' blocks straddle groups of
# rows
STRADDLE_CASES = [
    ("causal", [0, 300, 1200], 40, 8, 128, 0, 1, 0, 128, 0),       # G 5: 7, 7 and 6 blocks
    ("triangle", [0, 1250], 48, 8, 128, 8, 130, 40, 128, 0),       # G 6: 8, 8 and 8
    ("triangle", [0, 33, 750], 56, 8, 64, 8, 130, 70, 128, 2),     # G 7
    ("causal", [0, 333, 850], 40, 8, 64, 0, 1, 0, 128, 0),         # G 5, d 64
    ("triangle", [0, 3333], 24, 8, 64, 0, 130, 70, 128, 0),        # G 3, no sink
]


def _run(*args, **kw):
    o, lse, _ = run_pass(*args, poison=True, **kw)
    torch.cuda.synchronize()
    return o, lse


@pytest.mark.parametrize("kind,cu,hq,hkv,d,S,W,L,T,splits", CASES)
def test_row_blocks(kind, cu, hq, hkv, d, S, W, L, T, splits):
    log(f"case row blocks {kind} cu={cu} hq={hq} hkv={hkv} d={d} S={S} W={W} L={L} T={T}")
    _check_rows(kind, cu, hq, hkv, d, S, W, L, T, splits, range(hq))


# launches at d 64 that run eight-wave workgroups: dense causal ones of 769 to
# 1024 four-wave workgroups, Triangle ones without Last rows of 257 to 448
EIGHT_CASES = [
    ("causal", [0, 1201, 1700], 64, 8, 64, 0, 1, 0, 128, 0),   # G 8: 14 items of 32 blocks
    ("causal", [0, 1999], 56, 8, 64, 0, 1, 0, 128, 0),         # G 7: 16 items, 7 blocks each
    ("causal", [0, 3201], 32, 8, 64, 0, 1, 0, 64, 0),          # G 4, T 64: 51 items
    ("triangle", [0, 1150], 32, 4, 64, 0, 128, 0, 128, 0),     # G 8: 9 items
    ("triangle", [0, 2500], 15, 3, 64, 8, 128, 0, 128, 0),     # G 5: 20 items, 5 blocks each
]


@pytest.mark.parametrize("form,kind,cu,hq,hkv,d,S,W,L,T,splits", [
    *(("false, false, true>", *c) for c in STRADDLE_CASES),
    *(("<64, 8, false, false, false>", *c) for c in EIGHT_CASES)])
def test_forms_of_larger_launches(form, kind, cu, hq, hkv, d, S, W, L, T, splits):
    log(f"case larger launch {kind} cu={cu} hq={hq} hkv={hkv} d={d} S={S} W={W} L={L} T={T}")
    g = hq // hkv
    args = _check_rows(kind, cu, hq, hkv, d, S, W, L, T, splits,
                       [*range(g), *range(hq - g, hq)])
    names = [n for n in kernels_of(lambda: _run(*args)) if "attn_tile_kernel" in n]
    assert len(names) == 1 and form in names[0], names
    # the first kv head alone: a launch of one round, in another form
    o, lse = _run(*args)
    one = [args[0], args[1][:, :g].contiguous()] + [t[:, :1].contiguous() for t in args[2:4]]
    names = [n for n in kernels_of(lambda: _run(*one, *args[4:])) if "attn_tile_kernel" in n]
    assert len(names) == 1 and form not in names[0], names
    o1, lse1 = _run(*one, *args[4:])
    assert torch.equal(o[:, :g], o1) and torch.equal(lse[:g], lse1)


def _check_rows(kind, cu, hq, hkv, d, S, W, L, T, splits, heads):
    q, k, v = draw_qkv(cu, hq, hkv, d, seed=31 + hq + S)
    args = [kind] + [t.cuda() for t in (q, k, v)] + [cu, S, W, L, T, splits]
    o, lse = _run(*args)
    assert not torch.isnan(o).any() and not torch.isnan(lse).any()
    compare(kind, q, k, v, cu, S, W, L, 1 / math.sqrt(d), o, lse, np.arange(cu[-1]),
            heads, label=f"{kind} cu={cu}", p_bound=True)
    o16, _ = _run(*args, out_dtype=torch.bfloat16)
    assert torch.equal(o16, o.bfloat16())
    return args


@pytest.mark.parametrize("hq,d,T,bound", [(5, 128, 128, 0), (3, 64, 64, 3)])
def test_lists_equal_causal(hq, d, T, bound):
    """Full lists, an odd number of tiles among them: uncut they give the
    causal pass's rows bit for bit; cut into items of three tiles they meet the
    parity bar."""
    cu = [0, 450, 1100]
    q, k, v = draw_qkv(cu, hq, 1, d, seed=77)
    qg, kg, vg = (t.cuda() for t in (q, k, v))
    ptr, idx = [0], []
    for n in np.diff(cu):
        for t in range(-(-int(n) // T)):
            idx += range(t + 1)
            ptr.append(len(idx))
    plan = binding.Plan("blocksparse", cu, 0, 1, 0, T, hq, d, splits=bound, blocks=(ptr, idx))
    o = torch.full((cu[-1], hq, d), math.nan, device="cuda")
    lse = torch.full((hq, cu[-1]), math.nan, device="cuda")
    plan.run(qg, kg, vg, o, lse)
    ref, ref_lse = _run("causal", qg, kg, vg, cu, 0, 1, 0, T, 0)
    if bound == 0:
        assert torch.equal(o, ref) and torch.equal(lse, ref_lse)
    compare("causal", q, k, v, cu, 0, 1, 0, 1 / math.sqrt(d), o, lse, np.arange(cu[-1]),
            range(hq), label=f"lists hq={hq} d={d} T={T}", p_bound=True)


@pytest.mark.parametrize("upw", [None, 1, 3])
@pytest.mark.parametrize("cu,hq,d,T,splits", [
    ([0, 513], 4, 128, 128, 0),            # the second Last q-tile has one row
    ([0, 0, 40, 900, 901], 8, 64, 64, 0),  # sequences shorter than L
    ([0, 5000], 2, 128, 128, 1),           # one split by request
])
def test_one_split_needs_no_merge(cu, hq, d, T, splits, upw):
    """Where every Last q-tile has one split the fused call writes its rows
    in the tile pass: bit for bit what tiles and merge give, in every form of
    the kernel, and a split that does not cover its rows is rejected."""
    S, W, L = 5, 200, 129
    q, k, v = (t.cuda() for t in draw_qkv(cu, hq, 1, d, seed=5))
    if upw is not None:
        os.environ[ENV] = str(upw)
    try:
        plan = binding.Plan("triangle", cu, S, W, L, T, hq, d, splits)
        assert plan.info.max_splits == 1
        for dtype in (torch.float32, torch.bfloat16):
            o = torch.full((cu[-1], hq, d), math.nan, device="cuda", dtype=dtype)
            lse = torch.full((hq, cu[-1]), math.nan, device="cuda")
            o2, lse2 = o.clone(), lse.clone()
            plan.run(q, k, v, o, lse)
            args = (plan.sched, plan.info)
            binding.triangle_attn_tiles(q, k, v, o2, lse2, *args, d ** -0.5, plan.workspace)
            binding.triangle_attn_merge(o2, lse2, *args, plan.workspace)
            torch.cuda.synchronize()
            assert not torch.isnan(o).any() and not torch.isnan(lse).any()
            assert torch.equal(o, o2) and torch.equal(lse, lse2)
        plan.sched[binding.HDR_WORDS + 4] = 1  # the first split misses k-tile 0
        plan.run(q, k, v, o, lse)
        torch.cuda.synchronize()
        assert torch.isnan(o).any()
    finally:
        os.environ.pop(ENV, None)


@pytest.mark.parametrize("upw", [None, 3])
def test_one_split_checks_the_whole_schedule(upw, monkeypatch):
    """The fused call over one split per Last q-tile launches no merge, but
    rejects what the merge would: another tile in the header (every row NaN)
    and a malformed merge item."""
    cu, hq, d, T = [0, 700, 901], 4, 128, 128
    q, k, v = (t.cuda() for t in draw_qkv(cu, hq, 1, d, seed=6))
    if upw is not None:
        monkeypatch.setenv(ENV, str(upw))
    plan = binding.Plan("triangle", cu, 5, 64, 129, T, hq, d)
    info = plan.info
    assert info.max_splits == 1 and info.n_merge_items >= 3
    good = plan.sched.clone()
    merge = binding.HDR_WORDS + binding.ITEM_WORDS * info.n_items
    last = merge + 8 * (info.n_merge_items - 1)
    for word, value, every in ((3, 64, True), (merge, -1, False), (last, cu[-1], False),
                               (last + 1, -1, False), (last + 2, 1 << 20, False),
                               (last + 3, 0, False), (last + 3, 1 << 20, False),
                               (last + 4, -1, False), (last + 4, 1 << 20, False)):
        o = torch.zeros(q.shape, device="cuda")
        lse = torch.zeros((hq, cu[-1]), device="cuda")
        plan.sched.copy_(good)
        plan.run(q, k, v, o, lse)
        assert not torch.isnan(o).any() and not torch.isnan(lse).any()
        plan.sched[word] = value
        plan.run(q, k, v, o, lse)
        torch.cuda.synchronize()
        bad = torch.isnan(o)
        assert bool(bad.all() if every else bad.any()), word
        assert bool(torch.isnan(lse).all() if every else torch.isnan(lse).any()), word
