"""GPU parity of the HIP passes against the fp64 oracle on small and edge-case
shapes (full outputs), plus the structural properties of the split pass:
split invariance, packing invariance, determinism, every row written, and no
leak through the mask."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2507_21526_amd import binding
from paper_2507_21526_amd.inputs import WORKLOADS, draw_qkv, workload_qkv
from tests.parity import MAX_ABS, P_BOUND_ABS, P_ROUND_U, compare, log, run_pass

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _cuda(*ts):
    return [t.to(DEV) for t in ts]


def _full_check(kind, cu, hq, hkv, d, S, W, L, T, splits=0, seed=0,
                label="", p_bound=False):
    q, k, v = draw_qkv(cu, hq, hkv, d, seed)
    qg, kg, vg = _cuda(q, k, v)
    scale = 1.0 / math.sqrt(d)
    o, lse, _ = run_pass(kind, qg, kg, vg, cu, S, W, L, T, splits,
                         poison=True)
    torch.cuda.synchronize()
    total = cu[-1]
    if total == 0:
        return
    assert not torch.isnan(o).any(), "unwritten output rows"
    compare(kind, q, k, v, cu, S, W, L, scale, o, lse, np.arange(total),
            range(hq), label=label or f"{kind} cu={cu} S={S} W={W} L={L} T={T}",
            p_bound=p_bound)


@pytest.mark.parametrize("kind", ["triangle", "causal"])
def test_tiny_workload_full(kind):
    w = WORKLOADS["tiny_n1024_d64"]
    log(f"case tiny {kind}")
    _full_check(kind, list(w.cu_seqlens), w.hq, w.hkv, w.d, w.sink, w.window,
                w.last, w.tile, seed=w.seed, label=f"tiny {kind}")


EDGE = [
    # cu, hq, hkv, d, S, W, L, T
    ([0, 1], 4, 1, 64, 0, 1, 0, 64),
    ([0, 1], 8, 8, 128, 5, 1, 3, 128),
    ([0, 37], 2, 1, 128, 4, 8, 5, 64),
    ([0, 200], 7, 1, 128, 8, 64, 24, 64),          # G = 7
    ([0, 300], 28, 4, 128, 16, 100, 40, 128),      # Qwen group shape
    ([0, 33, 450], 14, 2, 64, 8, 96, 40, 128),     # G = 7, d 64: 28 dealt row blocks
    ([0, 700], 7, 1, 128, 8, 256, 128, 128),       # G = 7, sink tile split around the window
    ([0, 513], 4, 4, 64, 0, 70, 0, 64),            # streaming only, no sink
    ([0, 640], 8, 2, 128, 130, 65, 129, 128),      # sink not tile aligned
    ([0, 0, 100, 100, 357, 1000], 4, 2, 64, 3, 50, 77, 64),  # varlen + empty
    ([0, 90], 3, 1, 64, 2, 10, 500, 64),           # last > n: all causal
    ([0, 1500], 16, 2, 128, 1, 1, 1, 128),         # W = 1, L = 1: 2 keys/row
    ([0, 777], 5, 5, 64, 8, 512, 50, 128),         # MHA, paper's S/W
    ([0, 2000], 6, 3, 128, 64, 128, 128, 64),      # paper probing shape
    ([0, 1100], 3, 3, 128, 16, 300, 40, 64),       # G = 1, d 128, T 64: two waves
]


@pytest.mark.parametrize("kind", ["triangle", "causal"])
@pytest.mark.parametrize("cu,hq,hkv,d,S,W,L,T", EDGE)
def test_edge_shapes_full(kind, cu, hq, hkv, d, S, W, L, T):
    log(f"case edge {kind} cu={cu} hq={hq} hkv={hkv} d={d} S={S} W={W} L={L} T={T}")
    # Streaming rows with a 1- or 2-key window hold only a few keys, so a
    # single rounded probability can dominate: elements of those shapes may
    # exceed 1e-2 within their own bf16-P rounding bound.
    _full_check(kind, cu, hq, hkv, d, S, W, L, T, seed=len(cu) + hq + d,
                p_bound=kind == "triangle" and S + W <= 4)


def _bf16_matches_rounded_fp32(kind, q, k, v, cu, S, W, L, T, label):
    """The bf16 output mode (written through the LDS-staged epilogue, or by
    the merge) equals the fp32 output mode rounded to nearest even, within
    one bf16 ulp (the two modes are separate compilations of the same
    arithmetic); LSE is identical."""
    o32, l32, _ = run_pass(kind, q, k, v, cu, S, W, L, T)
    o16, l16, _ = run_pass(kind, q, k, v, cu, S, W, L, T, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    ref = o32.to(torch.bfloat16)
    diff = (o16.view(torch.int16).int() - ref.view(torch.int16).int()).abs()
    worst = int(diff.max()) if diff.numel() else 0
    log(f"{label}: bf16 output vs RNE(fp32 output): max {worst} ulp, "
        f"{int((diff > 0).sum())} of {diff.numel()} differ")
    assert worst <= 1, label
    assert torch.equal(l16, l32), label


def test_bf16_output_is_rounded_fp32_output():
    cu = [0, 700]
    q, k, v = _cuda(*draw_qkv(cu, 8, 2, 128, 21))
    for kind in ("triangle", "causal"):
        _bf16_matches_rounded_fp32(kind, q, k, v, cu, 16, 128, 64, 128,
                                   f"bf16 out {kind} 700")


@pytest.mark.parametrize("cu,hq,hkv,d,S,W,L,T", EDGE)
def test_bf16_output_edge_shapes(cu, hq, hkv, d, S, W, L, T):
    """bf16 output mode on every edge shape: d 64 and 128, groups 1 to 8
    (two-, four- and seven-wave workgroups), ragged and packed sequences."""
    q, k, v = _cuda(*draw_qkv(cu, hq, hkv, d, len(cu) + hq + d))
    for kind in ("triangle", "causal"):
        _bf16_matches_rounded_fp32(kind, q, k, v, cu, S, W, L, T,
                                   f"bf16 out {kind} cu={cu} hq={hq} hkv={hkv} d={d}")


@pytest.mark.parametrize("name", ["tiny_n1024_d64", "mha_n32k"])
def test_bf16_output_workloads(name):
    w = WORKLOADS[name]
    cu = list(w.cu_seqlens)
    q, k, v = _cuda(*workload_qkv(w))
    for kind in ("triangle", "causal"):
        _bf16_matches_rounded_fp32(kind, q, k, v, cu, w.sink, w.window, w.last, w.tile,
                                   f"bf16 out {kind} {name}")


def test_split_invariance():
    """Split counts 1, 2, 7, auto and one per k-tile (32) on a 4096-token
    sequence.  Streaming rows do not depend on the split count at all (bit
    for bit).  Last rows do, through the bf16 rounding of P: each split
    takes its probabilities against its own running maximum, so the same
    p_j is rounded at a different scale, independently in each
    configuration.  Per element, each result lies within u * absw of the
    exact output (u = 2^-8, absw = sum_j p_j |v_j|, tests/parity.py), so two
    results lie within 2 u absw.  Over a head the expected relative L2
    difference is sqrt(2 E[delta^2]) with delta the relative rounding error:
    for mantissas spread log-uniformly, E[delta^2] = u^2 (1/2 - 1/8) /
    (3 ln 2) = 2.75e-6, so about 2.35e-3 (rows that average many keys have
    |O|^2 and the error's variance in the same ratio); the test allows 3e-3.
    Each split count also meets the parity bar against the oracle."""
    cu = [0, 4096]
    hq, hkv, d = 8, 2, 128
    q, k, v = draw_qkv(cu, hq, hkv, d, 5)
    qg, kg, vg = _cuda(q, k, v)
    outs = {}
    for splits in (1, 2, 7, 0, 32):
        o, lse, plan = run_pass("triangle", qg, kg, vg, cu, 128, 512, 128,
                                128, splits, poison=True)
        outs[splits] = (o, lse)
        log(f"splits {splits}: max_splits {plan.info.max_splits}")
    torch.cuda.synchronize()
    base_o, base_l = outs[1]
    n_last = 128
    rows = np.arange(4096 - n_last, 4096)
    rt = np.repeat(rows, hq)
    rh = np.tile(np.arange(hq, dtype=np.int32), rows.size)
    _, _, absw = oracle.attn_rows(q, k, v, cu, "triangle", 128, 512, 128,
                                  1 / math.sqrt(d), rt, rh, with_absw=True)
    bound = torch.from_numpy(2 * P_ROUND_U * (1 + 2 ** -6) * absw + 2 * P_BOUND_ABS)
    bound = bound.reshape(n_last, hq, d)
    for s, (o, lse) in outs.items():
        assert torch.equal(o[:-n_last], base_o[:-n_last]), s
        assert torch.equal(lse[:, :-n_last], base_l[:, :-n_last]), s
        diff = (o[-n_last:] - base_o[-n_last:]).double().cpu()
        assert bool((diff.abs() <= bound).all()), (s, float((diff.abs() / bound).max()))
        rel = float(diff.norm() / base_o[-n_last:].double().norm().cpu())
        log(f"splits {s} vs 1: rel-L2 {rel:.2e}, max |diff| / bound "
            f"{float((diff.abs() / bound).max()):.3f}")
        assert rel <= 3e-3, (s, rel)
        assert float((lse - base_l).abs().max()) <= 1e-4
        compare("triangle", q, k, v, cu, 128, 512, 128, 1 / math.sqrt(128),
                o, lse, rows, range(8), label=f"splits={s} last rows")


@pytest.mark.parametrize("kind", ["triangle", "causal", "blocksparse"])
def test_corrupt_device_schedule_poisons_outputs(kind):
    """A device schedule that does not match the launch is rejected: with a
    bad header every workgroup fills its slice of O and LSE with NaN
    (together every element); a rejected item's workgroups fill the rows it
    names, which no other workgroup writes, so the NaN is there whatever
    order the workgroups run in.  Either way the caller sees the failure
    instead of stale values.  Cases: a wrong magic word in the device
    header, one malformed item (rows past its sequence), and an item whose
    mode the launch does not serve (a list item outside a block-sparse
    schedule, an unknown mode)."""
    cu = [0, 700, 1024]
    q, k, v = _cuda(*draw_qkv(cu, 8, 2, 128, 23))
    if kind == "blocksparse":
        ptr, idx = [0], []
        for n in (700, 324):  # every q-tile keeps its diagonal and tile 0
            for t in range(-(-n // 128)):
                idx.extend(sorted({0, t}))
                ptr.append(len(idx))
        plan = binding.Plan("blocksparse", cu, 0, 1, 0, 128, 8, 128, device=q.device,
                            blocks=(ptr, idx))
    else:
        plan = binding.Plan(kind, cu, 16, 128, 64, 128, 8, 128, device=q.device)
    for out_dtype in (torch.float32, torch.bfloat16):
        o = torch.zeros(q.shape, dtype=out_dtype, device=q.device)
        lse = torch.zeros((8, cu[-1]), dtype=torch.float32, device=q.device)
        plan.run(q, k, v, o, lse, 0.1)
        torch.cuda.synchronize()
        assert not torch.isnan(o).any() and not torch.isnan(lse).any()
        good = plan.sched.clone()
        plan.sched[0] ^= 1  # magic word
        plan.run(q, k, v, o, lse, 0.1)
        torch.cuda.synchronize()
        assert bool(torch.isnan(o).all()), (kind, out_dtype, "header")
        assert bool(torch.isnan(lse).all()), (kind, out_dtype, "header")
        plan.sched.copy_(good)
        o.zero_()
        lse.zero_()
        item = binding.HDR_WORDS + binding.ITEM_WORDS * (plan.info.n_items - 1)
        plan.sched[item + 3] = 1 << 20  # r1 (word 3) of the last item, past its sequence
        plan.run(q, k, v, o, lse, 0.1)
        torch.cuda.synchronize()
        assert bool(torch.isnan(o).any()), (kind, out_dtype, "item")
        plan.sched.copy_(good)
        # an item mode the launch does not serve: a list item (mode 2) outside
        # a block-sparse schedule, or an unknown mode
        modes = (2, 7) if kind != "blocksparse" else (7,)
        for mode in modes:
            o.zero_()
            lse.zero_()
            plan.sched[item + 8] = mode  # I_MODE (word 8) of the last item
            plan.run(q, k, v, o, lse, 0.1)
            torch.cuda.synchronize()
            assert bool(torch.isnan(o).any()), (kind, out_dtype, "mode", mode)
            plan.sched.copy_(good)
        log(f"corrupt schedule {kind} {out_dtype}: outputs poisoned")


def test_packing_invariance():
    cu = [0, 1000, 1000, 3100, 3300]
    q, k, v = _cuda(*draw_qkv(cu, 8, 2, 128, 6))
    for kind in ("triangle", "causal"):
        packed, plse, _ = run_pass(kind, q, k, v, cu, 32, 256, 100, 128)
        for b in range(len(cu) - 1):
            s, e = cu[b], cu[b + 1]
            if s == e:
                continue
            alone, alse, _ = run_pass(kind, q[s:e].contiguous(),
                                      k[s:e].contiguous(), v[s:e].contiguous(),
                                      [0, e - s], 32, 256, 100, 128)
            torch.cuda.synchronize()
            assert torch.equal(packed[s:e], alone), (kind, b)
            assert torch.equal(plse[:, s:e], alse), (kind, b)


@pytest.mark.parametrize("hq,hkv,d,T", [(32, 8, 128, 128), (7, 1, 128, 64), (5, 1, 128, 128),
                                        (32, 8, 64, 128), (4, 4, 64, 64), (4, 4, 128, 128)])
def test_packing_invariance_in_a_full_launch(hq, hkv, d, T):
    """Short sequences alone, whose few workgroups leave most of the chip
    idle, against the same ones in a batch of several rounds of workgroups:
    whatever form of the kernel each launch takes, the rows are the same bit
    for bit."""
    log(f"case packing hq={hq} hkv={hkv} d={d} T={T}")
    lens = [333, 1, 1024] + [3000] * max(1, 40 // hkv) + [2001]
    cu = [0] + [int(x) for x in np.cumsum(lens)]
    q, k, v = _cuda(*draw_qkv(cu, hq, hkv, d, 16))
    for kind in ("triangle", "causal"):
        packed, plse, _ = run_pass(kind, q, k, v, cu, 32, 256, 100, T)
        for b in (0, 1, 2, len(lens) - 1):
            s, e = cu[b], cu[b + 1]
            alone, alse, _ = run_pass(kind, *(t[s:e].contiguous() for t in (q, k, v)),
                                      [0, e - s], 32, 256, 100, T)
            assert torch.equal(packed[s:e], alone), (kind, b)
            assert torch.equal(plse[:, s:e], alse), (kind, b)


def test_determinism():
    cu = [0, 5000]
    q, k, v = _cuda(*draw_qkv(cu, 8, 2, 128, 7))
    for kind in ("triangle", "causal"):
        a, al, _ = run_pass(kind, q, k, v, cu, 128, 1024, 256, 128)
        b, bl, _ = run_pass(kind, q, k, v, cu, 128, 1024, 256, 128,
                            poison=True)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(al, bl), kind


def test_mask_does_not_leak():
    """V = identity: output row i is the attention row P_i, which must be
    exactly zero outside the mask."""
    n = d = 128
    cu = [0, n]
    S, W, L, T = 3, 20, 10, 64
    q, k, _ = draw_qkv(cu, 2, 1, d, 8)
    v = torch.eye(n, dtype=torch.bfloat16).view(n, 1, d)
    qg, kg, vg = _cuda(q, k, v)
    for kind in ("triangle", "causal"):
        o, _, _ = run_pass(kind, qg, kg, vg, cu, S, W, L, T)
        torch.cuda.synchronize()
        m = torch.from_numpy(oracle.mask_matrix(kind, n, S, W, L)).bool()
        for h in range(2):
            p = o[:, h, :].cpu()
            assert torch.all(p[~m] == 0), kind
            assert torch.all(p[m] > 0), kind
            np.testing.assert_allclose(p.sum(1).numpy(), 1.0, atol=2e-3)


def test_linearity_in_v():
    cu = [0, 600]
    q, k, v1 = draw_qkv(cu, 4, 2, 64, 9)
    gen = torch.Generator().manual_seed(3)
    # small integers: v1 + v2 is exact in bf16
    a = torch.randint(-8, 8, v1.shape, generator=gen).to(torch.bfloat16)
    b = torch.randint(-8, 8, v1.shape, generator=gen).to(torch.bfloat16)
    qg, kg, ag, bg, sg = _cuda(q, k, a, b, a + b)
    for kind in ("triangle", "causal"):
        oa, _, _ = run_pass(kind, qg, kg, ag, cu, 4, 64, 32, 64)
        ob, _, _ = run_pass(kind, qg, kg, bg, cu, 4, 64, 32, 64)
        os_, _, _ = run_pass(kind, qg, kg, sg, cu, 4, 64, 32, 64)
        torch.cuda.synchronize()
        assert float((os_ - oa - ob).abs().max()) <= 1e-4, kind


def test_lse_optional_and_default_stream():
    cu = [0, 300]
    q, k, v = _cuda(*draw_qkv(cu, 4, 1, 64, 10))
    plan = binding.Plan("triangle", cu, 4, 32, 16, 64, 4, 64)
    o = torch.empty(q.shape, dtype=torch.float32, device=DEV)
    plan.run(q, k, v, o, None)
    ref, _, _ = run_pass("triangle", q, k, v, cu, 4, 32, 16, 64)
    torch.cuda.synchronize()
    assert torch.equal(o, ref)


def test_side_stream():
    cu = [0, 900]
    q, k, v = _cuda(*draw_qkv(cu, 8, 2, 128, 11))
    ref, _, _ = run_pass("triangle", q, k, v, cu, 16, 128, 64, 128)
    plan = binding.Plan("triangle", cu, 16, 128, 64, 128, 8, 128)
    o = torch.empty(q.shape, dtype=torch.float32, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        plan.run(q, k, v, o, None, stream=s)
    s.synchronize()
    assert torch.equal(o, ref)


@pytest.mark.parametrize("kind", ["triangle", "causal", "blocksparse"])
def test_graph_replay_matches_eager(kind):
    # the passes enqueue kernels only (no memset, allocation or
    # synchronisation), so they can be captured in a HIP graph; each replay,
    # with eager work in between, must give the eager result bit for bit
    cu, hq, hkv, d, T = [0, 700, 1024], 8, 2, 128, 128
    log(f"case graph replay {kind}")
    q, k, v = _cuda(*draw_qkv(cu, hq, hkv, d, 31))
    blocks = None
    if kind == "blocksparse":
        from paper_2507_21526_amd.inputs import blocksparse_lists
        ptr, idx = [0], []
        for b in range(len(cu) - 1):
            n = cu[b + 1] - cu[b]
            p, i = blocksparse_lists(-(-n // T), 0.5, 32 + b)
            base = ptr[-1]
            idx.extend(i)
            ptr.extend(base + x for x in p[1:])
        blocks = (ptr, idx)
    plan = binding.Plan(kind, cu, 16, 128, 64, T, hq, d, 1 if kind != "causal" else 0,
                        device=DEV, blocks=blocks)
    scale = 1.0 / math.sqrt(d)
    o_ref = torch.empty(q.shape, dtype=torch.float32, device=DEV)
    l_ref = torch.empty((hq, cu[-1]), dtype=torch.float32, device=DEV)
    plan.run(q, k, v, o_ref, l_ref, scale)
    torch.cuda.synchronize()
    o = torch.zeros_like(o_ref)
    lse = torch.zeros_like(l_ref)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.run(q, k, v, o, lse, scale)
    for _ in range(3):
        o.fill_(float("nan"))
        lse.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, o_ref) and torch.equal(lse, l_ref)
