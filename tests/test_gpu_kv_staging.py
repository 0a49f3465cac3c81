"""GPU parity of the head-window forward (mmattn_fwd_heads) and of the
head-pipelined K/V staging built on it (paper section 4.3), against the float64
oracle and against the whole-launch forward.  Tolerances as for mmattn_fwd."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2503_11367_amd import binding as mb
from paper_2503_11367_amd import staging
from paper_2503_11367_amd import workloads as wl

from gpu_util import (DEV, bf16_to_f64, f64, fields, general_path, gpu_bits, make_tensors, max_abs, rel_l2,
                      spy_workspace)

pytestmark = pytest.mark.gpu

TOL_MAX, TOL_L2, TOL_LSE = 2e-2, 5e-3, 4.5e-3


def oracle_fwd(lay, blocks, block, t, Hq, Hkv):
    f = fields(lay)
    rows = oa.rows_of_blocks(blocks, block)
    Q, K, V = f64(t["q_bits"]), f64(t["k_bits"]), f64(t["v_bits"])
    return oa.forward(Q, K, V, rows, f[0], f[1], f[2], modality=f[3], attend=f[4])


def check(o, lse, o_ref, lse_ref):
    og, lg = bf16_to_f64(o), lse.cpu().numpy().astype(np.float64)
    assert np.isfinite(og).all()
    assert max_abs(og, o_ref) < TOL_MAX and rel_l2(og, o_ref) < TOL_L2
    assert max_abs(lg, lse_ref) < TOL_LSE


@pytest.mark.parametrize("Hq,Hkv,D,hps,ncs", [(8, 4, 128, 1, 1), (8, 4, 64, 2, 2), (4, 4, 128, 1, 3),
                                              (12, 2, 128, 1, 2)])
def test_pipelined_equals_oracle(Hq, Hkv, D, hps, ncs):
    lay = wl.layout_random(120 + Hq + D, S=1024, n_samples=2, max_spans=5, deny_prob=0.3)
    blocks = [9, 1, 4, 6, 14, 3]
    t = make_tensors(300 + Hq, len(blocks) * 64, lay.S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    # the staging buffers start as NaN: a kernel that ran ahead of its window's
    # arrival would read them
    ks = torch.full_like(t["k"], float("nan"))
    vs = torch.full_like(t["v"], float("nan"))
    o, lse = staging.fwd_head_pipelined(t["q"], t["k"], t["v"], bits, bl, 64, heads_per_stage=hps,
                                        k_stage=ks, v_stage=vs, compute_streams=ncs)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle_fwd(lay, blocks, 64, t, Hq, Hkv)
    check(o, lse, o_ref, lse_ref)
    assert torch.equal(ks, t["k"]) and torch.equal(vs, t["v"])
    # same share through the whole-launch entry point: same values up to the
    # summation order of split lists
    o2, lse2 = mb.fwd(t["q"], t["k"], t["v"], bits, bl, 64)
    assert max_abs(bf16_to_f64(o), bf16_to_f64(o2)) < TOL_MAX
    assert max_abs(lse.cpu().numpy().astype(np.float64), lse2.cpu().numpy().astype(np.float64)) < 1e-4


@pytest.mark.parametrize("Hq,Hkv,D,hps", [(8, 4, 128, 1), (8, 4, 64, 2), (6, 2, 128, 2), (16, 8, 128, 1)])
def test_staged_entry_point(Hq, Hkv, D, hps):
    """mmattn_fwd_staged: copies and windows enqueued by the library itself."""
    lay = wl.layout_random(140 + Hq + D, S=1024, n_samples=2, max_spans=5, deny_prob=0.3)
    blocks = [2, 11, 4, 7, 15]
    t = make_tensors(400 + Hq, len(blocks) * 64, lay.S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    ks = torch.full_like(t["k"], float("nan"))
    vs = torch.full_like(t["v"], float("nan"))
    copy = torch.cuda.Stream()
    o_ref, lse_ref = oracle_fwd(lay, blocks, 64, t, Hq, Hkv)
    for _ in range(2):                   # second call: buffers reused straight away
        o, lse = mb.fwd_staged(t["q"], t["k"], t["v"], ks, vs, bits, bl, 64, hps, copy)
        torch.cuda.synchronize()
        check(o, lse, o_ref, lse_ref)
        assert torch.equal(ks, t["k"]) and torch.equal(vs, t["v"])
        ks.fill_(float("nan")); vs.fill_(float("nan"))


def test_staged_inputs_written_on_the_copy_stream():
    """Mask words and block list that earlier work on the copy stream writes, behind some
    milliseconds of other work: the plan waits for them."""
    Hq, Hkv, D = 8, 4, 128
    lay = wl.layout_random(152, S=1024, n_samples=2, max_spans=5)
    blocks = [3, 14, 6, 9]
    t = make_tensors(412, len(blocks) * 64, lay.S, Hq, Hkv, D)
    bits_late = gpu_bits(lay)
    bl_late = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    bits, bl = torch.zeros_like(bits_late), torch.zeros_like(bl_late)
    ks, vs = torch.empty_like(t["k"]), torch.empty_like(t["v"])
    a = torch.randn(4096, 4096, device=DEV)
    copy = torch.cuda.Stream()
    copy.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(copy):
        for _ in range(8):
            a = a @ a
            a = a / a.norm()
        bits.copy_(bits_late)
        bl.copy_(bl_late)
    o, lse = mb.fwd_staged(t["q"], t["k"], t["v"], ks, vs, bits, bl, 64, 1, copy)
    torch.cuda.synchronize()
    check(o, lse, *oracle_fwd(lay, blocks, 64, t, Hq, Hkv))


def test_staged_in_place():
    """k_stage / v_stage may be the source buffers themselves: no copies, same result."""
    lay = wl.layout_random(151, S=512, n_samples=1, max_spans=3)
    blocks = [1, 6, 3]
    t = make_tensors(411, len(blocks) * 64, lay.S, 8, 4, 128)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    k0, v0 = t["k"].clone(), t["v"].clone()
    o, lse = mb.fwd_staged(t["q"], t["k"], t["v"], t["k"], t["v"], bits, bl, 64, 2, torch.cuda.Stream())
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle_fwd(lay, blocks, 64, t, 8, 4)
    check(o, lse, o_ref, lse_ref)
    assert torch.equal(t["k"], k0) and torch.equal(t["v"], v0)


@pytest.mark.parametrize("S,Hq,Hkv,D,hps", [
    (16384, 36, 9, 128, 1),      # 72 MiB, 4608 (tile, head) pairs: two transfers, of five heads and of four
    (16384, 16, 16, 64, 4),      # 64 MiB, 2048 pairs: everything at once
    (512, 16, 16, 128, 1),       # one kernel after one transfer
])
@pytest.mark.parametrize("in_place", ["neither", "k", "v", "both"])
def test_staged_windows_together(S, Hq, Hkv, D, hps, in_place):
    """Windows that travel together, their last group smaller; K or V already in its place."""
    lay = wl.layout_random(154, S=S, n_samples=3, max_spans=5, deny_prob=0.3)
    nb = S // 128
    blocks = np.random.default_rng(154).permutation(nb).tolist()
    t = make_tensors(414, S, S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    ks = t["k"] if in_place in ("k", "both") else torch.full_like(t["k"], float("nan"))
    vs = t["v"] if in_place in ("v", "both") else torch.full_like(t["v"], float("nan"))
    k0, v0 = t["k"].clone(), t["v"].clone()
    o, lse = mb.fwd_staged(t["q"], t["k"], t["v"], ks, vs, bits, bl, 128, hps, torch.cuda.Stream())
    torch.cuda.synchronize()
    assert torch.equal(ks, k0) and torch.equal(vs, v0)
    f = fields(lay)
    rows = oa.rows_of_blocks(blocks, 128)
    sel = np.sort(np.random.default_rng(7).choice(S, size=96, replace=False))
    Q, K, V = f64(t["q_bits"]), f64(t["k_bits"]), f64(t["v_bits"])
    rep = Hq // Hkv
    for g in sorted({0, 4, 5, Hkv - 1}):
        h = g * rep + rep - 1
        o_ref, lse_ref = oa.forward(Q[sel][:, h:h + 1], K[:, g:g + 1], V[:, g:g + 1], rows[sel], f[0], f[1], f[2],
                                    modality=f[3], attend=f[4])
        check(o[sel][:, h:h + 1], lse[h:h + 1][:, sel], o_ref, lse_ref)


@pytest.mark.parametrize("S", [1024, 4224])
def test_staged_from_pinned_memory(S):
    """Sources in pinned host memory take the runtime's copies, window by window; at 4224 tokens on the
    general path, which forms the key norms of each window behind its arrival."""
    lay = wl.layout_random(155, S=S, n_samples=2, max_spans=5)
    Hq, Hkv, D, blocks = 8, 4, 128, [3, 14, 6, 9]
    t = make_tensors(415, len(blocks) * 64, lay.S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    k_src, v_src = (torch.empty(t[x].shape, dtype=t[x].dtype, pin_memory=True) for x in "kv")
    k_src.copy_(t["k"]); v_src.copy_(t["v"])
    ks, vs = torch.full_like(t["k"], float("nan")), torch.full_like(t["v"], float("nan"))
    o, lse = torch.empty_like(t["q"]), torch.empty(Hq, t["q"].shape[0], dtype=torch.float32, device=DEV)
    ws = spy_workspace(mb.OP_FWD_HEADS, lay.S, len(blocks), 64, Hq, Hkv, D)
    copy = torch.cuda.Stream()
    rc = mb.lib().mmattn_fwd_staged(t["q"].data_ptr(), k_src.data_ptr(), v_src.data_ptr(), ks.data_ptr(), vs.data_ptr(),
                                    bits.data_ptr(), bl.data_ptr(), len(blocks), 64, lay.S, Hq, Hkv, D, D ** -0.5, mb.BF16, 2,
                                    o.data_ptr(), lse.data_ptr(), ws.data_ptr(), ws.numel(), copy.cuda_stream,
                                    torch.cuda.current_stream().cuda_stream)
    assert rc == mb.OK
    torch.cuda.synchronize()
    assert general_path(ws) == (S > 1024)
    assert torch.equal(ks, t["k"]) and torch.equal(vs, t["v"])
    check(o, lse, *oracle_fwd(lay, blocks, 64, t, Hq, Hkv))


@pytest.mark.parametrize("S,Hq,Hkv", [(512, 8, 4), (4096, 32, 8)])
def test_staged_in_a_graph(S, Hq, Hkv):
    """One captured call, replayed over new inputs with eager work in between."""
    lay = wl.layout_random(156, S=S, n_samples=2, max_spans=4)
    t = make_tensors(416, S, S, Hq, Hkv, 128)
    bits = gpu_bits(lay)
    bl = torch.arange(S // 64, dtype=torch.int32, device=DEV)
    ks, vs = torch.empty_like(t["k"]), torch.empty_like(t["v"])
    ws = torch.empty(mb.workspace_size(mb.OP_FWD_HEADS, S, S // 64, 64, Hq, Hkv, 128), dtype=torch.uint8, device=DEV)
    out = (torch.empty_like(t["q"]), torch.empty(Hq, S, dtype=torch.float32, device=DEV))
    copy = torch.cuda.Stream()
    args = (t["q"], t["k"], t["v"], ks, vs, bits, bl, 64, 1, copy)
    mb.fwd_staged(*args, out=out, ws=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mb.fwd_staged(*args, out=out, ws=ws)
    for _ in range(3):
        t["k"].neg_(); t["v"].mul_(0.5)
        ks.fill_(float("nan")); vs.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        o, lse = out[0].clone(), out[1].clone()
        o2, lse2 = mb.fwd_staged(*args)
        assert torch.equal(o, o2) and torch.equal(lse, lse2)


def test_window_touches_only_its_heads():
    """Heads outside the window are neither read (NaN there is harmless) nor
    written (sentinel survives); windows in any order, plan reused."""
    Hq, Hkv, D = 8, 4, 128
    lay = wl.layout_random(131, S=512, n_samples=1, max_spans=3)
    blocks = list(range(8))
    t = make_tensors(77, 512, lay.S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    o_ref, lse_ref = oracle_fwd(lay, blocks, 64, t, Hq, Hkv)
    ws = torch.empty(mb.workspace_size(mb.OP_FWD_HEADS, lay.S, 8, 64, Hq, Hkv, D), dtype=torch.uint8, device=DEV)
    o = torch.full_like(t["q"], 7.0)
    lse = torch.full((Hq, 512), 7.0, dtype=torch.float32, device=DEV)
    for n, (g0, c) in enumerate([(2, 1), (0, 2), (3, 1)]):
        k = torch.full_like(t["k"], float("nan"))
        v = torch.full_like(t["v"], float("nan"))
        k[:, g0:g0 + c] = t["k"][:, g0:g0 + c]
        v[:, g0:g0 + c] = t["v"][:, g0:g0 + c]
        before = o.clone()
        mb.fwd_heads(t["q"], k, v, bits, bl, 64, g0, c, plan_ready=n > 0, out=(o, lse), ws=ws)
        torch.cuda.synchronize()
        hs = slice(2 * g0, 2 * (g0 + c))
        outside = torch.ones(Hq, dtype=torch.bool)
        outside[hs] = False
        assert torch.equal(o[:, outside], before[:, outside])
        check(o[:, hs], lse[hs], o_ref[:, hs], lse_ref[hs])
    check(o, lse, o_ref, lse_ref)


@pytest.mark.parametrize("order", [[(0, 4), (4, 1), (5, 2), (7, 1)], [(7, 1), (0, 4), (4, 1), (5, 2)], "staged"])
def test_windows_share_a_plan_across_kernels(order):
    """4096 rows of 64 / 8 heads: windows of four KV heads put pairs of heads into a workgroup and
    walk whole lists, windows of one and two run single heads and cut them; each reuses the plan
    that another left, whatever slice length that chose.  `staged`: two windows of four in
    mmattn_fwd_staged, where 16 MiB of keys and values travel and are attended together."""
    Hq, Hkv, D, S = 64, 8, 128, 4096
    lay = wl.layout_packed(153, S=S, n_samples=4, span_lo=40, span_hi=300)
    blocks = np.random.default_rng(153).permutation(S // 64).tolist()
    t = make_tensors(413, S, S, Hq, Hkv, D)
    bits = gpu_bits(lay)
    bl = torch.tensor(blocks, dtype=torch.int32, device=DEV)
    if order == "staged":
        o, lse = mb.fwd_staged(t["q"], t["k"], t["v"], torch.empty_like(t["k"]), torch.empty_like(t["v"]), bits, bl, 64, 4,
                               torch.cuda.Stream())
        order = [(0, 4), (4, 4)]
    else:
        ws = torch.empty(mb.workspace_size(mb.OP_FWD_HEADS, S, len(blocks), 64, Hq, Hkv, D), dtype=torch.uint8, device=DEV)
        o, lse = torch.full_like(t["q"], 7.0), torch.full((Hq, S), 7.0, dtype=torch.float32, device=DEV)
        for n, (g0, c) in enumerate(order):
            mb.fwd_heads(t["q"], t["k"], t["v"], bits, bl, 64, g0, c, plan_ready=n > 0, out=(o, lse), ws=ws)
    torch.cuda.synchronize()
    f = fields(lay)
    rows = oa.rows_of_blocks(blocks, 64)
    sel = np.sort(np.random.default_rng(6).choice(S, size=160, replace=False))
    Q, K, V = f64(t["q_bits"]), f64(t["k_bits"]), f64(t["v_bits"])
    for g0, c in order:
        for g, h in ((g0, 8 * g0), (g0 + c - 1, 8 * (g0 + c) - 1)):
            o_ref, lse_ref = oa.forward(Q[sel][:, h:h + 1], K[:, g:g + 1], V[:, g:g + 1], rows[sel], f[0], f[1], f[2],
                                        modality=f[3], attend=f[4])
            check(o[sel][:, h:h + 1], lse[h:h + 1][:, sel], o_ref, lse_ref)


def test_workload2_pipelined_sampled():
    """The 8k workload in the configuration bench.py times: whole sequence,
    one KV head per stage; sampled rows and heads against the oracle."""
    w = wl.workload(2)
    lay = w.layout
    nb = lay.S // w.N_B
    t = make_tensors(w.tensor_seed, lay.S, lay.S, w.Hq, w.Hkv, w.D)
    bits = gpu_bits(lay)
    bl = torch.arange(nb, dtype=torch.int32, device=DEV)
    o, lse = staging.fwd_head_pipelined(t["q"], t["k"], t["v"], bits, bl, w.N_B, heads_per_stage=1,
                                        compute_streams=2)
    torch.cuda.synchronize()
    f = fields(lay)
    rng = np.random.default_rng(5)
    sel = np.sort(rng.choice(lay.S, size=192, replace=False))
    Q, K, V = f64(t["q_bits"]), f64(t["k_bits"]), f64(t["v_bits"])
    rep = w.Hq // w.Hkv
    for h in (0, 13, 31):
        g = h // rep
        o_ref, lse_ref = oa.forward(Q[sel][:, h:h + 1], K[:, g:g + 1], V[:, g:g + 1], sel, f[0], f[1], f[2],
                                    modality=f[3], attend=f[4])
        check(o[sel][:, h:h + 1], lse[h:h + 1][:, sel], o_ref, lse_ref)
