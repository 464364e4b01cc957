"""GPU parity of the fused decode attention + score path (kv_append, kv_attend_score, kv_evict_finish).

The attention output of every layer, sequence and query head is compared with the oracle's float64
attention: |o_gpu - o_ref| <= 1e-3 * sum_i a(i) |v(i)| (the scale of the weighted sum, which bounds its
rounding; 1e-3 is the probability tolerance of the scores) + 2^-8 |o_ref| when the output is rounded to bf16.
The scores, utilities, retention sets and compacted rows follow the same rules as the separate-pass step
(scores/utilities 1e-3 relative, retention equal outside the 1e-4 band with lockstep adoption, positions and
K/V rows bit-exact)."""
import zlib

import numpy as np
import pytest
import torch

from oracle import attention_output, evict_step, layer_scores, refresh_due, to_f64
from parity import assert_close, assert_o, check_norm_cache, lockstep_adopter, oracle_cache, oracle_params, to_device
from workload import LLAMA8B, LLAMA8B_LAZY, QWEN, TINY, Workload, raw_numpy

pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2609_03515_amd.binding")

def attend_layers(shape, cfg, n, q, k, v, pos, cur_pos, emit, ws, per_layer):
    o = torch.empty_like(q)
    if per_layer:
        for l in range(cfg.layers):
            B.kv_attend_score(shape, l, 1, n, q[l], k, v, pos, cur_pos, cfg.recency_bias, cfg.recency_window,
                              emit, o[l], ws)
    else:
        B.kv_attend_score(shape, 0, cfg.layers, n, q, k, v, pos, cur_pos, cfg.recency_bias, cfg.recency_window,
                          emit, o, ws)
    return o


def run_fused_lockstep(cfg, steps, per_layer, vnorm=False, entropy=False, emit_norms=False, merge=0,
                       norm_cache=False):
    w = Workload(cfg)
    cap = max(cfg.prefill_len, cfg.budget) + 1
    st = w.prefill(capacity=cap)
    oc = oracle_cache(st, cfg.dtype)
    dev = to_device(st)
    shape = B.make_shape(cfg.batch, cfg.layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cap, cfg.dtype)
    params = B.make_params(cfg.alpha, cfg.budget, cfg.refresh_period, cfg.score_free, cfg.nonrefresh_init,
                           cfg.recency_bias, cfg.recency_window, vnorm=vnorm, entropy=entropy,
                           norms_emitted=emit_norms, score_merge=merge)
    op = oracle_params(cfg, vnorm=vnorm, entropy=entropy)
    ws = B.workspace(shape, cap)
    n = st["n"]
    norms = None
    if norm_cache:
        norms = torch.full((cfg.layers, cfg.batch, cfg.n_kv_heads, cap), -1.0, device="cuda")
        B.kv_value_norms(shape, n, dev["v"], norms)
    flips = 0
    for t in range(1, steps + 1):
        si = w.step_inputs(t)
        sig = to_device(si)
        refresh = refresh_due(t, cfg.refresh_period, cfg.score_free)
        print(f"{cfg.name} t={t} refresh={refresh} per_layer={per_layer} n_in={n}", flush=True)
        B.kv_append(shape, params, t, n, si["new_pos"], sig["k_new"], sig["v_new"], dev["k"], dev["v"], dev["u"],
                    dev["pos"], v_norms=norms)
        emit = (B.KV_EMIT_SCORES | (B.KV_EMIT_VNORMS if emit_norms else 0)) if refresh else 0
        o = attend_layers(shape, cfg, n + 1, sig["q"], dev["k"], dev["v"], dev["pos"], si["new_pos"], emit, ws,
                          per_layer)
        keep = torch.zeros(cfg.batch, cap, dtype=torch.uint8, device="cuda")
        s_out = torch.full((cfg.layers, cfg.batch, n + 1), -1.0, device="cuda")
        n_out = B.kv_evict_finish(shape, params, t, n + 1, dev["k"], dev["v"], dev["u"], dev["pos"], ws,
                                  keep_out=keep, s_out=s_out, v_norms=norms)
        torch.cuda.synchronize()
        keep_g = keep.cpu().numpy()[:, : n + 1].astype(bool)
        step_flips = []
        ref = evict_step(oc, raw_numpy(si["q"]), raw_numpy(si["k_new"]), raw_numpy(si["v_new"]), t, si["new_pos"],
                         op, keep_override=lockstep_adopter(keep_g, cfg.budget, f"{cfg.name} t={t}", step_flips),
                         attention=True)
        assert n_out == ref.n_out == min(cfg.budget, n + 1)
        flips += sum(step_flips)
        assert_o(o, ref.o, ref.o_scale, cfg.dtype, f"{cfg.name} t={t} attention")
        if ref.refreshed:
            assert_close(s_out.cpu().numpy(), ref.s_layers, f"{cfg.name} t={t} scores")
        n = n_out
        assert_close(dev["u"][:, :n].cpu().numpy(), oc.u[:, :n], f"{cfg.name} t={t} utilities")
        np.testing.assert_array_equal(dev["pos"][:, :n].cpu().numpy(), oc.pos[:, :n])
        np.testing.assert_array_equal(raw_numpy(dev["k"])[:, :, :, :n], oc.k[:, :, :, :n])
        np.testing.assert_array_equal(raw_numpy(dev["v"])[:, :, :, :n], oc.v[:, :, :, :n])
        if norms is not None:
            check_norm_cache(B, shape, dev["v"], norms, n, oc.v, cfg.dtype, f"{cfg.name} t={t}")
    return flips


CASES = {
    "tiny": (TINY, 6),
    "llama8b_reduced": (LLAMA8B.scaled(batch=2, layers=3, prefill_len=1200, budget=120), 4),
    "llama8b_split_step1": (LLAMA8B.scaled(batch=1, layers=2, prefill_len=6000, budget=600), 2),
    "lazy_r4_min": (LLAMA8B_LAZY.scaled(batch=2, layers=2, prefill_len=800, budget=80), 6),
    "qwen_reduced": (QWEN.scaled(batch=2, layers=2, prefill_len=1000, budget=250), 3),
}


@pytest.mark.parametrize("per_layer", [True, False], ids=["per_layer", "all_layers"])
@pytest.mark.parametrize("name", list(CASES))
def test_fused_step_lockstep(name, per_layer):
    cfg, steps = CASES[name]
    flips = run_fused_lockstep(cfg, steps, per_layer)
    print(f"{name}: in-band flips {flips}")


@pytest.mark.parametrize("emit_norms", [False, True], ids=["norms_from_v", "norms_emitted"])
@pytest.mark.parametrize("name", ["tiny", "llama8b_reduced", "llama8b_split_step1", "qwen_reduced"])
def test_fused_step_scorer_variants(name, emit_norms):
    """VNorm + entropy weighting on the fused path: the perturbations are applied by kv_evict_finish to the
    scores the attention emitted, with the value norms either read from V by the finish or emitted by the
    attention's V pass (one and several chunks per slab)."""
    cfg, steps = CASES[name]
    run_fused_lockstep(cfg, steps, per_layer=True, vnorm=True, entropy=True, emit_norms=emit_norms)
    if emit_norms:
        run_fused_lockstep(cfg, 2, per_layer=False, vnorm=True, entropy=False, emit_norms=True)


@pytest.mark.parametrize("per_layer", [True, False], ids=["per_layer", "all_layers"])
@pytest.mark.parametrize("name", ["tiny", "llama8b_reduced", "llama8b_split_step1", "lazy_r4_min", "qwen_reduced"])
def test_fused_step_value_norm_cache(name, per_layer):
    """VNorm + entropy on the fused path with the value-norm cache: kv_append caches the newcomer's norm, the
    finish reads the cached norms (neither the attention nor the finish reads V for them) and keeps the cache
    through the placement and the compaction."""
    cfg, steps = CASES[name]
    run_fused_lockstep(cfg, steps, per_layer, vnorm=True, entropy=True, norm_cache=True)


@pytest.mark.parametrize("name,merge", [("llama8b_reduced", 4), ("llama8b_split_step1", 8), ("qwen_reduced", 2)])
def test_fused_step_merged_fold(name, merge):
    """The finish folds the attention's per-KV-head scores in the blocks a merging scorer would add (one and
    several chunks per slab)."""
    cfg, steps = CASES[name]
    run_fused_lockstep(cfg, steps, per_layer=True, entropy=True, merge=merge)


# ---- one call on random inputs over the supported geometries -------------------------------------------
GEOMS = [  # (dtype, head_dim, n_q, n_kv, n)
    ("bf16", 128, 32, 8, 1), ("bf16", 128, 32, 8, 15), ("bf16", 128, 32, 8, 256), ("bf16", 128, 32, 8, 257),
    ("bf16", 128, 32, 8, 3278), ("bf16", 128, 8, 8, 700), ("bf16", 128, 16, 8, 700), ("bf16", 128, 28, 4, 2049),
    ("bf16", 128, 16, 2, 300), ("bf16", 128, 16, 1, 520), ("bf16", 64, 8, 8, 333), ("bf16", 64, 16, 4, 1000),
    ("bf16", 64, 16, 2, 999), ("f32", 64, 4, 2, 513), ("f32", 128, 4, 4, 600), ("f32", 128, 8, 2, 1025),
    ("f32", 64, 16, 1, 200), ("bf16", 128, 32, 8, 5200),  # LDS limit: more than 5120 rows per chunk
    ("bf16", 128, 10, 2, 701), ("bf16", 128, 24, 2, 611), ("bf16", 64, 12, 2, 803),  # groups 5, 12, 6
]


@pytest.mark.parametrize("dtype,d,hq,hkv,n", GEOMS)
def test_attend_geometries(dtype, d, hq, hkv, n):
    L, b = 2, 2
    gen = torch.Generator(device="cpu").manual_seed(zlib.crc32(repr((dtype, d, hq, hkv, n)).encode()))
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cap = n + 3
    k = (torch.randn(L, b, hkv, cap, d, generator=gen) * 1.5).to(tdt)
    v = torch.randn(L, b, hkv, cap, d, generator=gen).to(tdt)
    q = torch.randn(L, b, hq, d, generator=gen).to(tdt)
    pos = torch.randperm(4 * cap, generator=gen)[:cap].to(torch.int32).repeat(b, 1).contiguous()
    cur = int(pos[0, :n].max())
    bias, window = 0.5, 64
    shape = B.make_shape(b, L, hq, hkv, d, cap, dtype)
    ws = B.workspace(shape, n)
    dk, dv, dq, dpos = k.cuda(), v.cuda(), q.cuda(), pos.cuda()
    print(f"attend {dtype} d={d} hq={hq} hkv={hkv} n={n}", flush=True)
    o_all = torch.empty_like(dq)
    B.kv_attend_score(shape, 0, L, n, dq, dk, dv, dpos, cur, bias, window, 1, o_all, ws)
    u = torch.zeros(b, cap, device="cuda")
    s_out = torch.empty(L, b, n, device="cuda")
    params = B.make_params(0.5, n, recency_bias=bias, recency_window=window)
    assert B.kv_evict_finish(shape, params, 1, n, dk, dv, u, dpos, ws, s_out=s_out) == n
    o_one = torch.empty_like(dq)
    for l in range(L):
        B.kv_attend_score(shape, l, 1, n, dq[l], dk, dv, dpos, cur, bias, window, 0, o_one[l], ws)
    torch.cuda.synchronize()
    kr, vr, qr = raw_numpy(k), raw_numpy(v), raw_numpy(q)
    pr = pos.numpy().astype(np.int64)
    o_ref = np.zeros((L, b, hq, d))
    sc = np.zeros_like(o_ref)
    s_ref = np.zeros((L, b, n))
    for l in range(L):
        for bb in range(b):
            keys = to_f64(kr[l, bb, :, :n], dtype)
            ql = to_f64(qr[l, bb], dtype)
            o_ref[l, bb], sc[l, bb] = attention_output(ql, keys, to_f64(vr[l, bb, :, :n], dtype), pr[bb, :n], cur,
                                                       bias, window)
            s_ref[l, bb] = layer_scores(ql, keys, pr[bb, :n], cur, bias, window)
    assert_o(o_all, o_ref, sc, dtype, "all layers in one call")
    assert_o(o_one, o_ref, sc, dtype, "one call per layer")
    assert_close(s_out.cpu().numpy(), s_ref, "scores from the attention")


@pytest.mark.parametrize("group", [3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("n", [1, 15, 17, 255, 257, 1033])
def test_attend_value_pass_edges(group, n):
    """The value pass on the matrix cores (bf16, d = 128, padded groups of 4 to 16) at the edges of its 16-row
    units and of the chunks, one chunk per slab and several, with rows whose scales differ by 2^20; then with an
    infinity and a NaN among the values, which reach their own column of every head and no other.

    Bound per output, relative to sum_i a(i) |v_i|: a logit is a sum of 128 products of fp32 rounding, at most
    128 * 2^-24 of sum |q k| / sqrt(d) <= 16, and moves its probability by as much: 1.3e-4; the products and their
    sum add n * 2^-24 <= 6.2e-5; together 2e-4, and 2^-8 of the output for its rounding to bf16."""
    b, hkv, d = 2, 2, 128
    hq = group * hkv
    gen = torch.Generator(device="cpu").manual_seed(1000 * group + n)
    cap = n + 5
    k = torch.randn(1, b, hkv, cap, d, generator=gen).clamp_(-4, 4).to(torch.bfloat16)
    v = torch.randn(1, b, hkv, cap, d, generator=gen)
    v *= 2.0 ** torch.randint(-10, 11, (1, b, hkv, cap, 1), generator=gen)
    v = v.to(torch.bfloat16)
    q = (0.5 * torch.randn(1, b, hq, d, generator=gen)).clamp_(-2, 2).to(torch.bfloat16)
    pos = torch.arange(cap, dtype=torch.int32).repeat(b, 1).contiguous()
    shape = B.make_shape(b, 1, hq, hkv, d, cap, "bf16")
    ws = B.workspace(shape, n)
    dk, dq, dpos = k.cuda(), q.cuda(), pos.cuda()

    def attend(values):
        o = torch.empty_like(dq)
        B.kv_attend_score(shape, 0, 1, n, dq, dk, values.cuda(), dpos, n - 1, 0.0, 0, B.KV_EMIT_SCORES, o, ws)
        torch.cuda.synchronize()
        return to_f64(raw_numpy(o), "bf16")

    print(f"value pass group={group} n={n}", flush=True)
    kr, vr, qr = raw_numpy(k), raw_numpy(v), raw_numpy(q)
    ref, scale = np.zeros((1, b, hq, d)), np.zeros((1, b, hq, d))
    for bb in range(b):
        ref[0, bb], scale[0, bb] = attention_output(to_f64(qr[0, bb], "bf16"), to_f64(kr[0, bb, :, :n], "bf16"),
                                                    to_f64(vr[0, bb, :, :n], "bf16"), pos.numpy()[bb, :n].astype(np.int64),
                                                    n - 1, 0.0, 0)
    got = attend(v)
    assert np.all(np.abs(got - ref) <= 2e-4 * scale + 2.0 ** -8 * np.abs(ref))
    odd = v.clone()
    odd[0, 0, 1, n // 2, 7] = float("inf")
    odd[0, 1, 0, n - 1, 100] = float("nan")
    odd[0, 1, 0, 0, 9] = float("-inf")
    got2 = attend(odd)
    assert np.all(np.isposinf(got2[0, 0, group:, 7])) and np.all(np.isnan(got2[0, 1, :group, 100]))
    assert np.all(np.isneginf(got2[0, 1, :group, 9]))
    same = np.ones_like(got, dtype=bool)
    same[0, 0, group:, 7] = same[0, 1, :group, 100] = same[0, 1, :group, 9] = False
    assert np.all(np.abs(got2 - got)[same] <= (4e-4 * scale + 2.0 ** -7 * np.abs(ref))[same])


@pytest.mark.parametrize("emit", [0, 1])
@pytest.mark.parametrize("group", [4, 7, 16])
@pytest.mark.parametrize("n", [200, 700])
def test_attend_infinite_value_weights(n, group, emit):
    """An infinity among the values, with and without the score and with one chunk per slab and several, on a row whose
    probability underflows to zero for the group's first head and for no other: 0 * inf is NaN for that head and an
    infinity for the others, whatever is done with the probabilities afterwards (with one chunk, they are replaced by
    the score's group sums).  Columns without an infinity, and the scores, are those of finite values."""
    b, hkv, d = 2, 2, 128
    hq = group * hkv
    gen = torch.Generator(device="cpu").manual_seed(100 * n + 10 * group + emit)
    k = torch.randn(1, b, hkv, n, d, generator=gen).clamp_(-4, 4).to(torch.bfloat16)
    v = torch.randn(1, b, hkv, n, d, generator=gen).to(torch.bfloat16)
    q = (0.5 * torch.randn(1, b, hq, d, generator=gen)).clamp_(-2, 2).to(torch.bfloat16)
    rows = torch.arange(0, n, 3)
    k[:, :, :, rows, 0] = 4.0      # logit 4 * -500 / sqrt(128) = -177 for the first heads
    k[:, :, :, 1, 0] = 0.0         # (their maximum is no lower than this row's)
    q[:, :, ::group, 0] = -500.0
    pos = torch.arange(n, dtype=torch.int32).repeat(b, 1).contiguous()
    shape = B.make_shape(b, 1, hq, hkv, d, n, "bf16")
    ws = B.workspace(shape, n)
    dk, dq, dpos = k.cuda(), q.cuda(), pos.cuda()

    def attend(values):
        o = torch.empty_like(dq)
        u, s_out = torch.zeros(b, n, device="cuda"), torch.zeros(1, b, n, device="cuda")
        dv = values.cuda()
        B.kv_attend_score(shape, 0, 1, n, dq, dk, dv, dpos, n - 1, 0.0, 0, emit, o, ws)
        if emit:
            B.kv_evict_finish(shape, B.make_params(0.5, n), 1, n, dk, dv, u, dpos, ws, s_out=s_out)
        torch.cuda.synchronize()
        return to_f64(raw_numpy(o), "bf16"), s_out.cpu().numpy()

    print(f"infinite value n={n} group={group} emit={emit}", flush=True)
    finite, scores = attend(v)
    odd = v.clone()
    cols = torch.arange(0, d, 5)   # columns in every workgroup's waves, each with the infinity in a row of its own
    for i, c in enumerate(cols.tolist()):
        odd[0, :, :, rows[(7 * i) % len(rows)], c] = float("inf") if i % 2 == 0 else float("-inf")
    odd[0, :, :, 0, 3], odd[0, :, :, n - 1, 3] = float("inf"), float("-inf")  # both signs: NaN
    odd[0, :, :, n // 2, 126] = float("nan")
    got, scores2 = attend(odd)
    first = np.zeros(hq, dtype=bool)
    first[::group] = True
    assert np.all(np.isnan(got[:, :, first][..., cols])) and np.all(np.isnan(got[..., [3, 126]]))
    assert np.all(np.isposinf(got[:, :, ~first][..., cols[::2]])) and np.all(np.isneginf(got[:, :, ~first][..., cols[1::2]]))
    # the waves claim their rows, so two calls add in different orders: n * 2^-24 <= 4.2e-5 of the weighted values
    # (at most the largest) on each side, and a step of bf16; of the scores on each side
    rest = np.setdiff1d(np.arange(d), [3, 126, *cols.tolist()])
    bound = 1e-4 * v.abs().max().item() + 2.0 ** -7 * np.abs(finite)
    assert np.all(np.abs(got - finite)[..., rest] <= bound[..., rest])
    np.testing.assert_allclose(scores2, scores, rtol=1e-4)


@pytest.mark.parametrize("emit", [0, 1])
@pytest.mark.parametrize("L,b,hkv,group", [(1, 3, 4, 4), (1, 3, 3, 1), (3, 1, 5, 7), (2, 11, 1, 2)])
def test_attend_slab_counts_beyond_eights(L, b, hkv, group, emit):
    """Slabs are numbered in groups of eight, a group's chunks eight workgroups apart, and the last slabs in order: 12, 9,
    15 and 22 slabs of several chunks, where both numberings meet in one launch of the attention and of its combine.
    Bounds as in the geometries above; every slab has inputs of its own."""
    d, n, hq = 128, 1100, hkv * group
    gen = torch.Generator(device="cpu").manual_seed(100 * hkv + 10 * group + b)
    k, v = (torch.randn(L, b, hkv, n, d, generator=gen).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(L, b, hq, d, generator=gen).to(torch.bfloat16)
    pos = torch.arange(n, dtype=torch.int32).repeat(b, 1).contiguous()
    shape = B.make_shape(b, L, hq, hkv, d, n, "bf16")
    ws = B.workspace(shape, n)
    dk, dv, dq, dpos = k.cuda(), v.cuda(), q.cuda(), pos.cuda()
    o = torch.full_like(dq, float("nan"))
    s_out = torch.full((L, b, n), float("nan"), device="cuda")
    print(f"slabs L={L} b={b} hkv={hkv} group={group} emit={emit}", flush=True)
    B.kv_attend_score(shape, 0, L, n, dq, dk, dv, dpos, n - 1, 0.0, 0, emit, o, ws)
    if emit:
        B.kv_evict_finish(shape, B.make_params(0.5, n), 1, n, dk, dv, torch.zeros(b, n, device="cuda"), dpos, ws,
                          s_out=s_out)
    torch.cuda.synchronize()
    pr = np.arange(n)
    for l in range(L):
        for bb in range(b):
            keys, ql = to_f64(raw_numpy(k)[l, bb], "bf16"), to_f64(raw_numpy(q)[l, bb], "bf16")
            ref, scale = attention_output(ql, keys, to_f64(raw_numpy(v)[l, bb], "bf16"), pr, n - 1, 0.0, 0)
            assert_o(o[l : l + 1, bb : bb + 1], ref[None, None], scale[None, None], "bf16", f"outputs of {l}, {bb}")
            if emit:
                assert_close(s_out[l, bb].cpu().numpy(), layer_scores(ql, keys, pr, n - 1, 0.0, 0), f"scores of {l}, {bb}")


@pytest.mark.parametrize("hq,hkv,n", [(4, 1, 700), (4, 1, 6000), (4, 1, 16384), (16, 1, 90000)])
def test_attend_infinite_logit(hq, hkv, n):
    """An infinite logit makes its head's softmax undefined: the outputs are NaN, and so are the scores of the rows that
    share its chunk, however many chunks there are (3, 24, 64 and 256 here: the combine takes up to 16, up to 64 and more
    in different ways), not an ordinary score of zero."""
    d, row = 128, n // 2 + 100  # (28 rows or more from either end of its chunk of 240, 256, 256 or 352 rows)
    gen = torch.Generator(device="cpu").manual_seed(n)
    k, v = (torch.randn(1, 1, hkv, n, d, generator=gen).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(1, 1, hq, d, generator=gen).to(torch.bfloat16)
    k[..., row, 0] = float("inf")
    q[0, 0, :, 0] = -1.0
    q[0, 0, 1, 0] = 1.0        # of the heads, one takes +inf, the others -inf (a probability of zero)
    pos = torch.arange(n, dtype=torch.int32).repeat(1, 1).contiguous()
    shape = B.make_shape(1, 1, hq, hkv, d, n, "bf16")
    ws = B.workspace(shape, n)
    dk, dv, dq, dpos = k.cuda(), v.cuda(), q.cuda(), pos.cuda()
    o, u, s_out = torch.empty_like(dq), torch.zeros(1, n, device="cuda"), torch.zeros(1, 1, n, device="cuda")
    print(f"infinite logit hq={hq} n={n}", flush=True)
    B.kv_attend_score(shape, 0, 1, n, dq, dk, dv, dpos, n - 1, 0.0, 0, B.KV_EMIT_SCORES, o, ws)
    B.kv_evict_finish(shape, B.make_params(0.5, n), 1, n, dk, dv, u, dpos, ws, s_out=s_out)
    torch.cuda.synchronize()
    assert torch.isnan(o[0, 0, 1]).all() and torch.isfinite(o[0, 0, 0].float()).all()
    assert torch.isnan(s_out[0, 0, row - 4 : row + 5]).all()


@pytest.mark.parametrize("what", ["query", "key", "values", "infinities"])
@pytest.mark.parametrize("emit", [0, 1])
def test_attend_nonfinite_inputs_are_not_slow(what, emit):
    """One sequence with a NaN query, key or values, or an infinity in every value column, does not hold up the others'
    call: at most twice the time of finite inputs (20 to 22 us a call; 32 with the infinities; 43 and more, in every case,
    where each such output was summed again by its thread row by row), the least of several runs of each."""
    b, hq, hkv, n, d = 8, 32, 8, 3278, 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    k, v = (torch.randn(1, b, hkv, n, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(1, b, hq, d, generator=gen, device="cuda").to(torch.bfloat16)
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(b, 1).contiguous()
    shape = B.make_shape(b, 1, hq, hkv, d, n, "bf16")
    ws = B.workspace(shape, n)
    o = torch.empty_like(q)

    def best():
        times = []
        for _ in range(8):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(20):
                B.kv_attend_score(shape, 0, 1, n, q, k, v, pos, n - 1, 0.0, 0, emit, o, ws)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1) / 20)
        return min(times)

    print(f"non-finite {what} emit={emit}", flush=True)
    clean = best()
    if what == "query":
        q[0, 0] = float("nan")
    elif what == "key":
        k[0, 0, :, 5] = float("nan")
    elif what == "values":
        v[0, 0] = float("nan")
    else:
        v[0, 0, :, torch.arange(d), torch.arange(d)] = float("inf")
    got = best()
    print(f"{clean * 1e3:.1f} us, non-finite {got * 1e3:.1f}", flush=True)
    assert got <= 2.0 * clean


@pytest.mark.parametrize("hq,hkv,n", [(1, 1, 4096), (16, 1, 4100), (7, 1, 4361), (1, 1, 8192), (3, 1, 16384),
                                      (16, 1, 90000), (3, 1, 331000)])
def test_attend_chunk_counts(hq, hkv, n):
    """The combine's ways of taking the chunks' statistics: up to 16 chunks per slab (16, 17 and 18 here), up to 64
    (32 and 64) and more (256, twice: one per CU for a single slab).  Bounds as in the geometries above (the oracle's own
    tolerance)."""
    d = 128
    gen = torch.Generator(device="cpu").manual_seed(n)
    k = torch.randn(1, 1, hkv, n, d, generator=gen).to(torch.bfloat16)
    v = torch.randn(1, 1, hkv, n, d, generator=gen).to(torch.bfloat16)
    q = torch.randn(1, 1, hq, d, generator=gen).to(torch.bfloat16)
    pos = torch.arange(n, dtype=torch.int32).repeat(1, 1).contiguous()
    shape = B.make_shape(1, 1, hq, hkv, d, n, "bf16")
    ws = B.workspace(shape, n)
    dk, dv, dq, dpos = k.cuda(), v.cuda(), q.cuda(), pos.cuda()
    o, u = torch.empty_like(dq), torch.zeros(1, n, device="cuda")
    s_out = torch.empty(1, 1, n, device="cuda")
    print(f"attend chunks hq={hq} n={n}", flush=True)
    B.kv_attend_score(shape, 0, 1, n, dq, dk, dv, dpos, n - 1, 0.0, 0, B.KV_EMIT_SCORES, o, ws)
    B.kv_evict_finish(shape, B.make_params(0.5, n), 1, n, dk, dv, u, dpos, ws, s_out=s_out)
    torch.cuda.synchronize()
    keys, ql, pr = to_f64(raw_numpy(k)[0, 0], "bf16"), to_f64(raw_numpy(q)[0, 0], "bf16"), np.arange(n)
    ref, scale = attention_output(ql, keys, to_f64(raw_numpy(v)[0, 0], "bf16"), pr, n - 1, 0.0, 0)
    assert_o(o, ref[None, None], scale[None, None], "bf16", "outputs")
    assert_close(s_out.cpu().numpy(), layer_scores(ql, keys, pr, n - 1, 0.0, 0)[None, None], "scores")


@pytest.mark.parametrize("merge,entropy", [(0, False), (1, False), (2, False), (4, False), (8, False), (4, True)],
                         ids=["auto", "merge1", "merge2", "merge4", "merge8", "merge4_entropy"])
def test_fused_scores_equal_separate_pass_bitwise(merge, entropy):
    """With one chunk per slab the attention computes its scores with the scorer's arithmetic in the same
    order, so the fused step and kv_evict_step leave bit-identical utilities and caches; also when the scorer
    adds the group sums of several KV heads in one workgroup (the finish adds the attention's per-KV-head rows
    in the same blocks), and with entropy weighting (computed from those sums)."""
    cfg = LLAMA8B.scaled(batch=8, layers=16, prefill_len=500, budget=400)
    w = Workload(cfg)
    cap = cfg.prefill_len + 1
    st = to_device(w.prefill(capacity=cap))
    st2 = {k: (v.clone() if isinstance(v, torch.Tensor) else v) for k, v in st.items()}
    shape = B.make_shape(cfg.batch, cfg.layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cap, cfg.dtype)
    params = B.make_params(cfg.alpha, cfg.budget, 1, False, "mean", cfg.recency_bias, cfg.recency_window,
                           entropy=entropy, score_merge=merge)
    ws = B.workspace(shape, cap)
    n = st["n"]
    si = to_device(w.step_inputs(1))
    s1 = torch.empty(cfg.layers, cfg.batch, n + 1, device="cuda")
    s2 = torch.empty_like(s1)
    n1 = B.kv_evict_step(shape, params, 1, n, si["new_pos"], si["q"], si["k_new"], si["v_new"], st["k"], st["v"],
                         st["u"], st["pos"], ws, s_out=s1)
    B.kv_append(shape, params, 1, n, si["new_pos"], si["k_new"], si["v_new"], st2["k"], st2["v"], st2["u"],
                st2["pos"])
    o = torch.empty_like(si["q"])
    B.kv_attend_score(shape, 0, cfg.layers, n + 1, si["q"], st2["k"], st2["v"], st2["pos"], si["new_pos"],
                      cfg.recency_bias, cfg.recency_window, 1, o, ws)
    n2 = B.kv_evict_finish(shape, params, 1, n + 1, st2["k"], st2["v"], st2["u"], st2["pos"], ws, s_out=s2)
    torch.cuda.synchronize()
    assert n1 == n2 == cfg.budget
    assert torch.equal(s1, s2)
    assert torch.equal(st["u"], st2["u"]) and torch.equal(st["pos"], st2["pos"])
    assert torch.equal(st["k"], st2["k"]) and torch.equal(st["v"], st2["v"])


def test_attend_without_scores_leaves_other_layers_alone():
    """emit_scores = 0 writes no score: a later finish folds what the emitting calls left (here: layer 0
    emitted, layer 1 not, so layer 1's scores are the previous step's)."""
    cfg = TINY
    w = Workload(cfg)
    st = to_device(w.prefill())
    shape = B.make_shape(cfg.batch, cfg.layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.capacity,
                         cfg.dtype)
    ws = B.workspace(shape, cfg.capacity)
    n = st["n"]
    si = to_device(w.step_inputs(1))
    params = B.make_params(cfg.alpha, n + 5)
    o = torch.empty_like(si["q"])
    B.kv_attend_score(shape, 0, 2, n, si["q"], st["k"], st["v"], st["pos"], 0, 0.0, 0, 1, o, ws)
    s_a = torch.empty(cfg.layers, cfg.batch, n, device="cuda")
    B.kv_evict_finish(shape, params, 1, n, st["k"], st["v"], st["u"].clone(), st["pos"], ws, s_out=s_a)
    q2 = torch.flip(si["q"], dims=[0]).contiguous()
    B.kv_attend_score(shape, 0, 1, n, q2[0], st["k"], st["v"], st["pos"], 0, 0.0, 0, 1, o[0], ws)
    B.kv_attend_score(shape, 1, 1, n, q2[1], st["k"], st["v"], st["pos"], 0, 0.0, 0, 0, o[1], ws)
    s_b = torch.empty_like(s_a)
    B.kv_evict_finish(shape, params, 1, n, st["k"], st["v"], st["u"].clone(), st["pos"], ws, s_out=s_b)
    torch.cuda.synchronize()
    assert torch.equal(s_b[1], s_a[1])          # layer 1 kept the first call's scores
    assert not torch.equal(s_b[0], s_a[0])      # layer 0 was re-scored with another query
