"""GPU parity of the decode step (voxzip_decode_attend_score) and of the whole
path with eviction, state-synced against the fp64 oracle: before every step
the oracle starts from the GPU's own state, and every eviction selects on the
oracle's scores rounded to float32 (so a near tie cannot flip the kept set)."""
import numpy as np
import pytest

import oracle
import synth
from vzt import RTOL, GpuCache, check_close, check_rel, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu


def synced_step(g, q, kn, vn, gamma, layers=None):
    """One GPU step checked against the oracle on ``layers`` (all by default).
    Only those layers are copied to the host; returns the oracle's scores and
    the GPU's state after the step, both for those layers."""
    sel = list(range(g.L)) if layers is None else list(layers)
    K, V, S, P = g.snapshot(sel)
    n0 = g.len
    ref_o, ref_s, ref_p, _ = oracle.decode_step(q[sel], kn[sel], vn[sel], K, V, S.astype(np.float64), P, n0,
                                                g.next_pos, gamma, g.dtype)
    g.step(to_dev(q), to_dev(kn), to_dev(vn), gamma)
    K2, V2, S2, P2 = g.snapshot(sel)
    o = from_dev(g.out)[sel]
    rt = RTOL[g.dtype]
    check_close(widen(o, g.dtype), ref_o, rt, "attention output")
    check_rel(S2[:, : n0 + 1], ref_s, rt, "decayed score")
    assert np.array_equal(P2[:, : n0 + 1], ref_p)
    assert np.array_equal(K2[:, :, n0], kn[sel]) and np.array_equal(V2[:, :, n0], vn[sel])   # Eq. 1 append
    assert np.array_equal(K2[:, :, :n0], K[:, :, :n0]) and np.array_equal(V2[:, :, :n0], V[:, :, :n0])
    return ref_s, (K2, V2, S2, P2)


def synced_evict(g, ref_s, state, budget, layers=None):
    """Evict on the oracle's float32 scores (written into the GPU state for the
    checked layers; the other layers keep the GPU's own); on the checked
    layers the kept set is bit-exact and the rows position-keyed."""
    t = __import__("torch")
    sel = list(range(g.L)) if layers is None else list(layers)
    K2, V2, S2, P2 = state
    T = g.len
    sc32 = S2.copy()
    sc32[:, :T] = ref_s.astype(np.float32)
    idx = t.tensor(sel, dtype=t.long, device="cuda")
    g.score.index_copy_(0, idx, t.from_numpy(sc32).cuda())
    keep, nl = oracle.evict_select(sc32.astype(np.float64), P2, T, budget, 4, -1, g.next_pos)
    kept = t.full((g.L, budget), -1, dtype=t.int32, device="cuda")
    new_len = g.evict(budget, kept=kept)
    assert new_len == nl == min(T, budget)
    K3, V3, S3, P3 = g.snapshot(sel)
    kept = from_dev(kept)[sel]
    for i in range(len(sel)):
        ref_pos = P2[i][keep[i]]
        assert np.array_equal(kept[i, :nl], ref_pos), "kept position set"
        order = np.argsort(P3[i, :nl], kind="stable")
        assert np.array_equal(P3[i, :nl][order], ref_pos)
        assert np.array_equal(K3[i][:, :nl][:, order], K2[i][:, keep[i]])
        assert np.array_equal(V3[i][:, :nl][:, order], V2[i][:, keep[i]])
        assert np.array_equal(S3[i, :nl][order], sc32[i, keep[i]])
    return T - nl


def _run_workload(w, g, steps, start_step=0, layers=None, budget=None, interval=1):
    """Steps (with the eviction rule of Sec. 3.2.2: after the score update,
    every `interval` steps, when len > B) state-synced against the oracle;
    returns the number of evictions and of rows they removed."""
    budget = w.budget if budget is None else budget
    bias = synth.q_bias(w) if w.q_bias else None
    n_ev = rows = 0
    for t in range(start_step, start_step + steps):
        q, kn, vn = synth.decode_inputs(w, t, bias=bias)
        ref_s, state = synced_step(g, q, kn, vn, w.gamma, layers)
        if (t + 1) % interval == 0 and g.len > budget:
            rows += synced_evict(g, ref_s, state, budget, layers)
            n_ev += 1
    return n_ev, rows


def test_tiny_fused_no_eviction_needed():
    """Tiny fp32 case: 64 fused spans + 32 steps stay within B = 128 (no eviction)."""
    w = synth.workload("tiny")
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    g = GpuCache(w.n_layers, w.n_q_heads, w.kv_heads, w.d, 200, w.dtype)
    g.fuse(to_dev(synth.prefill_kv(w, "k")), to_dev(synth.prefill_kv(w, "v")), to_dev(off))
    _run_workload(w, g, w.steps)
    assert g.len == 64 + 32


def test_tiny_unfused_evicts_every_step():
    """Stage 2 alone on 512 unfused tokens with B = 128 (M = 25, N = 99): evicts from step one."""
    w = synth.workload("tiny")
    off = np.arange(513, dtype=np.int32)
    g = GpuCache(w.n_layers, w.n_q_heads, w.kv_heads, w.d, 520, w.dtype)
    g.fuse(to_dev(synth.prefill_kv(w, "k")), to_dev(synth.prefill_kv(w, "v")), to_dev(off))
    _run_workload(w, g, w.steps)
    assert g.len == 128


def test_layer_bf16_real_head_shape():
    """One layer, 32Q/4KV, d = 128, bf16: ~1280 fused tokens, B = 1024, 128 steps."""
    w = synth.workload("layer")
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    n = len(off) - 1
    g = GpuCache(w.n_layers, w.n_q_heads, w.kv_heads, w.d, n + w.steps + 1, w.dtype)
    g.fuse(to_dev(synth.prefill_kv(w, "k")), to_dev(synth.prefill_kv(w, "v")), to_dev(off))
    _run_workload(w, g, w.steps)
    assert g.len == w.budget


@pytest.mark.parametrize("dtype,d,Hq,Hkv", [(synth.DT_BF16, 128, 64, 4), (synth.DT_BF16, 64, 6, 2),
                                            (synth.DT_F32, 128, 8, 8), (synth.DT_F32, 64, 16, 1),
                                            (synth.DT_BF16, 128, 32, 4), (synth.DT_BF16, 128, 16, 1),
                                            (synth.DT_BF16, 128, 6, 2), (synth.DT_BF16, 128, 64, 8)])
@pytest.mark.parametrize("length", [0, 1, 15, 255, 256, 257, 1000, 5000])
def test_shapes_and_ragged_lengths(dtype, d, Hq, Hkv, length):
    L, cap = 2, length + 3
    key = synth.stream_key(21, dtype, d, Hq, Hkv, length)
    k, v, s, p = synth.random_state(21, L, Hkv, d, cap, length, dtype, next_pos=length + 9)
    g = GpuCache(L, Hq, Hkv, d, cap, dtype)
    g.load(k, v, s, p, length, length + 9)
    for t in range(2):
        mk = lambda tag, shape: synth.as_storage(
            synth.normal_f32(synth.stream_key(key, tag, t), int(np.prod(shape))).reshape(shape) * np.float32(1.7),
            dtype)
        synced_step(g, mk("q", (L, Hq, d)), mk("k", (L, Hkv, d)), mk("v", (L, Hkv, d)), 0.95)


def test_gamma_edges_and_explicit_scale():
    dtype, L, Hq, Hkv, d, length = synth.DT_BF16, 1, 32, 4, 128, 700
    k, v, s, p = synth.random_state(3, L, Hkv, d, length + 2, length, dtype)
    for gamma in (0.0, 1.0):
        g = GpuCache(L, Hq, Hkv, d, length + 2, dtype)
        g.load(k, v, s, p, length, length)
        q, kn, vn = (synth.as_storage(synth.normal_f32(synth.stream_key(3, x), n).reshape(sh), dtype)
                     for x, n, sh in (("q", L * Hq * d, (L, Hq, d)), ("k", L * Hkv * d, (L, Hkv, d)),
                                      ("v", L * Hkv * d, (L, Hkv, d))))
        synced_step(g, q, kn, vn, gamma)
        # total mass: gamma * previous + Hq
        S = from_dev(g.score)[0, : length + 1].astype(np.float64)
        expect = gamma * s[0, :length].astype(np.float64).sum() + Hq
        assert abs(S.sum() - expect) <= 1e-4 * expect


@pytest.mark.parametrize("length,cap", [(16383, 16384), (16383, 16385), (16384, 16386)])
def test_single_and_ragged_calls_agree_on_long_sequences(length, cap):
    """T = 16,384 and 16,385 keys (128 and 129 chunks) in planes of 128 chunks
    (one finishing launch) and of 129 (two): the single-sequence call against
    the oracle and bit for bit against the ragged call on the same data."""
    import torch
    import paper_2608_08569_amd as vz
    dtype, L, Hq, Hkv, d = synth.DT_BF16, 1, 32, 4, 128
    k, v, s, p = synth.random_state(31, L, Hkv, d, cap, length, dtype, next_pos=length + 5)
    w = synth.workload("layer")
    q, kn, vn = synth.decode_inputs(w, 1)
    g = GpuCache(L, Hq, Hkv, d, cap, dtype)
    g.load(k, v, s, p, length, length + 5)
    synced_step(g, q, kn, vn, 0.95)
    K1, V1, S1, P1 = g.snapshot()
    out1 = from_dev(g.out)
    r = GpuCache(L, Hq, Hkv, d, cap, dtype)
    r.load(k, v, s, p, length, length + 5)
    dev = lambda a, dt: torch.tensor(a, dtype=dt, device="cuda")
    ws = vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, d, cap, 1)
    out = torch.zeros(1, L, Hq, d, dtype=torch.bfloat16, device="cuda")
    vz.voxzip_decode_attend_score_ragged(to_dev(q[None]), to_dev(kn[None]), to_dev(vn[None]), r.k, r.v, r.score,
                                         r.pos, out, dev([0], torch.int64), dev([cap], torch.int32),
                                         dev([length], torch.int32), dev([length + 5], torch.int32), 0.95,
                                         workspace=ws)
    K2, V2, S2, P2 = r.snapshot()
    assert np.array_equal(from_dev(out)[0], out1)
    assert np.array_equal(S2, S1) and np.array_equal(P2, P1) and np.array_equal(K2, K1)


def test_many_chunks_per_layer():
    """65,535 resident keys: 512 chunks of 128 keys per layer on the fused path."""
    dtype, L, Hq, Hkv, d, length = synth.DT_BF16, 1, 32, 4, 128, 65535
    k, v, s, p = synth.random_state(12, L, Hkv, d, length + 1, length, dtype)
    g = GpuCache(L, Hq, Hkv, d, length + 1, dtype)
    g.load(k, v, s, p, length, length)
    w = synth.workload("layer")
    q, kn, vn = synth.decode_inputs(w, 3)
    synced_step(g, q, kn, vn, 0.95)


def test_small_and_large_chunked_grids_agree():
    """A chunked call over 20 layers (32 chunks each: 2560 workgroups) and
    one-layer calls of the same data (128 workgroups) give the same bits; the
    first layer also against the oracle."""
    dtype, L, Hq, Hkv, d, length = synth.DT_BF16, 20, 32, 4, 128, 4000
    k, v, s, p = synth.random_state(14, L, Hkv, d, length + 2, length, dtype, next_pos=length + 9)
    key = synth.stream_key(14, "grids")
    mk = lambda tag, shape: synth.as_storage(synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape)))
                                             .reshape(shape), dtype)
    q, kn, vn = mk("q", (L, Hq, d)), mk("k", (L, Hkv, d)), mk("v", (L, Hkv, d))
    g = GpuCache(L, Hq, Hkv, d, length + 2, dtype)
    g.load(k, v, s, p, length, length + 9)
    ref_s, _ = synced_step(g, q, kn, vn, 0.95, layers=[0])
    out_all = from_dev(g.out)
    K_all, V_all, S_all, P_all = g.snapshot()
    for l in range(L):
        h = GpuCache(1, Hq, Hkv, d, length + 2, dtype)
        h.load(k[l:l + 1], v[l:l + 1], s[l:l + 1], p[l:l + 1], length, length + 9)
        h.step(to_dev(q[l:l + 1]), to_dev(kn[l:l + 1]), to_dev(vn[l:l + 1]), 0.95)
        Kh, Vh, Sh, Ph = h.snapshot()
        assert np.array_equal(from_dev(h.out)[0], out_all[l]), f"layer {l} output"
        assert np.array_equal(Sh[0], S_all[l]) and np.array_equal(Ph[0], P_all[l])
        assert np.array_equal(Kh[0], K_all[l]) and np.array_equal(Vh[0], V_all[l])


def test_deterministic_bits():
    """Two identical steps from the same state give identical bits."""
    w = synth.workload("layer")
    k, v, s, p = synth.random_state(8, 1, 4, 128, 2100, 2048, synth.DT_BF16, next_pos=3000)
    q, kn, vn = synth.decode_inputs(w, 0)
    outs = []
    for _ in range(2):
        g = GpuCache(1, 32, 4, 128, 2100, synth.DT_BF16)
        g.load(k, v, s, p, 2048, 3000)
        g.step(to_dev(q), to_dev(kn), to_dev(vn), 0.95)
        outs.append((from_dev(g.out), *g.snapshot()))
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def test_long32k_full_size_sampled_layers():
    """The 48-layer 32k-token workload at full size: fuse (8,150 spans), then
    decode steps until the cache has crossed the budget B = 8192 and been
    evicted for several steps (one row per layer and step, T = 8193: the
    steady state that bench.py times); layers 0, 23 and 47 are checked against
    the oracle at every step and every eviction."""
    w = synth.workload("long32k")
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    n = len(off) - 1
    assert n < w.budget
    steps = w.budget - n + 8          # the last 8 steps each evict one row
    cap = max(n, w.budget) + 32
    g = GpuCache(w.n_layers, w.n_q_heads, w.kv_heads, w.d, cap, w.dtype)
    g.fuse(to_dev(synth.prefill_kv(w, "k")), to_dev(synth.prefill_kv(w, "v")), to_dev(off))
    n_ev, rows = _run_workload(w, g, steps, layers=[0, 23, 47])
    assert (n_ev, rows) == (8, 8)
    assert g.len == w.budget


def test_aggr64k_full_size_sampled_layers():
    """The 48-layer 64k-token workload at full size (20x compression, queries
    biased towards ~5% of the keys): 65,536 tokens fused into ~13.1k spans; the
    first eviction removes ~9.8k rows per layer (radix select, grid-wide
    compaction), the later ones one row; layers 0 and 47 are checked against
    the oracle every step."""
    w = synth.workload("aggr64k")
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    n = len(off) - 1
    cap = max(n, w.budget) + 32
    g = GpuCache(w.n_layers, w.n_q_heads, w.kv_heads, w.d, cap, w.dtype)
    g.fuse(to_dev(synth.prefill_kv(w, "k")), to_dev(synth.prefill_kv(w, "v")), to_dev(off))
    _run_workload(w, g, 4, layers=[0, 47])
    assert g.len == w.budget


def test_batch16_per_sequence_calls():
    """The batched workload, one call sequence per sequence (16 caches of 2k-32k
    audio tokens, budget len/4, eviction every 16 steps), on the first 2 of the
    48 layers at the real head shape; every sequence is checked against the
    oracle every step for 32 steps (two evictions of ~16 rows each)."""
    layers = range(2)
    for i, w in enumerate(synth.batch_workloads()):
        off = synth.offsets_from_lengths(synth.span_lengths(w, seq=i))
        n = len(off) - 1
        g = GpuCache(len(layers), w.n_q_heads, w.kv_heads, w.d, max(n, w.budget) + 17, w.dtype)
        g.fuse(to_dev(synth.prefill_kv(w, "k", seq=i, layers=layers)),
               to_dev(synth.prefill_kv(w, "v", seq=i, layers=layers)), to_dev(off))
        for t in range(32):
            q, kn, vn = synth.decode_inputs(w, t, seq=i)
            ref_s, state = synced_step(g, q[:2], kn[:2], vn[:2], w.gamma)
            if (t + 1) % w.interval == 0 and g.len > w.budget:
                synced_evict(g, ref_s, state, w.budget)
        assert g.len == min(n + 32, w.budget)


def test_concurrent_calls_on_separate_streams():
    """Eight sequences decode at the same time, each on its own stream and
    workspace, with no synchronisation between the calls: no kernel of the
    library waits for another workgroup, so concurrent kernels cannot starve
    each other.  Every sequence is checked against the oracle after 3 steps."""
    import torch
    L, Hq, Hkv, d, dtype = 4, 32, 4, 128, synth.DT_BF16
    lens = [6000, 3000, 9000, 257, 8000, 1200, 7000, 4500]
    caches, refs, streams = [], [], []
    for i, n in enumerate(lens):
        k, v, s, p = synth.random_state(60 + i, L, Hkv, d, n + 4, n, dtype, next_pos=n + 7)
        g = GpuCache(L, Hq, Hkv, d, n + 4, dtype)
        g.load(k, v, s, p, n, n + 7)
        caches.append(g)
        refs.append([k, v, s.astype(np.float64), p])
        streams.append(torch.cuda.Stream())
    torch.cuda.synchronize()
    steps = []
    for t in range(3):
        key = synth.stream_key(61, "concurrent", t)
        mk = lambda tag, shape: synth.as_storage(
            synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape), dtype)
        steps.append([(mk(f"q{i}", (L, Hq, d)), mk(f"k{i}", (L, Hkv, d)), mk(f"v{i}", (L, Hkv, d)))
                      for i in range(len(lens))])
    dev_steps = [[tuple(to_dev(x) for x in trip) for trip in st] for st in steps]
    torch.cuda.synchronize()
    import paper_2608_08569_amd as vz
    for t in range(3):
        for i, g in enumerate(caches):  # all sequences' calls in flight together
            q, kn, vn = dev_steps[t][i]
            vz.voxzip_decode_attend_score(q, kn, vn, g.k, g.v, g.score, g.pos, g.out, g.len, g.next_pos, 0.95,
                                          workspace=g.ws_dec, stream=streams[i])
            g.len += 1
            g.next_pos += 1
    torch.cuda.synchronize()
    for i, g in enumerate(caches):
        k, v, s, p = refs[i]
        n = lens[i]
        K, V = k.copy(), v.copy()
        S, P = s.copy(), p.copy()
        for t in range(3):  # the oracle steps from its own state (no eviction: lengths only grow)
            q, kn, vn = steps[t][i]
            ro, rs, rp, _ = oracle.decode_step(q, kn, vn, K, V, S, P, n + t, n + 7 + t, 0.95, dtype)
            K[:, :, n + t], V[:, :, n + t] = kn, vn
            S[:, : n + t + 1] = rs
            P[:, : n + t + 1] = rp
        check_close(widen(from_dev(g.out), dtype), ro, RTOL[dtype], f"sequence {i} output")
        check_rel(from_dev(g.score)[:, : n + 3], S[:, : n + 3], RTOL[dtype], f"sequence {i} score")
        assert np.array_equal(from_dev(g.pos)[:, : n + 3], P[:, : n + 3])
