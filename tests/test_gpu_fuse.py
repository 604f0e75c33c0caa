"""GPU parity of Stage-1 fusion (voxzip_fuse_spans) against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import synth
from vzt import RTOL, GpuCache, bf16_ulp, check_close, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu


def _run(k_in, v_in, off, dtype, cap, anchor=None, Hq=None):
    L, H, T, d = k_in.shape
    g = GpuCache(L, Hq or H, H, d, cap, dtype)
    sentinel = 7.0
    g.k.fill_(sentinel)
    g.v.fill_(sentinel)
    g.score.fill_(-1.0)
    g.pos.fill_(-5)
    ak = av = None
    if anchor is not None:
        ak, av = to_dev(anchor[0]), to_dev(anchor[1])
    g.fuse(to_dev(k_in), to_dev(v_in), to_dev(off), ak, av)
    k, v, s, p = g.snapshot()
    return g, k, v, s, p, sentinel


def _verify(k_in, v_in, off, dtype, k, v, s, p, sentinel, anchor=None):
    n = len(off) - 1
    for name, x_in, got, a in (("K", k_in, k, None if anchor is None else anchor[0]),
                               ("V", v_in, v, None if anchor is None else anchor[1])):
        ref = oracle.fuse(x_in, off, dtype, anchor=a)
        g = widen(got[:, :, :n], dtype)
        check_close(g, ref, RTOL[dtype], f"fused {name}")
        if dtype == synth.DT_BF16:  # one rounding of a float32 result: within one bf16 ulp
            assert np.all(np.abs(g - ref) <= bf16_ulp(ref) + 1e-6 * np.abs(ref))
        if anchor is None:  # length-1 spans are copies, bit for bit
            one = np.nonzero(np.diff(off) == 1)[0]
            assert np.array_equal(got[:, :, one], x_in[:, :, off[one]])
        assert np.all(widen(got[:, :, n:], dtype) == sentinel)  # slots past n_spans untouched
    assert np.array_equal(p[:, :n], np.broadcast_to(np.arange(n, dtype=np.int32), (p.shape[0], n)))
    assert np.all(s[:, :n] == 0.0) and np.all(p[:, n:] == -5) and np.all(s[:, n:] == -1.0)


@pytest.mark.parametrize("name", ["tiny", "layer"])
def test_fuse_workload_shapes(name):
    w = synth.workload(name)
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    k_in, v_in = synth.prefill_kv(w, "k"), synth.prefill_kv(w, "v")
    n = len(off) - 1
    _, k, v, s, p, sen = _run(k_in, v_in, off, w.dtype, n + 40)
    _verify(k_in, v_in, off, w.dtype, k, v, s, p, sen)


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 64), (synth.DT_BF16, 128), (synth.DT_F32, 64),
                                     (synth.DT_F32, 128)])
def test_fuse_ragged_spans_with_anchor(dtype, d):
    L, H = 3, 2
    key = synth.stream_key(11, "fuse-ragged", dtype, d)
    lens = synth.uniform_int(key, 0, 97, 1, 41)          # tails of the 4-row unroll, long spans
    lens[::7] = 1
    off = synth.offsets_from_lengths(lens)
    T, n = int(off[-1]), len(lens)
    mk = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape) * np.float32(2.5), dtype)
    k_in, v_in = mk("k", (L, H, T, d)), mk("v", (L, H, T, d))
    anchor = (mk("ak", (L, H, n, d)), mk("av", (L, H, n, d)))
    _, k, v, s, p, sen = _run(k_in, v_in, off, dtype, n + 3, anchor=anchor)
    _verify(k_in, v_in, off, dtype, k, v, s, p, sen, anchor=anchor)
    _, k, v, s, p, sen = _run(k_in, v_in, off, dtype, n)      # cap exactly n_spans
    _verify(k_in, v_in, off, dtype, k, v, s, p, sen)


def test_fuse_single_span_and_all_identity():
    dtype, d = synth.DT_BF16, 128
    x = synth.as_storage(synth.normal_f32(synth.stream_key(5, "one"), 2 * 1 * 300 * d).reshape(2, 1, 300, d), dtype)
    y = synth.as_storage(synth.normal_f32(synth.stream_key(6, "one"), 2 * 1 * 300 * d).reshape(2, 1, 300, d), dtype)
    off = np.array([0, 300], dtype=np.int32)                 # one span over everything
    _, k, v, s, p, sen = _run(x, y, off, dtype, 4)
    _verify(x, y, off, dtype, k, v, s, p, sen)
    off = np.arange(301, dtype=np.int32)                     # every token its own span
    _, k, v, s, p, sen = _run(x, y, off, dtype, 300)
    assert np.array_equal(k, x) and np.array_equal(v, y)


def test_fuse_full_size_sampled_layers():
    """32k-token, 48-layer cache fused in one launch; layers 0, 23, 47 checked in full."""
    w = synth.workload("long32k")
    off = synth.offsets_from_lengths(synth.span_lengths(w))
    n = len(off) - 1
    k_in, v_in = synth.prefill_kv(w, "k"), synth.prefill_kv(w, "v")
    g, k, v, s, p, sen = _run(k_in, v_in, off, w.dtype, n + 300, Hq=w.n_q_heads)
    for l in (0, 23, 47):
        _verify(k_in[l:l + 1], v_in[l:l + 1], off, w.dtype, k[l:l + 1], v[l:l + 1], s[l:l + 1], p[l:l + 1], sen)
    assert np.all(p[:, :n] == np.arange(n)) and np.all(s[:, :n] == 0)


def test_fuse_with_offsets_from_the_span_builder():
    """End to end Stage 1: ASR segments -> voxzip_build_span_offsets (host) ->
    voxzip_fuse_spans (GPU), against the oracle's fusion of the oracle's offsets."""
    import paper_2608_08569_amd as vz
    key = synth.stream_key(5, "stage1-e2e")
    r = synth.uniform01(key, 0, 256)
    t_total, L_a, n = 120000, 1500, 30
    starts = np.sort((r[:n] * (t_total - 5000)).astype(np.int64))
    ends = starts + 800 + (r[n:2 * n] * 4000).astype(np.int64)
    conf = (0.1 + 0.9 * r[2 * n:3 * n]).astype(np.float32)
    tl = 1 + (r[3 * n:4 * n] * 12).astype(np.int32)
    off = vz.voxzip_build_span_offsets(starts, ends, conf, tl, t_total, L_a)
    assert np.array_equal(off, oracle.build_offsets(starts, ends, conf, tl, t_total, L_a))
    dtype, L, H, d = synth.DT_BF16, 2, 4, 128
    x = synth.as_storage(synth.normal_f32(synth.stream_key(key, "k"), L * H * L_a * d).reshape(L, H, L_a, d), dtype)
    y = synth.as_storage(synth.normal_f32(synth.stream_key(key, "v"), L * H * L_a * d).reshape(L, H, L_a, d), dtype)
    _, k, v, s, p, sen = _run(x, y, off, dtype, len(off) + 7)
    _verify(x, y, off, dtype, k, v, s, p, sen)


def _fuse_wide(x_k, x_v, off, dtype, cap, anchor_k=None, anchor_v=None):
    """Direct call for row sizes the decode path does not take (no workspaces)."""
    import torch
    import paper_2608_08569_amd as vz
    L, H, T, d = x_k.shape
    tdt = torch.float32 if dtype == synth.DT_F32 else torch.bfloat16
    sentinel = 7.0
    k_out = torch.full((L, H, cap, d), sentinel, dtype=tdt, device="cuda")
    v_out = None if x_v is None else torch.full((L, H, cap, d), sentinel, dtype=tdt, device="cuda")
    score = torch.full((L, cap), -1.0, dtype=torch.float32, device="cuda")
    pos = torch.full((L, cap), -5, dtype=torch.int32, device="cuda")
    dev = lambda a: None if a is None else to_dev(a)
    vz.voxzip_fuse_spans(to_dev(x_k), dev(x_v), to_dev(off), k_out, v_out, score, pos,
                         anchor_k=dev(anchor_k), anchor_v=dev(anchor_v))
    torch.cuda.synchronize()
    return from_dev(k_out), None if v_out is None else from_dev(v_out), from_dev(score), from_dev(pos), sentinel


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 256), (synth.DT_BF16, 1000), (synth.DT_BF16, 3584),
                                     (synth.DT_F32, 260), (synth.DT_F32, 2048)])
@pytest.mark.parametrize("with_anchor", [False, True])
def test_fuse_wide_rows(dtype, d, with_anchor):
    """Row sizes other than 64 and 128 (the wide-row kernel): K and V, span
    lengths 1..13 (tails of the 4-row unroll), columns past one block of
    threads (3584 bf16 = 448 vectors), against the oracle."""
    L, H = 2, 2
    key = synth.stream_key(17, "fuse-wide", dtype, d)
    lens = synth.uniform_int(key, 0, 45, 1, 14)
    lens[::5] = 1
    off = synth.offsets_from_lengths(lens)
    T, n = int(off[-1]), len(lens)
    mk = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape) * np.float32(1.5), dtype)
    k_in, v_in = mk("k", (L, H, T, d)), mk("v", (L, H, T, d))
    anchor = (mk("ak", (L, H, n, d)), mk("av", (L, H, n, d))) if with_anchor else None
    k, v, s, p, sen = _fuse_wide(k_in, v_in, off, dtype, n + 5, *(anchor or (None, None)))
    _verify(k_in, v_in, off, dtype, k, v, s, p, sen, anchor=anchor)


def test_embedding_space_stage1():
    """Sec. 3.2.1 in its literal, embedding-space form: ASR segments (with
    low-confidence and overlapping ones) give the span offsets through the
    library's span builder, the audio-token embeddings [L_a][d_model] are
    pooled per span and the text-token embeddings are added as anchors (zero
    rows for background tokens, which the kernel then copies bit for bit);
    one tensor only (v_in = v_out = NULL), d_model = 3584, bf16."""
    import paper_2608_08569_amd as vz
    dtype, d_model, L_a, t_total = synth.DT_BF16, 3584, 1500, 30000
    key = synth.stream_key(23, "embedding-stage1")
    n_seg = 14
    u = synth.uniform01(key, 0, 4 * n_seg)
    ts = np.sort((u[:n_seg] * t_total * 0.95).astype(np.int64))
    te = ts + (400 + u[n_seg:2 * n_seg] * 2600).astype(np.int64)
    conf = (0.1 + 0.9 * u[2 * n_seg:3 * n_seg]).astype(np.float32)
    tl = (1 + u[3 * n_seg:4 * n_seg] * 25).astype(np.int32)
    off = vz.voxzip_build_span_offsets(ts, te, conf, tl, t_total, L_a, 0.3)
    assert np.array_equal(off, oracle.build_offsets(ts, te, conf, tl, t_total, L_a, 0.3))
    n = len(off) - 1
    lens = np.diff(off)
    assert 1 < n < L_a and lens.max() > 1
    emb = synth.as_storage(synth.normal_f32(synth.stream_key(key, "audio"), L_a * d_model).reshape(
        1, 1, L_a, d_model), dtype)
    text = synth.as_storage(synth.normal_f32(synth.stream_key(key, "text"), n * d_model).reshape(
        1, 1, n, d_model) * np.float32(0.5), dtype)
    text[:, :, lens == 1] = 0           # background (and one-token) spans carry no text anchor
    k, v, s, p, sen = _fuse_wide(emb, None, off, dtype, n + 3, anchor_k=text)
    assert v is None
    ref = oracle.fuse(emb, off, dtype, anchor=text)
    got = widen(k[:, :, :n], dtype)
    check_close(got, ref, RTOL[dtype], "fused embeddings")
    assert np.all(np.abs(got - ref) <= bf16_ulp(ref) + 1e-6 * np.abs(ref))
    one = np.nonzero(lens == 1)[0]
    assert np.array_equal(k[:, :, one], emb[:, :, off[one]])        # copies, bit for bit
    assert np.all(widen(k[:, :, n:], dtype) == sen)
    assert np.array_equal(p[0, :n], np.arange(n, dtype=np.int32)) and np.all(s[0, :n] == 0)


def test_fuse_ragged_wide_rows_k_only():
    """The ragged twin with wide rows and k alone: three sequences of
    embeddings (d_model = 1024, bf16) fused into one packed output."""
    import torch
    import paper_2608_08569_amd as vz
    dtype, d, L, H = synth.DT_BF16, 1024, 1, 1
    key = synth.stream_key(29, "fuse-ragged-wide")
    T_in = [37, 1, 90]
    lens = [synth.uniform_int(synth.stream_key(key, "lens", i), 0, t, 1, 6) for i, t in enumerate(T_in)]
    offs = []
    for t, ln in zip(T_in, lens):
        o = synth.offsets_from_lengths(ln)
        o = o[o <= t]
        if o[-1] != t:
            o = np.append(o, t)
        offs.append(o.astype(np.int32))
    n_sp = [len(o) - 1 for o in offs]
    in_base = np.concatenate([[0], np.cumsum(T_in)[:-1]]).astype(np.int64)
    off_base = np.concatenate([[0], np.cumsum([len(o) for o in offs])[:-1]]).astype(np.int64)
    caps = [n + 2 for n in n_sp]
    seq_base = np.concatenate([[0], np.cumsum(caps)[:-1]]).astype(np.int64)
    total_in, total = int(sum(T_in)), int(sum(caps))
    x = synth.as_storage(synth.normal_f32(synth.stream_key(key, "x"), total_in * d).reshape(L, H, total_in, d), dtype)
    anc = synth.as_storage(synth.normal_f32(synth.stream_key(key, "a"), total * d).reshape(L, H, total, d), dtype)
    dev = lambda a, dt: torch.tensor(np.asarray(a), dtype=dt, device="cuda")
    k_out = torch.zeros(L, H, total, d, dtype=torch.bfloat16, device="cuda")
    score = torch.zeros(L, total, dtype=torch.float32, device="cuda")
    pos = torch.zeros(L, total, dtype=torch.int32, device="cuda")
    status = torch.full((3,), 99, dtype=torch.int32, device="cuda")
    vz.voxzip_fuse_spans_ragged(to_dev(x), None, dev(in_base, torch.int64), dev(T_in, torch.int32),
                                to_dev(np.concatenate(offs)), dev(off_base, torch.int64), dev(n_sp, torch.int32),
                                max(n_sp), k_out, None, score, pos, dev(seq_base, torch.int64),
                                dev(caps, torch.int32), status=status, anchor_k=to_dev(anc))
    assert np.all(from_dev(status) == 0)
    k = from_dev(k_out)
    for i in range(3):
        n, b, ib = n_sp[i], int(seq_base[i]), int(in_base[i])
        ref = oracle.fuse(x[:, :, ib:ib + T_in[i]], offs[i], dtype, anchor=anc[:, :, b:b + n])
        check_close(widen(k[:, :, b:b + n], dtype), ref, RTOL[dtype], f"sequence {i}")


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 8), (synth.DT_BF16, 520), (synth.DT_BF16, 2048),
                                     (synth.DT_BF16, 2056), (synth.DT_BF16, 4096), (synth.DT_BF16, 4104),
                                     (synth.DT_F32, 1024), (synth.DT_F32, 1028), (synth.DT_F32, 2052)])
def test_fuse_wide_rows_at_the_column_rounds(dtype, d):
    """1, 65, 256, 257, 512 and 513 vectors per row: one column per thread, two
    at a time, and a second column or round that only some threads have; one
    tensor, rows that end in infinities behind the spans that must not see
    them."""
    key = synth.stream_key(19, "fuse-rounds", dtype, d)
    lens = np.array([1, 2, 3, 4, 5, 7, 8, 9, 1, 6], dtype=np.int64)
    off = synth.offsets_from_lengths(lens)
    T, n = int(off[-1]), len(lens)
    x = synth.as_storage(synth.normal_f32(key, T * d).reshape(1, 1, T, d), dtype)
    x[0, 0, off[3] - 1] = np.float32(np.inf) if dtype == synth.DT_F32 else 0x7F80  # last row of a 3-row span
    k, _, s, p, sen = _fuse_wide(x, None, off, dtype, n + 2)
    inf = synth.storage_to_f64(k, dtype)[0, 0, :n]
    assert np.all(np.isposinf(inf[2])) and np.all(np.isfinite(np.delete(inf, 2, axis=0)))
    ref = oracle.fuse(x, off, dtype)[0, 0]
    for j in range(n):
        if j != 2:
            assert np.all(np.abs(inf[j] - ref[j]) <= RTOL[dtype] * (np.abs(ref[j]) + np.sqrt(np.mean(ref[j] ** 2)))), j


@pytest.mark.parametrize("dtype,d", [(synth.DT_BF16, 2552), (synth.DT_BF16, 2560), (synth.DT_BF16, 2816),
                                     (synth.DT_BF16, 3584), (synth.DT_BF16, 6144), (synth.DT_BF16, 8192),
                                     (synth.DT_F32, 1276), (synth.DT_F32, 1280), (synth.DT_F32, 4096)])
def test_fuse_wide_rows_one_and_two_columns_per_thread(dtype, d):
    """319, 320, 352 (a wave with a second column in half its lanes), 448, 768
    and 1024 vectors per row: spans of mean length 4 (from 320 vectors on two
    columns per thread) and the same spans with single rows behind them, which
    bring the mean below 1.2 (one column in bfloat16), give the same bits."""
    lens = np.array([1, 2, 3, 4, 5, 7, 8, 9, 1, 6], dtype=np.int64)
    n, tail = len(lens), 400
    key = synth.stream_key(23, "fuse-columns", dtype, d)
    T = int(lens.sum()) + tail
    x = synth.as_storage(synth.normal_f32(key, T * d).reshape(1, 1, T, d), dtype)
    short = x[:, :, : T - tail].copy()
    _, k, v, s, p, sen = _run(short, short, synth.offsets_from_lengths(lens), dtype, n + 1)
    _verify(short, short, synth.offsets_from_lengths(lens), dtype, k, v, s, p, sen)
    off = synth.offsets_from_lengths(np.concatenate([lens, np.ones(tail, dtype=np.int64)]))
    _, k1, v1, s, p, sen = _run(x, x, off, dtype, n + tail + 1)
    assert np.array_equal(k1[:, :, :n], k[:, :, :n]) and np.array_equal(v1[:, :, :n], v[:, :, :n])
    assert np.array_equal(k1[:, :, n: n + tail], x[:, :, T - tail:])
