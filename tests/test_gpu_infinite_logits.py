"""Decode steps over keys whose logits are minus infinity: they get probability
0, whether they are a few keys of a wave's 32, all of them, a lone last key, or
a whole 128-key chunk, as long as the sequence has a finite logit."""
import numpy as np
import pytest

import oracle
import synth
from vzt import RTOL, GpuCache, check_close, check_rel, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu

MINUS_INF = {synth.DT_F32: np.float32(-np.inf), synth.DT_BF16: np.uint16(0xFF80)}
ONE = {synth.DT_F32: np.float32(1), synth.DT_BF16: np.uint16(0x3F80)}
LENGTHS = [  # resident keys before the step, the keys [a, b) without a finite logit (b = length + 1: the new one too)
    (96, 96, 97),        # the new key, alone in its wave
    (200, 37, 60),       # part of a wave's 32 keys
    (200, 32, 64),       # all of them
    (300, 256, 301),     # the whole last chunk
    (1500, 0, 700),      # five chunks and a part of the sixth
    (1500, 128, 1501),   # every chunk but the first
    (17000, 96, 4000)]   # more than 128 chunks
CHUNKED = [(synth.DT_BF16, 128, 32, 4, 1), (synth.DT_BF16, 128, 6, 2, 2)]
GENERAL = [(synth.DT_F32, 128, 16, 4, 1), (synth.DT_BF16, 64, 14, 2, 2), (synth.DT_BF16, 128, 9, 1, 1)]


@pytest.mark.parametrize("length,first,last", LENGTHS)
@pytest.mark.parametrize("dtype,d,Hq,Hkv,L", CHUNKED + GENERAL)
def test_keys_without_a_finite_logit(dtype, d, Hq, Hkv, L, length, first, last):
    import torch
    import paper_2608_08569_amd as vz
    cap, gamma, nxt = length + 3, 0.95, length + 5
    k, v, s, p = synth.random_state(53, L, Hkv, d, cap, length, dtype, next_pos=nxt)
    key = synth.stream_key(53, dtype, d, Hq, Hkv, length)
    mk = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape), dtype)
    q, kn, vn = mk("q", (L, Hq, d)), mk("k", (L, Hkv, d)), mk("v", (L, Hkv, d))
    q[..., 5] = ONE[dtype]  # every head's query: positive on the channel that is infinite
    k[:, :, first: min(last, length), 5] = MINUS_INF[dtype]
    if last > length:
        kn[..., 5] = MINUS_INF[dtype]
    ref_o, ref_s, _, _ = oracle.decode_step(q, kn, vn, k, v, s.astype(np.float64), p, length, nxt, gamma, dtype)
    assert np.isfinite(ref_o).all() and np.isfinite(ref_s).all()
    g = GpuCache(L, Hq, Hkv, d, cap, dtype)
    g.load(k, v, s, p, length, nxt)
    g.step(to_dev(q), to_dev(kn), to_dev(vn), gamma)
    out, S = from_dev(g.out), from_dev(g.score)
    check_close(widen(out, dtype), ref_o, RTOL[dtype], "output")
    check_rel(S[:, : length + 1], ref_s, RTOL[dtype], "score")

    # the same bits as the second sequence of a batch, and as a batch of one
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    for lead in (7, 0):
        at = lead + 2 if lead else 0
        n = 2 if lead else 1
        shift = lambda a: np.concatenate([a[:, :, :at], a], axis=2) if a.ndim == 4 else np.concatenate([a[:, :at], a], 1)
        K, V, A, P = (to_dev(shift(x)) for x in (k, v, s, p))
        o = torch.zeros(n, L, Hq, d, dtype=K.dtype, device="cuda")
        rep = lambda a: to_dev(np.stack([a] * n))
        vz.voxzip_decode_attend_score_ragged(
            rep(q), rep(kn), rep(vn), K, V, A, P, o, torch.tensor([0, at][2 - n:], dtype=torch.int64, device="cuda"),
            i32([at, cap][2 - n:]), i32([lead, length][2 - n:]), i32([lead, nxt][2 - n:]), gamma,
            workspace=vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, d, at + cap, n))
        torch.cuda.synchronize()
        assert np.array_equal(from_dev(o[n - 1]), out)
        assert np.array_equal(from_dev(A)[:, at: at + length + 1], S[:, : length + 1])


@pytest.mark.parametrize("Hq,Hkv,L", [(32, 4, 32), (6, 2, 64)])
@pytest.mark.parametrize("T,first,last", [
    (300, 0, 130),       # the first chunk of a wave and keys of the next
    (300, 256, 300),     # the partial chunk
    (1500, 128, 1500),   # all chunks but the first
    (8224, 0, 8000),     # whole waves
    (9001, 0, 4608),     # the first of two parts
    (9001, 4000, 9001)]) # the second, and the end of the first
def test_keys_without_a_finite_logit_on_the_whole_range_path(Hq, Hkv, L, T, first, last):
    import math

    import torch
    import paper_2608_08569_amd as vz
    g = torch.Generator(device="cuda").manual_seed(T + first)
    n, d, gamma, bf, base = T - 1, 128, 0.95, torch.bfloat16, 9
    mk = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=bf)
    K, V, q, kn, vn = mk(L, Hkv, base + T, d), mk(L, Hkv, base + T, d), mk(2, L, Hq, d), mk(2, L, Hkv, d), mk(2, L, Hkv, d)
    q[..., 5] = 1.0  # every head's query: positive on the channel that is infinite
    K[:, :, base + first: base + min(last, n), 5] = -math.inf
    if last == T:
        kn[1, ..., 5] = -math.inf
    S = torch.rand(L, base + T, generator=g, device="cuda")
    P = torch.arange(base + T, dtype=torch.int32, device="cuda").repeat(L, 1)
    k1, v1, s1, p1 = (x[:, :, base:].contiguous() if x.dim() == 4 else x[:, base:].contiguous() for x in (K, V, S, P))
    out = torch.zeros(L, Hq, d, dtype=bf, device="cuda")
    vz.voxzip_decode_attend_score(q[1], kn[1], vn[1], k1, v1, s1, p1, out, n, n, gamma,
                                  workspace=vz.workspace(vz.VZ_OP_DECODE, L, Hq, Hkv, d, T))
    for l in (0, L - 1):
        ref_o, ref_s = [], gamma * S[l, base:].double()
        ref_s[n] = 0
        for h in range(Hkv):
            kd, vd = k1[l, h].double(), v1[l, h].double()
            s = (q[1, l].view(Hkv, -1, d)[h].double()[:, None] * kd[None]).sum(-1) / math.sqrt(d)
            a = torch.softmax(s, -1)
            ref_o.append(a @ vd)
            ref_s += a.sum(0)
        check_close(out[l].double().cpu().numpy(), torch.cat(ref_o).cpu().numpy(), RTOL[synth.DT_BF16], f"layer {l} output")
        check_rel(s1[l].double().cpu().numpy(), ref_s.cpu().numpy(), RTOL[synth.DT_BF16], f"layer {l} score")
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    o = torch.zeros(2, L, Hq, d, dtype=bf, device="cuda")
    vz.voxzip_decode_attend_score_ragged(q, kn, vn, K, V, S, P, o, torch.tensor([0, base], device="cuda"),
                                         i32([base, T]), i32([base - 1, n]), i32([base - 1, n]), gamma,
                                         workspace=vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, d, base + T, 2))
    torch.cuda.synchronize()
    assert torch.equal(o[1], out) and torch.equal(S[:, base:], s1)
