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
