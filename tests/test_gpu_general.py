"""GPU parity of the general decode path (float32 caches, d = 64, groups of up
to 16 query heads, any number of KV heads): 128-key chunks, runs of chunks and
their remainders, one head per KV head, one KV head (scores folded with the
outputs), and planes of more than 128 chunks (statistics in a launch of their
own).  Single-sequence and ragged calls give the same bits; what the cache
holds past the resident slots is never used."""
import numpy as np
import pytest

import oracle
import synth
from vzt import RTOL, GpuCache, check_close, check_rel, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu

# Scores are float32 throughout in both element types.  Each p carries the
# rounding of its logit (d products: |s| d 2^-24 at worst, a few 2^-24 in
# practice), one of exp and one of 1 / Z: the float32 bound of the other tests.
SCORE_RTOL = RTOL[synth.DT_F32]

CASES = [  # dtype, d, Hq, Hkv, resident keys before the step
    (synth.DT_F32, 64, 4, 1, 126), (synth.DT_F32, 64, 4, 1, 127), (synth.DT_F32, 64, 4, 1, 128),
    (synth.DT_F32, 128, 6, 3, 0), (synth.DT_F32, 128, 6, 3, 383), (synth.DT_F32, 128, 16, 1, 511),
    (synth.DT_F32, 128, 18, 2, 512), (synth.DT_F32, 64, 3, 3, 700),
    (synth.DT_BF16, 64, 14, 2, 15), (synth.DT_BF16, 64, 14, 2, 900), (synth.DT_BF16, 64, 32, 2, 641),
    (synth.DT_BF16, 128, 9, 1, 260), (synth.DT_BF16, 128, 32, 2, 1023), (synth.DT_BF16, 128, 5, 5, 300),
    (synth.DT_F32, 64, 4, 2, 16899), (synth.DT_BF16, 64, 16, 1, 17100),
]
# 128 chunks in planes of 128, whose workgroups merge the statistics themselves
# (the ragged twin's planes have 129: a launch of its own), and of 129
EDGES = [(synth.DT_F32, 64, 4, 2, 16383, 1), (synth.DT_F32, 64, 4, 2, 16383, 2), (synth.DT_F32, 64, 4, 2, 16384, 1),
         (synth.DT_BF16, 64, 14, 2, 16383, 1), (synth.DT_BF16, 64, 4, 1, 16383, 1)]


@pytest.mark.parametrize("dtype,d,Hq,Hkv,length,slots", [c + (3,) for c in CASES] + EDGES)
def test_general_path_against_oracle_and_ragged_twin(dtype, d, Hq, Hkv, length, slots):
    import torch
    import paper_2608_08569_amd as vz
    L, cap, gamma, nxt = 2, length + slots, 0.95, length + 9
    k, v, s, p = synth.random_state(31, L, Hkv, d, cap, length, dtype, next_pos=nxt)
    key = synth.stream_key(31, dtype, d, Hq, Hkv, length)
    mk = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape) * np.float32(1.7), dtype)
    q, kn, vn = mk("q", (L, Hq, d)), mk("k", (L, Hkv, d)), mk("v", (L, Hkv, d))
    ref_o, ref_s, ref_p, _ = oracle.decode_step(q, kn, vn, k, v, s.astype(np.float64), p, length, nxt, gamma, dtype)
    for a in (k, v):  # past the resident slots: not a number
        a[:, :, length:] = np.float32(np.nan) if dtype == synth.DT_F32 else 0x7FC0
    g = GpuCache(L, Hq, Hkv, d, cap, dtype)
    g.load(k, v, s, p, length, nxt)
    g.ws_dec.fill_(0xFF)  # the workspace needs no initialisation (here: NaNs)
    g.step(to_dev(q), to_dev(kn), to_dev(vn), gamma, check_ws=False)
    K1, V1, S1, P1 = g.snapshot()
    out = from_dev(g.out)
    check_close(widen(out, dtype), ref_o, RTOL[dtype], "output")
    check_rel(S1[:, : length + 1], ref_s, SCORE_RTOL, "score")
    assert np.array_equal(P1[:, : length + 1], ref_p)
    assert np.array_equal(K1[:, :, length], kn) and np.array_equal(V1[:, :, length], vn)
    assert np.array_equal(K1[:, :, :length], k[:, :, :length]) and np.array_equal(V1[:, :, :length], v[:, :, :length])

    # the same sequence second in a ragged call, behind a short one
    short, base = 5, 9
    total = base + cap + 4
    plane = lambda a, b: np.concatenate([b, a, np.zeros_like(a[:, :, :4])], axis=2)
    rows = lambda a: np.concatenate([a[:, :1].repeat(base, 1), a, a[:, :4] * 0], axis=1)
    lead = mk("lead", (L, Hkv, base, d))
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    K, V = to_dev(plane(k, lead)), to_dev(plane(v, lead))
    S, P = to_dev(rows(s)), to_dev(rows(p))
    o = torch.zeros(2, L, Hq, d, dtype=K.dtype, device="cuda")
    status = i32([-99, -99])
    vz.voxzip_decode_attend_score_ragged(
        to_dev(np.stack([q, q])), to_dev(np.stack([kn, kn])), to_dev(np.stack([vn, vn])), K, V, S, P, o,
        torch.tensor([0, base], dtype=torch.int64, device="cuda"), i32([base, cap]), i32([short, length]),
        i32([short, nxt]), gamma, status=status, workspace=vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, d, total, 2))
    torch.cuda.synchronize()
    assert from_dev(status).tolist() == [vz.VZ_OK, vz.VZ_OK]
    assert np.array_equal(from_dev(o[1]), out)
    at = slice(base, base + length + 1)
    assert np.array_equal(from_dev(S)[:, at], S1[:, : length + 1])
    assert np.array_equal(from_dev(P)[:, at], P1[:, : length + 1])
    assert np.array_equal(from_dev(K)[:, :, at], K1[:, :, : length + 1])
    assert np.array_equal(from_dev(V)[:, :, at], V1[:, :, : length + 1])
