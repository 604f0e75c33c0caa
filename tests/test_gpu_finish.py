"""The chunked path's finishing launches (outputs and scores from the chunks'
partial results): one launch or two, by the call's sizes, give the same bits
for each sequence, also one of more than 128 chunks inside a batch that takes
the one launch; every case also against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from vzt import RTOL, GpuCache, check_close, check_rel, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu

D = 128


def _i32(a):
    import torch
    return torch.tensor(np.asarray(a), dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("Hq,Hkv,L,lens,slots", [
    (32, 4, 1, [130, 1700, 1, 5, 260, 2047], 2),       # one launch, several sequences
    (64, 8, 1, [900, 127], 2),                         # 64 heads: four rounds of 16
    (6, 2, 2, [300, 31], 2),                           # heads that do not fill a wave's quarter
    (8, 1, 1, [17000, 40, 90, 1000], 2),               # 133 chunks in a batch of one launch
    (32, 4, 1, [300] * 70, 2),                         # too many blocks for one launch
    (16, 4, 1, [16383], 1),                            # 128 chunks of one sequence in planes of 128: one launch
    (16, 4, 1, [16383], 2), (16, 4, 1, [16384], 1),    # 128 and 129 chunks in planes of 129: two launches
    (16, 4, 1, [16384], 2)])
def test_ragged_calls_match_single_calls_and_the_oracle(Hq, Hkv, L, lens, slots):
    import torch
    import paper_2608_08569_amd as vz
    n, gamma, dt = len(lens), 0.95, synth.DT_BF16
    key = synth.stream_key(41, Hq, Hkv, L, n, lens[0])
    noise = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape), dt)
    caps = np.asarray(lens) + slots  # at least one free slot
    base = np.concatenate([[0], np.cumsum(caps)[:-1]])
    total = int(caps.sum())
    K, V = noise("K", (L, Hkv, total, D)), noise("V", (L, Hkv, total, D))
    S = synth.uniform01(synth.stream_key(key, "S"), 0, L * total).reshape(L, total).astype(np.float32)
    P = np.zeros((L, total), dtype=np.int32)
    for b, m in zip(base, lens):
        P[:, b: b + m] = np.arange(m)
    q, kn, vn = noise("q", (n, L, Hq, D)), noise("kn", (n, L, Hkv, D)), noise("vn", (n, L, Hkv, D))
    Kd, Vd, Sd, Pd, out = to_dev(K), to_dev(V), to_dev(S), to_dev(P), to_dev(np.zeros_like(q))
    status = _i32([-9] * n)
    vz.voxzip_decode_attend_score_ragged(
        to_dev(q), to_dev(kn), to_dev(vn), Kd, Vd, Sd, Pd, out, torch.tensor(base, device="cuda"), _i32(caps),
        _i32(lens), _i32(lens), gamma, status=status,
        workspace=vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, D, total, n))
    torch.cuda.synchronize()
    assert from_dev(status).tolist() == [vz.VZ_OK] * n
    o, s1 = from_dev(out), from_dev(Sd)
    for i in sorted({0, n // 2, n - 1}):
        m, at = int(lens[i]), slice(int(base[i]), int(base[i] + caps[i]))
        ref_o, ref_s, _, _ = oracle.decode_step(q[i], kn[i], vn[i], K[:, :, at], V[:, :, at],
                                                S[:, at].astype(np.float64), P[:, at], m, m, gamma, dt)
        check_close(widen(o[i], dt), ref_o, RTOL[dt], f"sequence {i} output")
        check_rel(s1[:, at][:, : m + 1], ref_s, RTOL[dt], f"sequence {i} score")
        g = GpuCache(L, Hq, Hkv, D, int(caps[i]), dt)
        g.load(K[:, :, at], V[:, :, at], S[:, at], P[:, at], m, m)
        g.step(to_dev(q[i]), to_dev(kn[i]), to_dev(vn[i]), gamma)
        assert np.array_equal(from_dev(g.out), o[i])
        _, _, sg, _ = g.snapshot()
        assert np.array_equal(sg[:, : m + 1], s1[:, at][:, : m + 1])
