"""Sequences of more than 2^24 slots, where a row's offset in its plane passes
2^31 elements (d = 128) or bytes (d = 64): the appended row, the output, the
scores and an eviction's moved row, of single and ragged calls."""
import numpy as np
import pytest

import synth
from vzt import RTOL, check_close, check_rel, from_dev, to_dev, widen

pytestmark = pytest.mark.gpu

# float32: an output accumulator takes 2048 chunks of a run, eight matrix
# instructions each, one after the other: 2^14 roundings of 2^-24 at most.
# (A lane's sum of exp takes 2^17 / 16 chunks: half as many.)
RTOL = {**RTOL, synth.DT_F32: 2.0 ** -10}


@pytest.mark.parametrize("dtype,d,Hq", [(synth.DT_BF16, 128, 8), (synth.DT_F32, 64, 4)])
def test_appended_and_moved_rows_past_two_to_the_24_slots(dtype, d, Hq):
    import torch
    import paper_2608_08569_amd as vz
    n, gamma, lead = 1 << 24, 0.5, 5  # `lead` slots in front: the ragged call's base
    key = synth.stream_key(61, dtype)
    mk = lambda tag, shape: synth.as_storage(
        synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape), dtype)
    q, vn = mk("q", (1, Hq, d)), mk("v", (1, 1, d))
    # one channel decides: logit 0 for every resident key, about ln n for the new one
    q[..., 0] = synth.as_storage(np.linspace(0.9, 1.1, Hq, dtype=np.float32), dtype)
    kn = synth.as_storage(np.zeros((1, 1, d), dtype=np.float32), dtype)
    kn[..., 0] = synth.as_storage(np.full(1, 16.0 * np.sqrt(d), dtype=np.float32), dtype)[0]
    e = np.exp(widen(q[0, :, 0], dtype) * widen(kn[0, 0, 0], dtype) / np.sqrt(d))
    p_new, p_old = e / (e + n), 1.0 / (e + n)
    ref = p_new[:, None] * widen(vn[0, 0], dtype)[None] + (n * p_old)[:, None] * 0.5
    tdt = torch.float32 if dtype == synth.DT_F32 else torch.bfloat16
    for ragged in (False, True):
        cap = n + 2 + lead
        K = torch.zeros(1, 1, cap, d, dtype=tdt, device="cuda")
        V = torch.full((1, 1, cap, d), 0.5, dtype=tdt, device="cuda")
        S = torch.full((1, cap), 1e-3, device="cuda")
        P = torch.arange(cap, dtype=torch.int32, device="cuda")[None].contiguous()
        base = lead if ragged else 0
        S[0, base + 777] = 0.0  # the slot that an eviction takes
        out = torch.zeros((1, 1, Hq, d) if ragged else (1, Hq, d), dtype=tdt, device="cuda")
        i32 = lambda x: torch.tensor([x], dtype=torch.int32, device="cuda")
        if ragged:
            P.sub_(lead)
            seq = torch.tensor([base], dtype=torch.int64, device="cuda"), i32(n + 2)
            vz.voxzip_decode_attend_score_ragged(
                to_dev(q[None]), to_dev(kn[None]), to_dev(vn[None]), K, V, S, P, out, *seq, i32(n), i32(n), gamma,
                workspace=vz.workspace_ragged(vz.VZ_OP_DECODE, 1, Hq, 1, d, cap, 1))
            vz.voxzip_evict_compact_ragged(K, V, S, P, *seq, i32(n + 1), i32(n), i32(n + 1),
                                           workspace=vz.workspace_ragged(vz.VZ_OP_EVICT, 1, Hq, 1, d, cap, 1))
        else:
            assert vz.voxzip_decode_evict(to_dev(q), to_dev(kn), to_dev(vn), K, V, S, P, out, n, n, gamma, n, n_sink=4,
                                          workspace=vz.workspace(vz.VZ_OP_DECODE_EVICT, 1, Hq, 1, d, cap)) == n
        torch.cuda.synchronize()
        got = from_dev(out).reshape(Hq, d)
        check_close(widen(got, dtype), ref, RTOL[dtype], f"ragged {ragged}: output")
        rows = torch.tensor([base, base + 776, base + 777, base + n - 1, base + n], device="cuda")
        k, v, s, p = (from_dev(x.index_select(2 if x.dim() == 4 else 1, rows)) for x in (K, V, S, P))
        new = [False, False, True, False, True]  # appended at slot n, moved to the freed slot 777
        for i, is_new in enumerate(new):
            assert np.array_equal(k[0, 0, i], kn[0, 0] if is_new else 0 * kn[0, 0]), (ragged, i)
            assert np.array_equal(widen(v[0, 0, i], dtype), widen(vn[0, 0], dtype) if is_new else np.full(d, 0.5)), (ragged, i)
        check_rel(s[0], np.where(new, p_new.sum(), gamma * 1e-3 + p_old.sum()), RTOL[dtype], f"ragged {ragged}: score")
        assert p[0].tolist() == [0, 776, n, n - 1, n]
        assert int(torch.count_nonzero(K).item()) == 2  # nothing else was written
        del K, V, S, P
        torch.cuda.empty_cache()
