"""The generation step of calls that take the chunked or the general decode
path: with one eviction due it runs inside the folding launch, and gives the
bits of the decode call followed by the eviction call, step after step."""
import numpy as np
import pytest

import synth
from vzt import GpuCache, from_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,Hq,Hkv,L,budget,n_sink,n_recent", [
    (synth.DT_BF16, 128, 32, 4, 1, 1024, 4, -1),
    (synth.DT_BF16, 128, 32, 4, 3, 255, 4, 0),       # no recent window: the new token may be the one that goes
    (synth.DT_BF16, 128, 8, 8, 2, 129, 4, 125),      # sinks and recent fill the budget: no slot competes
    (synth.DT_BF16, 128, 16, 2, 2, 8223, 4, -1),     # the last length the folding launch takes
    (synth.DT_BF16, 128, 16, 2, 1, 8224, 4, -1),     # ... and the first it does not
    (synth.DT_F32, 64, 4, 1, 1, 128, 4, -1),         # one KV head, one run: the values launch
    (synth.DT_F32, 64, 4, 1, 5, 700, 0, 0),          # one KV head, several runs
    (synth.DT_BF16, 64, 14, 2, 3, 900, 4, -1),
    (synth.DT_F32, 128, 16, 4, 2, 127, 4, -1),
    (synth.DT_F32, 128, 3, 3, 2, 300, 1, 5)])
def test_step_equals_decode_then_evict(dtype, d, Hq, Hkv, L, budget, n_sink, n_recent):
    compare_steps(dtype, d, Hq, Hkv, L, budget, n_sink, n_recent, budget + 2)


@pytest.mark.parametrize("dtype,d,Hq,Hkv,L,budget,cap", [
    (synth.DT_F32, 64, 8, 2, 2, 7167, 7170),         # general path: the last length the folding launch takes
    (synth.DT_F32, 64, 8, 2, 2, 7168, 7170),         # ... and the first it does not
    (synth.DT_F32, 64, 2, 1, 2, 8223, 8225),         # ... with one KV head
    (synth.DT_BF16, 64, 16, 16, 2, 2559, 2561),      # ... with sixteen
    (synth.DT_BF16, 64, 16, 16, 2, 2560, 2562),
    (synth.DT_F32, 64, 8, 2, 3, 300, 16384),         # planes of 128 chunks: the blocks' own statistics
    (synth.DT_F32, 64, 8, 2, 3, 300, 16385),         # 129: statistics in a launch of their own, counters elsewhere
    (synth.DT_F32, 64, 4, 1, 3, 7000, 16385),
    (synth.DT_BF16, 128, 16, 2, 3, 300, 16384),      # chunked path: one finishing launch
    (synth.DT_BF16, 128, 16, 2, 3, 300, 16385)])     # ... two, and the eviction after them
def test_step_at_the_lines_of_its_dispatch(dtype, d, Hq, Hkv, L, budget, cap):
    compare_steps(dtype, d, Hq, Hkv, L, budget, 4, -1, cap)


def compare_steps(dtype, d, Hq, Hkv, L, budget, n_sink, n_recent, cap):
    import torch
    import paper_2608_08569_amd as vz
    nxt, steps = budget + 40, 3
    k, v, s, p = synth.random_state(budget, L, Hkv, d, cap, budget, dtype, next_pos=nxt)
    a, b = (GpuCache(L, Hq, Hkv, d, cap, dtype) for _ in range(2))
    for g in (a, b):
        g.load(k, v, s, p, budget, nxt)
    ws = vz.workspace(vz.VZ_OP_DECODE_EVICT, L, Hq, Hkv, d, cap)
    ws.fill_(0xA5)  # needs no initialisation
    for t in range(steps):
        key = synth.stream_key(budget, "step-small", t)
        mk = lambda tag, shape: to_dev(synth.as_storage(
            synth.normal_f32(synth.stream_key(key, tag), int(np.prod(shape))).reshape(shape), dtype))
        q, kn, vn = mk("q", (L, Hq, d)), mk("k", (L, Hkv, d)), mk("v", (L, Hkv, d))
        n = vz.voxzip_decode_evict(q, kn, vn, a.k, a.v, a.score, a.pos, a.out, budget, nxt + t, 0.95, budget,
                                   n_sink=n_sink, n_recent=n_recent, workspace=ws)
        assert n == budget
        b.step(q, kn, vn, 0.95)
        assert b.evict(budget, n_sink=n_sink, n_recent=n_recent) == budget
        torch.cuda.synchronize()
        assert np.array_equal(from_dev(a.out), from_dev(b.out)), f"step {t}: outputs"
        for x, y, what in zip(a.snapshot(), b.snapshot(), ("K", "V", "score", "position")):
            assert np.array_equal(x[..., :budget, :] if x.ndim == 4 else x[:, :budget],
                                  y[..., :budget, :] if y.ndim == 4 else y[:, :budget]), f"step {t}: {what}"
