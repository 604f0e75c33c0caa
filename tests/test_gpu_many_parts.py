"""Long sequences on the whole-range path: up to 4 parts the finishing launch
forms the heads' statistics itself, more take a launch of their own, in rounds
of 16 parts at 8 KV heads.  Against 64 bits on sampled layers, and bit for bit
against the ragged call, whose planes decide which of the two it takes."""
import math

import numpy as np
import pytest

import synth
from vzt import RTOL, check_close, check_rel

pytestmark = pytest.mark.gpu

D, GAMMA = 128, 0.95


@pytest.mark.parametrize("Hq,Hkv,L,T,tail", [
    (32, 4, 32, 32768, 33000),  # 4 parts; in the ragged call's longer planes with the factors' launch
    (32, 4, 32, 32769, 1),      # 5 parts; in the ragged call without it
    (6, 2, 64, 66001, 1),       # heads that do not fill their columns
    (64, 8, 16, 135001, 1)])    # 17 parts: a second round
def test_many_parts(Hq, Hkv, L, T, tail):
    import torch
    import paper_2608_08569_amd as vz
    g = torch.Generator(device="cuda").manual_seed(T)
    n, lead, bf = T - 1, 300, torch.bfloat16
    total = lead + T + tail
    mk = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=bf)
    K, V = mk(L, Hkv, total, D), mk(L, Hkv, total, D)
    S = torch.rand(L, total, generator=g, device="cuda")
    P = torch.arange(total, dtype=torch.int32, device="cuda").repeat(L, 1)
    q, kn, vn = mk(2, L, Hq, D), mk(2, L, Hkv, D), mk(2, L, Hkv, D)
    at = slice(lead, lead + T)
    k1, v1 = K[:, :, at].contiguous(), V[:, :, at].contiguous()
    s1, p1 = S[:, at].contiguous(), P[:, at].contiguous()
    s0 = s1.clone()
    out = torch.zeros(L, Hq, D, dtype=bf, device="cuda")
    ws = vz.workspace(vz.VZ_OP_DECODE, L, Hq, Hkv, D, T)
    ws.fill_(0xFF)  # needs no initialisation
    vz.voxzip_decode_attend_score(q[1], kn[1], vn[1], k1, v1, s1, p1, out, n, n, GAMMA, workspace=ws)
    for l in (0, L - 1):
        ref_o, ref_s = [], GAMMA * s0[l, :T].double()
        ref_s[n] = 0
        for h in range(Hkv):
            kd, vd = k1[l, h, :T].double(), v1[l, h, :T].double()
            kd[n], vd[n] = kn[1, l, h].double(), vn[1, l, h].double()
            a = torch.softmax(q[1, l].view(Hkv, -1, D)[h].double() @ kd.t().contiguous() / math.sqrt(D), -1)
            ref_o.append(a @ vd)
            ref_s += a.sum(0)
        check_close(out[l].double().cpu().numpy(), torch.cat(ref_o).cpu().numpy(), RTOL[synth.DT_BF16], f"layer {l} output")
        check_rel(s1[l, :T].double().cpu().numpy(), ref_s.cpu().numpy(), RTOL[synth.DT_BF16], f"layer {l} score")

    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    o = torch.zeros(2, L, Hq, D, dtype=bf, device="cuda")
    ws = vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, D, total, 2)
    ws.fill_(0xFF)
    status = i32([-9, -9])
    vz.voxzip_decode_attend_score_ragged(q, kn, vn, K, V, S, P, o, torch.tensor([0, lead], device="cuda"),
                                         i32([lead, T]), i32([lead - 1, n]), i32([lead - 1, n]), GAMMA,
                                         status=status, workspace=ws)
    assert status.tolist() == [vz.VZ_OK] * 2
    assert torch.equal(o[1], out) and torch.equal(S[:, at], s1)
    assert np.isfinite(o.float().cpu().numpy()).all()
