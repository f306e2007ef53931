"""Multi-layer steps whose layers share launches: every layer's indices, cache rows and attention against the oracle."""
import numpy as np
import pytest
import torch

from oracle import pafu_oracle as orc
from paper_2601_21896_amd import binding as B
from paper_2601_21896_amd import workloads as wl
from tests.gpu_util import ATTN_MAX_ABS, ATTN_REL_FRO, DEV, attn_errors, dev, host, step_workspace

pytestmark = pytest.mark.gpu

EK, EV = -5, -6


@pytest.mark.parametrize("layers,n,Lc,L_B,N,D,kv,ws", [
    # 18 items of 35, 36 and 36 units: 642 units in 256 runs, which cross from item to item and from layer to layer
    (3, 8000, 600, 200, 2, 128, "bf16", True),
    (3, 8000, 600, 200, 2, 64, "bf16", True),
    (3, 8000, 600, 200, 2, 128, "e4m3", True),
    (3, 8000, 600, 200, 2, 128, "bf16", False),   # the same items whole
    (3, 900, 300, 300, 3, 128, "e4m3", False),
    (33, 96, 40, 40, 2, 64, "bf16", True),        # more layers than a launch takes
    (34, 700, 70, 30, 1, 128, "e4m3", True),
])
def test_layers_that_share_launches_match_the_oracle(layers, n, Lc, L_B, N, D, kv, ws):
    rng = np.random.Generator(np.random.PCG64(layers + n))
    draw = lambda *s: rng.standard_normal(s, dtype=np.float32)
    k, M, fp8 = n // 2, 64, kv == "e4m3"
    args, held = [], []
    for _ in range(layers):
        K, V, Q, Kn, Vn = (wl.round_to_bf16(draw(r, N, D)) for r in (n, n, Lc, Lc, Lc))
        SL = draw(n)
        if fp8:
            K, V = orc.quantise_e4m3(K.reshape(n, -1), EK), orc.quantise_e4m3(V.reshape(n, -1), EV)
            cache = [torch.from_numpy(a).to(DEV) for a in (K, V)]
            out = [torch.zeros(k + Lc, N * D, device=DEV, dtype=torch.uint8) for _ in range(2)]
        else:
            cache = [dev(a, "bf16") for a in (K, V)]
            out = [torch.zeros(k + Lc, N, D, device=DEV, dtype=torch.bfloat16) for _ in range(2)]
        ids = torch.zeros(k, dtype=torch.int32, device=DEV)
        SLo, O = torch.zeros(k + Lc, device=DEV), torch.zeros(Lc, N, D, device=DEV, dtype=torch.float32)
        a = B.make_step_args(B.PAFU_MODE_ROLLOUT, N, D, n, Lc, k, L_B, None, dev(draw(Lc, N * D), "bf16"),
                             dev(draw(M, N * D), "bf16"), None, dev(draw(1, M)), None, cache[0], cache[1], dev(SL),
                             dev(Q, "bf16"), dev(Kn, "bf16"), dev(Vn, "bf16"), None, ids, out[0], out[1], SLo, O,
                             kv_dtype=B.PAFU_FP8_E4M3 if fp8 else B.PAFU_BF16, k_scale_log2=EK if fp8 else 0,
                             v_scale_log2=EV if fp8 else 0)
        if ws and args:
            a.workspace, a.workspace_bytes = args[0].workspace, args[0].workspace_bytes
        elif ws:
            step_workspace(a)
        args.append(a)
        held.append((K, V, Q, Kn, Vn, SL, ids, out, SLo, O))
    B.pafu_step_layers(args)
    torch.cuda.synchronize()
    dq = lambda c, e: orc.dequantise_e4m3(c, e).reshape(-1, N, D)
    for l, (K, V, Q, Kn, Vn, SL, ids, out, SLo, O) in enumerate(held):
        want = orc.select_topk(SL, k)
        assert np.array_equal(host(ids), want), l
        assert np.array_equal(host(SLo[:k]), SL[want]), l
        if fp8:
            Kn, Vn = orc.quantise_e4m3(Kn.reshape(Lc, -1), EK), orc.quantise_e4m3(Vn.reshape(Lc, -1), EV)
        rows = [np.concatenate([K[want], Kn]), np.concatenate([V[want], Vn])]
        for got, r in zip(out, rows):
            assert np.array_equal(got.cpu().numpy() if fp8 else host(got), r), l
        if fp8:
            rows = [dq(rows[0], EK), dq(rows[1], EV)]
        O_want = orc.chunk_attention(Q, rows[0][:k], rows[1][:k], rows[0][k:], rows[1][k:], block_len=L_B)
        max_abs, rel = attn_errors(host(O), O_want)
        assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (l, max_abs, rel)


# A layer alone takes the attention kernel for few queries over few keys, the layers together pass its line: the same bits
@pytest.mark.parametrize("layers,N,D", [(6, 12, 128), (10, 7, 64)])
def test_short_layers_have_the_bits_of_single_steps(layers, N, D):
    n, Lc, k, M = 400, 128, 200, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(layers)
    draw = lambda *s: torch.randn(*s, device=DEV, generator=g)
    bf = lambda *s: draw(*s).to(torch.bfloat16)

    def args(t):
        out = dict(scores=torch.zeros(n + Lc, device=DEV), ids=torch.zeros(k, dtype=torch.int32, device=DEV),
                   K_out=torch.zeros(k, N, D, device=DEV, dtype=torch.bfloat16),
                   V_out=torch.zeros(k, N, D, device=DEV, dtype=torch.bfloat16), SL_out=torch.zeros(k, device=DEV),
                   O=torch.zeros(Lc, N, D, device=DEV))
        return out, B.make_step_args(B.PAFU_MODE_SINGLE, N, D, n, Lc, k, 50, t["xc"], t["x"], t["W1"], None, t["W2"], None,
                                     t["K"], t["V"], None, t["Q"], t["Kn"], t["Vn"], out["scores"], out["ids"],
                                     out["K_out"], out["V_out"], out["SL_out"], out["O"])

    given = [dict(xc=bf(n, 64), x=bf(Lc, 64), W1=bf(M, 64), W2=draw(1, M), K=bf(n, N, D), V=bf(n, N, D), Q=bf(Lc, N, D),
                  Kn=bf(Lc, N, D), Vn=bf(Lc, N, D)) for _ in range(layers)]
    together = [args(t) for t in given]
    B.pafu_step_layers([a for _, a in together])
    for t, (out, _) in zip(given, together):
        alone, a = args(t)
        B.pafu_step(a)
        torch.cuda.synchronize()
        for key in alone:
            assert torch.equal(alone[key], out[key]), key
