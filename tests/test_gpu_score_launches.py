"""The ways a step's scoring is launched: hidden units of a token group shared by workgroups (rollout), layers that share a
launch; and that none of them changes a bit of a score, because selections compare scores of different launches."""
import numpy as np
import pytest
import torch

from oracle import pafu_oracle as orc
from paper_2601_21896_amd import binding as B
from paper_2601_21896_amd import workloads as wl
from tests.gpu_util import DEV, bits, dev, host, step_workspace

pytestmark = pytest.mark.gpu


def _steps(mode, layers, n, Lc, N, D, M, n_out, n_seg, bias, dt="bf16", shared_ws=True):
    """Argument structs of `layers` steps, what they hold, and where each layer's fresh scores land."""
    rng = np.random.Generator(np.random.PCG64(layers * 1000 + M + Lc))
    single, k = mode == B.PAFU_MODE_SINGLE, max(1, n // 2)
    rnd = wl.round_to_bf16 if dt == "bf16" else (lambda a: a)
    draw = lambda *shape: rng.standard_normal(shape, dtype=np.float32)
    T = Lc + (n if single else 0)
    args, held, fresh = [], [], []
    for _ in range(layers):
        X = [rnd(draw(T, N * D)) for _ in range(n_seg)]
        W1 = rnd(draw(M, n_seg * N * D) * np.float32(0.05))
        W2 = draw(n_out, M) * np.float32(0.1)
        b1, b2 = (draw(M) * np.float32(0.1), draw(n_out)) if bias else (None, None)
        xs = [dev(x, dt) for x in X]
        kv = [dev(rnd(draw(r, N, D)), "bf16") for r in (n, n, Lc, Lc, Lc)]
        SL = dev(draw(n))
        scores = torch.full((T + 4,), -9.0, device=DEV)
        ids = torch.zeros(k, dtype=torch.int32, device=DEV)
        Ko, Vo = (torch.zeros(k + Lc, N, D, device=DEV, dtype=torch.bfloat16) for _ in range(2))
        SLo = torch.full((k + Lc + 4,), -9.0, device=DEV)
        O = torch.zeros(Lc, N, D, device=DEV, dtype=torch.bfloat16)
        w = [dev(W1, dt), None if b1 is None else dev(b1), dev(W2), None if b2 is None else dev(b2)]
        lead = n if single else 0
        a = B.make_step_args(mode, N, D, n, Lc, k, Lc, tuple(x[:lead] for x in xs) if single else None,
                             tuple(x[lead:] for x in xs), w[0], w[1], w[2], w[3], kv[0], kv[1], None if single else SL,
                             kv[2], kv[3], kv[4], scores if single else None, ids, Ko, Vo, SLo, O)
        if shared_ws and args:
            a.workspace, a.workspace_bytes = args[0].workspace, args[0].workspace_bytes
        else:
            step_workspace(a)
        args.append(a)
        held.append((X, W1, b1, W2, b2, xs, kv, SL, scores, ids, Ko, Vo, SLo, O, w))
        fresh.append(scores if single else SLo[k:])
    return args, held, fresh


@pytest.mark.parametrize("layers,Lc,N,D,M,n_out,n_seg,bias,shared_ws", [
    (1, 33, 2, 128, 128, 1, 1, False, True),      # one pass of 128 units, a tile of one token
    (1, 1, 2, 64, 384, 12, 1, True, True),        # three passes of 128, one token
    (1, 500, 12, 128, 1024, 12, 3, True, True),   # long rows: eight workgroups share a token group
    (1, 700, 4, 128, 512, 20, 1, True, True),     # more output rows than the kernel averages itself
    (1, 3000, 2, 128, 768, 16, 1, False, True),   # few slabs, many groups (the last ones not a multiple of 8)
    (1, 9000, 1, 64, 256, 1, 1, False, True),     # one slab only
    (3, 300, 4, 64, 128, 4, 1, True, True),       # layers in one launch, with a common workspace
    (3, 300, 4, 64, 1024, 4, 2, True, False),     # ... each with its own: one by one
    (33, 40, 2, 64, 512, 2, 1, False, True),      # more layers than a launch takes
])
def test_rollout_chunk_scores(layers, Lc, N, D, M, n_out, n_seg, bias, shared_ws):
    """fp32 sums of up to 4608 products of order 0.05 and up to 1024 units: roundings of 2^-24 that add up like a random
    walk, sqrt(4608) 2^-24 = 4e-6 of the sums; 1e-5 of the largest score is allowed."""
    args, held, fresh = _steps(B.PAFU_MODE_ROLLOUT, layers, 96, Lc, N, D, M, n_out, n_seg, bias, shared_ws=shared_ws)
    B.pafu_step(args[0]) if layers == 1 else B.pafu_step_layers(args)
    torch.cuda.synchronize()
    for h, s in zip(held, fresh):
        want = orc.smlp_score(np.concatenate(h[0], axis=1), *h[1:5])
        got = host(s)
        assert np.all(got[Lc:] == -9.0)
        err = np.abs(got[:Lc] - want).max()
        assert err <= 1e-5 * max(np.abs(want).max(), 1.0), err


@pytest.mark.parametrize("layers,n,Lc,N,D,M,n_out,n_seg,dt", [
    (1, 300, 100, 4, 128, 1024, 12, 1, "bf16"),
    (4, 301, 77, 4, 64, 128, 4, 1, "bf16"),
    (4, 301, 77, 4, 64, 256, 4, 3, "bf16"),
    (2, 301, 77, 2, 64, 96, 2, 1, "bf16"),
    (1, 256, 64, 2, 64, 32, 1, 1, "fp32"),
    (3, 40, 17, 2, 64, 37, 5, 2, "fp32"),
])
def test_scores_that_select_do_not_depend_on_the_launch(layers, n, Lc, N, D, M, n_out, n_seg, dt):
    args, held, fresh = _steps(B.PAFU_MODE_SINGLE, layers, n, Lc, N, D, M, n_out, n_seg, True, dt)
    B.pafu_step(args[0]) if layers == 1 else B.pafu_step_layers(args)
    for h, s in zip(held, fresh):
        alone = torch.empty(n + Lc, device=DEV)
        ws = torch.empty(M + 4, device=DEV)
        B.pafu_score(tuple(h[5]), h[14][0], h[14][1], h[14][2], h[14][3], alone, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(bits(alone), bits(s[:n + Lc]))
        want = orc.smlp_score(np.concatenate(h[0], axis=1), *h[1:5])
        assert np.abs(host(alone) - want).max() <= 1e-5 * max(np.abs(want).max(), 1.0)


@pytest.mark.parametrize("Lc,N,D,M,n_out,n_seg,bias", [
    (700, 12, 128, 1024, 12, 3, True),   # eight workgroups share a token group
    (2000, 4, 128, 512, 20, 1, True),    # more output rows than the kernels average themselves
    (1100, 12, 128, 256, 1, 1, False),   # one pass of 256 units, or two halves of it
    (333, 2, 64, 768, 16, 1, True),
    (500, 2, 64, 384, 3, 2, True),       # a hidden layer that 256 does not divide
    (300, 4, 64, 128, 1, 1, False),
])
def test_a_chunks_scores_are_those_of_any_other_launch(Lc, N, D, M, n_out, n_seg, bias):
    """A rollout stores the chunk's scores among those of other chunks: bit for bit what pafu_score gives, with and without
    scratch, for several layers in a launch, and for a shorter chunk of the same tokens."""
    def launch(length, layers, ws):
        args, held, fresh = _steps(B.PAFU_MODE_ROLLOUT, layers, 96, Lc, N, D, M, n_out, n_seg, bias)
        for a in args:
            a.Lc = length
            if not ws:
                a.workspace_bytes = (B.pafu_score_workspace_bytes(M) + 255) // 256 * 256
        B.pafu_step(args[0]) if layers == 1 else B.pafu_step_layers(args)
        torch.cuda.synchronize()
        for h, s in zip(held, fresh):
            alone, w = torch.empty(Lc, device=DEV), torch.empty(M + 4, device=DEV)
            B.pafu_score(tuple(h[5]), h[14][0], h[14][1], h[14][2], h[14][3], alone, workspace=w)
            torch.cuda.synchronize()
            assert np.array_equal(bits(alone[:length]), bits(s[:length])), (length, layers, ws)
            assert torch.all(s[length:] == -9.0)

    for layers in (1, 3):
        for ws in (True, False):
            launch(Lc, layers, ws)
    launch(Lc // 7, 1, True)


@pytest.mark.parametrize("T,Fs,n_seg,M,n_out", [
    (1, 4, 1, 1, 1), (16, 132, 1, 32, 1), (17, 260, 3, 37, 3), (333, 100, 2, 64, 12), (50, 1000, 1, 31, 20)])
def test_fp32_tiles_form_the_sums_of_the_plain_kernel(T, Fs, n_seg, M, n_out):
    """The same values as bf16 (rows whose length 64 does not divide take the plain kernel) and as fp32: the same bits."""
    assert Fs % 64 != 0
    rng = np.random.Generator(np.random.PCG64(T + Fs))
    pad = (Fs + 7) // 8 * 8
    X = [wl.round_to_bf16(rng.standard_normal((T, pad), dtype=np.float32)) for _ in range(n_seg)]
    W1 = wl.round_to_bf16(rng.standard_normal((M, n_seg * Fs), dtype=np.float32) * np.float32(0.05))
    W2, b1, b2 = (dev(rng.standard_normal(s, dtype=np.float32)) for s in ((n_out, M), (M,), (n_out,)))
    got = []
    for dt in ("bf16", "fp32"):
        out, ws = torch.full((T + 1,), -9.0, device=DEV), torch.empty(M + 4, device=DEV)
        B.pafu_score(tuple(dev(x, dt)[:, :Fs] for x in X), dev(W1, dt), b1, W2, b2, out[:T], workspace=ws)
        torch.cuda.synchronize()
        assert float(out[T]) == -9.0
        got.append(bits(out))
    assert np.array_equal(got[0], got[1])
