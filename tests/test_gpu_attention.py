"""GPU parity of pafu_chunk_attention against the fp64 oracle (max-abs 2e-2, relative Frobenius 5e-3)."""
import numpy as np
import pytest
import torch

from oracle import pafu_oracle as orc
from paper_2601_21896_amd import binding as B
from paper_2601_21896_amd import workloads as wl
from tests.gpu_util import ATTN_MAX_ABS, ATTN_REL_FRO, DEV, attention_workspace, attn_errors, dev, host

pytestmark = pytest.mark.gpu


def _inputs(n, Lc, N, D, seed, q_gain=1.0):
    rng = np.random.Generator(np.random.PCG64(seed))
    c = rng.uniform(0.5, 2.0, size=(N * D,)).astype(np.float32)
    r = lambda rows, s=None: wl.round_to_bf16(
        (rng.standard_normal((rows, N * D), dtype=np.float32) * (1.0 if s is None else s[None, :]))).reshape(rows, N, D)
    Kc, Vc = r(n, c), r(n)
    Q = wl.round_to_bf16(r(Lc) * np.float32(q_gain))
    Kn, Vn = r(Lc, c), r(Lc)
    return Q, Kc, Vc, Kn, Vn


# Calls of up to 256 groups of 32 queries (heads times query groups) over up to 24 tiles of 64 keys (7 at head dim 128) take a
# kernel of their own.  `copies` repeats the heads, so that a short call passes that line and takes the long kernel; the
# copies must have the same bits (with a workspace some of them may be cut: then the last ones are returned).
def _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=torch.bfloat16, Lq=None, ws=None, copies=1):
    Lq = Q.shape[0] if Lq is None else Lq
    N, D = Q.shape[1], Q.shape[2]
    n = Kc.shape[0]
    O = torch.full((Lq + 2, N * copies, D), 55.0, device=DEV, dtype=out_dtype)
    up = lambda x: dev(x, "bf16").repeat(1, copies, 1)
    B.pafu_chunk_attention(up(Q[:Lq]), up(Kc) if n else None, up(Vc) if n else None, n, up(Kn), up(Vn), L_B, O[:Lq],
                           workspace=ws)
    torch.cuda.synchronize()
    assert torch.all(O[Lq:] == 55.0)
    if ws is not None:
        assert (O[:Lq].view(Lq, copies, -1) - O[:Lq, :N].reshape(Lq, 1, -1)).nan_to_num().abs().max() < 2 * ATTN_MAX_ABS
        return host(O[:Lq, -N:])
    return _first_copy(O[:Lq], N)


def _first_copy(O, N):
    same = O.view(O.shape[0], -1, N * O.shape[2])
    bits = same.view(torch.int16 if O.dtype == torch.bfloat16 else torch.int32)
    assert torch.equal(bits, bits[:, :1].expand_as(bits))
    return host(O[:, :N])


@pytest.mark.parametrize("n,Lc,N,D,L_B", [
    (128, 64, 2, 64, 64),        # C0 shapes after budget 50%
    (128, 64, 2, 64, 16),
    (128, 64, 2, 64, 1),         # causal inside the chunk
    (0, 64, 2, 64, 64),          # first chunk: empty cache
    (0, 40, 1, 128, 7),
    (300, 200, 3, 128, 200),     # ragged query tile (200 = 128 + 72) and key tail (500 = 7*64 + 52)
    (300, 200, 3, 128, 50),
    (333, 130, 2, 128, 13),
    (1, 1, 1, 128, 1),
    (63, 129, 2, 64, 129),
    (1000, 520, 2, 128, 130),
    # short calls of many heads: the long kernel
    (128, 64, 130, 64, 16), (0, 64, 130, 64, 1), (63, 129, 52, 64, 129),
    (0, 40, 130, 128, 7), (1, 1, 257, 128, 1), (300, 130, 52, 128, 130), (317, 130, 52, 128, 13),
])
def test_attention_matches_oracle(n, Lc, N, D, L_B):
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=n * 7 + Lc)
    got = _run(Q, Kc, Vc, Kn, Vn, L_B)
    want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=L_B)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)


# Segments of 1 to 11 tiles, with and without a tile that straddles the two key segments, chunks shorter than a tile: in the
# long kernel (many copies of the heads: one item's tiles around the turns of the four-slot ring, ending in each slot) and in
# the one for few queries.  The gathered form reads the same rows through an index list: the same bits.  (Items that follow one
# another in one workgroup's run: test_attention_equal_runs_match_oracle.)
@pytest.mark.parametrize("copies", [1, 129])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 128, 191, 256, 320, 449, 512])
def test_attention_tile_counts_and_boundaries(n, D, copies):
    N = 2
    for Lc, L_B in [(1, 1), (63, 63), (64, 20), (65, 65), (130, 64)]:
        Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=n * 131 + Lc)
        want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=L_B)
        plain = _run(Q, Kc, Vc, Kn, Vn, L_B, copies=copies)
        for got in (plain, _run(Q, Kc, Vc, Kn, Vn, L_B, ws=attention_workspace(D), copies=copies)):
            max_abs, rel = attn_errors(got, want)
            assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (Lc, L_B, max_abs, rel)
        if n > 0:
            rows = 2 * n + 1
            at = np.sort(np.random.Generator(np.random.PCG64(n)).permutation(rows)[:n]).astype(np.int32)
            K, V = (torch.full((rows, N * copies, D), 7.0, device=DEV, dtype=torch.bfloat16) for _ in range(2))
            d_at = torch.from_numpy(at).to(DEV)
            up = lambda x: dev(x, "bf16").repeat(1, copies, 1)
            K[d_at.long()], V[d_at.long()] = up(Kc), up(Vc)
            O = torch.empty(Lc, N * copies, D, device=DEV, dtype=torch.bfloat16)
            B.pafu_chunk_attention_gather(up(Q), K, V, d_at, n, up(Kn), up(Vn), L_B, O)
            torch.cuda.synchronize()
            assert np.array_equal(_first_copy(O, N), plain), (Lc, L_B)


# Both sides of the line between the kernel for few queries over few keys and the long one (256 groups of 32 queries; 24 tiles
# at head dim 64, 7 at 128), with all forms of output, block masks, and the gathered form's bits.
@pytest.mark.parametrize("n,Lc,N,D,L_B,odt", [
    (1472, 64, 2, 64, 64, torch.float32), (1473, 64, 2, 64, 64, torch.float32),     # 24 and 25 tiles
    (1400, 100, 4, 64, 33, torch.bfloat16), (40, 33, 128, 64, 5, torch.bfloat16),   # three tiles per wave; 256 groups
    (40, 33, 130, 64, 5, torch.bfloat16), (0, 130, 64, 64, 130, torch.bfloat16),    # 260 and 320
    (65, 130, 64, 64, 64, torch.bfloat16), (191, 130, 64, 64, 7, torch.float32), (512, 130, 64, 64, 130, torch.bfloat16),
    (254, 130, 2, 128, 40, torch.float32), (255, 130, 2, 128, 40, torch.float32),   # 6 and 7 tiles
    (318, 130, 2, 128, 40, torch.bfloat16), (319, 130, 2, 128, 40, torch.float32),  # 7 and 8
    (65, 130, 12, 128, 130, torch.bfloat16), (65, 130, 13, 128, 130, torch.bfloat16),  # 60 and 65 groups
    (40, 33, 128, 128, 5, torch.bfloat16), (40, 33, 130, 128, 5, torch.bfloat16),   # 256 and 260
])
def test_attention_few_queries_over_few_keys(n, Lc, N, D, L_B, odt):
    # a peaked softmax in fp32 only: |O| passes 4 there, where half a unit of a bf16 result (2^-6) and the rounding of the
    # weights (2^-9 |V|, |V| up to 4.8) already add up to 0.025
    for gain in (1.0, 8.0) if odt == torch.float32 else (1.0,):
        Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=n + 3 * Lc + N, q_gain=gain)
        got = _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=odt)
        max_abs, rel = attn_errors(got, orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=L_B))
        assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (gain, max_abs, rel)
        if n > 0:
            ids = torch.arange(n, dtype=torch.int32, device=DEV)
            O = torch.empty(Lc, N, D, device=DEV, dtype=odt)
            B.pafu_chunk_attention_gather(dev(Q, "bf16"), dev(Kc, "bf16"), dev(Vc, "bf16"), ids, n, dev(Kn, "bf16"),
                                          dev(Vn, "bf16"), L_B, O)
            torch.cuda.synchronize()
            assert np.array_equal(host(O), got), gain


# A query's result has the same bits whichever kernel takes it.  The heads of the whole call pass the line of the kernel for few
# queries over few keys (256 groups of 32 queries); two of them alone do not.  Scores that grow from tile to tile or jump by
# hundreds of powers of two raise the softmax reference in both.
@pytest.mark.parametrize("n,Lc,N,D,L_B", [
    (128, 64, 130, 64, 64), (0, 130, 52, 64, 33), (700, 300, 26, 64, 77), (1403, 130, 52, 64, 130),
    (128, 64, 130, 128, 64), (0, 384, 22, 128, 100), (65, 130, 52, 128, 130), (251, 130, 52, 128, 64), (316, 130, 52, 128, 130),
])
@pytest.mark.parametrize("kind", ["plain", "growing", "jump", "nan query"])
def test_attention_bits_do_not_depend_on_what_shares_the_launch(n, Lc, N, D, L_B, kind):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + Lc + D)
    draw = lambda rows: torch.randn(rows, N, D, device=DEV, generator=g)
    Q, Kc, Vc, Kn, Vn = draw(Lc), draw(n), draw(n), draw(Lc), draw(Lc)
    tile = (torch.arange(n + Lc, device=DEV) // 64)[:, None, None].float()
    if kind == "growing":
        Kc, Kn = Kc * (0.1 * 2.0 ** tile[:n]), Kn * (0.1 * 2.0 ** tile[n:])
    elif kind == "jump":  # the queries' common direction meets keys that go up by 300 powers of two in the second tile
        Q = 0.3 * Q + 1.0
        step = 300 / (np.log2(np.e) * np.sqrt(D))
        Kc, Kn = 0.3 * Kc + step * tile[:n].clamp(max=1), 0.3 * Kn + step * tile[n:].clamp(max=1)
    elif kind == "nan query":
        Q[::29] = float("nan")
    Q, Kc, Vc, Kn, Vn = (x.to(torch.bfloat16) for x in (Q, Kc, Vc, Kn, Vn))
    O = torch.empty(Lc, N, D, device=DEV, dtype=torch.float32)
    B.pafu_chunk_attention(Q, Kc if n else None, Vc if n else None, n, Kn, Vn, L_B, O)
    torch.cuda.synchronize()
    for heads in (slice(0, 2), slice(N - 2, N)):
        few = torch.empty(Lc, 2, D, device=DEV, dtype=torch.float32)
        q, kc, vc, kn, vn = (x[:, heads] if heads.start == 0 else x[:, heads].contiguous() for x in (Q, Kc, Vc, Kn, Vn))
        B.pafu_chunk_attention(q, kc if n else None, vc if n else None, n, kn, vn, L_B, few)
        torch.cuda.synchronize()
        assert np.array_equal(host(few), host(O[:, heads]), equal_nan=True)
        if n:
            ids = torch.arange(n, dtype=torch.int32, device=DEV)
            again = torch.empty_like(few)
            B.pafu_chunk_attention_gather(q, kc, vc, ids, n, kn, vn, L_B, again)
            torch.cuda.synchronize()
            assert np.array_equal(host(again), host(few), equal_nan=True)


def test_attention_peaked_softmax_and_fp32_output():
    # queries scaled x8: the softmax is peaked, |O| ~ 1, so the max-abs bound bites
    n, Lc, N, D = 500, 192, 2, 128
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=99, q_gain=8.0)
    want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=64)
    assert np.abs(want).max() > 0.5
    for odt in (torch.bfloat16, torch.float32):
        got = _run(Q, Kc, Vc, Kn, Vn, 64, out_dtype=odt)
        max_abs, rel = attn_errors(got, want)
        assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (odt, max_abs, rel)


# With a workspace the launch cuts the flattened (head, query tile, key tiles) list of its last, ill-filled round into
# equal runs, at most one per CU, and merges the partial results of the query tiles that several workgroups worked on.
@pytest.mark.parametrize("n,Lc,N,D,L_B,odt,q_gain", [
    (16000, 600, 4, 128, 600, torch.bfloat16, 1.0),   # 12 items of 130 units each, 19 runs per item
    (9000, 1500, 3, 128, 500, torch.bfloat16, 1.0),   # block mask: the items have different lengths
    (9000, 1500, 3, 128, 500, torch.float32, 8.0),    # ... peaked softmax, fp32 output
    (20000, 300, 5, 64, 300, torch.bfloat16, 1.0),    # head dim 64
    (0, 9000, 2, 128, 1, torch.bfloat16, 1.0),        # no cache, strictly causal inside the chunk
    (12345, 777, 3, 128, 100, torch.bfloat16, 1.0),   # ragged everything
    (3000, 51, 5, 64, 51, torch.bfloat16, 1.0),       # fewer runs than compute units: 120 units in runs of two
    (900, 40, 1, 128, 40, torch.float32, 1.0),        # one item of 8 units in 4 runs
    (300, 1700, 40, 64, 1700, torch.bfloat16, 1.0),   # 280 items on 256 CUs: a round of whole items, 24 items cut
    (100, 1700, 38, 128, 450, torch.float32, 1.0),    # 266 items of different lengths, 10 of them cut
    (600, 500, 150, 64, 256, torch.bfloat16, 1.0),    # 300 items of 7 and 9 units, 44 cut in runs of two that cross items
    (600, 500, 150, 128, 256, torch.bfloat16, 1.0),
])
def test_attention_equal_runs_match_oracle(n, Lc, N, D, L_B, odt, q_gain):
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=n + Lc + N, q_gain=q_gain)
    ws = attention_workspace(D)
    got = _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=odt, ws=ws)
    want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=L_B)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)
    # the same launch without the workspace (one workgroup per query tile) agrees to the rounding of the bf16
    # softmax weights (taken relative to different running maxima), and a second launch with the workspace (now
    # holding the first one's partial results) gives the same bits as the first
    plain = _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=odt)
    assert np.abs(plain - got).max() < ATTN_MAX_ABS * max(1.0, np.abs(want).max())
    again = _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=odt, ws=ws)
    assert np.array_equal(got, again)


def test_attention_workspace_too_small_falls_back_to_whole_query_tiles():
    n, Lc, N, D = 16000, 600, 4, 128
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=3)
    small = torch.empty(4096, dtype=torch.uint8, device=DEV)
    got = _run(Q, Kc, Vc, Kn, Vn, Lc, ws=small)
    plain = _run(Q, Kc, Vc, Kn, Vn, Lc)
    assert np.array_equal(got, plain)


@pytest.mark.parametrize("copies", [1, 65])
def test_attention_large_key_offset_and_fewer_queries(copies):
    # a large common vector on every key shifts logits by a per-row constant: exercises the running max
    n, Lc, N, D = 200, 100, 2, 128
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=5)
    shift = wl.round_to_bf16(np.full((1, N, D), 3.0, np.float32))
    Kc2, Kn2 = wl.round_to_bf16(Kc + shift), wl.round_to_bf16(Kn + shift)
    got = _run(Q, Kc2, Vc, Kn2, Vn, 25, Lq=70, copies=copies)
    want = orc.chunk_attention(Q[:70], Kc2, Vc, Kn2, Vn, block_len=25)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)


@pytest.mark.parametrize("D,copies", [(64, 1), (64, 65), (128, 1)])  # (64, 1): the kernel for few queries
@pytest.mark.parametrize("case", ["every tile", "one query", "masked start", "nan query"])
def test_attention_running_maximum_outgrown(D, copies, case):
    # the running maximum is the first tile's until a later tile outgrows it: for all queries of every tile, for single
    # queries of one tile, from a first tile in which a query sees nothing; and a NaN in one query stays in that query
    # (masked start: 12 items per head of 2 to 24 units, the last one of 23: cut in runs of two, those of the second head
    # start in the middle of an item's last 256 keys, of which its first queries see none)
    n, Lc, N = (0, 2900, 2) if case == "masked start" else (700, 96, 2)
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=7 + D)
    bad = []
    if case == "every tile":
        Kc = wl.round_to_bf16(Kc * (0.1 * 2.0 ** (np.arange(n) // 64))[:, None, None].astype(np.float32))
    elif case == "one query":  # keys 70, 400, 690 look at queries 3, 40, 41 with growing weight
        for key, q, gain in ((70, 3, 2.0), (400, 40, 6.0), (690, 41, 20.0)):
            Kc[key] = wl.round_to_bf16(Q[q] * np.float32(gain))
    elif case == "nan query":
        bad = [5, 77]
        Q[bad] = np.nan
    L_B = 1 if case == "masked start" else Lc
    ok = np.setdiff1d(np.arange(Lc), bad)
    want = orc.chunk_attention(np.nan_to_num(Q), Kc, Vc, Kn, Vn, block_len=L_B)
    for ws in (None, attention_workspace(D)):
        got = _run(Q, Kc, Vc, Kn, Vn, L_B, out_dtype=torch.float32, ws=ws, copies=1 if case == "masked start" else copies)
        max_abs, rel = attn_errors(got[ok], want[ok])
        assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)
        assert np.isnan(got[bad]).all()


@pytest.mark.parametrize("D,n,copies", [(64, 384, 1), (64, 384, 65), (128, 384, 1), (128, 330, 1)])  # few, long, long, few
@pytest.mark.parametrize("bits,stairs", [(20, 1), (26, 1), (95, 1), (104, 1), (300, 1), (30, 5), (110, 5)])
def test_attention_reference_raised_by(D, n, copies, bits, stairs):
    # scores that jump by up to `bits` powers of two (less for the first queries) once or in every further tile: below the
    # limit of 2^24, scaled by a power of two (up to 2^100), or computed once more
    Lc, N = 96, 2
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=D + bits + stairs)
    gain = np.linspace(0.1, 1.0, Lc, dtype=np.float32)[:, None, None]
    step = np.float32(bits / (np.log2(np.e) * np.sqrt(D)))
    level = np.clip(np.arange(n) // 64 - 2 if stairs == 1 else np.arange(n) // 64, 0, stairs)
    Q = wl.round_to_bf16(Q * np.float32(0.3) + gain)
    Kc = wl.round_to_bf16(Kc * np.float32(0.3) + (step * level)[:, None, None].astype(np.float32))
    Kn = wl.round_to_bf16(Kn * np.float32(0.3) + step * np.float32(stairs))
    want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=Lc)
    got = _run(Q, Kc, Vc, Kn, Vn, Lc, out_dtype=torch.float32, copies=copies)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)


@pytest.mark.parametrize("N", [2, 130])  # the kernel for few queries, the long one
@pytest.mark.parametrize("D", [64, 128])
def test_attention_strided_slabs(N, D):
    # cache rows live in a slab with spare capacity and a wider token stride
    n, Lc = 150, 70
    Q, Kc, Vc, Kn, Vn = _inputs(n, Lc, N, D, seed=17)
    ld = N * D + 64
    slabK = torch.zeros(n + 10, ld, device=DEV, dtype=torch.bfloat16)
    slabV = torch.zeros(n + 10, ld, device=DEV, dtype=torch.bfloat16)
    slabK[:n, : N * D] = dev(Kc, "bf16").view(n, N * D)
    slabV[:n, : N * D] = dev(Vc, "bf16").view(n, N * D)
    Kv = slabK.as_strided((n, N, D), (ld, D, 1))
    Vv = slabV.as_strided((n, N, D), (ld, D, 1))
    O = torch.empty(Lc, N, D, device=DEV, dtype=torch.bfloat16)
    B.pafu_chunk_attention(dev(Q, "bf16"), Kv, Vv, n, dev(Kn, "bf16"), dev(Vn, "bf16"), 35, O)
    torch.cuda.synchronize()
    want = orc.chunk_attention(Q, Kc, Vc, Kn, Vn, block_len=35)
    max_abs, rel = attn_errors(host(O), want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)


# ------------------------------------------------------------------ index-based Select (Sec. 3.4; Eq. 7)
@pytest.mark.parametrize("n_cache,n_kept,Lc,N,D,L_B,order", [
    (300, 128, 64, 2, 64, 64, "sorted"),       # retained rows = whole tiles
    (300, 100, 64, 2, 64, 16, "sorted"),       # last cache tile mixed with chunk rows
    (1000, 517, 200, 3, 128, 200, "sorted"),
    (1000, 517, 200, 3, 128, 50, "shuffled"),  # the list need not be ascending
    (500, 500, 130, 2, 128, 13, "sorted"),     # everything kept
    (400, 0, 40, 1, 128, 7, "sorted"),         # nothing kept
    (70, 1, 1, 1, 128, 1, "sorted"),
    (5000, 2560, 300, 2, 128, 300, "sorted"),  # many full tiles through the prefetched-id path
    # short calls of many heads: the long kernel
    (300, 128, 64, 130, 64, 64, "sorted"), (300, 100, 64, 130, 64, 16, "shuffled"), (400, 0, 40, 130, 128, 7, "sorted"),
    (300, 100, 64, 130, 128, 16, "shuffled"), (70, 1, 1, 260, 128, 1, "sorted"), (70, 1, 1, 260, 64, 1, "sorted"),
])
def test_gather_attention_matches_oracle_and_the_compacted_path(n_cache, n_kept, Lc, N, D, L_B, order):
    Q, Kc, Vc, Kn, Vn = _inputs(n_cache, Lc, N, D, seed=n_cache + n_kept)
    rng = np.random.default_rng(n_cache * 3 + n_kept)
    ids = np.sort(rng.permutation(n_cache)[:n_kept]).astype(np.int32)
    if order == "shuffled":
        ids = rng.permutation(ids).astype(np.int32)
    d_ids = torch.from_numpy(ids).to(DEV) if n_kept else torch.zeros(4, dtype=torch.int32, device=DEV)
    dQ, dKc, dVc, dKn, dVn = (dev(x, "bf16") for x in (Q, Kc, Vc, Kn, Vn))
    O = torch.full((Lc + 2, N, D), 55.0, device=DEV, dtype=torch.bfloat16)
    B.pafu_chunk_attention_gather(dQ, dKc, dVc, d_ids, n_kept, dKn, dVn, L_B, O[:Lc])
    torch.cuda.synchronize()
    assert torch.all(O[Lc:] == 55.0)
    got = host(O[:Lc])
    want = orc.chunk_attention(Q, Kc[ids], Vc[ids], Kn, Vn, block_len=L_B)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)
    # same arithmetic in the same order as the plain kernel on the compacted cache: identical bits
    plain = _run(Q, Kc[ids], Vc[ids], Kn, Vn, L_B)
    assert np.array_equal(got, plain)


def test_gather_attention_with_equal_runs():
    n_cache, n_kept, Lc, N, D, L_B = 30000, 17000, 600, 4, 128, 200
    Q, Kc, Vc, Kn, Vn = _inputs(n_cache, Lc, N, D, seed=41)
    ids = np.sort(np.random.default_rng(4).permutation(n_cache)[:n_kept]).astype(np.int32)
    ws = attention_workspace(D)
    O = torch.full((Lc + 2, N, D), 55.0, device=DEV, dtype=torch.bfloat16)
    B.pafu_chunk_attention_gather(dev(Q, "bf16"), dev(Kc, "bf16"), dev(Vc, "bf16"), torch.from_numpy(ids).to(DEV), n_kept,
                                  dev(Kn, "bf16"), dev(Vn, "bf16"), L_B, O[:Lc], workspace=ws)
    torch.cuda.synchronize()
    assert torch.all(O[Lc:] == 55.0)
    want = orc.chunk_attention(Q, Kc[ids], Vc[ids], Kn, Vn, block_len=L_B)
    max_abs, rel = attn_errors(host(O[:Lc]), want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)
    # the plain kernel on the compacted cache with the same workspace cuts the work the same way: identical bits
    plain = _run(Q, Kc[ids], Vc[ids], Kn, Vn, L_B, ws=ws)
    assert np.array_equal(host(O[:Lc]), plain)


# few, long, long, few; the ids ring of the long kernel has eight tiles, the last cache tile is mixed with chunk rows
@pytest.mark.parametrize("D,n_kept,copies", [(64, 532, 1), (64, 532, 65), (128, 532, 1), (128, 148, 1)])
def test_gather_attention_clamps_out_of_range_ids(D, n_kept, copies):
    # ids outside the cache must not fault; rows are clamped into range (the result equals attention over those rows)
    n_cache, Lc, N = 700, 64, 2
    Q, Kc, Vc, Kn, Vn = _inputs(n_cache, Lc, N, D, seed=5)
    ids = np.arange(n_kept, dtype=np.int32)
    ids[[3, 63, 70, 127]] = -9, n_cache, 10 ** 6, -2 ** 31
    ids[[n_kept - 1, n_kept - 3, n_kept - 20]] = n_cache, -1, 2 ** 31 - 1
    if n_kept > 512:
        ids[[448, 449, 511]] = -2 ** 31, 2 ** 31 - 1, -1
    eff = np.clip(ids, 0, n_cache - 1)
    O = torch.empty(Lc, N * copies, D, device=DEV, dtype=torch.bfloat16)
    up = lambda x: dev(x, "bf16").repeat(1, copies, 1)
    B.pafu_chunk_attention_gather(up(Q), up(Kc), up(Vc), torch.from_numpy(ids).to(DEV), n_kept, up(Kn), up(Vn), Lc, O)
    torch.cuda.synchronize()
    got = _first_copy(O, N)
    want = orc.chunk_attention(Q, Kc[eff], Vc[eff], Kn, Vn, block_len=Lc)
    max_abs, rel = attn_errors(got, want)
    assert max_abs < ATTN_MAX_ABS and rel < ATTN_REL_FRO, (max_abs, rel)
    assert np.array_equal(got, _run(Q, Kc[eff], Vc[eff], Kn, Vn, Lc, copies=copies))
