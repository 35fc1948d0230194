"""GPU parity of each kernel of the step, through the C ABI, against the oracle.

* scoring + selection: bit-exact scores, index sets and position map (Eqs. 2,
  6, 7; Algorithm 1 SSC), including ties, NaN, quota 0 / N and ragged batches,
  up to 32768 tokens per sample;
* projections (MFMA GEMM, each epilogue) and attention (self, ragged varlen,
  cross with a non-tile-multiple key count) against float64 on the same
  bf16-rounded operands; bf16 bound 2e-2 max-rel, f32 bound 1e-4;
* LayerNorm/modulation and the timestep modulation path;
* gather + embedding and the final LayerNorm + output projection against
  float64; merge + Euler + cache rotation bit-exact against the oracle step.
"""
import numpy as np
import pytest

from helpers import (F32_GEMM_TILES, GEMM_TILES, bf16_round, gemm_f32_tile, gemm_tile, max_rel, oracle_selection, say,
                     to_dev)
from oracle import dit, ssc
from paper_2511_22533_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    from paper_2511_22533_amd import f3c
    f3c.lib()
    return t


def _run_select(torch, vc, vp, n_cache, omega):
    from paper_2511_22533_amd import f3c
    B, N = vc.shape[:2]
    total = int(sum(N - c for c in n_cache))
    d_vc, d_vp = to_dev(vc), to_dev(vp)
    idx = torch.full((max(total, 1),), -7, dtype=torch.int32, device="cuda")
    pos = torch.full((B, N), -7, dtype=torch.int32, device="cuda")
    score = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    f3c.op_select(d_vc, d_vp, omega, n_cache, idx, pos, score)
    torch.cuda.synchronize()
    return idx.cpu().numpy()[:total], pos.cpu().numpy(), score.cpu().numpy()


def _check_select(torch, vc, vp, n_cache, omega=0.7):
    B, N = vc.shape[:2]
    idx, pos, score = _run_select(torch, vc, vp, n_cache, omega)
    ref = oracle_selection(vc, vp, n_cache, omega)
    row = 0
    for b in range(B):
        s_ref, active = ref[b]
        n = len(active)
        assert n == N - n_cache[b]
        assert np.array_equal(idx[row:row + n], active), f"sample {b}"
        want_pos = np.full(N, -1, np.int64)
        want_pos[active] = row + np.arange(n)
        assert np.array_equal(pos[b], want_pos), f"sample {b}"
        if s_ref is not None:
            assert np.array_equal(score[b].view(np.uint32), s_ref.view(np.uint32)), f"scores sample {b}"
        row += n


@pytest.mark.parametrize("B,N", [(1, 512), (1, 4096), (4, 4096), (1, 32768), (3, 1000), (2, 1), (5, 3000), (16, 32768)])
def test_select_bit_exact_random(torch, B, N):
    rng = np.random.default_rng(N + B)
    vc = rng.standard_normal((B, N, 8)).astype(np.float32)
    vp = (vc + 0.1 * rng.standard_normal((B, N, 8))).astype(np.float32)
    for quotas in ([0] * B, [N] * B, [1] * B, [N - 1] * B,
                   [int(q) for q in rng.integers(0, N + 1, size=B)],
                   [int(N * f) for f in np.linspace(0.4, 0.85, B)]):
        say("select", B, N, quotas)
        _check_select(torch, vc, vp, quotas)


@pytest.mark.parametrize("omega", [0.0, 0.3, 0.7, 1.0])
def test_select_ties_and_sticky_cache(torch, omega):
    rng = np.random.default_rng(11)
    B, N = 2, 4096
    vc = (rng.integers(-2, 3, size=(B, N, 8)) * 0.5).astype(np.float32)   # many equal scores
    vp = vc.copy()
    moved = rng.random((B, N)) < 0.3
    vp[moved] += 0.5                                                      # A = 0 for the rest
    say("select ties", omega)
    _check_select(torch, vc, vp, [1000, 3000], omega)


def test_select_degenerate_and_nan(torch):
    B, N = 3, 2048
    vc = np.ones((B, N, 8), np.float32)
    vp = np.ones((B, N, 8), np.float32)             # max == min for both terms
    rng = np.random.default_rng(3)
    vc[1] = rng.standard_normal((N, 8)).astype(np.float32)
    vp[1] = rng.standard_normal((N, 8)).astype(np.float32)
    vc[1, 17, 3] = np.nan
    vc[1, 900, :] = np.inf
    vc[2] = rng.standard_normal((N, 8)).astype(np.float32)
    vp[2] = vc[2]
    say("select degenerate/nan")
    _check_select(torch, vc, vp, [100, 1500, 2047])


# The selection alone from given scores (f3c_op_select_scores) against the
# oracle's stable sort of the same scores: ragged quotas including 0, 1, N - 1
# and N; heavy ties (a few distinct values), NaN, +-inf, +-0 and subnormals.
@pytest.mark.parametrize("B,N", [(1, 1), (3, 1000), (4, 4096), (2, 32768)])
def test_select_from_given_scores(torch, B, N):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(7 * N + B)
    cases = {
        "continuous": rng.standard_normal((B, N)).astype(np.float32),
        "ties": (rng.integers(0, 5, size=(B, N)) * 0.25).astype(np.float32),
    }
    special = rng.random((B, N)).astype(np.float32)
    picks = rng.integers(0, N, size=(B, 6 * max(1, N // 64)))
    for b in range(B):
        for j, i in enumerate(picks[b]):
            special[b, i] = [np.nan, np.inf, -np.inf, 0.0, -0.0, np.float32(1e-45)][j % 6]
    cases["special"] = special
    for name, sc in cases.items():
        quota_sets = [[0] * B, [N] * B, [min(1, N)] * B, [max(N - 1, 0)] * B,
                      [int(q) for q in rng.integers(0, N + 1, size=B)]]
        for quotas in quota_sets:
            say("select scores", name, B, N, quotas)
            tot = sum(N - c for c in quotas)
            idx = torch.full((max(tot, 1),), -7, dtype=torch.int32, device="cuda")
            pos = torch.full((B, N), -7, dtype=torch.int32, device="cuda")
            f3c.op_select_scores(to_dev(sc), quotas, idx, pos)
            torch.cuda.synchronize()
            got_idx, got_pos = idx.cpu().numpy(), pos.cpu().numpy()
            row = 0
            for b in range(B):
                _, active = ssc.select(sc[b], quotas[b])
                n = len(active)
                assert np.array_equal(got_idx[row:row + n], active), (name, quotas, b)
                want_pos = np.full(N, -1, np.int64)
                want_pos[active] = row + np.arange(n)
                assert np.array_equal(got_pos[b], want_pos), (name, quotas, b)
                row += n


def _gemm_case(torch, dt, epi, M, N, K, seed):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = (0.05 * rng.standard_normal((N, K))).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    gate = rng.standard_normal(N).astype(np.float32)
    if dt == f3c.F3C_BF16:
        A, W = bf16_round(A), bf16_round(W)
        tdt = torch.bfloat16
    else:
        tdt = torch.float32
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    dA, dW, db, dg = to_dev(A, tdt), to_dev(W, tdt), to_dev(bias), to_dev(gate)
    say("gemm", dt, epi, M, N, K)
    if epi == 2:
        r0 = rng.standard_normal((M, N)).astype(np.float32)
        dr = to_dev(r0)
        f3c.op_gemm(dt, 2, dA, dW, db, resid=dr, gate=dg)
        torch.cuda.synchronize()
        got = dr.cpu().numpy().astype(np.float64) - r0
        want = gate * ref
    else:
        out = torch.empty((M, N), dtype=tdt, device="cuda")
        f3c.op_gemm(dt, epi, dA, dW, db, out=out)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        want = dit.gelu_tanh(ref) if epi == 1 else ref
    return got, want


# Few and ragged rows, one and several column tiles, one K tile and many (the tile
# shapes follow the size: see gemm_tile; the tests below cross all of them).
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (37, 384, 128), (128, 1024, 1024), (820, 3072, 1024),
                                   (4096, 1024, 4096), (2057, 4096, 1024), (1310, 3072, 1024)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_bf16(torch, M, N, K, epi):
    from paper_2511_22533_amd import f3c
    got, want = _gemm_case(torch, f3c.F3C_BF16, epi, M, N, K, seed=M * 7 + N + epi)
    assert max_rel(got, want) < 1e-2


# Long K: ragged M, few rows, every epilogue, and bit-reproducible
# repeats.
@pytest.mark.parametrize("M,N,K", [(1, 128, 4096), (37, 1024, 4096), (820, 1024, 4096), (1500, 1024, 4096),
                                   (2048, 1024, 4096), (300, 2048, 8192)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_bf16_long_k(torch, M, N, K, epi):
    from paper_2511_22533_amd import f3c
    got, want = _gemm_case(torch, f3c.F3C_BF16, epi, M, N, K, seed=M + K + epi)
    assert max_rel(got, want) < 1e-2
    got2, _ = _gemm_case(torch, f3c.F3C_BF16, epi, M, N, K, seed=M + K + epi)
    assert np.array_equal(got, got2)


def _gemm_big_case(torch, epi, M, N, K, seed, rows=None):
    """bf16 projection at many rows; the float64 reference on sampled rows."""
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(seed)
    A = bf16_round(rng.standard_normal((M, K)).astype(np.float32))
    W = bf16_round((0.05 * rng.standard_normal((N, K))).astype(np.float32))
    bias = rng.standard_normal(N).astype(np.float32)
    gate = rng.standard_normal(N).astype(np.float32)
    dA, dW, db, dg = to_dev(A, torch.bfloat16), to_dev(W, torch.bfloat16), to_dev(bias), to_dev(gate)
    say("gemm big", epi, M, N, K)
    if epi == 2:
        r0 = rng.standard_normal((M, N)).astype(np.float32)
        dr = to_dev(r0)
        f3c.op_gemm(f3c.F3C_BF16, 2, dA, dW, db, resid=dr, gate=dg)
        torch.cuda.synchronize()
        got = dr.cpu().numpy()
        base = r0
    else:
        out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        f3c.op_gemm(f3c.F3C_BF16, epi, dA, dW, db, out=out)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        base = None
    if rows is None:
        rows = np.unique(np.concatenate([rng.choice(M, 384, replace=False), np.arange(M - 130, M)]))
    ref = A[rows].astype(np.float64) @ W.astype(np.float64).T + bias
    if epi == 2:
        return got, (got[rows].astype(np.float64) - base[rows], gate * ref)
    return got, (got[rows], dit.gelu_tanh(ref) if epi == 1 else ref)


# Many rows (the 32^3 workload's active sets), on 256 x 256 and 256 x 128 tiles:
# ragged row counts, every epilogue, sampled rows against float64.
@pytest.mark.parametrize("M,N,K", [(8300, 3072, 1024), (9831, 1024, 4096), (16500, 1024, 4096),
                                   (9831, 4096, 1024), (16400, 4096, 1024)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_bf16_many_rows(torch, M, N, K, epi):
    _, (got, want) = _gemm_big_case(torch, epi, M, N, K, seed=M + epi)
    assert max_rel(got, want) < 1e-2


# The tile choice moves with the row count, not the results: every tile shape
# sums K in the same order with the same instruction, so runs on different tiles
# agree bit for bit in the rows they share. The row counts take all five tiles, for
# every epilogue and over 32 and 64 K tiles.
@pytest.mark.parametrize("N,K,rows", [(1024, 4096, (9831, 8191, 4096, 2047, 820)),
                                      (512, 2048, (16400, 9831, 8191, 4095, 2048))])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_bf16_tile_switch_bit_identical(torch, N, K, rows, epi):
    from paper_2511_22533_amd import f3c
    assert {gemm_tile(m, N, K, epi) for m in rows} == set(range(len(GEMM_TILES)))
    M = rows[0]
    rng = np.random.default_rng(M + N + epi)
    A = to_dev(rng.standard_normal((M, K)).astype(np.float32), torch.bfloat16)
    W = to_dev((0.05 * rng.standard_normal((N, K))).astype(np.float32), torch.bfloat16)
    bias = to_dev(rng.standard_normal(N).astype(np.float32))
    gate = to_dev(rng.standard_normal(N).astype(np.float32))
    whole = None
    for m in rows:
        say("gemm tile switch", epi, m, N, K, GEMM_TILES[gemm_tile(m, N, K, epi)])
        if epi == 2:
            r = torch.zeros((m, N), dtype=torch.float32, device="cuda")
            f3c.op_gemm(f3c.F3C_BF16, 2, A[:m], W, bias, resid=r, gate=gate)
        else:
            r = torch.empty((m, N), dtype=torch.bfloat16, device="cuda")
            f3c.op_gemm(f3c.F3C_BF16, epi, A[:m], W, bias, out=r)
        torch.cuda.synchronize()
        if whole is None:
            whole = r
        assert torch.equal(r.view(torch.int32 if epi == 2 else torch.int16),
                           whole[:m].view(torch.int32 if epi == 2 else torch.int16)), m


# The same at the edges of tiles, with short K and column counts that the wider
# tiles do not divide, and in f32: a prefix of the rows gives a prefix of the
# result. (Plain stores of 1024 columns take all five tiles, f32 calls of 640 columns
# all three.)
@pytest.mark.parametrize("dt_name,N,K", [("bf16", 1024, 1024), ("bf16", 384, 64), ("bf16", 640, 192),
                                         ("f32", 384, 32), ("f32", 640, 96)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_row_prefix_bit_identical(torch, dt_name, N, K, epi):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(N + K + epi)
    M = 9831
    dt, tdt = (f3c.F3C_BF16, torch.bfloat16) if dt_name == "bf16" else (f3c.F3C_F32, torch.float32)
    A = to_dev(rng.standard_normal((M, K)).astype(np.float32), tdt)
    W = to_dev((0.05 * rng.standard_normal((N, K))).astype(np.float32), tdt)
    bias = to_dev(rng.standard_normal(N).astype(np.float32))

    def run(rows):
        say("gemm rows", dt_name, epi, rows, N, K)
        r = torch.zeros((rows, N), dtype=torch.float32 if epi == 2 else tdt, device="cuda")
        f3c.op_gemm(dt, epi, A[:rows], W, bias, **({"resid": r} if epi == 2 else {"out": r}))
        torch.cuda.synchronize()
        return r

    shapes = {gemm_tile(m, N, K, epi) if dt_name == "bf16" else gemm_f32_tile(m, N, K)
              for m in (M, 1, 63, 64, 65, 333, 1639, 2100, 4097, 6000)}
    assert (dt_name, N, epi) != ("bf16", 1024, 0) or shapes == set(range(len(GEMM_TILES)))
    assert (dt_name, N) != ("f32", 640) or shapes == set(range(len(F32_GEMM_TILES)))
    whole = run(M)
    ref = A[::29].double().cpu().numpy() @ W.double().cpu().numpy().T + bias.double().cpu().numpy()
    tol = 1e-2 if dt_name == "bf16" else 1e-5
    assert max_rel(whole[::29].double().cpu().numpy(), dit.gelu_tanh(ref) if epi == 1 else ref) < tol
    for rows in (1, 63, 64, 65, 333, 1639, 2100, 4097, 6000):
        assert torch.equal(run(rows), whole[:rows]), rows


# Output rows aligned to 8 bytes only, and row strides beyond what 32-bit offsets
# span within a tile.
@pytest.mark.parametrize("epi", [0, 1])
@pytest.mark.parametrize("pad,stride", [(4, 0), (0, (1 << 22) + 8), (12, (1 << 22) + 8)])
def test_gemm_bf16_strides(torch, epi, pad, stride):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(pad + epi)
    M, N, K = 67, 256, 192
    a = to_dev(rng.standard_normal((M, K)).astype(np.float32), torch.bfloat16)
    W = to_dev((0.05 * rng.standard_normal((N, K))).astype(np.float32), torch.bfloat16)
    bias = to_dev(rng.standard_normal(N).astype(np.float32))
    want = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    f3c.op_gemm(f3c.F3C_BF16, epi, a, W, bias, out=want)
    if stride:
        A = torch.zeros(((M - 1) * stride + K,), dtype=torch.bfloat16, device="cuda").as_strided((M, K), (stride, 1))
        A.copy_(a)
    else:
        A = a
    out = torch.full((M, N + pad), 7.0, dtype=torch.bfloat16, device="cuda")
    say("gemm strides", epi, pad, stride)
    f3c.op_gemm(f3c.F3C_BF16, epi, A, W, bias, out=out[:, :N])
    torch.cuda.synchronize()
    assert torch.equal(out[:, :N], want) and bool((out[:, N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [(1, 128, 32), (300, 384, 128), (513, 512, 128)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_f32(torch, M, N, K, epi):
    from paper_2511_22533_amd import f3c
    got, want = _gemm_case(torch, f3c.F3C_F32, epi, M, N, K, seed=M + N + K + epi)
    assert max_rel(got, want) < 1e-5


def _attn_case(torch, dt, heads, hd, q_lens, k_lens, seed, sample_queries=None, workspace=False, outputs=None,
               key_ramp=0.0, prescaled=False):
    """key_ramp > 0 scales key j of each sample by 1 + key_ramp * (j // 64): every
    64-key tile then has larger scores than the ones before it. prescaled: the
    queries go in multiplied by log2(e)/sqrt(hd) (rounded once, as the step's
    projections store them) and the reference takes the stored values divided
    by that factor."""
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(seed)
    d = heads * hd
    q_off = np.concatenate([[0], np.cumsum(q_lens)]).astype(int)
    k_off = np.concatenate([[0], np.cumsum(k_lens)]).astype(int)
    q = (1.5 * rng.standard_normal((q_off[-1], d))).astype(np.float32)
    k = (1.5 * rng.standard_normal((k_off[-1], d))).astype(np.float32)
    v = rng.standard_normal((k_off[-1], d)).astype(np.float32)
    if key_ramp:
        j = np.concatenate([np.arange(n) for n in k_lens]) if k_off[-1] else np.zeros(0, int)
        k *= (1.0 + key_ramp * (j // 64)).astype(np.float32)[:, None]
    tdt = torch.bfloat16 if dt == f3c.F3C_BF16 else torch.float32
    cq = f3c.attention_q_scale(hd) if prescaled else 1.0
    q_in = (q * np.float32(cq)).astype(np.float32)
    if dt == f3c.F3C_BF16:
        q_in, k, v = bf16_round(q_in), bf16_round(k), bf16_round(v)
    q = (q_in.astype(np.float64) / cq) if prescaled else q_in     # what the kernel's input means
    o = torch.zeros((max(q_off[-1], 1), d), dtype=tdt, device="cuda")
    ws = torch.empty(8 << 20, dtype=torch.float32, device="cuda") if workspace else None
    say("attention", dt, heads, hd, list(q_lens), list(k_lens), "workspace" if workspace else "")
    f3c.op_attention(dt, heads, hd, q_off.tolist(), k_off.tolist(), to_dev(q_in, tdt), to_dev(k, tdt),
                     to_dev(v, tdt), o, workspace=ws, q_prescaled=prescaled)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy()
    if outputs is not None:
        outputs.append(got)
    worst = 0.0
    for b in range(len(q_lens)):
        if q_lens[b] == 0:
            continue
        rows = np.arange(q_off[b], q_off[b + 1])
        if sample_queries and len(rows) > sample_queries:
            rows = np.sort(rng.choice(rows, sample_queries, replace=False))
        kk = k[k_off[b]:k_off[b + 1]].astype(np.float64)
        vv = v[k_off[b]:k_off[b + 1]].astype(np.float64)
        want = dit.attention(q[rows].astype(np.float64), kk, vv, heads)
        worst = max(worst, max_rel(got[rows], want))
    return worst


# 1024 and 1025 queries sit on either side of the switch from four-wave to
# eight-wave key-group workgroups (16 x 16 = 256 workgroups of 64 queries is
# the last grid that fits one round).
@pytest.mark.parametrize("q_lens,k_lens", [([64], [64]), ([1], [1]), ([200], [200]), ([0, 37, 300], [0, 37, 300]),
                                           ([820], [820]), ([615, 1536, 2458, 1003], [615, 1536, 2458, 1003]),
                                           ([1024], [1024]), ([1025], [1025])])
@pytest.mark.parametrize("prescaled", [False, True])
def test_self_attention_bf16(torch, q_lens, k_lens, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, k_lens, seed=sum(q_lens), prescaled=prescaled) < 2e-2


@pytest.mark.parametrize("prescaled", [False, True])
def test_self_attention_bf16_full_size_sampled(torch, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, [4096], [4096], seed=5, sample_queries=96,
                      prescaled=prescaled) < 2e-2
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, [9831], [9831], seed=6, sample_queries=64,
                      prescaled=prescaled) < 2e-2


@pytest.mark.parametrize("q_lens", [[820], [5, 1000, 0, 77]])
@pytest.mark.parametrize("prescaled", [False, True])
def test_cross_attention_bf16(torch, q_lens, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, [1374] * len(q_lens), seed=len(q_lens),
                      prescaled=prescaled) < 2e-2


# With a workspace, launches with few query tiles may split the key range
# over workgroups and merge the partial results in a fixed order; they do
# when that shortens each wave's chain of key tiles by more than five tiles
# against two key groups in one workgroup. Chosen for these cases (bf16, 16
# heads): key groups of four waves for the first four, 4 splits, 8 splits,
# key groups of eight waves, key groups of four waves.
@pytest.mark.parametrize("q_lens,k_lens", [([1000], [1000]), ([820], [1374]), ([5, 300, 0, 77], [1374] * 4),
                                           ([300], [1374]), ([1, 40], [4096, 2000]), ([64], [8192]),
                                           ([1310], [1310]), ([820], [820])])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_bf16_split_keys(torch, q_lens, k_lens, prescaled):
    from paper_2511_22533_amd import f3c
    outs = []
    for rep in range(2):
        assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, k_lens, seed=sum(k_lens), workspace=True,
                          outputs=outs, prescaled=prescaled) < 2e-2
    assert np.array_equal(outs[0], outs[1])


# Scores that grow from tile to tile: the running reference max of the
# matrix-core path is too small for later tiles, so its fix-up branch
# (rescale what was accumulated, redo the tile) runs, for some queries of a
# wave and not others; in the four-wave key-group, eight-wave and key-split
# (300 x 4096 keys: 4 splits) launches.
@pytest.mark.parametrize("q_lens,k_lens,ramp,ws", [([300], [300], 2.0, False), ([1000], [1000], 0.5, False),
                                                   ([820], [1374], 1.0, False), ([300], [4096], 0.5, True),
                                                   ([37, 3000], [37, 3000], 0.3, False), ([640], [640], 0.12, False)])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_bf16_growing_scores(torch, q_lens, k_lens, ramp, ws, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, k_lens, seed=int(10 * ramp) + len(q_lens),
                      workspace=ws, key_ramp=ramp, sample_queries=128, prescaled=prescaled) < 2e-2


# Waves of 64 queries (from 12 key tiles up): workgroups of 512 queries (6000 and
# 6400), of 256 (9000), partial waves and blocks at their end, one more key than
# 12 and 13 whole tiles; a second sample of one query. With a ramp the sums
# overflow after some tiles and the workgroup starts over.
@pytest.mark.parametrize("q_lens,k_lens,ramp", [([6000], [769], 0.0), ([6400], [833], 0.0), ([9000], [705], 0.0),
                                                ([9011, 1], [1374, 800], 0.0), ([6000], [1374], 1.0),
                                                ([9000], [1000], 2.0)])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_bf16_wide_waves(torch, q_lens, k_lens, ramp, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, k_lens, seed=sum(q_lens) + sum(k_lens), key_ramp=ramp,
                      sample_queries=96, prescaled=prescaled) < 2e-2


# Scores (base 2) near `level` for every key: above and below what a raw pass
# takes from its first tile, for a few queries or all of them. And queries that
# are NaN or infinite, which change no other query of their wave. One launch per
# shape: 64 and 128 queries with key groups, 256 and 512, key splits.
@pytest.mark.parametrize("n,nk", [(820, 900), (1639, 900), (3000, 900), (9000, 900), (6000, 900), (200, 4096)])
@pytest.mark.parametrize("level,bad", [(90.0, False), (-90.0, False), (20.0, True)])
def test_attention_bf16_score_range(torch, n, nk, level, bad):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(n)
    heads, d = 16, 1024
    q = rng.standard_normal((n, heads, 64)) * 0.2
    k = rng.standard_normal((nk, heads, 64))
    q[:, :, 0] = np.where(rng.random(n) < 0.02, level / 8, 0.5)[:, None] if not bad else level / 8
    k[:, :, 0] = 8.0
    q, k = (bf16_round(a.reshape(-1, d).astype(np.float32)) for a in (q, k))
    v = bf16_round(rng.standard_normal((nk, d)).astype(np.float32))
    hurt = np.zeros(n, bool)
    if bad:
        hurt[[5, 40, n // 2, n - 1]] = True
        q[[5, n // 2]] = np.nan
        q[[40, n - 1]] = np.inf
    o = torch.zeros((n, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(8 << 20, dtype=torch.float32, device="cuda")
    say("attention range", n, nk, level, bad)
    f3c.op_attention(f3c.F3C_BF16, heads, 64, [0, n], [0, nk], to_dev(q, torch.bfloat16), to_dev(k, torch.bfloat16),
                     to_dev(v, torch.bfloat16), o, workspace=ws, q_prescaled=True)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy()
    assert np.isnan(got[hurt]).all()
    near = np.unique(np.concatenate([np.flatnonzero(~hurt)[:80], np.flatnonzero(q[:, 0] > 1)[:40],
                                     rng.choice(n, 60)]))
    rows = near[~hurt[near]]
    want = dit.attention(q[rows].astype(np.float64) * 8 * np.log(2.0), k.astype(np.float64), v.astype(np.float64), heads)
    assert max_rel(got[rows], want) < 2e-2


# Values near both ends of bf16's range, with scores (base 2) near `level` for
# every key or, late, for all but the first tile's: what the kernels keep
# unnormalised must neither overflow nor underflow. One launch per shape, as
# above, and key ranges of one and two tiles; the values are 2^vexp N(0, 1).
@pytest.mark.parametrize("n,nk", [(820, 900), (1639, 900), (3000, 900), (9000, 900), (6000, 900), (200, 4096),
                                  (300, 64), (300, 128)])
@pytest.mark.parametrize("level,late,vexp", [(34.0, False, 100), (60.0, True, 100), (110.0, True, 100),
                                             (150.0, True, 100), (-34.0, False, -100), (-14.0, False, -100)])
def test_attention_bf16_value_range(torch, n, nk, level, late, vexp):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(n)
    heads, d = 16, 1024
    q = rng.standard_normal((n, heads, 64)) * 0.2
    k = rng.standard_normal((nk, heads, 64))
    q[:, :, 0] = level / 8
    k[:, :, 0] = 8.0
    if late:
        k[:64, :, 0] = 0.0
    q, k = (bf16_round(a.reshape(-1, d).astype(np.float32)) for a in (q, k))
    v = bf16_round(np.ldexp(rng.standard_normal((nk, d)), vexp).astype(np.float32))
    o = torch.zeros((n, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(8 << 20, dtype=torch.float32, device="cuda")
    say("attention values", n, nk, level, late, vexp)
    f3c.op_attention(f3c.F3C_BF16, heads, 64, [0, n], [0, nk], to_dev(q, torch.bfloat16), to_dev(k, torch.bfloat16),
                     to_dev(v, torch.bfloat16), o, workspace=ws, q_prescaled=True)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(40), rng.choice(n, 40), [n - 1]]))
    want = dit.attention(q[rows].astype(np.float64) * 8 * np.log(2.0), k.astype(np.float64), v.astype(np.float64), heads)
    assert max_rel(o.float().cpu().numpy()[rows], want) < 2e-2


# Two key groups with one or two key tiles: the second group's only tile lies
# past the end (all keys masked) or is the ragged last one; four-wave
# workgroups up to 1024 queries, eight-wave ones in the last two cases (1100
# queries to one key tile go without key groups).
@pytest.mark.parametrize("q_lens,k_lens", [([600], [50]), ([600], [64]), ([700], [100]), ([5, 600], [1, 65]),
                                           ([1100], [50]), ([1100], [100]), ([1000, 100], [100, 50])])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_bf16_key_groups_short_keys(torch, q_lens, k_lens, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 16, 64, q_lens, k_lens, seed=sum(k_lens), prescaled=prescaled) < 2e-2


@pytest.mark.parametrize("hd,heads", [(32, 4), (64, 2)])
def test_attention_f32_split_keys(torch, hd, heads):
    from paper_2511_22533_amd import f3c
    # 2 key splits
    assert _attn_case(torch, f3c.F3C_F32, heads, hd, [512, 70], [2048, 1100], seed=hd, workspace=True) < 1e-4


@pytest.mark.parametrize("hd,heads", [(32, 4), (64, 2)])
@pytest.mark.parametrize("q_lens,k_lens", [([512], [512]), ([3, 256, 130], [64, 64, 64]), ([100], [1])])
@pytest.mark.parametrize("prescaled", [False, True])
def test_attention_f32(torch, hd, heads, q_lens, k_lens, prescaled):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_F32, heads, hd, q_lens, k_lens, seed=hd + len(q_lens),
                      prescaled=prescaled) < 1e-4


def test_attention_f32_eight_waves_sampled(torch):
    # enough query tiles (21 x 8 heads) for the 8-wave workgroup
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_F32, 8, 64, [5200], [5200], seed=11, sample_queries=64) < 1e-4


def test_attention_bf16_hd32(torch):
    from paper_2511_22533_amd import f3c
    assert _attn_case(torch, f3c.F3C_BF16, 4, 32, [300, 64], [300, 64], seed=9) < 2e-2


@pytest.mark.parametrize("dt_name,d", [("f32", 128), ("bf16", 1024), ("bf16", 2048)])
def test_ln_mod(torch, dt_name, d):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(d)
    rows = 333
    h = (3 * rng.standard_normal((rows, d)) + 1).astype(np.float32)
    shift = rng.standard_normal(d).astype(np.float32)
    scale = rng.standard_normal(d).astype(np.float32)
    dt = f3c.F3C_BF16 if dt_name == "bf16" else f3c.F3C_F32
    tdt = torch.bfloat16 if dt_name == "bf16" else torch.float32
    for mod in (True, False):
        out = torch.empty((rows, d), dtype=tdt, device="cuda")
        say("ln", dt_name, d, mod)
        f3c.op_ln_mod(dt, to_dev(h), out, to_dev(shift) if mod else None, to_dev(scale) if mod else None)
        torch.cuda.synchronize()
        want = dit.layer_norm(h.astype(np.float64))
        if mod:
            want = want * (1 + scale) + shift
        tol = 8e-3 if dt_name == "bf16" else 1e-5
        assert max_rel(out.float().cpu().numpy(), want) < tol


@pytest.mark.parametrize("cfg", [synth.TINY, synth.ModelConfig(grid=4, width=1024, depth=3, heads=16, cond_tokens=8,
                                                              cond_width=64, dtype="bf16")])
def test_modulation(torch, cfg):
    from paper_2511_22533_amd import f3c
    W = synth.make_weights(cfg, seed=2, scale=0.05)
    m = f3c.Model(cfg).load(W)
    om = dit.Model(cfg, W)
    for t in (1.0, 0.73, 0.111, 0.0):
        say("modulation", cfg.dtype, t)
        got = m.modulation(t).cpu().numpy()
        torch.cuda.synchronize()
        tol = 1e-4 if cfg.dtype == "f32" else 5e-3
        assert max_rel(got, om.modulation(t)) < tol


_EMBED_CFGS = [synth.TINY, synth.ModelConfig(grid=16, width=1024, depth=1, heads=16, cond_tokens=8, cond_width=64,
                                             dtype="bf16")]


@pytest.mark.parametrize("cfg", _EMBED_CFGS, ids=["tiny_f32", "g16_w1024_bf16"])
def test_embed_gather(torch, cfg):
    from paper_2511_22533_amd import f3c
    W = synth.make_weights(cfg, seed=4, scale=0.05)
    m = f3c.Model(cfg).load(W)
    om = dit.Model(cfg, W)
    N, d = cfg.grid ** 3, cfg.width
    rng = np.random.default_rng(17)
    B = 3
    x = rng.standard_normal((B, N, 8)).astype(np.float32)
    # ragged active sets: a large one, a tiny one, an empty one (ascending indices)
    sets = [np.sort(rng.choice(N, N - N // 5, replace=False)), np.array([0, N - 1]), np.zeros(0, np.int64)]
    off = np.concatenate([[0], np.cumsum([len(a) for a in sets])]).astype(int)
    idx = np.concatenate(sets).astype(np.int32)
    h = torch.full((off[-1], d), float("nan"), dtype=torch.float32, device="cuda")
    say("embed", cfg.dtype, off.tolist())
    f3c.op_embed(m, to_dev(x), off.tolist(), h, idx_active=to_dev(idx))
    torch.cuda.synchronize()
    got = h.cpu().numpy()
    for b in range(B):
        if len(sets[b]):
            want = om.embed(x[b][sets[b]], sets[b])
            assert max_rel(got[off[b]:off[b + 1]], want) < 1e-5
    # identity gather (full step): every token of each sample, no index list
    h2 = torch.empty((2 * N, d), dtype=torch.float32, device="cuda")
    say("embed identity", cfg.dtype)
    f3c.op_embed(m, to_dev(x[:2]), [0, N, 2 * N], h2)
    torch.cuda.synchronize()
    got2 = h2.cpu().numpy()
    for b in range(2):
        assert max_rel(got2[b * N:(b + 1) * N], om.embed(x[b], np.arange(N))) < 1e-5


@pytest.mark.parametrize("cfg", _EMBED_CFGS, ids=["tiny_f32", "g16_w1024_bf16"])
@pytest.mark.parametrize("rows", [1, 333])
def test_final_projection(torch, cfg, rows):
    from paper_2511_22533_amd import f3c
    W = synth.make_weights(cfg, seed=5, scale=0.05)
    m = f3c.Model(cfg).load(W)
    rng = np.random.default_rng(rows)
    h = (2 * rng.standard_normal((rows, cfg.width)) + 0.5).astype(np.float32)
    v = torch.full((rows, 8), float("nan"), dtype=torch.float32, device="cuda")
    say("final", cfg.dtype, rows)
    f3c.op_final(m, to_dev(h), v)
    torch.cuda.synchronize()
    want = dit.linear(dit.layer_norm(h.astype(np.float64)), W["out_w"], W["out_b"])
    assert max_rel(v.cpu().numpy(), want) < 1e-5


@pytest.mark.parametrize("N,n_cache", [(512, [0, 100, 512]), (4096, [3276, 0]), (32768, [22937])])
def test_euler_merge_rotate_bit_exact(torch, N, n_cache):
    """Merge + Euler + rotation equal the oracle's step bit for bit, with the
    oracle's own selection and the same fresh velocities for the active rows."""
    from oracle import sampler
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(N)
    B = len(n_cache)
    x = rng.standard_normal((B, N, 8)).astype(np.float32)
    vc = rng.standard_normal((B, N, 8)).astype(np.float32)
    vp = rng.standard_normal((B, N, 8)).astype(np.float32)
    sel = oracle_selection(vc, vp, n_cache)
    act = [a for _, a in sel]
    off = np.concatenate([[0], np.cumsum([len(a) for a in act])]).astype(int)
    v_act = rng.standard_normal((max(off[-1], 1), 8)).astype(np.float32)
    pos = np.full((B, N), -1, np.int32)
    for b in range(B):
        pos[b, act[b]] = off[b] + np.arange(len(act[b]))
    t, t_next = 0.7310585786, 0.6224593312
    st = sampler.State(x.copy(), vc.copy(), vp.copy())
    sampler.step(st, lambda b, xa, idx, tt: v_act[off[b]:off[b + 1]], t, t_next, n_cache)
    d_x, d_vn = to_dev(x), torch.full((B, N, 8), float("nan"), dtype=torch.float32, device="cuda")
    say("euler", N, n_cache)
    f3c.op_euler(d_x, to_dev(vc), to_dev(v_act), to_dev(pos), off.tolist(), t, t_next, d_vn)
    torch.cuda.synchronize()
    assert np.array_equal(d_x.cpu().numpy(), st.x)
    assert np.array_equal(d_vn.cpu().numpy(), st.v_cache)


def test_euler_all_active_without_pos(torch):
    from oracle import sampler
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(3)
    B, N = 2, 512
    x = rng.standard_normal((B, N, 8)).astype(np.float32)
    vc = rng.standard_normal((B, N, 8)).astype(np.float32)
    v_act = rng.standard_normal((B * N, 8)).astype(np.float32)
    st = sampler.State(x.copy(), vc.copy(), vc.copy())
    sampler.step(st, lambda b, xa, idx, tt: v_act[b * N:(b + 1) * N], 1.0, 0.96, [0, 0])
    d_x, d_vn = to_dev(x), torch.empty((B, N, 8), dtype=torch.float32, device="cuda")
    say("euler identity")
    f3c.op_euler(d_x, to_dev(vc), to_dev(v_act), None, [0, N, 2 * N], 1.0, 0.96, d_vn)
    torch.cuda.synchronize()
    assert np.array_equal(d_x.cpu().numpy(), st.x)
    assert np.array_equal(d_vn.cpu().numpy(), st.v_cache)


def _occupancy_logits(B, n, seed):
    """Decoder-like logits: a smooth blob (occupied core) plus noise, with the
    comparison's edge values planted: 0, -0, NaN, +-inf, the smallest subnormal."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, n)).astype(np.float32)
    x += np.linspace(1.5, -1.5, n, dtype=np.float32)[None, :]
    special = np.array([0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45], np.float32)
    for b in range(B):
        at = rng.choice(n, size=min(n, len(special)), replace=False)
        x[b, at] = special[:len(at)]
    return x


@pytest.mark.parametrize("B,n", [(1, 1), (2, 31), (1, 32), (3, 33), (3, 1028), (2, 8191), (1, 8192), (2, 8193), (2, 8196),
                                 (2, 64 ** 3), (1, 64 ** 3 + 5)])
def test_pack_occupancy_bit_exact(torch, B, n):
    """Packed occupancy equals the oracle's packing word for word, tail bits zero."""
    from oracle import occupancy
    from paper_2511_22533_amd import f3c
    say(f"pack_occupancy B={B} n={n}")
    x = _occupancy_logits(B, n, seed=B * 1000 + n)
    n_words = (n + 31) // 32
    bits = torch.full((B, n_words), -1, dtype=torch.int32, device="cuda")
    f3c.op_pack_occupancy(to_dev(x), bits)
    torch.cuda.synchronize()
    got = bits.cpu().numpy().view(np.uint32)
    for b in range(B):
        assert np.array_equal(got[b], occupancy.pack(occupancy.occupancy(x[b]))), f"sample {b}"


@pytest.mark.parametrize("B,n,offset", [(1, 1, 0), (3, 33, 0), (2, 64 ** 3, 0), (2, 64 ** 3, 1),
                                        (1, 64 ** 3 + 5, 0), (4, 1000, 3)])
def test_dynamic_voxels_exact(torch, B, n, offset):
    """Eq. (1) count per sample equals the oracle's, for grids that differ in a
    few voxels (late steps) and in many (early steps); offset shifts the rows
    off 16-byte alignment so the word-at-a-time path runs too."""
    from oracle import occupancy
    from paper_2511_22533_amd import f3c
    say(f"dynamic_voxels B={B} n={n} offset={offset}")
    rng = np.random.default_rng(n + offset)
    prev = _occupancy_logits(B, n, seed=7 + n)
    nxt = prev.copy()
    for b in range(B):
        flips = rng.choice(n, size=max(1, n // (10 ** (b + 1))), replace=False)
        nxt[b, flips] = -nxt[b, flips]
    n_words = (n + 31) // 32
    packed = torch.zeros(2, B * n_words + offset, dtype=torch.int32, device="cuda")
    a = packed[0, offset:].view(B, n_words)
    p = packed[1, offset:].view(B, n_words)
    f3c.op_pack_occupancy(to_dev(nxt), a)
    f3c.op_pack_occupancy(to_dev(prev), p)
    counts = torch.full((B,), -1, dtype=torch.int64, device="cuda")
    f3c.op_dynamic_voxels(a, p, counts)
    torch.cuda.synchronize()
    got = counts.cpu().numpy()
    for b in range(B):
        want = occupancy.dynamic_voxels(occupancy.occupancy(nxt[b]), occupancy.occupancy(prev[b]))
        assert got[b] == want, f"sample {b}"


def test_dynamic_voxels_all_bits(torch):
    """Complementary grids: every voxel counts, including full 32-bit words."""
    from paper_2511_22533_amd import f3c
    n_words = 4096 + 3
    a = torch.zeros((2, n_words), dtype=torch.int32, device="cuda")
    b = torch.full((2, n_words), -1, dtype=torch.int32, device="cuda")
    b[1] = 0
    counts = torch.full((2,), -1, dtype=torch.int64, device="cuda")
    f3c.op_dynamic_voxels(a, b, counts)
    torch.cuda.synchronize()
    assert counts.cpu().tolist() == [32 * n_words, 0]


def test_sigma_calibration_drives_schedule(torch):
    """sigma of the predictive schedule (Sec. 3.2) from two decoded 64^3 grids
    at the anchor step and the step before it: count on the GPU, then the host
    plan for a 16^3 latent (64 output voxels per latent token), equal to the
    oracle's plan from the oracle's count."""
    from oracle import occupancy
    from oracle import schedule as osched
    from paper_2511_22533_amd import f3c
    G = 64
    z, y, x = np.meshgrid(*(np.arange(G, dtype=np.float32),) * 3, indexing="ij")
    r = np.sqrt((z - 31.5) ** 2 + (y - 30.0) ** 2 + (x - 33.0) ** 2)
    rng = np.random.default_rng(11)
    prev = (20.0 - r + 0.8 * rng.standard_normal(r.shape)).astype(np.float32).reshape(1, -1)
    nxt = (20.6 - r + 0.8 * rng.standard_normal(r.shape)).astype(np.float32).reshape(1, -1)
    words = torch.zeros((2, 1, G ** 3 // 32), dtype=torch.int32, device="cuda")
    f3c.op_pack_occupancy(to_dev(nxt), words[0])
    f3c.op_pack_occupancy(to_dev(prev), words[1])
    counts = torch.zeros((1,), dtype=torch.int64, device="cuda")
    f3c.op_dynamic_voxels(words[0], words[1], counts)
    torch.cuda.synchronize()
    sigma = int(counts.item())
    want_sigma = occupancy.dynamic_voxels(occupancy.occupancy(nxt), occupancy.occupancy(prev))
    assert sigma == want_sigma and sigma > 0
    for tau in (0, 3):
        got = f3c.schedule_plan(25, 16 ** 3, float(sigma), gamma_up=64.0, tau=tau)
        assert got.tolist() == osched.plan(25, 16 ** 3, float(want_sigma), gamma_up=64.0, tau=tau)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [128, 256, 512, 2048])
def test_final_projection_widths(torch, dtype, width):
    """Every width's column split, a ragged last workgroup, and rows that start at a 4-byte offset. Bound: float32
    sums of `width` products, 2^-24 sqrt(width) per term twice over (LN, dot), below 1e-5 at width 2048."""
    from paper_2511_22533_amd import f3c
    cfg = synth.ModelConfig(grid=8, width=width, depth=1, heads=width // 32, cond_tokens=64, cond_width=64, dtype=dtype)
    W = synth.make_weights(cfg, seed=6, scale=0.05)
    m = f3c.Model(cfg).load(W)
    rows = 7
    h = (2 * np.random.default_rng(width).standard_normal((rows, width)) + 0.5).astype(np.float32)
    flat = torch.empty(rows * width + 1, dtype=torch.float32, device="cuda")
    hd = flat[1:].view(rows, width)
    hd.copy_(to_dev(h))
    v = torch.full((rows + 1, 8), float("nan"), dtype=torch.float32, device="cuda")
    say("final widths", dtype, width)
    f3c.op_final(m, hd, v[:rows])
    torch.cuda.synchronize()
    want = dit.linear(dit.layer_norm(h.astype(np.float64)), W["out_w"], W["out_b"])
    assert max_rel(v[:rows].cpu().numpy(), want) < 1e-5
    assert torch.isnan(v[rows]).all()


@pytest.mark.parametrize("N", [1, 63, 65, 1025, 4095, 4097, 8192, 8193, 9261, 16384, 16385, 27000, 32767])
def test_select_edges(torch, N):
    """Selection on both sides of every size at which its kernels change, bit-exact: spread scores, scores crowded
    into one histogram bin (all but a far one), mostly equal scores, and NaN / infinite velocities."""
    rng = np.random.default_rng(N)
    B = 4
    vc = rng.standard_normal((B, N, 8)).astype(np.float32)
    vp = (vc + 0.1 * rng.standard_normal((B, N, 8))).astype(np.float32)
    vc[1] = 1.0 + 1e-5 * vc[1]
    vp[1] = vc[1]
    vc[1, N // 2] *= 50.0
    vc[2] = vc[2, :1]
    vp[2] = vc[2]
    vp[2, N // 3] += 1.0
    vc[3, N // 2] = np.nan
    vp[3, N // 3, 2] = np.inf
    for omega in (0.7, 0.0):
        for quotas in ([N // 3] * B, [min(1, N)] * B, [N - 1, 0, N // 2, N], [N - 1] * B):
            say("select edges", N, omega, quotas)
            _check_select(torch, vc, vp, quotas, omega)


@pytest.mark.parametrize("N", [127, 129, 1024, 1025, 4097, 8193, 9261, 16385])
def test_select_from_given_scores_edges(torch, N):
    """Given scores on both sides of every size at which the kernel changes, bit-exact: spread over all keys, crowded
    around one value (neighbouring floats, and a few of them many times) with far ones on both sides, two values, one."""
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(N)
    near = np.float32(0.3) + np.float32(2.0 ** -25) * rng.integers(0, 300, N)
    few = np.where(rng.random(N) < 0.9, rng.integers(0, 3, N) * 0.125, rng.standard_normal(N))
    spread = np.ldexp(rng.standard_normal(N), rng.integers(-100, 100, N))
    near[N // 3], near[N // 2] = -1e30, np.nan
    sc = np.stack([near, few, spread, np.where(np.arange(N) % 3 == 0, -2.5, 1e-3), np.full(N, -0.0)]).astype(np.float32)
    B = sc.shape[0]
    for quotas in ([N // 3] * B, [N - 1] * B, [1] * B, [N // 2, 0, N, N // 7, 2 * N // 3]):
        say("select scores edges", N, quotas)
        idx = torch.full((sum(N - c for c in quotas),), -7, dtype=torch.int32, device="cuda")
        pos = torch.full((B, N), -7, dtype=torch.int32, device="cuda")
        f3c.op_select_scores(to_dev(sc), quotas, idx, pos)
        torch.cuda.synchronize()
        row = 0
        for b in range(B):
            active = ssc.select(sc[b], quotas[b])[1]
            want_pos = np.full(N, -1, np.int64)
            want_pos[active] = row + np.arange(len(active))
            assert np.array_equal(idx.cpu().numpy()[row:row + len(active)], active), (quotas, b)
            assert np.array_equal(pos.cpu().numpy()[b], want_pos), (quotas, b)
            row += len(active)


def _kernel_us(torch, fn, calls=20, repeats=7):
    """Fastest of several replays of `calls` captured calls, us per call (no host time)."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            fn()
    best = float("inf")
    for _ in range(repeats):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


# Row strides beyond 32-bit offsets, of either operand, with both tiles such calls
# take: bit for bit the contiguous call's result. The large one is not held to the
# smallest tile (1000 x 4096 x 1024: 14 us, 21 with 64 x 64, contiguous 13).
@pytest.mark.parametrize("which,M,N,K,epi", [("A", 1000, 4096, 1024, 0), ("A", 130, 256, 64, 2), ("W", 300, 256, 192, 1)])
def test_gemm_bf16_wide_rows(torch, which, M, N, K, epi):
    from paper_2511_22533_amd import f3c
    g = torch.Generator(device="cuda").manual_seed(M)
    a = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
    bias = torch.randn(N, generator=g, device="cuda")

    def wide(x):
        stride = (1 << 22) + 8
        y = torch.empty((x.shape[0] - 1) * stride + K, dtype=x.dtype, device="cuda").as_strided(x.shape, (stride, 1))
        y.copy_(x)
        return y

    def call(A, W):
        r = torch.zeros(M, N, dtype=torch.float32 if epi == 2 else torch.bfloat16, device="cuda")
        run = lambda: f3c.op_gemm(f3c.F3C_BF16, epi, A, W, bias, **({"resid": r} if epi == 2 else {"out": r}))
        say("gemm wide rows", which, M, N, K, epi)
        run()
        torch.cuda.synchronize()
        return run, r

    _, want = call(a, w)
    A, W = (wide(a), w) if which == "A" else (a, wide(w))
    run, got = call(A, W)
    assert torch.equal(got, want)
    if M == 1000:
        assert _kernel_us(torch, run) < 1.45 * _kernel_us(torch, call(a, w)[0])


# Twice the K takes no more than twice the time: long rows of weights are split over
# the XCDs in column groups, too. (8192 x 1024: 68 and 121 us; the longer one 161 us
# when every XCD takes whole row panels.)
def test_gemm_column_groups_cost(torch):
    from paper_2511_22533_amd import f3c
    g = torch.Generator(device="cuda").manual_seed(0)
    M, N = 8192, 1024
    r = torch.zeros(M, N, device="cuda")
    bias = torch.randn(N, generator=g, device="cuda")
    us = {}
    for K in (4096, 8192):
        A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
        W = (0.05 * torch.randn(N, K, generator=g, device="cuda")).bfloat16()
        say("gemm column groups cost", M, N, K)
        us[K] = _kernel_us(torch, lambda: f3c.op_gemm(f3c.F3C_BF16, 2, A, W, bias, resid=r), calls=5)
    assert us[8192] < 2.04 * us[4096], us


# More samples than the lookup of a workgroup's sample walks one by one, with empty
# ones at both ends and in between; bf16 on each path, and f32.
@pytest.mark.parametrize("dt_name,hd", [("bf16", 64), ("bf16", 32), ("f32", 64)])
@pytest.mark.parametrize("B", [5, 64])
def test_attention_many_samples(torch, dt_name, hd, B):
    from paper_2511_22533_amd import f3c
    rng = np.random.default_rng(B + hd)
    q_lens = [int(x) for x in rng.integers(0, 150, B)]
    q_lens[0] = q_lens[1] = q_lens[-1] = 0
    q_lens[B // 2] = 129
    k_lens = [int(x) for x in rng.integers(1, 200, B)]
    dt = f3c.F3C_BF16 if dt_name == "bf16" else f3c.F3C_F32
    assert _attn_case(torch, dt, 4, hd, q_lens, k_lens, seed=B) < (2e-2 if dt_name == "bf16" else 1e-4)


# Few keys and many queries: the launch shape follows what a round of workgroups
# costs besides its key tiles, so one key tile is not slower than three. (9831
# queries: 18 and 22 us; with the shape of longer key ranges 31 and 33.)
@pytest.mark.parametrize("n", [6000, 9831])
def test_attention_few_keys_cost(torch, n):
    from paper_2511_22533_amd import f3c
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(rows, 1024, generator=g, device="cuda").bfloat16() for rows in (n, 192, 192))
    o = torch.empty_like(q)
    us = {}
    for nk in (64, 192):
        say("attention few keys cost", n, nk)
        us[nk] = _kernel_us(torch, lambda: f3c.op_attention(f3c.F3C_BF16, 16, 64, [0, n], [0, nk], q, k[:nk], v[:nk], o,
                                                            q_prescaled=True))
    assert us[64] < 0.9 * us[192], us


# Scores crowded into one bin, or all equal, take a few more passes over the keys
# than spread ones (512 tokens: 7.7 and 7.6 us against 6.0); a radix select behind
# the histogram took 2.2 times the spread ones' time.
def test_select_crowded_scores_cost(torch):
    from paper_2511_22533_amd import f3c
    N = 512
    rng = np.random.default_rng(N)
    spread = rng.standard_normal((1, N, 8)).astype(np.float32)
    crowd = (1.0 + 1e-5 * spread).astype(np.float32)
    crowd[0, N // 2] *= 50.0
    us = {}
    for name, vc in (("spread", spread), ("crowd", crowd), ("equal", np.ones_like(spread))):
        a = to_dev(vc)
        b = a + 0.1 if name == "spread" else a.clone()
        idx = torch.empty(N, dtype=torch.int32, device="cuda")
        pos = torch.empty((1, N), dtype=torch.int32, device="cuda")
        ws = torch.empty(f3c.select_workspace_bytes(1, N), dtype=torch.uint8, device="cuda")
        say("select cost", N, name)
        us[name] = _kernel_us(torch, lambda: f3c.op_select(a, b, 0.7, [int(0.7 * N)], idx, pos, None, ws))
    assert us["crowd"] < 1.75 * us["spread"] and us["equal"] < 1.75 * us["spread"], us
