"""GPU parity of the prefill attention with cumulative attention scores (Section 3.2, Algorithm 1 line 2)
against the fp64 oracle: X_O to 2e-3, LSE to 1e-3, A_cumul to 1e-3 relative (+1e-4 absolute); then
Algorithm 1 lines 2-5 and 17-19 chained on the GPU and checked stage by stage."""
import math

import numpy as np
import pytest
import torch

from paper_2411_18077_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL_O, TOL_LSE, RTOL_A, ATOL_A = 2e-3, 1e-3, 1e-3, 1e-4


@pytest.fixture(scope="module")
def g():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


def run_gpu(Q, K, V, sm, want_cumul=True):
    from paper_2411_18077_amd import api
    B, Hq, L, D = Q.shape
    xo = torch.full((B, Hq, L, D), float("nan"), dtype=torch.float16, device="cuda")
    lse = torch.full((B, Hq, L), float("nan"), dtype=torch.float32, device="cuda")
    acc = torch.full((B, Hq, L), float("nan"), dtype=torch.float32, device="cuda") if want_cumul else None
    ws = torch.empty(api.selective_flash_attn_workspace_bytes(B, K.shape[1], L), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)                                           # no initial state needed (0xFFFF is an fp16 NaN)
    api.selective_flash_attn(B, Hq, K.shape[1], L, Q, K, V, sm, xo, lse, acc, ws)
    torch.cuda.synchronize()
    return xo, lse, acc


def check(g, B, Hq, Hkv, L, seed, gain=1.0, sm=None):
    from oracle import ref
    sm = 1.0 / math.sqrt(128) if sm is None else sm
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, seed, device="cuda", gain=gain)
    xo, lse, acc = run_gpu(Q, K, V, sm)
    _, xo64, lse64, acc64 = ref.selective_flash_attn(g.to_np(Q), g.to_np(K), g.to_np(V), sm)
    got_o, got_l, got_a = (g.to_np(t).astype(np.float64) for t in (xo, lse, acc))
    assert np.isfinite(got_o).all() and np.isfinite(got_l).all() and np.isfinite(got_a).all()
    assert np.max(np.abs(got_o - xo64)) <= TOL_O
    assert np.max(np.abs(got_l - lse64)) <= TOL_LSE
    assert np.all(np.abs(got_a - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)
    assert np.allclose(got_a.sum(-1), L, rtol=1e-4)          # the rows of the attention matrix sum to one


@pytest.mark.parametrize("B,Hq,Hkv,L", [(1, 1, 1, 1), (1, 2, 1, 31), (1, 1, 1, 64), (1, 2, 2, 65), (1, 1, 1, 128),
                                         (2, 4, 2, 129), (1, 8, 2, 300), (1, 2, 1, 777), (1, 4, 4, 1024)])
def test_prefill_matches_the_oracle(g, B, Hq, Hkv, L):
    check(g, B, Hq, Hkv, L, seed=100 + L)


@pytest.mark.parametrize("gain,sm", [(2.0, None), (1.0, 1.0), (0.0, None)])
def test_peaked_and_flat_softmax_rows(g, gain, sm):
    """gain 2: scores ~ N(0, 4^2/...) (peaked rows); sm_scale 1: very peaked; gain 0: all scores equal, so the
    column sums are differences of harmonic numbers."""
    check(g, 1, 4, 2, 500, seed=7, gain=gain, sm=sm)


def test_random_shapes(g):
    """Seeded sweep over batch, head counts, prompt lengths around the tile sizes (64 keys, 128 queries) and
    softmax sharpness."""
    rng = np.random.default_rng(7)
    for case in range(16):
        Hkv = int(rng.choice([1, 2, 3]))
        rep = int(rng.choice([1, 2, 4, 5]))
        L = int(rng.choice([rng.integers(1, 70), rng.integers(120, 136), rng.integers(190, 260), rng.integers(300, 900)]))
        check(g, int(rng.integers(1, 3)), Hkv * rep, Hkv, L, seed=300 + case, gain=float(rng.choice([0.5, 1.0, 1.7])))


@pytest.mark.parametrize("B,Hq,Hkv,L", [(64, 16, 4, 1), (64, 16, 4, 65), (32, 16, 16, 257), (32, 16, 2, 320), (32, 16, 4, 447)])
def test_launches_with_256_queries_per_workgroup(g, B, Hq, Hkv, L):
    """Many heads and short prompts, at least 1024 blocks of 256 queries (which serve long prompts only, below): tile and
    block edges; the oracle recomputes the first and the last sequence."""
    from oracle import ref
    assert B * Hq * ((L + 255) // 256) >= 1024
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 900 + L, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    assert torch.isfinite(xo).all() and torch.isfinite(lse).all()
    assert torch.allclose(acc.double().sum(-1), torch.full((B, Hq), float(L), dtype=torch.float64, device="cuda"), rtol=1e-4)
    sel = [0, B - 1]
    _, xo64, lse64, acc64 = ref.selective_flash_attn(g.to_np(Q[sel]), g.to_np(K[sel]), g.to_np(V[sel]), sm)
    assert np.max(np.abs(g.to_np(xo[sel]).astype(np.float64) - xo64)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse[sel]).astype(np.float64) - lse64)) <= TOL_LSE
    assert np.all(np.abs(g.to_np(acc[sel]) - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)


@pytest.mark.parametrize("B,Hq,Hkv", [(1, 2, 1), (4, 16, 4), (4, 32, 8), (5, 32, 16)])
@pytest.mark.parametrize("L", [1, 63, 64, 127, 129, 192, 321])
def test_every_division_of_a_launch(g, B, Hq, Hkv, L):
    """2 to 160 heads at lengths around a tile, a pair of tiles and a block (two sets of waves share a block on longer
    prompts, below)."""
    from oracle import ref
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 950 + L, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    assert torch.isfinite(xo).all() and torch.isfinite(lse).all() and torch.isfinite(acc).all()
    sel = [B - 1]
    _, xo64, lse64, acc64 = ref.selective_flash_attn(g.to_np(Q[sel]), g.to_np(K[sel]), g.to_np(V[sel]), sm)
    assert np.max(np.abs(g.to_np(xo[sel]).astype(np.float64) - xo64)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse[sel]).astype(np.float64) - lse64)) <= TOL_LSE
    assert np.all(np.abs(g.to_np(acc[sel]) - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)


def check_last(g, B, Hq, Hkv, L, seed):
    """Everything finite, every column sum's total right; the last sequence against the oracle."""
    from oracle import ref
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, seed, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    assert torch.isfinite(xo).all() and torch.isfinite(lse).all()
    assert torch.allclose(acc.double().sum(-1), torch.full((B, Hq), float(L), dtype=torch.float64, device="cuda"), rtol=1e-4)
    sel = [B - 1]
    _, xo64, lse64, acc64 = ref.selective_flash_attn(g.to_np(Q[sel]), g.to_np(K[sel]), g.to_np(V[sel]), sm)
    assert np.max(np.abs(g.to_np(xo[sel]).astype(np.float64) - xo64)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse[sel]).astype(np.float64) - lse64)) <= TOL_LSE
    assert np.all(np.abs(g.to_np(acc[sel]) - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(1, 2, 1, 385), (1, 2, 2, 447), (1, 2, 1, 448), (2, 4, 1, 449), (8, 4, 2, 512), (1, 2, 1, 577), (1, 1, 1, 1000)])
def test_two_sets_of_waves_on_64_queries(g, B, Hq, Hkv, L):
    """More than 96 tokens and at most 256 blocks of 64 queries: an odd and an even number of tiles, ragged ends."""
    check_last(g, B, Hq, Hkv, L, 1100 + L)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(16, 1, 1, 1024), (8, 2, 1, 1025), (15, 1, 1, 1151), (14, 1, 1, 1217)])
def test_two_sets_of_waves_on_128_queries(g, B, Hq, Hkv, L):
    """From 1024 tokens on, more than 256 blocks of 64 queries (or just as many) and at most 256 of 128."""
    check_last(g, B, Hq, Hkv, L, 1200 + L)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(4, 32, 8, 65), (2, 32, 8, 256), (5, 32, 8, 129), (8, 1, 1, 2049), (16, 1, 1, 2048), (11, 1, 1, 2689), (11, 1, 1, 3009),
                                         (33, 1, 1, 449), (19, 2, 1, 385), (5, 8, 4, 512), (10, 4, 4, 513), (7, 4, 1, 640), (12, 2, 1, 1217), (32, 1, 1, 1024), (16, 2, 1, 1025)])
def test_launches_of_up_to_two_long_row_blocks_per_compute_unit(g, B, Hq, Hkv, L):
    """Either side of the lines between 64 queries and two sets of waves (two buffers or one), 128 and two sets, and 128 alone:
    an odd and an even number of tiles, ragged ends."""
    check_last(g, B, Hq, Hkv, L, 1250 + L)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(64, 1, 1, 4096), (61, 1, 1, 4223)])
def test_256_queries_per_workgroup_on_long_prompts(g, B, Hq, Hkv, L):
    """From 4096 tokens and 1024 blocks of 256 queries on."""
    assert B * Hq * ((L + 255) // 256) >= 1024
    check_last(g, B, Hq, Hkv, L, 1300 + L)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(33, 16, 4, 1), (33, 16, 16, 31), (33, 16, 8, 63), (33, 16, 4, 64), (33, 16, 4, 65), (32, 16, 4, 64)])
def test_short_prompts_of_many_heads(g, B, Hq, Hkv, L):
    """Prompts of one or two key tiles on 512 heads and more: the launch that forms the column sums as well, with more
    workgroups than run at once."""
    check_last(g, B, Hq, Hkv, L, 1400 + L)


@pytest.mark.parametrize("L", [2, 32, 33, 63, 95, 96, 97, 127, 128])
def test_one_launch_for_prompts_of_one_row_block(g, L):
    check(g, 2, 6, 2, L, 1500 + L, gain=1.5)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(1, 2, 1, 191), (1, 2, 1, 193), (1, 1, 1, 255), (1, 1, 1, 257), (16, 1, 1, 1025), (20, 1, 1, 1601),
                                         (20, 1, 1, 1599), (64, 1, 1, 256), (64, 1, 1, 257), (21, 1, 1, 767), (21, 1, 1, 769)])
def test_column_sums_of_64_keys_per_workgroup(g, B, Hq, Hkv, L):
    """Either side of the lines between 64 and 128 keys per workgroup, key blocks that begin in the second half of a tile of 128
    queries, ragged last tiles."""
    check_last(g, B, Hq, Hkv, L, 1600 + L)


@pytest.mark.parametrize("per_tile", [-3.0, 0.02, 0.7, 3.0, 30.0])
def test_scores_that_rise_or_fall_along_the_keys(g, per_tile):
    """Scores whose level moves by `per_tile` (in powers of e) every 64 keys, so that the running maximum is raised, and the
    output rescaled, on the first tile only, now and then, or on every tile."""
    from oracle import ref
    B, Hq, Hkv, L = 1, 4, 2, 700
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 41, device="cuda", gain=0.3)
    Q[..., 0] = 8.0
    K[..., 0] = (torch.arange(L, device="cuda") * (per_tile / 64.0 / 8.0 * math.sqrt(128))).to(torch.float16)
    xo, lse, acc = run_gpu(Q, K, V, 1.0 / math.sqrt(128))
    _, xo64, lse64, acc64 = ref.selective_flash_attn(g.to_np(Q), g.to_np(K), g.to_np(V), 1.0 / math.sqrt(128))
    assert np.max(np.abs(g.to_np(xo).astype(np.float64) - xo64)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse).astype(np.float64) - lse64)) <= TOL_LSE
    assert np.all(np.abs(g.to_np(acc) - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)


@pytest.mark.parametrize("B,Hq,Hkv,L", [(1, 2, 1, L) for L in (1, 31, 48, 64, 65, 96, 97, 127, 128, 129, 200, 1000)] +
                                       [(9, 32, 8, L) for L in (1, 48, 96, 97, 128, 129)] +
                                       [(5, 8, 4, 512), (10, 4, 4, 513), (32, 1, 1, 1024), (16, 1, 1, 3000), (64, 1, 1, 4096)])
def test_first_pass_alone(g, B, Hq, Hkv, L):
    """Without column sums: one row block on few heads and on many (128 queries from 97 tokens on only there), a block of 64
    shared by two sets of waves with two buffers and with one, 128 shared by two sets, 256; the last sequence against the oracle."""
    from oracle import ref
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 5, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, 0.09, want_cumul=False)
    assert torch.isfinite(xo).all() and torch.isfinite(lse).all()
    xo, lse = xo[-1:], lse[-1:]
    _, xo64, lse64, _ = ref.selective_flash_attn(g.to_np(Q[-1:]), g.to_np(K[-1:]), g.to_np(V[-1:]), 0.09)
    assert np.max(np.abs(g.to_np(xo).astype(np.float64) - xo64)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse).astype(np.float64) - lse64)) <= TOL_LSE


def test_long_prompt_on_sampled_rows_and_columns(g):
    """L = 8192 (the longest length of the paper's kernel tables), 32 query / 8 KV heads: the oracle would
    need minutes for all of it, so a few heads are recomputed by it on a strided subset of the prompt:
    every 37th query row (its X_O and LSE need only that row's scores), and the exact property sum_j
    A_cumul[j] = L on all heads; A_cumul itself is compared on one head with numpy in float64."""
    B, Hq, Hkv, L = 1, 32, 8, 8192
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 11, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    assert np.allclose(g.to_np(acc).astype(np.float64).sum(-1), L, rtol=1e-4)
    for hq in (0, 13, 31):
        q = g.to_np(Q[0, hq]).astype(np.float64)
        k = g.to_np(K[0, hq // 4]).astype(np.float64)
        v = g.to_np(V[0, hq // 4]).astype(np.float64)
        rows = np.arange(5, L, 37)
        S = (q[rows] @ k.T) * np.float64(np.float32(sm))
        S[np.arange(L)[None, :] > rows[:, None]] = -np.inf
        m = S.max(-1, keepdims=True)
        E = np.exp(S - m)
        P = E / E.sum(-1, keepdims=True)
        assert np.max(np.abs(g.to_np(xo[0, hq])[rows].astype(np.float64) - P @ v)) <= TOL_O
        assert np.max(np.abs(g.to_np(lse[0, hq])[rows].astype(np.float64) - (m[:, 0] + np.log(E.sum(-1))))) <= TOL_LSE
    # one head in full, in float64 with numpy, row block by row block (the matrix is 8192 x 8192)
    hq = 7
    q = g.to_np(Q[0, hq]).astype(np.float64); k = g.to_np(K[0, hq // 4]).astype(np.float64)
    col = np.zeros(L)
    for r0 in range(0, L, 1024):
        rows = np.arange(r0, r0 + 1024)
        S = (q[rows] @ k.T) * np.float64(np.float32(sm))
        S[np.arange(L)[None, :] > rows[:, None]] = -np.inf
        E = np.exp(S - S.max(-1, keepdims=True))
        col += (E / E.sum(-1, keepdims=True)).sum(0)
    got = g.to_np(acc[0, hq]).astype(np.float64)
    assert np.all(np.abs(got - col) <= RTOL_A * np.abs(col) + ATOL_A)


def test_million_token_prompt_addressing(g):
    """One head, 2^20 + 77 tokens: the tile offsets are 32-bit byte offsets per head (268 MB of K, 2 MB rows of
    the transposed V), so this checks them at scale.  Compared in float64 with numpy: X_O and LSE of sampled
    query rows over the whole prompt, A_cumul of the last 150 columns (they only need the last 150 rows), and
    the exact property sum_j A_cumul[j] = L."""
    L = (1 << 20) + 77
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(1, 1, 1, L, 31, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    got_a = g.to_np(acc[0, 0]).astype(np.float64)
    assert np.isfinite(got_a).all() and abs(got_a.sum() - L) <= 1e-4 * L
    k = g.to_np(K[0, 0]).astype(np.float64)
    v = g.to_np(V[0, 0]).astype(np.float64)
    scale = np.float64(np.float32(sm))

    def rows_ref(rows):
        S = (g.to_np(Q[0, 0][rows]).astype(np.float64) @ k.T) * scale
        S[np.arange(L)[None, :] > rows[:, None]] = -np.inf
        m = S.max(-1, keepdims=True)
        E = np.exp(S - m)
        den = E.sum(-1, keepdims=True)
        return E / den, (m + np.log(den))[:, 0]

    rows = np.array([0, 63, 64, 4095, 65536, 65537, 524288, 1000003, L - 129, L - 2, L - 1])
    P, lse_ref = rows_ref(rows)
    assert np.max(np.abs(g.to_np(xo[0, 0][rows]).astype(np.float64) - P @ v)) <= TOL_O
    assert np.max(np.abs(g.to_np(lse[0, 0][rows]).astype(np.float64) - lse_ref)) <= TOL_LSE
    tail = np.arange(L - 150, L)
    P, _ = rows_ref(tail)
    col = P[:, L - 150:].sum(0)
    assert np.all(np.abs(got_a[L - 150:] - col) <= RTOL_A * np.abs(col) + ATOL_A)


def test_prefill_select_quantize_decode_chain(g):
    """Algorithm 1 lines 2-5, then a decode step (lines 9, 17-19), all on the GPU; each stage is checked
    against the oracle fed with the GPU's input to that stage (the selection decides on the GPU's fp32
    A_cumul on both sides, so the kept positions are bit-exact)."""
    from paper_2411_18077_amd import api
    from oracle import ref
    B, Hq, Hkv, L, G = 2, 8, 2, 1024, 32
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 21, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    _, xo64, _, acc64 = ref.selective_flash_attn(g.to_np(Q), g.to_np(K), g.to_np(V), sm)
    assert np.max(np.abs(g.to_np(xo).astype(np.float64) - xo64)) <= TOL_O
    assert np.all(np.abs(g.to_np(acc) - acc64) <= RTOL_A * np.abs(acc64) + ATOL_A)
    U, rep = B * Hkv, Hq // Hkv
    n_hh = torch.full((U,), 256, dtype=torch.int32, device="cuda")
    n_rw = torch.full((U,), 256, dtype=torch.int32, device="cuda")
    idx = torch.zeros(U, 512, dtype=torch.int32, device="cuda"); n_tok = torch.zeros(U, dtype=torch.int32, device="cuda")
    ws = torch.empty(api.kv_select_workspace_bytes(U, rep, L), dtype=torch.uint8, device="cuda")
    A2 = acc.view(U * rep, L)
    api.kv_select_hh_rw(U, rep, L, A2, n_hh, n_rw, idx, 512, n_tok, ws)
    ridx, rn = ref.select_hh_rw(g.to_np(A2), g.to_np(n_hh), g.to_np(n_rw), rep=rep, idx_stride=512)
    assert np.array_equal(g.to_np(idx), ridx) and np.array_equal(g.to_np(n_tok), rn)
    s = api.make_shape(B, Hq, Hkv, 128, G, 640, 32)
    rs = ref.RefShape(B, Hq, Hkv, 128, G, 640, 32)
    gc = api.Cache(s)
    Ku, Vu = K.view(U, L, 128), V.view(U, L, 128)
    api.kv_quantize_pack(s, Ku, Vu, L, idx, 512, n_tok, 512, gc)
    gen = torch.Generator(device="cuda"); gen.manual_seed(3)
    kn = torch.randn(U, 128, generator=gen, device="cuda").to(torch.float16)
    vn = torch.randn(U, 128, generator=gen, device="cuda").to(torch.float16)
    qn = torch.randn(B, Hq, 128, generator=gen, device="cuda").to(torch.float16)
    api.kv_append_residual(s, kn, vn, gc)
    out = torch.empty(B, Hq, 128, dtype=torch.float16, device="cuda")
    api.minikv_decode_attn(s, qn, gc, sm, out)
    torch.cuda.synchronize()
    rc = ref.RefCache(rs)
    assert ref.quantize_pack(rc, g.to_np(Ku), g.to_np(Vu), rn, ridx) == 0
    assert ref.append_residual(rc, g.to_np(kn), g.to_np(vn)) == 0
    g.assert_cache_bit_exact(gc, rc, what=("Kc", "Ks", "Kz", "Vc", "Vs", "Vz", "q_len", "r_len"))
    want, _, _ = ref.decode_attn(rc, g.to_np(qn), sm)
    assert np.max(np.abs(g.to_np(out).astype(np.float64) - want)) <= 2e-3


def test_benchmarked_shape_on_sampled_rows_and_late_columns(g):
    """The shape bench.py times (one sequence of 32768 tokens, 32 query / 8 KV heads): the whole matrix is out of
    the oracle's reach, so query rows are sampled (tile edges, the first and last rows, random ones) for X_O and
    LSE, the cumulative scores of the last 96 columns are rebuilt from the oracle's weights of the last 96 rows,
    and every head must satisfy what holds at any size: the column sums add up to L, the first column gets at
    least its own row, the last column exactly the last row's own weight."""
    from oracle import ref
    B, Hq, Hkv, L = 1, 32, 8, 32768
    sm = 1.0 / math.sqrt(128)
    Q, K, V = W.make_prefill_inputs(B, Hq, Hkv, L, 1013, device="cuda")
    xo, lse, acc = run_gpu(Q, K, V, sm)
    assert torch.isfinite(xo).all() and torch.isfinite(lse).all() and torch.isfinite(acc).all()
    accd = acc.double()
    assert torch.allclose(accd.sum(-1), torch.full((B, Hq), float(L), dtype=torch.float64, device="cuda"), rtol=1e-4)
    assert (accd[..., 0] >= 1.0 - 1e-3).all()
    rng = np.random.default_rng(5)
    tail = 96
    for hq in (0, 13, 31):
        hk = hq // (Hq // Hkv)
        q, k, v = g.to_np(Q[0, hq]), g.to_np(K[0, hk]), g.to_np(V[0, hk])
        rows = np.unique(np.concatenate([[0, 1, 63, 64, 127, 128, 129, 8191, 8192, 16383, 16384, L - 129, L - 128, L - 2, L - 1],
                                         rng.integers(0, L, 12)])).astype(np.int64)
        want_o, want_l, _ = ref.selective_flash_attn_rows(q, k, v, sm, rows)
        got_o = g.to_np(xo[0, hq]).astype(np.float64)[rows]
        got_l = g.to_np(lse[0, hq]).astype(np.float64)[rows]
        assert np.max(np.abs(got_o - want_o)) <= TOL_O
        assert np.max(np.abs(got_l - want_l)) <= TOL_LSE
        late = np.arange(L - tail, L, dtype=np.int64)
        _, _, pt = ref.selective_flash_attn_rows(q, k, v, sm, late, tail=tail)
        want_a = pt.sum(axis=0)
        got_a = g.to_np(acc[0, hq]).astype(np.float64)[L - tail:]
        assert np.all(np.abs(got_a - want_a) <= RTOL_A * np.abs(want_a) + ATOL_A)
