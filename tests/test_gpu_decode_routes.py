"""The forms of the decode kernel -- a workgroup per unit, or the work line -- by the calls that each is chosen for, seen by
whether partials went through the workspace (a workgroup per unit leaves it as it was): attention against the oracle, the fused
step against append + attend, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2411_18077_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.fixture(scope="module")
def g():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


def bar(want):
    """2e-3, or one fp16 step of a larger result (two correctly rounded results of nearly equal sums)."""
    return np.maximum(TOL, 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 2.0 ** -14))) - 10))


def cache_and_oracle(g, w, Tcap, r_len, lengths=None):
    """The cache of capacity Tcap, and the oracle's answer for it."""
    from oracle import ref
    inp = W.make_inputs(w, "cuda")
    if lengths is not None:
        inp.n_tok.copy_(torch.minimum(inp.n_tok.cpu(), torch.as_tensor(lengths, dtype=torch.int32)))
    s, _ = g.shapes_for(w, Tcap)
    _, rs = g.shapes_for(w, inp.Tcap)
    cache, rc = g.gpu_build_cache(inp, s, r_len=r_len), g.ref_build_cache(inp, rs, r_len=r_len)
    want, _, _ = ref.decode_attn(rc, g.to_np(inp.q), g.sm_scale())
    return inp, s, cache, want.astype(np.float64)


def attend(g, w, inp, s, cache, want):
    """Attention on a zeroed workspace; returns whether it took the work line."""
    from paper_2411_18077_amd import api
    assert not cache.workspace.any()
    out = torch.full((w.B, w.Hq, w.D), float("nan"), dtype=torch.float16, device="cuda")
    api.minikv_decode_attn(s, inp.q, cache, g.sm_scale(), out)
    torch.cuda.synchronize()
    assert np.all(np.abs(g.to_np(out).astype(np.float64) - want) <= bar(want))
    return bool(cache.workspace.any())


def step(g, w, inp, s, cache):
    """The fused step, then append + attend on the same cache: the same bits and the same lengths."""
    from paper_2411_18077_amd import api
    k_new, v_new = inp.Rk[:, -1].contiguous(), inp.Rv[:, 0].contiguous()
    one = torch.full((w.B, w.Hq, w.D), float("nan"), dtype=torch.float16, device="cuda")
    two, r_next = torch.full_like(one, float("nan")), torch.full((w.units,), -1, dtype=torch.int32, device="cuda")
    api.minikv_decode_step(s, inp.q, k_new, v_new, cache, r_next, g.sm_scale(), one)
    api.kv_append_residual(s, k_new, v_new, cache)
    api.minikv_decode_attn(s, inp.q, cache, g.sm_scale(), two)
    torch.cuda.synchronize()
    assert torch.equal(one.view(torch.int16), two.view(torch.int16)) and torch.equal(r_next, cache.r_len)
    assert torch.isfinite(one).all()


@pytest.mark.parametrize("behind", [0, 1])
@pytest.mark.parametrize("G,rep,units,items", [
    (32, 8, 144, 32), (32, 4, 144, 36), (32, 2, 144, 42), (32, 4, 256, 52), (64, 8, 176, 42), (64, 3, 136, 39), (64, 1, 200, 52),
    (128, 4, 208, 66), (128, 8, 208, 53), (128, 1, 132, 42), (32, 4, 96, 24), (64, 2, 128, 26), (128, 4, 100, 30),
    (16, 4, 24, 10), (16, 2, 24, 11), (16, 1, 64, 12), (16, 4, 120, 20), (16, 4, 136, 26), (16, 8, 192, 20), (16, 1, 196, 35),
])
def test_either_side_of_a_workgroup_per_unit(g, G, rep, units, items, behind):
    """Capacities at each limit and an item behind it: a workgroup per unit, then the work line.  Units of all lengths up to the
    capacity, one of them without any token, 0 to 2 residual items."""
    kv = units // (2 if rep > 4 else 1)                    # (five heads and more are two units)
    Tcap = (items + behind - 2) * 128
    w = W.Workload(name="t", B=kv // 4, Hq=4 * rep, Hkv=4, L=Tcap, keep=None, keep_range=(0.02, 1.0), G=G, Rcap=128, seed=2000 + items,
                   n_outlier=3, outlier_scale=8.0)
    r_len = np.arange(kv) * 37 % 129
    r_len[1] = 0
    lengths = np.full(kv, Tcap)
    lengths[1] = 0
    inp, s, cache, want = cache_and_oracle(g, w, Tcap, r_len, lengths)
    assert attend(g, w, inp, s, cache, want) == bool(behind)
    cache.r_len.clamp_(max=127)                            # (there is room for the token)
    step(g, w, inp, s, cache)


@pytest.mark.parametrize("rep", [1, 2, 3, 4])
@pytest.mark.parametrize("G,Tcap", [(16, 2944), (32, 3840), (64, 4608), (128, 5120)])
def test_a_workgroup_per_unit_with_the_streaming_hint(g, G, Tcap, rep):
    """256 units of more than 88 MiB of packed capacity: every group size, one to four heads, an even and an odd number of passes
    (0 to 12), units without tokens and with residual tokens only."""
    units = 256
    assert units * Tcap * (64 + 1024 // G) > 88 << 20
    w = W.Workload(name="t", B=16, Hq=16 * rep, Hkv=16, L=1536, keep=None, keep_range=(0.02, 1.0), G=G, Rcap=128, seed=2100 + G + rep,
                   n_outlier=3, outlier_scale=8.0)
    r_len = np.arange(units) * 41 % 129 * (np.arange(units) % 4 != 2)
    lengths = np.full(units, w.L)
    lengths[2::7] = 0
    r_len[[2, 9, 255]] = 0
    inp, s, cache, want = cache_and_oracle(g, w, Tcap, r_len, lengths)
    assert not attend(g, w, inp, s, cache, want)
    cache.r_len.clamp_(max=127)
    step(g, w, inp, s, cache)
    assert not cache.workspace.any()


@pytest.mark.parametrize("line", [0, 1])
@pytest.mark.parametrize("G,Tcap", [(16, 1024), (32, 1152), (64, 1152), (128, 1152)])
@pytest.mark.parametrize("Hq,Hkv,B", [(2, 2, 32), (8, 2, 33), (16, 2, 17)])
def test_anything_behind_the_lengths(g, G, Tcap, Hq, Hkv, B, line):
    """What the cache holds past the lengths -- infinities and NaN in the scales, the zero-points and the residual rows, those of an
    empty residual included -- reaches no output of either form, alone and as a fused step."""
    from paper_2411_18077_amd import api
    w = W.Workload(name="t", B=B, Hq=Hq, Hkv=Hkv, L=Tcap - 128, keep=None, keep_range=(0.02, 1.0), G=G, Rcap=256, seed=2200 + G,
                   n_outlier=3, outlier_scale=8.0)
    r_len = np.arange(w.units) * 53 % 256 * (np.arange(w.units) % 4 != 2)
    lengths = np.full(w.units, w.L)
    lengths[2::5] = 0
    inp, s, cache, want = cache_and_oracle(g, w, Tcap, r_len, lengths)
    n, r = inp.n_tok.tolist(), r_len.tolist()
    for name, value in (("Ks", float("nan")), ("Kz", float("nan")), ("Vs", float("inf")), ("Vz", float("nan"))):
        rows = cache.t[name].view(w.units, -1)
        per = rows.shape[1] // Tcap if name[0] == "V" else 0
        for u in range(w.units):
            rows[u, (n[u] * per if per else n[u] // G * w.D):] = value
    for rows in (cache.Rk.view(w.units, w.Rcap, w.D), cache.Rv.view(w.units, w.Rcap, w.D)):
        for u in range(w.units):
            rows[u, r[u]:] = float("nan")
    api.minikv_diag_decode_weights(line)
    try:
        assert attend(g, w, inp, s, cache, want) == bool(line)
        step(g, w, inp, s, cache)
    finally:
        api.minikv_diag_decode_weights(0)


WORKSPACE_SLOTS, COMPUTE_UNITS = 4096, 256                 # (of the library)


def line_partials(w, hsets, Tcap, n_tok, r_len, mode):
    """(first workgroup, number of workgroups) that share each unit on the work line, by the rules of the launch and of the kernel: the
    line's weights, its cut into 2^k ranges of a workgroup, the ranges that hold a unit's first and last item."""
    waves = 4 if w.G == 16 else 8
    nu, passes_cap, res_cap = w.units * hsets, (Tcap + 127) // 128, (w.Rcap + 63) // 64
    cap_items = nu * (passes_cap + res_cap)
    light = mode == 0 and (nu * (2 * passes_cap + 8 * res_cap) < 8 * COMPUTE_UNITS or 2048 < cap_items <= 3584)
    wq, wr = (1, 1) if mode == 2 else (2, 4 if light else 8)
    groups = min(cap_items, COMPUTE_UNITS, max(16 * nu, cap_items // 8))
    nq, nr = [(int(t) + 127) // 128 for t in n_tok for _ in range(hsets)], [(int(r) + 63) // 64 for r in r_len for _ in range(hsets)]
    P = sum(a * wq + b * wr for a, b in zip(nq, nr))
    nw_log = max(1, min(groups, P // wr)).bit_length() - 1 + waves.bit_length() - 1
    starts = np.array([(k * waves // 2 * P) >> (nw_log - 1) for k in range(1 << (nw_log - waves.bit_length() + 1))])
    out, ib = [], 0
    for a, b in zip(nq, nr):
        if a + b == 0:
            out.append((0, 0))
            continue
        end = ib + a * wq + b * wr
        last = end - (wr if b > 1 or a == 0 else wq)
        first = int(np.searchsorted(starts, ib, "right")) - 1
        out.append((first, int(np.searchsorted(starts, last, "right")) - first))
        ib = end
    return out


@pytest.mark.parametrize("weights", [0, 1, 2])
@pytest.mark.parametrize("G,Hq,Hkv,B,L,Tcap,second,rounds", [
    (16, 2, 1, 1, 40000, 40064, 1.0, "one level, two round trips"),
    (32, 4, 1, 1, 33000, 33024, 1.0, "one level, two round trips"),
    (32, 4, 1, 1, 100000, 100096, 1.0, "two levels"),
    (32, 4, 1, 2, 65536, 65536, 0.43, "two levels, last set not full"),
    (128, 1, 1, 2, 65536, 65536, 0.38, "two levels, last set not full"),
    (64, 8, 1, 1, 65536, 65536, 1.0, "two levels"),
    (64, 8, 2, 1, 50000, 50048, 0.3, "two levels, last set not full"),
    (32, 8, 1, 1, 33000, 33024, 1.0, "one level, two round trips"),
])
def test_units_shared_by_many_workgroups(g, G, Hq, Hkv, B, L, Tcap, second, rounds, weights):
    """Units over 17 to 32 workgroups, which merge at once in two round trips, and over more, which merge in sets of 16 and once
    more.  How many share a unit is worked out on the host, found again in the workspace, and must be what the case is for."""
    from paper_2411_18077_amd import api
    w = W.Workload(name="t", B=B, Hq=Hq, Hkv=Hkv, L=L, keep=0.998, G=G, Rcap=128, seed=2300 + G, n_outlier=3, outlier_scale=8.0)
    hsets = 2 if Hq // Hkv > 4 else 1
    lengths = np.array([L, int(L * second)][: w.units]) // G * G
    r_len = np.array([128, 70][: w.units])
    inp, s, cache, want = cache_and_oracle(g, w, Tcap, r_len, lengths)
    shared = line_partials(w, hsets, Tcap, inp.n_tok.tolist(), r_len, weights)
    counts = [n for _, n in shared]
    api.minikv_diag_decode_weights(weights)
    try:
        assert attend(g, w, inp, s, cache, want)
        written = cache.workspace.view(torch.float32)[(3 * w.units * hsets + WORKSPACE_SLOTS + 1 + 63) // 64 * 64:]
        slots = written[: written.numel() // 528 * 528].view(-1, 528).ne(0).any(dim=1).nonzero().flatten().tolist()
        # (slot = workgroup + 2 * unit)
        assert slots == sorted(k + 2 * u for u, (first, n) in enumerate(shared) for k in range(first, first + n) if n > 1)
        step(g, w, inp, s, cache)
    finally:
        api.minikv_diag_decode_weights(0)
    if rounds.startswith("one level"):
        assert any(16 < n <= 32 for n in counts), counts
    else:
        assert any(n > 32 for n in counts), counts
    if "not full" in rounds:
        assert any(n > 32 and n % 16 for n in counts), counts
