"""GPU parity for kv_quantize_pack / kv_append_residual / kv_flush_residual: codes, packed words, scale
and zero-point must equal the oracle's bit for bit (Section 3.1.1 / 3.3; Algorithm 1 lines 3-5, 9-15)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2411_18077_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_common
    assert torch.cuda.is_available()
    return gpu_common


def small(G, **kw):
    base = dict(name="t", B=2, Hq=4, Hkv=2, L=640, keep=0.5, G=G, Rcap=max(G, 32), seed=40 + G,
                n_outlier=3, outlier_scale=8.0)
    base.update(kw)
    return W.Workload(**base)


@pytest.mark.parametrize("G", [16, 32, 64, 128])
def test_prefill_quantize_bit_exact(g, G):
    w = small(G)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, inp.Tcap)
    gc = g.gpu_build_cache(inp, s)
    rc = g.ref_build_cache(inp, rs)
    assert int(gc.q_len[0]) == int(inp.n_tok[0]) > 0
    g.assert_cache_bit_exact(gc, rc)


def test_ragged_lengths_student_t_and_no_gather(g):
    w = small(64, keep=None, keep_range=(0.05, 1.0), dist="student_t4", L=1024, B=3, Hkv=2, Hq=2, n_outlier=0)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, inp.Tcap)
    g.assert_cache_bit_exact(g.gpu_build_cache(inp, s), g.ref_build_cache(inp, rs))
    # idx == NULL takes rows 0..n-1
    from paper_2411_18077_amd import api
    from oracle import ref
    cache = api.Cache(s)
    api.kv_quantize_pack(s, inp.K, inp.V, w.L, None, 0, inp.n_tok, int(inp.n_tok.max()), cache)
    torch.cuda.synchronize()
    c = ref.RefCache(rs)
    assert ref.quantize_pack(c, g.to_np(inp.K), g.to_np(inp.V), g.to_np(inp.n_tok), None) == 0
    g.assert_cache_bit_exact(cache, c)


def test_lattice_and_ties_bit_exact(g):
    """Exact half-way cases (round half to even) and degenerate groups reach the GPU rounding path."""
    w = small(16, L=256, keep=1.0, n_outlier=0)
    inp = W.make_inputs(w, "cuda")
    gen = torch.Generator(device="cuda"); gen.manual_seed(5)
    lev = torch.randint(0, 13, inp.K.shape, generator=gen, device="cuda").to(torch.float16) * 0.25   # 0..3 in steps of 1/4
    lev[:, 0::16] = 0; lev[:, 1::16] = 3
    inp.K.copy_(lev)
    v = torch.randint(0, 7, inp.V.shape, generator=gen, device="cuda").to(torch.float16) * 0.5
    v[:, :, 0::16] = 0; v[:, :, 1::16] = 3
    v[:, 5] = 1.25                                      # degenerate groups: max == min
    v[:, 6] = -0.0
    inp.V.copy_(v)
    s, rs = g.shapes_for(w, inp.Tcap)
    g.assert_cache_bit_exact(g.gpu_build_cache(inp, s), g.ref_build_cache(inp, rs))


def test_refused_units_are_left_unchanged(g):
    from paper_2411_18077_amd import api
    w = small(32, L=256, keep=1.0)
    inp = W.make_inputs(w, "cuda")
    s, _ = g.shapes_for(w, inp.Tcap)
    cache = api.Cache(s)
    n = inp.n_tok.clone(); n[1] = 40                     # not a multiple of G
    cache.q_len[2] = inp.Tcap - 32                       # would overflow the capacity
    api.kv_quantize_pack(s, inp.K, inp.V, w.L, None, 0, n, 256, cache)
    torch.cuda.synchronize()
    q = cache.q_len.cpu().tolist()
    assert q[0] == 256 and q[1] == 0 and q[2] == inp.Tcap - 32 and q[3] == 256


def test_unit_above_the_host_bound_is_left_unchanged(g):
    """max_tok sizes the launch; a unit whose device-side n_tok exceeds it must not be half-written with its
    length bumped: it is left alone, the others match the oracle bit for bit."""
    from paper_2411_18077_amd import api
    from oracle import ref
    w = small(32, L=512, keep=1.0)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, inp.Tcap)
    cache = api.Cache(s)
    n = torch.full_like(inp.n_tok, 128)
    n[2] = 256                                           # above the bound passed below
    api.kv_quantize_pack(s, inp.K, inp.V, w.L, None, 0, n, 128, cache)
    torch.cuda.synchronize()
    assert cache.q_len.cpu().tolist() == [128, 128, 0, 128]
    rc = ref.RefCache(rs)
    n_ref = g.to_np(n).copy(); n_ref[2] = 0              # what the library must have done
    assert ref.quantize_pack(rc, g.to_np(inp.K), g.to_np(inp.V), n_ref, None) == 0
    g.assert_cache_bit_exact(cache, rc, what=("Kc", "Ks", "Kz", "Vc", "Vs", "Vz", "q_len"))


def test_decode_loop_append_and_flush_bit_exact(g):
    """Algorithm 1 lines 9-15 over 2*n_r + 5 steps on both sides; every buffer equal after every flush."""
    from paper_2411_18077_amd import api
    from oracle import ref
    w = small(32, L=256, keep=0.5, Rcap=32)
    inp = W.make_inputs(w, "cuda")
    Tcap = 384
    s, rs = g.shapes_for(w, Tcap)
    gc = g.gpu_build_cache(inp, s)
    rc = g.ref_build_cache(inp, rs)
    gen = torch.Generator(device="cuda"); gen.manual_seed(9)
    steps = 2 * w.Rcap + 5
    for i in range(steps):
        k = torch.randn(w.units, w.D, generator=gen, device="cuda").to(torch.float16)
        v = torch.randn(w.units, w.D, generator=gen, device="cuda").to(torch.float16)
        api.kv_append_residual(s, k, v, gc)
        api.kv_flush_residual(s, gc)
        assert ref.append_residual(rc, g.to_np(k), g.to_np(v)) == 0
        assert ref.flush_residual(rc) == 0
        if (i + 1) % w.Rcap in (0, 1) or i == steps - 1:
            torch.cuda.synchronize()
            assert gc.r_len.cpu().tolist() == rc.r_len.tolist()
            assert gc.q_len.cpu().tolist() == rc.q_len.tolist()
            g.assert_cache_bit_exact(gc, rc, what=("Kc", "Ks", "Kz", "Vc", "Vs", "Vz"))
            r = int(rc.r_len[0])
            assert np.array_equal(g.to_np(gc.Rk).reshape(w.units, w.Rcap, w.D)[:, :r], rc.Rk[:, :r])
    # a full residual refuses a further token
    for i in range(w.Rcap):
        api.kv_append_residual(s, k, v, gc)
    torch.cuda.synchronize()
    assert gc.r_len.cpu().tolist() == [w.Rcap] * w.units
    before = gc.Rk.clone()
    api.kv_append_residual(s, k + 1, v, gc)
    torch.cuda.synchronize()
    assert gc.r_len.cpu().tolist() == [w.Rcap] * w.units and torch.equal(before, gc.Rk)


@pytest.mark.parametrize("G,Rcap", [(16, 16), (16, 64), (16, 80), (16, 192), (16, 272), (32, 128), (32, 256), (64, 64),
                                    (64, 192), (128, 128), (128, 256), (128, 384)])
def test_flush_of_one_to_five_blocks(g, G, Rcap):
    """Residuals that one workgroup quantizes and counts by itself (up to 256 tokens) and longer ones: units that are
    full, that are not, and that have no room left."""
    from paper_2411_18077_amd import api
    from oracle import ref
    w = small(G, B=3, L=512, keep=0.5, Rcap=Rcap)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, inp.Tcap)
    r = np.full(w.units, Rcap, np.int32)
    r[1], r[4] = Rcap - 1, 0
    gc, rc = g.gpu_build_cache(inp, s), g.ref_build_cache(inp, rs)
    for c in (gc, rc):
        c.q_len[5] = inp.Tcap - Rcap + G                 # no room for the residual
    gc.Rk.view(w.units, Rcap, w.D).copy_(inp.Rk), gc.Rv.view(w.units, Rcap, w.D).copy_(inp.Rv)
    gc.r_len.copy_(torch.from_numpy(r))
    rc.Rk[:], rc.Rv[:], rc.r_len[:] = g.to_np(inp.Rk), g.to_np(inp.Rv), r
    api.kv_flush_residual(s, gc)
    torch.cuda.synchronize()
    assert ref.flush_residual(rc) == 0
    assert gc.r_len.cpu().tolist() == rc.r_len.tolist() == [0, Rcap - 1, 0, 0, 0, Rcap]
    g.assert_cache_bit_exact(gc, rc)


@pytest.mark.parametrize("G", [16, 128])
def test_short_calls_with_lengths_up_to_the_bound(g, G):
    """kv_quantize_pack with a host bound of at most 256 tokens: every length below it, gathered."""
    w = small(G, B=2, Hkv=4, Hq=4, L=300, keep=256 / 300)
    inp = W.make_inputs(w, "cuda")
    inp.n_tok.copy_(torch.tensor([0, G, 2 * G, 128, 256, 256 - G, 128 + G if G < 128 else 256, 128], dtype=torch.int32))
    s, rs = g.shapes_for(w, inp.Tcap)
    g.assert_cache_bit_exact(g.gpu_build_cache(inp, s), g.ref_build_cache(inp, rs))


@pytest.mark.parametrize("G,T,B", [(16, 256, 64), (16, 192, 65), (32, 256, 65), (32, 256, 16), (64, 256, 17), (64, 192, 64), (32, 128, 128), (16, 128, 129),
                                   (64, 128, 129), (32, 64, 260), (128, 256, 8), (128, 128, 65), (16, 144, 95), (32, 192, 96), (16, 160, 128), (16, 160, 129),
                                   (16, 176, 129), (64, 256, 256), (32, 192, 257)])
def test_short_calls_of_many_units(g, G, T, B):
    """Up to four blocks per unit at the unit counts where three or four of them are one workgroup or two launches (256, 384, 512
    and 1024) and beyond, with lengths of every kind; the oracle takes sampled units."""
    w = small(G, B=B, Hkv=4, Hq=4, L=T, keep=1.0)
    inp = W.make_inputs(w, "cuda")
    n = torch.tensor([T, 0, G, T - G, T // 2 // G * G], dtype=torch.int32, device="cuda")
    inp.n_tok.copy_(n.repeat(w.units // 5 + 1)[: w.units])
    s, rs = g.shapes_for(w, inp.Tcap)
    units = sorted(set([0, 1, 2, 3, 4, w.units // 2] + list(range(w.units - 6, w.units))))
    one = small(G, B=len(units), Hkv=1, Hq=1, L=T, keep=1.0)
    _, rs = g.shapes_for(one, inp.Tcap)
    gc = g.gpu_build_cache(inp, s)
    assert gc.q_len.cpu().tolist() == inp.n_tok.cpu().tolist()
    g.assert_cache_bit_exact(gc, g.ref_build_cache(inp, rs, units=units), unit_map=units)


@pytest.mark.parametrize("G,first,second", [(16, 16, 32), (16, 48, 16), (16, 80, 96), (16, 32, 304), (32, 32, 32), (32, 96, 64), (32, 32, 352),
                                            (64, 64, 64), (64, 192, 320), (128, 128, 128), (128, 384, 512)])
def test_append_behind_every_offset(g, G, first, second):
    """A second call writes behind a first one whose length is no multiple of a block or a code tile; an odd number of units
    (the last has no partner where two short ones share a wave), units of every length, rows gathered and not."""
    from paper_2411_18077_amd import api
    from oracle import ref
    w = small(G, B=5, Hkv=1, Hq=1, L=600, keep=1.0)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, 1024)
    n1 = torch.tensor([first, 0, first, G, first], dtype=torch.int32, device="cuda")
    n2 = torch.tensor([second, second, 0, second - G, second], dtype=torch.int32, device="cuda")
    idx = torch.arange(w.L - second, w.L, dtype=torch.int32, device="cuda").repeat(w.units, 1).contiguous()
    gc, rc = api.Cache(s), ref.RefCache(rs)
    api.kv_quantize_pack(s, inp.K, inp.V, w.L, None, 0, n1, first, gc)
    api.kv_quantize_pack(s, inp.K, inp.V, w.L, idx, second, n2, second, gc)
    torch.cuda.synchronize()
    assert ref.quantize_pack(rc, g.to_np(inp.K), g.to_np(inp.V), g.to_np(n1), None) == 0
    assert ref.quantize_pack(rc, g.to_np(inp.K), g.to_np(inp.V), g.to_np(n2), g.to_np(idx)) == 0
    g.assert_cache_bit_exact(gc, rc, what=("Kc", "Ks", "Kz", "Vc", "Vs", "Vz", "q_len"))
