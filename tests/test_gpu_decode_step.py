"""GPU test of minikv_decode_step (Algorithm 1 lines 9 and 17-19 in one launch) against the two calls it stands
for, kv_append_residual followed by minikv_decode_attn, on identical caches: the attention output bit for bit,
the residual buffers bit for bit, the lengths it leaves in the second array equal to the ones the append leaves
in place; and, through those two calls, against the oracle."""
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


@pytest.fixture(params=[0, 1, 2], ids=["by-shape", "work-line", "work-line-equal-weights"])
def weights(request):
    """The work cut as the library chooses (a workgroup per unit at most of these sizes), then along the work line with
    either weights, as larger calls have it."""
    from paper_2411_18077_amd import api
    api.minikv_diag_decode_weights(request.param)
    yield request.param
    api.minikv_diag_decode_weights(0)


def both_ways(g, w, r_len, seed_offset=0, mutate=None):
    """Two identical caches; one takes append + attend, the other the fused step.  Returns the caches, the
    outputs and the length array the fused step wrote."""
    from paper_2411_18077_amd import api
    inp = W.make_inputs(w, "cuda", seed_offset=seed_offset)
    if mutate:
        mutate(inp)
    s, _ = g.shapes_for(w, inp.Tcap)
    ca = g.gpu_build_cache(inp, s, r_len=0)
    cb = g.gpu_build_cache(inp, s, r_len=0)
    r = torch.as_tensor(np.broadcast_to(np.asarray(r_len, np.int32), (w.units,)).copy(), device="cuda")
    ca.r_len.copy_(r)
    cb.r_len.copy_(r)
    gen = torch.Generator(device="cuda").manual_seed(4242 + seed_offset)
    k_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
    v_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
    sm = g.sm_scale()
    oa = torch.full((w.B, w.Hq, w.D), float("nan"), dtype=torch.float16, device="cuda")
    ob = torch.full_like(oa, float("nan"))
    api.kv_append_residual(s, k_new, v_new, ca)
    api.minikv_decode_attn(s, inp.q, ca, sm, oa)
    nxt = torch.full((w.units,), -77, dtype=torch.int32, device="cuda")
    api.minikv_decode_step(s, inp.q, k_new, v_new, cb, nxt, sm, ob)
    torch.cuda.synchronize()
    return s, inp, ca, cb, oa, ob, nxt, r


def assert_same(w, ca, cb, oa, ob, nxt, r_before):
    assert torch.equal(oa.view(torch.int16), ob.view(torch.int16))                 # the output, bit for bit
    assert torch.equal(ca.r_len, nxt)                                              # lengths after the append
    assert torch.equal(cb.r_len, r_before)                                         # ... the fused step's input array untouched
    # the residual rows below the new lengths (rows beyond are never read)
    Rk_a, Rk_b = ca.Rk.view(w.units, w.Rcap, w.D), cb.Rk.view(w.units, w.Rcap, w.D)
    Rv_a, Rv_b = ca.Rv.view(w.units, w.Rcap, w.D), cb.Rv.view(w.units, w.Rcap, w.D)
    n = nxt.clamp(0, w.Rcap).cpu().tolist()
    for u in range(w.units):
        assert torch.equal(Rk_a[u, : n[u]].view(torch.int16), Rk_b[u, : n[u]].view(torch.int16)), u
        assert torch.equal(Rv_a[u, : n[u]].view(torch.int16), Rv_b[u, : n[u]].view(torch.int16)), u


def tiny(G=32, **kw):
    base = dict(name="t", B=2, Hq=4, Hkv=2, L=1536, keep=0.5, G=G, Rcap=64, seed=170 + G, n_outlier=3,
                outlier_scale=8.0)
    base.update(kw)
    return W.Workload(**base)


@pytest.mark.usefixtures("weights")
@pytest.mark.parametrize("r", [0, 1, 31, 62, 63, 64])
def test_every_fill_of_the_residual(g, r):
    """Empty, one row, the last free row (the append fills the buffer), and a full buffer (nothing is appended:
    the lengths stay, the output is the attention without the new token)."""
    w = tiny()
    s, inp, ca, cb, oa, ob, nxt, rb = both_ways(g, w, r)
    assert_same(w, ca, cb, oa, ob, nxt, rb)
    assert nxt.cpu().tolist() == [min(r + 1, 64)] * w.units


@pytest.mark.usefixtures("weights")
@pytest.mark.parametrize("G,Hq,Hkv,B", [(32, 8, 8, 1), (16, 4, 2, 2), (64, 16, 2, 1), (128, 12, 3, 1), (32, 5, 5, 2),
                                        (32, 14, 2, 1)])
def test_head_layouts_and_ragged_lengths(g, G, Hq, Hkv, B):
    """Multi-head, grouped (1, 2, 4, 7, 8 heads per KV head: one and two sets of four), every group size; lengths
    differ from unit to unit, one unit holds no quantized token, one no residual token, one neither."""
    w = tiny(G, Hq=Hq, Hkv=Hkv, B=B, Rcap=max(G, 64), keep=None, keep_range=(0.05, 1.0))
    rng = np.random.default_rng(5 + Hq)
    r = rng.integers(0, w.Rcap + 1, w.units)
    r[0] = 0

    def mutate(inp):
        inp.n_tok[0] = 0                       # unit 0: nothing at all before the append
        inp.n_tok[-1] = 0

    s, inp, ca, cb, oa, ob, nxt, rb = both_ways(g, w, r, mutate=mutate)
    assert_same(w, ca, cb, oa, ob, nxt, rb)
    assert np.isfinite(ob.float().cpu().numpy()).all()


@pytest.mark.parametrize("G,Hq,Hkv,B", [(16, 2, 2, 16), (16, 16, 2, 16), (16, 5, 1, 40), (128, 8, 2, 2), (128, 16, 2, 1), (64, 8, 1, 3),
                                        (32, 16, 2, 50), (32, 2, 1, 100)])
def test_a_workgroup_per_unit_appends(g, G, Hq, Hkv, B):
    """Calls of few items per unit (at G = 16 from 32 units on), one and two sets of heads: residuals of every length, full
    ones among them, and units without any quantized token."""
    w = tiny(G, Hq=Hq, Hkv=Hkv, B=B, L=1000, Rcap=max(G, 64), keep=None, keep_range=(0.05, 0.8))
    rng = np.random.default_rng(7 + G + Hq)
    r = rng.integers(0, w.Rcap + 1, w.units)
    r[0], r[1 % w.units] = w.Rcap, 0

    def mutate(inp):
        inp.n_tok[0] = 0                       # unit 0: a full residual and nothing else
        inp.n_tok[1 % w.units] = 0             # unit 1: the appended token alone

    s, inp, ca, cb, oa, ob, nxt, rb = both_ways(g, w, r, mutate=mutate)
    assert_same(w, ca, cb, oa, ob, nxt, rb)
    assert torch.isfinite(ob).all()


@pytest.mark.usefixtures("weights")
def test_against_the_oracle(g):
    """The fused step against Algorithm 1 as the oracle runs it (append, then attention in fp64)."""
    from oracle import ref
    from paper_2411_18077_amd import api
    w = tiny(32, Hq=8, Hkv=2)
    inp = W.make_inputs(w, "cuda")
    s, rs = g.shapes_for(w, inp.Tcap)
    gc = g.gpu_build_cache(inp, s, r_len=40)
    rc = g.ref_build_cache(inp, rs, r_len=40)
    gen = torch.Generator(device="cuda").manual_seed(9)
    k_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
    v_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
    out = torch.empty(w.B, w.Hq, w.D, dtype=torch.float16, device="cuda")
    nxt = torch.zeros(w.units, dtype=torch.int32, device="cuda")
    api.minikv_decode_step(s, inp.q, k_new, v_new, gc, nxt, g.sm_scale(), out)
    torch.cuda.synchronize()
    assert ref.append_residual(rc, g.to_np(k_new), g.to_np(v_new)) == 0
    want, _, _ = ref.decode_attn(rc, g.to_np(inp.q), g.sm_scale())
    assert np.max(np.abs(g.to_np(out).astype(np.float64) - want)) <= TOL
    assert nxt.cpu().tolist() == [41] * w.units


@pytest.mark.usefixtures("weights")
def test_many_steps_with_flushes(g):
    """70 fused steps on one cache, the two length arrays swapped from step to step, a flush whenever the residual
    is full; next to it the same steps as separate calls.  Outputs and the whole cache state agree at the end."""
    from paper_2411_18077_amd import api
    w = tiny(32, Rcap=32, keep=0.25)
    inp = W.make_inputs(w, "cuda")
    s, _ = g.shapes_for(w, (inp.Tcap + 3 * 32 + 127) // 128 * 128)
    ca = g.gpu_build_cache(inp, s, r_len=30)
    cb = g.gpu_build_cache(inp, s, r_len=30)
    spare = torch.zeros(w.units, dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(11)
    oa = torch.empty(w.B, w.Hq, w.D, dtype=torch.float16, device="cuda")
    ob = torch.empty_like(oa)
    sm = g.sm_scale()
    for step in range(70):
        k_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
        v_new = torch.randn(w.units, w.D, generator=gen, device="cuda").half()
        q = torch.randn(w.B, w.Hq, w.D, generator=gen, device="cuda").half()
        api.kv_flush_residual(s, ca)                     # (acts only when the residual is full: Algorithm 1 line 10)
        api.kv_append_residual(s, k_new, v_new, ca)
        api.minikv_decode_attn(s, q, ca, sm, oa)
        api.kv_flush_residual(s, cb)
        api.minikv_decode_step(s, q, k_new, v_new, cb, spare, sm, ob)
        spare = cb.swap_r_len(spare)
        assert torch.equal(oa.view(torch.int16), ob.view(torch.int16)), step
    torch.cuda.synchronize()
    assert torch.equal(ca.r_len, cb.r_len) and torch.equal(ca.q_len, cb.q_len)
    assert int(ca.q_len[0]) == int(inp.n_tok[0]) + 3 * 32          # 30 + 70 tokens: three flushes, 4 tokens left
    assert int(ca.r_len[0]) == 4
    for name in ("Kc", "Ks", "Kz", "Vc", "Vs", "Vz"):
        assert torch.equal(ca.t[name], cb.t[name]), name


def test_arguments_are_checked_on_the_host(g):
    from paper_2411_18077_amd import api
    w = tiny()
    inp = W.make_inputs(w, "cuda")
    s, _ = g.shapes_for(w, inp.Tcap)
    c = g.gpu_build_cache(inp, s, r_len=3)
    k = torch.zeros(w.units, w.D, dtype=torch.float16, device="cuda")
    out = torch.empty(w.B, w.Hq, w.D, dtype=torch.float16, device="cuda")
    with pytest.raises(Exception):
        api.minikv_decode_step(s, inp.q, k, k, c, c.r_len, g.sm_scale(), out)     # the same array for both lengths
    with pytest.raises(Exception):
        api.minikv_decode_step(s, inp.q, None, k, c, torch.zeros_like(c.r_len), g.sm_scale(), out)


@pytest.mark.usefixtures("weights")
def test_two_fused_steps_captured_in_a_graph_and_replayed(g):
    """The length arrays alternate from step to step, so a HIP graph holds TWO steps (lengths A -> B, then B -> A),
    each with the flush in front.  The graph is replayed with new inputs in its static buffers, with eager work
    and synchronisations between the replays; a twin cache runs the same steps eagerly as separate calls, and
    every output and, at the end, the whole cache state agree bit for bit."""
    from paper_2411_18077_amd import api
    w = tiny(32, Rcap=32, keep=0.25)
    inp = W.make_inputs(w, "cuda")
    s, _ = g.shapes_for(w, (inp.Tcap + 2 * 32 + 127) // 128 * 128)
    ca = g.gpu_build_cache(inp, s, r_len=29)               # the twin, driven eagerly with the separate calls
    cb = g.gpu_build_cache(inp, s, r_len=29)
    len_a, len_b = cb.r_len, torch.zeros_like(cb.r_len)
    sm = g.sm_scale()
    ks = [torch.zeros(w.units, w.D, dtype=torch.float16, device="cuda") for _ in range(2)]
    vs = [torch.zeros_like(ks[0]) for _ in range(2)]
    qs = [torch.zeros(w.B, w.Hq, w.D, dtype=torch.float16, device="cuda") for _ in range(2)]
    outs = [torch.zeros_like(qs[0]) for _ in range(2)]
    oa = torch.zeros_like(qs[0])
    gen = torch.Generator(device="cuda").manual_seed(13)

    def fresh():
        for t in ks + vs + qs:
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda").to(torch.float16))

    def two_steps():
        api.kv_flush_residual(s, cb)                        # cb.r_len is len_a here
        api.minikv_decode_step(s, qs[0], ks[0], vs[0], cb, len_b, sm, outs[0])
        cb.swap_r_len(len_b)
        api.kv_flush_residual(s, cb)
        api.minikv_decode_step(s, qs[1], ks[1], vs[1], cb, len_a, sm, outs[1])
        cb.swap_r_len(len_a)

    def twin(i):
        api.kv_flush_residual(s, ca)
        api.kv_append_residual(s, ks[i], vs[i], ca)
        api.minikv_decode_attn(s, qs[i], ca, sm, oa)
        return oa.clone()

    fresh()
    two_steps()                                             # eagerly first (warm-up), then captured
    want = [twin(0), twin(1)]
    torch.cuda.synchronize()
    assert all(torch.equal(outs[i].view(torch.int16), want[i].view(torch.int16)) for i in range(2))
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        two_steps()
    for rep in range(20):                                   # 40 more tokens: crosses a flush
        fresh()
        graph.replay()
        torch.cuda.synchronize()
        want = [twin(0), twin(1)]
        torch.cuda.synchronize()
        for i in range(2):
            assert torch.equal(outs[i].view(torch.int16), want[i].view(torch.int16)), (rep, i)
        (ks[0].float().sum() + qs[1].float().sum()).item()  # unrelated eager work between replays
    assert torch.equal(ca.r_len, cb.r_len) and torch.equal(ca.q_len, cb.q_len)
    for name in ("Kc", "Ks", "Kz", "Vc", "Vs", "Vz", "Rk", "Rv"):
        assert torch.equal(ca.t[name], cb.t[name]), name
