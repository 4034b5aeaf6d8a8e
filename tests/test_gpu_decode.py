"""GPU parity of the decode step (locret_decode_step: Eq. 1 with B = 1 on the retained cache)
against the oracle, which runs the same token through its general chunk step with T = 1 and no
eviction.  A teacher-forced prefill stream first brings both caches to the same state."""
import numpy as np
import pytest
import torch

from paper_2410_01805_amd import synth
from tests.gpu_util import DEV, assert_close, dev, host, kappa_for, make_layer, make_oracle
from tests.test_gpu_prefill import _run_stream

pytestmark = pytest.mark.gpu

N_DEC = 7

CASES = [
    dict(name="dec_f32_gqa", dtype="f32", h=8, h_kv=2, d=64, N=1000, B=200, b=400, n_s=32, d_R=64, rope=False),
    dict(name="dec_f32_rope_d32", dtype="f32", h=4, h_kv=2, d=32, N=800, B=160, b=300, n_s=40, d_R=64, rope=True),
    dict(name="dec_f32_mha_d16", dtype="f32", h=3, h_kv=3, d=16, N=500, B=100, b=150, n_s=0, d_R=40, rope=True),
    dict(name="dec_f32_d128", dtype="f32", h=4, h_kv=2, d=128, N=700, B=128, b=333, n_s=10, d_R=64, rope=True),
    dict(name="dec_bf16_llama_like", dtype="bf16", h=8, h_kv=2, d=128, N=1500, B=300, b=700, n_s=100, d_R=128,
         theta=500000.0),
    dict(name="dec_bf16_phi_like", dtype="bf16", h=4, h_kv=4, d=96, N=1200, B=256, b=600, n_s=64, d_R=128),
    dict(name="dec_bf16_g8_norope", dtype="bf16", h=8, h_kv=1, d=64, N=1100, B=250, b=500, n_s=50, d_R=128,
         rope=False),
    dict(name="dec_bf16_g3", dtype="bf16", h=6, h_kv=2, d=128, N=900, B=128, b=641, n_s=30, d_R=128),
    dict(name="dec_bf16_short_cache", dtype="bf16", h=8, h_kv=2, d=128, N=40, B=64, b=256, n_s=8, d_R=128),
]


def _prefill(w):
    """Teacher-forced prefill of the first N - N_DEC tokens."""
    n_pre = w.N - N_DEC
    sizes = [w.B] * (n_pre // w.B) + ([n_pre % w.B] if n_pre % w.B else [])
    layer, o, _ = _run_stream(w, teacher_forced=True, chunk_sizes=sizes)
    assert layer.cache_len == o.n_c
    return layer, o, n_pre


@pytest.mark.parametrize("kw", CASES, ids=[c["name"] for c in CASES])
def test_decode_tokens_with_scores(kw):
    w = synth.tiny(**kw)
    layer, o, n_pre = _prefill(w)
    n0 = o.n_c
    for i in range(N_DEC):
        q, k, v = synth.tokens(w, n_pre + i, n_pre + i + 1)
        out_ref, sc_ref, _ = o.prefill_chunk(q, k, v, 0, evict=False)
        out, sc = layer.decode_step(dev(q, w), dev(k, w), dev(v, w), with_score=True)
        tag = f"{w.name} token {i}"
        assert_close(host(out), out_ref, w.dtype, tag + " attention", per_row=True)
        assert_close(sc.cpu().numpy(), sc_ref[:, 0], w.dtype, tag + " score")
        assert layer.cache_len == o.n_c == n0 + i + 1
    K, V, S, P = layer.cache_tensors()
    for m in range(w.h_kv):
        np.testing.assert_array_equal(P[m].cpu().numpy(), o.P[m])
        np.testing.assert_array_equal(host(K[m]), o.K[m].astype(np.float32))
        np.testing.assert_array_equal(host(V[m]), o.V[m].astype(np.float32))
        s = S[m].cpu().numpy()
        np.testing.assert_array_equal(s[:n0], o.S[m][:n0])          # prefill part: teacher-forced, exact
    layer.close()


@pytest.mark.parametrize("h,h_kv,d,d_R", [(1, 1, 64, 128), (4, 2, 64, 256), (8, 2, 128, 384), (6, 6, 96, 128), (33, 33, 64, 128), (16, 2, 64, 128)])
def test_scores_of_one_token(h, h_kv, d, d_R):
    """The single-token form of the retaining head: contractions shorter than and no multiple of a wavefront's 512 elements, more
    than 32 KV heads; locret_score, locret_score_static, a decode step and a chunk of one token give the same score.
    All sums are float32 over exact products of bf16 values, so the float32 bound applies."""
    from paper_2410_01805_amd import binding as B
    w = synth.tiny(name="one_token", dtype="bf16", h=h, h_kv=h_kv, d=d, N=3, B=4, b=8, n_s=1, d_R=d_R)
    layer, W1, W2 = make_layer(w)
    o = make_oracle(w, W1, W2)
    q, k, v = synth.tokens(w, 0, 1)
    ref = o.score(q, k, v)
    x = [dev(t, w) for t in (q, k, v)]
    sc = layer.score(*x).cpu().numpy()
    assert_close(sc, ref, "f32", "one token")
    static = torch.empty(h_kv, 1, device=DEV)
    B.locret_score_static(layer.ctx, *x, 1, static)
    np.testing.assert_array_equal(static.cpu().numpy(), sc)
    _, chunk, _ = layer.prefill_chunk(*x, 0)
    np.testing.assert_array_equal(chunk.cpu().numpy(), sc)
    _, token = layer.decode_step(*x, with_score=True)
    np.testing.assert_array_equal(token.cpu().numpy(), sc[:, 0])
    S = layer.cache_tensors()[2].cpu().numpy()
    np.testing.assert_array_equal(S, np.repeat(sc, 2, axis=1))
    layer.close()


def test_decode_without_scores_then_evicting_chunk():
    # generated units carry NaN scores; a later evicting chunk drops them before any scored unit
    w = synth.tiny(name="dec_nan", dtype="bf16", h=8, h_kv=2, d=128, N=1400, B=200, b=500, n_s=40, d_R=128)
    layer, o, n_pre = _prefill(w)
    n0 = o.n_c
    for i in range(N_DEC):
        q, k, v = synth.tokens(w, n_pre + i, n_pre + i + 1)
        out_ref, _, _ = o.prefill_chunk(q, k, v, 0, evict=False)
        out, sc = layer.decode_step(dev(q, w), dev(k, w), dev(v, w), with_score=False)
        assert sc is None
        assert_close(host(out), out_ref, w.dtype, f"token {i} attention", per_row=True)
    for m in range(w.h_kv):
        o.S[m][n0:] = np.nan                                          # what the library stores for them
    K, V, S, P = layer.cache_tensors()
    for m in range(w.h_kv):
        s = S[m].cpu().numpy()
        assert np.isnan(s[n0:]).all() and not np.isnan(s[:n0]).any()
        np.testing.assert_array_equal(host(K[m]), o.K[m].astype(np.float32))
    q, k, v = synth.tokens(w, 0, w.B - N_DEC)                         # a further chunk that still fits, teacher-forced
    out_ref, sc_ref, kept_ref = o.prefill_chunk(q, k, v, w.n_s)
    out, sc, kept = layer.prefill_chunk(dev(q, w), dev(k, w), dev(v, w), w.n_s,
                                        scores_in=torch.from_numpy(sc_ref).to(DEV))
    np.testing.assert_array_equal(kept.cpu().numpy()[:, :w.b], kept_ref)
    assert not np.isin(np.arange(n0, n0 + N_DEC), kept_ref[0]).any()   # the generated units went first
    assert_close(host(out), out_ref, w.dtype, "chunk after decode", per_row=True)
    layer.close()


def test_decode_capacity_and_argument_errors():
    from paper_2410_01805_amd import binding as B
    w = synth.tiny(name="dec_err", dtype="f32", h=4, h_kv=2, d=32, N=600, B=4, b=8, n_s=2, d_R=64)
    layer = B.LocretLayer(B.config_from_workload(w), DEV)
    q, k, v = (dev(x, w) for x in synth.tokens(w, 0, 1))
    with pytest.raises(B.LocretError) as e:        # scoring needs weights
        layer.decode_step(q, k, v, with_score=True)
    assert e.value.code == B.LOCRET_ESTATE
    for _ in range(12):                            # capacity = budget + chunk_max = 12 units
        layer.decode_step(q, k, v, with_score=False)
    assert layer.cache_len == 12
    with pytest.raises(B.LocretError) as e:
        layer.decode_step(q, k, v, with_score=False)
    assert e.value.code == B.LOCRET_ESTATE
    with pytest.raises(B.LocretError) as e:
        B.locret_decode_step(layer.ctx, q.data_ptr() + 4, k, v, 0, torch.empty_like(q))
    assert e.value.code == B.LOCRET_EALIGN
    layer.close()


def test_decode_on_the_full_budget_of_config3():
    # the headline layer with its cache at the budget: one generated token over 16384 units
    w = synth.WORKLOADS["cfg3_llama_128k"]
    layer, W1, W2 = make_layer(w)
    o = make_oracle(w, W1, W2)
    for c in range(5):                             # 5 chunks: cache full and compacted once
        q, k, v = synth.chunk(w, c)
        sc_ref = o.score(q, k, v)
        o.evict_compact(sc_ref, k, v, w.n_s)
        layer.prefill_chunk(dev(q, w), dev(k, w), dev(v, w), w.n_s, scores_in=torch.from_numpy(sc_ref).to(DEV))
    assert layer.cache_len == o.n_c == w.b
    for i in range(3):
        q, k, v = synth.tokens(w, 5 * w.B + i, 5 * w.B + i + 1)
        out_ref, _, _ = o.prefill_chunk(q, k, v, 0, evict=False)
        out, _ = layer.decode_step(dev(q, w), dev(k, w), dev(v, w), with_score=False)
        assert_close(host(out), out_ref, w.dtype, f"cfg3 decode token {i}", per_row=True, kappa=kappa_for(w))
    layer.close()


@pytest.mark.parametrize("h,h_kv,d", [(2, 2, 128), (4, 2, 96), (8, 2, 128), (12, 2, 64), (4, 1, 32)])
def test_decode_block_edges(h, h_kv, d):
    """Cache lengths around the 32-key blocks of a wavefront, the four of a workgroup and the first lengths with two splits, for one,
    two and four heads a launch; an infinite value (of the last key in the cache, where spare rows repeat it) stays infinite and alone."""
    w = synth.tiny(name=f"dec_edges_{h}_{h_kv}_{d}", dtype="bf16", h=h, h_kv=h_kv, d=d, N=400, B=200, b=400, n_s=0, d_R=128)
    layer, W1, W2 = make_layer(w)
    o = make_oracle(w, W1, W2)
    n = 0
    for upto in (1, 31, 32, 33, 63, 95, 127, 128, 129, 160, 191, 255, 256, 257, 319):
        while n < upto:
            end = min(upto, n + w.B)
            x = synth.tokens(w, n, end)
            o.prefill_chunk(*x, 0, evict=False)
            layer.evict_compact(torch.zeros(h_kv, end - n, device=DEV), dev(x[1], w), dev(x[2], w), 0)
            n = end
        x = synth.tokens(w, n, n + 1)
        ref, _, _ = o.prefill_chunk(*x, 0, evict=False)
        out, _ = layer.decode_step(*(dev(t, w) for t in x))
        n += 1
        assert_close(host(out), ref, w.dtype, f"{w.name} {upto}", per_row=True)
    # the same cache with one infinite element in a value row that every head sees
    q, k, v = (dev(t, w) for t in synth.tokens(w, n, n + 1))
    v[0, 0, 5] = float("inf")
    layer.evict_compact(torch.zeros(h_kv, 1, device=DEV), k, v, 0)
    out = layer.decode_step(*(dev(t, w) for t in synth.tokens(w, n + 1, n + 2)))[0][0].float().cpu()
    g = h // h_kv
    expect = torch.zeros(h, d, dtype=torch.bool)
    expect[:g, 5] = True
    assert torch.equal(out == float("inf"), expect) and bool(torch.isfinite(out[~expect]).all())
    layer.close()


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 96), ("bf16", 128), ("bf16", 64)])
def test_decode_merge_of_many_splits(dtype, d, monkeypatch):
    """Splits of 64 keys (LOCRET_DEC_KEYS), 3 ... 260 of them, around what the merge requests at once (96) and holds the weights of
    (128), against splits at least four times as long.  Same arithmetic on the keys, so float32 results differ by the order
    of sums of convex weights (2^-20 is 16 roundings), bf16 ones by that before one rounding (2^-7: two neighbours)."""
    w = synth.tiny(name="merge", dtype=dtype, h=4, h_kv=2, d=d, N=17000, B=17000, b=17000, n_s=0, d_R=128)
    layers = []
    for keys in ("64", "320"):
        monkeypatch.setenv("LOCRET_DEC_KEYS", keys)
        layers.append(make_layer(w)[0])
    gen = torch.Generator(device=DEV).manual_seed(3)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=gen).to(tdt)
    n = 0
    for splits in (2, 63, 64, 65, 94, 95, 96, 97, 126, 127, 128, 129, 130, 191, 259):
        k, v = rnd(64 * splits - n, 2, d), rnd(64 * splits - n, 2, d)
        token = rnd(1, 4, d), rnd(1, 2, d), rnd(1, 2, d)
        outs = []
        for layer in layers:
            layer.evict_compact(torch.zeros(2, len(k), device=DEV), k, v, 0)
            outs.append(layer.decode_step(*token)[0].float())
        n = 64 * splits + 1
        err = (outs[0] - outs[1]).abs().max() / outs[1].abs().max()
        assert err <= (2.0 ** -20 if dtype == "f32" else 2.0 ** -7), (splits, float(err))
    for layer in layers:
        layer.close()


@pytest.mark.parametrize("d", [64, 96, 128])
def test_decode_merge_sums_the_splits_in_eight_chains(d, monkeypatch):
    """64 splits of equal weight whose results are odd whole numbers near 2^21, of alternating sign: split s in the chain s mod 8 meets
    eight of one sign, which stay below 2^24 and therefore exact, and so do all sums of chains; sixteen of one sign would not."""
    monkeypatch.setenv("LOCRET_DEC_KEYS", "64")
    w = synth.tiny(name=f"chains_{d}", dtype="f32", h=2, h_kv=1, d=d, N=4096, B=4095, b=4096, n_s=0, d_R=64, rope=False)
    layer, _, _ = make_layer(w)
    V = torch.zeros(4095, 1, d, dtype=torch.float64)
    s = torch.arange(64)[:, None]
    V[::64, 0] = ((-1.0) ** s) * (2 ** 21 - 1 - 2 * ((s * 37 + torch.arange(d) * 11) % 512))
    layer.evict_compact(torch.zeros(1, 4095, device=DEV), torch.zeros(4095, 1, d, device=DEV), V.float().to(DEV), 0)
    zero = lambda n: torch.zeros(1, n, d, device=DEV)
    out = layer.decode_step(zero(2), zero(1), zero(1))[0].cpu().double()       # the token's own value is 0, its weight that of any unit
    assert torch.equal(out[0, 0], V.sum(0)[0] / 4096) and torch.equal(out[0, 1], out[0, 0])
    layer.close()
