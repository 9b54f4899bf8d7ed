"""What a repaired row may depend on, and with how many bits: the attention of
64-wide heads carries its probabilities in full, and no row sees a later slot."""
import numpy as np
import pytest
import torch

import paper_2609_17983_amd as kvr
import synth
from oracle import decoder as od
from tests.gpu_util import TOL, Engine, OracleWeights, relmax, say, to_device_weights

pytestmark = pytest.mark.gpu
F32, BF16 = kvr.KVR_F32, kvr.KVR_BF16


def bf16(x):
    return torch.as_tensor(np.asarray(x, dtype=np.float64)).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("items", ["split", "unsplit"])
def test_probabilities_keep_all_bits(monkeypatch, items):
    """One row over 200 stale keys whose value rows nearly cancel, so that the roundings of the probabilities and of
    the sums show some thousand times as large in the output.

    The query is exact (one non-zero dimension whose rotary angle is zero to fp32, embeddings of +-1 and no epsilon), the
    scores are exact bf16 numbers, the output projection is the identity and the MLP is zero, so that what differs from
    the oracle is the softmax and P V.  The same sums in numpy: fp32 probabilities added up one by one in fp32 are off by
    2.9e-3 of the largest output, probabilities rounded to 16 bits (a pair of bf16) and summed exactly by 5.9e-2."""
    monkeypatch.setenv("KVR_ATT_TARGET", "100000" if items == "split" else "1")
    hd, hq, hkv, n = 64, 4, 2, 201
    d = hq * hd
    shape = synth.ModelShape("exact query", 1, d, hq, hkv, hd, 64, 16, 0.0, 1e30)
    rng = np.random.default_rng(5)
    zeros = lambda *s: torch.zeros(s, dtype=torch.bfloat16)
    wq = zeros(hq * hd, d)
    wq[31::hd, 0] = 8.0  # q = 8 in dimension 31 of every head: score = key's dimension 31
    lw = dict(attn_norm=torch.ones(d, dtype=torch.bfloat16), wq=wq, wk=zeros(hkv * hd, d), wv=zeros(hkv * hd, d), bq=None,
              bk=None, bv=None, wo=torch.eye(d, dtype=torch.bfloat16), mlp_norm=torch.ones(d, dtype=torch.bfloat16),
              w_gate=zeros(64, d), w_up=zeros(64, d), w_down=zeros(d, 64))
    embed = torch.from_numpy(rng.choice([-1.0, 1.0], size=(16, d))).to(torch.bfloat16)
    embed[:, 0] = 1.0
    w = dict(embed=embed, final_norm=torch.ones(d, dtype=torch.bfloat16), layers=[lw])

    cache = np.zeros((1, 2, hkv, n, hd))
    score = bf16(rng.uniform(-3, 3, size=(hkv, n - 1)))
    score[:, 5], score[:, 9] = 3.0, 2.0
    p = np.exp(score)
    v = bf16(rng.uniform(-1, 1, size=(hkv, n - 1, hd)) * 2**18)
    for g in range(hkv):  # two rows take the sum to about 2^-12 of what it was
        v[g, [5, 9]] = 0
        v[g, 5] = bf16(-(p[g] @ v[g]) / p[g, 5])
        left = -(p[g] @ v[g]) / p[g, 9]
        v[g, 9] = np.ldexp(np.rint(np.ldexp(left, 4 - np.frexp(left)[1])), np.frexp(left)[1] - 4)  # four bits of it
    cache[0, 0, :, : n - 1, 31] = score
    cache[0, 1, :, : n - 1] = v
    assert np.array_equal(bf16(cache), cache)

    tokens = torch.arange(n, dtype=torch.int32) % 16
    eng = Engine(shape, to_device_weights(w), BF16, max_ctx=n, max_rows=64)
    try:
        dev = torch.from_numpy(cache).to(torch.bfloat16).cuda()
        out = torch.zeros((1, d), device="cuda")
        say(f"case: cancelling values, {items}")
        eng.repair([dict(cache=dev, tokens=tokens.cuda(), edit_start=n - 1, edit_end=n, positions=[], hidden=out)])
        torch.cuda.synchronize()
        y = od.repair(shape, OracleWeights(w), cache, tokens.numpy(), n - 1, n, [])
        e = relmax(out.cpu().numpy(), y)
        say(f"  largest error {e:.2e} of {np.abs(y).max():.2f}")
        assert e <= 1e-2
    finally:
        eng.close()


# bf16 heads of 64 (two key groups, one and two pairs per wavefront), the generic kernel in both types, both paddings,
# head widths that are not multiples of four, and one, two and four wavefronts per pair
POISON = [(BF16, 64, 4, 4), (BF16, 64, 8, 2), (BF16, 64, 14, 2), (BF16, 80, 4, 2), (BF16, 18, 4, 2), (F32, 64, 4, 4),
          (F32, 64, 4, 2), (F32, 64, 8, 2), (F32, 128, 4, 4), (F32, 6, 6, 2), (F32, 96, 4, 1)]


@pytest.mark.parametrize("items", ["split", "unsplit"])
@pytest.mark.parametrize("dtype,hd,hq,hkv", POISON, ids=[f"{'bf16' if t else 'f32'}-{d}x{a}/{b}" for t, d, a, b in POISON])
def test_rows_do_not_see_later_slots(monkeypatch, dtype, hd, hq, hkv, items):
    """Slots of the stale cache hold infinities and NaN: the rows before them, in the same row tile as rows behind them,
    are what they are without, and the rows behind them show it."""
    monkeypatch.setenv("KVR_ATT_TARGET", "100000" if items == "split" else "1")
    shape = synth.ModelShape(f"poison {hd}x{hq}/{hkv} {items}", 2, 64, hq, hkv, hd, 64, 128, 1e-5, 10000.0)
    n, bad = 400, 170
    tdt = torch.bfloat16 if dtype == BF16 else torch.float32
    w = synth.make_weights(shape, dtype=tdt, seed=hd)
    A = [3, 90, 150, 169, 172, 230, 231, 232, 399]
    P = np.asarray(od.repaired_set(100, 104, A))
    before = P < bad
    clean = synth.make_stale_cache(shape, n).to(tdt)
    stale = clean.clone()
    stale[:, 0, :, bad, hd - 1] = float("nan")
    stale[:, 1, 0, bad, 0] = float("inf")
    stale[:, 1, :, bad + 1, hd // 2] = float("nan")
    stale[:, 1, :, n - 2, 1] = -float("inf")
    toks = synth.make_tokens(n, shape.vocab, seed=1)
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=n, max_rows=64)
    try:
        dev, out = stale.cuda(), torch.zeros((len(P), shape.d_model), device="cuda")
        say(f"case: {shape.name}")
        eng.repair([dict(cache=dev, tokens=toks.cuda(), edit_start=100, edit_end=104, positions=A, hidden=out)])
        torch.cuda.synchronize()
        ref = clean.to(torch.float64).numpy()
        y = od.repair(shape, OracleWeights(w), ref, toks.numpy(), 100, 104, A)
        got, after = out.cpu().numpy(), dev.to(torch.float64).cpu().numpy()
        assert np.isfinite(got[before]).all() and not np.isfinite(got[~before]).all(axis=1).any()
        assert relmax(got[before], y[before]) <= TOL[dtype]
        for l in range(2):
            for kv in range(2):
                rows = P[before]
                assert relmax(after[l, kv][:, rows], ref[l, kv][:, rows]) <= TOL[dtype]
    finally:
        eng.close()


# (dtype, d_model, query / kv heads, head_dim, tokens): K in one slice and in several, with and without a remainder of 16
# and of 4; both tile sizes of the many-row kernel, the larger one with two slices (added up in memory) in both types
K_ORDERS = [(F32, 256, 4, 4, 64, 1501), (F32, 200, 3, 1, 12, 700), (F32, 1044, 2, 1, 6, 700), (BF16, 268, 4, 2, 12, 700),
            (F32, 272, 28, 2, 128, 2060), (BF16, 272, 46, 2, 80, 2060), (BF16, 272, 41, 1, 80, 1800)]


@pytest.mark.parametrize("dtype,d,hq,hkv,hd,n", K_ORDERS, ids=[f"{'bf16' if c[0] else 'f32'}-{c[1]}-{c[5]}" for c in K_ORDERS])
def test_projection_rows_do_not_depend_on_the_pass(dtype, d, hq, hkv, hd, n):
    """Keys and values of layer 0 depend on a row's token and position only: CacheBlend's deviations there are exactly
    zero whether the suffix has a few rows or hundreds, and its rule falls to the lowest positions."""
    shape = synth.ModelShape(f"generic {d}", 1, d, hq, hkv, hd, 64, 256, 1e-5, 10000.0)
    w = synth.make_weights(shape, dtype=torch.bfloat16 if dtype == BF16 else torch.float32, seed=d)
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=n, max_rows=64)
    try:
        toks = synth.make_tokens(n, shape.vocab, seed=1)
        cache = eng.new_cache(n)
        say(f"case: {shape.name} prefill n={n}")
        eng.prefill(toks.cuda(), cache)
        for rows in (18, 40, 64, 65, 250, 685):
            s0, K = n - rows, min(8, rows - 5)
            new = synth.apply_edit(toks, s0, 4, shape.vocab).cuda()
            out = torch.full((K,), -1, dtype=torch.int32, device="cuda")
            dev = torch.full((n - 1 - s0 - 4,), -1.0, device="cuda")
            say(f"case: suffix of {rows} rows")
            kvr.kvr_select_cacheblend(eng.ctx, cache.data_ptr(), n, n, new.data_ptr(), s0, s0 + 4, K, 0, out.data_ptr(),
                                      dev.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert torch.count_nonzero(dev).item() == 0, (rows, dev.max().item())
            assert out.cpu().tolist() == list(range(s0 + 4, s0 + 4 + K))
    finally:
        eng.close()


@pytest.mark.parametrize("dtype,d,hq,hkv,hd,n", [(F32, 256, 4, 4, 64, 1100), (F32, 200, 6, 2, 12, 700), (BF16, 268, 4, 1, 20, 700)],
                         ids=["f32-256", "f32-200", "bf16-268"])
def test_rows_do_not_depend_on_the_rows_beside_them(monkeypatch, dtype, d, hq, hkv, hd, n):
    """With whole key ranges for every row (no split of the attention), rows recomputed over the cache of a prefill of the
    same tokens are that prefill's bit for bit, every layer and the hidden rows, whether few or hundreds: the projections
    add up K alike for every row count, and no step looks at a row's neighbours."""
    monkeypatch.setenv("KVR_ATT_TARGET", "1")
    shape = synth.ModelShape(f"rows {d}", 2, d, hq, hkv, hd, 4 * d + 24, 256, 1e-5, 10000.0)
    w = synth.make_weights(shape, dtype=torch.bfloat16 if dtype == BF16 else torch.float32, seed=d)
    for lw in w["layers"]:
        lw["wq"] *= 100  # scores spread over tens, so that rows raise their running maxima at different keys
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=n, max_rows=n)
    try:
        toks = synth.make_tokens(n, shape.vocab, seed=1).cuda()
        cache, full = eng.new_cache(n), torch.zeros((n, shape.d_model), device="cuda")
        say(f"case: {shape.name} prefill n={n}")
        eng.prefill(toks, cache, full)
        rng = np.random.default_rng(d)
        for extra in (0, 40, 61, 62, 300, n - 4):
            pool = np.setdiff1d(np.arange(n - 1), [100, 101, 102])
            A = sorted(rng.choice(pool, size=min(extra, len(pool)), replace=False).tolist())
            P = od.repaired_set(100, 103, A)
            again, out = cache.clone(), torch.zeros((len(P), shape.d_model), device="cuda")
            say(f"case: {len(P)} rows")
            eng.repair([dict(cache=again, tokens=toks, edit_start=100, edit_end=103, positions=A, hidden=out)])
            torch.cuda.synchronize()
            assert torch.equal(again, cache), (len(P), (again - cache).abs().max().item())
            assert torch.equal(out, full[P]), (len(P), (out - full[P]).abs().max().item())
    finally:
        eng.close()
