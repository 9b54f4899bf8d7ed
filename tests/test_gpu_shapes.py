"""GPU parity of the kernels' shape edges against the fp64 oracle: head widths,
groupings, ragged matrix sizes and row counts at which a kernel or a branch of
its dispatch can go wrong.  Same measure and tolerances as the other parity
tests (1e-5 for fp32, 2e-2 for bf16, relative to the group's largest value)."""
import numpy as np
import pytest
import torch

import paper_2609_17983_amd as kvr
import synth
from oracle import decoder as od
from oracle import select as osel
from tests.gpu_util import TOL, Engine, OracleWeights, compare_repair, relmax, say, to_device_weights

pytestmark = pytest.mark.gpu


def prefill_and_repair(shape, dtype, n, edit, K, policy="edit_local", seed=0):
    """kvr_prefill of n tokens, then kvr_repair of the oracle's own prefill, both against the oracle."""
    tdt = torch.bfloat16 if dtype == kvr.KVR_BF16 else torch.float32
    w = synth.make_weights(shape, dtype=tdt, seed=seed)
    ow = OracleWeights(w, cache=True)
    s0, s1 = edit
    A = osel.select_edit_local(n, s0, s1, K) if policy == "edit_local" else osel.select_random(n, s0, s1, K, seed)
    P = od.repaired_set(s0, s1, A)
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=n + 3, max_rows=max(64, len(P)))
    try:
        toks = synth.make_tokens(n, shape.vocab, seed=seed + 1)
        say(f"case: {shape.name} prefill n={n}")
        cache = eng.new_cache(n + 3)
        hidden = torch.empty((n, shape.d_model), device="cuda")
        eng.prefill(toks.cuda(), cache, hidden)
        torch.cuda.synchronize()
        oc, oy = od.prefill(shape, ow, toks.numpy())
        got = cache.to(torch.float64).cpu().numpy()
        errs = {(l, kv): relmax(got[l, kv, :, :n], oc[l, kv]) for l in range(shape.n_layers) for kv in range(2)}
        errs["hidden"] = relmax(hidden.cpu().numpy(), oy)
        assert max(errs.values()) <= TOL[dtype], errs
        assert not got[:, :, :, n:].any()  # slots past the context stay as they were
        say(f"case: {shape.name} repair of {len(P)} rows")
        new = synth.apply_edit(toks, s0, s1 - s0, shape.vocab)
        stale = torch.from_numpy(oc).to(tdt).cuda()
        ref = stale.to(torch.float64).cpu().numpy()
        after = stale.clone()
        out = torch.full((len(P), shape.d_model), float("nan"), device="cuda")
        eng.repair([dict(cache=after, tokens=new.cuda(), edit_start=s0, edit_end=s1, positions=A, hidden=out)])
        torch.cuda.synchronize()
        y = od.repair(shape, ow, ref, new.numpy(), s0, s1, A)
        compare_repair(shape, None, stale, after, out, ref, y, P, n, TOL[dtype], shape.name)
    finally:
        eng.close()


F32, BF16 = kvr.KVR_F32, kvr.KVR_BF16
# (dtype, head_dim, query heads, kv heads): the bf16 MFMA kernel takes head_dim 64 (one and two (head, row tile) pairs
# per wavefront, two key groups) and 128; the generic kernel the rest: widths that are not multiples of four or of 16,
# both paddings (64 and 128), more than 16 query heads per kv head, one to many pairs per item
HEADS = [(BF16, 64, 4, 4), (BF16, 64, 8, 2), (BF16, 64, 14, 2), (BF16, 64, 16, 1), (BF16, 64, 17, 1), (BF16, 80, 4, 2),
         (BF16, 18, 4, 2), (BF16, 128, 18, 1), (F32, 64, 4, 4), (F32, 128, 8, 2), (F32, 6, 6, 2), (F32, 50, 6, 2),
         (F32, 96, 3, 1), (F32, 20, 33, 1)]


@pytest.mark.parametrize("items", ["split", "unsplit"])
@pytest.mark.parametrize("dtype,hd,hq,hkv", HEADS, ids=[f"{'bf16' if t else 'f32'}-{d}x{a}/{b}" for t, d, a, b in HEADS])
def test_attention_head_shapes(monkeypatch, dtype, hd, hq, hkv, items):
    """Short items of two key tiles that a combine merges, and items over all keys of a row block (49 rows and a ragged
    prefill: the last row tile holds one row)."""
    monkeypatch.setenv("KVR_ATT_TARGET", "100000" if items == "split" else "1")
    shape = synth.ModelShape(f"heads {hd}x{hq}/{hkv} {items}", 2, 64, hq, hkv, hd, 64, 128, 1e-5, 10000.0)
    prefill_and_repair(shape, dtype, 337, (201, 217), 33, seed=hd + hq)


# (dtype, d_model, kv heads, ffn, rows of the prefill, repaired rows): the generic projection's tiles (1 to 4 row tiles
# with K split over the wavefronts; 64 x 64 and 128 x 128 with a last row or column past the edge), K that is not a
# multiple of 32, of 16, of 4, or is shorter than one step per wavefront, and STORE launches cut into K slices
LINEARS = [(F32, 12, 1, 10, 65, 3), (F32, 100, 2, 262, 97, 17), (F32, 256, 4, 1003, 129, 48), (BF16, 132, 2, 70, 200, 64),
           (BF16, 36, 1, 2051, 66, 33), (F32, 1024, 4, 1500, 260, 64), (F32, 2048, 4, 2060, 1030, 65)]


@pytest.mark.parametrize("dtype,d,hkv,ffn,n,rows", LINEARS, ids=[f"{'bf16' if c[0] else 'f32'}-d{c[1]}-f{c[3]}-n{c[4]}" for c in LINEARS])
def test_generic_projection_shapes(dtype, d, hkv, ffn, n, rows):
    shape = synth.ModelShape(f"generic d{d} f{ffn}", 2 if d < 1000 else 1, d, 2 * hkv, hkv, 6 if d < 200 else 32, ffn, 96,
                             1e-5, 10000.0)
    prefill_and_repair(shape, dtype, n, (20, 20 + min(rows, 8)), rows - min(rows, 8), "random", seed=d)


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
def test_wide_residual_long_pass(dtype):
    """d_model wider than the fused Q|K|V row, and more rows than the partial buffer's fixed part holds: the output and
    down projections' results fill it up to R x d_model floats."""
    shape = synth.ModelShape("wide residual", 1, 512, 2, 1, 64, 128, 128, 1e-5, 10000.0)
    prefill_and_repair(shape, dtype, 2309, (100, 116), 40)


@pytest.mark.parametrize("n", [40, 1300, 9001], ids=lambda n: f"n{n}")
def test_topk_sizes(n):
    """The selection follows from the deviations the call returns: fewer keys than threads, and more than the block
    holds in LDS; one key, ties in bulk (duplicated cache rows) and the whole pool."""
    shape = synth.ModelShape("topk", 1, 16, 2, 1, 8, 16, 64, 1e-5, 10000.0)
    w = synth.make_weights(shape, dtype=torch.float32, seed=5)
    eng = Engine(shape, to_device_weights(w), F32, max_ctx=n, max_rows=64)
    try:
        toks = torch.full((n,), 3, dtype=torch.int32, device="cuda")  # equal values: V deviates alike at layer 0
        cache = torch.randn((1, 2, 1, n, 8), device="cuda")
        cache[:, :, :, : n // 2] = 0
        m = n - 1 - 5
        for K in (1, 7, m // 2, m):
            sel = torch.full((K,), -1, dtype=torch.int32, device="cuda")
            dev = torch.empty(m, device="cuda")
            say(f"case: top-{K} of {m}")
            got = kvr.kvr_select_cacheblend(eng.ctx, cache.data_ptr(), n, n, toks.data_ptr(), 2, 5, K, 0, sel.data_ptr(),
                                            dev.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            d = dev.cpu().numpy()
            want = np.sort(np.lexsort((np.arange(m), -d))[:K]) + 5
            assert got == K and np.array_equal(sel.cpu().numpy(), want)
    finally:
        eng.close()


# (dtype, layers, kv heads, head_dim): cache rows of 16-byte units and of 4-byte ones, planes that fill no group of four
@pytest.mark.parametrize("dtype,L,hkv,hd", [(F32, 1, 1, 6), (BF16, 3, 3, 18), (F32, 2, 1, 64), (BF16, 5, 1, 128)],
                         ids=["f32-6", "bf16-18", "f32-64", "bf16-128"])
def test_transplant_segments(dtype, L, hkv, hd):
    """Runs longer than a segment, single positions, and more segments than one launch carries."""
    shape = synth.ModelShape("copy", L, 4 if hd < 64 else 64, 2 * hkv, hkv, hd, 64, 64, 1e-5, 10000.0)
    w = synth.make_weights(shape, dtype=torch.float32 if dtype == F32 else torch.bfloat16)
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=3000, max_rows=1)
    try:
        rng = np.random.default_rng(hd)
        src = torch.randn((L, 2, hkv, 2900, hd), device="cuda").to(eng.tdtype)
        for pos in ([0], list(range(7, 7 + 33)), sorted(rng.choice(2800, size=1700, replace=False).tolist()),
                    list(range(0, 2800, 2)), list(range(2800))):
            dst = torch.randn((L, 2, hkv, 2800, hd), device="cuda").to(eng.tdtype)
            ref = dst.clone()
            ref[:, :, :, pos] = src[:, :, :, pos]
            say(f"case: transplant of {len(pos)} positions")
            kvr.kvr_transplant(eng.ctx, src.data_ptr(), 2900, dst.data_ptr(), 2800, pos,
                               torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert torch.equal(dst, ref)
    finally:
        eng.close()


# 448 x 3136: an odd number of k-steps per row (14, 98), a gate/up matrix of 24.5 column blocks, bias, seven heads per group
TILED = synth.ModelShape("tiled", 2, 448, 14, 2, 128, 3136, 256, 1e-6, 1e6, qkv_bias=True)


@pytest.mark.parametrize("rt", ["", "4", "5", "6", "7", "8"], ids=lambda r: r or "planned")
def test_tiled_row_tiles(monkeypatch, rt):
    """Each of the tiled kernel's block heights (the last row block holds one to seven row tiles, the last row tile one
    row) and the planned one; the repair's projections are cut into K slices of unequal length."""
    monkeypatch.setenv("KVR_TILED_RT", rt)
    prefill_and_repair(TILED, BF16, 785, (301, 317), 234, "random", seed=2)


# rows, documents: the first kernel takes positions from its argument, or reads the tables from host memory (several
# documents, more rows than the argument holds), or finds them on the device (tables too large to be uploaded by it)
@pytest.mark.parametrize("K,docs", [(20, 1), (20, 3), (300, 1), (1500, 3)], ids=["argument", "documents", "rows", "copied"])
def test_pass_tables_and_graph_replay(K, docs):
    """A repair captured into a graph (relaxed mode) and replayed, with eager repairs of the same edits (the same tables)
    and synchronisations between the replays: every replay equals the eager result bit for bit."""
    shape = synth.ModelShape("tables", 2, 256, 4, 2, 64, 256, 256, 1e-5, 10000.0)
    n = 2000
    w = synth.make_weights(shape, dtype=torch.bfloat16, seed=3)
    eng = Engine(shape, to_device_weights(w), BF16, max_ctx=n, max_rows=docs * (K + 16))
    try:
        toks = [synth.make_tokens(n, shape.vocab, seed=7 + i).cuda() for i in range(docs)]
        stale = [synth.make_stale_cache(shape, n, label=i).cuda() for i in range(docs)]
        caches = [s.clone() for s in stale]
        hidden = [torch.zeros((K + 16, shape.d_model), device="cuda") for _ in range(docs)]
        A = osel.select_random(n, 100, 116, K, 1)
        jobs = [dict(cache=c, tokens=t, edit_start=100, edit_end=116, positions=A, hidden=h)
                for c, t, h in zip(caches, toks, hidden)]
        say(f"case: eager repair of {docs} x {K + 16} rows")
        eng.repair(jobs)
        torch.cuda.synchronize()
        want = [h.clone() for h in hidden]
        ow = OracleWeights(w, cache=True)
        for i in range(docs):
            ref = stale[i].to(torch.float64).cpu().numpy()
            y = od.repair(shape, ow, ref, toks[i].cpu().numpy(), 100, 116, A)
            compare_repair(shape, None, stale[i], caches[i], hidden[i], ref, y, od.repaired_set(100, 116, A), n, TOL[BF16],
                           f"document {i}")
        say("case: captured repair")
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=side, capture_error_mode="relaxed"):
            eng.repair(jobs)
        for k in range(4):
            for c, s, h in zip(caches, stale, hidden):
                c.copy_(s)
                h.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(hidden, want)), f"replay {k}"
            eng.repair(jobs)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(hidden, want)), f"eager after replay {k}"
        del g
    finally:
        eng.close()


@pytest.mark.parametrize("K,docs", [(20, 1), (20, 3), (300, 1), (1500, 3)], ids=["argument", "documents", "rows", "copied"])
def test_graph_replay_after_other_work(K, docs):
    """Between the replays the context repairs another document at other positions, as many rows and fewer: a replay
    repeats the captured call on its own buffers and leaves the other cache alone."""
    shape = synth.ModelShape("tables", 2, 256, 4, 2, 64, 256, 256, 1e-5, 10000.0)
    n = 2000
    w = synth.make_weights(shape, dtype=torch.bfloat16, seed=3)
    eng = Engine(shape, to_device_weights(w), BF16, max_ctx=n, max_rows=docs * (K + 16))
    try:
        def job(i, at, count, seed):
            return dict(cache=synth.make_stale_cache(shape, n, label=i).cuda(), tokens=synth.make_tokens(n, shape.vocab, seed=i).cuda(),
                        edit_start=at, edit_end=at + 16, positions=osel.select_random(n, at, at + 16, count, seed),
                        hidden=torch.zeros((count + 16, shape.d_model), device="cuda"))

        def state(jobs):
            torch.cuda.synchronize()
            return [x.clone() for j in jobs for x in (j["cache"], j["hidden"])]

        def reset(jobs, start):
            for x, v in zip((x for j in jobs for x in (j["cache"], j["hidden"])), start):
                x.copy_(v)

        jobs = [job(i, 100, K, 1) for i in range(docs)]
        others = [[job(10 + i, 400, K, 2) for i in range(docs)], [job(20, 700, K // 2, 3)]]
        start, ostart = state(jobs), [state(o) for o in others]
        say(f"case: eager repairs of {docs} x {K + 16} rows")
        eng.repair(jobs)
        want = state(jobs)
        owant = []
        for o in others:
            eng.repair(o)
            owant.append(state(o))
        say("case: captured repair")
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=side, capture_error_mode="relaxed"):
            eng.repair(jobs)
        for k in range(4):
            for o, ow, os_ in zip(others, owant, ostart):
                reset(jobs, start)
                reset(o, os_)
                eng.repair(o)
                g.replay()
                assert all(torch.equal(a, b) for a, b in zip(state(jobs), want)), f"replay {k}"
                assert all(torch.equal(a, b) for a, b in zip(state(o), ow)), f"other document after replay {k}"
        del g
    finally:
        eng.close()


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
def test_graph_of_several_passes(dtype):
    """One call that makes many passes (a query block, then a pass per generated token), captured and replayed between
    eager repairs on the same context: each pass keeps its own tables."""
    shape = synth.ModelShape("generate", 2, 256, 4, 2, 64, 256, 256, 1e-5, 10000.0)
    n, q, new = 300, 20, 6
    w = synth.make_weights(shape, dtype=torch.bfloat16 if dtype == BF16 else torch.float32, seed=3)
    eng = Engine(shape, to_device_weights(w), dtype, max_ctx=512, max_rows=64)
    try:
        toks = synth.make_tokens(n + q + new, shape.vocab, seed=7).cuda()
        toks[n + q:] = -1
        cache = eng.new_cache(512)
        eng.prefill(toks, cache, n=n)
        other, otoks = cache.clone(), synth.make_tokens(n, shape.vocab, seed=8).cuda()
        start, tstart = cache.clone(), toks.clone()

        def generate():
            kvr.kvr_generate(eng.ctx, cache.data_ptr(), n, 512, toks.data_ptr(), q, new, torch.cuda.current_stream().cuda_stream)

        say("case: eager generation")
        generate()
        torch.cuda.synchronize()
        want, twant = cache.clone(), toks.clone()
        assert (twant[n + q:] >= 0).all()
        say("case: captured generation")
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=side, capture_error_mode="relaxed"):
            generate()
        for k in range(4):
            cache.copy_(start)
            toks.copy_(tstart)
            eng.repair([dict(cache=other, tokens=otoks, edit_start=10 + k, edit_end=20 + k, positions=[40, 50, 60], n=n)])
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(toks, twant) and torch.equal(cache, want), f"replay {k}"
        del g
    finally:
        eng.close()


@pytest.mark.parametrize("dtype,hd,hq,hkv", [(F32, 64, 4, 4), (F32, 128, 8, 4), (BF16, 80, 12, 4)],
                         ids=["f32-64", "f32-128", "bf16-80"])
def test_generic_attention_many_rows(dtype, hd, hq, hkv):
    """The generic kernel's planned items of 64 rows (their last row block holds 12 rows), split over the keys."""
    shape = synth.ModelShape(f"generic attention {hd}x{hq}/{hkv}", 1, 64, hq, hkv, hd, 64, 128, 1e-5, 10000.0)
    prefill_and_repair(shape, dtype, 1100, (700, 716), 250, "random", seed=hd)
