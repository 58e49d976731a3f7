"""GPU parity of synera_verify against the CPU oracle, through the C ABI.

Tolerances are the benchmark spec's: logits max |delta| <= 2e-2, token ids / accept lengths /
corrections exact except where the oracle's top-2 logit margin is below 1e-2, entropy within
1e-3 relative; KV page indexing bit-exact (slots that must not be written keep their NaN fill).
"""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import oracle
import workloads as wl
from helpers import oracle_model

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _report(name, rep, kv=None):
    print(f"\n[{name}] rows={rep['rows_checked']} requests={rep['requests_checked']} "
          f"max|dlogit|={rep['max_logit_err']:.3e} max rel dH={rep['max_entropy_rel']:.3e} "
          f"max rel dp={rep['max_prob_rel']:.3e} exempt rows/requests={rep['exempt_rows']}/{rep['exempt_requests']}"
          + (f" max|dKV|={kv['max_kv_err']:.3e}" if kv else ""), flush=True)


def test_config1_tiny_decoder_verify():
    case = gh.build_case(wl.config(1), DEV)
    out = gh.run_verify(case)
    rep = gh.compare_with_oracle(case, out)
    kv = gh.compare_kv(case)
    _report("c1", rep, kv)
    assert rep["ok"], rep["fail"]
    assert kv["ok"], kv["fail"]
    assert rep["rows_checked"] == 16 and rep["requests_checked"] == 4


def _mini_shape():
    return wl.ModelShape("mini_gqa", 3, 128, 4, 2, 64, 256, 256)


def test_ragged_chunks_with_uncached_tokens_and_edge_lengths():
    """Requests carrying u >= 0 uncached accepted tokens plus k drafts, chunk lengths 1..32, contexts
    from empty to several key ranges, pages permuted; compared request by request with the oracle."""
    import paper_2511_07423_amd as synera
    shape = _mini_shape()
    head = wl.draw_head_weights(shape, 21, DEV)
    layers = [wl.draw_layer_weights(shape, 21, l, DEV) for l in range(shape.n_layers)]
    model = oracle_model(shape, head, layers, np.float64)
    rng = np.random.default_rng(22)
    ctx = np.array([0, 1, 15, 16, 17, 100, 255, 256, 257, 700, 1500, 33], np.int32)
    unc = np.array([1, 0, 3, 0, 31, 0, 5, 16, 0, 2, 0, 0], np.int32)
    k = np.array([4, 1, 2, 32, 1, 7, 9, 16, 3, 8, 11, 5], np.int32)
    B = len(ctx)
    need = (ctx + unc + k + 15) // 16
    n_pages = int(need.sum()) + 7
    perm = rng.permutation(n_pages)
    max_pages = int(need.max()) + 1
    bt = np.full((B, max_pages), -1, np.int32)
    at = 0
    for i in range(B):
        bt[i, :need[i]] = perm[at:at + need[i]]
        at += int(need[i])
    okv = oracle.PagedKV(shape.n_layers, n_pages, shape.n_kv_heads, shape.head_dim)
    anchors = np.zeros(B, np.int32)
    toks, reqs = [], []
    for i in range(B):
        c = rng.integers(0, shape.vocab, int(ctx[i]))
        anchors[i] = oracle.prefill_context(model, okv, bt[i], c) if ctx[i] > 0 else int(rng.integers(0, shape.vocab))
        u = rng.integers(0, shape.vocab, int(unc[i]))
        d = rng.integers(0, shape.vocab, int(k[i]))
        if unc[i] == 0:
            d[0] = anchors[i]                                   # at least one draft can be accepted
        reqs.append({"block_table": bt[i], "ctx_len": int(ctx[i]), "uncached": u, "drafts": d, "anchor": int(anchors[i])})
        toks += [u, d]
    kp = gh.nan_pool(shape, n_pages, DEV, False)
    vp = gh.nan_pool(shape, n_pages, DEV, True)
    kd, vd = gh._oracle_pool_to_device(okv, DEV)
    for i in range(B):
        for t0 in range(0, int(ctx[i]), 16):
            m = min(16, int(ctx[i]) - t0)
            kp[:, bt[i, t0 // 16], :, :m, :] = kd[:, bt[i, t0 // 16], :, :m, :]
            vp[:, bt[i, t0 // 16], :, :, :m] = vd[:, bt[i, t0 // 16], :, :, :m]
    want = oracle.verify_chunks(model, okv, reqs)
    ver = synera.Verifier(shape, head, layers, max_batch=B, max_tokens=int((unc + k).sum()), max_pages=max_pages)
    tokens = torch.from_numpy(np.concatenate(toks).astype(np.int32)).to(DEV)
    out = ver.verify(ctx, unc, k, tokens, torch.from_numpy(anchors).to(DEV), bt, n_pages, kp, vp)
    torch.cuda.synchronize()
    got = {n: v.cpu().numpy() for n, v in out.items()}
    err = np.abs(got["logits"].astype(np.float64) - want["logits"]).max()
    print(f"\n[ragged+uncached] max|dlogit|={err:.3e}", flush=True)
    assert np.isfinite(got["logits"]).all() and err <= gh.LOGIT_TOL
    safe = want["margin"] >= gh.MARGIN
    assert np.array_equal(got["argmax"][safe], want["argmax"][safe])
    assert np.all(np.abs(got["entropy"] - want["entropy"]) <= gh.ENTROPY_RTOL * want["entropy"])
    assert np.all(np.abs(got["top1_prob"] - want["top1_prob"]) <= 2.5e-2 * want["top1_prob"] + 1e-6)
    cu = np.concatenate([[0], np.cumsum(k)])
    n_exact = 0
    for i in range(B):
        n = int(want["accept_len"][i])
        rows_ok = np.all(want["margin"][cu[i]:cu[i] + min(n + 1, int(k[i]))] >= gh.MARGIN)
        if rows_ok and want["first_margin"][i] >= gh.MARGIN:
            assert got["accept_len"][i] == n and got["correction"][i] == want["correction"][i], i
            n_exact += 1
    assert n_exact >= B // 2          # tiny vocabulary and logit spread: near-ties are common here
    # appended K/V (uncached and draft positions) land where the oracle put them; nothing else is written
    gk = kp.view(torch.int16).cpu().numpy().view(np.uint16)
    gv = vp.view(torch.int16).cpu().numpy().view(np.uint16)
    live_k = np.zeros(gk.shape, bool)                           # slots that hold a position < L + u + k
    live_v = np.zeros(gv.shape, bool)
    for i in range(B):
        for t in range(int(ctx[i] + unc[i] + k[i])):
            live_k[:, bt[i, t // 16], :, t % 16, :] = True
            live_v[:, bt[i, t // 16], :, :, t % 16] = True
    assert np.array_equal(gk != gh.NAN_BITS, live_k) and np.array_equal(gv != gh.NAN_BITS, live_v)
    dk = np.abs(oracle.bf16_from_bits(gk) - oracle.bf16_from_bits(okv.k))[live_k]
    dv = np.abs(oracle.bf16_from_bits(gv) - oracle.bf16_from_bits(okv.v))[live_v]
    assert dk.max() <= 0.05 and dv.max() <= 0.05
    # error paths launch nothing
    with pytest.raises(synera.SyneraError) as e:
        ver.verify(ctx, unc, np.where(k == 32, 33, k).astype(np.int32), tokens, torch.from_numpy(anchors).to(DEV), bt,
                   n_pages, kp, vp)
    assert e.value.status == synera.EUNSUP
    ver.close()


def test_chunked_verify_equals_sequential_decodes_on_gpu():
    """The method's own invariant on the HIP path: verifying a k-token chunk gives the rows of k
    single-token verifies with the context length advanced by one each time."""
    import paper_2511_07423_amd as synera
    case = gh.build_case(wl.config(1), DEV)
    chunk = gh.run_verify(case)
    b = case.batch
    B = len(b["ctx_len"])
    kmax = int(b["n_draft"].max())
    rows = [[] for _ in range(B)]
    for j in range(kmax):
        live = [i for i in range(B) if b["n_draft"][i] > j]
        toks = torch.tensor([int(case.drafts[i][j]) for i in live], dtype=torch.int32, device=DEV)
        out = case.verifier.verify((b["ctx_len"][live] + j).astype(np.int32), np.zeros(len(live), np.int32),
                                   np.ones(len(live), np.int32), toks,
                                   torch.zeros(len(live), dtype=torch.int32, device=DEV), b["block_table"][live],
                                   b["n_pages"], case.k_pool, case.v_pool)
        lg = out["logits"].cpu().numpy()
        for n, i in enumerate(live):
            rows[i].append(lg[n])
    seq = np.concatenate([np.stack(r) for r in rows])
    assert np.abs(seq - chunk["logits"]).max() < 2e-3


def test_out_of_range_token_ids_are_clamped_not_followed():
    """Token ids live in device memory, the host cannot validate them: ids outside [0, vocab) are
    clamped into the embedding table (regression test: such an id used to index out of bounds)."""
    case = gh.build_case(wl.config(1), DEV)
    b, V = case.batch, case.shape.vocab
    drafts = [d.copy() for d in case.drafts]
    drafts[0][0], drafts[1][1], drafts[2][2] = -7, V, 2 ** 31 - 1
    clamped = [np.clip(d, 0, V - 1) for d in drafts]
    outs = []
    for ds in (drafts, clamped):
        toks = torch.from_numpy(np.concatenate(ds).astype(np.int32)).to(DEV)
        o = case.verifier.verify(b["ctx_len"], case.n_uncached, b["n_draft"], toks,
                                 torch.from_numpy(case.anchor.astype(np.int32)).to(DEV), b["block_table"],
                                 b["n_pages"], case.k_pool, case.v_pool)
        torch.cuda.synchronize()
        outs.append(o["logits"].cpu().numpy())
    assert np.isfinite(outs[0]).all()
    assert np.allclose(outs[0], outs[1], rtol=0, atol=1e-5)


def test_model_wider_than_the_register_resident_rmsnorm():
    """d_model = 8320 > 8192: RMSNorm takes its two-pass form (the row no longer fits the registers of one
    block); a one-layer decoder, two requests, compared with the oracle."""
    import paper_2511_07423_amd as synera
    shape = wl.ModelShape("wide", 1, 8320, 2, 2, 64, 256, 256)
    head = wl.draw_head_weights(shape, 51, DEV)
    layers = [wl.draw_layer_weights(shape, 51, 0, DEV)]
    model = oracle_model(shape, head, layers, np.float64)
    rng = np.random.default_rng(52)
    ctx, unc, k = np.array([0, 21], np.int32), np.array([2, 0], np.int32), np.array([3, 5], np.int32)
    bt = np.array([[0, 1, -1], [2, 3, 4]], np.int32)
    n_pages = 5
    okv = oracle.PagedKV(1, n_pages, 2, 64)
    anchors = np.array([0, oracle.prefill_context(model, okv, bt[1], rng.integers(0, 256, 21))], np.int32)
    kp, vp = gh.nan_pool(shape, n_pages, DEV, False), gh.nan_pool(shape, n_pages, DEV, True)
    kd, vd = gh._oracle_pool_to_device(okv, DEV)
    for t0 in range(0, 21, 16):
        m = min(16, 21 - t0)
        kp[:, bt[1, t0 // 16], :, :m, :] = kd[:, bt[1, t0 // 16], :, :m, :]
        vp[:, bt[1, t0 // 16], :, :, :m] = vd[:, bt[1, t0 // 16], :, :, :m]
    toks = [rng.integers(0, 256, int(unc[i] + k[i])) for i in range(2)]
    reqs = [{"block_table": bt[i], "ctx_len": int(ctx[i]), "uncached": toks[i][:unc[i]], "drafts": toks[i][unc[i]:],
             "anchor": int(anchors[i])} for i in range(2)]
    want = oracle.verify_chunks(model, okv, reqs)
    ver = synera.Verifier(shape, head, layers, max_batch=2, max_tokens=16, max_pages=3)
    out = ver.verify(ctx, unc, k, torch.from_numpy(np.concatenate(toks).astype(np.int32)).to(DEV),
                     torch.from_numpy(anchors).to(DEV), bt, n_pages, kp, vp)
    torch.cuda.synchronize()
    err = np.abs(out["logits"].double().cpu().numpy() - want["logits"]).max()
    print(f"\n[wide d=8320] max|dlogit|={err:.3e}", flush=True)
    assert err <= gh.LOGIT_TOL
    safe = want["margin"] >= gh.MARGIN
    assert np.array_equal(out["argmax"].cpu().numpy()[safe], want["argmax"][safe])
    ver.close()


def test_a_request_with_nan_in_its_cache_leaves_the_others_untouched(monkeypatch):
    """Requests are independent: NaN in one request's cached K/V makes that request's outputs NaN and
    changes no bit of any other request's.  The attention kernel is cut down to 2 persistent blocks, so that
    every block runs many streams one after another and the poisoned request's streams come first in them:
    whatever a stream leaves in a block's registers must not reach the next one."""
    import paper_2511_07423_amd as synera
    monkeypatch.setenv("SYNERA_ATTN_BLOCKS", "2")
    shape = _mini_shape()
    head = wl.draw_head_weights(shape, 31, DEV)
    layers = [wl.draw_layer_weights(shape, 31, l, DEV) for l in range(shape.n_layers)]
    g = torch.Generator(device=DEV).manual_seed(32)
    rng = np.random.default_rng(33)
    ctx = np.array([90, 40, 300, 17, 64, 1, 700, 33], np.int32)
    k = np.array([5, 16, 1, 8, 32, 3, 9, 12], np.int32)
    B = len(ctx)
    need = (ctx + k + 15) // 16
    n_pages, max_pages = int(need.sum()), int(need.max())
    bt = np.full((B, max_pages), -1, np.int32)
    at = 0
    for i in range(B):
        bt[i, :need[i]] = np.arange(at, at + need[i])
        at += int(need[i])
    pool = (shape.n_layers, n_pages, shape.n_kv_heads)
    k_pool = torch.randn(pool + (wl.PAGE_SIZE, shape.head_dim), generator=g, device=DEV).to(torch.bfloat16)
    v_pool = torch.randn(pool + (shape.head_dim, wl.PAGE_SIZE), generator=g, device=DEV).to(torch.bfloat16)
    toks = torch.from_numpy(rng.integers(0, shape.vocab, int(k.sum())).astype(np.int32)).to(DEV)
    anchor = torch.from_numpy(rng.integers(0, shape.vocab, B).astype(np.int32)).to(DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=B, max_tokens=int(k.sum()), max_pages=max_pages)
    zeros = np.zeros(B, np.int32)

    def run(kp, vp):
        out = ver.verify(ctx, zeros, k, toks, anchor, bt, n_pages, kp, vp, want_logits=True)
        torch.cuda.synchronize()
        return {n: v.cpu().numpy() for n, v in out.items() if v is not None}

    clean = run(k_pool.clone(), v_pool.clone())
    assert all(np.isfinite(v).all() for v in clean.values())
    bad_k, bad_v = k_pool.clone(), v_pool.clone()
    bad_k[:, int(bt[0, 0]), :, :8, :] = float("nan")        # positions 0..7 of request 0: inside its context
    bad_v[:, int(bt[0, 1]), :, :, :4] = float("inf")        # positions 16..19
    dirty = run(bad_k, bad_v)
    ver.close()
    cu = np.concatenate([[0], np.cumsum(k)])
    assert not np.isfinite(dirty["logits"][:cu[1]]).all()    # the poisoned request shows it
    for name in ("logits", "argmax", "top1_prob", "entropy"):
        assert np.array_equal(clean[name][cu[1]:], dirty[name][cu[1]:]), name
    for name in ("accept_len", "correction"):
        assert np.array_equal(clean[name][1:], dirty[name][1:]), name


@pytest.mark.parametrize("heads", [(4, 4, 64), (16, 4, 128)], ids=["hd64", "hd128"])
@pytest.mark.parametrize("ctx,k", [(100, 1), (180, 4), (400, 4), (900, 16), (3000, 4), (6000, 16)])
def test_streams_cut_over_blocks_merge_to_the_whole(heads, ctx, k):
    """A lone request's keys cut into anything from one share to dozens (the merge takes eight at a time) against the same
    verify with at most two blocks in the plan.  A share rounds its probabilities to bf16 pairs (2^-17) against its own
    reference maximum: 2^-16 sum(p |v|) in o, whose size is that sum over sqrt(keys) or more: 1e-3."""
    import paper_2511_07423_amd as synera
    Hq, Hkv, hd = heads
    shape = wl.ModelShape("cut", 1, 512, Hq, Hkv, hd, 256, 256)
    head = wl.draw_head_weights(shape, 91, DEV)
    layers = [wl.draw_layer_weights(shape, 91, 0, DEV)]
    g = torch.Generator(device=DEV).manual_seed(92)
    pages = (ctx + k + 15) // 16
    k_pool = torch.randn((1, pages, Hkv, 16, hd), generator=g, device=DEV).to(torch.bfloat16)
    v_pool = torch.randn((1, pages, Hkv, hd, 16), generator=g, device=DEV).to(torch.bfloat16)
    bt = np.random.default_rng(93).permutation(pages).astype(np.int32).reshape(1, pages)
    args = [np.array([n], np.int32) for n in (ctx, 0, k)]
    toks = torch.arange(k, dtype=torch.int32, device=DEV)
    anchor = torch.zeros(1, dtype=torch.int32, device=DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=1, max_tokens=k, max_pages=pages)

    def run():
        out = ver.verify(*args, toks, anchor, bt, pages, k_pool, v_pool, want_logits=True)
        imp = ver.importance(*args, pages, k_pool, i_th=0.05)
        torch.cuda.synchronize()
        return out["logits"].cpu().double(), imp["scores"].cpu().double()

    got = run()
    ver.debug_set_attention_plan(attn_blocks=2)
    want = run()
    ver.close()
    for a, b in zip(got, want):
        assert torch.isfinite(a).all() and torch.isfinite(b).all()
        assert (a - b).norm().item() <= 1e-3 * b.norm().item()


def test_both_forms_of_the_activation_pair_give_the_same_bits():
    """A projection whose stage holds one 32-wide K block reads its (hi, lo) activations as one array of whole
    128-byte lines, written that way by RMSNorm, by the attention's normalising store and by the SwiGLU epilogue;
    otherwise as two arrays.  Same tile, same MFMAs in the same order: with the tile forced, the verify must give
    the same bits in both forms (the two-array form is kept by the low-part switch of the LM head's input, which
    changes no arithmetic: the LM head runs on the high part either way), and the planner's own choice for this
    small shape (64-wide stages, two arrays) must agree to rounding."""
    import paper_2511_07423_amd as synera
    shape = wl.ModelShape("pairs", 2, 512, 8, 2, 64, 1024, 512)
    head = wl.draw_head_weights(shape, 61, DEV)
    layers = [wl.draw_layer_weights(shape, 61, l, DEV) for l in range(shape.n_layers)]
    g = torch.Generator(device=DEV).manual_seed(62)
    rng = np.random.default_rng(63)
    B = 20
    ctx = rng.integers(0, 400, B).astype(np.int32)
    k = rng.integers(1, 33, B).astype(np.int32)
    k[0], k[1] = 32, 1
    T = int(k.sum())
    assert T > 144
    need = (ctx + k + 15) // 16
    n_pages, max_pages = int(need.sum()), int(need.max())
    bt = np.full((B, max_pages), -1, np.int32)
    perm, at = rng.permutation(n_pages), 0
    for i in range(B):
        bt[i, :need[i]] = perm[at:at + need[i]]
        at += int(need[i])
    pool = (shape.n_layers, n_pages, shape.n_kv_heads)
    k_pool = torch.randn(pool + (wl.PAGE_SIZE, shape.head_dim), generator=g, device=DEV).to(torch.bfloat16)
    v_pool = torch.randn(pool + (shape.head_dim, wl.PAGE_SIZE), generator=g, device=DEV).to(torch.bfloat16)
    toks = torch.from_numpy(rng.integers(0, shape.vocab, T).astype(np.int32)).to(DEV)
    anchor = torch.from_numpy(rng.integers(0, shape.vocab, B).astype(np.int32)).to(DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=B, max_tokens=T, max_pages=max_pages)
    zeros = np.zeros(B, np.int32)
    qkv_n = (shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim

    def run(tile, lo_off):
        synera.debug_set_gemm_tile(tile)
        ver.debug_set_lo_off(lo_off)
        try:
            stage_k = [synera.debug_gemm_plan_bk(T, n, kk, epi, 1) for n, kk, epi in
                       ((qkv_n, shape.d_model, 0), (shape.d_model, shape.n_q_heads * shape.head_dim, 1),
                        (2 * shape.d_ffn, shape.d_model, 2), (shape.d_model, shape.d_ffn, 1))]
            kp, vp = k_pool.clone(), v_pool.clone()
            out = ver.verify(ctx, zeros, k, toks, anchor, bt, n_pages, kp, vp, want_logits=True)
            torch.cuda.synchronize()
        finally:
            synera.debug_set_gemm_tile(-1)
            ver.debug_set_lo_off(0)
        res = {n: v.cpu().numpy() for n, v in out.items() if v is not None}
        res["k_pool"], res["v_pool"] = kp.view(torch.int16).cpu().numpy(), vp.view(torch.int16).cpu().numpy()
        return res, stage_k

    planned, sk0 = run(-1, [])
    paired, sk1 = run(108, [])                     # 128 x 128 tiles, one 32-wide K block per stage: one paired array
    two, sk2 = run(108, ["lm_head_in"])            # the same tiles on two arrays
    ver.close()
    assert sk1 == [32, 32, 32, 32] and sk2 == [32, 32, 32, 32], (sk1, sk2)
    assert all(np.isfinite(v).all() for n, v in paired.items() if n not in ("k_pool", "v_pool"))
    for name in paired:
        assert np.array_equal(paired[name], two[name]), name
    assert np.abs(paired["logits"] - planned["logits"]).max() < 1e-4, sk0
    assert np.array_equal(paired["accept_len"], planned["accept_len"])


def test_pools_that_are_not_16_byte_aligned_are_refused():
    """The attention kernel copies 16 bytes per lane straight out of the pools: a pool pointer off that alignment is
    an argument error, raised before anything is launched."""
    import paper_2511_07423_amd as synera
    shape = _mini_shape()
    head = wl.draw_head_weights(shape, 71, DEV)
    layers = [wl.draw_layer_weights(shape, 71, l, DEV) for l in range(shape.n_layers)]
    ctx, k = np.array([20], np.int32), np.array([4], np.int32)
    bt = np.array([[0, 1]], np.int32)
    n = shape.n_layers * 2 * shape.n_kv_heads * wl.PAGE_SIZE * shape.head_dim
    flat_k = torch.zeros(n + 8, dtype=torch.bfloat16, device=DEV)
    flat_v = torch.zeros(n + 8, dtype=torch.bfloat16, device=DEV)
    shp_k = (shape.n_layers, 2, shape.n_kv_heads, wl.PAGE_SIZE, shape.head_dim)
    shp_v = (shape.n_layers, 2, shape.n_kv_heads, shape.head_dim, wl.PAGE_SIZE)
    toks = torch.zeros(4, dtype=torch.int32, device=DEV)
    anchor = torch.zeros(1, dtype=torch.int32, device=DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=1, max_tokens=4, max_pages=2)
    zeros = np.zeros(1, np.int32)
    good = ver.verify(ctx, zeros, k, toks, anchor, bt, 2, flat_k[:n].view(shp_k), flat_v[:n].view(shp_v))
    torch.cuda.synchronize()
    assert good["argmax"].shape[0] == 4
    for kp, vp in ((flat_k[1:n + 1].view(shp_k), flat_v[:n].view(shp_v)), (flat_k[:n].view(shp_k), flat_v[4:n + 4].view(shp_v))):
        with pytest.raises(synera.SyneraError) as e:
            ver.verify(ctx, zeros, k, toks, anchor, bt, 2, kp, vp)
        assert e.value.status == synera.EINVAL
    ver.close()
