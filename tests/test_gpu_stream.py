"""Whole calls of up to 16 rows (stream.hip: the projections with RMSNorm, rotary embedding, append and residual sums folded
in) against the same calls with a GEMM tile forced, at the edges of the kernels' range: row counts around 8 and 16, one half
to eight 16-row weight units per block with ragged last blocks, one to eight stages of K per wavefront."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [  # (d_model, Hq, Hkv, head_dim, d_ffn, vocab)
    (128, 2, 2, 64, 128, 128),                # one stage; half a unit
    (640, 10, 2, 64, 1152, 4224),             # uneven stages; 1 1/2 units (LM head, SwiGLU)
    (4096, 32, 8, 128, 6272, 16512),          # 1 1/2 units (QKV), 4 (SwiGLU), 5 (LM head)
    (8192, 16, 1, 128, 10240, 32000),         # the widest norm; 2 units and a row's squares of both
    (1024, 16, 4, 64, 14336, 70272),          # 7 units; 8 and several rounds of blocks
]


@pytest.mark.parametrize("chunks", [[(0, 0, 1)], [(37, 3, 4), (0, 0, 1)], [(15, 0, 5), (63, 1, 3)], [(16, 8, 8)]])
@pytest.mark.parametrize("dims", SHAPES, ids=str)
def test_small_batch_agrees_with_the_tile_kernels(dims, chunks):
    import paper_2511_07423_amd as synera
    shape = wl.ModelShape("stream", 2, *dims)
    head = wl.draw_head_weights(shape, 71, DEV)
    layers = [wl.draw_layer_weights(shape, 71, l, DEV) for l in range(shape.n_layers)]
    g = torch.Generator(device=DEV).manual_seed(72)
    rng = np.random.default_rng(73)
    ctx, u, k = (np.array(v, np.int32) for v in zip(*chunks))      # cached, uncached and draft tokens of each request
    B, T = len(chunks), int((u + k).sum())
    pages = int(max(ctx + u + k) + 15) // 16
    bt = rng.permutation(B * pages).astype(np.int32).reshape(B, pages)
    pool = (shape.n_layers, B * pages, shape.n_kv_heads)
    k_pool = torch.randn(pool + (wl.PAGE_SIZE, shape.head_dim), generator=g, device=DEV).to(torch.bfloat16)
    v_pool = torch.randn(pool + (shape.head_dim, wl.PAGE_SIZE), generator=g, device=DEV).to(torch.bfloat16)
    toks = torch.from_numpy(rng.integers(0, shape.vocab, T).astype(np.int32)).to(DEV)
    anchor = torch.from_numpy(rng.integers(0, shape.vocab, B).astype(np.int32)).to(DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=B, max_tokens=T, max_pages=pages)

    def run(tile):
        synera.debug_set_gemm_tile(tile)
        try:
            kp, vp = k_pool.clone(), v_pool.clone()
            out = ver.verify(ctx, u, k, toks, anchor, bt, B * pages, kp, vp, want_logits=True)
            torch.cuda.synchronize()
        finally:
            synera.debug_set_gemm_tile(-1)
        return out["logits"].cpu(), kp.float().cpu(), vp.float().cpu()

    got, again, tiles = run(-1), run(-1), run(101)
    ver.close()
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    scale = tiles[0].abs().max().item()
    # the LM head of the tile kernels takes the high parts alone; a bf16 flip of a cached value is carried on
    assert (got[0] - tiles[0]).abs().max().item() < 2e-3 * max(scale, 1.0)
    for a, b in zip(got[1:], tiles[1:]):           # the whole pools, what neither wrote included
        assert ((a[0] - b[0]).abs() <= 2.0 ** -7 * b[0].abs() + 1e-4).all()     # a bf16 rounding apart
        assert ((a[1] - b[1]).abs() <= 2.0 ** -7 * b[1].abs() + 1e-2).all()


@pytest.mark.parametrize("d_ffn,shift", [(192, 0), (64, 0), (256, 4)], ids=["ffn192", "ffn64", "gain8"])
def test_models_outside_the_kernels_forms_take_the_tile_kernels(d_ffn, shift):
    """An FFN width that is an odd multiple of 64, and RMSNorm gains that start 8 bytes past a 16-byte boundary, are served
    at every batch size."""
    import paper_2511_07423_amd as synera
    shape = wl.ModelShape("stream", 2, 256, 4, 4, 64, d_ffn, 128)
    head = wl.draw_head_weights(shape, 81, DEV)
    layers = [wl.draw_layer_weights(shape, 81, l, DEV) for l in range(shape.n_layers)]
    if shift:                                      # elements of 2 bytes
        moved = torch.zeros(shape.d_model + 8, dtype=torch.bfloat16, device=DEV)
        moved[shift: shift + shape.d_model] = layers[1]["mlp_norm"]
        layers[1]["mlp_norm"] = moved[shift: shift + shape.d_model]
    ctx, u, k = (np.array([v], np.int32) for v in (20, 1, 4))
    bt = np.arange(2, dtype=np.int32).reshape(1, 2)
    toks = torch.arange(5, dtype=torch.int32, device=DEV)
    anchor = torch.zeros(1, dtype=torch.int32, device=DEV)
    ver = synera.Verifier(shape, head, layers, max_batch=1, max_tokens=5, max_pages=2)

    def run(tile):
        g = torch.Generator(device=DEV).manual_seed(82)
        kp = torch.randn((2, 2, 4, wl.PAGE_SIZE, 64), generator=g, device=DEV).to(torch.bfloat16)
        vp = torch.randn((2, 2, 4, 64, wl.PAGE_SIZE), generator=g, device=DEV).to(torch.bfloat16)
        synera.debug_set_gemm_tile(tile)
        try:
            out = ver.verify(ctx, u, k, toks, anchor, bt, 2, kp, vp, want_logits=True)
            torch.cuda.synchronize()
        finally:
            synera.debug_set_gemm_tile(-1)
        return out["logits"].cpu(), kp.cpu(), vp.cpu()

    got, tiles = run(-1), run(101)
    ver.close()
    assert all(torch.isfinite(t.float()).all() for t in got)
    assert (got[0] - tiles[0]).abs().max().item() < 2e-3 * max(tiles[0].abs().max().item(), 1.0)
    for a, b in zip(got[1:], tiles[1:]):
        assert ((a[0].float() - b[0].float()).abs() <= 2.0 ** -7 * b[0].float().abs() + 1e-4).all()


@pytest.mark.parametrize("slices", range(1, 9))
def test_rotary_kernel_adds_every_number_of_slices(slices):
    """The tile kernels cut K = 256 s into s slices here, and the rotary kernel adds them; the streams have none.  384
    values per token: its last block of threads is half empty."""
    import paper_2511_07423_amd as synera
    synera.debug_set_gemm_tile(101)
    try:
        assert synera.debug_gemm_plan(12, 384, 256 * slices, 0, True)[2] == slices
    finally:
        synera.debug_set_gemm_tile(-1)
    test_small_batch_agrees_with_the_tile_kernels((256 * slices, 2, 2, 64, 128, 128), [(37, 3, 4), (15, 0, 5)])
