"""Host logic of the projection GEMM's tile planner (no GPU call): the plans of the headline batch, and
properties every plan must have for the launch to be valid."""
import pytest

import paper_2511_07423_amd as synera

STORE, ADD, SWIGLU = 0, 1, 2
# the projections of one decoder layer and the LM head at the 8B shape (Section 6.1's cloud model class)
D, F, QKV, VOCAB = 4096, 14336, 6144, 32000


def test_headline_batch_plans():
    """532 draft rows: every projection on 256-column tall tiles; the few-tile ones split K into stored slices."""
    T = 532
    assert synera.debug_gemm_plan(T, QKV, D, STORE) == (272, 256, 5)
    assert synera.debug_gemm_plan(T, D, D, ADD) == (144, 256, 4)
    assert synera.debug_gemm_plan(T, 2 * F, D, SWIGLU) == (272, 256, 1)
    assert synera.debug_gemm_plan(T, D, F, ADD) == (272, 256, 8)
    assert synera.debug_gemm_plan(T, VOCAB, D, STORE, stored_slices=False) == (272, 256, 1)
    for n, k, e in ((QKV, D, STORE), (D, D, ADD), (2 * F, D, SWIGLU), (D, F, ADD)):
        assert synera.debug_gemm_plan_bk(T, n, k, e) == 32          # the tall tiles fill the LDS with 64-byte rows


def test_small_batches_take_the_narrow_tiles():
    """About 140 rows: 128-column tiles double the blocks that stream the weights, and those tiles are short
    enough for two MFMA K steps per stage (half the barriers, full 128-byte rows per copy)."""
    for n, k, e in ((QKV, D, STORE), (D, D, ADD), (2 * F, D, SWIGLU), (D, F, ADD)):
        assert synera.debug_gemm_plan(144, n, k, e)[1] == 128
        assert synera.debug_gemm_plan_bk(144, n, k, e) == 64
        assert synera.debug_gemm_plan_bk(128, n, k, e) == 64


def test_decode_sized_batches_use_tiles_of_their_own_height_and_never_atomics():
    """Below 128 rows the tile is as tall as the batch (one M tile); K may only be split into stored slices,
    and without a slice buffer (the stand-alone mode) it is not split at all: no path adds with atomics."""
    for M in (1, 8, 16, 17, 64, 96):
        for n, k, e in ((QKV, D, STORE), (D, D, ADD), (2 * F, D, SWIGLU), (D, F, ADD), (VOCAB, D, STORE)):
            bm, bn, split = synera.debug_gemm_plan(M, n, k, e)
            assert bm == (M + 15) // 16 * 16
            assert synera.debug_gemm_plan(M, n, k, e, stored_slices=False)[2] == 1


# The K slices of the projections that may be sliced, from the first row count each number holds for (17 to 1100 rows); with the
# stage's k where it moves the cuts.  They are the order of the sums, and with it the bits of every K and V row a layer appends.
SLICES = {
    (QKV, D, STORE): [(17, 5, 64), (145, 5, 32), (417, 3, 32), (433, 5, 32), (513, 3, 32), (529, 5, 32), (545, 2, 0)],
    (D, D, ADD): [(17, 8, 0), (185, 4, 0), (289, 8, 0), (307, 4, 0), (321, 5, 32), (433, 4, 0), (493, 2, 0), (513, 4, 0), (555, 2, 0),
                  (577, 4, 0), (705, 3, 32), (721, 4, 0), (769, 3, 32), (801, 4, 0), (833, 3, 32), (881, 4, 0), (917, 2, 0),
                  (986, 1, 0), (1025, 3, 32), (1041, 2, 0)],
    (D, F, ADD): [(17, 8, 0), (545, 4, 0), (705, 5, 32), (721, 4, 0), (1089, 3, 32)],
    (10240, 8192, STORE): [(17, 3, 64), (81, 6, 32), (241, 3, 32), (257, 6, 32), (273, 3, 32), (417, 2, 0), (433, 3, 32), (513, 2, 0),
                           (529, 3, 32), (545, 2, 0), (817, 1, 0)],
    (8192, 8192, ADD): [(17, 4, 0), (81, 8, 0), (93, 4, 0), (97, 8, 0), (108, 4, 0), (113, 8, 0), (124, 4, 0), (129, 8, 0), (139, 4, 0),
                        (145, 8, 0), (230, 4, 0), (545, 2, 0), (1089, 1, 0)],
    (8192, 28672, ADD): [(17, 4, 0), (81, 8, 0), (273, 4, 0), (545, 2, 0), (1089, 1, 0)],
    (768, 256, STORE): [(17, 1, 0)],
    (256, 256, ADD): [(17, 1, 0)],
    (256, 1024, ADD): [(17, 4, 0)],
}


@pytest.mark.parametrize("N,K,epi", SLICES, ids=[f"{n}x{k}" for n, k, _ in SLICES])
def test_slices_of_the_models_are_pinned(N, K, epi):
    """Another number of slices gives other bits everywhere: the 8B, 70B and tiny decoder's, row count by row count."""
    seen = []
    for M in range(17, 1101):
        split = synera.debug_gemm_plan(M, N, K, epi)[2]
        stage = synera.debug_gemm_plan_bk(M, N, K, epi) if (K // 64) % split else 0
        if not seen or seen[-1][1:] != (split, stage):
            seen.append((M, split, stage))
    assert seen == SLICES[N, K, epi]


@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("M", [1, 17, 96, 97, 130, 200, 333, 532, 777, 1030, 2048])
@pytest.mark.parametrize("N,K,epi", [(QKV, D, STORE), (D, D, ADD), (2 * F, D, SWIGLU), (D, F, ADD), (VOCAB, D, STORE),
                                     (128, 64, STORE), (1792, 4096, ADD), (8320, 8320, STORE)])
def test_plans_are_launchable(M, N, K, epi, stored):
    bm, bn, split = synera.debug_gemm_plan(M, N, K, epi, stored)
    assert bm % 16 == 0 and bn in (128, 256) and N % bn == 0
    assert 1 <= split <= K // 32
    if epi == SWIGLU:
        assert split == 1
    assert split <= 8                           # SYNERA_MAX_GEMM_SLICES
    bk = synera.debug_gemm_plan_bk(M, N, K, epi, stored)
    assert bk in (32, 64) and K % bk == 0
    if bk == 64:                                # three stages of (2 bm + bn) rows of 128 bytes fit the 160 KB of LDS
        assert 3 * (2 * bm + bn) * 128 <= 163840
    if not stored:
        assert split == 1


def test_plan_rejects_bad_shapes():
    with pytest.raises(synera.SyneraError):
        synera.debug_gemm_plan(0, 128, 64)
    with pytest.raises(synera.SyneraError):
        synera.debug_gemm_plan(16, 192, 64)     # N % 128
    with pytest.raises(synera.SyneraError):
        synera.debug_gemm_plan(16, 384, 64, SWIGLU)   # N % 256 for SwiGLU
    with pytest.raises(synera.SyneraError):
        synera.debug_gemm_plan(16, 128, 96)     # K % 64
