"""Kernel forms at their edges: the rows form of the small-M codes; the 128 x
128 group-scale tile (1 to 7 steps on its 3-deep
stage ring, ragged row and column tails) against the oracle, and the sizes at
which the planner turns from one group tile to the other."""
import numpy as np
import pytest

import paper_2608_12932_amd as w
from paper_2608_12932_amd import inputs as I
from helpers import check_all_outputs


@pytest.mark.gpu
@pytest.mark.parametrize("M,N", [(2000, 6160), (1793, 6128)])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7])
def test_group_tile_edges(steps, M, N):
    K = 128 * steps
    assert "largem<128x128,group>" in w.w4a8_linear_describe(M, N, K, w.SCALE_GROUP_F16)
    x = I.activations(M, K, 840 + M + steps)
    W, s = I.weights(N, K, 850 + N + steps, group=True)
    rows = np.unique(np.concatenate([np.arange(0, M, 61), np.arange(M - 40, M)]))  # with the ragged last row tile
    check_all_outputs(x, W, s, group=True, rows=rows, label="group tile")


# With at most one 128 x 128 tile per CU and a long K, the form that reads its
# operands a step ahead: every remainder of its 4-deep ring.
@pytest.mark.gpu
@pytest.mark.parametrize("rest", [0, 1, 2, 3])
def test_lone_group_tiles(rest):
    from test_gpu_swiglu import check as check_gated
    M, N, K = 1793, 2000, 8192 + 128 * rest
    assert "largem<128x128,group,ahead>" in w.w4a8_linear_describe(M, N, K, w.SCALE_GROUP_F16)
    x = I.activations(M, K, 880 + rest)
    W, s = I.weights(N, K, 884 + rest, group=True)
    rows = np.concatenate([np.arange(0, M, 120), np.arange(M - 10, M)])
    check_all_outputs(x, W, s, group=True, rows=rows, label="lone group tile")
    M, F, K = 201, 176, 2048 + 128 * rest
    assert "largem<128x128,group,swiglu,ahead>" in w.w4a8_linear_swiglu_describe(M, 2 * F, K, w.SCALE_GROUP_F16)
    check_gated(M, F, K, True, rest % 2 == 1, 888 + rest, "lone group tile")


@pytest.mark.parametrize("M,N,K,form", [(1024, 4096, 8192, "group,ahead"), (1024, 4096, 8064, "group"), (1400, 4096, 8192, "group")])
def test_lone_group_tile_choice(M, N, K, form):
    assert f"largem<128x128,{form}>" in w.w4a8_linear_describe(M, N, K, w.SCALE_GROUP_F16)


@pytest.mark.parametrize("M,F,K,form", [(1024, 2048, 2048, ",ahead"), (1024, 2048, 1920, ""), (1025, 2048, 2048, "")])
def test_lone_gated_tile_choice(M, F, K, form):
    assert f"largem<128x128,group,swiglu{form}>" in w.w4a8_linear_swiglu_describe(M, 2 * F, K, w.SCALE_GROUP_F16)


@pytest.mark.parametrize("M,N,tile", [(768, 6144, 64), (1024, 6144, 128), (320, 24576, 64), (384, 24576, 128),
                                      (768, 4096, 64), (1024, 4096, 128), (256, 24576, 128), (192, 24576, 64)])
def test_group_tile_choice(M, N, tile):
    assert f"largem<{tile}x{tile},group" in w.w4a8_linear_describe(M, N, 4096, w.SCALE_GROUP_F16)


# The small-M kernels load the codes as whole rows from 12 rows on, for some
# tiles only where the rows and blocks are worth it (both forms occur here):
# the turn, the edges of the 8-row halves and 16-row tiles, one and several
# column tiles, K splits that leave waves without a block.
@pytest.mark.gpu
@pytest.mark.parametrize("group", [False, True])
@pytest.mark.parametrize("M", [11, 12, 15, 16, 17, 25, 33, 40, 48, 57, 64])
def test_rows_of_codes(M, group):
    for K, N in ((128, 48), (1152, 4096), (2048, 8192), (6272, 2064)):
        x = I.activations(M, K, 860 + M)
        W, s = I.weights(N, K, 861 + N, group=group)
        check_all_outputs(x, W, s, group=group, label="rows of codes")


# The norm's codes come from a corrected reciprocal product, near halves from
# IEEE division: enough values (3 M) that ~700 quotients lie within 2^-12 of a
# half, and gains small and large enough for the scales that always divide.
@pytest.mark.gpu
@pytest.mark.parametrize("gain", [1.0, 2.0 ** -70, 2.0 ** 70])
def test_norm_codes_near_halves(gain):
    import oracle
    import torch
    from helpers import bf16_dev
    M, K = (256, 12288) if gain == 1.0 else (8, 1152)
    x = I.activations(M, K, 870)
    g = I.to_bf16_bits((gain * (1 + 0.1 * np.random.Generator(np.random.PCG64(871)).standard_normal(K))).astype(np.float32))
    q, s = w.w4a8_rmsnorm_quantize_act(bf16_dev(x), bf16_dev(g), 1e-6)
    rq, rs = oracle.rmsnorm_quantize(x, g, 1e-6)[:2]
    np.testing.assert_array_equal(s.cpu().numpy().view(np.uint32), np.asarray(rs, np.float32).view(np.uint32))
    np.testing.assert_array_equal(q.cpu().numpy(), rq)
