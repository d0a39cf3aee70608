"""GPU tests of the matrix-core GEMV's row-tile groups: grids where a workgroup holds 2, 3 or
5 row tiles (chosen from the row count on a 256-CU device), with remainders in the rows, the
16-row tiles, the group and the k-tiles, with and without the split over K and the
LayerNorm prologue."""
import numpy as np
import pytest

import oracle
import synth
from common import np_from_dev, torch_dev_from_np
from gpu_model import Model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hg = pytest.importorskip("paper_2403_01164_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hg.hetegen_create(0)
    yield c
    hg.hetegen_destroy(c)


# row tiles per workgroup on 256 CUs: 2 for the first three and 6991 rows, 3 for 11985 (750 tiles) of
# 296, 9190 (575) and 10007 (626) unsplit and 2550 in 8 splits, 5 for 9190 in 2 splits, 1 for 11985 and
# 12288 (768) rows of 1056; K: odd numbers of k-tiles, partial chunks of 4, K % 32 != 0
@pytest.mark.parametrize("N,K", [(5999, 40), (5999, 552), (8192, 72), (11985, 296), (11985, 1056), (10007, 2088),
                                 (9190, 4136), (2550, 10248), (9190, 1064), (6991, 1096), (12288, 1056)])
@pytest.mark.parametrize("B", [1, 5, 8])
def test_row_groups_integer_inputs_bit_exact(ctx, N, K, B):
    # x, W in {-1, 0, 1}, bias in {-4..4}: every partial sum is exact, so any order of the
    # sums gives the oracle's bits
    dtype = synth.F16
    W = synth.integers((N, K), dtype, 0, 21, -1, 1)
    b = synth.integers((N,), dtype, 0, 22, -4, 4)
    x = synth.integers((B, K), dtype, 0, 23, -1, 1)
    Wd, xd, bd = torch_dev_from_np(W), torch_dev_from_np(x), torch_dev_from_np(b)
    Wt = torch.empty((hg.hetegen_tiled_bytes(N, K) // 2,), dtype=torch.int16, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    hg.hetegen_tile_weights(ctx, Wd.data_ptr(), N, K, Wt.data_ptr(), s)
    y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    hg.hetegen_linear_tiled(ctx, xd.data_ptr(), B, K, Wt.data_ptr(), N, dtype, bd.data_ptr(), y.data_ptr(), hg.F32, s)
    torch.cuda.synchronize()
    ref = oracle.linear(x, W, b, dtype)
    assert np.array_equal(np_from_dev(y, np.float32).view(np.uint32), ref.view(np.uint32))


# qkv [3H, H] and fc1 [F, H] with the LayerNorm prologue: (2000, 11984) 2 and 3 row tiles per
# workgroup, (4136, 9192) fc1 split in 2 with 5, (2056, 520) K = 2056 with a last group of 8
@pytest.mark.parametrize("H,F", [(2000, 11984), (4136, 9192), (2056, 520)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_row_groups_layernorm_prologue(ctx, dtype, H, F):
    m = Model(ctx, 2 if H < 4096 else 1, H, F, dtype, 0.0, 1, max_batch=8)
    try:
        x = synth.normal((8, H), dtype, 0, synth.act_id(0))
        out, tr = m.step(x, trace=True)
        last, _ = m.check_teacher_forced(x, tr, sample=256)
        assert np.array_equal(out, last)
        for B in (2, 3, 7):  # a batch row's bits do not depend on the batch size
            assert np.array_equal(m.step(np.ascontiguousarray(x[:B])), out[:B]), B
    finally:
        m.free()
