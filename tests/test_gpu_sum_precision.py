"""GPU tests of how the matrix-core GEMVs sum over K: short rows bit for bit as the tree of their
k-tiles' products that the kernel documents, longer ones by their error against 64-bit sums."""
import numpy as np
import pytest

import bench
import oracle
import synth
from common import np_from_dev, torch_dev_from_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hg = pytest.importorskip("paper_2403_01164_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hg.hetegen_create(0)
    yield c
    hg.hetegen_destroy(c)


def _tiled(ctx, x, W, dtype):
    (B, K), N = x.shape, W.shape[0]
    s = torch.cuda.current_stream().cuda_stream
    xd, Wd = torch_dev_from_np(x), torch_dev_from_np(W)
    Wt = torch.empty((hg.hetegen_tiled_bytes(N, K) // 2,), dtype=torch.int16, device="cuda")
    hg.hetegen_tile_weights(ctx, Wd.data_ptr(), N, K, Wt.data_ptr(), s)
    y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    hg.hetegen_linear_tiled(ctx, xd.data_ptr(), B, K, Wt.data_ptr(), N, dtype, 0, y.data_ptr(), hg.F32, s)
    torch.cuda.synchronize()
    return np_from_dev(y, np.float32)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("K", [40, 72, 128, 136, 256])
def test_short_rows_add_their_tiles_pairwise(ctx, dtype, K):
    # up to 8 k-tiles no product continues another's sum: the tiles' sums (one-tile calls) are
    # added two by two.  The order is the kernel's own, so the bits are the same.
    N, B = 300, 8
    W, x = synth.normal((N, K), dtype, 0, 81, 0, 0.02), synth.normal((B, K), dtype, 0, 82)
    t = [_tiled(ctx, np.ascontiguousarray(x[:, k:k + 32]), np.ascontiguousarray(W[:, k:k + 32]), dtype)
         for k in range(0, K, 32)]
    t += [np.zeros((B, N), np.float32)] * (8 - len(t))
    want = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]))
    assert np.array_equal(_tiled(ctx, x, W, dtype), want)


@pytest.mark.parametrize("K", [4104, 8160])
def test_rows_of_an_uneven_grid_keep_their_four_splits(ctx, K):
    # 400 row tiles load 256 compute units 1.28x unevenly and take 4 splits, as the same rows do in
    # a linear of 63 row tiles: the same partial sums, added in the same order.  (Unsplit, their
    # error against 64 bits is 1.3-1.4 times as large.)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the shapes are chosen for a 256-CU device")
    assert bench.mfma_splits(6400, K, 256) == bench.mfma_splits(1000, K, 256) == 4
    W, x = synth.normal((6400, K), synth.F16, 0, 83, 0, 0.02), synth.normal((8, K), synth.F16, 0, 84)
    assert np.array_equal(_tiled(ctx, x, W, synth.F16)[:, :1000],
                          _tiled(ctx, x, np.ascontiguousarray(W[:1000]), synth.F16))


def _rows(ctx, x, W, dtype):
    (B, K), N = x.shape, W.shape[0]
    xd, Wd = torch_dev_from_np(x), torch_dev_from_np(W)
    y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    hg.hetegen_linear(ctx, xd.data_ptr(), B, K, Wd.data_ptr(), Wd.data_ptr(), N, dtype, 0, 0, 0.0, y.data_ptr(), hg.F32,
                      torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return np_from_dev(y, np.float32)


# 16 rows per workgroup but for the shapes of up to 2000 rows (8, where that is no less precise: not
# bfloat16 at 1032); K: one step of 256 or 512 columns and a little more, the middle of a step, several steps
@pytest.mark.parametrize("dtype,N,K", [(synth.BF16, 4096, 264), (synth.BF16, 4096, 520), (synth.BF16, 4096, 784),
                                       (synth.BF16, 1000, 1032), (synth.BF16, 2000, 1032), (synth.BF16, 2000, 1160),
                                       (synth.BF16, 2000, 2056), (synth.BF16, 4096, 1544), (synth.BF16, 4096, 2056),
                                       (synth.BF16, 4096, 4096), (synth.F16, 4096, 520), (synth.F16, 1000, 1032)])
def test_row_major_rows_are_as_precise_at_batch_8_as_alone(ctx, dtype, N, K):
    # batch 8 sums on the matrix cores (where that is no less precise), a single batch row of as few
    # rows on the vector GEMV.  The two errors are taken over 8 N = 8000 .. 32768 outputs; 1.02 leaves
    # room for the sampling error of their ratio (below 0.8 %), 1.02-1.09 being what chained products
    # gave bfloat16 at these lengths.
    W, x = synth.normal((N, K), dtype, 0, 85, 0, 0.02), synth.normal((8, K), dtype, 0, 86)
    ref = oracle.decode(x, dtype).astype(np.float64) @ oracle.decode(W, dtype).astype(np.float64).T
    together = _rows(ctx, x, W, dtype)
    alone = np.concatenate([_rows(ctx, np.ascontiguousarray(x[b:b + 1]), W, dtype) for b in range(8)])
    e = [np.sqrt(np.mean((y.astype(np.float64) - ref) ** 2)) for y in (together, alone)]
    assert e[0] <= 1.02 * e[1], e[0] / e[1]
