"""GPU tests of hetegen_linear on resident row-major weights through the matrix cores: 8 and
16 rows per workgroup, remainders in the rows, the steps of 256 / 512 columns and the k-tile
pairs, values that must not leak from past a row's end, independence of the batch and of alpha,
and the shapes that stay on the vector GEMV."""
import numpy as np
import pytest

import oracle
import synth
from common import TOL, np_from_dev, rel_err, torch_dev_from_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hg = pytest.importorskip("paper_2403_01164_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hg.hetegen_create(0)
    yield c
    hg.hetegen_destroy(c)


def _run(ctx, x, W, b, dtype):
    (B, K), N = x.shape, W.shape[0]
    Wd, xd = torch_dev_from_np(W), torch_dev_from_np(x)
    bd = torch_dev_from_np(b) if b is not None else None
    y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    hg.hetegen_linear(ctx, xd.data_ptr(), B, K, W.ctypes.data, Wd.data_ptr(), N, dtype,
                      b.ctypes.data if b is not None else 0, bd.data_ptr() if b is not None else 0, 0.0, y.data_ptr(),
                      hg.F32, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return np_from_dev(y, np.float32)


def _aligned(a):
    """Copy of a on a 16-byte boundary (the entry point refuses other host weights)."""
    buf = np.empty(a.nbytes + 16, np.uint8)
    o = -buf.ctypes.data % 16
    out = buf[o:o + a.nbytes].view(a.dtype).reshape(a.shape)
    out[...] = a
    return out


# on 256 CUs: 8 rows per workgroup for up to 2048 rows of K >= 1024 (1, 9, 37, 1001); 16 for the
# others (K < 1024, rows shorter than 3584 on an uneven grid, grids of one workgroup per CU).  Batches
# 1 and, up to 1024 rows, 2 run on the vector GEMV and are here as its counterpart
SHAPES = [(1, 1024), (9, 1032), (37, 3080), (1001, 1544), (5001, 1096), (4096, 8200), (37, 8), (33, 264), (2569, 520),
          (4095, 2056), (17, 1016)]


@pytest.mark.parametrize("N,K", SHAPES)
@pytest.mark.parametrize("B", [1, 2, 5, 8])
def test_rows_integer_inputs_bit_exact(ctx, N, K, B):
    dtype = synth.F16
    W = _aligned(synth.integers((N, K), dtype, 0, 21, -1, 1))
    b = synth.integers((N,), dtype, 0, 22, -4, 4)
    x = synth.integers((B, K), dtype, 0, 23, -1, 1)
    ref = oracle.linear(x, W, b, dtype)
    assert np.array_equal(_run(ctx, x, W, b, dtype).view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("N,K", [(37, 3080), (4095, 2056), (2569, 520)])
def test_rows_parity_and_batch_independence(ctx, dtype, N, K):
    W = _aligned(synth.normal((N, K), dtype, 0, 31, 0, 0.02))
    x = synth.normal((8, K), dtype, 0, 33)
    y8 = _run(ctx, x, W, None, dtype)
    assert rel_err(y8, oracle.linear(x, W, None, dtype)) <= TOL
    for B in (2, 3, 7) if N > 1024 else (3, 7):  # below that batch 2 is on the vector GEMV
        y = _run(ctx, np.ascontiguousarray(x[8 - B:]), W, None, dtype)
        assert np.array_equal(y.view(np.uint32), y8[8 - B:].view(np.uint32)), B


@pytest.mark.parametrize("N,K", [(24, 1096), (40, 520)])
def test_rows_infinity_stays_in_its_row(ctx, N, K):
    # the last columns of a row are reread where a step runs past K: an infinity there must
    # reach its own row's result only, and a zero x times it must give the NaN it is
    dtype = synth.F16
    W = synth.integers((N, K), dtype, 0, 41, -1, 1)
    W[5, K - 1] = 0x7C00
    W = _aligned(W)
    x = synth.encode(np.ones((3, K), np.float32), dtype)
    x[1, K - 1] = 0
    y = _run(ctx, x, W, None, dtype)
    assert np.isposinf(y[0, 5]) and np.isnan(y[1, 5]) and np.isposinf(y[2, 5])
    assert np.isfinite(np.delete(y, 5, axis=1)).all()


# Batch 1 from 16385 rows on (below it a single batch row is on the vector GEMV, as are 1 and 2
# above for up to 1024 rows): 16 rows per workgroup, the same with several steps per wavefront, and 8
# (1063 groups of 16, 1.2x uneven on 256 CUs)
MANY = [(16385, 264), (20481, 2120), (17001, 3592)]


# (and 8 rows per workgroup on a stride of 16 KiB, from batch 2)
@pytest.mark.parametrize("N,K", MANY + [(4081, 8192)])
@pytest.mark.parametrize("B", [1, 2, 8])
def test_many_rows_integer_inputs_bit_exact(ctx, N, K, B):
    dtype = synth.F16
    W = _aligned(synth.integers((N, K), dtype, 0, 51, -1, 1))
    b = synth.integers((N,), dtype, 0, 52, -4, 4)
    x = synth.integers((B, K), dtype, 0, 53, -1, 1)
    ref = oracle.linear(x, W, b, dtype)
    assert np.array_equal(_run(ctx, x, W, b, dtype).view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("N,K", MANY)
def test_many_rows_parity_and_batch_1_on_the_matrix_cores(ctx, dtype, N, K):
    W = _aligned(synth.normal((N, K), dtype, 0, 54, 0, 0.02))
    x = synth.normal((8, K), dtype, 0, 55)
    y8 = _run(ctx, x, W, None, dtype)
    assert rel_err(y8, oracle.linear(x, W, None, dtype)) <= TOL
    y1 = _run(ctx, np.ascontiguousarray(x[3:4]), W, None, dtype)
    assert np.array_equal(y1.view(np.uint32), y8[3:4].view(np.uint32))
    # few rows run on the vector GEMV, which adds in another order
    vec = _run(ctx, np.ascontiguousarray(x[3:4]), _aligned(W[:1000]), None, dtype)
    assert not np.array_equal(y1[:, :1000], vec)


# (N, K, B) where the matrix cores are slower: a row gets the vector GEMV's bits, those of few rows
# at batch 1.  Stride of 4 KiB at batch 1 and 3, a skewed stride, long rows of an uneven grid, x
# beyond the LDS on an uneven grid
@pytest.mark.parametrize("N,K,B", [(16400, 2048, 1), (12288, 2048, 3), (4096, 8160, 4), (4200, 8064, 4), (4200, 10248, 3),
                                   (4200, 10248, 8), (600, 6152, 4), (1000, 2048, 2)])
def test_rows_left_to_the_vector_gemv(ctx, N, K, B):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the shapes are chosen for a 256-CU device")
    dtype = synth.BF16
    W = _aligned(synth.normal((N, K), dtype, 0, 56, 0, 0.02))
    x = synth.normal((B, K), dtype, 0, 57)
    y = _run(ctx, x, W, None, dtype)
    few = _aligned(W[:500])
    for b in range(B):
        vec = _run(ctx, np.ascontiguousarray(x[b:b + 1]), few, None, dtype)
        assert np.array_equal(y[b:b + 1, :500].view(np.uint32), vec.view(np.uint32)), b


@pytest.mark.parametrize("N,K,B", [(20480, 264, 1), (2048, 1032, 3), (10000, 3592, 8)])
def test_gpu_rows_keep_their_bits_when_alpha_changes(ctx, N, K, B):
    dtype = synth.F16
    W = _aligned(synth.normal((N, K), dtype, 0, 58, 0, 0.02))
    x = synth.normal((B, K), dtype, 0, 59)
    full = _run(ctx, x, W, None, dtype)
    Wd, xd = torch_dev_from_np(W), torch_dev_from_np(x)
    for alpha in (0.3, 0.9):
        y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
        hg.hetegen_linear(ctx, xd.data_ptr(), B, K, W.ctypes.data, Wd.data_ptr(), N, dtype, 0, 0, alpha, y.data_ptr(),
                          hg.F32, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        n_gpu = int(N * (1 - alpha)) - 1  # rows that are on the GPU however the split rounds
        got = np_from_dev(y, np.float32)
        assert np.array_equal(got[:, :n_gpu].view(np.uint32), full[:, :n_gpu].view(np.uint32)), alpha
        assert rel_err(got, full) <= TOL
