"""GPU tests of hetegen_model_kv_write / hetegen_model_kv_read: every value lands where the
cache layout says (a window read back from a written range, neighbours untouched), for
device buffers (one kernel) and for the others (2-D copies): off a 16-byte boundary, in host memory,
overlapping."""
import ctypes

import numpy as np
import pytest

import synth
from gpu_model import Model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hg = pytest.importorskip("paper_2403_01164_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hg.hetegen_create(0)
    yield c
    hg.hetegen_destroy(c)


def _buf(shape, offset):
    """Uninitialised device tensor whose data starts `offset` elements past a 16-byte boundary."""
    n = int(np.prod(shape))
    return torch.empty(n + offset, dtype=torch.int16, device="cuda")[offset:].view(shape)


@pytest.mark.parametrize("H,D", [(192, 64), (640, 128), (4224, 128), (2112, 64)])  # 3, 5, 33 and 33 heads
@pytest.mark.parametrize("B,pos0,n", [(1, 0, 1), (3, 5, 7), (2, 1, 64), (3, 17, 4)])
@pytest.mark.parametrize("woff,roff", [(0, 0), (1, 0), (0, 3)])
def test_kv_write_read_round_trip(ctx, H, D, B, pos0, n, woff, roff):
    max_seq, s = 70, torch.cuda.current_stream().cuda_stream
    m = Model(ctx, 2, H, 64, synth.F16, 0.0, 0, max_batch=3)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, max_seq, D)
        g = torch.Generator(device="cuda").manual_seed(1)
        want = torch.zeros((2, 3, max_seq, H), dtype=torch.int16, device="cuda")  # the cache starts as zeros
        k, v = _buf((B, n, H), woff), _buf((B, n, H), woff)
        for i, t in enumerate((k, v)):
            t.copy_(torch.randint(-30000, 30000, (B, n, H), generator=g, device="cuda", dtype=torch.int16))
            want[i, :B, pos0:pos0 + n] = t
        hg.hetegen_model_kv_write(ctx, m.m, 1, B, pos0, n, k.data_ptr(), v.data_ptr(), s)
        for layer in (0, 1):
            for q0, q in ((0, max_seq), (pos0, n), (max(pos0 - 1, 0), 3)):
                kr, vr = _buf((3, q, H), roff), _buf((3, q, H), roff)
                kr.fill_(-1), vr.fill_(-1)
                hg.hetegen_model_kv_read(ctx, m.m, layer, 3, q0, q, kr.data_ptr(), vr.data_ptr(), s)
                torch.cuda.synchronize()
                for i, t in enumerate((kr, vr)):
                    assert torch.equal(t, want[i, :, q0:q0 + q] if layer else torch.zeros_like(t)), (layer, q0, q)
    finally:
        m.free()


def test_kv_pinned_buffers(ctx):
    # pinned memory goes through the 2-D copies, in and out, on either side of a device buffer
    H, D, B, n, pos0, max_seq = 640, 128, 2, 5, 3, 16
    s = torch.cuda.current_stream().cuda_stream
    m = Model(ctx, 1, H, 64, synth.F16, 0.0, 0, max_batch=B)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, max_seq, D)
        g = torch.Generator().manual_seed(2)
        k, v = (torch.randint(-30000, 30000, (B, n, H), generator=g, dtype=torch.int16, pin_memory=True)
                for _ in range(2))
        vd = v.cuda()
        hg.hetegen_model_kv_write(ctx, m.m, 0, B, pos0, n, k.data_ptr(), vd.data_ptr(), s)
        torch.cuda.synchronize()
        kr = torch.full((B, max_seq, H), -1, dtype=torch.int16, pin_memory=True)
        vr = torch.full((B, max_seq, H), -1, dtype=torch.int16, device="cuda")
        hg.hetegen_model_kv_read(ctx, m.m, 0, B, 0, max_seq, kr.data_ptr(), vr.data_ptr(), s)
        torch.cuda.synchronize()
        for got, want in ((kr, k), (vr.cpu(), v)):
            assert torch.equal(got[:, pos0:pos0 + n], want)
            got[:, pos0:pos0 + n] = 0
            assert not got.any()
    finally:
        m.free()


def test_kv_pageable_buffers_are_refused(ctx):
    H, D = 640, 128
    s = torch.cuda.current_stream().cuda_stream
    m = Model(ctx, 1, H, 64, synth.F16, 0.0, 0, max_batch=1)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, 4, D)
        host, dev = torch.zeros(1, 4, H, dtype=torch.int16), torch.zeros(1, 4, H, dtype=torch.int16, device="cuda")
        for copy in (hg.hetegen_model_kv_write, hg.hetegen_model_kv_read):
            with pytest.raises(hg.HetegenError) as e:
                copy(ctx, m.m, 0, 1, 0, 4, host.data_ptr(), dev.data_ptr(), s)
            assert e.value.status == hg.ERR_HIP
        torch.cuda.synchronize()
    finally:
        m.free()


@pytest.mark.parametrize("n", [1, 7, 64])
def test_kv_buffers_that_end_with_their_allocation(ctx, n):
    # allocations of exactly the bytes moved (not from torch's pools), and of 16 bytes more
    H, D, B = 2176, 64, 2
    s = torch.cuda.current_stream().cuda_stream
    hip = ctypes.CDLL(hg.LIB_PATH)  # its HIP runtime's symbols
    m = Model(ctx, 1, H, 64, synth.F16, 0.0, 0, max_batch=B)
    nbytes = B * n * H * 2
    ptrs = []
    try:
        hg.hetegen_model_kv_create(ctx, m.m, 64, D)
        for extra in (0, 0, 0, 16):
            p = ctypes.c_void_p()
            assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(nbytes + extra)) == 0
            ptrs.append(p)
        ki, vi, ko, vo = (p.value for p in ptrs)
        vo += 16
        g = torch.Generator(device="cuda").manual_seed(4)
        k, v = (torch.randint(-30000, 30000, (B, n, H), generator=g, device="cuda", dtype=torch.int16) for _ in range(2))
        torch.cuda.synchronize()
        for d, t in ((ki, k), (vi, v)):
            assert hip.hipMemcpy(ctypes.c_void_p(d), ctypes.c_void_p(t.data_ptr()), ctypes.c_size_t(nbytes), 3) == 0
        hg.hetegen_model_kv_write(ctx, m.m, 0, B, 64 - n, n, ki, vi, s)
        hg.hetegen_model_kv_read(ctx, m.m, 0, B, 64 - n, n, ko, vo, s)
        torch.cuda.synchronize()
        for d, t in ((ko, k), (vo, v)):
            out = torch.empty_like(t)
            assert hip.hipMemcpy(ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(d), ctypes.c_size_t(nbytes), 3) == 0
            torch.cuda.synchronize()
            assert torch.equal(out, t)
    finally:
        for p in ptrs:
            hip.hipFree(p)
        m.free()


@pytest.mark.parametrize("shift", [0, 8, 640])
def test_kv_read_into_overlapping_buffers(ctx, shift):
    # a read writes the keys, then the values: where the buffers overlap the values stay
    H, D, B, n = 640, 64, 2, 6
    s = torch.cuda.current_stream().cuda_stream
    m = Model(ctx, 1, H, 64, synth.F16, 0.0, 0, max_batch=B)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, n, D)
        g = torch.Generator(device="cuda").manual_seed(3)
        k, v = (torch.randint(-30000, 30000, (B, n, H), generator=g, device="cuda", dtype=torch.int16) for _ in range(2))
        hg.hetegen_model_kv_write(ctx, m.m, 0, B, 0, n, k.data_ptr(), v.data_ptr(), s)
        buf = torch.full((B * n * H + shift,), -1, dtype=torch.int16, device="cuda")
        hg.hetegen_model_kv_read(ctx, m.m, 0, B, 0, n, buf.data_ptr(), buf[shift:].data_ptr(), s)
        torch.cuda.synchronize()
        want = torch.cat([k.flatten(), torch.full((shift,), -1, dtype=torch.int16, device="cuda")])
        want[shift:] = v.flatten()
        assert torch.equal(buf, want)
    finally:
        m.free()
