"""GPU tests of hetegen_model_kv_write / hetegen_model_kv_read: every value lands where the
cache layout says (a window read back from a written range, neighbours untouched), for
device buffers (one kernel) and for buffers off a 16-byte boundary (2-D copies)."""
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
