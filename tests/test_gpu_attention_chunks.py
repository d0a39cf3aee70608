"""GPU tests of the decode attention where it can go wrong: at the edges of its chunks (64, 128
and 256 positions), of the switches between them (384 and 2048 positions) and of a wavefront's
rows, with scores that are far apart (a chunk or wavefront whose weights all vanish against
another's) and without leaks from positions past the new token's."""
import numpy as np
import pytest

import oracle
import synth
from common import TOL, U_ACT, rel_err, torch_dev_from_np
from gpu_model import Model
from test_gpu_decode import _attn_ref, _fill_cache

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hg = pytest.importorskip("paper_2403_01164_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hg.hetegen_create(0)
    yield c
    hg.hetegen_destroy(c)


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("P", [3, 319, 382, 383, 384, 511, 512, 2046, 2047, 2303, 2304])
def test_chunk_edges(ctx, dtype, head_dim, P):
    B, H = 2, 256
    m = Model(ctx, 1, H, 512, dtype, 0.0, 1, max_batch=2)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, P + 70, head_dim)
        kc, vc = _fill_cache(m, B, P)
        # positions past the new token's hold infinities: none may reach the result
        inf = torch_dev_from_np(np.full((B, 64, H), 0x7C00 if dtype == synth.F16 else 0x7F80, np.uint16))
        hg.hetegen_model_kv_write(ctx, m.m, 0, B, P + 1, 64, inf.data_ptr(), inf.data_ptr(),
                                  torch.cuda.current_stream().cuda_stream)
        x = synth.normal((B, H), dtype, 0, synth.act_id(P))
        out, tr = m.step_kv(x, P, trace=True)
        last, _ = m.check_teacher_forced(x, tr, attn=_attn_ref(m, kc, vc, head_dim))
        assert np.array_equal(out, last)
        assert np.array_equal(m.step_kv(x, P), out)  # the new token's own position is rewritten, not read
    finally:
        m.free()


# the last position of caches that end just before and at a larger chunk (6 chunks of 64, 3 of 128; 16 of
# 128, 8 of 256), and at 16 and 17 chunks of 256, around what the merge requests at once: the partial
# buffer holds the most chunks of any position of that cache, so earlier ones run too
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("P,earlier", [(63, []), (382, [319]), (383, [382]), (2046, [382]), (2047, [2046]), (2100, [2046]),
                                       (4095, [2046]), (4096, [2046])])
def test_full_caches(ctx, head_dim, P, earlier):
    B, H, dtype = 2, 256, synth.F16
    m = Model(ctx, 1, H, 512, dtype, 0.0, 1, max_batch=2)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, P + 1, head_dim)
        kc, vc = _fill_cache(m, B, P)
        x = synth.normal((B, H), dtype, 0, synth.act_id(P))
        for p in [P] + earlier:
            out, tr = m.step_kv(x, p, trace=True)
            last, _ = m.check_teacher_forced(x, tr, attn=_attn_ref(m, [kc[0][:, :p]], [vc[0][:, :p]], head_dim))
            assert np.array_equal(out, last), p
    finally:
        m.free()


@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("P,hot", [(60, 17), (400, 131), (2100, 0), (2100, 2099)])
def test_scores_far_apart(ctx, dtype, P, hot):
    # one cached position's key is 40 times larger than the others': its score is either far
    # above or far below all of them, per head
    B, H, D = 1, 256, 64
    m = Model(ctx, 1, H, 512, dtype, 0.0, 1, max_batch=1)
    try:
        hg.hetegen_model_kv_create(ctx, m.m, P + 1, D)
        kc, vc = _fill_cache(m, B, P)
        kf = oracle.decode(kc[0], dtype)
        kf[:, hot] *= 40.0
        kc[0] = synth.encode(kf.astype(np.float32), dtype)
        kd, vd = torch_dev_from_np(kc[0]), torch_dev_from_np(vc[0])
        hg.hetegen_model_kv_write(ctx, m.m, 0, B, 0, P, kd.data_ptr(), vd.data_ptr(),
                                  torch.cuda.current_stream().cuda_stream)
        x = synth.normal((B, H), dtype, 0, synth.act_id(1))
        _, tr = m.step_kv(x, P, trace=True)
        items = m.split_trace(tr, B)
        got, want = oracle.decode(items[1][2], dtype), _attn_ref(m, kc, vc, D)(0, items[0][3])
        assert rel_err(got, want) <= TOL + U_ACT[dtype]
    finally:
        m.free()
