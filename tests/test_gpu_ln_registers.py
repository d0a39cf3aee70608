"""GPU tests of the batch-1 GEMV that normalises its input in registers, for rows that do not
fill their last 512-element chunk: the bits of the persistent step (whose GEMV stages x in LDS
and sums in the same order), the oracle, and nothing read from past a row's end."""
import numpy as np
import pytest

import oracle
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


# 1 to 14 chunks of 512, the last one of 8 to 504 elements (7160: the widest in registers)
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("H", [8, 504, 520, 1528, 2056, 3592, 7160])
def test_partial_last_chunk(ctx, dtype, H):
    F = 2 * H if H < 4096 else 520
    m = Model(ctx, 1, H, F, dtype, 0.0, 1, max_batch=1)
    try:
        x = synth.normal((1, H), dtype, 0, synth.act_id(0))
        out, tr = m.step(x, trace=True)
        last, _ = m.check_teacher_forced(x, tr, sample=128)
        assert np.array_equal(out, last)
        hg.hetegen_model_set_exec(m.m, hg.EXEC_PERSISTENT)
        assert np.array_equal(m.step(x), out)
    finally:
        m.free()


@pytest.mark.parametrize("H", [40, 1000])
def test_infinity_stays_in_its_row(ctx, H):
    dtype = synth.F16
    ref = Model(ctx, 1, H, 64, dtype, 0.0, 1, max_batch=1)
    try:
        ref.W[0].a[5, H - 1] = 0x7C00  # an infinity in the last column of a qkv row
        m = Model(ctx, 1, H, 64, dtype, 0.0, 1, max_batch=1, weights=(ref.W, ref.b))
        try:
            x = synth.normal((1, H), dtype, 0, synth.act_id(0))
            _, tr = m.step(x, trace=True)
            q = oracle.decode(m.split_trace(tr, 1)[0][3], dtype)[0]
            assert np.isinf(q[5]) and np.isfinite(np.delete(q, 5)).all()
        finally:
            m.free()
    finally:
        ref.free()
