"""Partial evaluation at the sizes where its helpers change over, against the oracle: the table of a point in one
launch up to 16 coordinates and in several from 17 on, and few or many chunks of a long axis summed at the end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,lo,hi", [
    ((1, 64), 0, 1), ((2, 64), 0, 1), ((64, 1), 0, 1), ((8192, 64), 0, 1), ((16384, 32), 0, 1), ((16384, 1), 0, 1),
    ((512, 128), 0, 1), ((4096, 4), 0, 1), ((4, 4096), 1, 2), ((4, 256, 8), 1, 2), ((2, 4096, 64), 1, 2), ((64, 4, 128, 2), 0, 3),
])
@pytest.mark.parametrize("kind", ["i32", "i64", "fr"])
def test_partial_eval_sizes(lib, ctx, shape, lo, hi, kind):
    import torch
    from oracle.field import R_MOD, fr_array, fr_array_from_le, array_to_le
    from oracle.mle import partial_eval
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(sum(shape))
    n = int(np.prod(shape))
    if kind == "fr":
        raw = uniform_fr_limbs(rng, n).tobytes()
        ref = fr_array_from_le(raw, n)
        t = lib.fr_tensor_upload(ctx, raw, shape)
    else:
        src = rng.integers(-2 ** 31, 2 ** 31, n, dtype=np.int64) if kind == "i32" else rng.integers(-2 ** 47, 2 ** 47, n, dtype=np.int64)
        src[0] = -2 ** 31 if kind == "i32" else -2 ** 47
        ref = fr_array(src)
        t = lib.tensor_wrap_int(ctx, torch.from_numpy(src.astype(np.int32) if kind == "i32" else src).cuda(), shape)
    m = sum(int(s).bit_length() - 1 for s in shape[lo:hi])
    point = [int(x) for x in fr_array_from_le(uniform_fr_limbs(rng, max(m, 1)).tobytes(), max(m, 1))][:m]
    if m > 1:
        point[-1] = R_MOD - 1
    out = lib.mle_partial_eval(ctx, t, lo, hi, point)
    expect, oshape = partial_eval(ref, shape, lo, hi, point)
    assert list(out.shape) == oshape
    assert out.download() == array_to_le(expect)


# 64-bit integers at the ends of their range: their three limbs and the column sums are as large as they get
@pytest.mark.parametrize("shape,axis", [((64, 256), 1), ((2, 4096), 1), ((256, 64), 0), ((2, 64, 4), 1)])
@pytest.mark.parametrize("value", [-2 ** 63, 2 ** 63 - 1, -2 ** 58, 2 ** 29 - 1])
def test_partial_eval_int64_range(lib, ctx, shape, axis, value):
    import torch
    from oracle.field import R_MOD, fr_array, array_to_le
    from oracle.mle import partial_eval
    src = np.full(shape, value, dtype=np.int64)
    src.reshape(-1)[::7] = -1 - value
    t = lib.tensor_wrap_int(ctx, torch.from_numpy(src).cuda(), shape)
    for u in (R_MOD - 1, 2, R_MOD // 2):
        point = [u] * (shape[axis].bit_length() - 1)
        expect, _ = partial_eval(fr_array(src.reshape(-1)), shape, axis, axis + 1, point)
        assert lib.mle_partial_eval(ctx, t, axis, axis + 1, point).download() == array_to_le(expect)


# on either side of the line between a wave along a row and a lane per row, the ends of the range among the values
@pytest.mark.parametrize("shape", [(8, 1 << 16), (32, 1 << 13), (32, 1 << 14), (1024, 256), (1024, 512), (8192, 64)])
@pytest.mark.parametrize("value", [-2 ** 63, 2 ** 29 - 1])
def test_partial_eval_int64_rows(lib, ctx, shape, value):
    import torch
    from oracle.field import R_MOD, fr_array, array_to_le
    from oracle.mle import partial_eval
    src = np.full(shape, value, dtype=np.int64)
    src.reshape(-1)[::7] = -1 - value
    t = lib.tensor_wrap_int(ctx, torch.from_numpy(src).cuda(), shape)
    point = [R_MOD - 1 - 3 * k for k in range(shape[1].bit_length() - 1)]
    expect, _ = partial_eval(fr_array(src.reshape(-1)), shape, 1, 2, point)
    assert lib.mle_partial_eval(ctx, t, 1, 2, point).download() == array_to_le(expect)


# partial sums of 16, 32 | 64, 256 | 512 and 2048 chunks: at the lines between the three widths of the kernel that adds them, with
# fewer outputs than a block takes, as many, and several blocks of them
@pytest.mark.parametrize("shape", [(64, 256), (128, 16), (128, 64), (128, 256), (256, 2), (256, 16), (256, 64), (1024, 1), (1024, 32), (2048, 2),
                                   (2048, 4), (2048, 16), (8192, 1)])
@pytest.mark.parametrize("kind", ["i32", "fr"])
def test_partial_eval_chunk_sums(lib, ctx, shape, kind):
    test_partial_eval_sizes(lib, ctx, shape, 0, 1, kind)


# the longest points whose table is one launch, and the first that takes several
@pytest.mark.parametrize("coords", [15, 16, 17])
def test_partial_eval_long_points(lib, ctx, coords):
    test_partial_eval_sizes(lib, ctx, (1 << coords, 2), 0, 1, "i32")


# a point too long for the launch's arguments is copied from the caller's memory, which is the caller's again after the call
@pytest.mark.parametrize("coords", [16, 17, 19])
def test_partial_eval_point_memory_is_free_after_the_call(lib, ctx, coords):
    import ctypes as C
    import torch
    from oracle.field import R_MOD, array_to_le, fr_array
    from oracle.mle import beta_eval
    src = np.zeros((1 << coords, 2), dtype=np.int32)
    rows = (0, 1, (1 << coords) - 1, 12345)
    for i, row in enumerate(rows):
        src[row] = (i + 3, -7 * i - 1)
    t = lib.tensor_wrap_int(ctx, torch.from_numpy(src).cuda(), src.shape)
    point = [(R_MOD // 3 + 17 * k) % R_MOD for k in range(coords)]
    expect = [sum(int(src[row][i]) * beta_eval(point, row) for row in rows) % R_MOD for i in range(2)]
    raw = b"".join(p.to_bytes(32, "little") for p in point)
    for _ in range(3):
        buf, out = C.create_string_buffer(raw, len(raw)), C.c_void_p()
        assert lib.load_library().mle_partial_eval(ctx.handle, t.handle, 0, 1, buf, coords, C.byref(out)) == 0
        C.memset(buf, 0xff, len(raw))
        assert lib.FrTensor(ctx, out).download() == array_to_le(fr_array(expect))
