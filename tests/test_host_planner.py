"""CPU-side checks of the host logic that shapes the projection launches (no GPU needed): the plan must
cover every row and the whole contraction for any shape, keep the kernel's structural assumptions, and pick
the measured-best shapes at the two benchmark models."""
import itertools
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2509_23094_amd", "libd2c.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libd2c.so not built (run __graft_entry__.build())")


def _plan(*a, **k):
    from paper_2509_23094_amd import binding as B
    return B.d2c_plan_projection(*a, **k)


ROWS = [1, 15, 16, 17, 46, 64, 69, 96, 127, 128, 129, 150, 160, 161, 185, 192, 193, 200, 256, 257, 300, 512, 640,
        856, 1024, 3072, 12288]
SHAPES = [(12288, 4096), (4096, 4096), (24576, 4096), (4096, 12288), (126464, 4096),          # LLaDA-8B
          (4608, 3584), (3584, 3584), (37888, 3584), (3584, 18944), (152064, 3584),           # Dream-7B
          (768, 256), (1376, 256), (256, 688), (40, 20), (100, 132), (200, 264), (3000, 520), (33000, 256), (144, 64)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_plan_covers_rows_and_contraction_and_keeps_the_kernel_assumptions(dtype):
    elem_per_chunk = 128 if dtype == "bf16" else 64
    for (N, K), m, single in itertools.product(SHAPES, ROWS, (False, True)):
        if K % (8 if dtype == "bf16" else 4):
            continue                                   # the launcher refuses rows that are not whole 16-byte pieces
        p = _plan(dtype, m, N, K, single)
        where = f"{dtype} m={m} N={N} K={K} single={single}: {p}"
        assert p["row_tiles"] * 16 * p["row_chunks"] >= m, where
        assert (p["row_tiles"] * 16) * (p["row_chunks"] - 1) < m, where              # no empty row chunk
        assert p["k_per_split"] * p["splits"] >= K and p["k_per_split"] * (p["splits"] - 1) < K, where
        assert p["k_per_split"] % elem_per_chunk == 0, where                        # splits start on chunk boundaries
        assert 1 <= p["splits"] <= 8 and (not single or p["splits"] == 1), where
        assert p["waves"] in (4, 6, 7, 8, 10) and p["col_tiles_per_wave"] in (1, 2, 3, 4), where
        wide = p["col_tiles_per_wave"] > 2 and p["waves"] == 8
        cols = 16 * p["col_tiles_per_wave"] * p["waves"] // (2 if wide else 1)
        assert p["workgroups"] == -(-N // cols) * p["splits"] * p["row_chunks"], where
        if wide:
            # the kernel for many rows: bf16, 8 waves, 5-8 row tiles for each half of them, whole chunks of k
            assert dtype == "bf16" and p["row_tiles"] in (10, 12, 14, 16) and p["waves"] == 8 and m >= 193, where
            assert K % 128 == 0 and (m < 257 or (K % 256 == 0 and p["k_per_split"] % 256 == 0)), where
            if m < 257:                                # one workgroup row, where it fills three quarters of the chip
                assert p["row_chunks"] == 1 and p["workgroups"] >= 192, where
            continue
        if p["col_tiles_per_wave"] == 4:
            # the hand-pipelined loop of one row chunk per workgroup: 6-8 row tiles, 4 waves, chunks taken in pairs
            assert dtype == "bf16" and p["row_tiles"] in (6, 7, 8) and p["waves"] == 4 and m >= 257, where
            assert K % 256 == 0 and p["k_per_split"] % 256 == 0, where
        if p["row_tiles"] > 8:
            # the tall single chunk: bf16 only, even tile counts up to 12, 8 waves, one column tile per wave
            assert dtype == "bf16" and p["row_tiles"] in (10, 12) and p["row_chunks"] == 1, where
            assert p["waves"] == 8 and p["col_tiles_per_wave"] == 1 and 129 <= m <= 192, where
        if p["row_chunks"] == 1 and p["row_tiles"] <= 8:
            assert p["row_tiles"] == -(-m // 16), where


def test_plan_rows_per_workgroup_for_many_rows():
    """Rows are dealt evenly to the halves of all workgroups: (row tiles per workgroup, workgroup rows) as launched."""
    for m, tiles, blocks in ((257, 10, 2), (288, 10, 2), (330, 12, 2), (400, 14, 2), (512, 16, 2), (700, 12, 4), (777, 14, 4),
                             (856, 14, 4), (1000, 16, 4), (1100, 14, 5), (1500, 12, 8), (2048, 16, 8), (12288, 16, 48)):
        for (N, K) in ((12288, 4096), (4096, 12288)):
            p = _plan("bf16", m, N, K)
            assert (p["row_tiles"], p["row_chunks"]) == (tiles, blocks), (m, N, K, p)
    # the head on all masked rows of a first step; a block's matrices on as many rows keep two columns tiles per wave
    p = _plan("bf16", 256, 126464, 4096, True)
    assert (p["row_tiles"], p["row_chunks"], p["col_tiles_per_wave"], p["waves"], p["workgroups"]) == (16, 1, 4, 8, 494)
    assert _plan("bf16", 256, 12288, 4096)["col_tiles_per_wave"] == 2


def test_plan_many_rows_one_or_two_row_chunks_per_workgroup():
    """Sizes measured in both kernels for many rows, where they differ by 10 % and more: two row chunks per workgroup where
    that fills the chip, one where it does not."""
    for m, N, K, single, waves in ((777, 5632, 1024, False, 4), (1024, 8192, 4096, False, 4), (860, 8192, 3584, False, 4),
                                   (1500, 4096, 4096, False, 4), (512, 2048, 256, True, 4), (1024, 11264, 2048, True, 8),
                                   (512, 24576, 4096, True, 8), (512, 12288, 4096, False, 8), (300, 4096, 12288, False, 8),
                                   (640, 3584, 18944, False, 8), (3440, 3584, 3584, False, 8), (2048, 11264, 2048, False, 8)):
        p = _plan("bf16", m, N, K, single)
        assert p["waves"] == waves and p["col_tiles_per_wave"] in ((4,) if waves == 4 else (3, 4)), (m, N, K, single, p)


def test_plan_depends_on_the_tile_count_alone():
    """The workspace of a context is sized from the first and the last row count of every 16: all of them have one plan."""
    for (N, K), single in itertools.product([s for s in SHAPES if s[1] % 8 == 0], (False, True)):
        for t in (1, 3, 8, 9, 12, 13, 16, 17, 18, 19, 21, 25, 31, 32, 33, 40, 47, 54, 61, 64, 80, 97, 150, 215, 768):
            first, mid, last = (_plan("bf16", 16 * t - d, N, K, single) for d in (15, 6, 0))
            assert first == last and mid == last, (t, N, K, single, first, mid, last)


def test_plan_at_the_benchmark_shapes():
    """One round of equal workgroups over the 256 compute units where the shape allows it (the shapes
    measured fastest on the MI355X)."""
    # LLaDA-8B, 46 rows
    assert _plan("bf16", 46, 12288, 4096)["workgroups"] == 256 and _plan("bf16", 46, 12288, 4096)["waves"] == 6
    assert _plan("bf16", 46, 4096, 4096)["workgroups"] == 256 and _plan("bf16", 46, 4096, 4096)["splits"] == 8
    gu = _plan("bf16", 46, 24576, 4096, True)
    assert (gu["workgroups"], gu["waves"], gu["splits"]) == (256, 6, 1)
    assert _plan("bf16", 46, 4096, 12288)["workgroups"] == 256
    # Dream-7B, 69 rows: the gate/up projection in one round of 10-wave workgroups instead of 296 8-wave ones
    gu = _plan("bf16", 69, 37888, 3584, True)
    assert (gu["workgroups"], gu["waves"], gu["splits"]) == (237, 10, 1)
    assert _plan("bf16", 69, 4608, 3584)["workgroups"] == 252
    # 3584 output columns: 7-wave workgroups (112 columns) make 32 column blocks x 8 splits = one full round
    dn = _plan("bf16", 69, 3584, 18944)
    assert (dn["waves"], dn["splits"], dn["workgroups"]) == (7, 8, 256)
    assert _plan("bf16", 69, 37888, 3584, True)["waves"] != 7        # the gated epilogue pairs neighbouring waves
    # row-count regimes
    assert _plan("bf16", 150, 12288, 4096)["row_tiles"] == 10 and _plan("bf16", 185, 12288, 4096)["row_tiles"] == 12
    p = _plan("bf16", 200, 12288, 4096)
    assert (p["row_chunks"], p["col_tiles_per_wave"]) == (2, 2)
    p = _plan("bf16", 856, 12288, 4096)
    assert (p["row_tiles"], p["row_chunks"], p["col_tiles_per_wave"], p["waves"]) == (14, 4, 3, 8)
    p = _plan("f32", 856, 768, 256)
    assert p["col_tiles_per_wave"] == 2 and p["row_chunks"] == 7


def test_plan_rejects_bad_arguments():
    from paper_2509_23094_amd import binding as B
    import ctypes
    shape = (ctypes.c_int32 * 7)()
    assert B._lib.d2c_plan_projection(1, 0, 16, 16, 0, shape) == B.D2C_EINVAL
    assert B._lib.d2c_plan_projection(5, 4, 16, 16, 0, shape) == B.D2C_EINVAL
    assert B._lib.d2c_plan_projection(1, 4, 16, 16, 0, None) == B.D2C_EINVAL


def test_launchers_take_an_empty_array():
    """Nothing to copy or to add is no launch and no error (a launch of no workgroups would be one)."""
    import ctypes
    from paper_2509_23094_amd import binding as B
    copy = getattr(B._lib, "_ZN3d2c15launch_copy_f32EPfPKfmP12ihipStream_t")
    copy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    add = getattr(B._lib, "_ZN3d2c17launch_sum_splitsEPfPKfimmP12ihipStream_t")
    add.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t, ctypes.c_size_t, ctypes.c_void_p]
    assert copy(None, None, 0, None) == 0 and add(None, None, 2, 0, 0, None) == 0
