"""The tile a grouped GEMM launch takes, by its sizes alone (no GPU: the rule is
host code)."""
import ctypes
import os

import pytest

# Tile numbers of the kernels no override reaches.
SKINNY_16, SKINNY_32, SKINNY_64, DECODE_128 = 32, 33, 34, 35
F32_32x64, F32_32x64_S3, F32_64x64 = 36, 37, 38
PP_256, PP_128 = 30, 39
INT32_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def tile():
    from paper_2410_19123_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("libreadme.so not built")
    fn = _lib.load().readme_internal_gemm_tile
    fn.restype = ctypes.c_int32
    fn.argtypes = [ctypes.c_int32] + [ctypes.c_int64] * 3 + [ctypes.c_int32] * 4
    return lambda T, N, K, E, f32=False, shared=0, m32=0, stack=False: fn(f32, T, N, K, E, shared,
                                                                          m32, stack)


@pytest.mark.parametrize("T,N,K,E,want", [
    (4 << 20, 1024, 8192, 8, F32_64x64),
    (1 << 28, 64, 128, 1, F32_64x64),
    (256, 1024, 512, 4, F32_32x64),
])
def test_fp32_keeps_its_tiles_past_32_bit_offsets(tile, T, N, K, E, want):
    assert tile(T, N, K, E, f32=True) == want


def test_bf16_past_32_bit_offsets(tile):
    """Tiles whose activation offsets are 32-bit give way to 64-bit ones."""
    T = 4 << 20
    assert T * 8192 // 8 > INT32_MAX
    assert tile(T // 8, 1024, 8192, 8) == PP_256
    assert tile(T, 1024, 8192, 8) == 24


@pytest.mark.parametrize("T,N,E,shared", [(1 << 21, 1 << 15, 4, 0), ((1 << 21) - 512, 1 << 15, 1, 0),
                                          (1 << 20, 1 << 15, 4, 1), (1 << 26, 1 << 12, 256, 0)])
def test_fp32_grids_stay_below_2_to_32_threads(tile, T, N, E, shared):
    """Tiles (rounded up to 8) times threads of the chosen tile: a grid's size
    in threads is a 32-bit number."""
    rows_cols_threads = {F32_64x64: (64, 64, 256), 1: (256, 256, 512)}
    h, w, threads = rows_cols_threads[tile(T, N, 64, E, f32=True, shared=shared)]
    m = (T + E * (h - 1)) // h + shared * -(-T // h)
    assert -(-m * -(-N // w) // 8) * 8 * threads < 2 ** 32


@pytest.mark.parametrize("d,I", [(512, 256), (1024, 2816), (4096, 1376), (8192, 3584)])
@pytest.mark.parametrize("E", [8, 16, 64, 256])
def test_few_rows_per_expert_take_32_row_tiles(tile, d, I, E):
    """Under 8 rows per expert, however many experts: a taller tile would be
    mostly padding and leave fewer workgroups to stream the weights."""
    Ip = (I + 63) // 64 * 64
    for per in (1, 4, 7):
        for N, K in ((2 * Ip, d), (d, Ip)):
            assert tile(per * E, N, K, E) in (SKINNY_16, SKINNY_32, SKINNY_64, DECODE_128, 27)


def test_a_row_group_is_at_least_one_tile(tile):
    """Many experts whose rows fill a small part of a tall tile: the estimate
    counts a tile for each, not the rows' share of one."""
    for E, N, K in ((64, 1024, 1024), (32, 2816, 4096), (16, 7168, 8192)):
        assert tile(E * 40, N, K, E) != PP_256


@pytest.mark.parametrize("T,E", [(32, 16), (200, 8), (500, 64), (3, 3)])
def test_32x128_decode_tile_of_layers_and_stacks(tile, T, E):
    """A stack's tile has one summation order with the weight streams, whatever
    counts are known; a layer, which knows none, takes the faster tile."""
    streams = (SKINNY_16, SKINNY_32, SKINNY_64)
    N, K = 2816, 4096
    layer, stack = tile(T, N, K, E), tile(T, N, K, E, stack=True)
    assert stack in streams + (DECODE_128,)
    assert layer == (27 if stack == DECODE_128 else stack)
    for m32 in range(1, min(E, T) + 1):
        assert tile(T, N, K, E, stack=True, m32=m32) in streams + (DECODE_128,)


def test_tile_31_runs_the_tallest_tiles(tile):
    """A stored choice of 31 (made when it meant 192-row tiles) keeps a launch of
    tall tiles at every size."""
    from paper_2410_19123_amd import _lib
    try:
        for forced in (30, 31):
            _lib.readme_set_gemm_tile(forced)
            assert tile(8192, 7168, 8192, 8) == tile(512, 1024, 1024, 8) == PP_256
    finally:
        _lib.readme_set_gemm_tile(0)
