"""The kernels that no public override reaches (the decode tiles 32 to 35, the
fp32 tiles 36 to 38, the 128-row two-phase launch 39), each forced at the row
counts, widths and K-steps where it can go wrong, whatever the automatic rule
would choose there."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2410_19123_amd import workloads as wl
from tests import _util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2410_19123_amd import _lib
    _lib.load()
    return _lib


@pytest.fixture(scope="module")
def oracle_mod():
    from oracle import oracle
    return oracle


@contextlib.contextmanager
def forced(L, tile):
    print(f"tile {tile}", flush=True)
    assert L.load().readme_internal_set_gemm_tile(tile) == 0
    try:
        yield
    finally:
        L.load().readme_internal_set_gemm_tile(0)


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def _stack(L, tile, w, x0, packed, counts):
    """One residual layer on the fp32 rows x0."""
    xr = U.to_dev(x0)
    with forced(L, tile):
        L.readme_moe_ffn_stack(xr, U.to_dev(_offsets(counts)), [packed], w.E, w.I)
        torch.cuda.synchronize()
    return U.from_dev(xr)


def _layer(L, tile, w, x, weights, counts, seed):
    """Grouped rows of a layer, in its grouped form and through the row maps
    (asserted equal)."""
    T = sum(counts)
    perm = np.random.default_rng(seed).permutation(T).astype(np.int32)
    offs = U.to_dev(_offsets(counts))
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    xt = np.empty_like(x)
    xt[perm] = x  # token order: grouped row j is token perm[j]
    with forced(L, tile):
        y = U.from_dev(L.readme_moe_ffn(U.to_dev(x), offs, packed, w.E, w.I))
        yt = U.from_dev(L.readme_moe_ffn_fused(U.to_dev(xt), U.to_dev(perm), offs, packed, w.E,
                                               w.I))
    assert (yt[perm] == y).all()
    return y


# K-steps (of 64) of the two GEMMs: 1 to 9, below, at and past what each kernel
# keeps in flight; outputs of one 64-column unit to several tiles.
@pytest.mark.parametrize("d,I", [(64, 64), (128, 40), (192, 192), (320, 250), (576, 330)])
def test_two_phase_tiles_equal_the_register_streamed_ones(L, oracle_mod, d, I):
    """256- and 128-row launches on blocks around every tile height: the oracle's
    values, and the bits of tile 24, which adds K in the same order."""
    counts = [0, 1, 63, 64, 65, 127, 129, 255, 256, 257, 385]
    w = wl.Workload("t", T=sum(counts), d=d, E=len(counts), I=I, dtype="bf16")
    x, weights = wl.make_x(w, d), wl.make_experts(w, d)
    y = _layer(L, 39, w, x, weights, counts, d)
    U.close(y, oracle_mod.moe_ffn(x, _offsets(counts), *weights), "tile 39")
    x0 = wl.bf16_bits_to_f32(x).astype(np.float32)
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    ys = _stack(L, 39, w, x0, packed, counts)
    for tile in (24, 30):
        assert (_layer(L, tile, w, x, weights, counts, d) == y).all()
        assert (_stack(L, tile, w, x0, packed, counts) == ys).all()


@pytest.mark.parametrize("d,I", [(64, 64), (128, 150), (576, 1040), (1088, 700)])
@pytest.mark.parametrize("counts", [[1], [0, 16, 17], [31, 0, 32, 33], [65, 15]])
def test_decode_tiles_equal_each_other(L, oracle_mod, d, I, counts):
    """One summation order: every width gives the same bits, in a layer (store)
    and in a stack (residual)."""
    w = wl.Workload("t", T=sum(counts), d=d, E=len(counts), I=I, dtype="bf16")
    x, weights = wl.make_x(w, 3), wl.make_experts(w, 3)
    y = _layer(L, 35, w, x, weights, counts, d)
    U.close(y, oracle_mod.moe_ffn(x, _offsets(counts), *weights), f"counts {counts}")
    for tile in (32, 33, 34):
        assert (_layer(L, tile, w, x, weights, counts, d) == y).all()

    x0 = wl.bf16_bits_to_f32(x).astype(np.float32)
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    ys = _stack(L, 35, w, x0, packed, counts)
    U.close(ys.astype(np.float64) - x0,
            oracle_mod.layer(x0, _offsets(counts), *weights, eps=1e-5), "stack")
    for tile in (32, 33, 34):
        assert (_stack(L, tile, w, x0, packed, counts) == ys).all()


@pytest.mark.parametrize("d,I", [(64, 40), (128, 64), (192, 250), (576, 330)])
@pytest.mark.parametrize("counts", [[1], [0, 31, 33], [129, 0, 64, 95], [1] * 60 + [33] * 10])
def test_fp32_tiles_equal_the_32x128_tile(L, oracle_mod, d, I, counts):
    w = wl.Workload("t", T=sum(counts), d=d, E=len(counts), I=I, dtype="f32")
    x, weights = wl.make_x(w, d), wl.make_experts(w, d)
    y = _layer(L, 6, w, x, weights, counts, d)
    # Two fp32 sums of at most 640 terms: sqrt(640) * 2^-24 each, four times over.
    rel, _ = U.close(y, oracle_mod.moe_ffn(x, _offsets(counts), *weights), f"counts {counts}")
    assert rel <= 8 * 640 ** 0.5 * 2.0 ** -24
    for tile in (36, 37, 38):
        assert (_layer(L, tile, w, x, weights, counts, d) == y).all()


@pytest.mark.parametrize("dtype,same,tiles", [("f32", 6, (36, 37, 38)), ("bf16", 24, (30, 39)),
                                              ("bf16", 35, (32, 33, 34))])
def test_permanent_slices_and_pairs(L, oracle_mod, dtype, same, tiles):
    """Row groups over all rows (gate/up), K in segments (down) and top-2 pair
    rows through the maps: the bits of the tile of the same summation order."""
    counts = [70, 0, 2, 130]
    w = wl.Workload("t", T=sum(counts), d=320, E=4, I=200, P=400, dtype=dtype)
    x, e, p = wl.make_x(w, 9), wl.make_experts(w, 9), wl.make_permanent(w, 9)
    order = np.random.default_rng(9).permutation(w.T).astype(np.int32)
    packed = L.readme_pack_experts_permanent(*U.weights_to_dev(*e), *U.weights_to_dev(*p))
    plain = L.readme_pack_experts(*U.weights_to_dev(*e))
    offs, perm, xd = U.to_dev(_offsets(counts)), U.to_dev(order), U.to_dev(x)
    out = {}
    for tile in (same,) + tiles:
        with forced(L, tile):
            y = U.from_dev(L.readme_moe_ffn_permanent_fused(xd, perm, offs, packed, w.E, w.I, w.P))
            # Pair rows: token perm[j] // 2, so only the first half of x is read.
            yp = U.from_dev(L.readme_moe_ffn_topk(xd[:w.T // 2], perm, offs, plain, w.E, w.I, 2))
        out[tile] = (y, yp)
        assert (y == out[same][0]).all() and (yp == out[same][1]).all()
    U.close(out[same][1][order], oracle_mod.moe_ffn(x[order // 2], _offsets(counts), *e), "pairs")
    ref = oracle_mod.moe_ffn_permanent(x[order], _offsets(counts), *e, *p)
    U.close(out[same][0][order], ref, "permanent")
