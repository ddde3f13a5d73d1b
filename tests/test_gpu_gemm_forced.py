"""Kernels that no public override reaches (the 128-row two-phase launch 39),
each forced at the row counts, widths and K-steps where it can go wrong,
whatever the automatic rule would choose there."""
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
