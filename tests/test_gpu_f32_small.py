"""The fp32 tiles of 32 x 32 waves (32 x 64 and 64 x 64; gate and up sums meet
in LDS) where its rows, columns and K-steps can go wrong:
against the oracle, and the same bits as the 32 x 128 tile, which adds K in
the same order."""
import numpy as np
import pytest

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


# K-steps (of 32) below, at and past the six in flight; one column tile to many.
@pytest.mark.parametrize("d,I", [(64, 40), (128, 64), (192, 250), (576, 330)])
@pytest.mark.parametrize("counts", [[1], [0, 31, 0], [32, 33, 1], [129, 0, 64, 95],
                                    [65], [1] * 60 + [33] * 10])
def test_rows_columns_and_k_steps(L, oracle_mod, d, I, counts):
    E, T = len(counts), sum(counts)
    w = wl.Workload("t", T=T, d=d, E=E, I=I, dtype="f32")
    x, weights = wl.make_x(w, d), wl.make_experts(w, d)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    perm = np.random.default_rng(d).permutation(T).astype(np.int32)
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    offs = U.to_dev(offsets)
    xt = np.empty_like(x)
    xt[perm] = x  # token order: grouped row j is token perm[j]

    def layer(tile):
        L.readme_set_gemm_tile(tile)
        try:
            y = U.from_dev(L.readme_moe_ffn(U.to_dev(x), offs, packed, E, I))
            yt = U.from_dev(L.readme_moe_ffn_fused(U.to_dev(xt), U.to_dev(perm), offs, packed,
                                                   E, I))
        finally:
            L.readme_set_gemm_tile(0)
        return y, yt

    y, yt = layer(0)
    # Two fp32 sums of at most 640 terms: sqrt(640) * 2^-24 each, four times over.
    rel, _ = U.close(y, oracle_mod.moe_ffn(x, offsets, *weights), f"counts {counts} d {d} I {I}")
    assert rel <= 8 * 640 ** 0.5 * 2.0 ** -24
    assert (yt[perm] == y).all()
    assert (layer(6)[0] == y).all()
