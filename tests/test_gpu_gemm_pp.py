"""The two-phase grouped GEMM (tiles 30 and 31, one launch) at the sizes where its loop,
its row classes and its row maps can go wrong, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2410_19123_amd import workloads as wl
from tests import _util as U

pytestmark = pytest.mark.gpu

# Rows of an expert around every tile height; K-steps (of 64) below, at and
# past the four the loop keeps in flight, odd and even; output widths of one
# to five 64-column pairs of weight groups.
COUNTS = [0, 1, 63, 64, 65, 127, 129, 255, 256, 257, 385]


@pytest.fixture(scope="module")
def L():
    from paper_2410_19123_amd import _lib
    _lib.load()
    return _lib


@pytest.fixture(scope="module")
def oracle_mod():
    from oracle import oracle
    return oracle


@pytest.mark.parametrize("tile", [30, 31])
@pytest.mark.parametrize("d,I", [(64, 64), (128, 40), (192, 192), (320, 250), (576, 330)])
def test_heights_and_k_steps(L, oracle_mod, tile, d, I):
    """Every row against the oracle, grouped and through the row maps; the
    same bits both ways."""
    E, T = len(COUNTS), sum(COUNTS)
    w = wl.Workload("t", T=T, d=d, E=E, I=I, dtype="bf16")
    x = wl.make_x(w, d)
    weights = wl.make_experts(w, d)
    offsets = np.concatenate([[0], np.cumsum(COUNTS)]).astype(np.int32)
    perm = np.random.default_rng(d).permutation(T).astype(np.int32)
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    offs = U.to_dev(offsets)
    print(f"tile {tile} d {d} I {I}", flush=True)
    L.readme_set_gemm_tile(tile)
    try:
        y = U.from_dev(L.readme_moe_ffn(U.to_dev(x), offs, packed, E, I))
        xt = np.empty_like(x)
        xt[perm] = x  # token order: grouped row j is token perm[j]
        yt = U.from_dev(L.readme_moe_ffn_fused(U.to_dev(xt), U.to_dev(perm), offs, packed, E, I))
    finally:
        L.readme_set_gemm_tile(0)
    U.close(y, oracle_mod.moe_ffn(x, offsets, *weights), f"tile {tile}")
    assert (yt[perm] == y).all()


@pytest.mark.parametrize("tile", [30, 31])
def test_residual_rows(L, oracle_mod, tile):
    """The residual epilogue (a two-layer stack) on ragged blocks."""
    counts = [130, 0, 70, 300]
    w = wl.Workload("t", T=sum(counts), d=320, E=4, I=200, dtype="bf16", layers=2)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    host = [wl.make_experts(w, 7, layer=k) for k in range(2)]
    packed = [L.readme_pack_experts(*U.weights_to_dev(*h)) for h in host]
    x0 = wl.bf16_bits_to_f32(wl.make_x(w, 7)).astype(np.float32)
    xr = U.to_dev(x0)
    L.readme_set_gemm_tile(tile)
    try:
        L.readme_moe_ffn_stack(xr, U.to_dev(offsets), packed, w.E, w.I)
        torch.cuda.synchronize()
    finally:
        L.readme_set_gemm_tile(0)
    ref = x0.copy()
    for k in range(2):
        ref = (ref.astype(np.float64) + oracle_mod.layer(ref, offsets, *host[k], eps=1e-5))
        ref = ref.astype(np.float32)
    U.close(U.from_dev(xr).astype(np.float64) - x0, ref.astype(np.float64) - x0, "stack")
