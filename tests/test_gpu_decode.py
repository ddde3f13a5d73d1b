"""The decode GEMMs (weight streams that split K over a workgroup's waves, and
the 32 x 128 tile in the same summation order) at the sizes where their K
ranges, row tiles and column tiles can go wrong, against the oracle."""
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


def _ids(T, E, spread, seed=5):
    if spread == "one":
        return np.full(T, E // 2, np.int32)
    return np.random.default_rng(seed).integers(0, E, T).astype(np.int32)


# K-steps of 64 in the two GEMMs: fewer than the four ranges (1, 2, 3), not a
# multiple of them (9, 17, 22), and enough that every kernel's loop turns.
@pytest.mark.parametrize("d,I", [(64, 64), (128, 150), (576, 1040), (1088, 1376), (4096, 96)])
@pytest.mark.parametrize("T,E,spread", [(1, 8, "one"), (2, 2, "any"), (5, 3, "any"),
                                        (16, 4, "one"), (17, 1, "one"), (33, 2, "one"),
                                        (64, 16, "any")])
def test_layer_rows(L, oracle_mod, d, I, T, E, spread):
    """Every row of a layer, grouped and through the row maps (same bits)."""
    w = wl.Workload("t", T=T, d=d, E=E, I=I, dtype="bf16")
    x = wl.make_x(w, 3)
    weights = wl.make_experts(w, 3)
    ids = _ids(T, E, spread)
    packed = L.readme_pack_experts(*U.weights_to_dev(*weights))
    xd = U.to_dev(x)
    counts, offs, perm, inv, xg = L.readme_group_by_expert(U.to_dev(ids), E, x=xd)
    y = U.from_dev(L.readme_ungroup(L.readme_moe_ffn(xg, offs, packed, E, I), inv))
    yf = U.from_dev(L.readme_moe_ffn_fused(xd, perm, offs, packed, E, I))
    order = np.argsort(ids, kind="stable")
    offsets = np.concatenate([[0], np.cumsum(np.bincount(ids, minlength=E))]).astype(np.int32)
    ref = oracle_mod.moe_ffn(x[order], offsets, *weights)
    U.close(y[order], ref, f"T {T} E {E} d {d} I {I}")
    assert (yf == y).all()


@pytest.mark.parametrize("T,d,I", [(1, 192, 64), (1, 8192, 130), (2, 1088, 700), (3, 1088, 700),
                                   (40, 2048, 1500), (64, 4096, 1000)])
@pytest.mark.parametrize("spread", ["one", "any"])
def test_stack_counts_and_offload_agree(L, oracle_mod, T, d, I, spread):
    """Counts known or not, weights resident or cached, the norm inside the
    gate/up (one row) or before it: the same bits, and the oracle's."""
    E, layers = 8, 2
    w = wl.Workload("t", T=T, d=d, E=E, I=I, dtype="bf16", layers=layers)
    host = [wl.make_experts(w, 11, layer=k) for k in range(layers)]
    packed = [L.readme_pack_experts(*U.weights_to_dev(*h)) for h in host]
    ids = _ids(T, E, spread)
    cnt = np.bincount(ids, minlength=E)
    x0 = wl.bf16_bits_to_f32(wl.make_x(w, 11)).astype(np.float32)
    _, offs, perm, inv, xg = L.readme_group_by_expert(U.to_dev(ids), E, x=U.to_dev(x0))
    a, b, c = xg.clone(), xg.clone(), xg.clone()
    L.readme_moe_ffn_stack(a, offs, packed, E, I)
    L.readme_moe_ffn_stack(b, offs, packed, E, I, counts=cnt)
    ex = L.Offload(packed, E, d, I, 2 * E)
    try:
        ex.stack(c, offs, cnt)
        torch.cuda.synchronize()
    finally:
        ex.close()
    a, b, c = (U.from_dev(t) for t in (a, b, c))
    assert (a == b).all() and (a == c).all()
    start = x0[np.argsort(ids, kind="stable")]
    offsets = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    ref = start.copy()
    for k in range(layers):
        ref = (ref.astype(np.float64) +
               oracle_mod.layer(ref, offsets, *host[k], eps=1e-5)).astype(np.float32)
    U.close(a.astype(np.float64) - start, ref.astype(np.float64) - start, "stack")


def test_permanent_and_topk_rows(L, oracle_mod):
    """The K segments of a permanent expert and the pair rows of top-K at
    decode sizes."""
    w = wl.Workload("t", T=6, d=576, E=4, I=200, P=400, dtype="bf16")
    x, ids = wl.make_x(w, 9), _ids(6, 4, "any")
    e, p = wl.make_experts(w, 9), wl.make_permanent(w, 9)
    packed = L.readme_pack_experts_permanent(*U.weights_to_dev(*e), *U.weights_to_dev(*p))
    xd = U.to_dev(x)
    _, offs, perm, _, _ = L.readme_group_by_expert(U.to_dev(ids), w.E)
    y = U.from_dev(L.readme_moe_ffn_permanent_fused(xd, perm, offs, packed, w.E, w.I, w.P))
    order = np.argsort(ids, kind="stable")
    offsets = np.concatenate([[0], np.cumsum(np.bincount(ids, minlength=w.E))]).astype(np.int32)
    U.close(y[order], oracle_mod.moe_ffn_permanent(x[order], offsets, *e, *p), "permanent")

    K = 2
    pair_ids = np.stack([ids, (ids + 1) % 4], 1).reshape(-1).astype(np.int32)
    packed = L.readme_pack_experts(*U.weights_to_dev(*e))
    _, offs, perm, _, _ = L.readme_group_by_expert(U.to_dev(pair_ids), w.E)
    yp = U.from_dev(L.readme_moe_ffn_topk(xd, perm, offs, packed, w.E, w.I, K))
    order = np.argsort(pair_ids, kind="stable")
    offsets = np.concatenate([[0], np.cumsum(np.bincount(pair_ids, minlength=4))]).astype(np.int32)
    U.close(yp[order], oracle_mod.moe_ffn(x[order // K], offsets, *e), "pairs")
