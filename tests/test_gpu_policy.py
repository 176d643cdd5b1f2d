"""GPU parity of the block-size policy (sd_block_size_policy) against the fp64 oracle.

Tolerance: p and the activations are fp32 and every product accumulates in fp32 (the weights
are bf16 on both sides), so the scores agree to about 1e-5 relative; the test allows
1e-4 + 1e-4 |o|.  The chosen block size must be the oracle's unless its best two scores lie
within that band (counted, then the device's choice must be one of the two)."""
import numpy as np
import pytest
import torch

import gpu_util as G
import oracle.policy as OP
import paper_2606_31315_amd as sd
from paper_2606_31315_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(pp):
    dev = G.dev()
    G.log(f"sd_block_size_policy P={pp.P} V={pp.V} H={pp.H} k={pp.radius} dtype={pp.dtype}")
    sc, bs = sd.block_size_policy(pp.logits.to(dev), pp.w1.to(dev), torch.from_numpy(pp.b1).to(dev), pp.w2.to(dev),
                                  torch.from_numpy(pp.b2).to(dev), pp.w3.to(dev), torch.from_numpy(pp.b3).to(dev),
                                  pp.base_block)
    torch.cuda.synchronize()
    ref = OP.block_size_policy(pp.logits, pp.w1, pp.b1, pp.w2, pp.b2, pp.w3, pp.b3, pp.base_block, pp.radius)
    sc = sc.cpu().numpy().astype(np.float64)
    bs = bs.cpu().numpy()
    tol = 1e-4 + 1e-4 * np.abs(ref.scores)
    assert (np.abs(sc - ref.scores) <= tol).all(), np.abs(sc - ref.scores).max()
    near = ref.margin < 2 * tol.max()
    assert np.array_equal(bs[~near], ref.block_size[~near])
    for i in np.nonzero(near)[0]:
        top2 = np.argsort(ref.scores[i])[-2:] + pp.base_block - pp.radius
        assert bs[i] in top2
    G.log(f"  max score error {np.abs(sc - ref.scores).max():.2e}; near-ties {int(near.sum())}")
    return sc, bs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_small_shapes(dtype):
    _check(W.make_policy(61, P=3, V=4096, H=256, radius=2, dtype=dtype))


def test_vocab_not_a_chunk_multiple_and_wide_radius():
    _check(W.make_policy(62, P=2, V=1000, H=72, radius=7, base_block=10, dtype="bf16"))


@pytest.mark.parametrize("P", [1, 5, 11])
def test_qwen3_vocab_hidden_2048(P):
    """The paper's predictor: V = 151936 (Qwen3), two hidden layers of 2048, k = 2 around B = 16; one
    pass of the matrix layers, and with a workspace of the dense kernels' size those (11 prompts: two
    groups of their passes)."""
    pp = W.make_policy(63 + P, P=P, V=151936, H=2048, radius=2, dtype="bf16")
    sc, _ = _check(pp)
    dense, _ = _call(pp, _dense_bytes(P, 2048))
    # both within the fp64 oracle's band of 1e-4 + 1e-4 |o|, so within twice that of each other
    assert (np.abs(sc - dense) <= 2e-4 + 2e-4 * np.abs(dense)).all()


def _dense_bytes(P, H):
    """Workspace of the dense kernels alone: chunk records, then two layers of activations."""
    up = lambda n: (n + 255) // 256 * 256
    return up(P * 64 * 8) + 2 * up(P * H * 4)


def _call(pp, ws=None):
    dev = G.dev()
    f = lambda x: torch.from_numpy(x).to(dev)
    sc, bs = sd.block_size_policy(pp.logits.to(dev), pp.w1.to(dev), f(pp.b1), pp.w2.to(dev), f(pp.b2), pp.w3.to(dev),
                                  f(pp.b3), pp.base_block,
                                  workspace=None if ws is None else torch.empty(ws, dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    return sc.cpu().numpy(), bs.cpu().numpy()


@pytest.mark.parametrize("P,V,H,dtype", [(1, 64, 8, "bf16"), (3, 8, 8, "f32"), (3, 72, 24, "bf16"), (16, 632, 520, "f32"),
                                         (17, 1288, 72, "bf16"), (4, 2040, 1032, "bf16"), (1, 4160, 512, "f32"),
                                         (2, 1000, 64, "bf16")])
def test_matrix_layers_edges(P, V, H, dtype):
    """Vocabularies below, at and past a 64-element tile, partial rows of the 64- and 512-row groups
    and of the 16-row tiles, one more prompt than a pass holds (up to four prompts take the dense
    kernels here: test_layers_rule_edges has these edges with more); and the dense kernels, which a
    workspace of their size alone still gets, on the same inputs."""
    pp = W.make_policy(80 + P, P=P, V=V, H=H, radius=2, dtype=dtype)
    sc, _ = _check(pp)
    dense, _ = _call(pp, _dense_bytes(P, H))
    # both within the fp64 oracle's band of 1e-4 + 1e-4 |o|, so within twice that of each other
    assert (np.abs(sc - dense) <= 2e-4 + 2e-4 * np.abs(dense)).all()


def test_matrix_layers_special_values():
    """Prompts with -inf logits (a whole chunk of them too), only -inf, +inf and NaN; weights that are
    infinite, NaN, or infinite where p underflows to 0: the dense kernels' values, NaN for NaN."""
    P, V, H = 6, 4096, 64
    pp = W.make_policy(97, P=P, V=V, H=H, radius=2, dtype="bf16")
    pp.logits[1, :1500] = float("-inf")
    pp.logits[2, :] = float("-inf")
    pp.logits[3, 77] = float("inf")
    pp.logits[4, 4000] = float("nan")
    dense, _ = _call(pp, _dense_bytes(P, H))
    sc, bs = _call(pp)
    assert np.allclose(sc, dense, rtol=2e-4, atol=2e-4, equal_nan=True)
    ok = _check(W.PolicyProblem(pp.logits[:2], *[getattr(pp, k) for k in ("w1", "b1", "w2", "b2", "w3", "b3", "base_block",
                                                                          "radius", "dtype")]))
    assert np.isfinite(ok[0]).all()
    pp.w1[5, 100] = float("inf")
    pp.w1[6, 4095] = float("-inf")
    pp.w1[7, 9] = float("nan")
    pp.logits[5, 100] = -1e4  # p = 0 there: 0 times infinity
    dense, _ = _call(pp, _dense_bytes(P, H))
    sc, _ = _call(pp)
    assert np.array_equal(np.isnan(sc), np.isnan(dense)) and np.array_equal(np.isinf(sc), np.isinf(dense))
    fin = np.isfinite(dense)
    assert np.allclose(sc[fin], dense[fin], rtol=2e-4, atol=2e-4)


def test_matrix_layers_large_weights():
    """Weights near the largest bf16: sums over a chunk overflow before softmax's normaliser, the layer's
    output does not.  The dense kernels' values."""
    P, V, H = 6, 4096, 64
    pp = W.make_policy(98, P=P, V=V, H=H, radius=2, dtype="bf16")
    pp.w1[5, :] = 3e38
    pp.w1[6, ::2] = -3e38
    pp.w1[40, 17:1900] = 2e38
    dense, _ = _call(pp, _dense_bytes(P, H))
    sc, _ = _call(pp)
    assert np.isfinite(dense).all() and np.isfinite(sc).all()
    # fp32 sums of the same products in another order, as in _check
    assert (np.abs(sc - dense) <= 2e-4 * np.abs(dense).max()).all()


# On both sides of the rule that chooses between the dense and the matrix layers, and the matrix layers' edges
# (vocabularies below, at and past a tile; partial row groups) at prompt counts that take them.
@pytest.mark.parametrize("P,V,H,dtype", [(1, 59968, 72, "bf16"), (1, 60032, 72, "f32"), (2, 60008, 24, "bf16"),
                                         (1, 65536, 8, "bf16"), (2, 65600, 520, "bf16"), (3, 16320, 64, "bf16"),
                                         (3, 16384, 520, "f32"), (4, 8192, 1032, "bf16"),
                                         (4, 8128, 1032, "bf16"), (4, 8192, 1024, "f32"), (4, 24568, 24, "bf16"), (4, 24584, 72, "bf16"),
                                         (5, 64, 8, "bf16"), (5, 8, 8, "f32"), (6, 72, 24, "bf16"), (8, 2040, 1032, "bf16"),
                                         (5, 4160, 512, "f32"), (7, 1000, 64, "bf16")])
def test_layers_rule_edges(P, V, H, dtype):
    pp = W.make_policy(120 + P, P=P, V=V, H=H, radius=2, dtype=dtype)
    sc, _ = _check(pp)
    dense, _ = _call(pp, _dense_bytes(P, H))
    # both within the fp64 oracle's band of 1e-4 + 1e-4 |o|, so within twice that of each other
    assert (np.abs(sc - dense) <= 2e-4 + 2e-4 * np.abs(dense)).all()
