"""The block-sweep inverse where it can go wrong: every count of token-range partials that its loads group
differently, more matrices than one round of the compute units (the waves' roles rotate), a large condition number;
its off-diagonal blocks are exact transposes of each other; and B's partials are folded in range order."""
import numpy as np
import pytest

from vda_testutil import fold_partials, from_operand_tiles, rel_max_err, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    from paper_2609_20744_amd import vda
    return vda


@pytest.mark.parametrize("dk,count,tail,splits", [(32, 3, 0, 1), (32, 2, 2, 5), (64, 5, 3, 2), (64, 2, 1, 4),
                                                  (128, 3, 3, 3), (128, 2, 2, 4), (128, 2, 1, 8), (128, 530, 18, 4)])
def test_inverse(V, dk, count, tail, splits):
    import torch
    rng = np.random.default_rng(dk + count)
    K = rng.standard_normal((count, 2 * dk, dk)) + 2.0 * rng.standard_normal((count, 1, dk))
    K /= np.linalg.norm(K, axis=-1, keepdims=True)
    A = np.matmul(K.transpose(0, 2, 1) * rng.random((count, 1, 2 * dk)), K)
    A[0] *= 30.0
    w = rng.random((splits, count)) + 0.1  # the partials' shares of each split frame
    w /= w.sum(0)
    nparts = count + tail * (splits - 1)
    parts = np.empty((nparts, dk, dk), np.float32)
    parts[:count] = A
    for i in range(count - tail, count):
        for s in range(splits):
            parts[i + s * tail] = w[s, i] * A[i]
    A32 = parts[:count].astype(np.float64)
    for s in range(1, splits):
        A32[count - tail:] += parts[count + (s - 1) * tail:count + s * tail]
    ref = np.linalg.inv(np.eye(dk) + A32)
    cond = np.linalg.cond(np.eye(dk) + A32)
    B = rng.standard_normal((nparts, 32, dk)).astype(np.float32)
    args = dict(count=count, tail_frames=tail, splits=splits)
    Bi, Bt = to_device(B, "f32"), to_device(B, "f32")
    inv = V.frame_inverse(to_device(parts, "f32"), Bi, **args).double().cpu().numpy()
    tiles = V.frame_inverse(to_device(parts, "f32"), Bt, tiles=True, **args)
    tiles = from_operand_tiles(tiles, dk)
    # Both fold B's partials into the first in range order, in fp32.
    folded = fold_partials(torch.from_numpy(B), count, tail, splits)
    assert torch.equal(Bi[:count].cpu(), folded) and torch.equal(Bt[:count].cpu(), folded)
    for i in range(count):
        # As the stage test's bound: fp32 elimination's error grows with the condition number.
        assert rel_max_err(inv[i], ref[i]) < 2e-6 * cond[i], (i, cond[i])
        # The tiles hold the same values to bf16 hi + lo, 2^-17 of each.
        assert rel_max_err(tiles[i], inv[i].T) < 2.0 ** -16, i
    off = np.kron(1 - np.eye(dk // 16), np.ones((16, 16))).astype(bool)
    assert np.array_equal(inv[:, off], inv.transpose(0, 2, 1)[:, off])
