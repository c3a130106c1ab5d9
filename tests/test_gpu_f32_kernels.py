"""The fp32 storage path's kernels at the edges of their tiles, against fp64 on the CPU, each within the bound that
its own rounding gives: u = 2^-24 per operation of the longest chain of sums, over the sum of the terms' magnitudes.
"""
import numpy as np
import pytest

import oracle.vda_oracle as O
from vda_testutil import TOL_F32, fold_partials, rel_max_err, to_device

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def V():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    from paper_2609_20744_amd import vda
    return vda


# Tokens: one, around the tile (32) and the accumulator chain (256) of a range, and ranges of every remainder.
@pytest.mark.parametrize("N,tail,splits", [(1, 0, 1), (31, 0, 1), (32, 0, 1), (33, 0, 1), (255, 0, 1), (257, 0, 1),
                                           (520, 2, 2), (1025, 1, 8)])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 32), (32, 128), (128, 64)])
def test_stats(V, N, tail, splits, dk, dv):
    rng = np.random.default_rng(N + dk + dv)
    k, v = (rng.standard_normal((1, 3, N, d)).astype(np.float32) for d in (dk, dv))
    beta = rng.random((1, 3, N)).astype(np.float32)
    beta[:, :, ::7] = 0.0
    A, B = V.frame_stats(to_device(k, "f32"), to_device(v, "f32"), to_device(beta, "f32"), splits=splits,
                         tail_frames=tail)
    A = fold_partials(A.double(), 3, tail, splits).cpu().numpy()
    B = fold_partials(B.double(), 3, tail, splits).cpu().numpy()
    # beta * k, 256 sums in a chain, the chains' sums, and one spare.
    rel = U * (1 + min(N, 256) + -(-N // 256) + 1)
    for t in range(3):
        As, Bs = O.frame_statistics(*(x[0, t].astype(np.float64) for x in (k, v, beta)))
        Aa, Ba = O.frame_statistics(*(np.abs(x[0, t]).astype(np.float64) for x in (k, v, beta)))
        assert np.all(np.abs(A[t] - As) <= rel * Aa)
        assert np.all(np.abs(B[t] - Bs) <= rel * Ba)


# Tokens: one, around a wave's 16, a step's 64, and workgroups with and without a last step.
@pytest.mark.parametrize("H,N", [(1, 1), (2, 15), (1, 17), (2, 64), (1, 65), (3, 129), (70, 200)])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 32), (32, 128), (128, 64)])
def test_readout(V, H, N, dk, dv):
    F = 2
    rng = np.random.default_rng(N + dk + dv)
    q = rng.standard_normal((H, F, N, dk)).astype(np.float32)
    sf, sr = (rng.standard_normal((H, F, dv, dk)).astype(np.float32) for _ in range(2))
    gate = rng.random(H).astype(np.float32)
    y = V.readout(*(to_device(x, "f32") for x in (q, sf, sr, gate))).double().cpu().numpy()
    S = sf.astype(np.float64) + sr
    o = np.einsum("hftk,hfvk->hftv", q.astype(np.float64), S)
    # S~'s sum and the d_k products' chain.
    do = U * (dk + 2) * np.einsum("hftk,hfvk->hftv", np.abs(q).astype(np.float64), np.abs(S))
    rms = np.sqrt((o * o).mean(-1, keepdims=True) + 1e-6)
    g = gate.astype(np.float64)[:, None, None, None]
    ref = g * o / rms
    # The norm's own sum of d_v squares (relative error U * d_v / 2), root, quotient and product.
    bound = g / rms * (do + np.abs(o) / rms * do.max(-1, keepdims=True)) + U * (dv / 2 + 8) * np.abs(ref)
    assert np.all(np.abs(y - ref) <= bound)


# The scan from fp32 operand tiles (vda_forward) does the sums of the scan from rows (the stage) in the same order, so
# the two passes agree bit for bit: one step and no step in flight, every depth of the ring, and more heads than XCDs;
# frames of one range, of three (all of whose partials the inverse loads and folds at once) and of up to eight.
@pytest.mark.parametrize("H,F", [(1, 1), (2, 2), (1, 3), (3, 5), (9, 8)])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 32), (32, 128), (128, 64)])
@pytest.mark.parametrize("N,ranges", [(33, 1), (400, 3), (1536, 8)])
def test_scan_tiles(V, H, F, dk, dv, N, ranges):
    import torch
    rng = np.random.default_rng(H + F + dk + dv)
    q, k = (to_device((x / np.linalg.norm(x, axis=-1, keepdims=True)).astype(np.float32), "f32")
            for x in (rng.standard_normal((H, F, N, dk)) for _ in range(2)))
    v = to_device(rng.standard_normal((H, F, N, dv)).astype(np.float32), "f32")
    beta, gate = (to_device(rng.random(s).astype(np.float32), "f32") for s in ((H, F, N), (H,)))
    tail, splits = V.default_split_plan(F, N, H, dk, dv, is_f32=True)
    # (The partial round is one range per compute unit.)
    assert splits == min(ranges, torch.cuda.get_device_properties(0).multi_processor_count // (H * F))
    A, B = V.frame_stats(k, v, beta, splits=splits, tail_frames=tail)
    inv = V.frame_inverse(A, B, count=H * F, tail_frames=tail, splits=splits)
    sf, sr = V.state_scan(inv.view(H, F, dk, dk), B[:H * F].view(H, F, dv, dk), exact_f32=True)
    assert torch.equal(V.forward(q, k, v, beta, gate), V.readout(q, sf, sr, gate, d_v=dv))


# The whole pass with frames of three, six and eight ranges, against the oracle (the bar of the fp32 parity tests).
@pytest.mark.parametrize("N,ranges", [(400, 3), (1100, 6), (1536, 8)])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 32)])
def test_forward_ranges(V, N, ranges, dk, dv):
    H, F = 2, 3
    assert V.default_split_plan(F, N, H, dk, dv, is_f32=True) == (H * F, ranges)
    rng = np.random.default_rng(N + dk)
    q, k = ((x / np.linalg.norm(x, axis=-1, keepdims=True)).astype(np.float32)
            for x in (rng.standard_normal((H, F, N, dk)) for _ in range(2)))
    v = rng.standard_normal((H, F, N, dv)).astype(np.float32)
    beta, gate = (rng.random(s).astype(np.float32) for s in ((H, F, N), (H,)))
    y = V.forward(*(to_device(x, "f32") for x in (q, k, v, beta, gate))).double().cpu().numpy()
    ref = O.vda_forward(*(x.astype(np.float64) for x in (q, k, v, beta, gate)))
    assert rel_max_err(y, ref) <= TOL_F32


# Ranges are whole tiles of 64 tokens: with ceil(N / S) rounded up to them, S - 1 ranges may hold all N tokens (1025 and
# 1100 tokens in eight of 192).  The default plan has no range without tokens, and no more than the header states.
@pytest.mark.parametrize("is_f32,most,least", [(True, 8, 128), (False, 4, 256)])
def test_default_plan_ranges(V, is_f32, most, least):
    seen = set()
    for F, H, dk, dv in [(1, 1, 128, 128), (1, 16, 128, 128), (21, 4, 128, 128), (36, 16, 128, 128), (30, 6, 64, 64),
                         (64, 3, 64, 32)]:
        for N in list(range(1, 2600, 3)) + [512, 1000, 1024, 1100, 3840, 4032, 100001]:
            tail, splits = V.default_split_plan(F, N, H, dk, dv, is_f32=is_f32)
            seen.add(splits)
            if splits == 1:
                continue
            size = -(-(-(-N // splits)) // 64) * 64
            assert (splits - 1) * size < N and splits <= min(most, N // least) and 1 <= tail <= F * H, (F, H, dk, N)
    assert {1, 2, most} <= seen
