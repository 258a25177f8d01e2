"""GPU parity at the sizes where a kernel's tiles, masks and dispatch rules
change: each case is small and compared with the oracle at the same bars as
the stage and end-to-end parity tests."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from gpu_harness import SMALL, inputs, log, problem_of, to_device
from oracle import pipeline
from paper_2609_32628_amd import api
from test_gpu_parity import _check_end_to_end, _gpu, _run_gpu  # noqa: F401  (_gpu: module fixture)
from test_gpu_parity import test_draft_map_row_lengths as _check_draft_map, test_prep_operands as _check_operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("fmt4", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("n", [1, 4, 15, 16, 17, 31, 32, 33, 48, 49, 63])
def test_partial_block_masks(n, fmt4, d):
    """Three one-block frames of n tokens, one 16-bit, one 8-bit and one 4-bit
    key block per row: every phase masks the padding slots from n on, at both
    lane halves and both logit tiles."""
    w = replace(SMALL, name=f"mask-{n}-{fmt4}-d{d}", B=1, H=2, d=d, T=3, Hg=1, Wg=n, partition="ragged", scope="row",
                num16=34, budgets=(33, 33, 100), fmt4=fmt4)
    _check_end_to_end(w, *inputs(w))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("R", [1, 15, 17, 64, 65, 128, 129, 256, 257])
def test_draft_map_short_rows(R, d):
    """R one-block frames: the edges of the short-row kernel's column tiles and
    the first length that takes the tiled kernel."""
    _check_draft_map(replace(SMALL, name=f"draft-R{R}-d{d}", B=1, H=2, d=d, T=R, Hg=7, Wg=8))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("R,H", [(1, 2), (17, 2), (65, 2), (128, 2), (129, 2), (256, 2), (257, 2), (48, 172),
                                 (49, 128), (49, 129), (241, 16), (241, 17)])
def test_draft_workspace_holds_the_logits(R, H, d):
    """S_avg and S_max of da2_ws_draft_offsets are the logits of the pooled
    descriptors beside them, for both kernels: their row lengths and the numbers
    of workgroups at which one takes over from the other."""
    w = replace(SMALL, name=f"draft-ws-R{R}-h{H}-d{d}", B=1, H=H, d=d, T=R, Hg=1, Wg=3)
    Q, K, _ = inputs(w)
    p = problem_of(w)
    buf = api.alloc(p, w.scope)
    buf.ws_draft.fill_(0xA5)
    api.da2_draft_map(to_device(Q, w), to_device(K, w), buf.layout, p, w.lam, buf.A, buf.stats, buf.ws_draft)
    torch.cuda.synchronize()
    ws, off = buf.ws_draft.cpu().numpy(), api.da2_ws_draft_offsets(p)
    at = [ws[off[i]:off[i] + 8 * H * R * n].view(np.float64).reshape(H, R, n) for i, n in enumerate([d] * 4 + [R] * 2)]
    for i in (0, 1):   # average and maximum pooling
        q, k, S = at[i], at[2 + i].transpose(0, 2, 1), at[4 + i]
        # float64 sums of d products in any order, scaled by a rounded 1 / sqrt d
        bound = (d + 4) * 2.0 ** -53 * (np.abs(q) @ np.abs(k)) / np.sqrt(d)
        assert (np.abs(S - q @ k / np.sqrt(d)) <= 2 * bound).all()
    # and the map is their softmaxes' mixture
    e = [np.exp(S - S.max(axis=2, keepdims=True)) for S in at[4:]]
    A = (1 - w.lam) * e[0] / e[0].sum(axis=2, keepdims=True) + w.lam * e[1] / e[1].sum(axis=2, keepdims=True)
    np.testing.assert_allclose(buf.A.cpu().numpy()[0], A, rtol=2.0 ** -23, atol=1e-37)


@pytest.mark.parametrize("dtype,d,n", [("fp32", 128, 2048), ("fp32", 128, 2049), ("fp32", 64, 4096), ("fp32", 64, 4097),
                                       ("bf16", 128, 4096), ("bf16", 128, 4097), ("bf16", 64, 1), ("bf16", 64, 1025)])
def test_value_statistics_split(dtype, d, n):
    """Heads whose V has up to 1 MiB take their channel maxima inside the Q/K
    launch, larger ones in launches of their own: both sides of the limit, one
    token, and one token beyond a whole round of loads."""
    _check_operands(replace(SMALL, name=f"vstats-{dtype}-d{d}-n{n}", B=1, H=2, d=d, T=1, Hg=1, Wg=n, dtype=dtype,
                            partition="ragged"))


@pytest.mark.parametrize("dtype,n,H", [("bf16", 2048, 42), ("bf16", 2048, 43), ("fp32", 4096, 34), ("fp32", 4096, 35)])
def test_value_statistics_split_by_heads(dtype, n, H):
    """The numbers of heads from which narrow rows (d = 64) leave the Q/K launch."""
    _check_operands(replace(SMALL, name=f"vstats-{dtype}-h{H}", B=1, H=H, d=64, T=1, Hg=1, Wg=n, dtype=dtype,
                            partition="ragged"))


@pytest.mark.parametrize("B,H,T", [(1, 1, 1), (1, 1, 9), (1, 2, 5), (1, 3, 7), (1, 5, 11), (1, 7, 4), (3, 3, 13)])
def test_rows_dealt_to_xcds(B, H, T):
    """Head counts whose half-heads the eight segments of the work order cut in
    none, two or more parts: every row is computed."""
    w = replace(SMALL, name=f"deal-{B}x{H}x{T}", B=B, H=H, T=T, Hg=8, Wg=8, scope="head")
    _check_end_to_end(w, *inputs(w))


# Relative error of an output whose key logits are all equal. 4-bit pairs: the
# float32 exponent of a weight may be off by an ulp of the running maximum (half
# of it from the maximum, half from the fused offset), and the denominator sums
# what the quantizer then saturates. 8-bit pairs: weight and denominator share
# that error, and the weight, 448 less up to three such ulps (2^-8 at 2^25), is
# rounded to a normal E4M3 value.
def _equal_logits_bound(w, value):
    x = np.float32(value * value * np.sqrt(w.d) * np.log2(np.e))
    return (2.0 ** float(np.spacing(x)) - 1.0 if w.budgets[1] else 2.0 ** -4) + 5e-3


def _check_equal_logits(w, value, sign=1):
    Q, K, V = inputs(w)
    Q, K = np.full_like(Q, value), np.full_like(K, sign * value)
    O = _run_gpu(w, Q, K, V)[2].cpu().numpy().reshape(w.H, w.N, w.d)
    _, outs = pipeline.run(w, Q, K, V)
    for h, o in enumerate(outs):
        assert np.isfinite(O[h]).all(), (h, np.isnan(O[h]).any(axis=-1).sum())
        rel = np.abs(O[h] - o["O"]).max() / np.abs(o["O"]).max()
        log(f"  head {h}: rel {rel:.2e}, bound {_equal_logits_bound(w, value):.2e}")
        assert rel <= _equal_logits_bound(w, value)


@pytest.mark.parametrize("d,value", [(64, 344.0), (64, 500.0), (128, 250.0), (128, 344.0), (128, 352.0)])
def test_large_equal_logits_nvfp4(d, value):
    """Constant Q and K whose logits reach 2^20 in log2 units: a group's scaled
    maximum may pass the largest E4M3 value and has to saturate, not to become
    NaN."""
    _check_equal_logits(replace(SMALL, name=f"equal-{value:g}-d{d}", B=1, d=d, budgets=(0, 100, 100), scope="row"), value)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("d,value", [(64, 250.0), (64, 1000.0), (64, 2000.0), (128, 215.0), (128, 500.0),
                                     (128, 1000.0), (128, 1600.0)])
def test_large_equal_logits_int8(d, value, sign):
    """The same for 8-bit weights, of which the largest may pass 464; logits of
    either sign."""
    w = replace(SMALL, name=f"equal8-{value:g}-d{d}", B=1, d=d, budgets=(100, 0, 100), scope="row")
    _check_equal_logits(w, value, sign)


@pytest.mark.parametrize("fmt4,budgets", [("nvfp4", (0, 100, 100)), ("mxfp4", (0, 100, 100)), ("nvfp4", (100, 0, 100)),
                                          ("nvfp4", (30, 70, 100)), ("mxfp4", (30, 70, 100))])
@pytest.mark.parametrize("scale", [200.0, 400.0, 800.0, 3000.0])
def test_large_logits_stay_finite(scale, fmt4, budgets):
    """Different logits of up to 2^28 in log2 units, each phase and both."""
    w = replace(SMALL, name=f"large-{scale:g}-{fmt4}", B=1, fmt4=fmt4, budgets=budgets, scope="row")
    rng = np.random.default_rng(5)
    Q, K, V = inputs(w)
    Q = (scale * (1 + rng.standard_normal(Q.shape))).astype(Q.dtype)
    K = (scale * (1 + 0.01 * rng.standard_normal(K.shape))).astype(K.dtype)
    assert torch.isfinite(_run_gpu(w, Q, K, V)[2]).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_queries_beyond_half_precision(d, dtype):
    """Queries with a value of -70,144 (infinite in fp16) in a channel where
    every key is positive: their 16-bit logits are -inf, on partial blocks too,
    and the 4-bit and 8-bit pairs alone make the output."""
    w = replace(SMALL, name=f"half-inf-{dtype}-d{d}", B=1, d=d, dtype=dtype, num16=30, budgets=(30, 40, 100),
                scope="row")
    Q, K, V = inputs(w)
    Q[:, :, ::7, 0] = -70144.0
    K[..., 0] = 2.0 ** -6
    _check_end_to_end(w, Q, K, V)
