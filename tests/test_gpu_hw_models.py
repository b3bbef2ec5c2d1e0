"""Measures the hardware error models the certified fast paths rest on.

* v_exp_f32 (PAMA's and attention's exponentials): for an exactly known float
  argument x in PAMA's range, relative error <= 2^-23 (2 + 1.5 |x|) where the
  result is a normal float (the retrieval bound charges 1.5 |x| for the
  rounding of the argument it computes; the instruction alone is measured
  here), and at most FLT_MIN absolute below the normal range (the selection's
  absolute term).  PAMA's exponents reach 8 above the bias of its weights (at
  most 31), and at an integer the result is exact: its sums move between
  references by such powers of two without a rounding.
* v_mfma_f32_32x32x16_bf16 accumulation chains (k-means scores) and
  v_mfma_f32_32x32x16_f16 ones (PAMA scores): the bounds assume every addition errs by at most 2^-23 of the magnitudes
  involved, i.e. |C^ - C| <= (K + 1) 2^-23 (|C0| + sum_k |a_k b_k|) for a
  chain of K products started from C0.  PAMA's bound lets an f16 operand below
  the normal range count as zero; the test states what the card does with it.

The references are float64 (exp2 of the float argument; products of bf16
values are exact in float64 and summed with compensation)."""
import numpy as np
import pytest
import torch

from paper_2609_38978_amd import park as P
from paper_2609_38978_amd import synth

pytestmark = pytest.mark.gpu

FLT_MIN = float(np.finfo(np.float32).tiny)
U23 = 2.0 ** -23


def test_exp2_relative_error_model():
    rng = np.random.default_rng(0)
    x = np.concatenate([
        rng.uniform(-150.0, 8.0, 1 << 22).astype(np.float32),
        np.arange(-150, 9, dtype=np.float32),                     # integers
        np.nextafter(np.arange(-150, 9, dtype=np.float32), np.float32(np.inf)),
        np.nextafter(np.arange(-150, 9, dtype=np.float32), np.float32(-np.inf)),
        rng.uniform(-1e-3, 1e-3, 1 << 16).astype(np.float32),      # near zero
    ])
    y = P.park_probe_exp2(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    ref = np.exp2(x.astype(np.float64))
    normal = ref >= FLT_MIN
    rel = np.abs(y[normal] - ref[normal]) / ref[normal]
    bound = U23 * (2.0 + 1.5 * np.abs(x[normal].astype(np.float64)))
    worst_ulp = float((rel / U23).max())
    print(f"[exp2] {normal.sum()} normal results: worst relative error {worst_ulp:.3f} x 2^-23; "
          f"worst error / model bound {float((rel / bound).max()):.3g}")
    assert np.all(rel <= bound)
    sub = ~normal
    err_sub = np.abs(y[sub] - ref[sub])
    print(f"[exp2] {sub.sum()} subnormal results: worst absolute error {err_sub.max():.3g} "
          f"(FLT_MIN {FLT_MIN:.3g})")
    assert np.all(err_sub <= FLT_MIN)


def test_exp2_at_pama_exponents():
    rng = np.random.default_rng(1)
    x = rng.uniform(8.0, 40.0, 1 << 22).astype(np.float32)
    y = P.park_probe_exp2(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    ref = np.exp2(x.astype(np.float64))
    bound = U23 * (2.0 + 1.5 * x.astype(np.float64))
    rel = np.abs(y - ref) / ref
    print(f"[exp2] 8 .. 40: worst relative error {float((rel / U23).max()):.3f} x 2^-23")
    assert np.all(rel <= bound)
    n = np.arange(-126, 128, dtype=np.float32)
    y = P.park_probe_exp2(torch.from_numpy(n).cuda()).cpu().numpy()
    assert np.array_equal(y.astype(np.float64), np.exp2(n.astype(np.float64)))
    low = np.array([-127, -149, -1000, -1e30, -np.inf], np.float32)  # at most FLT_MIN
    y = P.park_probe_exp2(torch.from_numpy(low).cuda()).cpu().numpy()
    assert np.all((y >= 0.0) & (y <= FLT_MIN))


def _exact_chain(A, Bt, C0):
    """C0 + sum_k A[:, i, k] Bt[:, j, k] in float64 with Neumaier compensation,
    and sum_k |a_k b_k|."""
    A64, B64 = A.astype(np.float64), Bt.astype(np.float64)
    s = C0.astype(np.float64).copy()
    comp = np.zeros_like(s)
    mag = np.abs(s)
    for k in range(A.shape[2]):
        p = A64[:, :, k][:, :, None] * B64[:, :, k][:, None, :]  # exact products
        t = s + p
        comp += np.where(np.abs(s) >= np.abs(p), (s - t) + p, (p - t) + s)
        s = t
        mag = mag + np.abs(p)
    return s + comp, mag


def _bf16(a):
    return synth.bf16_round(np.asarray(a, np.float32))


@pytest.mark.parametrize("kind", ["random", "cancel", "wide", "on_top"])
@pytest.mark.parametrize("K", [128, 384])
def test_mfma_bf16_chain_error_model(kind, K):
    rng = np.random.default_rng(K + len(kind))
    Pn = 96
    if kind == "wide":  # products spread over 2^-24 .. 2^24
        A = rng.standard_normal((Pn, 32, K)) * 2.0 ** rng.integers(-12, 13, (Pn, 32, K))
        B = rng.standard_normal((Pn, 32, K)) * 2.0 ** rng.integers(-12, 13, (Pn, 32, K))
    else:
        A = rng.standard_normal((Pn, 32, K))
        B = rng.standard_normal((Pn, 32, K))
    A, B = _bf16(A), _bf16(B)
    if kind == "cancel":  # the second half cancels the first up to one small term
        h = K // 2
        A[:, :, h:] = -A[:, :, :h]
        B[:, :, h:] = B[:, :, :h]
        A[:, :, -1] = _bf16(A[:, :, -1] * 2.0 ** -10)
    C0 = np.zeros((Pn, 32, 32), np.float32)
    if kind == "on_top":  # a chain continued on an accumulator (the split-part chains)
        C0 = (rng.standard_normal((Pn, 32, 32)) * 4.0).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = P.park_probe_mfma_bf16(t(A).to(torch.bfloat16), t(B).to(torch.bfloat16),
                                 t(C0)).cpu().numpy().astype(np.float64)
    exact, mag = _exact_chain(A, B, C0)
    err = np.abs(got - exact)
    ratio = err / (U23 * mag)
    print(f"[mfma {kind} K={K}] worst error {float(ratio.max()):.3f} x 2^-23 (|C0| + sum|ab|); "
          f"model allows {K + 1}")
    assert np.all(err <= (K + 1) * U23 * mag)


def test_mfma_overflow_masks_scores():
    # attention masks a key by one bf16 MFMA before its score's chain: -3.39e38
    # (or 0) times 2^127 in the row's own column, every other column 0.  The
    # product must overflow to -inf, the zeros must not turn into NaN, and no
    # finite score may bring the sum back
    rng = np.random.default_rng(5)
    big = float(np.finfo(np.float32).max)
    A = np.zeros((4, 32, 32), np.float32)
    B = np.zeros((4, 32, 32), np.float32)
    masked = rng.random((4, 32, 16)) < 0.5
    A[:, :, :16] = np.where(masked, -(2.0 - 2.0 ** -7) * 2.0 ** 127, 0.0)
    own = rng.integers(0, 16, (4, 32))
    np.put_along_axis(B, own[:, :, None], 2.0 ** 127, axis=2)
    A[:, :, 16:] = _bf16(rng.standard_normal((4, 32, 16)) * 2.0 ** rng.integers(-60, 50, (4, 32, 16)))
    B[:, :, 16:] = _bf16(rng.standard_normal((4, 32, 16)) * 2.0 ** rng.integers(-60, 50, (4, 32, 16)))
    A[0, :, 31], B[0, :, 31] = 2.0 ** 64, (2.0 - 2.0 ** -7) * 2.0 ** 63  # next to FLT_MAX
    C0 = np.zeros((4, 32, 32), np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = P.park_probe_mfma_bf16(t(A).to(torch.bfloat16), t(B).to(torch.bfloat16),
                                 t(C0)).cpu().numpy().astype(np.float64)
    want = np.take_along_axis(masked, np.broadcast_to(own[:, None, :], (4, 32, 32)), axis=2)
    exact, mag = _exact_chain(A[:, :, 16:], B[:, :, 16:], C0)
    assert mag.max() <= big
    assert np.all(np.isneginf(got[want]))
    assert np.all(np.abs(got[~want] - exact[~want]) <= (17 * U23 * mag)[~want])


@pytest.mark.parametrize("kind", ["random", "cancel", "wide", "on_top", "split", "subnormal"])
@pytest.mark.parametrize("K", [32, 128, 384])
def test_mfma_f16_chain_error_model(kind, K):
    # operands as PAMA scales them: the largest element in [2^14, 2^15)
    rng = np.random.default_rng(K + len(kind))
    Pn = 96
    scale = lambda a: a * 2.0 ** (14 - np.floor(np.log2(np.abs(a).max((1, 2), keepdims=True))))
    f16 = lambda a: np.asarray(a, np.float32).astype(np.float16).astype(np.float32)
    A, B = (rng.standard_normal((Pn, 32, K)) for _ in range(2))
    if kind in ("wide", "subnormal"):  # down to the smallest normal, or below it
        low = -24 if kind == "wide" else -36
        A, B = (a * 2.0 ** rng.integers(low, 1, a.shape) for a in (A, B))
    A, B = scale(A), scale(B)
    if kind == "wide":
        A, B = (np.where(np.abs(a) < 2.0 ** -13, 2.0 ** -13, a) for a in (A, B))
    C0 = np.zeros((Pn, 32, 32), np.float32)
    if kind == "split":  # the second part of a float, 11 bits below the first
        B = B - B.astype(np.float16)
    if kind == "on_top":  # a chain continued on an accumulator of the second part's size
        C0 = (rng.standard_normal((Pn, 32, 32)) * 2.0 ** 20).astype(np.float32)
    A, B = f16(A), f16(B)
    if kind == "cancel":  # the second half cancels the first up to one small term
        h = K // 2
        A[:, :, h:] = -A[:, :, :h]
        B[:, :, h:] = B[:, :, :h]
        A[:, :, -1] = f16(A[:, :, -1] * 2.0 ** -10)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = P.park_probe_mfma_f16(t(A).half(), t(B).half(), t(C0)).cpu().numpy().astype(np.float64)
    exact, mag = _exact_chain(A, B, C0)
    err = np.abs(got - exact)
    model = (K + 1) * U23 * mag
    print(f"[mfma f16 {kind} K={K}] worst error {float((err / (U23 * mag)).max()):.3f} x 2^-23 "
          f"(|C0| + sum|ab|); model allows {K + 1}")
    # what may be lost: products of an operand below the smallest normal
    tiny = lambda a: np.where(np.abs(a) < 2.0 ** -14, np.abs(a), 0.0).astype(np.float64)
    A64, B64 = np.abs(A).astype(np.float64), np.abs(B).astype(np.float64)
    lost = tiny(A) @ B64.transpose(0, 2, 1) + A64 @ tiny(B).transpose(0, 2, 1)
    print(f"    without the allowance for subnormal operands: {bool(np.all(err <= model))}, "
          f"largest allowance {float((lost / mag).max()):.3g} of the magnitudes")
    assert np.all(err <= model + lost)
