"""fp32 caches scored as sums of six bf16 products under every option, against the oracle and to fp32 accuracy: the automatic choice,
which sends most of these calls to the direct kernels (those that stay with longer slices: test_gpu_score_split_large)."""
import math

import numpy as np
import pytest
import torch

from oracle import ccd_oracle as O
from paper_2410_01518_amd import infinipot as ip
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# (units, G, P, n, d, options).  Row blocks of 32 query rows: one, two, three, four, five to eight, more than 256 rows; one
# token, just around a tile of 32 and a stage of 64, several slices of 256; 260 units: more than places on the chip.
CASES = [
    (1, 1, 1, 1, 128, ""), (2, 1, 5, 31, 128, ""), (2, 1, 32, 33, 128, "lse"), (1, 1, 33, 64, 128, "kcat"),
    (2, 2, 40, 65, 128, "kcat"), (1, 3, 32, 255, 128, "window"), (1, 4, 32, 257, 128, "kcat window"),
    (2, 3, 43, 449, 128, "lse window"), (1, 2, 128, 1000, 128, "kcat window"), (3, 4, 64, 769, 128, ""),
    (1, 2, 129, 520, 128, "kcat"), (1, 8, 70, 333, 128, "window"), (1, 8, 64, 1409, 128, "lse"),
    (260, 1, 2, 700, 128, "kcat"), (260, 2, 3, 700, 128, "window"),
    (1, 1, 3, 7001, 64, ""), (2, 2, 20, 300, 64, "kcat"), (1, 4, 80, 515, 64, "kcat window"), (3, 1, 33, 130, 64, "window"),
    (260, 1, 2, 700, 64, "window"), (1, 1, 2100, 2600, 64, "window"),
]


@pytest.mark.parametrize("units,G,P,n,d,options", CASES)
def test_scores(units, G, P, n, d, options):
    rng = np.random.default_rng(units * n + G * P)
    Q = rng.standard_normal((1, 1, units * G, P, d)).astype(np.float32)
    K = rng.standard_normal((1, 1, units, n, d)).astype(np.float32)
    K[:, :, :, rng.integers(0, n, max(1, n // 50))] *= 4.0
    Kc = rng.standard_normal((1, 1, units, P, d)).astype(np.float32) if "kcat" in options else None
    window = max(P, n * 2 // 3) if "window" in options else 0
    lse = (3.0 + rng.random((1, 1, units * G, P))).astype(np.float32) if "lse" in options else None
    dK = gu.to_dev(K)
    shape = ip.make_shape(gu.to_dev(Q), dK, None, k=n, T=0, pool_w=1, window=window)
    ws = ip.alloc_workspace(shape)
    ws.fill_(0xFF)                                             # nothing relied on, and NaN where it is read too early
    scores = torch.empty((1, 1, units, n), dtype=torch.float32, device="cuda")
    print(f"split units={units} G={G} P={P} n={n} d={d} {options}", flush=True)
    if lse is not None:
        rc = ip.ccd_score_lse(shape, gu.to_dev(Q), dK, gu.to_dev(lse), None, scores, ws)
    elif Kc is not None:
        rc = ip.ccd_score_kcat(shape, gu.to_dev(Q), dK, gu.to_dev(Kc), None, scores, ws)
    else:
        rc = ip.ccd_score(shape, gu.to_dev(Q), dK, None, scores, ws)
    assert rc == ip.CCD_OK
    got = gu.to_host(scores).reshape(units, n).astype(np.float64)
    scale = 1.0 / math.sqrt(d)
    Qu, Ku = Q.reshape(units, G * P, d).astype(np.float64), K.reshape(units, n, d).astype(np.float64)
    for i in range(units):
        if lse is not None:
            ref = O.cap_scores_given_lse(Qu[i], Ku[i], scale, lse.reshape(units, -1)[i], P=P, window=window)
        else:
            ref = O.cap_scores(Qu[i], Ku[i], scale, K_cap=None if Kc is None else Kc[0, 0, i].astype(np.float64), P=P, window=window)
        _assert_close(got[i], ref, Qu[i], Ku[i], scale, i)


def _assert_close(got, ref, Q, K, scale, what, rounds=10):
    # A logit rounds at most ten times (eight additions of the large products, the small ones' sum, the scale), each by
    # 2^-24 of sum |q k| scale log2(e) at most; a probability carries that twice (logit and normaliser), times ln 2.
    # Behind that, 64 roundings of sums, exponentials and merges.
    size = (np.abs(Q) @ np.abs(K).T).max() * scale / math.log(2.0)
    bound = (2.0 * math.log(2.0) * rounds * size + 64.0) * 2.0 ** -24
    err = np.abs(got - ref)
    assert (err <= bound * ref + 2.0 * len(Q) * gu.FLT_MIN).all(), (what, float((err / np.maximum(ref, 1e-30)).max()), bound)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("units,G,P,n,d", [(2, 2, 5, 40, 128), (1, 3, 33, 129, 64), (1, 9, 32, 300, 128)])
def test_normaliser_of_a_row_that_sees_no_token(units, G, P, n, d, dtype):
    """window == P hides every cached token from the last CaP token of a head; its normaliser over the cached tokens is
    -inf.  It adds nothing to any score."""
    rng = np.random.default_rng(n)
    Q = rng.standard_normal((1, 1, units * G, P, d)).astype(np.float32)
    K = rng.standard_normal((1, 1, units, n, d)).astype(np.float32)
    if dtype == "bf16":
        Q, K = (O.round_bf16_bits(x) for x in (Q, K))
    scale = 1.0 / math.sqrt(d)
    Qu, Ku = O.to_f64(Q).reshape(units, G * P, d), O.to_f64(K).reshape(units, n, d)
    hidden = np.arange(n)[None, :] < (n + np.arange(G * P) % P + 1 - P)[:, None]
    with np.errstate(divide="ignore"):
        lse = np.stack([np.log(np.where(hidden, 0.0, np.exp(scale * Qu[i] @ Ku[i].T)).sum(1)) for i in range(units)])
    assert (np.isneginf(lse).sum(1) == G).all()
    lse = lse.astype(np.float32).reshape(1, 1, units * G, P)
    dQ, dK = gu.to_dev(Q), gu.to_dev(K)
    shape = ip.make_shape(dQ, dK, None, k=n, T=0, pool_w=1, window=P)
    ws = ip.alloc_workspace(shape)
    scores = torch.empty((1, 1, units, n), dtype=torch.float32, device="cuda")
    print(f"no token seen: {dtype} units={units} G={G} P={P} n={n} d={d}", flush=True)
    assert ip.ccd_score_lse(shape, dQ, dK, gu.to_dev(lse), None, scores, ws) == ip.CCD_OK
    got = gu.to_host(scores).reshape(units, n).astype(np.float64)
    for i in range(units):
        rows = np.isfinite(lse.reshape(units, -1)[i])
        A = np.exp(scale * Qu[i][rows] @ Ku[i].T - lse.reshape(units, -1)[i][rows, None].astype(np.float64))
        ref = np.where(hidden[rows], 0.0, A).sum(0)
        assert (got[i][: n - P + 1] == 0.0).all()
        _assert_close(got[i], ref, Qu[i], Ku[i], scale, i)


@pytest.mark.parametrize("kind", ["large keys", "large queries", "infinite keys"])
@pytest.mark.parametrize("units,G,P,n,d,options", [(2, 2, 5, 40, 128, ""), (1, 5, 60, 700, 128, "kcat"), (1, 2, 33, 300, 64, "kcat window"),
                                                   (2, 1, 20, 333, 128, "lse window"), (1, 4, 64, 520, 128, "window")])
def test_elements_beyond_the_largest_bf16(units, G, P, n, d, options, kind):
    """A finite element above the largest bf16 counts with its value (the elements it meets are small: moderate logits); an
    infinite one that takes a token's logits to -inf leaves that token a score of zero and the others theirs."""
    rng = np.random.default_rng(units * n + d)
    Q = rng.standard_normal((1, 1, units * G, P, d)).astype(np.float32)
    K = rng.standard_normal((1, 1, units, n, d)).astype(np.float32)
    Kc = rng.standard_normal((1, 1, units, P, d)).astype(np.float32) if "kcat" in options else None
    tokens, col, big, small = rng.integers(0, n, 5), 7, np.float32(3.4e38), lambda m: (1.2e-38 * (1.0 + 3.0 * rng.random(m))).astype(np.float32)
    if kind == "large queries":
        K[..., col] = small(K.shape[:-1])
        Q[0, 0, :, P // 2, col] = big
        if Kc is not None:
            Kc[..., col] = small(Kc.shape[:-1])
    else:
        Q[..., col] = small(Q.shape[:-1])
        K[0, 0, :, tokens, col] = -np.inf if kind == "infinite keys" else big
        if Kc is not None and kind == "large keys":
            Kc[0, 0, :, P // 3, col] = big
    window = max(P, n * 2 // 3) if "window" in options else 0
    lse = (3.0 + rng.random((1, 1, units * G, P))).astype(np.float32) if "lse" in options else None
    dQ, dK = gu.to_dev(Q), gu.to_dev(K)
    shape = ip.make_shape(dQ, dK, None, k=n, T=0, pool_w=1, window=window)
    ws = ip.alloc_workspace(shape)
    scores = torch.empty((1, 1, units, n), dtype=torch.float32, device="cuda")
    print(f"{kind}: units={units} G={G} P={P} n={n} d={d} {options}", flush=True)
    if lse is not None:
        ip.ccd_score_lse(shape, dQ, dK, gu.to_dev(lse), None, scores, ws)
    elif Kc is not None:
        ip.ccd_score_kcat(shape, dQ, dK, gu.to_dev(Kc), None, scores, ws)
    else:
        ip.ccd_score(shape, dQ, dK, None, scores, ws)
    got = gu.to_host(scores).reshape(units, n).astype(np.float64)
    scale = 1.0 / math.sqrt(d)
    Qu, Ku = Q.reshape(units, G * P, d).astype(np.float64), K.reshape(units, n, d).astype(np.float64)
    for i in range(units):
        if lse is not None:
            ref = O.cap_scores_given_lse(Qu[i], Ku[i], scale, lse.reshape(units, -1)[i], P=P, window=window)
        else:
            ref = O.cap_scores(Qu[i], Ku[i], scale, K_cap=None if Kc is None else Kc[0, 0, i].astype(np.float64), P=P, window=window)
        fin = np.where(np.isinf(Ku[i]), 0.0, Ku[i])
        _assert_close(got[i], ref, Qu[i], fin, scale, i, rounds=d + 2)      # a chain of d fmas, and the scale
        if kind == "infinite keys":
            assert (got[i][tokens] == 0.0).all()


# window == P: the last CaP token of a head sees no cached token, the one before it only the last; one token in all; a call with too many
# blocks of tokens and query rows for the direct kernels
@pytest.mark.parametrize("units,G,P,n,d,window,infinite", [
    (2, 2, 5, 40, 128, 5, 1), (1, 3, 33, 300, 64, 33, 1), (3, 1, 20, 333, 128, 24, 6), (1, 1, 1, 1, 64, 0, 1), (2, 4, 16, 96, 128, 0, 96),
    (12, 8, 128, 700, 128, 128, 1)])
def test_a_row_none_of_whose_visible_keys_is_finite_adds_nothing(units, G, P, n, d, window, infinite):
    """The last `infinite` tokens take every logit to -inf: a row that sees only such tokens has no weight to give, and the scores of
    the others are what they are without it."""
    rng = np.random.default_rng(units * n + P)
    Q = rng.standard_normal((1, 1, units * G, P, d)).astype(np.float32)
    K = rng.standard_normal((1, 1, units, n, d)).astype(np.float32)
    Q[..., 7] = np.abs(Q[..., 7]) + np.float32(0.1)
    K[0, 0, :, n - infinite:, 7] = -np.inf
    dQ, dK = gu.to_dev(Q), gu.to_dev(K)
    shape = ip.make_shape(dQ, dK, None, k=n, T=0, pool_w=1, window=window)
    ws = ip.alloc_workspace(shape)
    scores = torch.empty((1, 1, units, n), dtype=torch.float32, device="cuda")
    print(f"rows without a finite key: units={units} G={G} P={P} n={n} d={d} window={window}", flush=True)
    assert ip.ccd_score(shape, dQ, dK, None, scores, ws) == ip.CCD_OK
    got = gu.to_host(scores).reshape(units, n).astype(np.float64)
    scale = 1.0 / math.sqrt(d)
    Qu, Ku = Q.reshape(units, G * P, d).astype(np.float64), K.reshape(units, n, d).astype(np.float64)
    for i in range(units):
        ref = O.cap_scores(Qu[i], Ku[i], scale, P=P, window=window)
        assert (got[i][n - infinite:] == 0.0).all()
        _assert_close(got[i], ref, Qu[i], np.where(np.isinf(Ku[i]), 0.0, Ku[i]), scale, i, rounds=d + 2)
