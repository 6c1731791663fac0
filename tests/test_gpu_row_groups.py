"""GPU parity of the unit kernel with its waves side by side over row groups (units of more than 256 query rows), at the edges of the
groups, of the parts of the tokens and of the blocks of token sums; scores against the fp64 oracle at the suite's 1e-3."""
import numpy as np
import pytest
import torch

from oracle import ccd_oracle as O
from paper_2410_01518_amd import infinipot as ip
from paper_2410_01518_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(units, N, G, P, d, dtype="bf16", option="", window=0, gains=None):
    print(f"row groups {units} {N} {G} {P} {d} {dtype} {option} {window} {gains}", flush=True)
    cfg = synth.CCDConfig("t", 1, units, G, 1, d, N, max(1, N // 3), P, N // 8, 5, dtype, "normal", N + P)
    inp = synth.make_inputs(cfg)
    for start, gain in gains or []:          # keys from a token on, so many times as long
        K = gu.to_dev(inp["K"])
        K[:, :, :, start:] *= gain
        inp["K"] = gu.to_host(K)
    K_cap = synth.cap_keys(cfg) if option == "kcat" else None
    given = np.random.default_rng(5).normal(6.0, 0.5, (1, units, G, P)).astype(np.float32) if option == "lse" else None
    dev = {k: gu.to_dev(v) for k, v in inp.items()}
    shape = ip.make_shape(dev["Q_cat"], dev["K"], dev["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, window=window,
                          score_path=ip.CCD_PATH_MFMA_UNIT)
    ws = ip.alloc_workspace(shape)
    ws.fill_(0xFF)
    scores = torch.empty((1, units, 1, N), dtype=torch.float32, device="cuda")
    call = {"": lambda: ip.ccd_score(shape, dev["Q_cat"], dev["K"], dev["novelty"], scores, ws),
            "kcat": lambda: ip.ccd_score_kcat(shape, dev["Q_cat"], dev["K"], gu.to_dev(K_cap), dev["novelty"], scores, ws),
            "lse": lambda: ip.ccd_score_lse(shape, dev["Q_cat"], dev["K"], gu.to_dev(given), dev["novelty"], scores, ws)}[option]
    stages = gu.stages_run(call)
    assert "score_unit" in stages
    ref = O.compress(inp["Q_cat"], inp["K"], inp["V"], inp["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, K_cap=K_cap,
                     window=window, lse=given)
    if gains and dtype == "fp32":
        # three products leave 2^-16 of sum |q k|, here up to 64 times 8 E|q| E|k| 1.44 = 500 binary orders of logit: 5e-3, and what a token's
        # own normaliser is off by as much again; 5e-2 as for the single-group kernel
        got, want = gu.to_host(scores), ref["scores"]
        assert np.array_equal(np.isposinf(got), np.isposinf(want))
        np.testing.assert_allclose(got[np.isfinite(want)], want[np.isfinite(want)], rtol=5e-2, atol=2 * G * P * gu.FLT_MIN)
        return stages
    gu.assert_scores_close(gu.to_host(scores), ref["scores"], G * P)
    return stages


# rows: one over a sweep of 256, a sweep of 384 / 512 / 768 / 1024 one short, whole and one over, three sweeps of 384, five of 256;
# tokens: less than a tile, one short of and one over a tile per part, blocks of 128 tiles with one tile over in one part or in all
@pytest.mark.parametrize("units,N,G,P,d,dtype", [
    (3, 1, 1, 257, 128, "bf16"), (2, 31, 3, 128, 64, "bf16"), (2, 65, 5, 77, 128, "bf16"), (2, 8225, 2, 192, 128, "bf16"), (1, 8192, 8, 64, 64, "bf16"),
    (2, 127, 3, 171, 128, "bf16"), (1, 4129, 6, 128, 64, "bf16"), (2, 4096, 6, 127, 128, "bf16"), (2, 33, 1, 769, 128, "bf16"),
    (2, 4127, 8, 128, 128, "bf16"), (2, 129, 8, 128, 64, "bf16"), (1, 333, 5, 205, 128, "bf16"), (1, 160, 5, 256, 128, "bf16"),
    (2, 100, 3, 86, 64, "fp32"), (2, 8225, 8, 64, 64, "fp32"), (1, 4129, 3, 255, 64, "fp32"), (2, 64, 8, 128, 64, "fp32"), (1, 4100, 9, 129, 64, "fp32")])
def test_edges_of_groups_parts_and_blocks(units, N, G, P, d, dtype):
    _check(units, N, G, P, d, dtype)


@pytest.mark.parametrize("N,G,P,d", [(95, 4, 65, 128), (300, 3, 200, 64), (200, 4, 256, 128), (70, 5, 205, 128)])
@pytest.mark.parametrize("option", ["kcat", "lse"])
def test_cap_keys_and_given_normalisers(N, G, P, d, option):
    _check(2, N, G, P, d, option=option)


# heads of 96 and 128 tokens inside the kernel, of 64 and 160 by kernels of their own; the last row that sees nothing
@pytest.mark.parametrize("option", ["", "kcat", "lse"])
@pytest.mark.parametrize("N,G,P,d,window", [
    (400, 4, 90, 128, 400), (301, 8, 48, 64, 230), (500, 8, 128, 128, 500), (500, 8, 128, 128, 480), (333, 8, 64, 128, 333),
    (100, 10, 75, 64, 75)])
def test_windows(N, G, P, d, window, option):
    _check(2, N, G, P, d, option=option, window=window)


# two sweeps of 768 and of 1024 rows, the last one partly filled: token sums of several sweeps and several groups
@pytest.mark.parametrize("N,G,P,d,dtype,option", [(*case, option) for case in [
    (1, 13, 100, 128, "bf16"), (333, 13, 100, 128, "bf16"), (4129, 10, 130, 64, "bf16"), (255, 16, 96, 64, "bf16"), (161, 16, 125, 128, "bf16"),
    (4100, 15, 129, 64, "bf16"), (200, 16, 128, 128, "bf16"), (333, 13, 100, 64, "fp32"), (4129, 16, 125, 64, "fp32")]
    for option in (["", "kcat", "lse"] if case[4] == "bf16" else ["", "lse"])])        # (CaP keys of fp32 caches go to other kernels)
def test_several_sweeps_of_row_groups(N, G, P, d, dtype, option):
    _check(2, N, G, P, d, dtype, option)


# windowed heads over several sweeps, of 384 (1025, 1026 and 1152 rows), 256 (1280), 768 (1300) and 1024 rows (2000): of 64 tokens, by kernels of
# their own, and of 96 and 128 tokens inside
@pytest.mark.parametrize("option", ["", "kcat", "lse"])
@pytest.mark.parametrize("G,P,d,apart", [
    (25, 41, 128, True), (9, 114, 64, False), (12, 96, 128, False), (20, 64, 64, True), (10, 128, 128, False), (26, 50, 64, True), (20, 65, 128, False),
    (13, 100, 64, False), (40, 50, 128, True), (16, 125, 64, False), (25, 80, 128, False)])
def test_windowed_heads_over_several_sweeps(G, P, d, apart, option):
    for N, window in ((301, 301), (160, 140)):
        stages = _check(2, N, G, P, d, option=option, window=window)
        if window == N:
            assert ("window_head" in stages) == apart


# logits that leave the range of the first tile's reference in the first run of a part, in a later one, in its last or ragged tile; and where
# some parts do and others do not
@pytest.mark.parametrize("N,gains", [(1000, [(40, 64.0)]), (4130, [(64, 8.0), (600, 16.0)]), (4129, [(2200, 64.0)]), (1040, [(1010, 64.0)]), (515, [(512, 64.0)])])
@pytest.mark.parametrize("G,P,d,dtype", [(4, 128, 128, "bf16"), (8, 128, 64, "bf16"), (6, 128, 64, "fp32")])
def test_sums_that_leave_the_range(N, gains, G, P, d, dtype):
    _check(2, N, G, P, d, dtype, gains=gains)


@pytest.mark.parametrize("G,P,dtype", [(8, 32, "bf16"), (8, 48, "bf16"), (8, 64, "bf16"), (8, 96, "bf16"), (8, 128, "bf16"), (8, 64, "fp32"), (8, 128, "fp32")])
def test_the_normaliser_of_many_rows_is_as_close_as_that_of_few(G, P, dtype):
    """All query rows of a unit are one row (a sum of three key elements, in log2 units), so a token's score is G P times one
    probability, and what the scores of a unit have in common against fp64 is the error of its normaliser.
    Bound, from three parts.  With the tokens in four parts a sum is made of 16 chains (parts, lane halves, two per lane) of m = n / 16 additions; a
    chain's rms error is 0.72 x 2^-24 sqrt(m) / 3 (0.72: the mean of ulp / 2 over a binade), their sum's a quarter of it: 1.6e-7.  The
    log2-sum-exp is between 8 and 16, a number of 2^-20 steps: ln 2 x 2^-20 / sqrt(12) = 1.9e-7.  The merges add eight times, 2^-24 sqrt(8 / 3), and
    take exp2 and log2, good to an ulp: 1.2e-7 together.  In all 2.8e-7; the rms over 128 units has a standard deviation of 6 %, and the
    bound leaves 40 %.  (One chain per lane over two parts or the whole row: 4.7e-7 and 9.4e-7.)"""
    units, n, d = 128, 32768, 64
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    print(f"normalisers G={G} P={P} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(G * P)
    K = torch.zeros((1, units, 1, n, d), dtype=dt, device="cuda")
    K[..., :2] = (torch.randn((1, units, 1, n, 2), generator=g, device="cuda") * 0.5).bfloat16()
    K[..., 2] = (-4.0 * torch.rand((1, units, 1, 1), generator=g, device="cuda")).bfloat16()        # (the log2-sum-exps: 11.2 to 15.2)
    Q = torch.zeros((1, units, G, P, d), dtype=dt, device="cuda")
    Q[..., :3] = 1.0
    nov = torch.zeros((1, n), device="cuda")
    shape = ip.make_shape(Q, K, nov, k=1, T=0, pool_w=1, scale=float(np.log(2.0)), score_path=ip.CCD_PATH_MFMA_UNIT)
    scores = torch.empty((1, units, 1, n), dtype=torch.float32, device="cuda")
    assert "score_unit" in gu.stages_run(lambda: ip.ccd_score(shape, Q, K, nov, scores, ip.alloc_workspace(shape)))
    x = K[0, :, 0, :, :3].double().sum(-1) * np.log(2.0)
    ref = G * P * torch.exp(x - torch.logsumexp(x, -1, keepdim=True))
    err = (scores[0, :, 0].double() / ref - 1.0).mean(-1)
    rms = float(err.square().mean().sqrt())
    print(f"rms {rms:.2e} max {float(err.abs().max()):.2e}", flush=True)
    assert rms < 1.4 * np.sqrt((0.72 * 2.0**-24 * np.sqrt(n / 16) / 12) ** 2 + (np.log(2.0) * 2.0**-20) ** 2 / 12 + 1.2e-7**2)
