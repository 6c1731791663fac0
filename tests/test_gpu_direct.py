"""GPU parity of the score kernels for calls that do not fill the chip (ccd_score_direct.hip), at the edges of their tiles, row
blocks and slices, and on either side of the rules that lead there; scores against the fp64 oracle at the suite's 1e-3."""
import numpy as np
import pytest
import torch

from oracle import ccd_oracle as O
from paper_2410_01518_amd import infinipot as ip
from paper_2410_01518_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(cfg, *, window=0, kcat=False, lse=False):
    print(f"direct {cfg} window={window} kcat={kcat} lse={lse}", flush=True)
    inp = synth.make_inputs(cfg)
    K_cap = synth.cap_keys(cfg) if kcat else None
    dev = {k: gu.to_dev(v) for k, v in inp.items()}
    shape = ip.make_shape(dev["Q_cat"], dev["K"], dev["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, window=window)
    ws = ip.alloc_workspace(shape)
    ws.fill_(0xFF)                                        # nothing in it may have to start at zero
    scores = torch.empty((cfg.B, cfg.L, cfg.Hkv, cfg.N), dtype=torch.float32, device="cuda")
    given = None
    if lse:
        given = np.random.default_rng(5).normal(6.0, 0.5, (cfg.B, cfg.L, cfg.Hq, cfg.P)).astype(np.float32)
        rc = ip.ccd_score_lse(shape, dev["Q_cat"], dev["K"], gu.to_dev(given), dev["novelty"], scores, ws)
    elif kcat:
        rc = ip.ccd_score_kcat(shape, dev["Q_cat"], dev["K"], gu.to_dev(K_cap), dev["novelty"], scores, ws)
    else:
        rc = ip.ccd_score(shape, dev["Q_cat"], dev["K"], dev["novelty"], scores, ws)
    assert rc == ip.CCD_OK
    torch.cuda.synchronize()
    ref = O.compress(inp["Q_cat"], inp["K"], inp["V"], inp["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, K_cap=K_cap,
                     window=window, lse=given)
    gu.assert_scores_close(gu.to_host(scores), ref["scores"], cfg.G * cfg.P)


def _cfg(units, N, G, P, d, **kw):
    base = dict(name="t", B=1, L=units, Hq=G, Hkv=1, d=d, N=N, k=max(1, N // 3), P=P, T=N // 8, w=5, dtype="bf16", keys="normal", seed=N + P)
    base.update(kw)
    return synth.CCDConfig(**base)


# (units, tokens, heads per unit, CaP tokens, head dimension): one row, one token; tiles, row blocks (64), sweeps (256) and slices
# (256 in pass 1; 64, 128 or 256 in pass 2) one short, whole, one over; row counts that the slice kernels would waste or fill
@pytest.mark.parametrize("units,N,G,P,d", [
    (1, 1, 1, 1, 128), (1, 33, 1, 1, 64), (3, 255, 1, 63, 128), (9, 256, 1, 64, 64), (7, 257, 1, 65, 128), (5, 63, 2, 64, 128),
    (2, 513, 3, 43, 64), (2, 129, 3, 64, 128), (3, 385, 4, 48, 64), (2, 449, 4, 49, 128), (4, 320, 4, 64, 64), (3, 191, 1, 257, 128),
    (2, 300, 8, 40, 128), (3, 96, 9, 64, 64), (17, 512, 4, 64, 128)])
def test_edges_of_tiles_blocks_and_slices(units, N, G, P, d):
    _check(_cfg(units, N, G, P, d))


# slices of several batches of tiles in either pass (fp32 rows of 128 elements: a batch is one tile a wave); fp32 with one block of 32
# rows (whatever the number of tokens) and with two
@pytest.mark.parametrize("units,N,G,P,d,dtype", [
    (40, 4500, 1, 8, 64, "bf16"), (40, 8200, 1, 8, 64, "bf16"), (41, 2100, 2, 40, 128, "bf16"), (80, 1601, 4, 64, 64, "bf16"),
    (40, 4500, 1, 8, 64, "fp32"), (41, 2100, 1, 32, 128, "fp32"), (30, 2100, 1, 33, 128, "fp32"), (20, 1601, 2, 48, 64, "fp32")])
def test_long_slices(units, N, G, P, d, dtype):
    _check(_cfg(units, N, G, P, d, dtype=dtype))


@pytest.mark.parametrize("kcat", [False, True])
@pytest.mark.parametrize("units,N,G,P,d,window", [
    (3, 300, 1, 20, 64, 20),        # the last CaP token sees nothing
    (2, 700, 4, 33, 128, 700), (5, 1100, 2, 64, 128, 500), (2, 600, 5, 64, 64, 610),
    (36, 2500, 1, 16, 64, 1200)])   # whole slices that nobody sees
def test_windows(units, N, G, P, d, window, kcat):
    _check(_cfg(units, N, G, P, d), window=window, kcat=kcat)


@pytest.mark.parametrize("units,N,G,P,d,window", [(3, 257, 1, 65, 128, 0), (7, 500, 4, 60, 64, 0), (4, 333, 2, 64, 128, 200)])
def test_given_normalisers(units, N, G, P, d, window):
    _check(_cfg(units, N, G, P, d), window=window, lse=True)


# Calls on either side of the rule that sends them to the direct kernels.  bf16: the scores of the slice kernels, which can be named,
# bit for bit or not.  fp32: the six-product kernels by longer slices have a merge kernel, the direct ones have none.
@pytest.mark.parametrize("units,N,G,P,d,dtype,option,direct", [
    (8, 2048, 4, 64, 128, "bf16", "", True), (64, 2560, 4, 64, 128, "bf16", "", True), (12, 20000, 4, 25, 128, "bf16", "", True),
    (64, 2048, 4, 64, 128, "bf16", "", False), (64, 1024, 4, 64, 128, "bf16", "lse", False), (64, 4096, 4, 64, 64, "bf16", "", False),
    (128, 1024, 3, 44, 128, "bf16", "", False), (110, 1024, 4, 50, 128, "bf16", "kcat", False),
    (280, 250, 4, 64, 128, "bf16", "", False), (264, 256, 1, 80, 64, "bf16", "kcat", False), (300, 500, 2, 64, 128, "bf16", "lse", False),
    (4, 820, 4, 25, 128, "fp32", "", True), (4, 12000, 4, 40, 64, "fp32", "", True), (256, 700, 1, 2, 128, "fp32", "kcat", True),
    (48, 1024, 4, 40, 128, "fp32", "", False), (120, 256, 4, 50, 128, "fp32", "kcat", False), (87, 376, 4, 42, 64, "fp32", "kcat", False)])
def test_calls_that_the_direct_kernels_take(units, N, G, P, d, dtype, option, direct):
    print(f"route {units} {N} {G} {P} {d} {dtype} {option}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(units + N)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, K_cap = (torch.empty((1, units, h, m, d), dtype=dt, device="cuda").normal_(generator=g) for h, m in ((G, P), (1, N), (1, P)))
    lse = torch.full((1, units, G, P), 8.0, device="cuda")

    def run(path):
        shape = ip.make_shape(Q, K, None, k=N, score_path=path)
        scores, ws = torch.empty((1, units, 1, N), device="cuda"), ip.alloc_workspace(shape)
        call = {"": lambda: ip.ccd_score(shape, Q, K, None, scores, ws), "lse": lambda: ip.ccd_score_lse(shape, Q, K, lse, None, scores, ws),
                "kcat": lambda: ip.ccd_score_kcat(shape, Q, K, K_cap, None, scores, ws)}[option]
        return gu.stages_run(call), scores

    stages, scores = run(ip.CCD_PATH_AUTO)
    assert "score_prob" in stages and "score_unit" not in stages
    if dtype == "fp32":
        assert ("score_merge" in stages) == (not direct)
    else:
        assert torch.equal(scores, run(ip.CCD_PATH_MFMA_SLICES)[1]) == (not direct)
