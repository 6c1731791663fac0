"""Calls with a few more units than whole rounds of the chip: the unit kernel takes the whole rounds and slices of tokens the rest."""
import numpy as np
import pytest
import torch

from oracle import ccd_oracle as O
from paper_2410_01518_amd import infinipot as ip
from paper_2410_01518_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# 264 = 256 + 8 units: rest through the direct kernels; with a window, CaP keys, given normalisers
@pytest.mark.parametrize("option", ["plain", "kcat_window", "lse", "per_head"])
def test_rest_of_a_round_matches_oracle(option):
    cfg = synth.CCDConfig("t", 3, 11, 16, 8, 128, 1030, 400, 5, 100, 5, "bf16", "normal", 7)
    print(f"rounds {cfg} {option}", flush=True)
    inp = synth.make_inputs(cfg)
    window = 900 if option == "kcat_window" else 0
    K_cap = synth.cap_keys(cfg) if option == "kcat_window" else None
    lse = np.random.default_rng(1).normal(6.0, 0.5, (cfg.B, cfg.L, cfg.Hq, cfg.P)).astype(np.float32) if option == "lse" else None
    if option == "per_head":
        inp["novelty"] = np.random.default_rng(2).random((cfg.B, cfg.L, cfg.Hkv, cfg.N)).astype(np.float32)
    dev = {k: gu.to_dev(v) for k, v in inp.items()}
    shape = ip.make_shape(dev["Q_cat"], dev["K"], dev["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, window=window)
    ws = ip.alloc_workspace(shape)
    ws.fill_(0xFF)
    keep = torch.empty((cfg.B, cfg.L, cfg.Hkv, cfg.k), dtype=torch.int32, device="cuda")
    scores = torch.empty((cfg.B, cfg.L, cfg.Hkv, cfg.N), dtype=torch.float32, device="cuda")
    if lse is not None:
        rc = ip.ccd_compress_lse(shape, dev["Q_cat"], dev["K"], dev["V"], gu.to_dev(lse), dev["novelty"], keep, ws, scores=scores)
    elif K_cap is not None:
        rc = ip.ccd_compress_kcat(shape, dev["Q_cat"], dev["K"], dev["V"], gu.to_dev(K_cap), dev["novelty"], keep, ws, scores=scores)
    else:
        rc = ip.ccd_compress(shape, dev["Q_cat"], dev["K"], dev["V"], dev["novelty"], keep, ws, scores=scores)
    assert rc == ip.CCD_OK
    torch.cuda.synchronize()
    alone = ip.make_shape(dev["Q_cat"], dev["K"], dev["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, window=window)
    ran = gu.stages_run(lambda: ip.ccd_score(alone, dev["Q_cat"], dev["K"], dev["novelty"], torch.empty_like(scores), ws))
    assert {"score_unit", "score_prob"} <= ran                    # (1030 * 128 is just above what a rest has to be worth: 128000)
    ref = O.compress(inp["Q_cat"], inp["K"], inp["V"], inp["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, K_cap=K_cap, window=window,
                     lse=lse)
    got, kh = gu.to_host(scores), gu.to_host(keep)
    gu.assert_scores_close(got, ref["scores"], cfg.G * cfg.P)
    np.testing.assert_array_equal(kh, gu.replay_select(got, cfg.k))
    want = np.take_along_axis(inp["K"], kh.astype(np.int64)[..., None], axis=3)
    np.testing.assert_array_equal(gu.to_host(dev["K"])[..., :cfg.k, :], want)


# Rests up to half of the chip when a unit is long work, by each of the kernels that take one: against the unit kernel for all units.
# Two orders of fp32 sums of fp32 exponentials: 2e-7 to 4e-7 apart in the 2-norm, 1.3e-6 at most (four times that is asked for).  fp32:
# the unit kernel's logits are good to 2^-16 of sum |q k| (1e-5 and 3.4e-5 apart, four times that).  The stages tell the kernels: a rest
# under a window by slice kernels has head kernels (the unit kernel masks a head of 64 tokens itself), an fp32 rest by longer slices
# without given normalisers a merge.
@pytest.mark.parametrize("units,N,G,P,d,dtype,option,window,stage,rel,most", [
    (384, 4100, 1, 1024, 64, torch.bfloat16, "", 0, None, 1.6e-6, 1e-5), (320, 1100, 1, 256, 128, torch.bfloat16, "", 0, None, 1.6e-6, 1e-5),
    (320, 1100, 4, 64, 128, torch.bfloat16, "kcat", 0, None, 1.6e-6, 1e-5), (320, 2048, 4, 64, 128, torch.bfloat16, "lse", 0, None, 1.6e-6, 1e-5),
    (320, 8192, 4, 64, 128, torch.bfloat16, "kcat", 8100, "window_head", 1.6e-6, 1e-5),
    (320, 8192, 4, 64, 128, torch.bfloat16, "lse", 8192, "window_head", 1.6e-6, 1e-5),
    (320, 8192, 4, 64, 128, torch.bfloat16, "", 8192, "window_head", 1.6e-6, 1e-5),
    (264, 2100, 1, 16, 64, torch.float32, "", 0, None, 4e-5, 1.4e-4), (300, 2500, 4, 64, 64, torch.float32, "", 0, "score_merge", 4e-5, 1.4e-4),
    (300, 2500, 4, 64, 64, torch.float32, "lse", 0, None, 4e-5, 1.4e-4)])
def test_rest_of_a_round_against_the_unit_kernel(units, N, G, P, d, dtype, option, window, stage, rel, most):
    print(f"rounds {units} {N} {G} {P} {d} {option} {window}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(units)
    K, Q, K_cap = (torch.empty((1, units, h, m, d), dtype=dtype, device="cuda").normal_(generator=g) for h, m in ((1, N), (G, P), (1, P)))
    lse = torch.full((1, units, G, P), 8.0, device="cuda")
    out = []
    for path in (ip.CCD_PATH_AUTO, ip.CCD_PATH_MFMA_UNIT):
        shape = ip.make_shape(Q, K, None, k=N // 2, window=window, score_path=path)
        scores, ws = torch.empty((1, units, 1, N), dtype=torch.float32, device="cuda"), ip.alloc_workspace(shape)
        call = {"": lambda: ip.ccd_score(shape, Q, K, None, scores, ws), "lse": lambda: ip.ccd_score_lse(shape, Q, K, lse, None, scores, ws),
                "kcat": lambda: ip.ccd_score_kcat(shape, Q, K, K_cap, None, scores, ws)}[option]
        stages = gu.stages_run(call)
        assert "score_unit" in stages and ("score_prob" in stages) == (path == ip.CCD_PATH_AUTO)
        assert ("window_head" in stages, "score_merge" in stages) == ((stage == "window_head", stage == "score_merge") if path == ip.CCD_PATH_AUTO else (False, False))
        out.append(scores.double())
    torch.cuda.synchronize()
    a, b = out
    seen = b > 0.0
    assert torch.equal(a > 0.0, seen)
    assert float((a - b).norm() / b.norm()) < rel and float(((a - b).abs()[seen] / b[seen]).max()) < most
