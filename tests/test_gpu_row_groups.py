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


def _check(units, N, G, P, d, dtype="bf16", option="", window=0):
    print(f"row groups {units} {N} {G} {P} {d} {dtype} {option} {window}", flush=True)
    cfg = synth.CCDConfig("t", 1, units, G, 1, d, N, max(1, N // 3), P, N // 8, 5, dtype, "normal", N + P)
    inp = synth.make_inputs(cfg)
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
    assert "score_unit" in gu.stages_run(call)
    ref = O.compress(inp["Q_cat"], inp["K"], inp["V"], inp["novelty"], k=cfg.k, T=cfg.T, pool_w=cfg.w, K_cap=K_cap,
                     window=window, lse=given)
    gu.assert_scores_close(gu.to_host(scores), ref["scores"], G * P)


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
