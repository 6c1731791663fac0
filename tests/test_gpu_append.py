"""GPU parity of ccd_append (Sec. 3.2: filling the pot between two distillations) through the C ABI: bit copies."""
import numpy as np
import pytest
import torch

from oracle import ccd_oracle as O
from paper_2410_01518_amd import infinipot as ip
from paper_2410_01518_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    base = dict(name="t", B=2, L=2, Hq=4, Hkv=2, d=128, N=700, k=300, P=4, T=100, w=1, dtype="bf16", keys="normal", seed=7)
    base.update(kw)
    return synth.CCDConfig(**base)


# (cache type, head dimension, pot size, cached tokens, chunk length): chunk shares of a unit below, at and above four and more of
# the 16 KiB a workgroup moves, not multiples of it, an empty pot, a chunk that fills the pot exactly, an empty chunk
CASES = [
    ("bf16", 128, 700, 300, 100), ("bf16", 128, 700, 0, 700), ("bf16", 128, 4096, 2048, 2048), ("bf16", 64, 515, 3, 509),
    ("fp32", 64, 600, 100, 257), ("fp32", 128, 300, 299, 1), ("bf16", 128, 700, 300, 0), ("bf16", 128, 1300, 7, 1033),
]


@pytest.mark.parametrize("per_head", [True, False])
@pytest.mark.parametrize("dtype,d,N,n_valid,m", CASES)
def test_append_bit_exact(dtype, d, N, n_valid, m, per_head):
    cfg = _cfg(dtype=dtype, d=d, N=N, B=1 if N > 2000 else 2)
    print(f"append {cfg} n_valid={n_valid} m={m} per_head={per_head}", flush=True)
    inp = synth.make_inputs(cfg, per_head_novelty=per_head)
    rng = np.random.default_rng(5)
    new = synth.make_inputs(synth.scaled(cfg, N=max(m, 1), k=1, T=0, seed=99))
    K_new, V_new = new["K"][..., :m, :], new["V"][..., :m, :]
    nov_new = rng.random((cfg.B, m), dtype=np.float32)
    dev = {k: gu.to_dev(v) for k, v in inp.items()}
    shape = ip.make_shape(None, dev["K"], dev["novelty"], k=1, n_valid=n_valid)
    rc = ip.ccd_append(shape, dev["K"], dev["V"], dev["novelty"], gu.to_dev(np.ascontiguousarray(K_new)),
                       gu.to_dev(np.ascontiguousarray(V_new)), gu.to_dev(nov_new))
    torch.cuda.synchronize()
    assert rc == ip.CCD_OK
    np.testing.assert_array_equal(gu.to_host(dev["K"]), O.append(inp["K"], n_valid, K_new))
    np.testing.assert_array_equal(gu.to_host(dev["V"]), O.append(inp["V"], n_valid, V_new))
    nov_chunk = nov_new[:, None, None, :] if per_head else nov_new
    np.testing.assert_array_equal(gu.to_host(dev["novelty"]).view(np.uint32),
                                  O.append(inp["novelty"], n_valid, nov_chunk).view(np.uint32))


def test_append_into_a_strided_pot_leaves_the_padding_alone():
    """K and V as views of larger buffers (more heads, more rows per head): only the chunk's rows of the viewed units
    change."""
    cfg = _cfg(N=400)
    inp = synth.make_inputs(cfg)
    n_valid, m = 150, 200
    big = torch.full((cfg.B, cfg.Hkv + 1, cfg.L, cfg.N + 8, cfg.d), 7.0, dtype=torch.bfloat16, device="cuda")
    bigv = torch.full_like(big, 9.0)
    Kview = big[:, :cfg.Hkv, :, :cfg.N].permute(0, 2, 1, 3, 4)
    Vview = bigv[:, :cfg.Hkv, :, :cfg.N].permute(0, 2, 1, 3, 4)
    Kview.copy_(gu.to_dev(inp["K"]))
    Vview.copy_(gu.to_dev(inp["V"]))
    before_k, before_v = big.clone(), bigv.clone()
    new = synth.make_inputs(synth.scaled(cfg, N=m, k=1, T=0, seed=98))
    shape = ip.make_shape(None, Kview, None, k=1, n_valid=n_valid)
    assert ip.ccd_append(shape, Kview, Vview, None, gu.to_dev(new["K"]), gu.to_dev(new["V"]), None) == ip.CCD_OK
    torch.cuda.synchronize()
    np.testing.assert_array_equal(gu.to_host(Kview.contiguous()), O.append(inp["K"], n_valid, new["K"]))
    np.testing.assert_array_equal(gu.to_host(Vview.contiguous()), O.append(inp["V"], n_valid, new["V"]))
    mask = torch.ones_like(big, dtype=torch.bool)
    mask[:, :cfg.Hkv, :, n_valid:n_valid + m] = False
    assert torch.equal(big[mask], before_k[mask]) and torch.equal(bigv[mask], before_v[mask])


def test_streaming_pot_appends_and_distils_like_the_oracle():
    """Three chunks through a small pot (append, append, distil, append): the pot's K, V and carried novelty equal the
    oracle's after every step."""
    from paper_2410_01518_amd.pot import MemoryPot
    cfg = _cfg(B=1, L=2, Hq=4, Hkv=2, d=64, N=512, k=256, P=8, T=64, w=3)
    pot = MemoryPot(cfg.B, cfg.L, cfg.Hkv, cfg.d, cfg.N, cfg.k, cfg.T, pool_w=cfg.w)
    hK = np.zeros((cfg.B, cfg.L, cfg.Hkv, cfg.N, cfg.d), dtype=np.uint16)
    hV, hn, n = hK.copy(), np.zeros((cfg.B, cfg.L, cfg.Hkv, cfg.N), dtype=np.float32), 0
    rng = np.random.default_rng(3)
    for step in range(3):
        if n + 256 > cfg.N:
            q = synth.make_inputs(synth.scaled(cfg, seed=50 + step))["Q_cat"]
            ref = O.compress(q, hK, hV, hn, k=cfg.k, T=cfg.T, pool_w=cfg.w)
            assert pot.distill(gu.to_dev(q)) == ip.CCD_OK
            hK[..., :cfg.k, :], hV[..., :cfg.k, :] = ref["K"], ref["V"]
            hn[..., :cfg.k] = np.take_along_axis(hn, ref["keep_idx"].astype(np.int64), axis=3)
            n = cfg.k
            np.testing.assert_array_equal(gu.to_host(pot.keep_idx), ref["keep_idx"])
        new = synth.make_inputs(synth.scaled(cfg, N=256, k=1, T=0, seed=60 + step))
        nv = rng.random((cfg.B, 256), dtype=np.float32)
        pot.append(gu.to_dev(new["K"]), gu.to_dev(new["V"]), gu.to_dev(nv))
        hK, hV, hn = O.append(hK, n, new["K"]), O.append(hV, n, new["V"]), O.append(hn, n, nv[:, None, None, :])
        n += 256
        torch.cuda.synchronize()
        assert pot.n_valid == n
        np.testing.assert_array_equal(gu.to_host(pot.K)[..., :n, :], hK[..., :n, :])
        np.testing.assert_array_equal(gu.to_host(pot.V)[..., :n, :], hV[..., :n, :])
        np.testing.assert_array_equal(gu.to_host(pot.novelty)[..., :n], hn[..., :n])


def test_append_to_more_units_than_one_grid_has_threads_for():
    """Four million units whose shares of 16.5 KiB take two workgroups a tensor: more than 2^32 threads, so several launches.  The
    layers of a sequence are one piece of memory, and K and V are one chunk: 69 GB of it."""
    B, L, rows = 2, (1 << 21) + 1, 129
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 69 GB of device memory")
    K, V = (torch.zeros((B, 1, 1, rows, 64), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    new = torch.empty((B, L, 1, rows, 64), dtype=torch.bfloat16, device="cuda")
    new[0], new[1] = 1.0, 2.0
    shape = ip.make_shape(None, K.expand(B, L, 1, rows, 64), None, k=1, n_valid=0)
    print(f"append units={B * L} rows={rows}", flush=True)
    assert ip.ccd_append(shape, K, V, None, new, new, None) == ip.CCD_OK
    torch.cuda.synchronize()
    del new
    torch.cuda.empty_cache()
    for t in (K, V):
        assert bool((t[0] == 1.0).all()) and bool((t[1] == 2.0).all())


# chunks that fill an empty pot and are more than the memory-side cache holds, moved as one stretch: units that end inside a segment, rows of novelty that
# end inside a piece of 1024 tokens, units of just a segment; and pots that are no stretch (heads further apart, a token left empty, units
# of less than a segment)
@pytest.mark.parametrize("novelty", ["per_head", "shared", "none"])
@pytest.mark.parametrize("B,L,Hkv,m,d,fp32,apart,left", [
    (2, 4, 2, 33001, 64, False, 0, 0), (1, 3, 3, 29129, 128, False, 0, 0), (3, 1, 2, 22999, 128, True, 0, 0), (1, 16, 8, 1025, 128, True, 0, 0),
    (2, 253, 8, 130, 64, False, 0, 0), (1, 510, 8, 129, 64, False, 0, 0), (2, 4, 2, 33001, 64, False, 3, 0), (2, 4, 2, 33001, 64, False, 0, 1),
    (1, 640, 8, 103, 64, False, 0, 0)])
def test_append_that_fills_an_empty_pot(B, L, Hkv, m, d, fp32, apart, left, novelty):
    print(f"append whole pot {B} {L} {Hkv} {m} {d} {fp32} {apart} {left} {novelty}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m)
    dt, it = (torch.float32, torch.int32) if fp32 else (torch.bfloat16, torch.int16)
    assert 4 * B * L * Hkv * m * d * (4 if fp32 else 2) >= 256 << 20
    K_new, V_new = (torch.randint(-32768, 32767, (B, L, Hkv, m, d), generator=g, device="cuda", dtype=torch.int16).to(it) for _ in range(2))
    nov_new = torch.rand((B, m), generator=g, device="cuda")
    cap = m + left
    K, V = (torch.zeros((B, L, Hkv + apart, cap, d), dtype=it, device="cuda") for _ in range(2))
    nov = torch.zeros((B, L, Hkv, cap) if novelty == "per_head" else (B, cap), device="cuda")
    Kh = K[:, :, :Hkv]
    shape = ip.make_shape(None, Kh.view(dt), None if novelty == "none" else nov, k=1, n_valid=0)
    has = novelty != "none"
    assert ip.ccd_append(shape, Kh.view(dt), V[:, :, :Hkv].view(dt), nov if has else None, K_new.view(dt), V_new.view(dt), nov_new if has else None) == ip.CCD_OK
    torch.cuda.synchronize()
    for have, new in ((K, K_new), (V, V_new)):
        assert torch.equal(have[:, :, :Hkv, :m], new) and not bool(have[:, :, Hkv:].any()) and not bool(have[..., m:, :].any())
    if has:
        assert torch.equal(nov[..., :m], nov_new[:, None, None, :].expand(B, L, Hkv, m) if novelty == "per_head" else nov_new)
        assert not bool(nov[..., m:].any())


# chunk and pot are just less than what the memory-side cache holds, and just as much: keys and values in turn, values first
@pytest.mark.parametrize("m", [8191, 8192])
def test_append_of_chunks_as_large_as_the_memory_side_cache(m):
    B, L, Hkv, d, n_valid = 2, 16, 2, 64, 5
    print(f"append m={m}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m)
    K_new, V_new = (torch.randint(-32768, 32767, (B, L, Hkv, m, d), generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16) for _ in range(2))
    nov_new = torch.rand((B, m), generator=g, device="cuda")
    K, V = (torch.zeros((B, L, Hkv, m + 9, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    nov = torch.zeros((B, L, Hkv, m + 9), device="cuda")
    shape = ip.make_shape(None, K, nov, k=1, n_valid=n_valid)
    assert ip.ccd_append(shape, K, V, nov, K_new, V_new, nov_new) == ip.CCD_OK
    torch.cuda.synchronize()
    for have, new in ((K.view(torch.int16), K_new.view(torch.int16)), (V.view(torch.int16), V_new.view(torch.int16)),
                      (nov[..., None], nov_new[:, None, None, :, None].expand(B, L, Hkv, m, 1))):
        assert torch.equal(have[..., n_valid:n_valid + m, :], new)
        assert not bool(have[..., :n_valid, :].any()) and not bool(have[..., n_valid + m:, :].any())
