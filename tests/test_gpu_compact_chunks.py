"""Compaction in place by one workgroup per unit (more than 128 units): row counts one short of, equal to and one over its chunks of rows, the
kept list in LDS and (long rows) in keep_idx.  Rows and carried novelty are copies: the same bits."""
import pytest
import torch

from paper_2410_01518_amd import infinipot as ip
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# a chunk is four passes of 1024 threads: 512 rows of 128 bytes, 256 of 256, 128 of 512
@pytest.mark.parametrize("units,N,d,dtype,k", [
    (130, 1100, 64, torch.bfloat16, 511), (130, 1100, 64, torch.bfloat16, 512), (130, 1100, 64, torch.bfloat16, 513),
    (129, 700, 128, torch.bfloat16, 255), (129, 700, 128, torch.bfloat16, 257), (129, 700, 128, torch.float32, 127),
    (129, 700, 128, torch.float32, 129), (260, 5000, 64, torch.float32, 1), (130, 8300, 64, torch.bfloat16, 1025)])
def test_rows_and_novelty_move_up(units, N, d, dtype, k):
    print(f"chunks {units} {N} {d} {dtype} {k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    K = torch.empty((1, units, 1, N, d), dtype=dtype, device="cuda").normal_(generator=g)
    V = torch.empty_like(K).normal_(generator=g)
    Q = torch.empty((1, units, 1, 16, d), dtype=dtype, device="cuda").normal_(generator=g)
    novelty = torch.rand((1, units, 1, N), generator=g, device="cuda")
    K[:, :, :, :k // 8] *= 8.0                            # some rows at the start that stay where they are
    novelty[..., :k // 8] += 1.0
    K0, V0, nov0 = K.clone(), V.clone(), novelty.clone()
    shape = ip.make_shape(Q, K, novelty, k=k, T=k // 2, pool_w=3)
    keep = torch.empty((1, units, 1, k), dtype=torch.int32, device="cuda")
    scores = torch.empty((1, units, 1, N), dtype=torch.float32, device="cuda")
    ws = ip.alloc_workspace(shape)
    assert ip.ccd_compress(shape, Q, K, V, novelty, keep, ws, scores=scores) == ip.CCD_OK
    torch.cuda.synchronize()
    assert (gu.to_host(keep) == gu.replay_select(gu.to_host(scores), k)).all()
    idx = keep.long()
    rows = idx[..., None].expand(-1, -1, -1, -1, d)
    assert torch.equal(K[..., :k, :], K0.gather(3, rows)) and torch.equal(V[..., :k, :], V0.gather(3, rows))
    assert torch.equal(K[..., k:, :], K0[..., k:, :]) and torch.equal(V[..., k:, :], V0[..., k:, :])
    assert torch.equal(novelty[..., :k], nov0.gather(3, idx))
