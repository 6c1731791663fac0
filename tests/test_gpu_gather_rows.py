"""Out-of-place compaction at the edges of its runs of destination rows, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2410_01518_amd import infinipot as ip

pytestmark = pytest.mark.gpu

# a run is 4 x 256 x 16 bytes of destination rows: 128, 64 or 32 of them
@pytest.mark.parametrize("dtype,d,run", [(torch.bfloat16, 64, 128), (torch.float32, 64, 64), (torch.bfloat16, 128, 64),
                                         (torch.float32, 128, 32)])
def test_runs(dtype, d, run):
    g = torch.Generator(device="cuda").manual_seed(d + run)
    for n, k in ((1, 1), (run, run - 1), (run + 9, run), (2 * run, run + 1), (7 * run + 3, 5 * run + 1)):
        print(f"gather {dtype} d={d} n={n} k={k}", flush=True)
        K = torch.randn((2, 3, 2, n, d), generator=g, device="cuda").to(dtype)
        V = torch.randn((2, 3, 2, n, d), generator=g, device="cuda").to(dtype)
        keep = torch.stack([torch.randperm(n, generator=g, device="cuda")[:k].sort().values for _ in range(12)])
        keep = keep.reshape(2, 3, 2, k)
        K_out, V_out = torch.full_like(K, 7.0), torch.full_like(V, 7.0)
        shape = ip.make_shape(None, K, None, k=k)
        assert ip.ccd_compact(shape, K, V, keep.to(torch.int32).contiguous(), K_out, V_out) == ip.CCD_OK
        torch.cuda.synchronize()
        rows = keep[..., None].expand(-1, -1, -1, -1, d)
        for src, out in ((K, K_out), (V, V_out)):
            want = torch.full_like(src, 7.0)
            want[:, :, :, :k] = torch.gather(src, 3, rows)
            np.testing.assert_array_equal(out.float().cpu().numpy(), want.float().cpu().numpy())
