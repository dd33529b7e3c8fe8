"""Frame generation at the edges of its launch forms: the dense frame by blocks of the view's
rows (1 to 24 of them, odd and even row lengths, several passes, R1 in LDS or not) or by whole
vectors, and the seeded factors in registers (1 to 16 rows a thread) or in memory."""
import numpy as np
import pytest

import oracle as O
from fq_testutil import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,rho,d1", [
    (64, 17, 4, 1),        # one view row: whole vectors
    (64, 17, 4, 64),       # view rows of one element: whole vectors
    (90, 19, 6, 6),        # d2 = 15, odd
    (128, 40, 4, 8),       # blocks of 64 = 4 rows of 16
    (400, 27, 16, 16),     # blocks of 50 in rows of 25: 2 and 3 rows
    (2112, 150, 16, 132),  # d1 > 128: R1 read from memory; 17 or 18 rows a block
    (1536, 99, 16, 3),     # d2 = 512, a block within one or two rows, 1584 columns
    (90, 19, 6, 2),        # two view rows: whole vectors
    (90, 19, 6, 3),        # blocks of 30 in rows of 30
    (4096, 257, 16, 64),   # 4112 columns
])
def test_dense_frame_forms(d, k, rho, d1):
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    rng = np.random.default_rng(d + d1)
    R = []
    for n in (d1, d // d1):
        q, t = np.linalg.qr(rng.standard_normal((n, n)))
        R.append((q * np.sign(np.diag(t))).astype(np.float32))
    F = fq.Frame(d, k, rho, *(torch.from_numpy(r).cuda() for r in R))
    ws = torch.full((fq.fq_tff_materialize_workspace_bytes(F),), 0xFF, dtype=torch.uint8, device="cuda")
    # rows of a wider matrix stay as they are beyond the frame's columns
    ld = F.K + 5
    wide = torch.full((d, ld), 7.0, device="cuda")
    lib = fq.lib()
    import ctypes
    st = lib.fq_tff_materialize(None, ctypes.byref(F.c), ctypes.c_void_p(wide.data_ptr()), ld,
                                ctypes.c_void_p(ws.data_ptr()), ws.numel())
    torch.cuda.synchronize()
    assert st == 0
    m = d // rho
    s = torch.arange(k, device="cuda", dtype=torch.float64)
    T = torch.zeros((d, k, rho), dtype=torch.float64, device="cuda")
    j = torch.arange(d // 2, device="cuda")
    ang = 2.0 * np.pi / k * ((j[:, None] * torch.arange(k, device="cuda")[None, :]) % k).double()
    for c in range(rho // 2):
        rows = torch.arange(c * m, (c + 1) * m, device="cuda")
        cs, sn = torch.cos(ang[rows]) / np.sqrt(k), torch.sin(ang[rows]) / np.sqrt(k)
        T[2 * rows, :, 2 * c], T[2 * rows + 1, :, 2 * c] = cs, sn
        T[2 * rows, :, 2 * c + 1], T[2 * rows + 1, :, 2 * c + 1] = -sn, cs
    R1, R2 = (torch.from_numpy(r).cuda().double() for r in R)
    M = T.reshape(d1, d // d1, -1).permute(2, 0, 1).contiguous()
    P = (R1 @ M @ R2.t().contiguous()).reshape(k * rho, d).t()
    # fp32 sums of d2 and then a block's rows, fp32 twiddles (2^-21 rad)
    assert ((wide[:, :F.K].double() - P).norm() / P.norm()).item() < 1e-6
    if (d, d1) == (4096, 64):
        # partial sums of 8 terms, then of those 8, then of a block's 9 rows, every operation
        # correctly rounded: 1.1e-7 (simulated on the host; 1.8e-7 with 64 terms in one chain)
        assert ((wide[:, :F.K].double() - P).norm() / P.norm()).item() < 2.05 * 2.0 ** -24
    assert (wide[:, :F.K].double() - P).abs().max().item() < 1e-6
    assert (wide[:, F.K:] == 7.0).all()


@pytest.mark.parametrize("d1,d2", [(1, 1), (1, 2), (2, 33), (31, 32), (64, 64), (65, 90), (91, 128),
                                   (128, 129), (129, 40), (86, 128)])
def test_seeded_factors_forms(d1, d2):
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    ws = torch.full((fq.fq.fq_tff_rotation_factors_workspace_bytes(d1, d2),), 0xFF, dtype=torch.uint8,
                    device="cuda")
    R1, R2 = fq.fq_tff_rotation_factors(12345 + d1, d1, d2, ws=ws)
    for f, (R, n) in enumerate(((R1, d1), (R2, d2))):
        ref = O.seeded_haar(12345 + d1, f, n)
        got = R.cpu().numpy().astype(np.float64)
        assert np.abs(got - ref).max() < 1e-6
        assert np.abs(got @ got.T - np.eye(n)).max() < 1e-5
