"""The structured transforms and layer outputs over token counts and frame shapes at which
their launch forms change: rotations by rows or by 16-row tiles, DFTs of 1, 2, 4 or 8 vectors a
work-group, one or several token blocks, long rows of the rotation's view."""
import numpy as np
import pytest

from fq_testutil import need_gpu

pytestmark = pytest.mark.gpu


def _frame(torch, fq, d, k, rho, d1, seed):
    rng = np.random.default_rng(seed)
    R = []
    for n in (d1, d // d1):
        q, t = np.linalg.qr(rng.standard_normal((n, n)))
        R.append((q * np.sign(np.diag(t))).astype(np.float32))
    F = fq.Frame(d, k, rho, torch.from_numpy(R[0]).cuda(), torch.from_numpy(R[1]).cuda())
    # the dense frame in float64, column s rho + 2c + e
    m = d // rho
    P = np.zeros((d, k * rho))
    for c in range(rho // 2):
        j = c * m + np.arange(m)
        ph = np.exp(2j * np.pi * ((j[:, None] * np.arange(k)) % k) / k) / np.sqrt(k)
        for e, w in ((0, ph), (1, 1j * ph)):
            P[2 * j, 2 * c + e::rho] = w.real
            P[2 * j + 1, 2 * c + e::rho] = w.imag
    M = P.T.reshape(k * rho, d1, d // d1)
    P = (R[0].astype(np.float64) @ M @ R[1].astype(np.float64).T).reshape(k * rho, d).T
    return F, P


SHAPES = [
    (96, 13, 8, 8),          # d2 = 12: many thread groups a column
    (400, 55, 8, 16),        # d2 = 25, odd
    (1200, 80, 16, 2),       # d2 = 600 > 512 threads, rows of one block a part of a view row
    (520, 70, 8, 260),       # d1 = 260 > 128, d2 = 2: view rows much shorter than a tile
    (2112, 150, 16, 33),     # d2 = 64, odd d1
]


@pytest.mark.parametrize("d,k,rho,d1", SHAPES)
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 9, 81])
def test_transforms_every_launch_form(d, k, rho, d1, n):
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    F, P = _frame(torch, fq, d, k, rho, d1, d + k)
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, d), generator=g, device="cuda")
    Pd = torch.from_numpy(P).cuda()
    ws = torch.full((fq.fq_tff_analysis_workspace_bytes(n, F),), 0xFF, dtype=torch.uint8, device="cuda")
    U = fq.fq_tff_analysis(X, F, ws=ws)
    ref = X.double() @ Pd
    # fp32 factors and twiddles (about 2^-23 each) and fp32 sums of d1 + d2 + m terms
    tol = 2.0 ** -24 * (8.0 + 2.0 * np.sqrt(d1 + d // d1 + d // rho))
    assert ((U.double() - ref).norm() / ref.norm()).item() < tol
    ws.fill_(0xFF)
    Y = fq.fq_tff_synthesis(U, F, ws=ws)
    back = U.double() @ Pd.t().contiguous()
    tol = 2.0 ** -24 * (8.0 + 2.0 * np.sqrt(d1 + d // d1 + k))
    assert ((Y.double() - back).norm() / back.norm()).item() < tol


@pytest.mark.parametrize("d,k,rho,d1", SHAPES + [
    (768, 53, 16, 24), (4096, 282, 16, 64), (11008, 757, 16, 86),
    (2016, 139, 16, 2),      # d2 = 1008, the longest view row of the tiles
    (2080, 143, 16, 2),      # d2 = 1040: rows at any count
    (64, 17, 4, 1), (64, 17, 4, 64),
    (16400, 1128, 16, 8200), # the left factor's rows read from memory
])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -124])      # results in the subnormal range too
def test_a_vector_alone_and_in_a_batch(d, k, rho, d1, scale):
    """A vector's transform is the same bits whatever other vectors share its call."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    g = torch.Generator(device="cuda").manual_seed(d)
    F = fq.Frame(d, k, rho, *(torch.randn((n, n), generator=g, device="cuda") / np.sqrt(n) for n in (d1, d // d1)))
    for dtype in (torch.float32, torch.float16, torch.bfloat16):
        X = (torch.randn((20, d), generator=g, device="cuda") * (scale if dtype != torch.float16 else 1.0)).to(dtype)
        V = torch.randn((20, F.K), generator=g, device="cuda") * scale
        U, Y = fq.fq_tff_analysis(X, F), fq.fq_tff_synthesis(V, F)
        for n in (1, 2, 7, 8, 17):
            assert torch.equal(fq.fq_tff_analysis(X[:n], F), U[:n]), n
            assert torch.equal(fq.fq_tff_synthesis(V[:n], F), Y[:n]), n
        assert torch.equal(fq.fq_tff_analysis(X[19:], F), U[19:])
        assert torch.equal(fq.fq_tff_synthesis(V[19:], F), Y[19:])


@pytest.mark.parametrize("bits", [2, 4])
def test_a_token_alone_and_in_a_batch(bits):
    """Layer outputs too, with float and with rounded activations (where one bit can move a
    rounded value)."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    g = torch.Generator(device="cuda").manual_seed(bits)
    mk = lambda d, k, d1: fq.Frame(d, k, 16, *(torch.randn((n, n), generator=g, device="cuda") / np.sqrt(n)
                                               for n in (d1, d // d1)))
    Fo, Fi = mk(768, 53, 24), mk(1104, 76, 24)
    words = torch.randint(-2 ** 31, 2 ** 31 - 1, (Fo.K, fq.fq.words_per_row(Fi.K, bits)), generator=g,
                          device="cuda").to(torch.int32)
    sc, ze = torch.rand(Fo.K, generator=g, device="cuda"), torch.full((Fo.K,), 1.0, device="cuda")
    X = torch.randn((90, 1104), generator=g, device="cuda").bfloat16()
    for f in (lambda x: fq.fq_frame_apply_tff(x, words, sc, ze, Fo, Fi, bits=bits),
              lambda x: fq.fq_frame_apply_tff_actq(x, words, sc, ze, Fo, Fi, 8, bits=bits)):
        Y = f(X)
        for n in (1, 5, 6, 7, 8, 16, 17, 80):
            assert torch.equal(f(X[:n]), Y[:n]), n


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("n", [1, 5, 6, 16, 17, 80, 81, 163])
def test_layer_outputs_token_blocks(bits, n):
    """The same outputs, bit for bit, with any accepted workspace: the size the query states,
    and the smallest accepted (blocks of fewer tokens)."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    Fo, Po = _frame(torch, fq, 400, 27, 16, 16, 3)
    Fi, Pi = _frame(torch, fq, 336, 23, 16, 16, 4)
    rng = np.random.default_rng(bits)
    codes = rng.integers(0, 1 << bits, size=(Fo.K, Fi.K))
    cpw = 32 // bits
    w = np.zeros((Fo.K, (Fi.K + cpw - 1) // cpw), np.uint32)
    for j in range(Fi.K):
        w[:, j // cpw] |= codes[:, j].astype(np.uint32) << np.uint32(bits * (j % cpw))
    scale = rng.uniform(0.01, 0.1, Fo.K).astype(np.float32)
    zero = rng.integers(0, 1 << bits, Fo.K).astype(np.float32)
    words, sc, ze = (torch.from_numpy(a).cuda() for a in (w.view(np.int32), scale, zero))
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, 336), generator=g, device="cuda").bfloat16()
    D = scale[:, None].astype(np.float64) * (codes - zero[:, None])
    T = torch.from_numpy(Po @ D @ Pi.T).cuda()
    ref = X.double() @ T.t().contiguous()
    full = fq.fq_frame_apply_tff_workspace_bytes(Fo, Fi)
    least = 4 * (8 * (336 + 400 + Fo.K + (Fi.K + 15) // 16 * 16) + Fo.R2.shape[0] ** 2) + 6 * 256
    ys = []
    for size in (full, least):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        ys.append(fq.fq_frame_apply_tff(X, words, sc, ze, Fo, Fi, ws=ws, bits=bits))
    assert torch.equal(ys[0], ys[1])
    assert ((ys[0].double() - ref).norm() / ref.norm()).item() < 2e-6
    # rounded activations: equal for every block size too
    full = fq.fq_frame_apply_tff_actq_workspace_bytes(Fo, Fi)
    least += 8 * ((Fi.K + 15) // 16 * 16) + 8 * 8 + 4 * 256
    ys = []
    for size in (full, least):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        ys.append(fq.fq_frame_apply_tff_actq(X, words, sc, ze, Fo, Fi, 8, ws=ws, bits=bits))
    assert torch.equal(ys[0], ys[1])
    assert ((ys[0].double() - ref).norm() / ref.norm()).item() < 2e-2


@pytest.mark.parametrize("d,k,rho,d1,n", [
    (13824, 950, 16, 108, 17),    # 8 vectors of 950 subspaces a work-group: 68 KB of LDS
    (6016, 1639, 4, 64, 3),       # 4 of 1639: 66 KB
    (4000, 2457, 2, 50, 5),       # the most 4 take, 96 KB
    (4000, 2458, 2, 50, 5),       # 2 from here on
    (1456, 1365, 2, 26, 17),      # the most 8 take, 96 KB
    (1456, 1366, 2, 26, 17),      # 4 from here on
])
def test_transforms_beyond_64_kb_of_lds(d, k, rho, d1, n):
    """Synthesis and analysis against 64 bits where the vectors of a work-group need a raised LDS
    limit, and where fewer vectors are taken, also replayed from a graph."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    g = torch.Generator(device="cuda").manual_seed(k)
    R1, R2 = (torch.linalg.qr(torch.randn((s, s), generator=g, device="cuda", dtype=torch.float64))[0].float().contiguous()
              for s in (d1, d // d1))
    F = fq.Frame(d, k, rho, R1, R2)
    X = torch.randn((n, d), generator=g, device="cuda")
    V = torch.randn((n, F.K), generator=g, device="cuda")
    m, nb = d // rho, rho // 2
    ph = (torch.arange(d // 2, device="cuda")[:, None] * torch.arange(k, device="cuda")[None, :]) % k
    E = torch.polar(torch.full(ph.shape, k ** -0.5, dtype=torch.float64, device="cuda"), ph.double() * (-2.0 * np.pi / k))
    z = R1.double().t().contiguous() @ X.double().reshape(n, d1, d // d1) @ R2.double()
    z = torch.view_as_complex(z.reshape(n, d // 2, 2).contiguous())
    U = torch.stack([z[:, c * m:(c + 1) * m].contiguous() @ E[c * m:(c + 1) * m] for c in range(nb)], 2)
    U = torch.view_as_real(U.contiguous()).reshape(n, F.K)
    v = torch.view_as_complex(V.double().reshape(n, k, nb, 2).contiguous())
    y = torch.cat([v[:, :, c].contiguous() @ E[c * m:(c + 1) * m].conj().t().resolve_conj().contiguous() for c in range(nb)], 1)
    Y = torch.view_as_real(y.contiguous()).reshape(n, d1, d // d1)
    Y = (R1.double() @ Y @ R2.double().t().contiguous()).reshape(n, d)
    ws = torch.full((max(fq.fq_tff_analysis_workspace_bytes(n, F), fq.fq_tff_synthesis_workspace_bytes(n, F)),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    u, o = torch.empty((n, F.K), device="cuda"), torch.empty((n, d), device="cuda")
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        fq.fq_tff_analysis(X, F, u, ws=ws)
        fq.fq_tff_synthesis(V, F, o, ws=ws)
    for _ in range(3):
        u.fill_(0.0), o.fill_(0.0), ws.fill_(0xFF)
        graph.replay()
        torch.cuda.synchronize()
        # fp32 factors and twiddles and fp32 sums of d1 + d2 + m (k) terms, as above
        tol = lambda terms: 2.0 ** -24 * (8.0 + 2.0 * np.sqrt(d1 + d // d1 + terms))
        assert ((u.double() - U).norm() / U.norm()).item() < tol(m)
        assert ((o.double() - Y).norm() / Y.norm()).item() < tol(k)
    assert torch.equal(fq.fq_tff_analysis(X, F, ws=ws), u) and torch.equal(fq.fq_tff_synthesis(V, F, ws=ws), o)
