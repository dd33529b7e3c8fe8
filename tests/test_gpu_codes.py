"""The code product V = U (codes - zero)^T diag(scale) at the edges of its tiles and steps,
through the dense entry point with identity frames (so U = X and Y = V)."""
import numpy as np
import pytest

from fq_testutil import need_gpu

pytestmark = pytest.mark.gpu


def _layer(torch, K_out, K_in, bits, seed):
    rng = np.random.default_rng(seed)
    cpw = 32 // bits
    codes = rng.integers(0, 1 << bits, size=(K_out, K_in))
    w = np.zeros((K_out, (K_in + cpw - 1) // cpw), np.uint32)
    for j in range(K_in):
        w[:, j // cpw] |= codes[:, j].astype(np.uint32) << np.uint32(bits * (j % cpw))
    scale = rng.uniform(0.01, 0.1, K_out).astype(np.float32)
    zero = rng.uniform(0, (1 << bits) - 1, K_out).astype(np.float32)     # any float is taken
    up = lambda a: torch.from_numpy(a).cuda()
    D = up(scale.astype(np.float64)[:, None] * (codes - zero.astype(np.float64)[:, None]))
    eye = lambda n: torch.eye(n, device="cuda")
    return up(w.view(np.int32)), up(scale), up(zero), eye(K_out), eye(K_in), D


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("K_out", [1, 31, 32, 47, 95])       # one short of, at and past a tile
@pytest.mark.parametrize("K_in", [1, 31, 64, 65, 255, 257, 2049])   # words, quads, steps, waves
def test_code_product_edges(bits, K_out, K_in):
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    w, sc, ze, Po, Pi, D = _layer(torch, K_out, K_in, bits, K_out * 7 + K_in)
    for n in (1, 5, 6, 8):
        g = torch.Generator(device="cuda").manual_seed(n)
        X = torch.randn((n, K_in), generator=g, device="cuda")
        X *= 10.0 ** (torch.arange(n, device="cuda") * 4 - 14.0)[:, None]    # 1e-14 .. 1e14
        Y = fq.fq_frame_apply(X, w, sc, ze, Po, Pi, bits=bits)
        ref = X.double() @ D.t().contiguous()
        # per entry: fp32 sums of exact products, and the fp32 zero and scale factors
        bound = (X.double().abs() @ (D / sc.double()[:, None]).abs().t().contiguous() +
                 2.0 * ze.double() * X.double().sum(1, keepdim=True).abs() +
                 ((1 << bits) - 1) * X.double().abs().sum(1, keepdim=True)) * sc.double()
        assert ((Y.double() - ref).abs() <= 2.0 ** -23 * (2.0 + np.sqrt(K_in)) * bound).all()


@pytest.mark.parametrize("bits", [2, 4])
def test_code_product_special_values(bits):
    """A NaN or an infinity stays in its own token; values that need all 24 bits are exact."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    w, sc, ze, Po, Pi, D = _layer(torch, 40, 130, bits, 3)
    X = torch.randn((7, 130), device="cuda")
    clean = fq.fq_frame_apply(X, w, sc, ze, Po, Pi, bits=bits)
    X[2, 5] = float("nan")
    X[4, 129] = float("inf")
    Y = fq.fq_frame_apply(X, w, sc, ze, Po, Pi, bits=bits)
    ok = [0, 1, 3, 5, 6]
    assert torch.equal(Y[ok], clean[ok])
    assert not torch.isfinite(Y[2]).any() and not torch.isfinite(Y[4]).any()
    # one non-zero entry: q u, with the code's row scale 1 and zero 0, has no rounding at all
    one = torch.ones_like(sc)
    X = torch.zeros((3, 130), device="cuda")
    vals = torch.tensor([1.0 + 2.0 ** -23, -(3.0 - 2.0 ** -22), 1.1754945e-30], device="cuda")
    X[torch.arange(3), torch.tensor([0, 64, 129])] = vals
    Y = fq.fq_frame_apply(X, w, one, torch.zeros_like(ze), Po, Pi, bits=bits)
    q = torch.round(D / sc.double()[:, None] + ze.double()[:, None])
    assert torch.equal(Y.double(), (X.double() @ q.t().contiguous()).float().double())


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("K_out", [7936, 7952, 8192, 8208, 12032, 12048, 12288, 12304])
def test_row_tiles_of_one_token_tile(bits, K_out):
    """Row counts at which a single token tile takes 2 or 3 row tiles a work-group (31, 32, 47 and
    48 times 256 rows): 5 tokens, one tile of float columns, as in 6, two tiles, and as in 64 bits."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    from test_gpu_tff_block import _frame
    K_in = 16 * 9
    w, sc, ze, _, Pi, D = _layer(torch, K_out, K_in, bits, K_out)
    g = torch.Generator(device="cuda").manual_seed(K_out)
    Po = torch.randn((8, K_out), generator=g, device="cuda") / np.sqrt(K_out)
    X = torch.randn((6, K_in), generator=g, device="cuda")
    Y = fq.fq_frame_apply(X, w, sc, ze, Po, Pi, bits=bits)
    assert torch.equal(fq.fq_frame_apply(X[:5], w, sc, ze, Po, Pi, bits=bits), Y[:5])
    ref = (X.double() @ D.t().contiguous()) @ Po.double().t().contiguous()
    assert ((Y.double() - ref).norm() / ref.norm()).item() < 2e-6
    # rounded activations: 16 tokens a tile
    Fo, Pod = _frame(torch, fq, 96, K_out // 16, 16, 8, 1)
    Fi, _ = _frame(torch, fq, 128, 9, 16, 8, 2)
    X = torch.randn((17, 128), generator=g, device="cuda")
    Y = fq.fq_frame_apply_tff_actq(X, w, sc, ze, Fo, Fi, 8, bits=bits)
    assert torch.equal(fq.fq_frame_apply_tff_actq(X[:16], w, sc, ze, Fo, Fi, 8, bits=bits), Y[:16])
    U = fq.fq_tff_analysis(X, Fi)
    C, delta = fq.fq_act_quantize(U, 8)
    ref = (C.double() * delta.double()[:, None]) @ D.t().contiguous() @ torch.from_numpy(Pod).cuda().t().contiguous()
    assert ((Y.double() - ref).norm() / ref.norm()).item() < 2e-6
