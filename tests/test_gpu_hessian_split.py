"""The Hessian's token split: whole K steps of 32 tokens in the asynchronous product, the
rest with the reduction, splits and tiles chosen from the sizes, and fp32 sums that no choice
makes longer."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from fq_testutil import need_gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,d,ld", [
    (1, 64, 64),          # the reduction alone
    (31, 264, 272),       # the longest remainder, two tiles, rows of a wider buffer
    (32, 256, 256),       # one K step, no remainder
    (33, 520, 520),       # one K step and one token
    (2047, 512, 512),     # several splits and 31 tokens
    (4099, 96, 96),       # one tile, many splits
    (65, 52, 52),         # extent not a multiple of 8
    (100, 40, 45),        # rows not 16-byte aligned: the register-staged product
    (9000, 136, 136),     # two 128-column tiles, the second of 8 columns; many splits
    (2500, 640, 640),     # five 128-column tiles: the last 256 x 256 tile has one quarter
    (2600, 1160, 1160),
    (600, 5768, 5768),    # two splits, 24 tokens left over: all in the register-staged product
])
def test_token_remainders(dtype, n, d, ld):
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    g = torch.Generator(device="cuda").manual_seed(n * 1000 + d)
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    X = torch.randn((n, ld), generator=g, device="cuda").to(dt)[:, :d]
    X[:, 1] *= 50.0
    ref = X.double().t().contiguous() @ X.double()
    code = {"f32": fq.FQ_F32, "f16": fq.FQ_F16, "bf16": fq.FQ_BF16}[dtype]
    ws = torch.full((fq.fq_hessian_workspace_bytes(code, n, d),), 0xFF, dtype=torch.uint8, device="cuda")
    H = torch.full((d, d), float("nan"), device="cuda")
    fq.fq_hessian_accumulate(X, H, ws=ws)
    # fp32 sums of n exact products (n 2^-24 at worst, sqrt(n) 2^-24 for random signs); for
    # fp32 inputs a bf16 pair each (2^-17 a product)
    tol = (4.0 * np.sqrt(n) + 4.0) * 2.0 ** -24 + (2.0 ** -16 if dtype == "f32" else 0.0)
    scale = ref.diagonal().sqrt()
    err = ((H.double() - ref).abs() / (scale[:, None] * scale[None, :]).clamp_min(1e-30)).max().item()
    assert err <= tol, err
    assert torch.equal(H, H.t())
    H0 = H.clone()
    fq.fq_hessian_accumulate(X, H, accumulate=True, ws=ws)
    assert ((H.double() - 2.0 * H0.double()).abs() <= 2.0 ** -22 * H0.double().abs()).all()


def _longest_sum(n, d):
    """Tokens of the longest fp32 sum: those of as many splits as the workspace holds."""
    t = (d + 255) // 256
    tiles, kt = t * (t + 1) // 2, (n + 63) // 64
    splits = min(kt, max(1, (2048 + tiles // 2) // tiles))
    return 64 * -(-kt // splits)


@pytest.mark.parametrize("dtype,n,d", [("f16", 2037, 2048), ("bf16", 2048, 4096), ("bf16", 8192, 2048),
                                       ("bf16", 25216, 768), ("bf16", 16384, 2048), ("f16", 40000, 256)])
def test_error_of_the_fp32_sums(dtype, n, d):
    """Off the diagonal (whose entries, all of one sign, are larger), against 64 bits, in units of
    sqrt(H_ii H_jj), for Gaussian tokens.  Sums of L tokens in steps of 16, each rounded (c 2^-24
    of the partial sum, c^2 = 1/3 on average), n / L of them added in fp64, and H rounded:
    c 2^-24 sqrt((1 + L / 32) / n); c at most 0.85."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    dt = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    code = {"f16": fq.FQ_F16, "bf16": fq.FQ_BF16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, d), generator=g, device="cuda").to(dt)
    H = torch.empty((d, d), device="cuda")
    ws = torch.full((fq.fq_hessian_workspace_bytes(code, n, d),), 0xFF, dtype=torch.uint8, device="cuda")
    fq.fq_hessian_accumulate(X, H, ws=ws)
    ref = X.double().t().contiguous() @ X.double()
    s = ref.diagonal().sqrt()
    err = (((H.double() - ref) / (s[:, None] * s[None, :])).fill_diagonal_(0.0)).norm().item() / d
    assert err < 0.85 * 2.0 ** -24 * np.sqrt((1.0 + _longest_sum(n, d) / 32.0) / n), err


@pytest.mark.parametrize("n,d", [(2048, 2048), (2500, 640), (9000, 136), (65536, 256)])
def test_overflow_and_special_values(n, d):
    """A sum beyond fp32 is an infinity, a NaN or an infinity stays in its column and row."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn((n, d), generator=g, device="cuda").bfloat16()
    X[:, 3] = 1e19 * torch.sign(X[:, 3].float()).bfloat16()
    X[n // 2, 70] = float("nan")
    X[n // 3, 100] = float("inf")
    H = torch.empty((d, d), device="cuda")
    fq.fq_hessian_accumulate(X, H)
    assert H[3, 3] == float("inf")
    assert torch.isnan(H[70]).all() and torch.isnan(H[:, 70]).all()
    assert (~torch.isfinite(H[100])).all() and H[100, 100] == float("inf")
    ok = [j for j in range(d) if j not in (70, 100)]
    rest = H[ok][:, ok].clone()
    rest[3, 3] = 0.0
    assert torch.isfinite(rest).all()


def test_split_count_is_small_for_few_tiles():
    """A workspace sized for the longest chunk serves every shorter one."""
    torch = need_gpu()
    import paper_2403_06082_amd as fq
    sizes = [fq.fq_hessian_workspace_bytes(fq.FQ_BF16, n, 768) for n in range(0, 40000, 97)]
    assert sizes == sorted(sizes)
    ws = torch.empty(sizes[-1], dtype=torch.uint8, device="cuda")
    for n in (5, 300, 4000, 25216):
        X = torch.randn((n, 768), device="cuda").bfloat16()
        H = torch.empty((768, 768), device="cuda")
        fq.fq_hessian_accumulate(X, H, ws=ws)
        ref = X.double().t().contiguous() @ X.double()
        assert ((H.double() - ref).norm() / ref.norm()).item() < 1e-6
