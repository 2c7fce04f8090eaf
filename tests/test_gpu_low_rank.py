"""The narrow products of the low-rank branch (tl_k_low_rank), and the small frozen ones that take the same kernel (tl_k_frozen), against
fp64 sums of the same bf16 operands.

Every tile the rule can pick, with rows and columns that end inside one, contractions that end inside a 64-wide piece or leave some of the
eight waves without one, and the products that go on to the general kernel.  Tolerance: one bf16 rounding of the result has a relative
error of 2^-9 / sqrt(3) = 1.1e-3 in the L2 sense and at most 2^-9 of the element; 2e-3 and 2e-2 of the RMS leave room for fp32 sums and
elements of 4.5 RMS."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_11504_amd import synth  # noqa: E402

SCRATCH = 16 << 20
#        M, N, K, batch, tile
CASES = [(1024, 64, 4096, 1, "16x16"), (37, 24, 1000, 1, "16x16"), (1, 8, 8, 1, "16x16"), (200, 48, 72, 3, "16x16"), (300, 40, 4096, 2, "16x16"),
         (1024, 96, 4096, 1, "16x32"), (1030, 128, 4104, 1, "32x32"), (1020, 120, 4104, 1, "16x32"), (1000, 32, 4096, 3, "16x32"),
         (1024, 192, 4096, 1, "32x32"), (1020, 56, 2048, 3, "32x32"), (2048, 192, 4096, 1, "32x48"), (2048, 64, 4096, 3, "32x64"), (2044, 60, 4096, 3, "32x64"),
         (3000, 192, 4096, 1, "48x64"), (2990, 188, 4096, 1, "48x64"), (5120, 192, 4096, 1, "64x64"), (5101, 192, 2048, 1, "64x64"),
         (2048, 64, 11008, 2, "general")]


def test_the_cases_reach_every_tile():
    from paper_2401_11504_amd import api
    for M, N, K, nb, tile in CASES:
        assert api.tl_k_low_rank_plan(M, N, K, nb, SCRATCH) == tile, (M, N, K, nb)
    assert {c[4] for c in CASES} == {"16x16", "16x32", "32x32", "32x48", "32x64", "48x64", "64x64", "general"}


def test_the_other_side_is_what_the_general_kernel_would_do():
    """without scratch, or with too little, it does not split; many rows of 192 columns take its 128-wide tiles; what it refuses it gets"""
    from paper_2401_11504_amd import api
    assert [api.tl_k_low_rank_plan(2048, 64, 11008, 2, n) for n in (SCRATCH, 2048 * 64 * 2 - 1, 1, 0)] == ["general", "32x32", "32x32", "32x32"]
    assert [api.tl_k_low_rank_plan(64, 64, 11008, 2, n) for n in (SCRATCH, 0)] == ["general", "16x16"]
    assert [api.tl_k_low_rank_plan(M, 192, 4096, 1, SCRATCH) for M in (5120, 12000, 16384)] == ["64x64", "general", "general"]
    assert api.tl_k_low_rank_plan(200, 16, 1001, 1, SCRATCH) == "general"


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,nb", [(2044, 60, 11000, 2), (64, 64, 11008, 2), (5120, 64, 2048, 2)])
def test_without_scratch(M, N, K, nb):
    test_low_rank(M, N, K, nb, None, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,nb,tile", CASES)
def test_low_rank(M, N, K, nb, tile, scratch=SCRATCH):
    from paper_2401_11504_amd import api, harness as H
    # what lies behind the contraction in memory is NaN: it must not be multiplied, not even by zero
    lda, ldb = (nb * K + 71) // 8 * 8, (K + 71) // 8 * 8
    a, b = np.full((M, lda), np.nan), np.full((nb * N, ldb), np.nan)
    a[:, :nb * K] = synth.normal(1, (61, M, N), (M, nb * K), 1.0, True)
    b[:, :K] = synth.normal(2, (62, M, N), (nb * N, K), 0.05, True)
    A, B = H.to_dev_bf16(a)[:, :nb * K], H.to_dev_bf16(b)[:, :K]
    out = torch.full((M + 1, nb * N), 3.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(scratch, dtype=torch.float32, device="cuda") if scratch else None
    for _ in range(2):                  # twice: the same bits
        last = out.clone()
        api.tl_k_low_rank(A, B, out, nb, 0.5, ws)
        torch.cuda.synchronize()
    assert torch.equal(last, out)
    assert torch.all(out[M] == 3.0)
    A64, B64 = A.double(), B.double()
    ref = torch.cat([A64[:, i * K:(i + 1) * K] @ B64[i * N:(i + 1) * N].T for i in range(nb)], 1) * 0.5
    err = out[:M].double() - ref
    assert err.norm() <= 2e-3 * ref.norm()
    assert err.abs().max() <= 2e-2 * ref.norm() / ref.numel() ** 0.5


#         M, N, K, K2, batch, tile
FROZEN = [(200, 256, 256, 16, 1, "16x16"), (200, 256, 688, 16, 1, "16x16"), (1, 8, 8, 8, 1, "16x16"), (45, 100, 2000, 40, 1, "16x16"),
          (200, 688, 256, 16, 1, "32x32"), (300, 512, 1408, 8, 1, "32x32"), (290, 508, 1400, 72, 1, "32x32"), (100, 500, 4096, 64, 1, "16x16"),
          (300, 400, 2048, 0, 1, "16x32"), (500, 636, 1024, 192, 1, "32x48"), (512, 1024, 2816, 16, 1, "32x64"), (1024, 1024, 1024, 16, 1, "general"),
          (128, 4096, 4096, 64, 1, "general"),
          # one input, three outputs side by side, each with its own share of the second input: the q|k|v product
          (200, 256, 256, 16, 3, "32x32"), (37, 100, 704, 8, 3, "16x16"), (190, 252, 248, 24, 3, "32x32"), (300, 508, 1000, 24, 3, "32x32"),
          (200, 512, 512, 64, 3, "32x48"), (300, 1024, 1024, 16, 3, "general"),
          # few rows that share many columns of cold weights
          (200, 2048, 2048, 16, 1, "general"), (256, 1792, 1792, 16, 1, "general"), (85, 2048, 2048, 16, 3, "general"), (16, 2044, 2048, 8, 3, "16x32")]


def test_the_frozen_cases_reach_their_tiles():
    from paper_2401_11504_amd import api
    for *sizes, tile in FROZEN:
        for scratch in (0, SCRATCH):
            assert api.tl_k_frozen_plan(*sizes, scratch) == tile, sizes
    assert {c[5] for c in FROZEN} == {"16x16", "16x32", "32x32", "32x48", "32x64", "general"}


def frozen_operands(M, N, K, K2, nb, f32):
    """operands with NaN around them, an output with a row and 8 columns more than it needs, the fp64 product"""
    from paper_2401_11504_amd import harness as H

    def draw(i, rows, cols, std):
        full = np.full((rows + 8, cols + 8), np.nan)
        full[:rows, :cols] = synth.normal(i, (63, M, N), (rows, cols), std, True)
        return H.to_dev_bf16(full)[:rows, :cols]
    A, B = draw(1, M, K, 1.0), draw(2, nb * N, K, 0.05)
    A2, B2 = (draw(3, M, nb * K2, 1.0), draw(4, nb * N, K2, 0.05)) if K2 else (None, None)
    full = torch.full((M + 1, nb * N + 8), 3.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    R = None
    if f32:
        R = torch.full((M, nb * N + 8), float("nan"), device="cuda")
        R[:, :nb * N] = torch.randn(M, nb * N, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    ref = A.double() @ B.double().T
    if K2:
        ref += torch.cat([A2.double()[:, b * K2:(b + 1) * K2] @ B2.double()[b * N:(b + 1) * N].T for b in range(nb)], 1)
    return A, B, A2, B2, full, R, ref + R[:, :nb * N].double() if f32 else ref


def check_frozen(got, ref, tol):
    err = got.double() - ref
    assert err.norm() <= tol * ref.norm()
    assert err.abs().max() <= 10 * tol * ref.norm() / ref.numel() ** 0.5


@pytest.mark.gpu
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("M,N,K,K2,nb,tile", FROZEN)
def test_frozen(M, N, K, K2, nb, tile, f32):
    """bf16 output as above; fp32 output with a residual: fp32 sums of bf16 products, 1e-5 in the L2 sense (2^-24 times a few roundings of up to
    4288 terms)."""
    from paper_2401_11504_amd import api
    A, B, A2, B2, full, R, ref = frozen_operands(M, N, K, K2, nb, f32)
    api.tl_k_frozen(A, B, full[:M, :nb * N], A2, B2, R, nb)
    torch.cuda.synchronize()
    assert torch.all(full[M] == 3.0) and torch.all(full[:, nb * N:] == 3.0)
    check_frozen(full[:M, :nb * N], ref, 1e-5 if f32 else 2e-3)


#           M, N, K, K2, tile, partial tiles
DEFERRED = [(200, 256, 688, 16, "16x16", 0), (290, 508, 1400, 72, "32x32", 0), (512, 1024, 2816, 16, "32x64", 0), (1024, 1024, 1024, 16, "general", 0),
            (256, 2048, 8192, 64, "general", 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,K2,tile,parts", DEFERRED)
def test_frozen_deferred(M, N, K, K2, tile, parts):
    """What is handed over: no partial tiles and an output that is complete, residual included, or the tiles and an output that is untouched."""
    from paper_2401_11504_amd import api
    assert api.tl_k_frozen_plan(M, N, K, K2, 1, SCRATCH, True) == tile
    A, B, A2, B2, full, R, ref = frozen_operands(M, N, K, K2, 1, True)
    ws = torch.full((SCRATCH,), float("nan"), device="cuda")
    assert api.tl_k_frozen(A, B, full[:M, :N], A2, B2, R, 1, ws, deferred=True) == parts
    torch.cuda.synchronize()
    assert torch.all(full[M] == 3.0) and torch.all(full[:, N:] == 3.0)
    if parts:
        assert torch.all(full == 3.0)
        check_frozen(ws[:parts * M * N].view(parts, M, N).double().sum(0) + R[:, :N].double(), ref, 1e-5)
    else:
        check_frozen(full[:M, :N], ref, 1e-5)
