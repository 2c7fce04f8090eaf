"""The direct-to-LDS GEMM where its contraction does not divide by 64: the low-rank pair and the ragged end of the main
pair travel as edge tiles, zero-filled in LDS, ahead of the whole tiles.  Reference: the same bf16 operands in fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_kernels import BF16_TOL, H, api, check, rnd  # noqa: E402,F401  (api, H: fixtures)

# bf16 products are exact in fp32; a sum of K of them in another order differs by about sqrt(K) 2^-24 of its 2-norm, and
# K <= 16384 here: 128 x 6e-8 = 7.6e-6, doubled
F32_TOL = 1.6e-5

CASES = [
    # M, N, K, K2, workspace, plan
    (1000, 2056, 264, 8, False, "128x128"),           # one chunk of each operand pair in two edge tiles
    (1024, 1024, 1024, 16, False, "64x64"),           # rank 16
    (130, 136, 256, 24, False, "64x64"),              # ragged tiles, shortest contraction the path takes
    (333, 520, 328, 200, False, "64x64"),             # more edge tiles (4 + 1) than the prologue fetches (4)
    (1000, 8184, 320, 136, False, "256x128"),         # as many (3) as it fetches
    (1000, 11008, 264, 248, False, "256x192"),        # 4 + 1, prologue 2
    (1024, 16384, 256, 256, False, "256x256"),        # 4 whole edge tiles, prologue 2
    (1024, 16384, 264, 8, False, "256x256"),
    (1000, 4072, 11016, 56, True, "256x128-split"),   # edge tiles belong to the first split
    (520, 4104, 16384, 48, False, "128x128"),
]


@pytest.mark.parametrize("M,N,K,K2,ws,plan", CASES)
def test_edge_tiles(api, H, M, N, K, K2, ws, plan):  # noqa: F811
    assert api.tl_k_gemm_nt_plan(M, N, K, K2, (1 << 26) if ws else 0)[0] == plan
    A, B, A2, B2 = rnd(1, (M, K)), rnd(2, (N, K), 0.05), rnd(3, (M, K2)), rnd(4, (N, K2), 0.05)
    R = rnd(5, (M, N), 1.0, False)
    # operands as column blocks of wider buffers: what lies behind a row's last element must not leak in
    wide = [H.to_dev_bf16(np.concatenate([x, np.full((x.shape[0], 64), 3.0, np.float32)], axis=1)) for x in (A, B, A2, B2)]
    Ad, Bd, A2d, B2d = (w[:, :x.shape[1]] for w, x in zip(wide, (A, B, A2, B2)))
    ref = (torch.from_numpy(A).double() @ torch.from_numpy(B).double().T
           + torch.from_numpy(A2).double() @ torch.from_numpy(B2).double().T).numpy()
    scratch = torch.empty(1 << 26, dtype=torch.float32, device="cuda") if ws else None
    Cf = torch.empty(M, N, dtype=torch.float32, device="cuda")
    Cb = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    api.tl_k_gemm_nt(Ad, Bd, Cf, A2d, B2d, alpha=1.0, R=H.to_dev_f32(R), workspace=scratch)
    api.tl_k_gemm_nt(Ad, Bd, Cb, A2d, B2d, alpha=0.5, workspace=scratch)
    torch.cuda.synchronize()
    check(Cf.cpu().numpy() - R, ref, F32_TOL + 2.0 ** -24 * np.abs(R).max() / ref.std(), "C f32 + R")
    check(H.bf16_to_np(Cb), 0.5 * ref, BF16_TOL, "C bf16")


@pytest.mark.parametrize("M,N,K,K2,ws,plan", [CASES[i] for i in (0, 2, 3, 5, 8)])
def test_undefined_values_beside_the_operands(api, M, N, K, K2, ws, plan):  # noqa: F811
    """What lies behind a row's last element may be anything: the product is bit for bit the same."""
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    wide = [torch.randn(r, c + 64, generator=gen, device="cuda").bfloat16() for r, c in ((M, K), (N, K), (M, K2), (N, K2))]
    scratch = torch.empty(1 << 26, dtype=torch.float32, device="cuda") if ws else None
    out = []
    for behind in (3.0, float("nan"), float("-inf")):
        for w, c in zip(wide, (K, K, K2, K2)):
            w[:, c:] = behind
        C = torch.empty(M, N, dtype=torch.float32, device="cuda")
        api.tl_k_gemm_nt(wide[0][:, :K], wide[1][:, :K], C, wide[2][:, :K2], wide[3][:, :K2], workspace=scratch)
        out.append(C)
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


# contractions split over several workgroups in the two tile shapes that only the model of launch times picks, and products that go
# out as two launches: over two ranges of rows (the second split) and of columns.  F32_TOL holds up to K = 16384.
PARTS = [
    # M, N, K, K2, workspace, plan (of the first launch), launches
    (300, 1096, 8200, 64, True, ("128x128-split", 8, 1)),
    (130, 1096, 16320, 64, True, ("128x128-split", 8, 1)),
    (1000, 2056, 16320, 64, True, ("256x256-split", 4, 1)),
    (1250, 4072, 8200, 64, True, ("256x256-split", 3, 1)),
    (1250, 2040, 11272, 120, True, ("256x128-split", 3, 1)),
    (380, 3064, 8200, 56, True, ("128x128-split", 3, 1)),
    (4300, 4104, 8200, 64, True, ("256x256", 1, 2)),
    (1000, 17000, 4104, 40, False, ("256x256", 1, 2)),
]


@pytest.mark.parametrize("M,N,K,K2,ws,plan", PARTS)
def test_split_tiles_and_two_launches(api, M, N, K, K2, ws, plan):  # noqa: F811
    assert api.tl_k_gemm_nt_plan(M, N, K, K2, (1 << 26) if ws else 0) == plan
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    A, B, A2, B2 = (torch.randn(r, c, generator=gen, device="cuda").bfloat16() for r, c in ((M, K), (N, K), (M, K2), (N, K2)))
    R = torch.randn(M, N, generator=gen, device="cuda")
    scratch = torch.empty(1 << 26, dtype=torch.float32, device="cuda") if ws else None
    Cf, Cb = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda").bfloat16()
    api.tl_k_gemm_nt(A, B, Cf, A2, B2, alpha=1.0, R=R, workspace=scratch)
    api.tl_k_gemm_nt(A, B, Cb, A2, B2, alpha=0.5, workspace=scratch)
    # every row against a sample of columns, the edges of tiles and both ranges among them; and the other way round
    rows, cols = (sorted({i for i in (0, 127, 128, 255, 256, *seam, n - 1) if i < n} | set(range(0, n, step)))
                  for n, seam, step in ((M, (4095, 4096), 97), (N, (16383, 16384), 89)))
    assert max(rows) < M and max(cols) < N
    full = lambda a, b, a2, b2: (a.double().cpu() @ b.double().cpu().T + a2.double().cpu() @ b2.double().cpu().T).numpy()  # noqa: E731
    for r, c in ((slice(None), cols), (rows, slice(None))):
        ref, res = full(A[r], B[c], A2[r], B2[c]), R[r][:, c].cpu().numpy()
        check(Cf[r][:, c].cpu().numpy() - res, ref, F32_TOL + 2.0 ** -24 * np.abs(res).max() / ref.std(), "C f32 + R")
        check(Cb[r][:, c].float().cpu().numpy(), 0.5 * ref, BF16_TOL, "C bf16")
