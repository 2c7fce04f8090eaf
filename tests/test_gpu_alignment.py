"""Operands of the single kernels that start anywhere: one, two or four elements (2, 4, 8 bytes) behind a multiple of 16 bytes.

Direct-to-LDS loads take multiples of 4 bytes; an operand that starts between them comes through registers.  Attention and the products over
the tokens add in the same order either way: the same bits as aligned.  The products of two contiguous contractions may take another tile: a
tolerance as in test_gpu_low_rank.py (one bf16 rounding of the result)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import H, api  # noqa: E402,F401

OFFSETS = [1, 2, 4]


def at(x, n):
    """x in memory that starts n elements behind a multiple of 16 bytes, rows 8 elements further apart; NaN around it"""
    rows, cols = x.shape
    ld = (cols + 15) // 8 * 8
    flat = torch.full((rows * ld + 64,), float("nan"), dtype=x.dtype, device="cuda")
    view = flat[n:n + rows * ld].view(rows, ld)[:, :cols]
    view.copy_(x)
    assert view.data_ptr() % 16 == n * x.element_size()
    return view


def draw(H, seed, rows, cols, std=1.0):
    return H.to_dev_bf16(synth.normal(seed, (98, rows, cols), (rows, cols), std, True))


@pytest.mark.parametrize("n", OFFSETS)
@pytest.mark.parametrize("T,Mo,No", [(1, 8, 8), (200, 72, 136), (449, 64, 8)])
def test_products_over_the_tokens(api, H, T, Mo, No, n):
    P, Q = draw(H, 1, T, Mo), draw(H, 2, T, No)
    outs = [torch.zeros(Mo, No, device="cuda") for _ in range(4)]
    for out, p, q in zip(outs, (P, at(P, n), at(P, n), P), (Q, Q, at(Q, n), at(Q, n))):
        api.tl_k_gemm_tn(p, q, out)
    torch.cuda.synchronize()
    assert all(torch.equal(outs[0], o) for o in outs[1:])


@pytest.mark.parametrize("n", OFFSETS)
@pytest.mark.parametrize("T,nh,dh", [(1, 2, 64), (100, 2, 64), (321, 2, 64), (33, 2, 128), (129, 2, 128), (333, 2, 128)])
def test_attention(api, H, T, nh, dh, n):
    d = nh * dh
    x, do = [draw(H, i, T, d) for i in range(3)], draw(H, 4, T, d)

    def run(place):
        q, k, v = (place(t) for t in x)
        o, dq, dk, dv = (place(torch.zeros_like(do)) for _ in range(4))
        lse, delta = (torch.zeros(nh, T, device="cuda") for _ in range(2))
        api.tl_k_attention_fwd(q, k, v, nh, dh, o, lse)
        api.tl_k_attention_bwd(q, k, v, o, place(do), lse, nh, dh, dq, dk, dv, delta)
        torch.cuda.synchronize()
        return o, lse, dq, dk, dv
    for a, b in zip(run(lambda t: at(t, 0)), run(lambda t: at(t, n))):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", OFFSETS)
@pytest.mark.parametrize("M,N,K,nb", [(37, 24, 1000, 1), (200, 48, 72, 3), (300, 64, 4096, 1), (1020, 56, 2048, 3)])
def test_low_rank(api, H, M, N, K, nb, n):
    A, B = draw(H, 1, M, nb * K), draw(H, 2, nb * N, K, 0.05)
    out = torch.zeros(M, nb * N, dtype=torch.bfloat16, device="cuda")
    api.tl_k_low_rank(at(A, n), at(B, n), out, nb, 0.5, torch.empty(16 << 20, device="cuda"))
    torch.cuda.synchronize()
    A64, B64 = A.double(), B.double()
    ref = torch.cat([A64[:, i * K:(i + 1) * K] @ B64[i * N:(i + 1) * N].T for i in range(nb)], 1) * 0.5
    err = out.double() - ref
    assert err.norm() <= 2e-3 * ref.norm()
    assert err.abs().max() <= 2e-2 * ref.norm() / ref.numel() ** 0.5


@pytest.mark.parametrize("n", OFFSETS)
@pytest.mark.parametrize("M,N,K,K2", [(200, 256, 688, 16), (300, 320, 1000, 72), (1024, 1024, 1024, 64), (1200, 2560, 512, 0)])
def test_frozen(api, H, M, N, K, K2, n):
    """two operand pairs, as tl_k_gemm_nt takes them"""
    A, B = draw(H, 1, M, K), draw(H, 2, N, K, 0.05)
    A2, B2 = (draw(H, 3, M, K2), draw(H, 4, N, K2, 0.05)) if K2 else (None, None)
    out = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
    api.tl_k_gemm_nt(at(A, n), at(B, n), out, *((at(A2, n), at(B2, n)) if K2 else ()))
    torch.cuda.synchronize()
    ref = A.double() @ B.double().T
    if K2:
        ref += A2.double() @ B2.double().T
    err = out.double() - ref
    assert err.norm() <= 2e-3 * ref.norm()
    assert err.abs().max() <= 2e-2 * ref.norm() / ref.numel() ** 0.5
