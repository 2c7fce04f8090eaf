"""Backward attention at the edges of its tiles, against the fp64 oracle.

A part of the launch is a block of 128 (d_head 128) or 64 (d_head 64) keys or queries against 64-row tiles, each taken in two halves of 32
rows; a wave holds 64 or 32 rows of the block.  The lengths lie on both sides of every one of these edges.  What follows row T in memory
is NaN: a row read beyond the last one, and used, shows in the gradients."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import templora_oracle as O  # noqa: E402
from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import BF16_TOL, H, api, check  # noqa: E402,F401


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("T", [2, 31, 32, 33, 63, 65, 95, 97, 127, 128, 160, 191, 193, 257, 320])
def test_edges(api, H, T, dh):
    nh = 3
    d = nh * dh
    rows = T + 70

    def draw(seed, width):
        x = synth.normal(seed, (91, T, width), (T, width), 1.0, True)
        full = np.full((rows, width), np.nan)
        full[:T] = x
        return x, H.to_dev_bf16(full)[:T]
    qkv, qkvd = draw(1, 3 * d)
    do, dod = draw(2, d)
    q, k, v = (qkv[:, i * d:(i + 1) * d].reshape(T, nh, dh) for i in range(3))
    o = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros(nh, T, dtype=torch.float32, device="cuda")
    delta = torch.zeros(nh, T, dtype=torch.float32, device="cuda")
    grads = torch.full((rows, 3 * d), 7.0, dtype=torch.bfloat16, device="cuda")
    args = [qkvd[:, i * d:(i + 1) * d] for i in range(3)]
    api.tl_k_attention_fwd(*args, nh, dh, o, lse)
    api.tl_k_attention_bwd(*args, o, dod, lse, nh, dh, *(grads[:T, i * d:(i + 1) * d] for i in range(3)), delta)
    torch.cuda.synchronize()
    _, P = O.attention_fwd(q, k, v)
    refs = O.attention_bwd(do.reshape(T, nh, dh), q, k, v, P)
    g = H.bf16_to_np(grads)
    assert np.all(g[T:] == 7.0)                    # nothing is written behind the last row
    for i, name in enumerate(("dq", "dk", "dv")):
        check(g[:T, i * d:(i + 1) * d], refs[i].reshape(T, d), BF16_TOL, name, per_row=True)


def gradients(api, H, T, dh, do_edit):
    q, k, v, do = (H.to_dev_bf16(synth.normal(i, (95, T, dh), (T, dh), 1.0, True)) for i in range(4))
    o, dq, dk, dv = (torch.zeros(T, dh, dtype=torch.bfloat16, device="cuda") for _ in range(4))
    lse, delta = (torch.zeros(1, T, dtype=torch.float32, device="cuda") for _ in range(2))
    do_edit(do)
    api.tl_k_attention_fwd(q, k, v, 1, dh, o, lse)
    api.tl_k_attention_bwd(q, k, v, o, do, lse, 1, dh, dq, dk, dv, delta)
    torch.cuda.synchronize()
    return dq, dk, dv


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("T", [1, 33, 100, 193])
def test_infinity_in_the_last_row(api, H, T, dh):
    """One value of the last token's dO is infinite: so is that column of dV for every key, all of which the last token sees, and no other."""
    def edit(do):
        do[-1, 5] = float("inf")
    dv0, dv1 = (gradients(api, H, T, dh, e)[2] for e in (lambda do: None, edit))
    assert torch.all(dv1[:, 5] == float("inf"))
    others = torch.arange(dh, device="cuda") != 5
    assert torch.equal(dv0[:, others], dv1[:, others])


@pytest.mark.parametrize("T,dh", [(100, 64), (100, 128), (128, 128), (200, 128)])
def test_no_number_in_the_first_row_of_a_tile(api, H, T, dh):
    """Keys from 96 on follow token 64 by more than the 32 rows of a piece: what is not a number there stays away from them, also by way of
    the rows that fill a ragged tile up behind the last."""
    def edit(do):
        do[64] = float("nan")
    plain, edited = gradients(api, H, T, dh, lambda do: None), gradients(api, H, T, dh, edit)
    for a, b in zip(plain, edited):
        assert torch.equal(a[96:], b[96:])


def test_rows_far_apart(api, H):
    """Rows so far apart that 127 of them exceed 4 GiB (64 do not): the same as with the rows side by side."""
    T, dh, ld = 150, 128, (1 << 24) + (1 << 20)
    x = H.to_dev_bf16(synth.normal(1, (97, T), (T, 3 * dh), 1.0, True))
    do = H.to_dev_bf16(synth.normal(2, (97, T), (T, dh), 1.0, True))
    outs = []
    for step in (3 * dh, ld):
        src, grads = (torch.empty(T * step, dtype=torch.bfloat16, device="cuda").view(T, step)[:, :3 * dh] for _ in range(2))
        src.copy_(x)
        o, (lse, delta) = torch.zeros_like(do), (torch.zeros(1, T, dtype=torch.float32, device="cuda") for _ in range(2))
        args, outs_ = ([t[:, i * dh:(i + 1) * dh] for i in range(3)] for t in (src, grads))
        api.tl_k_attention_fwd(*args, 1, dh, o, lse)
        api.tl_k_attention_bwd(*args, o, do, lse, 1, dh, *outs_, delta)
        torch.cuda.synchronize()
        outs.append(grads.contiguous())
        del src, grads, args, outs_
    assert torch.equal(outs[0], outs[1])
