"""Forward attention at the edges of its tiles, against the fp64 oracle.

A block is 128 queries, a wave 32 of them; two groups of waves take the 64-key tiles in turn, and the queries come through the buffer
that the second pair of tiles lands in.  The lengths lie on both sides of these edges: one tile (the second group has none), an odd and
an even number, a ragged last one.  What follows row T in memory is NaN: a row read beyond the last one, and used, shows in the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import templora_oracle as O  # noqa: E402
from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import BF16_TOL, H, api, check  # noqa: E402,F401


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("T", [1, 31, 33, 63, 64, 65, 97, 127, 128, 129, 192, 193, 256, 321])
def test_edges(api, H, T, dh):
    nh = 3
    d = nh * dh
    x = synth.normal(1, (92, T, 3 * d), (T, 3 * d), 1.0, True)
    full = np.full((T + 140, 3 * d), np.nan)
    full[:T] = x
    qkvd = H.to_dev_bf16(full)[:T]
    out = torch.full((T + 140, d), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros(nh, T, dtype=torch.float32, device="cuda")
    api.tl_k_attention_fwd(*(qkvd[:, i * d:(i + 1) * d] for i in range(3)), nh, dh, out[:T], lse)
    torch.cuda.synchronize()
    q, k, v = (x[:, i * d:(i + 1) * d].reshape(T, nh, dh).astype(np.float64) for i in range(3))
    ref, _ = O.attention_fwd(q, k, v)
    got = H.bf16_to_np(out)
    assert np.all(got[T:] == 7.0)                  # nothing is written behind the last row
    check(got[:T], ref.reshape(T, d), BF16_TOL, "o", per_row=True)
    S = np.einsum("thd,uhd->htu", q, k) / np.sqrt(dh)
    S = np.where(np.triu(np.ones((T, T), bool), 1)[None], -np.inf, S)
    ref_lse = np.logaddexp.reduce(S, axis=-1)
    assert np.abs(lse.cpu().numpy() - ref_lse).max() < 2e-3


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("T", [1, 33, 100, 193])
def test_infinity_in_the_last_row(api, H, T, dh):
    """One value of the last token is infinite: so is the output that it has a weight in, and no other output of that row changes.  (Rows that fill a
    tile up behind the last have weights of 0, and 0 x inf is no number.)"""
    q, k, v = (H.to_dev_bf16(synth.normal(i, (94, T, dh), (T, dh), 1.0, True)) for i in range(3))
    lse = torch.zeros(1, T, dtype=torch.float32, device="cuda")
    out = [torch.zeros(T, dh, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    api.tl_k_attention_fwd(q, k, v, 1, dh, out[0], lse)
    v[-1, 5] = float("inf")
    api.tl_k_attention_fwd(q, k, v, 1, dh, out[1], lse)
    torch.cuda.synchronize()
    assert out[1][-1, 5] == float("inf")
    others = torch.arange(dh, device="cuda") != 5
    assert torch.equal(out[0][:, others], out[1][:, others])


def test_rows_far_apart(api, H):
    """Rows so far apart that 127 of them exceed 4 GiB (64 do not): the same as with the rows side by side."""
    T, dh = 150, 64
    x = H.to_dev_bf16(synth.normal(1, (96, T), (T, 3 * dh), 1.0, True))
    ld = (1 << 24) + (1 << 20)
    far = torch.empty(T * ld, dtype=torch.bfloat16, device="cuda").view(T, ld)[:, 8:8 + 3 * dh]
    far.copy_(x)
    outs = []
    for src in (x, far):
        o, lse = torch.zeros(T, dh, dtype=torch.bfloat16, device="cuda"), torch.zeros(1, T, dtype=torch.float32, device="cuda")
        api.tl_k_attention_fwd(*(src[:, i * dh:(i + 1) * dh] for i in range(3)), 1, dh, o, lse)
        outs.append((o, lse))
    torch.cuda.synchronize()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
