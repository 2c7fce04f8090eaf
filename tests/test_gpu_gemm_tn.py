"""P^T Q over the tokens (gradients of the adapters) at the edges of its 64 x 64 tiles and of the ring of token tiles, against fp64.

The token counts lie on both sides of one tile, of the ring's depth and of a ragged last tile; the widths are single 8-column chunks, whole
tiles and a chunk more.  Everything around the operands is NaN: a row behind the last token, or a column behind the last, that is used
shows in the result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import H, api  # noqa: E402,F401


@pytest.mark.parametrize("Mo,No", [(8, 8), (8, 72), (64, 64), (72, 136), (128, 8)])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 128, 192, 193, 256, 257, 320, 449])
def test_edges(api, H, T, Mo, No):
    def draw(seed, width):
        x = synth.normal(seed, (93, T, width), (T, width), 1.0, True)
        full = np.full((T + 64, width + 64), np.nan)
        full[:T, 8:8 + width] = x
        return x.astype(np.float64), H.to_dev_bf16(full)[:T, 8:8 + width]
    P, Pd = draw(1, Mo)
    Q, Qd = draw(2, No)
    C = torch.full((Mo + 8, No + 8), 7.0, dtype=torch.float32, device="cuda")
    api.tl_k_gemm_tn(Pd, Qd, C[:Mo, :No], alpha=0.5)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    # bf16 products are exact in fp32: T terms of fp32 rounding, 2^-24 each, against the sum of their magnitudes
    bound = 0.5 * (np.abs(P).T @ np.abs(Q)) * (T + 8) * 2.0 ** -24
    assert np.all(np.abs(got[:Mo, :No] - 0.5 * (P.T @ Q)) <= bound)
    assert np.all(got[Mo:] == 7.0) and np.all(got[:, No:] == 7.0)
