"""The loss kernel where its row forms meet: rows of up to 8192 and up to 32768 entries stay in registers, longer ones are
read twice.  Reference: the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import templora_oracle as O  # noqa: E402
from test_gpu_kernels import BF16_TOL, F32_TOL, H, api, check, rnd  # noqa: E402,F401


@pytest.mark.parametrize("T,V,n_ctx", [(5, 8, 0), (17, 8192, 3), (17, 8200, 3), (9, 32768, 0), (9, 32776, 0)])
def test_row_forms(api, H, T, V, n_ctx):  # noqa: F811
    z = rnd(1, (T, V), 3.0, False)
    labels = np.roll(np.arange(T) * 7919 % V, -1)
    labels[0], labels[-1] = V - 1, -1
    first = max(n_ctx, 1) - 1
    N = T - 1 - first
    nll, dl = torch.empty(T, device="cuda"), torch.full((T, V), 3.0, dtype=torch.bfloat16, device="cuda")
    ls = torch.empty(4, device="cuda")
    api.tl_k_cross_entropy(H.to_dev_f32(z), torch.from_numpy(labels.astype(np.int32)).cuda(), first, N, nll, dl, ls)
    mask = np.zeros(T, bool)
    mask[first:T - 1] = True
    loss, rnll, rdl = O.cross_entropy(z, labels, mask)
    check(nll.cpu().numpy(), rnll, F32_TOL, "nll")
    check(H.bf16_to_np(dl), rdl, BF16_TOL, "dlogits")
    assert abs(float(ls[0]) / N - loss) <= F32_TOL * loss
