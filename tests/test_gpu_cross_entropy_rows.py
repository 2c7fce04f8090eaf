"""The loss kernel where its row forms meet: rows of up to 32768 entries stay in registers, in seven sizes, longer ones are read
twice.  Reference: the oracle."""
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


# the edges of the register forms, with and without a gradient; 600 rows without one take the two-pass form above 24576 entries
@pytest.mark.parametrize("T,V", [(4, 1024), (4, 1032), (4, 4096), (4, 4104), (3, 12288), (3, 12296), (3, 16384), (3, 16392),
                                 (3, 24576), (3, 24584), (260, 16392), (600, 24576), (600, 24584)])
def test_register_forms(api, H, T, V):  # noqa: F811
    z = rnd(V, (T, V), 3.0, False)
    labels = np.roll(np.arange(T) * 7919 % V, -1)
    labels[0], labels[-1] = V - 1, -1
    mask = np.ones(T, bool)
    mask[-1] = False
    loss, rnll, rdl = O.cross_entropy(z, labels, mask)
    zd, ld = H.to_dev_f32(z), torch.from_numpy(labels.astype(np.int32)).cuda()
    for dl in (torch.full((T, V), 3.0, dtype=torch.bfloat16, device="cuda"), None):
        nll, ls = torch.empty(T, device="cuda"), torch.empty(4, device="cuda")
        api.tl_k_cross_entropy(zd, ld, 0, T - 1, nll, dl, ls)
        check(nll.cpu().numpy(), rnll, F32_TOL, "nll")
        assert abs(float(ls[0]) / (T - 1) - loss) <= F32_TOL * loss
        if dl is not None:      # entry by entry (1/N at the labels, 1e-8 elsewhere): half a bf16 ulp, 2^-9, and the exponential's 1e-5
            assert (np.abs(H.bf16_to_np(dl) - rdl) <= 2.0 ** -8 * np.abs(rdl)).all()


# An infinite or undefined logit shows in its own row's loss and gradient, whatever the form, and in no other row.
@pytest.mark.parametrize("V", [1000, 8200, 20000, 32768, 32776])
def test_non_finite_logits(api, H, V):  # noqa: F811
    T = 6
    z = rnd(V, (T, V), 3.0, False)
    z[0, V // 2], z[1, 0], z[2, V - 1], z[3, 1:] = np.nan, np.inf, -np.inf, -np.inf
    labels = np.full(T, 2)
    labels[3], labels[-1] = 0, -1
    dl, nll = torch.empty((T, V), dtype=torch.bfloat16, device="cuda"), torch.empty(T, device="cuda")
    ls = torch.empty(4, device="cuda")
    api.tl_k_cross_entropy(H.to_dev_f32(z), torch.from_numpy(labels.astype(np.int32)).cuda(), 0, T - 1, nll, dl, ls)
    nll, dl = nll.cpu().numpy(), H.bf16_to_np(dl)
    assert np.isnan(nll[:2]).all() and np.isnan(dl[0]).all() and np.isnan(dl[1, 0])
    ok = np.array([False, False, True, False, True, False])         # rows whose value the oracle has
    z[:2] = z[3] = 0.0
    z[2, V - 1] = -1e4                                              # its exponential is zero as well
    _, rnll, rdl = O.cross_entropy(z, labels, np.arange(T) < T - 1)
    check(nll[ok], rnll[ok], F32_TOL, "nll")
    assert (np.abs(dl[ok] - rdl[ok]) <= 2.0 ** -8 * np.abs(rdl[ok])).all()      # as above
