"""The input gradient of gate|up, at ranks that are multiples of 64 with the contraction of the low-rank pair (2 r) and at others:
its sum is kept in fp32 wherever the contraction is cut.  The case is built so that the gate half and the up half of the sum are large and nearly cancel: partial sums rounded to
bf16 leave an error of the size of the halves.  One size for every instance that leaves partial tiles to the norm.  Reference: fp64 from
the same bf16 operands."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import H, api  # noqa: E402,F401

G = -2.2178     # silu(g) + g silu'(g) = 0 here: with u = -g the two halves are opposite
# dgate and dup are stored in bf16: F independent roundings of 2^-9 / sqrt(3) at most, averaged: 1.5e-5 of a half (F 704: 4.3e-5).  Halves
# rounded to bf16 would be off by about 2^-9 / sqrt(3) x 0.7 each, 1e-3 in all.
TOL = 1e-4


CASES = [(1024, 2048, 5632, rank, ("256x128-split", 4)) for rank in (8, 16, 32, 40, 64)] + [
    (520, 4096, 5632, 32, ("256x256-split", 4)),
    (1250, 4096, 5632, 64, ("256x256-split", 3)),
    (300, 1024, 5632, 64, ("128x128-split", 8)),
    (200, 128, 704, 16, ("64x64-split", 5)),
]


@pytest.mark.parametrize("T,D,F,rank,plan", CASES)
def test_gate_up_input_gradient_is_summed_in_fp32(api, H, T, D, F, rank, plan):  # noqa: F811
    assert api.tl_k_gemm_nt_plan(T, D, 2 * F, 2 * rank, D * max(4 * T, 8 * min(T, 1024)))[:2] == plan     # (a session's scratch)
    rng = np.random.default_rng(rank)
    z = np.repeat(rng.normal(0, 0.02, D // 2), 2) * np.tile([1.0, -1.0], D // 2)     # no component along the rows of h
    row = synth.round_bf16((G / D + z).astype(np.float32))
    w_down = synth.round_bf16(rng.uniform(0.5, 1.0, F).astype(np.float32) / D)
    tau = synth.round_bf16(rng.uniform(0.5, 1.0, T).astype(np.float32))
    zero = torch.zeros(D, D, dtype=torch.bfloat16, device="cuda")      # no attention branch: the FFN sees h_in itself
    gate = H.to_dev_bf16(np.tile(row, (F, 1)))
    ones = torch.ones(D, device="cuda")
    weights = [zero, zero, zero, zero, gate, -gate, H.to_dev_bf16(np.tile(w_down, (D, 1))), ones, ones, None, None, None]
    model = api.tl_model_create(1, D, D // 128, 128, F, 0, T, weights, 1e-5, 10000.0)
    lora = api.tl_lora_init(model, rank, float(rank), seed=1)          # B = 0
    h_in = torch.ones(T, D, device="cuda")
    dh_out = H.to_dev_f32(np.tile(tau[:, None], (1, D)))
    h_out, dh_in = torch.empty_like(h_in), torch.empty_like(h_in)
    api.tl_layer_step(lora, 0, h_in, dh_out, h_out, dh_in)
    torch.cuda.synchronize()

    r64 = lambda x: synth.round_bf16(np.asarray(x, np.float32)).astype(np.float64)  # noqa: E731
    a = row.astype(np.float64)
    g = float(r64([a.sum()])[0])                                       # x = bf16(1 / sqrt(1 + 1e-5)) = 1
    sig = 1.0 / (1.0 + np.exp(-g))
    da = r64(np.outer(tau, w_down.astype(np.float64)) * D)
    dgate, dup = r64(da * -g * (sig + g * sig * (1.0 - sig))), r64(da * g * sig)
    dx = np.outer(dgate.sum(1) - dup.sum(1), a)
    rho = 1.0 / np.sqrt(1.0 + 1e-5)
    xn = rho * np.ones(D)
    want = tau[:, None] + rho * (dx - xn * (dx @ xn / D)[:, None])
    half = np.linalg.norm(np.outer(dup.sum(1), a))
    got = dh_in.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(dx) < 0.05 * half                            # the halves do cancel
    err = np.linalg.norm(got - want) / half
    assert err < TOL, err
    api.tl_lora_free(lora)
    api.tl_model_destroy(model)


@pytest.mark.parametrize("max_tokens", [1001, 1024, 1025, 1500])
def test_a_longer_window_splits_a_sample_no_less(api, H, max_tokens):  # noqa: F811
    """dX of gate|up is cut in eight here; the scratch for that does not shrink where the window grows."""
    shape, n = synth.Shape(1, 256, 4, 64, 4096, 0, 16, 16.0), 1000
    h, dy = H.to_dev_f32(synth.hidden(6500, n, 256)), H.to_dev_f32(synth.upstream_grad(6500, n, 256))
    out = []
    for window in (n, max_tokens):
        model = H.Model(shape, 6500, max_tokens=window)
        lora, _ = H.new_lora(model, 6500, b_std=0.05)
        h_out, dh_in = torch.empty_like(h), torch.empty_like(h)
        api.tl_layer_step(lora, 0, h, dy, h_out, dh_in)
        out.append((h_out, dh_in))
        api.tl_lora_free(lora)
        model.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
