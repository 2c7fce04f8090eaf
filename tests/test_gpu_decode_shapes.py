"""One decoded token at shapes where its launches can go wrong: feed-forward widths that do not fill the last SwiGLU piece,
ranks that do not divide a workgroup or exceed a wave, one and several key ranges, a key range longer than one trip.
Reference: the same window through the chunk path, which shares none of those kernels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import templora_oracle as O  # noqa: E402
from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import BF16_TOL, H, api, check, rnd  # noqa: E402,F401


@pytest.mark.parametrize("heads,d_head,d_ffn,rank,n", [
    (2, 64, 328, 24, 2), (3, 64, 1000, 8, 129), (2, 128, 8, 200, 300), (4, 128, 1416, 72, 383), (2, 64, 136, 256, 384),
    (1, 128, 264, 40, 1000), (2, 128, 2048, 64, 4200), (5, 64, 520, 16, 8300)])
def test_decoded_token_is_the_chunk_path_s(api, H, heads, d_head, d_ffn, rank, n):  # noqa: F811
    shape = synth.Shape(2, heads * d_head, heads, d_head, d_ffn, 504, rank, float(rank))
    model = H.Model(shape, 77, max_tokens=n + 2)
    lora, _ = H.new_lora(model, 77, b_std=0.02)
    tok = synth.zipf_tokens(77, n + 1, shape.vocab)
    api.tl_prefill(lora, tok[:n - 1], shape.vocab)
    nxt, first = api.tl_decode_step(lora, int(tok[n - 1]), shape.vocab)
    assert nxt == int(np.argmax(first))
    _, second = api.tl_decode_step(lora, int(tok[n]), shape.vocab)       # reads the key and value the first one wrote
    _, want = api.tl_prefill(lora, tok[:n], shape.vocab)
    check(first, want, 1e-2, "first token")
    _, want = api.tl_prefill(lora, tok[:n + 1], shape.vocab)
    check(second, want, 1e-2, "second token")
    api.tl_lora_free(lora)
    model.close()


# The down projection's input vector is kept in LDS (160 KB): up to 80896 entries the sums of the low-rank shares fit behind
# it, beyond that they take its place after the product, and 81888 is the widest vector (a norm's block sums stand beside it).
@pytest.mark.parametrize("d_ffn,rank", [(80896, 8), (80904, 256), (80904, 8), (81888, 40)])
def test_widest_feed_forward(api, H, d_ffn, rank):  # noqa: F811
    shape = synth.Shape(1, 128, 2, 64, d_ffn, 504, rank, float(rank))
    model = H.Model(shape, 78, max_tokens=12)
    lora, _ = H.new_lora(model, 78, b_std=0.02)
    tok = synth.zipf_tokens(78, 10, shape.vocab)
    api.tl_prefill(lora, tok[:9], shape.vocab)
    _, got = api.tl_decode_step(lora, int(tok[9]), shape.vocab)
    _, want = api.tl_prefill(lora, tok, shape.vocab)
    check(got, want, 1e-2, "logits")
    api.tl_lora_free(lora)
    model.close()


def test_wider_input_vectors_are_refused(api, H):  # noqa: F811
    W, x, y = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for n in (81896, 81896, 8))
    with pytest.raises(api.TlError):
        api.tl_k_gemv(W.view(1, -1), x, y[:1])
    h = torch.zeros(81896, device="cuda")
    with pytest.raises(api.TlError):
        api.tl_k_gemv_pre(W.view(1, -1), h[:1], 1, h=h, gain=h, eps=1e-5)


# on both sides of where a product behind a norm changes kernels (512 rows of more than 4096 columns), and where a long row's last
# trip changes length (4096 columns a trip, 1024 a step of the last one); two rows per wave from 8192 rows on
@pytest.mark.parametrize("N,K", [(520, 1024), (520, 1032), (512, 1032), (512, 4096), (512, 4104), (516, 4104), (3, 8), (514, 5120),
                                 (514, 5128), (514, 6144), (514, 6152), (514, 7176), (514, 8192), (514, 8200), (514, 9224),
                                 (514, 12288), (514, 13824), (514, 16392), (8195, 5120), (8193, 9216)])
def test_product_behind_a_norm(api, H, N, K):  # noqa: F811
    W, h, gain = rnd(1, (N, K), 0.05), rnd(2, (1, K), 2.0, False), 1.0 + rnd(3, (1, K), 0.1, False)[0]
    y, xo = torch.empty(N, device="cuda"), torch.empty(K, dtype=torch.bfloat16, device="cuda")
    api.tl_k_gemv_pre(H.to_dev_bf16(W), y, 1, h=H.to_dev_f32(h[0]), gain=H.to_dev_f32(gain), eps=1e-5, x_out=xo)
    x = H.bf16_to_np(xo).astype(np.float64)
    check(x, O.rmsnorm_fwd(h, gain, 1e-5)[0], BF16_TOL, "x")
    # K products summed in fp32: sqrt(16392) 2^-24 = 7.6e-6 of the sum's 2-norm; the lanes' chains are K / 64 long
    check(y.cpu().numpy(), W.astype(np.float64) @ x, 1e-5, "y")


# values are read sixteen bytes at a time from 16384 on, if they start on such a boundary
@pytest.mark.parametrize("n", [1, 1025, 16383, 16384, 16387, 32769])
@pytest.mark.parametrize("off", [0, 1])
def test_argmax_takes_the_first_of_equal_values(api, n, off):  # noqa: F811
    x = rnd(n, (1, n + 1), 1.0, False)[0]
    at = sorted({n - 1, n // 2, (n - 1) // 3})
    out = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for first in range(len(at)):
        x[off:][at[first:]] = 9.0 + first
        api.tl_k_argmax(torch.from_numpy(x).cuda()[off:off + n], out)
        assert int(out[0]) == at[first], (n, off, at)


# What the attention entry refuses: more than 30208 keys without scratch, and ranges of more than 13312 keys where the scratch
# holds too few of them.
@pytest.mark.parametrize("n_keys,ranges,ok", [(30208, 0, True), (30209, 0, False), (26624, 2, True), (26625, 2, False),
                                              (26625, 3, True), (40001, 3, False)])
def test_key_counts_that_attention_takes(api, n_keys, ranges, ok):  # noqa: F811
    dh = 64
    kv = torch.randn(n_keys, 2 * dh, device="cuda").bfloat16()
    q, o = torch.randn(dh, device="cuda").bfloat16(), torch.zeros(dh, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(ranges * (dh + 2), device="cuda") if ranges else None
    call = lambda: api.tl_k_attention_decode(q, kv[:, :dh], kv[:, dh:], 1, dh, o, workspace=ws)  # noqa: E731
    if not ok:
        with pytest.raises(api.TlError):
            call()
        return
    call()
    k, v = kv[:, :dh].double(), kv[:, dh:].double()
    want = torch.softmax(k @ q.double() / dh ** 0.5, 0) @ v
    check(o.double().cpu().numpy(), want.cpu().numpy(), BF16_TOL, "o")


# Values that are not finite: behind the last key they are not seen (the rest of a cache holds anything), in a key they make the
# whole head undefined, in a value the columns they stand in.
@pytest.mark.parametrize("n_keys,ranges", [(1, 0), (5, 0), (129, 0), (400, 0), (400, 32), (4100, 32)])
@pytest.mark.parametrize("dh", [64, 128])
def test_attention_and_non_finite_values(api, n_keys, ranges, dh):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(n_keys)
    kv = torch.full((n_keys + 300, 4 * dh), float("nan"), device="cuda").bfloat16()     # two heads: k k v v
    kv[:n_keys] = torch.randn(n_keys, 4 * dh, generator=gen, device="cuda").bfloat16()
    q, o = torch.randn(2 * dh, generator=gen, device="cuda").bfloat16(), torch.zeros(2 * dh, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(2 * ranges * (dh + 2), device="cuda") if ranges else None

    def run():
        api.tl_k_attention_decode(q, kv[:n_keys, :2 * dh], kv[:n_keys, 2 * dh:], 2, dh, o, workspace=ws)
        return o.double().cpu().view(2, dh)

    k, v = kv[:n_keys, :2 * dh].double().cpu().view(-1, 2, dh), kv[:n_keys, 2 * dh:].double().cpu().view(-1, 2, dh)
    want = torch.stack([torch.softmax(k[:, h] @ q.double().cpu().view(2, dh)[h] / dh ** 0.5, 0) @ v[:, h] for h in range(2)])
    check(run().numpy(), want.numpy(), BF16_TOL, "o")
    at = (n_keys - 1) // 2
    keep = kv[at].clone()
    kv[at, 2 * dh + 3] = float("inf")             # a value of head 0
    got = run()
    assert not torch.isfinite(got[0, 3]) and torch.isfinite(got).sum() == 2 * dh - 1
    kv[at] = keep
    kv[at, dh + 3] = float("nan")                 # a key of head 1
    got = run()
    assert torch.isfinite(got[0]).all() and torch.isnan(got[1]).all()


# o and down at every length of a long row's last trip, a norm of more than 4096 entries in front of q|k|v and gate|up, and outputs
# of 8192 rows and more, two per wave
@pytest.mark.parametrize("heads,d_head,d_ffn", [(2, 64, 4104), (2, 64, 5128), (2, 64, 6152), (2, 64, 7176), (2, 64, 8200), (2, 64, 13824),
                                                (36, 128, 520), (66, 128, 1032)])
def test_long_rows_of_one_token(api, H, heads, d_head, d_ffn):  # noqa: F811
    shape = synth.Shape(1, heads * d_head, heads, d_head, d_ffn, 504, 24, 24.0)
    model = H.Model(shape, 79, max_tokens=34)
    lora, _ = H.new_lora(model, 79, b_std=0.02)
    tok = synth.zipf_tokens(79, 33, shape.vocab)
    api.tl_prefill(lora, tok[:32], shape.vocab)
    _, got = api.tl_decode_step(lora, int(tok[32]), shape.vocab)
    _, want = api.tl_prefill(lora, tok, shape.vocab)
    check(got, want, 1e-2, "logits")
    api.tl_lora_free(lora)
    model.close()


# more key ranges than fit on the chip at once are made fewer and longer: on both sides of the line, in one and two trips over a range
@pytest.mark.parametrize("n_keys,heads,dh", [(2048, 32, 128), (2049, 32, 128), (4095, 32, 64), (3000, 40, 64), (1500, 70, 64)])
def test_attention_in_one_round_of_ranges(api, n_keys, heads, dh):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(n_keys + heads)
    kv = torch.randn(n_keys, 2 * heads * dh, generator=gen, device="cuda").bfloat16()
    q, o = torch.randn(heads * dh, generator=gen, device="cuda").bfloat16(), torch.zeros(heads * dh, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(heads * 32 * (dh + 2), device="cuda")
    api.tl_k_attention_decode(q, kv[:, :heads * dh], kv[:, heads * dh:], heads, dh, o, workspace=ws)
    k, v = (x.double().cpu().view(n_keys, heads, dh) for x in (kv[:, :heads * dh], kv[:, heads * dh:]))
    w = torch.softmax(torch.einsum("khd,hd->hk", k, q.double().cpu().view(heads, dh)) / dh ** 0.5, 1)
    want = torch.einsum("hk,khd->hd", w, v)
    check(o.double().cpu().view(heads, dh).numpy(), want.numpy(), BF16_TOL, "o")
