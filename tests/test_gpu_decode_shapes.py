"""One decoded token at shapes where its launches can go wrong: feed-forward widths that do not fill the last SwiGLU piece,
ranks that do not divide a workgroup or exceed a wave, one and several key ranges, a key range longer than one trip.
Reference: the same window through the chunk path, which shares none of those kernels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_kernels import H, api, check  # noqa: E402,F401


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
# it, beyond that they take its place after the product, and 81920 is the widest vector.
@pytest.mark.parametrize("d_ffn,rank", [(80896, 8), (80904, 256), (80904, 8), (81888, 40), (81920, 16)])
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
    W, x, y = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for n in (81928, 81928, 8))
    with pytest.raises(api.TlError):
        api.tl_k_gemv(W.view(1, -1), x, y[:1])
    h = torch.zeros(81896, device="cuda")               # a norm also needs its block sums there
    with pytest.raises(api.TlError):
        api.tl_k_gemv_pre(W[:81896].view(1, -1), h[:1], 1, h=h, gain=h, eps=1e-5)
