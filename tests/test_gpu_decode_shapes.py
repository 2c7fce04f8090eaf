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
