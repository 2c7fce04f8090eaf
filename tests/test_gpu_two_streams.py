"""Updates whose dA / dB products and AdamW steps run on the second stream (2^20 values of a layer's input or more, but for the bottom
layer): the gradients and the carried state against the oracle, the same bits from the same state, a loss that is not finite."""
import os
import sys

import numpy as np
import pytest
import torch  # noqa: F401

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from paper_2401_11504_amd import synth  # noqa: E402
from test_gpu_dropout import test_chunk_update_with_dropout_matches_oracle as two_updates  # noqa: E402
from test_gpu_kernels import H, api  # noqa: E402,F401

pytestmark = pytest.mark.gpu
T, LR = 1024, 1e-3
WIDE = synth.Shape(3, 1024, 16, 64, 704, 1000, 16, 16.0)
SELECT = ("FACTOR_A", "M_A", "V_A", "GRAD_A", "FACTOR_B", "M_B", "V_B", "GRAD_B")


def _state(api, lora, which=SELECT):  # noqa: F811
    return [api.tl_get_factor(lora, l, i, getattr(api, w), (WIDE.rank, WIDE.proj_dims(p)[1]) if w[-1] == "A" else
                              (WIDE.proj_dims(p)[0], WIDE.rank))
            for l in range(WIDE.n_layers) for i, p in enumerate(synth.PROJ) for w in which]


@pytest.mark.parametrize("p,n_ctx", [(0.0, 0), (0.05, 100)])
def test_two_updates_match_the_oracle(api, H, monkeypatch, p, n_ctx):  # noqa: F811
    monkeypatch.setitem(synth.SHAPES, "wide", WIDE)
    two_updates(api, H, "wide", T, n_ctx, p)


@pytest.mark.parametrize("p", [0.0, 0.05])
def test_same_bits_from_the_same_state(api, H, p):  # noqa: F811
    model = H.Model(WIDE, 6406, max_tokens=T)
    tok = synth.uniform_tokens(6406, T, WIDE.vocab)
    out = []
    for _ in range(2):
        lora, _ = H.new_lora(model, 6406, b_std=0.01, dropout=p)
        losses = [api.tl_chunk_update(lora, tok, 0, LR)[0] for _ in range(3)]
        out.append((losses, _state(api, lora)))
        api.tl_lora_free(lora)
    assert out[0][0] == out[1][0]
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)
    model.close()


@pytest.mark.parametrize("layer", [0, 2])
def test_a_loss_that_is_not_finite_changes_nothing(api, H, layer):  # noqa: F811
    model = H.Model(WIDE, 6407, max_tokens=T)
    tok = synth.uniform_tokens(6407, T, WIDE.vocab)
    lora, _ = H.new_lora(model, 6407, b_std=0.01)
    api.tl_chunk_update(lora, tok, 0, LR)
    healthy = api.tl_get_factor(lora, layer, 3, api.FACTOR_B, (WIDE.d_model, WIDE.rank))
    poisoned = healthy.copy()
    poisoned[3, 2] = np.inf
    kept = tuple(w for w in SELECT if "GRAD" not in w)
    want = _state(api, lora, kept)
    api.tl_set_factor(lora, layer, 3, api.FACTOR_B, poisoned)
    with pytest.raises(api.TlError) as e:
        api.tl_chunk_update(lora, tok, 0, LR)
    assert e.value.status == -5 and api.tl_get_step(lora) == 1
    api.tl_set_factor(lora, layer, 3, api.FACTOR_B, healthy)
    for a, b in zip(want, _state(api, lora, kept)):
        assert np.array_equal(a, b)
    assert np.isfinite(api.tl_chunk_update(lora, tok, 0, LR)[0])
    api.tl_lora_free(lora)
    model.close()
