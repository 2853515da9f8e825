"""The encoder's recurrence over the rows valid at each position: masks with holes, sentences
without a valid position, row counts around the 32-row groups and the 16-row blocks, depths that
are no multiple of a k-step, against the oracle's encoder at every position."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mtref
from paper_1804_00344_amd import synth
from parity_util import TOL, maxerr

if torch.cuda.is_available():
    from paper_1804_00344_amd import mtstep as mt
    from paper_1804_00344_amd.runner import Decoder

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def encoder(gemm, E, H, src_V, T, ln):
    p = synth.with_sizes(synth.PRESETS["tiny_bf16_ln" if gemm == "bf16" else "tiny_f32"], E=E, H=H, A=32)
    w = synth.make_weights(p)
    ew = synth.make_encoder_weights(p, src_V, transitions=T, layer_norm=ln)
    dec = Decoder(p.E, p.H, p.A, p.V, {**w, **ew}, gemm=gemm, layer_norm=p.layer_norm, k_max=4, src_V=src_V,
                  enc_transitions=T, enc_layer_norm=ln)
    return p, ew, dec


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,T,ln", [(1, 64, 0, False), (16, 80, 0, False), (17, 208, 0, False), (33, 64, 0, False),
                                      (65, 1024, 0, False), (33, 80, 1, True), (65, 64, 0, True)])
def test_encoder_masks_with_holes(B, H, T, ln, gemm):
    S, src_V = 6, 60
    p, ew, dec = encoder(gemm, 48, H, src_V, T, ln)
    rng = np.random.default_rng(B + H)
    mask = (rng.random((B, S)) < 0.6).astype(np.float32)
    mask[:, S - 2] = 1.0       # a position with every row,
    mask[:, 2] = 0.0           # one with none
    mask[0, 1:] = 0.0
    mask[0, 0] = 1.0
    if B > 1:
        mask[B - 1] = 0.0      # a sentence without a valid position
    src = rng.integers(0, src_V, size=(B, S)).astype(np.int32)
    dec.set_source(src, mask, 1)
    got = dec.ctx.float().cpu().numpy()
    assert mt.mt_device_errors(dec.model) == 0
    trans = tuple(ew[k] for k in synth.ENCODER_TRANSITION_NAMES) if T else None
    lnp = tuple(ew[k] for k in synth.ENCODER_LN_NAMES if k in ew) if ln else None
    ref = mtref.encode(src, mask, *[ew[k] for k in synth.ENCODER_NAMES], transitions=trans, ln=lnp, eps=1e-5)
    err = maxerr(got, ref)
    print(f"encoder {gemm} B={B} H={H} T={T} ln={ln}: max error {err:.3g}", flush=True)
    assert err <= TOL[gemm]["state"]


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,H,T,ln", [(256, 5, 64, 0, False), (257, 5, 64, 0, False), (300, 5, 1024, 0, False),
                                        (1030, 3, 64, 0, False), (200, 4, 1024, 1, False), (200, 4, 1024, 2, True)])
def test_encoder_of_many_sentences(B, S, H, T, ln, gemm):
    """Both sides of the one-launch form's 256 sentences; lists of more than 1024 sentences at a
    position; recurrent products of both directions in one launch of the tiled kernel, over rows
    counted on the device.  A sample of the sentences is compared at every position."""
    src_V = 60
    p, ew, dec = encoder(gemm, 48, H, src_V, T, ln)
    rng = np.random.default_rng(B + H)
    mask = (rng.random((B, S)) < 0.6).astype(np.float32)
    mask[:, 0] = 1.0
    mask[B - 2] = 0.0
    src = rng.integers(0, src_V, size=(B, S)).astype(np.int32)
    dec.set_source(src, mask, 1)
    got = dec.ctx.float().cpu().numpy()
    assert mt.mt_device_errors(dec.model) == 0
    pick = [0, 1, 31, 32, B // 2, B - 3, B - 2, B - 1]
    trans = tuple(ew[k] for k in synth.ENCODER_TRANSITION_NAMES) if T else None
    lnp = tuple(ew[k] for k in synth.ENCODER_LN_NAMES if k in ew) if ln else None
    ref = mtref.encode(src[pick], mask[pick], *[ew[k] for k in synth.ENCODER_NAMES], transitions=trans, ln=lnp, eps=1e-5)
    assert maxerr(got[pick], ref) <= TOL[gemm]["state"]
    assert np.isfinite(got).all() and np.abs(got).max() <= 1.0


# the same through products and cells (tests/test_routes.py has the rule): tiles of consecutive rows beside
# tiles with holes, in both tile kernels and with the last tile partly filled
@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,H,T,holes", [(1030, 3, 1024, 0, 0.4), (330, 4, 1024, 0, 0.0), (330, 4, 1024, 0, 0.01),
                                           (200, 4, 1024, 1, 0.0), (200, 4, 1024, 1, 0.01), (97, 4, 2048, 0, 0.02),
                                           (160, 4, 768, 1, 0.02)])
def test_encoder_products_store_runs_and_holes(B, S, H, T, holes, gemm):
    from routes import encoder_form
    assert T or encoder_form(B, H, gemm == "bf16") == "products"
    src_V = 60
    p, ew, dec = encoder(gemm, 48, H, src_V, T, False)
    rng = np.random.default_rng(B + H)
    mask = (rng.random((B, S)) >= holes).astype(np.float32)
    mask[:, S - 1] = 1.0
    src = rng.integers(0, src_V, size=(B, S)).astype(np.int32)
    dec.set_source(src, mask, 1)
    got = dec.ctx.float().cpu().numpy()
    assert mt.mt_device_errors(dec.model) == 0
    short = [int(b) for b in np.flatnonzero(mask.min(1) == 0)[:6]]
    pick = sorted({0, 31, 32, 63, 64, 95, 96, B - 1, *short, *(min(b + 1, B - 1) for b in short)})
    trans = tuple(ew[k] for k in synth.ENCODER_TRANSITION_NAMES) if T else None
    ref = mtref.encode(src[pick], mask[pick], *[ew[k] for k in synth.ENCODER_NAMES], transitions=trans, ln=None, eps=1e-5)
    assert maxerr(got[pick], ref) <= TOL[gemm]["state"]
    assert np.isfinite(got).all() and np.abs(got).max() <= 1.0


def test_encoder_flags_padded_tokens_out_of_range():
    p, ew, dec = encoder("f32", 48, 64, 50, 0, False)
    mask = np.array([[1, 1, 0]], np.float32)
    dec.set_source(np.array([[3, 4, 50]], np.int32), mask, 1)  # at padding: flagged, not read
    assert mt.mt_device_errors(dec.model) == 8
    good = dec.ctx.cpu().numpy()
    dec.set_source(np.array([[3, 4, 0]], np.int32), mask, 1)
    assert mt.mt_device_errors(dec.model) == 0
    assert np.array_equal(good, dec.ctx.cpu().numpy())
    dec.set_source(np.array([[3, -1, 0]], np.int32), mask, 1)
    assert mt.mt_device_errors(dec.model) == 8
