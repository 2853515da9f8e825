"""Attention of several hypotheses per sentence (the beam form): masks with holes, empty
sentences, tiles of positions at their edges, hypothesis groups, feature counts that are no
multiple of a wave's 512, and queries and keys beyond the shared-exponential range, against the
oracle's step (context, weights, state)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1804_00344_amd import synth
from parity_util import TOL, maxerr, oracle_model, oracle_sentences
from test_gpu_parity import T, run_step

if torch.cuda.is_available():
    from paper_1804_00344_amd.runner import Decoder

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def check(gemm, B, K, S, A, H, scale_q=1.0, shift_p=0.0):
    p = synth.with_sizes(synth.PRESETS["nematus_bf16_ln"], E=32, H=H, A=A, V=64, B=B, K=K, gemm=gemm, layer_norm=False)
    w = synth.make_weights(p)
    rng = np.random.default_rng(B * 1000 + K * 10 + S)
    w["Wa"] = (w["Wa"] * scale_q).astype(np.float32)
    w["ba"] = (shift_p * rng.standard_normal(A)).astype(np.float32)
    ctx = synth.round_bf16(np.tanh(rng.standard_normal((B, S, 2 * H))).astype(np.float32))
    mask = (rng.random((B, S)) < 0.7).astype(np.float32)
    mask[0] = 1.0
    if B > 1:
        mask[B - 1] = 0.0
    if B > 2 and S > 3:
        mask[1] = 0.0
        mask[1, S - 1] = 1.0
        ctx[1, :S - 1] = np.nan  # padding is never used
    dec = Decoder.from_preset(p, w)
    dec.set_batch(ctx, mask, K)
    dec.precompute()
    tok, src, state, score = synth.mid_decode_inputs(p)
    gpu = run_step(dec, p, tok, src, T(state), p.M)
    torch.cuda.synchronize()
    orc = oracle_sentences(oracle_model(p, w), K, list(range(B)), np.nan_to_num(ctx), mask, tok, src, state)
    for b in range(B):
        rows = slice(b * K, (b + 1) * K)
        for k, tol in (("alpha", "alpha"), ("c", "tap"), ("state", "state")):
            err = maxerr(gpu[k][rows].float().cpu().numpy(), orc[b][k])
            assert err <= TOL[gemm][tol], (b, k, err)
        assert np.all(gpu["alpha"][rows].cpu().numpy()[:, mask[b] == 0] == 0)


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("B,K,S,A,H", [(3, 2, 1, 512, 64), (2, 3, 300, 512, 64), (2, 9, 70, 512, 64), (5, 4, 9, 528, 272), (4, 5, 65, 1024, 128), (3, 6, 17, 2048, 64),
                                       (3, 8, 130, 1040, 64), (4, 12, 33, 2064, 128), (3, 13, 24, 4096, 64),
                                       (2, 16, 7, 512, 144), (700, 3, 16, 512, 64)])
def test_attention_beam_parity(B, K, S, A, H, gemm):
    check(gemm, B, K, S, A, H)


# sizes that take the beam form (tests/test_routes.py checks it): the fewest positions it takes with
# two and with three hypotheses, every hypothesis group size (one to three groups of 2..6), feature
# counts off a wave's 512, position counts at the edges of the context kernel's 64, 128 and 256 and
# of the score tiles (1, 2 and 4 positions), the most weights its LDS holds, many sentences
BEAM = [(1, 2, 11, 4096, 16), (2, 3, 12, 4096, 16), (2, 3, 300, 512, 128), (3, 2, 64, 512, 64), (5, 4, 41, 528, 272),
        (4, 5, 65, 1024, 128), (3, 6, 21, 2048, 64), (3, 8, 128, 1040, 64), (3, 8, 129, 1040, 64), (2, 9, 70, 512, 64),
        (4, 12, 33, 2064, 128), (3, 13, 24, 4096, 64), (2, 16, 70, 512, 144), (2, 3, 256, 512, 96),
        (2, 5, 257, 512, 96), (1, 16, 1020, 512, 352), (3, 4, 1024, 512, 352), (100, 4, 32, 4096, 16),
        (70, 2, 40, 4096, 16)]


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("B,K,S,A,H", BEAM)
def test_attention_beam_form_parity(B, K, S, A, H, gemm):
    check(gemm, B, K, S, A, H)


@pytest.mark.parametrize("scale_q,shift_p", [(40.0, 0.0), (1.0, 12.0), (30.0, 60.0)])
def test_attention_beam_out_of_range_operands(scale_q, shift_p):
    """|q| or |P| past the range of the shared exponentials (30 ln2 / 2 = 10.4)."""
    check("f32", 4, 5, 11, 576, 64, scale_q, shift_p)


# operands beyond the shared-exponential range, in both types: everywhere, in one feature (infinite
# once scaled), at one position of one sentence, in one hypothesis beside others in range, and a
# hypothesis of NaN beside finite ones
EXTREMES = ["queries", "keys", "feature", "position", "hypothesis", "nan"]
EXTREME_SIZES = dict(B=4, K=5, S=44, A=1040, H=64)


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("where", EXTREMES)
def test_attention_beam_extremes_match_the_row_form(where, gemm):
    """The same hypotheses as sentences of one hypothesis each run the row form on the same keys and
    queries: weights and contexts agree to fp32 rounding (scores of magnitude 30: 1e-4), and are NaN
    in the same places."""
    B, K, S, A, H = (EXTREME_SIZES[k] for k in "BKSAH")
    p = synth.with_sizes(synth.PRESETS["nematus_bf16_ln"], E=32, H=H, A=A, V=64, B=B, K=K, gemm=gemm, layer_norm=False)
    w = synth.make_weights(p)
    rng = np.random.default_rng(5)
    if where == "queries":
        w["Wa"] = synth.round_bf16((w["Wa"] * 60.0).astype(np.float32))
    if where == "keys":
        w["ba"] = (20.0 * rng.standard_normal(A)).astype(np.float32)
    if where == "feature":
        w["Wa"][:, 700] = 0.0
        w["Wa"][3, 700] = 3e38
    ctx = synth.round_bf16(np.tanh(rng.standard_normal((B, S, 2 * H))).astype(np.float32))
    mask = (rng.random((B, S)) < 0.8).astype(np.float32)
    mask[:, 7] = 1.0
    if where == "position":
        ctx[2, 7] *= 256.0
    tok, src, state, _ = synth.mid_decode_inputs(p)
    state = state[src].copy()
    if where == "hypothesis":
        w["Wa"] = synth.round_bf16((w["Wa"] * 8.0).astype(np.float32))
        state *= np.float32(0.02)
        state[K + 2] = np.sign(state[K + 2])
    if where == "nan":
        state[K + 2] = np.nan
    rows = np.arange(p.M, dtype=np.int32)
    out = []
    for k in (K, 1):
        dec = Decoder.from_preset(synth.with_sizes(p, B=p.M // k, K=k), w)
        dec.set_batch(np.repeat(ctx, K // k, axis=0), np.repeat(mask, K // k, axis=0), k)
        dec.precompute()
        if out:
            dec.pctx.copy_(out[0][1].repeat_interleave(K, 0))
        q = run_step(dec, synth.with_sizes(p, B=p.M // k, K=k), tok, rows, T(state), p.M)
        torch.cuda.synchronize()
        out.append(({n: q[n].float().cpu().numpy() for n in ("alpha", "c", "s1")}, dec.pctx.clone()))
    beam, row = out[0][0], out[1][0]
    assert np.array_equal(beam["s1"], row["s1"], equal_nan=True)
    for n in ("alpha", "c"):
        assert np.array_equal(np.isnan(beam[n]), np.isnan(row[n])), n
        assert np.isnan(beam[n]).any() == (where == "nan")
        ok = ~np.isnan(row[n])
        assert maxerr(beam[n][ok], row[n][ok]) <= (1e-4 if n == "alpha" or where != "position" else 256e-4), n


def test_attention_row_form_still_serves():
    """Sizes the beam form leaves to the row form: A < 512, and weights beyond its LDS."""
    check("f32", 3, 4, 12, 496, 64)
    check("f32", 2, 16, 1024, 512, 64)
