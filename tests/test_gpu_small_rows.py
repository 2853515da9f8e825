"""Decoder steps of few rows: the matrix products' split-depth kernel at the edges of its row
groups (32), of its 16-row blocks and of its k-split over eight waves, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1804_00344_amd import synth
from parity_util import TOL, oracle_model, oracle_sentences, sample_sentences
from test_gpu_parity import T, compare_rows, run_step

if torch.cuda.is_available():
    from paper_1804_00344_amd.runner import Decoder

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# (E, H, A): the Nematus sizes; depths of 5 and 13 k-steps of 16, fewer than or no multiple of 8
DIMS = {"nematus": dict(E=512, H=1024, A=2048), "odd": dict(E=48, H=80, A=208)}


@pytest.mark.parametrize("gemm", ["f32", "bf16"])
@pytest.mark.parametrize("dims,B,K", [("odd", 1, 1), ("odd", 3, 11), ("nematus", 1, 5), ("nematus", 1, 16),
                                      ("nematus", 17, 1), ("nematus", 4, 8), ("nematus", 11, 3), ("nematus", 13, 5),
                                      ("nematus", 24, 4)])
def test_step_parity_few_rows(dims, B, K, gemm):
    p = synth.with_sizes(synth.PRESETS["nematus_bf16_ln"], V=1200, B=B, K=K, gemm=gemm, len_b=20, len_a=9, **DIMS[dims])
    w = synth.make_weights(p)
    ctx, mask, lens = synth.make_source(p)
    dec = Decoder.from_preset(p, w)
    dec.set_batch(ctx, mask, K)
    dec.precompute()
    tok, src, state, score = synth.mid_decode_inputs(p)
    gpu = run_step(dec, p, tok, src, T(state), p.M)
    torch.cuda.synchronize()
    sents = sample_sentences(lens, 4)
    orc = oracle_sentences(oracle_model(p, w), K, sents, ctx, mask, tok, src, state)
    compare_rows(p, gpu, orc, sents, TOL[gemm], f"{dims} {gemm} {B}x{K}")
    for b in sents:  # the start state's product (tanh epilogue)
        err = float(np.max(np.abs(dec.s0[b].cpu().numpy() - orc[b]["s0"])))
        assert err <= TOL[gemm]["state"], (b, err)


# Start states of many sentences in bf16, S = 1: fp32 rows (the context itself) against the tiles of 32,
# 64, 96 and 128 rows (the last for depths from 2048 on), whole and partly filled last tiles
@pytest.mark.parametrize("B,H", [(1504, 512), (2048, 512), (3001, 512), (4100, 512), (6144, 512), (5000, 512),
                                 (1791, 2048), (1792, 2048), (1793, 2048), (2050, 1024), (3700, 1024)])
def test_start_state_of_many_sentences(B, H):
    p = synth.with_sizes(synth.PRESETS["tiny_bf16_ln"], E=16, H=H, A=16, V=50)
    w = synth.make_weights(p)
    dec = Decoder.from_preset(p, w)
    rng = np.random.default_rng(B)
    ctx = synth.round_bf16(np.tanh(rng.standard_normal((B, 1, 2 * H))).astype(np.float32))
    dec.set_batch(ctx, np.ones((B, 1), np.float32), 1)
    dec.precompute()
    Wi, bi = (torch.from_numpy(w[k]).double().cuda() for k in ("Wi", "bi"))
    ref = torch.tanh(torch.from_numpy(ctx[:, 0]).double().cuda() @ Wi + bi)
    # both operands are bf16 values, the sums fp32
    assert float((dec.s0.double() - ref).abs().max()) <= TOL["f32"]["state"]
