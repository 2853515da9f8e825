"""The joint vocabulary pass of two bf16 members with two chunks per workgroup: odd chunk counts
(a workgroup without its second chunk), row blocks with one and with several rows, vocabularies
that end inside a tile; against the per-member pass and the oracle's combination."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mtref
from paper_1804_00344_amd import synth
from parity_util import TOL, oracle_model, topk_gap_check

if torch.cuda.is_available():
    from paper_1804_00344_amd.runner import Decoder, Ensemble

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# sizes that take two chunks per workgroup (tests/test_routes.py checks it), the second and the last
# with an odd chunk count
PAIRS = [(512, 8191, 64, 16), (512, 14001, 28, 16), (512, 10011, 48, 16), (256, 20011, 64, 12), (128, 30011, 64, 16),
         (512, 72001, 64, 5)]


@pytest.mark.parametrize("E,V,B,K", [(64, 1200, 2, 4), (512, 1200, 13, 5), (512, 3001, 5, 16), (128, 20011, 33, 4)])
def test_joint_pair_parity(E, V, B, K):
    check(E, V, B, K)


@pytest.mark.parametrize("E,V,B,K", PAIRS)
def test_joint_pair_of_two_chunks_parity(E, V, B, K):
    check(E, V, B, K)


@pytest.mark.parametrize("E,V,B,K", [(512, 1200, 13, 5), (512, 14001, 28, 16)])
def test_joint_pair_of_unbounded_logits(E, V, B, K):
    """Output matrices whose logits have no bound in [-40, 40]: the running-maximum form, against the
    per-member pass (scores of magnitude 100: sums of fp32 in another order)."""
    check(E, V, B, K, wo_scale=60.0, tol=1e-3)


def check(E, V, B, K, wo_scale=1.0, tol=1e-4):
    ws = [0.6, 0.4]
    ps = [synth.with_sizes(synth.PRESETS["tiny_bf16_ln"], index=5 + 100 * i, E=E, V=V, B=B, K=K) for i in range(2)]
    p = ps[0]
    wts = [synth.make_weights(q, peaked_bias=True) for q in ps]
    for w in wts:
        w["Wo"] = synth.round_bf16(w["Wo"] * np.float32(wo_scale))
    ctx, mask, _ = synth.make_source(p)
    tok0 = synth.bounded_zipf(np.random.default_rng(3), V, p.M)
    score0 = np.tile(-0.3 * np.arange(K, dtype=np.float32), B)
    out = []
    for joint in (True, False):
        ens = Ensemble([Decoder.from_preset(q, w) for q, w in zip(ps, wts)], ws, joint=joint)
        assert ens.joint == joint
        ens.set_batch(ctx, mask, K)
        ens.precompute()
        ens.start(tok0, score0)
        states = ens.advance()
        torch.cuda.synchronize()
        lead = ens.lead
        out.append((lead.score.cpu().numpy(), lead.tok.cpu().numpy(), lead.bp.cpu().numpy(),
                    [s.cpu().numpy() for s in states]))
    assert np.max(np.abs(out[0][0] - out[1][0])) <= tol  # the same members, sums in another order
    for a, b in zip(out[0][3], out[1][3]):
        assert np.array_equal(a, b)
    if wo_scale != 1.0:
        return
    oms = [oracle_model(q, w) for q, w in zip(ps, wts)]
    for b in sorted({0, B // 2, B - 1}):
        rows = slice(b * K, (b + 1) * K)
        lps = []
        for om in oms:
            P, s0 = om.precompute(ctx[b:b + 1], mask[b:b + 1])
            lps.append(om.step(K, tok0[rows], np.zeros(K, np.int32), s0, ctx[b:b + 1], P, mask[b:b + 1])["logp"])
        topk_gap_check(K, score0[rows], mtref.ensemble_logp(lps, ws), out[0][0][rows], out[0][1][rows],
                       out[0][2][rows], TOL["bf16"]["logp"])
