"""The rules that choose a kernel's form by the sizes of a call (host code, no GPU)."""
import pytest

import ctypes as C

from routes import _fn, attention_form, encoder_form, joint_chunks, vocab_chunks
from test_gpu_attention_beam import BEAM, EXTREME_SIZES
from test_gpu_joint_pairs import PAIRS

NEMATUS = dict(E=512, H=1024, A=2048)


@pytest.mark.parametrize("B,K,S,A,H", BEAM)
def test_attention_beam_cases_take_the_beam_form(B, K, S, A, H):
    assert attention_form(B, K, S, 32, H, A) == "beam"


def test_attention_beam_extremes_take_both_forms():
    B, K, S, A, H = (EXTREME_SIZES[k] for k in "BKSAH")
    assert attention_form(B, K, S, 32, H, A) == "beam" and attention_form(B * K, 1, S, 32, H, A) == "row"


@pytest.mark.parametrize("B,K,S,dims,form", [
    (1, 5, 25, NEMATUS, "beam"), (8, 5, 60, NEMATUS, "beam"), (64, 12, 80, NEMATUS, "beam"),
    (128, 5, 100, NEMATUS, "beam"),
    # short sentences, or rows enough to fill the chip: measured slower with the beam form
    (1, 5, 10, NEMATUS, "row"), (64, 12, 25, NEMATUS, "row"), (64, 12, 50, NEMATUS, "row"), (300, 2, 30, NEMATUS, "row"),
    (300, 3, 30, NEMATUS, "row"), (48, 16, 50, NEMATUS, "row"), (48, 8, 30, NEMATUS, "row"),
    (1, 16, 25, dict(E=256, H=256, A=512), "row"), (64, 16, 80, dict(E=256, H=256, A=512), "row"),
    # one hypothesis; fewer features than a wave's; weights beyond the LDS; scores beyond their scratch
    (64, 1, 80, NEMATUS, "row"), (3, 4, 100, dict(E=512, H=1024, A=496), "row"),
    (2, 16, 1020, NEMATUS, "beam"), (2, 16, 1021, NEMATUS, "row"), (2, 12, 1024, NEMATUS, "beam"),
    (2, 3, 224, dict(E=32, H=64, A=512), "beam"), (2, 3, 225, dict(E=32, H=64, A=512), "row"),
    (65536, 2, 1024, NEMATUS, "row"),
])
def test_attention_form(B, K, S, dims, form):
    assert attention_form(B, K, S, **dims) == form


@pytest.mark.parametrize("E,V,B,K", PAIRS)
def test_joint_pair_cases_take_two_chunks(E, V, B, K):
    assert joint_chunks(E, V, B * K)[1] == 2


def test_joint_pair_cases_have_odd_chunk_counts():
    assert [joint_chunks(E, V, B * K)[0] % 2 for E, V, B, K in (PAIRS[1], PAIRS[-1])] == [1, 1]


@pytest.mark.parametrize("E", [64, 128, 256, 512])
@pytest.mark.parametrize("V", [500, 1000, 10000, 30000, 50000, 85000])
def test_joint_pair_of_few_rows_keeps_one_chunk_per_workgroup(E, V):
    """Up to 64 rows are one row block: two chunks per workgroup would only halve the workgroups."""
    for M in (1, 5, 20, 40, 64):
        n, group = joint_chunks(E, V, M)
        assert group == 1 and n == min(256, (V + 255) // 256)


def test_joint_chunks_fit_the_single_models_workspace():
    for E, V, M in ((512, 50000, 768), (512, 50000, 160), (512, 85000, 320), (128, 1000, 5), (512, 72001, 320)):
        assert joint_chunks(E, V, M)[0] <= vocab_chunks(E, V, M)
    assert joint_chunks(512, 50000, 768)[1] == 2
    # another type, another number of members, 32-row blocks: one chunk
    assert joint_chunks(512, 50000, 768, bf16=0)[1] == 1
    assert joint_chunks(512, 50000, 768, n=3)[1] == 1
    assert joint_chunks(1024, 50000, 768)[1] == 1


@pytest.mark.parametrize("bf16,E,V,M,chunks", [
    # one block per wave where the lists allow it, whatever the vocabulary
    (1, 512, 1000, 1, 8), (1, 512, 2000, 1, 16), (1, 512, 8000, 40, 63), (0, 512, 8000, 64, 63), (1, 512, 50000, 5, 256),
    (0, 64, 2000, 1, 16), (1, 64, 2049, 1, 17),
    # a narrow row and a small vocabulary: few lists, selected by sentence
    (1, 64, 2000, 1, 8), (1, 64, 1000, 1, 8),
    # rows wider than 2 KB: one block per wave or tiles of two
    (1, 2048, 32768, 32, 256), (1, 2048, 33000, 32, 129), (1, 1536, 85000, 32, 256), (1, 2048, 16384, 33, 128),
    (1, 2048, 20000, 33, 79), (0, 1024, 32768, 5, 256), (0, 1024, 33000, 5, 129), (1, 1024, 33000, 5, 256),
    # more rows: tiles of two
    (1, 512, 8000, 65, 32), (0, 512, 50000, 65, 128),
])
def test_vocab_chunks(bf16, E, V, M, chunks):
    assert vocab_chunks(E, V, M, bf16) == chunks


def test_weights_beyond_a_buffer_views_reach():
    """Output weights of 4 GiB or more: no joint pass (and no unrolled k-loop) reads them through 32-bit
    offsets."""
    fits = _fn("_ZN2mt15vocab_fits_viewEiii", C.c_bool, 3)
    rows = _fn("_ZN2mt16vocab_joint_rowsEiiii", C.c_int, 4)
    for bf16, V in ((0, 1 << 21), (1, 1 << 22)):  # x 512 x 4 or 2 bytes
        assert fits(bf16, V - 64, 512) and not fits(bf16, V, 512)
        assert rows(bf16, V - 64, 512, 2) > 0 and rows(bf16, V, 512, 2) == 0


@pytest.mark.parametrize("bf16,H,most", [
    # sentences up to which one kernel per position is the faster form, full lengths included
    (1, 64, 4096), (1, 256, 1024), (1, 512, 512), (1, 1024, 256), (1, 1536, 160), (1, 2048, 96),
    (0, 64, 4096), (0, 256, 1024), (0, 512, 512), (0, 768, 256), (0, 1024, 128), (0, 1536, 32), (0, 2048, 16),
])
def test_encoder_form(bf16, H, most):
    assert [B for B in range(1, 5000) if encoder_form(B, H, bf16) == "fused"] == list(range(1, most + 1))
