"""The rules that choose a kernel's form by the sizes of a call (host code, no GPU)."""
import pytest

from routes import attention_form
from test_gpu_attention_beam import BEAM

NEMATUS = dict(E=512, H=1024, A=2048)


@pytest.mark.parametrize("B,K,S,A,H", BEAM)
def test_attention_beam_cases_take_the_beam_form(B, K, S, A, H):
    assert attention_form(B, K, S, 32, H, A) == "beam"


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
