"""Which form of a kernel a call takes: the library's own rules (host code, no GPU), called by their
C++ names."""
import ctypes as C

from paper_1804_00344_amd import mtstep as mt


def _fn(symbol, restype, nargs):
    f = getattr(mt.lib(), symbol)
    f.restype, f.argtypes = restype, [C.c_int] * nargs
    return f


def attention_form(B, K, S, E, H, A):
    """"beam" or "row": the attention of a step (its scores need rows of 3H + E floats of scratch)."""
    takes = _fn("_ZN2mt20attention_takes_beamEiiiii", C.c_bool, 5)
    return "beam" if S <= 3 * H + E and takes(B, K, S, A, 2 * H) else "row"


def joint_chunks(E, V, M, n=2, bf16=1, num_cu=256):
    """(chunks, chunks per workgroup) of the joint vocabulary pass."""
    f = mt.lib()._ZN2mt18vocab_joint_chunksEiiiiiiPi
    f.restype, f.argtypes = C.c_int, [C.c_int] * 6 + [C.POINTER(C.c_int)]
    group = C.c_int(0)
    return f(bf16, M, V, E, n, num_cu, C.byref(group)), group.value


def encoder_form(B, H, bf16):
    """"fused" (one kernel per position) or "products": a shallow encoder cell without layer norm."""
    return "fused" if _fn("_ZN2mt14enc_step_takesEiii", C.c_bool, 3)(bf16, B, H) else "products"


def vocab_chunks(E, V, M, bf16=1, num_cu=256):
    return _fn("_ZN2mt12vocab_chunksEiiiii", C.c_int, 5)(bf16, M, V, E, num_cu)
