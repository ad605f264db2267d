"""The library's choice of kernel form, asked without a GPU: its host functions
by their C++ names (csrc/fwd_forms.h), so that a test can say which form a shape
takes and fails when a rule retargets it."""
import ctypes

import paper_2608_01563_amd as mg
from paper_2608_01563_amd import _binding

FWD_FORMS = ("few_wave", "few", "few_long", "rows32", "rows32_quad", "rows64", "rows64_pair",
             "rows128", "rows256")
FWD_ROWS = {"few_wave": 16, "few": 16, "few_long": 16, "rows32": 32, "rows32_quad": 32,
            "rows64": 64, "rows64_pair": 64, "rows128": 128, "rows256": 256}


class Problem(ctypes.Structure):
    """AttnProblem of csrc/launch.h."""
    _fields_ = [(n, ctypes.c_int) for n in ("B", "H", "Lq", "Lk", "d", "causal")] + \
        [("scale", ctypes.c_float), ("key_len", ctypes.c_void_p)]


def _ask(name, B, H, Lq, Lk, d, mode):
    f = getattr(mg.load_library(), "_ZN2mg%d%sERKNS_11AttnProblemE" % (len(name), name))
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(Problem)]
    return f(ctypes.byref(Problem(B, H, Lq, Lk, d, mode == "causal", 1.0,
                                  16 if mode == "padded" else None)))   # never dereferenced


def fwd_form(*shape):
    return FWD_FORMS[_ask("strict_fwd_form", *shape)]


BWD_FORMS = ("fused", "wide", "pair", "eight")


def bwd_form(*shape):
    return BWD_FORMS[_ask("split_bwd_form", *shape)]


def few_rows(contract, B, H, Lq, Lk, d, mode):
    """Whether a bf16 or accelerated forward takes 16 rows per workgroup."""
    f = mg.load_library()._ZN2mg12use_few_rowsERKNS_11AttnProblemE13mg_contract_t
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(Problem), ctypes.c_int]
    return f(ctypes.byref(Problem(B, H, Lq, Lk, d, mode == "causal", 1.0, None)),
             _binding.CONTRACTS[contract])
