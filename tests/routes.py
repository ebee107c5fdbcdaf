"""Which kernels a call's streaming passes, its gather and a decoding step go to: the library's own dispatch rules, asked on the host (no GPU).  They are
C++ functions inside libmixkv.so; the shape they take is filled in by the library and never looked into here."""
import ctypes as C

from paper_2510_20707_amd import binding as B


def _function(name, *argtypes):
    f = getattr(B.lib(), name)
    f.argtypes, f.restype = argtypes, C.c_int
    return lambda *a: f(*a) & 0xff                   # a C++ bool is the low byte


def _shape(p):
    shape = C.create_string_buffer(1024)             # larger than mixkv::Shape
    make = getattr(B.lib(), "_ZN5mixkv10make_shapeEPK12mixkv_paramsPNS_5ShapeE")
    make.argtypes, make.restype = [C.POINTER(B.MixkvParams), C.c_void_p], C.c_int
    assert make(C.byref(p), shape) == B.MIXKV_OK
    return shape


def passes(p: B.MixkvParams, n_layers: int, num_cus: int = 256, stride_n: int = 0, given_lse: bool = False):
    """(first pass, second pass) of a launch of `n_layers` layers (given softmax normalisers: the first pass only streams)."""
    assert n_layers <= 32                            # one launch group
    shape = _shape(p)
    units = n_layers * p.batch * p.n_kv_heads
    keysplit = _function("_ZN5mixkv18keysplit_supportedERKNS_5ShapeEi", C.c_void_p, C.c_int)
    qstats = _function("_ZN5mixkv16qstats_supportedERKNS_5ShapeEiiil", C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int64)
    keystat = _function("_ZN5mixkv17keystat_supportedERKNS_5ShapeEiii", C.c_void_p, C.c_int, C.c_int, C.c_int)
    if keysplit(shape, p.dtype):
        return "stats" if given_lse else "ks_stats", "ks_attn"
    return ("qs_stats" if not given_lse and qstats(shape, p.dtype, units, num_cus, stride_n or p.head_dim) else "stats",
            "kst_attn" if keystat(shape, p.dtype, units, num_cus) else "attn")


def decode_reads_once(heads_per_group: int, dtype: str):
    """Whether a decoding step's row loads are non-temporal."""
    return bool(_function("_ZN5mixkv17decode_reads_onceEii", C.c_int, C.c_int)(heads_per_group, B.DTYPE[dtype]))


def few_rows_read_once(p: B.MixkvParams, n_layers: int):
    """Whether the two passes for few query rows load keys and values non-temporally."""
    return bool(_function("_ZN5mixkv13keysplit_onceERKNS_5ShapeEii", C.c_void_p, C.c_int, C.c_int)(_shape(p), p.dtype, n_layers * p.batch * p.n_kv_heads))


def gathers_apart(p: B.MixkvParams, n_layers: int, most_rows: int):
    """Whether the rows that a fused selection keeps (of the best-endowed head: `most_rows`) are copied by a kernel behind it."""
    apart = _function("_ZN5mixkv12gather_apartERKNS_5ShapeEiil", C.c_void_p, C.c_int, C.c_int, C.c_int64)
    return bool(apart(_shape(p), 2 if p.dtype == B.DTYPE["bf16"] else 4, most_rows, n_layers * p.batch * p.n_kv_heads))
