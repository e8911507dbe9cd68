"""What a call takes from a tune cache file, by the file's format: the library's own lookup, without
a GPU.  Lines of the present format are taken as they stand.  Lines of earlier formats were measured
with other kernels and chunk rules: only a list threshold below the default is taken from them."""
import ctypes as C

import pytest

import paper_1111_7171_amd as P


class Params(C.Structure):
    _fields_ = [(k, C.c_int32) for k in ("verify_waves_per_cu", "seg_chunk", "big_list",
                                         "probe_blocks_per_cu", "lane_cands", "probe_map")]


DEFAULT = (32, 4, 32, 8, 1, 1)
LINE = (512, 256, 128, 16, 2, 0)


def _lookup(path, tau, mean):
    fn = C.CDLL(P.LIB_PATH)["_ZN2pj11tune_lookupEPKcid"]     # pj::tune_lookup(const char*, int, double)
    fn.argtypes, fn.restype = [C.c_char_p, C.c_int, C.c_double], Params
    p = fn(str(path).encode() if path else None, tau, mean)
    return tuple(getattr(p, k) for k, _ in Params._fields_)


def _arch():
    import torch
    if not torch.cuda.is_available():
        return "unknown"
    return torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]


@pytest.mark.parametrize("header, line, expected", [
    ("# passjoin tune cache v4: arch tau", LINE, LINE),
    ("# passjoin tune cache v4", (512, 3, 128, 16, 2, 0), DEFAULT),          # out of range
    ("# passjoin tune cache v4", LINE[:5], DEFAULT),                         # a column missing
    ("# passjoin tune cache v3: arch tau", LINE, DEFAULT),
    ("# passjoin tune cache v3: arch tau", (8, 2048, 16, 4, 2, 0), (32, 4, 16, 8, 1, 1)),
    ("# passjoin tune cache v2", (32, 4, 16, 4, 2), (32, 4, 16, 8, 1, 1)),
    ("# no version", LINE, DEFAULT),
])
def test_formats(tmp_path, header, line, expected):
    path = tmp_path / "tune.txt"
    path.write_text(f"{header}\n{_arch()} 61 4 {' '.join(map(str, line))} 112.300\n")
    assert _lookup(path, 61, 15.0) == expected
    assert _lookup(path, 62, 15.0) == DEFAULT
    assert _lookup(None, 61, 15.0) == DEFAULT
