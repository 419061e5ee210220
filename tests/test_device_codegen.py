"""What the device code tells the compiler, read from the LLVM IR and the assembly of small kernels
compiled here from the library's headers."""
import re
import subprocess
from pathlib import Path

from paper_2206_01299_amd import build as _build

ROOT = Path(__file__).resolve().parent.parent


def _compile(tmp_path, text, *flags):
    src = tmp_path / "probe.hip"
    src.write_text(text)
    r = subprocess.run([_build.HIPCC, *_build.FLAGS, "--cuda-device-only", "-S", *flags, str(src), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


def test_pieces_at_any_element_are_stored_without_a_promise_of_alignment(tmp_path):
    """Rows and groups that are no whole 16-byte pieces start at any element: a store of such a piece may
    promise the element's alignment and no more, and is one instruction all the same."""
    text = """
#include "aqsgd_anygroup.h"
using namespace aqsgd;
extern "C" __global__ void raw(char* p, u32x4_t a, f32x4_t b) { store16(p, a, false); store16(p + 64, b, false); }
extern "C" __global__ void f16(char* p, float x) { float v[8] = {x, x, x, x, x, x, x, x}; store_piece<AQSGD_F16, 8>(p, v); }
extern "C" __global__ void f32(char* p, float x) { float v[4] = {x, x, x, x}; store_piece<AQSGD_F32, 4>(p, v); }
extern "C" __global__ void units(char* p, Raw<AQSGD_F32> r) { store_raw_units(p, p + 100, r, false); }
"""
    ir = _compile(tmp_path, text, "-emit-llvm")
    stores = re.findall(r"store <\d x (\w+)> .*?align (\d+),.*!nontemporal", ir)
    assert len(stores) == 6, ir
    for kind, align in stores:
        assert int(align) <= (4 if kind == "float" else 2), stores
    asm = _compile(tmp_path, text)
    wide = [l for l in asm.splitlines() if re.search(r"global_store_dwordx4 .*\bnt\b", l)]
    assert len(wide) == len(stores), asm
