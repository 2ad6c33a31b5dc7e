"""Forms of kernels that no result shows, in the metadata and the code of the built library."""
import os
import re
import subprocess

import pytest

from paper_2509_06040_amd import binding as br
from test_matrix_instructions import code_objects

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernel_metadata(tmp_path, part):
    """name -> metadata text of the kernels whose name holds `part`."""
    out = {}
    for i, obj in enumerate(code_objects(br.LIB_PATH)):
        if part.encode() not in obj:
            continue
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(obj)
        text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"\n\s+- \.(?=agpr_count|args)", text):
            m = re.search(r"\.name:\s+(\S+)", entry[entry.rfind(".kernarg_segment_size"):])
            if m and part in m[1]:
                out[m[1]] = entry
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is missing")
def test_attention_that_reads_no_weights_ahead_carries_no_list_of_them(tmp_path):
    """Short sequences, the loop at head dim 64 and in both forms of 128, queries scaled ahead or not: no list of ranges (five numbers, two
    pointers and a factor); and scaled ahead with one, in the loops that launches with idle units have."""
    sizes = sorted(int(re.search(r"\.kernarg_segment_size:\s+(\d+)", e)[1]) for e in kernel_metadata(tmp_path, "attn_bf16").values())
    assert len(sizes) == 2 + 2 + 4 + 2 and sizes[7] <= 48 and sizes[8] > 64


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump is missing")
def test_layer_norm_of_long_rows_past_the_caches_sums_in_the_lds_unit(tmp_path):
    """Lane permutations everywhere (DPP) but in the launches that store past the caches: bf16 from 1536 columns, fp32 at 1024 and from 2048.  (Rows held
    in VPL registers of 256 columns each; 0: any length.)"""
    forms = {}
    for i, obj in enumerate(code_objects(br.LIB_PATH)):
        if b"ln_modulate_kernel" not in obj:
            continue
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            m = re.match(r"[0-9a-f]+ <_ZN2br18ln_modulate_kernelI(f|DF16b)Li(\d+)ELb([01])E", part)
            if m:
                forms[m[1] == "f", int(m[2]), m[3] == "1"] = "ds_bpermute" in part or "ds_swizzle" in part
    assert len(forms) == 2 * 2 * 8
    for (f32, vpl, stream), lds in forms.items():
        assert lds == (stream and (vpl in (4, 8, 12) if f32 else vpl >= 6)), (f32, vpl, stream)
