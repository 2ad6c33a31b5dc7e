"""Forms of kernels that no result shows, in the metadata and the code of the built library."""
import os
import re
import subprocess

import pytest

from paper_2509_06040_amd import binding as br
from test_matrix_instructions import code_objects

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


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
    """Head dim 64 in two loops and 128, queries scaled ahead or not: no list of ranges (five numbers, two pointers and a factor); and scaled
    ahead with one, in the loops that launches with idle units have."""
    sizes = sorted(int(re.search(r"\.kernarg_segment_size:\s+(\d+)", e)[1]) for e in kernel_metadata(tmp_path, "attn_bf16").values())
    assert len(sizes) == 8 and sizes[5] <= 48 and sizes[6] > 64
