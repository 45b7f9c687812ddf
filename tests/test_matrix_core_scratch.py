"""The matrix-core kernels for any row length keep all they hold in registers: what the compiler says of the built library."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_15563_amd import kmq
from tests.test_lds_reads_in_flight import device_code

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not os.path.exists(READELF), reason="no reader for the notes of code built here")
def test_no_instance_spills(tmp_path):
    path, seen, spilled = tmp_path / "code", 0, []
    for code in device_code(kmq.LIB_PATH):
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n  - \.", notes)[1:]:
            name = re.search(r"\.name:\s+(\S*gemm_canon_kernel\S*)", kernel)
            if name:
                seen += 1
                if re.search(r"\.private_segment_fixed_size:\s+[1-9]", kernel):
                    spilled.append(name[1])
    assert seen >= 100
    assert not spilled
