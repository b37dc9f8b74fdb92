"""The addresses that the products with M + G take from the pointer table have to arrive in scalar registers.  A store in
front of the table's loads makes the compiler use vector loads, whose results take vector registers for as long as the kernel
runs: the 128 x 128 tile of (M + G)^T P in fp32 then misses three waves per SIMD by two registers."""
import os
import re
import subprocess

import pytest

from paper_2504_05295_amd import build


@pytest.mark.parametrize("source", ["gemm_k1", "gemm_k2"])
def test_table_is_read_by_scalar_loads(source, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "out.s")
    subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, source + ".hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = open(out).read()
    vector_loads = re.findall(r"global_load_dwordx2 v\[\d+:\d+\], v\d+, s\[.*", text)
    assert not vector_loads, (len(vector_loads), vector_loads[:3])
    # (512 registers per SIMD: three waves up to 168 each)
    counts = {m.group(1): int(m.group(2)) for m in re.finditer(r"\.name:\s+(\S*gemm_kernel\S*)(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)", text, re.S)}
    assert len(counts) == 24
    if source == "gemm_k2":
        tile = [v for k, v in counts.items() if "TileCfgILi128ELi128ELi32ELi2ELi2EEELb0ELi3ELi1E" in k]
        assert len(tile) == 4 and max(tile) <= 168, tile
