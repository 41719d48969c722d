"""Prefill kernels that address registers by name across their asm statements, on the assembly the compiler makes of them."""
import re

import pytest

from paper_2509_23410_amd import build


@pytest.mark.parametrize("source,kernel,first,count", [("quant4_kgroups.hip", "prefill4_kgroups_kernel", 161, 4), ("gemm_prefill_128.hip", "prefill_kernel_r128", 160, 4)])
def test_named_registers_are_left_alone(tmp_path, source, kernel, first, count):
    """From the first asm statement that names them to the wait in front of the output stage, loads are in flight into registers v<first> and up
    and the statements hand values on in them: compiler-generated code may touch none of them, nor m0, may issue no vector memory instruction but
    the reload of the table entries (a single dword, waited for at once: the statements count their loads), and nothing may be spilled."""
    text = open(build.device_asm(source, str(tmp_path / "a.s"))).read()
    bodies = re.findall(r"^(_ZN5patch\d+" + kernel + r"\w*):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M)
    assert len(bodies) == count
    for name, body in bodies:
        lines = body.splitlines()
        begin = next(i for i, l in enumerate(lines) if re.search(r"v\[\d+\+", l))
        end = next(i for i in range(begin, len(lines)) if "s_nop 15" in lines[i])
        inasm, statements = True, 0
        for line in lines[begin:end]:
            if "#ASMSTART" in line or "#ASMEND" in line:
                inasm = "#ASMSTART" in line
                statements += inasm
                continue
            code = line.split(";")[0]
            if inasm or not code.strip() or code.strip().startswith("."):
                continue
            used = [int(v) for v in re.findall(r"\bv(\d+)\b", code)] + [int(v) for r in re.findall(r"\bv\[(\d+):(\d+)\]", code) for v in r]
            assert all(v < first for v in used), f"{name}: {line}"
            assert not re.search(r"\bm0\b", code) or "prefill4" not in kernel, f"{name}: {line}"
            assert not re.match(r"\s*(scratch|buffer|flat)_", code), f"{name}: {line}"
            assert not re.match(r"\s*global_(load|store)", code) or re.match(r"\s*global_load_dword ", code) or re.match(r"\s*global_load_lds", code), f"{name}: {line}"
        assert statements > 15, name
    kernels = [k for k in re.split(r"(?m)^  - \.a", text[text.index("amdhsa.kernels"):]) if kernel in k]
    assert len(kernels) == count
    for k in kernels:
        assert re.search(r"\.vgpr_spill_count:\s+0\b", k) and re.search(r"\.private_segment_fixed_size:\s+0\b", k)
