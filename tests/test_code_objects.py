"""What the compiler made of the kernels: properties of the built gfx950 code objects that the
kernels count on and that no output shows."""

import os
import re
import struct
import subprocess

import pytest

from paper_2606_21238_amd import _lib

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects in libarckv.so (an offload bundle for each kernel source)."""
    data, out, d = open(_lib.LIB_PATH, "rb").read(), [], tmp_path_factory.mktemp("co")
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            ofs, size, ln = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + ln].decode()
            p += 24 + ln
            if "gfx950" in name:
                path = os.path.join(d, f"{len(out)}.co")
                with open(path, "wb") as f:
                    f.write(data[at + ofs:at + ofs + size])
                out.append(path)
    assert len(out) == 3
    return out


def test_no_kernel_uses_private_memory(code_objects):
    """The library allocates no device memory; a kernel with spilled registers would have the
    runtime allocate their backing at its first launch, also under graph capture."""
    seen = []
    for path in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readobj", "--notes", path], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"\.symbol:\s+'?(\S+?)\.kd", notes)
        private = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
        assert len(names) == len(private) > 0
        seen += [(n, int(b)) for n, b in zip(names, private)]
    assert any("prefill_attn_pp_kernelILi64ELi2ELb1" in n for n, _ in seen)
    assert [(n, b) for n, b in seen if b] == []


def test_wide_attention_loops_are_placed_well(code_objects):
    """head_dim 128: a step whose 32 MFMAs begin at 16 modulo 32 bytes measured 5 to 10 % slower."""
    found = {}
    for path in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", path], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            name = re.match(r"[0-9a-f]{16} <(.*prefill_attn_pp_kernelILi128E.*)>:", part)
            if not name:
                continue
            code = re.findall(r"^\s+(\S+).*// ([0-9A-F]{12}):", part, re.M)
            at = [i for i, (op, _) in enumerate(code) if op.startswith("v_mfma")]
            runs, first = [], 0                       # MFMAs less than 40 instructions apart
            for k in range(1, len(at) + 1):
                if k == len(at) or at[k] - at[k - 1] > 40:
                    runs.append((k - first, int(code[at[first]][1], 16)))
                    first = k
            found[name.group(1)] = [a % 32 for n, a in runs if n == 32]
    assert len(found) == 10 and all(len(v) == 2 for v in found.values()), found   # plain and masked steps
    assert [k for k, v in found.items() if 16 in v] == []
