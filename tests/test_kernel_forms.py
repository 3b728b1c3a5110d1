"""What the built kernels are: which form of requantisation a window takes, that the depthwise kernels keep the
registers that 7 wavefronts per SIMD allow, and that the grouped kernels keep their loops out of scratch memory."""
import os
import shutil
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_forms_of_requantisation():
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    cmd = [hipcc, "--cuda-host-only", "-fsyntax-only", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(ROOT, "paper_2505_03254_amd", "csrc"), "-x", "hip", os.path.join(ROOT, "tests", "pair_forms.hip")]
    p = subprocess.run(cmd, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr


def _kernels(path):
    """name -> metadata of every kernel in the device code objects (ELF images) of a library built here."""
    data = open(path, "rb").read()
    out, at = {}, data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:  # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, count = struct.unpack_from("<HH", data, at + 58)
            for i in range(count):
                kind, off, length = (struct.unpack_from("<I", data, at + shoff + i * size + 4)[0],
                                     *struct.unpack_from("<QQ", data, at + shoff + i * size + 24))
                pos = at + off
                while kind == 7 and pos < at + off + length:  # SHT_NOTE
                    n, d, t = struct.unpack_from("<III", data, pos)
                    desc = pos + 12 + (n + 3) // 4 * 4
                    if t == 32:  # NT_AMDGPU_METADATA
                        for k in msgpack.unpackb(data[desc:desc + d])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    pos = desc + (d + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


def _found(*names):
    import paper_2505_03254_amd as P
    if not os.path.exists(P.library_path()):
        from paper_2505_03254_amd.build import build
        build()
    found = {k: v for k, v in _kernels(P.library_path()).items() if any(n in k for n in names)}
    if not found:
        pytest.skip("no readable kernel metadata")
    return found


def test_depthwise_registers():
    found = _found("dw_kernel_v4", "dw_batch_kernel")
    assert len(found) == 4, sorted(found)
    for name, k in found.items():
        assert k[".vgpr_count"] <= 72 and k[".private_segment_fixed_size"] == 0, (name, k[".vgpr_count"])


def test_grouped_kernels_use_no_scratch():
    found = _found("gconv_tapk_kernel", "gconv_tapk_batch_kernel")
    assert len(found) == 4, sorted(found)
    for name, k in found.items():
        assert k[".private_segment_fixed_size"] == 0, (name, k[".private_segment_fixed_size"])


def test_weight_loads_leave_together(tmp_path):
    """The loads of a batch of the weight staging stand in one basic block, 16 or 4 words per lane, 4 and 4 more in the
    row kernel, and nothing in that block waits for all loads before the last of them has left."""
    from paper_2505_03254_amd.build import HIPCC_FLAGS, _hipcc
    out = str(tmp_path / "weight_loads.s")
    p = subprocess.run([_hipcc()] + HIPCC_FLAGS + ["--cuda-device-only", "-S", "-x", "hip",
                                                   os.path.join(ROOT, "tests", "weight_loads.hip"), "-o", out],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    runs, name, run, waited = {}, None, 0, False
    for line in open(out):
        s = line.strip()
        if line[0] == "_" and ":" in line:
            name, run, waited = line.split(":")[0], 0, False
            runs[name] = []
        if name is None or not s or s[0] == ";" or (s[0] == "." and ":" not in s):
            continue
        op = s.split()[0]
        if op == "buffer_load_dword":  # a word of codes (activations and parameters have other loads)
            run += 1
            assert not waited, (name, s)
        elif op.endswith(":") or op.startswith(("s_cbranch", "s_branch", "v_mfma")):
            runs[name] += [run] if run else []
            run, waited = 0, False
            if op.startswith("v_mfma"):
                name = None
        elif op == "s_waitcnt" and "vmcnt(0)" in s:
            waited = True
    stream, = (v for k, v in runs.items() if "pw_stream_kernel" in k)
    rows, = (v for k, v in runs.items() if "rows_staging" in k)
    assert sorted(stream) == [4, 16, 16], runs
    assert sorted(rows) == [4, 4, 4, 4], runs
