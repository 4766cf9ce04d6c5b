"""Kernels that spill registers to scratch memory, from the metadata of the code objects in the built library (no GPU)."""
import os
import struct
import subprocess

import msgpack

from paper_2101_06983_amd import build

# bytes of scratch a lane may use; every kernel that is not named here uses none
SPILLS = {"gemm_nt_kernel<true, ": 72, "grad128_kernel<true, true>": 12, "planes_grad_kernel<1, 2, 8, false>": 124, "mlp_dh_tiled_kernel<64>": 232,
          "stats_mfma_kernel<(gc::StatsMode)1, 256>": 20}
NT_AMDGPU_METADATA, SHT_NOTE, EM_AMDGPU = 32, 7, 224


def scratch_bytes(path):
    """name -> bytes of scratch of every kernel: the notes of the 64-bit AMDGPU ELF images inside the library."""
    lib = open(path, "rb").read()
    out, at = {}, lib.find(b"\x7fELF", 1)   # (the first image is the library's own)
    while at >= 0:
        machine, = struct.unpack_from("<H", lib, at + 18)
        shoff, = struct.unpack_from("<Q", lib, at + 40)
        shsize, shnum = struct.unpack_from("<HH", lib, at + 58)
        for k in range(shnum if machine == EM_AMDGPU else 0):
            kind, = struct.unpack_from("<I", lib, at + shoff + k * shsize + 4)
            off, = struct.unpack_from("<Q", lib, at + shoff + k * shsize + 24)
            if kind != SHT_NOTE:
                continue
            name_len, desc_len, note = struct.unpack_from("<III", lib, at + off)
            if note == NT_AMDGPU_METADATA:
                desc = at + off + 12 + (name_len + 3) // 4 * 4
                for kernel in msgpack.unpackb(lib[desc:desc + desc_len])["amdhsa.kernels"]:
                    out[kernel[".name"]] = kernel[".private_segment_fixed_size"]
        at = lib.find(b"\x7fELF", at + 4)
    return out


def test_no_kernel_spills_that_is_not_known_to():
    if not os.path.exists(build.OUT):
        build.build()
    found = scratch_bytes(build.OUT)
    names = subprocess.run(["c++filt"] + list(found), capture_output=True, text=True, check=True).stdout.splitlines()
    assert any("planes_grad_kernel<3, 2, 8, false>" in n for n in names) and len(found) > 50
    bad = {n: s for n, s in zip(names, found.values()) if s > max([b for key, b in SPILLS.items() if key in n], default=0)}
    assert not bad, bad
