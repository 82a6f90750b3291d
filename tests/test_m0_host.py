"""The load from memory straight to the LDS takes its LDS address in the register M0.  Compiled here for gfx950, not run:
what the compiler's own code had in M0 must not be taken for still there behind such a load."""

import os
import subprocess

from paper_2605_17862_amd import build as b

SOURCE = """
#include "fopd_lm_head.hip"
typedef const __attribute__((address_space(1))) unsigned* from;
typedef __attribute__((address_space(3))) unsigned* to;
__global__ void around(const unsigned* p, unsigned* out) {
  __shared__ unsigned lds[4096];
  __builtin_amdgcn_global_load_lds((from)p + threadIdx.x, (to)lds, 4, 0, 0);
  fopd::load_to_lds(reinterpret_cast<const char*>(p), threadIdx.x * 16, 8192);
  __builtin_amdgcn_global_load_lds((from)p + 64 + threadIdx.x, (to)lds, 4, 1024, 0);
  __syncthreads();
  out[threadIdx.x] = lds[threadIdx.x] + lds[256 + threadIdx.x];
}
"""


def test_m0_is_written_again_behind_a_load_to_the_lds(tmp_path):
    src, asm = tmp_path / "around.hip", tmp_path / "around.s"
    src.write_text(SOURCE)
    flags = [f for f in b.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-I", os.path.join(b.ROOT, "include"), "-I", os.path.join(b.PKG, "csrc"), "--cuda-device-only", "-S",
                    str(src), "-o", str(asm)], check=True, capture_output=True)
    lines = [l.strip() for l in asm.read_text().splitlines()]
    body = lines[next(i for i, l in enumerate(lines) if l.startswith("_Z6around")):]
    loads = [i for i, l in enumerate(body) if l.startswith("global_load_lds_dword")][:3]
    assert [body[i].split()[0] for i in loads] == ["global_load_lds_dword", "global_load_lds_dwordx4",
                                                   "global_load_lds_dword"]
    writes = lambda a, z: any(l.startswith("s_") and l.split()[1:2] == ["m0,"] for l in body[a:z])
    assert writes(0, loads[0]) and writes(loads[0], loads[1]) and writes(loads[1], loads[2])
