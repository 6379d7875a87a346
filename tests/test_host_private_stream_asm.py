"""CPU test of the direct-to-LDS loads that are written in assembly (PrivateStream): a small kernel around
them is compiled for gfx950 and its device assembly is checked for what the compiler cannot know by itself."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_17051_amd.build import CSRC, HIPCC_FLAGS

SOURCE = """
#include "mfma_common.hpp"
using namespace astro;
// the compiler's own loads to one LDS address (held in m0) before and after the loads from assembly
extern "C" __global__ void __launch_bounds__(64) own_load_after(const __bf16* a, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * 4096];
  const RowSegment s = make_segment(a, 64, n, 64);
  TileStreamer<64, 8, 1> ts;
  ts.init();
  PrivateStream<64> ps;
  ps.init(threadIdx.x & 63);
  ts.issue(s, ts.lane_offset(s), 0, lds);
  ps.issue(segment_words(a, 64, n, 64), 128, 32, lds + 4096);
  ts.issue(s, ts.lane_offset(s), 64, lds);
  wait_vmem();
  __syncthreads();
  out[threadIdx.x] = *(int*)(lds + threadIdx.x * 4) + *(int*)(lds + 4096 + threadIdx.x * 4);
}
// the descriptor's words come out of vector registers right before the loads
extern "C" __global__ void __launch_bounds__(64) descriptor_from_lanes(const u32x4* words, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[4096];
  PrivateStream<64> ps;
  ps.init(threadIdx.x & 63);
  const u32x4 w = words[threadIdx.x];
  u32x4 r;
  for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_readfirstlane(w[i]);
  ps.issue(r, 128, 0, lds);
  wait_vmem();
  __syncthreads();
  out[threadIdx.x] = *(int*)(lds + threadIdx.x * 4);
}
"""


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """kernel name -> its instructions, each with whether it comes from an asm block"""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")
    (d / "t.hip").write_text(SOURCE)
    r = subprocess.run([hipcc, *HIPCC_FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(d / "t.hip"), "-o", str(d / "t.s")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found, name, in_asm = {}, None, False
    for line in (d / "t.s").read_text().splitlines():
        if line and not line[0].isspace() and line.split(":")[0].isidentifier():
            name = line.split(":")[0]
            found[name] = []
        text = line.strip()
        if text.startswith((";;#ASMSTART", ";APP")):
            in_asm = True
        elif text.startswith((";;#ASMEND", ";NO_APP")):
            in_asm = False
        elif name and line[:1].isspace() and text[:2] in ("s_", "v_", "bu", "ds", "gl"):
            found[name].append((text.split(";")[0].strip(), in_asm))
            if text.startswith("s_endpgm"):
                name = None
    return found


def test_the_compilers_own_load_sets_its_lds_address_again_after_the_assembly(kernels):
    code = kernels["own_load_after"]
    loads = [i for i, (t, _) in enumerate(code) if t.startswith("buffer_load") and t.endswith("lds")]
    from_asm = [i for i in loads if code[i][1]]
    own_after = [i for i in loads if not code[i][1] and i > from_asm[-1]]
    assert len(from_asm) == 4 and len(own_after) == 1 and len(loads) == 6
    between = [t for t, _ in code[from_asm[-1] + 1:own_after[0]]]
    assert any(t.startswith("s_mov_b32 m0,") for t in between), between


def test_wait_states_between_a_descriptor_written_by_a_vector_instruction_and_its_use(kernels):
    """A buffer load that reads a scalar register a vector instruction wrote needs five wait states in between;
    the compiler inserts them before its own loads only."""
    code = [t for t, _ in kernels["descriptor_from_lanes"]]
    load = next(i for i, t in enumerate(code) if t.startswith("buffer_load"))
    first, last = map(int, re.search(r"s\[(\d+):(\d+)\]", code[load]).groups())
    words = {f"s{r}" for r in range(first, last + 1)}
    write = max(i for i in range(load) if code[i].startswith("v_read") and code[i].split()[1].rstrip(",") in words)
    states = sum(int(t.split()[1]) + 1 if t.startswith("s_nop") else 1 for t in code[write + 1:load])
    assert states >= 5, code[write:load + 1]
