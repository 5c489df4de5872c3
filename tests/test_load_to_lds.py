"""The staging load of the attention kernels (load_to_lds, inline assembly that the compiler's own hazard pass does not look
into): its scalar operands may come straight from a vector instruction, which needs five wait states in front of the load, and
m0, which it goes by, may belong to one of the compiler's own loads before and after it.  Compiled here, read as assembly."""
import os
import re
import subprocess

import pytest

from paper_2602_03216_amd import build

SOURCE = r"""
#include "attend_common.h"
using namespace tsa;
using namespace tsa::attend_detail;
using lds_ptr = __attribute__((address_space(3))) char*;

__global__ void operand_from_vector(const float* p, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[4096];
  const float a = p[threadIdx.x], b = p[threadIdx.x + 64];
  load_to_lds(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, __builtin_bit_cast(int, a * b), (int)(uintptr_t)(lds_ptr)lds);
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}

__global__ void slot_from_vector(const float* p, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[4096];
  const float a = p[threadIdx.x], b = p[threadIdx.x + 64];
  load_to_lds(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, 0, __builtin_bit_cast(int, a * b));
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}

__global__ void between_builtins(const int* p, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[8192];
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, n, 0x00020000);
  auto* at = (__attribute__((address_space(3))) void*)lds;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, 16 * threadIdx.x, 0, 0, 0);
  load_to_lds(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, 1024, (int)(uintptr_t)(lds_ptr)lds + 4096);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, 16 * threadIdx.x, 2048, 0, 0);
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}
"""
CSRC = build.CSRC


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """kernel name -> its instructions"""
    try:
        hipcc = build.hipcc_path()
    except RuntimeError as e:
        pytest.skip(str(e))
    src = tmp_path_factory.mktemp("isa") / "staging.hip"
    src.write_text(SOURCE)
    run = subprocess.run([hipcc, *build.FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", "-"], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    code, name = {}, None
    for line in run.stdout.splitlines():
        line = line.split(";")[0].strip()
        label = re.match(r"_Z\d+(\w+?)PK\w+:$", line)
        if label:
            name = label.group(1)
            code[name] = []
        elif line.startswith("s_endpgm"):
            name = None
        elif name and line and not line.startswith(".") and not line.endswith(":"):
            code[name].append(line)
    assert set(code) == {"operand_from_vector", "slot_from_vector", "between_builtins"}
    return code


def _lds_loads(code):
    at = [i for i, line in enumerate(code) if line.startswith("buffer_load") and line.endswith(" lds")]
    assert at
    return at


def _scalars(text):
    """numbers of the scalar registers named in `text`, m0 as -1"""
    regs = {int(n) for n in re.findall(r"\bs(\d+)\b", text)}
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs | ({-1} if re.search(r"\bm0\b", text) else set())


@pytest.mark.parametrize("name", ["operand_from_vector", "slot_from_vector", "between_builtins"])
def test_wait_states_behind_vector_writes(kernels, name):
    code = kernels[name]
    for at in _lds_loads(code):
        reads, waited = _scalars(code[at]) | {-1}, 0
        for line in reversed(code[:at]):
            if waited >= 5:
                break
            op, _, args = line.partition(" ")
            if op.startswith("v_"):
                assert not (_scalars(args.split(",")[0]) & reads), (line, code[at], waited)
            waited += int(args, 0) + 1 if op == "s_nop" else 1


def test_m0_is_set_for_every_load(kernels):
    code = kernels["between_builtins"]
    loads = _lds_loads(code)
    assert len(loads) == 3
    for first, second in zip(loads, loads[1:]):
        assert any(_scalars(line.partition(" ")[2].split(",")[0]) == {-1} for line in code[first:second]), code[first:second + 1]
