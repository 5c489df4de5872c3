"""The staging load of the attention kernels (load_to_lds, inline assembly that the compiler's own hazard pass does not look
into): a load needs five wait states behind a vector instruction that wrote one of its scalar operands, and m0, which it goes
by, may belong to one of the compiler's own loads before and after it.  Compiled here with the library's flags and read as
assembly: small kernels around the padded form, where the operands do come out of vector instructions, and every load of the
kernels themselves."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

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
  load_to_lds<true>(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, __builtin_bit_cast(int, a * b), (int)(uintptr_t)(lds_ptr)lds);
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}

__global__ void slot_from_vector(const float* p, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[4096];
  const float a = p[threadIdx.x], b = p[threadIdx.x + 64];
  load_to_lds<true>(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, 0, __builtin_bit_cast(int, a * b));
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}

template <bool PAD>
__global__ void between_builtins(const int* p, int n, int* out) {
  __shared__ __attribute__((aligned(1024))) char lds[8192];
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, n, 0x00020000);
  auto* at = (__attribute__((address_space(3))) void*)lds;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, 16 * threadIdx.x, 0, 0, 0);
  load_to_lds<PAD>(rsrc_words((const __bf16*)p, n), 16 * threadIdx.x, 1024, (int)(uintptr_t)(lds_ptr)lds + 4096);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, 16 * threadIdx.x, 2048, 0, 0);
  wait_loads();
  __syncthreads();
  out[threadIdx.x] = ((int*)lds)[threadIdx.x];
}
template __global__ void between_builtins<true>(const int*, int, int*);
template __global__ void between_builtins<false>(const int*, int, int*);
"""
CSRC = build.CSRC


def _assembly(src, extra=()):
    """kernel name -> its lines, labels among them"""
    run = subprocess.run([build.hipcc_path(), *build.FLAGS, *extra, "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", "-"],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    kernels, name = {}, None
    for line in run.stdout.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            name = line[:-1]
            kernels[name] = []
        elif line.startswith((".section", ".end_amdhsa_kernel")):
            name = None
        elif name and line and (line.endswith(":") or not line.startswith(".")):
            kernels[name].append(line)
    return kernels


@pytest.fixture(scope="module")
def hipcc():
    try:
        return build.hipcc_path()
    except RuntimeError as e:
        pytest.skip(str(e))


@pytest.fixture(scope="module")
def small(hipcc, tmp_path_factory):
    src = tmp_path_factory.mktemp("isa") / "staging.hip"
    src.write_text(SOURCE)
    return _assembly(src)


@pytest.fixture(scope="module")
def library(hipcc):
    files = ["attend.hip", "attend_split.hip"]
    with ThreadPoolExecutor(len(files)) as pool:
        parts = pool.map(lambda f: _assembly(os.path.join(CSRC, f), build.EXTRA[f]), files)
    return {name: code for part in parts for name, code in part.items()}


def _loads(code):
    return [i for i, line in enumerate(code) if line.startswith("buffer_load") and line.endswith(" lds")]


def _scalars(text):
    """numbers of the scalar registers named in `text`, m0 as -1"""
    regs = {int(n) for n in re.findall(r"\bs(\d+)\b", text)}
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs | ({-1} if re.search(r"\bm0\b", text) else set())


def _target(line):
    return _scalars(line.partition(" ")[2].split(",")[0])


def _short_waits(code):
    """(vector instruction, load) pairs with fewer than five wait states between them on some way to the load"""
    jumps = {}
    for i, line in enumerate(code):
        if line.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(line.split()[-1] + ":", []).append(i)
    bad = []
    for load in _loads(code):
        reads = _scalars(code[load]) | {-1}
        todo, seen = [(load, 0)], set()
        while todo:
            i, waited = todo.pop()
            if (i, waited) in seen or waited >= 5:
                continue
            seen.add((i, waited))
            if code[i].endswith(":"):                          # `i` itself is counted; now what comes before it
                todo += [(j, waited + 1) for j in jumps.get(code[i], [])]
            if i == 0 or code[i - 1].startswith(("s_branch", "s_endpgm", "s_setpc")):
                continue
            before = code[i - 1]
            op, _, args = before.partition(" ")
            if op.startswith("v_") and _target(before) & reads:
                bad.append((before, code[load], waited))
                continue
            todo.append((i - 1, waited + (0 if before.endswith(":") else int(args, 0) + 1 if op == "s_nop" else 1)))
    return bad


def test_the_padded_form_behind_vector_writes(small):
    for name, code in small.items():
        assert _loads(code) and not _short_waits(code), name
    assert any(_target(line) & (_scalars(code[_loads(code)[0]]) | {-1}) and line.startswith("v_readfirstlane")
               for code in small.values() for line in code)      # (there is one to be behind of)


def test_m0_is_set_for_every_load(small):
    for name in [n for n in small if "between_builtins" in n]:
        code = small[name]
        loads = _loads(code)
        assert len(loads) == 3
        for first, second in zip(loads, loads[1:]):
            writes = [i for i in range(first, second) if _target(code[i]) == {-1}]
            assert writes and writes[-1] < second - 1, code[first:second + 1]         # (a wait state behind it)


def test_every_load_of_the_attention_kernels(library):
    kernels = [n for n in library if "attend" in n]
    assert len(kernels) == 24
    for name in kernels:
        assert len(_loads(library[name])) >= 7 and not _short_waits(library[name]), (name, _short_waits(library[name])[:3])


def test_the_search_sees_what_it_looks_for():
    """on listings made up here: a short wait straight, across a label, and on the way of a jump; a long one; another register"""
    load = "buffer_load_dwordx4 v1, s[4:7], s8 offen lds"
    pad = ["s_nop 4"]
    assert _short_waits(["v_readlane_b32 s8, v2, 1", "s_nop 3", load])
    assert _short_waits(["v_readlane_b32 s5, v2, 1", ".L1:", "s_nop 0", load])
    assert _short_waits(["v_readfirstlane_b32 m0, v2", "s_nop 0", load])
    assert _short_waits(["v_readlane_b32 s8, v2, 1", "s_cbranch_scc1 .L1", *pad, "s_endpgm", ".L1:", "s_nop 0", load])
    assert not _short_waits(["v_readlane_b32 s8, v2, 1", "s_branch .L2", ".L1:", "s_nop 0", load])
    assert not _short_waits(["v_readlane_b32 s8, v2, 1", *pad, load])
    assert not _short_waits(["v_readlane_b32 s9, v2, 1", load])
    assert not _short_waits(["v_mov_b32_e32 v8, s8", load])
