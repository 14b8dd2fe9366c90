"""What the compiler makes of load_to_lds and wait_vm (csrc/common.hpp), read from
the assembly of small kernels compiled here for gfx950.  No GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2408_11052_amd import build as B

SOURCE = r'''
#include "common.hpp"
using namespace crl;
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* global_ptr;

// the compiler's own loads into LDS, to one address, around ours to another
extern "C" __global__ void own_loads_around(const char* a, char* o) {
  __shared__ __attribute__((aligned(1024))) char sm[4096];
  __builtin_amdgcn_global_load_lds((global_ptr)(a + threadIdx.x * 16), (lds_ptr)sm, 16, 0, 0);
  load_to_lds(a, threadIdx.x * 16, lds_address(sm + 2048));
  __builtin_amdgcn_global_load_lds((global_ptr)(a + 2048 + threadIdx.x * 16), (lds_ptr)sm, 16, 1024, 0);
  __syncthreads();
  o[threadIdx.x] = sm[threadIdx.x ^ 5];
}
// a base that vector instructions write just ahead of the load
extern "C" __global__ void base_from_lanes(const uint32_t* p, char* o) {
  __shared__ __attribute__((aligned(1024))) char sm[4096];
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)p[threadIdx.x]);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)p[threadIdx.x + 64]);
  const char* base = (const char*)(((uint64_t)hi << 32) | lo);
  bases_ready(base);
  load_to_lds(base, threadIdx.x * 16, lds_address(sm));
  wait_vm<0>();
  __syncthreads();
  o[threadIdx.x] = sm[threadIdx.x ^ 5];
}
// an LDS read before a counted wait and a barrier, its value used behind them:
// other waves may refill the tile once the barrier is passed
extern "C" __global__ void read_before_barrier(const char* a, float* o, int n) {
  __shared__ __attribute__((aligned(1024))) float sm[1024];
  load_to_lds(a, threadIdx.x * 16, lds_address(sm));
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  const float x = sm[threadIdx.x ^ 33];
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  if (n > 3) o[threadIdx.x] = x;
}
'''


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """Kernel name -> its instructions."""
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")
    (d / "k.hip").write_text(SOURCE)
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", str(d / "k.hip"), "-o", str(d / "k.s")],
                   check=True, capture_output=True)
    out = {}
    for name, body in re.findall(r"^(\w+):\s+; @\1$(.*?)^\.Lfunc_end", (d / "k.s").read_text(), re.S | re.M):
        lines = (l.split(";")[0].strip() for l in body.splitlines())
        out[name] = [l for l in lines if l and not l.startswith(".")]
    return out


def test_the_compiler_sets_m0_again_after_ours(asm):
    ins = asm["own_loads_around"]
    loads = [i for i, l in enumerate(ins) if l.startswith("global_load_lds")]
    assert len(loads) == 3
    between = ins[loads[1] + 1:loads[2]]
    assert any(re.match(r"s_\w+ m0,", l) for l in between), "\n".join(ins)


def _short_waits(ins):
    """Loads into LDS whose SGPR base a vector instruction writes fewer than five
    wait states ahead (looked back along the listing, past labels too)."""
    loads = bad = 0
    for i, l in enumerate(ins):
        m = re.match(r"global_load_lds_dwordx4 v\S+ s\[(\d+):(\d+)\]", l)
        if not m:
            continue
        loads += 1
        regs = {f"s{k}" for k in range(int(m[1]), int(m[2]) + 1)}
        states, k = 0, i - 1
        while k >= 0 and states < 5:
            op, _, args = ins[k].partition(" ")
            if op.startswith("v_read") and args.split(",")[0].strip() in regs:
                bad += 1
                break
            states += int(args, 0) + 1 if op == "s_nop" else 1
            k -= 1
    return loads, bad


def test_wait_states_between_a_lane_read_and_the_load(asm):
    # a vector instruction's SGPR result may be read by a vector-memory
    # instruction five wait states later
    ins = asm["base_from_lanes"]
    assert sum(l.startswith("v_readfirstlane") for l in ins) >= 2
    assert _short_waits(ins) == (1, 0), "\n".join(ins)


def test_wait_states_in_the_built_library(tmp_path):
    tools = [os.path.join(os.path.dirname(os.path.realpath(B.HIPCC)), "..", "llvm", "bin", t)
             for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]
    if not all(os.path.exists(t) for t in tools) or not os.path.exists(B.OUT):
        pytest.skip("no LLVM tools or no built library")
    fat = tmp_path / "fat"
    subprocess.run([tools[0], "--dump-section", f".hip_fatbin={fat}", B.OUT, str(tmp_path / "rest")], check=True)
    # one bundle a source file, each on a boundary of 4 KB
    data, magic, loads = fat.read_bytes(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    starts = [m.start() for m in re.finditer(magic, data)]
    for a, b in zip(starts, starts[1:] + [len(data)]):
        (tmp_path / "bundle").write_bytes(data[a:b])
        subprocess.run([tools[1], "--unbundle", "--type=o", f"--targets=hipv4-amdgcn-amd-amdhsa--{B.ARCH}",
                        f"--input={tmp_path / 'bundle'}", f"--output={tmp_path / 'obj'}"], check=True)
        text = subprocess.run([tools[2], "-d", "--no-show-raw-insn", str(tmp_path / "obj")], check=True,
                              capture_output=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\w+)>:$(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.S | re.M):
            n, bad = _short_waits([l.split("//")[0].strip() for l in body.splitlines() if l.strip()])
            loads += n
            assert bad == 0, name
    assert loads > 100


def test_lds_reads_stay_before_the_counted_wait(asm):
    ins = asm["read_before_barrier"]
    read = next(i for i, l in enumerate(ins) if l.startswith("ds_read"))
    barriers = [i for i, l in enumerate(ins) if l == "s_barrier"]
    assert len(barriers) == 2 and barriers[0] < read < barriers[1], "\n".join(ins)
    # and the read has arrived by then
    assert any(l.startswith("s_waitcnt") and "lgkmcnt(0)" in l for l in ins[read:barriers[1]])
