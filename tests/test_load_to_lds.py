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
