"""The instruction forms that teams of workgroups on one XCD rely on (team.h), read
from the compiler's output: a store for the XCD's L2 writes through the L1 and
no further (sc0), a store for all XCDs goes on (sc1), loads pass over the L1, and
a read-modify-write is the same instruction at workgroup and agent scope."""
import os
import re
import subprocess

import pytest

from paper_1812_10499_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCE = """
#include "team.h"
using namespace sssp;
extern "C" {
__global__ void near32(int32_t *p) { put(p, 1, true); stores_done(); }
__global__ void far32(int32_t *p) { put(p, 1, false); }
__global__ void near64(unsigned long long *p) { put64(p, 1ull, true); }
__global__ void far64(unsigned long long *p) { put64(p, 1ull, false); }
__global__ void look32(const int32_t *p, int32_t *o) { *o = ld_relaxed(p); }
__global__ void look64(const unsigned long long *p, unsigned long long *o) { *o = ld_relaxed64(p); }
__global__ void swap_wg(unsigned long long *p, unsigned long long *o) {
  *o = __hip_atomic_exchange(p, 5ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__global__ void swap_agent(unsigned long long *p, unsigned long long *o) {
  *o = __hip_atomic_exchange(p, 5ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_instruction_forms(tmp_path):
    src, asm = tmp_path / "forms.hip", tmp_path / "forms.s"
    src.write_text(SOURCE)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([HIPCC] + flags + ["-I", build.CSRC, "--cuda-device-only", "-S", "-o",
                                             str(asm), str(src)], stderr=subprocess.DEVNULL)
    text = asm.read_text()

    def line(name, op):
        body = text[text.index("\n%s:" % name):]
        body = body[:body.index("s_endpgm")]
        found = re.findall(r"^\s+(%s\S*)\s[^;\n]*?((?: sc[01]| nt)*)\s*$" % op, body, re.M)
        assert found, (name, body)
        return found[0][0], set(found[0][1].split()), body

    for name in ("near32", "near64"):
        assert line(name, "global_store")[1] == {"sc0"}, name
    for name in ("far32", "far64"):
        assert line(name, "global_store")[1] == {"sc1"}, name
    for name in ("look32", "look64"):
        assert "sc1" in line(name, "global_load")[1], name
    assert line("swap_wg", "global_atomic")[:2] == line("swap_agent", "global_atomic")[:2]
    body = line("near32", "global_store")[2]
    assert body.index("global_store") < body.index("s_waitcnt vmcnt(0)")
