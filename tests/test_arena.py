"""Device memory of a context after a failed allocation: the next call asks for the buffers
that are still missing and for no other, and none is left without memory.  The allocator of
ctx.h against a stand-in for the runtime that fails on demand (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1606_06201_amd", "csrc")

PROGRAM = r"""
#include "ctx.h"
#include <cstdio>
#include <cstdlib>
static int calls = 0, fail_at = -1, last = 0;
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (++calls == fail_at) { last = 1; return hipErrorOutOfMemory; }
  *p = std::malloc(n);
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
extern "C" hipError_t hipGetLastError() { const int l = last; last = 0; return l ? hipErrorOutOfMemory : hipSuccess; }
using namespace ipmg;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  for (int at = 1; at <= 4; ++at) {
    Arena a;
    void* S[4] = {nullptr, nullptr, nullptr, nullptr};
    const size_t bytes[4] = {Arena::SMALL, 1000, 3 * Arena::SMALL, Arena::SMALL};
    auto ensure = [&] { for (int k = 0; k < 4; ++k) a.need(S[k], bytes[k]); };
    calls = 0;
    fail_at = at;
    bool failed = false;
    try { ensure(); } catch (const Error& e) { failed = e.code == IPMG_E_NOMEM; }
    CHECK(failed && last == 0);
    for (int k = 0; k < 4; ++k) CHECK((S[k] != nullptr) == (k < at - 1));
    void* had[4] = {S[0], S[1], S[2], S[3]};
    ensure();
    CHECK(calls == 5);
    for (int k = 0; k < 4; ++k) CHECK(S[k] != nullptr && (had[k] == nullptr || had[k] == S[k]));
    ensure();
    CHECK(calls == 5);
    a.release();
  }
  return 0;
}
"""


@pytest.mark.skipif(not shutil.which("hipcc"), reason="hipcc not found")
def test_buffers_after_a_failed_allocation(tmp_path):
    src, exe = tmp_path / "arena.cpp", tmp_path / "arena"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", "--offload-host-only", "-x", "hip", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
