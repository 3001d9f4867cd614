"""CPU-only checks of what the library asks the HIP runtime for: in a process of its own the runtime's launch calls are answered by a stand-in that
notes them, so nothing is launched and no pointer is followed."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>
struct dim3 { uint32_t x, y, z; };
static std::map<const void*, std::string> names;
static std::map<const void*, size_t> allowed;
static std::map<const void*, long> launches;
static long beyond = 0, total = 0;
static struct { dim3 grid, block; size_t lds; void* stream; } config;
extern "C" {
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[host] = name; }
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void* kernel, int attribute, int value) {
    if (attribute == 8) allowed[kernel] = (size_t)value;              // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) { config = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) { *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream; return 0; }
int hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t lds, void*) {
    ++total;
    ++launches[kernel];
    const size_t most = allowed.count(kernel) ? allowed[kernel] : 64 * 1024;
    if (lds > most) {
        if (beyond++ < 5) printf("%zu bytes of LDS, %zu allowed: %s\n", lds, most, names[kernel].c_str());
    }
    return 0;
}
long launches_seen() { return total; }
long launches_beyond() { return beyond; }
void print_never_launched(const char* part) {
    for (auto& k : names)
        if (!launches.count(k.first) && k.second.find(part) != std::string::npos) printf("never launched: %s\n", k.second.c_str());
}
}
"""

CALLS = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)             # before the library: its calls are looked up here first
sys.path.insert(0, sys.argv[2])
import paper_2406_10181_amd as L
fake, big = 0x1000, 1 << 40
for r in (16, 256, 260, 512, 516, 1024, 1028, 2048):                 # small ones first: what a kernel was allowed must not depend on the first call
    for m in (300, 2000, 3000, 4096, 4100, 9000, 20000):
        for n in (264, 266, 267, 4096, 4104):
            for d in (2, 3, 4, 8, 16, 64):
                if d > r: continue
                for code in (0, 1, 2):
                    L.lsp_decompress_apply(fake, fake, fake, fake, fake, fake, m, n, r, d, code)
                    L.lsp_estimation_bias(fake, fake, fake, fake, fake, fake, m, n, r, d, fake, fake, big, code)
                    L.lsp_compress_planned(fake, fake, m, n, r, d, fake, code, fake, big)
                L.lsp_plan_build_async(fake, fake, fake, fake, m, n, r, d, fake, big, fake, big, None)
    L.lsp_compress(fake, fake, fake, fake, fake, 4096, 4096, r, 8, fake, 2, fake, big)
shim.launches_seen.restype = shim.launches_beyond.restype = ctypes.c_long
print("launches", shim.launches_seen() > 5000, "beyond", shim.launches_beyond())
shim.print_never_launched(b"k_decompress")
sys.stdout.flush()
"""


@pytest.fixture(scope="module")
def outcome(tmp_path_factory):
    where = tmp_path_factory.mktemp("stand_in")
    src, so = where / "stand_in.cpp", where / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    out = subprocess.run([sys.executable, "-c", CALLS, str(so), ROOT], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, (out.returncode, out.stdout[-2000:], out.stderr[-2000:])
    return out.stdout


def test_no_launch_asks_for_more_lds_than_its_kernel_was_allowed(outcome):
    assert "launches True beyond 0" in outcome, outcome[-2000:]


def test_every_kernel_of_the_expand_side_is_launched_for_some_shape(outcome):
    assert "never launched" not in outcome, outcome[-2000:]
