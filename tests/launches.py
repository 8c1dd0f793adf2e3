"""What a product launches, without a GPU: a program that links the library with launch calls of its own, which note the kernel and do nothing."""
import os
import re
import subprocess

from paper_2501_04012_amd import build

# the runtime calls of the library: launches are noted, memory is an address
STUBS = r"""
#include <dlfcn.h>
#include <cstdio>
#include <string>
#include "common.h"
#define STUB extern "C" __attribute__((visibility("default"))) hipError_t
static std::string seen;
static size_t address = 1 << 20;
STUB hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  Dl_info info;
  seen += std::string(" ") + (dladdr(f, &info) && info.dli_sname ? info.dli_sname : "unknown");
  return hipSuccess;
}
STUB __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
STUB __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
STUB hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
STUB hipGetLastError() { return hipSuccess; }
STUB hipMalloc(void** p, size_t n) { *p = (void*)address; address += (n + 4095) / 4096 * 4096; return hipSuccess; }
STUB hipFree(void*) { return hipSuccess; }
STUB hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
STUB hipMemGetInfo(size_t* free, size_t* total) { *free = *total = (size_t)288 << 30; return hipSuccess; }
STUB hipDeviceSynchronize() { return hipSuccess; }
STUB hipGetDevice(int* d) { *d = 0; return hipSuccess; }
"""
SOURCE = STUBS + r"""
int main() {
  using namespace fc;
  int mode, M, N, K, packed;
  size_t lent;
  while (scanf("%d %d %d %d %d %zu", &mode, &M, &N, &K, &packed, &lent) == 6) {
    EpiParams ep;                                        // addresses that are never used
    ep.out = ep.q = ep.k = ep.v = (void*)4096;
    ep.ldo = N; ep.D = mode == EPI_HEADS ? N / 3 : N; ep.hd = 32; ep.heads = ep.D / 32; ep.tokens = M; ep.layer_stride = (size_t)M * N;
    ep.T = 1; ep.H = M; ep.W = 1; ep.p = 1; ep.C = N; ep.eps = (float*)4096;
    void* const scratch = lent ? (void*)4096 : nullptr;
    seen.clear();
    const hipError_t e = launch_gemm(1, mode, (void*)4096, (void*)4096, M, N, K, ep, nullptr, scratch, lent, packed ? (void*)4096 : nullptr);
    printf("%d %d%s\n", (int)e, (int)bf16_form(M, N, K, packed, scratch, lent), seen.c_str());
  }
}
"""


def program(folder, source):
    """Compiles a host program against the library's headers and links the library."""
    src, exe = str(folder / "program.hip"), str(folder / "program")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run([build.HIPCC, "-std=c++17", "-O1", "-w", "--offload-host-only", "-I" + build.CSRC, "-I" + os.path.join(build.HERE, "..", "include"), "-c", src, "-o", exe + ".o"], check=True)
    subprocess.run([build.HIPCC, "-rdynamic", exe + ".o", build.LIB_PATH, "-Wl,-rpath," + os.path.dirname(build.LIB_PATH), "-ldl", "-o", exe], check=True)
    return exe


def kernels(symbols):
    """[(kernel, first two of its numbers: rows and columns of a tile)]"""
    parts = [re.match(r"_ZN2fc\d+(k_[a-z0-9_]+?)(?:ILi(\d+)ELi(\d+)E|I|E)", n).groups() for n in symbols]
    return [(k, int(a or 0), int(b or 0)) for k, a, b in parts]


class Launches:
    def __init__(self, folder):
        self.exe = program(folder, SOURCE)

    def __call__(self, products):
        """products: (mode, M, N, K, packed weights, bytes of scratch memory).  For each: status, bf16_form, [(kernel, tile rows, columns)]."""
        text = "".join("%d %d %d %d %d %d\n" % tuple(map(int, p)) for p in products)
        out = subprocess.run([self.exe], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        assert len(out) == len(products)
        found = []
        for line in out:
            status, form, *names = line.split()
            found.append((int(status), int(form), kernels(names)))
        return found
