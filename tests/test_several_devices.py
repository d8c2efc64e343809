"""What the library asks the runtime for on a second device, on the CPU: a program with a HIP runtime of its own (two
devices, host memory, launches that are only noted) loads the built library and calls the matrix entry points."""
import subprocess

import paper_2605_30010_amd as et
from paper_2605_30010_amd.build import LIB, ROOT

PROGRAM = r"""
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <map>
#include <utility>
struct Dim3 { uint32_t x, y, z; };
static int device, launches, big, refused;
static std::map<std::pair<int, const void *>, int> allowed;      // dynamic LDS by device and kernel
static Dim3 pushed[2];
static size_t pushed_lds;
static void *pushed_stream;
extern "C" {
// Handles are passed through; nothing is registered, copied or launched.
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) {
  pushed[0] = grid; pushed[1] = block; pushed_lds = lds; pushed_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream) {
  *grid = pushed[0]; *block = pushed[1]; *lds = pushed_lds; *stream = pushed_stream;
  return 0;
}
int hipLaunchKernel(const void *kernel, Dim3, Dim3, void **, size_t lds, void *) {
  ++launches;
  if (lds <= 64 * 1024) return 0;
  ++big;
  auto it = allowed.find({device, kernel});
  if (it == allowed.end() || (size_t)it->second < lds) ++refused;
  return 0;
}
int hipFuncSetAttribute(const void *kernel, int, int bytes) { allowed[{device, kernel}] = bytes; return 0; }
int hipGetDevice(int *d) { *d = device; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return ""; }
int hipMalloc(void **p, size_t n) { return (*p = malloc(n)) ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
}
int main(int, char **argv) {
  void *lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) { fprintf(stderr, "%s\n", dlerror()); return 2; }
  auto gemm = (int (*)(const void *, const void *, const float *, const void *, int, int, int, int, int, void *, void *))dlsym(lib, "et_gemm_bf16");
  auto attention = (int (*)(const void *, int, int, int, int, void *, void *))dlsym(lib, "et_attention_uniform");
  static char buf[64];                                           // (never looked into)
  for (device = 0; device < 2; ++device) {
    for (int cfg = -1; cfg < 6; ++cfg)
      for (int epilogue = 0; epilogue < 3; ++epilogue)
        if (gemm(buf, buf, (const float *)buf, buf, 300, 512, 128, epilogue, cfg, buf, nullptr)) return 3;
    for (int frames : {1, 2, 30})
      if (attention(buf, frames, 729, 16, 72, buf, nullptr)) return 4;
  }
  printf("%d %d %d\n", launches, big, refused);
  return 0;
}
"""


def test_each_device_is_asked_for_the_lds_of_its_own_launches(tmp_path):
    """More than 64 KiB of dynamic LDS are allowed by kernel and device: a launch on the second device has to have asked
    there as well."""
    et.load_library()
    src, exe = str(tmp_path / "devices.cpp"), str(tmp_path / "devices")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", src, "-o", exe, "-ldl"], check=True)
    run = subprocess.run([exe, LIB], capture_output=True, text=True, cwd=ROOT, timeout=120)
    assert run.returncode == 0, run.stderr
    launches, big, refused = map(int, run.stdout.split())
    assert launches >= 2 * (7 * 3 + 3) and big >= 2 * 15
    assert refused == 0, "%d of %d launches" % (refused, big)
