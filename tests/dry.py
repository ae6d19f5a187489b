"""The library's host code without a GPU: its object files linked with a HIP runtime that launches nothing and writes down every
call, so that a test on the CPU can say which kernels a call enqueues, and with which grid.  Pointers are never dereferenced."""
import ctypes
import os
import re
import subprocess

from paper_2604_24013_amd import binding, build

# launches and copies go into the log, one line each, and with their streams and the events between these into another; the number
# of compute units is COMMFUSE_DRY_CUS, and with COMMFUSE_DRY_CAPTURING every stream is being captured
RUNTIME = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
struct dim3 { uint32_t x, y, z; };
static std::string text, order;
static std::string at(void *stream) { return std::to_string((unsigned long)stream) + " "; }
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static dim3 g_grid, g_block; static size_t g_shared; static void *g_stream; static char sym[16]; static long events;
extern "C" {
const char *dry_log() { return text.c_str(); }
const char *dry_order() { return order.c_str(); }
void dry_clear() { text.clear(); order.clear(); }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{ names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) { g_grid = g; g_block = b; g_shared = s; g_stream = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) { *g = g_grid; *b = g_block; *s = g_shared; *st = g_stream; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, void *s)
{ order += "launch " + at(s) + "0\n"; text += names()[f] + " " + std::to_string(g.x) + " " + std::to_string(b.x) + "\n"; return 0; }
int hipMemcpyAsync(void *, const void *, size_t n, int, void *s) { order += "copy " + at(s) + "0\n"; text += "memcpy " + std::to_string(n) + " 0\n"; return 0; }
int hipMemsetAsync(void *, int, size_t n, void *) { text += "memset " + std::to_string(n) + " 0\n"; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { const char *e = getenv("COMMFUSE_DRY_CUS"); *v = e ? atoi(e) : 256; return 0; }
int hipGetDevice(int *d) { const char *e = getenv("COMMFUSE_DRY_CUS"); *d = e ? atoi(e) / 8 % 64 : 0; return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "dry"; }
int hipGetSymbolAddress(void **p, const void *) { *p = sym; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = (void *)++events; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *e, void *s) { order += "record " + at(s) + at(e) + "\n"; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned) { order += "wait " + at(s) + at(e) + "\n"; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamIsCapturing(void *, int *v) { *v = getenv("COMMFUSE_DRY_CAPTURING") != nullptr; return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = sym; return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphInstantiate(void **g, void *, void *, char *, size_t) { *g = sym; return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
}
"""


class Dry:
    """``binding``'s functions on the dry library: ``calls(f)`` runs ``f()`` and returns [(kernel or copy, grid or bytes, block)]."""

    def __init__(self, folder):
        objs = [os.path.join(build.CSRC, s.replace(".hip", ".o")) for s in build.SOURCES]
        if not all(os.path.exists(o) for o in objs):
            build.build()
        src, so = os.path.join(folder, "runtime.cpp"), os.path.join(folder, "libdry.so")
        with open(src, "w") as f:
            f.write(RUNTIME)
        subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-Wl,-Bsymbolic", "-o", so, src] + objs, check=True)
        real, binding._lib, path = binding._lib, None, binding.LIB_PATH
        try:
            binding.LIB_PATH = so
            self.lib = binding.load()
        finally:
            binding.LIB_PATH, binding._lib = path, real
        self.lib.dry_log.restype = self.lib.dry_order.restype = ctypes.c_char_p
        self.names = {}

    def calls(self, f):
        real, binding._lib = binding._lib, self.lib
        try:
            self.lib.dry_clear()
            f()
            lines = [l.split() for l in self.lib.dry_log().decode().splitlines()]
        finally:
            binding._lib = real
        new = sorted({l[0] for l in lines if l[0].startswith("_Z")} - set(self.names))
        if new:
            out = subprocess.run(["c++filt"], input="\n".join(new), capture_output=True, text=True, check=True).stdout.splitlines()
            self.names.update(zip(new, (re.sub(r"\(anonymous namespace\)::|cf::|^void ", "", n).split("(")[0] for n in out)))
        return [(self.names.get(l[0], l[0]), int(l[1]), int(l[2])) for l in lines]

    def order(self, f):
        """[(launch, copy, record or wait, stream, event)] of ``f()``."""
        self.calls(f)
        return [(l[0], int(l[1]), int(l[2])) for l in (x.split() for x in self.lib.dry_order().decode().splitlines())]
