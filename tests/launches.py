"""Which kernels a call of the library launches, without a GPU: a process of its own loads libwersa.so on a stand-in for the HIP runtime
that notes launches and runs nothing."""
import json
import os
import re
import subprocess
import sys
import tempfile

STAND_IN = r"""
#include <stddef.h>
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void *host; const char *name; } kernels[4096];
static int count, last_error, fail_attributes;
static dim3 pushed_grid, pushed_block;
static size_t pushed_lds;
static void *pushed_stream;
static FILE *out;
void stand_in_setup(const char *path, int fail) { out = fopen(path, "w"); fail_attributes = fail; }
void stand_in_call(int status) { fprintf(out, "= %d %d\n", status, last_error); last_error = 0; fflush(out); }
void **__hipRegisterFatBinary(const void *d) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void **m, const void *host, char *d, const char *name, unsigned t, void *a, void *b, void *c, void *e, int *w) {
  kernels[count].host = host;
  kernels[count++].name = name;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *st) { pushed_grid = g; pushed_block = b; pushed_lds = lds; pushed_stream = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **st) { *g = pushed_grid; *b = pushed_block; *lds = pushed_lds; *st = pushed_stream; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *st) {
  const char *name = "?";
  for (int i = 0; i < count; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  fprintf(out, "%s %u %u %u %u %zu\n", name, g.x, g.y, g.z, b.x * b.y * b.z, lds);
  return 0;
}
int hipFuncSetAttribute(const void *f, int a, int v) { if (fail_attributes) last_error = 1; return fail_attributes; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
int hipPeekAtLastError(void) { return last_error; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)4096; return 0; }
int hipEventCreate(void **e) { return 0; }
int hipEventDestroy(void *e) { return 0; }
int hipEventElapsedTime(float *t, void *a, void *b) { return 0; }
int hipEventRecord(void *e, void *s) { return 0; }
int hipEventSynchronize(void *e) { return 0; }
"""

CALLS = r"""
import ctypes, json, sys
stand_in = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # in the place of libamdhip64, by its name
lib = ctypes.CDLL(sys.argv[2])
job = json.load(open(sys.argv[3]))
stand_in.stand_in_setup(sys.argv[4].encode(), job["fail_attributes"])
lib.wersa_workspace_bytes.restype = lib.wersa_block_workspace_bytes.restype = ctypes.c_size_t
one = ctypes.c_void_p(1 << 20)   # never dereferenced
for what, desc in job["calls"]:
    d = ctypes.create_string_buffer(bytes.fromhex(desc))
    entry = getattr(lib, "wersa_" + what)
    pointers = {"forward": 10, "backward": 18, "block_forward": 12, "block_backward": 20}[what]
    size = (lib.wersa_block_workspace_bytes if what.startswith("block") else lib.wersa_workspace_bytes)(d, int(what.endswith("backward")))
    stand_in.stand_in_call(entry(d, *[one] * (pointers + 1), ctypes.c_size_t(size), None))
"""


def launches(calls, lib=None, fail_attributes=False):
    """calls: (what, descriptor) with what "forward", "backward", "block_forward" or "block_backward"; of each (status, HIP's error that is left,
    [(kernel, grid, threads of a workgroup, bytes of dynamic LDS)]).  fail_attributes: hipFuncSetAttribute fails."""
    from paper_2507_08637_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    with tempfile.TemporaryDirectory(prefix="wersa_launches_") as tmp:
        path = lambda name: os.path.join(tmp, name)
        with open(path("hip.c"), "w") as f:
            f.write(STAND_IN)
        with open(path("hip.map"), "w") as f:
            f.write("hip_4.2 { global: *; };")
        subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script," + path("hip.map"), path("hip.c"),
                        "-o", path("hip.so")], check=True)
        with open(path("job.json"), "w") as f:
            json.dump(dict(fail_attributes=int(fail_attributes), calls=[(what, bytes(d).hex()) for what, d in calls]), f)
        subprocess.run([sys.executable, "-c", CALLS, path("hip.so"), lib or binding.LIB_PATH, path("job.json"), path("out")], check=True)
        with open(path("out")) as f:
            lines = f.read().splitlines()
    results, kernels = [], []
    for line in lines:
        name, *numbers = line.split(" ")
        if name == "=":
            results.append((int(numbers[0]), int(numbers[1]), kernels))
            kernels = []
        else:
            x, y, z, threads, lds = (int(v) for v in numbers)
            kernels.append((plain(name), (x, y, z), threads, lds))
    return results


def plain(symbol):
    """rows_kernel<0,256,0,1,0,4>: a kernel's name and its template's numbers and truth values."""
    length, rest = re.match(r"_ZN5wersa12_GLOBAL__N_1(\d+)(\w+)", symbol).groups()
    name, args = rest[:int(length)], re.match(r"I\w*?((?:L[ib]\d+E)+)E", rest[int(length):])
    return name + ("<" + ",".join(re.findall(r"L[ib](\d+)E", args.group(1))) + ">" if args else "")
