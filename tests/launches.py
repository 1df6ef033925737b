"""What the built library launches for a call, on the CPU.

A child process (this file run as a script) loads a small C library that defines the HIP
functions libxshare.so calls, ahead of the HIP runtime, then the library itself: its host code
runs as it is, and every launch is recorded by kernel name and grid instead of reaching a GPU.
``kernels`` reads the register, spill and LDS figures of the kernels from the built library.
"""
import json
import os
import re
import struct
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2602_07265_amd", "libxshare.so")
CUS = 256

RECORDER = r"""
#include <stddef.h>
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void* fn; const char* name; int per_cu; } reg[512];
static int n_reg;
static char text[1 << 16];
static size_t used;
static dim3 g_grid, g_block;
static size_t g_shared;
static void* g_stream;
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned lim,
                           void* t, void* b, void* bd, void* gd, int* w) {
  (void)m; (void)dev; (void)lim; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  if (n_reg < 512) { reg[n_reg].fn = fn; reg[n_reg].name = name; reg[n_reg++].per_cu = 0; }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) {
  g_grid = g; g_block = b; g_shared = s; g_stream = st; return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) {
  *g = g_grid; *b = g_block; *s = g_shared; *st = g_stream; return 0;
}
int hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t shared, void* st) {
  (void)args; (void)shared; (void)st;
  for (int i = 0; i < n_reg; ++i)
    if (reg[i].fn == fn && used + 512 < sizeof(text))
      used += (size_t)snprintf(text + used, sizeof(text) - used, "%s %u %u %u %u\n", reg[i].name,
                               g.x, g.y, g.z, b.x);
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* fn, int b, size_t s) {
  (void)b; (void)s;
  *n = 0;
  for (int i = 0; i < n_reg; ++i) if (reg[i].fn == fn) *n = reg[i].per_cu;
  return *n ? 0 : 1;
}
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = CUS; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipStreamGetDevice(void* s, int* d) { (void)s; *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)(1 << 20); return 0; }
void recorder_blocks(const char* name, int per_cu) {
  for (int i = 0; i < n_reg; ++i) if (!strcmp(reg[i].name, name)) reg[i].per_cu = per_cu;
}
void recorder_clear(void) { used = 0; text[0] = 0; }
const char* recorder_text(void) { return text; }
"""


def short_names(mangled):
    """Demangled names without namespaces and arguments, for instance down_kernel<2, 0, 4>."""
    out = subprocess.run(["c++filt"], input="\n".join(mangled), capture_output=True, text=True,
                         check=True).stdout.split("\n")
    return [re.sub(r"^void |xs::|\(anonymous namespace\)::|\([^()]*\)$", "", n) for n in out]


def kernels(lib=LIB):
    """{mangled name: metadata} of the gfx950 kernels in the built library."""
    import yaml
    data, found, pos = open(lib, "rb").read(), {}, 0
    while (pos := data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)) >= 0:
        count, at = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + n]
            at += 24 + n
            if b"gfx950" not in target or size == 0:
                continue
            with tempfile.NamedTemporaryFile() as f:
                f.write(data[pos + off:pos + off + size])
                f.flush()
                notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", f.name],
                                       capture_output=True, text=True, check=True).stdout
            meta = notes[notes.index("---"):]
            for k in yaml.safe_load(meta[:meta.rindex("...")])["amdhsa.kernels"]:
                found[k[".name"]] = k
        pos += 24
    return found


def blocks_per_cu(k):
    """Blocks of a kernel that a CU holds: its registers (512 a SIMD lane, eight waves at most)
    and 160 KB of LDS."""
    waves = k[".max_flat_workgroup_size"] // 64
    per_simd = min(8, 512 // ((max(k[".vgpr_count"], 1) + 7) // 8 * 8))
    lds = k[".group_segment_fixed_size"]
    return max(1, min(per_simd * 4 // waves, (160 << 10) // lds if lds else 8))


def launches(cases, lib=LIB):
    """For each case the launches of one call: [(kernel, (x, y, z), threads)].

    A case is a dict: T, N, k, d, f, M and, where they differ from the defaults of ``call``,
    op (route | forward | layer), fmt, mode, score, k0, tau, reqs, m_r, groups, local, shared."""
    meta = kernels(lib)
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "recorder.so")
        subprocess.run(["gcc", f"-DCUS={CUS}", "-shared", "-fPIC", "-O1", "-x", "c", "-", "-o", so],
                       input=RECORDER, text=True, check=True)
        request = dict(so=so, lib=lib, cases=cases,
                       blocks={n: blocks_per_cu(k) for n, k in meta.items()})
        res = subprocess.run([sys.executable, os.path.abspath(__file__)], text=True, check=True,
                             input=json.dumps(request), stdout=subprocess.PIPE)
    names = list(meta)
    short = dict(zip(names, short_names(names)))
    return [[(short[n], tuple(g), t) for n, g, t in one] for one in json.loads(res.stdout)]


def call(X, L, c):
    """One layer or selection call with pointers that nothing dereferences."""
    import ctypes
    fake = ctypes.c_void_p(1 << 20)
    mode = c.get("mode", "per_group" if c.get("groups") else "total")
    p = X.RouteParams(c["N"], c["k"], c.get("k0", 1), c["M"], X.BUDGET[mode],
                      X.SCORE[c.get("score", "topk")], c.get("m_r", 0), c.get("tau", 0.0), None)
    big = 1 << 44
    if c.get("op") == "route":
        if c.get("reqs"):
            return L.xshare_select_hier(fake, c["T"], fake, None, c["reqs"], ctypes.byref(p), fake,
                                        fake, fake, fake, fake, big, None)
        return L.xshare_route(fake, c["T"], ctypes.byref(p), fake, fake, fake, fake, fake, big, None)
    a = X.LayerArgs()
    a.struct_size = ctypes.sizeof(a)
    a.T, a.d, a.f = c["T"], c["d"], c["f"]
    a.weight_format = X.WEIGHTS[c.get("fmt", "bf16")]
    for field in ("x", "w1", "w3", "w2", "w1_scale", "w3_scale", "w2_scale", "y", "ws"):
        setattr(a, field, fake)
    if c.get("op") == "layer":
        a.w_gate = fake
    else:
        a.logits = fake
    a.params = ctypes.pointer(p)
    if c.get("reqs"):
        a.req_offsets, a.R = fake, c["reqs"]
    if c.get("groups"):
        a.ep = ctypes.pointer(X.EpLayout(c["groups"], c.get("local", -1), None, None))
    if c.get("shared"):
        a.shared = ctypes.pointer(X.SharedExperts(c["shared"], fake, fake, fake))
    a.ws_bytes = big
    return L.xshare_moe_forward_v2(ctypes.byref(a))


def _child():
    import ctypes
    import types
    request = json.load(sys.stdin)
    rec = ctypes.CDLL(request["so"], mode=ctypes.RTLD_GLOBAL)   # ahead of the HIP runtime
    rec.recorder_text.restype = ctypes.c_char_p
    sys.modules["torch"] = types.ModuleType("torch")            # the binding's types only
    sys.path.insert(0, os.path.join(ROOT, "paper_2602_07265_amd"))
    import xshare as X
    X.LIB_PATH = request["lib"]
    L = X.lib()
    for name, n in request["blocks"].items():
        rec.recorder_blocks(name.encode(), n)
    out = []
    for c in request["cases"]:
        rec.recorder_clear()
        status = call(X, L, c)
        if status != 0:
            raise RuntimeError(f"status {status} for {c}")
        rows = [r.split() for r in rec.recorder_text().decode().splitlines()]
        out.append([(r[0], [int(v) for v in r[1:4]], int(r[4])) for r in rows])
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child()
