"""What the library would launch, without a GPU.

A small program defines the HIP entry points that libugbs.so imports, so the
library runs on the CPU up to its launches: every kernel is recorded with its
grid, block and dynamic LDS, and none is started (the pointers it is given are
not memory).  The static LDS of each kernel comes from the metadata of the
gfx950 objects built here.
"""
import functools
import json
import os
import re
import subprocess
import tempfile

import pytest

import paper_2607_07724_amd as ugbs
from paper_2607_07724_amd import build

LDS_BYTES = 160 * 1024          # per CU (and per workgroup) on gfx950
LDS_GRANULE = 1280              # allocated in units of 320 dwords

_SRC = r"""
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include "ugbs.h"
struct dim3 { uint32_t x, y, z; };
// (the library registers its kernels before this program's own globals exist)
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static dim3 g_grid, g_block;
static size_t g_smem;
static bool fail_attribute, first;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int st;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  names()[f] = d ? d : name;
  free(d);
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t smem, void*) { g_grid = g; g_block = b; g_smem = smem; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* smem, void** s) { *g = g_grid; *b = g_block; *smem = g_smem; *s = nullptr; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t smem, void*) {
  printf("%s{\"kernel\": \"%s\", \"grid\": %u, \"block\": %u, \"dynamic\": %zu}", first ? "" : ", ", names()[f].c_str(), g.x, b.x, smem);
  first = false;
  return 0;
}
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return fail_attribute ? 1 : 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x10000; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }
}
int main() {
  char fn[64];
  ugbs_problem p;
  memset(&p, 0, sizeof p);
  int extra, fail;
  char* m = (char*)0x100000;   // stands for every tensor; nothing reads it
  while (scanf("%63s %d %d %d %d %d %d %d %lf %d %d %d", fn, &p.batch, &p.n_heads, &p.n_kv_heads, &p.seq_len,
               &p.head_dim, &p.k_budget, &p.backbone, &p.q, &p.rho, &extra, &fail) == 12) {
    p.block = 64;
    fail_attribute = fail != 0;
    first = true;
    printf("{\"launches\": [");
    int st = -1;
    const size_t ws = ugbs_workspace_bytes(&p);
    if (!strcmp(fn, "attend")) st = ugbs_attend(&p, m, m, m, (int32_t*)m, extra, m, nullptr);
    else if (!strcmp(fn, "attend_select")) st = ugbs_attend_select(&p, m, m, m, nullptr, nullptr, m, ws, m, nullptr);
    else if (!strcmp(fn, "attend_bitmap")) st = ugbs_attend_bitmap(&p, m, m, m, (uint32_t*)m, m, nullptr);
    else if (!strcmp(fn, "bai_tiles")) st = ugbs_bai_tiles(&p, (float*)m, (float*)m, (float*)m, extra, (ugbs_bai_tile*)m, nullptr);
    else if (!strcmp(fn, "score_select")) st = ugbs_score_select(&p, m, m, nullptr, nullptr, (int32_t*)m, (float*)m, m, ws, nullptr);
    printf("], \"status\": %d}\n", st);
  }
}
"""


@functools.lru_cache(None)
def _program():
    where = tempfile.mkdtemp(prefix="ugbs_launches_")
    src, exe = os.path.join(where, "launches.cpp"), os.path.join(where, "launches")
    with open(src, "w") as f:
        f.write(_SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(build.ROOT, "include"), src, "-o", exe,
                    ugbs.library_path(), "-Wl,-rpath," + build.PKG, "-Wl,--allow-shlib-undefined"], check=True)
    return exe


def launches(calls):
    """calls: (function, problem, extra=0, fail_attribute=False) tuples; extra is
    kv_width (attend) or n_samples (bai_tiles).  One (status, launches) each."""
    text = ""
    for fn, p, *rest in calls:
        extra, fail = (list(rest) + [0, False][len(rest):])[:2]
        text += (f"{fn} {p.batch} {p.n_heads} {p.n_kv_heads} {p.seq_len} {p.head_dim} {p.k_budget} {p.backbone} "
                 f"{p.q!r} {p.rho} {extra} {int(fail)}\n")
    r = subprocess.run([_program()], input=text, check=True, capture_output=True, text=True)
    out = [json.loads(x) for x in r.stdout.splitlines()]
    assert len(out) == len(calls)
    for o in out:
        for x in o["launches"]:
            x["kernel"] = re.sub(r"^void |ugbs::|\(anonymous namespace\)::|\(ugbs::\w+.*\)$", "", x["kernel"])
            x["kernel"] = re.sub(r"\(.*\)$", "", x["kernel"])
    return [(o["status"], o["launches"]) for o in out]


@functools.lru_cache(None)
def static_lds():
    """Static LDS bytes of every kernel, by name without arguments."""
    res = {}
    for s in build.SOURCES:
        obj = os.path.join(build.BUILD, os.path.splitext(s)[0] + ".o")
        if not os.path.exists(obj):
            pytest.skip("objects not built here (run __graft_entry__.build())")
        notes = build.device_notes(obj)
        for k in re.split(r"\n  - ", notes)[1:]:
            name, lds = re.search(r"\.name:\s+(\S+)", k), re.search(r"\.group_segment_fixed_size:\s+(\d+)", k)
            if name and lds:
                d = subprocess.run(["c++filt", name.group(1)], check=True, capture_output=True, text=True).stdout.strip()
                d = re.sub(r"^void |ugbs::|\(anonymous namespace\)::", "", d)
                res[re.sub(r"\(.*\)$", "", d)] = int(lds.group(1))
    return res


def workgroups_per_cu(launch):
    """Workgroups of a launch that the LDS of one CU holds."""
    n = static_lds()[launch["kernel"]] + launch["dynamic"]
    return LDS_BYTES // max(1, -(-n // LDS_GRANULE) * LDS_GRANULE)
