"""Buffers that the runtime moves, so that they may lie in any memory it reaches: the residual stream that eagle3_tree_verify_layers is given may be in
another GPU's memory, which a kernel of this one cannot read, and the last feature of eagle3_prefill may go there.  The library runs here without a GPU, on a stand-in of the runtime that writes down
copies and launches; no address is dereferenced."""
import os
import subprocess

import pytest

import paper_2503_01840_amd as E

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HOST = r"""
#include <dlfcn.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>
#include "eagle3.h"
// ---- the runtime's entry points that the library calls; a program's own come before those of the libraries it opens
struct Dim { uint32_t x, y, z; };
static std::map<const void*, std::string> names;
static char* const X = (char*)0x7100000000;            // the caller's buffer
static struct { Dim g, b; size_t lds; void* st; } pushed;
static void launch(const void* f, void** args) {
  const std::string& name = names[f];
  bool given = false;
  if (name.find("begin_rows_kernel") != std::string::npos)       // its first argument is a block of at least eight words
    for (int i = 0; i < 8; ++i) given = given || ((char**)args[0])[i] == X;
  printf("launch %s%s\n", name.c_str(), given ? " with the caller's buffer" : "");
}
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[f] = name; }
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* st) { pushed = {g, b, lds, st}; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** st) { *g = pushed.g; *b = pushed.b; *lds = pushed.lds; *st = pushed.st; return 0; }
int hipLaunchKernel(const void* f, Dim, Dim, void** args, size_t, void*) { launch(f, args); return 0; }
int hipExtLaunchKernel(const void* f, Dim, Dim, void** args, size_t, void*, void*, void*, int) { launch(f, args); return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
  printf("copy %zu bytes from %s to %s\n", n, src == X ? "the caller's buffer" : "elsewhere", dst == X ? "the caller's buffer" : "elsewhere");
  return 0;
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
const char* hipGetErrorString(int) { return ""; }
}
#define NEED(call) do { const int rc = (call); if (rc) { printf("%s: %d\n", #call, rc); return 1; } } while (0)
int main(int, char** argv) {
  void* so = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (!so) { puts(dlerror()); return 1; }
#define GET(name) auto name = (decltype(&::name))dlsym(so, #name)
  GET(eagle3_create); GET(eagle3_workspace_bytes); GET(eagle3_set_workspace); GET(eagle3_set_weights); GET(eagle3_tree_verify_layers); GET(eagle3_prefill);
  const int L = 3, H = 512;
  eagle3_config c = {H, 4, 2, 128, 512, 1024, 512, L, {0, 0, 1}, atoi(argv[2]), 1e4f, 1e-5f, 20, 16, 2, 2, 4};
  eagle3_ctx* ctx;
  NEED(eagle3_create(&c, &ctx));
  size_t bytes;
  NEED(eagle3_workspace_bytes(ctx, &bytes));
  NEED(eagle3_set_workspace(ctx, (void*)0x7200000000, bytes));
  void* p = (void*)0x7000000000;                       // everything else, on this GPU
  const eagle3_layer_weights w = {p, p, p, p, p, p, p, p, p};
  const std::vector<eagle3_layer_weights> layers(L, w);
  const eagle3_target_weights t = {layers.data(), p, p, p};
  const eagle3_draft_weights d = {p, w, p, p, p, p, (int32_t*)p};
  NEED(eagle3_set_weights(ctx, &t, &d));
  void* caches[L] = {p, p, p};
  const eagle3_kv kv = {caches, caches, (int32_t*)p, (int32_t*)p, 40};
  auto number = [&](int i) { return atoi(argv[4 + i]); };
  if (*argv[3] == 's')
    NEED(eagle3_tree_verify_layers(ctx, number(0), number(1), (int32_t*)p, (int32_t*)p, &kv, (float*)X, number(2), number(3), (float*)p, nullptr, nullptr));
  else
    NEED(eagle3_prefill(ctx, (int32_t*)p, number(0), &kv, &kv, (float*)X, (float*)p, nullptr));
  return 0;
}
"""


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    """(dtype, call, its numbers) -> the copies and launches it makes"""
    if not os.path.exists(E.LIB_PATH):
        from paper_2503_01840_amd.build import build_library
        build_library()
    d = tmp_path_factory.mktemp("calls")
    (d / "m.cpp").write_text(HOST)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(d / "m.cpp"), "-o", str(d / "m"), "-ldl"], check=True)

    def run(*args):
        r = subprocess.run([str(d / "m"), E.LIB_PATH, *map(str, args)], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout.splitlines()
    return run


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("B,N,l0,l1", [(1, 1, 1, 2), (2, 15, 0, 1), (20, 16, 1, 3), (3, 5, 2, 2)])
def test_a_stage_reads_its_residual_stream_through_the_runtime(calls, dtype, B, N, l0, l1):
    lines = calls(dtype, "stage", B, N, l0, l1)
    moved = [i for i, line in enumerate(lines) if line.startswith("copy")]
    assert [lines[i] for i in moved] == [f"copy {B * N * 512 * 4} bytes from the caller's buffer to elsewhere"]
    begins = [i for i, line in enumerate(lines) if "begin_rows_kernel" in line]
    assert len(begins) == 1 and begins[0] > moved[0] and "caller" not in lines[begins[0]]


# one chunk and several (256 rows in fp32, 2048 in bf16)
@pytest.mark.parametrize("dtype,T", [(0, 1), (0, 77), (0, 513), (1, 1), (1, 77), (1, 300), (1, 4100)])
def test_the_last_feature_of_a_prompt_leaves_through_the_runtime(calls, dtype, T):
    lines = calls(dtype, "prompt", T)
    assert [line for line in lines if line.startswith("copy")] == [f"copy {512 * 4} bytes from elsewhere to the caller's buffer"]
