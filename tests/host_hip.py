"""Runs calls of libppll.so on the CPU against a stand-in for the HIP runtime, and gives what the library asked of it, in order: kernel
launches with their grids, event records and waits, copies, queries.  Nothing is computed; device addresses are never read."""
import os
import subprocess

from host_cpp import ROOT
from paper_2411_12780_amd import binding as P

LIB = os.path.join(ROOT, "paper_2411_12780_amd", "libppll.so")

# The program defines the runtime's entry points itself, so that the library it loads binds to these.
SOURCE = r"""
#include <dlfcn.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <string>
#include <vector>
struct dim3 { uint32_t x, y, z; };
static std::map<const void*, std::string> kernels;
static bool logging = false;
static long events = 0;
#define SAY(...) do { if (logging) std::printf(__VA_ARGS__); } while (0)
static dim3 grid_, block_; static size_t lds_; static void* stream_;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) { grid_ = g; block_ = b; lds_ = lds; stream_ = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) { *g = grid_; *b = block_; *lds = lds_; *s = stream_; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, void* s) {
  SAY("launch %ld %u %u %u %u %zu %s\n", (long)(intptr_t)s, g.x, g.y, g.z, b.x, lds, kernels[f].c_str());
  return 0;
}
int hipGetDevice(int* d) { *d = 0; SAY("device\n"); return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)(intptr_t)(1L << 42); return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "?"; }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t n, int, void* s) { SAY("copy %ld %zu\n", (long)(intptr_t)s, n); return 0; }
int hipEventCreate(void** e) { *e = (void*)(intptr_t)++events; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)(intptr_t)++events; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) { *t = 0; return 0; }
int hipEventRecord(void* e, void* s) { SAY("record %ld %ld\n", (long)(intptr_t)s, (long)(intptr_t)e); return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)(intptr_t)99; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned) { SAY("wait %ld %ld\n", (long)(intptr_t)s, (long)(intptr_t)e); return 0; }
}
static void* lib;
template <class R = int, class... A> static R call(const char* name, A... a) {
  auto f = (R (*)(A...))dlsym(lib, name);
  if (!f) { std::fprintf(stderr, "%s is not there\n", name); std::exit(3); }
  return f(a...);
}
static void ok(int status, const char* what) {
  if (status) { std::fprintf(stderr, "%s: %s\n", what, call<const char*>("ppll_last_error")); std::exit(4); }
}
static std::vector<char> bytes(const std::string& hex) {
  std::vector<char> v;
  for (size_t i = 0; i + 1 < hex.size(); i += 2) v.push_back((char)std::stoi(hex.substr(i, 2), nullptr, 16));
  return v;
}
int main(int, char** argv) {
  lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (!lib) { std::fprintf(stderr, "%s\n", dlerror()); return 2; }
  int n;
  std::string hex;
  std::cin >> n;
  std::vector<char> cfgs;                       // n configurations, one behind the other
  for (int j = 0; j < n; ++j) { std::cin >> hex; const auto v = bytes(hex); cfgs.insert(cfgs.end(), v.begin(), v.end()); }
  const size_t one = cfgs.size() / n;
  void* const ws = (void*)(intptr_t)(1L << 40);
  void* const x = (void*)(intptr_t)(1L << 38);
  void* const out = (void*)(intptr_t)(3L << 38);
  void* const y = (void*)(intptr_t)(1L << 37);
  void *pipe = nullptr, *block = nullptr;
  size_t need = 0;
  if (n > 1) {
    std::vector<void*> streams;
    for (int j = 0; j < n; ++j) streams.push_back((void*)(intptr_t)(j + 1));
    std::vector<std::vector<float>> zero;
    std::vector<const float*> params;
    for (int j = 0; j < n; ++j) { size_t b; ok(call("ppll_block_param_bytes", (void*)(cfgs.data() + j * one), &b), "size"); zero.emplace_back(b / 4); }
    for (auto& z : zero) params.push_back(z.data());
    ok(call("ppll_pipeline_workspace_bytes", (void*)cfgs.data(), n, 2, &need), "size");
    ok(call("ppll_pipeline_init", (void*)cfgs.data(), n, 2, ws, need, (void*)streams.data(), (void*)params.data(), &pipe), "init");
    ok(call("ppll_pipeline_block", pipe, n - 1, &block), "block");
  } else {
    size_t b;
    ok(call("ppll_block_param_bytes", (void*)cfgs.data(), &b), "size");
    std::vector<float> zero(b / 4);
    ok(call("ppll_block_workspace_bytes", (void*)cfgs.data(), &need), "size");
    ok(call("ppll_block_init", (void*)cfgs.data(), ws, need, (void*)zero.data(), (void*)nullptr, &block), "init");
  }
  std::string what;
  while (std::cin >> what) {
    std::printf("== %s\n", what.c_str());
    logging = true;
    if (what == "batch") ok(call("ppll_pipeline_step", pipe, x, y, 0.1f, (void*)nullptr), "batch");
    else if (what == "step") ok(call("ppll_block_step", block, x, y, 0.1f, out, (void*)nullptr, (void*)nullptr), "step");
    else if (what == "eval") ok(call("ppll_block_forward_eval", block, x, out, (void*)((char*)out + (1L << 36)), (void*)nullptr), "eval");
    else if (what == "eval_noalloc") ok(call("ppll_block_forward_eval_noalloc", block, x, out, (void*)((char*)out + (1L << 36)), (void*)nullptr), "eval");
    else return 5;
    logging = false;
  }
}
"""


def compile_runtime(directory):
    src, exe = os.path.join(directory, "runtime.cpp"), os.path.join(directory, "runtime")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", src, "-o", exe, "-ldl"], check=True)
    return exe


def calls(exe, workloads, *what):
    """What the runtime was asked by each call of `what`: "step", "eval", "eval_noalloc" of the (last) block, "batch" of the pipeline that
    several workloads make.  Records are tuples: ("launch", stream, grid, threads, lds, kernel), ("record", stream, event), ("copy", stream,
    bytes), ("wait", stream, event), ("device",)."""
    text = "%d\n%s\n%s\n" % (len(workloads), "\n".join(bytes(P.make_config(wl)).hex() for wl in workloads), "\n".join(what))
    r = subprocess.run([exe, LIB], input=text, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    out = []
    for line in r.stdout.splitlines():
        f = line.split()
        if f[0] == "==":
            out.append([])
        elif f[0] == "launch":
            out[-1].append(("launch", int(f[1]), tuple(map(int, f[2:5])), int(f[5]), int(f[6]), f[7]))
        else:
            out[-1].append((f[0], *map(int, f[1:])))
    return out
