"""The library's host layer (sfcgemm_api.cpp, sfc_model.cpp) compiled with g++ against
a stand-in for the HIP runtime that hands out memory addresses and prints every
allocation and launch: what a call would do on the device, checked without one.

``run(exe, lines)`` takes one command per line and returns its events, a list of
(name, {key: value}) per command:
  gemm <entry> M N K lda ldb ldc out ca tile ws stream    entry: ex, fused, noalloc, f8
  capture <stream> <0|1>                                  a capture begins or ends
  fail <n>                                                the n-th allocation from here fails
  notready <0|1>                                          events report unfinished work
Every command ends with a ``ret`` event that holds the return code.  Addresses are
numbers counted up from 2^40; ``ws`` is 1 for a caller's workspace, else 0."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = f"{ROOT}/paper_2601_16294_amd/csrc"

HIP = r'''
#pragma once
#include <stddef.h>
#include <stdint.h>
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&x)
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorNotReady = 600,
                  hipErrorStreamCaptureUnsupported = 900, hipErrorStreamCaptureIsolation = 905, hipErrorStreamCaptureImplicit = 906 };
typedef struct ihipStream_t* hipStream_t;
typedef struct ihipEvent_t* hipEvent_t;
enum { hipEventDisableTiming = 2, hipDeviceAttributeMultiprocessorCount = 1, hipMemcpyDeviceToHost = 2 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1,
                              hipStreamCaptureStatusInvalidated = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal = 0, hipStreamCaptureModeThreadLocal = 1,
                            hipStreamCaptureModeRelaxed = 2 };
extern "C" {
const char* hipGetErrorString(hipError_t);
hipError_t hipGetLastError();
hipError_t hipGetDevice(int*);
hipError_t hipDeviceGetAttribute(int*, int, int);
hipError_t hipEventQuery(hipEvent_t);
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned);
hipError_t hipEventRecord(hipEvent_t, hipStream_t);
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned);
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus*);
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*);
hipError_t hipFree(void*);
hipError_t hipFreeAsync(void*, hipStream_t);
hipError_t hipMemcpy(void*, const void*, size_t, int);
}
hipError_t hip_malloc(void** p, size_t n);
hipError_t hip_malloc_async(void** p, size_t n, hipStream_t s);
template <typename T> hipError_t hipMalloc(T** p, size_t n) { return hip_malloc((void**)p, n); }
template <typename T> hipError_t hipMallocAsync(T** p, size_t n, hipStream_t s) { return hip_malloc_async((void**)p, n, s); }
hipError_t hipGetSymbolAddress(void** p, const void*);
'''

MAIN = r'''
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>
#include <set>
#include "sfc_params.h"
#include "sfcgemm.h"
static uintptr_t next_addr = (uintptr_t)1 << 40;
static std::set<hipStream_t> capturing;
static hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
static int fail_in = 0, not_ready = 0;
static hipError_t take(const char* what, void** p, size_t n, hipStream_t s) {
  if (fail_in && --fail_in == 0) return hipErrorOutOfMemory;
  *p = (void*)next_addr;
  next_addr += (n + 4095) / 4096 * 4096;
  printf("%s p=%lu n=%zu stream=%lu\n", what, (unsigned long)(uintptr_t)*p, n, (unsigned long)(uintptr_t)s);
  return hipSuccess;
}
// a plain allocation is refused while any stream is captured, but in the relaxed mode
hipError_t hip_malloc(void** p, size_t n) {
  if (!capturing.empty() && mode != hipStreamCaptureModeRelaxed) return hipErrorStreamCaptureUnsupported;
  return take("malloc", p, n, 0);
}
hipError_t hip_malloc_async(void** p, size_t n, hipStream_t s) {
  return take(capturing.count(s) ? "malloc_in_graph" : "malloc_async", p, n, s);
}
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)((uintptr_t)1 << 39); return hipSuccess; }
extern "C" {
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) {
  if (!capturing.empty() && mode != hipStreamCaptureModeRelaxed) return hipErrorStreamCaptureUnsupported;
  return not_ready ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
  return capturing.count(s) ? hipErrorStreamCaptureIsolation : hipSuccess;   // an event from outside the capture
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return !s && !capturing.empty() ? hipErrorStreamCaptureImplicit : hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  const hipStreamCaptureMode old = mode;
  mode = *m;
  *m = old;
  return hipSuccess;
}
hipError_t hipFree(void* p) { printf("free p=%lu\n", (unsigned long)(uintptr_t)p); return hipSuccess; }
hipError_t hipFreeAsync(void* p, hipStream_t s) {
  printf("free p=%lu stream=%lu captured=%d\n", (unsigned long)(uintptr_t)p, (unsigned long)(uintptr_t)s, (int)capturing.count(s));
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, int) { return hipSuccess; }
}
namespace sfc {
static unsigned long u(const void* p) { return (unsigned long)(uintptr_t)p; }
hipError_t launch_sfc_order(int gm, int gn, int order, int32_t* d, hipStream_t) {
  printf("order gm=%d gn=%d d=%lu\n", gm, gn, u(d));
  return hipSuccess;
}
hipError_t launch_gemm(const Variant& v, const GemmParams& p, int grid, hipStream_t) {
  printf("gemm tile=%d bf16=%d loads=%d f8=%d deep=%d M=%ld N=%ld K=%ld layers=%d out=%lu counters=%lu grid=%d table=%lu\n", v.tile,
         (int)v.out_bf16, v.loads, v.f8, (int)v.deep, (long)p.M, (long)p.N, (long)p.K, p.layers, u(p.out), u(p.counters), grid, u(p.table));
  return hipSuccess;
}
hipError_t gemm_occupancy(const Variant& v, int* n) { *n = v.tile == kT128x128 && !v.deep ? 2 : 1; return hipSuccess; }
hipError_t launch_small(const SmallParams& p, int fm, bool ob, hipStream_t) {
  printf("small fm=%d bf16=%d M=%d N=%d K=%d layers=%d W=%lu counters=%lu\n", fm, (int)ob, p.M, p.N, p.K, p.layers, u(p.W),
         u(p.counters));
  return hipSuccess;
}
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t) {
  printf("fill p=%lu n=%ld\n", u(p), (long)n);
  return hipSuccess;
}
hipError_t launch_reduce(const float* W, int layers, int64_t, int64_t, void*, int64_t, bool, hipStream_t) {
  printf("reduce W=%lu layers=%d\n", u(W), layers);
  return hipSuccess;
}
hipError_t run_mfma_probe(int, int, float*, double*) { return hipErrorInvalidValue; }
}  // namespace sfc
int main() {
  char cmd[16], entry[16];
  while (scanf("%15s", cmd) == 1) {
    int rc = 0;
    if (!strcmp(cmd, "gemm")) {
      long M, N, K, lda, ldb, ldc;
      int out, ca, tile, ws;
      unsigned long stream;
      if (scanf("%15s %ld %ld %ld %ld %ld %ld %d %d %d %d %lu", entry, &M, &N, &K, &lda, &ldb, &ldc, &out, &ca, &tile, &ws,
                &stream) != 12) return 1;
      void *A = (void*)0x1000, *B = (void*)0x2000, *C = (void*)0x3000, *W = ws ? (void*)0x4000 : nullptr;
      const size_t wb = ws ? (size_t)1 << 50 : 0;
      void* s = (void*)stream;
      if (!strcmp(entry, "ex")) rc = sfc_gemm_ex(M, N, K, A, lda, B, ldb, C, ldc, out, ca, tile, 0, 0, W, wb, s);
      else if (!strcmp(entry, "fused")) rc = sfc_gemm_fused_ex(M, N, K, A, lda, B, ldb, C, ldc, out, ca, tile, 0, 0, W, wb, s);
      else if (!strcmp(entry, "noalloc")) rc = sfc_gemm_noalloc_ex(M, N, K, A, lda, B, ldb, C, ldc, out, ca, tile, 0, 0, s);
      else if (!strcmp(entry, "f8")) rc = sfc_gemm_f8_ex(M, N, K, A, lda, B, ldb, C, ldc, out, ca, tile, 0, 0, W, wb, s);
      else return 1;
    } else if (!strcmp(cmd, "capture")) {
      unsigned long stream; int on;
      if (scanf("%lu %d", &stream, &on) != 2) return 1;
      if (on) capturing.insert((hipStream_t)stream);
      else capturing.erase((hipStream_t)stream);
      if (mode != hipStreamCaptureModeGlobal) return 2;      // left as the library found it
    } else if (!strcmp(cmd, "notready")) {
      if (scanf("%d", &not_ready) != 1) return 1;
    } else if (!strcmp(cmd, "fail")) {
      if (scanf("%d", &fail_in) != 1) return 1;
    } else {
      return 1;
    }
    printf("ret rc=%d\n", rc);
  }
  return 0;
}
'''


def build(directory) -> str:
    """Compiles the stand-in and the host layer into `directory`; the program's path."""
    hip = os.path.join(directory, "hip")
    os.makedirs(hip, exist_ok=True)
    with open(os.path.join(hip, "hip_runtime.h"), "w") as f:
        f.write(HIP)
    main, exe = os.path.join(directory, "main.cpp"), os.path.join(directory, "host_api")
    with open(main, "w") as f:
        f.write(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", f"-I{directory}", f"-I{ROOT}/include", f"-I{CSRC}", main,
                    f"{CSRC}/sfcgemm_api.cpp", f"{CSRC}/sfc_model.cpp", "-o", exe], check=True)
    return exe


def run(exe, lines):
    out = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True).stdout
    calls, cur = [], []
    for line in out.splitlines():
        name, *kv = line.split()
        cur.append((name, {k: int(v) for k, v in (x.split("=") for x in kv)}))
        if name == "ret":
            calls.append(cur)
            cur = []
    return calls


def gemm(entry, M, N, K, out=0, ca=1, tile=0, ws=0, stream=1, lda=None, ldb=None, ldc=None) -> str:
    return (f"gemm {entry} {M} {N} {K} {K if lda is None else lda} {N if ldb is None else ldb} "
            f"{N if ldc is None else ldc} {out} {ca} {tile} {ws} {stream}")
