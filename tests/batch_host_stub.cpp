// A HIP runtime that records instead of running, for tests of rx_batch.cpp's host code on the CPU: device memory is
// host memory, and the kernel nodes of the last graph are kept for the test to read.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <vector>

#include "../include/rx.h"
#include "../paper_1901_07499_amd/csrc/rx_launch.h"

namespace {
struct Node {
  const void* func;
  unsigned grid, block, lds;
  std::vector<int> deps;
  const void* tiles;  // second argument (the tile map of estimate and demod kernels)
};
std::vector<Node> nodes;
int set_lds[64];          // last value of the maximum dynamic LDS of each kernel
char kernels[64];         // kernel "functions": &kernels[id]
int id_of(const void* f) { return (int)((const char*)f - kernels); }
enum { kReset = 0, kMergedDem = 1, kMergedEst = 5, kClassDem = 9, kClassEst = 30 };
int length_index(int N) { return __builtin_ctz(N) - 6; }
}  // namespace

namespace rx {
bool batch_kernels(int N, int, int waves, int jobs, int, int, BatchKernel& dem, BatchKernel& est) {
  const int tpw = waves * 1024 / N > 0 ? waves * 1024 / N : 1;
  dem = {kernels + kClassDem + length_index(N), 64 * waves, 36864, (size_t)tpw * 12 + 2, 0};
  est = {kernels + kClassEst + length_index(N), 256, 36864, 0, tpw * jobs};
  return true;
}
int fft_schedule_count(int N) { return N >= 512 ? 2 : 1; }
void fft_schedule_radices(int, int, int r[3]) { r[0] = r[1] = r[2] = 0; }
const void* batch_reset_func() { return kernels + kReset; }
bool batch_wide(int N, int U) { return 8 * U > 5 * N; }
BatchMerged batch_merged(bool wide, int waves) {
  BatchMerged m;
  const int v = (wide ? 1 : 0) + (waves == 8 ? 2 : 0);
  m.dem = kernels + kMergedDem + v;
  m.est = kernels + kMergedEst + v;
  m.dem_block = 64 * waves;
  m.est_block = 256;
  m.est_jobs = 2;

  for (int i = 0; i < 6; i++) {
    const int tpw = waves * 16 >> i > 0 ? waves * 16 >> i : 1;
    m.lds_fft[i] = m.est_lds[i] = 36864;
    m.lds_per_u[i] = (size_t)tpw * 12 + 2;
    m.est_ants[i] = 2 * tpw;
  }
  return m;
}
}  // namespace rx

extern "C" {
int rx_params_check(const rx_params*) { return RX_OK; }

int stub_nodes() { return (int)nodes.size(); }
void stub_node(int i, int64_t out[6]) {
  out[0] = id_of(nodes[i].func);
  out[1] = nodes[i].grid;
  out[2] = nodes[i].block;
  out[3] = nodes[i].lds;
  out[4] = (int64_t)nodes[i].tiles;
  out[5] = (int64_t)nodes[i].deps.size();
}
int stub_dep(int i, int k) { return nodes[i].deps[k]; }
int stub_lds(int kernel) { return set_lds[kernel]; }

hipError_t hipMalloc(void** p, size_t n) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) { set_lds[id_of(f)] = v; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// every class kernel takes the same time, the merged ones stub_set_merged_ms
float merged_ms = 1.f;
void stub_set_merged_ms(float ms) { merged_ms = ms; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  const int k = nodes.size() > 1 ? id_of(nodes[1].func) : kClassDem;
  *ms = k >= kMergedDem && k < kClassDem ? merged_ms : 1.f;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t* g, unsigned) {
  nodes.clear();
  *g = (hipGraph_t)&nodes;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)&nodes;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t* n, hipGraph_t, const hipGraphNode_t* deps, size_t n_deps,
                                 const hipKernelNodeParams* p) {
  Node x{p->func, p->gridDim.x, p->blockDim.x, p->sharedMemBytes, {}, *(const void* const*)p->kernelParams[1]};
  for (size_t i = 0; i < n_deps; i++) x.deps.push_back((int)(intptr_t)deps[i] - 1);
  nodes.push_back(x);
  *n = (hipGraphNode_t)(intptr_t)nodes.size();
  return hipSuccess;
}
}
