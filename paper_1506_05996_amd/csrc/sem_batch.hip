// Batched independent solves (many meshes, orders 2..15, one stream).
//
// Instances of the same order N are concatenated into one disjoint-union mesh:
// every operator, gather, patch and coarse kernel then covers all of them in
// one launch (work items = elements of all instances, in the union's Morton
// order; each component is its own tree of the coarse nested dissection, and
// nodes of all trees at one height share the coarse sweep launches).  The
// union's canonical numbering restricted to one instance is that instance's
// own numbering shifted by four offsets (vertices, edges, faces, interiors), so
// instance vectors map to union vectors by four contiguous copies.
//
// PCG (Algorithm 1) runs per instance: dot products are reduced per instance
// over fixed chunks in a fixed order (deterministic), alpha and beta are
// per-instance device scalars, and an instance stops updating the moment its
// own residual test passes, exactly where a single solve would stop.  The
// vector kernels take the chunks of all orders in one launch.  One whole
// batched iteration is captured once in a hipGraph and replayed; in it the
// orders' operators, and their preconditioners, are parallel branches: each is
// a chain of launches that leaves most of the chip idle.  16 instances of
// orders 3..8 and 2..20 hexahedra per side to 1e-10: 79 ms with the orders one
// after another and vector kernels per order over chunks of 16,384 nodes,
// 31.6 ms so; the launch rate of the graph's nodes (about 5 us each) bounds it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <memory>
#include <vector>

#include "sem_device.h"

namespace sem {

// per-instance scalar slots
enum : int {
  kRz = 0, kPw, kAlpha, kBeta, kRr, kBb, kActive, kIters, kTol2, kFlag, kNorm, kRestarts, kScal  // kScal = stride
};
// Nodes per reduction chunk, one workgroup each: 16 per lane (at 16,384 a
// middling mesh had 12-160 workgroups for 256 CUs, each with 64 dependent
// rounds of loads: 20-60 us a launch).
constexpr int64_t kChunk = 4096;
constexpr int kSeg = 256;  // lanes of the chunk kernels and of the per-instance sums

struct Chunk {
  int64_t begin, end;  // union index range in the group's vectors
  int64_t src;         // the range's first entry in the instance's own vectors
  int32_t inst;        // global instance index
  int32_t group;
};

// vectors of one group on the device: x, r, z, p, w, b (union-sized)
struct SegGroup {
  double* v64[6];
  float* v32[5];
  const uint8_t* dir;
};

template <typename T>
__device__ __forceinline__ T* seg_vec(const SegGroup& g, int i) {
  if constexpr (std::is_same<T, double>::value)
    return g.v64[i];
  else
    return g.v32[i];
}

// --- kernels ------------------------------------------------------------------
__device__ __forceinline__ double block_reduce(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) s += sh[q];
  return s;
}

// part[chunk] = sum over the chunk of v_ia * v_ib
template <typename T>
__global__ void __launch_bounds__(kSeg)
seg_dot_kernel(const SegGroup* __restrict__ groups, int ia, int ib, const Chunk* __restrict__ chunks,
               double* __restrict__ part) {
  __shared__ double sh[kSeg / 64];
  const Chunk c = chunks[blockIdx.x];
  const T* a = seg_vec<T>(groups[c.group], ia);
  const T* b = seg_vec<T>(groups[c.group], ib);
  double s = 0.0;
#pragma unroll 4
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) s += (double)a[q] * (double)b[q];
  s = block_reduce(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// an active instance stops: one fewer in the count (whole numbers, so the order does not matter)
__device__ __forceinline__ void seg_stop(double* S, double* nactive) {
  S[kActive] = 0.0;
  atomicAdd(nactive, -1.0);
}

// One workgroup per instance: s = sum of its chunks in a fixed order; then
//   mode 0: sc[dst] = s
//   mode 1: p^T w -> alpha (0 for stopped instances), breakdown flag
//   mode 2: z^T r -> beta, rz
//   mode 3: r^T r -> rr; an active instance that meets its tolerance stops;
//           active ones count the iteration
// nactive[0]: instances still active (set when a run starts, lowered as they stop)
__global__ void __launch_bounds__(kSeg)
seg_final_kernel(const double* __restrict__ part, const int32_t* __restrict__ inst_chunk_off,
                 double* __restrict__ sc, int dst, int mode, double* __restrict__ nactive) {
  __shared__ double sh[kSeg / 64];
  const int i = blockIdx.x;
  double s = 0.0;
  for (int32_t c = inst_chunk_off[i] + (int)threadIdx.x; c < inst_chunk_off[i + 1]; c += kSeg) s += part[c];
  s = block_reduce(s, sh);
  if (threadIdx.x != 0) return;
  double* S = sc + (int64_t)i * kScal;
  const bool act = S[kActive] != 0.0;
  if (mode == 0) {
    S[dst] = s;
  } else if (mode == 1) {
    S[kPw] = s;
    double a = 0.0;
    if (act) {
      a = S[kRz] / s;
      if (!(s > 0.0) || !isfinite(a)) {
        S[kFlag] = 1.0;
        seg_stop(S, nactive);
        a = 0.0;
      }
    }
    S[kAlpha] = a;
  } else if (mode == 2) {
    if (act) {
      const double b = s / S[kRz];
      if (!isfinite(b)) {
        S[kFlag] = 1.0;
        seg_stop(S, nactive);
      }
      S[kBeta] = b;
      S[kRz] = s;
    }
  } else if (mode == 3) {
    if (act) {
      S[kRr] = s;
      S[kIters] += 1.0;
      if (!isfinite(s)) {
        S[kFlag] = 1.0;
        seg_stop(S, nactive);
      } else if (s <= S[kTol2]) {
        seg_stop(S, nactive);
      }
    }
  }
}

// x += alpha p; r -= alpha w (active instances); partial sums of r^T r
template <typename T>
__global__ void __launch_bounds__(kSeg)
seg_update_xr_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks,
                     const double* __restrict__ sc, double* __restrict__ part) {
  __shared__ double sh[kSeg / 64];
  const Chunk c = chunks[blockIdx.x];
  const double* S = sc + (int64_t)c.inst * kScal;
  const SegGroup g = groups[c.group];
  T* __restrict__ x = seg_vec<T>(g, 0);
  T* __restrict__ r = seg_vec<T>(g, 1);
  const T* __restrict__ p = seg_vec<T>(g, 3);
  const T* __restrict__ w = seg_vec<T>(g, 4);
  const T al = (T)S[kAlpha];
  double s = 0.0;
  if (S[kActive] != 0.0) {
#pragma unroll 4
    for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) {
      x[q] += al * p[q];
      const T rn = r[q] - al * w[q];
      r[q] = rn;
      s += (double)rn * (double)rn;
    }
  }
  s = block_reduce(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;  // read for active instances alone
}

// p = z + beta p (active instances)
template <typename T>
__global__ void __launch_bounds__(kSeg)
seg_update_p_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks,
                    const double* __restrict__ sc) {
  const Chunk c = chunks[blockIdx.x];
  const double* S = sc + (int64_t)c.inst * kScal;
  if (S[kActive] == 0.0) return;
  T* __restrict__ p = seg_vec<T>(groups[c.group], 3);
  const T* __restrict__ z = seg_vec<T>(groups[c.group], 2);
  const T b = (T)S[kBeta];
#pragma unroll 4
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) p[q] = z[q] + b * p[q];
}

// p = z
template <typename T>
__global__ void __launch_bounds__(kSeg)
seg_start_p_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks) {
  const Chunk c = chunks[blockIdx.x];
  T* __restrict__ p = seg_vec<T>(groups[c.group], 3);
  const T* __restrict__ z = seg_vec<T>(groups[c.group], 2);
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) p[q] = z[q];
}

// the callers' right-hand sides into b and r (0 on the Dirichlet set: the
// values there do not take part), x = 0
__global__ void __launch_bounds__(kSeg)
seg_load_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks,
                const double* const* __restrict__ src) {
  const Chunk c = chunks[blockIdx.x];
  const SegGroup g = groups[c.group];
  const double* __restrict__ from = src[c.inst] + c.src;
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) {
    const double v = g.dir[q] ? 0.0 : from[q - c.begin];
    g.v64[5][q] = v;
    g.v64[1][q] = v;
    g.v64[0][q] = 0.0;
  }
}

// the solutions to the callers' vectors
__global__ void __launch_bounds__(kSeg)
seg_store_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks, double* const* __restrict__ dst) {
  const Chunk c = chunks[blockIdx.x];
  const double* __restrict__ x = groups[c.group].v64[0];
  double* __restrict__ to = dst[c.inst] + c.src;
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) to[q - c.begin] = x[q];
}

// start of an FP32 inner solve: r32 = r64 / ||r||, d = 0; instances that have
// stopped get a zero right-hand side (their inner solve is idle)
__global__ void __launch_bounds__(kSeg)
seg_scale_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks,
                 const double* __restrict__ sc) {
  const Chunk c = chunks[blockIdx.x];
  const SegGroup g = groups[c.group];
  const double* S = sc + (int64_t)c.inst * kScal;
  const double nrm = S[kNorm];
  const double f = (nrm > 0.0 && S[kActive] != 0.0) ? 1.0 / nrm : 0.0;
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) {
    g.v32[1][q] = (float)(g.v64[1][q] * f);
    g.v32[0][q] = 0.0f;
  }
}

// x64 += ||r||_inst * d32 for instances still refining
__global__ void __launch_bounds__(kSeg)
seg_correct_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks,
                   const double* __restrict__ sc_outer) {
  const Chunk c = chunks[blockIdx.x];
  const double* S = sc_outer + (int64_t)c.inst * kScal;
  if (S[kActive] == 0.0) return;
  const SegGroup g = groups[c.group];
  const double f = S[kNorm];
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) g.v64[0][q] += f * (double)g.v32[0][q];
}

// r = b - Ax (Ax in w) with partial sums of r^T r
__global__ void __launch_bounds__(kSeg)
seg_residual_kernel(const SegGroup* __restrict__ groups, const Chunk* __restrict__ chunks, double* __restrict__ part) {
  __shared__ double sh[kSeg / 64];
  const Chunk c = chunks[blockIdx.x];
  const SegGroup g = groups[c.group];
  double s = 0.0;
  for (int64_t q = c.begin + threadIdx.x; q < c.end; q += kSeg) {
    const double v = g.v64[5][q] - g.v64[4][q];
    g.v64[1][q] = v;
    s += v * v;
  }
  s = block_reduce(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// After a batched FP64 solve, rr holds each instance's true ||b - A x||^2:
// instances whose true residual is still above the tolerance become active
// again (PCG restarts from it), the others stay stopped; counts restarts.
__global__ void __launch_bounds__(64)
seg_restart_kernel(double* __restrict__ sc, int n, double* __restrict__ nactive) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double* S = sc + (int64_t)i * kScal;
    const double s = S[kRr];
    if (!isfinite(s)) S[kFlag] = 1.0;
    const bool act = S[kFlag] == 0.0 && S[kBb] > 0.0 && s > S[kTol2];
    S[kActive] = act ? 1.0 : 0.0;
    if (act) {
      S[kRestarts] += 1.0;
      atomicAdd(&cnt, 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) nactive[0] = (double)cnt;
}

// per-instance scalar initialisation of a PCG run from ||r||^2 in rr: active, tol2, counters
__global__ void __launch_bounds__(64)
seg_init_kernel(double* __restrict__ sc, int n, double rtol2, double* __restrict__ nactive) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double* S = sc + (int64_t)i * kScal;
    const double bb = S[kRr];
    S[kBb] = bb;
    S[kTol2] = rtol2 * bb;
    S[kIters] = 0.0;
    S[kRestarts] = 0.0;
    S[kFlag] = 0.0;
    const bool act = bb > 0.0 && isfinite(bb) && bb > S[kTol2];
    S[kActive] = act ? 1.0 : 0.0;
    if (act) atomicAdd(&cnt, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) nactive[0] = (double)cnt;
}

__global__ void seg_norm_kernel(double* __restrict__ sc, int n, int src_slot) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double* S = sc + (int64_t)i * kScal;
    S[kNorm] = sqrt(S[src_slot]);
  }
}

// --- host side ------------------------------------------------------------------
template <typename T>
struct Vecs {
  DBuf<T> v[6];
};

struct MeshDeleter {
  void operator()(sem_mesh_s* m) const { sem_mesh_destroy(m); }
};

struct Group {
  int N = 0;
  std::unique_ptr<sem_mesh_s, MeshDeleter> mesh;
  std::vector<int> inst;            // global instance indices, in concatenation order
  Vecs<double> f64;                 // x, r, z, p, w, b   (union-sized)
  Vecs<float> f32;                  // d, r, z, p, w
};

struct Run {  // one instance's run of union entries
  int inst, group;
  int64_t src, dst, len;
};

}  // namespace sem

using namespace sem;

struct sem_batch_s {
  int n = 0;
  std::vector<int64_t> ng;        // per instance
  std::vector<Group> groups;
  std::vector<Run> runs;
  std::vector<Chunk> chunks;      // ordered by instance
  std::vector<int32_t> inst_chunk_off;
  DBuf<Chunk> d_chunks;
  DBuf<int32_t> d_inst_chunk_off;
  DBuf<SegGroup> d_groups;
  DBuf<double*> d_ptr;            // the call's right-hand sides, then its solution vectors
  DBuf<double> part, sc, sc_outer, nactive;
  double** ptr_host = nullptr;    // pinned: staging of d_ptr
  double* active_host = nullptr;  // pinned: two read-backs of nactive
  hipEvent_t ev_active[2] = {nullptr, nullptr};
  hipStream_t cap = nullptr;
  std::vector<hipStream_t> branch;  // capture: one stream per order and phase (operator, preconditioner)
  std::vector<hipEvent_t> ev_branch;
  hipEvent_t ev_main[2] = {nullptr, nullptr};
  hipGraphExec_t it64 = nullptr, it32 = nullptr;
  int graph_pc = -1;
  ~sem_batch_s() {
    if (it64) (void)hipGraphExecDestroy(it64);
    if (it32) (void)hipGraphExecDestroy(it32);
    for (auto e : ev_branch) (void)hipEventDestroy(e);
    for (auto e : ev_active)
      if (e) (void)hipEventDestroy(e);
    for (auto e : ev_main)
      if (e) (void)hipEventDestroy(e);
    for (auto t : branch) (void)hipStreamDestroy(t);
    if (cap) (void)hipStreamDestroy(cap);
    if (ptr_host) (void)hipHostFree(ptr_host);
    if (active_host) (void)hipHostFree(active_host);
  }
};

namespace {

template <typename T>
Vecs<T>& vecs(Group& g) {
  if constexpr (std::is_same<T, double>::value)
    return g.f64;
  else
    return g.f32;
}

template <typename F, typename... A>
void seg_launch(sem_batch b, F kernel, hipStream_t s, A... args) {
  hipLaunchKernelGGL(kernel, dim3((unsigned)b->chunks.size()), dim3(kSeg), 0, s, (const SegGroup*)b->d_groups.p, args...);
  SEM_HIP(hipGetLastError());
}

// per instance v_ia . v_ib, then seg_final
template <typename T>
void seg_dot(sem_batch b, int ia, int ib, double* sc, int dst, int mode, hipStream_t s) {
  seg_launch(b, seg_dot_kernel<T>, s, ia, ib, (const Chunk*)b->d_chunks.p, b->part.p);
  hipLaunchKernelGGL(seg_final_kernel, dim3((unsigned)b->n), dim3(kSeg), 0, s, (const double*)b->part.p,
                     (const int32_t*)b->d_inst_chunk_off.p, sc, dst, mode, b->nactive.p);
  SEM_HIP(hipGetLastError());
}

void seg_final(sem_batch b, double* sc, int dst, int mode, hipStream_t s) {
  hipLaunchKernelGGL(seg_final_kernel, dim3((unsigned)b->n), dim3(kSeg), 0, s, (const double*)b->part.p,
                     (const int32_t*)b->d_inst_chunk_off.p, sc, dst, mode, b->nactive.p);
  SEM_HIP(hipGetLastError());
}

// f(group, stream) for every group: one after another on `s`, or, while `s` is
// being captured and there are several groups, as parallel branches of the
// graph.  Every branch stream is forked from the capturing stream once and
// joined into it once (hence streams of their own for each phase), and forks
// none itself.
template <typename F>
void for_groups(sem_batch b, hipStream_t s, int phase, F&& f) {
  const size_t G = b->groups.size();
  const bool fork = s == b->cap && G > 1;
  if (!fork) {
    for (auto& g : b->groups) f(g, s);
    return;
  }
  SEM_HIP(hipEventRecord(b->ev_main[phase], s));
  for (size_t g = 0; g < G; ++g) {
    hipStream_t t = b->branch[phase * G + g];
    SEM_HIP(hipStreamWaitEvent(t, b->ev_main[phase], 0));
    f(b->groups[g], t);
    SEM_HIP(hipEventRecord(b->ev_branch[phase * G + g], t));
  }
  for (size_t g = 0; g < G; ++g) SEM_HIP(hipStreamWaitEvent(s, b->ev_branch[phase * G + g], 0));
}

// one batched PCG iteration on vectors of type T (x, r, z, p, w = v[0..4])
template <typename T>
void batched_iteration(sem_batch b, int pc, hipStream_t s) {
  for_groups(b, s, 0, [&](Group& g, hipStream_t t) { apply_A<T>(g.mesh.get(), vecs<T>(g).v[3].p, vecs<T>(g).v[4].p, t); });
  seg_dot<T>(b, 3, 4, b->sc.p, 0, 1, s);
  seg_launch(b, seg_update_xr_kernel<T>, s, (const Chunk*)b->d_chunks.p, (const double*)b->sc.p, b->part.p);
  seg_final(b, b->sc.p, 0, 3, s);
  for_groups(b, s, 1, [&](Group& g, hipStream_t t) { precond<T>(g.mesh.get(), vecs<T>(g).v[1].p, vecs<T>(g).v[2].p, pc, t); });
  seg_dot<T>(b, 1, 2, b->sc.p, 0, 2, s);
  seg_launch(b, seg_update_p_kernel<T>, s, (const Chunk*)b->d_chunks.p, (const double*)b->sc.p);
}

template <typename T>
hipGraphExec_t capture_iteration(sem_batch b, int pc) {
  if (!b->cap) {
    SEM_HIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
    for (auto& e : b->ev_main) SEM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  }
  while (b->branch.size() < 2 * b->groups.size()) {
    hipStream_t t = nullptr;
    SEM_HIP(hipStreamCreateWithFlags(&t, hipStreamNonBlocking));
    b->branch.push_back(t);
    hipEvent_t e = nullptr;
    SEM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    b->ev_branch.push_back(e);
  }
  auto set_flags = [b](bool on) {
    for (auto& g : b->groups) {
      g.mesh->in_capture = on;
      g.mesh->one_stream = on && b->groups.size() > 1;  // the other orders' branches fill the chip
    }
  };
  set_flags(true);
  hipGraph_t graph = nullptr;
  SEM_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
  try {
    batched_iteration<T>(b, pc, b->cap);
  } catch (...) {
    (void)hipStreamEndCapture(b->cap, &graph);
    if (graph) (void)hipGraphDestroy(graph);
    set_flags(false);
    throw;
  }
  SEM_HIP(hipStreamEndCapture(b->cap, &graph));
  set_flags(false);
  hipGraphExec_t exec = nullptr;
  hipError_t err = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (err != hipSuccess) throw Error{SEM_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(err)};
  return exec;
}

double read_active(sem_batch b, hipStream_t s) {
  double v = 0.0;
  SEM_HIP(hipMemcpyAsync(&v, b->nactive.p, sizeof(double), hipMemcpyDeviceToHost, s));
  SEM_HIP(hipStreamSynchronize(s));
  return v;
}

// PCG on all instances: x, r given (r = rhs), returns the batched iterations
// performed.  restart: the scalars (tolerances, active flags, counters) come
// from seg_restart_kernel instead of a fresh start from ||r||.
// The count of active instances is read back one check late: the next
// iteration is enqueued before the host waits for it, so that the GPU works
// through the round trip; the one iteration that follows the last instance's
// stop changes nothing (every update is masked by its instance's flag).
template <typename T>
int batched_pcg(sem_batch b, double rtol, int max_iter, int pc, int check_every, hipStream_t s,
                bool restart = false) {
  if (!restart) {
    // per-instance ||r||^2 -> scalars, tolerance, active flags
    seg_dot<T>(b, 1, 1, b->sc.p, kRr, 0, s);
    hipLaunchKernelGGL(seg_init_kernel, dim3(1), dim3(64), 0, s, b->sc.p, b->n, rtol * rtol, b->nactive.p);
  }
  for (auto& g : b->groups) precond<T>(g.mesh.get(), vecs<T>(g).v[1].p, vecs<T>(g).v[2].p, pc, s);
  seg_launch(b, seg_start_p_kernel<T>, s, (const Chunk*)b->d_chunks.p);
  seg_dot<T>(b, 1, 2, b->sc.p, kRz, 0, s);
  hipGraphExec_t& exec = std::is_same<T, double>::value ? b->it64 : b->it32;
  if (!exec || b->graph_pc != pc) {
    if (b->it64) (void)hipGraphExecDestroy(b->it64);
    if (b->it32) (void)hipGraphExecDestroy(b->it32);
    b->it64 = b->it32 = nullptr;
    b->graph_pc = pc;
    exec = capture_iteration<T>(b, pc);
  }
  int k = 0, asked = 0, seen = 0;  // read-backs enqueued and looked at
  bool done = false;
  while (k < max_iter && !done) {
    SEM_HIP(hipGraphLaunch(exec, s));
    ++k;
    if (k % check_every == 0 && k < max_iter) {
      SEM_HIP(hipMemcpyAsync(b->active_host + (asked & 1), b->nactive.p, sizeof(double), hipMemcpyDeviceToHost, s));
      SEM_HIP(hipEventRecord(b->ev_active[asked & 1], s));
      ++asked;
    }
    if (asked - seen == 2 || (k == max_iter && asked > seen)) {
      SEM_HIP(hipEventSynchronize(b->ev_active[seen & 1]));
      done = b->active_host[seen & 1] == 0.0;
      ++seen;
    }
  }
  return done ? seen * check_every : k;
}

}  // namespace

extern "C" {

int sem_batch_setup(int n, const double* const* vtx, const int64_t* n_vtx, const int64_t* const* hex,
                    const int64_t* n_hex, const int* order, const sem_setup_opts* opts, sem_batch* out) {
  return guarded_call([&]() -> int {
    if (!out || n <= 0 || !vtx || !n_vtx || !hex || !n_hex || !order) throw Error{SEM_EINVAL, "batch arguments"};
    *out = nullptr;
    sem_setup_opts d;
    sem_default_setup_opts(&d);
    if (!opts) opts = &d;
    if (opts->host_only) throw Error{SEM_EUNSUPPORTED, "a batch needs a device"};
    auto B = std::make_unique<sem_batch_s>();
    B->n = n;
    B->ng.assign(n, 0);
    std::vector<int> orders;
    for (int i = 0; i < n; ++i) {
      if (order[i] < 2 || order[i] > 15) throw Error{SEM_EUNSUPPORTED, "order must be in 2..15"};
      if (!vtx[i] || !hex[i] || n_vtx[i] <= 0 || n_hex[i] <= 0) throw Error{SEM_EINVAL, "empty instance"};
      orders.push_back(order[i]);
    }
    std::sort(orders.begin(), orders.end());
    orders.erase(std::unique(orders.begin(), orders.end()), orders.end());
    for (int N : orders) {
      Group g;
      g.N = N;
      std::vector<double> V;
      std::vector<int64_t> H;
      for (int i = 0; i < n; ++i) {
        if (order[i] != N) continue;
        const int64_t voff = (int64_t)V.size() / 3;
        V.insert(V.end(), vtx[i], vtx[i] + 3 * n_vtx[i]);
        for (int64_t x = 0; x < 8 * n_hex[i]; ++x) {
          if (hex[i][x] < 0 || hex[i][x] >= n_vtx[i]) throw Error{SEM_EINVAL, "hexahedron vertex id out of range"};
          H.push_back(hex[i][x] + voff);
        }
        g.inst.push_back(i);
      }
      g.mesh.reset(create_mesh(V.data(), (int64_t)V.size() / 3, H.data(), (int64_t)H.size() / 8, N, opts));
      B->groups.push_back(std::move(g));
    }
    // instance <-> union maps: vertices, edges, faces, interiors
    for (size_t gi = 0; gi < B->groups.size(); ++gi) {
      Group& g = B->groups[gi];
      const HostTables& U = g.mesh->T;
      const int64_t m = g.N - 1;
      int64_t vo = 0, eo = 0, fo = 0, io = 0;
      for (int i : g.inst) {
        // the instance's own class sizes, from its referenced vertices and topology
        std::vector<char> used(n_vtx[i], 0);
        for (int64_t x = 0; x < 8 * n_hex[i]; ++x) used[hex[i][x]] = 1;
        int64_t Vi = 0;
        for (char c : used) Vi += c;
        // edges and faces of the instance = union entities of its elements
        std::vector<int64_t> eds, fcs;
        int64_t ebase = 0, fbase = 0;
        for (int j : g.inst) {
          if (j == i) break;
          ebase += n_hex[j];
        }
        (void)fbase;
        std::vector<char> eu, fu;
        int64_t nE = 0, nF = 0;
        {
          // count distinct edge / face ranks of this instance's elements in the union
          std::vector<int64_t> er, fr;
          for (int64_t e = ebase; e < ebase + n_hex[i]; ++e) {
            for (int cz = 0; cz < 3; ++cz)
              for (int cy = 0; cy < 3; ++cy)
                for (int cx = 0; cx < 3; ++cx) {
                  const int nb = (cx != 1) + (cy != 1) + (cz != 1);
                  if (nb != 2 && nb != 1) continue;
                  const int64_t gid = gid_of(U, e, cx == 2 ? g.N : (cx == 1 ? 1 : 0), cy == 2 ? g.N : (cy == 1 ? 1 : 0),
                                             cz == 2 ? g.N : (cz == 1 ? 1 : 0));
                  if (nb == 2)
                    er.push_back((gid - U.base_e) / m);
                  else
                    fr.push_back((gid - U.base_f) / (m * m));
                }
          }
          std::sort(er.begin(), er.end());
          er.erase(std::unique(er.begin(), er.end()), er.end());
          std::sort(fr.begin(), fr.end());
          fr.erase(std::unique(fr.begin(), fr.end()), fr.end());
          nE = (int64_t)er.size();
          nF = (int64_t)fr.size();
          if (nE && (er.front() != eo || er.back() != eo + nE - 1)) throw Error{SEM_EMESH, "batch edge map"};
          if (nF && (fr.front() != fo || fr.back() != fo + nF - 1)) throw Error{SEM_EMESH, "batch face map"};
        }
        const int64_t Ei = n_hex[i];
        const int64_t ng = Vi + nE * m + nF * m * m + Ei * m * m * m;
        B->ng[i] = ng;
        B->runs.push_back(Run{i, (int)gi, 0, vo, Vi});
        B->runs.push_back(Run{i, (int)gi, Vi, U.base_e + eo * m, nE * m});
        B->runs.push_back(Run{i, (int)gi, Vi + nE * m, U.base_f + fo * m * m, nF * m * m});
        B->runs.push_back(Run{i, (int)gi, Vi + nE * m + nF * m * m, U.base_i + io * m * m * m, Ei * m * m * m});
        vo += Vi;
        eo += nE;
        fo += nF;
        io += Ei;
      }
      if (vo != U.V || eo != U.n_edges || fo != U.n_faces || io != U.E) throw Error{SEM_EMESH, "batch maps"};
    }
    // reduction chunks, ordered by instance
    B->inst_chunk_off.assign(n + 1, 0);
    std::vector<std::vector<Chunk>> per(n);
    for (auto& r : B->runs)
      for (int64_t q = 0; q < r.len; q += kChunk)
        per[r.inst].push_back(Chunk{r.dst + q, r.dst + std::min(r.len, q + kChunk), r.src + q, r.inst, r.group});
    for (int i = 0; i < n; ++i) {
      for (auto& c : per[i]) B->chunks.push_back(c);
      B->inst_chunk_off[i + 1] = (int32_t)B->chunks.size();
    }
    SEM_HIP(hipSetDevice(opts->device));
    B->d_chunks.upload(B->chunks.data(), B->chunks.size());
    B->d_inst_chunk_off.upload(B->inst_chunk_off.data(), B->inst_chunk_off.size());
    std::vector<SegGroup> sg;
    for (auto& g : B->groups) {
      const int64_t ngu = g.mesh->T.n_global;
      for (auto& v : g.f64.v) v.alloc(ngu);
      if (opts->build_fp32)
        for (int q = 0; q < 5; ++q) g.f32.v[q].alloc(ngu);
      SegGroup d{};
      for (int q = 0; q < 6; ++q) d.v64[q] = g.f64.v[q].p;
      for (int q = 0; q < 5; ++q) d.v32[q] = g.f32.v[q].p;
      d.dir = g.mesh->dir.p;
      sg.push_back(d);
    }
    B->d_groups.upload(sg.data(), sg.size());
    B->d_ptr.alloc(2 * (size_t)n);
    SEM_HIP(hipHostMalloc((void**)&B->ptr_host, 2 * (size_t)n * sizeof(double*), hipHostMallocDefault));
    SEM_HIP(hipHostMalloc((void**)&B->active_host, 2 * sizeof(double), hipHostMallocDefault));
    for (auto& e : B->ev_active) SEM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    B->part.alloc(std::max<size_t>(1, B->chunks.size()));
    B->sc.alloc((size_t)n * kScal);
    B->sc_outer.alloc((size_t)n * kScal);
    B->nactive.alloc(1);
    *out = B.release();
    return SEM_OK;
  });
}

int sem_batch_destroy(sem_batch b) {
  if (!b) return SEM_OK;
  (void)hipDeviceSynchronize();
  delete b;
  return SEM_OK;
}

int sem_batch_sizes(sem_batch b, int64_t* n_global) {
  if (!b || !n_global) return SEM_EINVAL;
  for (int i = 0; i < b->n; ++i) n_global[i] = b->ng[i];
  return SEM_OK;
}

int sem_batch_solve(sem_batch b, const double* const* b_dev, double* const* x_dev, const sem_solve_opts* o,
                    sem_solve_stats* st, void* stream) {
  if (!b || !b_dev || !x_dev) return SEM_EINVAL;
  sem_solve_opts d;
  sem_default_solve_opts(&d);
  if (!o) o = &d;
  if (o->pc < 0 || o->pc > 3 || o->max_iter < 0 || !(o->rtol >= 0.0)) return SEM_EINVAL;
  for (int i = 0; i < b->n; ++i)
    if (!b_dev[i] || !x_dev[i]) return SEM_EINVAL;
  return guarded_call([&]() -> int {
    hipStream_t s = (hipStream_t)stream;
    auto t0 = std::chrono::steady_clock::now();
    const int check = std::max(1, o->check_every);
    const bool refined = o->mode == SEM_SOLVE_FP32_REFINED;
    if (refined && !b->groups.front().f32.v[0].p) throw Error{SEM_EUNSUPPORTED, "batch built without FP32 copies"};
    if (o->use_x0) throw Error{SEM_EUNSUPPORTED, "batched solves start from x = 0"};
    // b -> union slots 5 and 1 (zero on the Dirichlet set); x = 0
    for (int i = 0; i < b->n; ++i) {
      b->ptr_host[i] = const_cast<double*>(b_dev[i]);
      b->ptr_host[b->n + i] = x_dev[i];
    }
    SEM_HIP(hipMemcpyAsync(b->d_ptr.p, b->ptr_host, 2 * (size_t)b->n * sizeof(double*), hipMemcpyHostToDevice, s));
    seg_launch(b, seg_load_kernel, s, (const Chunk*)b->d_chunks.p, (const double* const*)b->d_ptr.p);
    // r = b - A x per instance, ||r||^2 by chunks
    auto true_residual = [&]() {
      for (auto& g : b->groups) apply_A<double>(g.mesh.get(), g.f64.v[0].p, g.f64.v[4].p, s);
      seg_launch(b, seg_residual_kernel, s, (const Chunk*)b->d_chunks.p, b->part.p);
    };
    std::vector<int> iters(b->n, 0), outer(b->n, 0);
    std::vector<double> host_sc((size_t)b->n * kScal), host_out((size_t)b->n * kScal);
    if (!refined) {
      int total = batched_pcg<double>(b, o->rtol, o->max_iter, o->pc, check, s);
      // the recursive residual can drift below the true one: b - A x per
      // instance, and PCG again from it for the instances still above their
      // tolerance (as the single solve does)
      for (;;) {
        true_residual();
        seg_final(b, b->sc.p, kRr, 0, s);
        hipLaunchKernelGGL(seg_restart_kernel, dim3(1), dim3(64), 0, s, b->sc.p, b->n, b->nactive.p);
        SEM_HIP(hipGetLastError());
        if (read_active(b, s) == 0.0 || total >= o->max_iter) break;
        total += batched_pcg<double>(b, o->rtol, o->max_iter - total, o->pc, check, s, true);
      }
      SEM_HIP(hipMemcpyAsync(host_sc.data(), b->sc.p, host_sc.size() * sizeof(double), hipMemcpyDeviceToHost, s));
      SEM_HIP(hipStreamSynchronize(s));
      for (int i = 0; i < b->n; ++i) {
        iters[i] = (int)host_sc[(size_t)i * kScal + kIters];
        outer[i] = (int)host_sc[(size_t)i * kScal + kRestarts];
      }
    } else {
      // outer: r = b - A x in FP64 per instance; inner: FP32 batched PCG on r / ||r||
      for (int it = 0; it <= o->max_outer; ++it) {
        true_residual();
        if (it == 0) {
          // ||b||^2 = ||r||^2 at x = 0: sets each instance's tolerance
          seg_final(b, b->sc_outer.p, kRr, 0, s);
          hipLaunchKernelGGL(seg_init_kernel, dim3(1), dim3(64), 0, s, b->sc_outer.p, b->n, o->rtol * o->rtol,
                             b->nactive.p);
        } else {
          // refreshed residuals: stop the instances that meet their tolerance
          seg_final(b, b->sc_outer.p, 0, 3, s);
        }
        SEM_HIP(hipMemcpyAsync(host_out.data(), b->sc_outer.p, host_out.size() * sizeof(double),
                               hipMemcpyDeviceToHost, s));
        SEM_HIP(hipStreamSynchronize(s));
        bool any = false;
        for (int i = 0; i < b->n; ++i) any |= host_out[(size_t)i * kScal + kActive] != 0.0;
        if (!any || it == o->max_outer) break;
        for (int i = 0; i < b->n; ++i)
          if (host_out[(size_t)i * kScal + kActive] != 0.0) outer[i]++;
        hipLaunchKernelGGL(seg_norm_kernel, dim3(1), dim3(64), 0, s, b->sc_outer.p, b->n, (int)kRr);
        seg_launch(b, seg_scale_kernel, s, (const Chunk*)b->d_chunks.p, (const double*)b->sc_outer.p);
        batched_pcg<float>(b, o->inner_rtol, o->max_iter, o->pc, check, s);
        SEM_HIP(hipMemcpyAsync(host_sc.data(), b->sc.p, host_sc.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        SEM_HIP(hipStreamSynchronize(s));
        for (int i = 0; i < b->n; ++i)
          if (host_out[(size_t)i * kScal + kActive] != 0.0) iters[i] += (int)host_sc[(size_t)i * kScal + kIters];
        seg_launch(b, seg_correct_kernel, s, (const Chunk*)b->d_chunks.p, (const double*)b->sc_outer.p);
      }
      host_sc = host_out;
    }
    seg_launch(b, seg_store_kernel, s, (const Chunk*)b->d_chunks.p, (double* const*)(b->d_ptr.p + b->n));
    SEM_HIP(hipStreamSynchronize(s));
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    int status = SEM_OK;
    for (int i = 0; i < b->n; ++i) {
      const double* S = &host_sc[(size_t)i * kScal];
      const double rel = S[kBb] > 0.0 ? std::sqrt(S[kRr] / S[kBb]) : 0.0;
      const bool flag = S[kFlag] != 0.0;
      const bool conv = S[kBb] == 0.0 || S[kRr] <= S[kTol2];
      if (st) {
        st[i].iterations = iters[i];
        st[i].outer_iterations = outer[i];
        st[i].rel_residual = rel;
        st[i].solve_ms = ms;
        st[i].history_len = 0;
      }
      if (flag)
        status = SEM_EBREAKDOWN;
      else if (!conv && status == SEM_OK)
        status = SEM_ENOCONV;
    }
    if (status == SEM_EBREAKDOWN) set_error("PCG breakdown in a batched instance");
    if (status == SEM_ENOCONV) set_error("a batched instance did not reach its tolerance");
    return status;
  });
}

}  // extern "C"
