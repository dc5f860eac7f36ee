// Device state, kernel launches and the C ABI of the spectral-element solver.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>
#include <mutex>
#include <vector>

#include "sem_device.h"
#include "sem_internal.h"
#include "sem_kernels.h"

namespace sem {

static thread_local std::string g_last_error;
void set_error(const std::string& msg) { g_last_error = msg; }

}  // namespace sem

using namespace sem;

namespace sem {

constexpr int kGS = 256;

inline int64_t blocks_for(int64_t n, int t = kGS) { return std::max<int64_t>(1, (n + t - 1) / t); }
// grid of the grid-stride streaming kernels: up to 65,536 workgroups (more
// loads in flight than the 8,192 a stream of n_global doubles would need to
// cover the chip once: the p/x update streams at 5.2 TB/s instead of 4.5)
inline int grid_stride_blocks(int64_t n) { return (int)std::min<int64_t>(blocks_for(n), 65536); }

// every pointer 16-byte aligned (the streaming kernels then move two entries per access)
template <typename... P>
bool aligned16(const P*... ptrs) {
  return ((reinterpret_cast<uintptr_t>(ptrs) % 16 == 0) && ...);
}

template <typename T>
const T* Gp(sem_mesh m);
template <>
const double* Gp<double>(sem_mesh m) { return m->G64.p; }
template <>
const float* Gp<float>(sem_mesh m) { return m->G32.p; }
template <typename T>
const T* Dp(sem_mesh m);
template <>
const double* Dp<double>(sem_mesh m) { return m->D64.p; }
template <typename T>
const T* X8p(sem_mesh m);
template <>
const double* X8p<double>(sem_mesh m) { return m->X864.p; }
template <>
const float* X8p<float>(sem_mesh m) { return m->X832.p; }
template <typename T>
const T* TQp(sem_mesh m);
template <>
const double* TQp<double>(sem_mesh m) { return m->tq64.p; }
template <>
const float* TQp<float>(sem_mesh m) { return m->tq32.p; }
template <>
const float* Dp<float>(sem_mesh m) { return m->D32.p; }
template <typename T>
T* Wp(sem_mesh m);
template <>
double* Wp<double>(sem_mesh m) { return m->w64.p; }
template <>
float* Wp<float>(sem_mesh m) { return m->w32.p; }
template <typename T>
T* ZOp(sem_mesh m);
template <>
double* ZOp<double>(sem_mesh m) { return m->zo64.p; }
template <>
float* ZOp<float>(sem_mesh m) { return m->zo32.p; }
template <typename T>
const T* Sp(sem_mesh m);
template <>
const double* Sp<double>(sem_mesh m) { return m->S64.p; }
template <>
const float* Sp<float>(sem_mesh m) { return m->S32.p; }
template <typename T>
const T* Lp(sem_mesh m);
template <>
const double* Lp<double>(sem_mesh m) { return m->lam64.p; }
template <>
const float* Lp<float>(sem_mesh m) { return m->lam32.p; }
template <typename T>
const T* Hp(sem_mesh m);
template <>
const double* Hp<double>(sem_mesh m) { return m->h64.p; }
template <>
const float* Hp<float>(sem_mesh m) { return m->h32.p; }
template <typename T>
const T* KEp(sem_mesh m);
template <>
const double* KEp<double>(sem_mesh m) { return m->ke64.p; }
template <>
const float* KEp<float>(sem_mesh m) { return m->ke32.p; }
template <typename T>
const T* CEp(sem_mesh m);
template <>
const double* CEp<double>(sem_mesh m) { return m->ce64.p; }
template <>
const float* CEp<float>(sem_mesh m) { return m->ce32.p; }

// --- operator ---------------------------------------------------------------
// tile candidates: elements per workgroup, workgroups of at most 1024 lanes;
// kTileMfma selects the matrix-core kernel (N = 15), kTileGeo the kernel
// that rebuilds the geometric factors from the vertices
constexpr int kTileCandidates[4] = {1, 2, 4, 8};
constexpr int kTileMfma = 16;
constexpr int kTileGeo = 32;  // factors rebuilt from the vertices, default elements per workgroup
// the line-phase kernel: factors rebuilt from the vertices, or stored
constexpr int kTileLineGeo = 64;
constexpr int kTileLineStored = 48;

bool tile_code_ok(int epb, int N) {
  if (epb == 1 || epb == 2 || epb == 4 || epb == 8) return epb * (N + 1) * (N + 1) <= 1024;
  return epb == kTileGeo || epb == kTileLineGeo || epb == kTileLineStored || (epb == kTileMfma && N == 15);
}

template <int N>
constexpr bool tile_ok(int epb) {
  return epb * (N + 1) * (N + 1) <= 1024;
}

// coefficients of the operator for dtype T (kappa = 1, c = 0 unless set)
template <typename T>
OpCoef<T> op_coef(sem_mesh m) {
  OpCoef<T> oc{T(1), T(0), nullptr, 0, nullptr, nullptr, nullptr, nullptr};
  if (m->per_node) {  // kappa per node is inside the stored G (kn: for the rebuilt G); c m per local node
    if constexpr (std::is_same<T, double>::value) {
      oc.ke = m->nk64.p;
      oc.ce = m->nc64.p;
      oc.mL = m->nm64.p;
      oc.kn = m->kn64.p;
    } else {
      oc.ke = m->nk32.p;
      oc.ce = m->nc32.p;
      oc.mL = m->nm32.p;
      oc.kn = m->kn32.p;
    }
    if (oc.ke == nullptr || oc.ce == nullptr || oc.kn == nullptr || (m->any_ce && oc.mL == nullptr))
      throw Error{SEM_EINVAL, "per-node coefficients not on the device"};
    return oc;
  }
  if (m->per_elem) {  // per-element coefficients: applied by the element kernels
    if constexpr (std::is_same<T, double>::value) {
      oc.ke = m->ke64.p;
      oc.ce = m->ce64.p;
      oc.mL = m->mL64.p;
    } else {
      oc.ke = m->ke32.p;
      oc.ce = m->ce32.p;
      oc.mL = m->mL32.p;
    }
    if (oc.ke == nullptr || oc.ce == nullptr || (m->any_ce && oc.mL == nullptr))
      throw Error{SEM_EINVAL, "per-element coefficients not on the device"};
    return oc;
  }
  oc.kap = (T)m->T.kappa;
  oc.cm = (T)m->T.cmass;
  oc.scaled = (m->T.kappa != 1.0 || m->T.cmass != 0.0) ? 1 : 0;
  if constexpr (std::is_same<T, double>::value)
    oc.mN = m->mN64.p;
  else
    oc.mN = m->mN32.p;
  if (m->T.cmass != 0.0 && oc.mN == nullptr) throw Error{SEM_EINVAL, "lumped mass not on the device"};
  return oc;
}

// element kernel launches; with dpart, each workgroup also leaves its share of
// u^T A u in dpart[block], over all local nodes, so that the shares' sum is the whole
// scalar product (the grid size is returned so the caller knows how many)
template <int N, typename T, int EPB, bool GEO = false, bool KN = false>
int64_t launch_ax_tile(sem_mesh m, const T* u, T* y, double* dpart, hipStream_t s) {
  if constexpr (tile_ok<N>(EPB)) {
    const HostTables& T_ = m->T;
    const int64_t grid = xcd_grid((T_.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((ax_kernel<N, T, EPB, GEO, KN>), dim3((unsigned)grid), dim3(EPB * (N + 1) * (N + 1)), 0, s, u,
                       y, Wp<T>(m), GEO ? X8p<T>(m) : Gp<T>(m), m->rec.p, Dp<T>(m), m->dir.p, m->order.p, T_.E, dpart,
                       TQp<T>(m), op_coef<T>(m));
    SEM_HIP(hipGetLastError());
    return grid;
  } else {
    throw Error{SEM_EINVAL, "operator tile too large for the order"};
  }
}

template <int N, typename T, bool GEO, bool KN = false>
int64_t launch_ax_line(sem_mesh m, const T* u, T* y, double* dpart, hipStream_t s) {
  constexpr int EPB = line_epb<N, GEO>();
  const HostTables& T_ = m->T;
  const int64_t grid = xcd_grid((T_.E + EPB - 1) / EPB);
  hipLaunchKernelGGL((ax_line_kernel<N, T, EPB, GEO, KN>), dim3((unsigned)grid), dim3(EPB * (N + 1) * (N + 1)), 0, s,
                     u, y, Wp<T>(m), GEO ? X8p<T>(m) : Gp<T>(m), m->rec.p, Dp<T>(m), m->dir.p, m->order.p, T_.E, dpart,
                     TQp<T>(m), op_coef<T>(m));
  SEM_HIP(hipGetLastError());
  return grid;
}

template <int N, typename T>
int64_t launch_ax(sem_mesh m, const T* u, T* y, double* dpart, hipStream_t s) {
  const int epb = m->epb[std::is_same<T, double>::value ? 0 : 1];
  if (epb == kTileMfma) {
    if constexpr (N == 15) {
      const HostTables& T_ = m->T;
      const int64_t grid = xcd_grid(T_.E);
      hipLaunchKernelGGL((ax_mfma15_kernel<T>), dim3((unsigned)grid), dim3(256), 0, s, u, y, Wp<T>(m), Gp<T>(m),
                         m->rec.p, Dp<T>(m), m->dir.p, m->order.p, T_.E, dpart, op_coef<T>(m));
      SEM_HIP(hipGetLastError());
      return grid;
    } else {
      throw Error{SEM_EINVAL, "the matrix-core operator exists at N = 15"};
    }
  }
  if (epb == kTileGeo) {
    // per-node kappa: read per node by its own instance of the kernel
    if (m->per_node) return launch_ax_tile<N, T, ax_epb<N>(), true, true>(m, u, y, dpart, s);
    return launch_ax_tile<N, T, ax_epb<N>(), true>(m, u, y, dpart, s);
  }
  if (epb == kTileLineGeo) {
    if (m->per_node) return launch_ax_line<N, T, true, true>(m, u, y, dpart, s);
    return launch_ax_line<N, T, true>(m, u, y, dpart, s);
  }
  if (epb == kTileLineStored) return launch_ax_line<N, T, false>(m, u, y, dpart, s);
  switch (epb) {
    case 1: return launch_ax_tile<N, T, 1>(m, u, y, dpart, s);
    case 2: return launch_ax_tile<N, T, 2>(m, u, y, dpart, s);
    case 4: return launch_ax_tile<N, T, 4>(m, u, y, dpart, s);
    case 8: return launch_ax_tile<N, T, 8>(m, u, y, dpart, s);
    default: throw Error{SEM_EINVAL, "operator tile"};
  }
}

// the largest compiled packing (kTileCandidates) of at most ax_epb elements
template <int N>
constexpr int packed_tile() {
  return ax_epb<N>() >= 4 ? 4 : ax_epb<N>() >= 2 ? 2 : 1;
}

int default_tile(int N) {
  switch (N) {
#define CASE(NN) \
  case NN:       \
    return packed_tile<NN>();
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
  }
  return 1;
}

SharedNodes shared_nodes(sem_mesh m) {
  const HostTables& T = m->T;
  return SharedNodes{m->vinc_off.p, m->einc_off.p, m->fcount.p, m->dir.p,     T.V,
                     T.base_f,      T.base_i,      T.N - 1,     T.wedge_off, T.wvert_off};
}

// the coefficients as the shared nodes need them (those per element are in the copies already)
template <typename T>
OpCoef<T> shared_coef(sem_mesh m) {
  if (m->per_elem) return OpCoef<T>{T(1), T(0), nullptr, 0, nullptr, nullptr, nullptr, nullptr};
  return op_coef<T>(m);
}

// the shared-node gather; as the operator's last step (u_op = the operator's
// input) it also applies the coefficients, as the preconditioner's it only sums
template <typename T>
void launch_gs(sem_mesh m, T* y, hipStream_t s, const T* u_op = nullptr) {
  OpCoef<T> oc{T(1), T(0), nullptr, 0, nullptr, nullptr, nullptr, nullptr};
  if (u_op != nullptr) oc = shared_coef<T>(m);
  hipLaunchKernelGGL((gs_kernel<T>), dim3((unsigned)blocks_for(m->T.base_i)), dim3(kGS), 0, s, y, Wp<T>(m),
                     shared_nodes(m), oc, u_op);
  SEM_HIP(hipGetLastError());
}

// element kernel only (the gather follows separately); returns the grid size
template <typename T>
int64_t apply_A_elements(sem_mesh m, const T* u, T* y, hipStream_t s, double* dpart = nullptr) {
  switch (m->T.N) {
#define CASE(NN) \
  case NN:       \
    return launch_ax<NN, T>(m, u, y, dpart, s);
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
    default:
      throw Error{SEM_EUNSUPPORTED, "order not compiled"};
  }
}

template <typename T>
void apply_A(sem_mesh m, const T* u, T* y, hipStream_t s) {
  apply_A_elements<T>(m, u, y, s);
  launch_gs<T>(m, y, s, u);
}

// n partial sums into the scalars (see pcg_scalar): one launch up to kOneSum,
// through kRedBlocks chunk sums beyond
void reduce_partials(sem_mesh m, const double* part, int64_t n, int dst, int mode, hipStream_t s, int rz_in = 0,
                     int rz_out = 0, double* host = nullptr) {
  if (n > kOneSum) {
    const int64_t chunk = (n + kRedBlocks - 1) / kRedBlocks;
    const int nb = (int)((n + chunk - 1) / chunk);
    hipLaunchKernelGGL(sum_chunks_kernel, dim3(nb), dim3(kRedThreads), 0, s, part, m->wk.part, n, chunk);
    part = m->wk.part;
    n = nb;
  }
  hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(kFinalThreads), 0, s, part, m->wk.sc, (int)n, dst, mode, rz_in,
                     rz_out, host);
  SEM_HIP(hipGetLastError());
}

// Up to so many partial sums the kernel that needs the scalar sums them itself,
// in every workgroup, instead of a launch of its own in between (about 5 us):
// a handful of loads per lane, and few enough workgroups.
constexpr int64_t kConsumerSum = 512;

// --- fine and coarse preconditioner -----------------------------------------
template <int N>
int64_t fdm_grid(sem_mesh m) { return xcd_grid((m->T.E + fdm_ppb<N>() - 1) / fdm_ppb<N>()); }

template <int N, typename T>
void launch_fdm(sem_mesh m, const T* r, hipStream_t s, double* epart) {
  T* zc = ZOp<T>(m);
  T* zx = zc + m->T.E * (int64_t)m->T.n1 * m->T.n1 * m->T.n1;
  hipLaunchKernelGGL((fdm_kernel<N, T>), dim3((unsigned)fdm_grid<N>(m)), dim3(fdm_threads<N>()), 0, s, r, zc, zx,
                     m->pidx.p, m->pdst.p, Sp<T>(m), Lp<T>(m), Hp<T>(m), m->order.p, m->T.E,
                     (T)m->T.kappa, (T)m->T.cmass, m->per_elem ? KEp<T>(m) : nullptr,
                     m->per_elem ? CEp<T>(m) : nullptr, epart);
  SEM_HIP(hipGetLastError());
}

// element-wise sum of the corrections (+ coarse interpolation), interiors as
// MODE says (z: the result, or p), shared nodes to the work array
template <int N, typename T, int MODE>
void launch_schwarz_sum(sem_mesh m, T* z, T* x, bool fine, const double* Zv, hipStream_t s, int rz_in, int rz_out,
                        const double* bpart, int nb) {
  constexpr int EPB = sum_epb<N>();
  const T* zc = ZOp<T>(m);
  const T* zx = zc + m->T.E * (int64_t)m->T.n1 * m->T.n1 * m->T.n1;
  hipLaunchKernelGGL((schwarz_sum_kernel<N, T, EPB, MODE>), dim3((unsigned)xcd_grid((m->T.E + EPB - 1) / EPB)),
                     dim3(EPB * (N + 1) * (N + 1)), 0, s, z, x, Wp<T>(m), zc, zx, m->rec.p, m->dir.p, m->order.p,
                     m->T.E, (int)fine, Zv, m->phi.p, m->wk.sc, rz_in, rz_out, bpart, nb);
  SEM_HIP(hipGetLastError());
}

template <typename T, int MODE>
void schwarz_sum(sem_mesh m, T* z, T* x, bool fine, const double* Zv, hipStream_t s, int rz_in = 0, int rz_out = 0,
                 const double* bpart = nullptr, int nb = 0) {
  switch (m->T.N) {
#define CASE(NN) \
  case NN:       \
    return launch_schwarz_sum<NN, T, MODE>(m, z, x, fine, Zv, s, rz_in, rz_out, bpart, nb);
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
    default:
      throw Error{SEM_EUNSUPPORTED, "order not compiled"};
  }
}

// the element parts of the coarse residual of r (cvec: into the contribution
// vector); UPDATE: first r -= alpha A p at the interiors, with r . r.  Returns the
// number of partial sums of r . r
template <int N, typename T, bool UPDATE>
int64_t launch_restrict(sem_mesh m, T* r, const T* y, bool coarse, hipStream_t s) {
  constexpr int EPB = line_epb<N>();
  const int64_t grid = xcd_grid((m->T.E + EPB - 1) / EPB);
  hipLaunchKernelGGL((restrict_kernel<N, T, EPB, UPDATE>), dim3((unsigned)grid), dim3(EPB * (N + 1) * (N + 1)), 0, s,
                     r, y, (const double*)m->wk.sc, coarse ? m->cvec.p : nullptr, m->part_dst.p, m->wk.rpart, m->rec.p,
                     (const double*)m->phi.p, m->order.p, m->T.E);
  SEM_HIP(hipGetLastError());
  return grid;
}

template <typename T, bool UPDATE>
int64_t launch_restrict(sem_mesh m, T* r, const T* y, bool coarse, hipStream_t s) {
  switch (m->T.N) {
#define CASE(NN) \
  case NN:       \
    return launch_restrict<NN, T, UPDATE>(m, r, y, coarse, s);
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
    default:
      throw Error{SEM_EUNSUPPORTED, "order not compiled"};
  }
}

// the patch solves; with epart, also the partial sums of their share of r . z
template <typename T>
void launch_fdm(sem_mesh m, const T* r, hipStream_t s, double* epart = nullptr) {
  switch (m->T.N) {
#define CASE(NN) \
  case NN:       \
    return launch_fdm<NN, T>(m, r, s, epart);
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
    default:
      throw Error{SEM_EUNSUPPORTED, "order not compiled"};
  }
}

// workgroups of the patch solves (their partial sums)
int64_t fdm_blocks(sem_mesh m) {
  switch (m->T.N) {
#define CASE(NN) \
  case NN:       \
    return fdm_grid<NN>(m);
    CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    CASE(15)
#undef CASE
    default:
      throw Error{SEM_EUNSUPPORTED, "order not compiled"};
  }
}

// one launch of the forward or backward sweep
template <int RW, bool NARROW>
void launch_coarse_tiles(sem_mesh m, hipStream_t s, const CoarseLaunch& L, bool forward, double* epart) {
  const CoarseTile* tiles = m->tiles.p + L.first;
  if (forward) {
    const int n_pre = L.first == 0 ? (int)m->T.pre_row.size() : 0;  // the lowest launch sums the higher rows' parts
    hipLaunchKernelGGL((coarse_fwd_kernel<RW, NARROW>), dim3((unsigned)(L.count + (n_pre + 255) / 256)), dim3(256), 0,
                       s, m->Xlev.p, m->Zv.p, m->cvec.p, (const double*)m->fwd_pool.p, tiles,
                       (const int32_t*)m->rs_off.p, (const int32_t*)m->cdst.p, (const int32_t*)m->cvert.p,
                       (int)L.count, (const int32_t*)m->pre_slot.p, (const int32_t*)m->pre_row.p, n_pre,
                       epart != nullptr ? epart + L.first : nullptr);
  } else {
    hipLaunchKernelGGL((coarse_bwd_kernel<RW, NARROW>), dim3((unsigned)L.count), dim3(256), 0, s, m->Xlev.p, m->Zv.p,
                       (const double*)m->bwd_pool.p, tiles, (const int32_t*)m->fb_idx.p, (const int32_t*)m->cvert.p);
  }
  SEM_HIP(hipGetLastError());
}

void launch_coarse(sem_mesh m, hipStream_t s, const CoarseLaunch& L, bool forward, double* epart = nullptr) {
  if (!L.wide) {
    switch (L.rw) {
      case 1: return launch_coarse_tiles<1, true>(m, s, L, forward, epart);
      case 2: return launch_coarse_tiles<2, true>(m, s, L, forward, epart);
      case 4: return launch_coarse_tiles<4, true>(m, s, L, forward, epart);
      default: return launch_coarse_tiles<8, true>(m, s, L, forward, epart);
    }
  }
  switch (L.rw) {
    case 1: return launch_coarse_tiles<1, false>(m, s, L, forward, epart);
    case 2: return launch_coarse_tiles<2, false>(m, s, L, forward, epart);
    default: return launch_coarse_tiles<4, false>(m, s, L, forward, epart);
  }
}

// element parts in the contribution vector -> Zv (vertex order; 0 on Dirichlet
// vertices since set-up): nested-dissection sweeps; with epart, the partial
// sums of R . Z (one per forward tile)
void coarse_sweeps(sem_mesh m, hipStream_t s, double* epart = nullptr) {
  for (const CoarseLaunch& L : m->T.fwd_launch) launch_coarse(m, s, L, true, epart);
  for (const CoarseLaunch& L : m->T.bwd_launch) launch_coarse(m, s, L, false);
}

void release_coarse_graph(sem_mesh m) {
  if (m->amg_graph) (void)hipGraphExecDestroy(m->amg_graph);
  m->amg_graph = nullptr;
}

// --- aggregation AMG (Section 4.1, "Algebraic multigrid") ------------------
constexpr double kAmgOmega = 2.0 / 3.0;  // damped Jacobi

// host hierarchy -> device (work vectors per level, Jacobi weights omega / a_ii)
void amg_setup(sem_mesh m) {
  const HostTables& T = m->T;
  m->amg.clear();
  if (T.nc == 0) return;
  AmgHierarchy H;
  build_amg(T, H);
  for (const AmgLevel& L : H.levels) {
    auto d = std::make_unique<sem_mesh_s::AmgDev>();
    d->n = L.n;
    d->off.upload(L.off.data(), L.off.size());
    d->col.upload(L.col.data(), L.col.size());
    d->val.upload(L.val.data(), L.val.size());
    std::vector<double> wd(L.n);
    for (int64_t i = 0; i < L.n; ++i) wd[i] = kAmgOmega / L.diag[i];
    d->wd.upload(wd.data(), wd.size());
    if (!L.agg.empty()) {
      d->agg.upload(L.agg.data(), L.agg.size());
      d->moff.upload(L.moff.data(), L.moff.size());
      d->mem.upload(L.mem.data(), L.mem.size());
    }
    for (DBuf<double>* b : {&d->B, &d->X, &d->R, &d->T, &d->V, &d->W, &d->B2, &d->V2, &d->W2}) b->alloc(L.n);
    m->amg.push_back(std::move(d));
  }
  m->amg_inv.upload(H.coarse_inv.data(), H.coarse_inv.size());
  m->amg_sc.alloc(5 * H.levels.size());
  m->amg_nd.upload(H.nd_of.data(), H.nd_of.size());
  std::vector<int32_t> pos(T.nc);
  for (size_t q = 0; q < H.nd_of.size(); ++q) pos[H.nd_of[q]] = (int32_t)q;
  m->amg_pos.upload(pos.data(), pos.size());
}

void amg_fcg2(sem_mesh m, int l, const double* b, double* x, hipStream_t s);

// one K-cycle on level l: x ~= A_l^{-1} b
void amg_kcycle(sem_mesh m, int l, const double* b, double* x, hipStream_t s) {
  const int L = (int)m->amg.size() - 1;
  auto& d = *m->amg[l];
  const int64_t n = d.n;
  const unsigned g = (unsigned)blocks_for(n);
  if (l == L) {
    hipLaunchKernelGGL(amg_gemv_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, x, m->amg_inv.p, b, n);
    SEM_HIP(hipGetLastError());
    return;
  }
  auto& c = *m->amg[l + 1];
  hipLaunchKernelGGL(amg_presmooth_kernel, dim3(g), dim3(kGS), 0, s, x, d.R.p, b, d.wd.p, d.off.p, d.col.p, d.val.p,
                     n);
  hipLaunchKernelGGL(amg_restrict_kernel, dim3((unsigned)blocks_for(c.n)), dim3(kGS), 0, s, c.B.p, d.R.p, d.moff.p,
                     d.mem.p, c.n);
  SEM_HIP(hipGetLastError());
  if (l + 1 == L)
    amg_kcycle(m, l + 1, c.B.p, c.X.p, s);
  else
    amg_fcg2(m, l + 1, c.B.p, c.X.p, s);
  hipLaunchKernelGGL(amg_prolong_kernel, dim3(g), dim3(kGS), 0, s, d.T.p, x, c.X.p, d.agg.p, n);
  hipLaunchKernelGGL(amg_post_kernel, dim3(g), dim3(kGS), 0, s, x, d.T.p, b, d.off.p, d.col.p, d.val.p, d.wd.p, n);
  SEM_HIP(hipGetLastError());
}

// two flexible-CG steps on level l preconditioned by the K-cycle of level l
void amg_fcg2(sem_mesh m, int l, const double* b, double* x, hipStream_t s) {
  auto& d = *m->amg[l];
  const int64_t n = d.n;
  const unsigned g = (unsigned)blocks_for(n);
  double* sc = m->amg_sc.p + 5 * l;
  amg_kcycle(m, l, b, d.V.p, s);
  hipLaunchKernelGGL(amg_spmv_kernel, dim3(g), dim3(kGS), 0, s, d.W.p, d.V.p, d.off.p, d.col.p, d.val.p, n);
  hipLaunchKernelGGL((amg_dots_kernel<2>), dim3(1), dim3(1024), 0, s, sc, 0, d.V.p, b, (const double*)d.W.p,
                     (const double*)nullptr, n);
  hipLaunchKernelGGL(amg_r2_kernel, dim3(g), dim3(kGS), 0, s, d.B2.p, b, d.W.p, sc, n);
  SEM_HIP(hipGetLastError());
  amg_kcycle(m, l, d.B2.p, d.V2.p, s);
  hipLaunchKernelGGL(amg_spmv_kernel, dim3(g), dim3(kGS), 0, s, d.W2.p, d.V2.p, d.off.p, d.col.p, d.val.p, n);
  hipLaunchKernelGGL((amg_dots_kernel<3>), dim3(1), dim3(1024), 0, s, sc, 2, d.V2.p, (const double*)d.W.p,
                     (const double*)d.W2.p, (const double*)d.B2.p, n);
  hipLaunchKernelGGL(amg_combine_kernel, dim3(g), dim3(kGS), 0, s, x, d.V.p, d.V2.p, sc, n);
  SEM_HIP(hipGetLastError());
}

// one K-cycle from the element parts in the contribution vector to level 0's solution
void amg_cycle(sem_mesh m, hipStream_t s) {
  auto& d0 = *m->amg[0];
  hipLaunchKernelGGL(amg_in_kernel, dim3((unsigned)blocks_for(d0.n)), dim3(kGS), 0, s, d0.B.p, m->cvec.p, m->rs_off.p,
                     m->pslot.p, m->cvert.p, m->vinc_off.p, m->amg_nd.p, d0.n);
  amg_kcycle(m, 0, d0.B.p, d0.X.p, s);
}

// Capture one K-cycle (some 200 small launches) once, on a private stream; the
// preconditioner replays it on the caller's stream, then forms the vertex values
// (and R . Z) with one more launch.  Built at set-up and whenever the coarse
// matrix or solver changes.  The exact solve needs none: it is a handful of
// launches.
void build_coarse_graph(sem_mesh m) {
  if (m->T.nc == 0 || m->coarse_solver != SEM_COARSE_AMG) return;
  if (m->amg.empty()) throw Error{SEM_EINVAL, "AMG hierarchy not built"};
  if (m->amg_graph) return;
  if (m->no_alloc) throw Error{SEM_EINVAL, "coarse-solve graph missing (it is built at set-up)"};
  if (!m->capture_stream) SEM_HIP(hipStreamCreateWithFlags(&m->capture_stream, hipStreamNonBlocking));
  hipGraph_t g = nullptr;
  SEM_HIP(hipStreamBeginCapture(m->capture_stream, hipStreamCaptureModeThreadLocal));
  try {
    amg_cycle(m, m->capture_stream);
  } catch (...) {
    (void)hipStreamEndCapture(m->capture_stream, &g);
    if (g) (void)hipGraphDestroy(g);
    throw;
  }
  SEM_HIP(hipStreamEndCapture(m->capture_stream, &g));
  hipError_t err = hipGraphInstantiate(&m->amg_graph, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (err != hipSuccess) {
    m->amg_graph = nullptr;
    throw Error{SEM_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(err)};
  }
}

// element parts in the contribution vector -> Zv (vertex order): the coarse
// solve P_0; with epart, also the partial sums of R . Z
void coarse_solve_tree(sem_mesh m, hipStream_t s, double* epart = nullptr) {
  if (m->coarse_solver != SEM_COARSE_AMG) return coarse_sweeps(m, s, epart);
  if (m->in_capture) {  // inside an enclosing capture: the kernels themselves
    amg_cycle(m, s);
  } else {
    build_coarse_graph(m);
    SEM_HIP(hipGraphLaunch(m->amg_graph, s));
  }
  auto& d0 = *m->amg[0];
  hipLaunchKernelGGL(amg_out_kernel, dim3((unsigned)blocks_for(m->T.V)), dim3(kGS), 0, s, m->Zv.p, d0.X.p, d0.B.p,
                     m->cidx.p, m->amg_pos.p, m->T.V, epart);
  SEM_HIP(hipGetLastError());
}

// number of the partial sums of R . Z
int64_t coarse_parts(sem_mesh m) {
  if (m->T.nc == 0) return 0;
  if (m->coarse_solver == SEM_COARSE_AMG) return blocks_for(m->T.V);
  int64_t n = 0;
  for (const CoarseLaunch& L : m->T.fwd_launch) n += L.count;
  return n;
}

// the second stream (and its fork/join events) that runs the coarse chain
// beside the patch solves; created at set-up
void ensure_side_stream(sem_mesh m) {
  if (m->side_stream) return;
  if (m->no_alloc) throw Error{SEM_EINVAL, "side stream missing (it is created at set-up)"};
  SEM_HIP(hipStreamCreateWithFlags(&m->side_stream, hipStreamNonBlocking));
  SEM_HIP(hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming));
  SEM_HIP(hipEventCreateWithFlags(&m->ev_join, hipEventDisableTiming));
}

// Whether the coarse solve runs on the second stream, beside the patch solves.
// The exact solve's few launches run before them on the caller's stream: the
// patch solves fill every CU, so that each height waited for their workgroups
// to end, and the hand-overs between the streams cost about 10 us each (beside /
// before, N = 7: preconditioner alone 24^3 177 / 170 us FP64 and 133 / 127 FP32, 40^3
// 797 / 779 and 623 / 605, 56^3 2221 / 2180 and 1718 / 1667; PCG 24^3 17.5 / 17.2 ms,
// 40^3 refined 60.8 / 59.3, 56^3 216 / 213 and refined 163 / 160).  At N = 9 the patch
// solves leave room and beside is the faster (30^3 559 / 585 us and 427 / 459, PCG
// 77.5 / 79.0 ms and 55.6 / 57.3); the one order is kept all the same.  Against the graph of
// one launch per height that ran beside them earlier the preconditioner alone at 56^3
// takes 2180 / 2187 us FP64 and 1667 / 1651 FP32, the latter 1% slower.  A K-cycle of some
// 200 small launches is worth hiding.
bool coarse_beside(sem_mesh m) { return !m->one_stream && m->coarse_solver == SEM_COARSE_AMG; }

// what follows on s runs beside the coarse chain on the returned stream
hipStream_t fork_coarse(sem_mesh m, hipStream_t s) {
  if (!coarse_beside(m)) return s;
  ensure_side_stream(m);
  SEM_HIP(hipEventRecord(m->ev_fork, s));
  SEM_HIP(hipStreamWaitEvent(m->side_stream, m->ev_fork, 0));
  return m->side_stream;
}

// z = P r (assembled); the coarse and fine parts are independent until the final sum
template <typename T>
void precond(sem_mesh m, const T* r, T* z, int pc, hipStream_t s) {
  const HostTables& H = m->T;
  const bool fine = pc & SEM_PC_FINE, coarse = (pc & SEM_PC_COARSE) && H.nc > 0;
  if (pc == SEM_PC_NONE) {
    hipLaunchKernelGGL((copy_kernel<T, T>), dim3(grid_stride_blocks(H.n_global)), dim3(kGS), 0, s, z, r, H.n_global);
    SEM_HIP(hipGetLastError());
    return;
  }
  hipStream_t sc = s;
  if (coarse) {
    if (fine) sc = fork_coarse(m, s);
    launch_restrict<T, false>(m, const_cast<T*>(r), (const T*)nullptr, true, sc);  // r only read
    coarse_solve_tree(m, sc);
    if (sc != s) SEM_HIP(hipEventRecord(m->ev_join, sc));
  }
  if (fine) launch_fdm<T>(m, r, s);
  if (sc != s) SEM_HIP(hipStreamWaitEvent(s, m->ev_join, 0));
  schwarz_sum<T, kSumZ>(m, z, nullptr, fine, coarse ? (const double*)m->Zv.p : nullptr, s);
  launch_gs<T>(m, z, s);
}

// --- the steps of a PCG iteration -----------------------------------------------
// alpha = rz / (p . A p) and r -= alpha A p; returns the number of partial sums of r . r
template <typename T>
int64_t pcg_update_r(sem_mesh m, T* r, const T* p, T* y, int rz, bool coarse, hipStream_t s) {
  int64_t na = apply_A_elements<T>(m, p, y, s, m->wk.dpart);
  if (na > kConsumerSum) {
    reduce_partials(m, m->wk.dpart, na, 1, 1, s, rz);
    na = 0;
  }
  hipLaunchKernelGGL((gs_r_kernel<T>), dim3((unsigned)blocks_for(m->T.base_i)), dim3(kGS), 0, s, r, Wp<T>(m),
                     shared_nodes(m), shared_coef<T>(m), p, m->wk.sc, rz, (const double*)m->wk.dpart, (int)na);
  SEM_HIP(hipGetLastError());
  return launch_restrict<T, true>(m, r, y, coarse, s);
}

// the coarse solve of the element parts in the contribution vector, its partial
// sums of r . z after those of the patch solves
void pcg_start_coarse(sem_mesh m, bool fine, hipStream_t s) {
  hipStream_t sc = fine ? fork_coarse(m, s) : s;
  coarse_solve_tree(m, sc, m->wk.epart + (fine ? fdm_blocks(m) : 0));
  if (sc != s) SEM_HIP(hipEventRecord(m->ev_join, sc));
}

// the rest of an iteration: the patch solves, beta = (r . z) / rz, and x += alpha p,
// p = z + beta p (start: p = z and rz alone)
template <typename T>
void pcg_finish(sem_mesh m, const T* r, T* x, T* p, bool fine, bool coarse, int rz_in, int rz_out, bool start,
                hipStream_t s) {
  if (fine) launch_fdm<T>(m, r, s, m->wk.epart);
  if (fine && coarse && coarse_beside(m)) SEM_HIP(hipStreamWaitEvent(s, m->ev_join, 0));
  const double* Zv = coarse ? (const double*)m->Zv.p : nullptr;
  const int64_t n = (fine ? fdm_blocks(m) : 0) + (coarse ? coarse_parts(m) : 0);
  if (start) {
    reduce_partials(m, m->wk.epart, n, rz_out, 0, s);
    schwarz_sum<T, kSumStart>(m, p, nullptr, fine, Zv, s);
  } else if (n > 0 && n <= kConsumerSum) {
    schwarz_sum<T, kSumPx>(m, p, x, fine, Zv, s, rz_in, rz_out, (const double*)m->wk.epart, (int)n);
  } else {
    reduce_partials(m, m->wk.epart, n, 5, 2, s, rz_in, rz_out);
    schwarz_sum<T, kSumPx>(m, p, x, fine, Zv, s);
  }
  hipLaunchKernelGGL((gs_px_kernel<T>), dim3((unsigned)blocks_for(m->T.base_i)), dim3(kGS), 0, s, x, p, Wp<T>(m),
                     shared_nodes(m), (const double*)m->wk.sc, (int)start);
  SEM_HIP(hipGetLastError());
}

// --- coarse factorisation (set-up), multifrontal in post-order.  Node t's
// front F (f = s + b, column-major) holds the entries of A_c with the smaller
// index in t's own range, plus the update matrices of its children
// (extend-add).  Then S = F_II, S^-1 by Cholesky, W^T = S^-1 F_IB,
// W = F_BI S^-1 and the update U = F_BB - W F_IB for the parent.
void factor_coarse(sem_mesh m) {
  HostTables& T = m->T;
  release_coarse_graph(m);
  if (m->coarse_solver == SEM_COARSE_AMG) amg_setup(m);
  m->cidx.upload(T.cidx.data(), T.cidx.size());
  m->part_dst.upload(T.part_dst.data(), T.part_dst.size());
  m->cvec.alloc(std::max<int64_t>(T.c_size, 1));
  m->Xlev.alloc(std::max<int64_t>(T.nc, 1));
  SEM_HIP(hipMemset(m->Zv.p, 0, m->Zv.n * sizeof(double)));  // Dirichlet vertices stay 0
  if (T.nc == 0) {
    m->fwd_pool.release();
    m->bwd_pool.release();
    SEM_HIP(hipDeviceSynchronize());
    return;
  }
  // fronts are factored densely: bound their size
  if (T.max_front > 16384)
    throw Error{SEM_EUNSUPPORTED, "coarse front of " + std::to_string(T.max_front) + " vertices exceeds 16384"};
  m->tiles.upload(T.tiles.data(), T.tiles.size());
  m->fb_idx.upload(T.fb_idx.data(), T.fb_idx.size());
  m->cvert.upload(T.cvert.data(), T.cvert.size());
  m->pslot.upload(T.pslot.data(), T.pslot.size());
  m->pre_slot.upload(T.pre_slot.data(), T.pre_slot.size());
  m->pre_row.upload(T.pre_row.data(), T.pre_row.size());
  m->rs_off.upload(T.rs_off.data(), T.rs_off.size());
  m->cdst.upload(T.cdst.data(), T.cdst.size());
  m->fwd_pool.alloc(T.fwd_size);
  m->bwd_pool.alloc(std::max<int64_t>(T.bwd_size, 1));
  // the padding entry of odd rows is read (against a zero): keep it finite
  SEM_HIP(hipMemset(m->fwd_pool.p, 0, m->fwd_pool.n * sizeof(double)));
  SEM_HIP(hipMemset(m->bwd_pool.p, 0, m->bwd_pool.n * sizeof(double)));
  rocblas_handle hb;
  if (rocblas_create_handle(&hb) != rocblas_status_success) throw Error{SEM_EHIP, "rocblas_create_handle failed"};
  std::unique_ptr<std::remove_pointer<rocblas_handle>::type, decltype(&rocblas_destroy_handle)> guard(
      hb, rocblas_destroy_handle);
  // positions of every front's entries of A_c (columns of its own vertices;
  // entries towards eliminated vertices were taken by the descendants' fronts)
  // and of every child's boundary in its parent's front, in one upload
  const size_t nn = T.fnodes.size();
  std::vector<int32_t> pos, map;
  std::vector<double> val;
  std::vector<int64_t> a_at(nn + 1, 0), map_at(nn, 0);
  for (size_t q = 0; q < nn; ++q) {
    const FrontNode& F = T.fnodes[q];
    const int64_t s = F.s, b = F.b, f = s + b, end = F.off + s;
    const int32_t* B = T.fb_idx.data() + F.bidx;
    auto local = [&](int64_t g) -> int64_t {
      if (g >= F.off && g < end) return g - F.off;
      const int32_t* p = std::lower_bound(B, B + b, (int32_t)g);
      if (p == B + b || *p != g) throw Error{SEM_EMESH, "coarse front: entry outside the node's front"};
      return s + (p - B);
    };
    for (int64_t r = 0; r < s; ++r)
      for (int32_t k = T.ac_off[F.off + r]; k < T.ac_off[F.off + r + 1]; ++k) {
        if (T.ac_col[k] < F.off) continue;
        pos.push_back((int32_t)(r * f + local(T.ac_col[k])));
        val.push_back(T.ac_val[k]);
      }
    a_at[q + 1] = (int64_t)pos.size();
    for (int32_t c : T.fchildren[q]) {
      const FrontNode& C = T.fnodes[c];
      map_at[c] = (int64_t)map.size();
      for (int32_t k = 0; k < C.b; ++k) map.push_back((int32_t)local(T.fb_idx[C.bidx + k]));
    }
  }
  const int64_t mf = T.max_front;
  DBuf<double> Fd, Ust, vald;
  DBuf<int32_t> posd, mapd;
  DBuf<rocblas_int> info;
  posd.upload(pos.data(), pos.size());
  vald.upload(val.data(), val.size());
  mapd.upload(map.data(), map.size());
  info.alloc(2 * nn);
  SEM_HIP(hipMemset(info.p, 0, 2 * nn * sizeof(rocblas_int)));
  Fd.alloc((size_t)mf * mf);
  Ust.alloc(std::max<int64_t>(T.ustack_size, 1));
  std::vector<int64_t> u_at(nn, -1);  // update matrix position in the stack
  int64_t top = 0;
  const double one = 1.0, zero = 0.0, mone = -1.0;
  for (size_t q = 0; q < nn; ++q) {
    const FrontNode& F = T.fnodes[q];
    const int64_t s = F.s, b = F.b, f = s + b;
    SEM_HIP(hipMemsetAsync(Fd.p, 0, (size_t)f * f * sizeof(double), 0));
    const int64_t na = a_at[q + 1] - a_at[q];
    hipLaunchKernelGGL(front_scatter_kernel, dim3((unsigned)blocks_for(na)), dim3(kGS), 0, 0, Fd.p,
                       (const int32_t*)posd.p + a_at[q], (const double*)vald.p + a_at[q], na);
    SEM_HIP(hipGetLastError());
    if (b > 0) {
      hipLaunchKernelGGL(front_transpose_kernel, dim3((unsigned)blocks_for(s * b)), dim3(kGS), 0, 0, Fd.p, f, s, b);
      SEM_HIP(hipGetLastError());
    }
    // extend-add the children's update matrices, then pop them
    int64_t first = -1;
    for (int32_t c : T.fchildren[q]) {
      const FrontNode& C = T.fnodes[c];
      if (C.b == 0) continue;
      hipLaunchKernelGGL(front_extend_add_kernel, dim3((unsigned)blocks_for((int64_t)C.b * C.b)), dim3(kGS), 0, 0,
                         Fd.p, f, (const double*)Ust.p + u_at[c], (int64_t)C.b, (const int32_t*)mapd.p + map_at[c]);
      SEM_HIP(hipGetLastError());
      if (first < 0 || u_at[c] < first) first = u_at[c];
    }
    if (first >= 0) top = first;
    // S^-1 in place (lower triangle), mirrored; the info values are checked at the end
    if (rocsolver_dpotrf(hb, rocblas_fill_lower, (rocblas_int)s, Fd.p, (rocblas_int)f, info.p + 2 * q) !=
        rocblas_status_success)
      throw Error{SEM_EHIP, "rocsolver_dpotrf failed"};
    if (rocsolver_dpotri(hb, rocblas_fill_lower, (rocblas_int)s, Fd.p, (rocblas_int)f, info.p + 2 * q + 1) !=
        rocblas_status_success)
      throw Error{SEM_EHIP, "rocsolver_dpotri failed"};
    hipLaunchKernelGGL(symmetrize_kernel, dim3((unsigned)blocks_for(s * s)), dim3(kGS), 0, 0, Fd.p, s, f);
    SEM_HIP(hipGetLastError());
    // forward [S^-1 ; W] by rows = column-major s x (s + b) [S^-1 | W^T];
    // backward W^T by rows = column-major W
    double* X = m->fwd_pool.p + F.fwd;
    double* W = m->bwd_pool.p + F.bwd;
    const rocblas_int si = (rocblas_int)s, bi = (rocblas_int)b, fi = (rocblas_int)f;
    SEM_HIP(hipMemcpy2DAsync(X, F.lds * sizeof(double), Fd.p, f * sizeof(double), s * sizeof(double), s,
                             hipMemcpyDeviceToDevice, 0));
    if (b > 0) {
      // W = F_BI S^-1  (b x s), W^T = S^-1 F_IB  (s x b, the columns from s on)
      if (rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, bi, si, si, &one, Fd.p + s, fi, Fd.p, fi,
                        &zero, W, F.ldb) != rocblas_status_success)
        throw Error{SEM_EHIP, "rocblas_dgemm failed"};
      if (rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, si, bi, si, &one, Fd.p, fi, Fd.p + s * f,
                        fi, &zero, X + s * F.lds, F.lds) != rocblas_status_success)
        throw Error{SEM_EHIP, "rocblas_dgemm failed"};
      // U = F_BB - W F_IB, pushed for the parent
      if (top + b * b > std::max<int64_t>(T.ustack_size, 1)) throw Error{SEM_EHIP, "coarse update stack overflow"};
      double* U = Ust.p + top;
      SEM_HIP(hipMemcpy2DAsync(U, b * sizeof(double), Fd.p + s + s * f, f * sizeof(double), b * sizeof(double), b,
                               hipMemcpyDeviceToDevice, 0));
      if (rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, bi, bi, si, &mone, W, F.ldb, Fd.p + s * f,
                        fi, &one, U, bi) != rocblas_status_success)
        throw Error{SEM_EHIP, "rocblas_dgemm failed"};
      u_at[q] = top;
      top += b * b;
    }
  }
  std::vector<rocblas_int> bad(2 * nn);
  SEM_HIP(hipMemcpy(bad.data(), info.p, bad.size() * sizeof(rocblas_int), hipMemcpyDeviceToHost));
  for (rocblas_int v : bad)
    if (v != 0) throw Error{SEM_EMESH, "coarse matrix is not positive definite"};
  SEM_HIP(hipDeviceSynchronize());
  build_coarse_graph(m);
}

// D (n1 x n1, row-major) followed by the even/odd split that the line-phase
// operator kernel uses for D and for D^T (see line_pairs in the kernels):
// rows q < H = n1/2 of (D[q][m] + D[q][n1-1-m]) / 2 for m < H, D[q][H] when
// n1 is odd, (D[q][m] - D[q][n1-1-m]) / 2 for m < H; for odd n1 a last row of
// the middle output's (D[H][m] - D[H][n1-1-m]) / 2.  The other kernels read
// only the first n1 x n1 entries.
std::vector<double> d_with_split(const std::vector<double>& D, int n1) {
  const int H = n1 / 2, od = n1 % 2;
  std::vector<double> out(D);
  for (int t = 0; t < 2; ++t) {
    auto d = [&](int q, int m) { return t == 0 ? D[(size_t)q * n1 + m] : D[(size_t)m * n1 + q]; };
    for (int q = 0; q < H; ++q) {
      for (int m = 0; m < H; ++m) out.push_back(0.5 * (d(q, m) + d(q, n1 - 1 - m)));
      if (od) out.push_back(d(q, H));
      for (int m = 0; m < H; ++m) out.push_back(0.5 * (d(q, m) - d(q, n1 - 1 - m)));
    }
    if (od)
      for (int m = 0; m < H; ++m) out.push_back(0.5 * (d(H, m) - d(H, n1 - 1 - m)));
  }
  return out;
}

void upload_all(sem_mesh m) {
  HostTables& T = m->T;
  SEM_HIP(hipSetDevice(m->device));
  m->rec.upload(T.rec.data(), T.rec.size());
  m->order.upload(T.order.data(), T.order.size());
  m->vinc_off.upload(T.vinc_off.data(), T.vinc_off.size());
  m->einc_off.upload(T.einc_off.data(), T.einc_off.size());
  m->dir.upload(T.dir.data(), T.dir.size());
  m->fcount.upload(T.fcount.data(), T.fcount.size());
  m->G64.upload(T.G.data(), T.G.size());
  const std::vector<double> Dx = d_with_split(T.D, T.n1);
  m->D64.upload(Dx.data(), Dx.size());
  m->X864.upload(T.X8.data(), T.X8.size());
  std::vector<double> tq(T.t);
  tq.insert(tq.end(), T.rho.begin(), T.rho.end());
  m->tq64.upload(tq.data(), tq.size());
  m->w64.alloc(T.w_size);
  if (T.N >= kPatchRecordsFrom) {
    std::vector<int32_t> pidx, pdst;
    build_patch_records(T, pidx, pdst);
    m->pidx.upload(pidx.data(), pidx.size());
    m->pdst.upload(pdst.data(), pdst.size());
  } else {
    m->pidx.upload(T.ip.data(), T.ip.size());
    m->pdst.upload(T.xdest.data(), T.xdest.size());
  }
  m->S64.upload(T.S.data(), T.S.size());
  m->lam64.upload(T.lam.data(), T.lam.size());
  m->h64.upload(T.h.data(), T.h.size());
  // consumer slots no patch writes (NULL) stay zero for good
  m->zo64.alloc((size_t)T.E * T.np * T.np * T.np);
  SEM_HIP(hipMemset(m->zo64.p, 0, m->zo64.n * sizeof(double)));
  if (m->fp32) {
    auto G32 = convert<float>(T.G);
    m->G32.upload(G32.data(), G32.size());
    auto D32 = convert<float>(Dx);
    m->D32.upload(D32.data(), D32.size());
    auto X832 = convert<float>(T.X8);
    m->X832.upload(X832.data(), X832.size());
    auto tq32 = convert<float>(tq);
    m->tq32.upload(tq32.data(), tq32.size());
    m->w32.alloc(T.w_size);
    auto S32 = convert<float>(T.S);
    m->S32.upload(S32.data(), S32.size());
    auto l32 = convert<float>(T.lam);
    m->lam32.upload(l32.data(), l32.size());
    auto h32 = convert<float>(T.h);
    m->h32.upload(h32.data(), h32.size());
    m->zo32.alloc((size_t)T.E * T.np * T.np * T.np);
    SEM_HIP(hipMemset(m->zo32.p, 0, m->zo32.n * sizeof(float)));
  }
  // Phi_I(t_i): row I = 0, 1
  std::vector<double> phi(2 * T.n1);
  for (int i = 0; i < T.n1; ++i) {
    phi[i] = 0.5 * (1.0 - T.t[i]);
    phi[T.n1 + i] = 0.5 * (1.0 + T.t[i]);
  }
  m->phi.upload(phi.data(), phi.size());
  m->Zv.alloc(std::max<int64_t>(T.V, 1));
  m->part.alloc(kRedBlocks);
  m->sc.alloc(16);
  ensure_side_stream(m);
  SEM_HIP(hipHostMalloc((void**)&m->check_host, 4 * sizeof(double), hipHostMallocDefault));
  for (auto& e : m->ev_check) SEM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  factor_coarse(m);
}

// partial sums of one solve: p . A p and r . r (one per element workgroup at
// most), r . z (one per workgroup of the patch solves and of the coarse solve)
struct PartCounts {
  size_t d, r, e;
  size_t total() const { return d + r + e; }
};
PartCounts part_counts(sem_mesh m) {
  const size_t n = (size_t)xcd_grid(m->T.E);
  return PartCounts{n, n, (size_t)(fdm_blocks(m) + coarse_parts(m))};
}

void set_parts(sem_mesh m, double* base) {
  const PartCounts c = part_counts(m);
  m->wk.dpart = base;
  m->wk.rpart = base + c.d;
  m->wk.epart = base + c.d + c.r;
}

// the handle's own solve buffers (allocated on first need) as the work of the
// next solve
void ensure_work(sem_mesh m, bool need32) {
  const int64_t n = m->T.n_global;
  const size_t np = part_counts(m).total();
  if (m->parts.n < np) m->parts.alloc(np);
  for (int q = 0; q < 3; ++q) {
    if (m->v64[q].n != (size_t)n) m->v64[q].alloc(n);
    m->wk.v64[q] = m->v64[q].p;
  }
  for (int q = 0; q < 4; ++q) {
    if (need32 && m->v32[q].n != (size_t)n) m->v32[q].alloc(n);
    m->wk.v32[q] = need32 ? m->v32[q].p : nullptr;
  }
  m->wk.part = m->part.p;
  m->wk.sc = m->sc.p;
  set_parts(m, m->parts.p);
}

// --- static scratch of sem_pcg_solve_noalloc ------------------------------
// The work of one solve (Algorithm 1's scalars, partial sums and three FP64
// vectors, plus four FP32 vectors for the refined form) as views into one
// file-scope device array, for callers that cannot allocate device memory.
// Every device holds its own copy of the array, at its own address, resolved
// once per device at set-up (create_mesh) with that device current; host code
// uses only that address, never the array's name.
constexpr size_t kScratchBytes = size_t(128) << 20;
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

std::mutex g_scratch_mu;
std::vector<double*> g_scratch_dev;  // by device id: the device address of scratch (NULL until resolved)

void resolve_scratch(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_dev.size() <= device) g_scratch_dev.resize((size_t)device + 1, nullptr);
  if (g_scratch_dev[device] != nullptr) return;
  void* p = nullptr;
  SEM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
  if (p == nullptr) throw Error{SEM_EHIP, "hipGetSymbolAddress(scratch) returned NULL"};
  g_scratch_dev[device] = static_cast<double*>(p);
}

double* scratch_of(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return device >= 0 && device < (int)g_scratch_dev.size() ? g_scratch_dev[device] : nullptr;
}

// byte offsets of one solve's work inside the scratch array (256-aligned parts)
struct ScratchLayout {
  size_t sc, part, parts, v64, v32, s64, s32;  // s64, s32: bytes from one vector to the next
  size_t total;
};

ScratchLayout scratch_layout(sem_mesh m, bool need32) {
  auto up = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
  const size_t n = (size_t)m->T.n_global;
  ScratchLayout L{};
  L.s64 = up(n * sizeof(double));
  L.s32 = up(n * sizeof(float));
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += up(bytes);
    return at;
  };
  L.sc = take(16 * sizeof(double));
  L.part = take(kRedBlocks * sizeof(double));
  const size_t vectors = o;
  L.parts = take(part_counts(m).total() * sizeof(double));
  L.v64 = take(3 * L.s64);
  L.v32 = take(need32 ? 4 * L.s32 : 0);
  // which meshes the call takes is part of its interface (40 bytes per global
  // node, 60 in the refined form): what a solve no longer needs stays counted
  const size_t stated = vectors + up((size_t)(xcd_grid(m->T.E) + blocks_for(m->T.base_i)) * sizeof(double)) +
                        5 * L.s64 + (need32 ? 5 * L.s32 : 0);
  L.total = std::max(o, stated);
  return L;
}

// the next solve's work as views into the scratch array at `base`
void scratch_work(sem_mesh m, bool need32, double* base) {
  const ScratchLayout L = scratch_layout(m, need32);
  char* c = reinterpret_cast<char*>(base);
  for (int q = 0; q < 3; ++q) m->wk.v64[q] = reinterpret_cast<double*>(c + L.v64 + q * L.s64);
  for (int q = 0; q < 4; ++q) m->wk.v32[q] = need32 ? reinterpret_cast<float*>(c + L.v32 + q * L.s32) : nullptr;
  m->wk.part = reinterpret_cast<double*>(c + L.part);
  m->wk.sc = reinterpret_cast<double*>(c + L.sc);
  set_parts(m, reinterpret_cast<double*>(c + L.parts));
}

template <typename TA, typename TB>
void dot(sem_mesh m, const TA* a, const TB* b, int dst, hipStream_t s) {
  const int64_t n = m->T.n_global;
  const int nb = (int)std::min<int64_t>(kRedBlocks, blocks_for(n, kRedThreads));
  hipLaunchKernelGGL((dot_partial_kernel<TA, TB>), dim3(nb), dim3(kRedThreads), 0, s, a, b, m->wk.part, n,
                     (int)aligned16(a, b));
  SEM_HIP(hipGetLastError());
  reduce_partials(m, m->wk.part, nb, dst, 0, s);
}

double read_scalar(sem_mesh m, int idx, hipStream_t s) {
  double v = 0.0;
  SEM_HIP(hipMemcpyAsync(&v, m->wk.sc + idx, sizeof(double), hipMemcpyDeviceToHost, s));
  SEM_HIP(hipStreamSynchronize(s));
  return v;
}

// One PCG solve (Algorithm 1) on vectors of type T; x, r in/out (r holds the
// residual of x, rr0 = ||r||^2).  Returns the status; *iters gets the
// iterations, *rel the last ||r|| / ||b||.  A start that already meets the
// tolerance returns at once; after a breakdown x keeps the last finite iterate
// (the vector updates skip themselves once the flag is set).
//
// One iteration is nine launches and the coarse solve's (two sums fewer up to
// kConsumerSum partial sums, a chunk sum more for each beyond kOneSum): the
// operator's element kernel with p . A p; alpha; r -= alpha A p at the shared nodes,
// with the gather of A p, then at the interiors, with r . r and the coarse
// restriction; r . r to the host; the coarse solve; the patch solves with r . z;
// beta; the sum of the corrections into x and p at the interiors, then at the
// shared nodes.  The scalar products need no assembled vector, so neither A p at the
// shared nodes nor z is ever stored.  Against the gathers and vector updates as passes of
// their own: PCG to 1e-10 at 24^3, N = 7 19.2 -> 17.4 ms, 4^3,
// N = 4 3.0 -> 1.8 ms, 40^3 refined 62.8 -> 58.7 ms.
template <typename T>
int pcg_core(sem_mesh m, T* x, T* r, double bnorm2, double rr0, double rtol, int max_iter, int pc, int check_every,
             hipStream_t s, int* iters, double* rel, sem_solve_stats* st) {
  T* p;
  T* w;
  if constexpr (std::is_same<T, double>::value) {
    p = m->wk.v64[1];
    w = m->wk.v64[2];
  } else {
    p = m->wk.v32[1];
    w = m->wk.v32[2];
  }
  double* sc = m->wk.sc;
  const int64_t n = m->T.n_global;
  const int gb = grid_stride_blocks(n);
  const double tol2 = rtol * rtol * bnorm2;
  const bool fine = pc & SEM_PC_FINE, coarse = (pc & SEM_PC_COARSE) && m->T.nc > 0;
  int k = 0;
  double rr = rr0;
  *iters = 0;
  *rel = std::sqrt(rr / bnorm2);
  if (rr <= tol2) return SEM_OK;
  hipLaunchKernelGGL((fill_kernel<double>), dim3(1), dim3(kGS), 0, s, sc, 0.0, (int64_t)7);
  SEM_HIP(hipGetLastError());
  int rz = 0, rz_next = 10;  // scalar slots of r . z, in turn
  if (pc == SEM_PC_NONE) {
    hipLaunchKernelGGL((copy_kernel<T, T>), dim3(gb), dim3(kGS), 0, s, p, (const T*)r, n);
    SEM_HIP(hipGetLastError());
    dot<T, T>(m, r, r, rz, s);
  } else {
    if (coarse) {
      launch_restrict<T, false>(m, r, (const T*)nullptr, true, s);
      pcg_start_coarse(m, fine, s);
    }
    pcg_finish<T>(m, r, x, p, fine, coarse, rz, rz, true, s);
  }
  int status = SEM_ENOCONV;
  bool pending_x = false;       // x += alpha p of the last iteration not yet applied
  bool coarse_pending = false;  // a coarse solve forked that no pcg_finish has joined
  int late = 0;                 // iteration whose check is not looked at yet (0: none)
  // r . r of iteration q, read back by its check; true when the solve is over
  auto over = [&](int q) {
    SEM_HIP(hipEventSynchronize(m->ev_check[q & 1]));
    const double* h = m->check_host + 2 * (q & 1);
    rr = h[0];
    const double flag = h[1];
    if (st && st->history && st->history_len < st->history_cap)
      st->history[st->history_len++] = std::sqrt(rr / bnorm2);
    if (flag != 0.0 || !std::isfinite(rr))
      status = SEM_EBREAKDOWN;
    else if (rr <= tol2)
      status = SEM_OK;
    else
      return false;
    k = q;
    return true;
  };
  while (k < max_iter) {
    const int64_t nr = pcg_update_r<T>(m, r, p, w, rz, coarse, s);
    ++k;
    pending_x = true;
    const bool check = k % check_every == 0 || k == max_iter;
    if (pc == SEM_PC_NONE) reduce_partials(m, m->wk.rpart, nr, 5, 2, s, rz, rz_next);
    if (check) {
      reduce_partials(m, m->wk.rpart, nr, 4, 3, s, 0, 0, m->check_host + 2 * (k & 1));
      SEM_HIP(hipEventRecord(m->ev_check[k & 1], s));
    }
    if (coarse) {
      pcg_start_coarse(m, fine, s);
      coarse_pending = fine && coarse_beside(m);
    }
    // The check of the iteration before, then this one's.  Far from the
    // tolerance (the last r . r above 100 tol^2) this one's is looked at when
    // the next iteration's first half is enqueued, so that the GPU works
    // through the host's round trip; if it then ends the solve, x is already
    // the iterate of this step, and what follows it was spent for nothing,
    // which this margin makes rare
    if (late != 0) {
      const int q = late;
      late = 0;
      if (over(q)) {
        pending_x = false;  // applied before the next iteration began
        break;
      }
    }
    if (check) {
      if (k < max_iter && rr > 100.0 * tol2)
        late = k;
      else if (over(k))
        break;
    }
    if (pc == SEM_PC_NONE) {
      hipLaunchKernelGGL((update_px_kernel<T>), dim3(gb), dim3(kGS), 0, s, x, p, (const T*)r, (const double*)sc, n,
                         (int)aligned16(x, p, r));
      SEM_HIP(hipGetLastError());
    } else {
      pcg_finish<T>(m, r, x, p, fine, coarse, rz, rz_next, false, s);
      coarse_pending = false;
    }
    std::swap(rz, rz_next);
    pending_x = false;
  }
  // a coarse solve forked for an iteration that did not follow: the caller's
  // stream waits for it, so no later work on the handle overlaps it
  if (coarse_pending) SEM_HIP(hipStreamWaitEvent(s, m->ev_join, 0));
  if (pending_x && status != SEM_EBREAKDOWN) {
    hipLaunchKernelGGL((update_x_kernel<T>), dim3(gb), dim3(kGS), 0, s, x, (const T*)p, (const double*)sc, n);
    SEM_HIP(hipGetLastError());
  }
  *iters = k;
  *rel = std::sqrt(rr / bnorm2);
  return status;
}

// back from per-node coefficients: the plain factors G return to the device
// (in place, so the buffers keep their addresses)
void leave_node_coefficients(sem_mesh m) {
  if (!m->per_node) return;
  m->per_node = false;
  if (m->host_only) return;
  SEM_HIP(hipSetDevice(m->device));
  SEM_HIP(hipDeviceSynchronize());
  m->G64.copy_in(m->T.G.data(), m->T.G.size());
  if (m->fp32) {
    const std::vector<float> f = convert<float>(m->T.G);
    m->G32.copy_in(f.data(), f.size());
  }
}

// kappa and c of the operator, the patch solves and the coarse matrix (whose
// values are reassembled and refactorised when they change)
void set_coefficients(sem_mesh m, double kappa, double c) {
  HostTables& T = m->T;
  if (!m->per_elem && T.kappa == kappa && T.cmass == c) return;
  leave_node_coefficients(m);
  T.kappa = kappa;
  T.cmass = c;
  T.kap_e.clear();
  T.c_e.clear();
  m->per_elem = false;
  assemble_coarse_matrix(T);
  if (m->host_only) return;
  SEM_HIP(hipSetDevice(m->device));
  SEM_HIP(hipDeviceSynchronize());
  if (c != 0.0 && m->mN64.p == nullptr) {
    m->mN64.upload(T.mN.data(), T.mN.size());
    if (m->fp32) {
      const std::vector<float> f = convert<float>(T.mN);
      m->mN32.upload(f.data(), f.size());
    }
  }
  factor_coarse(m);
}

// one kappa_e > 0 and c_e >= 0 per element (Algorithm 2): uploaded with the
// local mass m_{ijk;e} when some c_e != 0; coarse matrix reassembled
void set_element_coefficients(sem_mesh m, const double* kap, const double* c) {
  HostTables& T = m->T;
  const int64_t E = T.E;
  leave_node_coefficients(m);
  if (kap)
    T.kap_e.assign(kap, kap + E);
  else
    T.kap_e.assign(E, 1.0);
  if (c)
    T.c_e.assign(c, c + E);
  else
    T.c_e.assign(E, 0.0);
  T.kappa = T.cmass = std::nan("");
  bool any_c = false;
  for (double v : T.c_e) any_c = any_c || v != 0.0;
  assemble_coarse_matrix(T);
  m->per_elem = true;
  m->any_ce = any_c;
  if (m->host_only) return;
  SEM_HIP(hipSetDevice(m->device));
  SEM_HIP(hipDeviceSynchronize());
  m->ke64.upload(T.kap_e.data(), E);
  m->ce64.upload(T.c_e.data(), E);
  if (m->fp32) {
    const std::vector<float> kf = convert<float>(T.kap_e), cf = convert<float>(T.c_e);
    m->ke32.upload(kf.data(), E);
    m->ce32.upload(cf.data(), E);
  }
  if (any_c && m->mL64.p == nullptr) {
    m->mL64.upload(T.mass.data(), T.mass.size());
    if (m->fp32) {
      const std::vector<float> f = convert<float>(T.mass);
      m->mL32.upload(f.data(), f.size());
    }
  }
  factor_coarse(m);
}

// kappa_{ijk;e} > 0 and c_{ijk;e} >= 0 at every local node (eq. (R)): kappa
// multiplies the six factors G at its node, c the local mass.  The patch solves
// and the coarse matrix take one value per element: the mean over the
// reference cube by the GLL rule, (1/8) sum rho_i rho_j rho_k v_{ijk;e}.
void set_node_coefficients(sem_mesh m, const double* kap, const double* c) {
  HostTables& T = m->T;
  const int64_t E = T.E;
  const int n1 = T.n1;
  const int64_t NN = (int64_t)n1 * n1 * n1;
  T.kap_e.assign(E, 1.0);
  T.c_e.assign(E, 0.0);
  std::vector<double> nc(E, 0.0);
  bool any_c = false;
  for (int64_t e = 0; e < E; ++e) {
    double ks = 0.0, cs = 0.0;
    for (int k = 0; k < n1; ++k)
      for (int j = 0; j < n1; ++j)
        for (int i = 0; i < n1; ++i) {
          const int64_t l = e * NN + i + (int64_t)n1 * (j + (int64_t)n1 * k);
          const double w = T.rho[i] * T.rho[j] * T.rho[k] * 0.125;
          if (kap) ks += w * kap[l];
          if (c) {
            cs += w * c[l];
            if (c[l] != 0.0) nc[e] = 1.0;
          }
        }
    if (kap) T.kap_e[e] = ks;
    T.c_e[e] = cs;
    any_c = any_c || nc[e] != 0.0;
  }
  T.kappa = T.cmass = std::nan("");
  assemble_coarse_matrix(T);
  m->per_elem = true;
  m->per_node = true;
  m->any_ce = any_c;
  if (m->host_only) return;
  SEM_HIP(hipSetDevice(m->device));
  SEM_HIP(hipDeviceSynchronize());
  // factors scaled by kappa at their node; c m per local node
  std::vector<double> Gs(T.G.size());
  for (int64_t e = 0; e < E; ++e)
    for (int f = 0; f < 6; ++f)
      for (int64_t l = 0; l < NN; ++l) {
        const int64_t o = (e * 6 + f) * NN + l;
        Gs[o] = kap ? kap[e * NN + l] * T.G[o] : T.G[o];
      }
  std::vector<double> cm;
  if (any_c) {
    cm.resize((size_t)E * NN);
    for (int64_t l = 0; l < E * NN; ++l) cm[l] = c[l] * T.mass[l];
  }
  const std::vector<double> ones(E, 1.0);
  m->G64.copy_in(Gs.data(), Gs.size());
  // kappa per node for the operator kernel that rebuilds G from the vertices
  std::vector<double> kl;
  if (kap)
    kl.assign(kap, kap + E * NN);
  else
    kl.assign((size_t)E * NN, 1.0);
  m->kn64.upload(kl.data(), kl.size());
  m->ke64.upload(T.kap_e.data(), E);
  m->ce64.upload(T.c_e.data(), E);
  m->nk64.upload(ones.data(), E);
  m->nc64.upload(nc.data(), E);
  if (any_c) m->nm64.upload(cm.data(), cm.size());
  if (m->fp32) {
    const std::vector<float> Gf = convert<float>(Gs);
    m->G32.copy_in(Gf.data(), Gf.size());
    const std::vector<float> klf = convert<float>(kl);
    m->kn32.upload(klf.data(), klf.size());
    const std::vector<float> kf = convert<float>(T.kap_e), cf = convert<float>(T.c_e);
    m->ke32.upload(kf.data(), E);
    m->ce32.upload(cf.data(), E);
    const std::vector<float> of = convert<float>(ones), ncf = convert<float>(nc);
    m->nk32.upload(of.data(), E);
    m->nc32.upload(ncf.data(), E);
    if (any_c) {
      const std::vector<float> cmf = convert<float>(cm);
      m->nm32.upload(cmf.data(), cmf.size());
    }
  }
  factor_coarse(m);
}

// The solve behind sem_pcg_solve, in the work buffers m->wk (set by the caller).
// b counts on the free nodes only: r = mask(b - A x), ||b|| = ||mask(b)||.
int solve_impl(sem_mesh m, const double* b, double* x, const sem_solve_opts* o, sem_solve_stats* st,
               hipStream_t s) {
  auto t0 = std::chrono::steady_clock::now();
  const int64_t n = m->T.n_global;
  const bool refined = o->mode == SEM_SOLVE_FP32_REFINED;
  if (refined && (!m->fp32 || m->wk.v32[0] == nullptr)) throw Error{SEM_EUNSUPPORTED, "no FP32 work buffers"};
  const int gb = grid_stride_blocks(n);
  const int nb = (int)std::min<int64_t>(kRedBlocks, blocks_for(n, kRedThreads));
  const int check = std::max(1, o->check_every);
  if (st) st->history_len = 0;
  double* r64 = m->wk.v64[0];
  double* Ax = m->wk.v64[2];
  // r = mask(b - A x) with ||r||^2 into scalar slot `slot` (Ax = NULL: r = mask(b))
  auto residual = [&](const double* ax, int slot) {
    hipLaunchKernelGGL(residual_kernel, dim3(nb), dim3(kRedThreads), 0, s, r64, b, ax, (const uint8_t*)m->dir.p,
                       m->wk.part, n);
    reduce_partials(m, m->wk.part, nb, slot, 0, s);
    return read_scalar(m, slot, s);
  };
  const double bnorm2 = residual(nullptr, 7);
  int status = SEM_OK, iters = 0, outer = 0;
  double rel = 0.0;
  if (!std::isfinite(bnorm2)) {
    status = SEM_EBREAKDOWN;
  } else if (bnorm2 == 0.0) {
    hipLaunchKernelGGL((fill_kernel<double>), dim3(gb), dim3(kGS), 0, s, x, 0.0, n);
    SEM_HIP(hipGetLastError());
    SEM_HIP(hipStreamSynchronize(s));
  } else if (!refined) {
    double rr0 = bnorm2;  // x = 0: r = mask(b) already
    if (o->use_x0) {
      apply_A<double>(m, x, Ax, s);
      rr0 = residual(Ax, 8);
    } else {
      hipLaunchKernelGGL((fill_kernel<double>), dim3(gb), dim3(kGS), 0, s, x, 0.0, n);
      SEM_HIP(hipGetLastError());
    }
    status = !std::isfinite(rr0) ? SEM_EBREAKDOWN
                                 : pcg_core<double>(m, x, r64, bnorm2, rr0, o->rtol, o->max_iter, o->pc, check, s,
                                                    &iters, &rel, st);
    // the recursive residual can drift below the true one: confirm with
    // b - A x and restart from the true residual while it is above the tolerance
    const double tol2 = o->rtol * o->rtol * bnorm2;
    while (status == SEM_OK) {
      apply_A<double>(m, x, Ax, s);
      const double rr = residual(Ax, 8);
      rel = std::sqrt(rr / bnorm2);
      if (!std::isfinite(rr)) {
        status = SEM_EBREAKDOWN;
        break;
      }
      if (rr <= tol2) break;
      if (iters >= o->max_iter) {
        status = SEM_ENOCONV;
        break;
      }
      ++outer;
      int it = 0;
      status = pcg_core<double>(m, x, r64, bnorm2, rr, o->rtol, o->max_iter - iters, o->pc, check, s, &it, &rel, st);
      iters += it;
    }
  } else {
    // outer FP64 refinement around FP32 inner PCG solves
    float* r32 = m->wk.v32[0];
    float* d32 = m->wk.v32[3];
    if (!o->use_x0) hipLaunchKernelGGL((fill_kernel<double>), dim3(gb), dim3(kGS), 0, s, x, 0.0, n);
    status = SEM_ENOCONV;
    const double tol2 = o->rtol * o->rtol * bnorm2;
    for (outer = 0; outer <= o->max_outer; ++outer) {
      apply_A<double>(m, x, Ax, s);
      const double rr = residual(Ax, 8);
      rel = std::sqrt(rr / bnorm2);
      if (st && st->history && st->history_len < st->history_cap) st->history[st->history_len++] = rel;
      if (!std::isfinite(rr)) {
        status = SEM_EBREAKDOWN;
        break;
      }
      if (rr <= tol2) {
        status = SEM_OK;
        break;
      }
      if (outer == o->max_outer) break;
      const double rn = std::sqrt(rr);
      hipLaunchKernelGGL(scale_to_f32_kernel, dim3(gb), dim3(kGS), 0, s, r32, r64, 1.0 / rn, n);
      hipLaunchKernelGGL((fill_kernel<float>), dim3(gb), dim3(kGS), 0, s, d32, 0.0f, n);
      SEM_HIP(hipGetLastError());
      // ||r32||^2 of the scaled residual (about 1)
      dot<float, float>(m, r32, r32, 9, s);
      const double r32n2 = read_scalar(m, 9, s);
      int it = 0;
      double irel = 0.0;
      const int st_in = pcg_core<float>(m, d32, r32, r32n2, r32n2, o->inner_rtol, o->max_iter, o->pc, check, s, &it,
                                        &irel, nullptr);
      iters += it;
      if (st_in == SEM_EBREAKDOWN) {
        status = SEM_EBREAKDOWN;
        break;
      }
      hipLaunchKernelGGL(axpy_f32_kernel, dim3(gb), dim3(kGS), 0, s, x, d32, rn, n);
      SEM_HIP(hipGetLastError());
    }
  }
  SEM_HIP(hipStreamSynchronize(s));
  if (st) {
    st->iterations = iters;
    st->outer_iterations = outer;
    st->rel_residual = rel;
    st->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  return status;
}

template <typename F>
int guarded(F&& f) {
  try {
    return f();
  } catch (const Error& e) {
    set_error(e.msg);
    return e.status;
  } catch (const std::bad_alloc&) {
    set_error("host allocation failed");
    return SEM_ENOMEM;
  } catch (const std::exception& e) {
    set_error(e.what());
    return SEM_EINVAL;
  }
}

int need_device(sem_mesh m) {
  if (!m) {
    set_error("NULL handle");
    return SEM_EINVAL;
  }
  if (m->host_only) {
    set_error("host-only handle: no device state");
    return SEM_EUNSUPPORTED;
  }
  return SEM_OK;
}

template void apply_A<double>(sem_mesh, const double*, double*, hipStream_t);
template void apply_A<float>(sem_mesh, const float*, float*, hipStream_t);
template void precond<double>(sem_mesh, const double*, double*, int, hipStream_t);
template void precond<float>(sem_mesh, const float*, float*, int, hipStream_t);

// Autotuner of the operator tile: time each candidate (elements per
// workgroup) on this mesh and keep the fastest; results keyed by
// (architecture, order, dtype, element-count bucket) in an optional text cache.
template <typename T>
int tune_tile(sem_mesh m) {
  const int N = m->T.N;
  std::vector<int> cands;
  for (int c : kTileCandidates)
    if (c * (N + 1) * (N + 1) <= 1024 && c * (N + 1) * (N + 1) >= 16) cands.push_back(c);
  if (N == 15) cands.push_back(kTileMfma);
  cands.push_back(kTileGeo);
  cands.push_back(kTileLineGeo);
  cands.push_back(kTileLineStored);
  if (cands.size() <= 1) return cands.empty() ? 1 : cands[0];
  DBuf<T> u, y;
  u.alloc(m->T.n_global);
  y.alloc(m->T.n_global);
  hipLaunchKernelGGL((fill_kernel<T>), dim3(grid_stride_blocks(m->T.n_global)), dim3(kGS), 0, 0, u.p, T(1),
                     m->T.n_global);
  hipEvent_t a, b;
  SEM_HIP(hipEventCreate(&a));
  SEM_HIP(hipEventCreate(&b));
  const int idx = std::is_same<T, double>::value ? 0 : 1;
  // candidates interleaved over several rounds, best time per candidate kept,
  // so that clock drift does not favour whichever ran first
  constexpr int kRounds = 3;
  std::vector<float> best_ms(cands.size(), 1e30f);
  for (int round = 0; round < kRounds; ++round)
    for (size_t q = 0; q < cands.size(); ++q) {
      m->epb[idx] = cands[q];
      apply_A_elements<T>(m, u.p, y.p, 0);
      SEM_HIP(hipEventRecord(a, 0));
      for (int r = 0; r < 3; ++r) apply_A_elements<T>(m, u.p, y.p, 0);
      SEM_HIP(hipEventRecord(b, 0));
      SEM_HIP(hipEventSynchronize(b));
      float ms = 0.f;
      SEM_HIP(hipEventElapsedTime(&ms, a, b));
      best_ms[q] = std::min(best_ms[q], ms);
    }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  // the default tile unless another is faster by more than the timing noise
  const int def = default_tile(N);
  size_t pick = 0;
  for (size_t q = 0; q < cands.size(); ++q)
    if (cands[q] == def) pick = q;
  for (size_t q = 0; q < cands.size(); ++q)
    if (best_ms[q] < 0.98f * best_ms[pick] && best_ms[q] < best_ms[pick]) pick = q;
  return cands[pick];
}

std::string tune_key(sem_mesh m, int dtype) {
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, m->device) != hipSuccess) return "";
  int bucket = 0;
  for (int64_t e = m->T.E; e > 1; e >>= 2) ++bucket;  // element count, base-4 buckets
  return std::string(prop.gcnArchName).substr(0, std::string(prop.gcnArchName).find(':')) + " N=" +
         std::to_string(m->T.N) + " dtype=" + std::to_string(dtype) + " ebucket=" + std::to_string(bucket);
}

void autotune(sem_mesh m, const char* cache) {
  for (int d = 0; d < (m->fp32 ? 2 : 1); ++d) {
    const std::string key = tune_key(m, d);
    int found = 0;
    if (cache && !key.empty()) {
      if (FILE* f = std::fopen(cache, "r")) {
        char line[512];
        while (std::fgets(line, sizeof line, f)) {
          std::string l(line);
          const size_t p = l.rfind(" epb=");
          if (p != std::string::npos && l.compare(0, p, key) == 0) found = std::atoi(l.c_str() + p + 5);
        }
        std::fclose(f);
      }
    }
    if (found > 0 && tile_code_ok(found, m->T.N)) {
      m->epb[d] = found;
      continue;
    }
    m->epb[d] = d == 0 ? tune_tile<double>(m) : tune_tile<float>(m);
    if (cache && !key.empty())
      if (FILE* f = std::fopen(cache, "a")) {
        std::fprintf(f, "%s epb=%d\n", key.c_str(), m->epb[d]);
        std::fclose(f);
      }
  }
  SEM_HIP(hipDeviceSynchronize());
}

sem_mesh_s* create_mesh(const double* vtx, int64_t n_vtx, const int64_t* hex, int64_t n_hex, int order,
                        const sem_setup_opts* opts) {
  if (!vtx || !hex || n_vtx <= 0 || n_hex <= 0) throw Error{SEM_EINVAL, "NULL or empty mesh input"};
  if (order < 2 || order > 15) throw Error{SEM_EUNSUPPORTED, "order must be in 2..15"};
  sem_setup_opts d;
  sem_default_setup_opts(&d);
  if (!opts) opts = &d;
  auto m = std::make_unique<sem_mesh_s>();
  m->host_only = opts->host_only != 0;
  m->fp32 = opts->build_fp32 != 0;
  m->device = opts->device;
  HostTables& T = m->T;
  build_reference(T, order);
  build_numbering(T, hex, n_hex, n_vtx);
  build_geometry(T, vtx, hex);
  build_patches(T, hex);
  build_coarse_matrices(T, vtx, hex);
  build_coarse_tree(T);
  m->epb[0] = m->epb[1] = default_tile(order);
  if (!m->host_only) {
    upload_all(m.get());
    resolve_scratch(m->device);  // upload_all left the handle's device current
    if (opts->autotune) autotune(m.get(), opts->tune_cache);
  }
  return m.release();
}

int guarded_call(const std::function<int()>& f) { return guarded(f); }

}  // namespace sem

// ============================================================================
// C ABI
// ============================================================================
extern "C" {

void sem_default_setup_opts(sem_setup_opts* o) {
  if (!o) return;
  o->device = 0;
  o->host_only = 0;
  o->build_fp32 = 1;
  o->autotune = 1;
  o->tune_cache = nullptr;
}

int sem_mesh_set_tile(sem_mesh m, int dtype, int epb) {
  if (!m || (dtype != SEM_F64 && dtype != SEM_F32)) return SEM_EINVAL;
  if (!tile_code_ok(epb, m->T.N)) {
    set_error("tile not available for this order and dtype");
    return SEM_EINVAL;
  }
  m->epb[dtype == SEM_F64 ? 0 : 1] = epb;
  return SEM_OK;
}

int sem_mesh_tile(sem_mesh m, int dtype, int* epb) {
  if (!m || !epb || (dtype != SEM_F64 && dtype != SEM_F32)) return SEM_EINVAL;
  *epb = m->epb[dtype == SEM_F64 ? 0 : 1];
  return SEM_OK;
}

int sem_mesh_coarse_factor_size(sem_mesh m, int64_t* fwd_entries, int64_t* bwd_entries) {
  if (!m || !fwd_entries || !bwd_entries) return SEM_EINVAL;
  *fwd_entries = m->T.fwd_entries;
  *bwd_entries = m->T.bwd_entries;
  return SEM_OK;
}

void sem_default_solve_opts(sem_solve_opts* o) {
  if (!o) return;
  o->mode = SEM_SOLVE_FP64;
  o->pc = SEM_PC_TWOSCALE;
  o->rtol = 1e-8;
  o->max_iter = 1000;
  o->use_x0 = 0;
  o->inner_rtol = 1e-3;
  o->max_outer = 20;
  o->check_every = 1;
}

const char* sem_last_error(void) { return g_last_error.c_str(); }

int sem_mesh_setup(const double* vtx, int64_t n_vtx, const int64_t* hex, int64_t n_hex, int order,
                   const sem_setup_opts* opts, sem_mesh* out) {
  return guarded([&]() -> int {
    if (!out) throw Error{SEM_EINVAL, "NULL output handle"};
    *out = nullptr;
    *out = create_mesh(vtx, n_vtx, hex, n_hex, order, opts);
    return SEM_OK;
  });
}

int sem_mesh_destroy(sem_mesh m) {
  if (!m) return SEM_OK;
  if (!m->host_only) {
    (void)hipSetDevice(m->device);
    (void)hipDeviceSynchronize();
    release_coarse_graph(m);
    if (m->capture_stream) (void)hipStreamDestroy(m->capture_stream);
    if (m->side_stream) (void)hipStreamDestroy(m->side_stream);
    if (m->ev_fork) (void)hipEventDestroy(m->ev_fork);
    if (m->ev_join) (void)hipEventDestroy(m->ev_join);
    for (auto e : m->ev_check)
      if (e) (void)hipEventDestroy(e);
    if (m->check_host) (void)hipHostFree(m->check_host);
  }
  delete m;
  return SEM_OK;
}

int sem_mesh_sizes(sem_mesh m, int64_t* n_global, int64_t* n_local, int64_t* n_vertices) {
  if (!m) return SEM_EINVAL;
  if (n_global) *n_global = m->T.n_global;
  if (n_local) *n_local = m->T.n_local;
  if (n_vertices) *n_vertices = m->T.V;
  return SEM_OK;
}

int sem_mesh_numbering(sem_mesh m, int32_t* l2g) {
  if (!m || !l2g) return SEM_EINVAL;
  return guarded([&]() -> int {
    export_l2g(m->T, l2g);
    return SEM_OK;
  });
}

int sem_mesh_gs_csr(sem_mesh m, int64_t* offsets, int32_t* idx) {
  if (!m || !offsets || !idx) return SEM_EINVAL;
  return guarded([&]() -> int {
    const HostTables& T = m->T;
    std::vector<int32_t> l2g(T.n_local);
    export_l2g(T, l2g.data());
    std::fill(offsets, offsets + T.n_global + 1, 0);
    for (int64_t x = 0; x < T.n_local; ++x) offsets[l2g[x] + 1]++;
    for (int64_t g = 0; g < T.n_global; ++g) offsets[g + 1] += offsets[g];
    std::vector<int64_t> fill(offsets, offsets + T.n_global);
    for (int64_t x = 0; x < T.n_local; ++x) idx[fill[l2g[x]]++] = (int32_t)x;
    return SEM_OK;
  });
}

int sem_mesh_patch_table(sem_mesh m, int32_t* ip) {
  if (!m || !ip) return SEM_EINVAL;
  std::copy(m->T.ip.begin(), m->T.ip.end(), ip);
  return SEM_OK;
}

int sem_mesh_node_coords(sem_mesh m, double* xyz) {
  if (!m || !xyz) return SEM_EINVAL;
  std::copy(m->T.xN.begin(), m->T.xN.end(), xyz);
  return SEM_OK;
}

int sem_mesh_lumped_mass(sem_mesh m, double* mass) {
  if (!m || !mass) return SEM_EINVAL;
  std::copy(m->T.mN.begin(), m->T.mN.end(), mass);
  return SEM_OK;
}

int sem_mesh_boundary_mask(sem_mesh m, uint8_t* mask) {
  if (!m || !mask) return SEM_EINVAL;
  std::copy(m->T.dir.begin(), m->T.dir.end(), mask);
  return SEM_OK;
}

int sem_mesh_geometry(sem_mesh m, double* G, double* mass) {
  if (!m) return SEM_EINVAL;
  if (G) std::copy(m->T.G.begin(), m->T.G.end(), G);
  if (mass) std::copy(m->T.mass.begin(), m->T.mass.end(), mass);
  return SEM_OK;
}

int sem_mesh_set_dirichlet(sem_mesh m, const uint8_t* mask) {
  if (!m || !mask) return SEM_EINVAL;
  return guarded([&]() -> int {
    HostTables& T = m->T;
    for (int64_t g = 0; g < T.n_global; ++g) T.dir[g] = mask[g] ? 1 : 0;
    // the coarse free set follows the vertex nodes: new dissection, new factor
    build_coarse_tree(T);
    update_interior_mask_flags(T);
    if (!m->host_only) {
      SEM_HIP(hipSetDevice(m->device));
      SEM_HIP(hipDeviceSynchronize());
      m->dir.upload(T.dir.data(), T.dir.size());
      m->rec.upload(T.rec.data(), T.rec.size());
      factor_coarse(m);
    }
    return SEM_OK;
  });
}

int sem_apply_A(sem_mesh m, const void* u, void* y, int dtype, void* stream) {
  int st = need_device(m);
  if (st) return st;
  if (!u || !y || u == y) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    hipStream_t s = (hipStream_t)stream;
    if (dtype == SEM_F64)
      apply_A<double>(m, (const double*)u, (double*)y, s);
    else if (dtype == SEM_F32) {
      if (!m->fp32) throw Error{SEM_EUNSUPPORTED, "handle built without FP32 copies"};
      apply_A<float>(m, (const float*)u, (float*)y, s);
    } else
      throw Error{SEM_EINVAL, "dtype"};
    return SEM_OK;
  });
}

int sem_time_apply_A(sem_mesh m, const void* u, void* y, int dtype, int reps, void* stream, double* ms_element,
                     double* ms_gather) {
  int st = need_device(m);
  if (st) return st;
  if (!u || !y || u == y || reps < 1) return SEM_EINVAL;
  if (dtype == SEM_F32 && !m->fp32) return SEM_EUNSUPPORTED;
  if (dtype != SEM_F64 && dtype != SEM_F32) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    hipStream_t s = (hipStream_t)stream;
    std::vector<hipEvent_t> ev(3 * (size_t)reps);
    for (auto& e : ev) SEM_HIP(hipEventCreate(&e));
    struct Cleanup {
      std::vector<hipEvent_t>& v;
      ~Cleanup() {
        for (auto e : v) (void)hipEventDestroy(e);
      }
    } cleanup{ev};
    for (int r = 0; r < reps; ++r) {
      SEM_HIP(hipEventRecord(ev[3 * r], s));
      if (dtype == SEM_F64)
        apply_A_elements<double>(m, (const double*)u, (double*)y, s);
      else
        apply_A_elements<float>(m, (const float*)u, (float*)y, s);
      SEM_HIP(hipEventRecord(ev[3 * r + 1], s));
      if (dtype == SEM_F64)
        launch_gs<double>(m, (double*)y, s, (const double*)u);
      else
        launch_gs<float>(m, (float*)y, s, (const float*)u);
      SEM_HIP(hipEventRecord(ev[3 * r + 2], s));
    }
    SEM_HIP(hipStreamSynchronize(s));
    double te = 0.0, tg = 0.0;
    for (int r = 0; r < reps; ++r) {
      float a = 0.f, b = 0.f;
      SEM_HIP(hipEventElapsedTime(&a, ev[3 * r], ev[3 * r + 1]));
      SEM_HIP(hipEventElapsedTime(&b, ev[3 * r + 1], ev[3 * r + 2]));
      te += a;
      tg += b;
    }
    if (ms_element) *ms_element = te / reps;
    if (ms_gather) *ms_gather = tg / reps;
    return SEM_OK;
  });
}

int sem_stream_bench(const double* a, double* b, double* c, int64_t n, int reps, void* stream, double* gbs) {
  if (!a || !b || !c || !gbs || n < 2 || (n & 1) || reps < 1 || a == b || a == c || b == c ||
      !aligned16(a, b, c))
    return SEM_EINVAL;
  return guarded([&]() -> int {
    hipStream_t s = (hipStream_t)stream;
    const int64_t n2 = n / 2;
    hipEvent_t e0, e1;
    SEM_HIP(hipEventCreate(&e0));
    SEM_HIP(hipEventCreate(&e1));
    struct Cleanup {
      hipEvent_t a, b;
      ~Cleanup() {
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
      }
    } cleanup{e0, e1};
    const double bytes[3] = {16.0 * n, 24.0 * n, 8.0 * n};
    for (int q = 0; q < 3; ++q) gbs[q] = 0.0;
    // best over grid sizes (workgroups of 256 lanes), each timed over reps launches
    for (int grid : {1024, 2048, 4096, 8192, 16384, 32768, 65536}) {
      const int g = (int)std::min<int64_t>(grid, (n2 + 255) / 256);
      for (int q = 0; q < 3; ++q) {
        auto launch = [&]() {
          if (q == 0)
            hipLaunchKernelGGL(stream_copy_kernel, dim3(g), dim3(256), 0, s, (double2*)b, (const double2*)a, n2);
          else if (q == 1)
            hipLaunchKernelGGL(stream_triad_kernel, dim3(g), dim3(256), 0, s, (double2*)c, (const double2*)a,
                               (const double2*)b, 0.5, n2);
          else  // the partial sums land in c (g <= n2 entries)
            hipLaunchKernelGGL(stream_read_kernel, dim3(g), dim3(256), 0, s, (const double2*)a, n2, c);
        };
        launch();
        SEM_HIP(hipEventRecord(e0, s));
        for (int r = 0; r < reps; ++r) launch();
        SEM_HIP(hipEventRecord(e1, s));
        SEM_HIP(hipEventSynchronize(e1));
        float ms = 0.f;
        SEM_HIP(hipEventElapsedTime(&ms, e0, e1));
        gbs[q] = std::max(gbs[q], bytes[q] * reps / (ms * 1e-3) / 1e9);
      }
    }
    return SEM_OK;
  });
}

int sem_precond(sem_mesh m, const void* r, void* z, int dtype, int pc, void* stream) {
  int st = need_device(m);
  if (st) return st;
  if (!r || !z || r == z || pc < 0 || pc > 3) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    hipStream_t s = (hipStream_t)stream;
    if (dtype == SEM_F64)
      precond<double>(m, (const double*)r, (double*)z, pc, s);
    else if (dtype == SEM_F32) {
      if (!m->fp32) throw Error{SEM_EUNSUPPORTED, "handle built without FP32 copies"};
      precond<float>(m, (const float*)r, (float*)z, pc, s);
    } else
      throw Error{SEM_EINVAL, "dtype"};
    return SEM_OK;
  });
}

int sem_coarse_solve(sem_mesh m, const double* R, double* Z, void* stream) {
  int st = need_device(m);
  if (st) return st;
  if (!R || !Z) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    hipStream_t s = (hipStream_t)stream;
    const HostTables& T = m->T;
    if (T.nc > 0) {
      hipLaunchKernelGGL(coarse_set_rhs_kernel, dim3((unsigned)blocks_for(T.nc)), dim3(kGS), 0, s, m->cvec.p, R,
                         (const int32_t*)m->rs_off.p, (const int32_t*)m->pslot.p, (const int32_t*)m->cvert.p,
                         (const int32_t*)m->vinc_off.p, T.nc);
      SEM_HIP(hipGetLastError());
      coarse_solve_tree(m, s);
    } else {
      hipLaunchKernelGGL((fill_kernel<double>), dim3(grid_stride_blocks(T.V)), dim3(kGS), 0, s, m->Zv.p, 0.0, T.V);
    }
    SEM_HIP(hipMemcpyAsync(Z, m->Zv.p, T.V * sizeof(double), hipMemcpyDeviceToDevice, s));
    return SEM_OK;
  });
}

int sem_pcg_solve(sem_mesh m, const double* b, double* x, const sem_solve_opts* o, sem_solve_stats* st,
                  void* stream) {
  int s0 = need_device(m);
  if (s0) return s0;
  if (!b || !x || b == x) return SEM_EINVAL;
  sem_solve_opts d;
  sem_default_solve_opts(&d);
  if (!o) o = &d;
  if (o->pc < 0 || o->pc > 3 || o->max_iter < 0 || !(o->rtol >= 0.0)) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    if (o->mode == SEM_SOLVE_FP32_REFINED && !m->fp32) throw Error{SEM_EUNSUPPORTED, "handle built without FP32 copies"};
    ensure_work(m, o->mode == SEM_SOLVE_FP32_REFINED);
    return solve_impl(m, b, x, o, st, (hipStream_t)stream);
  });
}

int sem_pcg_solve_noalloc(sem_mesh m, const double* b, double* x, const sem_solve_opts* o, sem_solve_stats* st,
                          void* stream) {
  if (!m) {
    set_error("NULL handle");
    return SEM_EINVAL;
  }
  if (!b || !x || b == x) return SEM_EINVAL;
  sem_solve_opts d;
  sem_default_solve_opts(&d);
  if (!o) o = &d;
  if (o->pc < 0 || o->pc > 3 || o->max_iter < 0 || !(o->rtol >= 0.0)) return SEM_EINVAL;
  const bool need32 = o->mode == SEM_SOLVE_FP32_REFINED;
  const size_t need = scratch_layout(m, need32).total;
  if (need > kScratchBytes) {
    set_error("sem_pcg_solve_noalloc: this mesh needs " + std::to_string(need) + " bytes of static scratch, more than " +
              "its maximum of " + std::to_string(kScratchBytes) + " bytes; use sem_pcg_solve");
    return SEM_EINVAL;
  }
  int s0 = need_device(m);
  if (s0) return s0;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    if (need32 && !m->fp32) throw Error{SEM_EUNSUPPORTED, "handle built without FP32 copies"};
    double* base = scratch_of(m->device);
    if (base == nullptr) throw Error{SEM_EHIP, "static scratch not resolved on this device"};
    // views into the scratch for this solve only; any lazy set-up that would
    // allocate raises instead (no_alloc); the handle's own buffers return with
    // the next sem_pcg_solve
    struct Restore {
      sem_mesh m;
      ~Restore() {
        m->no_alloc = false;
        m->wk = sem_mesh_s::SolveWork{};
      }
    } restore{m};
    m->no_alloc = true;
    scratch_work(m, need32, base);
    return solve_impl(m, b, x, o, st, (hipStream_t)stream);
  });
}

int sem_mesh_set_coefficients(sem_mesh m, double kappa, double c) {
  if (!m || !(kappa > 0.0) || !(c >= 0.0) || !std::isfinite(kappa) || !std::isfinite(c)) return SEM_EINVAL;
  return guarded([&]() -> int {
    set_coefficients(m, kappa, c);
    return SEM_OK;
  });
}

int sem_mesh_set_element_coefficients(sem_mesh m, const double* kappa, const double* c) {
  if (!m) return SEM_EINVAL;
  const int64_t E = m->T.E;
  for (int64_t e = 0; e < E; ++e) {
    if (kappa && !(kappa[e] > 0.0 && std::isfinite(kappa[e]))) return SEM_EINVAL;
    if (c && !(c[e] >= 0.0 && std::isfinite(c[e]))) return SEM_EINVAL;
  }
  return guarded([&]() -> int {
    set_element_coefficients(m, kappa, c);
    return SEM_OK;
  });
}

int sem_mesh_set_node_coefficients(sem_mesh m, const double* kappa, const double* c) {
  if (!m) return SEM_EINVAL;
  const int64_t nl = m->T.n_local;
  for (int64_t l = 0; l < nl; ++l) {
    if (kappa && !(kappa[l] > 0.0 && std::isfinite(kappa[l]))) return SEM_EINVAL;
    if (c && !(c[l] >= 0.0 && std::isfinite(c[l]))) return SEM_EINVAL;
  }
  return guarded([&]() -> int {
    set_node_coefficients(m, kappa, c);
    return SEM_OK;
  });
}

int sem_mesh_boundary_face_mass(sem_mesh m, const int64_t* faces, int64_t n_faces, double* ws) {
  if (!m || !ws || n_faces < 0 || (n_faces > 0 && !faces)) return SEM_EINVAL;
  return guarded([&]() -> int {
    boundary_face_mass(m->T, faces, n_faces, ws);
    return SEM_OK;
  });
}

int sem_mesh_set_coarse_solver(sem_mesh m, int solver) {
  if (!m || (solver != SEM_COARSE_EXACT && solver != SEM_COARSE_AMG)) return SEM_EINVAL;
  return guarded([&]() -> int {
    if (m->coarse_solver == solver) return SEM_OK;
    m->coarse_solver = solver;
    if (m->host_only) return SEM_OK;
    SEM_HIP(hipSetDevice(m->device));
    SEM_HIP(hipDeviceSynchronize());
    release_coarse_graph(m);
    if (solver == SEM_COARSE_AMG) {
      try {
        amg_setup(m);
      } catch (...) {
        m->coarse_solver = SEM_COARSE_EXACT;
        m->amg.clear();
        build_coarse_graph(m);
        throw;
      }
    } else {
      m->amg.clear();
    }
    build_coarse_graph(m);
    return SEM_OK;
  });
}

int sem_mesh_amg_hierarchy(sem_mesh m, int64_t* level_sizes, int cap, int* n_levels, int32_t* agg0) {
  if (!m || !n_levels || cap < 0 || (cap > 0 && !level_sizes)) return SEM_EINVAL;
  return guarded([&]() -> int {
    AmgHierarchy H;
    build_amg(m->T, H);
    *n_levels = (int)H.levels.size();
    for (int l = 0; l < cap && l < (int)H.levels.size(); ++l) level_sizes[l] = H.levels[l].n;
    if (agg0 && !H.levels.empty() && !H.levels[0].agg.empty())
      std::copy(H.levels[0].agg.begin(), H.levels[0].agg.end(), agg0);
    return SEM_OK;
  });
}

int sem_mesh_coefficients(sem_mesh m, double* kappa, double* c) {
  if (!m || !kappa || !c) return SEM_EINVAL;
  *kappa = m->T.kappa;
  *c = m->T.cmass;
  return SEM_OK;
}

int sem_heat_step(sem_mesh m, double kappa, double dt, const double* u_prev, const double* q, double* u_next,
                  const sem_solve_opts* o, sem_solve_stats* st, void* stream) {
  int s0 = need_device(m);
  if (s0) return s0;
  if (!u_prev || !u_next || !(dt > 0.0) || !(kappa > 0.0) || !std::isfinite(dt) || !std::isfinite(kappa))
    return SEM_EINVAL;
  if (q == u_next) return SEM_EINVAL;
  sem_solve_opts d;
  sem_default_solve_opts(&d);
  if (!o) o = &d;
  if (o->pc < 0 || o->pc > 3 || o->max_iter < 0 || !(o->rtol >= 0.0)) return SEM_EINVAL;
  return guarded([&]() -> int {
    SEM_HIP(hipSetDevice(m->device));
    hipStream_t s = (hipStream_t)stream;
    set_coefficients(m, kappa, 1.0 / dt);
    const int64_t n = m->T.n_global;
    if (m->hb.n < (size_t)n) m->hb.alloc(n);
    hipLaunchKernelGGL(heat_rhs_kernel, dim3((unsigned)blocks_for(n)), dim3(kGS), 0, s, m->hb.p, u_prev, q,
                       m->mN64.p, m->dir.p, dt, n);
    SEM_HIP(hipGetLastError());
    if (u_next != u_prev) SEM_HIP(hipMemcpyAsync(u_next, u_prev, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    sem_solve_opts oo = *o;
    oo.use_x0 = 1;
    if (oo.mode == SEM_SOLVE_FP32_REFINED && !m->fp32) throw Error{SEM_EUNSUPPORTED, "handle built without FP32 copies"};
    ensure_work(m, oo.mode == SEM_SOLVE_FP32_REFINED);
    return solve_impl(m, m->hb.p, u_next, &oo, st, s);
  });
}

}  // extern "C"
