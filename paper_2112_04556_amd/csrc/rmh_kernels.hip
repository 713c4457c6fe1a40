// HIP kernels for gfx950 besides the stencil: layout conversion, element-wise kernels with
// deterministic reductions, the multi-shift CG vector and scalar kernels, mixed-precision
// reliable updates, and the link-derivative (force) kernel.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rmh_internal.h"
#include "rmh_reduce.h"

namespace rmh {

// ------------------------------------------------------------------------------------------
// element-wise helpers

int64_t field_reals(const Geom& g) { return 32 * (int64_t)g.V; }
int elem_num_blocks(int64_t n_reals) { return (int)((n_reals / 4 + kBlock - 1) / kBlock); }
int red_steps(int64_t n_reals) {
  const int64_t s = n_reals / (4LL * kBlock * 2048);   // keep at least ~2048 blocks
  return (int)std::max<int64_t>(1, std::min<int64_t>(8, s));
}
int red_num_blocks(int64_t n_reals) {
  const int64_t c = 4LL * kBlock * red_steps(n_reals);
  return (int)((n_reals + c - 1) / c);
}

template <typename T>
__global__ void k_dot(const T* __restrict__ a, const T* __restrict__ b, int64_t n, int32_t steps, double* partials) {
  const int32_t v = blockIdx.y;
  const T* av = a + (int64_t)v * n;
  const T* bv = b + (int64_t)v * n;
  double d[1] = {0.0};
  for (int32_t t = 0; t < steps; ++t) {
    const int64_t i0 = (((int64_t)blockIdx.x * steps + t) * blockDim.x + threadIdx.x) * 4;
    if (i0 < n) {
#pragma unroll
      for (int k = 0; k < 4; ++k) d[0] = fma((double)av[i0 + k], (double)bv[i0 + k], d[0]);
    }
  }
  __shared__ double lds[1][16];
  block_sum<1>(d, lds);
  if (threadIdx.x == 0) partials[(int64_t)v * gridDim.x + blockIdx.x] = d[0];
}

template <typename T>
hipError_t launch_dot(const T* a, const T* b, int64_t n_reals, int32_t n, double* partials, hipStream_t s) {
  if (n == 0) return hipSuccess;
  dim3 grid(red_num_blocks(n_reals), n);
  hipLaunchKernelGGL((k_dot<T>), grid, dim3(kBlock), 0, s, a, b, n_reals, red_steps(n_reals), partials);
  return hipGetLastError();
}
template hipError_t launch_dot<double>(const double*, const double*, int64_t, int32_t, double*, hipStream_t);
template hipError_t launch_dot<float>(const float*, const float*, int64_t, int32_t, double*, hipStream_t);

__global__ void k_reduce_rows(const double* partials, int32_t nblk, double* sums) {
  __shared__ double lds[1][16];
  const double v = block_sum_array(partials + (int64_t)blockIdx.x * nblk, nblk, lds);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

hipError_t launch_reduce_rows(const double* partials, int32_t nblk, int32_t m, double* sums, hipStream_t s) {
  if (m == 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_rows, dim3(m), dim3(kRedBlock), 0, s, partials, nblk, sums);
  return hipGetLastError();
}

// Fills stride over the grid: a launch holds fewer than 2^32 threads, and buffers of 16 GiB and
// more (a batch of FP64 link fields at 32^3 x 64) have more 4-byte words than that.
static unsigned fill_blocks(int64_t n) { return (unsigned)std::min<int64_t>((n + kBlock - 1) / kBlock, 1 << 20); }

__global__ void k_zero(uint32_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
  // every buffer is carved at 256-byte granularity, so bytes is a multiple of 4
  const int64_t n = (int64_t)(bytes / 4);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero, dim3(fill_blocks(n)), dim3(kBlock), 0, s, (uint32_t*)p, n);
  return hipGetLastError();
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(fill_blocks(n)), dim3(kBlock), 0, s, p, v, n);
  return hipGetLastError();
}

template <typename TI, typename TO>
__global__ void k_cast(const TI* __restrict__ in, TO* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (TO)in[i];  // FP64 -> FP32 rounds to nearest even
}

hipError_t launch_f64_to_f32(const double* in, float* out, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((k_cast<double, float>), dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     in, out, n);
  return hipGetLastError();
}
hipError_t launch_f32_to_f64(const float* in, double* out, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((k_cast<float, double>), dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     in, out, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_copy_cast(const double* in, T* out, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((k_cast<double, T>), dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, in,
                     out, n);
  return hipGetLastError();
}
template hipError_t launch_copy_cast<double>(const double*, double*, int64_t, hipStream_t);
template hipError_t launch_copy_cast<float>(const double*, float*, int64_t, hipStream_t);

__global__ void k_add(double* __restrict__ x, const double* __restrict__ e, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] += e[i];
}
hipError_t launch_add(double* x, const double* e, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_add, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, x, e, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// layout conversion (bitwise: pure data movement plus FP64 -> FP32 round to nearest even)

template <typename T>
__global__ void k_pack_links(Geom g, const double* __restrict__ aos, T* __restrict__ soa) {
  const int32_t mu = blockIdx.y;
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const double* src = aos + ((int64_t)mu * g.V + s) * 18;
#pragma unroll
  for (int c = 0; c < 18; ++c) soa[((int64_t)mu * 18 + c) * g.V + s] = (T)src[c];
}

__global__ void k_unpack_links(Geom g, const double* __restrict__ soa, double* __restrict__ aos) {
  const int32_t mu = blockIdx.y;
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  double* dst = aos + ((int64_t)mu * g.V + s) * 18;
#pragma unroll
  for (int c = 0; c < 18; ++c) dst[c] = soa[((int64_t)mu * 18 + c) * g.V + s];
}

hipError_t launch_pack_links(const Geom& g, const double* aos, void* soa, int dtype, hipStream_t s) {
  dim3 grid((g.V + kBlock - 1) / kBlock, 4);
  if (dtype == 0)
    hipLaunchKernelGGL((k_pack_links<double>), grid, dim3(kBlock), 0, s, g, aos, (double*)soa);
  else
    hipLaunchKernelGGL((k_pack_links<float>), grid, dim3(kBlock), 0, s, g, aos, (float*)soa);
  return hipGetLastError();
}

hipError_t launch_unpack_links(const Geom& g, const double* soa, double* aos, hipStream_t s) {
  dim3 grid((g.V + kBlock - 1) / kBlock, 4);
  hipLaunchKernelGGL(k_unpack_links, grid, dim3(kBlock), 0, s, g, soa, aos);
  return hipGetLastError();
}

// fields: AoS [n][V][4][8]  <->  SoA [n][4][8][V]
template <typename T>
__global__ void k_fields_aos_to_soa(Geom g, const double* __restrict__ aos, T* __restrict__ soa) {
  const int32_t n = blockIdx.y;
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const double* src = aos + ((int64_t)n * g.V + s) * 32;
  T* dst = soa + (int64_t)n * 32 * g.V;
#pragma unroll
  for (int c = 0; c < 32; ++c) dst[(int64_t)c * g.V + s] = (T)src[c];
}

template <typename T>
__global__ void k_fields_soa_to_aos(Geom g, const T* __restrict__ soa, double* __restrict__ aos) {
  const int32_t n = blockIdx.y;
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  double* dst = aos + ((int64_t)n * g.V + s) * 32;
  const T* src = soa + (int64_t)n * 32 * g.V;
#pragma unroll
  for (int c = 0; c < 32; ++c) dst[c] = (double)src[(int64_t)c * g.V + s];
}

hipError_t launch_fields_aos_to_soa(const Geom& g, int32_t n, const double* aos, void* soa, int dtype,
                                    hipStream_t s) {
  if (n == 0) return hipSuccess;
  dim3 grid((g.V + kBlock - 1) / kBlock, n);
  if (dtype == 0)
    hipLaunchKernelGGL((k_fields_aos_to_soa<double>), grid, dim3(kBlock), 0, s, g, aos, (double*)soa);
  else
    hipLaunchKernelGGL((k_fields_aos_to_soa<float>), grid, dim3(kBlock), 0, s, g, aos, (float*)soa);
  return hipGetLastError();
}

hipError_t launch_fields_soa_to_aos(const Geom& g, int32_t n, const void* soa, int dtype, double* aos,
                                    hipStream_t s) {
  if (n == 0) return hipSuccess;
  dim3 grid((g.V + kBlock - 1) / kBlock, n);
  if (dtype == 0)
    hipLaunchKernelGGL((k_fields_soa_to_aos<double>), grid, dim3(kBlock), 0, s, g, (const double*)soa, aos);
  else
    hipLaunchKernelGGL((k_fields_soa_to_aos<float>), grid, dim3(kBlock), 0, s, g, (const float*)soa, aos);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// multi-shift CG (Jegerlehner's shifted recurrences on a seed system; every shift's
// residual is zeta_j times the seed residual)

__global__ void k_cg_init(CgDev cg, const double* bn2_part, int32_t nblk, const double* tol_rel, double delta,
                          int32_t maxiter, int32_t fp32_start) {
  __shared__ double lds[1][16];
  const int32_t v = blockIdx.x;
  const double bn2 = block_sum_array(bn2_part + (int64_t)v * nblk, nblk, lds);
  __shared__ double s_bn2;
  if (threadIdx.x == 0) {
    double* sc = cg.sc + (int64_t)v * kScN;
    int32_t* fl = cg.flags + (int64_t)v * kFlN;
    sc[kScRR] = bn2;
    sc[kScBnorm2] = bn2;
    sc[kScAlphaPrev] = 1.0;
    sc[kScBetaPrev] = 0.0;
    sc[kScMaxR] = sqrt(bn2);
    sc[kScTolAbs] = tol_rel[v] * sqrt(bn2);
    sc[kScIters] = 0.0;
    sc[kScRU] = 0.0;
    sc[kScDelta] = delta;
    sc[kScMaxIter] = (double)maxiter;
    sc[kScZMax] = 1.0;
    fl[kFlRun] = (bn2 > 0.0) ? 1 : 0;
    fl[kFlStatus] = (bn2 == bn2) ? kStOk : kStBreakdown;   // NaN source
    if (!(bn2 == bn2)) fl[kFlRun] = 0;
    fl[kFlNeedRU] = 0;
    fl[kFlSum] = 0;
    fl[kFlDefer] = 0;
    fl[kFlBase] = 0;
    fl[kFlM] = 0;
    fl[kFlK64] = fp32_start ? 0 : kAllFp64;
    fl[kFlK0] = 0;
    fl[kFlBase32] = 0;
    s_bn2 = bn2;
  }
  __syncthreads();
  const int32_t nc = 2 + 2 * cg.cslots;
  for (int j = threadIdx.x; j < cg.n_shift; j += blockDim.x) {
    const int64_t vj = (int64_t)v * cg.n_shift + j;
    double* sh = cg.sh + vj * kShN;
    sh[kShZeta] = 1.0;
    sh[kShZetaPrev] = 1.0;
    sh[kShSeg] = 0.0;
    // x_j = 0, p_j = b = ring slot 0
    double* cf = cg.coef + vj * nc;
    for (int i = 0; i < nc; ++i) cf[i] = 0.0;
    cf[2 + cg.cslots] = 1.0;
    const int32_t on = (s_bn2 > 0.0) ? 1 : 0;
    cg.act[vj] = on;
    cg.act_next[vj] = on;
  }
}

hipError_t launch_cg_init(const CgDev& cg, const double* bn2_partials, int32_t nblk, const double* tol_rel,
                          double delta, int32_t maxiter, int32_t fp32_start, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_init, dim3(cg.n_rhs), dim3(kRedBlock), 0, s, cg, bn2_partials, nblk, tol_rel, delta,
                     maxiter, fp32_start);
  return hipGetLastError();
}

// One iteration is two launches: the stencil (Ap and the partials of <r, Ap>, <p, Ap>, <Ap, Ap>) and the
// update of r and p.  beta = <r', r'> / <r, r> needs the norm of a residual that the same launch computes;
// it is taken from <r', r'> = <r, r> - 2 alpha <r, Ap> + alpha^2 <Ap, Ap>, which holds for the vectors at
// hand whatever their conjugacy (a form without <r, Ap>, which the exact recurrences would allow, doubles
// its error every iteration).  r is the residual that this update takes: after a reliable update the FP64 one,
// which the stencil's dot then reads too (with the recursive one there, solves that reach FP32's digits in a
// few iterations broke down).  The residual that was computed gives alpha and the next prediction their <r, r>,
// so a prediction's rounding, a few ulps of <r, r>, is not handed on.  Where <r', r'> comes out below
// 1e-4 <r, r> more than four digits have cancelled: convergence is then decided by the next update from the
// sum (Defer), until then the norm counts as 1e-2 |r|, and mixed solves take a reliable update, which a smaller
// delta would ask for on the true norm (one iteration later the two residuals have parted, and solves broke down).
// Against residual and direction updates of their own, which read r' and p again (16^4, one field: 11.8 and
// 11.0 us; 12^4: 6.9 and 7.8), one pass over five streams takes 17.5 and 10.6 us, and the stencil 1 us more.
//
// Every block sums the partials itself (the same values in the same order, so every block gets the same
// bits) instead of waiting for a scalar kernel; the last block of each rhs carries out the scalar state and
// the shift coefficients meanwhile, into the other copy of the state, so no launch writes what its other
// blocks read.

// One array of partials, p[0, n): this thread's first four, loaded without a wait or a branch, so that the
// loads of all arrays, and the vectors' after them, are in flight together.
struct CgPart {
  const double* p;
  int32_t n;
  double t[4];
  __device__ __forceinline__ CgPart(const double* p_, int32_t n_) : p(p_), n(n_) {
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = p[min((int32_t)(threadIdx.x + k * blockDim.x), max(n - 1, 0))];
  }
  // this thread's part of the fixed-order sum
  __device__ __forceinline__ double sum() const {
    const int32_t B = blockDim.x;
    double a = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) a += (int32_t)threadIdx.x + k * B < n ? t[k] : 0.0;
    for (int32_t i = threadIdx.x + 4 * B; i < n; i += B) a += p[i];
    return a;
  }
};

// The scalars of an iteration.
struct CgStep {
  double rr, alpha;    // <r, r> the iteration starts from, and its step
  double rrn, beta;    // <r', r'> (predicted: at least 1e-4 rr) and the direction's coefficient
  double maxr;         // largest residual norm since the last reliable update
  bool done, ok;       // converged (or at its iteration limit) before this iteration; no breakdown
  bool defer, need_ru;
};

// The partials an update reads.  kNext: <r', r'> is the sum of nnew partials in part_e_next, else predicted
// (unused by the launch that writes them).  With ru the residual is the FP64 one of a reliable update issued at the end of the
// previous iteration (r64 = b - (Delta + sigma0) x_seed), which replaces the recursive residual from now on
template <bool kNext>
struct CgParts {
  CgPart pAp, rr, a, b;   // a, b: <r', r'> and nothing, or <r, Ap> and <Ap, Ap>
  __device__ __forceinline__ CgParts(const CgDev& cg, int32_t v, bool ru, int32_t sum, int32_t nnew)
      : CgParts(cg, cg.part + (int64_t)v * 3 * cg.nblk_hop, v, ru, sum, nnew) {}

 private:
  __device__ __forceinline__ CgParts(const CgDev& cg, const double* part, int32_t v, bool ru, int32_t sum, int32_t nnew)
      : pAp(part + cg.nblk_hop, cg.nblk_hop),
        rr(ru ? cg.part_ru + ((int64_t)v * 3 + 2) * cg.nblk_ru : cg.part_e + (int64_t)v * cg.nblk_e,
           ru ? cg.nblk_ru : sum),
        a(kNext ? cg.part_e_next + (int64_t)v * cg.nblk_e : part, kNext ? nnew : cg.nblk_hop),
        b(kNext ? part : part + 2 * (int64_t)cg.nblk_hop, kNext ? 0 : cg.nblk_hop) {}
};

template <bool kNext>
__device__ __forceinline__ CgStep cg_scalars(const CgDev& cg, int32_t v, bool ru, int32_t mixed,
                                             const CgParts<kNext>& pt, double (*lds)[16]) {
  const int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const double* sc = cg.sc + (int64_t)v * kScN;
  const int32_t sum = fl[kFlSum];
  double q[4] = {pt.pAp.sum(), pt.rr.sum(), pt.a.sum(), pt.b.sum()};
  block_sum_all<4>(q, lds);
  const double pAp = q[0];
  CgStep r;
  r.rr = ru || sum ? q[1] : sc[kScRR];
  r.done = fl[kFlDefer] != 0 &&
           (sc[kScZMax] * sqrt(r.rr) <= sc[kScTolAbs] || sc[kScIters] >= sc[kScMaxIter]);
  r.alpha = r.rr / pAp;
  r.ok = pAp > 0.0 && r.alpha == r.alpha && r.alpha < 1e300;
  const double rrn = kNext ? q[2] : fma(r.alpha, fma(r.alpha, q[3], -2.0 * q[2]), r.rr);
  r.defer = !kNext && rrn < 1e-4 * r.rr;
  r.beta = (rrn < 0.0 ? 0.0 : rrn) / r.rr;
  r.rrn = r.defer ? 1e-4 * r.rr : rrn;
  // a reliable update once the residual norm fell below delta times its largest value since the last one, or further
  // than the prediction tells
  r.maxr = ru ? sqrt(r.rr) : sc[kScMaxR];
  const double rnorm = sqrt(r.rrn);
  r.need_ru = mixed && (r.defer || rnorm < sc[kScDelta] * (rnorm > r.maxr ? rnorm : r.maxr));
  return r;
}

// The scalar side of the update (one block per rhs).  zeta_{k+1}^j, the x-update coefficient and the
// p-update coefficients of every active shift, applied to the segment coefficients of the non-seed shifts:
// x_j += cx_j p_j, then p_j = cr_j r' + cp_j p_j; convergence and freezing; the new residual becomes the
// current ring entry
__device__ __forceinline__ void cg_state(const CgDev& cg, int32_t v, bool ru, int32_t mixed, int32_t nsum,
                                         const CgStep& it) {
  const int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const double* sc = cg.sc + (int64_t)v * kScN;
  int32_t* fn = cg.flags_next + (int64_t)v * kFlN;
  double* sn = cg.sc_next + (int64_t)v * kScN;
  const int32_t ns = cg.n_shift;
  const int32_t nc = 2 + 2 * cg.cslots;
  const int32_t tid = threadIdx.x;
  const int32_t m = fl[kFlM];
  const int32_t seed = cg.seed[v];
  if (it.done || !it.ok) {
    if (tid == 0) {
      fn[kFlRun] = 0;
      fn[kFlNeedRU] = 0;
      const bool conv = it.done && sc[kScZMax] * sqrt(it.rr) <= sc[kScTolAbs];
      if (it.done && !conv) fn[kFlStatus] = kStNoConv;
      if (!it.done) fn[kFlStatus] = kStBreakdown;
    }
    return;
  }
  const double ap = sc[kScAlphaPrev], bp = sc[kScBetaPrev];
  const double alpha = it.alpha, beta = it.beta;
  const double tolabs = sc[kScTolAbs];
  const double rnorm = sqrt(it.rrn);
  __shared__ double s_cx[kMaxShifts], s_cp[kMaxShifts], s_cr[kMaxShifts], s_z[kMaxShifts];
  __shared__ int s_ux[kMaxShifts], s_up[kMaxShifts];   // coefficients updated
  __shared__ int s_seed_act, s_seed_keep;              // the seed's act and act_next, for thread 0
  const double s0 = cg.sigma[(int64_t)v * ns + seed];
  int any_other = 0;
  if (tid < ns) {
    const int64_t vj = (int64_t)v * ns + tid;
    const int32_t on = cg.act_next[vj];
    double* sh = cg.sh + vj * kShN;
    cg.act[vj] = on;
    int ux = 0, up = 0, keep = 0;
    double zn = 0.0;
    if (on) {
      const double z = sh[kShZeta], zp = sh[kShZetaPrev];
      const double ds = cg.sigma[vj] - s0;
      zn = z * zp * ap / (ap * zp * (1.0 + alpha * ds) + alpha * bp * (zp - z));
      const double ratio = zn / z;
      const double cx = alpha * zn / z;
      const bool in_ring = cg.ring_on && !(cg.seed_explicit && tid == seed);
      ux = in_ring && m < cg.nslot ? 1 : 0;
      if (ux) sh[kShSeg] = 1.0;
      s_cx[tid] = cx;
      s_cr[tid] = zn;
      s_cp[tid] = beta * ratio * ratio;
      keep = (fabs(zn) * rnorm > tolabs) ? 1 : 0;
      if (tid != seed) any_other |= keep;
      up = in_ring && keep && m + 1 < cg.nslot ? 1 : 0;
      sh[kShZetaPrev] = z;
      sh[kShZeta] = zn;
    }
    cg.act_next[vj] = keep;
    s_z[tid] = keep || tid == seed ? fabs(zn) : 0.0;
    if (tid == seed) {
      s_seed_act = on;
      s_seed_keep = keep;
    }
    s_ux[tid] = ux;
    s_up[tid] = up;
  }
  any_other = __syncthreads_or(any_other);
  if (tid == 0) {
    const int64_t vs = (int64_t)v * ns + seed;
    int32_t seed_next = s_seed_keep;
    if (any_other && !seed_next && s_seed_act) {
      // the seed carries the Krylov space for the others: its direction keeps being updated
      if (cg.ring_on && !cg.seed_explicit && m + 1 < cg.nslot) s_up[seed] = 1;
    }
    if (any_other) seed_next = 1;
    if (seed_next != s_seed_keep) cg.act_next[vs] = seed_next;
    const int32_t any = any_other | seed_next;
    const double iters = sc[kScIters] + 1.0;
    double zmax = 0.0;
    for (int j = 0; j < ns; ++j) zmax = s_z[j] > zmax ? s_z[j] : zmax;
    if (ru) sn[kScRU] = sc[kScRU] + 1.0;
    sn[kScAlphaPrev] = alpha;
    sn[kScBetaPrev] = beta;
    sn[kScRR] = it.rrn;
    sn[kScIters] = iters;
    sn[kScZMax] = zmax;
    if (mixed) sn[kScMaxR] = rnorm > it.maxr ? rnorm : it.maxr;
    fn[kFlM] = m + 1;
    fn[kFlSum] = nsum;
    fn[kFlDefer] = it.defer && any ? 1 : 0;
    fn[kFlNeedRU] = it.need_ru ? 1 : 0;
    if (!(it.rrn == it.rrn)) {
      fn[kFlStatus] = kStBreakdown;
      fn[kFlRun] = 0;
    } else if (!any) {
      fn[kFlRun] = 0;
    } else if (iters >= sc[kScMaxIter] && !it.defer) {
      fn[kFlStatus] = kStNoConv;
      fn[kFlRun] = 0;
    }
  }
  __syncthreads();
  // One (shift, coefficient) pair per thread and round.  The pairs: q = 0 the p_j0 coefficient (x_j0 += cx p_j0,
  // then scaled by cp), q = 1 + i the ring entry i <= m (d_ji += cx e_ji, e_ji scaled by cp), q = m + 2 the new
  // entry m + 1 (e set to cr).  x is updated only while m < nslot <= cslots, p while m + 1 < nslot; past that
  // (a single shift's segment index grows without flushes) the pairs stop at the last coefficient slot
  const int32_t per = min(m, cg.cslots - 1) + 3;
  for (int t = tid; t < ns * per; t += blockDim.x) {
    const int32_t jj = t / per, q = t - jj * per;
    double* cf = cg.coef + ((int64_t)v * ns + jj) * nc;
    double* e = cf + 2 + cg.cslots;
    if (q == m + 2) {
      if (s_up[jj]) e[m + 1] = s_cr[jj];
      continue;
    }
    double* pc = q == 0 ? cf + 1 : e + (q - 1);
    double* xc = q == 0 ? cf : cf + 1 + q;
    if (q - 1 >= cg.cslots) continue;
    if (s_ux[jj]) *xc = fma(s_cx[jj], *pc, *xc);
    if (s_up[jj]) *pc *= s_cp[jj];
  }
}

// ring slot i of rhs v in a ring region of rhs_bytes per rhs, viewed as T (slots of n_reals)
template <typename T>
__device__ __forceinline__ T* ring_slot(const void* ring, int64_t rhs_bytes, int32_t v, int32_t i, int64_t n) {
  return (T*)((char*)ring + (int64_t)v * rhs_bytes + (int64_t)i * n * (int64_t)sizeof(T));
}

// segment entry i of rhs v: in the FP64 ring from the segment's FP64 base slot, or in the FP32
// ring counted from entry k0, which sits in FP32 slot base32
__device__ __forceinline__ double* entry64(const CgDev& cg, int32_t v, int32_t base, int32_t i, int64_t n) {
  return ring_slot<double>(cg.ring64, cg.rb64, v, (base + i) % cg.nslot64, n);
}
__device__ __forceinline__ float* entry32(const CgDev& cg, int32_t v, int32_t base32, int32_t k0, int32_t i,
                                          int64_t n) {
  return ring_slot<float>(cg.ring32, cg.rb32, v, (base32 + i - k0) % cg.nslot32, n);
}
// entry i of the phase whose arithmetic type is T (the FP32 phase only touches entries >= k0)
template <typename T>
__device__ __forceinline__ T* entry(const CgDev& cg, int32_t v, const int32_t* st, int32_t i, int64_t n) {
  if constexpr (sizeof(T) == 8)
    return entry64(cg, v, st[0], i, n);
  else
    return entry32(cg, v, st[1], st[2], i, n);
}

template <typename T>
__global__ void k_cg_start(const double* __restrict__ b, void* ring, T* __restrict__ p, int64_t rhs_bytes,
                           int64_t n) {
  const int32_t v = blockIdx.y;
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
  T* r0 = ring_slot<T>(ring, rhs_bytes, v, 0, n);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const T x = (T)b[(int64_t)v * n + i0 + k];
    r0[i0 + k] = x;
    p[(int64_t)v * n + i0 + k] = x;
  }
}

template <typename T>
hipError_t launch_cg_start(const double* b, void* ring, T* p, int32_t nr, int64_t rhs_bytes, int64_t n_reals,
                           hipStream_t s) {
  if (nr == 0) return hipSuccess;
  dim3 grid(elem_num_blocks(n_reals), nr);
  hipLaunchKernelGGL((k_cg_start<T>), grid, dim3(kBlock), 0, s, b, ring, p, rhs_bytes, n_reals);
  return hipGetLastError();
}
template hipError_t launch_cg_start<double>(const double*, void*, double*, int32_t, int64_t, int64_t, hipStream_t);
template hipError_t launch_cg_start<float>(const double*, void*, float*, int32_t, int64_t, int64_t, hipStream_t);

// The update takes its vectors in pieces of 16 bytes per lane, consecutive lanes consecutive pieces: a block
// covers kCgChunk reals per step, all loads of a step in flight together, in enough steps that at most 1024
// blocks and as many partials remain per rhs.  Blocks of 1024 threads on as few partials are slower (21.1 us
// against 18.2 at 16^4, 16.9 against 11.8 at 12^4, before the block sums were rewritten): they start and
// stop together.
constexpr int kCgChunk = 2048;
static int cg_steps(int64_t n_reals) { return (int)std::max<int64_t>(1, n_reals / ((int64_t)kCgChunk * 1024)); }
int cg_num_blocks(int64_t n_reals) {
  const int64_t c = (int64_t)kCgChunk * cg_steps(n_reals);
  return (int)((n_reals + c - 1) / c);
}
template <typename T>
using Piece = T __attribute__((ext_vector_type(16 / sizeof(T))));

// the last block of a rhs: a copy of the state, to be changed by cg_state after a barrier
__device__ __forceinline__ void cg_state_copy(const CgDev& cg, int32_t v) {
  if (threadIdx.x < kScN) cg.sc_next[(int64_t)v * kScN + threadIdx.x] = cg.sc[(int64_t)v * kScN + threadIdx.x];
  if (threadIdx.x >= 64 && threadIdx.x < 64 + kFlN) {
    const int32_t i = threadIdx.x - 64;
    cg.flags_next[(int64_t)v * kFlN + i] = i == kFlNeedRU ? 0 : cg.flags[(int64_t)v * kFlN + i];
  }
}

// One launch of the update; PART 0: all of it, 1: alpha and r' alone, 2: beta, p, the seed's solution and the
// state (launch_cg_step2).
template <typename T, int PART>
__global__ void __launch_bounds__(256) k_cg_step(CgDev cg, const T* __restrict__ Ap, T* __restrict__ p,
                                                      float* __restrict__ x_lo, double* __restrict__ x_hi,
                                                      const double* __restrict__ r64, int64_t n, int32_t steps,
                                                      int32_t mixed, int32_t nsum) {
  constexpr int N = 16 / sizeof(T), U = kCgChunk / (256 * N);
  constexpr bool R = PART != 2, P = PART != 1;   // the residual, the direction
  __shared__ double lds[4][16], lds_r[1][16];
  const int32_t v = blockIdx.y;
  const int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const bool run = fl[kFlRun] != 0;
  const bool ru = cg.part_ru && fl[kFlNeedRU] != 0;
  const int32_t m = fl[kFlM], sum = fl[kFlSum];
  const int32_t st[3] = {fl[kFlBase], fl[kFlBase32], fl[kFlK0]};
  if (P && blockIdx.x + 1 == gridDim.x) {
    cg_state_copy(cg, v);
    if (!run) return;
    const CgParts<PART == 2> pt(cg, v, ru, sum, nsum);
    const CgStep it = cg_scalars<PART == 2>(cg, v, ru, mixed, pt, lds);
    cg_state(cg, v, ru, mixed, nsum, it);
    return;
  }
  if (!run) return;
  const T* rc = R ? entry<T>(cg, v, st, m, n) : nullptr;
  T* rn = entry<T>(cg, v, st, m + 1, n);
  const T* av = Ap + (int64_t)v * n;
  T* pv = p + (int64_t)v * n;
  const double* r64v = r64 ? r64 + (int64_t)v * n : nullptr;
  const bool from64 = r64 && ru;
  Piece<T> r4[U], a4[U], p4[U];
  auto load = [&](int64_t i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + (int64_t)u * 256 * N;
      if (i >= n) break;
      if (!R) {
        r4[u] = *(const Piece<T>*)(rn + i);
      } else if (from64) {
#pragma unroll
        for (int k = 0; k < N; ++k) r4[u][k] = (T)r64v[i + k];
      } else {
        r4[u] = *(const Piece<T>*)(rc + i);
      }
      if (R) a4[u] = *(const Piece<T>*)(av + i);
      if (P) p4[u] = *(const Piece<T>*)(pv + i);
    }
  };
  const int64_t b0 = (int64_t)blockIdx.x * steps * kCgChunk + threadIdx.x * N;
  const CgParts<PART == 2> pt(cg, v, ru, sum, nsum);
  load(b0);   // in flight while the partials are summed
  const CgStep it = cg_scalars<PART == 2>(cg, v, ru, mixed, pt, lds);
  if (it.done || !it.ok) return;
  const T alpha = (T)it.alpha, beta = (T)it.beta;
  float* xl = x_lo ? x_lo + (int64_t)v * n : nullptr;
  // with a reliable update due the seed's increment goes into its FP64 solution now (x_hi[seed] += x_lo,
  // x_lo = 0), ahead of the update's FP64 residual stencil
  double* xh = x_hi && (!x_lo || it.need_ru) ? x_hi + ((int64_t)v * cg.n_shift + cg.seed[v]) * n : nullptr;
  double d[1] = {0.0};
  for (int32_t t = 0; t < steps; ++t) {
    const int64_t i0 = b0 + (int64_t)t * kCgChunk;
    if (t > 0) load(i0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + (int64_t)u * 256 * N;
      if (i >= n) break;
      Piece<T> r1 = r4[u];
      if (R) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
          r1[k] = fmadd(-alpha, a4[u][k], r4[u][k]);
          d[0] = fma((double)r1[k], (double)r1[k], d[0]);
        }
        *(Piece<T>*)(rn + i) = r1;
      }
      if (!P) continue;
      Piece<T> p1;
#pragma unroll
      for (int k = 0; k < N; ++k) p1[k] = fmadd(beta, p4[u][k], r1[k]);
      *(Piece<T>*)(pv + i) = p1;
      if (sizeof(T) == 8) {
        if (xh) {
#pragma unroll
          for (int k = 0; k < N; ++k) xh[i + k] = fma(it.alpha, (double)p4[u][k], xh[i + k]);
        }
      } else {
        // the seed's increment of this iteration, alpha p, in FP32 until the next reliable update
        Piece<float> inc = *(const Piece<float>*)(xl + i);
#pragma unroll
        for (int k = 0; k < N; ++k) inc[k & 3] = fmaf((float)alpha, (float)p4[u][k], inc[k & 3]);
        if (xh) {
#pragma unroll
          for (int k = 0; k < N; ++k) {
            xh[i + k] += (double)inc[k & 3];
            inc[k & 3] = 0.0f;
          }
        }
        *(Piece<float>*)(xl + i) = inc;
      }
    }
  }
  if (R) {
    block_sum<1>(d, lds_r);
    if (threadIdx.x == 0) cg.part_e_next[(int64_t)v * cg.nblk_e + blockIdx.x] = d[0];
  }
}

template <typename T, int PART>
static hipError_t launch_cg_part(const CgDev& cg, const T* Ap, T* p, float* x_lo, double* x_hi, const double* r64,
                                 int32_t mixed, int64_t n_reals, hipStream_t s) {
  const int32_t nblk = cg_num_blocks(n_reals);
  if (cg.n_shift > kMaxShifts || cg.nblk_e < nblk) return hipErrorInvalidValue;
  if (sizeof(T) == 4 && (!cg.ring32 || !x_lo)) return hipErrorInvalidValue;
  dim3 grid(nblk + (PART == 1 ? 0 : 1), cg.n_rhs);
  hipLaunchKernelGGL((k_cg_step<T, PART>), grid, dim3(256), 0, s, cg, Ap, p, x_lo, x_hi, r64, n_reals,
                     cg_steps(n_reals), mixed, nblk);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_cg_step(const CgDev& cg, const T* Ap, T* p, float* x_lo, double* x_hi, const double* r64,
                          int32_t mixed, int64_t n_reals, hipStream_t s) {
  return launch_cg_part<T, 0>(cg, Ap, p, x_lo, x_hi, r64, mixed, n_reals, s);
}
template <typename T>
hipError_t launch_cg_step2(const CgDev& cg, const T* Ap, T* p, float* x_lo, double* x_hi, const double* r64,
                           int32_t mixed, int64_t n_reals, hipStream_t s) {
  const hipError_t e = launch_cg_part<T, 1>(cg, Ap, p, x_lo, x_hi, r64, mixed, n_reals, s);
  return e != hipSuccess ? e : launch_cg_part<T, 2>(cg, Ap, p, x_lo, x_hi, r64, mixed, n_reals, s);
}
#define RMH_CG(T)                                                                                                   \
  template hipError_t launch_cg_step<T>(const CgDev&, const T*, T*, float*, double*, const double*, int32_t, int64_t, \
                                        hipStream_t);                                                              \
  template hipError_t launch_cg_step2<T>(const CgDev&, const T*, T*, float*, double*, const double*, int32_t, int64_t, \
                                         hipStream_t);
RMH_CG(double)
RMH_CG(float)
#undef RMH_CG

// x_hi[seed] += x_lo, x_lo = 0, at the end of an FP32 phase
__global__ void k_cg_xfold(CgDev cg, float* __restrict__ x_lo, double* __restrict__ x_hi, int64_t n) {
  const int32_t v = blockIdx.y;
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
  float* xl = x_lo + (int64_t)v * n;
  double* xh = x_hi + ((int64_t)v * cg.n_shift + cg.seed[v]) * n;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    xh[i0 + k] += (double)xl[i0 + k];
    xl[i0 + k] = 0.0f;
  }
}

hipError_t launch_cg_xfold(const CgDev& cg, float* x_lo, double* x_hi, int64_t n_reals, hipStream_t s) {
  dim3 grid(elem_num_blocks(n_reals), cg.n_rhs);
  hipLaunchKernelGGL(k_cg_xfold, grid, dim3(kBlock), 0, s, cg, x_lo, x_hi, n_reals);
  return hipGetLastError();
}

// s + sum of c_i r_i over i <= m, in groups of eight (entries past m carry zero coefficients)
template <int NS>
__device__ __forceinline__ double fold(const double* __restrict__ c, const double (&r)[NS], int32_t m, double s) {
  double t[4] = {s, 0.0, 0.0, 0.0};
#pragma unroll
  for (int g = 0; g < NS; g += 8)
    if (g <= m) {
#pragma unroll
      for (int i = g; i < g + 8 && i < NS; ++i) t[i & 3] = fma(c[i], r[i], t[i & 3]);
    }
  return (t[0] + t[1]) + (t[2] + t[3]);
}

// One element per thread: the segment's residuals at this element are loaded once and every
// non-seed shift touched in the segment is folded from registers (seed_only: the seed alone,
// its solution only).  F32: an FP32-phase segment, whose entries from K64 on are FP32 (those
// below K64, in the segment that spans the switch of precision, are FP64).  NS: the entries a thread
// holds (33, or 48 for the long segments of small lattices).  They are loaded eight at a time, each
// group without conditions so that its loads overlap: entries past the segment's end re-read an
// existing one (a cache hit) against coefficients that are zero.  The coefficients are the same for a
// whole block and come through the scalar cache into scalar registers (read from LDS, with a branch
// per entry, the 36-entry fold of 12 shifts at 16^4 took 362 us).
template <bool F32, int NS>
__global__ void __launch_bounds__(256) k_cg_flush(CgDev cg, const double* __restrict__ coef,
                                                  const double* __restrict__ sh, const int32_t* __restrict__ act_next,
                                                  double* __restrict__ x_hi, double* __restrict__ pj, int32_t final_,
                                                  int32_t first, int32_t seed_only, int64_t n) {
  const int32_t v = blockIdx.y;
  const int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const int32_t m = min(fl[kFlM], cg.nslot - 1);   // the host flushes before m passes nslot - 1
  const int32_t base = fl[kFlBase], base32 = fl[kFlBase32], k0 = fl[kFlK0], k64 = fl[kFlK64];
  const int32_t seed = cg.seed[v];
  const int32_t nc = 2 + 2 * cg.cslots;
  const int32_t ns = cg.n_shift;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double rv[NS];
  if constexpr (!F32) {
#pragma unroll
    for (int g = 0; g < NS; g += 8)
      if (g <= m) {
#pragma unroll
        for (int i = g; i < g + 8 && i < NS; ++i) rv[i] = entry64(cg, v, base, min(i, m), n)[e];
      }
  } else {
    // below K64 the FP64 entries (only in the segment that spans the switch), from K0 on the FP32 ones
    const int32_t m64 = min(k64, m + 1) - 1;
#pragma unroll
    for (int g = 0; g < NS; g += 8) {
      if (g > m) continue;
      float rt[8];
      if (g + 7 > m64) {
#pragma unroll
        for (int i = 0; i < 8; ++i) rt[i] = entry32(cg, v, base32, k0, min(max(g + i, k0), m), n)[e];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (g + i < NS) rv[g + i] = (double)rt[i];
      }
      if (g <= m64) {
        double rd[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) rd[i] = entry64(cg, v, base, min(g + i, m64), n)[e];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (g + i < NS && g + i <= m64) rv[g + i] = rd[i];
      }
    }
  }
  for (int j = 0; j < ns; ++j) {
    if (seed_only ? j != seed : (cg.seed_explicit && j == seed)) continue;   // kept current by the residual update
    const int64_t vj = (int64_t)v * ns + j;
    const double* cf = coef + vj * nc;
    double* xj = x_hi + vj * n + e;
    double* pp = pj + vj * n + e;
    if (sh[vj * kShN + kShSeg] == 0.0) {
      if (first) *xj = 0.0;   // never updated (zero source)
      continue;
    }
    // p_j0 exists once a flush has written it; before that its coefficients are exactly zero
    const double p0 = (cf[0] != 0.0 || cf[1] != 0.0) ? *pp : 0.0;
    *xj = fold<NS>(cf + 2, rv, m, fma(cf[0], p0, first ? 0.0 : *xj));
    if (!final_ && !seed_only && act_next[vj]) *pp = fold<NS>(cf + 2 + cg.cslots, rv, m, cf[1] * p0);
  }
}

// after a flush: coefficients of the fresh segment (x_j = x_j0, p_j = p_j0), which starts at the
// current residual (fp32: in the FP32 ring, with no FP64 entries)
__global__ void k_cg_flush_reset(CgDev cg, int32_t fp32) {
  const int32_t v = blockIdx.x;
  int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const int32_t nc = 2 + 2 * cg.cslots;
  for (int j = threadIdx.x; j < cg.n_shift; j += blockDim.x) {
    const int64_t vj = (int64_t)v * cg.n_shift + j;
    double* cf = cg.coef + vj * nc;
    for (int i = 0; i < nc; ++i) cf[i] = 0.0;
    cf[1] = 1.0;
    cg.sh[vj * kShN + kShSeg] = 0.0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int32_t m = fl[kFlM];
    if (fp32) {
      fl[kFlBase32] = (fl[kFlBase32] + m - fl[kFlK0]) % cg.nslot32;
      fl[kFlK0] = 0;
      fl[kFlK64] = 0;
    } else {
      fl[kFlBase] = (fl[kFlBase] + m) % cg.nslot64;
    }
    fl[kFlM] = 0;
  }
}

hipError_t launch_cg_flush(const CgDev& cg, double* x_hi, double* pj, int32_t final_, int32_t first,
                           int32_t seed_only, int32_t fp32, int64_t n_reals, hipStream_t s) {
  if (cg.nslot > kMaxSlots || cg.nslot > cg.cslots || cg.cslots % 8 || cg.nslot64 > kMaxSlots) return hipErrorInvalidValue;
  if (fp32 && (!cg.ring32 || cg.nslot32 < cg.nslot || seed_only)) return hipErrorInvalidValue;
  dim3 grid((unsigned)((n_reals + kBlock - 1) / kBlock), cg.n_rhs);
  const auto kernel = cg.nslot <= kMaxBasis + 1 ? (fp32 ? k_cg_flush<true, kMaxBasis + 1> : k_cg_flush<false, kMaxBasis + 1>)
                                                : (fp32 ? k_cg_flush<true, kMaxSlots> : k_cg_flush<false, kMaxSlots>);
  hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, cg, cg.coef, cg.sh, cg.act_next, x_hi, pj, final_, first,
                     seed_only, n_reals);
  if (!seed_only) hipLaunchKernelGGL(k_cg_flush_reset, dim3(cg.n_rhs), dim3(kRedBlock), 0, s, cg, fp32);
  return hipGetLastError();
}

// the switch of precision: the current FP64 entry M -> FP32 slot 0, which holds entry K0 = M from
// now on; p64 -> p32
__global__ void k_cg_to_f32(CgDev cg, const double* __restrict__ p64, float* __restrict__ p32, int64_t n) {
  const int32_t v = blockIdx.y;
  const int32_t* fl = cg.flags + (int64_t)v * kFlN;
  const double* r = entry64(cg, v, fl[kFlBase], fl[kFlM], n);
  float* r32 = ring_slot<float>(cg.ring32, cg.rb32, v, 0, n);
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r32[i0 + k] = (float)r[i0 + k];
    p32[(int64_t)v * n + i0 + k] = (float)p64[(int64_t)v * n + i0 + k];
  }
}

__global__ void k_cg_to_f32_scalars(CgDev cg) {
  for (int v = threadIdx.x; v < cg.n_rhs; v += blockDim.x) {
    int32_t* fl = cg.flags + (int64_t)v * kFlN;
    double* sc = cg.sc + (int64_t)v * kScN;
    fl[kFlK64] = fl[kFlM] + 1;
    fl[kFlK0] = fl[kFlM];
    fl[kFlBase32] = 0;
    sc[kScMaxR] = sqrt(sc[kScRR]);
  }
}

hipError_t launch_cg_to_f32(const CgDev& cg64, const double* p64, float* p32, int64_t n_reals, hipStream_t s) {
  if (!cg64.ring32) return hipErrorInvalidValue;
  dim3 grid(elem_num_blocks(n_reals), cg64.n_rhs);
  hipLaunchKernelGGL(k_cg_to_f32, grid, dim3(kBlock), 0, s, cg64, p64, p32, n_reals);
  hipLaunchKernelGGL(k_cg_to_f32_scalars, dim3(1), dim3(kRedBlock), 0, s, cg64);
  return hipGetLastError();
}

// X[i] = x_hi[idx[i]], B[i] = b[idx[i] / ns] for the pairs of a refinement batch
__global__ void k_gather_pairs(const double* __restrict__ x_hi, const double* __restrict__ b,
                               const int32_t* __restrict__ idx, int32_t ns, double* __restrict__ X,
                               double* __restrict__ B, int64_t n) {
  const int32_t i = blockIdx.y;
  const int32_t q = idx[i];
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    X[(int64_t)i * n + i0 + k] = x_hi[(int64_t)q * n + i0 + k];
    B[(int64_t)i * n + i0 + k] = b[(int64_t)(q / ns) * n + i0 + k];
  }
}

hipError_t launch_gather_pairs(const double* x_hi, const double* b, const int32_t* idx, int32_t ns, double* X,
                               double* B, int32_t nb, int64_t n, hipStream_t s) {
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_pairs, dim3(elem_num_blocks(n), nb), dim3(kBlock), 0, s, x_hi, b, idx, ns, X, B, n);
  return hipGetLastError();
}

// x_hi[idx[i]] += E[i]
__global__ void k_scatter_add_pairs(double* __restrict__ x_hi, const int32_t* __restrict__ idx,
                                    const double* __restrict__ E, int64_t n) {
  const int32_t i = blockIdx.y;
  const int32_t q = idx[i];
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) x_hi[(int64_t)q * n + i0 + k] += E[(int64_t)i * n + i0 + k];
}

hipError_t launch_scatter_add_pairs(double* x_hi, const int32_t* idx, const double* E, int32_t nb, int64_t n,
                                    hipStream_t s) {
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_add_pairs, dim3(elem_num_blocks(n), nb), dim3(kBlock), 0, s, x_hi, idx, E, n);
  return hipGetLastError();
}

// y = c x + sum_j r_j x_j  (FP64) with partial <y, y>
__global__ void k_rational_combine(const double* __restrict__ x, const double* __restrict__ xp, int32_t n_poles,
                                   const double* __restrict__ coef, double* __restrict__ y, int64_t n,
                                   int32_t steps, double* partials) {
  const int32_t v = blockIdx.y;
  double d[1] = {0.0};
  const double c = coef[0];
  for (int32_t t = 0; t < steps; ++t) {
    const int64_t i0 = (((int64_t)blockIdx.x * steps + t) * blockDim.x + threadIdx.x) * 4;
    if (i0 < n) {
      double acc[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] = c * x[(int64_t)v * n + i0 + k];
      for (int j = 0; j < n_poles; ++j) {
        const double* xj = xp + ((int64_t)v * n_poles + j) * n + i0;
        const double rj = coef[1 + j];
        double t4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t4[k] = xj[k];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = fma(rj, t4[k], acc[k]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        y[(int64_t)v * n + i0 + k] = acc[k];
        d[0] = fma(acc[k], acc[k], d[0]);
      }
    }
  }
  if (partials) {
    __shared__ double lds[1][16];
    block_sum<1>(d, lds);
    if (threadIdx.x == 0) partials[(int64_t)v * gridDim.x + blockIdx.x] = d[0];
  }
}

hipError_t launch_rational_combine(const double* x, const double* xp, int32_t n_rhs, int32_t n_poles,
                                   const double* coef, double* y, int64_t n_reals, double* partials,
                                   hipStream_t s) {
  if (n_rhs == 0) return hipSuccess;
  dim3 grid(red_num_blocks(n_reals), n_rhs);
  hipLaunchKernelGGL(k_rational_combine, grid, dim3(kBlock), 0, s, x, xp, n_poles, coef, y, n_reals,
                     red_steps(n_reals), partials);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// link derivative
//
// For the link U = U_mu(x):  d<A, Delta B>/d omega^c = sum_{d,e} f^{dec} (R(U) C)^{de},
// C^{be} = B(x+mu)^b A(x)^e + A(x+mu)^b B(x)^e (summed over nu and over the pairs with
// weights w_k).  f^{abc} are the su(3) structure constants; with the antisymmetric part
// S = RC - (RC)^T each independent triple (a, b, c; f) contributes
// f S_ab to component c, f S_bc to component a and f S_ca to component b.

struct FTriple {
  int a, b, c;
  double f;
};
// compile-time table: with the loop over it unrolled every index is a constant, so the 8x8
// products stay in registers
constexpr FTriple kF[9] = {{0, 1, 2, 1.0},
                           {0, 3, 6, 0.5},
                           {0, 4, 5, -0.5},
                           {1, 3, 5, 0.5},
                           {1, 4, 6, 0.5},
                           {2, 3, 4, 0.5},
                           {2, 5, 6, -0.5},
                           {3, 4, 7, 0.86602540378443864676},
                           {5, 6, 7, 0.86602540378443864676}};

// G += R[:, b1] x C[b1, :] + R[:, b2] x C[b2, :] for the column group q of R(U) (columns b1, b2)
template <int q, int b1, int b2>
__device__ __forceinline__ void force_cross_cols(const double* u, const double* C, double* G) {
  double c1[8], c2[8];
  adjoint_columns<double, q>(u, c1, c2);
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int a = kF[t].a, b = kF[t].b, c = kF[t].c;
    const double f = kF[t].f;
    // (p x q)_c += f (p_a q_b - p_b q_a), cyclically in (a, b, c), both columns in one chain
    const auto cross = [&](int i, int j) {
      return fma(-c2[j], C[b2 * 8 + i],
                 fma(c2[i], C[b2 * 8 + j], fma(-c1[j], C[b1 * 8 + i], c1[i] * C[b1 * 8 + j])));
    };
    G[c] = fma(f, cross(a, b), G[c]);
    G[a] = fma(f, cross(b, c), G[a]);
    G[b] = fma(f, cross(c, a), G[b]);
  }
}

// One thread per (site, mu): a block of 256 threads is four waves, wave w taking direction mu = w for the
// block's 64 consecutive sites.  With every lane loading A and B at x and x+mu, 512 reals per site and pair,
// the path from the caches to the registers (32 bytes per clock and CU) bounds it: 12 us a pair at 16^4 and 26
// for the rest of the launch.  So the four waves load A and B at x once, a quarter each, into LDS, where a
// neighbour inside the block is read too: at 16^4 208 reals per site and pair.  One step is one nu of one
// pair; the loads of the next step are in flight during the 128 multiply-adds of this one (two steps ahead
// they spill: four pairs in 133 us instead of 71).  12 pairs 168 -> 111 us in a loop and 261 -> 172 after a solve
// (their 400 MB then come from HBM), at 12^4 111 -> 82 us; the two pairs of two reverse Chebyshev steps 41 to 43 us,
// against 38 for one.  What is left is the latency of a step, two waves per SIMD.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_force(const ForceArgs F, int32_t xcd) {
  __shared__ double own[2][16][64];   // A and B at the block's sites, by turns
  const int32_t o = blockIdx.y;
  const int32_t V = F.g.V;
  const int32_t blk = remap_block(blockIdx.x, gridDim.x, xcd);
  const int32_t mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t lane = threadIdx.x & 63;
  const bool live = blk * 64 + lane < V;
  const int32_t s = live ? blk * 64 + lane : blk * 64;   // lanes past the end go along with the first site
  int32_t xc[4];
  site_coords(F.g, s, xc);
  const int32_t r0 = F.per_rhs ? o : 0;
  const int32_t nr = F.per_rhs ? 1 : F.n_rhs;
  {
    const int32_t sf = site_shift(F.g, s, xc, mu, +1);
    const int32_t d = sf - blk * 64;
    const bool near = d >= 0 && d < 64;
    const uint32_t os = byte_off<double>(s), of = byte_off<double>(sf);
    double C[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) C[i] = 0.0;
    const int32_t steps = nr * F.n_pair * 4;
    // the step whose loads go out next
    int32_t rh = r0, k = 0, nu = 0;
    double q[4], fa[8], fb[8];
    auto load = [&]() {
      const int64_t off = rh * F.rhs_stride + (int64_t)nu * 8 * V;
      const double* Ak = F.A[k] + off;
      const double* Bk = F.B[k] + off;
      Rows<double> qr((mu < 2 ? Ak : Bk) + (int64_t)((mu & 1) * 4) * V, V, os);
#pragma unroll
      for (int a = 0; a < 4; ++a) q[a] = qr.get();
      if (!near) {
        Rows<double> ar(Ak, V, of), br(Bk, V, of);
#pragma unroll
        for (int a = 0; a < 8; ++a) fa[a] = ar.get();
#pragma unroll
        for (int a = 0; a < 8; ++a) fb[a] = br.get();
      }
      if (++nu == 4) {
        nu = 0;
        if (++k == F.n_pair) {
          k = 0;
          ++rh;
        }
      }
    };
    if (steps > 0) load();
#pragma unroll 1
    for (int32_t t = 0; t < steps; ++t) {
      double(*buf)[64] = own[t & 1];
      const double w = F.w[(t >> 2) % F.n_pair];
#pragma unroll
      for (int a = 0; a < 4; ++a) buf[mu * 4 + a][lane] = q[a];
      double af[8], bf[8];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        af[a] = fa[a];
        bf[a] = fb[a];
      }
      __syncthreads();
      if (t + 1 < steps) load();
      if (near) {
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          af[a] = buf[a][d];
          bf[a] = buf[8 + a][d];
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double ax = w * buf[e][lane], bx = w * buf[8 + e][lane];
#pragma unroll
        for (int b = 0; b < 8; ++b) C[b * 8 + e] = fma(af[b], bx, fma(bf[b], ax, C[b * 8 + e]));
      }
    }
    if (!live) return;
    // rows 0 and 1 of U_mu(x) (12 reals), row 2 rebuilt (SU(3))
    double u[18];
    const double* Um = F.U + (int64_t)mu * 18 * V;
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = (Um + (size_t)c * V)[s];
    su3_row2<double>(u);
    // G = sum_b R[:, b] x C[b, :], x the su(3) product (p x q)_c = sum_{a,e} f^{aec} p_a q_e, with
    // the columns of R(U) formed two at a time (the whole of R is never held)
    double G[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) G[c] = 0.0;
    force_cross_cols<0, 0, 1>(u, C, G);
    force_cross_cols<1, 3, 4>(u, C, G);
    force_cross_cols<2, 5, 6>(u, C, G);
    force_cross_cols<3, 2, 7>(u, C, G);
    double* go = F.grad + ((int64_t)o * 4 + mu) * 8 * V;
    if (F.accumulate) {
#pragma unroll
      for (int c = 0; c < 8; ++c) go[(int64_t)c * V + s] += G[c];
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) go[(int64_t)c * V + s] = G[c];
    }
  }
}

__global__ void k_cheb_source(double* __restrict__ tb, const double* __restrict__ Y, const double* __restrict__ coef,
                              int32_t n_rhs, int32_t n_y, int32_t n_k, int32_t k, int64_t n) {
  const int32_t v = blockIdx.y;
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i0 >= n) return;
  double acc[4];
  double* t = tb + (int64_t)v * n + i0;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = t[q];
  for (int32_t y = 0; y < n_y; ++y) {
    const double c = coef[((int64_t)v * n_y + y) * n_k + k];
    const double* yv = Y + ((int64_t)y * n_rhs + v) * n + i0;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = fma(c, yv[q], acc[q]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) t[q] = acc[q];
}

hipError_t launch_cheb_source(double* tb, const double* Y, const double* coef, int32_t n_rhs, int32_t n_y,
                              int32_t n_k, int32_t k, int64_t n_reals, hipStream_t s) {
  if (n_rhs == 0 || n_y == 0) return hipSuccess;
  dim3 grid(elem_num_blocks(n_reals), n_rhs);
  hipLaunchKernelGGL(k_cheb_source, grid, dim3(kBlock), 0, s, tb, Y, coef, n_rhs, n_y, n_k, k, n_reals);
  return hipGetLastError();
}

// Chebyshev filter fold: two consecutive elements per thread; the block's t_k are loaded once
// into registers and every window output is read, updated and written once per fold.
template <typename T>
__global__ void __launch_bounds__(256) k_cheb_fold(const T* __restrict__ x, const T* __restrict__ ring, int32_t R,
                                                   int32_t k0, int32_t cnt, int32_t first,
                                                   const double* __restrict__ coef, int32_t D1, int32_t nw,
                                                   T* __restrict__ y, int64_t n) {
  // this fold's coefficients (window w, vector j: coef[w][k0 + j]; column 0 for x on the first
  // fold) staged in LDS by the whole block, so the window loop reads no global scalars
  __shared__ double s_c[kMaxFilterWindows][kMaxFold + 1];
  for (int t = threadIdx.x; t < nw * (kMaxFold + 1); t += blockDim.x) {
    const int w = t / (kMaxFold + 1), j = t - w * (kMaxFold + 1);
    double c = 0.0;
    if (j == 0)
      c = first ? coef[(int64_t)w * D1] : 0.0;
    else if (j <= cnt)
      c = coef[(int64_t)w * D1 + k0 + j - 1];
    s_c[w][j] = c;
  }
  __syncthreads();
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 2;
  if (i0 >= n) return;
  // every load is issued unconditionally so they overlap: entries past cnt re-read the last
  // vector of the fold (a cache hit) and are never used
  T tt[kMaxFold][2];
#pragma unroll
  for (int j = 0; j < kMaxFold; ++j) {
    const T* t = ring + (int64_t)((k0 + min(j, cnt - 1)) % R) * n + i0;
    tt[j][0] = t[0];
    tt[j][1] = t[1];
  }
  double tv[kMaxFold][2];
#pragma unroll
  for (int j = 0; j < kMaxFold; ++j) {
    tv[j][0] = (double)tt[j][0];
    tv[j][1] = (double)tt[j][1];
  }
  double x0 = 0.0, x1 = 0.0;
  if (first) {
    x0 = (double)x[i0];
    x1 = (double)x[i0 + 1];
  }
  // windows four at a time: their outputs are loaded together
  for (int32_t w0 = 0; w0 < nw; w0 += 4) {
    double a[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t w = w0 + u;
      if (w < nw && !first) {
        const T* yw = y + (int64_t)w * n + i0;
        a[u][0] = (double)yw[0];
        a[u][1] = (double)yw[1];
      } else {
        a[u][0] = 0.0;
        a[u][1] = 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t w = w0 + u;
      if (w >= nw) break;
      const double* c = s_c[w];
      if (first) {
        a[u][0] = c[0] * x0;
        a[u][1] = c[0] * x1;
      }
      // branch-free: the coefficients past cnt are zero (their vectors are finite re-reads)
#pragma unroll
      for (int j = 0; j < kMaxFold; ++j) {
        a[u][0] = fma(c[1 + j], tv[j][0], a[u][0]);
        a[u][1] = fma(c[1 + j], tv[j][1], a[u][1]);
      }
      T* yw = y + (int64_t)w * n + i0;
      yw[0] = (T)a[u][0];
      yw[1] = (T)a[u][1];
    }
  }
}

template <typename T>
hipError_t launch_cheb_fold(const T* x, const T* ring, int32_t R, int32_t k0, int32_t cnt, int32_t first,
                            const double* coef, int32_t D, int32_t nw, T* y, int64_t n, hipStream_t s) {
  if (n == 0 || nw == 0) return hipSuccess;
  if (cnt < 1 || cnt > kMaxFold || nw > kMaxFilterWindows || (n & 1)) return hipErrorInvalidValue;
  const int64_t nb = (n / 2 + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_cheb_fold<T>, dim3((uint32_t)nb), dim3(kBlock), 0, s, x, ring, R, k0, cnt, first, coef, D + 1,
                     nw, y, n);
  return hipGetLastError();
}
template hipError_t launch_cheb_fold<double>(const double*, const double*, int32_t, int32_t, int32_t, int32_t,
                                             const double*, int32_t, int32_t, double*, int64_t, hipStream_t);
template hipError_t launch_cheb_fold<float>(const float*, const float*, int32_t, int32_t, int32_t, int32_t,
                                            const double*, int32_t, int32_t, float*, int64_t, hipStream_t);

hipError_t launch_force(const ForceArgs& a, hipStream_t s) {
  const int32_t n_out = a.per_rhs ? a.n_rhs : 1;
  if (a.n_pair < 0 || a.n_pair > (int32_t)(sizeof(a.w) / sizeof(a.w[0]))) return hipErrorInvalidValue;
  if (n_out == 0) return hipSuccess;
  dim3 grid((a.g.V + 63) / 64, n_out);
  hipLaunchKernelGGL(k_force, grid, dim3(256), 0, s, a, 1);
  return hipGetLastError();
}

}  // namespace rmh

namespace rmh {

// ------------------------------------------------------------------------------------------
// Wilson gauge force
//
// 3x3 complex matrices as separate real and imaginary parts, row-major.
struct M3 {
  double re[9], im[9];
};

// Rows 0 and 1 of the links at a block's 64 sites, by direction and component.
using OwnLinks = double[4][12][64];

// U_mu at site s: rows 0 and 1 (12 reals) from LDS where it holds the block's own links (kOwn) and s is one of the
// block's sites (from s0 on), else from memory; row 2 rebuilt from them (SU(3)).
template <bool kOwn>
__device__ __forceinline__ void load_link(const double* __restrict__ U, const OwnLinks& own, int32_t mu, int32_t s,
                                          int32_t s0, int32_t V, M3& m) {
  double u[18];
  const int32_t d = s - s0;
  if (kOwn && d >= 0 && d < 64) {
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = own[mu][c][d];
  } else {
    Rows<double> r(U + (int64_t)mu * 18 * V, V, byte_off<double>(s));
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = r.get();
  }
  su3_row2<double>(u);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    m.re[k] = u[2 * k];
    m.im[k] = u[2 * k + 1];
  }
}

// C = op(A) op(B) (kAcc: C += op(A) op(B)), op = identity or Hermitian conjugate
template <bool kDa, bool kDb, bool kAcc = false>
__device__ __forceinline__ void mul3(const M3& A, const M3& B, M3& C) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double re = kAcc ? C.re[i * 3 + j] : 0.0, im = kAcc ? C.im[i * 3 + j] : 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int ia = kDa ? k * 3 + i : i * 3 + k;
        const int ib = kDb ? j * 3 + k : k * 3 + j;
        const double ar = A.re[ia], ai = kDa ? -A.im[ia] : A.im[ia];
        const double br = B.re[ib], bi = kDb ? -B.im[ib] : B.im[ib];
        re = fma(ar, br, fma(-ai, bi, re));
        im = fma(ar, bi, fma(ai, br, im));
      }
      C.re[i * 3 + j] = re;
      C.im[i * 3 + j] = im;
    }
}

// F^c_mu(x) = -(beta/3) Im Tr(T^c U_mu(x) A_mu(x)), A the sum of the six staples; partials of
// sum_mu Re Tr(U_mu A_mu) per block (each plaquette enters four times).  A block is four waves over
// the same 64 consecutive sites, wave w computing the force on U_w: the direction is wave-uniform,
// every load is a coalesced 64-site row of one component, and a lattice gives four times as many
// waves as sites / 64 to hide the staples' dependent loads.
// Loaded by every wave for itself, the 76 links of a site take 912 reals through the path from the caches to the
// registers (32 bytes per clock and CU), 0.85 ms at 32^3x64: so the block's own links go to LDS once, and a
// link at one of the block's sites (all x0 neighbours and half the x1 neighbours there) is read from it: 46
// links, 552 reals, 1140 -> 1040 us.  With row 2 in LDS too the kernel needs 290 registers: one wave per SIMD, 1680 us.
// Where the lattice gives a CU one block at most, latency alone counts: with rows of x0 across wave and block ends
// a wave goes through both paths link by link, and every link from memory (kOwn false) is the faster (7x6x8x5 10.8 us
// against 12.0; 8^4, whose rows fit, 11.9 against 10.8 from LDS).
template <bool kOwn>
__global__ void __launch_bounds__(256) k_gauge_force(Geom g, const double* __restrict__ U, double beta,
                                                     double* __restrict__ F, double* __restrict__ partials) {
  __shared__ OwnLinks own;
  const int32_t V = g.V;
  const int32_t mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t s0 = blockIdx.x * 64, lane = threadIdx.x & 63;
  const int32_t s = s0 + lane;
  double tr[1] = {0.0};
  if (kOwn) {
    Rows<double> r(U + (int64_t)mu * 18 * V, V, byte_off<double>(min(s, V - 1)));
    double u[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = r.get();
#pragma unroll
    for (int c = 0; c < 12; ++c) own[mu][c][lane] = u[c];
    __syncthreads();
  }
  if (s < V) {
    int32_t xc[4];
    site_coords(g, s, xc);
    const int32_t s_pm = site_shift(g, s, xc, mu, +1);
    int32_t xm[4];
    site_coords(g, s_pm, xm);
    M3 A;
#pragma unroll
    for (int k = 0; k < 9; ++k) A.re[k] = A.im[k] = 0.0;
#pragma unroll 1
    for (int32_t nu = 0; nu < 4; ++nu) {
      if (nu == mu) continue;
      const int32_t s_pn = site_shift(g, s, xc, nu, +1);
      const int32_t s_mn = site_shift(g, s, xc, nu, -1);
      const int32_t s_pm_mn = site_shift(g, s_pm, xm, nu, -1);
      M3 a, b, t;
      // upper staple U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
      load_link<kOwn>(U, own, nu, s_pm, s0, V, a);
      load_link<kOwn>(U, own, mu, s_pn, s0, V, b);
      mul3<false, true>(a, b, t);
      load_link<kOwn>(U, own, nu, s, s0, V, a);
      mul3<false, true, true>(t, a, A);
      // lower staple U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
      load_link<kOwn>(U, own, nu, s_pm_mn, s0, V, a);
      load_link<kOwn>(U, own, mu, s_mn, s0, V, b);
      mul3<true, true>(a, b, t);
      load_link<kOwn>(U, own, nu, s_mn, s0, V, a);
      mul3<false, false, true>(t, a, A);
    }
    M3 u, m;
    load_link<kOwn>(U, own, mu, s, s0, V, u);
    mul3<false, false>(u, A, m);
    tr[0] = m.re[0] + m.re[4] + m.re[8];
    // Im Tr(lambda^c M) for the eight Gell-Mann matrices; T^c = lambda^c / 2
    double q[8];
    q[0] = m.im[3] + m.im[1];
    q[1] = m.re[1] - m.re[3];
    q[2] = m.im[0] - m.im[4];
    q[3] = m.im[6] + m.im[2];
    q[4] = m.re[2] - m.re[6];
    q[5] = m.im[7] + m.im[5];
    q[6] = m.re[5] - m.re[7];
    q[7] = (m.im[0] + m.im[4] - 2.0 * m.im[8]) * 0.57735026918962576451;
    if (F) {
      double* f = F + (int64_t)mu * 8 * V + s;
      const double k = -beta / 6.0;
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) f[(int64_t)cc * V] = k * q[cc];
    }
  }
  if (partials) {
    __shared__ double lds[1][16];
    block_sum<1>(tr, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = tr[0];
  }
}

int gauge_force_blocks(const Geom& g) { return (g.V + 63) / 64; }

hipError_t launch_gauge_force(const Geom& g, const double* U, double beta, double* F, double* partials,
                              hipStream_t s) {
  const int nblk = gauge_force_blocks(g);
  const auto kernel = nblk <= 256 && 64 % g.L0 ? k_gauge_force<false> : k_gauge_force<true>;
  hipLaunchKernelGGL(kernel, dim3(nblk), dim3(256), 0, s, g, U, beta, F, partials);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// molecular-dynamics updates of the implicit leapfrog

// 3x3 complex matrices as separate real and imaginary parts, row major
struct Cm3 {
  double re[9], im[9];
};

__device__ __forceinline__ void cm3_mul(const Cm3& a, const Cm3& b, Cm3& c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        sr = fma(a.re[3 * i + k], b.re[3 * k + j], fma(-a.im[3 * i + k], b.im[3 * k + j], sr));
        si = fma(a.re[3 * i + k], b.im[3 * k + j], fma(a.im[3 * i + k], b.re[3 * k + j], si));
      }
      c.re[3 * i + j] = sr;
      c.im[3 * i + j] = si;
    }
}

// exp(i H) U per link, H = sum_c a^c T^c: scaling and squaring of the Taylor series.  X = i H is
// scaled by 2^-q until its Frobenius norm is at most 1/4, the series is summed to degree 12 in
// Horner form (remainder below 0.25^13 / 13! < 3e-18 relative), and the result is squared q
// times.  The exponential of an anti-Hermitian traceless matrix is in SU(3), so U1 stays in SU(3)
// to rounding.
__global__ void k_link_exp(Geom g, const double* __restrict__ U0, const double* __restrict__ A,
                           const double* __restrict__ B, double h, double* __restrict__ U1) {
  const int32_t mu = blockIdx.y;
  const int64_t V = g.V;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= V) return;
  double a[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int64_t e = ((int64_t)mu * 8 + c) * V + s;
    a[c] = h * (B ? A[e] + B[e] : A[e]);
  }
  // H = sum_c a^c lambda^c / 2 (Gell-Mann), Hermitian traceless
  const double r3 = 0.57735026918962576451;   // 1 / sqrt(3)
  double hre[9], him[9];
  hre[0] = 0.5 * (a[2] + r3 * a[7]);
  hre[4] = 0.5 * (-a[2] + r3 * a[7]);
  hre[8] = -r3 * a[7];
  him[0] = him[4] = him[8] = 0.0;
  hre[1] = 0.5 * a[0]; him[1] = -0.5 * a[1];
  hre[2] = 0.5 * a[3]; him[2] = -0.5 * a[4];
  hre[5] = 0.5 * a[5]; him[5] = -0.5 * a[6];
  hre[3] = hre[1]; him[3] = -him[1];
  hre[6] = hre[2]; him[6] = -him[2];
  hre[7] = hre[5]; him[7] = -him[5];
  double nrm2 = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) nrm2 += hre[k] * hre[k] + him[k] * him[k];
  double nrm = sqrt(nrm2), scale = 1.0;
  int q = 0;
  while (nrm > 0.25 && q < 64) {   // false for NaN: a NaN momentum gives a NaN link
    nrm *= 0.5;
    scale *= 0.5;
    ++q;
  }
  // Y = i H * scale
  Cm3 Y, E, T;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    Y.re[k] = -him[k] * scale;
    Y.im[k] = hre[k] * scale;
  }
  // E = I + Y/1 (I + Y/2 (I + ... (I + Y/12)))
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    E.re[k] = (k % 4 == 0) ? 1.0 : 0.0;
    E.im[k] = 0.0;
  }
#pragma unroll 1
  for (int m = 12; m >= 1; --m) {
    cm3_mul(Y, E, T);
    const double w = 1.0 / (double)m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      E.re[k] = ((k % 4 == 0) ? 1.0 : 0.0) + w * T.re[k];
      E.im[k] = w * T.im[k];
    }
  }
#pragma unroll 1
  for (int i = 0; i < q; ++i) {
    cm3_mul(E, E, T);
    E = T;
  }
  Cm3 u;
  const double* um = U0 + (int64_t)mu * 18 * V + s;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    u.re[k] = um[(int64_t)(2 * k) * V];
    u.im[k] = um[(int64_t)(2 * k + 1) * V];
  }
  cm3_mul(E, u, T);
  double* uo = U1 + (int64_t)mu * 18 * V + s;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    uo[(int64_t)(2 * k) * V] = T.re[k];
    uo[(int64_t)(2 * k + 1) * V] = T.im[k];
  }
}

hipError_t launch_link_exp(const Geom& g, const double* U0, const double* A, const double* B, double h, double* U1,
                           hipStream_t s) {
  dim3 grid((unsigned)((g.V + kBlock - 1) / kBlock), 4);
  hipLaunchKernelGGL(k_link_exp, grid, dim3(kBlock), 0, s, g, U0, A, B, h, U1);
  return hipGetLastError();
}

// The transposed left-trivialised differential of the exponential map, per link:
// out = J(omega)^T g with exp(i(omega + eps e_c).T) = exp(i eps (J e_c).T + O(eps^2)) exp(i omega.T),
// so that d/d omega f(exp(i omega.T) U) = J^T (the derivative at the displaced link under left
// multiplication).  In the adjoint representation J = sum_k M^k / (k+1)!, (M v)^d = f^{adc} omega^a v^c,
// and M is antisymmetric, so J^T g = sum_k t_k with t_0 = g, t_k = (omega x t_{k-1}) / (k + 1) and
// (p x q)^d = sum f^{acd} p^a q^c.  The series is summed until a term no longer changes the sum
// (at most 64 terms: enough for |omega| up to about 10).
__global__ void k_dexp_vjp(Geom g, const double* __restrict__ omega, const double* __restrict__ gin,
                           double* __restrict__ gout) {
  const int32_t mu = blockIdx.y;
  const int64_t V = g.V;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= V) return;
  double w[8], t[8], acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int64_t e = ((int64_t)mu * 8 + c) * V + s;
    w[c] = omega[e];
    t[c] = gin[e];
    acc[c] = t[c];
  }
#pragma unroll 1
  for (int k = 1; k <= 64; ++k) {
    double n[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) n[c] = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int a = kF[q].a, b = kF[q].b, c = kF[q].c;
      const double f = kF[q].f;
      // (w x t)_c += f (w_a t_b - w_b t_a), cyclically in (a, b, c)
      n[c] += f * (w[a] * t[b] - w[b] * t[a]);
      n[a] += f * (w[b] * t[c] - w[c] * t[b]);
      n[b] += f * (w[c] * t[a] - w[a] * t[c]);
    }
    const double inv = 1.0 / (double)(k + 1);
    bool changed = false;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      t[c] = n[c] * inv;
      const double nxt = acc[c] + t[c];
      changed = changed || (nxt != acc[c]);
      acc[c] = nxt;
    }
    if (!changed) break;
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) gout[((int64_t)mu * 8 + c) * V + s] = acc[c];
}

hipError_t launch_dexp_vjp(const Geom& g, const double* omega, const double* gin, double* gout, hipStream_t s) {
  dim3 grid((unsigned)((g.V + kBlock - 1) / kBlock), 4);
  hipLaunchKernelGGL(k_dexp_vjp, grid, dim3(kBlock), 0, s, g, omega, gin, gout);
  return hipGetLastError();
}

__global__ void k_axpy_diff(const double* x, const double* __restrict__ y, const double* __restrict__ z, double h,
                            const double* prev, double* out, int64_t n, int32_t steps,
                            double* __restrict__ partials) {
  double d[2] = {0.0, 0.0};
  for (int32_t t = 0; t < steps; ++t) {
    const int64_t i0 = (((int64_t)blockIdx.x * steps + t) * blockDim.x + threadIdx.x) * 4;
    if (i0 < n) {
      double xv[4], yv[4], zv[4], ov[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        xv[k] = x[i0 + k];
        yv[k] = y[i0 + k];
        zv[k] = z[i0 + k];
        ov[k] = prev[i0 + k];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double o = fma(h, yv[k] - zv[k], xv[k]);
        const double e = o - ov[k];
        out[i0 + k] = o;
        d[0] = fma(e, e, d[0]);
        d[1] = fma(o, o, d[1]);
      }
    }
  }
  __shared__ double lds[2][16];
  block_sum<2>(d, lds);
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = d[0];
    partials[gridDim.x + blockIdx.x] = d[1];
  }
}

hipError_t launch_axpy_diff(const double* x, const double* y, const double* z, double h, const double* prev,
                            double* out, int64_t n, double* partials, hipStream_t s) {
  if (n % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_axpy_diff, dim3(red_num_blocks(n)), dim3(kBlock), 0, s, x, y, z, h, prev, out, n,
                     red_steps(n), partials);
  return hipGetLastError();
}

}  // namespace rmh
