// The adjoint-Laplacian stencil for gfx950: one hop per direction and sign, fused epilogues
// (axpby, dot products), the site-per-thread kernel, the hop-split kernel and the
// x3-walking kernel, and their launch dispatch.  Every kernel writes its output with
// non-temporal stores (and reads a per-field z input with non-temporal loads): neither is touched
// again in the launch, and streaming them past the L2 leaves that cache to the neighbour fields
// and links the blocks share.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "rmh_internal.h"
#include "rmh_reduce.h"

namespace rmh {

// ------------------------------------------------------------------------------------------
// the stencil

// Block -> (field v, lattice block lb). The grid is one-dimensional, nblk lattice blocks times
// n_rhs fields, taken in groups of fg fields (the largest divisor of n_rhs up to 4): within a
// group the fields are fastest, so consecutive blocks take the same sites of successive fields
// and a link loaded for the first is an L2 hit for the others (with the XCD remap each XCD owns
// a contiguous range); the groups are not interleaved, which keeps the neighbour fields of at
// most fg fields in the L2 at a time.
struct HopBlock {
  int32_t v, lb, nblk;
};
__host__ __device__ __forceinline__ int32_t hop_field_group(int32_t n_rhs) {
  for (int32_t f = 4; f > 1; --f)
    if (n_rhs % f == 0) return f;
  return 1;
}
__device__ __forceinline__ HopBlock hop_block(int32_t xcd, int32_t n_rhs) {
  const int32_t b = remap_block(blockIdx.x, gridDim.x, xcd);
  const int32_t fg = hop_field_group(n_rhs);
  HopBlock h;
  h.nblk = gridDim.x / n_rhs;
  const int32_t gsize = h.nblk * fg;   // blocks per field group
  const int32_t grp = b / gsize, r = b - grp * gsize;
  h.v = grp * fg + r % fg;
  h.lb = r / fg;
  return h;
}

// One hop's contribution to NV vectors: forward (kT = false, link U_mu(x), neighbour x+mu) or
// backward (kT = true, link U_mu(x-mu), neighbour x-mu).
template <typename T, int FORM, int NV, bool kT>
__device__ __forceinline__ void hop_apply(const T* u, const T (*phi)[8], T (*acc)[8]) {
  if (FORM == kFormAdjoint) {
    T R[64];
    adjoint_matrix<T>(u, R);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (!kT)
        adj_apply<T>(R, phi[v], acc[v]);
      else
        adj_apply_t<T>(R, phi[v], acc[v]);
    }
  } else if (FORM == kFormMatrix) {
#pragma unroll
    for (int v = 0; v < NV; ++v) mat_hop<T, kT>(u, phi[v], acc[v]);
  } else {
    adj_stream<T, NV, kT>(u, phi, acc);
  }
}

// The sum of all hops in components (the 3x3 form accumulates matrix elements).
template <typename T, int FORM, int NV>
__device__ __forceinline__ void hop_finish(T (*acc)[8]) {
  if (FORM == kFormMatrix) {
#pragma unroll
    for (int v = 0; v < NV; ++v) mat_components<T>(acc[v]);
  }
}

// Row 2 from rows 0 and 1 in the rounding the form uses (su3_row2).
template <typename T, int FORM>
__device__ __forceinline__ void link_row2(T* u) {
  su3_row2<T, sizeof(T) == 8 || FORM == kFormMatrix>(u);
}

// Rows 0 and 1 of the link at site s (component c at Um[c V + s]): row 2 is rebuilt from them (link_row2, SU(3)),
// so a hop moves 12 link reals instead of 18.  kUni: Um is the same for the whole wave.  The callers load the
// field before they rebuild row 2, so that all of a hop's loads are in flight together.
template <typename T, bool kUni = true, int N>
__device__ __forceinline__ void load_rows(const T* __restrict__ Um, int32_t s, int32_t V, T (&u)[N]) {
  if (kUni) {
    Rows<T> r(Um, V, byte_off<T>(s));
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = r.get();
  } else {
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] = (Um + (size_t)c * V)[s];
  }
}

// Directions nu0 .. nu0 + NV - 1 of the field at site s.  kScalar false: addressed per lane (the streamed form
// of the hop split: scalar rows made it 1 % slower, FP32 moments at 13x16x10x11, four fields).
template <typename T, int NV, bool kScalar = true>
__device__ __forceinline__ void load_field(const T* __restrict__ xf, int32_t s, int nu0, int32_t V, T (*f)[8]) {
  if (kScalar) {
    Rows<T> r(xf + (size_t)(nu0 * 8) * V, V, byte_off<T>(s));
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int b = 0; b < 8; ++b) f[i][b] = r.get();
  } else {
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int b = 0; b < 8; ++b) f[i][b] = (xf + (size_t)((nu0 + i) * 8 + b) * V)[s];
  }
}

// The residual of field v that dot 0 is taken with: the current one in the CG's ring (HopArgs::ring) or, after a
// reliable update, the FP64 one (HopArgs::ring_ru); neither without a ring.
template <typename T>
struct HopRing {
  const T* r;
  const double* ru;
  __device__ __forceinline__ explicit operator bool() const { return r || ru; }
};
template <typename T>
__device__ __forceinline__ HopRing<T> hop_ring_field(const HopArgs<T>& A, int32_t v) {
  HopRing<T> f{nullptr, nullptr};
  if (!A.ring) return f;
  const int32_t* fl = A.run - kFlRun + (int64_t)v * A.run_stride;
  if (sizeof(T) == 4 && A.ring_ru && fl[kFlNeedRU]) {
    f.ru = A.ring_ru + (int64_t)v * 32 * A.g.V;
    return f;
  }
  const int32_t i = sizeof(T) == 8 ? fl[kFlBase] + fl[kFlM] : fl[kFlBase32] + fl[kFlM] - fl[kFlK0];
  f.r = A.ring + ((int64_t)v * A.ring_slots + i % A.ring_slots) * 32 * (int64_t)A.g.V;
  return f;
}

// The epilogue at one site: out = a h + b x + c z for NV directions from nu0 on, and the partial dot
// products.  kLoadX: x is read back from the field, else it is handed over in xc.  kRing: the kernel takes
// HopArgs::ring and HopArgs::src (the walk has no registers left for them).  Per direction the
// loads of x and z come before the stores (z may be the output itself, each element read and
// written by this thread only), so they overlap.
template <typename T, int NV, bool DOTS, bool kLoadX, bool kRing>
__device__ __forceinline__ void hop_store(const HopArgs<T>& A, int32_t v, const T* __restrict__ xf, const T (*xc)[8],
                                          int nu0, int32_t s, bool store, const T (*acc)[8], double* dsum) {
  const int64_t V = A.g.V;
  const int64_t FV = 32 * V;
  const T ca = T(A.a);
  const T cb = T(A.b_rhs ? A.b_rhs[v] : A.b);
  const T cc = T(A.c);
  const T* zf = A.z ? A.z + (int64_t)(v / A.z_div) * FV : nullptr;  // may alias out
  T* outf = A.out + (int64_t)v * FV;
  HopRing<T> rf{nullptr, nullptr};
  if (DOTS && kRing) rf = hop_ring_field(A, v);   // z is null with it
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    T xs[8], zv[8];
    const int64_t r0 = (int64_t)((nu0 + i) * 8) * V;
    if (kLoadX) {
      Rows<T> xr(xf + r0, V, byte_off<T>(s));
#pragma unroll
      for (int a = 0; a < 8; ++a) xs[a] = xr.get();
    } else {
#pragma unroll
      for (int a = 0; a < 8; ++a) xs[a] = xc[i][a];
    }
    if (zf) {
      if (A.z_div == 1) {
        Rows<T> zr(zf + r0, V, byte_off<T>(s));
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          zv[a] = __builtin_nontemporal_load(zr.ptr());
          zr.next();
        }
      } else {
        Rows<T> zr(zf + r0, V, byte_off<T>(s));
#pragma unroll
        for (int a = 0; a < 8; ++a) zv[a] = zr.get();
      }
    }
    T w[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) w[a] = fmadd(ca, acc[i][a], cb * xs[a]);
    if (zf) {
#pragma unroll
      for (int a = 0; a < 8; ++a) w[a] = fmadd(cc, zv[a], w[a]);
    }
    if constexpr (!DOTS && kRing && sizeof(T) == 8) {
      if (A.src && v < A.src_rhs) {
        for (int32_t y = 0; y < A.src_n; ++y) {
          const double c = A.src_coef[((int64_t)v * A.src_n + y) * A.src_stride];
          Rows<T> yr(A.src + ((int64_t)y * A.src_rhs + v) * FV + r0, V, byte_off<T>(s));
          T yv[8];
#pragma unroll
          for (int a = 0; a < 8; ++a) yv[a] = yr.get();
#pragma unroll
          for (int a = 0; a < 8; ++a) w[a] = fma(c, yv[a], w[a]);
        }
      }
    }
    if (DOTS) {
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const double xd = (double)xs[a], od = (double)w[a];
        if (!kRing || !rf) dsum[0] = fma(xd, xd, dsum[0]);
        dsum[1] = fma(od, xd, dsum[1]);
        dsum[2] = fma(od, od, dsum[2]);
      }
    }
    if (store) {
      Rows<T> outr(outf + r0, V, byte_off<T>(s));
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        __builtin_nontemporal_store(w[a], outr.ptr());
        outr.next();
      }
    }
    if (DOTS && kRing && rf) {   // last, where the fewest registers are in use
      T rv[8];
      if (sizeof(T) == 4 && rf.ru) {
        Rows<double> rr(rf.ru + r0, V, byte_off<double>(s));
#pragma unroll
        for (int a = 0; a < 8; ++a) rv[a] = (T)rr.get();
      } else {
        Rows<T> rr(rf.r + r0, V, byte_off<T>(s));
#pragma unroll
        for (int a = 0; a < 8; ++a) rv[a] = rr.get();
      }
#pragma unroll
      for (int a = 0; a < 8; ++a) dsum[0] = fma((double)w[a], (double)rv[a], dsum[0]);
    }
  }
}

// The FP32 streamed form's link and field loads go out before any of the hop's arithmetic: left to itself the
// scheduler starts on the link and issues the field's loads between, a second exposed latency per hop (moments at
// 24^4, two fields: 134 us with all loads first, 141 without).  With two directions a thread the loads are half as
// many and all of them at once would cost a wave per SIMD.
template <typename T, int FORM, int NV>
__device__ __forceinline__ void all_loads_first() {
  if constexpr (sizeof(T) == 4 && FORM == kFormStream && NV == 4) __builtin_amdgcn_sched_barrier(0);
}

// out[v] = a (H x)[v] + b x[v] + c z[v]: a block of B threads covers B * NV / 4 sites; the
// 4 / NV thread groups of a site (direction subsets) are wave-aligned slices of the block.
// One backward hop: link and field both read at the neighbour site sb.
template <typename T, int FORM, int NV, bool kT, bool kUni = true>
__device__ __forceinline__ void hop_term(const T* __restrict__ Um, int32_t sb, const T* __restrict__ xf,
                                         int nu0, int32_t V, T (&acc)[NV][8]) {
  T u[18], phi[NV][8];
  load_rows<T, kUni>(Um, sb, V, u);
  load_field<T, NV, kUni || FORM == kFormMatrix>(xf, sb, nu0, V, phi);
  all_loads_first<T, FORM, NV>();
  link_row2<T, FORM>(u);
  hop_apply<T, FORM, NV, kT>(u, phi, acc);
}

// One forward hop: link at s, field at the neighbour sf.
template <typename T, int FORM, int NV, bool kUni = true>
__device__ __forceinline__ void hop_term_fwd(const T* __restrict__ Um, int32_t s, int32_t sf,
                                             const T* __restrict__ xf, int nu0, int32_t V,
                                             T (&acc)[NV][8]) {
  T u[18], phi[NV][8];
  load_rows<T, kUni>(Um, s, V, u);
  load_field<T, NV, kUni || FORM == kFormMatrix>(xf, sf, nu0, V, phi);
  all_loads_first<T, FORM, NV>();
  link_row2<T, FORM>(u);
  hop_apply<T, FORM, NV, false>(u, phi, acc);
}

template <typename T, int FORM, int NV, bool DOTS>
__global__ void __launch_bounds__(256) k_hop(const HopArgs<T> A, int32_t xcd, int32_t order) {
  constexpr int G = 4 / NV;  // thread groups per site
  const HopBlock hb = hop_block(xcd, A.n_rhs);
  const int32_t v = hb.v;
  if (A.run && A.run[(int64_t)v * A.run_stride] == 0) return;
  const int32_t V = A.g.V;
  const int32_t lb = hb.lb;
  const int32_t spb = blockDim.x / G;              // sites per block
  // direction subset of this thread: wave-uniform (spb is a multiple of the wave size), so the
  // per-component base addresses stay in scalar registers
  const int32_t grp = __builtin_amdgcn_readfirstlane(threadIdx.x / spb);
  int32_t blk = lb;
  if (order) {
    // lb = ((chunk * L2) + x2) * L3 + x3  ->  lexicographic block of that (x0 x1 chunk, x2, x3)
    const int32_t x3 = lb % A.g.L3;
    const int32_t t = lb / A.g.L3;
    const int32_t x2 = t % A.g.L2;
    const int32_t chunk = t / A.g.L2;
    const int32_t cpp = (A.g.L0 * A.g.L1) / spb;   // chunks per (x2, x3) plane
    blk = (x3 * A.g.L2 + x2) * cpp + chunk;
  }
  const int32_t s = blk * spb + (threadIdx.x - grp * spb);
  const int nu0 = grp * NV;
  double dsum[3] = {0.0, 0.0, 0.0};
  if (s < V) {
    const int64_t FV = 32 * (int64_t)V;
    const T* __restrict__ xf = A.x + ((int64_t)v * A.x_mul + A.x_add) * FV;
    const T* __restrict__ U = A.U;
    T acc[NV][8];
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int a = 0; a < 8; ++a) acc[i][a] = T(0);
    int32_t xc[4];
    site_coords(A.g, s, xc);
    // term order (shared with k_hop_walk, so every launch shape rounds alike): the x3
    // backward hop, the x0, x1, x2 forward and backward hops, the x3 forward hop
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      const int mb = (mu + 3) & 3;   // backward hop of the previous direction, x3 first
      hop_term<T, FORM, NV, true>(U + (int64_t)mb * 18 * V, site_shift(A.g, s, xc, mb, -1), xf, nu0, V, acc);
      hop_term_fwd<T, FORM, NV>(U + (int64_t)mu * 18 * V, s, site_shift(A.g, s, xc, mu, +1), xf, nu0, V, acc);
    }
    hop_finish<T, FORM, NV>(acc);
    hop_store<T, NV, DOTS, true, true>(A, v, xf, nullptr, nu0, s, A.store != 0, acc, dsum);
  }
  if (DOTS) {
    __shared__ double lds[3][16];
    block_sum<3>(dsum, lds);
    if (threadIdx.x == 0) {
      const int32_t nblk = hb.nblk;
      double* p = A.partials + (int64_t)v * 3 * nblk + lb;
      if (A.dot_mask & 1) p[0] = dsum[0];
      if (A.dot_mask & 2) p[nblk] = dsum[1];
      if (A.dot_mask & 4) p[2 * nblk] = dsum[2];
    }
  }
}

// Hop-split variant of k_hop for lattices too small to fill the chip with one thread per site:
// the four lanes l, l+16, l+32, l+48 of a wave share a site, lane group mu doing the forward and the
// backward hop along mu; two butterfly shuffles sum the four partial results (in the fixed order
// (mu0 + mu1) + (mu2 + mu3)), and each of the four lanes stores a quarter of the components.  A wave
// covers 16 consecutive sites for one direction group; a block of B threads has B/64 waves.
template <typename T, int FORM, int NV, bool DOTS>
__global__ void __launch_bounds__(256) k_hop_split(const HopArgs<T> A, int32_t xcd, int32_t order) {
  constexpr int G = 4 / NV;
  const HopBlock hb = hop_block(xcd, A.n_rhs);
  const int32_t v = hb.v;
  if (A.run && A.run[(int64_t)v * A.run_stride] == 0) return;
  const int32_t V = A.g.V;
  const int32_t lb = hb.lb;
  const int32_t wi = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t W = blockDim.x >> 6;
  const int32_t grp = wi % G;   // wave-uniform direction group
  const int32_t spb = (W / G) * 16;
  const int32_t lane = threadIdx.x & 63;
  const int32_t mu = lane >> 4;
  int32_t blk = lb;
  if (order) {
    // x3 fastest, then x2, then the (x0, x1) chunks: a contiguous range of blocks (one XCD's,
    // with the remap) sweeps whole x3 columns of a few chunks, so the x3 and x2 neighbours of a
    // block were loaded moments before by the same XCD
    const int32_t x3 = lb % A.g.L3;
    const int32_t t = lb / A.g.L3;
    const int32_t x2 = t % A.g.L2;
    const int32_t chunk = t / A.g.L2;
    const int32_t cpp = (A.g.L0 * A.g.L1) / spb;
    blk = (x3 * A.g.L2 + x2) * cpp + chunk;
  }
  const int32_t s = blk * spb + (wi / G) * 16 + (lane & 15);
  const int nu0 = grp * NV;
  const bool live = s < V;
  const int64_t FV = 32 * (int64_t)V;
  const T* __restrict__ xf = A.x + ((int64_t)v * A.x_mul + A.x_add) * FV;
  T acc[NV][8];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int a = 0; a < 8; ++a) acc[i][a] = T(0);
  if (live) {
    int32_t xc[4];
    site_coords(A.g, s, xc);
    const T* __restrict__ Um = A.U + (int64_t)mu * 18 * V;
    hop_term<T, FORM, NV, true, false>(Um, site_shift(A.g, s, xc, mu, -1), xf, nu0, V, acc);
    hop_term_fwd<T, FORM, NV, false>(Um, s, site_shift(A.g, s, xc, mu, +1), xf, nu0, V, acc);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      acc[i][a] += __shfl_xor(acc[i][a], 16, 64);
      acc[i][a] += __shfl_xor(acc[i][a], 32, 64);
    }
  hop_finish<T, FORM, NV>(acc);
  // lane group mu keeps the components 4q + mu of its direction group (q < 2 NV), picked with
  // bit masks (a select chain here tends to become a lane-indexed array in scratch), then one
  // full-wave load/store per q; every z value is loaded before the first store (z may be the
  // output itself, each element read and written by this lane only), so those loads overlap
  double dsum[3] = {0.0, 0.0, 0.0};
  if (live) {
    const T ca = T(A.a);
    const T cb = T(A.b_rhs ? A.b_rhs[v] : A.b);
    const T cc = T(A.c);
    const T* zf = A.z ? A.z + (int64_t)(v / A.z_div) * FV : nullptr;  // may alias out
    T* outf = A.out + (int64_t)v * FV;
    constexpr bool kRing = sizeof(T) == 8 || FORM == kFormMatrix;   // the FP32 moments' form does without
    HopRing<T> rf{nullptr, nullptr};
    if (DOTS && kRing) rf = hop_ring_field(A, v);   // z is null with it
    using Bits = typename std::conditional<sizeof(T) == 8, uint64_t, uint32_t>::type;
    const Bits m0 = mu == 0 ? ~Bits(0) : Bits(0), m1 = mu == 1 ? ~Bits(0) : Bits(0);
    const Bits m2 = mu == 2 ? ~Bits(0) : Bits(0), m3 = mu == 3 ? ~Bits(0) : Bits(0);
    T hs[2 * NV], xs[2 * NV], zv[2 * NV];
#pragma unroll
    for (int q = 0; q < 2 * NV; ++q) {
      const int i = q >> 1, a0 = (q & 1) * 4;
      const Bits hb_ = (m0 & __builtin_bit_cast(Bits, acc[i][a0])) | (m1 & __builtin_bit_cast(Bits, acc[i][a0 + 1])) |
                       (m2 & __builtin_bit_cast(Bits, acc[i][a0 + 2])) | (m3 & __builtin_bit_cast(Bits, acc[i][a0 + 3]));
      hs[q] = __builtin_bit_cast(T, hb_);
      const int64_t e = (int64_t)(nu0 * 8 + 4 * q + mu) * V + s;
      xs[q] = xf[e];
      zv[q] = !zf ? T(0) : A.z_div == 1 ? __builtin_nontemporal_load(&zf[e]) : zf[e];
    }
    if (kRing && rf) {
      if (sizeof(T) == 4 && rf.ru) {
#pragma unroll
        for (int q = 0; q < 2 * NV; ++q) zv[q] = (T)rf.ru[(int64_t)(nu0 * 8 + 4 * q + mu) * V + s];
      } else {
#pragma unroll
        for (int q = 0; q < 2 * NV; ++q) zv[q] = rf.r[(int64_t)(nu0 * 8 + 4 * q + mu) * V + s];
      }
    }
#pragma unroll
    for (int q = 0; q < 2 * NV; ++q) {
      hs[q] = fmadd(ca, hs[q], cb * xs[q]);
      if (zf) hs[q] = fmadd(cc, zv[q], hs[q]);
    }
    if constexpr (!DOTS && sizeof(T) == 8) {
      // one branch for all components (a branch in each kept the stores apart: 4^4 5.36 us against 5.04)
      if (A.src && v < A.src_rhs)
        for (int32_t y = 0; y < A.src_n; ++y) {
          const T c = A.src_coef[((int64_t)v * A.src_n + y) * A.src_stride];
          const T* sf = A.src + ((int64_t)y * A.src_rhs + v) * FV;
#pragma unroll
          for (int q = 0; q < 2 * NV; ++q) hs[q] = fma(c, sf[(int64_t)(nu0 * 8 + 4 * q + mu) * V + s], hs[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 2 * NV; ++q) {
      if (A.store) __builtin_nontemporal_store(hs[q], &outf[(int64_t)(nu0 * 8 + 4 * q + mu) * V + s]);
      if (DOTS) {
        const double xd = (double)xs[q], od = (double)hs[q];
        const double rd = kRing && rf ? (double)zv[q] : xd;
        dsum[0] = fma(kRing && rf ? od : xd, rd, dsum[0]);
        dsum[1] = fma(od, xd, dsum[1]);
        dsum[2] = fma(od, od, dsum[2]);
      }
    }
  }
  if (DOTS) {
    __shared__ double lds[3][16];
    block_sum<3>(dsum, lds);
    if (threadIdx.x == 0) {
      const int32_t nblk = hb.nblk;
      double* p = A.partials + (int64_t)v * 3 * nblk + lb;
      if (A.dot_mask & 1) p[0] = dsum[0];
      if (A.dot_mask & 2) p[nblk] = dsum[1];
      if (A.dot_mask & 4) p[2 * nblk] = dsum[2];
    }
  }
}

// Waves per SIMD the walking kernel is compiled for.  The FP32 3x3-form walk over all four
// directions needs about 170 registers left to itself (two waves per SIMD); capped at 168 it keeps
// three waves, and its batched Chebyshev sweeps ran 4-5 % faster (they move fewer bytes than one
// thread per site but were latency-bound at two waves).  Under the cap the variant with the fused
// dot products (the sweeps, the CG) does not spill; the plain one spills about 130 B per lane since
// the x0 hops take their neighbours from other lanes.  The other walks keep the compiler's choice
// (FP64 and the 8x8 forms do not fit three waves without spilling).
template <typename T, int FORM, int NV>
constexpr int hop_walk_waves() {
  return (sizeof(T) == 4 && FORM == kFormMatrix && NV == 4) ? 3 : 1;
}

// Walking variant of k_hop: a block of B threads covers B * NV / 4 columns (x0, x1, x2) of the
// lattice; each thread walks K consecutive x3 values of its column.  Per step the x1 and x2 hops
// load their links and neighbours as in k_hop, the x0 hops too unless lane_x0 (then they take the
// neighbours from the other lanes of the x0 row); the x3 forward hop loads U_3(x) and phi(x+3),
// which stay in registers as the backward link and the centre field of the next step.
template <typename T, int FORM, int NV, bool DOTS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(hop_walk_waves<T, FORM, NV>())))
k_hop_walk(const HopArgs<T> A, int32_t xcd, int32_t K, int32_t tile2, int32_t lane_x0) {
  constexpr int G = 4 / NV;
  const HopBlock hb = hop_block(xcd, A.n_rhs);
  const int32_t v = hb.v;
  if (A.run && A.run[(int64_t)v * A.run_stride] == 0) return;
  const int32_t V = A.g.V;
  const int32_t P = A.g.L0 * A.g.L1 * A.g.L2;            // sites per x3 plane
  const int32_t cpb = blockDim.x / G;                    // columns per block
  const int32_t nchunk = (P + cpb - 1) / cpb;
  const int32_t lb = hb.lb;
  const int32_t chunk = lb % nchunk;
  const int32_t x3_0 = (lb / nchunk) * K;
  const int32_t grp = __builtin_amdgcn_readfirstlane(threadIdx.x / cpb);  // wave-uniform
  const int32_t tc = threadIdx.x - grp * cpb;
  int32_t col;
  if (tile2 > 1) {
    // the block's columns form an L0 x R1 x tile2 tile of the (x0, x1, x2) plane (tiles with x1
    // fastest), so its x2 neighbours are partly its own columns; hop_walk_ok checks the tiling
    const int32_t R1 = cpb / (A.g.L0 * tile2);
    const int32_t nc1 = A.g.L1 / R1;
    const int32_t c1 = chunk % nc1, c2 = chunk / nc1;
    const int32_t x0 = tc % A.g.L0, r = tc / A.g.L0;
    col = x0 + A.g.L0 * ((c1 * R1 + r % R1) + A.g.L1 * (c2 * tile2 + r / R1));
  } else {
    col = chunk * cpb + tc;
  }
  const int nu0 = grp * NV;
  double dsum[3] = {0.0, 0.0, 0.0};
  if (col < P) {
    const int64_t FV = 32 * (int64_t)V;
    const T* __restrict__ xf = A.x + ((int64_t)v * A.x_mul + A.x_add) * FV;
    const T* __restrict__ U = A.U;
    const T* __restrict__ U3 = U + (int64_t)3 * 18 * V;
    int32_t xc[4];
    site_coords(A.g, col + x3_0 * P, xc);
    // carried state: the centre field, the x-3 field and the 12 loaded reals of the link U_3(x-3)
    // (this thread's forward x3 link of the step before; row 2 is rebuilt from them each step)
    T cen[NV][8], bwd[NV][8], l3[12];
    {
      const int32_t s0 = col + x3_0 * P;
      const int32_t sb = (x3_0 == 0) ? s0 + (A.g.L3 - 1) * P : s0 - P;
      load_rows<T>(U3, sb, V, l3);
      load_field<T, NV>(xf, s0, nu0, V, cen);
      load_field<T, NV>(xf, sb, nu0, V, bwd);
    }
#pragma unroll 1
    for (int32_t t = 0; t < K; ++t) {
      const int32_t x3 = x3_0 + t;
      const int32_t s = col + x3 * P;
      xc[3] = x3;
      T acc[NV][8];
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int a = 0; a < 8; ++a) acc[i][a] = T(0);
      // x3 backward hop: carried field, link U_3(x - 3)
      {
        T u[18];
#pragma unroll
        for (int c = 0; c < 12; ++c) u[c] = l3[c];
        link_row2<T, FORM>(u);
        hop_apply<T, FORM, NV, true>(u, bwd, acc);
      }
      int32_t mu_begin = 0;
      if (lane_x0) {
        // x0 hops from the other lanes of this x0 row (a row of L0 lanes lies within the wave):
        // the field at x +- 0 is that lane's carried centre, and the backward link U_0(x - 0) is
        // the forward link that lane loads, passed as its 12 loaded reals (row 2 rebuilt here, as
        // a hop of its own does) -- the same values the loads would give, in the same order of terms
        const int32_t lane = threadIdx.x & 63;
        const int32_t x0 = xc[0];
        const int32_t row = lane - x0;
        const int32_t lp = row + (x0 + 1 == A.g.L0 ? 0 : x0 + 1);
        const int32_t lm = row + (x0 == 0 ? A.g.L0 - 1 : x0 - 1);
        T u[18], u12[12], phi[NV][8];
        load_rows<T>(U, s, V, u12);
#pragma unroll
        for (int c = 0; c < 12; ++c) u[c] = u12[c];
        link_row2<T, FORM>(u);
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int b = 0; b < 8; ++b) phi[i][b] = __shfl(cen[i][b], lp, 64);
        hop_apply<T, FORM, NV, false>(u, phi, acc);
#pragma unroll
        for (int c = 0; c < 12; ++c) u[c] = __shfl(u12[c], lm, 64);
        link_row2<T, FORM>(u);
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int b = 0; b < 8; ++b) phi[i][b] = __shfl(cen[i][b], lm, 64);
        hop_apply<T, FORM, NV, true>(u, phi, acc);
        mu_begin = 1;
      }
#pragma unroll 1
      for (int mu = mu_begin; mu < 3; ++mu) {
        const T* __restrict__ Um = U + (int64_t)mu * 18 * V;
        hop_term_fwd<T, FORM, NV>(Um, s, site_shift(A.g, s, xc, mu, +1), xf, nu0, V, acc);
        hop_term<T, FORM, NV, true>(Um, site_shift(A.g, s, xc, mu, -1), xf, nu0, V, acc);
      }
      // x3 forward hop: phi(x + 3) becomes the centre of the next step
      T fwd[NV][8];
      {
        const int32_t sf = (x3 == A.g.L3 - 1) ? s - (A.g.L3 - 1) * P : s + P;
        T u[18];
        load_rows<T>(U3, s, V, l3);
#pragma unroll
        for (int c = 0; c < 12; ++c) u[c] = l3[c];
        link_row2<T, FORM>(u);
        load_field<T, NV>(xf, sf, nu0, V, fwd);
        hop_apply<T, FORM, NV, false>(u, fwd, acc);
      }
      hop_finish<T, FORM, NV>(acc);
      hop_store<T, NV, DOTS, false, false>(A, v, xf, cen, nu0, s, A.store != 0, acc, dsum);
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          bwd[i][b] = cen[i][b];
          cen[i][b] = fwd[i][b];
        }
    }
  }
  if (DOTS) {
    __shared__ double lds[3][16];
    block_sum<3>(dsum, lds);
    if (threadIdx.x == 0) {
      const int32_t nblk = hb.nblk;
      double* p = A.partials + (int64_t)v * 3 * nblk + lb;
      if (A.dot_mask & 1) p[0] = dsum[0];
      if (A.dot_mask & 2) p[nblk] = dsum[1];
      if (A.dot_mask & 4) p[2 * nblk] = dsum[2];
    }
  }
}


// Multi-field variant of k_hop (one thread per site, all four directions): the thread applies the
// operator at its site to NS consecutive fields of the batch.  The grid is lattice blocks times field
// groups of NS, laid out as hop_block lays out fields.  Per hop the link is loaded once and its
// adjoint matrix built once for all 4 NS vectors: form 0 keeps the 8x8 matrix in registers and
// streams the fields through it one at a time (registers: the matrix, one field, the NS
// accumulators); form 2 builds each column pair once and applies it to all 4 NS vectors.  Term order
// and per-vector arithmetic are those of k_hop, so every field's result is bitwise that of k_hop with
// the same form.
template <typename T, int FORM, int NS, bool kT>
__device__ __forceinline__ void hop_term_ns(const T* __restrict__ Um, int32_t sl, int32_t sn,
                                            const T* const (&xf)[NS], int32_t V, T (&acc)[NS * 4][8]) {
  T u[18];
  load_rows<T>(Um, sl, V, u);
  if (FORM == kFormAdjoint) {
    T R[64];
    link_row2<T, FORM>(u);
    adjoint_matrix<T>(u, R);
#pragma unroll
    for (int f = 0; f < NS; ++f) {
      T phi[4][8];
      load_field<T, 4>(xf[f], sn, 0, V, phi);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!kT)
          adj_apply<T>(R, phi[i], acc[f * 4 + i]);
        else
          adj_apply_t<T>(R, phi[i], acc[f * 4 + i]);
      }
    }
  } else {
    T phi[NS * 4][8];
#pragma unroll
    for (int f = 0; f < NS; ++f)
      load_field<T, 4>(xf[f], sn, 0, V, phi + f * 4);
    link_row2<T, FORM>(u);
    adj_stream<T, NS * 4, kT>(u, phi, acc);
  }
}

template <typename T, int FORM, int NS, bool DOTS>
__global__ void __launch_bounds__(256) k_hop_ns(const HopArgs<T> A, int32_t xcd, int32_t order) {
  const int32_t ngrp = A.n_rhs / NS;
  const HopBlock hb = hop_block(xcd, ngrp);
  const int32_t v0 = hb.v * NS;
  bool runs[NS];
  bool any = false;
#pragma unroll
  for (int f = 0; f < NS; ++f) {
    runs[f] = !A.run || A.run[(int64_t)(v0 + f) * A.run_stride] != 0;
    any = any || runs[f];
  }
  if (!any) return;
  const int32_t V = A.g.V;
  const int32_t lb = hb.lb;
  const int32_t spb = blockDim.x;
  int32_t blk = lb;
  if (order) {
    const int32_t x3 = lb % A.g.L3;
    const int32_t t = lb / A.g.L3;
    const int32_t x2 = t % A.g.L2;
    const int32_t chunk = t / A.g.L2;
    const int32_t cpp = (A.g.L0 * A.g.L1) / spb;
    blk = (x3 * A.g.L2 + x2) * cpp + chunk;
  }
  const int32_t s = blk * spb + threadIdx.x;
  double dsum[NS * 3];
#pragma unroll
  for (int q = 0; q < NS * 3; ++q) dsum[q] = 0.0;
  if (s < V) {
    const int64_t FV = 32 * (int64_t)V;
    const T* xf[NS];
#pragma unroll
    for (int f = 0; f < NS; ++f) xf[f] = A.x + ((int64_t)(v0 + f) * A.x_mul + A.x_add) * FV;
    const T* __restrict__ U = A.U;
    T acc[NS * 4][8];
#pragma unroll
    for (int i = 0; i < NS * 4; ++i)
#pragma unroll
      for (int a = 0; a < 8; ++a) acc[i][a] = T(0);
    int32_t xc[4];
    site_coords(A.g, s, xc);
    // the term order of k_hop: x3 backward, then x0, x1, x2 forward and backward, x3 forward
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      const int mb = (mu + 3) & 3;
      const int32_t sb = site_shift(A.g, s, xc, mb, -1);
      hop_term_ns<T, FORM, NS, true>(U + (int64_t)mb * 18 * V, sb, sb, xf, V, acc);
      hop_term_ns<T, FORM, NS, false>(U + (int64_t)mu * 18 * V, s, site_shift(A.g, s, xc, mu, +1), xf, V, acc);
    }
#pragma unroll
    for (int f = 0; f < NS; ++f)
      hop_store<T, 4, DOTS, true, true>(A, v0 + f, xf[f], nullptr, 0, s, A.store && runs[f], acc + f * 4, dsum + f * 3);
  }
  if (DOTS) {
    __shared__ double lds[NS * 3][16];
    block_sum<NS * 3>(dsum, lds);
    if (threadIdx.x == 0) {
      const int32_t nblk = hb.nblk;
#pragma unroll
      for (int f = 0; f < NS; ++f) {
        if (!runs[f]) continue;
        double* p = A.partials + (int64_t)(v0 + f) * 3 * nblk + lb;
        if (A.dot_mask & 1) p[0] = dsum[f * 3 + 0];
        if (A.dot_mask & 2) p[nblk] = dsum[f * 3 + 1];
        if (A.dot_mask & 4) p[2 * nblk] = dsum[f * 3 + 2];
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// the tiled walk
//
// A block takes a tile of L0 x R1 x R2 columns (x0 rows whole) and walks n3 values of x3.  The tile's
// plane of the field sits in LDS, double buffered, so the x0 neighbours and those x1 and x2 neighbours
// that lie in the tile come from LDS; only the tile's edge rows read theirs from memory, where each
// halo site is read by one thread only.  What bounds the other shapes is the load path (32 bytes
// per cycle and CU, measured, from L1 and L2 alike) and the traffic past L2: 384 reals per site go
// through it in the site-per-thread shapes, 240 in the walk, 160 here.
//
// A wave is 32 columns in two halves: lanes 0-31 take directions nu = 0, 1 and lanes 32-63 nu = 2, 3 of
// the same columns, and each half loads one of the two stored rows of a link, exchanged through the
// register file (v_permlane32_swap), so a site's links are loaded once.  Two directions per
// lane keep the kernel at 220 registers in FP64: two waves per SIMD (FP64 instructions issue every 4.4
// cycles with two or more waves, every 6-9 with one).
//
// Every load is issued a hop ahead of its use (pin() keeps the compiler from moving arithmetic across
// hops, which would need more registers than there are).  The x3 hop uses its link both ways:
// U phi(x+3) U^dag for this plane, U^dag phi(x) U for the next.  The x1 and x2 hops come first in a
// step and phi(x+3) is loaded last: the halo rows of a plane were then loaded by the neighbouring blocks
// moments ago and are still in the XCD's L2 (at 32^3x64 17.6 to 18.2 M misses of 128 bytes instead of 21.0 M
// with the opposite order; 1.24 times the algorithmic bytes).
//
// Measured per application against the walk (same card, both warm): FP64 32^3x64 494 us against 568,
// 24^4 x 4 fields (recursion step) 357 against 434, 16^4 x 2 35.5 against 41.4, 16^4 x 8 115 against 123;
// FP32 32^3x64 273 against 292.  In FP64 the unit that returns loaded data is busy 89 % of the time at
// 32^3x64 (78 % at 16^4 x 8) and vector instructions issue 63 % of it (58 %).

// Keeps x in registers here: later arithmetic is not moved before, earlier not after.
template <typename T, int N>
__device__ __forceinline__ void pin(T (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}
template <typename T>
__device__ __forceinline__ void pin(T (&x)[2][8]) {
  pin(x[0]);
  pin(x[1]);
}

template <typename T>
using Vec16 = T __attribute__((ext_vector_type(16 / sizeof(T))));

// One lane's 16 reals of a column in LDS.  A column takes kTilePitch elements: 32 and 16 bytes more, so
// that the 16 lanes of a 16-byte access phase fall into distinct banks.
template <typename T>
constexpr int kTilePitch = 32 + 16 / sizeof(T);
template <typename T>
__device__ __forceinline__ void lds_get(const char* p, T (&f)[2][8]) {
  constexpr int N = 16 / sizeof(T);
  const Vec16<T>* q = (const Vec16<T>*)p;
#pragma unroll
  for (int i = 0; i < 16 / N; ++i) {
    const Vec16<T> w = q[i];
#pragma unroll
    for (int k = 0; k < N; ++k) f[(i * N + k) >> 3][(i * N + k) & 7] = w[k];
  }
}
template <typename T>
__device__ __forceinline__ void lds_put(char* p, const T (&f)[2][8]) {
  constexpr int N = 16 / sizeof(T);
  Vec16<T>* q = (Vec16<T>*)p;
#pragma unroll
  for (int i = 0; i < 16 / N; ++i) {
    Vec16<T> w;
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = f[(i * N + k) >> 3][(i * N + k) & 7];
    q[i] = w;
  }
}

// 16 rows of a field (two directions), or the 6 reals of one stored row of a link, at a byte offset
// that includes the lane half's rows.
template <typename T>
__device__ __forceinline__ void get_half(const T* base, int64_t V, uint32_t o, T (&f)[2][8]) {
  Rows<T> r(base, V, o);
#pragma unroll
  for (int i = 0; i < 16; ++i) f[i >> 3][i & 7] = r.get();
}
template <typename T, bool kOnce = false>
__device__ __forceinline__ void get_row(const T* base, int64_t V, uint32_t o, T (&u)[6]) {
  Rows<T> r(base, V, o);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    u[i] = kOnce ? __builtin_nontemporal_load(r.ptr()) : *r.ptr();
    r.next();
  }
}

// a = the value of lanes 0-31 in both halves, b = that of lanes 32-63.
__device__ __forceinline__ void both_halves(float x, float& a, float& b) {
  const uint32_t w = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]);
  b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void both_halves(double x, double& a, double& b) {
  const uint64_t w = __builtin_bit_cast(uint64_t, x);
  const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)w, (uint32_t)w, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(w >> 32), (uint32_t)(w >> 32), false, false);
  a = __builtin_bit_cast(double, (uint64_t)(uint32_t)l[0] | ((uint64_t)(uint32_t)h[0] << 32));
  b = __builtin_bit_cast(double, (uint64_t)(uint32_t)l[1] | ((uint64_t)(uint32_t)h[1] << 32));
}

// The whole link from the half rows of the two lane halves.
template <typename T>
__device__ __forceinline__ void whole_link(T (&h)[6], T (&u)[18]) {
  pin(h);
#pragma unroll
  for (int i = 0; i < 6; ++i) both_halves(h[i], u[i], u[6 + i]);
  su3_row2<T, true>(u);
}

template <typename T, bool kT>
__device__ __forceinline__ void hop_pair(const T* u, T (&f)[2][8], T (&acc)[2][8]) {
  pin(f);
  mat_hop<T, kT>(u, f[0], acc[0]);
  pin(acc[0]);
  mat_hop<T, kT>(u, f[1], acc[1]);
  pin(acc[1]);
}

template <typename T, bool DOTS, bool Z>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4)))
k_hop_tile(const HopArgs<T> A, const HopTile S, int32_t xcd) {
  extern __shared__ __align__(16) char smem[];
  const HopBlock hb = hop_block(xcd, A.n_rhs);
  const int32_t v = hb.v;
  if (A.run && A.run[(int64_t)v * A.run_stride] == 0) return;
  constexpr uint32_t SZ = sizeof(T);
  constexpr uint32_t PB = kTilePitch<T> * SZ;      // LDS bytes per column
  const int64_t V = A.g.V;
  const int32_t L0 = A.g.L0, L1 = A.g.L1, L2 = A.g.L2, L3 = A.g.L3;
  const int32_t L01 = L0 * L1;
  const int32_t lb = hb.lb;
  const int32_t ntile = S.n1 * S.n2;
  const int32_t tile = lb % ntile;
  const int32_t x3_0 = (lb / ntile) * S.K;
  const int32_t n3 = min(S.K, L3 - x3_0);
  const int32_t y1 = (tile % S.n1) * S.R1, y2 = (tile / S.n1) * S.R2;   // the tile's first row
  const int32_t m1 = min(S.R1, L1 - y1), m2 = min(S.R2, L2 - y2);       // and its rows (cut at the lattice's end)
  const int32_t h = (threadIdx.x >> 5) & 1;
  int32_t tc = (threadIdx.x >> 6) * 32 + (threadIdx.x & 31);
  int32_t x0 = tc % L0, r1 = (tc / L0) % S.R1, r2 = tc / (L0 * S.R1);
  // lanes without a column go through the motions of the tile's first one and write nothing
  const bool live = r1 < m1 && r2 < m2;
  if (!live) x0 = r1 = r2 = 0;
  const int32_t x1 = y1 + r1, x2 = y2 + r2;
  const int32_t col = x0 + L0 * (x1 + L1 * x2);
  // LDS byte offsets of the neighbours in the tile
  auto lds_at = [&](int32_t c0, int32_t c1, int32_t c2) {
    return (uint32_t)(c0 + L0 * (c1 + S.R1 * c2)) * PB + (uint32_t)h * (16 * SZ);
  };
  const uint32_t lc = lds_at(x0, r1, r2);
  const uint32_t l0p = lds_at(x0 + 1 == L0 ? 0 : x0 + 1, r1, r2), l0m = lds_at(x0 == 0 ? L0 - 1 : x0 - 1, r1, r2);
  const uint32_t l1p = lds_at(x0, r1 + 1 < m1 ? r1 + 1 : 0, r2), l1m = lds_at(x0, r1 > 0 ? r1 - 1 : m1 - 1, r2);
  const uint32_t l2p = lds_at(x0, r1, r2 + 1 < m2 ? r2 + 1 : 0), l2m = lds_at(x0, r1, r2 > 0 ? r2 - 1 : m2 - 1);
  // a tile that spans the lattice in a direction holds all its neighbours there
  const bool i1p = r1 + 1 < m1 || m1 == L1, i1m = r1 > 0 || m1 == L1;
  const bool i2p = r2 + 1 < m2 || m2 == L2, i2m = r2 > 0 || m2 == L2;
  // byte offsets in a component of the global neighbours in the plane x3 = 0, and of the lane half's rows
  const uint32_t gc = (uint32_t)col * SZ;
  const uint32_t g0m = (uint32_t)(col + (x0 == 0 ? L0 - 1 : -1)) * SZ;
  const uint32_t g1p = (uint32_t)(col + (x1 + 1 == L1 ? L0 - L01 : L0)) * SZ;
  const uint32_t g1m = (uint32_t)(col + (x1 == 0 ? L01 - L0 : -L0)) * SZ;
  const uint32_t g2p = (uint32_t)(col + (x2 + 1 == L2 ? (1 - L2) * L01 : L01)) * SZ;
  const uint32_t g2m = (uint32_t)(col + (x2 == 0 ? (L2 - 1) * L01 : -L01)) * SZ;
  const uint32_t hf = (uint32_t)h * (uint32_t)(16 * V * SZ), hl = (uint32_t)h * (uint32_t)(6 * V * SZ);
  const uint32_t plane = (uint32_t)(L01 * L2) * SZ;
  const int64_t FV = 32 * V;
  const T* __restrict__ xf = A.x + ((int64_t)v * A.x_mul + A.x_add) * FV;
  const T* __restrict__ U0 = A.U;
  const T* __restrict__ U1 = U0 + 18 * V;
  const T* __restrict__ U2 = U0 + 36 * V;
  const T* __restrict__ U3 = U0 + 54 * V;
  const T ca = T(A.a), cb = T(A.b_rhs ? A.b_rhs[v] : A.b), cc = T(A.c);
  const T* zf = Z ? A.z + (int64_t)(v / A.z_div) * FV : nullptr;   // may alias out
  T* outf = A.out + (int64_t)v * FV;
  HopRing<T> rf{nullptr, nullptr};
  if (DOTS && !Z) rf = hop_ring_field(A, v);
  const uint32_t buf = (uint32_t)(S.R1 * S.R2 * L0) * PB;          // one plane of the tile in LDS
  double dsum[3] = {0.0, 0.0, 0.0};
  uint32_t pl = (uint32_t)x3_0 * plane;
  // acc: this plane's result; p, q, r: fields; la, lb2: link half rows; u: a link
  T acc[2][8], p[2][8], q[2][8], r[2][8], la[6], lb2[6], u[18];
  {
    // the first plane into LDS, and its x3 backward hop
    const uint32_t pb = (uint32_t)(x3_0 == 0 ? L3 - 1 : x3_0 - 1) * plane;
    get_half(xf, V, hf + gc + pl, r);
    get_row(U3, V, hl + gc + pb, la);
    get_half(xf, V, hf + gc + pb, q);
    get_row(U1, V, hl + gc + pl, lb2);
    pin(r);
    if (live) lds_put<T>(smem + lc, r);
#pragma unroll
    for (int a = 0; a < 8; ++a) acc[0][a] = acc[1][a] = T(0);
    whole_link(la, u);
    hop_pair<T, true>(u, q, acc);
#pragma unroll
    for (int i = 0; i < 6; ++i) la[i] = lb2[i];
  }
  __syncthreads();
#pragma unroll 1
  for (int32_t t = 0; t < n3; ++t) {
    const int32_t x3 = x3_0 + t;
    const char* cur = smem + (t & 1 ? buf : 0u);
    char* nxt = smem + (t & 1 ? 0u : buf);
    const uint32_t pf = (uint32_t)(x3 + 1 == L3 ? 0 : x3 + 1) * plane;
    // a neighbour: from the tile in LDS or, for an edge row, from memory
    auto near = [&](bool in, uint32_t l, uint32_t g, T (&f)[2][8]) {
      if (in)
        lds_get<T>(cur + l, f);
      else
        get_half(xf, V, hf + g + pl, f);
    };
    near(i1p, l1p, g1p, r);
    near(i1m, l1m, g1m, q);
    get_row(U1, V, hl + g1m + pl, lb2);
    whole_link(la, u);
    hop_pair<T, false>(u, r, acc);    // x1 forward
    get_row(U2, V, hl + gc + pl, la);
    near(i2p, l2p, g2p, r);
    whole_link(lb2, u);
    hop_pair<T, true>(u, q, acc);     // x1 backward
    get_row(U2, V, hl + g2m + pl, lb2);
    near(i2m, l2m, g2m, q);
    whole_link(la, u);
    hop_pair<T, false>(u, r, acc);    // x2 forward
    get_row(U0, V, hl + gc + pl, la);
    lds_get<T>(cur + l0p, r);
    whole_link(lb2, u);
    hop_pair<T, true>(u, q, acc);     // x2 backward
    get_row(U0, V, hl + g0m + pl, lb2);
    lds_get<T>(cur + l0m, q);
    get_half(xf, V, hf + gc + pf, p);
    whole_link(la, u);
    hop_pair<T, false>(u, r, acc);    // x0 forward
    get_row<T, true>(U3, V, hl + gc + pl, la);
    lds_get<T>(cur + lc, r);
    whole_link(lb2, u);
    hop_pair<T, true>(u, q, acc);     // x0 backward
    if (Z) {
      Rows<T> zr(zf, V, hf + gc + pl);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        q[i >> 3][i & 7] = A.z_div == 1 ? __builtin_nontemporal_load(zr.ptr()) : *zr.ptr();
        zr.next();
      }
    }
    if (DOTS && !Z && rf) {
      if (sizeof(T) == 4 && rf.ru) {
        Rows<double> rr(rf.ru, V, 2 * (hf + gc + pl));   // (at most 34 V bytes of FP32, 2^24 sites)
#pragma unroll
        for (int i = 0; i < 16; ++i) q[i >> 3][i & 7] = (T)rr.get();
      } else {
        get_half(rf.r, V, hf + gc + pl, q);
      }
    }
    whole_link(la, u);
    hop_pair<T, false>(u, p, acc);    // x3 forward; phi(x+3) is the next plane
    if (live) lds_put<T>(nxt + lc, p);
    T back[2][8];
#pragma unroll
    for (int a = 0; a < 8; ++a) back[0][a] = back[1][a] = T(0);
    hop_pair<T, true>(u, r, back);    // the next plane's x3 backward hop
    if (t + 1 < n3) get_row(U1, V, hl + gc + pf, la);
    mat_components<T>(acc[0]);
    mat_components<T>(acc[1]);
    T w[2][8];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      T o = fmadd(ca, acc[i >> 3][i & 7], cb * r[i >> 3][i & 7]);
      if (Z) o = fmadd(cc, q[i >> 3][i & 7], o);
      w[i >> 3][i & 7] = o;
      if (DOTS && live) {
        const double xd = (double)r[i >> 3][i & 7], od = (double)o;
        dsum[0] = !Z && rf ? fma(od, (double)q[i >> 3][i & 7], dsum[0]) : fma(xd, xd, dsum[0]);
        dsum[1] = fma(od, xd, dsum[1]);
        dsum[2] = fma(od, od, dsum[2]);
      }
    }
    if constexpr (!DOTS && Z && sizeof(T) == 8) {
      if (A.src && v < A.src_rhs) {
        for (int32_t y = 0; y < A.src_n; ++y) {
          const double c = A.src_coef[((int64_t)v * A.src_n + y) * A.src_stride];
          T yv[2][8];
          get_half(A.src + ((int64_t)y * A.src_rhs + v) * FV, V, hf + gc + pl, yv);
#pragma unroll
          for (int i = 0; i < 16; ++i) w[i >> 3][i & 7] = fma(c, yv[i >> 3][i & 7], w[i >> 3][i & 7]);
        }
      }
    }
    if (A.store && live) {
      Rows<T> outr(outf, V, hf + gc + pl);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        __builtin_nontemporal_store(w[i >> 3][i & 7], outr.ptr());
        outr.next();
      }
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      acc[0][a] = back[0][a];
      acc[1][a] = back[1][a];
    }
    pl = pf;
    // the next plane is complete in nxt, and nobody reads cur any more
    __syncthreads();
  }
  if (DOTS) {
    double(*lds)[16] = (double(*)[16])smem;
    block_sum<3>(dsum, lds);
    if (threadIdx.x == 0) {
      const int32_t nblk = hb.nblk;
      double* pp = A.partials + (int64_t)v * 3 * nblk + lb;
      if (A.dot_mask & 1) pp[0] = dsum[0];
      if (A.dot_mask & 2) pp[nblk] = dsum[1];
      if (A.dot_mask & 4) pp[2 * nblk] = dsum[2];
    }
  }
}

static int hop_tile_blocks(const Geom& g, const HopTile& t) { return t.n1 * t.n2 * ((g.L3 + t.K - 1) / t.K); }

// The tile of a configuration: cfg.tile2 rows of x2 and as many rows of x1 as cfg.block columns
// allow, evened out over the lattice; segments of cfg.walk planes, the last one shorter where
// walk does not divide L3.
bool hop_tile_of(const Geom& g, const HopConfig& cfg, HopTile* t) {
  if (cfg.order != 1 || cfg.walk < 1 || cfg.form != kFormMatrix || cfg.nv != 2 || cfg.ns != 1) return false;
  // byte offsets of half a field (17 V elements of 8 bytes) fit 32 bits; a row of columns fits a block
  if (g.V > (1 << 24) || g.L0 > cfg.block) return false;
  t->R2 = std::min<int32_t>(cfg.tile2, g.L2);
  while (g.L0 * t->R2 > cfg.block) --t->R2;
  t->R1 = std::min<int32_t>(cfg.block / (g.L0 * t->R2), g.L1);
  t->n1 = (g.L1 + t->R1 - 1) / t->R1;
  t->R1 = (g.L1 + t->n1 - 1) / t->n1;
  t->n2 = (g.L2 + t->R2 - 1) / t->R2;
  t->R2 = (g.L2 + t->n2 - 1) / t->n2;
  t->K = std::min(cfg.walk, g.L3);
  // small extents can leave a tile a handful of columns (4x3x6x7 in single rows and planes: 42 blocks of 12
  // sites), and the buffers of the partial sums hold hop_max_blocks: such a launch runs as if there were no tile
  return hop_tile_blocks(g, *t) <= hop_max_blocks(g);
}

template <typename T>
static hipError_t launch_hop_tile(const HopArgs<T>& A, const HopTile& t, int32_t xcd, dim3 grid, hipStream_t s) {
  const int32_t columns = A.g.L0 * t.R1 * t.R2;
  dim3 block((columns + 31) / 32 * 64);
  // two planes; the block sums of the dot products use the same memory at the end
  const size_t lds = std::max<size_t>(2 * (size_t)columns * kTilePitch<T> * sizeof(T), 3 * 16 * sizeof(double));
  const bool dots = A.partials && A.dot_mask;
  if (dots && A.z)
    hipLaunchKernelGGL((k_hop_tile<T, true, true>), grid, block, lds, s, A, t, xcd);
  else if (dots)
    hipLaunchKernelGGL((k_hop_tile<T, true, false>), grid, block, lds, s, A, t, xcd);
  else if (A.z)
    hipLaunchKernelGGL((k_hop_tile<T, false, true>), grid, block, lds, s, A, t, xcd);
  else
    hipLaunchKernelGGL((k_hop_tile<T, false, false>), grid, block, lds, s, A, t, xcd);
  return hipGetLastError();
}

int hop_walk_ok(const Geom& g, const HopConfig& cfg) {
  if (!(cfg.walk > 0 && (g.L3 % cfg.walk) == 0)) return 0;
  if (cfg.tile2 > 1) {
    // an L0 x R1 x tile2 column tile per block that tiles the (x0, x1, x2) plane exactly
    const int cpb = cfg.block * cfg.nv / 4;
    if (cpb % (g.L0 * cfg.tile2) || g.L2 % cfg.tile2) return 0;
    const int R1 = cpb / (g.L0 * cfg.tile2);
    if (R1 < 1 || g.L1 % R1) return 0;
  }
  return 1;
}

int hop_ns_ok(const HopConfig& cfg, int32_t n_rhs) {
  return (cfg.ns > 1 && n_rhs % cfg.ns == 0 && cfg.nv == 4 && cfg.walk == 0 && (cfg.order == 0 || cfg.order == 1) &&
          (cfg.form == kFormAdjoint || cfg.form == kFormStream))
             ? 1
             : 0;
}

// hop-split shape (order 2, or 3 with the x3-fastest block order): each wave covers 16 sites
// of one direction group
int hop_split_ok(const HopConfig& cfg) {
  return ((cfg.order == 2 || cfg.order == 3) && (cfg.block / 64) % (4 / cfg.nv) == 0) ? 1 : 0;
}
static int hop_split_spb(const HopConfig& cfg) { return (cfg.block / 64) / (4 / cfg.nv) * 16; }

bool hop_ring_ok(const Geom& g, const HopConfig& cfg, int bytes) {
  HopTile tile;
  if (hop_tile_of(g, cfg, &tile)) return true;
  if (hop_split_ok(cfg)) return bytes == 8 || cfg.form == kFormMatrix;
  return !hop_walk_ok(g, cfg);
}

int hop_num_blocks(const Geom& g, const HopConfig& cfg) {
  HopTile tile;
  if (hop_tile_of(g, cfg, &tile)) return hop_tile_blocks(g, tile);
  if (hop_split_ok(cfg)) {
    const int spb = hop_split_spb(cfg);
    return (g.V + spb - 1) / spb;
  }
  const int spb = cfg.block * cfg.nv / 4;
  if (hop_walk_ok(g, cfg)) {
    const int P = g.L0 * g.L1 * g.L2;
    return ((P + spb - 1) / spb) * (g.L3 / cfg.walk);
  }
  return (g.V + spb - 1) / spb;
}

int hop_order_ok(const Geom& g, const HopConfig& cfg) {
  const int spb = hop_split_ok(cfg) ? hop_split_spb(cfg) : cfg.block * cfg.nv / 4;
  return ((g.L0 * g.L1) % spb) == 0 ? 1 : 0;
}

template <typename T, int FORM, int NV>
static hipError_t launch_hop_form(const HopArgs<T>& A, const HopConfig& cfg, hipStream_t s) {
  const int64_t nblk = hop_num_blocks(A.g, cfg);
  // one-dimensional grid, fields fastest (hop_block)
  if (nblk * A.n_rhs > 0x7fffffff) return hipErrorInvalidValue;
  dim3 grid((uint32_t)(nblk * A.n_rhs)), block(cfg.block);
  const bool dots = A.partials && A.dot_mask;
  // the partial-sum buffers hold hop_max_blocks entries per field and dot product
  if (dots && nblk > hop_max_blocks(A.g)) return hipErrorInvalidValue;
  if constexpr (NV == 4 && FORM != kFormMatrix) {
    if (hop_ns_ok(cfg, A.n_rhs)) {
      const int32_t ord = (cfg.order == 1 && hop_order_ok(A.g, cfg)) ? 1 : 0;
      dim3 g2((uint32_t)(nblk * (A.n_rhs / cfg.ns)));
      if (cfg.ns == 2) {
        if (dots)
          hipLaunchKernelGGL((k_hop_ns<T, FORM, 2, true>), g2, block, 0, s, A, cfg.xcd_remap, ord);
        else
          hipLaunchKernelGGL((k_hop_ns<T, FORM, 2, false>), g2, block, 0, s, A, cfg.xcd_remap, ord);
      } else if (cfg.ns == 4) {
        // four fields per thread: FP32 only (the FP64 kernel would spill)
        if constexpr (sizeof(T) == 4) {
          if (dots)
            hipLaunchKernelGGL((k_hop_ns<T, FORM, 4, true>), g2, block, 0, s, A, cfg.xcd_remap, ord);
          else
            hipLaunchKernelGGL((k_hop_ns<T, FORM, 4, false>), g2, block, 0, s, A, cfg.xcd_remap, ord);
        } else {
          return hipErrorInvalidValue;
        }
      } else {
        return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
  }
  if constexpr (NV == 2 && FORM == kFormMatrix) {
    HopTile tile;
    if (hop_tile_of(A.g, cfg, &tile)) return launch_hop_tile<T>(A, tile, cfg.xcd_remap, grid, s);
  }
  if (hop_split_ok(cfg)) {
    const int32_t ord = (cfg.order == 3 && hop_order_ok(A.g, cfg)) ? 1 : 0;
    if (dots)
      hipLaunchKernelGGL((k_hop_split<T, FORM, NV, true>), grid, block, 0, s, A, cfg.xcd_remap, ord);
    else
      hipLaunchKernelGGL((k_hop_split<T, FORM, NV, false>), grid, block, 0, s, A, cfg.xcd_remap, ord);
    return hipGetLastError();
  }
  const int32_t order = (cfg.order == 1 && hop_order_ok(A.g, cfg)) ? 1 : 0;
  if (hop_walk_ok(A.g, cfg)) {
    const int32_t K = cfg.walk;
    // the x0 rows lie whole within a wave (L0 divides 64 and the columns per block): their x0
    // neighbours come from other lanes instead of the caches
    const int32_t cpb = cfg.block * cfg.nv / 4;
    const int32_t lane_x0 = (64 % A.g.L0 == 0 && cpb % A.g.L0 == 0) ? 1 : 0;
    if (dots)
      hipLaunchKernelGGL((k_hop_walk<T, FORM, NV, true>), grid, block, 0, s, A, cfg.xcd_remap, K, cfg.tile2, lane_x0);
    else
      hipLaunchKernelGGL((k_hop_walk<T, FORM, NV, false>), grid, block, 0, s, A, cfg.xcd_remap, K, cfg.tile2,
                         lane_x0);
    return hipGetLastError();
  }
  if (dots)
    hipLaunchKernelGGL((k_hop<T, FORM, NV, true>), grid, block, 0, s, A, cfg.xcd_remap, order);
  else
    hipLaunchKernelGGL((k_hop<T, FORM, NV, false>), grid, block, 0, s, A, cfg.xcd_remap, order);
  return hipGetLastError();
}

template <typename T, int FORM>
static hipError_t launch_hop_nv(const HopArgs<T>& A, const HopConfig& cfg, hipStream_t s) {
  if (cfg.nv == 1) {
    // one direction per thread: only the 3x3 form, whose work does not repeat across directions
    if constexpr (FORM == kFormMatrix) return launch_hop_form<T, FORM, 1>(A, cfg, s);
    return hipErrorInvalidValue;
  }
  if (cfg.nv == 2) return launch_hop_form<T, FORM, 2>(A, cfg, s);
  if (cfg.nv == 4) return launch_hop_form<T, FORM, 4>(A, cfg, s);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_hop(const HopArgs<T>& A, const HopConfig& cfg, hipStream_t s) {
  if (A.n_rhs == 0 || A.g.V == 0) return hipSuccess;
  if (A.ring && (A.z || !A.run || A.ring_slots < 1 || !hop_ring_ok(A.g, cfg, sizeof(T)))) return hipErrorInvalidValue;
  if (A.src && (sizeof(T) != 8 || A.dot_mask || !A.z || !hop_ring_ok(A.g, cfg, sizeof(T)))) return hipErrorInvalidValue;
  if (cfg.form == kFormMatrix) return launch_hop_nv<T, kFormMatrix>(A, cfg, s);
  if (cfg.form == kFormAdjoint) return launch_hop_nv<T, kFormAdjoint>(A, cfg, s);
  return launch_hop_nv<T, kFormStream>(A, cfg, s);
}
template hipError_t launch_hop<double>(const HopArgs<double>&, const HopConfig&, hipStream_t);
template hipError_t launch_hop<float>(const HopArgs<float>&, const HopConfig&, hipStream_t);

}  // namespace rmh
