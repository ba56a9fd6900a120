// kernels.hip -- gfx950 kernels of libcsmap.
//
// Hot path (paper Sec. II.A, Eq. (1)-(2), summed over every segment for every
// pixel of the HEALPix sky of Sec. II.D):
//
//   precompute : per segment, P = origin + x_rel, R = |P|, the light-cone slab
//                test eta_lo <= eta0 - R < eta_hi, eps, and the per-segment
//                constants of the pair formula, all in FP64; kept segments
//                are compacted in their original order.
//   forward    : one wavefront owns a tile of 64*K consecutive RING pixels
//                (K per lane), computes their directions in-kernel, and
//                streams the segment records of every box the tile sees
//                through scalar registers: each record is fetched once per
//                wavefront with scalar loads and used by all 64 lanes.
//   adjoint    : the transpose -- one lane owns one segment, pixels stream
//                through scalar registers -- so a segment's 13 running sums
//                stay in its lane and no cross-lane reduction is needed in
//                the loop; partial sums of pixel chunks are combined by a
//                separate kernel in a fixed order.
//
// Pair formula.  With d = R n - P = R (n - Ph), Ph = P/R, and
// m = (Xdot.d') b - a (X'.d'), d' = n - Ph, a = n.X', b = 1 + n.Xdot,
// Eq. (1)-(2) give the summand -4 eps dsigma (u.d)/|d|^2 = kappa m/(b q),
// q = |n - Ph|^2, kappa = -4 eps dsigma / R.  Since n and Ph are unit
// vectors, q = 2 w with w = 1 - n.Ph, and
//   kappa/2 * (Xdot.d') = kappa/2 * b - kappa/2 (1 + Ph.Xdot)
//   kappa/2 * (X'.d')   = kappa/2 * a - kappa/2 (Ph.X')
// so the FP32 form needs only the three dot products n.Ph, n.X', n.Xdot per
// pair and two per-segment constants.  That form loses accuracy as w -> 0
// (cancellation in 1 - n.Ph), so pairs with w below a threshold take the
// direction difference n - Ph in FP64 instead.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "healpix_dev.h"
#include "internal.h"
#include "segment_dev.h"

namespace csmap {

// Pixel visibility of a box (decided in FP64 with a fixed operation order).
__device__ __forceinline__ bool sees_box(double nx, double ny, double nz, const DevBox& bx,
                                         double eta0) {
  if (bx.vis == 0) return true;
  if (bx.vis == 2) {
    const double dot = (nx * bx.cap_dir[0] + ny * bx.cap_dir[1]) + nz * bx.cap_dir[2];
    return dot >= bx.cap_cos;
  }
  const double r_lo = eta0 - bx.eta_hi;
  const double r_hi = eta0 - bx.eta_lo;
  const double n3[3] = {nx, ny, nz};
  double t_in = 0.0, t_out = __builtin_inf();
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double lo = bx.origin[k];
    const double hi = bx.origin[k] + bx.ext[k];
    if (n3[k] == 0.0) {
      if (lo > 0.0 || hi < 0.0) return false;
      continue;
    }
    const double ta = lo / n3[k];
    const double tb = hi / n3[k];
    const double tmin = (ta < tb) ? ta : tb;
    const double tmax = (ta < tb) ? tb : ta;
    if (tmin > t_in) t_in = tmin;
    if (tmax < t_out) t_out = tmax;
  }
  return (t_in <= t_out) && (t_out > r_lo) && (t_in <= r_hi);
}

// ---------------------------------------------------------------------------
// Precompute: count kept segments per block, scan per box, emit records.
// ---------------------------------------------------------------------------
// Thread t of a block handles segments base + t + kPreThreads j, j < 4, so
// that every pass of the wavefront reads consecutive segments; the four
// segments' loads are in flight together.
constexpr int kPrePer = kPreBlock / kPreThreads;

// The pixel tests a block still needs are queued in LDS and run with every
// lane busy, rather than by the few lanes of each wavefront that need them.
// The few directions that neither the caps nor the edge planes settle
// (about 0.3% of the segments of a stacked grid) are queued in LDS by their
// position in the block and tested once the block's segments are done: their
// geometry is formed again and ang2pix runs with every lane busy.  Queuing
// positions rather than event coordinates keeps the block's LDS at 4 KB.
// A block belongs to one box, so its storage type and kind are uniform: the
// body is specialised on them, and the common case (positions stored, not
// slab-start snapshots) requests all of a thread's positions before using
// any of them.
struct PreShared {
  unsigned long long flags[kPreWords];
  int qpos[kPreBlock];
  int nq;
  ConeTest cone;
};

__device__ __forceinline__ void pre_keep(const PreArgs& A, const DevBox& bx, PreShared& sh,
                                         const SegGeom& g, int pos, bool& keep) {
  keep = g.keep;
  if (keep && A.flat_on) {
    const double D = (A.flat_dir[0] * g.P[0] + A.flat_dir[1] * g.P[1]) + A.flat_dir[2] * g.P[2];
    keep = (D > 0.0) && (D > A.flat_cos * g.R);
  }
  if (keep && bx.cone_nside > 0) {
    const int st = cone_state(sh.cone, g);
    keep = st == 1;
    if (st == 2) sh.qpos[atomicAdd(&sh.nq, 1)] = pos;
  }
}

template <typename T>
__device__ __forceinline__ void pre_count_pos(const PreArgs& A, const DevBox& bx, PreShared& sh,
                                              const T* x, int64_t base) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Indices past the box's end read its last segment (a block of the box
  // starts below n) and are not used: the loads carry no branch and are all
  // in flight together.
  T v[kPrePer][3];
#pragma unroll
  for (int j = 0; j < kPrePer; ++j) {
    const int64_t i = base + threadIdx.x + kPreThreads * j;
    const int64_t ic = i < bx.n ? i : bx.n - 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) v[j][k] = x[3 * ic + k];
  }
#pragma unroll
  for (int j = 0; j < kPrePer; ++j) {
    const int pos = threadIdx.x + kPreThreads * j;
    bool keep = false;
    if (base + pos < bx.n) {
      const double xd[3] = {(double)v[j][0], (double)v[j][1], (double)v[j][2]};
      pre_keep(A, bx, sh, seg_pos_at(bx, xd, A.eta0), pos, keep);
    }
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) sh.flags[(kPreThreads / 64) * j + wave] = bal;
  }
}

__device__ __forceinline__ void pre_count_snap(const PreArgs& A, const DevBox& bx, PreShared& sh,
                                               const char* raw, int64_t base) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int j = 0; j < kPrePer; ++j) {
    const int pos = threadIdx.x + kPreThreads * j;
    bool keep = false;
    if (base + pos < bx.n) pre_keep(A, bx, sh, seg_geom(bx, raw, base + pos, A.eta0), pos, keep);
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) sh.flags[(kPreThreads / 64) * j + wave] = bal;
  }
}

__global__ void __launch_bounds__(kPreThreads) k_pre_count(PreArgs A) {
  const int64_t blk = blockIdx.x;
  const int b = ((ci32p)A.blk_box)[blk];
  const DevBox bx = load_box(A.boxes, b);
  const int64_t base = (blk - bx.blk_off) * kPreBlock;
  const char* raw = (const char*)A.raw + A.raw_byte_off[b];
  __shared__ PreShared sh;
  if (threadIdx.x == 0) sh.nq = 0;
  if (bx.cone_nside > 0) load_cone(A.boxes, b, sh.cone);
  __syncthreads();
  if (bx.snapshot) pre_count_snap(A, bx, sh, raw, base);
  else if (bx.dtype == 0) pre_count_pos(A, bx, sh, (const float*)raw, base);
  else pre_count_pos(A, bx, sh, (const double*)raw, base);
  __syncthreads();
  for (int q = threadIdx.x; q < sh.nq; q += kPreThreads) {
    const int pos = sh.qpos[q];
    const SegGeom g = bx.snapshot ? seg_geom(bx, raw, base + pos, A.eta0)
                                  : seg_pos(bx, raw, base + pos, A.eta0);
    if (ang2pix_ring(bx.cone_nside, g.P[0], g.P[1], g.P[2]) == bx.cone_pix)
      atomicOr(&sh.flags[pos >> 6], 1ull << (pos & 63));
  }
  __syncthreads();
  if (threadIdx.x < kPreWords) {
    const unsigned long long w = sh.flags[threadIdx.x];
    A.blk_mask[blk * kPreWords + threadIdx.x] = w;
    int c = __popcll(w);
#pragma unroll
    for (int off = 1; off < kPreWords; off <<= 1) c += __shfl_xor(c, off);
    if (threadIdx.x == 0) A.blk_count[blk] = c;
  }
}

// Position of the set bit of rank r (0-based) in a 64-bit word holding more
// than r set bits.
__device__ __forceinline__ int select_bit(uint64_t w, int r) {
  int pos = 0;
#pragma unroll
  for (int width = 32; width >= 1; width >>= 1) {
    const int c = __popcll(w & ((1ull << width) - 1ull));
    if (r >= c) {
      r -= c;
      w >>= width;
      pos += width;
    }
  }
  return pos;
}

// One workgroup per box: exclusive prefix of the block counts of the box.
__global__ void __launch_bounds__(256) k_pre_scan(PreArgs A, int64_t nbox) {
  const int b = blockIdx.x;
  if (b >= nbox) return;
  const DevBox bx = A.boxes[b];
  const int64_t nb = (bx.n + kPreBlock - 1) / kPreBlock;
  __shared__ int64_t sh[256];
  int64_t running = 0;
  for (int64_t c0 = 0; c0 < nb; c0 += 256) {
    const int64_t k = c0 + threadIdx.x;
    const int64_t v = (k < nb) ? (int64_t)A.blk_count[bx.blk_off + k] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
      const int64_t add = (threadIdx.x >= (unsigned)off) ? sh[threadIdx.x - off] : 0;
      __syncthreads();
      sh[threadIdx.x] += add;
      __syncthreads();
    }
    if (k < nb) A.blk_prefix[bx.blk_off + k] = running + sh[threadIdx.x] - v;
    const int64_t tot = sh[255];
    __syncthreads();
    running += tot;
  }
  if (threadIdx.x == 0) {
    A.box_count[b].kept = running;
    A.box_count[b].pad = 0;
  }
}

// Records by rank: record li of box b (li < kept) is the kept segment of
// rank li among the box's segments in index order.  Its block k is the last
// with exclusive prefix <= li; its rank inside the block selects a set bit of
// the block's keep flags.  A thread writes records base + t + kPreThreads j,
// j < 4, so consecutive threads write consecutive records.
__device__ __forceinline__ void emit_record(const PreArgs& A, const DevBox& bx, const char* raw,
                                            int64_t li, int64_t k0);

// Last block k in [lo, hi] with pre[k] <= li (pre[lo] <= li must hold).
__device__ __forceinline__ int64_t block_of_rank(const int64_t* pre, int64_t lo, int64_t hi,
                                                 int64_t li) {
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= li) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The workgroup's records (ranks base .. base + kPreBlock - 1) come from a
// short run of consecutive source blocks: two searches over the box's block
// prefixes find the run, whose prefixes are then staged in LDS, and each
// record's block is found there (a run longer than the staging buffer is
// searched in global memory, within the run).
constexpr int kEmitStage = 1024;

__global__ void __launch_bounds__(kPreThreads) k_pre_emit(PreArgs A) {
  const int64_t blk = blockIdx.x;
  const int b = ((ci32p)A.blk_box)[blk];
  const DevBox bx = load_box(A.boxes, b);
  const int64_t kept = load_kept(A.box_count, b);
  const int64_t base = (blk - bx.blk_off) * kPreBlock;
  if (base >= kept) return;
  const char* raw = (const char*)A.raw + A.raw_byte_off[b];
  const int64_t nb = (bx.n + kPreBlock - 1) / kPreBlock;
  const int64_t* pre = A.blk_prefix + bx.blk_off;
  const int64_t last = (base + kPreBlock < kept ? base + kPreBlock : kept) - 1;
  __shared__ int64_t run[2];
  __shared__ int64_t spre[kEmitStage];
  if (threadIdx.x < 2) run[threadIdx.x] = block_of_rank(pre, 0, nb - 1, threadIdx.x ? last : base);
  __syncthreads();
  const int64_t r0 = run[0], r1 = run[1];
  const bool staged = r1 - r0 < kEmitStage;
  if (staged)
    for (int64_t k = threadIdx.x; k <= r1 - r0; k += kPreThreads) spre[k] = pre[r0 + k];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPrePer; ++j) {
    const int64_t li = base + threadIdx.x + kPreThreads * j;
    if (li < kept) {
      int64_t k0;
      if (staged) {
        int lo = 0, hi = (int)(r1 - r0);
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (spre[mid] <= li) lo = mid;
          else hi = mid - 1;
        }
        k0 = r0 + lo;
      } else {
        k0 = block_of_rank(pre, r0, r1, li);
      }
      emit_record(A, bx, raw, li, k0);
    }
  }
}

// Record li, from the kept segment of rank li - pre[k0] in block k0.
__device__ __forceinline__ void emit_record(const PreArgs& A, const DevBox& bx, const char* raw,
                                            int64_t li, int64_t k0) {
  const int64_t* pre = A.blk_prefix + bx.blk_off;
  int rank = (int)(li - pre[k0]);
  // The block's keep flags are requested together (128 contiguous bytes)
  // and scanned in registers.
  const uint64_t* mask = A.blk_mask + (bx.blk_off + k0) * kPreWords;
  uint64_t mw[kPreWords];
#pragma unroll
  for (int w = 0; w < kPreWords; ++w) mw[w] = mask[w];
  int word = 0;
  uint64_t bits = mw[0];
  bool found = false;
#pragma unroll
  for (int w = 0; w < kPreWords; ++w) {
    const int c = __popcll(mw[w]);
    if (!found) {
      if (rank < c || w == kPreWords - 1) {
        found = true;
        word = w;
        bits = mw[w];
      } else {
        rank -= c;
      }
    }
  }
  const int64_t i = k0 * kPreBlock + word * 64 + select_bit(bits, rank);
  if (i >= bx.n) return;   // unreachable when the counts and flags agree
  const SegGeom g = seg_geom(bx, raw, i, A.eta0);
  const int64_t r = bx.rec_off + li;
  double Ph[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) Ph[k] = g.P[k] / g.R;
  const double kappa = -4.0 * g.eps * g.ds / g.R;
  A.orig_index[r] = (int32_t)i;
  if (A.rec32) {
    const double kh = 0.5 * kappa;
    const double pv = (Ph[0] * g.V[0] + Ph[1] * g.V[1]) + Ph[2] * g.V[2];
    const double pt = (Ph[0] * g.T[0] + Ph[1] * g.T[1]) + Ph[2] * g.T[2];
    float4* o = (float4*)(A.rec32 + (size_t)r * kRec32);
    o[0] = make_float4((float)Ph[0], (float)Ph[1], (float)Ph[2], (float)g.T[0]);
    o[1] = make_float4((float)g.T[1], (float)g.T[2], (float)g.V[0], (float)g.V[1]);
    o[2] = make_float4((float)g.V[2], (float)kh, (float)(kh * (1.0 + pv)), (float)(kh * pt));
    const double vv = (g.V[0] * g.V[0] + g.V[1] * g.V[1]) + g.V[2] * g.V[2];
    const float force_near = (1.0 - sqrt(vv) < 0.05) ? 1.0f : 0.0f;
    o[3] = make_float4(__int_as_float((int)i), force_near, 0.f, 0.f);
    if (A.recm) {
      const double k = fabs(kh), root = sqrt(k), h = 0.5 * root * pt;
      // Beyond these bounds parts of the split rows leave FP32's exponents.
      const bool odd = !(k < 0x1p100) || (k < 0x1p-100 && k != 0.0);
      float4* m = (float4*)(A.recm + (size_t)r * kRecM);
      m[0] = make_float4((float)(k * g.V[0]), (float)(k * g.V[1]), (float)(k * g.V[2]),
                         (float)(1.0 + pv));
      m[1] = make_float4((float)(root * g.T[0]), (float)(root * g.T[1]), (float)(root * g.T[2]),
                         (float)h);
      m[2] = make_float4((float)(h * h), k != 0.0 ? (float)(1.0 / k) : 0.f,
                         kh < 0.0 ? -1.f : 1.f, (odd || force_near != 0.f) ? 1.f : 0.f);
    }
    if (A.adjc) {
      // The adjoint's constants, without kappa (every adjoint sum is linear
      // in kappa, which the finalize step applies in FP64).
      ((float4*)A.adjc)[r] = make_float4((float)(1.0 + pv), (float)pt, 0.f, 0.f);
    }
    double2* h = (double2*)(A.phat64 + (size_t)r * 4);
    h[0] = make_double2(Ph[0], Ph[1]);
    h[1] = make_double2(Ph[2], g.R);
  }
  if (A.rec64) {
    double2* o = (double2*)(A.rec64 + (size_t)r * kRec64);
    o[0] = make_double2(Ph[0], Ph[1]);
    o[1] = make_double2(Ph[2], g.T[0]);
    o[2] = make_double2(g.T[1], g.T[2]);
    o[3] = make_double2(g.V[0], g.V[1]);
    o[4] = make_double2(g.V[2], kappa);
    // P/R carried as an unevaluated sum hi + lo: lo is the exact remainder
    // of the rounded quotient divided by R, so that n - P/R can be formed
    // accurately for directions close to the event.
    double lo[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) lo[k] = fma(-Ph[k], g.R, g.P[k]) / g.R;
    o[5] = make_double2((double)i, g.R);
    o[6] = make_double2(lo[0], lo[1]);
    o[7] = make_double2(lo[2], 0.0);
  }
}

// ---------------------------------------------------------------------------
// Light-cone events of a snapshot box, on their own (the same crossing as the
// render path): per segment the observer-relative event position, D, and
// whether the event falls inside the slab.
// ---------------------------------------------------------------------------
// One segment per thread: any alignment of the caller's arrays.
__global__ void k_cone_events_1(int64_t n, int dtype, const void* x_rel, const void* xdot,
                                double o0, double o1, double o2, double eta0, double eta_lo,
                                double eta_hi, double* pos, double* delta, uint8_t* keep) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const char* xr = (const char*)x_rel;
  const char* xd = (const char*)xdot;
  double P0[3], V[3];
  const double o[3] = {o0, o1, o2};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    P0[k] = o[k] + raw_at(xr, dtype, 3 * i + k);
    V[k] = raw_at(xd, dtype, 3 * i + k);
  }
  const double vv = (V[0] * V[0] + V[1] * V[1]) + V[2] * V[2];
  double D;
  const bool in = snapshot_event(P0, V, eta0, eta_lo, eta_hi, vv, D);
  const double nan = __builtin_nan("");
#pragma unroll
  for (int k = 0; k < 3; ++k) pos[3 * i + k] = in ? P0[k] + V[k] * D : nan;
  delta[i] = in ? D : nan;
  keep[i] = in ? 1 : 0;
}

// Thread t handles segments 2t and 2t + 1: their six coordinates are
// contiguous, so loads and stores move 8- and 16-byte vectors (positions
// 48 bytes, D 16 bytes, keep flags 2 bytes per thread).
template <typename Tin, typename Tin2>
__global__ void k_cone_events(int64_t n, const Tin* x_rel, const Tin* xdot, double o0, double o1,
                              double o2, double eta0, double eta_lo, double eta_hi, double* pos,
                              double* delta, uint8_t* keep) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i0 = 2 * t;
  if (i0 >= n) return;
  const bool pair = i0 + 1 < n;
  double x[6], v[6];
  if (pair) {
    const Tin2* xr = (const Tin2*)(x_rel + 3 * i0);
    const Tin2* xd = (const Tin2*)(xdot + 3 * i0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const Tin2 a = xr[k], c = xd[k];
      x[2 * k] = (double)a.x;
      x[2 * k + 1] = (double)a.y;
      v[2 * k] = (double)c.x;
      v[2 * k + 1] = (double)c.y;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = (double)x_rel[3 * i0 + k];
      v[k] = (double)xdot[3 * i0 + k];
      x[3 + k] = 0.0;
      v[3 + k] = 0.0;
    }
  }
  const double o[3] = {o0, o1, o2};
  const double nan = __builtin_nan("");
  double p[6], d[2];
  bool in[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    double P0[3], V[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      P0[k] = o[k] + x[3 * s + k];
      V[k] = v[3 * s + k];
    }
    const double vv = (V[0] * V[0] + V[1] * V[1]) + V[2] * V[2];
    double D;
    in[s] = snapshot_event(P0, V, eta0, eta_lo, eta_hi, vv, D);
#pragma unroll
    for (int k = 0; k < 3; ++k) p[3 * s + k] = in[s] ? P0[k] + V[k] * D : nan;
    d[s] = in[s] ? D : nan;
  }
  if (pair) {
    double2* po = (double2*)(pos + 3 * i0);
    po[0] = make_double2(p[0], p[1]);
    po[1] = make_double2(p[2], p[3]);
    po[2] = make_double2(p[4], p[5]);
    *(double2*)(delta + i0) = make_double2(d[0], d[1]);
    *(uint16_t*)(keep + i0) = (uint16_t)((in[0] ? 1u : 0u) | (in[1] ? 0x100u : 0u));
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) pos[3 * i0 + k] = p[k];
    delta[i0] = d[0];
    keep[i0] = in[0] ? 1 : 0;
  }
}

hipError_t launch_cone_events(int64_t n, int dtype, const void* x_rel, const void* xdot,
                              const double origin[3], double eta0, double eta_lo, double eta_hi,
                              double* pos, double* delta, uint8_t* keep, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const size_t es = dtype == 0 ? 4 : 8;
  const bool aligned = ((uintptr_t)x_rel % (2 * es)) == 0 && ((uintptr_t)xdot % (2 * es)) == 0 &&
                       ((uintptr_t)pos % 16) == 0 && ((uintptr_t)delta % 16) == 0 &&
                       ((uintptr_t)keep % 2) == 0;
  if (!aligned) {
    k_cone_events_1<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(
        n, dtype, x_rel, xdot, origin[0], origin[1], origin[2], eta0, eta_lo, eta_hi, pos, delta,
        keep);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)(((n + 1) / 2 + 255) / 256)), block(256);
  if (dtype == 0)
    k_cone_events<float, float2><<<grid, block, 0, st>>>(n, (const float*)x_rel,
                                                         (const float*)xdot, origin[0], origin[1],
                                                         origin[2], eta0, eta_lo, eta_hi, pos,
                                                         delta, keep);
  else
    k_cone_events<double, double2><<<grid, block, 0, st>>>(
        n, (const double*)x_rel, (const double*)xdot, origin[0], origin[1], origin[2], eta0,
        eta_lo, eta_hi, pos, delta, keep);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small utility kernels (plain stores; used instead of memset so that the
// launches can be captured in a graph).
// ---------------------------------------------------------------------------
__global__ void k_fill_f64(double* p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = i; k < n; k += stride) p[k] = v;
}

// A box's four arrays (word counts n[k]) into its storage, one after another.
struct CopyBox {
  const uint32_t* src[4];
  uint32_t* dst;
  int64_t end[4];   // running word counts
};

__global__ void __launch_bounds__(256) k_copy_box(CopyBox c) {
  const int64_t first = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  uint32_t v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t w = first + 256 * j;
    const int k = w < c.end[0] ? 0 : (w < c.end[1] ? 1 : (w < c.end[2] ? 2 : 3));
    if (w < c.end[3]) v[j] = c.src[k][k ? w - c.end[k - 1] : w];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (first + 256 * j < c.end[3]) c.dst[first + 256 * j] = v[j];
}

__global__ void k_zero_counters(unsigned long long* c) {
  for (int i = threadIdx.x; i < kCounters; i += blockDim.x) c[i] = 0ull;
}

// Direction table in structure-of-arrays form (x, y, z each npix doubles).
__global__ void k_dir_table(int64_t nside, int64_t npix, double* x, double* y, double* z) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npix) return;
  double a, b, c;
  pix2vec_ring(nside, i, &a, &b, &c);
  x[i] = a;
  y[i] = b;
  z[i] = c;
}

__global__ void k_ang2pix(int64_t nside, int64_t n, const double* xyz, int64_t* pix) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  pix[i] = ang2pix_ring(nside, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]);
}

__global__ void k_pix2vec(int64_t nside, int64_t first, int64_t count, double* xyz) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  double x, y, z;
  pix2vec_ring(nside, first + i, &x, &y, &z);
  xyz[3 * i + 0] = x;
  xyz[3 * i + 1] = y;
  xyz[3 * i + 2] = z;
}

// ---------------------------------------------------------------------------
// Forward pair kernels.
// ---------------------------------------------------------------------------
// The wavefront's next item: each starts with the item of its own index.
__device__ __forceinline__ int64_t next_item(const FwdArgs& A, bool persistent, int lane,
                                             int64_t cur, int64_t stride) {
  if (!persistent || A.nitems <= kStaticRounds * stride) return cur + stride;
  uint32_t it = 0;
  if (lane == 0) it = atomicAdd(A.work_counter, 1u);
  return stride + (int64_t)__builtin_amdgcn_readfirstlane(__shfl(it, 0));
}

// The pixels of one lane in a tile: slot j is pixel first + pos0 + j step,
// present when pos0 + j step < cnt.  Ring-block tilings give each ring of
// the tile 64 / G lanes (G rings per tile) and read the ring's row from the
// table, so all K pixels of a lane lie on one ring; strips are 64 K
// consecutive pixels cut at the end of the map.  An empty row reports pixel
// 0 as its first, so that loads through it stay inside the map.
struct LaneRow {
  int64_t first;
  int32_t cnt, pos0, step;
};

template <int K>
__device__ __forceinline__ LaneRow lane_row(const FwdArgs& A, int64_t tile, int lane) {
  LaneRow r;
  if (A.rows) {
    const int g = lane >> A.ring_shift;
    const int64_t e = A.rows[tile * A.ring_g + g];
    r.first = e >> kRowCountBits;
    r.cnt = (int32_t)(e & ((1 << kRowCountBits) - 1));
    r.pos0 = lane - (g << A.ring_shift);
    r.step = 1 << A.ring_shift;
  } else {
    r.first = tile * (64 * K);
    const int64_t room = A.npix - r.first;
    r.cnt = room >= 64 * K ? 64 * K : (room > 0 ? (int32_t)room : 0);
    if (r.cnt == 0) r.first = 0;
    r.pos0 = lane;
    r.step = 64;
  }
  return r;
}

// Offset of slot j of a lane inside its row; slots past the end repeat the
// row's last pixel (or pixel `first` of an empty row).
__device__ __forceinline__ int32_t slot_off(const LaneRow& r, int j) {
  const int32_t pos = r.pos0 + j * r.step;
  return pos < r.cnt ? pos : (r.cnt > 0 ? r.cnt - 1 : 0);
}

// The records a work item takes: the records of every box its tile sees, one
// box after another in runs of kSliceUnit (a box's last run may be short), cut
// into w.slices nearly equal ranges of runs.  Whole runs keep a box's windows
// of four records as they are in one slice.  The range's first box is found
// by the wavefront's lanes, 64 boxes at a time: an item that asked every box
// in turn would wait on one scalar load each.
constexpr uint32_t kSliceUnit = 32;

struct SliceRange {
  uint32_t lo, hi;   // runs [lo, hi) of the tile's boxes
  int32_t bi;        // first box entry to visit
  uint32_t pos;      // runs before it
};

__device__ __forceinline__ uint32_t box_kept(const FwdArgs& A, int64_t b) {
  const int64_t n = A.box_count[b].kept;
  return (uint32_t)(A.seg_cap > 0 && n > A.seg_cap ? A.seg_cap : n);
}

__device__ __forceinline__ uint32_t runs_of(uint32_t records) {
  return (records + kSliceUnit - 1) / kSliceUnit;
}

// Runs of the box of list entry bi (0 past the end): one entry per lane.
__device__ __forceinline__ uint32_t entry_runs(const FwdArgs& A, bool list, int32_t bi,
                                               int32_t b1) {
  if (bi >= b1) return 0;
  return runs_of(box_kept(A, list ? A.tile_boxes[bi] : bi));
}

__device__ __forceinline__ SliceRange slice_range(const FwdArgs& A, const WorkItem& w, bool list,
                                                  int32_t b0, int32_t b1, int lane) {
  SliceRange r = {0u, ~0u, b0, 0u};
  if (w.slices <= 1) return r;
  uint32_t total = 0;
  for (int32_t c = b0; c < b1; c += 64) {
    uint32_t u = entry_runs(A, list, c + lane, b1);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) u += __shfl_xor(u, off);
    total += (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
  }
  r.lo = (uint32_t)((uint64_t)total * (uint32_t)w.slice / (uint32_t)w.slices);
  r.hi = (uint32_t)((uint64_t)total * ((uint32_t)w.slice + 1) / (uint32_t)w.slices);
  if (r.lo == 0) return r;
  uint32_t before = 0;
  for (int32_t c = b0; c < b1; c += 64) {
    const uint32_t u = entry_runs(A, list, c + lane, b1);
    uint32_t incl = u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    const unsigned long long past = __ballot(before + incl > r.lo);
    if (past) {
      const int l = __builtin_ctzll(past);
      r.bi = c + l;
      r.pos = before + (uint32_t)__builtin_amdgcn_readlane((int)(incl - u), l);
      return r;
    }
    before += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  }
  r.bi = b1;
  return r;
}

// Records [r0, r1) of box b inside the range (r1 <= r0: none), moving past it.
__device__ __forceinline__ void box_records(const FwdArgs& A, int32_t b, SliceRange& r,
                                            int64_t& r0, int64_t& r1) {
  r0 = ((cbox_p)A.boxes + b)->rec_off;
  const int64_t kept = load_kept(A.box_count, b);
  const uint32_t n = (uint32_t)(A.seg_cap > 0 && kept > A.seg_cap ? A.seg_cap : kept);
  const uint32_t u = runs_of(n);
  const uint32_t u0 = r.lo > r.pos ? r.lo - r.pos : 0;
  const uint32_t u1 = r.hi - r.pos < u ? r.hi - r.pos : u;
  r.pos += u;
  r1 = r0 + (u1 < u ? u1 * kSliceUnit : n);
  r0 += u0 * kSliceUnit;
}

// Work item `item` (uniform over the wavefront).
__device__ __forceinline__ WorkItem work_item(const FwdArgs& A, int64_t item) {
  WorkItem w;
  if (A.work) {
    const ci32p p = (ci32p)(A.work + item);
    w.tile = p[0];
    w.slice = p[1];
    w.slices = p[2];
    w.slot = p[3];
  } else {
    // 32-bit division: the launcher keeps the items below 2^31.
    const uint32_t at = (uint32_t)item / (uint32_t)A.nsplit;
    w.slice = (int32_t)((uint32_t)item - at * (uint32_t)A.nsplit);
    w.tile = A.items ? ((ci32p)A.items)[at] : (int32_t)at;
    w.slices = A.nsplit;
    w.slot = (int32_t)(at * (uint32_t)A.nsplit);
  }
  return w;
}

// Where the sum of pixel p (slot j of this lane) goes: the map, or the
// slice's partial tile.
template <int K>
__device__ __forceinline__ void store_pixel(const FwdArgs& A, const WorkItem& w, int64_t p, int j,
                                            int lane, double v) {
  if (w.slices > 1) A.part[(int64_t)(w.slot + w.slice) * (64 * K) + 64 * j + lane] = v;
  else A.map[p] = A.accumulate ? A.map[p] + v : v;
}

// Fold the term m/d into the running fraction fp/fq of a window; the first
// slot of a window starts it.
__device__ __forceinline__ void fold_term(bool first, float& fp, float& fq, float m, float d) {
  if (first) {
    fp = m;
    fq = d;
  } else {
    fp = fmaf(fp, d, m * fq);
    fq = fq * d;
  }
}

// A 64-bit value every lane holds alike, moved to scalar registers.
__device__ __forceinline__ int64_t uniform_i64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Terms of one segment for close pairs: the direction difference n - P/R
// is taken in FP64 (n from this wavefront's LDS slice, P/R from the FP64
// record) and the rest in FP32.  An exact coincidence gives m = 0 and a
// finite reciprocal, so that term is 0.
template <int K>
__device__ __forceinline__ void near_terms(const float (&nf)[K][3], const double* sdir, int lane,
                                           const v4f r0, const v4f r1, const v4f r2,
                                           const float (&a)[K], const float (&b)[K], cd2p hp,
                                           float (&part)[K]) {
  const v2d h0 = hp[0];
  const v2d h1 = hp[1];
  const float tx = r0.w, ty = r1.x, tz = r1.y;
  const float vx = r1.z, vy = r1.w, vz = r2.x;
  const float kap = r2.y;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const float dx = (float)(sdir[(j * 3 + 0) * 64 + lane] - h0.x);
    const float dy = (float)(sdir[(j * 3 + 1) * 64 + lane] - h0.y);
    const float dz = (float)(sdir[(j * 3 + 2) * 64 + lane] - h1.x);
    const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    const float t1 = kap * fmaf(vz, dz, fmaf(vy, dy, vx * dx));
    const float t2 = kap * fmaf(tz, dz, fmaf(ty, dy, tx * dx));
    const float m = fmaf(-a[j], t2, t1 * b[j]);
    const float den = b[j] * fmaxf(0.5f * q, 1e-30f);
    part[j] = fmaf(m, __builtin_amdgcn_rcpf(den), part[j]);
  }
  (void)nf;
}

// One box's kept records [r0, r1) against a wavefront's pixels, with the
// terms m/d of a pixel folded into one fraction over windows of four
// consecutive segments, (p/q) + m/d = (p d + m q)/(q d), divided once per
// window.  Folded terms have d = b w >= 0.05 near_w (b >= 0.05 unless the
// segment is flagged), so a product of four stays inside the FP32 range.
// Terms of the FP64 path are added one by one.  Each window slot is a
// separate copy of the step, so its update of (p, q) is fixed at compile
// time.  RING: the K pixels of every lane lie on one HEALPix ring and share
// z, so each dot product n.X takes its z part from a per-segment constant.
template <int K, bool RING>
__device__ __forceinline__ void frac_box(const FwdArgs& A, cf4p recs, cd2p ph64, int64_t r0,
                                         int64_t r1, const float (&nf)[K][3],
                                         const double* sdir, int lane, const float (&vis)[K],
                                         float (&S)[K], float (&C)[K],
                                         unsigned long long& near_steps,
                                         unsigned long long& mid_steps) {
  const float near_w = A.near_w, far_w = A.far_w;
  // 32-bit counts (a box holds fewer than 2^31 records) keep the loop tests
  // on the scalar unit, which has no 64-bit ordered compare.
  const int32_t nseg = (int32_t)(r1 - r0);
  const int32_t nwin = (nseg + 3) >> 2;
  const cf4p last = recs + 4 * (r1 - 1);
  cf4p rp = recs + 4 * r0;
  v4f q0 = rp[0], q1 = rp[1], q2 = rp[2], q3 = rp[3];
  float part[K], fp[K], fq[K];
#pragma unroll
  for (int j = 0; j < K; ++j) { part[j] = 0.f; fp[j] = 0.f; fq[j] = 1.f; }
  int32_t left = A.chunk;   // segments until the next Kahan update (multiple of 4)
  for (int32_t win = 0; win < nwin; ++win) {
    const int32_t nslot = (win + 1 < nwin) ? 4 : nseg - 4 * win;
#pragma unroll
    for (int slot = 0; slot < 4; ++slot) {
      if (slot < nslot) {
        const cf4p pf = (rp != last) ? rp + 4 : rp;
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): q0..q3 have arrived
        const v4f n0 = pf[0], n1 = pf[1], n2 = pf[2], n3 = pf[3];
        // Segment constants copied to vector registers once per step: FMAs
        // whose operands are all vector registers issue at twice the rate of
        // those reading a scalar register.
        const float px = to_vgpr(q0.x), py = to_vgpr(q0.y);
        const float tx = to_vgpr(q0.w), ty = to_vgpr(q1.x);
        const float vx = to_vgpr(q1.z), vy = to_vgpr(q1.w);
        const float kap = to_vgpr(q2.y), c1v = to_vgpr(q2.z), c2v = to_vgpr(q2.w);
        float pz, tz, vz;
        float w[K], a[K], bb[K];
        bool nearp = false;
        if constexpr (RING) {
          pz = q0.z;
          tz = q1.y;
          vz = q2.x;
          const float zz = nf[0][2];
          const float cw = fmaf(-zz, pz, 1.0f), ca = zz * tz, cb = fmaf(zz, vz, 1.0f);
#pragma unroll
          for (int j = 0; j < K; ++j) {
            w[j] = fmaf(-nf[j][1], py, fmaf(-nf[j][0], px, cw));
            a[j] = fmaf(nf[j][1], ty, fmaf(nf[j][0], tx, ca));
            bb[j] = fmaf(nf[j][1], vy, fmaf(nf[j][0], vx, cb));
            nearp |= (w[j] < far_w);
          }
        } else {
          pz = to_vgpr(q0.z);
          tz = to_vgpr(q1.y);
          vz = to_vgpr(q2.x);
#pragma unroll
          for (int j = 0; j < K; ++j) {
            w[j] = fmaf(-nf[j][2], pz, fmaf(-nf[j][1], py, fmaf(-nf[j][0], px, 1.0f)));
            a[j] = fmaf(nf[j][2], tz, fmaf(nf[j][1], ty, nf[j][0] * tx));
            bb[j] = fmaf(nf[j][2], vz, fmaf(nf[j][1], vy, fmaf(nf[j][0], vx, 1.0f)));
            nearp |= (w[j] < far_w);
          }
        }
        const bool force = __float_as_int(q3.y) != 0;
        // The far step is marked likely so that it runs without a taken
        // branch (1-2% on a full-sky launch).
        if (__builtin_expect(!force && !__any(nearp), 1)) {
          // Far step: kappa/2 times Xdot.(n - Ph) and X'.(n - Ph) from the
          // dot products.
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const float t1 = fmaf(kap, bb[j], -c1v);
            const float t2 = fmaf(kap, a[j], -c2v);
            const float m = fmaf(-a[j], t2, t1 * bb[j]);   // kappa/2 * m
            fold_term(slot == 0, fp[j], fq[j], m, bb[j] * w[j]);
          }
        } else {
          bool n64 = force;
#pragma unroll
          for (int j = 0; j < K; ++j) n64 |= (w[j] < near_w);
          if (!__any(n64)) {
            // Middle step: the direction difference in FP32 (its error,
            // about 1e-7 absolute, is small against |n - Ph| >= 0.01).
            ++mid_steps;
#pragma unroll
            for (int j = 0; j < K; ++j) {
              const float dx = nf[j][0] - px, dy = nf[j][1] - py, dz = nf[j][2] - pz;
              const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
              const float t1 = kap * fmaf(vz, dz, fmaf(vy, dy, vx * dx));
              const float t2 = kap * fmaf(tz, dz, fmaf(ty, dy, tx * dx));
              const float m = fmaf(-a[j], t2, t1 * bb[j]);
              fold_term(slot == 0, fp[j], fq[j], m, bb[j] * (0.5f * q));
            }
          } else {
            ++near_steps;
            near_terms<K>(nf, sdir, lane, q0, q1, q2, a, bb, ph64 + 2 * ((rp - recs) >> 2), part);
            if (slot == 0) {
#pragma unroll
              for (int j = 0; j < K; ++j) { fp[j] = 0.f; fq[j] = 1.f; }
            }
          }
        }
        q0 = n0;
        q1 = n1;
        q2 = n2;
        q3 = n3;
        rp = pf;
      }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = fmaf(fp[j], __builtin_amdgcn_rcpf(fq[j]), part[j]);
    left -= 4;
    if (left <= 0 || win + 1 == nwin) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        kahan_add(S[j], C[j], part[j] * vis[j]);
        part[j] = 0.f;
      }
      left = A.chunk;
    }
  }
}

template <int K, bool PERSISTENT, bool FRAC>
__global__ void __launch_bounds__(256) k_fwd32(FwdArgs A) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  // The wavefront index is uniform; say so, so that everything derived from
  // it (tile, box, segment index) lives in scalar registers.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t item = (int64_t)blockIdx.x * wpb + wave;
  const int64_t stride = (int64_t)gridDim.x * wpb;
  unsigned long long near_steps = 0, mid_steps = 0, all_steps = 0, pairs = 0;
  const float near_w = A.near_w, far_w = A.far_w;
  cf4p recs = (cf4p)A.rec32;
  cd2p ph64 = (cd2p)A.phat64;
  // Dynamic LDS: K x 3 x 64 doubles per wavefront of the workgroup.
  extern __shared__ double sdir_all[];
  double* const sdir = sdir_all + wave * (K * 3 * 64);
  while (item < A.nitems) {
    const WorkItem wi = work_item(A, item);
    const int64_t tile = wi.tile;
    // Pixel directions come from the table written by the RING pix2vec
    // kernel.  Slots past the end of a lane's row repeat its last pixel
    // (they are masked out of every sum and never written).  The FP64
    // directions are parked in this wavefront's slice of LDS for the
    // close-pair steps and visibility tests; only the FP32 copies stay in
    // registers across the segment loop.
    float nf[K][3];
    bool inmap[K];
    bool same_ring = true;   // this lane's K pixels share one ring (one z)
    double z0 = 0.0;
    const LaneRow lr = lane_row<K>(A, tile, lane);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      inmap[j] = lr.pos0 + j * lr.step < lr.cnt;
      const int64_t p = lr.first + slot_off(lr, j);
      const double x = A.dirx[p], y = A.diry[p], z = A.dirz[p];
      if (j == 0) z0 = z;
      same_ring = same_ring && z == z0;
      sdir[(j * 3 + 0) * 64 + lane] = x;
      sdir[(j * 3 + 1) * 64 + lane] = y;
      sdir[(j * 3 + 2) * 64 + lane] = z;
      nf[j][0] = (float)x;
      nf[j][1] = (float)y;
      nf[j][2] = (float)z;
    }
    // Ring z is computed from integers, so equal z means one ring.
    const bool ring = __all(same_ring);
    float S[K], C[K];
#pragma unroll
    for (int j = 0; j < K; ++j) { S[j] = 0.f; C[j] = 0.f; }

    int32_t b0 = 0, b1 = A.nbox;
    if (A.only_box >= 0) { b0 = A.only_box; b1 = A.only_box + 1; }
    else if (!A.all_boxes) { b0 = ((ci32p)A.tile_ptr)[tile]; b1 = ((ci32p)A.tile_ptr)[tile + 1]; }
    const bool list = !A.all_boxes && A.only_box < 0;
    SliceRange sr = slice_range(A, wi, list, b0, b1, lane);
    for (int32_t bi = sr.bi; bi < b1 && sr.pos < sr.hi; ++bi) {
      const int32_t b = list ? ((ci32p)A.tile_boxes)[bi] : bi;
      int64_t r0, r1;
      box_records(A, b, sr, r0, r1);
      if (r1 <= r0) continue;
      const DevBox bx = load_box(A.boxes, b);
      // Visibility as a per-lane 0/1 weight: partial sums of pixels that do
      // not see the box are multiplied by 0 before they reach the running
      // sum (the arithmetic on those lanes stays finite).
      float vis[K];
      unsigned long long nvis = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const bool v = inmap[j] && (bx.vis == 0 || sees_box(sdir[(j * 3 + 0) * 64 + lane],
                                                             sdir[(j * 3 + 1) * 64 + lane],
                                                             sdir[(j * 3 + 2) * 64 + lane], bx,
                                                             A.eta0));
        vis[j] = v ? 1.0f : 0.0f;
        nvis += __popcll(__ballot(v));
      }
      if (nvis == 0) continue;
      pairs += nvis * (unsigned long long)(r1 - r0);
      all_steps += (unsigned long long)(r1 - r0);
      if constexpr (FRAC) {
        if (ring)
          frac_box<K, true>(A, recs, ph64, r0, r1, nf, sdir, lane, vis, S, C, near_steps, mid_steps);
        else
          frac_box<K, false>(A, recs, ph64, r0, r1, nf, sdir, lane, vis, S, C, near_steps, mid_steps);
      } else {
      // Segment records stream through scalar registers.  The record of the
      // next step is requested before the current one is used; the explicit
      // wait at the top of each step covers exactly the previous request.
      cf4p rp = recs + 4 * r0;
      const cf4p re = recs + 4 * r1;
      v4f q0 = rp[0], q1 = rp[1], q2 = rp[2], q3 = rp[3];
      float part[K];
#pragma unroll
      for (int j = 0; j < K; ++j) part[j] = 0.f;
      int32_t left = A.chunk;   // steps until the next Kahan update
      while (true) {
        const cf4p nxt = rp + 4;
        const bool more = nxt != re;
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): q0..q2 have arrived
        const cf4p pf = more ? nxt : rp;
        const v4f n0 = pf[0], n1 = pf[1], n2 = pf[2], n3 = pf[3];
        const float px = q0.x, py = q0.y, pz = q0.z;
        const float tx = q0.w, ty = q1.x, tz = q1.y;
        const float vx = q1.z, vy = q1.w, vz = q2.x;
        const float kap = q2.y, c1v = q2.z, c2v = q2.w;
        float w[K], a[K], bb[K];
        bool nearp = false;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          w[j] = fmaf(-nf[j][2], pz, fmaf(-nf[j][1], py, fmaf(-nf[j][0], px, 1.0f)));
          a[j] = fmaf(nf[j][2], tz, fmaf(nf[j][1], ty, nf[j][0] * tx));
          bb[j] = fmaf(nf[j][2], vz, fmaf(nf[j][1], vy, fmaf(nf[j][0], vx, 1.0f)));
          nearp |= (w[j] < far_w);
        }
        // Segments flagged at precompute (|Xdot| close to 1, where b = 1 + n.Xdot
        // may be tiny) always take the FP64 form.
        const bool force = __float_as_int(q3.y) != 0;
        bool n64 = force;
        if (!force && __any(nearp)) {
#pragma unroll
          for (int j = 0; j < K; ++j) n64 |= (w[j] < near_w);
        }
        if (__builtin_expect(!force && !__any(nearp), 1)) {
          // kappa/2 times Xdot.(n - Ph) and X'.(n - Ph) from the dot products.
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const float t1 = fmaf(kap, bb[j], -c1v);
            const float t2 = fmaf(kap, a[j], -c2v);
            const float m = fmaf(-a[j], t2, t1 * bb[j]);   // kappa/2 * m
            part[j] = fmaf(m, __builtin_amdgcn_rcpf(bb[j] * w[j]), part[j]);
          }
        } else if (!__any(n64)) {
          // Middle pairs: the direction difference in FP32.
          ++mid_steps;
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const float dx = nf[j][0] - px, dy = nf[j][1] - py, dz = nf[j][2] - pz;
            const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const float t1 = kap * fmaf(vz, dz, fmaf(vy, dy, vx * dx));
            const float t2 = kap * fmaf(tz, dz, fmaf(ty, dy, tx * dx));
            const float m = fmaf(-a[j], t2, t1 * bb[j]);
            part[j] = fmaf(m, __builtin_amdgcn_rcpf(bb[j] * (0.5f * q)), part[j]);
          }
        } else {
          // Close pairs: the difference of directions in FP64.  An exact
          // coincidence (n == Ph) gives m = 0 and a finite reciprocal, so
          // the term is 0.
          ++near_steps;
          const cd2p hp = ph64 + 2 * ((rp - recs) >> 2);
          const v2d h0 = hp[0];
          const v2d h1 = hp[1];
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const float dx = (float)(sdir[(j * 3 + 0) * 64 + lane] - h0.x);
            const float dy = (float)(sdir[(j * 3 + 1) * 64 + lane] - h0.y);
            const float dz = (float)(sdir[(j * 3 + 2) * 64 + lane] - h1.x);
            const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const float t1 = kap * fmaf(vz, dz, fmaf(vy, dy, vx * dx));
            const float t2 = kap * fmaf(tz, dz, fmaf(ty, dy, tx * dx));
            const float m = fmaf(-a[j], t2, t1 * bb[j]);
            const float den = bb[j] * fmaxf(0.5f * q, 1e-30f);
            part[j] = fmaf(m, __builtin_amdgcn_rcpf(den), part[j]);
          }
        }
        --left;
        if (left == 0 || !more) {
#pragma unroll
          for (int j = 0; j < K; ++j) {
            kahan_add(S[j], C[j], part[j] * vis[j]);
            part[j] = 0.f;
          }
          left = A.chunk;
        }
        if (!more) break;
        q0 = n0;
        q1 = n1;
        q2 = n2;
        q3 = n3;
        rp = nxt;
      }
      }
    }
    const LaneRow lw = lane_row<K>(A, tile, lane);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (lw.pos0 + j * lw.step < lw.cnt) {
        // The running sum s carries the result; c is the negated rounding
        // error still owed to it, so the value is s - c.
        const int64_t p = lw.first + lw.pos0 + j * lw.step;
        store_pixel<K>(A, wi, p, j, lane, (double)S[j] - (double)C[j]);
      }
    }
    item = PERSISTENT ? next_item(A, true, lane, item, stride) : item + stride;
  }
  // One atomic per wavefront and counter: per box and tile they queued up on
  // one address.
  const int slot = kCounterStride * (int)(blockIdx.x % kCounterSlots);
  if (lane == 0 && pairs) atomicAdd(A.pairs + slot, pairs);
  if (lane == 0 && near_steps) atomicAdd(A.near_steps + slot, near_steps);
  if (lane == 0 && mid_steps) atomicAdd(A.mid_steps + slot, mid_steps);
  if (lane == 0 && all_steps) atomicAdd(A.steps + slot, all_steps);
}

// ---------------------------------------------------------------------------
// Forward, FP32C form, on the matrix cores.
//
// In the frame of a tile (centre c, tangent axes e1, e2) a pixel is
// n' = n - c = (x1, x2, x3), x3 = c.n - 1 = -|n'|^2/2, and a segment
// d = Ph - c.  The three forms a pair needs are affine in n':
//   w   = 1 - n.Ph = |n' - d|^2/2 = -n'.d - x3 + |d|^2/2,
//   v   = Xdot.(n - Ph)           =  Xdot.n' - Xdot.d,
//   u   = X'.(n - Ph)             =  X'.n'   - X'.d,
// three products of a row of four numbers per segment with a column
// (x1, x2, x3, 1) per pixel.  The term is kappa' m/(b w) with b = 1 + n.Xdot =
// v + b0, a = n.X' = u + a0 (b0 = 1 + Ph.Xdot, a0 = Ph.X') and m = v b - u a =
// v b - (u + a0/2)^2 + a0^2/4.  With k = |kappa'| the rows carry k v,
// y = sqrt(k) (u + a0/2) and -w (w where kappa' > 0), so that a pair takes
// b = (k v)/k + b0, k m = (k v) b + k a0^2/4 - y^2 and b w: four operations.
// Every number in a row or column is of the size it has in
// the tile, so that w and the differences keep FP32's relative accuracy down
// to angles of 1.5 tile radii from the centre, where the error of w is at
// most about 3 (theta + rho)^2/(theta - rho)^2 2^-24 <= 4.5e-6 (the far form
// of the vector kernel: 1.2e-5 at its threshold).
//
// The products run on the bf16 matrix cores without losing FP32's 24 bits:
// each number is split into three bf16 parts (8 bits each, exact), and the
// eight partial products above 2^-32 of the whole (parts (0,0), (0,1),
// (1,0), (1,1), (0,2), (2,0), (1,2), (2,1)) take eight of the instruction's
// 32 terms for each component, the constant's three parts three more.  They
// are summed in FP32 inside one v_mfma_f32_16x16x32_bf16: measured against
// 64 bits its error is 2.9e-8 rms, 1.1e-7 at most, of the summed magnitudes
// (the FP32 FMA chain: 3.3e-8 and 1.4e-7).  The FP32 matrix instruction
// would take twice the cycles.
//
// A workgroup of four wavefronts owns a tile of 512 pixels, 128 per
// wavefront: eight columns of 16 pixels, so that a 16 x 16 result leaves a
// lane four segments of one pixel, whose terms are folded into one fraction
// and divided once; the four lane groups hold partial sums of the same
// pixels, added at the end.  The rows of 64 segments at a time are formed by
// the whole workgroup (wavefront role g: component g of the lane's segment)
// and shared through LDS, one block ahead.  Segments closer than the limit
// above (and those flagged at precompute) get neutral rows there and go
// through the FP64 difference one by one, two pixels per lane.
//
// It is bound by instruction issue: per 256 pairs three matrix instructions
// (16 cycles each) and 27 vector ones with the reciprocal (60 cycles), which
// overlap hardly at all (interleaving them one to nine measured the same).
// One box of 50,000 segments at Nside 2048: 553 ms (4.55e12 pairs/s) against
// 720 ms on the vector kernel; 514 ms without staging the rows.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kMTile = 512;     // pixels of a tile
constexpr int kMCols = 8;       // 16-pixel columns per wavefront
constexpr int kMRows = 64;      // segments per LDS block
constexpr float kMReach = 1.5f; // closest segment, in tile radii from the centre

typedef const TileFrame __attribute__((address_space(4)))* cframe_p;

struct MBlock {
  bf16x8 a[3][kMRows / 16][64];   // rows of w, v, u: [form][segment / 16][lane]
  float b0[kMRows], hh[kMRows], g[kMRows];
  unsigned long long near, mid;   // segments for the FP64 path; below far_w (counted)
};

__device__ __forceinline__ void split_bf16(float x, __bf16& p0, __bf16& p1, __bf16& p2) {
  p0 = (__bf16)x;
  const float r = x - (float)p0;
  p1 = (__bf16)r;
  p2 = (__bf16)(r - (float)p1);
}

__device__ __forceinline__ bf16x8 row_parts(float y, bool constant) {
  __bf16 a, b, c;
  split_bf16(y, a, b, c);
  const __bf16 z = (__bf16)0.0f;
  return constant ? bf16x8{a, b, c, z, z, z, z, z} : bf16x8{a, b, a, b, c, a, c, b};
}

__device__ __forceinline__ bf16x8 column_parts(float x, bool constant) {
  __bf16 a, b, c;
  split_bf16(x, a, b, c);
  const __bf16 z = (__bf16)0.0f, o = (__bf16)1.0f;
  return constant ? bf16x8{o, o, o, z, z, z, z, z} : bf16x8{a, a, b, b, a, c, b, c};
}

// 2 sin^2(x/2) = 1 - cos x for an angle x, 2 from pi on.
__device__ __forceinline__ float versine(float x) {
  if (x >= 3.14159f) return 2.0f;
  const float s = sinf(0.5f * x);
  return 2.0f * s * s;
}

// One frame per tile: wavefront per tile, lane l taking slots 64 j + l.
template <int K>
__global__ void __launch_bounds__(256) k_tile_frames(FwdArgs A, int64_t ntiles, TileFrame* out) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= ntiles) return;
  const LaneRow lr = lane_row<K>(A, t, lane);
  double n[K][3], c[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int64_t p = lr.first + slot_off(lr, j);
    n[j][0] = A.dirx[p];
    n[j][1] = A.diry[p];
    n[j][2] = A.dirz[p];
    const double in = lr.pos0 + j * lr.step < lr.cnt ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] += in * n[j][k];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] += __shfl_xor(c[k], off);
  double r = sqrt((c[0] * c[0] + c[1] * c[1]) + c[2] * c[2]);
  if (!(r > 1e-6)) {   // a tile around the whole sky has no centre: any will do
    c[0] = c[1] = 0.0;
    c[2] = r = 1.0;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) c[k] /= r;
  double far = 0.0;   // largest |n - c|^2
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double x = n[j][0] - c[0], y = n[j][1] - c[1], z = n[j][2] - c[2];
    if (lr.pos0 + j * lr.step < lr.cnt) far = fmax(far, (x * x + y * y) + z * z);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) far = fmax(far, __shfl_xor(far, off));
  if (lane != 0) return;
  TileFrame f;
  const bool polar = fabs(c[2]) > 0.9;
  const double h = polar ? sqrt(c[1] * c[1] + c[2] * c[2]) : sqrt(c[0] * c[0] + c[1] * c[1]);
  f.e1[0] = polar ? 0.0 : -c[1] / h;
  f.e1[1] = polar ? -c[2] / h : c[0] / h;
  f.e1[2] = polar ? c[1] / h : 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f.c[k] = c[k];
    f.e2[k] = c[(k + 1) % 3] * f.e1[(k + 2) % 3] - c[(k + 2) % 3] * f.e1[(k + 1) % 3];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f.axis[0][k] = (float)f.e1[k];
    f.axis[1][k] = (float)f.e2[k];
    f.axis[2][k] = (float)c[k];
  }
  f.rho = 1.000001f * (float)(2.0 * asin(fmin(1.0, 0.5 * sqrt(far))));
  out[t] = f;
}

// The rows of one block: records r0 + lane, the first n of them real, by the
// wavefront of role g (0, 1, 2: component along the axis; 3: the constants).
__device__ __forceinline__ void stage_rows(const FwdArgs& A, MBlock& sh, int lane, int role,
                                           cframe_p fr, float t_near, float t_mid, int64_t r0,
                                           int32_t n) {
  const int64_t r = r0 + (lane < n ? lane : n - 1);
  const float4* M = (const float4*)(A.recm + (size_t)r * kRecM);
  const float4 mv = M[0], mt = M[1], mk = M[2];
  const double2 h0 = ((const double2*)A.phat64)[2 * r];
  const double pz = A.phat64[4 * r + 2];
  const float dx = (float)(h0.x - fr->c[0]), dy = (float)(h0.y - fr->c[1]);
  const float dz = (float)(pz - fr->c[2]);
  const float t = 0.5f * fmaf(dz, dz, fmaf(dy, dy, dx * dx));
  const bool real = lane < n;
  const bool near = real && (!(t >= t_near) || mk.w != 0.f);
  const bool neutral = !real || near;   // m = 0 and b w = 1 for every pixel
  bf16x8* const to = &sh.a[0][lane >> 4][role * 16 + (lane & 15)];
  constexpr int kForm = kMRows / 16 * 64;   // rows of the next form
  if (role < 3) {
    const float ex = fr->axis[role][0], ey = fr->axis[role][1], ez = fr->axis[role][2];
    const float dd = fmaf(ez, dz, fmaf(ey, dy, ex * dx));
    const float one = role == 2 ? -1.0f : 0.0f;
    const float yw = (one - dd) * mk.z;
    const float yv = fmaf(ez, mv.z, fmaf(ey, mv.y, ex * mv.x));
    const float yu = fmaf(ez, mt.z, fmaf(ey, mt.y, ex * mt.x));
    to[0] = row_parts(neutral ? 0.f : yw, false);
    to[kForm] = row_parts(neutral ? 0.f : yv, false);
    to[2 * kForm] = row_parts(neutral ? 0.f : yu, false);
  } else {
    const float yv = -fmaf(dz, mv.z, fmaf(dy, mv.y, dx * mv.x));
    const float yu = mt.w - fmaf(dz, mt.z, fmaf(dy, mt.y, dx * mt.x));
    to[0] = row_parts(neutral ? 1.f : t * mk.z, true);
    to[kForm] = row_parts(neutral ? 0.f : yv, true);
    to[2 * kForm] = row_parts(neutral ? 0.f : yu, true);
    sh.b0[lane] = neutral ? 1.f : mv.w;
    sh.hh[lane] = neutral ? 0.f : mk.x;
    sh.g[lane] = neutral ? 0.f : mk.y;
    const unsigned long long nm = __ballot(near), mm = __ballot(real && !near && t < t_mid);
    if (lane == 0) {
      sh.near = nm;
      sh.mid = mm;
    }
  }
}

template <bool PERSISTENT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_fwd32m(FwdArgs A) {
  __shared__ MBlock sh[2];
  __shared__ uint32_t next;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane >> 4, col = lane & 15;
  unsigned long long near_steps = 0, mid_steps = 0, all_steps = 0, pairs = 0;
  const cf4p recs = (cf4p)A.rec32;
  const cd2p ph64 = (cd2p)A.phat64;
  int64_t item = blockIdx.x;
  while (item < A.nitems) {
    const WorkItem wi = work_item(A, item);
    const int64_t tile = wi.tile;
    const cframe_p fr = (cframe_p)A.frames + tile;   // scalar loads
    const double c0 = fr->c[0], c1 = fr->c[1], c2 = fr->c[2];
    const float rho = fr->rho;
    const float t_near = versine(fmaxf(kMReach * rho, rho + acosf(fmaxf(-1.0f, 1.0f - A.near_w))));
    const float t_mid = versine(rho + acosf(fmaxf(-1.0f, 1.0f - A.far_w)));
    // Pixel slot s of the tile: position s % W of row s / W, W = 512 / rings.
    const int wshift = 3 + A.ring_shift;   // log2 W (64 / rings lanes of 8 slots)
    // This lane's pixels 16 (grp + 4 h) + col, h = 0, 1, of its wavefront:
    // written, tested for visibility and summed by the FP64 path.
    auto slot_pixel = [&](int s, bool& in, int64_t& p) {
      int64_t first;
      int32_t cnt, pos;
      if (A.rows) {
        const int64_t e = A.rows[tile * A.ring_g + (s >> wshift)];
        first = e >> kRowCountBits;
        cnt = (int32_t)(e & ((1 << kRowCountBits) - 1));
        pos = s & ((1 << wshift) - 1);
      } else {
        first = tile * kMTile;
        const int64_t room = A.npix - first;
        cnt = room >= kMTile ? kMTile : (room > 0 ? (int32_t)room : 0);
        if (cnt == 0) first = 0;
        pos = s;
      }
      in = pos < cnt;
      p = first + (in ? pos : (cnt > 0 ? cnt - 1 : 0));
    };
    bool in2[2];
    int32_t p2[2];   // pixel indices are below 2^30
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int64_t p;
      slot_pixel(wave * 128 + 16 * (grp + 4 * h) + col, in2[h], p);
      p2[h] = (int32_t)p;
    }
    // Columns: component grp of each pixel's n'.
    bf16x8 B[kMCols];
    {
      const double a0 = grp == 0 ? fr->e1[0] : (grp == 1 ? fr->e2[0] : c0);
      const double a1 = grp == 0 ? fr->e1[1] : (grp == 1 ? fr->e2[1] : c1);
      const double a2 = grp == 0 ? fr->e1[2] : (grp == 1 ? fr->e2[2] : c2);
#pragma unroll
      for (int j = 0; j < kMCols; ++j) {
        bool in;
        int64_t p;
        slot_pixel(wave * 128 + 16 * j + col, in, p);
        const double x = (a0 * (A.dirx[p] - c0) + a1 * (A.diry[p] - c1)) + a2 * (A.dirz[p] - c2);
        B[j] = column_parts((float)x, grp == 3);
      }
    }
    float S[kMCols], C[kMCols], part[kMCols];
#pragma unroll
    for (int j = 0; j < kMCols; ++j) S[j] = C[j] = part[j] = 0.f;
    int32_t b0 = 0, b1 = A.nbox;
    if (A.only_box >= 0) { b0 = A.only_box; b1 = A.only_box + 1; }
    else if (!A.all_boxes) { b0 = ((ci32p)A.tile_ptr)[tile]; b1 = ((ci32p)A.tile_ptr)[tile + 1]; }
    const bool list = !A.all_boxes && A.only_box < 0;
    SliceRange sr = slice_range(A, wi, list, b0, b1, lane);
    int buf = 0;
    for (int32_t bi = sr.bi; bi < b1 && sr.pos < sr.hi; ++bi) {
      const int32_t b = list ? ((ci32p)A.tile_boxes)[bi] : bi;
      int64_t r0, r1;
      box_records(A, b, sr, r0, r1);
      if (r1 <= r0) continue;
      // Visibility of the wavefront's 128 pixels, two per lane, as masks.
      unsigned long long vis[2];
      {
        const DevBox bx = load_box(A.boxes, b);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          bool v = in2[h];
          if (bx.vis != 0) v = v && sees_box(A.dirx[p2[h]], A.diry[p2[h]], A.dirz[p2[h]], bx, A.eta0);
          vis[h] = __ballot(v);
        }
        const int any = __popcll(vis[0]) + __popcll(vis[1]);
        if (bx.vis != 0 && !__syncthreads_or(any)) continue;
        if (any) {
          pairs += (unsigned long long)any * (unsigned long long)(r1 - r0);
          all_steps += (unsigned long long)(r1 - r0);
        }
      }
      const bool sees = (vis[0] | vis[1]) != 0;
      const int32_t nrec = (int32_t)(r1 - r0), nblk = (nrec + kMRows - 1) / kMRows;
      auto stage = [&](int32_t k, MBlock& to) {
        // Roles move on with the block, so that no SIMD always gets the same.
        const int role = (wave + k) & 3;
        const int32_t left = nrec - k * kMRows;
        stage_rows(A, to, lane, role, fr, t_near, t_mid, r0 + (int64_t)k * kMRows,
                   left < kMRows ? left : kMRows);
      };
      int32_t terms = 0;
      stage(0, sh[buf]);
      __syncthreads();
      for (int32_t k = 0; k < nblk; ++k) {
        if (k + 1 < nblk) stage(k + 1, sh[buf ^ 1]);
        const MBlock& m = sh[buf];
        if (sees) {
          const int32_t left = nrec - k * kMRows;
          const int nrt = left < kMRows ? (left + 15) >> 4 : kMRows / 16;
#pragma unroll 1
          for (int rt = 0; rt < nrt; ++rt) {
            const bf16x8 aw = m.a[0][rt][lane], av = m.a[1][rt][lane], au = m.a[2][rt][lane];
            const f32x4 kb = *(const f32x4*)&m.b0[16 * rt + 4 * grp];
            const f32x4 ka = *(const f32x4*)&m.hh[16 * rt + 4 * grp];
            const f32x4 kg = *(const f32x4*)&m.g[16 * rt + 4 * grp];
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < kMCols; ++j) {
              const f32x4 w = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, B[j], zero, 0, 0, 0);
              const f32x4 v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, B[j], zero, 0, 0, 0);
              const f32x4 u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(au, B[j], zero, 0, 0, 0);
              float n[4], d[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const float bb = fmaf(v[q], kg[q], kb[q]);
                n[q] = fmaf(-u[q], u[q], fmaf(v[q], bb, ka[q]));
                d[q] = bb * w[q];
              }
              const float n01 = fmaf(n[0], d[1], n[1] * d[0]), d01 = d[0] * d[1];
              const float n23 = fmaf(n[2], d[3], n[3] * d[2]), d23 = d[2] * d[3];
              part[j] = fmaf(fmaf(n01, d23, n23 * d01), __builtin_amdgcn_rcpf(d01 * d23), part[j]);
            }
          }
          mid_steps += __popcll(m.mid);
          // Close segments, in order: the terms of pixels (grp + 4 h, col)
          // go to this lane's partial sums of those columns.  The next
          // segment's record is requested before this one is used.
          unsigned long long todo = (unsigned long long)uniform_i64((int64_t)m.near);
          if (todo) {
            near_steps += __popcll(todo);
            double nd[2][3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              nd[h][0] = A.dirx[p2[h]];
              nd[h][1] = A.diry[p2[h]];
              nd[h][2] = A.dirz[p2[h]];
            }
            const int64_t rk = r0 + (int64_t)k * kMRows;
            int64_t r = rk + __builtin_ctzll(todo);
            v4f q0 = recs[4 * r], q1 = recs[4 * r + 1], q2 = recs[4 * r + 2];
            v2d h0 = ph64[2 * r], h1 = ph64[2 * r + 1];
            while (todo) {
              todo &= todo - 1;
              if (todo) r = rk + __builtin_ctzll(todo);
              __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this record has arrived
              const v4f n0 = recs[4 * r], n1 = recs[4 * r + 1], n2 = recs[4 * r + 2];
              const v2d g0 = ph64[2 * r], g1 = ph64[2 * r + 1];
              float term[2];
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const float fx = (float)nd[h][0], fy = (float)nd[h][1], fz = (float)nd[h][2];
                const float dx = (float)(nd[h][0] - h0.x), dy = (float)(nd[h][1] - h0.y);
                const float dz = (float)(nd[h][2] - h1.x);
                const float a = fmaf(fz, q1.y, fmaf(fy, q1.x, fx * q0.w));
                const float bb = fmaf(fz, q2.x, fmaf(fy, q1.w, fmaf(fx, q1.z, 1.0f)));
                const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const float t1 = q2.y * fmaf(q2.x, dz, fmaf(q1.w, dy, q1.z * dx));
                const float t2 = q2.y * fmaf(q1.y, dz, fmaf(q1.x, dy, q0.w * dx));
                const float mm = fmaf(-a, t2, t1 * bb);
                term[h] = mm * __builtin_amdgcn_rcpf(bb * fmaxf(0.5f * q, 1e-30f));
              }
#pragma unroll
              for (int j = 0; j < kMCols; ++j) part[j] += grp == (j & 3) ? term[j >> 2] : 0.0f;
              q0 = n0;
              q1 = n1;
              q2 = n2;
              h0 = g0;
              h1 = g1;
            }
          }
          terms += kMRows / 4;
          if (terms >= A.chunk || k + 1 == nblk) {
#pragma unroll
            for (int j = 0; j < kMCols; ++j) {
              const bool v = (vis[j >> 2] >> (16 * (j & 3) + col)) & 1;
              kahan_add(S[j], C[j], v ? part[j] : 0.0f);
              part[j] = 0.f;
            }
            terms = 0;
          }
        }
        __syncthreads();
        buf ^= 1;
      }
    }
    // The four lane groups' sums of each pixel, then lane group j mod 4
    // writes column j.
    double out[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kMCols; ++j) {
      double v = (double)S[j] - (double)C[j];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (grp == (j & 3)) out[j >> 2] = v;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!in2[h]) continue;
      if (wi.slices > 1) {
        // The partial tile's layout: row's lane and its slot (lane_row).
        const int s = wave * 128 + 16 * (grp + 4 * h) + col;
        const int row = A.rows ? s >> wshift : 0, pos = A.rows ? s & ((1 << wshift) - 1) : s;
        const int ln = (row << A.ring_shift) + (pos & ((1 << A.ring_shift) - 1));
        A.part[(int64_t)(wi.slot + wi.slice) * kMTile + 64 * (pos >> A.ring_shift) + ln] = out[h];
      } else {
        A.map[p2[h]] = A.accumulate ? A.map[p2[h]] + out[h] : out[h];
      }
    }
    if (PERSISTENT && A.nitems > kStaticRounds * gridDim.x) {
      if (threadIdx.x == 0) next = atomicAdd(A.work_counter, 1u);
      __syncthreads();
      item = (int64_t)gridDim.x + __builtin_amdgcn_readfirstlane(next);
      __syncthreads();
    } else {
      __syncthreads();   // every wavefront is done with the staged rows
      item += gridDim.x;
    }
  }
  const int slot = kCounterStride * (int)(blockIdx.x % kCounterSlots);
  if (lane == 0 && pairs) atomicAdd(A.pairs + slot, pairs);
  if (lane == 0 && near_steps) atomicAdd(A.near_steps + slot, near_steps);
  if (lane == 0 && mid_steps) atomicAdd(A.mid_steps + slot, mid_steps);
  if (lane == 0 && all_steps) atomicAdd(A.steps + slot, all_steps);
}

__device__ __forceinline__ double rcp_f64(double x) {
  // The hardware estimate r (relative error e = 1 - x r below 2^-24)
  // refined by one third-order step: 1/x = r / (1 - e) = r (1 + e + e^2 +
  // ...), truncated after e^2, leaves e^3 < 2^-72.  Three FMAs where two
  // Newton steps take four; both measure within 1 ulp of 1/x over 2^22
  // random operands spanning 2^-40 to 2^10.
  double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  r = fma(r, fma(e, e, e), r);
  return r;
}

// The terms kappa m/(b q) of one record at the lane's K pixels, as numerator
// and denominator.  An exact coincidence has m = 0; its q is raised to 1e-50
// (below any other pair's, and far enough from the range's end for a product
// of four) so that the term is 0.
template <int K, bool kRing>
__device__ __forceinline__ void fwd64_terms(cd2p rp, const double (&nd)[K][3], double (&num)[K],
                                            double (&den)[K]) {
  const v2d q0 = rp[0];
  const v2d q1 = rp[1];
  const v2d q2 = rp[2];
  const v2d q3 = rp[3];
  const v2d q4 = rp[4];
  const v2d q6 = rp[6];
  const v2d q7 = rp[7];
  const double px = q0.x, py = q0.y, pz = q1.x;
  const double lx = q6.x, ly = q6.y, lz = q7.x;
  const double tx = q1.y, ty = q2.x, tz = q2.y;
  const double vx = q3.x, vy = q3.y, vz = q4.x;
  const double kap = q4.y;
  // (n - hi) is exact for nearby directions; the lo part then enters with
  // a single rounding.
  double qz = 0.0, az = 0.0, bz = 1.0, vdz = 0.0, tdz = 0.0;
  if constexpr (kRing) {
    const double dz0 = (nd[0][2] - pz) - lz;
    qz = dz0 * dz0;
    az = nd[0][2] * tz;
    bz = fma(nd[0][2], vz, 1.0);
    vdz = vz * dz0;
    tdz = tz * dz0;
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double dx = (nd[j][0] - px) - lx;
    const double dy = (nd[j][1] - py) - ly;
    double q, a, b, vd, td;
    if constexpr (kRing) {
      q = fma(dy, dy, fma(dx, dx, qz));
      a = fma(nd[j][1], ty, fma(nd[j][0], tx, az));
      b = fma(nd[j][1], vy, fma(nd[j][0], vx, bz));
      vd = fma(vy, dy, fma(vx, dx, vdz));
      td = fma(ty, dy, fma(tx, dx, tdz));
    } else {
      const double dz = (nd[j][2] - pz) - lz;
      q = fma(dz, dz, fma(dy, dy, dx * dx));
      a = fma(nd[j][2], tz, fma(nd[j][1], ty, nd[j][0] * tx));
      b = fma(nd[j][2], vz, fma(nd[j][1], vy, fma(nd[j][0], vx, 1.0)));
      vd = fma(vz, dz, fma(vy, dy, vx * dx));
      td = fma(tz, dz, fma(ty, dy, tx * dx));
    }
    num[j] = kap * fma(vd, b, -(a * td));
    den[j] = b * fmax(q, 1e-50);
  }
}

// The FP64 pair steps over nk consecutive records (16 doubles each) into
// part[j].  The terms of W consecutive records are folded into one fraction,
// p/q + m/d = (p d + m q)/(q d), and divided once: the reciprocal with its
// refinement costs about eight FP64 instructions, a fold three
// (50,000 segments at Nside 512, K = 4: one term per division 135 ms, two
// 120, four 108).  kRing: every lane's K pixels share one z (ring-block tiles
// keep a lane on one ring), so the z parts of n - Ph, |n - Ph|^2, n.X',
// 1 + n.Xdot, Xdot.(n - Ph) and X'.(n - Ph) are formed once per record for
// the lane (3.5 fewer FP64 instructions per pair at K = 2; the sums are
// associated differently, within an ulp).
template <int K, bool kRing>
__device__ __forceinline__ void fwd64_steps(cd2p rp, int32_t nk, const double (&nd)[K][3],
                                            double (&part)[K]) {
  constexpr int W = 4;
  int32_t k = 0;
  for (; k + W <= nk; k += W, rp += 8 * W) {
    double fp[K], fq[K];
    fwd64_terms<K, kRing>(rp, nd, fp, fq);
#pragma unroll
    for (int r = 1; r < W; ++r) {
      double num[K], den[K];
      fwd64_terms<K, kRing>(rp + 8 * r, nd, num, den);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        fp[j] = fma(fp[j], den[j], num[j] * fq[j]);
        fq[j] = fq[j] * den[j];
      }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = fma(fp[j], rcp_f64(fq[j]), part[j]);
  }
  for (; k < nk; ++k, rp += 8) {
    double num[K], den[K];
    fwd64_terms<K, kRing>(rp, nd, num, den);
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = fma(num[j], rcp_f64(den[j]), part[j]);
  }
}

template <int K, bool PERSISTENT>
__global__ void __launch_bounds__(256) k_fwd64(FwdArgs A) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  // The wavefront index is uniform; say so, so that everything derived from
  // it (tile, box, segment index) lives in scalar registers.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t item = (int64_t)blockIdx.x * wpb + wave;
  const int64_t stride = (int64_t)gridDim.x * wpb;
  cd2p recs = (cd2p)A.rec64;
  unsigned long long pairs = 0;
  while (item < A.nitems) {
    const WorkItem wi = work_item(A, item);
    const int64_t tile = wi.tile;
    double nd[K][3];
    bool inmap[K];
    bool same_ring = true;   // this lane's K pixels share one ring (one z)
    const LaneRow lr = lane_row<K>(A, tile, lane);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      inmap[j] = lr.pos0 + j * lr.step < lr.cnt;
      const int64_t pc = lr.first + slot_off(lr, j);
      nd[j][0] = A.dirx[pc];
      nd[j][1] = A.diry[pc];
      nd[j][2] = A.dirz[pc];
      same_ring = same_ring && nd[j][2] == nd[0][2];
    }
    // Ring z is computed from integers, so equal z means one ring.
    const bool ring = __all(same_ring);
    double S[K], C[K];
#pragma unroll
    for (int j = 0; j < K; ++j) { S[j] = 0.0; C[j] = 0.0; }
    int32_t b0 = 0, b1 = A.nbox;
    if (A.only_box >= 0) { b0 = A.only_box; b1 = A.only_box + 1; }
    else if (!A.all_boxes) { b0 = ((ci32p)A.tile_ptr)[tile]; b1 = ((ci32p)A.tile_ptr)[tile + 1]; }
    const bool list = !A.all_boxes && A.only_box < 0;
    SliceRange sr = slice_range(A, wi, list, b0, b1, lane);
    for (int32_t bi = sr.bi; bi < b1 && sr.pos < sr.hi; ++bi) {
      const int32_t b = list ? ((ci32p)A.tile_boxes)[bi] : bi;
      int64_t r0, r1;
      box_records(A, b, sr, r0, r1);
      if (r1 <= r0) continue;
      const DevBox bx = load_box(A.boxes, b);
      bool vis[K];
      unsigned long long nvis = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        vis[j] = inmap[j] && (bx.vis == 0 || sees_box(nd[j][0], nd[j][1], nd[j][2], bx, A.eta0));
        nvis += __popcll(__ballot(vis[j]));
      }
      if (nvis == 0) continue;
      pairs += nvis * (unsigned long long)(r1 - r0);
      for (int64_t c0 = r0; c0 < r1; c0 += A.chunk) {
        const int64_t c1 = (c0 + A.chunk < r1) ? c0 + A.chunk : r1;
        double part[K];
#pragma unroll
        for (int j = 0; j < K; ++j) part[j] = 0.0;
        const int32_t nk = (int32_t)(c1 - c0);
        const cd2p rp = recs + 8 * c0;
        if (ring)
          fwd64_steps<K, true>(rp, nk, nd, part);
        else
          fwd64_steps<K, false>(rp, nk, nd, part);
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const double y = part[j] - C[j];
          const double t = S[j] + y;
          const double cn = (t - S[j]) - y;
          S[j] = vis[j] ? t : S[j];
          C[j] = vis[j] ? cn : C[j];
        }
      }
    }
    const LaneRow lw = lane_row<K>(A, tile, lane);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (lw.pos0 + j * lw.step < lw.cnt) {
        const int64_t p = lw.first + lw.pos0 + j * lw.step;
        store_pixel<K>(A, wi, p, j, lane, S[j] - C[j]);
      }
    }
    item = PERSISTENT ? next_item(A, true, lane, item, stride) : item + stride;
  }
  const int slot = kCounterStride * (int)(blockIdx.x % kCounterSlots);
  if (lane == 0 && pairs) atomicAdd(A.pairs + slot, pairs);
}

// The map's pixels of the sliced tiles: each the sum of its tile's partial
// sums.  A workgroup takes one pixel slot j of a tile's 64 lanes; its
// wavefronts each add a run of the slices in order, eight loads in flight,
// and the runs' sums are added in order.  The loads' latency bounds it (one
// wavefront adding 782 slices of two tiles took 1.5 ms), hence the
// wavefronts per workgroup grow with the slices.
template <int K>
__global__ void __launch_bounds__(1024) k_fwd_combine(FwdArgs A) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int32_t i = (int32_t)(blockIdx.x / K);
  const int j = (int)(blockIdx.x % K);
  int32_t tile = i, slices = A.nsplit, slot = i * A.nsplit;
  if (A.split) {
    const ci32p p = (ci32p)(A.split + i);
    tile = p[0];
    slices = p[2];
    slot = p[3];
  }
  __shared__ double sum[16][64];
  const int32_t s0 = slices * wave / nw, s1 = slices * (wave + 1) / nw;
  const double* part = A.part + (int64_t)(slot + s0) * (64 * K) + 64 * j + lane;
  double v = 0.0;
  int32_t s = s0;
  for (; s + 8 <= s1; s += 8, part += 8 * 64 * K) {
    double t[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) t[q] = part[q * 64 * K];
#pragma unroll
    for (int q = 0; q < 8; ++q) v += t[q];
  }
  for (; s < s1; ++s, part += 64 * K) v += *part;
  sum[wave][lane] = v;
  __syncthreads();
  if (wave != 0) return;
  for (int w = 1; w < nw; ++w) v += sum[w][lane];
  const LaneRow lr = lane_row<K>(A, tile, lane);
  const int32_t at = lr.pos0 + j * lr.step;
  if (at < lr.cnt) A.map[lr.first + at] = v;
}

// ---------------------------------------------------------------------------
// Adjoint.
// ---------------------------------------------------------------------------
// Pixel table: direction (FP32) and cotangent (FP32) per pixel, plus the FP64
// direction for close pairs and visibility decisions.
// The adjoint's pixel table: per pixel n (FP32) and the cotangent, and n in
// FP64 with the cotangent; one zero record past the last pixel lets the
// pixel loop read one record ahead without a bound.
__global__ void k_pixtab(int64_t nside, int64_t npix, const double* dmap, float* tab32,
                         double* tab64) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p == npix) {
    ((float4*)tab32)[p] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  if (p > npix) return;
  double x, y, z;
  pix2vec_ring(nside, p, &x, &y, &z);
  ((float4*)tab32)[p] = make_float4((float)x, (float)y, (float)z, (float)dmap[p]);
  ((double2*)tab64)[2 * p + 0] = make_double2(x, y);
  ((double2*)tab64)[2 * p + 1] = make_double2(z, dmap[p]);
}

// Accumulators of one segment (see the finalize kernel for their use).  All
// of them are linear in kappa' = -2 eps dsigma / R, which is left out here
// and applied in FP64 by the finalize step.  With s the pixel's cotangent,
// d = n - Ph the direction difference of the pair, w = 1 - n.Ph = |d|^2/2,
// a = n.X', b = 1 + n.Xdot, v = Xdot.d, u = X'.d, r = 1/(b w) and
// m = v b - a u (the Eq. (1) term is kappa' m r):
//   0 S1  = sum s/w                      1 S2 = sum s a r
//   2 SF  = sum s m r                    3 C2 = sum s a u r/b
//   4 C4  = sum s u r                    5..7   D3 = sum (s m r/w) d
//   8..10 DV = sum (s/w + s a u r/b) d   11..13 DT = sum s r (u + a) d
// Every vector sum multiplies d rather than n: the n-weighted sums of the
// close pixels are each of order 1/theta larger than the result and would
// cancel against Ph times a scalar sum.
constexpr int kAcc = 14;

// Add one pair to the accumulators (see their list above): s the pixel's
// cotangent, a, b, w, v = Xdot.d, u = X'.d, r = 1/(b w), d = n - Ph.
// With g = s r: S1 += g b, S2 += g a, SF += g m, C4 += g u,
// C2 += (g u) a (w r), D3 += (g m)(b r) d, DV += (g b + C2 term) d,
// DT += (g a + g u) d.  The z components of DV and DT are left out: over a
// run of pixels with one d_z they are d_z (S1 + C2) and d_z (S2 + C4), added
// when the run ends (a close pixel adds what its d_z differs by).
// 25 instructions.
__device__ __forceinline__ void adj_accumulate(float (&pa)[kAcc], float s, float a, float bb,
                                               float w, float v, float u, float r, float dx,
                                               float dy, float dz) {
  const float g = s * r;
  const float m = fmaf(-a, u, v * bb);
  const float gm = g * m;                       // s m r
  pa[2] += gm;
  pa[0] = fmaf(g, bb, pa[0]);
  pa[1] = fmaf(g, a, pa[1]);
  const float gu = g * u;                       // s u r
  pa[4] += gu;
  const float c2 = (gu * a) * (w * r);          // s a u r / b
  pa[3] += c2;
  const float d3 = gm * (bb * r);               // s m r / w
  pa[5] = fmaf(d3, dx, pa[5]);
  pa[6] = fmaf(d3, dy, pa[6]);
  pa[7] = fmaf(d3, dz, pa[7]);
  const float dv = fmaf(g, bb, c2);             // s/w + s a u r/b
  pa[8] = fmaf(dv, dx, pa[8]);
  pa[9] = fmaf(dv, dy, pa[9]);
  const float c3 = fmaf(g, a, gu);              // s r (u + a)
  pa[11] = fmaf(c3, dx, pa[11]);
  pa[12] = fmaf(c3, dy, pa[12]);
}

// Per-lane constants of the adjoint's segment (see k_adj32).
struct AdjSeg {
  float px, py, pz, tx, ty, tz, vx, vy, vz;
  float c1, c2;   // 1 + Ph.Xdot, Ph.X'
  double hx, hy, hz;   // Ph in FP64
};

// Ring (1 .. 4N-1) of RING pixel p.
__device__ __forceinline__ int64_t ring_of_pixel(int64_t N, int64_t npix, int64_t p) {
  const int64_t ncap = 2 * N * (N - 1);
  if (p >= ncap && p < npix - ncap) return N + (p - ncap) / (4 * N);
  const bool south = p >= ncap;
  const int64_t q = south ? npix - 1 - p : p;
  // Cap ring i holds pixels 2 i (i - 1) .. 2 i (i + 1) - 1.
  int64_t i = (int64_t)((1.0 + sqrt(1.0 + 2.0 * (double)q)) * 0.5);
  while (2 * i * (i - 1) > q) --i;
  while (2 * i * (i + 1) <= q) ++i;
  return south ? 4 * N - i : i;
}

// The adjoint's pixel loop over [p0, p1).  The wavefront copies 64 pixel
// records at a time into its own LDS slots, the next 64 requested meanwhile,
// and every lane reads them back one by one as vector registers (one
// broadcast read per pixel; streamed through scalar registers, each pixel
// took three copies to vector registers, whose FMAs run at twice the rate).
// The pixels of a ring share z, so that the z parts of w, a, b and d are
// formed once per run of one ring, whose ends are known from the ring
// numbers; whether every pair of a run is far is settled once for the run,
// so that the far loop has no test and no branch per pixel.  kVis: the box
// has a visibility rule, tested per pixel.  kForce: the group takes the FP64
// form against every pixel.
// The far loop takes 37 vector instructions per pixel, unrolled by four; the
// loop that streamed pixels through scalar registers and tested each pair
// took 44.  12,000 segments against Nside 256: 8.1 against 8.8 ms; 4,000
// against Nside 1024: 41.9 against 44.3.  (One loop with the test kept but
// the records in LDS was slower, 11.9 ms: the compiler copied the
// accumulators where the paths met.)
template <bool kVis, bool kForce>
__device__ __forceinline__ void adj_pixels(const AdjArgs& A, const DevBox& bx, const AdjSeg& g,
                                           int64_t p0, int64_t p1, float4* lds, int lane,
                                           double (&acc)[kAcc]) {
  const float near_w = A.near_w, far_w = A.far_w;
  const float4* tab = (const float4*)A.pixtab;
  cd2p tab64 = (cd2p)A.pix64;
  constexpr int J = 64;
  const int64_t N = A.nside;
  const float th_far = acosf(fmaxf(-1.0f, 1.0f - far_w));
  auto ring_len = [&](int64_t i) {
    const int64_t k = i < 4 * N - i ? i : 4 * N - i;
    return 4 * (k < N ? k : N);
  };
  int64_t ring = uniform_i64(ring_of_pixel(N, A.npix, p0));
  int64_t ring_end;   // one past the ring's last pixel
  {
    const int64_t ncap = 2 * N * (N - 1), k = 4 * N - ring;
    ring_end = ring < N ? 2 * ring * (ring + 1)
                        : (ring <= 3 * N ? ncap + (ring - N + 1) * 4 * N : A.npix - 2 * k * (k - 1));
  }
  auto request = [&](int64_t p) { return tab[p + lane < A.npix ? p + lane : A.npix]; };
  float4 nxt = request(p0);
  for (int64_t pc = p0; pc < p1; pc += J) {
    lds[lane] = nxt;
    __builtin_amdgcn_wave_barrier();
    nxt = request(pc + J);
    // 32-bit counts keep the loop tests on the scalar unit.
    const int32_t rest = (int32_t)(p1 - pc), np = rest < J ? rest : J;
    int32_t i = 0;
    while (i < np) {
      if (i == (int32_t)(ring_end - pc)) ring_end += ring_len(++ring);
      const int32_t to = (int32_t)(ring_end - pc);
      const int32_t end = __builtin_amdgcn_readfirstlane(to < np ? to : np);
      const float z = lds[i].z;
      const float wz = fmaf(-z, g.pz, 1.0f), az = z * g.tz, bz = fmaf(z, g.vz, 1.0f);
      const float dzr = z - g.pz;
      // Whether every pair of the run is far: its pixels lie within rho of
      // its middle one (chord to the farther end; runs of more than half a
      // ring, or of a chord past 1, are not asked).
      bool far = false;
      if (!kForce && 2 * (int64_t)(end - i) <= ring_len(ring)) {
        const float4 c = lds[(i + end) >> 1], e0 = lds[i], e1 = lds[end - 1];
        const float d0 = fmaf(c.x - e0.x, c.x - e0.x, (c.y - e0.y) * (c.y - e0.y));
        const float d1 = fmaf(c.x - e1.x, c.x - e1.x, (c.y - e1.y) * (c.y - e1.y));
        const float chord = sqrtf(fmaxf(d0, d1));
        const float w = fmaf(-c.y, g.py, fmaf(-c.x, g.px, wz));
        far = chord < 1.0f && !__any(w < versine(th_far + 1.05f * chord + 1e-6f));
      }
      float pa[kAcc];
#pragma unroll
      for (int k = 0; k < kAcc; ++k) pa[k] = 0.f;
      const int32_t from = __builtin_amdgcn_readfirstlane(i);
      i = end;
      if (far) {
#pragma unroll 4
        for (int32_t q = from; q < end; ++q) {
          const float4 pt = lds[q];
          if (kVis) {
            const v2d e0 = tab64[2 * (pc + q)];
            const v2d e1 = tab64[2 * (pc + q) + 1];
            if (!sees_box(e0.x, e0.y, e1.x, bx, A.eta0)) continue;
          }
          const float w = fmaf(-pt.y, g.py, fmaf(-pt.x, g.px, wz));
          const float a = fmaf(pt.y, g.ty, fmaf(pt.x, g.tx, az));
          const float bb = fmaf(pt.y, g.vy, fmaf(pt.x, g.vx, bz));
          // Xdot.d = b - (1 + Ph.Xdot), X'.d = a - Ph.X'.
          adj_accumulate(pa, pt.w, a, bb, w, bb - g.c1, a - g.c2, __builtin_amdgcn_rcpf(bb * w),
                         pt.x - g.px, pt.y - g.py, dzr);
        }
      } else {
        for (int32_t j = from; j < end; ++j) {
          const int64_t p = pc + j;
          const float4 pt = lds[j];
          if (kVis) {
            const v2d e0 = tab64[2 * p + 0];
            const v2d e1 = tab64[2 * p + 1];
            if (!sees_box(e0.x, e0.y, e1.x, bx, A.eta0)) continue;
          }
          const float nx = pt.x, ny = pt.y;
          float s = pt.w;
          float w = fmaf(-ny, g.py, fmaf(-nx, g.px, wz));
          const float a = fmaf(ny, g.ty, fmaf(nx, g.tx, az));
          const float bb = fmaf(ny, g.vy, fmaf(nx, g.vx, bz));
          float dx = nx - g.px, dy = ny - g.py, dz = dzr;
          float v = bb - g.c1, u = a - g.c2;
          if (kForce || __any(w < far_w)) {
            // Middle form: the direction difference in FP32 (see the forward
            // kernel); FP64 form: from the FP64 directions.
            if (kForce || __any(w < near_w)) {
              const v2d e0 = tab64[2 * p + 0];
              const v2d e1 = tab64[2 * p + 1];
              dx = (float)(e0.x - g.hx);
              dy = (float)(e0.y - g.hy);
              dz = (float)(e1.x - g.hz);
            }
            const float q = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            v = fmaf(g.vz, dz, fmaf(g.vy, dy, g.vx * dx));
            u = fmaf(g.tz, dz, fmaf(g.ty, dy, g.tx * dx));
            // An exact coincidence (q = 0) contributes nothing.
            w = (q > 0.0f) ? 0.5f * q : 1.0f;
            s = (q > 0.0f) ? s : 0.0f;
          }
          const float r = __builtin_amdgcn_rcpf(bb * w), gr = s * r, gu = gr * u, dze = dz - dzr;
          pa[10] = fmaf(fmaf(gr, bb, (gu * a) * (w * r)), dze, pa[10]);
          pa[13] = fmaf(fmaf(gr, a, gu), dze, pa[13]);
          adj_accumulate(pa, s, a, bb, w, v, u, r, dx, dy, dz);
        }
      }
      pa[10] = fmaf(dzr, pa[0] + pa[3], pa[10]);
      pa[13] = fmaf(dzr, pa[1] + pa[4], pa[13]);
#pragma unroll
      for (int k = 0; k < kAcc; ++k) acc[k] += (double)pa[k];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Work item: a group of 64 consecutive kept records of one box (one per
// lane) and one of `nsplit` contiguous pixel ranges.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_adj32(AdjArgs A) {
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int64_t item = (int64_t)blockIdx.x * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (item >= (int64_t)A.ngroups * A.nsplit) return;
  const int32_t at = (int32_t)(item / A.nsplit), split = (int32_t)(item - (int64_t)at * A.nsplit);
  const int32_t b = ((ci32p)A.groups)[2 * at + 0];
  const int32_t grp = ((ci32p)A.groups)[2 * at + 1];
  const DevBox bx = load_box(A.boxes, b);
  const int64_t kept = load_kept(A.box_count, b);
  const int64_t li = (int64_t)grp * 64 + lane;
  const bool active = li < kept;
  const int64_t rec = bx.rec_off + (active ? li : 0);
  // Segment constants (per lane).
  const float4* R4 = (const float4*)(A.rec32 + (size_t)rec * kRec32);
  const float4 q0 = R4[0], q1 = R4[1], q2 = R4[2], q3 = R4[3];
  // 1 + Ph.Xdot and Ph.X' (the sums leave out kappa' = -2 eps dsigma / R,
  // which the finalize step applies, so they stay finite at dsigma = 0).
  const float4 cu = ((const float4*)A.adjc)[rec];
  const double2 h0 = ((const double2*)A.phat64)[2 * rec + 0];
  const double2 h1 = ((const double2*)A.phat64)[2 * rec + 1];
  const AdjSeg g = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x,
                    cu.x, cu.y, h0.x, h0.y, h1.x};
  // The pixel range is uniform; computing it through readfirstlane keeps it
  // (and the loop bound) in scalar registers.
  const int64_t p0 = uniform_i64(A.npix * split / A.nsplit);
  const int64_t p1 = uniform_i64(A.npix * (split + 1) / A.nsplit);
  // A group holding a segment flagged at precompute takes the FP64 form
  // against every pixel.
  const bool force = __any(active && __float_as_int(q3.y) != 0);
  __shared__ float4 px[4][64];
  float4* const lds = px[threadIdx.x >> 6];
  double acc[kAcc];
#pragma unroll
  for (int k = 0; k < kAcc; ++k) acc[k] = 0.0;
  if (force) {
    if (bx.vis != 0)
      adj_pixels<true, true>(A, bx, g, p0, p1, lds, lane, acc);
    else
      adj_pixels<false, true>(A, bx, g, p0, p1, lds, lane, acc);
  } else {
    if (bx.vis != 0)
      adj_pixels<true, false>(A, bx, g, p0, p1, lds, lane, acc);
    else
      adj_pixels<false, false>(A, bx, g, p0, p1, lds, lane, acc);
  }
  // Lanes past the box's last record repeat its first and are not read.
  const int64_t slots = 64 * (int64_t)A.ngroups;
  double* o = A.partial + (int64_t)split * kAcc * slots + 64 * (int64_t)at + lane;
#pragma unroll
  for (int k = 0; k < kAcc; ++k) o[k * slots] = acc[k];
}

// Combine the pixel-chunk partials of each kept record (in chunk order) and
// apply the per-segment chain rule, then scatter to the caller's arrays.
// The partial sums leave out kappa' = -2 eps dsigma / R; with S the sums
// times k = -2 eps / R (kappa' per unit dsigma):
//   G_d   = V S1 - T S2 - D3                   (sum of s df/d(n - Ph))
//   dL/dP = dsigma [-(G_d - Ph (Ph.G_d))/R - SF Ph / R] (Ph = P/R, dR/dP = Ph)
//   dL/dV = dsigma [DV + Ph C2 + SF V/(1 - V^2)]        (the last term from eps)
//   dL/dT = dsigma [-DT - Ph C4 + SF T/T^2]             (the last term from eps)
//   dL/ddsigma = SF                            (Eq. (1) is linear in dsigma)
// One workgroup per group of 64 records, all boxes in one launch: its
// wavefronts each add a run of the chunks in order (28 loads of 512 bytes in
// flight), then the runs are added in order.  The loads' latency bounds it: a
// thread per record reading its chunks one after another, a launch per box,
// took 65-76 us per box (1,500 records, 86 chunks), eight such boxes 521-608;
// one launch over the eight takes 19.
constexpr int kFinWaves = 8;
__global__ void __launch_bounds__(64 * kFinWaves) k_adj_finalize(AdjArgs A, const void* raw_base,
                                                                 const int64_t* raw_byte_off,
                                                                 const int32_t* orig_index,
                                                                 const GradPtrs* grads) {
  __shared__ double sum[kFinWaves][kAcc][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int32_t at = blockIdx.x;
  const int64_t slots = 64 * (int64_t)A.ngroups;
  double S[kAcc];
#pragma unroll
  for (int k = 0; k < kAcc; ++k) S[k] = 0.0;
  const int32_t s1 = A.nsplit * (wave + 1) / nw;
  int32_t sp = A.nsplit * wave / nw;
  const double* pp = A.partial + (int64_t)sp * kAcc * slots + 64 * (int64_t)at + lane;
  for (; sp + 2 <= s1; sp += 2, pp += 2 * kAcc * slots) {
    double t[2 * kAcc];
#pragma unroll
    for (int k = 0; k < 2 * kAcc; ++k) t[k] = pp[k * slots];
#pragma unroll
    for (int k = 0; k < kAcc; ++k) S[k] = (S[k] + t[k]) + t[kAcc + k];
  }
  if (sp < s1)
#pragma unroll
    for (int k = 0; k < kAcc; ++k) S[k] += pp[k * slots];
#pragma unroll
  for (int k = 0; k < kAcc; ++k) sum[wave][k][lane] = S[k];
  __syncthreads();
  if (wave != 0) return;
  for (int w = 1; w < nw; ++w)
#pragma unroll
    for (int k = 0; k < kAcc; ++k) S[k] += sum[w][k][lane];
  const int32_t b = ((ci32p)A.groups)[2 * at];
  const DevBox bx = load_box(A.boxes, b);
  const int64_t li = 64 * (int64_t)((ci32p)A.groups)[2 * at + 1] + lane;
  if (li >= load_kept(A.box_count, b)) return;
  const int64_t rec = bx.rec_off + li;
  const char* raw = (const char*)raw_base + raw_byte_off[b];
  const double* phat64 = A.phat64;
  const GradPtrs out = grads[b];
  const int64_t i = orig_index[rec];
  const int dt = bx.dtype;
  const int64_t n = bx.n;
  double V[3], T[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    V[k] = raw_at(raw, dt, 3 * n + 3 * i + k);
    T[k] = raw_at(raw, dt, 6 * n + 3 * i + k);
  }
  if (bx.rotated) {
    const double v[3] = {V[0], V[1], V[2]}, t[3] = {T[0], T[1], T[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      V[k] = rot_row(bx.rot, k, v);
      T[k] = rot_row(bx.rot, k, t);
    }
  }
  const double ds = raw_at(raw, dt, 9 * n + i);
  const double Ph[3] = {phat64[4 * rec + 0], phat64[4 * rec + 1], phat64[4 * rec + 2]};
  const double R = phat64[4 * rec + 3];
  const double vv = (V[0] * V[0] + V[1] * V[1]) + V[2] * V[2];
  const double tt = (T[0] * T[0] + T[1] * T[1]) + T[2] * T[2];
  const double kunit = -2.0 * sqrt(tt / (1.0 - vv)) / R;
#pragma unroll
  for (int k = 0; k < kAcc; ++k) S[k] *= kunit;
  double G[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) G[k] = V[k] * S[0] - T[k] * S[1] - S[5 + k];
  const double pg = (Ph[0] * G[0] + Ph[1] * G[1]) + Ph[2] * G[2];
  const double SF = S[2];
  double gx[3], gv[3], gt[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    gx[k] = ds * (-(G[k] - Ph[k] * pg) / R - SF * Ph[k] / R);
    gv[k] = ds * (S[8 + k] + Ph[k] * S[3] + SF * V[k] / (1.0 - vv));
    gt[k] = ds * (-S[11 + k] - Ph[k] * S[4] + SF * T[k] / tt);
  }
  // A rotated box: sky = rot * box, so d/d(box) = rot^T d/d(sky).
  const bool rot = bx.rotated != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (out.x) out.x[3 * i + k] = rot ? rot_col(bx.rot, k, gx) : gx[k];
    if (out.xd) out.xd[3 * i + k] = rot ? rot_col(bx.rot, k, gv) : gv[k];
    if (out.xp) out.xp[3 * i + k] = rot ? rot_col(bx.rot, k, gt) : gt[k];
  }
  if (out.ds) out.ds[i] = SF;
}

// ---------------------------------------------------------------------------
// Host-side launchers (C++ linkage, used by the API layer).
// ---------------------------------------------------------------------------
hipError_t launch_precompute(const PreArgs& A, int64_t nbox, hipStream_t st) {
  if (nbox == 0) return hipSuccess;
  // The scan runs for every box, also when no box has segments, so that every
  // kept count the pair kernels read has been written.
  if (A.nblk) k_pre_count<<<dim3((unsigned)A.nblk), dim3(kPreThreads), 0, st>>>(A);
  k_pre_scan<<<dim3((unsigned)nbox), dim3(256), 0, st>>>(A, nbox);
  if (A.nblk) k_pre_emit<<<dim3((unsigned)A.nblk), dim3(kPreThreads), 0, st>>>(A);
  return hipGetLastError();
}

// Arrays of 3n, 3n, 3n and n elements of es bytes (device memory, aligned to
// 4 bytes) to dst, back to back.
hipError_t launch_copy_box(void* dst, const void* const src[4], int64_t n, size_t es,
                           hipStream_t st) {
  CopyBox c;
  const int64_t words = n * (int64_t)(es / 4);
  c.dst = (uint32_t*)dst;
  for (int k = 0; k < 4; ++k) {
    c.src[k] = (const uint32_t*)src[k];
    c.end[k] = k < 3 ? 3 * words * (k + 1) : 10 * words;
  }
  k_copy_box<<<dim3((unsigned)((10 * words + 1023) / 1024)), dim3(256), 0, st>>>(c);
  return hipGetLastError();
}

hipError_t launch_fill(double* p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  k_fill_f64<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_zero_counters(unsigned long long* c, hipStream_t st) {
  k_zero_counters<<<1, 256, 0, st>>>(c);
  return hipGetLastError();
}

hipError_t launch_dir_table(int64_t nside, int64_t npix, double* x, double* y, double* z,
                           hipStream_t st) {
  k_dir_table<<<dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, st>>>(nside, npix, x, y, z);
  return hipGetLastError();
}

hipError_t launch_ang2pix(int64_t nside, int64_t n, const double* xyz, int64_t* pix,
                          hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_ang2pix<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(nside, n, xyz, pix);
  return hipGetLastError();
}

hipError_t launch_pix2vec(int64_t nside, int64_t first, int64_t count, double* xyz,
                          hipStream_t st) {
  if (count <= 0) return hipSuccess;
  k_pix2vec<<<dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st>>>(nside, first, count,
                                                                          xyz);
  return hipGetLastError();
}

static size_t fwd32_lds(int K, unsigned block) {
  return sizeof(double) * 3 * 64 * (size_t)K * (block / 64);
}

template <int K, bool P>
static void fwd_launch(bool fp64, const FwdArgs& A, unsigned grid, unsigned block,
                       hipStream_t st) {
  if (fp64)
    k_fwd64<K, P><<<dim3(grid), dim3(block), 0, st>>>(A);
  else if (A.frac)
    k_fwd32<K, P, true><<<dim3(grid), dim3(block), fwd32_lds(K, block), st>>>(A);
  else
    k_fwd32<K, P, false><<<dim3(grid), dim3(block), fwd32_lds(K, block), st>>>(A);
}

template <int K, bool P>
static int fwd_occupancy(bool fp64, bool frac, unsigned block) {
  int nb = 0;
  hipError_t e;
  if (fp64)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd64<K, P>, (int)block, 0);
  else if (frac)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd32<K, P, true>, (int)block,
                                                      fwd32_lds(K, block));
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd32<K, P, false>, (int)block,
                                                      fwd32_lds(K, block));
  return e == hipSuccess ? nb : 0;
}

// Workgroups of the persistent forward kernel that fit on one CU at once.
int forward_blocks_per_cu(bool fp64, bool frac, int K, unsigned block) {
  switch (K) {
    case 1: return fwd_occupancy<1, true>(fp64, frac, block);
    case 2: return fwd_occupancy<2, true>(fp64, frac, block);
    case 4: return fwd_occupancy<4, true>(fp64, frac, block);
    case 8: return fwd_occupancy<8, true>(fp64, frac, block);
  }
  return 0;
}

// Frames of the ntiles tiles of A's tiling (K = 8).
hipError_t launch_tile_frames(const FwdArgs& A, int64_t ntiles, TileFrame* out, hipStream_t st) {
  if (ntiles > 0)
    k_tile_frames<8><<<dim3((unsigned)((ntiles + 3) / 4)), dim3(256), 0, st>>>(A, ntiles, out);
  return hipGetLastError();
}

// Workgroups of the persistent matrix-core forward kernel on one CU.
int forward_m_blocks_per_cu() {
  int nb = 0;
  const hipError_t e =
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd32m<true>, 256, 0);
  return e == hipSuccess ? nb : 0;
}

static hipError_t launch_combine(int K, const FwdArgs& A, hipStream_t st);

// One workgroup per work item, or the persistent grid of `grid` workgroups.
hipError_t launch_forward_m(bool persistent, const FwdArgs& A, unsigned grid, hipStream_t st) {
  if (persistent) k_fwd32m<true><<<dim3(grid), dim3(256), 0, st>>>(A);
  else k_fwd32m<false><<<dim3((unsigned)A.nitems), dim3(256), 0, st>>>(A);
  return launch_combine(8, A, st);
}

hipError_t launch_forward(bool fp64, int K, bool persistent, const FwdArgs& A, unsigned grid,
                          unsigned block, hipStream_t st) {
  switch (K) {
    case 1: persistent ? fwd_launch<1, true>(fp64, A, grid, block, st)
                       : fwd_launch<1, false>(fp64, A, grid, block, st); break;
    case 2: persistent ? fwd_launch<2, true>(fp64, A, grid, block, st)
                       : fwd_launch<2, false>(fp64, A, grid, block, st); break;
    case 4: persistent ? fwd_launch<4, true>(fp64, A, grid, block, st)
                       : fwd_launch<4, false>(fp64, A, grid, block, st); break;
    case 8: persistent ? fwd_launch<8, true>(fp64, A, grid, block, st)
                       : fwd_launch<8, false>(fp64, A, grid, block, st); break;
    default: return hipErrorInvalidValue;
  }
  return launch_combine(K, A, st);
}

static hipError_t launch_combine(int K, const FwdArgs& A, hipStream_t st) {
  const int64_t nt = A.split ? A.nsplit_tiles : (A.nsplit > 1 ? A.nitems / A.nsplit : 0);
  if (nt > 0) {
    // About eight slices (one round of loads) per wavefront, at most 16.
    int nw = 1;
    while (nw < 16 && 8 * nw < A.max_slices) nw *= 2;
    const dim3 cg((unsigned)(nt * K)), cb(64 * nw);
    switch (K) {
      case 1: k_fwd_combine<1><<<cg, cb, 0, st>>>(A); break;
      case 2: k_fwd_combine<2><<<cg, cb, 0, st>>>(A); break;
      case 4: k_fwd_combine<4><<<cg, cb, 0, st>>>(A); break;
      case 8: k_fwd_combine<8><<<cg, cb, 0, st>>>(A); break;
    }
  }
  return hipGetLastError();
}

hipError_t launch_pixtab(int64_t nside, int64_t npix, const double* dmap, float* tab32,
                         double* tab64, hipStream_t st) {
  k_pixtab<<<dim3((unsigned)((npix + 256) / 256)), dim3(256), 0, st>>>(nside, npix, dmap, tab32,
                                                                        tab64);
  return hipGetLastError();
}

// Workgroups (four wavefronts) of the adjoint pair kernel on one CU.
int adjoint_blocks_per_cu() {
  int nb = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_adj32, 256, 0);
  return e == hipSuccess ? nb : 0;
}

hipError_t launch_adjoint(const AdjArgs& A, hipStream_t st) {
  if (A.ngroups == 0) return hipSuccess;
  const unsigned grid = (unsigned)(((int64_t)A.ngroups * A.nsplit + 3) / 4);
  k_adj32<<<dim3(grid), dim3(256), 0, st>>>(A);
  return hipGetLastError();
}

hipError_t launch_adj_finalize(const AdjArgs& A, const void* raw, const int64_t* raw_byte_off,
                               const int32_t* orig_index, const GradPtrs* grads, hipStream_t st) {
  if (A.ngroups == 0) return hipSuccess;
  const int nw = A.nsplit < kFinWaves ? A.nsplit : kFinWaves;
  k_adj_finalize<<<dim3((unsigned)A.ngroups), dim3(64 * nw), 0, st>>>(A, raw, raw_byte_off,
                                                                     orig_index, grads);
  return hipGetLastError();
}

}  // namespace csmap
