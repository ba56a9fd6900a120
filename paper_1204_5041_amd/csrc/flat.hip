// flat.hip -- flat-sky small-angle maps on a gnomonic patch.
//
// The small-angle, flat-sky form of Eq. (1) (Sec. II.A: X n -> X, every
// photon path parallel to the patch axis c; Sec. III.B, Fig. 3 compares such
// maps with a gnomonic projection of the full-sky map).  A segment at P, at
// depth D = c.P, is seen at the plane position s = (e1.P, e2.P)/D; with u
// built from c instead of n, u = Xdot - (c.X')/(1 + c.Xdot) X', pixel t
// receives -4 eps dsigma (u_perp . (t - s)) / (D |t - s|^2).
//
//   records : per kept segment (the light-cone stage, with the patch's
//             acceptance cone, has compacted them), the plane position in
//             pixel units as an FP32 pair hi + lo and the two weights
//             a = -4 eps dsigma u_perp / (D h), from FP64 geometry.
//   far     : with z = x + i y and W = a_x + i a_y a pixel receives
//             Re sum_s W_s / (z - z_s), so the segments that lie beyond three
//             times a tile's radius rho from its centre c act on its pixels
//             through one power series: with d = z_s - c and r = rho/d,
//               sum_s W_s / (z - z_s) = sum_k L_k ((z - c)/rho)^k,
//               L_k = -sum_s (W_s r/rho) r^k,
//             of which kFlatTerms terms, in FP64, leave out less than 5e-10
//             of each segment's own term.  A (tile, segment) pair costs about
//             six FP64 operations a term where 32 x 32 pixels one by one cost
//             some 10,000 FP32 ones.  Large patches take a second series over
//             tiles of 128 x 128 for what is far from those, so that a tile's
//             own series runs over its surroundings only.
//   near    : the other segments pixel by pixel in FP32: a wavefront owns a
//             tile of 32 x 32 pixels (16 consecutive pixels of a row per
//             lane), and the terms of two records are folded into one
//             fraction before the division.
// A wavefront finds its records (far or near ones) by testing 256 plane
// positions at a time and stacks them in LDS, so that it always works on 64.
// At 1024 x 1024 pixels and 200,000 segments far takes 368 us and near 340;
// pixel by pixel for all, nine FP32 operations a pair, took 31.8 ms.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"
#include "segment_dev.h"

namespace csmap {

constexpr int kFlatTile = 32;        // tile side of the near sums and of the finer series
constexpr int kFlatTile1 = 128;      // tile side of the coarser series
constexpr int kFlatK = 16;           // pixels per lane
constexpr int kFlatTerms = 20;       // series terms
constexpr int kFlatCoef = 2 * kFlatTerms;
constexpr int kFlatChunk = 32;       // records per FP32 partial sum
constexpr float kFlatTiny = 1e-18f;  // floor of |t - s|^2 (pixel units): an exact hit gives 0

// 1/x for x in [2^-125, 2^125] on the ordinary FP32 pipeline: the hardware
// reciprocal is a transcendental instruction that costs the pair loop about
// ten ordinary ones.  Subtracting the bits of x = 2^E (1 + f) from those of
// 2^127 would negate the exponent and map the mantissa to 2 - f, a seed y0
// with x y0 in [1, 1.125]; the constant used, 0x7EF311C2, is that one less
// 847422, the shift that minimises max |1 - x y0| over all mantissas (5.05e-2).
// A Newton step of third order, y <- y + y (e + e^2) with e = 1 - x y, cubes
// the relative error (to 1.3e-4), one of second order, y <- y + y e, squares
// it (to 1.7e-8), which leaves the result within 0.8 ulp of 1/x (the hardware
// reciprocal is within 1 ulp).
__device__ __forceinline__ float recip_newton(float x) {
  float y = __uint_as_float(0x7EF311C2u - __float_as_uint(x));
  float e = fmaf(-x, y, 1.0f);
  y = fmaf(y, fmaf(e, e, e), y);
  e = fmaf(-x, y, 1.0f);
  return fmaf(y, e, y);
}

// Exclusive prefix over boxes of their kept counts.
__global__ void __launch_bounds__(256) k_flat_scan(FlatArgs A) {
  __shared__ int64_t sh[256];
  int64_t running = 0;
  for (int64_t c0 = 0; c0 < A.nbox; c0 += 256) {
    const int64_t b = c0 + threadIdx.x;
    const int64_t v = (b < A.nbox) ? A.box_count[b].kept : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
      const int64_t add = (threadIdx.x >= (unsigned)off) ? sh[threadIdx.x - off] : 0;
      __syncthreads();
      sh[threadIdx.x] += add;
      __syncthreads();
    }
    if (b < A.nbox) A.flat_off[b] = running + sh[threadIdx.x] - v;
    const int64_t tot = sh[255];
    __syncthreads();
    running += tot;
  }
  if (threadIdx.x == 0) A.flat_off[A.nbox] = running;
}

// One thread per kept record (four per thread, as the emit pass).
__global__ void __launch_bounds__(kPreThreads) k_flat_rec(FlatArgs A) {
  const int64_t blk = blockIdx.x;
  const int b = ((ci32p)A.blk_box)[blk];
  const DevBox bx = load_box(A.boxes, b);
  const int64_t kept = load_kept(A.box_count, b);
  const int64_t base = (blk - bx.blk_off) * kPreBlock;
  if (base >= kept) return;
  const char* raw = (const char*)A.raw + A.raw_byte_off[b];
  const int64_t out0 = A.flat_off[b];
  for (int j = 0; j < kPreBlock / kPreThreads; ++j) {
    const int64_t li = base + threadIdx.x + kPreThreads * j;
    if (li >= kept) break;
    const int64_t i = A.orig_index[bx.rec_off + li];
    const SegGeom g = seg_geom(bx, raw, i, A.eta0);
    const double D = (A.c[0] * g.P[0] + A.c[1] * g.P[1]) + A.c[2] * g.P[2];
    const double ca = (A.c[0] * g.T[0] + A.c[1] * g.T[1]) + A.c[2] * g.T[2];
    const double cb = 1.0 + ((A.c[0] * g.V[0] + A.c[1] * g.V[1]) + A.c[2] * g.V[2]);
    double u[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) u[k] = g.V[k] - (ca / cb) * g.T[k];
    const double kap = -4.0 * g.eps * g.ds / D * A.inv_h;
    const double sx = ((A.e1[0] * g.P[0] + A.e1[1] * g.P[1]) + A.e1[2] * g.P[2]) / D * A.inv_h +
                      A.off_x;
    const double sy = ((A.e2[0] * g.P[0] + A.e2[1] * g.P[1]) + A.e2[2] * g.P[2]) / D * A.inv_h +
                      A.off_y;
    const float sxh = (float)sx, syh = (float)sy;
    const float ax = (float)(kap * ((A.e1[0] * u[0] + A.e1[1] * u[1]) + A.e1[2] * u[2]));
    const float ay = (float)(kap * ((A.e2[0] * u[0] + A.e2[1] * u[1]) + A.e2[2] * u[2]));
    float4* o = (float4*)(A.rec + (size_t)(out0 + li) * kFlatRec);
    o[0] = make_float4(sxh, (float)(sx - (double)sxh), syh, (float)(sy - (double)syh));
    o[1] = make_float4(ax, ay, 0.f, 0.f);
    // The position that decides near or far; a weight that is not finite acts
    // pixel by pixel (a NaN position is far from nothing).
    const bool finite = fabsf(ax) + fabsf(ay) < INFINITY;
    A.pos[out0 + li] = finite ? make_float2(sxh, syh) : make_float2(NAN, NAN);
  }
}

// Blocks are numbered over a grid of two dimensions: a patch of 2^30 x 1
// pixels has more tiles than one dimension takes.
constexpr int64_t kGridX = int64_t(1) << 20;

__device__ __forceinline__ int64_t block_index() {
  return (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
}

// Centre of tile i of side T along one axis, and whether a position is near
// a tile: every kernel decides by these, so that no record is counted twice.
__device__ __forceinline__ float tile_centre(int64_t i, int T) {
  return (float)((double)(i * T) + 0.5 * (double)(T - 1));
}

__device__ __forceinline__ bool is_near(float2 p, float cx, float cy, float r2) {
  const float dx = p.x - cx, dy = p.y - cy;
  return !(fmaf(dx, dx, dy * dy) > r2);
}

// The records of one wavefront's range that `want` takes, 64 at a time: the
// range's positions are tested 256 at a time (four loads in flight per lane),
// the indices of those taken are stacked in LDS (kFlatQueue entries), and
// `work(index, have)` runs on all lanes whenever 64 wait, and once more on the
// rest, with `have` of the lanes holding one.  `work` stands in the code once,
// which a short launch has to fetch; indices within the range have 32 bits.
constexpr int kFlatQueue = 64 + 256;

template <typename Want, typename Work>
__device__ __forceinline__ void for_records(const float2* __restrict__ pos, int64_t rbeg,
                                            int64_t rend, uint32_t* queue, Want want, Work work) {
  const uint32_t lane = threadIdx.x & 63, n = (uint32_t)(rend - rbeg);
  const float2* const range = pos + rbeg;
  uint32_t waiting = 0;
  for (uint32_t base = 0; base < n; base += 256) {
    float2 p[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) p[g] = range[min(base + 64 * g + lane, n - 1)];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint32_t i = base + 64 * g + lane;
      const bool take = i < n && want(p[g]);
      const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
      if (take)
        queue[waiting + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0))] = i;
      waiting += (uint32_t)__builtin_popcountll(mask);
    }
    const bool last = base + 256 >= n;
    while (waiting >= 64 || (last && waiting > 0)) {
      const uint32_t have = min(waiting, 64u);
      __builtin_amdgcn_wave_barrier();
      const uint32_t now = queue[waiting - have + min(lane, have - 1)];
      __builtin_amdgcn_wave_barrier();
      waiting -= have;
      work(rbeg + now, (int)have);
    }
  }
}

// 1/x of a positive normal x: the hardware seed and one step of third order.
__device__ __forceinline__ double recip64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Series of one tile over one record range: work item w = 4 (block) +
// (wavefront) is tile w mod ntiles and range w / ntiles.  Each lane sums the
// terms of its own records and the wavefront adds its lanes at the end.
__global__ void __launch_bounds__(256) k_flat_far(FlatArgs A, FlatLevel lv, FlatLevel up) {
  __shared__ uint32_t queue_all[4][kFlatQueue];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t item = block_index() * 4 + wave;
  if (item >= lv.ntiles * lv.nsplit) return;
  const int64_t split = item / lv.ntiles, tile = item - split * lv.ntiles;
  const int64_t ty = tile / lv.tx, tx = tile - ty * lv.tx;
  const int64_t nrec = ((const int64_t __attribute__((address_space(4)))*)A.flat_off)[A.nbox];
  const int64_t rbeg = nrec * split / lv.nsplit, rend = nrec * (split + 1) / lv.nsplit;
  const float cx = tile_centre(tx, lv.side), cy = tile_centre(ty, lv.side);
  const int ratio = up.series ? up.side / lv.side : 1;
  const float ux = up.series ? tile_centre(tx / ratio, up.side) : 0.f;
  const float uy = up.series ? tile_centre(ty / ratio, up.side) : 0.f;
  const double cxd = (double)(tx * lv.side) + 0.5 * (double)(lv.side - 1);
  const double cyd = (double)(ty * lv.side) + 0.5 * (double)(lv.side - 1);
  double L[kFlatCoef];
#pragma unroll
  for (int k = 0; k < kFlatCoef; ++k) L[k] = 0.0;
  for_records(
      A.pos, rbeg, rend, queue_all[wave],
      [&](float2 p) {
        return !is_near(p, cx, cy, lv.near2) && (!up.series || is_near(p, ux, uy, up.near2));
      },
      [&](int64_t i, int have) {
        const float4* rec = (const float4*)(A.rec + (size_t)i * kFlatRec);
        const float4 s = rec[0], w = rec[1];
        const bool on = lane < have;
        const double dx = on ? ((double)s.x + (double)s.y) - cxd : 1.0;
        const double dy = on ? ((double)s.z + (double)s.w) - cyd : 0.0;
        const double inv = lv.rho * recip64(fma(dx, dx, dy * dy));
        const double rx = dx * inv, ry = -(dy * inv);   // r = rho / d
        const double wx = on ? -(double)w.x * lv.inv_rho : 0.0;
        const double wy = on ? -(double)w.y * lv.inv_rho : 0.0;
        double gx = fma(wx, rx, -(wy * ry)), gy = fma(wx, ry, wy * rx);
#pragma unroll
        for (int k = 0; k < kFlatTerms; ++k) {
          L[2 * k] += gx;
          L[2 * k + 1] += gy;
          const double t = fma(gx, rx, -(gy * ry));
          gy = fma(gx, ry, gy * rx);
          gx = t;
        }
      });
  // Sums over the lanes: three steps that halve the values a lane holds (bit
  // 5, 4, 3 of the lane picks the half), then three over whole sums.
  int held = kFlatCoef;
#pragma unroll
  for (int bit = 32; bit >= 8; bit >>= 1) {
    held /= 2;
    const bool high = (lane & bit) != 0;
#pragma unroll
    for (int k = 0; k < kFlatCoef / 2; ++k) {
      if (k < held) {
        const double give = high ? L[k] : L[k + held];
        const double keep = high ? L[k + held] : L[k];
        L[k] = keep + __shfl_xor(give, bit);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kFlatCoef / 8; ++k) {
    for (int bit = 4; bit >= 1; bit >>= 1) L[k] += __shfl_xor(L[k], bit);
  }
  if ((lane & 7) == 0) {
    const int first = ((lane & 32) ? kFlatCoef / 2 : 0) + ((lane & 16) ? kFlatCoef / 4 : 0) +
                      ((lane & 8) ? kFlatCoef / 8 : 0);
    double* out = lv.coef + (split * lv.ntiles + tile) * kFlatCoef + first;
#pragma unroll
    for (int k = 0; k < kFlatCoef / 8; ++k) out[k] = L[k];
  }
}

// Near records of one tile and one record range, pixel by pixel: lane l holds
// pixels 16 (l mod 2) .. + 15 of the tile's row l / 2.  The sums go to
// parts[range][pixel], with one range to the map.
__global__ void __launch_bounds__(256) k_flat_near(FlatArgs A, FlatLevel lv, double* parts) {
  __shared__ uint32_t queue_all[4][kFlatQueue];
  __shared__ float4 rec_all[4][2 * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t item = block_index() * 4 + wave;
  if (item >= lv.ntiles * lv.nsplit) return;
  const int64_t split = item / lv.ntiles, tile = item - split * lv.ntiles;
  const int64_t ty = tile / lv.tx, tx = tile - ty * lv.tx;
  const int64_t nrec = ((const int64_t __attribute__((address_space(4)))*)A.flat_off)[A.nbox];
  const int64_t rbeg = nrec * split / lv.nsplit, rend = nrec * (split + 1) / lv.nsplit;
  const float cx = tile_centre(tx, lv.side), cy = tile_centre(ty, lv.side);
  const int64_t y = ty * kFlatTile + lane / 2, x0 = tx * kFlatTile + (lane & 1) * kFlatK;
  const float fy = (float)y, fx = (float)x0;
  float4* const recs = rec_all[wave];
  float acc[kFlatK], cmp[kFlatK], part[kFlatK];
#pragma unroll
  for (int j = 0; j < kFlatK; ++j) {
    acc[j] = 0.f;
    cmp[j] = 0.f;
    part[j] = 0.f;
  }
  auto flush = [&]() {
#pragma unroll
    for (int j = 0; j < kFlatK; ++j) {
      kahan_add(acc[j], cmp[j], part[j]);
      part[j] = 0.f;
    }
  };
  for_records(
      A.pos, rbeg, rend, queue_all[wave], [&](float2 p) { return !lv.series || is_near(p, cx, cy, lv.near2); },
      [&](int64_t i, int have) {
        const float4* rec = (const float4*)(A.rec + (size_t)i * kFlatRec);
        recs[2 * lane] = rec[0];
        // A record without weight completes an odd count.
        recs[2 * lane + 1] = lane < have ? rec[1] : make_float4(0.f, 0.f, 0.f, 0.f);
        __builtin_amdgcn_wave_barrier();
        for (int r = 0; r < have; r += 2) {
          const float4 pa = recs[2 * r], wa = recs[2 * r + 1];
          const float4 pb = recs[2 * r + 2], wb = recs[2 * r + 3];
          // x - s = ((x0 - s_hi) + j) - s_lo: the first two steps are exact for
          // a pixel near the segment, so s_lo is subtracted at the scale of the
          // pixel's own offset (subtracting it before adding j would round at
          // the scale of x0 - s and cost nearly-coincident pairs their accuracy).
          const float hxa = fx - pa.x, dya = (fy - pa.z) - pa.w;
          const float hxb = fx - pb.x, dyb = (fy - pb.z) - pb.w;
          const float ya2 = fmaf(dya, dya, kFlatTiny), yb2 = fmaf(dyb, dyb, kFlatTiny);
          const float aya = wa.y * dya, ayb = wb.y * dyb;
          // Each stage runs over half the lane's pixels before the next starts,
          // so that independent operations separate dependent ones.
#pragma unroll
          for (int h = 0; h < kFlatK; h += kFlatK / 2) {
            float xa[kFlatK / 2], xb[kFlatK / 2], qa[kFlatK / 2], qb[kFlatK / 2], rq[kFlatK / 2];
#pragma unroll
            for (int j = 0; j < kFlatK / 2; ++j) {
              xa[j] = (hxa + (float)(h + j)) - pa.y;
              xb[j] = (hxb + (float)(h + j)) - pb.y;
            }
#pragma unroll
            for (int j = 0; j < kFlatK / 2; ++j) {
              qa[j] = fmaf(xa[j], xa[j], ya2);
              qb[j] = fmaf(xb[j], xb[j], yb2);
            }
#pragma unroll
            // qa qb >= kFlatTiny^2 = 1e-36 > 2^-125, and below 2^122 because the
            // entry point admits only patches whose pixel offsets stay below
            // 2^30: inside recip_newton's range.
            for (int j = 0; j < kFlatK / 2; ++j) rq[j] = recip_newton(qa[j] * qb[j]);
#pragma unroll
            for (int j = 0; j < kFlatK / 2; ++j) {
              const float na = fmaf(wa.x, xa[j], aya), nb = fmaf(wb.x, xb[j], ayb);
              const float num = fmaf(na, qb[j], nb * qa[j]);
              part[h + j] = fmaf(num, rq[j], part[h + j]);
            }
          }
          if ((r & (kFlatChunk - 2)) == kFlatChunk - 2) flush();
        }
        __builtin_amdgcn_wave_barrier();
      });
  flush();
  if (y >= A.ny) return;
  double* out = (lv.nsplit == 1 ? A.map : parts + split * (A.nx * A.ny)) + y * A.nx;
#pragma unroll
  for (int j = 0; j < kFlatK; ++j)
    if (x0 + j < A.nx) out[x0 + j] = (double)acc[j] - (double)cmp[j];
}

// The map of one tile, or of a kCut-th of it: the near sums in range order,
// plus the real part of the tile's series and of its coarser tile's, each
// summed over its ranges.  A pixel's ranges are cut over kGroups threads.
// A patch of few tiles has many ranges and leaves the chip to a few blocks:
// 32 x 32 pixels with 256 ranges took 250 us with one block per tile.
template <int kCut, int kGroups>
__global__ void __launch_bounds__(256) k_flat_combine(FlatArgs A, FlatLevel lv, FlatLevel up,
                                                      const double* __restrict__ parts) {
  constexpr int kPix = 256 / kGroups;   // pixels at a time
  __shared__ double near_sum[kGroups][kPix];
  __shared__ double sum[6][kFlatCoef], L[2][kFlatCoef];
  const int64_t tile = block_index() / kCut, ty = tile / lv.tx, tx = tile - ty * lv.tx;
  const int t = threadIdx.x;
  if (tile >= lv.ntiles) return;
  const int ratio = up.series ? up.side / lv.side : 1;
  for (int level = 0; level < lv.series + up.series; ++level) {
    const FlatLevel& v = level ? up : lv;
    const int64_t at = level ? (ty / ratio) * up.tx + tx / ratio : tile;
    if (t < 6 * kFlatCoef) {
      const int k = t % kFlatCoef, g = t / kFlatCoef;
      double acc = 0.0;
      for (int64_t s = g; s < v.nsplit; s += 6) acc += v.coef[(s * v.ntiles + at) * kFlatCoef + k];
      sum[g][k] = acc;
    }
    __syncthreads();
    if (t < kFlatCoef) {
      double acc = sum[0][t];
      for (int g = 1; g < 6; ++g) acc += sum[g][t];
      L[level][t] = acc;
    }
    __syncthreads();
  }
  const int64_t npix = A.nx * A.ny;
  const double* in = lv.nsplit == 1 ? A.map : parts;
  const int group = t / kPix;
  const int first = (int)(block_index() % kCut) * (kFlatTile * kFlatTile / kCut);
  for (int m0 = first; m0 < first + kFlatTile * kFlatTile / kCut; m0 += kPix) {
    const int m = m0 + t % kPix;
    const int64_t x = tx * kFlatTile + m % kFlatTile, y = ty * kFlatTile + m / kFlatTile;
    const bool inside = x < A.nx && y < A.ny;
    const int64_t p = y * A.nx + x;
    double v = 0.0;
    if (inside) {
      const int64_t s1 = lv.nsplit * (group + 1) / kGroups;
#pragma unroll 8
      for (int64_t s = lv.nsplit * group / kGroups; s < s1; ++s) v += in[s * npix + p];
    }
    if constexpr (kGroups > 1) {
      near_sum[group][t % kPix] = v;
      __syncthreads();
      if (group == 0)
        for (int g = 1; g < kGroups; ++g) v += near_sum[g][t];
    }
    if (!inside || group) continue;
    for (int level = 0; level < lv.series + up.series; ++level) {
      const FlatLevel& l = level ? up : lv;
      const int64_t ix = level ? tx / ratio : tx, iy = level ? ty / ratio : ty;
      const double zx = ((double)(x - ix * l.side) - 0.5 * (double)(l.side - 1)) * l.inv_rho;
      const double zy = ((double)(y - iy * l.side) - 0.5 * (double)(l.side - 1)) * l.inv_rho;
      double hx = L[level][kFlatCoef - 2], hy = L[level][kFlatCoef - 1];
#pragma unroll
      for (int k = kFlatTerms - 2; k >= 0; --k) {
        const double nx = fma(hx, zx, fma(-hy, zy, L[level][2 * k]));
        hy = fma(hx, zy, fma(hy, zx, L[level][2 * k + 1]));
        hx = nx;
      }
      v += hx;
    }
    A.map[p] = v;
  }
}

// Caller directions (n x 3, any positive length) as unit vectors in three
// arrays, the layout the forward kernels read pixel directions from.
__global__ void k_dirs_soa(int64_t n, const double* xyz, double* x, double* y, double* z) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double a = xyz[3 * i], b = xyz[3 * i + 1], c = xyz[3 * i + 2];
  const double r = sqrt((a * a + b * b) + c * c);
  x[i] = a / r;
  y[i] = b / r;
  z[i] = c / r;
}

hipError_t launch_dirs_soa(int64_t n, const double* xyz, double* x, double* y, double* z,
                           hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_dirs_soa<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(n, xyz, x, y, z);
  return hipGetLastError();
}

hipError_t launch_flat(const FlatArgs& A, hipStream_t st) {
  k_flat_scan<<<1, 256, 0, st>>>(A);
  if (A.nblk) k_flat_rec<<<dim3((unsigned)A.nblk), dim3(kPreThreads), 0, st>>>(A);
  return hipGetLastError();
}

// The tiles of one level on nx x ny pixels, with `nseg` records at most.
// A position is near within three radii; FP32 rounds positions and centres on
// a patch of n pixels by some n 2^-23, which the bound exceeds.
static FlatLevel flat_level(int64_t nx, int64_t ny, int side) {
  FlatLevel v;
  v.side = side;
  v.tx = (nx + side - 1) / side;
  v.ntiles = v.tx * ((ny + side - 1) / side);
  v.rho = 0.5 * (side - 1) * sqrt(2.0);
  v.inv_rho = 1.0 / v.rho;
  const double near = 3.0 * v.rho * (1.0 + 0x1p-16) + (double)(nx + ny) * 0x1p-20;
  v.near2 = (float)(near * near);
  v.coef = nullptr;
  v.nsplit = 1;
  v.series = 0;
  return v;
}

// The levels of a patch whose segments reach `reach` pixels from its axis.
// The finer series runs unless every segment is near every tile, or so few
// (tile, segment) pairs are left that its launch costs more than its pixels
// one by one (33 us of kernels either way at 256 x 128 pixels and 1000
// segments; 29 with it and 16 without at 45 x 1 and 1200).  The coarser one
// pays where most segments lie beyond its near bound (270 pixels) and the
// finer tiles meet many segments; a pass without and with it: 1508 and 720 us
// at 1024^2 pixels (reach 853), 672 and 560 at 512^2 (426), 200,000 segments;
// 151 and 159 us at 512^2, 5000 segments; 163 and 211 us at 400 x 13 (333),
// 200,000 segments.  Figures of one pass over all segments before: 32.1 ms at
// 1024^2 and 200,000 segments (770 us now), 2.35 ms at 256^2 and 100,000 (227).
FlatPlan flat_plan(int64_t nx, int64_t ny, int64_t nseg, double reach) {
  FlatPlan p;
  p.lv = flat_level(nx, ny, kFlatTile);
  p.up = flat_level(nx, ny, kFlatTile1);
  auto farthest = [](int64_t n) {   // tile centre from the axis, along one side
    const double off = 0.5 * (double)(n - 1), c = 0.5 * (kFlatTile - 1);
    return std::max(off - c, (double)((n - 1) / kFlatTile * kFlatTile) + c - off);
  };
  const double most = reach + sqrt(farthest(nx) * farthest(nx) + farthest(ny) * farthest(ny)) + 1.0;
  p.lv.series = most * most > (double)p.lv.near2 && p.lv.ntiles * nseg >= int64_t(1) << 15;
  p.up.series = p.lv.series && reach * reach >= 2.0 * (double)p.up.near2 &&
                p.lv.ntiles * nseg >= int64_t(1) << 24;
  // Record ranges per tile: enough that a launch has about 4096 wavefronts
  // (as many as are resident), at most 1024, each of at least 16 records or,
  // where a range's series must pay for the sum over its lanes, 32 (256^2
  // pixels, 1000 segments: 52 us of kernels with 16, 37 with 32), and of at
  // most 2^30.  With 8192 wavefronts a pass took 235 us at 256^2 pixels and
  // 100,000 segments (4096: 227) and 760 us at 1024^2 and 200,000 (776).
  const int64_t least = p.lv.series ? 32 : 16;
  for (FlatLevel* v : {&p.lv, &p.up})
    v->nsplit = std::max<int64_t>(
        1 + (nseg >> 30),
        std::min<int64_t>({(4096 + v->ntiles - 1) / v->ntiles, 1024, nseg / least}));
  p.part_doubles = p.lv.nsplit > 1 ? p.lv.nsplit * nx * ny : 0;
  p.lv_doubles = p.lv.series * p.lv.nsplit * p.lv.ntiles * kFlatCoef;
  p.up_doubles = p.up.series * p.up.nsplit * p.up.ntiles * kFlatCoef;
  return p;
}

// `scratch` holds part_doubles + lv_doubles + up_doubles.
hipError_t launch_flat_pairs(const FlatArgs& A, const FlatPlan& plan, double* scratch,
                             hipStream_t st) {
  FlatLevel lv = plan.lv, up = plan.up, none = plan.up;
  none.series = 0;
  lv.coef = scratch + plan.part_doubles;
  up.coef = lv.coef + plan.lv_doubles;
  auto grid = [](int64_t n) {
    return dim3((unsigned)std::min(n, kGridX), (unsigned)((n + kGridX - 1) / kGridX));
  };
  auto blocks = [&](const FlatLevel& v) { return grid((v.ntiles * v.nsplit + 3) / 4); };
  if (up.series) k_flat_far<<<blocks(up), dim3(256), 0, st>>>(A, up, none);
  if (lv.series) k_flat_far<<<blocks(lv), dim3(256), 0, st>>>(A, lv, up);
  k_flat_near<<<blocks(lv), dim3(256), 0, st>>>(A, lv, scratch);
  if (!lv.series && lv.nsplit == 1) return hipGetLastError();   // the map is the near sums
  if (lv.ntiles < 256)
    k_flat_combine<16, 4><<<grid(16 * lv.ntiles), dim3(256), 0, st>>>(A, lv, up, scratch);
  else
    k_flat_combine<1, 1><<<grid(lv.ntiles), dim3(256), 0, st>>>(A, lv, up, scratch);
  return hipGetLastError();
}

}  // namespace csmap
