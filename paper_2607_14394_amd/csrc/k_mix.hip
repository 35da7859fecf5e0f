// Mode-wise channel mix and its gradients (Sec. V-A Eq. partitioned_conv,
// Sec. V-C), on a flattened mode range [m0, m1):
//
//   mix      yhat[b,o,m] = sum_i xhat[b,i,m] w[m-m0,i,o]
//   mix_h    g_x[b,i,m]  = sum_o g_y[b,o,m] conj(w[m-m0,i,o])     (data gradient)
//   wgrad    g_w[m-m0,i,o] (+)= sum_b conj(xhat[b,i,m]) g_y[b,o,m]
//
// Row groups of lanes below; the column forms further down take C_out up to 64
// (mix) or 63 (mix_h, wgrad) except at 16, and mostly 32, columns and other widths
// and mode counts where the row groups measured faster (row_groups, row_groups_h,
// few_blocks, launch_mix, and `lines` in launch_wgrad), and where
// their LDS does not fit.
//
// With B <= 2 the arithmetic intensity is about 1-2 flop/byte, so all three
// are bound by HBM traffic on w / g_w (M C_in C_out complex values).
//
// Layout of the work: a "row group" of LPR lanes (the power of two >= C_out,
// at most 64) covers one row (m, i, 0..C_out) of w / g_w, lane l holding the
// columns o = l + LPR s (s < OPL), so every row is read or written with
// contiguous 8-byte accesses.  A 256-thread workgroup has 256 / LPR groups and
// handles that many consecutive modes at a time ("mode block"), one per
// group.  The spectra of a block (stride M between channels in HBM) are
// staged through LDS as [b][channel][mode + 1], which turns their strided
// reads into coalesced ones and gives each group its per-mode vectors.
//
// mix and mix_h (bound by the reads of w): one workgroup per mode block in
// an XCD-aware order; the first rows of w are loaded into registers before
// the staging barrier, so their HBM latency overlaps the staging.
// wgrad (bound by the writes of g_w): a grid of resident workgroups, each
// walking a contiguous run of mode blocks (its reads of the spectra advance
// through the same DRAM rows), fetching the next block's spectra into
// registers while the current block's rows are written, with the LDS area
// double-buffered so that one barrier per block separates writers and
// readers.
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "dtst_internal.h"

namespace dtst {
namespace {

struct MixArgs {
  int64_t M, m0, count;  // count = m1 - m0
  int64_t nblk;           // number of mode blocks
  int B, ci, co;
  int lpr, mpb;           // lanes per row group, modes per block (= 256 / lpr)
  int acc;
};

typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Spectrum entries of one batch chunk processed together.
constexpr int BCH = 2;

// w rows held in registers per chunk (times OPL columns per lane).
template <int OPL>
struct Rows {
  static constexpr int value = OPL >= 8 ? 2 : 16 / OPL;
};

// Spectra of a block's modes in LDS: entry (b, c, mm) at
// [(b * C + c) * (MPB + 1) + mm].  They are read from spec[b][c][mbase + mm]
// (channel stride M), MPB consecutive modes per (b, c) row; each thread
// fetches its PRE entries into registers one block ahead and writes them to
// LDS when that block starts (entries beyond 256 * PRE are copied directly).
constexpr int PRE = 4;

template <int MPB>
__device__ __forceinline__ int sidx(int bc, int mm) {
  return bc * (MPB + 1) + mm;
}

// Direct staging of a block's spectra (no register prefetch).
template <int MPB>
__device__ __forceinline__ void stage(float2* dst, const float2* __restrict__ spec, int BC, int64_t M,
                                      int64_t mbase, int nm) {
  for (int e = threadIdx.x; e < BC * MPB; e += 256) {
    const int mm = e % MPB, bc = e / MPB;
    if (mm < nm) dst[sidx<MPB>(bc, mm)] = spec[int64_t(bc) * M + mbase + mm];
  }
}

template <int MPB>
__device__ __forceinline__ void fetch(float2 (&pre)[PRE], const float2* __restrict__ spec, int BC, int64_t M,
                                      int64_t mbase, int nm) {
#pragma unroll
  for (int j = 0; j < PRE; ++j) {
    const int e = threadIdx.x + 256 * j;
    const int mm = e % MPB, bc = e / MPB;
    const bool ok = bc < BC && mm < nm;
    pre[j] = spec[ok ? int64_t(bc) * M + mbase + mm : 0];
  }
}

template <int MPB>
__device__ __forceinline__ void put(float2* dst, const float2 (&pre)[PRE], const float2* __restrict__ spec, int BC,
                                    int64_t M, int64_t mbase, int nm) {
#pragma unroll
  for (int j = 0; j < PRE; ++j) {
    const int e = threadIdx.x + 256 * j;
    const int mm = e % MPB, bc = e / MPB;
    if (bc < BC && mm < nm) dst[sidx<MPB>(bc, mm)] = pre[j];
  }
  for (int e = threadIdx.x + 256 * PRE; e < BC * MPB; e += 256) {
    const int mm = e % MPB, bc = e / MPB;
    if (mm < nm) dst[sidx<MPB>(bc, mm)] = spec[int64_t(bc) * M + mbase + mm];
  }
}

template <int MPB>
__device__ __forceinline__ void unstage(float2* __restrict__ spec, const float2* src, int BC, int64_t M,
                                        int64_t mbase, int nm) {
  for (int e = threadIdx.x; e < BC * MPB; e += 256) {
    const int mm = e % MPB, bc = e / MPB;
    if (mm < nm) spec[int64_t(bc) * M + mbase + mm] = src[sidx<MPB>(bc, mm)];
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Give each XCD a contiguous run of mode blocks, so that neighbouring
// blocks -- which read the two halves of the same 128-byte lines of the
// spectra -- share an L2 and each line is fetched from HBM once.
__device__ __forceinline__ int64_t first_block() {
  const int64_t grid = gridDim.x, bid = blockIdx.x;
  const int64_t per = grid / 8;
  if (bid >= per * 8) return bid;
  return (bid % 8) * per + bid / 8;
}

// The contiguous run of mode blocks [*k0, *k1) of this workgroup.
__device__ __forceinline__ void span(int64_t nblk, int64_t* k0, int64_t* k1) {
  *k0 = nblk * blockIdx.x / gridDim.x;
  *k1 = nblk * (blockIdx.x + 1) / gridDim.x;
}

// Loads rows i0 .. i0 + R - 1 of the (ci x co) matrix at `base` into v;
// rows or columns outside the matrix (and inactive groups) read its first
// element and are never used.
template <int OPL, int R>
__device__ __forceinline__ void load_rows(float2 (&v)[R][OPL], const float2* __restrict__ base, int i0, int ci,
                                          int co, int lr, int lpr, bool active) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int s = 0; s < OPL; ++s) {
      const int i = i0 + r, o = lr + lpr * s;
      const bool ok = active && i < ci && o < co;
      v[r][s] = base[ok ? int64_t(i) * co + o : 0];
    }
}

// Sum of v over each aligned group of LPR lanes (a power of two <= 64),
// with DPP steps: pairs and quads (quad_perm), 8 and 16 lanes (row half
// mirror, row mirror), then 32 and 64 lanes by broadcasting the last lane of
// a row into the next row(s).  The full sum is valid in the group's last
// lane (lanes >= 16 of a 32-lane group, >= 48 of a 64-lane group; every lane
// for groups up to 16).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  if (LPR > 1) v += dpp<0xB1, 0xf>(v);   // quad_perm [1, 0, 3, 2]
  if (LPR > 2) v += dpp<0x4E, 0xf>(v);   // quad_perm [2, 3, 0, 1]
  if (LPR > 4) v += dpp<0x141, 0xf>(v);  // row_half_mirror
  if (LPR > 8) v += dpp<0x140, 0xf>(v);  // row_mirror
  if (LPR > 16) v += dpp<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
  if (LPR > 32) v += dpp<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__device__ __forceinline__ float2 cjmul(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

// mix and mix_h: one mode block per workgroup (the grid covers every
// block), in the XCD-aware order above.
template <int LPR, int OPL>
__global__ void __launch_bounds__(256)
mix_kernel(const float2* __restrict__ x, const float2* __restrict__ w, float2* __restrict__ y, MixArgs a) {
  constexpr int R = Rows<OPL>::value;
  constexpr int MPB = 256 / LPR;
  extern __shared__ float2 sm[];
  float2* sx = sm;                                // B * ci rows
  float2* sy = sm + a.B * a.ci * (MPB + 1);       // B * co rows
  const int lr = threadIdx.x % LPR, mm = threadIdx.x / LPR;
  for (int64_t k = first_block(); k < a.nblk; k += gridDim.x) {
    const int64_t lm0 = k * MPB;  // local mode index in [0, count)
    const int nm = static_cast<int>(min(int64_t(MPB), a.count - lm0));
    const int64_t mbase = a.m0 + lm0;
    const bool active = mm < nm;
    const float2* wm = w + (lm0 + (active ? mm : 0)) * int64_t(a.ci) * a.co;
    float2 wv[R][OPL];
    load_rows<OPL, R>(wv, wm, 0, a.ci, a.co, lr, LPR, active);
    stage<MPB>(sx, x, a.B * a.ci, a.M, mbase, nm);
    __syncthreads();
    for (int i0 = 0; i0 < a.ci; i0 += R) {
      if (i0 > 0) load_rows<OPL, R>(wv, wm, i0, a.ci, a.co, lr, LPR, active);
      for (int b0 = 0; b0 < a.B; b0 += BCH) {
        float2 acc[BCH][OPL];
#pragma unroll
        for (int q = 0; q < BCH; ++q)
#pragma unroll
          for (int s = 0; s < OPL; ++s) acc[q][s] = make_float2(0.f, 0.f);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (i0 + r >= a.ci) continue;
#pragma unroll
          for (int q = 0; q < BCH; ++q) {
            if (b0 + q >= a.B) continue;
            const float2 xv = sx[sidx<MPB>((b0 + q) * a.ci + i0 + r, mm)];
#pragma unroll
            for (int s = 0; s < OPL; ++s) {
              const float2 p = cmul(xv, wv[r][s]);
              acc[q][s].x += p.x;
              acc[q][s].y += p.y;
            }
          }
        }
        if (active) {
#pragma unroll
          for (int q = 0; q < BCH; ++q) {
            if (b0 + q >= a.B) continue;
#pragma unroll
            for (int s = 0; s < OPL; ++s) {
              const int o = lr + LPR * s;
              if (o >= a.co) continue;
              float2* d = sy + sidx<MPB>((b0 + q) * a.co + o, mm);
              if (i0 > 0) {
                acc[q][s].x += d->x;
                acc[q][s].y += d->y;
              }
              *d = acc[q][s];
            }
          }
        }
      }
    }
    __syncthreads();
    unstage<MPB>(y, sy, a.B * a.co, a.M, mbase, nm);
    __syncthreads();
  }
}

// Data gradient: each row (m, i) of w gives g_x[b, i, m] for every b as a
// sum over the row's C_out columns, reduced across the row group's lanes.
template <int LPR, int OPL>
__global__ void __launch_bounds__(256)
mix_h_kernel(const float2* __restrict__ gy, const float2* __restrict__ w, float2* __restrict__ gx, MixArgs a) {
  constexpr int R = Rows<OPL>::value;
  constexpr int MPB = 256 / LPR;
  extern __shared__ float2 sm[];
  float2* sg = sm;                                // B * co rows
  float2* sx = sm + a.B * a.co * (MPB + 1);       // B * ci rows
  const int lr = threadIdx.x % LPR, mm = threadIdx.x / LPR;
  for (int64_t k = first_block(); k < a.nblk; k += gridDim.x) {
    const int64_t lm0 = k * MPB;
    const int nm = static_cast<int>(min(int64_t(MPB), a.count - lm0));
    const int64_t mbase = a.m0 + lm0;
    const bool active = mm < nm;
    const float2* wm = w + (lm0 + (active ? mm : 0)) * int64_t(a.ci) * a.co;
    float2 wv[R][OPL];
    load_rows<OPL, R>(wv, wm, 0, a.ci, a.co, lr, LPR, active);
    stage<MPB>(sg, gy, a.B * a.co, a.M, mbase, nm);
    __syncthreads();
    for (int i0 = 0; i0 < a.ci; i0 += R) {
      if (i0 > 0) load_rows<OPL, R>(wv, wm, i0, a.ci, a.co, lr, LPR, active);
      for (int b0 = 0; b0 < a.B; b0 += BCH) {
        // this lane's columns of g_y for the batch chunk
        float2 gv[BCH][OPL];
#pragma unroll
        for (int q = 0; q < BCH; ++q)
#pragma unroll
          for (int s = 0; s < OPL; ++s) {
            const int o = lr + LPR * s;
            gv[q][s] = (b0 + q < a.B && o < a.co && active) ? sg[sidx<MPB>((b0 + q) * a.co + o, mm)]
                                                             : make_float2(0.f, 0.f);
          }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (i0 + r >= a.ci) continue;
#pragma unroll
          for (int q = 0; q < BCH; ++q) {
            if (b0 + q >= a.B) continue;
            float2 t = make_float2(0.f, 0.f);
#pragma unroll
            for (int s = 0; s < OPL; ++s) {
              const float2 p = cjmul(wv[r][s], gv[q][s]);
              t.x += p.x;
              t.y += p.y;
            }
            t.x = group_sum<LPR>(t.x);
            t.y = group_sum<LPR>(t.y);
            if (lr == LPR - 1 && active) sx[sidx<MPB>((b0 + q) * a.ci + i0 + r, mm)] = t;
          }
        }
      }
    }
    __syncthreads();
    unstage<MPB>(gx, sx, a.B * a.ci, a.M, mbase, nm);
    __syncthreads();
  }
}

// Weight gradient: a grid of resident workgroups, each walking its run of
// mode blocks.  Per block its spectra go from registers to one half of a
// double-buffered LDS area, the next block's are fetched, one barrier; then
// each lane forms its columns of a chunk of rows (m, i) in registers -- its
// g_y values of the batch chunk held in registers, x broadcast from LDS --
// and streams the rows out with non-temporal stores (g_w is written once and
// not read back here, except for the accumulate read-modify-write).  With
// almost no reads to overlap, this keeps the stores flowing while the next
// block's spectra arrive.  W = 2: every lane holds the column pairs
// o = 2 (lr + LPR s) + {0, 1} and writes them with one 16-byte store (half
// the store instructions of W = 1 for the same bytes; needs an even C_out
// and a 16-byte aligned g_w).
template <int LPR, int OPL, int W, int ACC>
__global__ void __launch_bounds__(256)
wgrad_kernel(const float2* __restrict__ x, const float2* __restrict__ gy, float2* __restrict__ gw, MixArgs a) {
  constexpr int R = Rows<OPL>::value;
  constexpr int MPB = 256 / LPR;
  extern __shared__ float2 sm[];
  const int nx = a.B * a.ci * (MPB + 1), ng = a.B * a.co * (MPB + 1);
  const int lr = threadIdx.x % LPR, mm = threadIdx.x / LPR;
  auto col = [&](int s, int w) { return W * (lr + LPR * s) + w; };
  int64_t k0, k1;
  span(a.nblk, &k0, &k1);
  float2 prex[PRE], preg[PRE];
  if (k0 < k1) {
    const int nm0 = int(min(int64_t(MPB), a.count - k0 * MPB));
    fetch<MPB>(prex, x, a.B * a.ci, a.M, a.m0 + k0 * MPB, nm0);
    fetch<MPB>(preg, gy, a.B * a.co, a.M, a.m0 + k0 * MPB, nm0);
  }
  for (int64_t k = k0; k < k1; ++k) {
    float2* sx = sm + ((k - k0) & 1) * (nx + ng);  // B * ci rows
    float2* sg = sx + nx;                          // B * co rows
    const int64_t lm0 = k * MPB;
    const int nm = static_cast<int>(min(int64_t(MPB), a.count - lm0));
    const int64_t mbase = a.m0 + lm0;
    const bool active = mm < nm;
    float2* gm = gw + (lm0 + (active ? mm : 0)) * int64_t(a.ci) * a.co;
    // rows i0 .. i0 + R - 1 of this mode's (ci x co) block of g_w (the
    // accumulate read; rows or columns outside read its first element and
    // are never used)
    auto load_acc = [&](float2 (&v)[R][OPL][W], int i0) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < OPL; ++s) {
          const int i = i0 + r, o = col(s, 0);
          const bool ok = active && i < a.ci && o < a.co;
          const float2* src = gm + (ok ? int64_t(i) * a.co + o : 0);
          if (W == 2) {
            const float4 t = *reinterpret_cast<const float4*>(src);
            v[r][s][0] = make_float2(t.x, t.y);
            v[r][s][W - 1] = make_float2(t.z, t.w);
          } else {
            v[r][s][0] = *src;
          }
        }
    };
    float2 acc[R][OPL][W];
    if constexpr (ACC) load_acc(acc, 0);
    put<MPB>(sx, prex, x, a.B * a.ci, a.M, mbase, nm);
    put<MPB>(sg, preg, gy, a.B * a.co, a.M, mbase, nm);
    if (k + 1 < k1) {
      const int nm1 = int(min(int64_t(MPB), a.count - lm0 - MPB));
      fetch<MPB>(prex, x, a.B * a.ci, a.M, mbase + MPB, nm1);
      fetch<MPB>(preg, gy, a.B * a.co, a.M, mbase + MPB, nm1);
    }
    __syncthreads();
    if (!active) continue;
    for (int i0 = 0; i0 < a.ci; i0 += R) {
      if constexpr (ACC) {
        if (i0 > 0) load_acc(acc, i0);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int s = 0; s < OPL; ++s)
#pragma unroll
            for (int w = 0; w < W; ++w) acc[r][s][w] = make_float2(0.f, 0.f);
      }
      for (int b0 = 0; b0 < a.B; b0 += BCH) {
        float2 gv[BCH][OPL][W];
#pragma unroll
        for (int q = 0; q < BCH; ++q)
#pragma unroll
          for (int s = 0; s < OPL; ++s)
#pragma unroll
            for (int w = 0; w < W; ++w) {
              const int o = col(s, w);
              gv[q][s][w] =
                  (b0 + q < a.B && o < a.co) ? sg[sidx<MPB>((b0 + q) * a.co + o, mm)] : make_float2(0.f, 0.f);
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (i0 + r >= a.ci) continue;
#pragma unroll
          for (int q = 0; q < BCH; ++q) {
            if (b0 + q >= a.B) continue;
            const float2 xv = sx[sidx<MPB>((b0 + q) * a.ci + i0 + r, mm)];
#pragma unroll
            for (int s = 0; s < OPL; ++s)
#pragma unroll
              for (int w = 0; w < W; ++w) {
                const float2 p = cjmul(xv, gv[q][s][w]);
                acc[r][s][w].x += p.x;
                acc[r][s][w].y += p.y;
              }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = i0 + r;
        if (i >= a.ci) continue;
#pragma unroll
        for (int s = 0; s < OPL; ++s) {
          const int o = col(s, 0);
          if (o >= a.co) continue;
          if (W == 2)
            __builtin_nontemporal_store(v4f{acc[r][s][0].x, acc[r][s][0].y, acc[r][s][W - 1].x, acc[r][s][W - 1].y},
                                        reinterpret_cast<v4f*>(gm + int64_t(i) * a.co + o));
          else
            __builtin_nontemporal_store(v2f{acc[r][s][0].x, acc[r][s][0].y},
                                        reinterpret_cast<v2f*>(gm + int64_t(i) * a.co + o));
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// C_out up to 64: W columns a lane (2, one 16-byte access, for an even C_out and
// 16-byte aligned w / g_w; else 1).  mix and mix_h give every wave MPW = 64 / CP
// consecutive modes, CP = C_out / W lanes a mode: with row groups of a power of
// two lanes 12 of 32 lanes idled at C = 20 (the paper's width), and 8-byte loads
// kept half as many bytes in flight.  wgrad writes g_w as the flat array it is,
// 1 KiB a store instruction: rows of 160 bytes (C = 20) end inside 128-byte
// lines, and a wave writing several of them left lines in parts.
// 65536 modes, 20 -> 20 channels (210 MB of weights), B = 1, before and now:
// mix 56.6 -> 46.6 us, mix_h 61.6 -> 44.4, wgrad 81.1 -> 39.9 (5.25 TB/s).
// ---------------------------------------------------------------------------
struct PairArgs {
  int64_t M, m0, count, nblk;
  int B, ci, co;
  int cp, mpw, mpb;  // lanes per mode; modes per wave and per workgroup (4 waves)
};

// Rows [i0, i0 + R) of one mode's matrix, this lane's columns (rows past the
// end and idle lanes read the first entry and are never used).
template <int R, int W>
__device__ __forceinline__ void load_cols(float2 (&v)[R][W], const float2* __restrict__ wm, int i0, int ci, int co,
                                          int p, bool active) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = i0 + r;
    const float2* src = wm + (active && i < ci ? i * co + W * p : 0);
    if constexpr (W == 2) {
      const float4 t = *reinterpret_cast<const float4*>(src);
      v[r][0] = make_float2(t.x, t.y);
      v[r][1] = make_float2(t.z, t.w);
    } else {
      v[r][0] = *src;
    }
  }
}

__device__ __forceinline__ void stage_n(float2* dst, const float2* __restrict__ spec, int BC, int64_t M,
                                        int64_t mbase, int mpb, int nm) {
  const int per = 256 / mpb, mm = threadIdx.x % mpb, c0 = threadIdx.x / mpb;
  if (c0 >= per || mm >= nm) return;
  for (int bc = c0; bc < BC; bc += per) dst[bc * (mpb + 1) + mm] = spec[int64_t(bc) * M + mbase + mm];
}
__device__ __forceinline__ void unstage_n(float2* __restrict__ spec, const float2* src, int BC, int64_t M,
                                          int64_t mbase, int mpb, int nm) {
  const int per = 256 / mpb, mm = threadIdx.x % mpb, c0 = threadIdx.x / mpb;
  if (c0 >= per || mm >= nm) return;
  for (int bc = c0; bc < BC; bc += per) spec[int64_t(bc) * M + mbase + mm] = src[bc * (mpb + 1) + mm];
}

template <int R, int W>
__global__ void __launch_bounds__(256)
mix_cols_kernel(const float2* __restrict__ x, const float2* __restrict__ w, float2* __restrict__ y, PairArgs a) {
  extern __shared__ float2 sm[];
  const int st = a.mpb + 1;
  float2* sx = sm;                    // B * ci rows
  float2* sy = sm + a.B * a.ci * st;  // B * co rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ml = lane / a.cp, p = lane - ml * a.cp, mm = wave * a.mpw + ml;
  for (int64_t k = first_block(); k < a.nblk; k += gridDim.x) {
    const int64_t lm0 = k * a.mpb;
    const int nm = static_cast<int>(min(int64_t(a.mpb), a.count - lm0));
    const bool active = ml < a.mpw && mm < nm;
    const float2* wm = w + (lm0 + (active ? mm : 0)) * int64_t(a.ci) * a.co;
    float2 wv[R][W];
    load_cols<R, W>(wv, wm, 0, a.ci, a.co, p, active);
    stage_n(sx, x, a.B * a.ci, a.M, a.m0 + lm0, a.mpb, nm);
    __syncthreads();
    for (int i0 = 0; i0 < a.ci; i0 += R) {
      if (i0 > 0) load_cols<R, W>(wv, wm, i0, a.ci, a.co, p, active);
      if (!active) continue;
      for (int b = 0; b < a.B; ++b) {
        float2 acc[W];
#pragma unroll
        for (int c = 0; c < W; ++c) acc[c] = make_float2(0.f, 0.f);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (i0 + r >= a.ci) continue;
          const float2 xv = sx[(b * a.ci + i0 + r) * st + mm];
#pragma unroll
          for (int c = 0; c < W; ++c) {
            const float2 t = cmul(xv, wv[r][c]);
            acc[c].x += t.x;
            acc[c].y += t.y;
          }
        }
        float2* d = sy + (b * a.co + W * p) * st + mm;
#pragma unroll
        for (int c = 0; c < W; ++c) {
          if (i0 > 0) {
            acc[c].x += d[c * st].x;
            acc[c].y += d[c * st].y;
          }
          d[c * st] = acc[c];
        }
      }
    }
    __syncthreads();
    unstage_n(y, sy, a.B * a.co, a.M, a.m0 + lm0, a.mpb, nm);
    __syncthreads();
  }
}

// Orders a wave's LDS accesses before this point with those of its other lanes
// after it (no instruction on this hardware: a wave's LDS accesses stay in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Data gradient: the products of a row over a mode's CP lanes are summed
// through a wave's own LDS area (no workgroup barrier), R rows at a time.
template <int R, int W>
__global__ void __launch_bounds__(256)
mix_h_cols_kernel(const float2* __restrict__ gy, const float2* __restrict__ w, float2* __restrict__ gx, PairArgs a) {
  extern __shared__ float2 sm[];
  const int st = a.mpb + 1;
  float2* sg = sm;                    // B * co rows
  float2* sx = sm + a.B * a.co * st;  // B * ci rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float2* red = sx + a.B * a.ci * st + wave * R * 65;  // R rows of 64 lanes
  const int ml = lane / a.cp, p = lane - ml * a.cp, mm = wave * a.mpw + ml;
  for (int64_t k = first_block(); k < a.nblk; k += gridDim.x) {
    const int64_t lm0 = k * a.mpb;
    const int nm = static_cast<int>(min(int64_t(a.mpb), a.count - lm0));
    const bool active = ml < a.mpw && mm < nm;
    const float2* wm = w + (lm0 + (active ? mm : 0)) * int64_t(a.ci) * a.co;
    float2 wv[R][W];
    load_cols<R, W>(wv, wm, 0, a.ci, a.co, p, active);
    stage_n(sg, gy, a.B * a.co, a.M, a.m0 + lm0, a.mpb, nm);
    __syncthreads();
    for (int i0 = 0; i0 < a.ci; i0 += R) {
      if (i0 > 0) load_cols<R, W>(wv, wm, i0, a.ci, a.co, p, active);
      const int nr = min(R, a.ci - i0);
      for (int b = 0; b < a.B; ++b) {
        float2 gv[W];
#pragma unroll
        for (int c = 0; c < W; ++c)
          gv[c] = active ? sg[(b * a.co + W * p + c) * st + mm] : make_float2(0.f, 0.f);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float2 t = cjmul(wv[r][0], gv[0]);
          if constexpr (W == 2) {
            const float2 t1 = cjmul(wv[r][1], gv[1]);
            t.x += t1.x;
            t.y += t1.y;
          }
          red[r * 65 + lane] = t;
        }
        wave_sync();
        // sums of (mode, row): lane e of each pass
        for (int e = lane; e < a.mpw * nr; e += 64) {
          const int r = e / a.mpw, me = e - r * a.mpw, q = wave * a.mpw + me;
          float2 t = make_float2(0.f, 0.f);
          const float2* src = red + r * 65 + me * a.cp;
          for (int c = 0; c < a.cp; ++c) {
            const float2 v = src[c];
            t.x += v.x;
            t.y += v.y;
          }
          if (q < nm) sx[(b * a.ci + i0 + r) * st + q] = t;
        }
        wave_sync();
      }
    }
    __syncthreads();
    unstage_n(gx, sx, a.B * a.ci, a.M, a.m0 + lm0, a.mpb, nm);
    __syncthreads();
  }
}

// Weight gradient: the block's g_w is one run of W-column elements; thread f of
// a pass forms columns W p .. of row i of mode mm, f = (mm ci + i) CP + p, from
// the spectra in LDS ([mode][b][channel]).
template <int ACC, int W>
__global__ void __launch_bounds__(256)
wgrad_flat_kernel(const float2* __restrict__ x, const float2* __restrict__ gy, float2* __restrict__ gw, PairArgs a) {
  extern __shared__ float4 sm4[];
  const int sgx = a.B * a.ci + 1, sgy = (a.B * a.co + 3) / 2 * 2;  // mode strides (pairs stay 16-byte aligned)
  float2* sg = reinterpret_cast<float2*>(sm4);
  float2* sx = sg + a.mpb * sgy;
  const int rows = a.ci * a.cp;  // elements of one mode
  for (int64_t k = first_block(); k < a.nblk; k += gridDim.x) {
    const int64_t lm0 = k * a.mpb;
    const int nm = static_cast<int>(min(int64_t(a.mpb), a.count - lm0));
    const int64_t mbase = a.m0 + lm0;
    {
      const int per = 256 / a.mpb, mm = threadIdx.x % a.mpb, c0 = threadIdx.x / a.mpb;
      if (c0 < per && mm < nm) {
        for (int c = c0; c < a.B * a.ci; c += per) sx[mm * sgx + c] = x[int64_t(c) * a.M + mbase + mm];
        for (int c = c0; c < a.B * a.co; c += per) sg[mm * sgy + c] = gy[int64_t(c) * a.M + mbase + mm];
      }
    }
    __syncthreads();
    float2* out = gw + lm0 * int64_t(a.ci) * a.co;
    const int n = nm * rows;
    const int d_row = 256 / a.cp, d_p = 256 - d_row * a.cp;  // a pass further on
    int row = threadIdx.x / a.cp, p = threadIdx.x - row * a.cp;
    int mm = row / a.ci, i = row - mm * a.ci;
    const int d_mm = d_row / a.ci, d_i = d_row - d_mm * a.ci;
    for (int f = threadIdx.x; f < n; f += 256) {
      float2 acc[W];
      if constexpr (ACC && W == 2) {
        const float4 t = *reinterpret_cast<const float4*>(out + W * f);
        acc[0] = make_float2(t.x, t.y);
        acc[W - 1] = make_float2(t.z, t.w);
      } else {
#pragma unroll
        for (int c = 0; c < W; ++c) acc[c] = ACC ? out[W * f + c] : make_float2(0.f, 0.f);
      }
      for (int b = 0; b < a.B; ++b) {
        const float2 xv = sx[mm * sgx + b * a.ci + i];
#pragma unroll
        for (int c = 0; c < W; ++c) {
          const float2 t = cjmul(xv, sg[mm * sgy + b * a.co + W * p + c]);
          acc[c].x += t.x;
          acc[c].y += t.y;
        }
      }
      if constexpr (W == 2)
        __builtin_nontemporal_store(v4f{acc[0].x, acc[0].y, acc[1].x, acc[1].y}, reinterpret_cast<v4f*>(out + W * f));
      else
        __builtin_nontemporal_store(v2f{acc[0].x, acc[0].y}, reinterpret_cast<v2f*>(out + f));
      // element f + 256
      p += d_p;
      i += d_i;
      mm += d_mm;
      if (p >= a.cp) {
        p -= a.cp;
        ++i;
      }
      if (i >= a.ci) {
        i -= a.ci;
        ++mm;
      }
    }
    __syncthreads();
  }
}

int lanes_per_row(int64_t co) {
  int l = 1;
  while (l < co && l < 64) l <<= 1;
  return l;
}

int opl_of(int64_t co) {
  const int64_t o = (co + 63) / 64;
  return o <= 1 ? 1 : (o <= 2 ? 2 : (o <= 4 ? 4 : 8));
}

// cols: the columns one lane group spans per row slot (C_out, or C_out / 2
// for wgrad's column pairs).
MixArgs make_args(int64_t B, int64_t ci, int64_t co, int64_t M, int64_t m0, int64_t m1, int acc,
                  int64_t cols = 0) {
  MixArgs a;
  a.M = M;
  a.m0 = m0;
  a.count = m1 - m0;
  a.B = static_cast<int>(B);
  a.ci = static_cast<int>(ci);
  a.co = static_cast<int>(co);
  a.lpr = lanes_per_row(cols > 0 ? cols : co);
  a.mpb = 256 / a.lpr;
  a.acc = acc;
  a.nblk = (a.count + a.mpb - 1) / a.mpb;
  return a;
}

typedef void (*mix_fn)(const float2*, const float2*, float2*, MixArgs);

// Workgroups of kernel f with `lds` bytes of LDS the current device holds at
// once (cached per kernel, LDS size and device).
int64_t resident_workgroups(mix_fn f, size_t lds) {
  struct Entry {
    mix_fn f;
    size_t lds;
    int dev;
    int64_t n;
  };
  static std::mutex mu;
  static std::vector<Entry> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    for (const Entry& e : cache)
      if (e.f == f && e.lds == lds && e.dev == dev) return e.n;
  }
  int cus = 0, per_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, 256, lds) != hipSuccess) return 0;
  const int64_t n = int64_t(cus) * (per_cu > 0 ? per_cu : 1);
  std::lock_guard<std::mutex> lock(mu);
  cache.push_back(Entry{f, lds, dev, n});
  return n;
}

// LDS of one mode block's spectra (mode blocks of 256 / lanes_per_row(cols)
// modes; cols = C_out unless given).
size_t block_lds(int64_t B, int64_t ci, int64_t co, int64_t cols = 0) {
  const size_t mpb = size_t(256 / lanes_per_row(cols > 0 ? cols : co));
  return sizeof(float2) * size_t(B) * size_t(ci + co) * (mpb + 1);
}

// persistent: a grid of resident workgroups walking runs of blocks (wgrad);
// else one workgroup per block (capped at 2^22, the kernels loop beyond).
int launch(mix_fn f, size_t lds, bool persistent, const float2* p0, const float2* p1, float2* p2, const MixArgs& a,
           void* stream) {
  if (lds > 65536) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  int64_t cap = int64_t(1) << 22;
  if (persistent) {
    cap = resident_workgroups(f, lds);
    if (cap <= 0) return hipErrorInvalidConfiguration;
  }
  const int64_t blocks = a.nblk < cap ? a.nblk : cap;
  hipLaunchKernelGGL(f, dim3(static_cast<unsigned>(blocks)), dim3(256), lds, static_cast<hipStream_t>(stream), p0,
                     p1, p2, a);
  return hipGetLastError();
}

}  // namespace

// LDS a mix workgroup needs: wgrad's double-buffered spectra of one mode
// block (mix and mix_h use half of it; wgrad's column-pair form, taken only
// where it fits, twice as many modes).
size_t mix_lds_bytes(int64_t B, int64_t ci, int64_t co) { return 2 * block_lds(B, ci, co); }

namespace {

// Kernel instance for C_out: LPR lanes per row and OPL columns per lane.
template <template <int, int> class K>
mix_fn pick(int64_t co) {
  switch (lanes_per_row(co)) {
    case 1: return K<1, 1>::fn;
    case 2: return K<2, 1>::fn;
    case 4: return K<4, 1>::fn;
    case 8: return K<8, 1>::fn;
    case 16: return K<16, 1>::fn;
    case 32: return K<32, 1>::fn;
    default: break;
  }
  const int opl = opl_of(co);
  return opl == 1 ? K<64, 1>::fn : opl == 2 ? K<64, 2>::fn : opl == 4 ? K<64, 4>::fn : K<64, 8>::fn;
}
template <int L, int O>
struct MixK {
  static constexpr mix_fn fn = mix_kernel<L, O>;
};
template <int L, int O>
struct MixHK {
  static constexpr mix_fn fn = mix_h_kernel<L, O>;
};
// (accumulating and overwriting instances apart: the accumulate read and its
// conditions are not compiled into the overwriting kernel)
template <int L, int O>
struct WgradK {
  static constexpr mix_fn fn = wgrad_kernel<L, O, 1, 0>;
};
template <int L, int O>
struct WgradK2 {
  static constexpr mix_fn fn = wgrad_kernel<L, O, 2, 0>;
};
template <int L, int O>
struct WgradKA {
  static constexpr mix_fn fn = wgrad_kernel<L, O, 1, 1>;
};
template <int L, int O>
struct WgradK2A {
  static constexpr mix_fn fn = wgrad_kernel<L, O, 2, 1>;
};

// ---- column forms (C_out <= 64) ----
int cols_of(int64_t co, const void* w) {
  return co % 2 == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0 ? 2 : 1;
}

PairArgs pair_args(int64_t B, int64_t ci, int64_t co, int64_t M, int64_t m0, int64_t m1, int cols, int mpb) {
  PairArgs a;
  a.M = M;
  a.m0 = m0;
  a.count = m1 - m0;
  a.B = static_cast<int>(B);
  a.ci = static_cast<int>(ci);
  a.co = static_cast<int>(co);
  a.cp = static_cast<int>(co / cols);
  a.mpw = 64 / a.cp;
  a.mpb = mpb > 0 ? mpb : 4 * a.mpw;
  a.nblk = (a.count + a.mpb - 1) / a.mpb;
  return a;
}

typedef void (*pair_fn)(const float2*, const float2*, float2*, PairArgs);

int launch_pair(pair_fn f, size_t lds, const void* p0, const void* p1, void* p2, const PairArgs& a, void* stream) {
  if (lds > 65536) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  const int64_t cap = int64_t(1) << 22;
  const int64_t blocks = a.nblk < cap ? a.nblk : cap;
  hipLaunchKernelGGL(f, dim3(static_cast<unsigned>(blocks)), dim3(256), lds, static_cast<hipStream_t>(stream),
                     static_cast<const float2*>(p0), static_cast<const float2*>(p1), static_cast<float2*>(p2), a);
  return hipGetLastError();
}

// mix and mix_h by row groups of a power of two lanes: rows that fill their
// groups and are whole 128-byte lines, 16 columns (262144 modes of 16 -> 16, B =
// 2: mix 127 us and 137 by columns, mix_h 128 and 151) and 32 columns of weights
// under 1 GB (32768 modes, B = 1: 53 and 57; above, 262144 modes, B = 2: 471 and
// 448, 484 and 455).
bool row_groups(int64_t ci, int64_t co, int64_t modes) {
  return co == 16 || (co == 32 && modes * ci * co * 8 < (int64_t(1) << 30));
}

// mix_h over several batch entries by row groups too where a lane holds one
// column (an odd C_out): an element of w then costs two LDS accesses an entry,
// which the row groups' register sums do not, unless most of their lanes idle
// (65536 modes, B = 3: 13 -> 13 29.6 us and 42.9 by columns, 29 -> 29 121 and 170,
// 21 -> 21 80 and 76; 49152 modes, B = 3: 10 -> 29 35.7 and 52.5).
bool row_groups_h(int64_t B, int64_t ci, int64_t co) {
  return co % 2 != 0 && B > 1 && (B * ci >= 32 || co >= 25) && (co <= 7 || 10 * co >= 7 * lanes_per_row(co));
}

// Several batch entries and few modes: the column forms' blocks, of about twice
// the modes, leave CUs idle (2048 modes, B = 2, row groups and columns: 20 -> 20 mix
// 6.3 and 7.6 us, mix_h 8.0 and 9.1; 28 -> 28 mix_h 9.1 and 12.0; 7680 modes, B = 3:
// 14 -> 14 mix 6.5 and 8.1; with blocks enough columns are the faster, 8192 modes, B
// = 2, 20 -> 20 mix_h by row groups 1.3 times the columns' time).
bool few_blocks(int64_t B, int64_t blocks, int64_t least) { return B > 1 && blocks < least; }

// Rows of w in flight: as many as C_in, or the count that leaves the fewest
// unused ones; but 8 where the registers of 16 or 20 cost more waves than their
// loads hide: in mix for C_in of 13 to 20 (65536 modes of 20 -> 20: B = 1 38.1 and
// 34.8 us, B = 3 62.9 and 43.4; by row groups 40.1 and 61.3), in mix_h over
// several batch entries with two columns a lane, from 12 (B = 3: 80.1 and 55.7; at
// B = 1 34.9 and 35.4).
int rows_in_flight(int64_t ci, bool few) {
  if (few) return 8;
  if (ci <= 20) return static_cast<int>((ci + 3) / 4 * 4);
  int best = 16;
  for (int r : {20, 12})
    if ((ci + r - 1) / r * r < (ci + best - 1) / best * best) best = r;
  return best;
}
template <int W>
pair_fn pick_mix_cols(int r) {
  return r == 4 ? mix_cols_kernel<4, W> : r == 8 ? mix_cols_kernel<8, W> : r == 12 ? mix_cols_kernel<12, W>
       : r == 16 ? mix_cols_kernel<16, W> : mix_cols_kernel<20, W>;
}
template <int W>
pair_fn pick_mix_h_cols(int r) {
  return r == 4 ? mix_h_cols_kernel<4, W> : r == 8 ? mix_h_cols_kernel<8, W> : r == 12 ? mix_h_cols_kernel<12, W>
       : r == 16 ? mix_h_cols_kernel<16, W> : mix_h_cols_kernel<20, W>;
}

}  // namespace

int launch_mix(const void* xhat, const void* w, void* yhat, int64_t B, int64_t ci, int64_t co, int64_t M,
               int64_t m0, int64_t m1, void* stream) {
  if (B <= 0 || m1 <= m0) return hipSuccess;
  // (27 to 31 columns fill the row groups as well, which have twice the blocks: 28
  // -> 28, 7680 modes, B = 2: 11.4 us and 14.8 by columns; 32768, B = 1: 31.8 and
  // 32.8; 49152, B = 1: 60.5 and 57.9)
  if (co <= 64 && !row_groups(ci, co, m1 - m0) && !(co >= 27 && co < 32)) {
    const int cols = cols_of(co, w), r = rows_in_flight(ci, ci >= 13 && ci <= 20);
    const PairArgs a = pair_args(B, ci, co, M, m0, m1, cols, 0);
    const size_t lds = sizeof(float2) * size_t(B) * size_t(ci + co) * (a.mpb + 1);
    // (with up to four columns a block is up to 256 modes, whose input spectra then
    // fill the LDS: 65536 modes of 20 -> 3, B = 3: 26.9 us, by row groups 16.9)
    if (lds <= (co <= 4 && ci >= 12 ? 24 : 64) * 1024 && !few_blocks(B, a.nblk, 256))
      return launch_pair(cols == 2 ? pick_mix_cols<2>(r) : pick_mix_cols<1>(r), lds, xhat, w, yhat, a, stream);
  }
  const MixArgs a = make_args(B, ci, co, M, m0, m1, 0);
  return launch(pick<MixK>(co), block_lds(B, ci, co), false, static_cast<const float2*>(xhat),
                static_cast<const float2*>(w), static_cast<float2*>(yhat), a, stream);
}

int launch_mix_h(const void* gy, const void* w, void* gx, int64_t B, int64_t ci, int64_t co, int64_t M,
                 int64_t m0, int64_t m1, void* stream) {
  if (B <= 0 || m1 <= m0) return hipSuccess;
  // (a full wave per row, C_out = 64, sums it in registers faster: 32768 modes
  // of 12 -> 64, B = 3: 70 us below, 79 us through LDS; of 48 -> 48, B = 2: 165
  // below, 131 through LDS)
  if (co < 64 && !row_groups(ci, co, m1 - m0) && !row_groups_h(B, ci, co)) {
    const int cols = cols_of(co, w), r = rows_in_flight(ci, B > 1 && ci >= 13 && co % 2 == 0 && co >= 12);
    const PairArgs a = pair_args(B, ci, co, M, m0, m1, cols, 0);
    const size_t lds = sizeof(float2) * (size_t(B) * size_t(ci + co) * (a.mpb + 1) + size_t(4) * r * 65);
    if (lds <= 80 * 1024 && !few_blocks(B, a.nblk, 129))
      return launch_pair(cols == 2 ? pick_mix_h_cols<2>(r) : pick_mix_h_cols<1>(r), lds, gy, w, gx, a, stream);
  }
  const MixArgs a = make_args(B, ci, co, M, m0, m1, 0);
  return launch(pick<MixHK>(co), block_lds(B, ci, co), false, static_cast<const float2*>(gy),
                static_cast<const float2*>(w), static_cast<float2*>(gx), a, stream);
}

int launch_wgrad(const void* xhat, const void* gy, void* gw, int64_t B, int64_t ci, int64_t co, int64_t M,
                 int64_t m0, int64_t m1, int accumulate, void* stream) {
  if (B <= 0 || m1 <= m0) return hipSuccess;
  // Flat g_w, except where rows are whole 128-byte lines and the resident form
  // below is the faster one: 32 columns (262144 modes of 32 -> 32: 370 us there,
  // 389 flat); 16 columns of under 1 GB (within a backward step of a 64 x 32 x
  // 128 x 32 pencil 123 and 126; 4194304 modes alone: 1930 and 1767); and
  // accumulating 16 or more than 32 (65536 of 16 -> 16: 55 there, 67 flat; 32768
  // of 48 -> 48, B = 2: 263 and 275).
  const bool lines = co % 32 == 0 || (accumulate && (co == 16 || co > 32)) ||
                     (co == 16 && (m1 - m0) * ci * co * 8 < (int64_t(1) << 30));
  if (co < 64 && !lines) {
    const int cols = cols_of(co, gw);
    int mpb = 16;  // modes of a block: at least four passes of the workgroup
    while (mpb < 64 && mpb * ci * (co / cols) < 1024) mpb *= 2;
    const PairArgs a = pair_args(B, ci, co, M, m0, m1, cols, mpb);
    const size_t lds = sizeof(float2) * mpb * (size_t(B) * size_t(ci + co) + 4);
    if (lds <= 64 * 1024)
      return launch_pair(cols == 2 ? (accumulate ? wgrad_flat_kernel<1, 2> : wgrad_flat_kernel<0, 2>)
                                   : (accumulate ? wgrad_flat_kernel<1, 1> : wgrad_flat_kernel<0, 1>),
                         lds, xhat, gy, gw, a, stream);
  }
  // column pairs (16-byte stores) for an even C_out of at least 4 when g_w
  // is 16-byte aligned and the doubled mode block still fits the LDS
  const size_t lds2 = 2 * block_lds(B, ci, co, co / 2);
  if (co % 2 == 0 && co >= 4 && (reinterpret_cast<uintptr_t>(gw) & 15) == 0 && lds2 <= 160 * 1024) {
    const MixArgs a = make_args(B, ci, co, M, m0, m1, accumulate ? 1 : 0, co / 2);
    return launch(accumulate ? pick<WgradK2A>(co / 2) : pick<WgradK2>(co / 2), lds2, true,
                  static_cast<const float2*>(xhat),
                  static_cast<const float2*>(gy), static_cast<float2*>(gw), a, stream);
  }
  const MixArgs a = make_args(B, ci, co, M, m0, m1, accumulate ? 1 : 0);
  return launch(accumulate ? pick<WgradKA>(co) : pick<WgradK>(co), mix_lds_bytes(B, ci, co), true,
                static_cast<const float2*>(xhat),
                static_cast<const float2*>(gy), static_cast<float2*>(gw), a, stream);
}

}  // namespace dtst
