// Inverse z + t expansion fused with the block epilogue, one wave per task:
//
//   y[b,o,n] = GELU( sum_i w[o,i] x[b,i,n] + Re sum_{kz,kt} C_t C_z V[b,o,kz,kt] ),
//
// V the y-expanded spectrum (B, C_out, N_x, N_y, K_z, K_t), for few input channels.
// The chunked kernel (block_zt.h) runs one workgroup of two waves per SIMD in lock
// step, a barrier per chunk of z rows, and forms the bypass on 16-channel matrix
// tiles: with few channels most of its lanes idle and each step costs a memory
// latency (5 channels of 2 x 12 x 159 rows of 204 x 16, with the x and y
// expansions: 545 us, here 209 us).
//
// Here a workgroup of 8 waves takes a few (b, x, y) rows at a time.  First the
// waves expand t of the rows' spectra, a (row, channel) each, with t before z
// as in k_zrow.hip, and leave the cosine and sine parts in LDS in the layout of
// the z expansion's A operand.  After a barrier every wave takes tasks of its
// own, a (row, z tile, t group): it reads the C_in input chunks of its 16 z
// positions (and of their mirror rows) into registers, 16 bytes a lane, and
// for each output channel expands z on the matrix cores, adds the bypass with
// vector FMAs on the same lanes (weights broadcast from LDS), applies GELU and
// stores.  No values are exchanged between the matrix and the vector part, and
// tasks need no barrier.  Bound: HBM and the latency of a task's reads for few
// channels, the vector unit above (C_in C_out FMAs and 15 C_out GELU
// instructions per point), so plans take it up to 8 input channels (12 with one
// t group); above 8 output channels not for short rows, whose expansion a group
// pays per output channel (the rule, with figures, is where Derived::blk is set).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dtst_internal.h"

namespace dtst {
namespace {

#include "stream_ops.h"
#include "zrow_ops.h"
#include "gelu_as.h"

constexpr int kRowWaves = 8;

struct RowBlockArgs {
  int64_t rows, xy;  // B * N_x * N_y, N_x * N_y
  int ci, co;
  int rw;            // rows per group
  int ns, nt16;      // K steps of the z image; 16-mode tiles
  int kg;            // groups of four k_t in the t image
};

// CI: input channels padded to a multiple of 4 (zero weights).
template <int TH, int FOLD, int CI>
__global__ void __launch_bounds__(64 * kRowWaves)
inv_row_block_kernel(const float2* __restrict__ in, const float* __restrict__ x, const float* __restrict__ wb,
                     float* __restrict__ y, const float2* __restrict__ zimg, const float4* __restrict__ phase,
                     const float* __restrict__ timg, ZRowArgs a, RowBlockArgs ba) {
  constexpr int NP = 1 + FOLD;  // z row sets
  extern __shared__ float4 lds[];
  // LDS: the expanded t parts, the z image, the t image, the weights
  float4* ul = lds;
  const int n_u = ba.rw * ba.co * ba.nt16 * 2 * TH * 64;
  float2* zl2 = reinterpret_cast<float2*>(lds + n_u);
  const int n_z = a.units * ba.ns * 64;
  float* tl = reinterpret_cast<float*>(zl2 + n_z);
  const int n_t = TH * ba.kg * 2 * 64;
  float* wl = tl + n_t;
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < n_z; i += blockDim.x) zl2[i] = zimg[i];
  for (int i = threadIdx.x; i < n_t; i += blockDim.x) tl[i] = timg[i];
  for (int i = threadIdx.x; i < ba.co * CI; i += blockDim.x) {
    const int o = i / CI, c = i - o * CI;
    wl[i] = c < ba.ci ? wb[o * ba.ci + c] : 0.f;
  }
  __syncthreads();

  const int64_t row_len = int64_t(a.nz) * a.nt;
  const int64_t cs = ba.xy * row_len;  // channel stride of x and y
  const int spec_len = 2 * a.kmax * a.kt;
  const int64_t groups = (ba.rows + ba.rw - 1) / ba.rw;
  const int n_items = ba.rw * ba.co * ba.nt16;
  const int n_tasks = ba.rw * a.units * TH;

  for (int64_t gi = blockIdx.x; gi < groups; gi += gridDim.x) {
    const int64_t row0 = gi * ba.rw;
    // ---- t expansion of the group's rows: item (row, channel, mode tile) ----
    auto load = [&](int it, float2 (&un)[1][4][2]) __attribute__((always_inline)) {
      const int n = it % ba.nt16, q = it / ba.nt16, rw = q / ba.co, o = q - rw * ba.co;
      const int64_t row = row0 + rw < ba.rows ? row0 + rw : ba.rows - 1;
      const int64_t b = row / ba.xy, rxy = row - b * ba.xy;
      const float2* u = in + ((b * ba.co + o) * ba.xy + rxy) * spec_len;
#pragma unroll
      for (int kg = 0; kg < 4; ++kg)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          bool ok;
          const int i = zinv_index(a, m, g, n, kg, e, &ok);
          const float2 v = u[i];
          un[0][kg][e] = v;
        }
    };
    float2 cur[1][4][2];
    if (w < n_items) load(w, cur);
    for (int it = w; it < n_items; it += kRowWaves) {
      float2 nxt[1][4][2];
      load(it + kRowWaves < n_items ? it + kRowWaves : it, nxt);
      const int n = it % ba.nt16;
      const float4 ph = phase[n * 64 + lane];
      v4f A[TH], B[TH];
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        A[h] = v4f{0.f, 0.f, 0.f, 0.f};
        B[h] = v4f{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) {
        if (kg >= ba.kg) break;
        bool okp, okn;
        (void)zinv_index(a, m, g, n, kg, 0, &okp);
        (void)zinv_index(a, m, g, n, kg, 1, &okn);
        const float2 p = okp ? cur[0][kg][0] : make_float2(0.f, 0.f), q = okn ? cur[0][kg][1] : make_float2(0.f, 0.f);
        float a0, a1, b0, b1;
        zinv_ab<FOLD, 0>(p, q, ph, &a0, &a1, &b0, &b1);
#pragma unroll
        for (int h = 0; h < TH; ++h) {
          const float t0 = tl[((h * ba.kg + kg) * 2 + 0) * 64 + lane], t1 = tl[((h * ba.kg + kg) * 2 + 1) * 64 + lane];
          A[h] = mfma(a0, t0, A[h]);
          B[h] = mfma(b0, t0, B[h]);
          A[h] = mfma(a1, t1, A[h]);
          B[h] = mfma(b1, t1, B[h]);
        }
      }
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        ul[((it * 2 + 0) * TH + h) * 64 + lane] = make_float4(A[h][0], A[h][1], A[h][2], A[h][3]);
        ul[((it * 2 + 1) * TH + h) * 64 + lane] = make_float4(B[h][0], B[h][1], B[h][2], B[h][3]);
      }
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) {
        cur[0][kg][0] = nxt[0][kg][0];
        cur[0][kg][1] = nxt[0][kg][1];
      }
    }
    __syncthreads();

    // ---- tasks: (row, z tile, t group) ----
    for (int ti = w; ti < n_tasks; ti += kRowWaves) {
      const int h = ti % TH, q = ti / TH, rw = q / a.units, zt = q - rw * a.units;
      const int64_t row = row0 + rw;
      if (row >= ba.rows) break;
      const int64_t b = row / ba.xy, rxy = row - b * ba.xy;
      const int zl = 16 * zt + m, zc = min(zl, a.np - 1);
      const bool chunk = t_chunk<TH, 0>(h, g, a.nt);
      const int ts = t_start<TH, 0>(h, g, a.nt);
      const float* xr = x + b * ba.ci * cs + rxy * row_len;
      float* yr = y + b * ba.co * cs + rxy * row_len;
      const unsigned off[2] = {static_cast<unsigned>(zc * a.nt + ts), static_cast<unsigned>((a.nz - 1 - zc) * a.nt + ts)};
      const bool ok[2] = {chunk && zl < a.np, chunk && zl < a.np2};
      // cosine and sine of the tile's z positions for each K step
      float2 csv[2][4];
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          csv[n][s] = 4 * n + s < ba.ns ? zl2[(zt * ba.ns + 4 * n + s) * 64 + lane] : make_float2(0.f, 0.f);
      v4f xv[CI][NP];
#pragma unroll
      for (int c = 0; c < CI; ++c) {
        const float* xc = xr + (c < ba.ci ? c : ba.ci - 1) * cs;
#pragma unroll
        for (int p = 0; p < NP; ++p) xv[c][p] = *reinterpret_cast<const v4f_u*>(xc + off[p]);
      }
#pragma unroll 1
      for (int o = 0; o < ba.co; ++o) {
        v4f E = v4f{0.f, 0.f, 0.f, 0.f}, O = E;
        const float4* uo = ul + ((rw * ba.co + o) * ba.nt16 * 2 * TH + h) * 64 + lane;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          if (n >= ba.nt16) break;
          const float4 ua = uo[(2 * n) * TH * 64], ub = uo[(2 * n + 1) * TH * 64];
          const float uav[4] = {ua.x, ua.y, ua.z, ua.w}, ubv[4] = {ub.x, ub.y, ub.z, ub.w};
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            E = mfma(uav[s], csv[n][s].x, E);
            O = mfma(ubv[s], csv[n][s].y, O);
          }
        }
        v4f acc[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[p] = v4f{0.f, 0.f, 0.f, 0.f};
        const float4* wo = reinterpret_cast<const float4*>(wl + o * CI);
#pragma unroll
        for (int c4 = 0; c4 < CI / 4; ++c4) {
          const float4 wv = wo[c4];
          const float w4[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[p][i] = fmaf(w4[c], xv[4 * c4 + c][p][i], acc[p][i]);
        }
        float* yo = yr + o * cs;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          v4f r;
#pragma unroll
          for (int i = 0; i < 4; ++i) r[i] = gelu_as((p == 1 ? E[i] - O[i] : E[i] + O[i]) + acc[p][i]);
          if (ok[p]) *reinterpret_cast<v4f_u*>(yo + off[p]) = r;
        }
      }
    }
    __syncthreads();
  }
}

template <int TH, int FOLD>
const void* pick_ci(int64_t ci) {
  if (ci <= 4) return reinterpret_cast<const void*>(inv_row_block_kernel<TH, FOLD, 4>);
  if (ci <= 8) return reinterpret_cast<const void*>(inv_row_block_kernel<TH, FOLD, 8>);
  return reinterpret_cast<const void*>(inv_row_block_kernel<TH, FOLD, 12>);
}
const void* pick(const ZRowCfg& c, int64_t ci) {
  if (c.th == 1) return c.fold ? pick_ci<1, 1>(ci) : pick_ci<1, 0>(ci);
  return c.fold ? pick_ci<2, 1>(ci) : pick_ci<2, 0>(ci);
}

int ci_pad(int64_t ci) { return static_cast<int>((ci + 3) / 4 * 4); }
int tiles16(const ZRowCfg& c) { return (c.ns + 3) / 4; }

// LDS without the expanded parts, and the parts of one row.
size_t fixed_lds(const ZRowCfg& c, int64_t ci, int64_t co) {
  return size_t(c.units) * c.ns * 64 * 8 + size_t(c.th) * 2 * c.mk * 2 * 64 * 4 + size_t(co) * ci_pad(ci) * 4;
}
size_t row_lds(const ZRowCfg& c, int64_t co) { return size_t(co) * tiles16(c) * 2 * c.th * 64 * 16; }

// Rows per group: enough tasks for the 8 waves, within half of the LDS (two
// workgroups a CU) where one row fits it, else one row.
int rows_per_group(const ZRowCfg& c, int64_t ci, int64_t co) {
  const int tasks = c.units * c.th;
  int want = (kRowWaves + tasks - 1) / tasks;
  const size_t fixed = fixed_lds(c, ci, co), row = row_lds(c, co);
  while (want > 1 && fixed + want * row > 80 * 1024) --want;
  return want;
}

size_t lds_of(const ZRowCfg& c, int64_t ci, int64_t co) {
  return fixed_lds(c, ci, co) + rows_per_group(c, ci, co) * row_lds(c, co);
}

}  // namespace

bool block_row_supported(const ZRowCfg& c, int64_t ci, int64_t co) {
  return c.ns > 0 && ci <= 12 && co <= 32 && lds_of(c, ci, co) <= 160 * 1024;
}

int prepare_block_row(const ZRowCfg& c, int64_t ci, int64_t co, int* grid) {
  const void* fn = pick(c, ci);
  const size_t lds = lds_of(c, ci, co);
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * kRowWaves, lds);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) return hipErrorInvalidConfiguration;
  *grid = cus * per_cu;
  return hipSuccess;
}

int launch_inv_row_block(const ZRowCfg& c, const StreamCfg& s, int grid_resident, const void* in, const float* x,
                         const float* w, float* y, int64_t batch, int64_t nxy, int64_t ci, int64_t co,
                         const float* timg, const float* zimg, const float* phase, void* stream) {
  ZRowArgs a;
  a.rows = batch * nxy;
  if (a.rows <= 0) return hipSuccess;
  if (!block_row_supported(c, ci, co) || grid_resident <= 0) return hipErrorInvalidConfiguration;
  a.nt = s.nt;
  a.nz = s.nz;
  a.kt = s.kt;
  a.kmax = s.kz / 2;
  a.np = c.np;
  a.np2 = c.np2;
  a.steps = c.steps;
  a.units = c.units;
  RowBlockArgs ba;
  ba.rows = a.rows;
  ba.xy = nxy;
  ba.ci = static_cast<int>(ci);
  ba.co = static_cast<int>(co);
  ba.rw = rows_per_group(c, ci, co);
  ba.ns = c.ns;
  ba.nt16 = tiles16(c);
  ba.kg = 2 * c.mk;
  const int64_t groups = (a.rows + ba.rw - 1) / ba.rw;
  const int grid = static_cast<int>(groups < grid_resident ? groups : grid_resident);
  const float2* in2 = static_cast<const float2*>(in);
  const float2* z = reinterpret_cast<const float2*>(zimg);
  const float4* p = reinterpret_cast<const float4*>(phase);
  void* args[] = {&in2, &x, &w, &y, &z, &p, &timg, &a, &ba};
  return hipLaunchKernel(pick(c, ci), dim3(grid), dim3(64 * kRowWaves), args, lds_of(c, ci, co),
                         static_cast<hipStream_t>(stream));
}

}  // namespace dtst
