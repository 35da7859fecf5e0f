// Inverse y + t + z in one launch with z expanded last (the rows of k_zrow.hip,
// the plane structure of inv_yzt_kernel in k_stream.hip).
//
// A workgroup of 16 waves owns one part of one (b, c, x) plane: a run of groups
// of 16 y slots (a slot is the row pair (y, y + N_y/2) where y folds).  Each
// wave keeps 16 columns of the plane's (K_y x K_z K_t) spectrum as MFMA
// operands; per group it expands y for them into LDS, and after a barrier
// expands t and z of the row(s) of one slot; a second barrier frees the LDS
// rows.  Nothing but the spectrum is shared between the groups, so that a
// launch of few planes is divided into parts until it fills the CUs.  Against
// separate launches the (N_y x K_z K_t) intermediate stays out of HBM.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "dtst_internal.h"

namespace dtst {
namespace {

#include "stream_ops.h"
#include "zrow_ops.h"

template <int TH, int NS, int KG, int T32, int NCY, int JQY>
__global__ void __launch_bounds__(1024)
inv_yzrow_kernel(const float2* __restrict__ in, float* __restrict__ y, const float2* __restrict__ zimg,
                 const float4* __restrict__ phase, const float* __restrict__ timg, const float4* __restrict__ yimg,
                 ZRowArgs a, ZPlaneArgs f) {
  constexpr int NT = (NS + 3) / 4;
  // LDS: the y image, the z image, the exchanged rows
  extern __shared__ float4 lds[];
  const float4* ylds = lds;
  float2* zl2 = reinterpret_cast<float2*>(lds + f.yimg_n4);
  const int nimg = a.units * NS * 64;
  float2* vlds = zl2 + nimg;
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = blockIdx.x;
  if (item >= f.items) return;  // the host launches one workgroup per item
  const int pl = item / f.parts, q0 = (item - pl * f.parts) * f.gpp, q1 = min(q0 + f.gpp, f.jq);

  // B operands of the y expansion: spectrum row p (class cl, K index
  // 16q + 4g + i), column mc (lanes outside the spectrum read its first value
  // and are cleared).
  const int mc = 16 * w + m;
  const bool col_ok = mc < f.mcols;
  float2 u[NCY][JQY][4];
  constexpr int ACC = KG == 2;  // shorter chains (zrow_ops.h): K_t <= 8, where t-first rows fold z into four classes
  float4 ph[ACC ? 1 : NT];      // half-position phases: of the column (ACC), or of the row modes
#pragma unroll
  for (int n = 0; n < (ACC ? 1 : NT); ++n) ph[n] = phase[ACC ? min(mc, f.mcols - 1) : n * 64 + lane];
  {
    const float2* sp = in + pl * int64_t(f.ky) * f.mcols;
#pragma unroll
    for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
      for (int q = 0; q < JQY; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int kk = 16 * q + 4 * g + i;
          const int p = NCY == 2 ? 2 * kk + cl : kk;
          const bool ok = col_ok && p < f.ky;
          const float2 v = sp[ok ? int64_t(p) * f.mcols + mc : 0];
          u[cl][q][i] = ok ? v : make_float2(0.f, 0.f);
        }
  }
  float tb[TH][KG][2];
#pragma unroll
  for (int h = 0; h < TH; ++h)
#pragma unroll
    for (int kg = 0; kg < KG; ++kg)
#pragma unroll
      for (int e = 0; e < 2; ++e) tb[h][kg][e] = timg[((h * KG + kg) * 2 + e) * 64 + lane];
  for (int i = threadIdx.x; i < f.yimg_n4; i += blockDim.x) lds[i] = yimg[i];
  for (int i = threadIdx.x; i < nimg; i += blockDim.x) zl2[i] = zimg[i];
  __syncthreads();

  if constexpr (ACC) {  // (after the staging, so that the spectrum's loads stay in flight across it)
#pragma unroll
    for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
      for (int q = 0; q < JQY; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) u[cl][q][i] = turn<1>(u[cl][q][i].x, u[cl][q][i].y, conj_phase(ph[0]));
  }

  const int64_t row_len = int64_t(a.nz) * (T32 ? 32 : a.nt);
  for (int gq = q0; gq < q1; ++gq) {
    if (16 * w < f.mcols) {
      v4f er[NCY], ei[NCY], fr[NCY], fi[NCY];  // ACC: products of Re and of Im of the basis
#pragma unroll
      for (int cl = 0; cl < NCY; ++cl) {
        er[cl] = v4f{0.f, 0.f, 0.f, 0.f};
        ei[cl] = fr[cl] = fi[cl] = er[cl];
      }
#pragma unroll
      for (int q = 0; q < JQY; ++q)
#pragma unroll
        for (int cl = 0; cl < NCY; ++cl) {
          // image entry (((tile * JQ + q) * NCY + class) * 2 + part) * 64 + lane
          const int e = ((gq * JQY + q) * NCY + cl) * 2 * 64 + lane;
          const float4 br = ylds[e], bi = ylds[e + 64];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float2 v = u[cl][q][i];
            er[cl] = mfma(br[i], v.x, er[cl]);
            ei[cl] = mfma(br[i], v.y, ei[cl]);
            v4f& r = ACC ? fr[cl] : er[cl];
            v4f& s = ACC ? fi[cl] : ei[cl];
            r = mfma(bi[i], -v.y, r);
            s = mfma(bi[i], v.x, s);
          }
        }
      if constexpr (ACC) {
#pragma unroll
        for (int cl = 0; cl < NCY; ++cl) {
          er[cl] += fr[cl];
          ei[cl] += fi[cl];
        }
      }
      // accumulator register i holds slot 4g + i, column mc
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int sl = 4 * g + i;
        if constexpr (NCY == 2) {
          vlds[sl * f.mrow + mc] = make_float2(er[0][i] + er[1][i], ei[0][i] + ei[1][i]);
          vlds[(16 + sl) * f.mrow + mc] = make_float2(er[0][i] - er[1][i], ei[0][i] - ei[1][i]);
        } else {
          vlds[sl * f.mrow + mc] = make_float2(er[0][i], ei[0][i]);
        }
      }
    }
    __syncthreads();
    const int s = 16 * gq + w;
    if (s < f.slots) {
#pragma unroll
      for (int h = 0; h < NCY; ++h) {
        float2 un[NT][KG][2];
        zinv_load<NT, KG>(vlds + (h * 16 + w) * f.mrow, a, m, g, un);
        v4f A[NT][TH], B[NT][TH];
        if constexpr (ACC) zinv_t<TH, NT, KG, 0>(un, {}, tb, a, m, g, A, B);
        else zinv_t<TH, NT, KG, 1>(un, ph, tb, a, m, g, A, B);
        zinv_z<TH, NS, 1, T32>(A, B, zl2, a, m, g, y + (int64_t(pl) * f.ny + s + h * f.half) * row_len);
      }
    }
    __syncthreads();
  }
}

template <int TH, int NS, int KG, int T32>
const void* pick_y(const ZRowCfg& c) {
  if (c.ncy == 2) return reinterpret_cast<const void*>(inv_yzrow_kernel<TH, NS, KG, T32, 2, 1>);
  return reinterpret_cast<const void*>(c.kyt == 1 ? inv_yzrow_kernel<TH, NS, KG, T32, 1, 1>
                                                  : inv_yzrow_kernel<TH, NS, KG, T32, 1, 2>);
}
// (K_z K_t <= 256 bounds the modes at K_t > 8 to k_max <= 14)
template <int TH, int T32>
const void* pick_n(const ZRowCfg& c) {
  if (c.mk == 2) {
    if (c.ns == 2) return pick_y<TH, 2, 4, T32>(c);
    return c.ns == 3 ? pick_y<TH, 3, 4, T32>(c) : pick_y<TH, 4, 4, T32>(c);
  }
  if (c.ns == 2) return pick_y<TH, 2, 2, T32>(c);
  if (c.ns == 3) return pick_y<TH, 3, 2, T32>(c);
  if (c.ns == 4) return pick_y<TH, 4, 2, T32>(c);
  return c.ns == 6 ? pick_y<TH, 6, 2, T32>(c) : pick_y<TH, 8, 2, T32>(c);
}
const void* pick(const ZRowCfg& c, int nt) {
  if (c.th == 1) return pick_n<1, 0>(c);
  return nt == 32 ? pick_n<2, 1>(c) : pick_n<2, 0>(c);
}

}  // namespace

int prepare_inv_yzrow(const ZRowCfg& c, int nt) {
  int per_cu = 0;
  const void* fn = pick(c, nt);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(c.ifused_lds_bytes));
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 1024, c.ifused_lds_bytes);
  if (e != hipSuccess) return e;
  return per_cu > 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

int launch_inv_yzrow(const ZRowCfg& c, const StreamCfg& s, const AxisCfg& ay, const void* in, float* y, int64_t planes,
                     int ny, const float* timg, const float* zimg, const float* phase, const float* yimg,
                     void* stream) {
  if (planes <= 0) return hipSuccess;
  // the image must have the K steps and tiles the kernel assumes
  if (ay.JQ != c.kyt || (ay.fold == 2) != (c.ncy == 2) || ay.parts != 2) return hipErrorInvalidValue;
  ZRowArgs a;
  a.nt = s.nt;
  a.nz = s.nz;
  a.kt = s.kt;
  a.kmax = s.kz / 2;
  a.np = c.np;
  a.np2 = c.np2;
  a.steps = c.steps;
  a.units = c.units;
  ZPlaneArgs f;
  f.ny = ny;
  f.slots = ay.fold == 2 ? ny / 2 : ny;
  f.half = ay.fold == 2 ? ny / 2 : 0;
  f.jq = ay.ktiles;
  // A workgroup fills a CU (of 256): the parts that leave the least work on
  // the busiest one, counting a part's start (staging, the spectrum operands)
  // as a third of a slot group.
  int64_t best = 0;
  f.gpp = f.jq;
  for (int64_t parts = 1; parts <= f.jq && planes * parts <= 16384; ++parts) {
    const int64_t gpp = (f.jq + parts - 1) / parts;
    const int64_t cost = (planes * parts + 255) / 256 * (3 * gpp + 1);
    if (best == 0 || cost < best) {
      best = cost;
      f.gpp = static_cast<int>(gpp);
    }
  }
  f.parts = (f.jq + f.gpp - 1) / f.gpp;  // (1 where there are more planes than kInvPlanesPerLaunch)
  f.kth = 0;
  f.ky = ay.J;
  f.mcols = s.kz * s.kt;
  f.mrow = c.fused_mrow;
  f.yimg_n4 = ay.ktiles * ay.JQ * (ay.fold == 2 ? 2 : 1) * 2 * 64;
  const float2* z = reinterpret_cast<const float2*>(zimg);
  const float4* p = reinterpret_cast<const float4*>(phase);
  const float4* yi = reinterpret_cast<const float4*>(yimg);
  for (int64_t p0 = 0; p0 < planes; p0 += kInvPlanesPerLaunch) {
    const int64_t n = std::min(planes - p0, kInvPlanesPerLaunch);
    const float2* i = static_cast<const float2*>(in) + p0 * f.ky * f.mcols;
    float* yp = y + p0 * ny * s.nz * s.nt;
    a.rows = n * ny;
    f.items = static_cast<int>(n) * f.parts;
    void* args[] = {&i, &yp, &z, &p, &timg, &yi, &a, &f};
    const hipError_t e = hipLaunchKernel(pick(c, s.nt), dim3(f.items), dim3(1024), args, c.ifused_lds_bytes,
                                         static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dtst
