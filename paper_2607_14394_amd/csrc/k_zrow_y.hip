// Forward z + t + y in one launch with z contracted first (the rows of
// k_zrow.hip, the plane structure of fwd_tzy_kernel in k_stream.hip).
//
// A workgroup of 8 waves owns one part of one (b, c, x) plane at a time
// (persistent over parts): a plane's y rows come in groups of 16 slots (a
// slot is the row pair (y, y + N_y/2) where y folds) and a part is a run of
// groups.  Each wave contracts the rows of two slots of a group and leaves
// the (K_z x K_t) results in LDS; after a barrier the waves contract y for the
// group's slots, 16 columns of K_z K_t at a time, accumulating over the part's
// groups in registers; a second barrier frees the LDS rows.  The x contraction
// that follows sums the parts of a plane along with its N_x planes (its J is
// N_x times the parts, the parts of one x sharing the basis value).
//
// Against separate launches this keeps the (N_y x K_z K_t) intermediate out
// of HBM (written and read back: at K_z K_t = 256 a quarter as many bytes as
// the 128 x 32 rows themselves; storing it took 62 of the row kernel's 336 us
// on 20 channels of 32 x 128 x 128 x 32, and the y launch 46).  Parts exist
// because one workgroup fills a CU: 640 planes on 256 CUs would run as three
// rounds of which the last is half empty.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dtst_internal.h"

namespace dtst {
namespace {

#include "stream_ops.h"
#include "zrow_ops.h"

constexpr int kYWaves = 8;

// MODE 2: N_z a multiple of 32, whole units without masks.  ACC: shorter chains
// of roundings (zrow_ops.h), 1 of the y products alone, 2 of the rows' as well; the
// phases then go to the columns.  Two workgroups a CU where 128 registers hold the
// accumulators (one t group, one y tile): 28 channels of 21 x 21 x 28 x 8 19.3 us
// without ACC, 23.2 with it and 131 registers, 20.8 with it and 128.
template <int TH, int NT, int MK, int FOLD, int MODE, int NCY, int KYT, int ACC>
__global__ void __launch_bounds__(64 * kYWaves) __attribute__((amdgpu_waves_per_eu(TH == 1 && NCY == 1 && KYT == 1 ? 4 : 2)))
fwd_zty_kernel(const float* __restrict__ x, float2* __restrict__ out, const float4* __restrict__ zimg,
               const float4* __restrict__ phase, const float* __restrict__ timg, const float4* __restrict__ yimg,
               ZRowArgs a, ZPlaneArgs f) {
  constexpr int NB = kZBufs, NW = kYWaves;
  constexpr int SPW = 16 / NW;         // slots of a group per wave
  constexpr int MTW = 16 / NW;         // 16-column tiles of the y contraction per wave
  // LDS: the y image, the z image, the exchanged row results
  extern __shared__ float4 lds[];
  const float4* ylds = lds;
  float4* zl4 = lds + f.yimg_n4;
  const int nimg = a.units * NT * 2 * 64;
  float2* vlds = reinterpret_cast<float2*>(zl4 + nimg);
  for (int i = threadIdx.x; i < f.yimg_n4; i += blockDim.x) lds[i] = yimg[i];
  for (int i = threadIdx.x; i < nimg; i += blockDim.x) zl4[i] = zimg[i];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (static_cast<int>(blockIdx.x) >= f.items) return;  // the host never launches more workgroups than items

  float ta[TH * 4][MK];
#pragma unroll
  for (int s = 0; s < TH * 4; ++s)
#pragma unroll
    for (int k = 0; k < MK; ++k) ta[s][k] = timg[(s * MK + k) * 64 + lane];
  // half-position phases: of this lane's columns (ACC), or of its row modes
  float4 ph[ACC ? MTW : NT];
#pragma unroll
  for (int t = 0; t < (ACC ? MTW : NT); ++t)
    ph[t] = phase[ACC ? min(16 * (w + NW * t) + (lane & 15), f.mcols - 1) : t * 64 + lane];

  const ZLane l = zlane<TH>(a);
  const int m = l.m, g = l.g;
  const int64_t row_len = int64_t(a.nz) * a.nt;

  // Position of a unit: item (plane, part), slot group, slot of this wave,
  // row of the slot, unit (fastest).
  struct Cur {
    int it, pl, q0, q1, q, j, h, u;  // item, its plane and groups [q0, q1), group, slot, row, unit
  };
  auto at_item = [&](Cur& c) {
    const int it = c.it < f.items ? c.it : f.items - 1;
    c.pl = it / f.parts;
    c.q0 = (it - c.pl * f.parts) * f.gpp;
    c.q1 = min(c.q0 + f.gpp, f.jq);
    c.q = c.q0;
  };
  auto advance = [&](Cur c) {
    if (++c.u == a.units) {
      c.u = 0;
      if (++c.h == NCY) {
        c.h = 0;
        if (++c.j == SPW) {
          c.j = 0;
          if (++c.q == c.q1) {
            c.it += gridDim.x;
            at_item(c);
          }
        }
      }
    }
    return c;
  };
  // Slots past the plane's end read its first row and contribute zeros;
  // positions past the last item (loaded, never contracted) read the last one.
  auto row_of = [&](const Cur& c, bool* valid) {
    const int s = 16 * c.q + w + NW * c.j;
    *valid = s < f.slots;
    return int64_t(c.pl) * f.ny + (*valid ? s + c.h * f.half : 0);
  };

  float xb[NB][4][1 + FOLD][TH];
  bool vb[NB];
  Cur cb[NB];
  cb[0] = Cur{static_cast<int>(blockIdx.x), 0, 0, 0, 0, 0, 0, 0};
  at_item(cb[0]);
#pragma unroll
  for (int k = 1; k < NB; ++k) cb[k] = advance(cb[k - 1]);
#pragma unroll
  for (int k = 0; k < NB; ++k) zload<TH, FOLD, MODE>(x + row_of(cb[k], &vb[k]) * row_len, a, l, cb[k].u, xb[k]);
  __syncthreads();

  v4f yr[NCY][KYT][MTW], yi[NCY][KYT][MTW];
#pragma unroll
  for (int c = 0; c < NCY; ++c)
#pragma unroll
    for (int k = 0; k < KYT; ++k)
#pragma unroll
      for (int t = 0; t < MTW; ++t) {
        yr[c][k][t] = v4f{0.f, 0.f, 0.f, 0.f};
        yi[c][k][t] = v4f{0.f, 0.f, 0.f, 0.f};
      }
  constexpr int ZS = ACC == 2 ? 2 : 1;
  v4f R[ZS][NT][TH], I[ZS][NT][TH];

  // As fwd_tzy_kernel's process: contract buffer k's unit, refill the buffer,
  // at a row's end leave its results in LDS, and after the wave's last row of
  // a slot group run the group's y contraction.  (live is the same for the
  // whole workgroup.)
  auto process = [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const Cur c = cb[k];
    const bool valid = vb[k];
    const bool live = c.it < f.items;
    if (live) zunit<TH, NT, FOLD, MODE>(xb[k], zl4, a, l, c.u, R, I);
    const Cur far = advance(cb[(k + NB - 1) % NB]);
    cb[k] = far;
    zload<TH, FOLD, MODE>(x + row_of(far, &vb[k]) * row_len, a, l, far.u, xb[k]);
    if (!live || c.u != a.units - 1) return;
    float2* vrow = vlds + (c.h * 16 + w + NW * c.j) * f.mrow;
    const auto put = [&](int e, v4f_c v, bool both) __attribute__((always_inline)) {
      vrow[e] = valid ? make_float2(v[0], v[1]) : make_float2(0.f, 0.f);
      if (both) vrow[e + 1] = valid ? make_float2(v[2], v[3]) : make_float2(0.f, 0.f);
    };
    if constexpr (ACC) zfinish<TH, NT, MK, 0, ACC == 2>(R, I, {}, ta, a, l, put);
    else zfinish<TH, NT, MK, FOLD, 0>(R, I, ph, ta, a, l, put);
    if (c.h != NCY - 1 || c.j != SPW - 1) return;
    __syncthreads();
    float4 br[NCY][KYT], bi[NCY][KYT];
#pragma unroll
    for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
      for (int kk = 0; kk < KYT; ++kk) {
        const int kt = NCY == 2 ? cl * f.kth + kk : kk;
        const int e = (kt * f.jq + c.q) * 2 * 64 + lane;
        br[cl][kk] = ylds[e];
        bi[cl][kk] = ylds[e + 64];
      }
#pragma unroll
    for (int t = 0; t < MTW; ++t) {
      const int mt = w + NW * t;
      if (16 * mt >= f.mcols) continue;
      const int mc = 16 * mt + m;
      // (all of the tile's reads first: one LDS latency instead of four)
      float2 vs[NCY][4];
#pragma unroll
      for (int c2 = 0; c2 < NCY; ++c2)
#pragma unroll
        for (int i = 0; i < 4; ++i) vs[c2][i] = vlds[(16 * c2 + 4 * g + i) * f.mrow + mc];
      __builtin_amdgcn_sched_barrier(0);
      // ACC: the products of Im of the basis in a chain of their own per group
      v4f pr[NCY][KYT], pi[NCY][KYT];
#pragma unroll
      for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
        for (int kk = 0; kk < KYT; ++kk) {
          pr[cl][kk] = ACC ? v4f{0.f, 0.f, 0.f, 0.f} : yr[cl][kk][t];
          pi[cl][kk] = ACC ? v4f{0.f, 0.f, 0.f, 0.f} : yi[cl][kk][t];
        }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 va = vs[0][i];
        float2 xs[NCY];
        if constexpr (NCY == 2) {
          const float2 vh = vs[NCY - 1][i];
          xs[0] = make_float2(va.x + vh.x, va.y + vh.y);
          xs[1] = make_float2(va.x - vh.x, va.y - vh.y);
        } else {
          xs[0] = va;
        }
#pragma unroll
        for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
          for (int kk = 0; kk < KYT; ++kk) {
            v4f& r = ACC ? yr[cl][kk][t] : pr[cl][kk];
            v4f& q = ACC ? yi[cl][kk][t] : pi[cl][kk];
            r = mfma(br[cl][kk][i], xs[cl].x, r);
            q = mfma(br[cl][kk][i], xs[cl].y, q);
            pr[cl][kk] = mfma(bi[cl][kk][i], -xs[cl].y, pr[cl][kk]);
            pi[cl][kk] = mfma(bi[cl][kk][i], xs[cl].x, pi[cl][kk]);
          }
      }
#pragma unroll
      for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
        for (int kk = 0; kk < KYT; ++kk) {
          yr[cl][kk][t] = ACC ? yr[cl][kk][t] + pr[cl][kk] : pr[cl][kk];
          yi[cl][kk][t] = ACC ? yi[cl][kk][t] + pi[cl][kk] : pi[cl][kk];
        }
      if (c.q == c.q1 - 1) {
        // part done: rows p of K_y (class cl, slot 16kk + 4g + i), columns mc
        float2* op = out + c.it * int64_t(f.ky) * f.mcols;
#pragma unroll
        for (int cl = 0; cl < NCY; ++cl)
#pragma unroll
          for (int kk = 0; kk < KYT; ++kk) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int sl = 16 * kk + 4 * g + i;
              const int p = NCY == 2 ? 2 * sl + cl : sl;
              const float2 v = make_float2(yr[cl][kk][t][i], yi[cl][kk][t][i]);
              if (p < f.ky && mc < f.mcols) op[int64_t(p) * f.mcols + mc] = ACC ? turn<1>(v.x, v.y, ph[ACC ? t : 0]) : v;
            }
            yr[cl][kk][t] = v4f{0.f, 0.f, 0.f, 0.f};
            yi[cl][kk][t] = v4f{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
    __syncthreads();
  };
  static_assert(NB == 4, "four unit buffers");
  do {
    process(std::integral_constant<int, 0>{});
    process(std::integral_constant<int, 1>{});
    process(std::integral_constant<int, 2>{});
    process(std::integral_constant<int, 3>{});
  } while (cb[0].it < f.items);
}

template <int TH, int NT, int MK, int FOLD, int MODE, int ACC>
const void* pick_y(const ZRowCfg& c) {
  if (c.ncy == 2) return reinterpret_cast<const void*>(fwd_zty_kernel<TH, NT, MK, FOLD, MODE, 2, 1, ACC>);
  return reinterpret_cast<const void*>(c.kyt == 1 ? fwd_zty_kernel<TH, NT, MK, FOLD, MODE, 1, 1, ACC>
                                                  : fwd_zty_kernel<TH, NT, MK, FOLD, MODE, 1, 2, ACC>);
}
template <int TH, int NT, int MK>
const void* pick_fold(const ZRowCfg& c) {
  if (!c.fold) return pick_y<TH, NT, MK, 0, 1, 0>(c);
  if (c.acc == 2) return c.fmode == 2 ? pick_y<TH, NT, MK, 1, 2, 2>(c) : pick_y<TH, NT, MK, 1, 1, 2>(c);
  if constexpr (TH == 1) {
    if (c.acc) return c.fmode == 2 ? pick_y<TH, NT, MK, 1, 2, 1>(c) : pick_y<TH, NT, MK, 1, 1, 1>(c);
  }
  return c.fmode == 2 ? pick_y<TH, NT, MK, 1, 2, 0>(c) : pick_y<TH, NT, MK, 1, 1, 0>(c);
}
// The combinations that plans take (zty_covers in tables.cpp): two t groups
// with one mode tile, one t group with K_t <= 8.
const void* pick(const ZRowCfg& c) {
  if (c.th == 2) return c.mk == 1 ? pick_fold<2, 1, 1>(c) : pick_fold<2, 1, 2>(c);
  return c.ntl == 1 ? pick_fold<1, 1, 1>(c) : pick_fold<1, 2, 1>(c);
}

}  // namespace

int prepare_fwd_zty(ZRowCfg* c) {
  int dev = 0, cus = 0, per_cu = 0;
  const void* fn = pick(*c);
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(c->fused_lds_bytes));
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * kYWaves, c->fused_lds_bytes);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) return hipErrorInvalidConfiguration;
  c->grid_fused = cus * per_cu;
  return hipSuccess;
}

int launch_fwd_zty(const ZRowCfg& c, const StreamCfg& s, const AxisCfg& ay, const float* x, void* out, int64_t planes,
                   int ny, const float* timg, const float* zimg, const float* phase, const float* yimg, void* stream) {
  if (planes <= 0) return hipSuccess;
  if (planes * c.parts > 0x7fffffff) return hipErrorInvalidConfiguration;
  ZRowArgs a;
  a.rows = planes * ny;
  a.nt = s.nt;
  a.nz = s.nz;
  a.kt = s.kt;
  a.kmax = s.kz / 2;
  a.np = c.np;
  a.np2 = c.np2;
  a.steps = c.steps;
  a.units = c.units;
  ZPlaneArgs f;
  f.parts = c.parts;
  f.items = static_cast<int>(planes) * c.parts;
  f.ny = ny;
  f.slots = ay.fold == 1 ? ny / 2 : ny;
  f.half = ay.fold == 1 ? ny / 2 : 0;
  f.jq = ay.JQ;
  f.gpp = (ay.JQ + c.parts - 1) / c.parts;
  f.kth = ay.kth;
  f.ky = ay.KO;
  f.mcols = s.kz * s.kt;
  f.mrow = c.fused_mrow;
  f.yimg_n4 = ay.ktiles * ay.JQ * 2 * 64;
  const int grid = f.items < c.grid_fused ? f.items : c.grid_fused;
  float2* o = static_cast<float2*>(out);
  const float4* z = reinterpret_cast<const float4*>(zimg);
  const float4* p = reinterpret_cast<const float4*>(phase);
  const float4* yi = reinterpret_cast<const float4*>(yimg);
  void* args[] = {&x, &o, &z, &p, &timg, &yi, &a, &f};
  return hipLaunchKernel(pick(c), dim3(grid), dim3(64 * kYWaves), args, c.fused_lds_bytes,
                         static_cast<hipStream_t>(stream));
}

}  // namespace dtst
