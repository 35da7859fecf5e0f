// Row kernels of the split schedule that contract z before t (forward) and
// expand t before z (inverse); z_first_fwd_cost and z_first_inv_cost in
// tables.cpp say when a plan takes them instead of the t-first kernels of
// k_stream.hip.
//
// Contracting t first costs N_z K_t N_t products per row for t alone, and its
// z step is complex.  Contracting z first takes the real row, so that
// X[-k] = conj(X[k]) before t: only k = 0 .. k_max are formed, a cosine and a
// sine product each.  Where the shard holds all of z, the rows z and
// N_z - 1 - z share them too: with the angle taken at z + 1/2 (the phase
// f = exp(i pi k / N_z) of the mode makes up for it) the cosines multiply the
// sum of the two rows and the sines their difference, for any N_z, odd ones
// included.  The t step then works on K_z / 2 + 1 modes instead of N_z rows
// and serves k and -k at once.  Matrix instructions per row, t first -> z
// first: 160 -> 96 at N_z = 128, N_t = 32, K_z = K_t = 16 (the paper's model);
// 100 -> 28 (forward) at N_z = 75, N_t = 10, K_z = 22, K_t = 6.
//
// Forward.  M = t (lane m reads t = TH m .. TH m + TH - 1 of position g of a K
// step, 4 TH contiguous bytes; 16 lanes a whole row), N = mode k, K =
// position.  The accumulators are, register for register, the B operand of
// the t contraction (M = k_t, N = k, K = t), and the combination of P, Q and f
// stays in the lane (zfinish in zrow_ops.h).  Kernels that contract or expand y as
// well may apply f to the columns of the plane's spectrum instead, after (forward)
// or before (inverse) y: fewer values than the rows'.
//
// Inverse.  With V = conj(f) Y[k], f Y[-k] and U = V C_t, the row is
//   y(z) = sum_k cos(k z') (Re U+ + Re U-) + sin(k z') (Im U- - Im U+),
// z' = 2 pi (z + 1/2) / N_z: the sums and differences of V are the A operand
// (M = mode, K = k_t) of the t expansion with N = t, whose accumulators are the
// A operand (M = t, K = mode) of the z expansion with N = z.  Folded, the
// cosine part E and the sine part O give E + O at z and E - O at N_z - 1 - z.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dtst_internal.h"

namespace dtst {
namespace {

#include "stream_ops.h"
#include "zrow_ops.h"

// TH: t groups; NT: 16-mode tiles of k = 0 .. kmax; MK: 1 when K_t <= 8 (Br
// and Bi rows in one tile), else 2; ACC: shorter chains (zrow_ops.h).
//
// Three waves per SIMD where the accumulators would spill at four (two t groups
// with two k_t tiles or ACC: 5 channels of 34 x 239 x 126 x 21 193 us at three, 323
// at four; 10 of 17 x 40 x 191 x 32, K_t 13, 56 and 74).
//
// Every wave walks its (row, unit) pairs with NB unit buffers, loads are
// unconditional and past the last unit re-read the last row, as in
// fwd_tz_body: the waits for one unit then cover that unit's loads only.
template <int TH, int NT, int MK, int FOLD, int MODE, int ACC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT == 1 && !(TH == 2 && (ACC || MK == 2)) ? 4 : 3)))
fwd_zrow_kernel(const float* __restrict__ x, float2* __restrict__ out, const float4* __restrict__ zimg,
                const float4* __restrict__ phase, const float* __restrict__ timg, ZRowArgs a) {
  constexpr int NB = kZBufs;
  extern __shared__ float4 zl4[];
  const int nimg = a.units * NT * 2 * 64;
  for (int i = threadIdx.x; i < nimg; i += blockDim.x) zl4[i] = zimg[i];

  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int64_t wstride = int64_t(gridDim.x) * wpb;
  // (the same in every lane: row addresses and loop conditions stay scalar)
  const int64_t wave = int64_t(blockIdx.x) * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  float ta[TH * 4][MK];
#pragma unroll
  for (int s = 0; s < TH * 4; ++s)
#pragma unroll
    for (int k = 0; k < MK; ++k) ta[s][k] = timg[(s * MK + k) * 64 + lane];
  float4 ph[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) ph[n] = phase[n * 64 + lane];
  __syncthreads();
  if (wave >= a.rows) return;

  const ZLane l = zlane<TH>(a);
  const int64_t row_len = int64_t(a.nz) * a.nt;
  const int64_t n_rows = (a.rows - 1 - wave) / wstride + 1;
  const int64_t n_iter = n_rows * a.units;
  const int64_t last_row = wave + (n_rows - 1) * wstride;

  float xb[NB][4][1 + FOLD][TH];
  int64_t rn = wave, itn = 0;
  int un = 0;
  int64_t rp[NB], itp[NB];
  int up[NB];
  auto fetch = [&](int k) __attribute__((always_inline)) {
    rp[k] = rn;
    up[k] = un;
    itp[k] = itn++;
    zload<TH, FOLD, MODE>(x + (rn < last_row ? rn : last_row) * row_len, a, l, un, xb[k]);
    if (++un == a.units) {
      un = 0;
      rn += wstride;
    }
  };
#pragma unroll
  for (int k = 0; k < NB; ++k) fetch(k);

  constexpr int ZS = ACC && TH == 1 ? 2 : 1;
  v4f R[ZS][NT][TH], I[ZS][NT][TH];
  auto step = [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const bool live = itp[k] < n_iter;
    const int64_t r = rp[k];
    const int u = up[k];
    if (live) zunit<TH, NT, FOLD, MODE>(xb[k], zl4, a, l, u, R, I);
    fetch(k);
    if (!live || u != a.units - 1) return;
    float2* orow = out + r * int64_t(2 * a.kmax) * a.kt;
    zfinish<TH, NT, MK, FOLD, ACC>(R, I, ph, ta, a, l, [&](int e, v4f_c v, bool both) {
      if (both) *reinterpret_cast<v4f_c*>(orow + e) = v;
      else orow[e] = make_float2(v[0], v[1]);
    });
  };
  static_assert(NB == 4, "four unit buffers");
  do {
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
  } while (itp[0] < n_iter);
}

// Each row's spectrum is loaded one row ahead.
template <int TH, int NS, int KG, int FOLD, int T32>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NS <= 4 ? 4 : 3)))
inv_zrow_kernel(const float2* __restrict__ in, float* __restrict__ y, const float2* __restrict__ zimg,
                const float4* __restrict__ phase, const float* __restrict__ timg, ZRowArgs a) {
  constexpr int NT = (NS + 3) / 4;
  extern __shared__ float2 zl2[];
  const int nimg = a.units * NS * 64;
  for (int i = threadIdx.x; i < nimg; i += blockDim.x) zl2[i] = zimg[i];

  const int lane = threadIdx.x & 63;
  const int m = lane & 15, g = lane >> 4;
  const int wpb = blockDim.x >> 6;
  const int64_t wstride = int64_t(gridDim.x) * wpb;
  const int64_t wave = int64_t(blockIdx.x) * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // B operand of the t expansion: column t (m of group h), K index k_t = 4kg +
  // g, Re and Im of C_t
  float tb[TH][KG][2];
#pragma unroll
  for (int h = 0; h < TH; ++h)
#pragma unroll
    for (int kg = 0; kg < KG; ++kg)
#pragma unroll
      for (int e = 0; e < 2; ++e) tb[h][kg][e] = timg[((h * KG + kg) * 2 + e) * 64 + lane];
  float4 ph[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) ph[n] = phase[n * 64 + lane];
  __syncthreads();
  if (wave >= a.rows) return;

  const int64_t row_len = int64_t(a.nz) * (T32 ? 32 : a.nt);
  const int64_t spec_len = int64_t(2 * a.kmax) * a.kt;
  float2 un[NT][KG][2];
  zinv_load<NT, KG>(in + wave * spec_len, a, m, g, un);
  for (int64_t r = wave; r < a.rows; r += wstride) {
    v4f A[NT][TH], B[NT][TH];
    zinv_t<TH, NT, KG, FOLD>(un, ph, tb, a, m, g, A, B);
    zinv_load<NT, KG>(in + (r + wstride < a.rows ? r + wstride : r) * spec_len, a, m, g, un);
    zinv_z<TH, NS, FOLD, T32>(A, B, zl2, a, m, g, y + r * row_len);
  }
}

template <class F>
const void* kernel_of(F* f) {
  return reinterpret_cast<const void*>(f);
}

template <int TH, int NT, int MK, int ACC>
const void* pick_f4(const ZRowCfg& c) {
  return c.fmode == 2 ? kernel_of(fwd_zrow_kernel<TH, NT, MK, 1, 2, ACC>) : kernel_of(fwd_zrow_kernel<TH, NT, MK, 1, 1, ACC>);
}
template <int TH, int NT, int MK>
const void* pick_f3(const ZRowCfg& c) {
  if (!c.fold) return kernel_of(fwd_zrow_kernel<TH, NT, MK, 0, 1, 0>);
  return c.acc ? pick_f4<TH, NT, MK, 1>(c) : pick_f4<TH, NT, MK, 0>(c);
}
template <int TH>
const void* pick_f2(const ZRowCfg& c) {
  if (c.ntl == 1) return c.mk == 1 ? pick_f3<TH, 1, 1>(c) : pick_f3<TH, 1, 2>(c);
  return c.mk == 1 ? pick_f3<TH, 2, 1>(c) : pick_f3<TH, 2, 2>(c);
}
const void* pick_f(const ZRowCfg& c) { return c.th == 2 ? pick_f2<2>(c) : pick_f2<1>(c); }

template <int TH, int NS, int T32>
const void* pick_i3(const ZRowCfg& c) {
  if (c.mk == 1) return c.fold ? kernel_of(inv_zrow_kernel<TH, NS, 2, 1, T32>) : kernel_of(inv_zrow_kernel<TH, NS, 2, 0, T32>);
  return c.fold ? kernel_of(inv_zrow_kernel<TH, NS, 4, 1, T32>) : kernel_of(inv_zrow_kernel<TH, NS, 4, 0, T32>);
}
template <int TH, int T32>
const void* pick_i2(const ZRowCfg& c) {
  switch (c.ns) {
    case 2: return pick_i3<TH, 2, T32>(c);
    case 3: return pick_i3<TH, 3, T32>(c);
    case 4: return pick_i3<TH, 4, T32>(c);
    case 6: return pick_i3<TH, 6, T32>(c);
    default: return pick_i3<TH, 8, T32>(c);
  }
}
const void* pick_i(const ZRowCfg& c, int nt) {
  if (c.th == 1) return pick_i2<1, 0>(c);
  return nt == 32 ? pick_i2<2, 1>(c) : pick_i2<2, 0>(c);
}

size_t lds_fwd(const ZRowCfg& c) { return size_t(c.units) * c.ntl * 2 * 64 * 16; }
size_t lds_inv(const ZRowCfg& c) { return size_t(c.units) * c.ns * 64 * 8; }

ZRowArgs args_of(const ZRowCfg& c, const StreamCfg& s, int64_t rows) {
  ZRowArgs a;
  a.rows = rows;
  a.nt = s.nt;
  a.nz = s.nz;
  a.kt = s.kt;
  a.kmax = s.kz / 2;
  a.np = c.np;
  a.np2 = c.np2;
  a.steps = c.steps;
  a.units = c.units;
  return a;
}

int grid_for(int resident, int64_t rows) {
  const int64_t want = (rows + 3) / 4;
  return static_cast<int>(want < resident ? want : resident);
}

// Resident workgroups of `fn` with `lds` bytes on the current device.
hipError_t resident(const void* fn, size_t lds, int* grid) {
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, lds);
  if (e == hipSuccess && per_cu <= 0) e = hipErrorInvalidConfiguration;
  *grid = cus * per_cu;
  return e;
}

}  // namespace

int prepare_zrow(ZRowCfg* c, int nt) {
  hipError_t e = hipSuccess;
  if (c->fwd == 1) e = resident(pick_f(*c), lds_fwd(*c), &c->grid_fwd);
  if (e == hipSuccess && c->inv == 1) e = resident(pick_i(*c, nt), lds_inv(*c), &c->grid_inv);
  return e;
}

int launch_fwd_zrow(const ZRowCfg& c, const StreamCfg& s, const float* x, void* out, int64_t rows, const float* timg,
                    const float* zimg, const float* phase, void* stream) {
  if (rows <= 0) return hipSuccess;
  ZRowArgs a = args_of(c, s, rows);
  float2* o = static_cast<float2*>(out);
  const float4* z = reinterpret_cast<const float4*>(zimg);
  const float4* p = reinterpret_cast<const float4*>(phase);
  void* args[] = {&x, &o, &z, &p, &timg, &a};
  return hipLaunchKernel(pick_f(c), dim3(grid_for(c.grid_fwd, rows)), dim3(256), args, lds_fwd(c),
                         static_cast<hipStream_t>(stream));
}

int launch_inv_zrow(const ZRowCfg& c, const StreamCfg& s, const void* in, float* y, int64_t rows, const float* timg,
                    const float* zimg, const float* phase, void* stream) {
  if (rows <= 0) return hipSuccess;
  ZRowArgs a = args_of(c, s, rows);
  const float2* i = static_cast<const float2*>(in);
  const float2* z = reinterpret_cast<const float2*>(zimg);
  const float4* p = reinterpret_cast<const float4*>(phase);
  void* args[] = {&i, &y, &z, &p, &timg, &a};
  return hipLaunchKernel(pick_i(c, s.nt), dim3(grid_for(c.grid_inv, rows)), dim3(256), args, lds_inv(c),
                         static_cast<hipStream_t>(stream));
}

}  // namespace dtst
