// Device functions of the z-first rows (k_zrow.hip has the method), shared by
// the row kernels there and the kernels that contract or expand y as well
// (k_zrow_y.hip, k_zrow_yi.hip).  Included after stream_ops.h inside namespace
// dtst::{anonymous}.
#pragma once

// Pairs of floats at any 4-byte boundary; pairs of complex values, 8-byte
// aligned.
typedef float v2f_u __attribute__((ext_vector_type(2), aligned(4)));
typedef float v4f_c __attribute__((ext_vector_type(4), aligned(8)));

struct ZRowArgs {
  int64_t rows;
  int nt, nz, kt;
  int kmax;   // z modes 0 .. kmax - 1 and -kmax .. -1
  int np;     // z positions: ceil(N_z / 2) folded, else N_z
  int np2;    // positions with a partner row N_z - 1 - z: N_z / 2 folded
  int steps;  // K steps of four positions
  int units;  // 16-position units (forward), 16-row z tiles (inverse)
};

// Planes of the kernels that contract or expand y too.
struct ZPlaneArgs {
  int items;    // planes * parts
  int parts;    // parts per plane
  int gpp;      // slot groups (of 16 slots) per part
  int ny;       // rows per plane
  int slots;    // slots per plane: N_y / 2 folded, else N_y
  int half;     // N_y / 2 folded (second row of a slot), else 0
  int jq;       // slot groups per plane
  int kth;      // k tiles per y class in the y image
  int ky;       // K_y
  int mcols;    // K_z K_t
  int mrow;     // LDS row stride in complex values
  int yimg_n4;  // float4 entries of the y image
};

// Unit buffers per wave: NB - 1 units are in flight while one is contracted.
constexpr int kZBufs = 4;

// This lane's fixed part of the forward's accesses.
struct ZLane {
  int m, g;
  // byte offsets within a row (unsigned 32-bit: the loads take them beside the
  // row's scalar address)
  unsigned off0;  // position g, the lane's t
  unsigned last;  // the last position
  unsigned mir;   // offset + partner's offset
};
// t positions TH m .. TH m + TH - 1 (those past the extent: its last ones,
// with zero t basis values).
template <int TH>
__device__ __forceinline__ ZLane zlane(const ZRowArgs& a) {
  ZLane l;
  const int lane = threadIdx.x & 63;
  l.m = lane & 15;
  l.g = lane >> 4;
  const int t0 = min(TH * l.m, a.nt - TH);
  l.off0 = 4u * (l.g * a.nt + t0);
  l.last = 4u * ((a.np - 1) * a.nt + t0);
  l.mir = 4u * ((a.nz - 1) * a.nt + 2 * t0);
  return l;
}

// The four steps' values of unit u of the row at xr (positions 16u + 4st + g
// and, FOLD, their partners).  Unconditional: positions past the last one
// repeat it (MODE 2: there are none).
template <int TH, int FOLD, int MODE>
__device__ __forceinline__ void zload(const float* xr, const ZRowArgs& a, const ZLane& l, int u,
                                      float (&dst)[4][1 + FOLD][TH]) {
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const unsigned at = l.off0 + 4u * ((16 * u + 4 * st) * a.nt);
    const unsigned off = MODE == 2 ? at : min(at, l.last);
#pragma unroll
    for (int p = 0; p < 1 + FOLD; ++p) {
      const char* src = reinterpret_cast<const char*>(xr) + (p == 0 ? off : l.mir - off);
      if constexpr (TH == 2) {
        const v2f_u v = *reinterpret_cast<const v2f_u*>(src);
        dst[st][p][0] = v.x;
        dst[st][p][1] = v.y;
      } else {
        dst[st][p][0] = *reinterpret_cast<const float*>(src);
      }
    }
  }
}

// ACC: shorter chains of roundings, for rows whose t-first form folds z into
// classes and so has short chains too (ZRowCfg::acc).  The K steps of the z
// products then go to ZS = 2 accumulator sets in turn where the registers allow
// it, the t products of a row form two chains, and the phases are applied with
// what rounding them left out; the fused kernels keep the products of Re and Im
// of the y basis in chains of their own and apply the phases to the columns.  Forward of 16 x 24 x 144 x 12, modes
// 8/9/12/5, error against 64 bits: 2.16e-7 without, 1.79e-7 with (t first 1.86e-7);
// 64^3 x 16, 16 channels: 68.3 us without, 71.6 with (t first 76).

// Contracts one unit into the row's accumulators: R with the cosines of the
// sums, I with the (negative) sines of the differences.  zl4: float4 (four
// steps) of the unit's cosine and sine tiles.  MODE 2: every position and
// partner exists.
template <int TH, int NT, int FOLD, int MODE, int ZS>
__device__ __forceinline__ void zunit(const float (&xv)[4][1 + FOLD][TH], const float4* zl4, const ZRowArgs& a,
                                      const ZLane& l, int u, v4f (&R)[ZS][NT][TH], v4f (&I)[ZS][NT][TH]) {
  if (u == 0) {
#pragma unroll
    for (int p = 0; p < ZS; ++p)
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int j = 0; j < TH; ++j) {
          R[p][n][j] = v4f{0.f, 0.f, 0.f, 0.f};
          I[p][n][j] = v4f{0.f, 0.f, 0.f, 0.f};
        }
  }
  float4 c[NT], s[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    c[n] = zl4[((u * NT + n) * 2 + 0) * 64 + (threadIdx.x & 63)];
    s[n] = zl4[((u * NT + n) * 2 + 1) * 64 + (threadIdx.x & 63)];
  }
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    if (MODE != 2 && 4 * u + st >= a.steps) break;  // the same for the whole launch
    const int pos = 16 * u + 4 * st + l.g;
    float f[TH], d[TH];
#pragma unroll
    for (int j = 0; j < TH; ++j) {
      const float lo = MODE == 2 || pos < a.np ? xv[st][0][j] : 0.f;
      if constexpr (FOLD) {
        const float hi = MODE == 2 || pos < a.np2 ? xv[st][FOLD][j] : 0.f;
        f[j] = lo + hi;
        d[j] = lo - hi;
      } else {
        f[j] = lo;
        d[j] = lo;
      }
    }
    const auto at = [&](const float4& v) { return st == 0 ? v.x : (st == 1 ? v.y : (st == 2 ? v.z : v.w)); };
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < TH; ++j) {
        v4f& r = R[st % ZS][n][j];
        v4f& i = I[st % ZS][n][j];
        r = mfma(f[j], at(c[n]), r);
        i = mfma(d[j], at(s[n]), i);
      }
  }
}

// (x + i y) (c + i s) of a phase c + i s = (ph.x + ph.z) + i (ph.y + ph.w), the
// second parts what rounding the first left out (ACC = 0: without them).
template <int ACC>
__device__ __forceinline__ float2 turn(float x, float y, const float4& ph) {
  if constexpr (!ACC) return make_float2(fmaf(x, ph.x, -(y * ph.y)), fmaf(y, ph.x, x * ph.y));
  return make_float2(fmaf(x, ph.x, fmaf(-y, ph.y, fmaf(x, ph.z, -(y * ph.w)))),
                     fmaf(y, ph.x, fmaf(x, ph.y, fmaf(y, ph.z, x * ph.w))));
}
__device__ __forceinline__ float4 conj_phase(const float4& ph) { return make_float4(ph.x, -ph.y, ph.z, -ph.w); }

// Finishes a row.  Lane (m, g) holds mode k = 16n + m, t = TH (4g + i) + j in
// register i of R[.][n][j] (Re) and I[.][n][j] (Im).  The t contraction of both
// gives P and Q (k_t rows, B_t = Br + i Bi), and the modes are
//   X[k] = f (P + i Q),   X[-k] = conj(f) (P - i Q),
// f the mode's half-position phase (PH = 0: left to the caller, who applies it
// after the y contraction, to fewer values).  st(index, v) takes the coefficients
// of k_t and k_t + 1 at index = p K_t + k_t; `both` false: of k_t only.
template <int TH, int NT, int MK, int PH, int ACC, int ZS, class St>
__device__ __forceinline__ void zfinish(const v4f (&R)[ZS][NT][TH], const v4f (&I)[ZS][NT][TH],
                                        const float4 (&ph)[NT], const float (&ta)[TH * 4][MK], const ZRowArgs& a,
                                        const ZLane& l, St&& st) {
  constexpr int TC = ACC ? 2 : 1;  // chains
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    v4f P[MK], Q[MK];
#pragma unroll
    for (int c = 0; c < TC; ++c)
#pragma unroll
      for (int kk = 0; kk < MK; ++kk) {
        v4f p = v4f{0.f, 0.f, 0.f, 0.f}, q = p;
#pragma unroll
        for (int j = 0; j < TH; ++j)
#pragma unroll
          for (int i = 4 / TC * c; i < 4 / TC * (c + 1); ++i) {
            float r = R[0][n][j][i], im = I[0][n][j][i];
            if constexpr (ZS == 2) {
              r += R[ZS - 1][n][j][i];
              im += I[ZS - 1][n][j][i];
            }
            p = mfma(ta[4 * j + i][kk], r, p);
            q = mfma(ta[4 * j + i][kk], im, q);
          }
        P[kk] = c == 0 ? p : P[kk] + p;
        Q[kk] = c == 0 ? q : Q[kk] + q;
      }
    const int k = 16 * n + l.m;
#pragma unroll
    for (int e = 0; e < MK; ++e) {
      // k_t = 8e + 2g + i: Br products in register 2e + i of tile 0 (MK = 1:
      // register i), Bi products of tile 1 (MK = 1: register 2 + i)
      v4f_c up, dn;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r0 = MK == 2 ? 2 * e + i : i, r1 = MK == 2 ? 2 * e + i : 2 + i;
        const float pr = P[0][r0], pi = P[MK - 1][r1], qr = Q[0][r0], qi = Q[MK - 1][r1];
        float2 u = make_float2(pr - qi, pi + qr), d = make_float2(pr + qi, pi - qr);
        if constexpr (PH) {
          // (with two tiles of modes and two t groups the registers spill)
          u = turn<ACC && NT * TH < 4>(u.x, u.y, ph[n]);
          d = turn<ACC && NT * TH < 4>(d.x, d.y, conj_phase(ph[n]));
        }
        up[2 * i] = u.x;
        up[2 * i + 1] = u.y;
        dn[2 * i] = d.x;
        dn[2 * i + 1] = d.y;
      }
      const int kt = 8 * e + 2 * l.g;
      if (kt < a.kt) {
        const bool both = kt + 1 < a.kt;
        if (k < a.kmax) st(k * a.kt + kt, up, both);
        if (k >= 1 && k <= a.kmax) st((2 * a.kmax - k) * a.kt + kt, dn, both);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Inverse.  NT: 16-mode tiles; NS: K steps of four modes (k = 0 .. kmax within
// 4 NS); KG: groups of four k_t; T32: N_t = 32, streamed as whole 128-byte rows.
// Row m of tile n of the t expansion is mode k = 16n + 4(m & 3) + (m >> 2),
// which makes K step s of the z expansion the modes 4s .. 4s + 3.
// ---------------------------------------------------------------------------

// Spectrum index of Y[k] (neg = 0) or Y[-k] at k_t = 4kg + g, and whether the
// coefficient is retained (else index 0).
__device__ __forceinline__ int zinv_index(const ZRowArgs& a, int m, int g, int n, int kg, int neg, bool* ok) {
  const int k = 16 * n + 4 * (m & 3) + (m >> 2), kt = 4 * kg + g;
  *ok = kt < a.kt && (neg ? k >= 1 && k <= a.kmax : k < a.kmax);
  return *ok ? (neg ? 2 * a.kmax - k : k) * a.kt + kt : 0;
}

template <int NT, int KG>
__device__ __forceinline__ void zinv_load(const float2* u, const ZRowArgs& a, int m, int g, float2 (&un)[NT][KG][2]) {
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int kg = 0; kg < KG; ++kg)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        bool ok;
        const int i = zinv_index(a, m, g, n, kg, e, &ok);
        un[n][kg][e] = u[i];
      }
}

// A operands of the t expansion from p = Y[k], q = Y[-k] (zero where not
// retained) and the mode's phase f (PH = 0: p and q have it already): with
// V+ = conj(f) p and V- = f q,
//   a0 = Re V+ + Re V-,  a1 = -(Im V+ + Im V-),  b0 = Im V- - Im V+,  b1 = Re V- - Re V+.
template <int PH, int ACC>
__device__ __forceinline__ void zinv_ab(float2 p, float2 q, const float4& ph, float* a0, float* a1, float* b0,
                                        float* b1) {
  if constexpr (PH) {
    p = turn<ACC>(p.x, p.y, conj_phase(ph));
    q = turn<ACC>(q.x, q.y, ph);
  }
  *a0 = p.x + q.x;
  *a1 = -(p.y + q.y);
  *b0 = q.y - p.y;
  *b1 = q.x - p.x;
}

// t expansion of a row: A (cosine) and B (sine) parts, tb the B operand
// (column t, K index k_t = 4kg + g; Re and Im of C_t, with K_t <= 8 a chain of
// roundings each: the t-first form of such rows may fold z into four classes).
template <int TH, int NT, int KG, int PH>
__device__ __forceinline__ void zinv_t(const float2 (&un)[NT][KG][2], const float4 (&ph)[NT],
                                       const float (&tb)[TH][KG][2], const ZRowArgs& a, int m, int g,
                                       v4f (&A)[NT][TH], v4f (&B)[NT][TH]) {
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    constexpr int ACC = KG == 2;
    v4f A1[TH], B1[TH];
#pragma unroll
    for (int h = 0; h < TH; ++h) {
      A[n][h] = v4f{0.f, 0.f, 0.f, 0.f};
      B[n][h] = A1[h] = B1[h] = A[n][h];
    }
#pragma unroll
    for (int kg = 0; kg < KG; ++kg) {
      bool okp, okn;
      (void)zinv_index(a, m, g, n, kg, 0, &okp);
      (void)zinv_index(a, m, g, n, kg, 1, &okn);
      const float2 p = okp ? un[n][kg][0] : make_float2(0.f, 0.f), q = okn ? un[n][kg][1] : make_float2(0.f, 0.f);
      float a0, a1, b0, b1;
      zinv_ab<PH, ACC>(p, q, ph[n], &a0, &a1, &b0, &b1);
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        A[n][h] = mfma(a0, tb[h][kg][0], A[n][h]);
        B[n][h] = mfma(b0, tb[h][kg][0], B[n][h]);
        v4f& aa = ACC ? A1[h] : A[n][h];
        v4f& bb = ACC ? B1[h] : B[n][h];
        aa = mfma(a1, tb[h][kg][1], aa);
        bb = mfma(b1, tb[h][kg][1], bb);
      }
    }
    if constexpr (ACC) {
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        A[n][h] += A1[h];
        B[n][h] += B1[h];
      }
    }
  }
}

// z expansion and stores of a row.  zl2: (cosine, sine) per z tile and K step.
template <int TH, int NS, int FOLD, int T32>
__device__ __forceinline__ void zinv_z(const v4f (&A)[(NS + 3) / 4][TH], const v4f (&B)[(NS + 3) / 4][TH],
                                       const float2* zl2, const ZRowArgs& a, int m, int g, float* __restrict__ yrow) {
  const int nt = T32 ? 32 : a.nt;
  for (int zt = 0; zt < a.units; ++zt) {
    // E: cosine part, O: sine part (unfolded: both into E)
    v4f Y[1 + FOLD][TH];
#pragma unroll
    for (int p = 0; p < 1 + FOLD; ++p)
#pragma unroll
      for (int h = 0; h < TH; ++h) Y[p][h] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float2 cs = zl2[(zt * NS + s) * 64 + (threadIdx.x & 63)];
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        Y[0][h] = mfma(A[s / 4][h][s % 4], cs.x, Y[0][h]);
        Y[FOLD][h] = mfma(B[s / 4][h][s % 4], cs.y, Y[FOLD][h]);
      }
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int h = 0; h < TH; ++h) {
        const v4f s = Y[0][h] + Y[1][h], d = Y[0][h] - Y[1][h];
        Y[0][h] = s;
        Y[FOLD][h] = d;
      }
    }
    if constexpr (T32) {
      // lanes m and m^8 trade one 16-byte chunk so that each store writes 8
      // whole 128-byte rows
      const int za = 16 * zt + (m & 7), zb = za + 8;
      const int tch = (m < 8 ? 0 : 16) + 4 * g;
#pragma unroll
      for (int p = 0; p < 1 + FOLD; ++p) {
        float va[4], vb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          va[i] = ror8_into<0xC>(Y[p][0][i], Y[p][TH - 1][i]);
          vb[i] = ror8_into<0x3>(Y[p][TH - 1][i], Y[p][0][i]);
        }
        const int lim = p == 0 ? a.np : a.np2;
        if (za < lim) store_stream(yrow + (p == 0 ? za : a.nz - 1 - za) * 32 + tch, va[0], va[1], va[2], va[3]);
        if (zb < lim) store_stream(yrow + (p == 0 ? zb : a.nz - 1 - zb) * 32 + tch, vb[0], vb[1], vb[2], vb[3]);
      }
    } else {
      const int zl = 16 * zt + m;
#pragma unroll
      for (int p = 0; p < 1 + FOLD; ++p) {
        float* dst = yrow + (p == 0 ? zl : a.nz - 1 - zl) * nt;
        const bool ok = zl < (p == 0 ? a.np : a.np2);
#pragma unroll
        for (int h = 0; h < TH; ++h)
          if (ok && t_chunk<TH, 0>(h, g, nt)) *reinterpret_cast<v4f_u*>(dst + t_start<TH, 0>(h, g, nt)) = Y[p][h];
      }
    }
  }
}
