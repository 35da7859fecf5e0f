// Host-side geometry validation and basis tables of the DTST library.
//
// Everything here is plain C++ (no HIP): it derives the kernel
// configuration from a descriptor and builds, in fp64, the kernel-ready
// images of the per-dimension basis matrices of Sec. V-B Eq. (basis_matrix),
//   B_i[k, j] = exp(-2 pi i ((k * (offset_i + j)) mod N_i) / N_i),
// each value rounded once to fp32.  The exponent is reduced in exact
// integer arithmetic before the angle is formed, so no precision is lost to
// large k*n products (k*n reaches 2.6e5 at N = 512).
#include <algorithm>
#include <cmath>
#include <limits>

#include "dtst_internal.h"

namespace dtst {

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t round_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

// exp(-2 pi i r / N) of every r < N for the few N of one plan: the images take
// each value many times over (every lane of every tile).  Filled on demand
// while build_images runs, on its thread; larger N are evaluated directly.
struct TwiddleTables {
  struct Table {
    int64_t N;
    std::vector<double> v;  // (re, im), NaN until evaluated
  };
  std::vector<Table> tables;
  double* entry(int64_t N, int64_t r) {
    if (N > 4096) return nullptr;
    for (Table& t : tables)
      if (t.N == N) return &t.v[2 * r];
    tables.push_back({N, std::vector<double>(2 * N, std::numeric_limits<double>::quiet_NaN())});
    return &tables.back().v[2 * r];
  }
};
thread_local TwiddleTables* g_twiddles = nullptr;

// exp(-2 pi i r / N) with r = (k * n) mod N, k, n >= 0.
inline void twiddle(int64_t N, int64_t k, int64_t n, double* re, double* im) {
  const int64_t r = ((k % N) * (n % N)) % N;
  double* e = g_twiddles ? g_twiddles->entry(N, r) : nullptr;
  if (e && e[0] == e[0]) {
    *re = e[0];
    *im = e[1];
    return;
  }
  const double ang = kTwoPi * static_cast<double>(r) / static_cast<double>(N);
  *re = std::cos(ang);
  *im = -std::sin(ang);
  if (e) {
    e[0] = *re;
    e[1] = *im;
  }
}

// Real-inverse weight of stored t index kt (Sec. V-A inverse, half spectrum).
inline double half_weight(int64_t nt, int64_t kt) {
  if (kt == 0) return 1.0;
  if (nt % 2 == 0 && kt == nt / 2) return 1.0;
  return 2.0;
}

// Classes stacked in an inverse axis image entry (fold 2: parity, fold 4:
// k mod 4); the forward images hold one class per k tile.
inline int axis_image_classes(const AxisCfg& a) { return a.fold == 2 ? 2 : (a.fold == 4 ? 4 : 1); }

// z image blocks of 16 rows (forward) or 16 K entries (inverse) per (class,
// z tile): mt, plus mt / 2 when t folds (the three-product form's third
// operand, see z_forward_image and z_inverse_image).
inline int z_blocks(const StreamCfg& s) { return s.tf ? 3 * s.mt / 2 : s.mt; }

// Matrix instructions per row of the t-first kernels (either direction) and
// of the z-first ones.
int t_first_cost(const StreamCfg& s) {
  const int t = s.ncls * s.th * 4 * s.ct / (s.tf ? 2 : 1);
  const int z = s.ncls * (s.tf ? 3 * s.mt / 2 : s.mt * s.ct) * 4;
  return s.zt * (t + z);
}
int z_first_fwd_cost(const ZRowCfg& z) { return z.ntl * 2 * z.th * (z.steps + 4 * z.mk); }
int z_first_inv_cost(const ZRowCfg& z) { return 2 * z.th * (z.units * z.ns + (z.ns + 3) / 4 * 4 * z.mk); }

// The z-first row kernels' configuration (whole_z: the shard holds all of z).
// Returns false for rows they do not cover.
bool z_first(const StreamCfg& s, bool whole_z, ZRowCfg* out) {
  ZRowCfg z;
  z.th = s.th;
  const int modes = s.kz / 2 + 1;  // k = 0 .. k_max
  if (!s.vec || s.th > 2 || modes > 32) return false;
  z.ntl = modes <= 16 ? 1 : 2;
  z.ns = static_cast<int>(ceil_div(modes, 4));
  z.ns = z.ns <= 2 ? 2 : (z.ns <= 4 ? z.ns : (z.ns <= 6 ? 6 : 8));
  z.mk = s.kt <= 8 ? 1 : 2;
  z.fold = whole_z && s.nz >= 2 ? 1 : 0;
  z.np = z.fold ? (s.nz + 1) / 2 : s.nz;
  z.np2 = z.fold ? s.nz / 2 : 0;
  z.steps = static_cast<int>(ceil_div(z.np, 4));
  z.units = static_cast<int>(ceil_div(z.np, 16));
  z.fmode = z.fold && s.nz % 32 == 0 ? 2 : 1;
  // Where the t-first rows fold z their chains are short, and so are these rows'
  // (zrow_ops.h) unless the y chains alone make up for them: one t group and one
  // unit of z (layer of 32^3 x 8: error 2.5e-7 and 28.9 us, with both 2.4e-7 and
  // 29.7, with neither 2.7e-7 and 28.9; t first 2.5e-7).
  z.acc = s.ncls == 1 ? 0 : (z.th == 1 && z.units == 1 ? 1 : 2);
  // z bases in LDS, four workgroups a CU
  if (z.units * size_t(z.ntl) * 2 * 64 * 16 > 40 * 1024 || z.units * size_t(z.ns) * 64 * 8 > 40 * 1024) return false;
  *out = z;
  return true;
}

bool mul_ok(int64_t a, int64_t b, int64_t* out) {
  if (a < 0 || b < 0) return false;
  if (a != 0 && b > std::numeric_limits<int64_t>::max() / a) return false;
  *out = a * b;
  return true;
}

}  // namespace

int64_t retained_index(const dtst_desc& d, int dim, int64_t p) {
  if (dim == 3) return p;
  const int64_t k = d.kmax[dim];
  return p < k ? p : d.n_global[dim] - 2 * k + p;
}

dtst_status derive(const dtst_desc* d, uint32_t flags, Derived* out, std::string* err) {
  if (!d || !out) {
    *err = "null descriptor";
    return DTST_ERR_INVALID_ARG;
  }
  static const char* names[4] = {"x", "y", "z", "t"};
  for (int i = 0; i < 4; ++i) {
    if (d->n_global[i] < 1 || d->n_local[i] < 1 || d->offset[i] < 0 ||
        d->n_local[i] > d->n_global[i] || d->offset[i] > d->n_global[i] - d->n_local[i]) {
      *err = std::string("dimension ") + names[i] +
             ": need n_global >= 1, n_local >= 1, 0 <= offset, offset + n_local <= n_global";
      return DTST_ERR_INVALID_ARG;
    }
    if (d->n_global[i] > (int64_t(1) << 30)) {
      *err = std::string("dimension ") + names[i] + ": n_global above 2^30";
      return DTST_ERR_INVALID_ARG;
    }
  }
  for (int i = 0; i < 3; ++i) {
    if (d->kmax[i] < 1 || 2 * int64_t(d->kmax[i]) > d->n_global[i]) {
      *err = std::string("dimension ") + names[i] + ": need 1 <= 2*kmax <= n_global";
      return DTST_ERR_INVALID_ARG;
    }
  }
  if (d->kt < 1 || d->kt > d->n_global[3] / 2 + 1) {
    *err = "t: need 1 <= kt <= n_global_t/2 + 1";
    return DTST_ERR_INVALID_ARG;
  }
  if (d->batch < 0 || d->c_in < 1 || d->c_out < 1) {
    *err = "need batch >= 0, c_in >= 1, c_out >= 1";
    return DTST_ERR_INVALID_ARG;
  }
  if ((flags & ~uint32_t(DTST_PLAN_SPLIT_SCHEDULE | DTST_PLAN_UNFUSED_BLOCK)) != 0) {
    *err = "unknown plan flag";
    return DTST_ERR_INVALID_ARG;
  }

  Derived dv;
  dv.d = *d;
  for (int i = 0; i < 3; ++i) dv.K[i] = 2 * int64_t(d->kmax[i]);
  dv.K[3] = d->kt;
  dv.M = dv.K[0] * dv.K[1] * dv.K[2] * dv.K[3];

  // Element counts must stay far inside int64.
  const int64_t cmax = std::max(d->c_in, d->c_out);
  int64_t t = 1;
  bool ok = mul_ok(std::max<int64_t>(d->batch, 1), cmax, &t);
  for (int i = 0; i < 4 && ok; ++i) ok = mul_ok(t, d->n_local[i], &t);
  int64_t tm = 1;
  ok = ok && mul_ok(std::max<int64_t>(d->batch, 1), cmax, &tm) && mul_ok(tm, dv.M, &tm);
  int64_t tw = 1;
  ok = ok && mul_ok(dv.M, d->c_in, &tw) && mul_ok(tw, d->c_out, &tw);
  if (!ok || t > (int64_t(1) << 50) || tm > (int64_t(1) << 50) || tw > (int64_t(1) << 50)) {
    *err = "problem size overflows the supported element counts";
    return DTST_ERR_INVALID_ARG;
  }

  // ---- streaming t+z configuration ----
  StreamCfg& sc = dv.sc;
  sc.nt = static_cast<int>(d->n_local[3]);
  sc.nz = static_cast<int>(d->n_local[2]);
  sc.kt = d->kt;
  sc.kz = static_cast<int>(dv.K[2]);
  if (sc.kt <= 8) {
    sc.ct = 1;
  } else if (sc.kt <= 16) {
    sc.ct = 2;
  } else {
    *err = "kt > 16 is not covered by the streaming kernels";
    return DTST_ERR_UNSUPPORTED;
  }
  if (sc.nt <= 16) {
    sc.th = 1;
  } else if (sc.nt <= 32) {
    sc.th = 2;
  } else if (sc.nt <= 64) {
    sc.th = 4;
  } else {
    *err = "local N_t > 64 is not covered by the streaming kernels";
    return DTST_ERR_UNSUPPORTED;
  }
  // z folds when this shard holds the whole even z extent: into 2 classes by
  // mode parity, or into 4 by k mod 4 when N_z % 4 == 0 and the stored
  // position of a mode has its residue (k even).  The four-class fold takes
  // either Re / Im of k_t in separate column tiles (ct == 2, the factors +-i
  // swap tiles) with at most 16 modes per class (one Re and one Im row tile:
  // the kernels fit their registers only at that size), or one column tile
  // (ct == 1, the factors +-i trade lanes m and m ^ 8) with at most 8 modes
  // per class, whose Re and Im rows then share one 16-row tile (mt == 1).
  // The z products per row are (padded slots per class) x N_z whatever the
  // class count, so the count taken is the one with the fewest padded slots
  // per class, and of those the smallest (fewer class sums and differences):
  // with at most 16 modes every count pads to one 16-row tile.
  const bool fold = d->n_local[2] == d->n_global[2] && d->n_global[2] % 2 == 0;
  const bool fold4_base = fold && d->n_global[2] % 4 == 0 && d->kmax[2] % 2 == 0;
  const bool fold4_ct2 = fold4_base && sc.ct == 2 && sc.kz <= 4 * 16;
  const bool fold4_ct1 = fold4_base && sc.ct == 1 && sc.kz <= 4 * 8;
  auto padded = [&](int n) {
    if (n == 4 && sc.ct == 1) return 8;
    int k = static_cast<int>(round_up(ceil_div(sc.kz, n), 16));
    return k == 48 ? 64 : k;
  };
  sc.ncls = 1;
  if (fold && padded(2) < padded(sc.ncls)) sc.ncls = 2;
  if ((fold4_ct2 || fold4_ct1) && padded(4) < padded(sc.ncls)) sc.ncls = 4;
  int kcp = padded(sc.ncls);
  if (kcp > 64) {
    *err = "more than 64 retained z modes per parity class is not covered";
    return DTST_ERR_UNSUPPORTED;
  }
  sc.kcp = kcp;
  sc.mt = kcp / 8;
  sc.zh = sc.nz / sc.ncls;
  sc.zt = static_cast<int>(ceil_div(sc.zh, 16));
  sc.vec = sc.nt >= 4 ? 1 : 0;
  // t folds (even k_t from x(t) + x(t + N_t/2), odd k_t from the difference)
  // in the split kernels when the shard holds the whole N_t = 32.  Shorter even
  // N_t would fold too (each half is one 16-wide group from 18), 7% faster over 40
  // random geometries, but the three-product z step that goes with it made the
  // forward's error 10% larger (up to 20%: 32 x 16 x 154 x 28 2.4e-7 -> 2.9e-7) and the
  // inverse's 2%: only the block kernel, below, folds those, where its z image, half
  // as large again, fits the LDS.
  auto z_lds = [&] { return size_t(sc.ncls) * sc.zt * z_blocks(sc) * 64 * 16; };
  sc.tf = (sc.ct == 2 && sc.th == 2 && sc.nt % 2 == 0 && d->n_local[3] == d->n_global[3]) ? 1 : 0;
  StreamCfg folded = sc;
  if (sc.nt != 32) {
    if (z_lds() > 160 * 1024) folded.tf = 0;
    sc.tf = 0;
  }
  sc.lds_bytes = z_lds();
  if (sc.lds_bytes > 160 * 1024) {
    *err = "z basis image exceeds the 160 KiB LDS of a workgroup";
    return DTST_ERR_UNSUPPORTED;
  }

  // ---- axis contractions ----
  auto axis = [](int J, int KO, int64_t NN, int fold) {
    AxisCfg a;
    a.J = J;
    a.KO = KO;
    a.NN = static_cast<int>(NN);
    a.fold = fold;
    if (fold == 1) {
      a.JQ = static_cast<int>(ceil_div(J / 2, 16));
      a.kth = static_cast<int>(ceil_div(KO / 2, 16));
      a.ktiles = 2 * a.kth;
    } else if (fold == 2) {
      a.JQ = static_cast<int>(ceil_div(J / 2, 16));
      a.ktiles = static_cast<int>(ceil_div(KO / 2, 16));
    } else if (fold == 3) {
      a.JQ = static_cast<int>(ceil_div(J / 4, 16));
      a.kth = static_cast<int>(ceil_div(KO / 4, 16));
      a.ktiles = 4 * a.kth;
    } else if (fold == 4) {
      a.JQ = static_cast<int>(ceil_div(J / 4, 16));
      a.ktiles = static_cast<int>(ceil_div(KO / 4, 16));
    } else {
      a.JQ = static_cast<int>(ceil_div(J, 16));
      a.ktiles = static_cast<int>(ceil_div(KO, 16));
    }
    return a;
  };
  const int64_t nn_y = dv.K[2] * dv.K[3];
  const int64_t nn_x = dv.K[1] * nn_y;
  if (nn_x > (int64_t(1) << 30)) {
    *err = "retained mode count too large";
    return DTST_ERR_UNSUPPORTED;
  }
  // A dimension folds when this shard holds its whole even global extent.
  const bool fold_x = d->n_local[0] == d->n_global[0] && d->n_global[0] % 2 == 0;
  const bool fold_y = d->n_local[1] == d->n_global[1] && d->n_global[1] % 2 == 0;
  dv.ay_f = axis(static_cast<int>(d->n_local[1]), static_cast<int>(dv.K[1]), nn_y, fold_y ? 1 : 0);
  dv.ax_f = axis(static_cast<int>(d->n_local[0]), static_cast<int>(dv.K[0]), nn_x, fold_x ? 1 : 0);
  dv.ax_i = axis(static_cast<int>(dv.K[0]), static_cast<int>(d->n_local[0]), nn_x, fold_x ? 2 : 0);
  dv.ay_i = axis(static_cast<int>(dv.K[1]), static_cast<int>(d->n_local[1]), nn_y, fold_y ? 2 : 0);

  // ---- workspace: the complex intermediates of the largest channel count ----
  // W1 = (.., N_x, N_y, K_z, K_t) between the t+z and y steps, W2 = (.., N_x,
  // K_y, K_z, K_t) between the y and x steps (W1 only without the fused y).
  const int64_t bc = d->batch * cmax;
  const size_t w1 = round_up(size_t(bc) * d->n_local[0] * d->n_local[1] * nn_y * 8, 256);
  const size_t w2 = round_up(size_t(bc) * d->n_local[0] * dv.K[1] * nn_y * 8, 256);

  // ---- fused forward t + z + y ----
  // Taken when the y contraction fits the fused kernel's registers (one
  // 16-column tile of K_z K_t per wave of 16, at most two 16-row k tiles of
  // K_y per wave) and its LDS.  The plan flag DTST_PLAN_SPLIT_SCHEDULE keeps
  // the separate t + z and y launches.
  {
    const bool split = (flags & DTST_PLAN_SPLIT_SCHEDULE) != 0;
    sc.ncy = fold_y ? 2 : 1;
    sc.kyt = fold_y ? dv.ay_f.kth : dv.ay_f.ktiles;
    const int mcols = static_cast<int>(nn_y);
    sc.fused_mrow = static_cast<int>(round_up(mcols, 32)) + 16;
    // z image, the 16 slots' exchanged rows, and the larger of the forward and
    // inverse y images when that still fits (else the y images are read from
    // global memory)
    const size_t yf = size_t(dv.ay_f.ktiles) * dv.ay_f.JQ * 2 * 64 * 16;
    const size_t yi = size_t(dv.ay_i.ktiles) * dv.ay_i.JQ * (fold_y ? 2 : 1) * 2 * 64 * 16;
    sc.fused_lds_bytes = sc.lds_bytes + size_t(16) * sc.ncy * sc.fused_mrow * 8;
    sc.fused_y_lds = sc.fused_lds_bytes + std::max(yf, yi) <= 160 * 1024 ? 1 : 0;
    if (sc.fused_y_lds) sc.fused_lds_bytes += std::max(yf, yi);
    sc.fuse_y = (!split && sc.ct == 1 && ((sc.mt == 2 && sc.ncls <= 2) || (sc.mt == 1 && sc.ncls == 4)) &&
                 sc.th <= 2 && sc.vec && dv.K[1] <= 32 &&
                 mcols <= 256 && sc.kyt <= (fold_y ? 1 : 2) && sc.fused_lds_bytes <= 160 * 1024)
                    ? 1
                    : 0;
  }
  // W1 leaves the workspace where the y contraction is always fused: with
  // N_t % 4 != 0 the plans have W1 whatever their schedule.
  const bool has_w1 = !sc.fuse_y || sc.nt % 4 != 0;
  dv.w1_bytes = has_w1 ? w1 : 0;
  dv.ws_bytes = dv.w1_bytes + w2;
  // At N_t % 4 != 0 the fused forward's masked tiles cost it more than the W1
  // traffic it saves: 8 channels, B = 3, 26 x 19 rows of 210 x 30 155 us, separate
  // 97; 12 of 45 x 129 rows of 26 x 30 113 and 74; 24, B = 2, 21 x 41 of 29 x 26 49
  // and 48.
  sc.fuse_yf = sc.fuse_y && !has_w1 ? 1 : 0;

  // ---- z-first rows ----
  // Taken where they need fewer matrix instructions than the t-first kernels;
  // the forward contracts y in the same launch under the fused forward's
  // conditions on y (also for K_t > 8, which the t-first fused kernel does not
  // cover), with the plane in `parts` where the workspace holds the parts.
  if (ZRowCfg z; z_first(sc, d->n_local[2] == d->n_global[2], &z)) {
    // The forward goes z first only where that takes fewer than even t-folded rows
    // would: between the two counts the rows t first, unfolded, were 5% faster (40
    // geometries), and z first the inverse.
    const int tcost = t_first_cost(sc);
    z.ncy = fold_y ? 2 : 1;
    z.kyt = fold_y ? dv.ay_f.kth : dv.ay_f.ktiles;
    const int mcols = static_cast<int>(nn_y);
    z.fused_mrow = static_cast<int>(round_up(mcols, 32)) + 16;
    z.fused_lds_bytes = size_t(dv.ay_f.ktiles) * dv.ay_f.JQ * 2 * 64 * 16 + size_t(16) * z.ncy * z.fused_mrow * 8 +
                        size_t(z.units) * z.ntl * 2 * 64 * 16;
    // Against four z classes and K_t > 8 (so more than 32 modes: two mode tiles, two
    // chains of which would not fit) the rows z first took 10 to 15% less time, but
    // their error was 3 to 13% larger forward and 2 to 6% inverse: t first, except at
    // N_t = 32, whose folded rows' error is as large.
    const bool precise = !(sc.ct == 2 && sc.ncls == 4 && !sc.tf);
    const bool fwd_better = precise && z_first_fwd_cost(z) < t_first_cost(folded);
    // Separate launches (where the plan has W1) stay where the fused kernel's two
    // waves per SIMD do not carry the row work: two mode tiles (28 x 24 x 86 x 32,
    // K_z 36: 86 us separate), or one t group (99 x 90 x 75 x 10: 289, fused 333);
    // with one tile and two groups fused was faster (32 x 128 x 128 x 32, K_z 16:
    // 355 and 287; 32 x 128 x 64 x 30: 206 and 176) unless the last group of 16 y
    // slots leaves over a quarter of the slots empty (of 90 random geometries the
    // 19 such were 11% faster separate, 18 x 18 x 187 x 28 54 and 71, the others 1%
    // slower); rows of four z classes stay fused there too, for its shorter z chains
    // (16 x 16 x 148 x 26: 2.0e-7, separate 2.2e-7, t first 2.0e-7).  With one t group and the y contraction in the t-first kernel's
    // reach, rows z first in separate launches were faster than t first fused (45
    // geometries of N_t 5 to 15: 1.56 times, 0.98 to 5.1).  A plan whose workspace
    // has no W1 (fused t-first kernels otherwise) stays fused.
    const int64_t slots = fold_y ? d->n_local[1] / 2 : d->n_local[1];
    const bool zty_covers = z.th == 2 ? z.ntl == 1 : z.mk == 1;  // (the instances there are)
    const bool fused = (flags & DTST_PLAN_SPLIT_SCHEDULE) == 0 && zty_covers && mcols <= 256 && dv.K[1] <= 32 &&
                       z.kyt <= (fold_y ? 1 : 2) && z.fused_lds_bytes <= 160 * 1024 &&
                       bc * d->n_local[0] < (1 << 24) &&
                       (!has_w1 || (z.ntl == 1 && z.th == 2 && (z.acc || slots * 4 >= dv.ay_f.JQ * 16 * 3)));
    if (fwd_better && fused) {
      z.fwd = 2;
      // A workgroup fills a CU (of 256): the parts that leave the fewest slot
      // groups on the busiest one, the fewest of those within 5%.
      const int64_t planes = std::max<int64_t>(bc, 1) * d->n_local[0], jq = dv.ay_f.JQ;
      int64_t best = 0;
      for (int64_t parts = 1; parts <= jq; ++parts) {
        const int64_t gpp = ceil_div(jq, parts);
        if ((parts - 1) * gpp >= jq || size_t(parts) * w2 > dv.ws_bytes) continue;
        const int64_t cost = ceil_div(planes * parts, 256) * gpp;
        if (best == 0 || cost * 20 < best * 19) {
          best = cost;
          z.parts = static_cast<int>(parts);
        }
      }
    } else if (fwd_better && has_w1) {
      z.fwd = 1;
    }
    z.ifused_lds_bytes = size_t(dv.ay_i.ktiles) * dv.ay_i.JQ * (fold_y ? 2 : 1) * 2 * 64 * 16 +
                         size_t(16) * z.ncy * z.fused_mrow * 8 + size_t(z.units) * z.ns * 64 * 8;
    if (precise && z_first_inv_cost(z) < tcost) {
      if ((flags & DTST_PLAN_SPLIT_SCHEDULE) == 0 && mcols <= 256 && z.fold && dv.ay_i.JQ == z.kyt &&
          z.kyt <= (fold_y ? 1 : 2) && z.ifused_lds_bytes <= 160 * 1024 && bc * d->n_local[0] < (1 << 24))
        z.inv = 2;
      else if (has_w1)
        z.inv = 1;
    }
    dv.zr = z;
  }

  // Separate x and y launches fold in four classes (k mod 4, which is the
  // position mod 4 when N % 4 == 0 and k_max is even) when every class fills
  // whole 16-mode tiles (K % 64 == 0) and the inverse's class sums take at
  // most two K steps (K <= 128): a quarter of the direct MFMA work instead of
  // a half.
  {
    auto four = [&](int dim) {
      const int64_t n = d->n_global[dim], k = dv.K[dim];
      return d->n_local[dim] == n && n % 4 == 0 && k % 64 == 0 && k <= 128;
    };
    if (four(1) && !sc.fuse_y) {
      dv.ay_f = axis(static_cast<int>(d->n_local[1]), static_cast<int>(dv.K[1]), nn_y, 3);
      dv.ay_i = axis(static_cast<int>(dv.K[1]), static_cast<int>(d->n_local[1]), nn_y, 4);
    }
    if (four(0)) {
      dv.ax_f = axis(static_cast<int>(d->n_local[0]), static_cast<int>(dv.K[0]), nn_x, 3);
      dv.ax_i = axis(static_cast<int>(dv.K[0]), static_cast<int>(d->n_local[0]), nn_x, 4);
    }
  }

  // the parts of a plane are further columns of the x contraction
  if (dv.zr.fwd == 2) {
    dv.ax_f = axis(static_cast<int>(d->n_local[0]) * dv.zr.parts, static_cast<int>(dv.K[0]), nn_x, dv.ax_f.fold);
    dv.ax_f.jdup = dv.zr.parts;
  }

  // Two-part (Re, Im) images: the inverse expansions of the expand kernel
  // (fold 2 or 4 within two K steps) and the y images the fused stream
  // kernels read; dtst_inverse_block expands y with the axis kernels even
  // where the plan fuses y into the stream kernels.
  auto expand_parts = [](AxisCfg& a) {
    if ((a.fold == 2 || a.fold == 4) && a.JQ <= 2) a.parts = 2;
  };
  expand_parts(dv.ax_i);
  expand_parts(dv.ay_i);
  dv.ay_b = dv.ay_i;
  if (dv.zr.fwd == 2 || (dv.zr.fwd == 0 && sc.fuse_yf)) dv.ay_f.parts = 2;
  if (dv.zr.inv == 2 || (dv.zr.inv == 0 && sc.fuse_y)) dv.ay_i.parts = 2;

  // ---- fused inverse z + t expansion and block epilogue ----
  // The same z + t expansion as the split inverse, with z folded into at
  // most two classes (a chunk of the kernel is one z tile of every class),
  // fed by the separate y expansion: dtst_inverse_block's workspace holds W1
  // then W2 even where the layer's own calls fuse y.  The plan flag
  // DTST_PLAN_UNFUSED_BLOCK keeps the inverse and the epilogue separate.
  {
    StreamCfg sb = sc;
    sb.tf = folded.tf;
    sb.ncls = fold && round_up(ceil_div(sc.kz, 2), 16) < round_up(sc.kz, 16) ? 2 : 1;
    sb.kcp = static_cast<int>(round_up(ceil_div(sc.kz, sb.ncls), 16));
    sb.mt = sb.kcp / 8;
    sb.zh = sb.nz / sb.ncls;
    sb.zt = static_cast<int>(ceil_div(sb.zh, 16));
    auto fits = [&] {
      sb.lds_bytes = size_t(sb.ncls) * sb.zt * z_blocks(sb) * 64 * 16;
      return sb.kcp <= 32 && block_zt_supported(sb, d->c_in, d->c_out);
    };
    sb.fuse_y = 0;
    bool fused = fits();
    // Folding t makes the z image half as large again.  Where only the unfolded
    // one leaves the kernel its LDS, it runs with t unfolded if its waves are
    // well filled: one 16-mode tile a class and N_t > 24 with up to 20 channels
    // (20 channels of 16 x 32 rows of 288 x 28, K_z 16: 340 us in two launches,
    // 235 fused; 8 x 32 rows of 388 x 28: 205, 183; of 386 x 28 in two classes, 16
    // channels: 153, 133), or one class and unconditional passes (32 channels of
    // 480 x 28: 410, 327).  Two launches, measured with t folded, were faster elsewhere (28
    // channels of 402 x 28: 304, 316; 16 of 347 x 20, two tiles: 105, 149; 32 of
    // 384 x 20, two classes: 256, 306).  N_t = 32 is always folded.
    const int64_t cb = std::max(d->c_in, d->c_out);
    const bool whole = d->c_in == d->c_out && (cb == 16 || cb == 20 || cb == 32) && sb.zh % 16 == 0;
    if (!fused && sb.tf && sb.nt != 32 && sb.mt == 2 && ((sb.nt > 24 && cb <= 20) || (whole && sb.ncls == 1))) {
      sb.tf = 0;
      fused = fits();
    }
    dv.sb = sb;
    dv.blk = (flags & DTST_PLAN_UNFUSED_BLOCK) == 0 && fused ? 1 : 0;
    // Row tasks instead of chunks for few input channels, where a chunk's
    // matrix tiles and waves would mostly idle (chunks -> row tasks, with the
    // x and y expansions: 5 channels of 3816 rows of 204 x 16: 545 -> 209 us;
    // 7 of 5940 of 103 x 32: 493 -> 374; 12 of 1232 of 114 x 8: 110 -> 83);
    // above that the bypass on the vector unit is the slower one (10 channels
    // of 2184 rows of 42 x 32: 110 -> 136; 16 of 558 of 137 x 8: 88 -> 108).
    // So they are for rows short for more than 8 output channels, N_z N_t below 40
    // sqrt(C_in C_out) (16 x 65 rows of 16 x 32, 8 -> 30 channels: 76 -> 156; 18
    // such of 294 random blocks: 0.42 to 1.05 of the chunks' rate, but for one of
    // 1.7; 8 or fewer: 26 x 8, 6 channels, 41 -> 28), or of two t groups and up to 40
    // z, 48 with two k_t tiles to expand (23 x 60 rows of 38 x 32, K_t 5, 5 -> 16, B =
    // 2: 175 -> 215; 8 x 72 of 47 x 32, K_t 9, 5 -> 12, B = 2: 0.81 of the chunks' rate;
    // 24 such blocks 0.67 to 1.34, mean 0.89; longer rows 0.8 to 2.6, mean 1.4).
    const int64_t row = int64_t(sc.nz) * sc.nt;
    const bool filled = d->c_out <= 8 || (row * row >= int64_t(1600) * d->c_in * d->c_out &&
                                          !(sc.th == 2 && sc.nz <= (sc.kt > 8 ? 48 : 40)));
    if (dv.blk && (d->c_in <= 8 || (d->c_in <= 12 && sc.th == 1)) && filled &&
        block_row_supported(dv.zr, d->c_in, d->c_out))
      dv.blk = 2;
    dv.blk_w1_bytes = dv.blk ? w1 : dv.w1_bytes;
    dv.blk_ws_bytes = dv.blk ? w1 + w2 : dv.ws_bytes;
  }


  // ---- image offsets (floats, 256-byte aligned) ----
  Images& im = dv.img;
  size_t off = 0;
  auto take = [&off](size_t n) {
    size_t o = off;
    off = round_up(off + n, 64);
    return o;
  };
  const size_t t_img = size_t(sc.th) * 4 * sc.ct * 64;
  const size_t z_img = size_t(sc.ncls) * sc.zt * z_blocks(sc) * 64 * 4;
  if (!dv.zr.fwd) {  // the z-first kernels have images of their own
    im.t_fwd = take(t_img);
    im.t_fwd_adjoint_of_inverse = take(t_img);
    im.z_fwd = take(z_img);
  }
  if (!dv.zr.inv) {
    im.t_inv = take(t_img);
    im.t_inv_adjoint_of_forward = take(t_img);
    im.z_inv = take(z_img);
  }
  auto axis_img = [](const AxisCfg& a) {
    return size_t(a.ktiles) * a.JQ * axis_image_classes(a) * a.parts * 64 * 4;
  };
  im.y_fwd = take(axis_img(dv.ay_f));
  im.x_fwd = take(axis_img(dv.ax_f));
  im.y_inv = take(axis_img(dv.ay_i));
  im.x_inv = take(axis_img(dv.ax_i));
  im.y_blk = sc.fuse_y || dv.zr.inv == 2 ? take(axis_img(dv.ay_b)) : im.y_inv;
  im.z_blk = take(size_t(dv.sb.ncls) * dv.sb.zt * z_blocks(dv.sb) * 64 * 4);
  im.t_blk = take(t_img);
  if (dv.zr.fwd || dv.zr.inv || dv.blk == 2) {
    const ZRowCfg& z = dv.zr;
    im.zr_z_fwd = take(size_t(z.units) * z.ntl * 2 * 64 * 4);
    im.zr_phase = take(size_t(z.ntl) * 64 * 4);
    im.zr_t_fwd = take(size_t(z.th) * 4 * z.mk * 64);
    im.zr_t_fwd_adjoint_of_inverse = take(size_t(z.th) * 4 * z.mk * 64);
    im.zr_z_inv = take(size_t(z.units) * z.ns * 64 * 2);
    im.zr_phase_inv = take(ceil_div(z.ns, 4) * 64 * 4);
    im.zr_phase_col = take(size_t(nn_y) * 4);
    im.zr_t_inv = take(size_t(z.th) * 4 * z.mk * 64);
    im.zr_t_inv_adjoint_of_forward = take(size_t(z.th) * 4 * z.mk * 64);
  }
  im.total = off;

  *out = dv;
  return DTST_OK;
}

namespace {

// Complex basis value of dimension dim at (mode position p, local index j).
inline void bval(const dtst_desc& d, int dim, int64_t p, int64_t j, double* re, double* im) {
  twiddle(d.n_global[dim], retained_index(d, dim, p), d.offset[dim] + j, re, im);
}

// First t of the 16-byte chunk that starts at t0 of an extent of `lim`
// values: a chunk that would run past the end starts at the last four values
// (t_start of the kernels; extents below 4 have no such chunks).
int t_chunk_start(int t0, int lim) { return lim >= 4 ? std::min(t0, lim - 4) : t0; }

// t image of the forward streaming kernel (B operand of the first MFMA):
// entry ((h*4 + j)*CT + ct)*64 + lane holds Bt'[t][c] with t = 16h + 4g + j
// (the chunk's start plus j where the chunk starts early; zero for the values
// an earlier chunk also holds),
// c = 16ct + m (m = lane & 15, g = lane >> 4); c < 8CT is Re B_t[kt=c][t],
// otherwise Im B_t[kt = c - 8CT][t]; times scale(kt).  t-folded (tf), only
// t < N_t/2 is filled and column m of tile ct is k_t = 2(m & 7) + ct, Re for
// m < 8 and Im otherwise (the kernel forms x(t) +- x(t + N_t/2)).
void t_forward_image(const Derived& dv, bool adjoint_of_inverse, float* dst) {
  const StreamCfg& sc = dv.sc;
  const dtst_desc& d = dv.d;
  const int ktp = 8 * sc.ct;
  const double ntot = double(d.n_global[0]) * d.n_global[1] * d.n_global[2] * d.n_global[3];
  const int tlim = sc.tf ? sc.nt / 2 : sc.nt;
  for (int h = 0; h < sc.th; ++h)
    for (int j = 0; j < 4; ++j)
      for (int ct = 0; ct < sc.ct; ++ct)
        for (int lane = 0; lane < 64; ++lane) {
          const int m = lane & 15, g = lane >> 4;
          const int t0 = 16 * h + 4 * g, t = t_chunk_start(t0, tlim) + j;
          const int c = 16 * ct + m;
          const bool is_re = sc.tf ? m < 8 : c < ktp;
          const int kt = sc.tf ? 2 * (m & 7) + ct : (is_re ? c : c - ktp);
          double v = 0.0;
          if (t >= t0 && t < tlim && kt < sc.kt) {
            double re, im;
            bval(d, 3, kt, t, &re, &im);
            double s = adjoint_of_inverse ? half_weight(d.n_global[3], kt) / ntot : 1.0;
            v = s * (is_re ? re : im);
          }
          dst[((h * 4 + j) * sc.ct + ct) * 64 + lane] = static_cast<float>(v);
        }
}

// z image of the forward streaming kernel (A operand of the second MFMA,
// staged in LDS): float4 entry ((cl*ZT + zt)*MT + mt)*64 + lane, component
// i, holds row r = 16mt + m at z = 16zt + 4g + i of class cl; rows [0, KCP)
// are Re B_z[p][z], rows [KCP, 2KCP) are Im B_z[p][z], p = s*NCLS + cl.
// With MT = 1 (KCP = 8) row r holds slot s = 2(r >> 2) + ((r >> 1) & 1),
// Re for even r and Im for odd r, so that the products with Re B_z and Im B_z
// of one slot land in accumulator registers 2j and 2j + 1 of one lane.
// With t folded, the blocks hold the three-product operands of B = Br +
// i Bi: blocks mr < mt / 2 Br, the next mt / 2 blocks Bi - Br, the last
// mt / 2 Br + Bi, each for the rows (slots) of block mr.
void z_forward_image(const Derived& dv, float* dst) {
  const StreamCfg& sc = dv.sc;
  const dtst_desc& d = dv.d;
  const int nb = z_blocks(sc);
  for (int cl = 0; cl < sc.ncls; ++cl)
    for (int zt = 0; zt < sc.zt; ++zt)
      for (int mb = 0; mb < nb; ++mb)
        for (int lane = 0; lane < 64; ++lane)
          for (int i = 0; i < 4; ++i) {
            const int m = lane & 15, g = lane >> 4;
            const int z = 16 * zt + 4 * g + i;
            double v = 0.0;
            if (sc.tf) {
              const int half = sc.mt / 2, kind = mb / half, mr = mb % half;
              const int p = (16 * mr + m) * sc.ncls + cl;
              if (p < sc.kz && z < sc.zh) {
                double re, im;
                bval(d, 2, p, z, &re, &im);
                v = kind == 0 ? re : (kind == 1 ? im - re : re + im);
              }
            } else {
              const int row = 16 * mb + m;
              const bool is_re = sc.mt == 1 ? (row & 1) == 0 : row < sc.kcp;
              const int s = sc.mt == 1 ? 2 * (row >> 2) + ((row >> 1) & 1) : (is_re ? row : row - sc.kcp);
              const int p = s * sc.ncls + cl;
              if (p < sc.kz && z < sc.zh) {
                double re, im;
                bval(d, 2, p, z, &re, &im);
                v = is_re ? re : im;
              }
            }
            dst[((((size_t)cl * sc.zt + zt) * nb + mb) * 64 + lane) * 4 + i] = static_cast<float>(v);
          }
}

// t image of the inverse streaming kernel (A operand of its second MFMA):
// entry ((mt*CT + ct)*4 + i)*64 + lane holds A[t][c] with t = 16mt + m (rows
// 4q..4q+3 of a chunk that starts early, or past the end, are the last four t
// again: every store of such a chunk writes values of the row),
// c = 16ct + 4g + i: Re C_t[t][kt] for c < 8CT, -Im C_t[t][kt] otherwise,
// where C_t[t][kt] = scale(kt) conj(B_t[kt][t]).  t-folded (tf), only
// t < N_t/2 is filled and K index 4g + i of tile ct is
// k_t = 2(2g + (i & 1)) + (i >> 1), Re for ct = 0 and Im for ct = 1 (the
// rows of the three-product z expansion of the t-folded inverse).  With the
// four-class z fold of one column tile (MT = 1), K index 4g + i is
// k_t = 2g + (i & 1), Re for i < 2 and Im otherwise (Re and Im of one k_t in
// registers i and i + 2 of one lane of the z expansion).
void t_inverse_image(const Derived& dv, bool is_inverse, float* dst) {
  const StreamCfg& sc = dv.sc;
  const dtst_desc& d = dv.d;
  const int ktp = 8 * sc.ct;
  const double ntot = double(d.n_global[0]) * d.n_global[1] * d.n_global[2] * d.n_global[3];
  const int tlim = sc.tf ? sc.nt / 2 : sc.nt;
  for (int mt = 0; mt < sc.th; ++mt)
    for (int ct = 0; ct < sc.ct; ++ct)
      for (int i = 0; i < 4; ++i)
        for (int lane = 0; lane < 64; ++lane) {
          const int m = lane & 15, g = lane >> 4;
          const int t = t_chunk_start(16 * mt + (m & ~3), tlim) + (m & 3);
          const int c = 16 * ct + 4 * g + i;
          // t-folded: tile ct holds part ct (0 Re, 1 -Im) of k_t = 2(2g + (i & 1)) + (i >> 1)
          const bool is_re = sc.tf ? ct == 0 : (sc.mt == 1 ? i < 2 : c < ktp);
          const int kt = sc.tf ? 2 * (2 * g + (i & 1)) + (i >> 1)
                               : (sc.mt == 1 ? 2 * g + (i & 1) : (is_re ? c : c - ktp));
          double v = 0.0;
          if (t < tlim && kt < sc.kt) {
            double re, im;
            bval(d, 3, kt, t, &re, &im);  // B_t = re + i im; conj(B_t) = re - i im
            const double s = is_inverse ? half_weight(d.n_global[3], kt) / ntot : 1.0;
            v = is_re ? s * re : s * im;  // -Im(s conj B_t) = s * im
          }
          dst[((mt * sc.ct + ct) * 4 + i) * 64 + lane] = static_cast<float>(v);
        }
}

// z image of the inverse streaming kernel (B operand of its first MFMA,
// staged in LDS): float4 entry ((cl*ZT + zt)*MT + q)*64 + lane, component
// i, holds row kz' = 16q + 4g + i at z = 16zt + m: Re C_z[z][p] for
// kz' < KCP and Im C_z[z][p] otherwise, C_z[z][p] = conj(B_z[p][z]).
// With MT = 1 (KCP = 8) row kz' holds slot s = 2g + (i >> 1), Re for even i
// and Im for odd i.
// With t folded, the blocks hold the three-product operands of C_z = Cr +
// i Ci (Cr = Re B, Ci = -Im B): blocks qh < mt / 2 Cr, the next mt / 2
// blocks Ci - Cr, the last mt / 2 Cr + Ci, each for the K entries of block qh.
void z_inverse_image(const Derived& dv, float* dst) {
  const StreamCfg& sc = dv.sc;
  const dtst_desc& d = dv.d;
  const int nb = z_blocks(sc);
  for (int cl = 0; cl < sc.ncls; ++cl)
    for (int zt = 0; zt < sc.zt; ++zt)
      for (int q = 0; q < nb; ++q)
        for (int lane = 0; lane < 64; ++lane)
          for (int i = 0; i < 4; ++i) {
            const int m = lane & 15, g = lane >> 4;
            const int z = 16 * zt + m;
            if (sc.tf) {
              const int half = sc.mt / 2, kind = q / half, qh = q % half;
              const int p = (16 * qh + 4 * g + i) * sc.ncls + cl;
              double v = 0.0;
              if (p < sc.kz && z < sc.zh) {
                double re, im;
                bval(d, 2, p, z, &re, &im);
                const double cr = re, ci = -im;
                v = kind == 0 ? cr : (kind == 1 ? ci - cr : cr + ci);
              }
              dst[((((size_t)cl * sc.zt + zt) * nb + q) * 64 + lane) * 4 + i] = static_cast<float>(v);
              continue;
            }
            const int kzp = 16 * q + 4 * g + i;
            const bool is_re = sc.mt == 1 ? (i & 1) == 0 : kzp < sc.kcp;
            const int s = sc.mt == 1 ? 2 * g + (i >> 1) : (is_re ? kzp : kzp - sc.kcp);
            const int p = s * sc.ncls + cl;
            double v = 0.0;
            if (p < sc.kz && z < sc.zh) {
              double re, im;
              bval(d, 2, p, z, &re, &im);
              v = is_re ? re : -im;
            }
            dst[((((size_t)cl * sc.zt + zt) * nb + q) * 64 + lane) * 4 + i] = static_cast<float>(v);
          }
}

// Images of the z-first row kernels (k_zrow.hip).  Angles are taken at z + 1/2
// where z folds (2 pi k (2z + 1) / 2N_z), else at the global z.
//   forward z: float4 entry ((u*NT + n)*2 + part)*64 + lane, component st: Re
//     (part 0) or Im of exp(-i angle) of mode k = 16n + m at position 16u + 4st + g;
//   phases: float4 entry n*64 + lane: exp(i pi k / N_z) of k = 16n + m (forward)
//     or k = 16n + 4(m & 3) + (m >> 2) (inverse) where z folds, else 1; real and
//     imaginary part, then what rounding them to 32 bits left out;
//   column phases: the same for each column of K_z K_t (k of its z mode, signed);
//   forward t: entry ((4j + i)*MK + kk)*64 + lane: K index g of step (j, i) is
//     t = TH (4g + i) + j (lanes past the extent hold its last TH values
//     again, with zeros), rows M = 4g' + i': with MK = 2 tile kk is part kk of B_t at
//     k_t = 8(i' >> 1) + 2g' + (i' & 1); with MK = 1 part i' >> 1 at
//     k_t = 2g' + (i' & 1);
//   inverse z: float2 entry (zt*NS + s)*64 + lane: cosine and sine of mode
//     k = 4s + g at position 16zt + m;
//   inverse t: entry ((h*KG + kg)*2 + e)*64 + lane: C_t = scale conj(B_t) at
//     k_t = 4kg + g and the t of row m of group h, part e.
void zrow_images(const Derived& dv, float* base) {
  const StreamCfg& sc = dv.sc;
  const ZRowCfg& z = dv.zr;
  const dtst_desc& d = dv.d;
  const Images& im = dv.img;
  const double ntot = double(d.n_global[0]) * d.n_global[1] * d.n_global[2] * d.n_global[3];
  const int64_t N = d.n_global[2];
  const int kmax = sc.kz / 2, kg_n = 2 * z.mk;
  double re, im_;
  // exp(-i angle) of mode k at position pos
  auto zval = [&](int k, int pos) {
    if (k > kmax || pos >= z.np) re = im_ = 0.0;
    else if (z.fold) twiddle(2 * N, k, 2 * int64_t(pos) + 1, &re, &im_);
    else twiddle(N, k, d.offset[2] + pos, &re, &im_);
  };
  auto put_phase = [&](size_t at, int k) {
    re = 1.0;
    im_ = 0.0;
    if (z.fold) twiddle(2 * N, k, 1, &re, &im_);  // exp(-i pi k / N)
    base[at] = static_cast<float>(re);
    base[at + 1] = static_cast<float>(-im_);
    base[at + 2] = static_cast<float>(re - base[at]);
    base[at + 3] = static_cast<float>(-im_ - base[at + 1]);
  };
  for (int c = 0; c < sc.kz * sc.kt; ++c) {
    const int p = c / sc.kt, k = p < kmax ? p : 2 * kmax - p;  // |k| of the column
    float* e = base + im.zr_phase_col + size_t(c) * 4;
    put_phase(im.zr_phase_col + size_t(c) * 4, k);
    if (p >= kmax) e[1] = -e[1], e[3] = -e[3];
  }
  for (int lane = 0; lane < 64; ++lane) {
    const int m = lane & 15, g = lane >> 4;
    for (int n = 0; n < z.ntl; ++n) {
      put_phase(im.zr_phase + size_t(n * 64 + lane) * 4, 16 * n + m);
      for (int u = 0; u < z.units; ++u)
        for (int st = 0; st < 4; ++st) {
          zval(16 * n + m, 16 * u + 4 * st + g);
          float* e = base + im.zr_z_fwd + ((size_t(u * z.ntl + n) * 2) * 64 + lane) * 4 + st;
          e[0] = static_cast<float>(re);
          e[64 * 4] = static_cast<float>(im_);
        }
    }
    for (int n = 0; n < ceil_div(z.ns, 4); ++n)
      put_phase(im.zr_phase_inv + size_t(n * 64 + lane) * 4, 16 * n + 4 * (m & 3) + (m >> 2));
    for (int zt = 0; zt < z.units; ++zt)
      for (int s = 0; s < z.ns; ++s) {
        zval(4 * s + g, 16 * zt + m);
        float* e = base + im.zr_z_inv + (size_t(zt * z.ns + s) * 64 + lane) * 2;
        e[0] = static_cast<float>(re);
        e[1] = static_cast<float>(-im_);
      }
    for (int j = 0; j < z.th; ++j)
      for (int i = 0; i < 4; ++i)
        for (int kk = 0; kk < z.mk; ++kk) {
          // lane 4g + i of a row reads t0 .. t0 + TH - 1
          const int first = z.th * (4 * g + i), t = std::min(first, sc.nt - z.th) + j;
          const int gr = m >> 2, ir = m & 3;
          const bool is_re = z.mk == 2 ? kk == 0 : ir < 2;
          const int kt = z.mk == 2 ? 8 * (ir >> 1) + 2 * gr + (ir & 1) : 2 * gr + (ir & 1);
          double v = 0.0, w = 0.0;
          if (kt < sc.kt && t >= first) {
            bval(d, 3, kt, t, &re, &im_);
            v = is_re ? re : im_;
            w = v * (half_weight(d.n_global[3], kt) / ntot);
          }
          const size_t o = size_t((4 * j + i) * z.mk + kk) * 64 + lane;
          base[im.zr_t_fwd + o] = static_cast<float>(v);
          base[im.zr_t_fwd_adjoint_of_inverse + o] = static_cast<float>(w);
        }
    for (int h = 0; h < z.th; ++h)
      for (int kg = 0; kg < kg_n; ++kg)
        for (int e = 0; e < 2; ++e) {
          const int t = t_chunk_start(16 * h + (m & ~3), sc.nt) + (m & 3), kt = 4 * kg + g;
          double v = 0.0, w = 0.0;
          if (kt < sc.kt) {
            bval(d, 3, kt, t, &re, &im_);
            v = e == 0 ? re : -im_;
            w = v * (half_weight(d.n_global[3], kt) / ntot);
          }
          const size_t o = size_t((h * kg_n + kg) * 2 + e) * 64 + lane;
          base[im.zr_t_inv + o] = static_cast<float>(w);
          base[im.zr_t_inv_adjoint_of_forward + o] = static_cast<float>(v);
        }
  }
}

// Axis image, float4 entries indexed by lane (m = lane & 15, g = lane >> 4)
// and component i.  With 3 parts (the axis kernels) part 0 holds Br, part 1
// Bi - Br, part 2 Br + Bi of the basis value Br + i Bi; with 2 parts (the y
// images of the fused stream kernels) part 0 Re, part 1 Im.  Entry layouts
// below with 2 parts; 3 parts stride the same way.
//   fold 0: entry ((kt*JQ + q)*2 + part)*64 + lane = basis[k][j],
//           k = 16kt + m, j = 16q + 4g + i.
//   fold 1: same entry layout; tile kt holds parity class c = (kt >= kth),
//           mode p = 2 (16 (kt - c kth) + m) + c, column j = 16q + 4g + i < J/2.
//   fold 2: entry (((kt*JQ + q)*2 + c)*2 + part)*64 + lane = basis[y][p],
//           y = 16kt + m < KO/2, mode p = 2 (16q + 4g + i) + c.
//   fold 3: fold 0's entry layout; tile kt holds class c = kt mod 4, mode
//           p = 4 (16 (kt / 4) + m) + c, column j = 16q + 4g + i < J/4.
//   fold 4: entry (((kt*JQ + q)*4 + c)*2 + part)*64 + lane = basis[y][p],
//           y = 16kt + m < KO/4, mode p = 4 (16q + 4g + i) + c.
// forward: basis[k][j] = B_dim[k][j / jdup]; inverse: basis[y][p] = conj(B_dim[p][y]).
void axis_image(const Derived& dv, const AxisCfg& a, int dim, bool inverse, float* dst) {
  const dtst_desc& d = dv.d;
  const int ncls = axis_image_classes(a);
  for (int kt = 0; kt < a.ktiles; ++kt)
    for (int q = 0; q < a.JQ; ++q)
      for (int c = 0; c < ncls; ++c)
        for (int part = 0; part < a.parts; ++part)
          for (int lane = 0; lane < 64; ++lane)
            for (int i = 0; i < 4; ++i) {
              const int m = lane & 15, g = lane >> 4;
              int k, j;  // output row, contracted index (before the basis orientation)
              bool ok;
              if (a.fold == 1) {
                const int cls = kt >= a.kth ? 1 : 0;
                k = 2 * (16 * (kt - cls * a.kth) + m) + cls;
                j = 16 * q + 4 * g + i;
                ok = k < a.KO && j < a.J / 2;
              } else if (a.fold == 2) {
                k = 16 * kt + m;
                j = 2 * (16 * q + 4 * g + i) + c;
                ok = k < a.KO / 2 && j < a.J;
              } else if (a.fold == 3) {
                k = 4 * (16 * (kt >> 2) + m) + (kt & 3);
                j = 16 * q + 4 * g + i;
                ok = k < a.KO && j < a.J / 4;
              } else if (a.fold == 4) {
                k = 16 * kt + m;
                j = 4 * (16 * q + 4 * g + i) + c;
                ok = k < a.KO / 4 && j < a.J;
              } else {
                k = 16 * kt + m;
                j = 16 * q + 4 * g + i;
                ok = k < a.KO && j < a.J;
              }
              double v = 0.0;
              if (ok) {
                double re, im;
                if (inverse) {
                  bval(d, dim, j, k, &re, &im);
                  im = -im;
                } else {
                  bval(d, dim, k, j / a.jdup, &re, &im);
                }
                if (a.parts == 3) v = part == 0 ? re : (part == 1 ? im - re : re + im);
                else v = part == 0 ? re : im;
              }
              dst[(((((size_t)kt * a.JQ + q) * ncls + c) * a.parts + part) * 64 + lane) * 4 + i] =
                  static_cast<float>(v);
            }
}

}  // namespace

void build_images(const Derived& dv, std::vector<float>* blob) {
  TwiddleTables tables;
  struct Use {
    explicit Use(TwiddleTables* t) { g_twiddles = t; }
    ~Use() { g_twiddles = nullptr; }
  } use(&tables);
  blob->assign(dv.img.total, 0.0f);
  float* b = blob->data();
  if (!dv.zr.fwd) {
    t_forward_image(dv, false, b + dv.img.t_fwd);
    t_forward_image(dv, true, b + dv.img.t_fwd_adjoint_of_inverse);
    z_forward_image(dv, b + dv.img.z_fwd);
  }
  if (!dv.zr.inv) {
    t_inverse_image(dv, true, b + dv.img.t_inv);
    t_inverse_image(dv, false, b + dv.img.t_inv_adjoint_of_forward);
    z_inverse_image(dv, b + dv.img.z_inv);
  }
  if (dv.zr.fwd || dv.zr.inv || dv.blk == 2) zrow_images(dv, b);
  axis_image(dv, dv.ay_f, 1, false, b + dv.img.y_fwd);
  axis_image(dv, dv.ax_f, 0, false, b + dv.img.x_fwd);
  axis_image(dv, dv.ay_i, 1, true, b + dv.img.y_inv);
  axis_image(dv, dv.ax_i, 0, true, b + dv.img.x_inv);
  if (dv.img.y_blk != dv.img.y_inv) axis_image(dv, dv.ay_b, 1, true, b + dv.img.y_blk);
  // the fused inverse + block epilogue's z and t images: those of the
  // inverse for its own z configuration
  Derived db = dv;
  db.sc = dv.sb;
  z_inverse_image(db, b + dv.img.z_blk);
  t_inverse_image(db, true, b + dv.img.t_blk);
}

void plain_basis(const dtst_desc& d, int dim, int kind, float* out) {
  const int64_t K = dim < 3 ? 2 * int64_t(d.kmax[dim]) : d.kt;
  const int64_t n = d.n_local[dim];
  for (int64_t p = 0; p < K; ++p)
    for (int64_t j = 0; j < n; ++j) {
      double re, im;
      bval(d, dim, p, j, &re, &im);
      out[(p * n + j) * 2 + 0] = static_cast<float>(re);
      out[(p * n + j) * 2 + 1] = static_cast<float>(kind == 1 ? -im : im);
    }
}

}  // namespace dtst
