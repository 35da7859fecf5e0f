// Launcher of the fused inverse z + t expansion and block epilogue, and its
// instances with one column tile (K_t <= 8) and N_t != 32.  The kernel is in block_zt.h.
#include "block_zt.h"

namespace dtst {

// Instances of the other sources.
const void* block_zt_kernel1(int mt, int ncls, int kio);
const void* block_zt_kernel1s(int zp, int mt, int ncls, int kio);
const void* block_zt_kernel2(int th, int t32, int zp, int mt, int ncls, int kio);
const void* block_zt_kernel2f(int t32, int mt, int ncls, int kio);

namespace {

// float4 of a row's spectrum per thread for each (KI, OT) class.
constexpr int kSpf[3] = {4, 5, 8};

// (KI, OT) class of a channel count: 0 up to 16, 1 up to 20, 2 up to 32.
int kio_of(int64_t ci, int64_t co) {
  const int64_t c = ci > co ? ci : co;
  return c <= 16 ? 0 : (c <= 20 ? 1 : 2);
}

size_t lds_bytes(const StreamCfg& c, int64_t ci, int64_t co, int zp) {
  // chunk buffers of 16 channels where the instance makes two output passes
  const int64_t cb = kio_of(ci, co) == 2 ? 16 : co;
  return size_t(c.ncls) * c.zt * (c.tf ? 3 * c.mt / 2 : c.mt) * 64 * 16 + size_t(co) * c.kz * c.kt * 8 +
         2 * size_t(cb) * 16 * zp * c.nt * sizeof(float);
}

// z tiles per chunk.  More of them fill the 8 waves with points (16 ZP N_t <=
// 512) and halve the barriers, but the last chunk of a row then runs empty tiles,
// and channels above 20 make two passes a chunk as it is.  Against one tile, over
// 220 random blocks of one z class: N_t > 8, two tiles, an even number of tiles a
// row and up to 20 channels 1.00 to 1.10 times (22 x 16, 14: 0.93; 76 x 12, 16:
// 1.09), other rows 0.77 to 1.02 (78 x 236 rows of 35 x 12, 14 channels: 0.90;
// 66 x 26 of 101 x 16, 24: 0.89).  N_t <= 8, two: 1.0 to 1.36 (16 channels of 18 x 31
// rows of 137 x 8: 1.16), three tiles a row 0.78 to 1.06.  Four: above two only at N_t <= 6
// with up to 20 channels and chunks nearly full (40 x 48 rows of 111 x 4: 1.26,
// four 1.54; 60 x 6: 1.32, 1.39; 119 x 8: 1.24, 1.13).  One with two t groups, and
// with two z classes (the runs' expansions kept for the second class spilled: 28
// channels of 981 rows of 46 x 16 137 -> 147 us).
int z_tiles(const StreamCfg& c, int64_t ci, int64_t co) {
  if (c.th == 2 || c.nt > 16 || c.ncls == 2) return 1;
  const bool few = kio_of(ci, co) < 2;
  int zp = 1;
  if (c.nt > 8) {
    if (few && c.zt % 2 == 0) zp = 2;
  } else if (c.zt != 3) {
    zp = c.nt <= 6 && few && (c.zt + 1) % 4 <= 1 ? 4 : 2;
  }
  while (zp > 1 && (zp > c.zt || lds_bytes(c, ci, co, zp) > 160 * 1024)) zp /= 2;
  return zp;
}

const void* pick_blk(const StreamCfg& c, int64_t ci, int64_t co) {
  const int kio = kio_of(ci, co), zp = z_tiles(c, ci, co);
  const int t32 = c.nt == 32 ? 1 : 0;
  if (c.tf) return block_zt_kernel2f(t32, c.mt, c.ncls, kio);
  if (c.ct == 2) return block_zt_kernel2(c.th, t32, zp, c.mt, c.ncls, kio);
  if (c.th == 1) return block_zt_kernel1s(zp, c.mt, c.ncls, kio);
  return t32 ? block_zt_kernel1(c.mt, c.ncls, kio) : pick_mn<1, 2, 0, 0>(c.mt, c.ncls, kio);
}

}  // namespace

size_t block_zt_lds_bytes(const StreamCfg& c, int64_t ci, int64_t co) {
  return lds_bytes(c, ci, co, z_tiles(c, ci, co));
}

// N_t even, and N_z N_t / (z classes) a multiple of 4, which keeps every
// chunk, and the points of a ragged last one, in whole aligned groups of four.
// (Odd N_t keeps the two launches.)
bool block_zt_supported(const StreamCfg& c, int64_t ci, int64_t co) {
  if (!(c.vec && c.nt % 2 == 0 && (int64_t(c.zh) * c.nt) % 4 == 0 && c.th <= 2 && c.ncls <= 2 &&
        (c.mt == 2 || c.mt == 4) && (!c.tf || (c.ct == 2 && c.th == 2)) && ci <= 32 && co <= 32 && (c.kz * c.kt) % 2 == 0))
    return false;
  const int64_t n4 = co * c.kz * c.kt / 2;
  return n4 <= int64_t(64) * kBlkWaves * kSpf[kio_of(ci, co)] && block_zt_lds_bytes(c, ci, co) <= 160 * 1024;
}

int prepare_block_zt(const StreamCfg& c, int64_t ci, int64_t co, int* grid) {
  const void* fn = pick_blk(c, ci, co);
  const size_t lds = block_zt_lds_bytes(c, ci, co);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0, per_cu = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * kBlkWaves, lds)) != hipSuccess) return e;
  if (per_cu <= 0) return hipErrorInvalidConfiguration;
  *grid = cus * per_cu;
  return hipSuccess;
}

int launch_inv_zt_block(const StreamCfg& c, int grid_resident, const void* in, const float* x, const float* w,
                        float* y, int64_t batch, int64_t nxy, int64_t ci, int64_t co, const float* timg,
                        const float* zimg, void* stream) {
  const int64_t rows = batch * nxy;
  if (rows <= 0) return hipSuccess;
  if (!block_zt_supported(c, ci, co) || grid_resident <= 0) return hipErrorInvalidConfiguration;
  StreamArgs a;
  a.rows = rows;
  a.nt = c.nt;
  a.nz = c.nz;
  a.kt = c.kt;
  a.kz = c.kz;
  a.zh = c.zh;
  a.zt = c.zt;
  a.vec = c.vec;
  a.full = 0;
  BlockArgs ba;
  ba.rows = rows;
  ba.xy = nxy;
  ba.ci = static_cast<int>(ci);
  ba.co = static_cast<int>(co);
  ba.ostride = 16 * z_tiles(c, ci, co) * c.nt;
  if (c.nt > 4 * kBlkWaves) return hipErrorInvalidConfiguration;  // one 64-point group per wave
  const int64_t grid = rows < grid_resident ? rows : grid_resident;
  const float2* in2 = static_cast<const float2*>(in);
  const float4* zimg4 = reinterpret_cast<const float4*>(zimg);
  void* args[] = {&in2, &x, &w, &y, &timg, &zimg4, &a, &ba};
  return hipLaunchKernel(pick_blk(c, ci, co), dim3(static_cast<unsigned>(grid)), dim3(64 * kBlkWaves), args,
                         block_zt_lds_bytes(c, ci, co), static_cast<hipStream_t>(stream));
}

}  // namespace dtst
