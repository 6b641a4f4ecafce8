// Large-M W4A8 GEMM: tile planning, the per-channel kernel instances and the
// launch.  The kernel template is in largem_kernel.h; the group-scale
// instances are built in gemm_largem_group.hip.
#include <cstdio>

#include "largem_kernel.h"

namespace w4a8 {

namespace {

LargeMKernelFn channel_kernel(int cfg, bool swiglu) {
  if (swiglu) {
    switch (cfg) {
      case 1: return menu_kernel<1, false, true>();
      case 3: return menu_kernel<3, false, true>();
      default: return nullptr;
    }
  }
  switch (cfg) {
    case 0: return menu_kernel<0, false>();
    case 1: return menu_kernel<1, false>();
    case 2: return menu_kernel<2, false>();
    case kMenuKSplit: return menu_kernel<kMenuKSplit, false>();
    default: return nullptr;
  }
}

}  // namespace

// Gated plans (swiglu) take the tiles whose waves hold an even number of
// blocks (gate and up halves): a tile covers BN / 2 output columns.
LargeMPlan plan_largem(int M, int N, int K, bool group, bool swiglu) {
  LargeMPlan p{};
  p.group = group;
  p.swiglu = swiglu;
  double best = -1.0;
  for (int c = 0; c < kMenuSize && (!group || swiglu); ++c) {  // plain group scales choose below
    const TileCfg& t = kMenu[c];
    if (group && !t.group_ok) continue;
    if (t.ks > 1) continue;  // the k-split form replaces entry 2 below
    if (swiglu ? !t.gated_ok : !t.plain_ok) continue;
    const int BM = 32 * t.WM * t.GM, BN = 32 * t.WN * t.GN;
    const int tm = (M + BM - 1) / BM, tn = swiglu ? (N / 2 + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
    const int64_t tiles = (int64_t)tm * tn;
    const int64_t rounds = (tiles + 255) / 256;
    const double eff = (double)M * N / ((double)rounds * 256.0 * BM * BN);
    const double score = eff * t.quality;
    if (score > best + 1e-9) {
      best = score;
      p.cfg = c;
      p.BM = BM;
      p.BN = BN;
      p.threads = 64 * t.GM * t.GN * t.ks;
      p.tiles_m = tm;
      p.tiles_n = tn;
      p.tiles = tiles;
    }
  }
  // Plain group scales choose between the 128 x 128 and the 64 x 64 tile by
  // the time of the fullest CU, in us for 32 steps (K = 4096) beyond what
  // every call pays: a lone 128 x 128 tile 19.8 and one of several 16 (two
  // share the CU), a lone 64 x 64 tile 6.4 (its k-split form) and one of
  // several 5.5.  Fitted to a sweep of both over M = 80 .. 2048 and
  // N = 1536 .. 24576; at the turns, 128 x 128 against 64 x 64 in us:
  // qkv M = 768 34.3 / 30.4 (2 tiles a CU against 5), M = 1024 34.1 / 39.5
  // (2, 6); gate+up M = 320 50.8 / 47.7 (3, 8), M = 384 51.0 / 54.2 (3, 9);
  // o M = 768 23.6 / 20.6 (1, 3), M = 1024 24.1 / 28.1 (1, 4).  Both sides
  // scale with K alike: N = 4096, K = 1024 M = 512 8.9 / 6.3, M = 777 9.4 /
  // 10.3, K = 12288 M = 512 62.8 / 42.4, M = 777 60.7 / 77.4.
  if (group && !swiglu) {
    auto tiles_of = [&](int B) { return (int64_t)((M + B - 1) / B) * ((N + B - 1) / B); };
    auto cost = [](int64_t tiles, double lone, double each) {
      const double n = (double)((tiles + 255) / 256);
      return n <= 1 ? lone : n * each;
    };
    p.cfg = cost(tiles_of(128), 19.8, 16.0) < cost(tiles_of(64), 6.4, 5.5) ? 1 : 2;
    const int B = p.cfg == 1 ? 128 : 64;
    p.BM = p.BN = B;
    p.threads = 256;
    p.tiles_m = (M + B - 1) / B;
    p.tiles_n = (N + B - 1) / B;
    p.tiles = tiles_of(B);
  }
  // 64 x 64 tiles that fill at most one round: two k groups per tile
  // (measured at M = 256, group scales: o 12.4 -> 10.8 us, down 31.8 -> 24.4
  // us; channel scales: down 24.0 -> 21.7 us, o unchanged; with more tiles,
  // one 8-wave workgroup per CU loses to three 4-wave ones)
  if (!swiglu && p.cfg == 2 && p.tiles <= 256) {
    p.cfg = kMenuKSplit;
    p.threads = 64 * kMenu[p.cfg].GM * kMenu[p.cfg].GN * kMenu[p.cfg].ks;
  }
  const TileCfg& c = kMenu[p.cfg];
  // 128 x 128 group tiles: two workgroups per CU hide each other's latencies
  // (largem_group128); one alone does better reading its operands a step
  // ahead (largem_kernel.h), unless K is short and the start and the end
  // count.  us (paired / ahead), 256 tiles at most: gated, 16 tiles K = 512
  // 6.8 / 7.1, 1024 9.1 / 9.3, 2048 14.2 / 13.6, 4096 23.8 / 22.3, 12288 61.5
  // / 56.7; gated, 256 tiles K = 4096 24.3 / 24.2, 12288 68.4 / 66.3; plain,
  // 224 tiles K = 1024 9.5 / 9.9, 4096 23.9 / 23.8, 8192 42.8 / 41.9, 12288
  // 61.8 / 60.3.
  p.paired = group && p.cfg == 1 && (p.tiles > 256 || K < (swiglu ? 2048 : 8192));
  const int ring = p.paired ? kGroup128Ring : c.ring;
  p.lds_bytes = (size_t)ring * ((size_t)p.BM * 128 + (size_t)p.BN / 16 * kBlockBytes +
                                (group ? (size_t)(c.GM * c.GN) * 256 : 0));
  return p;
}

hipError_t launch_largem(const LargeMPlan& p, const LargeMArgs& a, hipStream_t stream) {
  LargeMKernelFn k = p.group ? largem_group_kernel(p.cfg, p.swiglu, p.paired) : channel_kernel(p.cfg, p.swiglu);
  if (!k || p.tiles < 1 || p.tiles > kMaxGrid) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)p.tiles;
  hipLaunchKernelGGL(k, dim3(grid), dim3(p.threads), p.lds_bytes, stream, a);
  return hipGetLastError();
}

const char* largem_kernel_name(const LargeMPlan& p) {
  static thread_local char buf[96];
  snprintf(buf, sizeof buf, "largem<%dx%d,%s%s%s%s> tiles=%dx%d", p.BM, p.BN, p.group ? "group" : "channel",
           p.swiglu ? ",swiglu" : "", kMenu[p.cfg].ks > 1 ? ",ksplit" : "",
           p.group && p.cfg == 1 && !p.paired ? ",ahead" : "", p.tiles_m, p.tiles_n);
  return buf;
}

}  // namespace w4a8
