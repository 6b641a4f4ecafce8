// Group-scale instances of the large-M W4A8 GEMM.
//
// This file is built with -mllvm -amdgpu-mfma-vgpr-form: the MFMAs then
// write their int32 partial sums to VGPRs, where the per-step rescale reads
// them directly (from AGPRs every element would first need a
// v_accvgpr_read, one more VALU instruction per element and step in a loop
// that is bound by its VALU work).  The per-channel instances keep the
// default AGPR form, which is faster for them.
//
// The 128 x 128 tile (plain and gated) has a kernel of its own here, held to
// 256 registers and 75 KiB of LDS so that two workgroups share a CU; where
// there is only one per CU it is an instance of largem_kernel.h, like the
// 64 x 64 tiles.
#include "largem_kernel.h"

namespace w4a8 {

namespace {

// 128 x 128 tile, 4 waves of 64 x 64, 128 k (one scale group) per step.
//
// What bounds it: a step's 16 matrix instructions per wave (33 cycles each)
// come with 128 vector instructions of rescale (convert, fma per output) and
// 48 of nibble unpack, and a vector instruction takes 4 cycles while matrix
// instructions run on the SIMD: 768 cycles a step, whatever the number of
// waves.  A wave alone on its SIMD also spends issue slots on its LDS reads,
// loads, waits and scalar instructions and waits out every latency: with the
// template's 296 registers (one workgroup per CU) a step took ~1430 cycles.
// Two workgroups per CU, which pass their barriers, prologues and epilogues
// independently, fill each other's gaps.  So registers are held to 256 (196
// are used): one operand set, read after the barrier instead of a step
// ahead, partial sums of two 32 x 32 blocks, no scales kept.  The stage ring
// is 3 deep: two stages of loads in flight under a step.
template <bool SW>
__global__ __launch_bounds__(256, 2) void largem_group128(const LargeMArgs a) {
  constexpr int kRing = kGroup128Ring, BM = 128, BN = 128, kThreads = 256;
  constexpr int kABytes = BM * 128, kBBytes = BN / 16 * kBlockBytes, kSBytes = 4 * 256;
  constexpr int kAReg = kRing * kABytes, kBReg = kRing * kBBytes;
  constexpr int OBN = SW ? BN / 2 : BN;  // output columns per tile
  constexpr int kPerStage = 7;           // vector-memory instructions per wave and stage: 4 A, 2 B, 1 scales
  extern __shared__ __align__(16) uint8_t lds[];

  int bid = blockIdx.x;
  const int total = (int)gridDim.x;
  if (a.xcd_remap) bid = (bid & 7) * (total >> 3) + (bid >> 3);
  const int tm = bid % a.tiles_m, tn = bid / a.tiles_m;
  // Gated tiles: tile columns [0, 64) are gate columns f0 .., [64, 128) the
  // up columns F + f0 ..; output columns f0 .. f0 + 64.
  const int m0 = tm * BM, n0 = tn * BN;
  const int f0 = tn * OBN, ft0 = f0 / 16, fu0 = a.F / 16 + ft0;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int M = a.M, N = a.N, K = a.K, KB = a.KB;
  const int l32 = lane & 31, g2 = lane >> 5;

  // Rows past M and tiles past N lie outside the descriptors and read as
  // zeros (gated: per half, the tiles and columns inside [0, F)).
  const int rows_here = min(BM, M - m0);
  const int tiles_here = SW ? min(OBN / 16, a.F / 16 - ft0) : min(BN / 16, N / 16 - n0 / 16);
  const int cols_here = SW ? min(OBN, a.F - f0) : min(BN, N - n0);
  const u32x4 ares = make_rsrc_words(a.xq + (size_t)m0 * K, (uint32_t)(rows_here * K));
  const u32x4 bres = make_rsrc_words(a.wp + (size_t)(SW ? ft0 : n0 / 16) * KB * kBlockBytes,
                                     (uint32_t)(tiles_here * KB * kBlockBytes));
  const u32x4 bres_u =
      SW ? make_rsrc_words(a.wp + (size_t)fu0 * KB * kBlockBytes, (uint32_t)(tiles_here * KB * kBlockBytes)) : bres;
  // group scales: wave w fetches tile columns [32 w, + 32), two per lane;
  // gated: waves 2 and 3 the up columns
  const bool s_up = SW && wave >= 2;
  const int sc0 = SW ? (s_up ? a.F + f0 : f0) : n0;
  const u32x4 sres =
      make_rsrc_words(static_cast<const uint16_t*>(a.w_scale) + sc0, (uint32_t)(((size_t)KB * N - sc0) * 2));
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

  // Loads of a stage: 16-byte chunk p = j * 256 + tid of the A tile is row
  // p / 8, physical chunk p % 8, which holds the logical chunk
  // (p % 8) ^ ((row >> 1) & 7) (see largem_kernel.h).
  uint32_t a_voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = j * kThreads + tid, row = p >> 3;
    a_voff[j] = (uint32_t)(row * K + (((p & 7) ^ ((row >> 1) & 7)) * 16));
  }
  uint32_t b_voff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    b_voff[j] = (uint32_t)(lane * 16 + (j * 4 + wave - (SW && j == 1 ? BN / 32 : 0)) * KB * kBlockBytes);
  const int scol = wave * 32 - (s_up ? OBN : 0) + 2 * lane;
  const uint32_t s_voff = 2 * lane < 32 && scol < cols_here ? (uint32_t)(scol * 2) : kOOB;
  // instruction d of step kb's stage (past the end: zeros without traffic)
  auto issue_one = [&](int kb, int stage, int d) {
    const bool ok = kb < KB;
    if (d < 4)
      lds_dma16(ares, lds_base + (uint32_t)(stage * kABytes + (d * 4 + wave) * 1024), a_voff[d], ok ? kb * 128 : kOOB);
    else if (d < 6)
      lds_dma16_nt(d == 5 ? bres_u : bres, lds_base + (uint32_t)(kAReg + stage * kBBytes + ((d - 4) * 4 + wave) * 1024),
                   b_voff[d - 4], ok ? kb * kBlockBytes : kOOB);
    else
      lds_dma4(sres, lds_base + (uint32_t)(kAReg + kBReg + stage * kSBytes + wave * 256), s_voff,
               ok ? (uint32_t)((size_t)kb * N * 2) : kOOB);
  };

  // LDS read addresses (stage, block and k half go in the immediate): the
  // activation chunks of row 64 wm + 32 i + l32, the weight chunk and scale
  // of column 64 wn + 32 j + l32 (gated: 64 j + 32 wn + l32).
  const uint8_t* a_rd[4];
#pragma unroll
  for (int tp = 0; tp < 2; ++tp)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      a_rd[2 * tp + h] = lds + (wm * 64 + l32) * 128 + (((2 * (2 * tp + g2) + h) ^ ((l32 >> 1) & 7)) << 4);
  const int col0 = (SW ? 32 : 64) * wn + l32;
  constexpr int kColStep = SW ? 64 : 32;  // tile columns between a wave's two blocks
  const uint8_t* b_rd = lds + kAReg + (col0 >> 4) * kBlockBytes + (col0 & 15) * 16 + g2 * 256;
  const uint8_t* s_rd = lds + kAReg + kBReg + (col0 >> 5) * 256 + (col0 & 31) * 2;

  float facc[2][2][16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) facc[i][j][r] = 0.0f;
  v16i part[2];  // partial sums of the block in the matrix core and of the one before it
#pragma unroll
  for (int r = 0; r < 16; ++r) part[1][r] = 0;
  float sg_last = 0.0f;  // the scale of part[1] at the start of a step (block (1, 1) of the last step)

  // the unpack as assembly, so that it stays in the slot it is dealt to
  auto unpack_word = [](uint32_t w, int& lo, int& hi) {
    asm volatile(
        "v_lshlrev_b32 %0, 4, %2\n\t"
        "v_and_b32 %0, 0xf0f0f0f0, %0\n\t"
        "v_and_b32 %1, 0xf0f0f0f0, %2"
        : "=&v"(lo), "=&v"(hi)
        : "v"(w));
  };
  auto word = [](const uint4& c, int e) { return e == 0 ? c.x : e == 1 ? c.y : e == 2 ? c.z : c.w; };

  // A step: wait for its stage (the younger stage stays in flight), barrier
  // (every wave's share has landed, and every wave is done with the stage
  // before it, which is refilled for step kb + 2), the operand reads, then
  // 16 slots of one matrix instruction, a quarter of the rescale of the
  // block before it (the last block's falls in the next step) and 3 words of
  // unpack.  Blocks in the order (0, 0) (1, 0) (0, 1) (1, 1): column block
  // 1 is unpacked under block 0's matrix instructions.
  auto step = [&](auto stage_c, int kb) {
    constexpr int S = decltype(stage_c)::value;
    wait_vmcnt<kPerStage>();
    lds_barrier();
    uint4 braw[2][2];
    v4i aop[2][4], lo[2][2], hi[2][2];
    float sg[2];
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) braw[0][tp] = *reinterpret_cast<const uint4*>(b_rd + S * kBBytes + tp * 512);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) aop[i][c] = *reinterpret_cast<const v4i*>(a_rd[c] + S * kABytes + i * 32 * 128);
#pragma unroll
    for (int tp = 0; tp < 2; ++tp)
      braw[1][tp] = *reinterpret_cast<const uint4*>(b_rd + S * kBBytes + kColStep / 16 * kBlockBytes + tp * 512);
    uint16_t sraw[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      sraw[j] = *reinterpret_cast<const uint16_t*>(s_rd + S * kSBytes + j * (kColStep / 32) * 256);
#pragma unroll
    for (int tp = 0; tp < 2; ++tp)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int l, h;
        unpack_word(word(braw[0][tp], e), l, h);
        lo[0][tp][e] = l;
        hi[0][tp][e] = h;
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int t = q / 4, i = t & 1, j = t >> 1, sub = q & 3, tp = sub >> 1, hn = sub & 1;
      v16i& p = part[t & 1];
      const v16i& prev = part[(t & 1) ^ 1];
      const v4i bop = hn ? hi[j][tp] : lo[j][tp];
      if (sub == 0)
        p = mfma32(aop[i][0], bop, v16i{});  // a block starts from zero: an inline constant
      else
        p = mfma32(aop[i][sub], bop, p);
      if (q < 14 && q % 2 == 0) issue_one(kb + 2, (S + 2) % kRing, q / 2);
      const int pi = (t + 3) & 1, pj = ((t + 3) & 3) >> 1;  // the block before
      const float ps = t == 0 ? sg_last : sg[pj];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 4 * sub + u;
        facc[pi][pj][r] = __fmaf_rn((float)prev[r], ps, facc[pi][pj][r]);
      }
      if (q < 8) {  // column block 1's words
        int l, h;
        unpack_word(word(braw[1][q >> 2], q & 3), l, h);
        lo[1][q >> 2][q & 3] = l;
        hi[1][q >> 2][q & 3] = h;
      }
      if (q == 2) {
        sg[0] = f16_to_f32(sraw[0]) * 0.0625f;  // the unpacked weights are 16 times too large
        sg[1] = f16_to_f32(sraw[1]) * 0.0625f;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    sg_last = sg[1];
  };

#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int d = 0; d < kPerStage; ++d) issue_one(st, st, d);
  for (int kb = 0; kb < KB; kb += 3) {
    step(std::integral_constant<int, 0>{}, kb);
    if (kb + 1 < KB) step(std::integral_constant<int, 1>{}, kb + 1);
    if (kb + 2 < KB) step(std::integral_constant<int, 2>{}, kb + 2);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) facc[1][1][r] = __fmaf_rn((float)part[1][r], sg_last, facc[1][1][r]);

  // token scales: rows 8 q + 4 g2 + e of block i
  const __amdgpu_buffer_rsrc_t xsres = make_rsrc(uniform_ptr(a.x_scale + m0), uniform_u32((uint32_t)(rows_here * 4)));
  uint4 sx4[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) sx4[i][q] = buf_load16(xsres, (uint32_t)((wm * 64 + i * 32 + 8 * q + 4 * g2) * 4));
  wait_vmcnt<0>();  // the stages issued past the end, the token scales
  lds_barrier();    // every wave is done with the ring

  // ---- epilogue: the scaled tile is staged in the idle ring and leaves as
  // 16-byte row chunks, as in largem_kernel.h
  auto result = [&](int i, int j, int r) -> float {
    const uint4 s4 = sx4[i][r >> 2];
    return __fmul_rn(facc[i][j][r], __uint_as_float(word(s4, r & 3)));
  };
  constexpr int OWN = SW ? 1 : 2;
  auto out_value = [&](int i, int j, int r) -> float {
    if constexpr (SW) {
      const float g = result(i, 0, r), u = result(i, 1, r);
      return __fmul_rn(__fdiv_rn(g, __fadd_rn(1.0f, __expf(-g))), u);
    } else {
      return result(i, j, r);
    }
  };
  const int ldy = SW ? a.F : N, oc0 = SW ? f0 : n0;
  auto store_tile = [&](auto es_tag) {
    constexpr int es = decltype(es_tag)::value;
    constexpr int kPitch = es == 2 ? OBN * 2 + 64 : OBN * 4 + 16;
    static_assert(BM * kPitch <= kRing * (kABytes + kBBytes + kSBytes), "output tile must fit the LDS ring");
    const bool odd = lane & 1;
    const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < OWN; ++j)
        if constexpr (es == 2) {
#pragma unroll
          for (int rp = 0; rp < 8; ++rp) {
            const uint32_t pair =
                bf16x2_bits(canonical_nan(out_value(i, j, 2 * rp)), canonical_nan(out_value(i, j, 2 * rp + 1)));
            const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)pair, 0xB1, 0xF, 0xF, false);
            const uint32_t w = __builtin_amdgcn_perm(recv, pair, sel);
            const int r = 2 * rp + (odd ? 1 : 0);
            const int row = wm * 64 + i * 32 + 8 * (r >> 2) + 4 * g2 + (r & 3);
            *reinterpret_cast<uint32_t*>(lds + row * kPitch + (wn * 32 * OWN + j * 32 + (l32 & ~1)) * 2) = w;
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = wm * 64 + i * 32 + 8 * (r >> 2) + 4 * g2 + (r & 3);
            *reinterpret_cast<float*>(lds + row * kPitch + (wn * 32 * OWN + j * 32 + l32) * 4) = out_value(i, j, r);
          }
        }
    lds_barrier();
    constexpr int kRowChunks = OBN * es / 16;
#pragma unroll
    for (int it = 0; it < BM * kRowChunks / kThreads; ++it) {
      const int p = it * kThreads + tid, row = p / kRowChunks, cc = p % kRowChunks;
      const uint4 v = *reinterpret_cast<const uint4*>(lds + row * kPitch + cc * 16);
      if (row < rows_here && cc * (16 / es) < cols_here)
        *reinterpret_cast<uint4*>(static_cast<uint8_t*>(a.y) + ((size_t)(m0 + row) * ldy + oc0) * es + cc * 16) = v;
    }
  };
  if (a.out_kind == kOutBF16)
    store_tile(std::integral_constant<int, 2>{});
  else
    store_tile(std::integral_constant<int, 4>{});
}

}  // namespace

LargeMKernelFn largem_group_kernel(int cfg, bool swiglu, bool paired) {
  if (swiglu)  // the gated tile that fits group mode
    return cfg != 1 ? nullptr : paired ? largem_group128<true> : menu_kernel<1, true, true>();
  switch (cfg) {
    case 1: return paired ? largem_group128<false> : menu_kernel<1, true>();
    case 2: return menu_kernel<2, true>();
    case kMenuKSplit: return menu_kernel<kMenuKSplit, true>();
    default: return nullptr;  // 128 x 192 does not fit the group accumulators
  }
}

}  // namespace w4a8
