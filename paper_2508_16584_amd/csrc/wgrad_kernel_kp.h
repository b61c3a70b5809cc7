// Weight gradient in tiles of 64 x 64 with the token blocks dealt to the waves (same operation, bounds and arithmetic per element
// as wgrad_kernel.h, so the same bits): for launches of so few tiles that each is a chain of token blocks.
//
// A tile of 256 x 128 goes through its token blocks one after the other, 1.1 to 2 us each, and few outputs are few tiles: 2 groups,
// 11472 tokens, 256 x 768, are 12 of them and up to 46 blocks, 96 us of which the operands take 2.  Only the last step of a block
// has to happen in the order of the blocks, acc = fma(p, sdy * sx, acc).  So, as in the fifth kernel of the forward pass, wave w of
// four takes blocks w, w + 4, ... of the group, each through LDS slots of its own without any barrier: fetch, clear the bytes outside the
// group, 16 matrix instructions; the products go where the operands were, and after one barrier per four blocks wave w adds up the
// rows of dY^T fragment w, in order.  A workgroup computes one tile and ends; the hardware deals them out.
// Measured, us per launch (narrow tiles -> these): those 2 groups 96.2 -> 25.9; 1 group of 944 tokens, 1280 x 512, 24.1 -> 6.9; 5 groups,
// 4000 tokens, 256 x 512, 24.5 -> 9.0; 3 groups, 448 tokens, 640 x 768, 11.2 -> 6.5 (fp32 all).
// What bounds it: in long chains the latency of the fetches.  A slot is free when its products have been added up, is fetched again behind
// the barrier of the next round and awaited in the round after: from the third round on a wave has at most one block on its way, behind the sums
// alone (those 12 rounds: 2 us each).  With many tiles LDS (operands in and out, products in and out: 64 KB per block) and a quarter of the
// operand reuse of a 256 x 256 tile, hence only where few outputs meet many tokens (see wgrad_chain in gg_fp8.hip).
#pragma once
#include "wgrad_kernel.h"

namespace gg {

struct WgradKpCfg {
  static constexpr int TK = 64, TN = 64, NW = 4, NT = 64 * NW, U = 2;
  static constexpr int X_BYTES = TK * 128, Y_BYTES = TN * 128;
  static constexpr int SX_BASE = X_BYTES + Y_BYTES, SY_BASE = SX_BASE + TK * 4, SLOT_BYTES = SY_BASE + TN * 4;
  static constexpr int ND = (TK + TN) / 8 + 2;                         // fetches per token block
  static constexpr int LDS_BYTES = NW * U * SLOT_BYTES;
  static_assert(16 * 1024 <= SX_BASE && ND * (U - 1) < 64 && LDS_BYTES <= 160 * 1024, "products over the operands; wait counter; LDS budget");
};

template <bool OUT16>
__global__ void __launch_bounds__(WgradKpCfg::NT) gg_wgrad_kp_kernel(const WgradArgs a) {
  using Cfg = WgradKpCfg;
  constexpr int NW = Cfg::NW, U = Cfg::U;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l = threadIdx.x & 63, r = l & 15, q = l >> 4;
  const int M = a.M_total;

  // Workgroup b runs on XCD b % 8: of every 64 tiles an XCD takes 8 neighbours, which share features.
  const int b = (int)blockIdx.x, T = (b & ~63) | (b & 7) << 3 | (b >> 3 & 7);
  if (T >= a.tiles) return;
  const int per_group = a.n_tiles * a.k_tiles;
  const int g = T / per_group, local = T - g * per_group, kt = local / a.n_tiles, nt = local - kt * a.n_tiles;
  const int k0 = kt * Cfg::TK, n0 = nt * Cfg::TN;
  const GG_CONST_I32* offc = (const GG_CONST_I32*)a.off;
  const int lo = clampi(offc[g], 0, M), hi = clampi(offc[g + 1], lo, M);
  const int j0 = lo >> 7, steps = hi > lo ? ((hi + 127) >> 7) - j0 : 0;

  // fetches, as in the narrow tiles: whole-tensor views; the features change places on their way into LDS, so that a lane of row r
  // holds four neighbouring features (slot 16 f + r is feature 4 r + f)
  const __amdgpu_buffer_rsrc_t dX = __builtin_amdgcn_make_buffer_rsrc((void*)a.XT, 0, a.K * M, GG_RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t dY = __builtin_amdgcn_make_buffer_rsrc((void*)a.DYT, 0, a.N * M, GG_RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t dSX = __builtin_amdgcn_make_buffer_rsrc((void*)a.SX, 0, a.K * a.MB * 4, GG_RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t dSY = __builtin_amdgcn_make_buffer_rsrc((void*)a.SDY, 0, a.N * a.MB * 4, GG_RSRC_FLAGS);
  int vX[2], vY[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * i + (l >> 3), o = ((l & 7) ^ swz_key_a(row)) << 4;      // of 16 rows; the keys repeat
    vX[i] = 4 * row * M + o;
    vY[i] = row * M + o;
  }
  uint8_t* const slots = lds + w * (U * Cfg::SLOT_BYTES);
  auto fetch = [&](int s, int slot) __attribute__((always_inline)) {           // token block s of the group
    const int j = j0 + s;
    uint8_t* const st = slots + slot * Cfg::SLOT_BYTES;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(dX, GG_LDS_PTR(st + i * 1024), 16, vX[i & 1], j * 128 + (k0 + (i >> 1)) * M, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(dY, GG_LDS_PTR(st + Cfg::X_BYTES + i * 1024), 16, vY[i & 1], j * 128 + (n0 + 16 * (i >> 1)) * M, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dSX, GG_LDS_PTR(st + Cfg::SX_BASE), 4, l * 4, (j * a.K + k0) * 4, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dSY, GG_LDS_PTR(st + Cfg::SY_BASE), 4, l * 4, (j * a.N + n0) * 4, 0, 0);
  };
  const int mine = (steps - w + NW - 1) / NW;             // token blocks of this wave
  int issued = 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < mine) {
      fetch(u * NW + w, u);
      issued = u + 1;
    }

  const int key = swz_key_a(r), rd0 = r * 128 + (((2 * q) ^ key) << 4), rd1 = r * 128 + (((2 * q + 1) ^ key) << 4);
  auto frag = [&](const uint8_t* p) __attribute__((always_inline)) -> v8i {
    const v4i x = *(const v4i*)(p + rd0), y = *(const v4i*)(p + rd1);
    return (v8i){x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
  };
  v4f acc[4];                                             // row 16 w + 4 q + i of the tile: four neighbouring features
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = (v4f){0.f, 0.f, 0.f, 0.f};
  const int rounds = (steps + NW - 1) / NW;
  int slot = 0, prev = 0;
  for (int c = 0; c < rounds; ++c) {
    uint8_t* const st = slots + slot * Cfg::SLOT_BYTES;
    if (c < mine) {
      wait_all_but_n<Cfg::ND, U - 1>(issued - 1 - c);
      v8i xf[4], yf[4];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        xf[f] = frag(st + f * 2048);
        yf[f] = frag(st + Cfg::X_BYTES + f * 2048);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read: it can be written
      __builtin_amdgcn_sched_barrier(0);
      const int first = (j0 + c * NW + w) * 128;
      if (lo > first || hi < first + 128) {               // tokens of other groups: in both operands, so that no NaN of theirs arrives
        const int lo4 = 4 * (lo - first - 32 * q), hi4 = 4 * (hi - first - 32 * q);
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const int m = bytes_from(lo4 - 16 * d) & bytes_below(hi4 - 16 * d);
#pragma unroll
          for (int f = 0; f < 4; ++f) {
            xf[f][d] &= m;
            yf[f][d] &= m;
          }
        }
      }
      v4f p[4][4];
#pragma unroll
      for (int nf = 0; nf < 4; ++nf)
#pragma unroll
        for (int kf = 0; kf < 4; ++kf)
          p[nf][kf] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(yf[nf], xf[kf], (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
#pragma unroll
      for (int nf = 0; nf < 4; ++nf)
#pragma unroll
        for (int kf = 0; kf < 4; ++kf) *(v4f*)(st + (nf * 4 + kf) * 1024 + l * 16) = p[nf][kf];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                         // the products of this round are there, those of the last one have been added up
    asm volatile("" ::: "memory");
    if (c > 0 && issued < mine) {
      fetch(issued * NW + w, prev);
      ++issued;
    }
    prev = slot;
    const uint8_t* const pr = lds + slot * Cfg::SLOT_BYTES;
    const int left = steps - c * NW;
    v4f p[NW][4], sx[NW], sy[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {                        // (past the last block: read and not used)
      const uint8_t* const pi = pr + i * (U * Cfg::SLOT_BYTES);
#pragma unroll
      for (int kf = 0; kf < 4; ++kf) p[i][kf] = *(const v4f*)(pi + (w * 4 + kf) * 1024 + l * 16);
      sx[i] = *(const v4f*)(pi + Cfg::SX_BASE + 16 * r);
      sy[i] = *(const v4f*)(pi + Cfg::SY_BASE + (16 * w + 4 * q) * 4);
    }
#pragma unroll
    for (int i = 0; i < NW; ++i)
      if (i < left) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int kf = 0; kf < 4; ++kf) acc[e][kf] = __builtin_fmaf(p[i][kf][e], sy[i][e] * sx[i][kf], acc[e][kf]);
      }
    slot = slot + 1 == U ? 0 : slot + 1;
  }
  constexpr int ES = OUT16 ? 2 : 4;      // bytes per element of dW
  const __amdgpu_buffer_rsrc_t dOut = __builtin_amdgcn_make_buffer_rsrc((void*)((uint8_t*)a.dW + (((int64_t)g * a.N + n0) * a.K + k0) * ES), 0, ((Cfg::TN - 1) * a.K + Cfg::TK) * ES, GG_RSRC_FLAGS);
  const int vOut = ((16 * w + 4 * q) * a.K + 4 * r) * ES;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (OUT16)
      __builtin_amdgcn_raw_buffer_store_b64((v2i){pack2_rne(acc[i][0], acc[i][1], false), pack2_rne(acc[i][2], acc[i][3], false)}, dOut, vOut, i * a.K * ES, kStoreStreaming);
    else
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, acc[i]), dOut, vOut, i * a.K * ES, kStoreStreaming);
  }
}

}  // namespace gg
