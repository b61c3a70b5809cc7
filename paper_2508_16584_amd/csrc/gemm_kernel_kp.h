// Fifth kernel of the padding-free block-scaled FP8 grouped GEMM (same operation, same bounds and the same arithmetic per
// element as gemm_kernel.h, so the same bits): for launches of so few tiles that each is a chain of K blocks.
//
// In the other kernels a workgroup goes through its K blocks one after the other, a barrier and an LDS round trip each (0.24 us
// in the smallest tile of the third kernel), with a ring of two to four of them on their way: one row of K = 7808 takes 19 us of
// which its bytes take 1.5, and 92 workgroups of 24 KB in flight stream at 1.4 TB/s.  What has to happen in the order of K is
// only the last step, acc = fma(p, s, acc) with the product p of a K block and its factor s.  So here the K blocks are dealt to
// the waves of a workgroup: wave w takes blocks w, w + NW, ..., each through LDS slots of its own without any barrier, and puts
// its products and factors into LDS; after one barrier per NW blocks the waves that own a fragment of the tile add them up in
// order.  A workgroup starts with NW x U K blocks on their way (two slots per wave); how far ahead it stays: see OVERLAY.
//
// A workgroup computes one tile and ends: the launch has as many as there may be tiles, the hardware deals them out, and nothing
// stands between the launch and the first fetch but the lookup of the group.  (With persistent workgroups whose fetches run on
// into the next tile the smallest launches take 1 us more, 2.9 -> 3.9 us at 3 rows, N = 512, K = 640, and only streams of 100 MB
// and more gain.)
//
// OVERLAY: the products go where their operands were, which leaves room for more workgroups per compute unit; a slot is then
// free only when they have been added up: it is fetched again behind the barrier of the next round and awaited in the round after, so
// from the third round on a wave has at most one block on its way, hidden behind the sums and the other workgroups of the compute unit
// alone.  Better for short K loops and many tiles; the long chains are better off with an area for the products and a slot that is
// refilled as soon as it has been read, two rounds ahead of its use (one row, N = 1280, K = 7808: 10.3 -> 7.3 us).
//
// Measured, us per launch in a graph (third kernel -> this one, bytes at 6.8 TB/s): 1 group of 16 rows, 5888 x 4224 22.0 -> 8.2
// (3.7); 4 groups, 65 rows, 640 x 5120 14.5 -> 6.5 (2.0); 4 groups, 600 rows, 256 x 256 4.6 -> 3.3; 54 groups, 193 rows,
// 1152 x 4608 39.3 -> 36.4 (30.7), which is too little for the choice to take it (kChainTimes in gg_fp8.hip).
#pragma once
#include "gemm_kernel.h"

namespace gg {

template <int MF_, int NF_, int NW_, int U_, int WGS_, bool OVERLAY_>
struct KpCfg {
  static constexpr int MF = MF_, NF = NF_, U = U_, NW = NW_, NT = 64 * NW;
  static constexpr bool OVERLAY = OVERLAY_;
  static constexpr int BM = 16 * MF, BN = 16 * NF, FRAGS = MF * NF;                           // fragments of 16 x 16 outputs
  static constexpr int A_BYTES = MF * 2048, B_BYTES = NF * 2048;
  static constexpr int SA_BASE = A_BYTES + B_BYTES, SB_BASE = SA_BASE + 256, SLOT_BYTES = SB_BASE + 256;
  static constexpr int ND = 2 * MF + 2 * NF + 2;                                              // fetches per K block
  static constexpr int P_BASE = NW * U * SLOT_BYTES, S_OFF = FRAGS * 1024, P_BYTES = S_OFF + 64 * MF;   // a wave's products, factors
  static constexpr int P_PITCH = OVERLAY ? U * SLOT_BYTES : P_BYTES;                          // from wave to wave
  static constexpr int LDS_BYTES = P_BASE + (OVERLAY ? 0 : 2 * NW * P_BYTES);
  static_assert(BM <= 64 && 128 % BN == 0, "one fetch for the scales of the rows, one scale block of columns");
  static_assert(FRAGS <= NW && U >= 2 && ND * (U - 1) < 64, "a fragment per wave; the wait counter");
  static_assert(P_BYTES <= SLOT_BYTES && LDS_BYTES * WGS_ <= 160 * 1024, "LDS budget");
};

template <class Cfg>
__global__ void __launch_bounds__(Cfg::NT) gg_gemm_kp_kernel(const GemmArgs a) {
  constexpr int MF = Cfg::MF, NF = Cfg::NF, U = Cfg::U, NW = Cfg::NW, BM = Cfg::BM, BN = Cfg::BN;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l = threadIdx.x & 63, r = l & 15, q = l >> 4;
  const int K = a.K, KB = a.KB, N = a.N;

  // Workgroup b runs on XCD b % 8: of every 64 tiles an XCD takes 8 neighbours, and neighbours are row tiles of one column tile,
  // which share its weights.
  const int b = (int)blockIdx.x, T = (b & ~63) | (b & 7) << 3 | (b >> 3 & 7);
  GroupRows groups;
  groups.init(a, BM, l, false);
  GroupRows::Group grp;
  if (!groups.find_once(a, BM, l, T, grp)) return;
  const int mtiles = row_tiles(grp.rows, BM), local = T - grp.tiles_before;
  const int ntile = local / mtiles, mtile = local - ntile * mtiles;
  const int n0 = ntile * BN, n_rem = N - n0;
  const int rows = grp.rows - mtile * BM < BM ? grp.rows - mtile * BM : BM;
  const int64_t grow = (int64_t)grp.row0 + mtile * BM;
  const int nb_all = (N + 127) >> 7;
  // bounded views, as in the first kernel
  const __amdgpu_buffer_rsrc_t dA = uniform_rsrc(a.A + grow * K, rows * K);
  const __amdgpu_buffer_rsrc_t dB = uniform_rsrc(a.B + ((int64_t)grp.g * N + n0) * K, (n_rem < BN ? n_rem : BN) * K);
  const __amdgpu_buffer_rsrc_t dSA = uniform_rsrc((const uint8_t*)a.SA + grow * a.sa_row_stride, sa_view_bytes(a, grow, rows));
  const __amdgpu_buffer_rsrc_t dSB = uniform_rsrc(a.SB + ((int64_t)grp.g * nb_all + (n0 >> 7)) * KB, KB * 4);
  const int rot = k_rotation(a, n0);
  const bool stream = mtiles == 1 && a.b_lines;        // weights that are fetched once: past the L2

  // fetches: lane l of a slab of 8 rows lands at byte 16 l of its 1 KB (row l / 8, chunk l % 8), swizzled as in the first kernel;
  // in a short last K block the lanes whose 16 bytes belong to the next row fetch zeros
  int v[2];
  bool tail[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * i + (l >> 3), o = ((l & 7) ^ swz_key_a(row)) << 4;
    v[i] = row * K + o;
    tail[i] = o >= a.k_rem;
  }
  const int vSA = l < BM ? l * a.sa_row_stride : GG_OOB_OFFSET, vSB = l == 0 ? 0 : GG_OOB_OFFSET;
  uint8_t* const slots = lds + w * (U * Cfg::SLOT_BYTES);
  auto fetch = [&](int i, int slot) __attribute__((always_inline)) {       // the i-th K block of the tile
    const int kb = k_wrapped(i + rot, KB);
    const bool last = kb == KB - 1;
    uint8_t* const st = slots + slot * Cfg::SLOT_BYTES;
    const int v0 = last && tail[0] ? GG_OOB_OFFSET : v[0], v1 = last && tail[1] ? GG_OOB_OFFSET : v[1];
#pragma unroll
    for (int s = 0; s < 2 * NF; ++s) {
      if (stream) __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(st + Cfg::A_BYTES + s * 1024), 16, s & 1 ? v1 : v0, kb * 128 + (s >> 1) * 16 * K, 0, 2 | 16);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(st + Cfg::A_BYTES + s * 1024), 16, s & 1 ? v1 : v0, kb * 128 + (s >> 1) * 16 * K, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 2 * MF; ++s)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(dA, GG_LDS_PTR(st + s * 1024), 16, s & 1 ? v1 : v0, kb * 128 + (s >> 1) * 16 * K, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dSA, GG_LDS_PTR(st + Cfg::SA_BASE), 4, vSA, kb * a.sa_kb_stride, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dSB, GG_LDS_PTR(st + Cfg::SB_BASE), 4, vSB, kb * 4, 0, 0);
  };
  const int mine = (KB - w + NW - 1) / NW;             // K blocks of this wave
  int issued = 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < mine) {
      fetch(u * NW + w, u);
      issued = u + 1;
    }

  const int key = swz_key_a(r), rd0 = r * 128 + (((2 * q) ^ key) << 4), rd1 = r * 128 + (((2 * q + 1) ^ key) << 4);
  auto frag = [&](const uint8_t* p) __attribute__((always_inline)) -> v8i {
    const v4i lo = *(const v4i*)(p + rd0), hi = *(const v4i*)(p + rd1);
    return (v8i){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  };
  const int fm = w / NF, fn = w - fm * NF;             // the fragment that this wave adds up (w < FRAGS)
  v4f acc = {0.f, 0.f, 0.f, 0.f};
  // (stated as fused operations: behind a branch the compiler may form a product and a sum, which round twice)
  auto add = [&](const v4f p, float s) __attribute__((always_inline)) { acc = __builtin_elementwise_fma(p, (v4f){s, s, s, s}, acc); };
  const int rounds = (KB + NW - 1) / NW;
  int slot = 0, prev = 0, half = 0;
  for (int c = 0; c < rounds; ++c) {
    uint8_t* const st = slots + slot * Cfg::SLOT_BYTES;
    uint8_t* const pw = Cfg::OVERLAY ? st : lds + Cfg::P_BASE + (half * NW + w) * Cfg::P_BYTES;
    if (c < mine) {
      wait_all_but_n<Cfg::ND, U - 1>(issued - 1 - c);
      v8i bf[NF], af[MF];
      float sa[MF];
#pragma unroll
      for (int j = 0; j < NF; ++j) bf[j] = frag(st + Cfg::A_BYTES + j * 2048);
#pragma unroll
      for (int m = 0; m < MF; ++m) af[m] = frag(st + m * 2048);
#pragma unroll
      for (int m = 0; m < MF; ++m) sa[m] = *(const float*)(st + Cfg::SA_BASE + (16 * m + r) * 4);
      const float sb = *(const float*)(st + Cfg::SB_BASE);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slot has been read: it can be written
      __builtin_amdgcn_sched_barrier(0);
      v4f p[MF][NF];
#pragma unroll
      for (int m = 0; m < MF; ++m)
#pragma unroll
        for (int j = 0; j < NF; ++j)
          p[m][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bf[j], af[m], (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
      if (!Cfg::OVERLAY && issued < mine) {
        fetch(issued * NW + w, slot);
        ++issued;
      }
#pragma unroll
      for (int m = 0; m < MF; ++m) {
#pragma unroll
        for (int j = 0; j < NF; ++j) *(v4f*)(pw + (m * NF + j) * 1024 + l * 16) = p[m][j];
        if (q == 0) *(float*)(pw + Cfg::S_OFF + (16 * m + r) * 4) = sa[m] * sb;
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                      // the products of this round are there, those of the last one have been added up
    asm volatile("" ::: "memory");
    if (Cfg::OVERLAY) {
      if (c > 0 && issued < mine) {
        fetch(issued * NW + w, prev);
        ++issued;
      }
      prev = slot;
    }
    if (w < Cfg::FRAGS) {
      const uint8_t* const pr = pw - w * Cfg::P_PITCH;
      const int left = KB - c * NW;
      v4f p[NW];
      float s[NW];
#pragma unroll
      for (int i = 0; i < NW; ++i) {                   // all reads before the first sum (past the last K block: read and not used)
        p[i] = *(const v4f*)(pr + i * Cfg::P_PITCH + w * 1024 + l * 16);
        s[i] = *(const float*)(pr + i * Cfg::P_PITCH + Cfg::S_OFF + (16 * fm + r) * 4);
      }
      if (left >= NW) {
#pragma unroll
        for (int i = 0; i < NW; ++i) add(p[i], s[i]);
      } else {
#pragma unroll
        for (int i = 0; i < NW - 1; ++i)
          if (i < left) add(p[i], s[i]);
      }
    }
    slot = slot + 1 == U ? 0 : slot + 1;
    half ^= 1;
  }
  if (w < Cfg::FRAGS) {
    // lane (q, r): row r of the fragment, columns 4 q .. + 3 (N is a multiple of 8: they exist together or not at all)
    const int col = 16 * fn + 4 * q;
    const __amdgpu_buffer_rsrc_t dC = uniform_rsrc(a.C + grow * N + n0, rows * N * 2 - n0 * 2);
    const bool f16 = a.out_f16 != 0;
    const v2i out = {pack2_rne(acc[0], acc[1], f16), pack2_rne(acc[2], acc[3], f16)};
    __builtin_amdgcn_raw_buffer_store_b64(out, dC, col < n_rem ? ((16 * fm + r) * N + col) * 2 : GG_OOB_OFFSET, 0, 0);
  }
}

}  // namespace gg
