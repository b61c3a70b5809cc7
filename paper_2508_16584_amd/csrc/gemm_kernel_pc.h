// Fourth kernel of the padding-free block-scaled FP8 grouped GEMM (same operation, same bounds and the same arithmetic per
// element as gemm_kernel.h, so the same bits): fetching and multiplying are the work of different waves.
//
// A wave whose fetch finds the compute unit's vector memory queue full waits at the issue of that instruction.  In the other
// kernels the waves that multiply issue the fetches too, so a full queue holds up matrix instructions, and while the waves
// read LDS, meet at a barrier or multiply the last fragments of a K block, nobody feeds the queue.  Here a workgroup has 12 waves:
//  * 3 only fetch operands: they walk the tile list with a cursor of their own, keep a ring of three LDS buffers full, wait
//    for their fetches and meet the others at one barrier per K block.  They run on from tile to tile;
//  * 1 only makes scale factors: it takes the scales of 8 K blocks at a time into registers, one such chunk ahead (either
//    storage order of SA; row-major, a row's 32 bytes are one request), and puts the products SA * SB of a K block beside its
//    operands, so a multiplying wave reads one factor per 16 rows and has no scale arithmetic;
//  * 8 (2 x 4) only multiply: they issue no fetch and wait for none.  The barrier that publishes K block kb + 1 stands
//    in front of the last row of matrix instructions of block kb, when a wave has read all it needs of block kb; during
//    that row the weight fragments are refilled in place, so no LDS latency stands between two K blocks.
// Short last K blocks, partial tiles and any number of K blocks are the fetching waves' business alone: one instantiation takes
// every shape.
//
// Tiles have the height of their rows: a group is cut into the fewest tiles of at most `bm` rows (a launch argument, a
// multiple of 32 up to 160), all of about the same number of 32-row steps, and a tile fetches, multiplies and stores only the
// steps that hold rows.
// Three waves per SIMD leave 168 registers per lane: 160 rows of 256 columns are the most that fit (80 accumulators, 32 for
// the weight fragments, 24 for the activation fragments).
//
// What bounds it: where weights are streamed, memory and nothing else (with every matrix instruction taken out the launch takes
// the same time): 256 groups of about 128 rows, N = 4096, K = 7168: 1385 us, of which the weights alone 1104 (6.8 TB/s), the
// activation tiles 55, the scales 40, the stores 175; what is missing to the sum is waiting for one another.  Where there is
// more to multiply, fetches and arithmetic side by side (8 groups of 1120 rows: 305 us; fetches alone 198, arithmetic alone
// 246).  Against the first kernel's 160 x 256 and 128 x 256 tiles, which it replaced: 1472 -> 1421 us on those 256 groups, 284
// -> 261 on 64 groups of 32 rows on average (height chosen), 160 -> 151 on 8 groups of 375, N = 4104, K = 7232; on 1530 random
// problems 0.924 of the time of the 160-row tile and 0.985 of the 128-row one.
#pragma once
#include "gemm_kernel.h"

namespace gg {

struct PcCfg {
  static constexpr int BM = 160, BN = 256, S = 3;                  // the tallest tile; buffers of the ring
  static constexpr int WM = 2, WN = 4, CW = WM * WN, FW = 3, NT = 64 * (CW + FW + 1);
  static constexpr int WTN = BN / WN, TM = BM / 32, TN = WTN / 16;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, S_BYTES = 2 * BM * 4;   // S: one factor per row and 128 columns
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES + S_BYTES;
  static constexpr int INFO_BASE = S * STAGE_BYTES;                // per buffer: the tile whose first K block it holds
  static constexpr int LDS_BYTES = INFO_BASE + S * 16;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// Height of the tallest tile: the one whose tiles fill the rounds over the workgroups best.  A tile's K step costs 4.24 and one
// for each 32 rows (0.56 + 0.13 us per 32 rows), a partly filled round nearly a full one.  On 2500 random problems of 60 GFLOP and
// more (`sweep.py --tiles 2500 --min-gflop 60 --seed 303`) the time is 1.008 of the best of the five heights; with 160 rows
// throughout it is 1.022, with 128 1.087, with 96 1.200.  (Smaller ones of 15 us and more: 1.025, 1.052, 1.066, 1.092.)
__device__ __forceinline__ int pc_height(const GemmArgs& a, const GroupIndex::Rows& rows, int l) {
  int t[5];
  count_row_tiles<32, 64, 96, 128, 160>(a, rows, l, t);
  int best = 160;
  float best_cost = 0.f;
#pragma unroll
  for (int i = 4; i >= 0; --i) {
    const float tiles = (float)t[i] * (float)a.n_tiles;
    const float cost = rounds_of(tiles, 0.91f) * (4.24f + (float)t[0] / (float)(t[i] > 0 ? t[i] : 1));
    if (i == 4 || (tiles < 2147483000.f && cost < best_cost)) {
      best = 32 * (i + 1);
      best_cost = cost;
    }
  }
  return __builtin_amdgcn_readfirstlane(best);
}

__global__ void __launch_bounds__(PcCfg::NT) gg_gemm_pc_kernel(const GemmArgs a) {
  using Cfg = PcCfg;
  constexpr int BM = Cfg::BM, BN = Cfg::BN, WN = Cfg::WN, TM = Cfg::TM, TN = Cfg::TN, S = Cfg::S;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int K = a.K, KB = a.KB, N = a.N;

  if (w >= Cfg::CW) {
    // ---- the tile list, as in the other kernels ------------------------------------------------------------------
    struct Tile {
      int g, n0, rows;       // rows: 0 when there is no tile
      int64_t grow;
      bool once;             // the group's only row tile: its weights are fetched once
    };
    GroupIndex::Rows group_rows;
    group_rows.load(a, l);
    const int bm = a.bm ? a.bm : pc_height(a, group_rows, l);
    GroupIndex groups;
    groups.init(a, group_rows, bm, l, a.split_last != 0);
    const GG_CONST_I32* offc = (const GG_CONST_I32*)a.off;
    auto tile_at = [&](int it) __attribute__((always_inline)) -> Tile {
      Tile t = {0, 0, 0, 0, false};
      const int T = groups.unit(a, it);
      if (T == GroupIndex::NONE) return t;
      int g = 0, base = 0;
      if (!groups.find(a, bm, T, g, base)) return t;
      const int row0 = clampi(offc[g], 0, a.M_total);
      const int Mg = clampi(offc[g + 1], row0, a.M_total) - row0;
      const int mtiles = row_tiles(Mg, bm);
      const int local = T - base;
      const int per_chunk = mtiles * a.n_chunk;
      const int nc = local / per_chunk;
      const int rem = local - nc * per_chunk;
      int csz = a.n_tiles - nc * a.n_chunk;
      csz = csz < a.n_chunk ? csz : a.n_chunk;
      const int mtile = rem / csz;
      const int h = even_height(Mg, mtiles);                             // height of the group's tiles: h * mtiles >= Mg, h <= bm
      t.g = g;
      t.n0 = (nc * a.n_chunk + (rem - mtile * csz)) * BN;
      t.rows = Mg - mtile * h < h ? Mg - mtile * h : h;
      t.grow = (int64_t)row0 + mtile * h;
      t.once = mtiles == 1;
      return t;
    };
    __builtin_amdgcn_s_setprio(3);           // a fetch that can be issued goes before arithmetic

    if (w < Cfg::CW + Cfg::FW) {
      // ======== fetching waves ===================================================================================
      // A K block is 8 + (32-row steps) units of 32 rows x 128 bytes, four fetches of 8 rows each; wave p takes units
      // p, p + 3, ...
      const int p = w - Cfg::CW;
      int vA[4], vB[4];                      // lane offsets of the fetches of a unit; in a short last K block ...
      bool tA[4], tB[4];                     // ... the lanes whose 16 bytes belong to the next row: they fetch zeros
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 8 * i + (l >> 3);    // the swizzle keys repeat every 32 rows
        const int oA = ((l & 7) ^ swz_key_a(row)) << 4, oB = ((l & 7) ^ swz_key_b(row)) << 4;
        vA[i] = row * K + oA;
        vB[i] = row * K + oB;
        tA[i] = oA >= a.k_rem;
        tB[i] = oB >= a.k_rem;
      }
      Tile F = tile_at(0);
      __amdgpu_buffer_rsrc_t dA, dB;
      int rotF = 0, steps = 0, nd = 0;       // nd: fetches of this wave per K block
      bool nt = false;
      auto point = [&]() __attribute__((always_inline)) {              // bounded views of tile F
        const int n_rem = N - F.n0;
        dA = uniform_rsrc(a.A + F.grow * K, F.rows * K);
        dB = uniform_rsrc(a.B + ((int64_t)F.g * N + F.n0) * K, (n_rem < BN ? n_rem : BN) * K);
        rotF = k_rotation(a, F.n0);
        steps = (F.rows + 31) >> 5;
        nd = (8 + steps - p + 2) / 3 * 4;
        nt = F.once && a.b_lines;
      };
      if (F.rows) point();
      int itF = 0, kF = 0, stF = 0, issued = 0;
      int out1 = 0;                          // fetches of the newest K block
      auto advance = [&]() __attribute__((always_inline)) {
        out1 = 0;
        if (F.rows) {
          const int kb = k_wrapped(kF + rotF, KB);
          const bool last = kb == KB - 1;
          uint8_t* const st = lds + stF * Cfg::STAGE_BYTES;
          // (the range check adds the scalar part of an offset: rows past the views' ends are not read)
#pragma unroll
          for (int u = 0; u < 3; ++u) {      // weight units p, p + 3, p + 6
            const int unit = p + 3 * u;
            if (unit < 8) {
              uint8_t* const dst = st + Cfg::A_BYTES + unit * 4096;
              const int so = kb * 128 + unit * 32 * K;
              if (nt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(dst + i * 1024), 16, last && tB[i] ? GG_OOB_OFFSET : vB[i], so, 0, 2 | 16);
              } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(dst + i * 1024), 16, last && tB[i] ? GG_OOB_OFFSET : vB[i], so, 0, 0);
              }
            }
          }
#pragma unroll
          for (int u = 2; u < 5; ++u) {      // activation units: p + 3 u - 8
            const int unit = p + 3 * u - 8;
            if (unit >= 0 && unit < steps) {
              uint8_t* const dst = st + unit * 4096;
              const int so = kb * 128 + unit * 32 * K;
#pragma unroll
              for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(dA, GG_LDS_PTR(dst + i * 1024), 16, last && tA[i] ? GG_OOB_OFFSET : vA[i], so, 0, 0);
            }
          }
          out1 = nd;
          ++issued;
          stF = stF + 1 == S ? 0 : stF + 1;
          if (++kF == KB) {
            kF = 0;
            F = tile_at(++itF);
            if (F.rows) point();
          }
        }
      };
#pragma nounroll
      for (int s = 0; s < S - 1; ++s) advance();
      for (int j = 0;; ++j) {
        // block j has landed: only the fetches of block j + 1 may still be in flight
        if (out1 == 20) wait_vmcnt<20>();
        else if (out1 == 16) wait_vmcnt<16>();
        else if (out1 == 12) wait_vmcnt<12>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();        // block j can be read; block j - 1 has been, its buffer is free
        asm volatile("" ::: "memory");
        if (j == issued) return;             // the barrier of a block that does not exist: see the multiplying waves
        advance();
      }
    }

    // ======== the wave that makes the factors ======================================================================
    // Lane 2 i + c takes K blocks 4 c .. 4 c + 3 of the chunk, of rows i, 32 + i, ...
    const bool km = a.sa_kmajor != 0;
    const int nb_all = (N + 127) >> 7;
    const int s_i = l >> 1, s_c = l & 1;
    constexpr int SG = BM / 32;
    v4f sa_c[SG], sb0_c, sb1_c, sa_n[SG], sb0_n, sb1_n;                // the chunk in use, the one after it
#pragma unroll
    for (int i = 0; i < SG; ++i) sa_c[i] = sa_n[i] = (v4f){0.f, 0.f, 0.f, 0.f};
    sb0_c = sb1_c = sb0_n = sb1_n = (v4f){0.f, 0.f, 0.f, 0.f};
    Tile L = tile_at(0);                     // tile and first K block of the chunk after the one in use
    int itL = 0, kL = 0;
    auto load4 = [](__amdgpu_buffer_rsrc_t d, int vo) __attribute__((always_inline)) -> v4f {
      return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(d, vo, 0, 0));
    };
    auto load_chunk = [&]() __attribute__((always_inline)) {
      const int nb_rem = nb_all - (L.n0 >> 7);
      const __amdgpu_buffer_rsrc_t dSA = uniform_rsrc((const uint8_t*)a.SA + L.grow * a.sa_row_stride, L.rows ? sa_view_bytes(a, L.grow, L.rows) : 0);
      const __amdgpu_buffer_rsrc_t dSB = uniform_rsrc(a.SB + ((int64_t)L.g * nb_all + (L.n0 >> 7)) * KB, L.rows ? (nb_rem < BN / 128 ? nb_rem : BN / 128) * KB * 4 : 0);
      // This lane's four K blocks.  (With a rotated K loop the number of K blocks is a multiple of four, so four neighbours
      // never wrap.)  What a piece takes from the next row, or past the last K block, meets no operand.
      const int k4 = kL + 4 * s_c, kp = k_wrapped(k4 + k_rotation(a, L.n0), KB);
#pragma unroll
      for (int i = 0; i < SG; ++i) {
        const int row = 32 * i + s_i;
        if (km) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            sa_n[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(dSA, k4 + e < KB && row < L.rows ? row * 4 + (kp + e) * a.sa_kb_stride : GG_OOB_OFFSET, 0, 0));
        } else {
          sa_n[i] = load4(dSA, k4 < KB ? row * a.sa_row_stride + kp * 4 : GG_OOB_OFFSET);
        }
      }
      sb0_n = load4(dSB, k4 < KB ? kp * 4 : GG_OOB_OFFSET);
      sb1_n = load4(dSB, k4 < KB ? (KB + kp) * 4 : GG_OOB_OFFSET);
    };
    load_chunk();
    auto pick = [](v4f x, int e) __attribute__((always_inline)) -> float { return e == 0 ? x[0] : e == 1 ? x[1] : e == 2 ? x[2] : x[3]; };
    int kW = 0, stW = 0, made = 0;
    bool ended = false;
    // the factors of the next K block, and its tile where it is the first of one
    auto advance = [&]() __attribute__((always_inline)) {
      if (ended) return;
      if (kW == 0) {
        if (l == 0) *(v4i*)(lds + Cfg::INFO_BASE + stW * 16) = (v4i){L.rows, L.n0, (int)L.grow, 0};
        if (L.rows == 0) { ended = true; return; }
      }
      if ((kW & 7) == 0) {
#pragma unroll
        for (int i = 0; i < SG; ++i) sa_c[i] = sa_n[i];
        sb0_c = sb0_n;
        sb1_c = sb1_n;
        kL += 8;
        if (kL >= KB) {
          kL = 0;
          L = tile_at(++itL);
        }
        load_chunk();
      }
      if (s_c == ((kW & 7) >> 2)) {
        float* const f = (float*)(lds + stW * Cfg::STAGE_BYTES + Cfg::A_BYTES + Cfg::B_BYTES) + s_i;
        const float sb0 = pick(sb0_c, kW & 3), sb1 = pick(sb1_c, kW & 3);
#pragma unroll
        for (int i = 0; i < SG; ++i) {
          const float sa = pick(sa_c[i], kW & 3);
          f[32 * i] = sa * sb0;
          f[32 * i + BM] = sa * sb1;
        }
      }
      ++made;
      stW = stW + 1 == S ? 0 : stW + 1;
      kW = kW + 1 == KB ? 0 : kW + 1;
    };
#pragma nounroll
    for (int s = 0; s < S - 1; ++s) advance();
    for (int j = 0;; ++j) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (ended && j == made) return;
      advance();
    }
  }

  // ======== multiplying waves ======================================================================================
  const int r = l & 15, q = l >> 4;
  const int wm = w / WN, wn = w % WN;
  // wave row wm takes the 16-row blocks wm, wm + 2, ... of a tile
  const int keyA = swz_key_a(r), rowB = 8 * (r >> 2) + (r & 3), keyB = swz_key_b(rowB);
  const int aRd0 = (wm * 16 + r) * 128 + (((2 * q) ^ keyA) << 4), aRd1 = (wm * 16 + r) * 128 + (((2 * q + 1) ^ keyA) << 4);
  const int bRd0 = Cfg::A_BYTES + (wn * Cfg::WTN + rowB) * 128 + (((2 * q) ^ keyB) << 4);
  const int bRd1 = Cfg::A_BYTES + (wn * Cfg::WTN + rowB) * 128 + (((2 * q + 1) ^ keyB) << 4);
  const int sRd = Cfg::A_BYTES + Cfg::B_BYTES + (((wn * Cfg::WTN) >> 7) * BM + wm * 16 + r) * 4;
  // Rows of matrix instructions: row i < TM - 1 is 32-row step TM - 1 - i of the tile, the last row is step 0, which every tile
  // has: the steps that a tile does not have are left out at the front.  Row i's activation fragment goes through register
  // set i % 2; with an odd number of rows the last has a set of its own, so that the next K block's first fragment always
  // finds set 0 free.
  auto step_of = [](int i) constexpr { return TM - 1 - i == 0 ? 0 : TM - 1 - i; };
  auto slot = [](int i) constexpr { return TM % 2 && i == TM - 1 ? 2 : i & 1; };
  // (of the K block that is multiplied next) the weight fragments, the first activation fragment, the factors
  v8i bfr[TN], afr[3];
  // Factors of the rows: of steps 1 .. 4 read with the fragments; that of step 0, which the last row needs, during the block
  // itself, so that the register still holds the block's factor when its last product is added in the next block.
  static_assert(TM == 5, "four factors and one");
  v2f s12, s34;
  float s0 = 0.f;
  auto s = [&](int m) __attribute__((always_inline)) -> float { return m == 0 ? s0 : m < 3 ? s12[m - 1] : s34[m - 3]; };
  auto read_s = [&](const uint8_t* st) __attribute__((always_inline)) {
    const float* const f = (const float*)(st + sRd);
    s12 = (v2f){f[32], f[64]};
    s34 = (v2f){f[96], f[128]};
  };
  auto frag = [&](const uint8_t* p0, const uint8_t* p1) __attribute__((always_inline)) -> v8i {
    const v4i lo = *(const v4i*)p0;
    const v4i hi = *(const v4i*)p1;
    return (v8i){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  };
  auto read_b = [&](int j, const uint8_t* st) __attribute__((always_inline)) -> v8i {
    const int o = (32 * (j >> 1) + 4 * (j & 1)) * 128;
    return frag(st + bRd0 + o, st + (bRd0 ^ 16) + o);
  };
  auto read_a = [&](int mt, const uint8_t* st) __attribute__((always_inline)) -> v8i { return frag(st + aRd0 + mt * 4096, st + (aRd0 ^ 16) + mt * 4096); };

  __builtin_amdgcn_s_barrier();              // block 0 can be read
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < TN; ++j) bfr[j] = read_b(j, lds);
  afr[0] = read_a(step_of(0), lds);
  read_s(lds);
  int stage = 0;

  for (;;) {
    const v4i info = *(const v4i*)(lds + Cfg::INFO_BASE + stage * 16);
    const int rows = __builtin_amdgcn_readfirstlane(info.x), n0 = __builtin_amdgcn_readfirstlane(info.y), grow = __builtin_amdgcn_readfirstlane(info.z);
    if (rows == 0) return;
    const int steps = (rows + 31) >> 5;
    v4f acc[TM][TN];
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[mt][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    // product of a row's last matrix instruction: added behind the next row's first.  (Where the row in front of a row was
    // left out, what is added there goes into accumulators that are never stored.)
    v4f pend = {0.f, 0.f, 0.f, 0.f};
    s0 = 0.f;

#pragma nounroll
    for (int kb = 0; kb < KB; ++kb) {
      const int stage1 = stage + 1 == S ? 0 : stage + 1;
      const uint8_t* const st = lds + stage * Cfg::STAGE_BYTES;
      const uint8_t* const st1 = lds + stage1 * Cfg::STAGE_BYTES;
      // One row: 4 matrix instructions, each with the 4 FMAs of the one before it behind it.  One scheduling region per
      // matrix instruction: the software pipeline is written out in the source.
      auto row = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, m = step_of(i), m_pend = step_of(i == 0 ? TM - 1 : i - 1);
        constexpr bool LAST = i == TM - 1;
        v4f p[TN];
        static_for<0, TN>([&](auto jc) __attribute__((always_inline)) {
          constexpr int j = decltype(jc)::value;
          p[j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bfr[j], afr[slot(i)], (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
          // (nothing in this block of code uses a row's last product: the empty asm keeps the instruction from being moved behind
          // the refill of its operand)
          if constexpr (j == TN - 1) asm volatile("" : "+v"(p[j]));
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (LAST) bfr[j] = read_b(j, st1);
          if constexpr (i > 0 && j == 0) acc[m_pend][TN - 1] += pend * s(m_pend);
          if constexpr (j > 0) acc[m][j - 1] += p[j - 1] * s(m);
          __builtin_amdgcn_sched_barrier(0);
        });
        pend = p[TN - 1];
      };
      acc[0][TN - 1] += pend * s0;
      asm volatile("" : "+v"(acc[0][TN - 1]));       // here, not where the accumulator is used next
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, TM - 1>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        afr[slot(i + 1)] = read_a(step_of(i + 1), st);
        if constexpr (i == 0) s0 = *(const float*)(st + sRd);
        __builtin_amdgcn_sched_barrier(0);
        if (steps > step_of(i)) row(ic);
        __builtin_amdgcn_sched_barrier(0);
      });
      // this wave has read all of block kb; block kb + 1 can be read (past the last block of the last tile: LDS that
      // nobody writes any more, read and not used)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      afr[0] = read_a(step_of(0), st1);
      __builtin_amdgcn_sched_barrier(0);
      row(std::integral_constant<int, TM - 1>{});
      read_s(st1);
      stage = stage1;
    }
    acc[0][TN - 1] += pend * s0;

    // ---- epilogue: bfloat16 (or binary16), round to nearest even.  The lane (q, r) holds 16 bytes of row r and columns 8 q ..,
    // and as much of columns 32 + 8 q .. .  Lane 8 i + c of a store takes piece c of row i (or 8 + i) instead, so that a store
    // writes 8 whole 128-byte lines: the halves of a 16-lane row trade registers, then the pieces change lanes.  (Stores of 64
    // bytes of 16 rows: 16 groups of 250 rows, N = 3328, K = 640 26.5 us, 22.5 with these; 32 of 512, N = 7168, K = 2048 297, 288.)
    const int n_rem = N - n0;
    const __amdgpu_buffer_rsrc_t dC = uniform_rsrc(a.C + (int64_t)grow * N + n0, rows * N * 2 - n0 * 2);
    const int cSrc = (16 * (l & 3) + (l >> 3) + 8 * ((l >> 2) & 1)) * 4;
    const int col = wn * Cfg::WTN + 8 * (l & 7);
    // (opaque: computed once per kernel, the offsets of all stores would be kept in memory, and reading one back waits for all
    // stores before it)
    unsigned vC = col < n_rem ? (unsigned)((16 * wm + (l >> 3)) * N + col) * 2 : GG_OOB_OFFSET;
    asm volatile("" : "+v"(vC));
    auto store = [&](auto f16_c, auto aux_c) __attribute__((always_inline)) {
      constexpr bool f16 = decltype(f16_c)::value;
      constexpr int kAux = decltype(aux_c)::value;
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
        if (mt < steps) {
          v4i x, y;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int lo = pack2_rne(acc[mt][e >> 1][2 * (e & 1)], acc[mt][e >> 1][2 * (e & 1) + 1], f16);
            const int hi = pack2_rne(acc[mt][2 + (e >> 1)][2 * (e & 1)], acc[mt][2 + (e >> 1)][2 * (e & 1) + 1], f16);
            x[e] = __builtin_amdgcn_ds_bpermute(cSrc, __builtin_amdgcn_update_dpp(lo, hi, 0x128, 0xF, 0xC, false));   // row_ror:8
            y[e] = __builtin_amdgcn_ds_bpermute(cSrc, __builtin_amdgcn_update_dpp(hi, lo, 0x128, 0xF, 0x3, false));
          }
          __builtin_amdgcn_raw_buffer_store_b128(x, dC, (int)(vC + mt * 64 * N), 0, kAux);
          __builtin_amdgcn_raw_buffer_store_b128(y, dC, (int)(vC + mt * 64 * N + 16 * N), 0, kAux);
        }
      }
    };
    // Streaming cache policy (nt sc1): C is written once and not read here.  Rows of C that are no whole lines take the default
    // policy instead, under which the L2 puts the pieces of a line together.
    constexpr std::integral_constant<int, 2 | 16> streamed{};
    constexpr std::integral_constant<int, 0> cached{};
    if (a.out_f16) {
      if (a.c_lines) store(std::true_type{}, streamed);
      else store(std::true_type{}, cached);
    } else {
      if (a.c_lines) store(std::false_type{}, streamed);
      else store(std::false_type{}, cached);
    }
  }
}

}  // namespace gg
