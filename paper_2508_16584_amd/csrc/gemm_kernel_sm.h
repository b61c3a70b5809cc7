// Third kernel of the padding-free block-scaled FP8 grouped GEMM (same operation, same bounds and the same arithmetic
// per element as gemm_kernel.h, so the same bits): small tiles, for problems whose tiles of the other two kernels would
// leave most of the chip idle, or whose K loop would be a chain of latencies.
//
// With few rows per group 256-wide tiles are few (8 groups of 8 rows, N = 4096: 128 tiles on 256 compute units), and a
// K step of the other kernels takes 0.4 (first) to 0.8 us (fourth) however little there is to multiply: wait for the fetches,
// barrier, LDS reads, matrix instructions and FMAs follow one another.  Here
//  * a workgroup has 4 waves and a tile of 32 x 64, 32 x 128 or 64 x 128 (with the activation epilogue 32 or 64 rows of 256
//    weight rows); several workgroups share a compute unit;
//  * a wave multiplies K block kb out of registers, into which the block was read during the step before; the barrier at
//    the top of the step publishes block kb + 1, whose fragments refill the registers right behind the matrix
//    instructions that used them, so no LDS latency stands between the barrier and the first matrix instruction;
//  * the buffer that block kb came from is free at once: its fetch of block kb + STAGES is issued in the same step;
//  * fetches are one stream of K blocks that runs on from tile to tile, with a cursor of its own on the tile list: no
//    prologue after a workgroup's first tile, whatever the number of K blocks (1 included);
//  * scales come four K blocks at a time into a ring of chunk buffers (row-major: 16-byte pieces of a row;
//    K-block-major: one K block per wave), outside the wait counts: a wave waits for a few operations more than it needs
//    at times, never for fewer.
#pragma once
#include "gemm_kernel.h"
#include "quant_kernel.h"

namespace gg {

// FUSE: the first GEMM of an expert MLP with the activation and the quantiser in its epilogue, as in the second kernel:
// the tile's 256 weight rows are 128 gate rows and the 128 matching up rows, and wave w holds gate and up of activation
// columns [32 w, 32 w + 32).
template <int BM_, int BN_, int WM_, int WN_, int STAGES_, bool FUSE_ = false>
struct SmCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, STAGES = STAGES_;
  static constexpr bool FUSE = FUSE_;
  static constexpr int NW = 4, NT = 256;
  static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
  static constexpr int A_ITERS = (BM + 31) / 32, B_ITERS = BN / 32;    // 8-row slabs per wave; rows past BM are past every tile's end: zeros, no traffic
  static constexpr int ND = A_ITERS + B_ITERS;                         // fetches per wave and K block
  static constexpr int A_BYTES = A_ITERS * 32 * 128, STAGE_BYTES = A_BYTES + BN * 128;
  // a chunk: four K blocks of scales.  K blocks kb + 1 .. kb + STAGES are live while block kb is multiplied, and each may
  // have a chunk of its own (K <= 128)
  static constexpr int SA_BANDS = (BM + 63) / 64, SA_CHUNK = SA_BANDS * 1024, CHUNK = SA_CHUNK + 256, CHUNKS = STAGES;
  static constexpr int CHUNK_BASE = STAGES * STAGE_BYTES;
  static constexpr int RED_BASE = CHUNK_BASE + CHUNKS * CHUNK;          // FUSE: per row, the 4 waves' partial maxima
  static constexpr int LDS_BYTES = RED_BASE + (FUSE ? BM * NW * 4 : 0);
  static constexpr int WG_PER_CU = 160 * 1024 / LDS_BYTES < 4 ? 160 * 1024 / LDS_BYTES : 4;
  static_assert(WM * WN == NW && BM % (16 * WM) == 0 && BN % (32 * WN) == 0 && (FUSE ? BN == 256 && WN == 4 : BN <= 128), "wave tiles of 16 x 32, one scale block of B");
  static_assert(STAGES >= 3 && (STAGES - 1) * ND + 2 * STAGES + 16 < 63, "vmcnt is a 6-bit counter");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// BSTREAM: weight fetches with the streaming cache policy (groups of one row tile on average); RAGGED: N not a multiple
// of the tile width or K of 128 - both as in the first kernel.
template <class Cfg, bool RAGGED = false, bool BSTREAM = false>
__global__ void __launch_bounds__(Cfg::NT, Cfg::WG_PER_CU) gg_gemm_sm_kernel(const GemmArgs a) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, WN = Cfg::WN, NW = Cfg::NW, TM = Cfg::TM, TN = Cfg::TN, S = Cfg::STAGES, ND = Cfg::ND;
  constexpr int kBAux = BSTREAM ? (2 | 16) : 0;
  constexpr int TILE_COLS = Cfg::FUSE ? 128 : BN;      // output columns of a tile
  static_assert(!(Cfg::FUSE && RAGGED), "the activation epilogue takes whole blocks only");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int r = l & 15, q = l >> 4;
  const int wm = w / WN, wn = w % WN;
  const int K = a.K, KB = a.KB, N = a.N;

  // ---- per-lane constants of the fetches and of the operand reads: see the first kernel
  const int f_row = w * 8 + (l >> 3);                                  // + 32 i; the swizzle keys repeat every 32 rows
  const int offA = ((l & 7) ^ swz_key_a(f_row)) << 4, offB = ((l & 7) ^ swz_key_b(f_row)) << 4;
  const int vA = f_row * K + offA, vB = f_row * K + offB;
  const bool a_tail = RAGGED && offA >= a.k_rem, b_tail = RAGGED && offB >= a.k_rem;
  const bool km = a.sa_kmajor != 0;
  const int vSA = l * a.sa_row_stride;                                 // + 64 rows per band
  const int inter = N >> 1;                                            // FUSE: activation columns (N = gate + up rows)
  const int vSB = (l & 3) * 4 + (Cfg::FUSE ? ((l >> 2) & 1) * (inter >> 7) * KB * 4 : 0);
  const int keyA = swz_key_a(r), rowB = 8 * (r >> 2) + (r & 3), keyB = swz_key_b(rowB);
  const int aRd0 = (wm * Cfg::WTM + r) * 128 + (((2 * q) ^ keyA) << 4), aRd1 = (wm * Cfg::WTM + r) * 128 + (((2 * q + 1) ^ keyA) << 4);
  const int bRd0 = Cfg::A_BYTES + (wn * (Cfg::FUSE ? 32 : Cfg::WTN) + rowB) * 128 + (((2 * q) ^ keyB) << 4);
  const int bRd1 = Cfg::A_BYTES + (wn * (Cfg::FUSE ? 32 : Cfg::WTN) + rowB) * 128 + (((2 * q + 1) ^ keyB) << 4);
  // a scale of the chunk: row * sa_rs + (K block % 4) * sa_js (row-major: a row's 16 bytes; K-block-major: a block's rows)
  const int sa_rs = km ? 4 : 16, sa_js = km ? Cfg::SA_BANDS * 256 : 4;
  const int saRd = (wm * Cfg::WTM + r) * sa_rs;

  // ---- the tile list, as in the other kernels; the fetch stream and the arithmetic each have a cursor on it
  struct Tile {
    bool valid;
    int g, n0, rows_valid;
    int64_t grow;
  };
  GroupRows groups;
  groups.init(a, BM, l, true);
  auto tile_at = [&](int it, GroupRows& walk) __attribute__((always_inline)) -> Tile {
    Tile t = {false, 0, 0, 0, 0};
    const int T = walk.unit(a, it);
    if (T == GroupIndex::NONE) return t;
    GroupRows::Group grp;
    if (!walk.find(a, BM, T, grp)) return t;
    const int g = grp.g, base = grp.tiles_before, row0 = grp.row0, Mg = grp.rows;
    const int mtiles = row_tiles(Mg, BM);
    const int local = T - base;
    const int per_chunk = mtiles * a.n_chunk;
    const int nc = local / per_chunk;
    const int rem = local - nc * per_chunk;
    int csz = a.n_tiles - nc * a.n_chunk;
    csz = csz < a.n_chunk ? csz : a.n_chunk;
    const int mtile = rem / csz;
    t.g = g;
    t.n0 = (nc * a.n_chunk + (rem - mtile * csz)) * TILE_COLS;
    t.rows_valid = Mg - mtile * BM < BM ? Mg - mtile * BM : BM;
    t.grow = (int64_t)row0 + mtile * BM;
    t.valid = true;
    return t;
  };
  // ---- the fetch stream
  const int nb_all = (N + 127) >> 7;
  GroupRows groupsF = groups;   // (the registers are shared: only the walk past 256 groups is a cursor's own)
  int itF = 0;
  Tile F = tile_at(0, groupsF);
  if (!F.valid) return;
  __amdgpu_buffer_rsrc_t dA, dB, dSA, dSB;
  int kF = 0, rotF = 0, ch_fetch = 0;
  auto point = [&]() __attribute__((always_inline)) {      // views of tile F (of length zero when there is none): see the first kernel
    const int n_rem = N - F.n0;
    dA = uniform_rsrc(a.A + F.grow * K, F.valid ? F.rows_valid * K : 0);
    dB = uniform_rsrc(a.B + ((int64_t)F.g * N + F.n0) * K, F.valid ? (Cfg::FUSE ? inter + 128 : RAGGED && n_rem < BN ? n_rem : BN) * K : 0);
    dSA = uniform_rsrc((const uint8_t*)a.SA + F.grow * a.sa_row_stride, F.valid ? sa_view_bytes(a, F.grow, F.rows_valid) : 0);
    dSB = uniform_rsrc(a.SB + ((int64_t)F.g * nb_all + (F.n0 >> 7)) * KB, F.valid ? (Cfg::FUSE ? (inter >> 7) + 1 : 1) * KB * 4 : 0);
    rotF = k_rotation(a, F.n0);
  };
  point();
  auto next_chunk = [](int c) __attribute__((always_inline)) -> int { return c + Cfg::CHUNK == Cfg::CHUNKS * Cfg::CHUNK ? 0 : c + Cfg::CHUNK; };
  auto fetch_next = [&](int stage) __attribute__((always_inline)) {
    const int kb = k_wrapped(kF + rotF, KB);
    if ((kF & 3) == 0) {
      // four K blocks of scales; those past the last K block, and what a 16-byte piece takes from the next row, are not read
      ch_fetch = next_chunk(ch_fetch);
      uint8_t* const ch = lds + Cfg::CHUNK_BASE + ch_fetch;
      if (km) {
#pragma unroll
        for (int b = 0; b < Cfg::SA_BANDS; ++b)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(dSA, GG_LDS_PTR(ch + (w * Cfg::SA_BANDS + b) * 256), 4, kF + w < KB ? vSA + b * 256 : GG_OOB_OFFSET, (kF + w < KB ? kb + w : 0) * a.sa_kb_stride, 0, 0);
      } else if (w < Cfg::SA_BANDS) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(dSA, GG_LDS_PTR(ch + w * 1024), 16, vSA + w * 64 * a.sa_row_stride, kb * 4, 0, 0);
      }
      if (w == NW - 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(dSB, GG_LDS_PTR(ch + Cfg::SA_CHUNK), 4, vSB, kb * 4, 0, 0);
    }
    uint8_t* const st = lds + stage * Cfg::STAGE_BYTES;
    const bool last = RAGGED && kb == KB - 1;
#pragma unroll
    for (int i = 0; i < Cfg::B_ITERS; ++i) {
      if constexpr (RAGGED)      // the row part in the lane offset: rows past N fail the range check
        __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(st + Cfg::A_BYTES + (w + i * NW) * 1024), 16, last && b_tail ? GG_OOB_OFFSET : vB + i * 32 * K, kb * 128, 0, kBAux);
      else {
        const int rows = i * 32 + (Cfg::FUSE && i >= 4 ? inter - 128 : 0);      // FUSE: slabs 4 .. 7 are the up rows
        __builtin_amdgcn_raw_ptr_buffer_load_lds(dB, GG_LDS_PTR(st + Cfg::A_BYTES + (w + i * NW) * 1024), 16, vB, kb * 128 + rows * K, 0, kBAux);
      }
    }
#pragma unroll
    for (int i = 0; i < Cfg::A_ITERS; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(dA, GG_LDS_PTR(st + (w + i * NW) * 1024), 16, last && a_tail ? GG_OOB_OFFSET : vA + i * 32 * K, kb * 128, 0, 0);
    if (++kF == KB) {
      kF = 0;
      if (F.valid) F = tile_at(++itF, groupsF);
      point();
    }
  };

  // ---- registers of the K block that is multiplied next
  v8i af[TM], bf[TN];
  float sa[TM], sb, sb_up = 0.f;       // sb_up: FUSE, the up rows' weight scale
  int ch_read = 0, sc = 0;       // chunk of that block, LDS offset of its scales
  auto frag = [&](const uint8_t* p0, const uint8_t* p1) __attribute__((always_inline)) -> v8i {
    const v4i lo = *(const v4i*)p0;
    const v4i hi = *(const v4i*)p1;
    return (v8i){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  };
  auto read_b = [&](int j, const uint8_t* st) __attribute__((always_inline)) {
    const int o = ((Cfg::FUSE ? 128 : 32) * (j >> 1) + 4 * (j & 1)) * 128;
    bf[j] = frag(st + bRd0 + o, st + bRd1 + o);
  };
  auto read_a = [&](int mt, const uint8_t* st) __attribute__((always_inline)) { af[mt] = frag(st + aRd0 + mt * 2048, st + aRd1 + mt * 2048); };
  auto read_scales = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) sa[mt] = *(const float*)(lds + sc + saRd + mt * 16 * sa_rs);
  };
  auto next_scales = [&](bool new_chunk) __attribute__((always_inline)) {
    if (new_chunk) ch_read = next_chunk(ch_read);
    sc = new_chunk ? Cfg::CHUNK_BASE + ch_read : sc + sa_js;
  };

  int k_read = 0;                // K block (within its tile) in the registers
  auto read_sb = [&]() __attribute__((always_inline)) {
    const uint8_t* const p = lds + Cfg::CHUNK_BASE + ch_read + Cfg::SA_CHUNK + (k_read & 3) * 4;
    sb = *(const float*)p;
    if constexpr (Cfg::FUSE) sb_up = *(const float*)(p + 16);
  };
#pragma nounroll
  for (int s = 0; s < S; ++s) fetch_next(s);
  wait_vmcnt<(S - 1) * ND>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  next_scales(true);
#pragma unroll
  for (int j = 0; j < TN; ++j) read_b(j, lds);
#pragma unroll
  for (int mt = 0; mt < TM; ++mt) read_a(mt, lds);
  read_scales();
  read_sb();
  int stage = 0;                 // the buffer the block in the registers came from

  for (int it = 0;; ++it) {
    const Tile cur = tile_at(it, groups);
    if (!cur.valid) break;
    v4f acc[TM][TN];
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[mt][j] = (v4f){0.f, 0.f, 0.f, 0.f};

    for (int kb = 0; kb < KB; ++kb) {
      // this wave's reads of block kb are back and its part of block kb + 1 has landed (newer: the fetches of blocks
      // kb + 2 .. kb + S - 1, and scales and stores that only make the wait longer) ...
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wait_vmcnt<(S - 2) * ND>();
      __builtin_amdgcn_s_barrier();       // ... and everybody's: block kb's buffer is free, block kb + 1 can be read
      asm volatile("" ::: "memory");
      fetch_next(stage);
      stage = stage + 1 == S ? 0 : stage + 1;
      const uint8_t* const st = lds + stage * Cfg::STAGE_BYTES;
      k_read = kb + 1 == KB ? 0 : kb + 1;
      next_scales((k_read & 3) == 0);
      __builtin_amdgcn_sched_barrier(0);

      float s[TM], s_up[TM];
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
        s[mt] = sa[mt] * sb;
        if constexpr (Cfg::FUSE) s_up[mt] = sa[mt] * sb_up;
      }
      v4f p[TM][TN];
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          p[mt][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bf[j], af[mt], (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
          if (mt == TM - 1) read_b(j, st);
        }
        read_a(mt, st);
      }
      read_scales();
      read_sb();
      __builtin_amdgcn_sched_barrier(0);  // the reads are on their way before the FMAs wait for the matrix instructions
#pragma unroll
      for (int mt = 0; mt < TM; ++mt)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[mt][j] += p[mt][j] * (Cfg::FUSE && j >= 2 ? s_up[mt] : s[mt]);
    }

    if constexpr (Cfg::FUSE) {
      // ---- epilogue of the second kernel's activation form: both projections rounded to bfloat16, act = silu(gate) * up,
      // the row's block maximum over lanes and waves, the quantiser.  Lane (q, r) holds 8 neighbouring columns of row r.
      uint8_t* const red = lds + Cfg::RED_BASE;
      int act[TM][4];
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const v4f g = acc[mt][i >> 1], u = acc[mt][2 + (i >> 1)];
          const int e = 2 * (i & 1);
          act[mt][i] = swiglu2(pack2_rne(g[e], g[e + 1], false), pack2_rne(u[e], u[e + 1], false));
          const unsigned t0 = amax_bits_of(__builtin_bit_cast(float, act[mt][i] << 16)), t1 = amax_bits_of(__builtin_bit_cast(float, act[mt][i] & (int)0xFFFF0000));
          top = top > t0 ? top : t0;
          top = top > t1 ? top : t1;
        }
        unsigned o = (unsigned)__shfl_xor((int)top, 16);
        top = top > o ? top : o;
        o = (unsigned)__shfl_xor((int)top, 32);
        top = top > o ? top : o;
        if (q == 0) *(unsigned*)(red + ((wm * Cfg::WTM + mt * 16 + r) * NW + wn) * 4) = top;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();        // the K steps' barriers keep the next tile's maxima away from this one's reads
      asm volatile("" ::: "memory");
      const __amdgpu_buffer_rsrc_t dQ = __builtin_amdgcn_make_buffer_rsrc((void*)(a.A2 + cur.grow * inter + cur.n0), 0, cur.rows_valid * inter - cur.n0, GG_RSRC_FLAGS);
      const __amdgpu_buffer_rsrc_t dAct = __builtin_amdgcn_make_buffer_rsrc((void*)(a.act_out + cur.grow * inter + cur.n0), 0, a.act_out ? (cur.rows_valid * inter - cur.n0) * 2 : 0, GG_RSRC_FLAGS);
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
        const int row = wm * Cfg::WTM + mt * 16 + r;
        const v4i m = *(const v4i*)(red + row * NW * 4);
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) top = top > (unsigned)m[i] ? top : (unsigned)m[i];
        const float amax = block_amax(top);
        const float scale = amax / 448.0f, inv = 448.0f / amax;
        float v[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[2 * i] = __builtin_bit_cast(float, act[mt][i] << 16);
          v[2 * i + 1] = __builtin_bit_cast(float, act[mt][i] & (int)0xFFFF0000);
        }
        const int o = row * inter + wn * 32 + 8 * q;
        __builtin_amdgcn_raw_buffer_store_b64((v2i){e4m3x4_of(v, inv), e4m3x4_of(v + 4, inv)}, dQ, o, 0, 0);
        if (a.act_out) __builtin_amdgcn_raw_buffer_store_b128((v4i){act[mt][0], act[mt][1], act[mt][2], act[mt][3]}, dAct, o * 2, 0, 0);
        if (wn == 0 && q == 0 && row < cur.rows_valid) a.SA2[(cur.grow + row) * a.sa2_row_stride + (int64_t)(cur.n0 >> 7) * a.sa2_kb_stride] = scale;
      }
      continue;
    }

    // ---- epilogue: as in the first kernel
    const int n_rem = N - cur.n0;
    const __amdgpu_buffer_rsrc_t dC = __builtin_amdgcn_make_buffer_rsrc((void*)(a.C + cur.grow * N + cur.n0), 0, cur.rows_valid * N * 2 - cur.n0 * 2, GG_RSRC_FLAGS);
    const int cSrc = (16 * (l & 3) + (l >> 2)) * 4;
    const bool f16 = a.out_f16 != 0;
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      const int row = wm * Cfg::WTM + 16 * mt + (l >> 2);
#pragma unroll
      for (int pr = 0; pr < TN / 2; ++pr) {
        const v4f x = acc[mt][2 * pr], y = acc[mt][2 * pr + 1];
        v4i out;
        out.x = __builtin_amdgcn_ds_bpermute(cSrc, pack2_rne(x[0], x[1], f16));
        out.y = __builtin_amdgcn_ds_bpermute(cSrc, pack2_rne(x[2], x[3], f16));
        out.z = __builtin_amdgcn_ds_bpermute(cSrc, pack2_rne(y[0], y[1], f16));
        out.w = __builtin_amdgcn_ds_bpermute(cSrc, pack2_rne(y[2], y[3], f16));
        const int col = wn * Cfg::WTN + 32 * pr + 8 * (l & 3);
        __builtin_amdgcn_raw_buffer_store_b128(out, dC, !RAGGED || col < n_rem ? row * N * 2 + col * 2 : GG_OOB_OFFSET, 0, 2 | 16);
      }
    }
  }
  wait_vmcnt<0>();     // fetches past the last tile still write zeros into this workgroup's LDS
}

}  // namespace gg
