// The weight-gradient GEMM in tiles of 256 features x 256 rows of dY^T, for groups of many tokens (definition, layouts and
// epilogue: wgrad_kernel.h; the same arithmetic per element, so the same bits).
//
// The 256 x 128 tiles fetch 48 KB per token block for 32768 outputs; here it is 64 KB for 65536, and the operand reads out of LDS
// per output fall by a quarter.  8 waves of 64 features x 128 rows hold 128 accumulators and, of a block, the feature
// fragments; of the eight dY^T fragments a wave holds the one it multiplies and the next.  A block is eight rows of four
// matrix instructions (a dY^T fragment with the four feature fragments), each followed by the four factors sdy * sx of its
// products and the FMAs of the product before it: one scheduling region per matrix instruction, the software pipeline is
// written out in the source.
//
// LDS holds two buffers of the X tile (the registers are the third), a ring of five halves of the dY^T tile and the scales of three
// blocks.  There are two barriers per block, in front of rows 3 and 7, and the fetches between two of them go to what the
// first has freed:
//   row 7 of block b - 1, rows 0 .. 2 of b:  half 0 of dY^T of block b + 2        (frees X of block b and half 0 of b)
//   rows 3 .. 6:                             X, scales and half 1 of block b + 2  (frees half 1 of b, publishes block b + 1)
// Tokens outside the group: a lane whose 16 tokens are all outside fetches zeros; where a bound lies inside 16 tokens the wave
// that fetched them clears the rest in LDS, before the barrier that publishes them.
// A tile's last block is a copy of its own that stores each row of sums behind the row after it: only the last four of 32
// stores per wave wait for the block's end (8 groups of 1000 tokens, 4096 x 7168, fp32: 348 -> 340 us).
//
// What bounds it: 8 vector instructions per matrix instruction (45 cycles for 32 of the matrix pipe, in a register-only loop: 175 us
// on those 8 groups; with LDS reads and barriers 225), stores (70) and fetches (55) that hide only in part (development builds
// with parts left out, which are not kept).  237 vector registers; 37 scalar ones are spilled into lanes of vector registers.
// Against the 256 x 128 tiles, inputs rotated through 276 MB: 8 groups, 8192 tokens, 4096 x 7168, fp32 451 -> 404 us, 389 with the
// operands brought in ahead, bfloat16 374 -> 337; one group of 8192, 8192 x 8192 618 -> 586.
#pragma once
#include "wgrad_kernel.h"

namespace gg {

// Brings the operands into the last-level cache ahead of their fetches.  Those take 128 bytes of each of 500 rows per token block,
// a row pitch apart, in the order in which the tiles come up and beside the stores of the gradients: from memory they cost far
// more than their bytes (8 groups, 8000 tokens, 4096 x 7168, fp32: 360 us with the operands in the cache, 433 without).  Here
// every wave of the launch fetches 1 KB pieces of single rows (1024 tokens), in the order of the tokens, into 1 KB of LDS that
// nobody reads: a dozen ahead of its first tile, eight ahead of each tile until all are there.  433 -> 381 us; where the
// operands are in the cache already, 359 -> 361.
struct OperandTouch {
  static constexpr int FIRST = 12, TILE = 8;
  int row, tok, step, first;
  __device__ __forceinline__ void init(const WgradArgs& a, int w) {
    step = 8 * (int)gridDim.x;
    row = first = 8 * (int)blockIdx.x + w;
    tok = a.touch ? 0 : a.M_total;
  }
  __device__ __forceinline__ bool left(const WgradArgs& a) const { return tok < a.M_total; }
  // one piece, or none past the last one: the same number of fetches either way
  __device__ __forceinline__ void piece(const WgradArgs& a, __amdgpu_buffer_rsrc_t dX, __amdgpu_buffer_rsrc_t dY, int l, uint8_t* dump) {
    const bool y = row >= a.K, in = row < a.K + a.N && left(a);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(y ? dY : dX, GG_LDS_PTR(dump), 16, in && tok + 16 * l < a.M_total ? 16 * l : GG_OOB_OFFSET,
                                             __builtin_amdgcn_readfirstlane(in ? (row - (y ? a.K : 0)) * a.M_total + tok : 0), 0, 0);
    if (!left(a)) return;
    row += step;
    if (row >= a.K + a.N) {
      row = first;
      tok = tok > a.M_total - 1024 ? a.M_total : tok + 1024;
    }
  }
};

struct WgradSqCfg {
  static constexpr int TK = 256, TN = 256, NW = 8, NT = 512;
  // X: two buffers of a token block (the registers are the third); dY^T: a ring of five halves of a block; scales of three blocks
  static constexpr int X_BYTES = TK * 128, YH_BYTES = TN / 2 * 128, S_BYTES = (TK + TN) * 4;
  static constexpr int X_BASE = 0, Y_BASE = 2 * X_BYTES, S_BASE = Y_BASE + 5 * YH_BYTES, DUMP_BASE = S_BASE + 3 * S_BYTES;
  static constexpr int LDS_BYTES = DUMP_BASE + 1024;
  static constexpr int ND1 = 2, ND2 = 7;       // fetches per wave in the first and in the second phase of a block
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

template <bool OUT16>
__global__ void __launch_bounds__(WgradSqCfg::NT) gg_wgrad_sq_kernel(const WgradArgs a) {
  using Cfg = WgradSqCfg;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int r = l & 15, q = l >> 4;
  const int wk = w >> 1, wn = w & 1;
  const int M = a.M_total;

  struct Tile {
    bool valid;
    int g, k0, n0, lo, hi, j0, steps;
  };
  const GG_CONST_I32* offc = (const GG_CONST_I32*)a.off;
  const int per_group = a.n_tiles * a.k_tiles;
  // ---- the tile list: group by group, inside a group in columns of 4 k tiles, so that the 32 tiles which an XCD's workgroups have
  // at one time share 1024 + 2048 operand rows in its L2.  Workgroup b runs on XCD b % 8; every XCD takes runs of `slots` tiles.
  //
  // Dealt round by round, a workgroup's share of long and short groups is left to chance: 8 groups of 27 to 2970 tokens, 1.75
  // rounds each, 1.07 to 1.11 of the mean.  With a.balanced the runs are dealt by cost instead, group by group from the most
  // tokens on, to the XCD that has least so far (1.005; 417 -> 401 us).  It takes every wave 0.1 us per group, hence only up to 64
  // groups and for launches of three token blocks per group and workgroup or more.
  // Lane i looks after the group of the (i + 1)th largest cost: `upto` are the tiles that this workgroup
  // gets of it and of those before it, `dealt` its number, this XCD's place among those that get one run of tiles more
  // than others, and the workgroup's tile of the group's last, partial run.
  int upto = 0, dealt = 0;
  const int xcd = (int)(blockIdx.x & 7), runs = a.balanced ? per_group / a.slots : 0, part = a.balanced ? per_group % a.slots : 0;
  if (a.balanced) {
    int cost = -1;
    if (l < a.G) {
      const int lo = clampi(a.off[l], 0, M), hi = clampi(a.off[l + 1], lo, M);
      cost = hi > lo ? 2 * (((hi + 127) >> 7) - (lo >> 7)) + 3 : 3;
    }
    int place = 0;
    for (int j = 0; j < a.G; ++j) {
      const int c = __builtin_amdgcn_readlane(cost, j);
      place += c > cost || (c == cost && j < l);
    }
    // lane 8 x + y compares the loads of XCDs x and y: bit y of byte x of the mask says that y comes before x
    const int x = l >> 3, y = l & 7;
    unsigned load_x = 0, load_y = 0;
    int start = 0;       // start: of this XCD's next partial run
    for (int i = 0; i < a.G; ++i) {
      const int g = __builtin_ctzll(__builtin_amdgcn_ballot_w64(l < a.G && place == i));
      const int c = __builtin_amdgcn_readlane(cost, g);
      const uint64_t before = __builtin_amdgcn_ballot_w64(load_y < load_x || (load_y == load_x && y < x));
      auto load_of = [&](int p) { return (unsigned)c * (unsigned)(a.slots * ((runs >> 3) + (p < (runs & 7))) + (p == (runs & 7) ? part : 0)); };
      load_x += load_of(__builtin_popcount((unsigned)(before >> (8 * x)) & 255));
      load_y += load_of(__builtin_popcount((unsigned)(before >> (8 * y)) & 255));
      const int own = __builtin_popcount((unsigned)(before >> (8 * xcd)) & 255);
      int n = (runs >> 3) + (own < (runs & 7)), in = 0;
      if (own == (runs & 7) && part) {
        in = (int)(blockIdx.x >> 3) - start;
        in += in < 0 ? a.slots : 0;
        n += in < part;
        start += part;
        start -= start >= a.slots ? a.slots : 0;
      }
      upto = l == i ? n : upto;
      dealt = l == i ? g | own << 8 | in << 16 : dealt;
    }
    for (int d = 1; d < 64; d *= 2) {
      const int o = __shfl_up(upto, d);
      upto += l >= d ? o : 0;
    }
  }
  auto tile_at = [&](int it) __attribute__((always_inline)) -> Tile {
    Tile t = {false, 0, 0, 0, 0, 0, 0, 0};
    int T;
    if (a.balanced) {
      const uint64_t past = __builtin_amdgcn_ballot_w64(upto > it);
      if (!past) return t;
      const int i = __builtin_ctzll(past), k = it - (i ? __builtin_amdgcn_readlane(upto, i - 1) : 0);
      const int d = __builtin_amdgcn_readlane(dealt, i), own = (d >> 8) & 255;
      const int local = k < runs >> 3                     ? (k * 8 + xcd) * a.slots + (int)(blockIdx.x >> 3)
                        : k == runs >> 3 && own < (runs & 7) ? ((runs & ~7) + own) * a.slots + (int)(blockIdx.x >> 3)
                                                             : runs * a.slots + (d >> 16);
      T = (d & 255) * per_group + local;
    } else if (a.slots > 0) T = (it * 8 + (int)(blockIdx.x & 7)) * a.slots + (int)(blockIdx.x >> 3);
    else T = it * (int)gridDim.x + (int)blockIdx.x;
    if (T >= a.tiles) return t;
    t.valid = true;
    t.g = T / per_group;
    const int local = T - t.g * per_group;
    const int kc = local / (4 * a.n_tiles), rem = local - kc * 4 * a.n_tiles;
    const int csz = a.k_tiles - 4 * kc < 4 ? a.k_tiles - 4 * kc : 4;
    const int nt = rem / csz;
    t.k0 = (4 * kc + rem - nt * csz) * Cfg::TK;
    t.n0 = nt * Cfg::TN;
    t.lo = clampi(offc[t.g], 0, M);
    t.hi = clampi(offc[t.g + 1], t.lo, M);
    t.j0 = t.lo >> 7;
    t.steps = t.hi > t.lo ? ((t.hi + 127) >> 7) - t.j0 : 0;     // token blocks [j0, j0 + steps)
    return t;
  };

  // ---- fetches
  const __amdgpu_buffer_rsrc_t dX = __builtin_amdgcn_make_buffer_rsrc((void*)a.XT, 0, a.K * M, GG_RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t dY = __builtin_amdgcn_make_buffer_rsrc((void*)a.DYT, 0, a.N * M, GG_RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t dS = w == 0 ? __builtin_amdgcn_make_buffer_rsrc((void*)a.SX, 0, a.K * a.MB * 4, GG_RSRC_FLAGS)
                                           : __builtin_amdgcn_make_buffer_rsrc((void*)a.SDY, 0, a.N * a.MB * 4, GG_RSRC_FLAGS);
  const int slab_row = w * 8 + (l >> 3);                           // + 64 i
  const int chunk = (l & 7) ^ swz_key_a(slab_row);                 // the 16 tokens of a block that this lane fetches
  auto feature_of_slot = [](int s) { return 64 * (s >> 6) + 4 * (s & 15) + ((s >> 4) & 3); };
  const int vX = feature_of_slot(slab_row) * M + chunk * 16;
  const int vY = slab_row * M + chunk * 16;
  const int s_pitch = (w == 0 ? a.K : a.N) * 4;

  Tile F = tile_at(0);
  int itF = 0, sF = 0;
  int f_x = 0, f_y = 0, f_s = 0, f_cut = 0;
  int vXsel = GG_OOB_OFFSET, vYsel = GG_OOB_OFFSET, vSsel = GG_OOB_OFFSET;
  auto fetch_prepare = [&]() __attribute__((always_inline)) {
    while (F.valid && sF >= F.steps) {
      ++itF;
      F = tile_at(itF);
      sF = 0;
    }
    const int first = (F.j0 + sF) * 128;
    f_x = __builtin_amdgcn_readfirstlane(first + F.k0 * M);
    f_y = __builtin_amdgcn_readfirstlane(first + F.n0 * M);
    f_s = __builtin_amdgcn_readfirstlane((F.j0 + sF) * s_pitch + (w == 0 ? F.k0 : F.n0) * 4);
    const int lo = clampi(F.lo - first, 0, 128), hi = clampi(F.hi - first, 0, 128);
    const bool in = F.valid && 16 * chunk < hi && 16 * chunk + 16 > lo;
    vXsel = in ? vX : GG_OOB_OFFSET;
    vYsel = in ? vY : GG_OOB_OFFSET;
    vSsel = F.valid && w < 2 ? l * 16 : GG_OOB_OFFSET;
    f_cut = __builtin_amdgcn_readfirstlane(F.valid && ((lo | hi) & 15) ? lo | hi << 8 : 0);
    ++sF;
  };
  auto fetch_y = [&](int half, int i, int slot) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dY, GG_LDS_PTR(lds + Cfg::Y_BASE + slot * Cfg::YH_BYTES + (w + i * 8) * 1024), 16, vYsel,
                                             f_y + (128 * i + 64 * half) * M, 0, 0);
  };
  auto fetch_x = [&](int i, int buf) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dX, GG_LDS_PTR(lds + buf * Cfg::X_BYTES + (w + i * 8) * 1024), 16, vXsel, f_x + 64 * i * M, 0, 0);
  };
  auto fetch_s = [&](int slot) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(dS, GG_LDS_PTR(lds + (w < 2 ? Cfg::S_BASE + slot * Cfg::S_BYTES + w * 1024 : Cfg::DUMP_BASE)), 16, vSsel, f_s, 0, 0);
  };
  // Clears the tokens outside the group in the NS slabs of this wave from `o` on, 8 KB apart.  cut: first and last + 1 token of the
  // block inside the group.
  auto patch = [&](auto nc, int cut, int o) __attribute__((always_inline)) {
    constexpr int NS = decltype(nc)::value;
    const int lo = cut & 255, hi = cut >> 8;
    const bool at_lo = (lo & 15) && chunk == lo >> 4, at_hi = (hi & 15) && chunk == hi >> 4;
    if (at_lo || at_hi) {
      v4i v[NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) v[i] = *(const v4i*)(lds + o + w * 1024 + l * 16 + i * 8192);
      v4i m;
#pragma unroll
      for (int d = 0; d < 4; ++d) m[d] = (at_lo ? bytes_from(4 * (lo & 15) - 16 * d) : -1) & (at_hi ? bytes_below(4 * (hi & 15) - 16 * d) : -1);
#pragma unroll
      for (int i = 0; i < NS; ++i) *(v4i*)(lds + o + w * 1024 + l * 16 + i * 8192) = v[i] & m;
    }
  };
  constexpr std::integral_constant<int, 2> TWO{};
  constexpr std::integral_constant<int, 4> FOUR{};
  // The waits for fetches.  In front of row 3 of block b: half 1 of its dY^T, whose fetches were the last two of block b - 2; in
  // front of row 7: what block b - 1 fetched but for its last two.  Newer are 2 + 2 + 7 fetches either way, and the stores
  // issued since (a wave's loads and stores complete in the order they were issued, see wait_vmcnt; where there are more than
  // are counted here, the wait is longer than it must be).
  // The counter holds 63.  Most is outstanding where a tile of one block follows another tile: what that one leaves, pieces of the
  // operands, the fetches of row 0 and the stores of rows 1 and 2 of the last block.  A tile of blocks leaves kNewer + 24 of the wait
  // in front of its row 7 and its last 8 stores; a tile without blocks kEmptyWait and its 32.
  constexpr int kNewer = 2 + Cfg::ND1 + Cfg::ND2, kEmptyWait = 12;
  static_assert(kNewer + 24 + 8 + OperandTouch::TILE + Cfg::ND1 + 8 <= 63 && kEmptyWait + 32 + OperandTouch::TILE + Cfg::ND1 + 8 <= 63,
                "more operations in flight than vmcnt counts");
  auto wait_fetched = [&](int stores) __attribute__((always_inline)) {
    if (__builtin_expect(stores < 8, 1)) wait_vmcnt<kNewer>();
    else if (stores < 16) wait_vmcnt<kNewer + 8>();
    else if (stores < 32) wait_vmcnt<kNewer + 16>();
    else wait_vmcnt<kNewer + 32>();
  };

  // ---- operand reads
  const int keyR = swz_key_a(r);
  const int rd0 = r * 128 + (((2 * q) ^ keyR) << 4), rd1 = r * 128 + (((2 * q + 1) ^ keyR) << 4);
  auto read_frag = [&](int o) __attribute__((always_inline)) -> v8i {
    const v4i x = *(const v4i*)(lds + o + rd0);
    const v4i y = *(const v4i*)(lds + o + rd1);
    return (v8i){x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
  };
  const int sxRd = Cfg::S_BASE + (wk * 64 + 4 * r) * 4, syRd = Cfg::S_BASE + 1024 + (wn * 128 + 4 * q) * 4;

  int xb = 0, yS = 0, sS = 0;           // buffers of the block that is multiplied: X, half 0 of dY^T, scales
  auto mod5 = [](int s) { return s >= 5 ? s - 5 : s; };
  auto mod3 = [](int s) { return s >= 3 ? s - 3 : s; };
  v8i xf[4], yf[2];
  v4f sx, sy[2];
  auto read_x = [&](int kf, int buf) __attribute__((always_inline)) { xf[kf] = read_frag(buf * Cfg::X_BYTES + (wk * 64 + kf * 16) * 128); };
  auto read_y = [&](auto nfc, int slot, int ss) __attribute__((always_inline)) {
    constexpr int nf = decltype(nfc)::value;
    yf[nf & 1] = read_frag(Cfg::Y_BASE + slot * Cfg::YH_BYTES + (wn * 64 + (nf & 3) * 16) * 128);
    sy[nf & 1] = *(const v4f*)(lds + syRd + ss * Cfg::S_BYTES + nf * 64);
  };

  OperandTouch touch;
  touch.init(a, w);
  for (int i = 0; i < OperandTouch::FIRST && touch.left(a); ++i) touch.piece(a, dX, dY, l, lds + Cfg::DUMP_BASE);
  // ---- prologue: blocks 0 and 1
  int cut0 = 0, cut1 = 0;               // of the block that is multiplied and of the next one
  for (int b = 0; b < 2; ++b) {
    fetch_prepare();
    fetch_y(0, 0, 2 * b);
    fetch_y(0, 1, 2 * b);
    for (int i = 0; i < 4; ++i) fetch_x(i, b);
    fetch_s(b);
    fetch_y(1, 0, 2 * b + 1);
    fetch_y(1, 1, 2 * b + 1);
    cut0 = cut1;
    cut1 = f_cut;
  }
  wait_fetched(0);
  if (cut0) {
    patch(FOUR, cut0, 0);
    patch(TWO, cut0, Cfg::Y_BASE);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int f = 0; f < 4; ++f) read_x(f, 0);
  sx = *(const v4f*)(lds + sxRd);
  read_y(std::integral_constant<int, 0>{}, 0, 0);
  int st_cur = 0, st_prev = 0;          // stores since the barrier in front of the last row 7, between that one and the one before

  for (int it = 0;; ++it) {
    const Tile cur = tile_at(it);
    if (!cur.valid) break;
    if (touch.left(a)) {
#pragma unroll
      for (int i = 0; i < OperandTouch::TILE; ++i) touch.piece(a, dX, dY, l, lds + Cfg::DUMP_BASE);
      st_cur += OperandTouch::TILE;       // they count like stores
    }
    v4f acc[8][4];
#pragma unroll
    for (int nf = 0; nf < 8; ++nf)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[nf][i] = (v4f){0.f, 0.f, 0.f, 0.f};
    v4f pend = {0.f, 0.f, 0.f, 0.f}, pf = {0.f, 0.f, 0.f, 0.f};      // the last product and its factors

    // ---- stores, as in wgrad_kernel.h
    constexpr int ES = OUT16 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t dOut = __builtin_amdgcn_make_buffer_rsrc((void*)((uint8_t*)a.dW + (((int64_t)cur.g * a.N + cur.n0) * a.K + cur.k0) * ES), 0, ((Cfg::TN - 1) * a.K + Cfg::TK) * ES, GG_RSRC_FLAGS);
    const int vOut = (4 * q * a.K + 4 * r) * ES;
    auto store = [&](auto tc) __attribute__((always_inline)) {      // row 4 q + i of fragment nf, 4 nf + i from 0 to 31
      constexpr int nf = decltype(tc)::value / 4, i = decltype(tc)::value % 4;
      const v4f v = acc[nf][i];
      const int row = ((wn * 128 + 16 * nf + i) * a.K + wk * 64) * ES;
      if constexpr (OUT16)
        __builtin_amdgcn_raw_buffer_store_b64((v2i){pack2_rne(v[0], v[1], false), pack2_rne(v[2], v[3], false)}, dOut, vOut, row, kStoreStreaming);
      else
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), dOut, vOut, row, kStoreStreaming);
    };

    auto block = [&](auto lastc) __attribute__((always_inline)) {
      constexpr bool LAST = decltype(lastc)::value;
      const int y1 = mod5(yS + 1), y2 = mod5(yS + 2), y4 = mod5(yS + 4), s1 = mod3(sS + 1), s2 = mod3(sS + 2);
      fetch_prepare();
      auto row = [&](auto nfc) __attribute__((always_inline)) {
        constexpr int nf = decltype(nfc)::value;
        if constexpr (nf < 7) read_y(std::integral_constant<int, (nf + 1) & 7>{}, nf + 1 < 4 ? yS : y1, sS);
        else read_y(std::integral_constant<int, 0>{}, y2, s1);
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, 4>([&](auto kfc) __attribute__((always_inline)) {
          constexpr int kf = decltype(kfc)::value;
          v4f p = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(yf[nf & 1], xf[kf], (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
          asm volatile("" : "+v"(p));
          __builtin_amdgcn_sched_barrier(0);
          v4f f;
#pragma unroll
          for (int i = 0; i < 4; ++i) f[i] = sy[nf & 1][i] * sx[kf];
          asm volatile("" : "+v"(f));
          __builtin_amdgcn_sched_barrier(0);
          constexpr int pn = kf > 0 ? nf : (nf + 7) & 7, pk = (kf + 3) & 3;
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[pn][i][pk] += pend[i] * pf[i];
#pragma unroll
          for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(acc[pn][i]));
          if constexpr (nf == 7) {
            read_x(kf, xb ^ 1);
            if constexpr (kf == 3) sx = *(const v4f*)(lds + sxRd + s1 * Cfg::S_BYTES);
          }
          if constexpr (nf == 0 && (kf == 1 || kf == 3)) fetch_y(0, kf >> 1, y4);
          if constexpr ((nf == 3 || nf == 4) && (kf == 0 || kf == 2)) fetch_x((nf - 3) * 2 + (kf >> 1), xb);
          if constexpr (nf == 5 && kf == 0) fetch_s(s2);
          if constexpr (nf == 5 && (kf == 1 || kf == 3)) fetch_y(1, kf >> 1, yS);
          if constexpr (LAST && nf > 0) store(std::integral_constant<int, 4 * (nf - 1) + kf>{});
          pend = p;
          pf = f;
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      static_for<0, 2>(row);
      if (cut0) {
        wait_fetched(st_prev + st_cur);
        patch(TWO, cut0, Cfg::Y_BASE + y1 * Cfg::YH_BYTES);
        __builtin_amdgcn_sched_barrier(0);
      }
      row(std::integral_constant<int, 2>{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if constexpr (LAST) wait_vmcnt<kNewer + 8>();
      else wait_fetched(st_prev + st_cur);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      static_for<3, 6>(row);
      if (cut1) {
        if constexpr (LAST) wait_vmcnt<kNewer + 20>();
        else wait_fetched(st_cur);
        patch(FOUR, cut1, (xb ^ 1) * Cfg::X_BYTES);
        patch(TWO, cut1, Cfg::Y_BASE + y2 * Cfg::YH_BYTES);
        __builtin_amdgcn_sched_barrier(0);
      }
      row(std::integral_constant<int, 6>{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if constexpr (LAST) wait_vmcnt<kNewer + 24>();
      else wait_fetched(st_cur);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      static_for<7, 8>(row);
      st_prev = st_cur + (LAST ? 24 : 0);
      st_cur = 0;
      cut0 = cut1;
      cut1 = f_cut;
      xb ^= 1;
      yS = y2;
      sS = s1;
    };
    const bool early = cur.steps > 0;
#pragma nounroll
    for (int s = 0; s < cur.steps - (early ? 1 : 0); ++s) block(std::false_type{});
    if (early) block(std::true_type{});
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[7][i][3] += pend[i] * pf[i];

    if (early) {
      static_for<28, 32>(store);
      st_cur = 8;
    } else {
      wait_vmcnt<kEmptyWait>();
      static_for<0, 32>(store);
      st_cur = 32;
    }
  }
  wait_vmcnt<0>();     // the fetches past the last block still write zeros into this workgroup's LDS: let them land
}

}  // namespace gg
