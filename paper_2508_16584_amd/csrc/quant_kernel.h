// The step in front of the grouped GEMM: bf16 rows -> e4m3 bytes + one fp32 scale per 1x128 block (the scaling
// of A stated below Table 1 of the paper), gathered straight into group-contiguous order.  With the
// padding-free GEMM this kernel runs on the valid rows only; nothing is padded and nothing is copied again.
//
// Per output row r and K block kb, in fp32:
//     amax  = max( max |x| over the 128 values with NaNs skipped, 2^-100 )
//     scale = amax / 448                                       (a dequantisation multiplier)
//     byte  = e4m3( clamp(x * (448 / amax), -448, 448) )       round to nearest even; NaN -> 0x7F
// The two divisions per block, the product and the conversion are the hardware's correctly rounded ones, so the
// bytes and scales are reproducible bit for bit on the host.
//
// Mapping: 8 lanes own one block.  A lane loads 16 bytes of either half of it (a half is one 128-byte line for the
// eight lanes), reduces amax over its 16 values and the eight lanes, and after an exchange of 8 bytes with its
// neighbour stores 16 bytes.  A workgroup of 256 threads takes up to 64 blocks in one pass, all its loads issued before
// any arithmetic: a piece of one row, or several short rows.  One pass per workgroup: the grid covers the tensor.
// Few blocks are a chain of latencies (load, reduce, divide, convert, store), in which 16 values per lane cost more than the
// second store request: there 16 lanes own one block, 16 bytes in and 8 bytes out each, and a workgroup takes up to 16
// blocks (few_blocks in gg_fp8.hip; one row of 512: 2.75 us, 2.95 with eight lanes, 64 rows of 7168 3.2, 3.9).
// HBM-bound: 2K bytes in, K + K/32 out per row.  8192 x 7168 gathered: 33.5 us (5.3 TB/s), 16384 x 7168 out of 8192 rows
// 57 (6.3), 32768 x 7168 118 (6.0); with 16 lanes and 8-byte stores per block, row pairs strided over 8 workgroups per
// compute unit and no streaming policy they took 40, 72 and 146 us.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gg {

constexpr int Q_THREADS = 256;

typedef int q_v4i __attribute__((ext_vector_type(4)));
typedef int q_v2i __attribute__((ext_vector_type(2)));

// max over the 8 lanes of half a DPP row, result in every lane
__device__ __forceinline__ unsigned max8(unsigned v) {
  unsigned t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);       // quad_perm [1, 0, 3, 2]
  v = v > t ? v : t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);       // quad_perm [2, 3, 0, 1]
  v = v > t ? v : t;
  t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);      // row_half_mirror: the other quad of the eight
  return v > t ? v : t;
}

// The block quantiser's arithmetic for callers that hold a block's values spread over lanes in a way of their own:
// amax_bits_of() of every value, reduced by the caller with an integer max, then block_amax() and e4m3x4_of().
__device__ __forceinline__ unsigned amax_bits_of(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v) & 0x7FFFFFFFu;
  return u > 0x7F800000u ? 0u : u;                             // a NaN (quiet or signalling) counts as zero
}
__device__ __forceinline__ float block_amax(unsigned top) {
  top = top > 0x0D800000u ? top : 0x0D800000u;                 // floor 2^-100: 448 / amax stays finite
  return __builtin_bit_cast(float, top);
}
// four values -> four e4m3 bytes in a dword (value 0 in the low byte); SPECIAL: NaNs and infinities may be among them
template <bool SPECIAL = true>
__device__ __forceinline__ int e4m3x4_of(const float* v, float inv) {
  float y[4];
  unsigned nan = 0;                                            // 0x7F in the byte of every NaN, whatever its sign or payload
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float t = v[i] * inv;
    if constexpr (SPECIAL) {
      const bool is_nan = t != t;
      y[i] = is_nan ? 0.f : __builtin_fminf(__builtin_fmaxf(t, -448.0f), 448.0f);
      nan |= is_nan ? (0x7Fu << (8 * i)) : 0u;
    } else {
      y[i] = __builtin_amdgcn_fmed3f(t, -448.0f, 448.0f);
    }
  }
  int w = 0;
  w = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], w, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], w, true);
  return w | (int)nan;
}

// One block.  LANES 8: lane `sub` of its eight holds bf16 columns 8 sub .. + 7 in lo and 64 + 8 sub .. + 7 in hi.  LANES 16:
// lane `sub` of its sixteen holds columns 8 sub .. + 7 in lo.
template <bool SNT, int LANES>
__device__ __forceinline__ void quantize_block(const q_v4i lo, const q_v4i hi, uint8_t* dst, float* dst_scale, int sub) {
  constexpr int NV = 128 / LANES;
  float v[NV];
  unsigned top = 0;
#pragma unroll
  for (int i = 0; i < NV / 2; ++i) {
    const unsigned two = (unsigned)(i < 4 ? lo[i & 3] : hi[i & 3]);
    v[2 * i] = __builtin_bit_cast(float, two << 16);
    v[2 * i + 1] = __builtin_bit_cast(float, two & 0xFFFF0000u);
    const unsigned a0 = (two << 16) & 0x7FFFFFFFu, a1 = two & 0x7FFF0000u;      // |x| of non-NaN values orders like its bit pattern
    top = top > a0 ? top : a0;
    top = top > a1 ? top : a1;
  }
  // NaNs and infinities are rare: one wave-uniform branch keeps their handling out of the common path
  const bool special = __builtin_amdgcn_ballot_w64(top >= 0x7F800000u) != 0;
  if (special) {
    top = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const unsigned t = amax_bits_of(v[i]);
      top = top > t ? top : t;
    }
  }
  top = max8(top);
  if constexpr (LANES == 16) {
    const unsigned t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)top, 0x128, 0xF, 0xF, false);      // row_ror 8: the other eight
    top = top > t ? top : t;
  }
  const float amax = block_amax(top);
  const float scale = amax / 448.0f;
  const float inv = 448.0f / amax;
  int w[NV / 4];
#pragma unroll
  for (int d = 0; d < NV / 4; ++d) w[d] = special ? e4m3x4_of(v + 4 * d, inv) : e4m3x4_of<false>(v + 4 * d, inv);
  if (sub == 0) *dst_scale = scale;
  if constexpr (LANES == 16) *(q_v2i*)(dst + 8 * sub) = (q_v2i){w[0], w[1]};
  // w[0], w[1] are bytes 8 sub .. + 7 of the block and w[2], w[3] bytes 64 + 8 sub .. + 7: an even lane gives the latter
  // away for its neighbour's former, so that every lane has 16 consecutive bytes
  if constexpr (LANES == 8) {
    const bool odd = sub & 1;
    const int r0 = __builtin_amdgcn_update_dpp(0, odd ? w[0] : w[2], 0xB1, 0xF, 0xF, false);
    const int r1 = __builtin_amdgcn_update_dpp(0, odd ? w[1] : w[3], 0xB1, 0xF, 0xF, false);
    const q_v4i out = odd ? (q_v4i){r0, r1, w[2], w[3]} : (q_v4i){w[0], w[1], r0, r1};
    q_v4i* const p = (q_v4i*)(dst + (odd ? 64 + 8 * (sub - 1) : 8 * sub));
    if constexpr (SNT) __builtin_nontemporal_store(out, p);
    else *p = out;
  }
}

// Work of a workgroup: up to 64 blocks (16 with sixteen lanes each), `rows` adjacent rows of `blocks` blocks (rows > 1 only where a row has few).
// Which rows depends on the storage order of the scales:
//   sector == 0: workgroup b takes piece b of the row-major list of pieces;
//   sector == 8 or 32: with K-block-major scales the 4-byte scale stores of 8 adjacent rows make up a 32-byte piece of
//     memory (of 32 rows a line).  Runs of `sector` adjacent row groups go to ONE XCD (workgroup b runs on XCD b % 8) in
//     neighbouring slots, which run at about the same time, so that they leave that XCD's L2 together; dealt out one by
//     one, every XCD's L2 would write a masked piece of its own.
struct RowWork {
  int rows;          // rows of one workgroup
  int blocks;        // blocks of a row it takes
  int pieces;        // pieces of a row: ceil(KB / blocks)
  unsigned magic;    // ceil(2^16 / blocks): v / blocks = v * magic >> 16 for v < 64
  int sector;
  unsigned groups;   // workgroups' worth of work: groups of rows x pieces, rounded up to whole runs of sectors
};

struct RowSlot {
  bool valid;
  int row, blk;
};
// slot v (of rows * blocks) of work item `id`
__device__ __forceinline__ RowSlot row_slot(const RowWork& rw, unsigned id, int v, int KB, int M_total) {
  unsigned g = id, piece = 0;
  if (rw.pieces > 1) {
    g = id / (unsigned)rw.pieces;
    piece = id - g * (unsigned)rw.pieces;
  }
  if (rw.sector) {
    const unsigned x = g & 7, i = g >> 3, n = (unsigned)rw.sector;
    g = (i / n) * (8 * n) + x * n + i % n;
  }
  const int rr = (int)((unsigned)v * rw.magic >> 16);
  const int64_t row = (int64_t)g * rw.rows + rr;
  RowSlot s;
  s.blk = (int)piece * rw.blocks + (v - rr * rw.blocks);
  s.valid = v < rw.rows * rw.blocks && row < M_total && s.blk < KB;
  s.row = (int)row;
  return s;
}

template <bool NT>
__device__ __forceinline__ q_v4i load_16(const uint16_t* p) {
  if constexpr (NT) return __builtin_nontemporal_load((const q_v4i*)p);
  return *(const q_v4i*)p;
}

// LNT, SNT: the rows are read, the bytes written, with the streaming policy (see bytes_stream() in gg_fp8.hip)
template <bool LNT, bool SNT, int LANES = 8>
__global__ void __launch_bounds__(Q_THREADS) gg_quantize_rows_kernel(const uint16_t* __restrict__ X,
                                                                     const int32_t* __restrict__ row_src,
                                                                     uint8_t* __restrict__ A, float* __restrict__ SA,
                                                                     int64_t T, int M_total, int K, int KB,
                                                                     int64_t sa_rs, int64_t sa_ks,     // SA[row * sa_rs + blk * sa_ks]
                                                                     RowWork rw) {
  constexpr int U = LANES == 8 ? 2 : 1, GROUPS = Q_THREADS / LANES;      // blocks per lane, blocks per workgroup / U
  const int grp = threadIdx.x / LANES, sub = threadIdx.x % LANES;
  for (unsigned id = blockIdx.x; id < rw.groups; id += gridDim.x) {
    RowSlot s[U];
    int64_t src[U];
    q_v4i lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = row_slot(rw, id, u * GROUPS + grp, KB, M_total);              // uniform over the lanes of a block
      src[u] = !s[u].valid ? -1 : row_src ? (int64_t)row_src[s[u].row] : (int64_t)s[u].row;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      lo[u] = hi[u] = (q_v4i){0, 0, 0, 0};
      if (src[u] >= 0 && src[u] < T) {                                     // a source outside [0, T) stands for a row of zeros
        const uint16_t* p = X + src[u] * K + s[u].blk * 128 + sub * 8;
        lo[u] = load_16<LNT>(p);
        if constexpr (LANES == 8) hi[u] = load_16<LNT>(p + 64);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s[u].valid) quantize_block<SNT, LANES>(lo[u], hi[u], A + (int64_t)s[u].row * K + s[u].blk * 128, SA + s[u].row * sa_rs + s[u].blk * sa_ks, sub);
  }
}

// The activation between the two grouped GEMMs of an expert MLP, fused with the quantiser above: H [M, 2I] bf16
// (columns [0, I): gate projection, [I, 2I): up projection) ->
//     act = bf16_rne( silu(gate) * up ),  silu(g) = g / (1 + exp(-g))   in fp32
// and then exactly quantize_block on the bf16 bits of act.  act is also written out when act_out is not null.
// Same mapping: 8 lanes own one block of 128 activation columns, a lane loads 16 gate and 16 up values (of few blocks: 16
// lanes, 8 and 8).
// two (gate, up) pairs, each a dword of two bf16 -> one dword of two bf16 activations
__device__ __forceinline__ int swiglu2(const int g_raw, const int u_raw) {
  float g[2] = {__builtin_bit_cast(float, g_raw << 16), __builtin_bit_cast(float, g_raw & (int)0xFFFF0000)};
  float u[2] = {__builtin_bit_cast(float, u_raw << 16), __builtin_bit_cast(float, u_raw & (int)0xFFFF0000)};
  float a[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // sigmoid through t = exp(-|g|) in [0, 1]: no overflow for any g; the hardware exponential (a few fp32
    // ulps, denormal results flushed: t = 0 below g = -87.3) and the hardware reciprocal (1 ulp; 1 + t lies in
    // [1, 2]) are far inside the bf16 rounding.  A division here compiles to the 10-instruction correctly
    // rounded sequence, which made this kernel bound by vector arithmetic.
    const float t = __expf(-__builtin_fabsf(g[h]));
    const float sig = (g[h] >= 0.f ? 1.0f : t) * __builtin_amdgcn_rcpf(1.0f + t);
    a[h] = g[h] * sig * u[h];
  }
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  const bf2 r = __builtin_convertvector((f2){a[0], a[1]}, bf2);     // round to nearest even
  return __builtin_bit_cast(int, r);
}

__device__ __forceinline__ q_v4i swiglu8(const q_v4i g_raw, const q_v4i u_raw) {
  q_v4i out;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = swiglu2(g_raw[i], u_raw[i]);
  return out;
}

// The producer of the weight-gradient GEMM's operands: the same block quantiser ALONG THE TOKENS, with the transpose
// that GEMM wants.  X [T, K] bf16 (token-major) -> XT [K, M_total] e4m3 (token index contiguous) and SX [MB, K]:
// output token r is input row row_src[r]; feature k's block j holds tokens [128 j, 128 j + 128) of the output order,
// the last block those that exist.  (The paper defines neither this operation nor its layouts.)
// A workgroup takes tiles of one token block x 64 features: 128 rows of 128 bytes go through LDS (every group of 16
// rows shifted by 32 bytes (sixteen lanes: of 8 by 16), so that the eight lanes of a feature pair read from different banks); lane 8 f + p then
// owns tokens 16 p .. 16 p + 15 of features 2 f and 2 f + 1 (one 4-byte LDS read per token): amax over its 16 values
// per feature and over the eight lanes, 16 bytes out per feature - the eight lanes of a feature write one 128-byte
// line of XT.  Few tiles are a chain of latencies (token index, row, LDS, reduction, divisions, store): there sixteen lanes own a
// feature pair, 8 tokens each, and a workgroup has twice the threads (few_tiles in gg_fp8.hip; 1264 x 1280 out of 640 rows
// 4.6 us, 3.9).
// Tiles are listed token block by token block, or (strips) in strips of QC_STRIP feature tiles, a strip's token blocks one after the
// other: the workgroups at work at one time then write neighbouring lines of a few rows of XT instead of lines of all rows, a row
// pitch apart, and read 512 bytes of a token instead of all of it.  Where that pays: see cols_in_strips() in gg_fp8.hip.
constexpr int QC_FEATS = 64, QC_STRIP = 4;
constexpr int QC_LDS_BYTES = 128 * 128 + 15 * 16;

// SNT: the bytes are written with the streaming policy (see cols_bytes_stream() in gg_fp8.hip).
template <bool SNT, int LANES = 8>
__global__ void __launch_bounds__(32 * LANES) gg_quantize_cols_kernel(const uint16_t* __restrict__ X,
                                                                     const int32_t* __restrict__ row_src,
                                                                     uint8_t* __restrict__ XT, float* __restrict__ SX,
                                                                     int64_t T, int M_total, int K, int MB, int strips) {
  constexpr int NT = 32 * LANES, TOKS = 128 / LANES, LOADS = 1024 / NT;      // threads, tokens of a lane, 16-byte pieces it brings in
  __shared__ __attribute__((aligned(16))) uint8_t tile[QC_LDS_BYTES];
  const int t = threadIdx.x;
  const int kt = K / QC_FEATS;
  const int64_t tiles = (int64_t)MB * kt;
  const int fp = t / LANES, part = t % LANES;
  // piece t + NT i of a tile: token (t + NT i) / 8 of the block, features 8 (t % 8) .. + 7
  q_v4i raw[LOADS];
  auto place = [&](int64_t id, int& j, int& k0) __attribute__((always_inline)) {      // token block and first feature of a tile
    if (!strips) {
      j = (int)(id / kt);
      k0 = (int)(id - (int64_t)j * kt) * QC_FEATS;
      return;
    }
    const int strip = (int)(id / ((int64_t)QC_STRIP * MB));
    const unsigned in = (unsigned)(id - (int64_t)strip * QC_STRIP * MB);
    const unsigned width = (unsigned)(kt - strip * QC_STRIP < QC_STRIP ? kt - strip * QC_STRIP : QC_STRIP);
    j = (int)(in / width);
    k0 = (strip * QC_STRIP + (int)(in - (unsigned)j * width)) * QC_FEATS;
  };
  auto load_tile = [&](int64_t id) __attribute__((always_inline)) {
    int j, k0;
    place(id, j, k0);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int r = 128 * j + ((t + NT * i) >> 3);
      raw[i] = (q_v4i){0, 0, 0, 0};                        // a token past the end or a source outside [0, T): zeros
      if (r < M_total) {
        const int64_t src = row_src ? (int64_t)row_src[r] : (int64_t)r;
        if (src >= 0 && src < T) raw[i] = *(const q_v4i*)(X + src * K + k0 + 8 * (t & 7));
      }
    }
  };
  if ((int64_t)blockIdx.x < tiles) load_tile(blockIdx.x);
  for (int64_t id = blockIdx.x; id < tiles; id += gridDim.x) {
    int j, k0;
    place(id, j, k0);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int tok = (t + NT * i) >> 3;
      *(q_v4i*)(tile + tok * 128 + tok / TOKS * (2 * TOKS) + 16 * (t & 7)) = raw[i];
    }
    __syncthreads();
    if (id + gridDim.x < tiles) load_tile(id + gridDim.x);      // the next tile's rows are on their way during this one's arithmetic
    float v[2][TOKS];
    unsigned top[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < TOKS; ++i) {
      const unsigned two = *(const unsigned*)(tile + (TOKS * part + i) * 128 + part * (2 * TOKS) + 4 * fp);
      v[0][i] = __builtin_bit_cast(float, two << 16);
      v[1][i] = __builtin_bit_cast(float, two & 0xFFFF0000u);
      const unsigned a0 = two & 0x7FFFu, a1 = (two >> 16) & 0x7FFFu;      // |x| of non-NaN values orders like its bit pattern
      top[0] = top[0] > a0 ? top[0] : a0;
      top[1] = top[1] > a1 ? top[1] : a1;
    }
    // NaNs and infinities are rare: one wave-uniform branch keeps their handling out of the common path
    const bool special = __builtin_amdgcn_ballot_w64((top[0] > top[1] ? top[0] : top[1]) >= 0x7F80u) != 0;
    int out[2][TOKS / 4];
    float scale[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      unsigned m = top[f];
      if (special) {
        m = 0;
#pragma unroll
        for (int i = 0; i < TOKS; ++i) {
          const unsigned a = amax_bits_of(v[f][i]) >> 16;               // a NaN counts as zero
          m = m > a ? m : a;
        }
      }
      m = max8(m);
      if constexpr (LANES == 16) {
        const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x128, 0xF, 0xF, false);      // row_ror 8: the other eight
        m = m > o ? m : o;
      }
      const float amax = block_amax(m << 16);
      scale[f] = amax / 448.0f;
      const float inv = 448.0f / amax;
#pragma unroll
      for (int d = 0; d < TOKS / 4; ++d) {
        out[f][d] = special ? e4m3x4_of(v[f] + 4 * d, inv) : e4m3x4_of<false>(v[f] + 4 * d, inv);
      }
    }
    // M_total is a multiple of 16: a lane's piece of a row of XT exists whole or not at all
    const int tok0 = 128 * j + TOKS * part;
    if (tok0 < M_total) {
      uint8_t* dst = XT + (int64_t)(k0 + 2 * fp) * M_total + tok0;
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        typedef int piece __attribute__((ext_vector_type(TOKS / 4)));
        piece o;
#pragma unroll
        for (int d = 0; d < TOKS / 4; ++d) o[d] = out[f][d];
        if constexpr (SNT) __builtin_nontemporal_store(o, (piece*)(dst + f * (int64_t)M_total));
        else *(piece*)(dst + f * (int64_t)M_total) = o;
      }
    }
    if (part == 0) *(q_v2i*)(SX + (int64_t)j * K + k0 + 2 * fp) = (q_v2i){__builtin_bit_cast(int, scale[0]), __builtin_bit_cast(int, scale[1])};
    __syncthreads();                                        // before the next tile's rows overwrite these
  }
}

template <bool LNT, bool SNT, int LANES = 8>
__global__ void __launch_bounds__(Q_THREADS) gg_swiglu_quantize_rows_kernel(const uint16_t* __restrict__ H,
                                                                            uint8_t* __restrict__ A, float* __restrict__ SA,
                                                                            uint16_t* __restrict__ act_out,
                                                                            int M_total, int I, int IB,
                                                                            int64_t sa_rs, int64_t sa_ks,     // SA[row * sa_rs + blk * sa_ks]
                                                                            RowWork rw) {
  const int grp = threadIdx.x / LANES, sub = threadIdx.x % LANES;
  for (unsigned id = blockIdx.x; id < rw.groups; id += gridDim.x) {
    const RowSlot s = row_slot(rw, id, grp, IB, M_total);
    if (!s.valid) continue;
    const uint16_t* p = H + (int64_t)s.row * 2 * I + s.blk * 128 + sub * 8;
    const int64_t o = (int64_t)s.row * I + s.blk * 128;
    q_v4i lo, hi = {0, 0, 0, 0};
    if constexpr (LANES == 8) {
      const q_v4i g0 = load_16<LNT>(p), g1 = load_16<LNT>(p + 64), u0 = load_16<LNT>(p + I), u1 = load_16<LNT>(p + I + 64);
      lo = swiglu8(g0, u0);
      hi = swiglu8(g1, u1);
    } else {
      const q_v4i g0 = load_16<LNT>(p), u0 = load_16<LNT>(p + I);
      lo = swiglu8(g0, u0);
    }
    if (act_out) {       // for the backward pass: past the caches (with the GEMM behind this kernel 0.6 to 2 % faster than through them)
      __builtin_nontemporal_store(lo, (q_v4i*)(act_out + o + sub * 8));
      if constexpr (LANES == 8) __builtin_nontemporal_store(hi, (q_v4i*)(act_out + o + 64 + sub * 8));
    }
    quantize_block<SNT, LANES>(lo, hi, A + o, SA + s.row * sa_rs + s.blk * sa_ks, sub);
  }
}

}  // namespace gg
