// HIP kernels for gfx950 (CDNA4, wave64) and the exported calls that launch
// them: decoding (lfc_decode_blocks, lfc_decode_progressive), rendering
// (lfc_render_views, lfc_render_views_ex, lfc_render_tune, the render
// plans), and the launchers the batch context and server use.
//
// Decoding a block (Alg. 2, Sec. 3.5) is: read the top-level key-view block,
// then for every level below, locate the node's residual block inside the
// group of its spatial location (one level of indirection through the
// block offsets, Sec. 3.4), unpack its BISE values (Sec. 3.3), undo the
// zigzag and the quantiser step, and add it.  All integer work; no MFMA.
//
// Work mapping of the whole-field kernel: a workgroup owns a strip of 64/B
// blocks of one block row and channel; one lane decodes a whole stored
// residual block into LDS, then each lane gathers and stores 16 bytes of an
// output row (key view + ancestors + leaf).  Random access and rendering
// give one lane one channel of a block (random access to 8 x 8 blocks: one
// row of it).  Samples travel as packed
// int16 pairs: the residual tail (zigzag undo, step 2^q, adding the parent)
// runs on both halves of a register at once, and the sums wrap modulo 2^16
// exactly as the final int16 store of a 32-bit sum would.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "serve.h"

// Device memory of lfc_render_views_noalloc: the decoded source views of
// its decode-then-interpolate path, for callers that cannot allocate.  Each
// device that runs the library holds its own copy until the process ends;
// host code reaches it only through the address hipGetSymbolAddress returns
// on that device.
static __device__ __align__(256) uint8_t scratch[LFC_NOALLOC_SCRATCH_BYTES];

namespace {

using lfc::kMaxLevels;
constexpr uint32_t kAbsent = 0xFFFFFFFFu;
constexpr int kLutEntries = 384;  // 256 trit-field values, then 128 quint-field values
constexpr int kThreads = 256;

template <int S>
struct Planes {
  static constexpr uint32_t trit = (8 * S + 4) / 5;    // digit-plane bits, trit blocks
  static constexpr uint32_t quint = (7 * S + 2) / 3;   // digit-plane bits, quint blocks
};

// Digits of a trit field (entries 0..255: five 2-bit digits) or of a quint
// field (entries 256..383: three 3-bit digits).  Out-of-range fields map to 0;
// streams holding them are rejected before upload.
constexpr uint32_t lut_value(int t) {
  uint32_t v = 0;
  if (t < 256) {
    if (t < 243)
      for (int r = 0, x = t, p = 0; r < 5; r++, x /= 3, p += 2) v |= (uint32_t)(x % 3) << p;
  } else if (t - 256 < 125) {
    for (int r = 0, x = t - 256, p = 0; r < 3; r++, x /= 5, p += 3) v |= (uint32_t)(x % 5) << p;
  }
  return v;
}

// The LUT, two entries per word, as a table in device memory (the
// whole-field kernel copies it into LDS instead of computing it).
struct LutWords {
  uint32_t w[kLutEntries / 2];
};
constexpr LutWords make_lut_words() {
  LutWords l{};
  for (int t = 0; t < kLutEntries; t++) l.w[t / 2] |= lut_value(t) << (16 * (t & 1));
  return l;
}
__device__ constexpr LutWords kLutTable = make_lut_words();

// 64 bits of a group's bit stream starting at bit pos (bit p is bit p%32 of word p/32).
__device__ __forceinline__ uint64_t window64(const uint32_t *gw, uint32_t pos) {
  const uint32_t *p = gw + (pos >> 5);
  const uint32_t a = p[0], b = p[1], c = p[2];
  const uint32_t sh = pos & 31u;
  const uint32_t lo = __builtin_amdgcn_alignbit(b, a, sh);
  const uint32_t hi = __builtin_amdgcn_alignbit(c, b, sh);
  return ((uint64_t)hi << 32) | lo;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 as_u16x2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t as_u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// two samples at once: a + b modulo 2^16 per half
__device__ __forceinline__ uint32_t add_pk(uint32_t a, uint32_t b) { return as_u32(as_u16x2(a) + as_u16x2(b)); }

// Two zigzagged values (0,1,2,3,.. -> 0,-1,1,-2,..) in the 16-bit halves of
// z, back to signed and times 2^q (0 <= q <= 4), as int16 pairs.  A value's
// magnitude times 2^q is (z >> 1) << q = z rotated left by q - 1 (right by
// 1 for q = 0) with the low half's top bit and the word's top bit cleared;
// a negative value's bits from q - 1 up are then inverted, which also clears
// bit q - 1 (its zigzag parity bit).  Every zigzag value of a valid stream is
// below 2^12 (at most 12 plain bits, or 6 bits below a trit or quint digit),
// so nothing crosses between the halves; equal, for all such pairs and every
// q, to unzigzagging each half and shifting it left by q (checked
// exhaustively on the host by tests/arith_identities.c).  Five VALU
// operations per pair against seven with packed 16-bit shifts.
__device__ __forceinline__ uint32_t unzigzag_pk(uint32_t z, int q) {
  const uint32_t rot = (uint32_t)(33 - q) & 31u;
  const uint32_t inv = q ? (0xFFFFu << (q - 1)) & 0xFFFFu : 0xFFFFu;   // the bits a negative value inverts
  const uint32_t t = __builtin_amdgcn_alignbit(z, z, rot) & 0x7FFF7FFFu;
  return t ^ ((z & 0x00010001u) * inv);
}

// Where the digits of row y (values 8 y .. 8 y + 7) sit in a trit or quint 8 x 8
// block: bits 0..7 the bit offset of the row's first digit field in the
// digit plane, bits 8..15 the offset of the row's first digit in the
// concatenated digits of those fields, bits 16+4i the width of the row's i-th
// field (the last group of a block can be short; 0 = no such field).
// Computed once per lane.
__device__ __forceinline__ uint32_t digit_plan(int y, bool trit) {
  constexpr int B = 8, S = B * B;
  const int glen = trit ? 5 : 3, fw = trit ? 8 : 7, dbits = trit ? 2 : 3;
  const int rem = S % glen, last = S / glen;
  const int pw = trit ? (8 * rem + 4) / 5 : (7 * rem + 2) / 3;
  const int i0 = y * B, a = i0 / glen, a_end = (i0 + B - 1) / glen;
  uint32_t plan = (uint32_t)(a * fw) | ((uint32_t)((i0 - a * glen) * dbits) << 8);
  for (int i = 0; i <= a_end - a && i < 4; i++)
    plan |= (uint32_t)((rem && a + i == last) ? pw : fw) << (16 + 4 * i);
  return plan;
}

// Row y of an 8 x 8 block of any kind: its BISE fields read (digit << m | low
// bits), zigzag undone, times 2^q; d holds the residuals as packed int16 pairs.
__device__ __forceinline__ void decode_row(const uint32_t *gw, uint32_t e, uint32_t plan_t, uint32_t plan_q, int y,
                                           int q, const uint16_t *lut, uint32_t d[4]) {
  constexpr int B = 8, S = B * B;
  const uint32_t code = e & 31u, rel = e >> 5;
  const bool is_bits = code < 12u, is_trit = code - 12u < 7u;
  const uint32_t m = is_bits ? code + 1u : (is_trit ? code - 12u : code - 19u);
  const uint32_t hdr = is_bits ? 0u : (is_trit ? Planes<S>::trit : Planes<S>::quint);
  const uint32_t p = rel + hdr + (uint32_t)(y * B) * m, lmask = (1u << m) - 1u;
  const uint32_t plan = is_trit ? plan_t : plan_q, pd = rel + (is_bits ? 0u : (plan & 0xffu));
  const uint32_t *qd = gw + (pd >> 5);
  const uint64_t v = window64(gw, p), v2 = window64(gw, p + 4u * m);   // low bits of values 0..3, 4..7
  const uint32_t win = __builtin_amdgcn_alignbit(qd[1], qd[0], pd & 31u);
  // the row's digit fields through the LUT, concatenated, then one digit per value
  const uint32_t fw = is_trit ? 8u : 7u, gb = is_trit ? 10u : 9u, db = is_trit ? 2u : 3u;
  const uint32_t lb = is_trit ? 0u : 256u;
  uint64_t D = 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint32_t f = __builtin_amdgcn_ubfe(win, i * fw, (plan >> (16 + 4 * i)) & 15u);
    D |= (uint64_t)lut[lb + f] << (i * gb);
  }
  const uint64_t rowd = D >> ((plan >> 8) & 0xffu);
  const uint32_t dmask = is_bits ? 0u : (is_trit ? 3u : 7u);
  uint32_t u[B];
#pragma unroll
  for (int k = 0; k < B; k++) {
    const uint32_t low = (uint32_t)((k < 4 ? v : v2) >> ((k & 3) * m)) & lmask;
    u[k] = ((((uint32_t)(rowd >> (k * db))) & dmask) << m) | low;
  }
#pragma unroll
  for (int i = 0; i < B / 2; i++) d[i] = unzigzag_pk(u[2 * i] | (u[2 * i + 1] << 16), q);
}

// a row of B int16 samples as B/2 packed words
template <int B>
__device__ __forceinline__ void load_row(const int16_t *p, uint32_t x[B / 2]) {
  if constexpr (B == 2) {
    x[0] = *reinterpret_cast<const uint32_t *>(p);
  } else if constexpr (B == 4) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    x[0] = v.x;
    x[1] = v.y;
  } else {
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  }
}

template <int B>
__device__ __forceinline__ void store_row(int16_t *p, const uint32_t x[B / 2]) {
  if constexpr (B == 2) {
    *reinterpret_cast<uint32_t *>(p) = x[0];
  } else if constexpr (B == 4) {
    *reinterpret_cast<uint2 *>(p) = make_uint2(x[0], x[1]);
  } else {
    *reinterpret_cast<uint4 *>(p) = make_uint4(x[0], x[1], x[2], x[3]);
  }
}

// Stores of output that no kernel of the same call reads again, with the
// non-temporal hint when NT: streamed to HBM without displacing what L2 and
// the Infinity Cache hold (the compressed input of the next call).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ void put4(int16_t *p, const uint32_t x[4]) {
  if constexpr (NT) {
    const u32x4_t v = {x[0], x[1], x[2], x[3]};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(p));
  } else {
    *reinterpret_cast<uint4 *>(p) = make_uint4(x[0], x[1], x[2], x[3]);
  }
}
template <int B, bool NT>
__device__ __forceinline__ void put_row(int16_t *p, const uint32_t x[B / 2]) {
  if constexpr (!NT) {
    store_row<B>(p, x);
  } else if constexpr (B == 2) {
    __builtin_nontemporal_store(x[0], reinterpret_cast<uint32_t *>(p));
  } else if constexpr (B == 4) {
    const u32x2_t v = {x[0], x[1]};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x2_t *>(p));
  } else {
    put4<true>(p, x);
  }
}

// ---------------------------------------------------------------------------
// whole light field, images layout
// ---------------------------------------------------------------------------

constexpr int kLFThreads = 512;
constexpr int kLFWaves = kLFThreads / 64;
constexpr int kLFHeadWords = 448;     // LDS words before the residual tile (LUT, per-block extents)
constexpr int kStagePad = 8;          // zero words after the staged group words
using lfc::kRunWords;

// LDS words of the whole-field kernel's compact tile: tile_cap slots of
// stored blocks and one zero slot, rounded up to 16 bytes.
__host__ __device__ constexpr int lf_tile_words(int tile_cap, int S) { return ((tile_cap + 1) * (S / 2) + 3) & ~3; }

struct LFArgs {
  const int16_t *rkv;
  const uint32_t *srv;
  const uint32_t *sched;      // decode schedule: one record per strip (see build_schedule on the host)
  const uint32_t *order;      // [n_strips][order_words] strip of each workgroup, costliest first
  const int32_t *batch;       // [nbatch][kBatchWords] runs of sibling leaves (see internal.h)
  int16_t *out;               // [nv][3][hp][wp]
  int nbx, L, q, wp, hp, nb, nbatch;
  int stage_cap;              // LDS words available for staging the strip
  int vec_store;              // output rows may be stored 16 bytes at a time
  int n_top, key_words;       // key views; LDS words of the strip's key-view rows (0: not staged)
  int tile_cap;               // blocks of the compact residual tile
  int tab_words;              // LDS words of a chunk's gather table and run records
  int stream_out;             // store the output with the non-temporal hint
};

// A whole block of a known kind (0 plain bits, 1 trit, 2 quint) decoded by one
// lane, row by row from memory (8 x 8 blocks, and plain ones too wide for a
// window): d holds the B*B residuals as packed int16 pairs, row-major.  With the
// kind and the row fixed at compile time, every field position except the
// m-dependent low-bit offsets is a constant.
template <int B, int KIND>
__device__ __forceinline__ void decode_block_k(const uint32_t *gw, uint32_t e, int q, const uint16_t *lut,
                                               uint32_t d[B * B / 2]) {
  constexpr int S = B * B;
  constexpr uint32_t HDR = KIND == 0 ? 0u : (KIND == 1 ? Planes<S>::trit : Planes<S>::quint);
  constexpr uint32_t FW = KIND == 1 ? 8u : 7u, GB = KIND == 1 ? 10u : 9u, DB = KIND == 1 ? 2u : 3u;
  constexpr uint32_t LB = KIND == 1 ? 0u : 256u, DMASK = KIND == 1 ? 3u : 7u;
  static_assert(B == 8 || KIND == 0);
  const uint32_t code = e & 31u, rel = e >> 5;
  const uint32_t m = KIND == 0 ? code + 1u : (KIND == 1 ? code - 12u : code - 19u);
  const uint32_t lmask = (1u << m) - 1u;
#pragma unroll
  for (int y = 0; y < B; y++) {
    uint32_t u[B];
    const uint32_t p = rel + HDR + (uint32_t)(y * B) * m;
    {
      const uint64_t v = window64(gw, p);
#pragma unroll
      for (int k = 0; k < (B < 4 ? B : 4); k++) u[k] = (uint32_t)(v >> (k * m)) & lmask;
      if constexpr (B > 4) {
        const uint64_t v2 = window64(gw, p + 4u * m);
#pragma unroll
        for (int k = 4; k < B; k++) u[k] = (uint32_t)(v2 >> ((k - 4) * m)) & lmask;
      }
    }
    if constexpr (KIND != 0) {
      const uint32_t plan = digit_plan(y, KIND == 1);   // a constant once unrolled
      const uint32_t pd = rel + (plan & 0xffu);
      const uint32_t *qd = gw + (pd >> 5);
      const uint32_t win = __builtin_amdgcn_alignbit(qd[1], qd[0], pd & 31u);
      uint64_t D = 0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const uint32_t wdt = (plan >> (16 + 4 * i)) & 15u;
        if (wdt) D |= (uint64_t)lut[LB + ((win >> (i * FW)) & ((1u << wdt) - 1u))] << (i * GB);
      }
      const uint64_t rowd = D >> ((plan >> 8) & 0xffu);
#pragma unroll
      for (int k = 0; k < B; k++) u[k] |= (((uint32_t)(rowd >> (k * DB))) & DMASK) << m;
    }
#pragma unroll
    for (int i = 0; i < B / 2; i++) d[y * (B / 2) + i] = unzigzag_pk(u[2 * i] | (u[2 * i + 1] << 16), q);
  }
}

// A 2 x 2 or 4 x 4 block whose bits are read at once, in one window of
// window_words: every trit and quint block, and plain ones of at most 7 bits
// (others decode row by row from memory).  Pairs of values are taken out by
// packed 16-bit shifts of the word that holds their low bits, digits likewise;
// a pair takes eight operations, five without a digit, against twelve and
// seven, and a block two reads instead of up to fourteen.
template <int B>
constexpr int window_words() { return B == 2 ? 3 : (B == 4 ? 6 : 1); }
template <int B>
struct Window {
  uint32_t w[window_words<B>()];
};
template <int B>
__device__ __forceinline__ void fetch_window(const uint32_t *p, Window<B> &s) {
  if constexpr (B <= 4) {
#pragma unroll
    for (int i = 0; i < window_words<B>(); i++) s.w[i] = p[i];
  }
}

// two shifted copies of a 16-bit field: v's low (HI: high) half >> s per half
template <bool HI>
__device__ __forceinline__ uint32_t shr_both(uint32_t v, uint32_t s) {
  const u16x2 x = as_u16x2(v);
  const unsigned short f = HI ? x[1] : x[0];
  return as_u32((u16x2){f, f} >> as_u16x2(s));
}

// the digits of the pairs of a trit or quint block whose bits are in b, one per
// half, with bits of their neighbours above them
template <int B, int KIND>
__device__ __forceinline__ void pair_digits(const uint32_t *b, const uint16_t *lut, uint32_t dg[B * B / 2]) {
  constexpr int NP = B * B / 2;
  if constexpr (KIND == 1) {
    uint32_t D = lut[b[0] & (B == 4 ? 255u : 127u)];
    if constexpr (B == 4)
      D |= (uint32_t)lut[(b[0] >> 8) & 255u] << 10 | (uint32_t)lut[(b[0] >> 16) & 255u] << 20 |
           (uint32_t)lut[(b[0] >> 24) & 3u] << 30;
#pragma unroll
    for (int i = 0; i < NP; i++) {
      const uint32_t at = 4u * (i % 4);
      dg[i] = i < 4 ? shr_both<false>(D, at | (at + 2u) << 16) : shr_both<true>(D, at | (at + 2u) << 16);
    }
  } else {
    auto field = [&](uint32_t f) { return (uint32_t)lut[256u + f]; };
    if constexpr (B == 4) {
      const uint32_t f1 = field((b[0] >> 7) & 127u), f2 = field((b[0] >> 14) & 127u);
      const uint32_t w0 = field(b[0] & 127u) | f1 << 9, w1 = f1 | f2 << 9;   // digits 0..5, 3..8
      const uint32_t w2 = f2 >> 6 | field((b[0] >> 21) & 127u) << 3 |
                          field(__builtin_amdgcn_alignbit(b[1], b[0], 28) & 127u) << 12;   // 8..14
      const uint32_t w3 = w2 >> 12 | field((b[1] >> 3) & 7u) << 9;                         // 12..15
      dg[0] = shr_both<false>(w0, 0u | 3u << 16);
      dg[1] = shr_both<false>(w0, 6u | 9u << 16);
      dg[2] = shr_both<false>(w1, 3u | 6u << 16);
      dg[3] = shr_both<false>(w1, 9u | 12u << 16);
      dg[4] = shr_both<false>(w2, 0u | 3u << 16);
      dg[5] = shr_both<false>(w2, 6u | 9u << 16);
      dg[6] = shr_both<false>(w3, 0u | 3u << 16);
      dg[7] = shr_both<false>(w3, 6u | 9u << 16);
    } else {
      const uint32_t w0 = field(b[0] & 127u) | field((b[0] >> 7) & 7u) << 9;
      dg[0] = shr_both<false>(w0, 0u | 3u << 16);
      dg[1] = shr_both<false>(w0, 6u | 9u << 16);
    }
  }
}

// the values of a block from its NL words of low bits, m (at most MAXM) a value,
// and its pairs' digits (DIGITS), of which dmask are valid: zigzag undone, times 2^q
template <int B, int NL, int MAXM, bool DIGITS>
__device__ __forceinline__ void pair_values(uint32_t (&l)[NL], const uint32_t *dg, uint32_t m, uint32_t dmask, int q,
                                            uint32_t d[B * B / 2]) {
  constexpr int NP = B * B / 2;
  const uint32_t s01 = m << 16, lm = ((1u << m) - 1u) * 0x10001u;
  const uint32_t zm = DIGITS ? (((dmask + 1u) << m) - 1u) * 0x10001u : lm;
#pragma unroll
  for (int y = 0; y < NP / 2; y++) {   // four values, at most 28 bits, at a time
    const uint32_t v[2] = {shr_both<false>(l[0], s01), shr_both<false>(l[0] >> (2u * m), s01)};
#pragma unroll
    for (int i = 0; i < 2; i++) {
      // digit << m | low bits (what the shift carries into the upper half is
      // below its digit), then the zigzag undone, doubled: z for even z, ~z for odd
      uint32_t z = v[i];
      if constexpr (DIGITS) z = __builtin_amdgcn_bitop3_b32(lm, v[i], dg[2 * y + i] << m, 0xCA);   // lm ? v : digit
      const uint32_t odd = as_u32((u16x2){0, 0} - as_u16x2(z & 0x00010001u));
      d[2 * y + i] = __builtin_amdgcn_bitop3_b32(z, zm, odd, 0x6A);   // (z & zm) ^ odd
    }
#pragma unroll
    for (int i = 0; i < NL; i++)
      if (i < ((NP / 2 - 1 - y) * 4 * MAXM + 31) / 32)
        l[i] = i + 1 < NL ? __builtin_amdgcn_alignbit(l[i + 1], l[i], 4u * m) : l[i] >> (4u * m);
  }
  if (q) {
    const unsigned short k = (unsigned short)(q - 1);
#pragma unroll
    for (int i = 0; i < NP; i++) d[i] = as_u32(as_u16x2(d[i]) << (u16x2){k, k});
  } else {
#pragma unroll
    for (int i = 0; i < NP; i++) d[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, d[i]) >> (i16x2){1, 1});
  }
}

template <int B, int KIND>
__device__ __forceinline__ void decode_window(const Window<B> &s, uint32_t e, int q, const uint16_t *lut,
                                              uint32_t d[B * B / 2]) {
  static_assert(B <= 4);
  constexpr int NP = B * B / 2, MAXM = KIND == 0 ? 7 : 6;
  constexpr int HDR = KIND == 0 ? 0 : (int)(KIND == 1 ? Planes<B * B>::trit : Planes<B * B>::quint);
  constexpr int NB = (HDR + B * B * MAXM + 31) / 32, NL = (B * B * MAXM + 31) / 32;   // words of the block, of its low bits
  static_assert(NB < window_words<B>());
  uint32_t b[NB + 1], l[NL], dg[NP];
#pragma unroll
  for (int i = 0; i < NB; i++) b[i] = __builtin_amdgcn_alignbit(s.w[i + 1], s.w[i], e >> 5);
  b[NB] = 0;
  if constexpr (KIND != 0) pair_digits<B, KIND>(b, lut, dg);
#pragma unroll
  for (int i = 0; i < NL; i++)
    l[i] = HDR % 32 ? __builtin_amdgcn_alignbit(b[i + HDR / 32 + 1], b[i + HDR / 32], HDR % 32) : b[i + HDR / 32];
  const uint32_t m = KIND == 0 ? (e & 31u) + 1u : (KIND == 1 ? (e & 31u) - 12u : (e & 31u) - 19u);
  pair_values<B, NL, MAXM, KIND != 0>(l, dg, m, KIND == 1 ? 3u : 7u, q, d);
}

// A block of any kind (but a plain one too wide), where the lanes of a wave hold
// blocks of all kinds: what the kinds share is done once.
template <int B>
__device__ __forceinline__ void decode_window_any(const Window<B> &s, uint32_t e, int q, const uint16_t *lut,
                                                  uint32_t d[B * B / 2]) {
  constexpr int NP = B * B / 2, NL = (B * B * 7 + 31) / 32, NB = window_words<B>() - 1;
  constexpr uint32_t HT = Planes<B * B>::trit, HQ = Planes<B * B>::quint;
  const uint32_t code = e & 31u;
  const bool plain = code < 12u, trit = code - 12u < 7u;
  uint32_t b[NB + 1], l[NL], dg[NP];
#pragma unroll
  for (int i = 0; i < NB; i++) b[i] = __builtin_amdgcn_alignbit(s.w[i + 1], s.w[i], e >> 5);
  b[NB] = s.w[NB] >> ((e >> 5) & 31u);
#pragma unroll
  for (int i = 0; i < NP; i++) dg[i] = 0;
  if (trit) pair_digits<B, 1>(b, lut, dg);
  else if (!plain) pair_digits<B, 2>(b, lut, dg);
  // the low bits start at bit 0, HT or HQ of the block
  const uint32_t at = plain ? 0u : (trit ? HT : HQ);
  uint32_t c[NL + 1];
#pragma unroll
  for (int i = 0; i <= NL; i++) {
    const uint32_t lo = i <= NB ? b[i] : 0u;
    c[i] = HQ >= 32 && at >= 32u ? (i + 1 <= NB ? b[i + 1] : 0u) : lo;
  }
#pragma unroll
  for (int i = 0; i < NL; i++) l[i] = __builtin_amdgcn_alignbit(c[i + 1], c[i], at & 31u);
  const uint32_t m = code - (plain ? ~0u : (trit ? 12u : 19u));
  pair_values<B, NL, 7, true>(l, dg, m, plain ? 0u : (trit ? 3u : 7u), q, d);
}

// A block of a known kind whose window has been read; base is its group's first word.
template <int B, int KIND>
__device__ __forceinline__ void decode_fetched(const Window<B> &s, const uint32_t *words, uint32_t base, uint32_t e,
                                               int q, const uint16_t *lut, uint32_t d[B * B / 2]) {
  if constexpr (B <= 4) {
    if (KIND != 0 || lfc::window_code(e & 31u)) {
      decode_window<B, KIND>(s, e, q, lut, d);
      return;
    }
  }
  if constexpr (B == 8 || KIND == 0) decode_block_k<B, KIND>(words + base, e, q, lut, d);
}

// A whole 8 x 8 block of any kind decoded by one lane, row by row (one code for
// the three kinds, the row plans constant).
__device__ __forceinline__ void decode_block(const uint32_t *gw, uint32_t e, int q, const uint16_t *lut, uint32_t d[32]) {
#pragma unroll
  for (int y = 0; y < 8; y++) decode_row(gw, e, digit_plan(y, true), digit_plan(y, false), y, q, lut, d + 4 * y);
}

// n words from global memory into LDS, without a round trip through
// registers: lane i of each wave-wide load writes dst[i0 + i].
__device__ __forceinline__ void lds_copy(uint32_t *dst, const uint32_t *src, uint32_t n, int lane) {
  for (uint32_t i0 = 0; i0 < n; i0 += 64)
    if (i0 + (uint32_t)lane < n)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + i0 + lane),
                                       (__attribute__((address_space(3))) void *)(dst + i0), 4, 0, 0);
}

// A workgroup barrier for data exchanged through LDS only: this wave's LDS
// operations complete before it, but its global stores stay in flight (a
// __syncthreads() would also wait for every outstanding store of the wave,
// and the whole-field kernel's stores need not be visible to other waves).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0); vmcnt and expcnt not waited on
  __builtin_amdgcn_s_barrier();
}

// Tables that every lane of a wave reads at the same address (tree runs,
// chunk records) are read through the scalar unit: a vector load would make
// the wave wait for all of its outstanding stores as well.
typedef const __attribute__((address_space(4))) int32_t *uniform_i32;
__device__ __forceinline__ uniform_i32 as_uniform(const int32_t *p) { return (uniform_i32)p; }

// One workgroup = one channel c, one row of blocks by, one strip of 64/B
// consecutive blocks (64 pixels).  Phase A copies into LDS what fits of the
// strip's data: its groups and its decode schedule (tier 1), else the
// schedule only (tier 2: payload read through bit windows from global
// memory), else nothing (tier 3, the default), plus its key-view rows.  Phase B
// walks the strip's chunks (runs of sibling leaves in serial order whose
// stored blocks fit the compact tile): (3) every stored block of the chunk is
// decoded once, whole, by one lane, with the decoder of its range kind, into
// its slot of the tile; (4) per sibling run, key-view row + ancestor rows +
// leaf row (absent blocks add nothing), stored 16 bytes per lane.
// What bounds it is memory where the light field is sparse (289 views of
// 512 x 512 at 40 dB: 105 -> 101 us, 5.2 TB/s) and was, where it is dense, the
// vector-memory path (eleven short reads per block), LDS bank conflicts and the
// issue of vector instructions.  Hence one window per block, entries in an order
// in which a wave's windows adjoin, a tile of 16-byte planes, node masks whose
// bits lie as the lanes that test them, tables read from LDS alone, and
// everything a chunk needs read before the chunk before it stores (a load waits
// for older stores).  At 50 dB (15.9 M blocks): 172 -> 121 us, 635 MB at
// 5.2 TB/s; 62 -> 49 million vector instructions, LDS conflicts 40 -> 16 million
// cycles.  Staged (STAGED: the caller gave LDS for it), a strip's chunks are
// read when they are decoded.
// (B <= 4: at most 80 VGPRs, six waves per SIMD, so three workgroups share a
// compute unit whenever their LDS fits; B = 8 keeps its registers)
template <int B, bool STAGED, bool KEYS>
__global__ __launch_bounds__(kLFThreads, B <= 4 ? 6 : 1) void k_decode_lf(LFArgs a) {
  constexpr int S = B * B, NBLK = 64 / B, H = B / 2;
  constexpr int PB = 8 / B;                            // blocks per 16-byte row segment (1 for B = 8)
  extern __shared__ uint32_t smem[];
  const uint16_t *lut = reinterpret_cast<const uint16_t *>(smem);   // 384 x u16 = 192 words
  uint32_t *s_o0 = smem + 192;                         // group start word in the SRV section
  uint32_t *s_len = smem + 256;                        // group length in words
  uint32_t *s_wo = smem + 320;                         // staged group words
  uint32_t *s_cnt = smem + 384;                        // [0] tier, [1] staged group words, [2] schedule words
  uint32_t *tile = smem + kLFHeadWords;                // compact tile, the last slot zero (tile_quad)
  uint32_t *keys = tile + lf_tile_words(a.tile_cap, S); // [n_top][B][NBLK][H]
  uint32_t *s_tab = keys + a.key_words;                 // two chunks' gather tables (tier 3) and run records
  uint32_t *stage = s_tab + 2 * a.tab_words;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the workgroup's strip (strips are taken costliest first, so the last
  // workgroups to start are short ones)
  // (its order entry: the strip, its schedule, its groups; one load)
  constexpr int OW = lfc::order_words(B);
  const uint32_t *ent = a.order + (size_t)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * OW;
  const uniform_i32 uent = as_uniform(reinterpret_cast<const int32_t *>(ent));
  const int st = uent[0];
  const int sx = st % (int)gridDim.x, by = (st / (int)gridDim.x) % (int)gridDim.y, c = st / ((int)gridDim.x * (int)gridDim.y);
  const uint32_t sched0 = (uint32_t)uent[1], sched_len = (uint32_t)uent[2];
  // the strip's chunk count and chunk headers (scalar loads)
  const uint32_t *gs = a.sched + sched0;
  const uniform_i32 head = as_uniform(reinterpret_cast<const int32_t *>(gs));
  const int nck = head[0];
  struct Header {
    int at, q0, nq, nn;
    uint32_t n0, n01, n;
    int words;   // of the gather table
  };
  auto header = [&](int ci) {
    const uniform_i32 h = head + 8 + 8 * ci;
    Header r{h[0], h[1], h[2], h[3], (uint32_t)h[4], (uint32_t)h[5], (uint32_t)h[6], 0};
    r.words = (B == 2 ? r.nn + (r.nn + 1) / 2 : r.nn) + 3 * r.nq;
    return r;
  };
  // h: the chunk being decoded, hn: the one after it.  Unless staged, the lane
  // holds its first two entries of each, (e, t) and (f, u).  (A lane past a
  // chunk's last entry takes that entry: it decodes the same block into the same
  // slot.)
  Header h{}, hn{};
  uint32_t e[2] = {}, t[2] = {}, f[2] = {}, u[2] = {};
  auto entry = [&](const Header &r, uint32_t it, uint32_t &en, uint32_t &item) {
    const uint32_t *ents = gs + r.at + r.words;
    const uint32_t i = min(it, r.n - 1);
    en = ents[i];
    item = reinterpret_cast<const uint16_t *>(ents + r.n)[i];
  };
  // a chunk's gather table, unless it is staged, and after it its run records into LDS
  auto tables_to_lds = [&](const Header &r, uint32_t *dst, bool tab) {
    if (tab) {
      for (int w = wave * 64; w < r.words; w += kLFThreads)
        if (w + lane < r.words)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gs + r.at + w + lane),
                                           (__attribute__((address_space(3))) void *)(dst + w), 4, 0, 0);
      dst += r.words;
    }
    const uint32_t *recs = reinterpret_cast<const uint32_t *>(a.batch + (size_t)a.nbatch * lfc::kBatchWords) +
                           (size_t)r.q0 * kRunWords;
    for (int w = wave * 64; w < kRunWords * r.nq; w += kLFThreads)
      if (w + lane < kRunWords * r.nq)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(recs + w + lane),
                                         (__attribute__((address_space(3))) void *)(dst + w), 4, 0, 0);
  };
  if (a.L > 1) {
    h = header(0);
    if (nck > 1) hn = header(1);
    if constexpr (!STAGED) {
#pragma unroll
      for (int k = 0; k < 2; k++) {
        if (h.n) entry(h, tid + k * kLFThreads, e[k], t[k]);
        if (hn.n) entry(hn, tid + k * kLFThreads, f[k], u[k]);
      }
      tables_to_lds(h, s_tab, true);
    }
  }
  // the LUT from its table (a copy straight into LDS)
  if (tid < kLutEntries / 2) __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void *)(kLutTable.w + tid),
      (__attribute__((address_space(3))) void *)(smem + (tid & ~63)), 4, 0, 0);
  // 16-byte quad k of tile slot s (B = 2: a slot is 8 bytes): a slot's quads lie
  // tile_cap + 1 quads apart, so that lanes at neighbouring slots reach
  // different banks
  const int plane = 4 * (a.tile_cap + 1);
  if (tid < S / 2) tile[B == 2 ? a.tile_cap * (S / 2) + tid : (tid / 4) * plane + a.tile_cap * 4 + tid % 4] = 0u;
  if constexpr (!STAGED) {
    if (tid < NBLK) s_o0[tid] = ent[4 + tid];
  } else if (tid < 64) {
    // wave 0: the strip's group offsets and lengths, their exclusive prefix
    // sum (a wave scan) and the staging tier
    uint32_t o0 = 0, len = 0;
    if (lane < NBLK) {
      o0 = ent[4 + lane];
      len = ent[4 + NBLK + lane];
    }
    uint32_t incl = len;
#pragma unroll
    for (int d = 1; d < NBLK; d <<= 1) {
      const uint32_t v = __shfl_up(incl, d);
      if (lane >= d) incl += v;
    }
    const uint32_t words = __shfl(incl, NBLK - 1);
    if (lane < NBLK) {
      s_o0[lane] = o0;
      s_len[lane] = len;
      s_wo[lane] = incl - len;
    }
    if (lane == 0) {
      // tier 1: [group words][pad][schedule]; tier 2: [schedule]
      const uint32_t tier = words + kStagePad + sched_len <= (uint32_t)a.stage_cap ? 1u
                            : (sched_len <= (uint32_t)a.stage_cap ? 2u : 3u);
      s_cnt[0] = tier;
      s_cnt[1] = tier == 1u ? words : 0u;
      s_cnt[2] = tier == 1u ? words + kStagePad : 0u;
    }
  }
  if constexpr (KEYS) {
    // the strip's key-view rows, [root][row][block][H]: a wave's load covers two
    // rows (64 words) of a root
    const uint32_t *rk = reinterpret_cast<const uint32_t *>(a.rkv) +
                         ((size_t)(by * a.nbx + sx * NBLK + (lane & 31) / H) * 3 + c) * (S / 2) + (lane >> 5) * H + lane % H;
    const bool in = sx * NBLK + (lane & 31) / H < a.nbx;
    for (int f = wave; f < a.n_top * (B / 2); f += kLFWaves)
      if (in)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)(rk + (size_t)(f / (B / 2)) * a.nb * (3 * S / 2) + f % (B / 2) * B),
            (__attribute__((address_space(3))) void *)(keys + f * 64), 4, 0, 0);
  }
  uint32_t tier = 3, sched_at = 0;
  if constexpr (STAGED) {
    __syncthreads();
    tier = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cnt[0]);
    sched_at = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cnt[2]);
    // every copy goes straight from global memory to LDS, all in flight at once
    if (tier == 1u)
      for (int j = wave; j < NBLK; j += kLFWaves)
        if (s_len[j]) lds_copy(stage + s_wo[j], a.srv + s_o0[j], s_len[j], lane);
    if (tier < 3u) {
      // the schedule, split over the waves in pieces of whole 64-word rows
      const uint32_t rows = (sched_len + 63) / 64, per = (rows + kLFWaves - 1) / kLFWaves;
      const uint32_t r0 = min(rows, (uint32_t)wave * per), r1 = min(rows, r0 + per);
      if (r1 > r0) lds_copy(stage + sched_at + r0 * 64, a.sched + sched0 + r0 * 64, min(sched_len, r1 * 64) - r0 * 64, lane);
    }
    if (tier == 1u && tid < kStagePad) stage[s_cnt[1] + tid] = 0;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const uint32_t vstride = 3u * (uint32_t)a.hp * (uint32_t)a.wp;
  const uint64_t cplane = (uint64_t)c * a.hp * a.wp;
  if (a.L == 1) {
    // no residual levels: every view is a stored key view
    const int j = lane % NBLK, y = lane / NBLK, bx = sx * NBLK + j;
    if (bx >= a.nbx) return;
    const int b = by * a.nbx + bx;
    const int per = (a.nbatch + kLFWaves - 1) / kLFWaves;
    for (int qb = wave * per; qb < min(a.nbatch, wave * per + per); qb++) {
      const uniform_i32 rec = as_uniform(a.batch + (size_t)qb * lfc::kBatchWords);
      uint32_t x[H];
      load_row<B>(a.rkv + ((size_t)(rec[5] * a.nb + b) * 3 + c) * S + y * B, x);
      int16_t *dst = a.out + (size_t)rec[1] * vstride + cplane + (size_t)(by * B + y) * a.wp + bx * B;
      if (a.stream_out) put_row<B, true>(dst, x);
      else put_row<B, false>(dst, x);
    }
    return;
  }
  // store-side lane mapping: run of the wave's pair (lane / 32), sibling in
  // the run, segment of PB blocks (16 bytes of each of the B rows)
  const int half = lane >> 5, so = (lane >> 3) & 3, jq = lane & 7;
  const int bx0 = sx * NBLK + jq * PB;
  const int nact = max(0, min(PB, a.nbx - bx0));       // blocks of the segment inside the image
  const bool wide = nact == PB && a.vec_store;          // a 16-byte store is aligned
  const uint64_t lane_off = cplane + (uint64_t)(by * B) * a.wp + (uint64_t)bx0 * B;
  const uint32_t zslot = (uint32_t)a.tile_cap;          // the zeroed slot

  // (3) one entry: its block's residuals into its tile slot
  auto decode_to_tile = [&](uint32_t it, const Window<B> &w, const uint32_t *words, uint32_t base, uint32_t en, uint32_t item) {
    uint32_t d[S / 2];
    if (it < h.n0) decode_fetched<B, 0>(w, words, base, en, a.q, lut, d);
    else if (it < h.n01) decode_fetched<B, 1>(w, words, base, en, a.q, lut, d);
    else decode_fetched<B, 2>(w, words, base, en, a.q, lut, d);
    uint32_t *dst = tile + (item >> 5) * (B == 2 ? 2 : 4);
    if constexpr (B == 2) {
      *reinterpret_cast<uint2 *>(dst) = make_uint2(d[0], d[1]);
    } else {
#pragma unroll
      for (int k = 0; k < S / 8; k++)
        *reinterpret_cast<uint4 *>(dst + k * plane) = make_uint4(d[4 * k], d[4 * k + 1], d[4 * k + 2], d[4 * k + 3]);
    }
  };
  // (4) a wave takes two runs at a time, one per half; a lane owns one sibling
  // of its run and one 16-byte segment (PB blocks) of the strip's rows.  Node
  // tables and run records come from LDS (a vector load would wait for the
  // wave's outstanding stores); an absent block reads the zeroed slot (no
  // masking).  nodes_c: nodes of a path, -1 if found at run time.
  auto gather = [&](auto nodes_c, int nq, int nn, const uint32_t *tab, const uint32_t *rec) {
    constexpr int NC = decltype(nodes_c)::value, NM = NC < 0 ? lfc::kMaxLevels - 1 : NC;
    const int nodes = NC < 0 ? a.L - 1 : NC;
    const uint16_t *firsts = reinterpret_cast<const uint16_t *>(tab + nn);   // (B = 2)
    const uint32_t *runs = tab + (B == 2 ? nn + (nn + 1) / 2 : nn);
    for (int qp = wave; 2 * qp < nq; qp += kLFWaves) {
      const int qi = min(2 * qp + half, nq - 1);
      const int vi = rec[kRunWords * qi + so], root = rec[kRunWords * qi + 4];
      const bool live = 2 * qp + half < nq && vi >= 0;
      int node[NM];
      {
        const uint32_t w0 = runs[3 * qi];
        node[0] = min((int)(w0 & 0xFFFFu) + so, nn - 1);
        if constexpr (NM > 1) node[1] = (int)(w0 >> 16);
        if constexpr (NM > 2) {
          const uint32_t w1 = runs[3 * qi + 1], w2 = runs[3 * qi + 2];
          node[2] = (int)(w1 & 0xFFFFu);
          node[3] = (int)(w1 >> 16);
          node[4] = (int)(w2 & 0xFFFFu);
        }
      }
      uint32_t slot[NM][PB];
#pragma unroll
      for (int k = 0; k < NM; k++) {
        if (NC < 0 && k >= nodes) continue;
        const uint32_t w = tab[node[k]];
        const uint32_t first = B == 2 ? firsts[node[k]] : w >> 16;
#pragma unroll
        for (int b = 0; b < PB; b++) {
          const uint32_t bit = (uint32_t)(jq + 8 * b);
          const uint32_t sl = first + (uint32_t)__popc(w & ((1u << bit) - 1u));
          slot[k][b] = ((w >> bit) & 1u ? sl : zslot) * (B == 2 ? 2 : 4);
        }
      }
      // key-view rows
      uint32_t x[B][4];
      if constexpr (KEYS) {
#pragma unroll
        for (int y = 0; y < B; y++) {
          const uint4 k4 = reinterpret_cast<const uint4 *>(keys)[(((root * B + y) * NBLK + jq * PB) * H) / 4];
          x[y][0] = k4.x;
          x[y][1] = k4.y;
          x[y][2] = k4.z;
          x[y][3] = k4.w;
        }
      } else {
#pragma unroll
        for (int y = 0; y < B; y++) {
#pragma unroll
          for (int w = 0; w < 4; w++) x[y][w] = 0;
#pragma unroll
          for (int k = 0; k < PB; k++)
            if (k < nact)
              load_row<B>(a.rkv + ((size_t)(root * a.nb + by * a.nbx + bx0 + k) * 3 + c) * S + y * B, x[y] + k * H);
        }
      }
      // node rows added to every row of the lane's blocks
#pragma unroll
      for (int k = 0; k < NM; k++) {
        if (NC < 0 && k >= nodes) continue;
#pragma unroll
        for (int b = 0; b < PB; b++) {
          const uint32_t *t = tile + slot[k][b];
          if constexpr (B == 2) {
            const uint2 v = *reinterpret_cast<const uint2 *>(t);
            x[0][b] = add_pk(x[0][b], v.x);
            x[1][b] = add_pk(x[1][b], v.y);
          } else {
#pragma unroll
            for (int i = 0; i < S / 8; i++) {
              const uint4 v = *reinterpret_cast<const uint4 *>(t + i * plane);
              const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int z = 0; z < 4; z++) {
                uint32_t &xw = x[(4 * i + z) / H][H * b + (4 * i + z) % H];
                xw = add_pk(xw, w[z]);
              }
            }
          }
        }
      }
      if (!live) continue;
      int16_t *dst = a.out + ((uint64_t)(uint32_t)vi * vstride + lane_off);
      // separate loops, so that the 16-byte stores stay whole
      if (wide && a.stream_out) {
#pragma unroll
        for (int y = 0; y < B; y++) put4<true>(dst + (size_t)y * a.wp, x[y]);
      } else if (wide) {
#pragma unroll
        for (int y = 0; y < B; y++) put4<false>(dst + (size_t)y * a.wp, x[y]);
      } else if (nact > 0) {
#pragma unroll
        for (int y = 0; y < B; y++)
#pragma unroll
          for (int k = 0; k < PB; k++)
            if (k < nact) {
              if (a.stream_out) put_row<B, true>(dst + (size_t)y * a.wp + k * B, x[y] + k * H);
              else put_row<B, false>(dst + (size_t)y * a.wp + k * B, x[y] + k * H);
            }
      }
    }
  };
  auto fetch = [&](uint32_t en, uint32_t item, Window<B> &w) { fetch_window<B>(a.srv + (s_o0[item & 31u] + (en >> 10)), w); };
  Window<B> w[2] = {};
  if (!STAGED && h.n) {
    fetch(e[0], t[0], w[0]);
    fetch(e[1], t[1], w[1]);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // landed (in the loop no wait for them would tell them from stores)
  }
  for (int ci = 0; ci < nck; ci++) {
    const int nq = h.nq, nn = h.nn;
    const uint32_t n = h.n;
    uint32_t *tab = s_tab + (ci & 1) * a.tab_words, *rec = tab + h.words;
    if constexpr (!STAGED) {
      // the first two blocks of a lane have been read; the next chunk's are
      // requested here, with its tables and the entries of the one after it, so
      // that all have landed before the gather's stores (a load waits for older
      // stores)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        if ((uint32_t)(wave * 64 + k * kLFThreads) < n)
          decode_to_tile(min((uint32_t)(tid + k * kLFThreads), n - 1), w[k], a.srv, s_o0[t[k] & 31u], e[k], t[k]);
        e[k] = f[k], t[k] = u[k];
        if (hn.n) fetch(e[k], t[k], w[k]);
      }
      for (uint32_t b = wave * 64 + 2 * kLFThreads; b < n; b += kLFThreads) {
        uint32_t en, item;
        entry(h, b + lane, en, item);
        Window<B> wb;
        fetch(en, item, wb);
        decode_to_tile(min(b + lane, n - 1), wb, a.srv, s_o0[item & 31u], en, item);
      }
    } else {
      // tier 3: tables, entries and payload from global memory; tier 2: payload
      if (tier < 3u) {
        rec = s_tab;
        tab = stage + sched_at + h.at;
      }
      tables_to_lds(h, tier < 3u ? rec : tab, tier == 3u);
      if (tier == 1u) {
        const uint32_t *ents = tab + h.words;
        const uint16_t *items = reinterpret_cast<const uint16_t *>(ents + n);
        for (uint32_t it = tid; it < n; it += kLFThreads) {
          const uint32_t en = ents[it], item = items[it], base = s_wo[item & 31u];
          Window<B> wb;
          fetch_window<B>(stage + (base + (en >> 10)), wb);
          decode_to_tile(it, wb, stage, base, en, item);
        }
      } else {
        for (uint32_t it = tid; it < n; it += kLFThreads) {
          uint32_t en, item;
          if (tier == 2u) {
            const uint32_t *ents = tab + h.words;
            en = ents[it];
            item = reinterpret_cast<const uint16_t *>(ents + n)[it];
          } else {
            entry(h, it, en, item);
          }
          Window<B> wb;
          fetch(en, item, wb);
          decode_to_tile(it, wb, a.srv, s_o0[item & 31u], en, item);
        }
      }
    }
    h = hn;
    hn.n = 0;
    if (ci + 2 < nck) hn = header(ci + 2);
    if constexpr (!STAGED) {
#pragma unroll
      for (int k = 0; k < 2; k++)
        if (hn.n) entry(hn, tid + k * kLFThreads, f[k], u[k]);
      if (ci + 1 < nck) tables_to_lds(h, s_tab + (~ci & 1) * a.tab_words, true);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's reads have landed
    lds_barrier();
    __builtin_amdgcn_s_setprio(2);   // gather issue first; another workgroup's decode fills the gaps
    if (a.L == 2) gather(std::integral_constant<int, 1>{}, nq, nn, tab, rec);
    else if (a.L == 3) gather(std::integral_constant<int, 2>{}, nq, nn, tab, rec);
    else gather(std::integral_constant<int, -1>{}, nq, nn, tab, rec);
    __builtin_amdgcn_s_setprio(0);
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// random access: one (view, block) at a time through the directory
// ---------------------------------------------------------------------------

struct RAArgs {
  const int16_t *rkv;
  const uint32_t *off;
  const uint32_t *srv;
  const uint32_t *poff;
  const int32_t *path;
  const int32_t *root;
  int nb, nbx, nv, nbw, L, q;
  const uint32_t *dir2;   // [nb][nbw][3] (bitmap word, directory index of its first stored node) pairs
};

// Row y of 8 x 8 block b, channel c, of view vi (Alg. 2): key-view row plus the
// residual rows of the view's ancestors on levels L-2 down to stop (0: the
// view itself; a higher stop is progressive decompression, Sec. 3.6), as
// packed int16 pairs.
__device__ __forceinline__ void gather_row(const RAArgs &a, int vi, int b, int c, int y, int stop, uint32_t plan_t,
                                           uint32_t plan_q, const uint16_t *lut, uint32_t x[4]) {
  constexpr int B = 8, S = B * B;
  const int root = a.root[vi];
  load_row<B>(a.rkv + ((size_t)(root * a.nb + b) * 3 + c) * S + y * B, x);
  const int g = 3 * b + c;
  const uint32_t o0 = a.off[g], o1 = a.off[g + 1];
  if (o0 == o1) return;
  const uint32_t *gw = a.srv + o0;
  const int depth = a.L - 1;
  for (int l = depth - 1; l >= stop; --l) {
    const int s = a.path[vi * depth + l];
    // the bitmap word and the directory index of its first stored node, read together
    const uint2 bd = *reinterpret_cast<const uint2 *>(a.dir2 + (((size_t)b * a.nbw + (s >> 5)) * 3 + c) * 2);
    const uint32_t bm = bd.x;
    const uint32_t bit = (uint32_t)s & 31u;
    if ((bm >> bit) & 1u) {
      const uint32_t idx = bd.y + __popc(bm & ((1u << bit) - 1u));
      uint32_t d[B / 2];
      decode_row(gw, a.poff[idx], plan_t, plan_q, y, a.q, lut, d);
#pragma unroll
      for (int i = 0; i < B / 2; i++) x[i] = add_pk(x[i], d[i]);
    }
  }
}

// Block b, channel c, of view vi whole (B <= 4), by one lane: as gather_row, two
// levels' directory entries, offsets and windows read side by side (an absent
// block reads the first ones and is not added).
template <int B>
__device__ __forceinline__ void gather_block(const RAArgs &a, int vi, int b, int c, int stop, const uint16_t *lut,
                                             uint32_t x[B * B / 2]) {
  constexpr int S = B * B;
  const int root = a.root[vi], g = 3 * b + c, depth = a.L - 1;
  const uint32_t *key = reinterpret_cast<const uint32_t *>(a.rkv + ((size_t)(root * a.nb + b) * 3 + c) * S);
  if constexpr (B == 4) {
    const uint4 k0 = *reinterpret_cast<const uint4 *>(key), k1 = *reinterpret_cast<const uint4 *>(key + 4);
    x[0] = k0.x, x[1] = k0.y, x[2] = k0.z, x[3] = k0.w;
    x[4] = k1.x, x[5] = k1.y, x[6] = k1.z, x[7] = k1.w;
  } else {
    const uint2 k0 = *reinterpret_cast<const uint2 *>(key);
    x[0] = k0.x, x[1] = k0.y;
  }
  const uint32_t o0 = a.off[g];
  const bool any = o0 != a.off[g + 1];
  for (int top = depth - 1; top >= stop; top -= 2) {
    uint2 bd[2];
    uint32_t bit[2], e[2];
    bool in[2];
    Window<B> w[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const int s = a.path[vi * depth + max(top - k, stop)];
      bit[k] = (uint32_t)s & 31u;
      // the bitmap word and the directory index of its first stored node, read together
      bd[k] = *reinterpret_cast<const uint2 *>(a.dir2 + (((size_t)b * a.nbw + (s >> 5)) * 3 + c) * 2);
    }
#pragma unroll
    for (int k = 0; k < 2; k++) {
      in[k] = any && top - k >= stop && ((bd[k].x >> bit[k]) & 1u);
      e[k] = a.poff[in[k] ? bd[k].y + __popc(bd[k].x & ((1u << bit[k]) - 1u)) : 0u];
    }
#pragma unroll
    for (int k = 0; k < 2; k++) fetch_window<B>(a.srv + (in[k] ? o0 + (e[k] >> 10) : 0u), w[k]);
#pragma unroll
    for (int k = 0; k < 2; k++) {
      if (!in[k]) continue;
      uint32_t d[S / 2];
      if (lfc::window_code(e[k] & 31u)) decode_window_any<B>(w[k], e[k], a.q, lut, d);
      else decode_block_k<B, 0>(a.srv + o0, e[k], a.q, lut, d);
#pragma unroll
      for (int i = 0; i < S / 2; i++) x[i] = add_pk(x[i], d[i]);
    }
  }
}

// Lanes per request: one per channel, which decodes the whole block (B <= 4), or
// one per channel and row.  Random accesses are bound by the latency of their
// chain of reads (request - path - directory - offset - window) and by the lines
// they read past L2, about eight; with three lanes a request four times as many
// are in flight as with one per row, and the levels' chains run side by side.
// 10^6 blocks of 289 views of 512 x 512: 167 -> 135 us, sorted by block 142 -> 47.
template <int B>
constexpr int request_lanes() { return B <= 4 ? 3 : 3 * B; }

// the LUT, copied to LDS by the whole workgroup
__device__ __forceinline__ void load_lut(uint32_t *lut) {
  for (int t = threadIdx.x; t < kLutEntries / 2; t += kThreads) lut[t] = kLutTable.w[t];
  __syncthreads();
}

// Request r = (vi, b) by its lanes, of which this one is sub: the block, or zeros
// and the error flag if the request is out of range (out is aligned to 16 bytes).
template <int B>
__device__ __forceinline__ void serve_request(const RAArgs &ra, bool valid, int vi, int b, int64_t r, int sub, int stop,
                                              const uint16_t *lut, int16_t *out, int32_t *err) {
  constexpr int S = B * B;
  if (!valid && sub == 0) atomicOr(err, 1);
  if constexpr (B <= 4) {
    uint32_t x[S / 2] = {};
    if (valid) gather_block<B>(ra, vi, b, sub, stop, lut, x);
    int16_t *dst = out + ((size_t)r * 3 + sub) * S;
    if constexpr (B == 4) {
      *reinterpret_cast<uint4 *>(dst) = make_uint4(x[0], x[1], x[2], x[3]);
      *reinterpret_cast<uint4 *>(dst + 8) = make_uint4(x[4], x[5], x[6], x[7]);
    } else {
      *reinterpret_cast<uint2 *>(dst) = make_uint2(x[0], x[1]);
    }
  } else {
    const int c = sub / B, y = sub % B;
    uint32_t x[B / 2] = {};
    if (valid) gather_row(ra, vi, b, c, y, stop, digit_plan(y, true), digit_plan(y, false), lut, x);
    store_row<B>(out + ((size_t)r * 3 + c) * S + y * B, x);
  }
}

struct BlocksArgs {
  RAArgs ra;
  const int32_t *req;  // [n][2] or null
  int16_t *out;        // [n][3][S]
  int32_t *err;
  int64_t n;
  int stop;            // lowest tree level whose residuals are added
};

template <int B>
__global__ __launch_bounds__(kThreads) void k_decode_blocks(BlocksArgs a) {
  constexpr int LPR = request_lanes<B>(), RPW = 64 / LPR;
  __shared__ uint32_t lut[kLutEntries / 2];
  load_lut(lut);
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int slot = lane / LPR, sub = lane % LPR;
  if (slot >= RPW) return;
  const int64_t r = wave * RPW + slot;
  if (r >= a.n) return;
  int vi, b;
  if (a.req) {
    vi = a.req[2 * r];
    b = a.req[2 * r + 1];
  } else {
    vi = (int)(r / a.ra.nb);
    b = (int)(r % a.ra.nb);
  }
  const bool valid = vi >= 0 && vi < a.ra.nv && b >= 0 && b < a.ra.nb;
  serve_request<B>(a.ra, valid, vi, b, r, sub, a.stop, reinterpret_cast<const uint16_t *>(lut), a.out, a.err);
}

// The same for a long list over a light field whose tables exceed an L2 several
// times.  The blocks fall into eight bands, by a hash of four neighbouring ones,
// and the workgroups of one die (blockIdx % 8 is its number) serve the requests
// of one band, so that its 4 MB L2 sees an eighth of the tables.  Each die's
// workgroup reads a piece of 512 requests, picks its band's, 64 or so, and serves
// them.  Where a piece's requests crowd into few bands (one holds twice its
// share), its workgroups take equal parts of it instead; all of them see the same
// piece and decide alike.  10^6 random blocks of 289 views of 512 x 512: 135 ->
// 97 us (sorted by block, which no list here need be, 47 -> 64).
constexpr int64_t kBandRequests = 1 << 17, kBandBytes = (int64_t)13 << 20;

template <int B>
__global__ __launch_bounds__(kThreads) void k_decode_banded(BlocksArgs a) {
  constexpr int LPR = request_lanes<B>(), RPW = 64 / LPR, NW = kThreads / 64, PER = 2, PIECE = PER * kThreads, SHARE = PIECE / 8;
  __shared__ uint32_t lut[kLutEntries / 2];
  __shared__ int s_count[NW][8];
  __shared__ uint16_t s_at[PIECE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), mine = blockIdx.x % 8;
  const int64_t r0 = (int64_t)(blockIdx.x / 8) * PIECE;
  const int n = (int)min((int64_t)PIECE, a.n - r0);
  const int32_t *req = a.req + 2 * r0;
  int band[PER];
#pragma unroll
  for (int i = 0; i < PER; i++) {
    const int k = i * kThreads + threadIdx.x;
    band[i] = k < n ? (int)(((uint32_t)req[2 * k + 1] / 4u * 0x9E3779B1u) >> 29) : -1;
  }
  for (int t = threadIdx.x; t < kLutEntries / 2; t += kThreads) lut[t] = kLutTable.w[t];
  int count = 0;   // lane k: the wave's requests of band k
#pragma unroll
  for (int k = 0; k < 8; k++) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < PER; i++) c += __popcll(__ballot(band[i] == k));
    if (lane == k) count = c;
  }
  if (lane < 8) s_count[wave][lane] = count;
  __syncthreads();
  int first = 0, total = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < NW; w++) {
    if (w < wave) first += s_count[w][mine];
    total += s_count[w][mine];
    sum += s_count[w][lane & 7];
  }
  const bool crowded = __any(sum > 2 * SHARE);
  if (crowded) {
    total = min(SHARE, max(0, n - mine * SHARE));
  } else {
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const uint64_t m = __ballot(band[i] == mine);
      const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (band[i] == mine) s_at[first + below] = (uint16_t)(i * kThreads + threadIdx.x);
      first += __popcll(m);
    }
  }
  __syncthreads();
  const int slot = lane / LPR, sub = lane % LPR;
  if (slot >= RPW) return;
  for (int i = wave * RPW + slot; i < total; i += NW * RPW) {
    const int k = crowded ? mine * SHARE + i : (int)s_at[i];
    const int vi = req[2 * k], b = req[2 * k + 1];
    const bool valid = vi >= 0 && vi < a.ra.nv && b >= 0 && b < a.ra.nb;
    serve_request<B>(a.ra, valid, vi, b, r0 + k, sub, a.stop, reinterpret_cast<const uint16_t *>(lut), a.out, a.err);
  }
}

// Random access over many light fields of one block size in one launch:
// request r = (light field, view, block) indexes a table of the light
// fields' device tables; otherwise as k_decode_blocks.
struct MultiArgs {
  const RAArgs *lfs;
  int32_t n_lf;
  const int32_t *req;  // [n][3]
  int16_t *out;        // [n][3][S]
  int32_t *err;
  int64_t n;
};

template <int B>
__global__ __launch_bounds__(kThreads) void k_decode_multi(MultiArgs a) {
  constexpr int LPR = request_lanes<B>(), RPW = 64 / LPR;
  __shared__ uint32_t lut[kLutEntries / 2];
  load_lut(lut);
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int slot = lane / LPR, sub = lane % LPR;
  if (slot >= RPW) return;
  const int64_t r = wave * RPW + slot;
  if (r >= a.n) return;
  const int li = a.req[3 * r], vi = a.req[3 * r + 1], b = a.req[3 * r + 2];
  const bool known = li >= 0 && li < a.n_lf;
  RAArgs la{};
  if (known) la = a.lfs[li];   // the light field's record, read once
  const bool valid = known && vi >= 0 && vi < la.nv && b >= 0 && b < la.nb;
  serve_request<B>(la, valid, vi, b, r, sub, 0, reinterpret_cast<const uint16_t *>(lut), a.out, a.err);
}

// ---------------------------------------------------------------------------
// novel views: footprint decode into LDS, then quadrilinear interpolation
// ---------------------------------------------------------------------------

struct RenderArgs {
  RAArgs ra;
  const lfc_view *views;
  float *out;  // [n][3][ho][wo]
  int wo, ho, U, V, W, H, TX, TY, fbx_max, fby_max;
  float disp;  // focal disparity: image-plane shift per unit of camera-grid offset
};

// lower grid index, upper index and fraction of x on [0, n-1], after clamping
__device__ __forceinline__ void cell(float x, int n, int &i0, int &i1, float &f) {
  x = fminf(fmaxf(x, 0.0f), (float)(n - 1));
  if (n == 1) {
    i0 = i1 = 0;
    f = 0.0f;
    return;
  }
  int i = (int)floorf(x);
  i = min(max(i, 0), n - 2);
  i0 = i;
  i1 = i + 1;
  f = x - (float)i;
}

__device__ __forceinline__ float lerpf(float a, float b, float f) { return a + f * (b - a); }

// The residual-block entry (payload offset << 5 | code) of node s in group g,
// or kAbsent, through the directory built at initialisation.
__device__ __forceinline__ uint32_t locate(const RAArgs &a, int g, int s, const uint32_t **gw_out) {
  const uint32_t o0 = a.off[g], o1 = a.off[g + 1];
  if (o0 == o1) return kAbsent;
  const uint2 bd = *reinterpret_cast<const uint2 *>(a.dir2 + ((size_t)(g / 3 * a.nbw + (s >> 5)) * 3 + g % 3) * 2);
  const uint32_t bm = bd.x, bit = (uint32_t)s & 31u;
  if (!((bm >> bit) & 1u)) return kAbsent;
  *gw_out = a.srv + o0;
  return a.poff[bd.y + __popc(bm & ((1u << bit) - 1u))];
}

// Threads of a render-tile workgroup: 8 waves, so that a tile's footprint
// decode (a chain of dependent reads per level) and its interpolation run
// in half the passes of a 4-wave workgroup at the same LDS per tile.
constexpr int kRenderThreads = 512;

// One workgroup per (view, output tile).  The tile's source footprint in the
// four nearest views is reconstructed in LDS, a lane summing one channel of one
// block of one view in registers (gather_block); 8 x 8 blocks first by their
// key-view rows, then, level by level, every distinct stored residual block is
// decoded by one lane and added for each of the four views whose path passes
// through its node.  The sums are converted to RGB (inverse YCoCg-R, clamped) in
// place, then every output pixel interpolates its 16 taps in FP32.  A tile is
// bound by its chains of reads: one chain per pass of the workgroup over the
// footprint, where the key rows took ten passes and every level three more, took
// a 512 x 512 view from 22.4 to 16.9 us (13.7 with best_plan's tile).

// Inverse YCoCg-R (Sec. 4) of two pixels in packed 16-bit samples, clamped to
// 8 bits and packed R | G << 8 | B << 16 each.  With h = cg >> 1 and k = co >> 1:
//   G = y + (cg - h),  B = y - (h + k),  R = y - (h - (co - k)),
// where every bracket fits 16 bits for all samples, so that each channel is one
// saturating operation, whose clamp to 8 bits is that of the exact value
// (tests/test_colour_packed.py).  Six operations a pixel against fourteen in 32
// bits.
__device__ __forceinline__ uint32_t sat_bytes(i16x2 v) {   // both halves to 8 bits, in the two low bytes
  uint32_t r;
  asm("v_sat_pk_u8_i16 %0, %1" : "=v"(r) : "v"(v));
  return r;
}
__device__ __forceinline__ void rgb_pack2(uint32_t yw, uint32_t cow, uint32_t cgw, uint32_t &p0, uint32_t &p1) {
  const i16x2 y = __builtin_bit_cast(i16x2, yw), co = __builtin_bit_cast(i16x2, cow), cg = __builtin_bit_cast(i16x2, cgw);
  const i16x2 h = cg >> 1, k = co >> 1;
  const uint32_t g = sat_bytes(__builtin_elementwise_add_sat(y, (i16x2)(cg - h)));
  const uint32_t b = sat_bytes(__builtin_elementwise_sub_sat(y, (i16x2)(h + k)));
  const uint32_t r = sat_bytes(__builtin_elementwise_sub_sat(y, (i16x2)(h - (co - k))));
  const uint32_t rg = __builtin_amdgcn_perm(g, r, 0x05010400u);   // R0 G0 R1 G1
  p0 = __builtin_amdgcn_perm(b, rg, 0x0c040100u);
  p1 = __builtin_amdgcn_perm(b, rg, 0x0c050302u);
}

// Source views of an output pixel: k = 0: (u0, v0), 1: (u1, v0), 2: (u0, v1),
// 3: (u1, v1); its taps in each are (y0,x0), (y0,x1), (y1,x0), (y1,x1).
// Camera-plane position (clamped to the grid) and the image-plane shift of
// source view k (0: lower column/row, 1: upper) for focal disparity d: a
// novel camera focused at disparity d samples source camera (iu, jv) at
// (s + d (iu - u), t + d (jv - v)).
// FOCAL false compiles the plain render, where every source view shares one
// footprint and one set of fractions.
template <bool FOCAL>
__device__ __forceinline__ float focal_shift(float d, float x, int n, int i) {
#pragma clang fp contract(off)
  if constexpr (!FOCAL) return 0.0f;
  return d * ((float)i - fminf(fmaxf(x, 0.0f), (float)(n - 1)));
}

// Source-image position of output pixel X: each operation rounded on its
// own (no fused multiply-add), so every renderer samples the same positions.
__device__ __forceinline__ float src_pos(float s, int X, float scale) {
#pragma clang fp contract(off)
  return s + ((float)X + 0.5f) * scale - 0.5f;
}

// The interpolation works on taps scaled by 2^-24 (exact throughout: a power
// of two): a byte in the low half of a 16-bit lane is the fp16 number byte x
// 2^-24, so a byte permute makes two taps into packed fp16, their differences
// are exact there, and a mixed-precision fma lerps them in fp32.  Five
// operations for two taps pairs against eight with conversions.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x2 tap_pair(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(hi, lo, sel));
}

// lerp along s of the tap pairs (a[k], b[k]) of the four source views, at that
// view's fraction fs[k % NS]: h[view][channel]
template <int NS>
__device__ __forceinline__ void slerp_taps(const uint32_t (&a)[4], const uint32_t (&b)[4], const float (&fs)[NS],
                                           float (&h)[4][3]) {
#pragma unroll
  for (int k = 0; k < 4; k++) {   // red and green
    const f16x2 p = tap_pair(a[k], a[k], 0x0c010c00u), d = tap_pair(b[k], b[k], 0x0c010c00u) - p;
    h[k][0] = __builtin_fmaf((float)d.x, fs[k % NS], (float)p.x);
    h[k][1] = __builtin_fmaf((float)d.y, fs[k % NS], (float)p.y);
  }
#pragma unroll
  for (int k = 0; k < 4; k += 2) {   // blue, of two views
    const f16x2 p = tap_pair(a[k + 1], a[k], 0x0c060c02u), d = tap_pair(b[k + 1], b[k], 0x0c060c02u) - p;
    h[k][2] = __builtin_fmaf((float)d.x, fs[k % NS], (float)p.x);
    h[k + 1][2] = __builtin_fmaf((float)d.y, fs[(k + 1) % NS], (float)p.y);
  }
}

// lerp along v, then u, of the four views' values
__device__ __forceinline__ void blend_views(const float (&h)[4][3], float fu, float fv, float (&r)[3]) {
#pragma unroll
  for (int ch = 0; ch < 3; ch++) r[ch] = lerpf(lerpf(h[0][ch], h[2][ch], fv), lerpf(h[1][ch], h[3][ch], fv), fu);
}

// x / 255 for 0 <= x <= 255 given x 2^-24, rounded as the IEEE quotient: the
// product with the rounded reciprocal, corrected by one fused residual step
// (equal to the division for every float of the range, checked on the host by
// tests/arith_identities.c, where the powers of two are left out; negative
// inputs mirror it); three VALU operations instead of a full division.
__device__ __forceinline__ float div255(float x) {
  constexpr float r = 1.0f / 255.0f * 16777216.0f, k = 255.0f / 16777216.0f;
  const float q = x * r;
  return __builtin_fmaf(__builtin_fmaf(-q, k, x), r, q);
}

// quadrilinear interpolation of the 16 RGB taps P[view][tap] (taps 00, 01,
// 10, 11 of each view, at that view's fractions fs[k], ft[k]).  The lerps go
// along s, v, u and t: the first three depend on the source row only, so
// consecutive output rows can share them; with a focal shift, where the views
// have fractions of their own, along s, t, v and u.
template <bool FOCAL>
__device__ __forceinline__ void interp_store(const uint32_t P[4][4], const float fs[4], const float ft[4], float fu,
                                             float fv, float *o, size_t plane) {
  const float f[4] = {fs[0], fs[1], fs[2], fs[3]};
  const uint32_t t0[4] = {P[0][0], P[1][0], P[2][0], P[3][0]}, t1[4] = {P[0][1], P[1][1], P[2][1], P[3][1]};
  const uint32_t b0[4] = {P[0][2], P[1][2], P[2][2], P[3][2]}, b1[4] = {P[0][3], P[1][3], P[2][3], P[3][3]};
  float top[4][3], bot[4][3], r[2][3];
  slerp_taps<4>(t0, t1, f, top);
  slerp_taps<4>(b0, b1, f, bot);
  if constexpr (FOCAL) {
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
      for (int ch = 0; ch < 3; ch++) top[k][ch] = lerpf(top[k][ch], bot[k][ch], ft[k]);
    blend_views(top, fu, fv, r[0]);
#pragma unroll
    for (int ch = 0; ch < 3; ch++) o[ch * plane] = div255(r[0][ch]);
  } else {
    blend_views(top, fu, fv, r[0]);
    blend_views(bot, fu, fv, r[1]);
#pragma unroll
    for (int ch = 0; ch < 3; ch++) o[ch * plane] = div255(lerpf(r[0][ch], r[1][ch], ft[0]));
  }
}

// One output tile (tile column tbx, tile row tby) of view vw into outn
// ([3][ho][wo] floats); smem holds the LUT and the footprint accumulators.
template <int B, bool FOCAL>
__device__ __forceinline__ void render_tile(const RenderArgs &a, const lfc_view vw, float *outn, int tbx, int tby,
                                            uint32_t *smem) {
  constexpr int S = B * B, SLOT = 3 * S / 2;   // words per (view, block): 3 channels of packed int16
  const uint16_t *lut = reinterpret_cast<const uint16_t *>(smem);
  uint32_t *acc = smem + kLutEntries / 2;       // [4][fbx_max*fby_max][SLOT]
  const int tid = threadIdx.x;
  if (tid < kLutEntries / 2) smem[tid] = kLutTable.w[tid];
  int iu0, iu1, jv0, jv1;
  float fu, fv;
  cell(vw.u, a.U, iu0, iu1, fu);
  cell(vw.v, a.V, jv0, jv1, fv);
  const float sxs = (float)a.W / (float)a.wo, tys = (float)a.H / (float)a.ho;
  const int tx0 = tbx * a.TX, ty0 = tby * a.TY;
  const int tx1 = min(tx0 + a.TX, a.wo) - 1, ty1 = min(ty0 + a.TY, a.ho) - 1;
  int vis[4];
  vis[0] = jv0 * a.U + iu0;
  vis[1] = jv0 * a.U + iu1;
  vis[2] = jv1 * a.U + iu0;
  vis[3] = jv1 * a.U + iu1;
  // per source view: image-plane shift (focal disparity) and the tile's
  // source footprint, one pixel wider on each side than needed
  float shx[4], shy[4];
  int fbx0[4], fby0[4], FBX[4], FBY[4], FB[4];
  int FBmax = 0;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    shx[k] = focal_shift<FOCAL>(a.disp, vw.u, a.U, (k & 1) ? iu1 : iu0);
    shy[k] = focal_shift<FOCAL>(a.disp, vw.v, a.V, (k & 2) ? jv1 : jv0);
    const float sa = fminf(fmaxf(src_pos(vw.s, tx0, sxs) + shx[k], 0.0f), (float)(a.W - 1));
    const float sb = fminf(fmaxf(src_pos(vw.s, tx1, sxs) + shx[k], 0.0f), (float)(a.W - 1));
    const float ta = fminf(fmaxf(src_pos(vw.t, ty0, tys) + shy[k], 0.0f), (float)(a.H - 1));
    const float tb = fminf(fmaxf(src_pos(vw.t, ty1, tys) + shy[k], 0.0f), (float)(a.H - 1));
    const int xlo = max((int)floorf(sa) - 1, 0), xhi = min((int)floorf(sb) + 2, a.W - 1);
    const int ylo = max((int)floorf(ta) - 1, 0), yhi = min((int)floorf(tb) + 2, a.H - 1);
    fbx0[k] = xlo / B;
    fby0[k] = ylo / B;
    FBX[k] = min(xhi / B - fbx0[k] + 1, a.fbx_max);
    FBY[k] = min(yhi / B - fby0[k] + 1, a.fby_max);
    FB[k] = FBX[k] * FBY[k];
    FBmax = max(FBmax, FB[k]);
  }
  const int FBM = a.fbx_max * a.fby_max;
  const int depth = a.ra.L - 1;
  __syncthreads();

  // a quotient by FBmax and by the footprint's width, for numerators below 2^16
  const uint32_t div_fb = 0xFFFFFFFFu / (uint32_t)FBmax + 1u;
  if constexpr (B <= 4) {
    // (1, 2) item = (view k, block, channel): the lane sums the block's key view
    // and residuals in registers
    uint32_t div_x[FOCAL ? 4 : 1];
#pragma unroll
    for (int k = 0; k < (FOCAL ? 4 : 1); k++) div_x[k] = 0xFFFFFFFFu / (uint32_t)FBX[k] + 1u;
    for (int it = tid; it < 4 * FBmax * 3; it += kRenderThreads) {
      const int c = it % 3, r1 = it / 3, k = FBmax == 1 ? r1 : (int)__umulhi((uint32_t)r1, div_fb), bb = r1 - k * FBmax;
      const int kf = FOCAL ? k : 0;
      if (bb >= FB[kf]) continue;
      const int by = FBX[kf] == 1 ? bb : (int)__umulhi((uint32_t)bb, div_x[kf]);
      const int b = (fby0[kf] + by) * a.ra.nbx + fbx0[kf] + bb - by * FBX[kf];
      uint32_t x[S / 2];
      gather_block<B>(a.ra, vis[k], b, c, 0, lut, x);
      uint32_t *slot = acc + (k * FBM + bb) * SLOT + c * (S / 2);
      if constexpr (B == 4) {
        *reinterpret_cast<uint4 *>(slot) = make_uint4(x[0], x[1], x[2], x[3]);
        *reinterpret_cast<uint4 *>(slot + 4) = make_uint4(x[4], x[5], x[6], x[7]);
      } else {
        *reinterpret_cast<uint2 *>(slot) = make_uint2(x[0], x[1]);
      }
    }
    __syncthreads();
  } else {
    // (1) key-view rows: item = (view k, block, channel, row)
    for (int it = tid; it < 4 * FBmax * 3 * B; it += kRenderThreads) {
      const int y = it % B, r1 = it / B, c = r1 % 3, r2 = r1 / 3, bb = r2 % FBmax, k = r2 / FBmax;
      if (bb >= FB[k]) continue;
      const int b = (fby0[k] + bb / FBX[k]) * a.ra.nbx + fbx0[k] + bb % FBX[k];
      uint32_t x[B / 2];
      load_row<B>(a.ra.rkv + ((size_t)(a.ra.root[vis[k]] * a.ra.nb + b) * 3 + c) * S + y * B, x);
#pragma unroll
      for (int h = 0; h < B / 2; h++) acc[(k * FBM + bb) * SLOT + c * (S / 2) + y * (B / 2) + h] = x[h];
    }
    __syncthreads();

    // (2) residual levels, one at a time (each (view, block, channel) slot gets
    // one block per level, so the adds never race)
    for (int l = depth - 1; l >= 0; --l) {
      int node[4], owner[4];
#pragma unroll
      for (int k = 0; k < 4; k++) node[k] = a.ra.path[vis[k] * depth + l];
#pragma unroll
      for (int k = 0; k < 4; k++) {
        // views with one ancestor share its decoded blocks when their
        // footprints coincide (no focal shift)
        owner[k] = k;
        if (!FOCAL)
          for (int k2 = k - 1; k2 >= 0; --k2)
            if (node[k2] == node[k]) owner[k] = k2;
      }
      for (int it = tid; it < 4 * FBmax * 3; it += kRenderThreads) {
        const int c = it % 3, r1 = it / 3, bb = r1 % FBmax, k = r1 / FBmax;
        if (owner[k] != k || bb >= FB[k]) continue;
        const int b = (fby0[k] + bb / FBX[k]) * a.ra.nbx + fbx0[k] + bb % FBX[k];
        const uint32_t *gw = nullptr;
        const uint32_t e = locate(a.ra, 3 * b + c, node[k], &gw);
        if (e == kAbsent) continue;
        uint32_t d[S / 2];
        decode_block(gw, e, a.ra.q, lut, d);
#pragma unroll
        for (int k2 = 0; k2 < 4; k2++) {
          if (owner[k2] != k) continue;
          uint32_t *slot = acc + (k2 * FBM + bb) * SLOT + c * (S / 2);
#pragma unroll
          for (int h = 0; h < S / 2; h++) slot[h] = add_pk(slot[h], d[h]);
        }
      }
      __syncthreads();
    }

  }

  // (3) YCoCg-R -> RGB in place: item = (view, block)
  for (int it = tid; it < 4 * FBmax; it += kRenderThreads) {
    const int k = it / FBmax, bb = it % FBmax;
    if (bb >= FB[k]) continue;
    uint32_t *slot = acc + (k * FBM + bb) * SLOT;
    uint32_t v[SLOT];
#pragma unroll
    for (int w = 0; w < SLOT; w++) v[w] = slot[w];
#pragma unroll
    for (int i = 0; i < S / 2; i++) {
      uint32_t p0, p1;
      rgb_pack2(v[i], v[S / 2 + i], v[S + i], p0, p1);
      slot[2 * i] = p0;
      slot[2 * i + 1] = p1;
    }
  }
  __syncthreads();

  // (4) quadrilinear interpolation of every output pixel of the tile
  const size_t plane = (size_t)a.ho * a.wo;
  for (int p = tid; p < a.TX * a.TY; p += kRenderThreads) {
    const int X = tx0 + p % a.TX, Yp = ty0 + p / a.TX;
    if (X >= a.wo || Yp >= a.ho) continue;
    const float sx = src_pos(vw.s, X, sxs), ty = src_pos(vw.t, Yp, tys);
    uint32_t P[4][4];
    float fs[4], ft[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
      int x0, x1, y0, y1;
      cell(sx + shx[k], a.W, x0, x1, fs[k]);
      cell(ty + shy[k], a.H, y0, y1, ft[k]);
      const int FW = FBX[k] * B, FH = FBY[k] * B;
      const int lx0 = min(max(x0 - fbx0[k] * B, 0), FW - 1), lx1 = min(max(x1 - fbx0[k] * B, 0), FW - 1);
      const int ly0 = min(max(y0 - fby0[k] * B, 0), FH - 1), ly1 = min(max(y1 - fby0[k] * B, 0), FH - 1);
      // word of footprint pixel (lx, ly) within the view's part of the tile
      const uint32_t *img = acc + k * FBM * SLOT;
      P[k][0] = img[((ly0 / B) * FBX[k] + lx0 / B) * SLOT + (ly0 % B) * B + lx0 % B];
      P[k][1] = img[((ly0 / B) * FBX[k] + lx1 / B) * SLOT + (ly0 % B) * B + lx1 % B];
      P[k][2] = img[((ly1 / B) * FBX[k] + lx0 / B) * SLOT + (ly1 % B) * B + lx0 % B];
      P[k][3] = img[((ly1 / B) * FBX[k] + lx1 / B) * SLOT + (ly1 % B) * B + lx1 % B];
    }
    interp_store<FOCAL>(P, fs, ft, fu, fv, outn + (size_t)Yp * a.wo + X, plane);
  }
}

template <int B, bool FOCAL>
__global__ __launch_bounds__(kRenderThreads) void k_render(RenderArgs a) {
  extern __shared__ uint32_t smem[];
  const int n = blockIdx.z;
  render_tile<B, FOCAL>(a, a.views[n], a.out + (size_t)n * 3 * a.ho * a.wo, blockIdx.x, blockIdx.y, smem);
}

// Many render requests in one launch, possibly of different light fields and
// output sizes: workgroup (x, r) renders tile x of request r, and exits when
// the request has fewer tiles.
struct RenderReq {
  RenderArgs a;        // the request's light field, output size, tiling and output (views unused)
  lfc_view view;
  int ntx, ntiles;     // tile columns, tiles
};

template <int B>
__global__ __launch_bounds__(kRenderThreads) void k_render_multi(const RenderReq *reqs) {
  extern __shared__ uint32_t smem[];
  // one read of the record, at the start: every wave then works from the
  // same copy, however late it uses a field
  const RenderReq r = reqs[blockIdx.y];
  const int t = blockIdx.x;
  if (t >= r.ntiles) return;
  render_tile<B, false>(r.a, r.view, r.a.out, t % r.ntx, t / r.ntx, smem);
}

// ---------------------------------------------------------------------------
// whole light field as 8-bit RGB (the decode-then-interpolate render's input)
// ---------------------------------------------------------------------------

// LDS words before the tile: LUT; the start words of the strip's 3 x 64/B
// groups; a flag and a bit per node of the chunk for the views a render
// reads; then, sized for the light field, the view mask, a chunk's gather table
// (masks and first slots, run node positions), its runs' views and roots, and
// the list of the pairs that are wanted.
using lfc::kRGBNodeCap;
constexpr int kRGBNeedWords = 128;        // views a render may mask: at most 32 x 128
constexpr int kRGBFixedWords = 192 + 96 + 4 + kRGBNodeCap / 32;
__host__ __device__ constexpr int rgb_head_words(int need_words, int tab_cap, int run_cap) {
  return (kRGBFixedWords + need_words + tab_cap + (kRunWords + 2) * run_cap + 3) & ~3;
}
struct RGBArgs {
  const int16_t *rkv;
  const uint32_t *off;
  const uint32_t *srv;
  const uint32_t *sched;      // colour decode schedule: one record per strip (build_schedule_rgb on the host)
  const uint32_t *order;      // [n_strips][2] strip and first word of its record, costliest first
  const int32_t *batch;       // [nbatch][kBatchWords] runs of sibling leaves
  const uint32_t *vneed;      // [ceil(nv/32)] bit per view to write (nv <= 32 kRGBNeedWords), or null: every view
  uint32_t *out;              // [nv][hp][wp] pixels R | G << 8 | B << 16
  int nbx, nsx, L, q, wp, hp, nb, nbatch, nv;
  int n_top, key_roots;       // key views; those whose rows (all channels) the LDS holds: all, else a chunk's
  int tile_cap;
  int parts;                  // workgroups per strip: part p takes the chunks ci with ci % parts == p
  int need_words, tab_cap, run_cap;   // sizes of the LDS tables: view mask, gather table, runs
  // with vneed null: the cameras of a render, whose four grid neighbours
  // each workgroup marks itself (null: every view, unless vneed is given)
  const lfc_view *views = nullptr;
  int nviews = 0, U = 0, V = 0;
};

// One workgroup = one strip of 64/B blocks of one block row, all three
// channels, or every parts-th chunk of it (a strip of three channels holds
// three times the blocks of a one-channel strip, so strips alone would not
// fill the chip).  Phase A copies the LUT, the strip's group starts, the view
// mask and the key-view rows to LDS.  Per chunk of the strip's runs: its node
// masks, first slots, run positions and views are copied to LDS while (3) every
// stored residual block of the chunk, of any channel (with a view mask: of a
// node that a wanted view reads), is decoded once into the compact tile; then
// (4) four (run, sibling) pairs per wave: a lane owns 4 pixels of the strip's
// rows, sums key row + ancestor rows + leaf row of each channel, converts the
// pixels to RGB (inverse YCoCg-R, clamped) and stores 16 bytes per row.
// What bounds it is the issue of vector instructions and, per chunk, the chain
// header - entry - window - decode - barrier - gather; hence the packed colour
// conversion, a gather without branches on the path's length (one body for each
// depth of the tree), tables and key views that the gather reads from LDS alone,
// the next chunk's header and first entries read before this chunk's stores
// (loads wait for older stores), 16-byte planes of the tile against bank
// conflicts, and at most 80 registers and 53 KB, which let three workgroups share
// a compute unit (two at 8 x 8).  81 views of 625 x 434: 66 -> 43 us (12 against
// 26 million vector instructions), 2.5 TB/s of output and payload; the views that
// 64 cameras read of 17 x 17 of 512 x 512: 132 -> 90 us; 8 x 8 blocks, 80 views
// of 317 x 521: 92 -> 49 us.
template <int B>
__device__ __forceinline__ void rgb_strip(const RGBArgs &a, int wg, uint32_t *smem) {
  constexpr int S = B * B, NBLK = 64 / B, HR = B;   // HR rows per lane
  const uint16_t *lut = reinterpret_cast<const uint16_t *>(smem);   // 384 x u16 = 192 words
  uint32_t *s_o0 = smem + 192;                          // [3][NBLK] group start words
  uint32_t *s_nlist = smem + 288;                       // [0] listed pairs of the chunk
  uint32_t *s_node = s_nlist + 4;                       // wanted nodes of the chunk, a bit each
  uint32_t *s_need = smem + kRGBFixedWords;             // the view mask
  uint32_t *s_mf = s_need + a.need_words;               // masks and first slots [3][nn], run node positions[nq][3]
  int32_t *s_rec = reinterpret_cast<int32_t *>(s_mf + a.tab_cap);   // [nq][kRunWords]
  uint16_t *s_list = reinterpret_cast<uint16_t *>(s_rec + kRunWords * a.run_cap);
                                                        // (run << 2 | sibling) pairs of the chunk
  uint32_t *tile = smem + rgb_head_words(a.need_words, a.tab_cap, a.run_cap);   // residual tile
  uint32_t *keys = tile + lf_tile_words(a.tile_cap, S); // [n_top][NBLK][3][S/2], blocks as in the tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the workgroup's strip and part, and its first chunk's header (scalar loads)
  const uniform_i32 ent = as_uniform(reinterpret_cast<const int32_t *>(a.order) + 2 * (wg / a.parts));
  const int st = ent[0], part = wg % a.parts;
  const uint32_t *gs = a.sched + (uint32_t)ent[1];
  const uniform_i32 head = as_uniform(reinterpret_cast<const int32_t *>(gs));
  const int nck = head[0];
  int h_at = 0, q0 = 0, nq = 0, nr = 0, nn = 0, r0 = 0;
  uint32_t n0 = 0, n01 = 0, n = 0;
  auto header = [&](int ci) {
    const uniform_i32 h = head + 8 + 8 * ci;
    h_at = h[0], q0 = h[1], nq = h[2] & 0xFFFF, nr = h[2] >> 16, nn = h[3], r0 = h[7];
    n0 = (uint32_t)h[4], n01 = (uint32_t)h[5], n = (uint32_t)h[6];
  };
  // a chunk's entries and items follow its masks, first slots and run positions
  auto tables = [&](const uint32_t *&chunk, int &mf_words, const uint32_t *&ents, const uint32_t *&items) {
    chunk = gs + h_at;
    mf_words = B == 2 ? 3 * nn + (3 * nn + 1) / 2 : 3 * nn;
    ents = chunk + mf_words + 3 * nq;
    items = ents + n;
  };
  uint32_t e_nx = 0, t_nx = 0;   // the lane's next entry, requested ahead
  auto request_first = [&] {
    const uint32_t *chunk, *ents, *items;
    int mf_words;
    tables(chunk, mf_words, ents, items);
    if ((uint32_t)tid < n) {
      e_nx = ents[tid];
      t_nx = items[tid];
    }
  };
  if (part < nck) {
    header(part);
    request_first();
  }
  const int sx = st % a.nsx, by = st / a.nsx;
  const bool masked = a.vneed != nullptr || a.views != nullptr;
  if (tid < kLutEntries / 2) __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void *)(kLutTable.w + tid),
      (__attribute__((address_space(3))) void *)(smem + (tid & ~63)), 4, 0, 0);
  // 16-byte quad k of tile slot s (B = 2: a slot is 8 bytes) at k * plane + 4 s;
  // the last slot is zero
  const int plane = 4 * (a.tile_cap + 1);
  if (tid < S / 2) tile[B == 2 ? a.tile_cap * 2 + tid : (tid / 4) * plane + a.tile_cap * 4 + tid % 4] = 0u;
  if (tid < 64)
    for (int k = lane; k < 3 * NBLK; k += 64) {
      const int c = k / NBLK, bx = sx * NBLK + k % NBLK;
      s_o0[k] = bx < a.nbx ? a.off[3 * (by * a.nbx + bx) + c] : 0u;
    }
  if (a.vneed) {
    for (int w = tid; w < (a.nv + 31) / 32; w += kLFThreads) s_need[w] = a.vneed[w];
  } else if (a.views) {
    // the source views the cameras read: each camera's four grid neighbours
    for (int w = tid; w < (a.nv + 31) / 32; w += kLFThreads) s_need[w] = 0u;
    lds_barrier();
    for (int i = tid; i < a.nviews; i += kLFThreads) {
      int iu0, iu1, jv0, jv1;
      float fu, fv;
      cell(a.views[i].u, a.U, iu0, iu1, fu);
      cell(a.views[i].v, a.V, jv0, jv1, fv);
      const int vs[4] = {jv0 * a.U + iu0, jv0 * a.U + iu1, jv1 * a.U + iu0, jv1 * a.U + iu1};
#pragma unroll
      for (int k = 0; k < 4; k++) atomicOr(&s_need[vs[k] >> 5], 1u << (vs[k] & 31));
    }
  }
  // key views r0 .. r0 + nr - 1: a key view's blocks of the strip, of all channels, lie together
  auto stage_keys = [&](int r0, int nr) {
    constexpr int KW = 3 * NBLK * (S / 2);
    const uint32_t *rk = reinterpret_cast<const uint32_t *>(a.rkv) +
                         ((size_t)r0 * a.nb + by * a.nbx + sx * NBLK) * (3 * S / 2);
    const int valid = min(NBLK, a.nbx - sx * NBLK) * (3 * S / 2);
    for (int f = wave; f < nr * (KW / 64); f += kLFWaves) {
      const int r = f / (KW / 64), w0 = f % (KW / 64) * 64;
      if (w0 + lane < valid)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)(rk + (size_t)r * a.nb * (3 * S / 2) + w0 + lane),
            (__attribute__((address_space(3))) void *)(keys + f * lfc::rgb_key_step(B)), 4, 0, 0);
    }
  };
  const bool all_keys = a.n_top <= a.key_roots;
  if (all_keys) stage_keys(0, a.n_top);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // gather lane mapping: listed pair lane / 16, 4-pixel segment jseg (word pairs pp = 2 jseg,
  // 2 jseg + 1 of the strip's 32-word rows); the block and the word inside its row of each pair
  const int jseg = lane & 15;
  int jb[2], wib[2];
#pragma unroll
  for (int w = 0; w < 2; w++) {
    const int pp = 2 * jseg + w;
    jb[w] = (2 * pp) / B;
    wib[w] = ((2 * pp) % B) / 2;
  }
  const int px0 = sx * 64 + 4 * jseg;                   // first pixel of the segment
  const bool seg_in = sx * NBLK + jb[0] < a.nbx;        // the segment's first block is inside the image
  const uint32_t zslot = (uint32_t)a.tile_cap;
  const uint32_t vplane = (uint32_t)a.hp * (uint32_t)a.wp;
  auto wanted_view = [&](int vi) { return !masked || ((s_need[vi >> 5] >> (vi & 31)) & 1u); };
  for (int ci = part; ci < nck; ci += a.parts) {
    const uint32_t *chunk, *ents, *items;
    int mf_words;
    tables(chunk, mf_words, ents, items);
    const uniform_i32 runs = as_uniform(reinterpret_cast<const int32_t *>(chunk)) + mf_words;
    // with a view mask, the chunk's (run, sibling) pairs of wanted views are
    // listed in LDS and the nodes they read are marked (a chunk with none is
    // skipped whole); without one, pair e is sibling e % 4 of run e / 4
    int n_list = 4 * nq;
    if (masked) {
      for (int w = tid; w < kRGBNodeCap / 32; w += kLFThreads) s_node[w] = 0u;
      if (tid == 0) *s_nlist = 0u;
      // (barriers on LDS only: a full barrier would also wait for the stores
      // of the previous chunk's gather)
      lds_barrier();
      for (int qi = wave; qi < nq; qi += kLFWaves) {
        const uniform_i32 rec = as_uniform(a.batch + (size_t)(q0 + qi) * lfc::kBatchWords);
        const int nsib = rec[0];
        bool wanted[4];
#pragma unroll
        for (int k = 0; k < 4; k++) wanted[k] = k < nsib && wanted_view(max(rec[1 + k], 0));
        if (!(wanted[0] || wanted[1] || wanted[2] || wanted[3])) continue;
        const bool mine = lane == 0 ? wanted[0] : (lane == 1 ? wanted[1] : (lane == 2 ? wanted[2] : wanted[3]));
        if (lane < 4 && mine) s_list[atomicAdd(s_nlist, 1u)] = (uint16_t)(qi << 2 | lane);
        const uint32_t w0 = (uint32_t)runs[3 * qi], w1 = (uint32_t)runs[3 * qi + 1], w2 = (uint32_t)runs[3 * qi + 2];
        const int anc_ln[4] = {(int)(w0 >> 16), (int)(w1 & 0xFFFFu), (int)(w1 >> 16), (int)(w2 & 0xFFFFu)};
        int ln = -1;
        if (lane < 4 && a.L > 1 && mine)
          ln = (int)(w0 & 0xFFFFu) + lane;
        else if (lane >= 4 && lane < 8 && lane - 4 < a.L - 2)
          ln = lane == 4 ? anc_ln[0] : (lane == 5 ? anc_ln[1] : (lane == 6 ? anc_ln[2] : anc_ln[3]));
        if (ln >= 0) atomicOr(&s_node[ln >> 5], 1u << (ln & 31));
      }
      lds_barrier();
      n_list = __builtin_amdgcn_readfirstlane((int)*s_nlist);
      if (n_list == 0) {
        lds_barrier();   // every wave has read the count before the next chunk clears it
        if (ci + a.parts < nck) {
          header(ci + a.parts);
          request_first();
        }
        continue;
      }
    }
    // the chunk's node masks, first slots, run positions, views and roots into
    // LDS, in flight during the decode (the gather then reads no global memory)
    const int tab_words = mf_words + 3 * nq;
    for (int w0 = wave * 64; w0 < tab_words; w0 += kLFThreads)
      if (w0 + lane < tab_words)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(chunk + w0 + lane),
                                         (__attribute__((address_space(3))) void *)(s_mf + w0), 4, 0, 0);
    const uint32_t *recs = reinterpret_cast<const uint32_t *>(a.batch + (size_t)a.nbatch * lfc::kBatchWords) + (size_t)q0 * kRunWords;
    for (int w0 = wave * 64; w0 < kRunWords * nq; w0 += kLFThreads)
      if (w0 + lane < kRunWords * nq)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(recs + w0 + lane),
                                         (__attribute__((address_space(3))) void *)(s_rec + w0), 4, 0, 0);
    if (!all_keys) stage_keys(r0, nr);
    // (3) decode every stored block of the chunk (that a wanted view reads) into its tile slot
    for (uint32_t it = tid; it < n; it += kLFThreads) {
      const uint32_t e = e_nx, t = t_nx;
      const uint32_t base = s_o0[((t >> 6) & 3u) * NBLK + (t & 63u)];
      Window<B> w;
      fetch_window<B>(a.srv + (base + (e >> 10)), w);
      if (it + kLFThreads < n) {
        e_nx = ents[it + kLFThreads];
        t_nx = items[it + kLFThreads];
      }
      if (masked) {
        const uint32_t ln = (t >> 8) & 4095u;
        if (!((s_node[ln >> 5] >> (ln & 31u)) & 1u)) continue;
      }
      uint32_t d[S / 2];
      if (it < n0) decode_fetched<B, 0>(w, a.srv, base, e, a.q, lut, d);
      else if (it < n01) decode_fetched<B, 1>(w, a.srv, base, e, a.q, lut, d);
      else decode_fetched<B, 2>(w, a.srv, base, e, a.q, lut, d);
      uint32_t *dst = tile + (t >> 20) * (B == 2 ? 2 : 4);
      if constexpr (B == 2) {
        *reinterpret_cast<uint2 *>(dst) = make_uint2(d[0], d[1]);
      } else {
#pragma unroll
        for (int q = 0; q < S / 8; q++)
          *reinterpret_cast<uint4 *>(dst + q * plane) = make_uint4(d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]);
      }
    }
    // the next chunk's header and first entries, taken before this chunk's stores
    const int nn_c = nn, nn3 = 3 * nn, root0 = all_keys ? 0 : r0;
    if (ci + a.parts < nck) {
      header(ci + a.parts);
      request_first();
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's copies of the node table have landed
    lds_barrier();
    const uint16_t *firsts = reinterpret_cast<const uint16_t *>(s_mf + nn3);   // (B = 2)
    const uint32_t *s_runs = s_mf + mf_words;
    // (4) four listed (run, sibling) pairs per wave at a time, one per 16-lane
    // group.  Everything comes from LDS and without branches, in three steps
    // whose reads are in flight together: the pair's run; the masks and first
    // slots of its path's nodes (nodes_c of them; -1: found at run time) for
    // all channels; per channel the key row and the nodes' rows.
    auto gather = [&](auto nodes_c) {
      constexpr int NC = decltype(nodes_c)::value, NM = NC < 0 ? lfc::kMaxLevels - 1 : NC;
      const int nodes = NC < 0 ? a.L - 1 : NC;
      constexpr int NS = B == 2 ? 2 : 1;   // blocks of a lane's four pixels of a row
      for (int e0 = wave * 4; e0 < n_list; e0 += 4 * kLFWaves) {
        const int e = min(e0 + (lane >> 4), n_list - 1);
        const uint32_t en = masked ? s_list[e] : (uint32_t)e;
        const int qi = (int)(en >> 2), so = (int)(en & 3u);
        const int vi = s_rec[kRunWords * qi + so], root = s_rec[kRunWords * qi + 4] - root0;
        const bool live = seg_in && e0 + (lane >> 4) < n_list && vi >= 0;
        // the path's nodes: the lane's own leaf, then its ancestors
        int node[NM > 0 ? NM : 1] = {};
        if constexpr (NM > 0) {
          const uint32_t w0 = s_runs[3 * qi];
          node[0] = min((int)(w0 & 0xFFFFu) + so, max(nn_c - 1, 0));
          if constexpr (NM > 1) node[1] = (int)(w0 >> 16);
          if constexpr (NM > 2) {
            const uint32_t w1 = s_runs[3 * qi + 1], w2 = s_runs[3 * qi + 2];
            node[2] = (int)(w1 & 0xFFFFu);
            node[3] = (int)(w1 >> 16);
            node[4] = (int)(w2 & 0xFFFFu);
          }
        }
        // tile slots of the lane's blocks; an absent block's is the zeroed one
        uint32_t slot[3][NM > 0 ? NM : 1][NS];
#pragma unroll
        for (int c = 0; c < 3; c++)
#pragma unroll
          for (int k = 0; k < NM; k++) {
            if (NC < 0 && k >= nodes) continue;
            const uint32_t w = s_mf[c * nn_c + node[k]];
            const uint32_t first = B == 2 ? firsts[c * nn_c + node[k]] : w >> 16;
#pragma unroll
            for (int b = 0; b < NS; b++) {
              const uint32_t sl = first + (uint32_t)__popc(w & ((1u << jb[b]) - 1u));
              slot[c][k][b] = ((w >> jb[b]) & 1u ? sl : zslot) * (B == 2 ? 2 : 4);
            }
          }
        uint32_t x[3][HR][2];
        // the lane's words of a block, at the given distance of its 16-byte quads:
        // B = 4, the whole 4 x 4 block in two 16-byte reads; B = 2, both rows
        // of each of its two blocks in one 8-byte read; B = 8, half of each row
        auto read_slot = [&](const uint32_t *slot0, const uint32_t *slot1, int quads, bool add, uint32_t (&xc)[HR][2]) {
          if constexpr (B == 4) {
            const uint4 v0 = *reinterpret_cast<const uint4 *>(slot0), v1 = *reinterpret_cast<const uint4 *>(slot0 + quads);
            const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
            for (int y = 0; y < 4; y++)
#pragma unroll
              for (int k = 0; k < 2; k++) xc[y][k] = add ? add_pk(xc[y][k], w[2 * y + k]) : w[2 * y + k];
          } else if constexpr (B == 2) {
            const uint2 v0 = *reinterpret_cast<const uint2 *>(slot0), v1 = *reinterpret_cast<const uint2 *>(slot1);
            const uint32_t w[2][2] = {{v0.x, v1.x}, {v0.y, v1.y}};
#pragma unroll
            for (int y = 0; y < 2; y++)
#pragma unroll
              for (int k = 0; k < 2; k++) xc[y][k] = add ? add_pk(xc[y][k], w[y][k]) : w[y][k];
          } else {
#pragma unroll
            for (int y = 0; y < HR; y++) {
              const uint2 v = *reinterpret_cast<const uint2 *>(slot0 + y * quads + wib[0]);
              xc[y][0] = add ? add_pk(xc[y][0], v.x) : v.x;
              xc[y][1] = add ? add_pk(xc[y][1], v.y) : v.y;
            }
          }
        };
#pragma unroll
        for (int c = 0; c < 3; c++) {
          {
            const uint32_t *kb = keys + root * lfc::rgb_key_words(B);
            const int k0 = jb[0] * (3 * S / 2) + c * (S / 2), k1 = jb[1] * (3 * S / 2) + c * (S / 2);
            read_slot(kb + k0 + k0 / 64 * (lfc::rgb_key_step(B) - 64), kb + k1, 4, false, x[c]);
          }
#pragma unroll
          for (int k = 0; k < NM; k++) {
            if (NC < 0 && k >= nodes) continue;
            read_slot(tile + slot[c][k][0], tile + slot[c][k][NS - 1], plane, true, x[c]);
          }
        }
        if (!live) continue;
        uint32_t *dst = a.out + (uint32_t)vi * vplane + (uint32_t)(by * B) * (uint32_t)a.wp + (uint32_t)px0;
#pragma unroll
        for (int y = 0; y < HR; y++) {
          uint32_t p[4];
#pragma unroll
          for (int w = 0; w < 2; w++) rgb_pack2(x[0][y][w], x[1][y][w], x[2][y][w], p[2 * w], p[2 * w + 1]);
          uint32_t *row = dst + (uint32_t)y * (uint32_t)a.wp;
          if constexpr (B >= 4) {   // (the padded width is a multiple of four)
            *reinterpret_cast<uint4 *>(row) = make_uint4(p[0], p[1], p[2], p[3]);
          } else {
            *reinterpret_cast<uint2 *>(row) = make_uint2(p[0], p[1]);
            if (px0 + 2 < a.wp) *reinterpret_cast<uint2 *>(row + 2) = make_uint2(p[2], p[3]);
          }
        }
      }
    };
    switch (a.L) {
      case 1: gather(std::integral_constant<int, 0>{}); break;
      case 2: gather(std::integral_constant<int, 1>{}); break;
      case 3: gather(std::integral_constant<int, 2>{}); break;
      default: gather(std::integral_constant<int, -1>{});
    }
    lds_barrier();
  }
}

template <int B>
__global__ __launch_bounds__(kLFThreads, B <= 4 ? 6 : 4) void k_decode_rgb(RGBArgs a) {
  extern __shared__ uint32_t smem[];
  rgb_strip<B>(a, (int)blockIdx.x, smem);
}

// The colour decode of several light fields in one launch: the workgroups are
// every light field's (strip, part) pairs, each light field's strips costliest
// first.  (Workgroups that stayed resident and took items from a device counter
// needed 20 registers more, which kept a third of them off the chip: the 4 x 4
// fields of a mixed batch 99 -> 55 us, its 8 x 8 field 23 -> 14 us, with the
// changes above.)
struct RGBMultiArgs {
  const RGBArgs *lfs;      // [n_lf], every one of block size B
  const int32_t *first;    // [n_lf + 1] first work item of each light field (items = strips x parts)
  int n_lf;
};

template <int B>
__global__ __launch_bounds__(kLFThreads, B <= 4 ? 6 : 4) void k_decode_rgb_multi(RGBMultiArgs m) {
  extern __shared__ uint32_t smem[];
  const uniform_i32 first = as_uniform(m.first);
  const int item = blockIdx.x;
  int lf = 0;
  while (lf + 1 < m.n_lf && first[lf + 1] <= item) lf++;
  const RGBArgs a = m.lfs[lf];
  const int local = item - first[lf];
  rgb_strip<B>(a, local, smem);
}

// Novel views from fully decoded 8-bit RGB source views ([nv][hp][wp]): one
// thread per output column and R consecutive output rows, the same lerps as
// render_tile.  Used when a batch of views needs about as many source blocks
// as the whole light field holds.
// What bounds it: the traffic of the taps (four source views of 4 bytes a
// pixel) and of the output.  The lerps along s, v and u depend on the column
// and the source row only, and consecutive output rows mostly share a source
// row, so a thread keeps the blended values of two source rows and takes a new
// one when the output row moves on: at equal scale half of the tap reads and
// lerps.  Taps are read as pairs (x1 = x0 + 1) in one 8-byte read, all of a
// thread's before its first store: a load issued after stores waits for them
// too (a loop over the rows, each with its own reads, took as long as one row
// per thread).
// Measured, 64 views of 512 x 512 from 17 x 17 x 512 x 512 (167 MB of decoded
// views, 201 MB out): 82 us, 5.1 TB/s of what the counters see, about the rate
// of a copy (112 us with one row per thread and conversions); one row per
// thread 129 us, two 106, eight 81.
struct InterpRGBArgs {
  const uint32_t *rgb;
  uint32_t rgb_bytes;   // bytes of the decoded views (below 4 GiB)
  const lfc_view *views;
  float *out;
  int wo, ho, U, V, W, H, wp, hp;
  float disp;       // focal disparity (as RenderArgs)
  float sxs, tys;   // W / wo and H / ho, rounded once on the host as the other renderers round them
  int stream_out;   // store the output with the non-temporal hint
};

// Output pixels (X, Yb..Yb + R - 1) of view vw into o (its view's [3][ho][wo]
// planes), as far as they are inside.
template <bool FOCAL, int R>
__device__ __forceinline__ void interp_rgb_rows(const InterpRGBArgs &a, const lfc_view &vw, float *o, int X, int Yb) {
  constexpr int NS = FOCAL ? 4 : 1;   // source positions: of each view, or shared
  int iu0, iu1, jv0, jv1, x0, x1;
  float fu, fv;
  cell(vw.u, a.U, iu0, iu1, fu);
  cell(vw.v, a.V, jv0, jv1, fv);
  // (lanes past the row's end, in its last wave, follow the last column: the
  // row positions below come from the wave's first lanes, whatever they hold)
  const float sx = src_pos(vw.s, min(X, a.wo - 1), a.sxs);
  // taps through a buffer resource: 32-bit byte offsets from one base (the
  // decoded views take less than 4 GiB); a row's offset goes in the load's
  // scalar offset, the column in the per-lane one, and the hardware adds them;
  // the stores likewise (a view's planes take at most 3 GiB)
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.rgb), 0, a.rgb_bytes, 0x00020000);
  const uint32_t plane = (uint32_t)a.ho * (uint32_t)a.wo;
  const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(o, 0, 12u * plane, 0x00020000);
  const uint32_t vbytes = 4u * (uint32_t)a.hp * (uint32_t)a.wp, rbytes = 4u * (uint32_t)a.wp;
  const uint32_t vis[4] = {(uint32_t)(jv0 * a.U + iu0), (uint32_t)(jv0 * a.U + iu1), (uint32_t)(jv1 * a.U + iu0),
                           (uint32_t)(jv1 * a.U + iu1)};
  uint32_t vo[4], c0[NS];
  float fs[NS];
#pragma unroll
  for (int k = 0; k < 4; k++) vo[k] = __builtin_amdgcn_readfirstlane(vis[k] * vbytes);
#pragma unroll
  for (int k = 0; k < NS; k++) {
    // (the pair's second pixel is x0 + 1; where the image is one pixel wide,
    // the padding's, at fraction zero)
    cell(sx + focal_shift<FOCAL>(a.disp, vw.u, a.U, (k & 1) ? iu1 : iu0), a.W, x0, x1, fs[k]);
    c0[k] = 4u * (uint32_t)x0;
  }
  // the rows' source positions, the same for the whole wave: lane l finds row
  // l % R's, and they go to scalar registers
  int y0[R][NS], y1[R][NS];
  float ft[R][NS];
  {
    const int l = R == 1 ? 0 : (int)(threadIdx.x & 63) % R;
    const float ty = src_pos(vw.t, min(Yb + l, a.ho - 1), a.tys);
#pragma unroll
    for (int k = 0; k < NS; k++) {
      int u0, u1;
      float f;
      cell(ty + focal_shift<FOCAL>(a.disp, vw.v, a.V, (k & 2) ? jv1 : jv0), a.H, u0, u1, f);
#pragma unroll
      for (int i = 0; i < R; i++) {
        y0[i][k] = R == 1 ? __builtin_amdgcn_readfirstlane(u0) : __builtin_amdgcn_readlane(u0, i);
        y1[i][k] = R == 1 ? __builtin_amdgcn_readfirstlane(u1) : __builtin_amdgcn_readlane(u1, i);
        ft[i][k] = __uint_as_float(R == 1 ? __builtin_amdgcn_readfirstlane(__float_as_uint(f))
                                          : __builtin_amdgcn_readlane(__float_as_uint(f), i));
      }
    }
  }
  // which rows to read: a row's upper source row is read if the row above has
  // it neither as its upper nor as its lower one, the lower unless the row
  // above has it in the same part
  bool nu[R], nl[R];
  u32x2_t wu[R][4], wl[R][4];
  auto read = [&](u32x2_t (&w)[4], const int (&y)[NS]) {
#pragma unroll
    for (int k = 0; k < 4; k++)
      w[k] = __builtin_amdgcn_raw_buffer_load_b64(rs, c0[k % NS], vo[k] + (uint32_t)y[k % NS] * rbytes, 0);
  };
#pragma unroll
  for (int i = 0; i < R; i++) {
    nu[i] = i == 0 || (y0[i][0] != y0[i - 1][0] && y0[i][0] != y1[i - 1][0]);
    nl[i] = i == 0 || y0[i][0] != y0[i - 1][0] || y1[i][0] != y1[i - 1][0];
    if (nu[i]) read(wu[i], y0[i]);
    if (nl[i]) read(wl[i], y1[i]);
  }
  auto slerp = [&](const u32x2_t (&w)[4], float (&h)[4][3]) {
    const uint32_t p[4] = {w[0].x, w[1].x, w[2].x, w[3].x}, q[4] = {w[0].y, w[1].y, w[2].y, w[3].y};
    slerp_taps<NS>(p, q, fs, h);
  };
  auto put = [&](int i, const float (&x)[3]) {
    if (Yb + i >= a.ho || X >= a.wo) return;
    const uint32_t at = 4u * (uint32_t)X, row = 4u * (uint32_t)(Yb + i) * (uint32_t)a.wo;
    if (a.stream_out)
#pragma unroll
      for (uint32_t ch = 0; ch < 3; ch++)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(div255(x[ch])), ro, at, 4u * ch * plane + row, 2 /* nt */);
    else
#pragma unroll
      for (uint32_t ch = 0; ch < 3; ch++)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(div255(x[ch])), ro, at, 4u * ch * plane + row, 0);
  };
  float h[4][3];
  if constexpr (FOCAL) {
    static_assert(R == 1, "the source rows of a refocused pixel are each view's own");
    float g[4][3], x[3];
    slerp(wu[0], h);
    slerp(wl[0], g);
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
      for (int ch = 0; ch < 3; ch++) h[k][ch] = lerpf(h[k][ch], g[k][ch], ft[0][k]);
    blend_views(h, fu, fv, x);
    put(0, x);
  } else {
    // the blended source rows: row i's upper one in place i % 2, its lower one
    // in the other, so that moving on by one source row moves no value
    float row[2][3];
#pragma unroll
    for (int i = 0; i < R; i++) {
      const int U = i & 1;
      if (nu[i]) {
        slerp(wu[i], h);
        blend_views(h, fu, fv, row[U]);
      } else if (i > 0 && y0[i][0] == y0[i - 1][0]) {   // (magnified: the same upper row again)
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
          const float t = row[U][ch];
          row[U][ch] = row[1 - U][ch];
          row[1 - U][ch] = t;
        }
      }
      if (nl[i]) {
        slerp(wl[i], h);
        blend_views(h, fu, fv, row[1 - U]);
      }
      float x[3];
#pragma unroll
      for (int ch = 0; ch < 3; ch++) x[ch] = lerpf(row[U][ch], row[1 - U][ch], ft[i][0]);
      put(i, x);
    }
  }
}

// The grid of the interpolation: workgroups go to the eight dies in turn, and
// the bands of R output rows with them, so that all views' workgroups of a
// band run on one die about together and its L2 serves a source row once for
// every view that reads it (64 views of 512 x 512: 82 us; bands in launch
// order 85; an eighth of the rows per die in one run 86).
struct InterpGrid {
  int pieces, n;   // workgroups per output row, views
  __device__ __forceinline__ void at(int &x, int &view, int &band) const {
    const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
    const int j = (int)(id / 8u), per = pieces * n;
    band = j / per * 8 + (int)(id % 8u);
    x = (j % per % pieces) * kThreads + (int)threadIdx.x;
    view = j % per / pieces;
  }
  // (a grid dimension holds fewer than 2^32 threads; bands past the last exit)
  static constexpr uint32_t kRow = 1u << 23;   // most workgroups in a row of the grid
  dim3 grid(int bands) const {
    const uint64_t blocks = (uint64_t)8 * ((bands + 7) / 8) * pieces * n;
    const uint32_t x = (uint32_t)std::min<uint64_t>(blocks, kRow);
    return dim3(x, (uint32_t)((blocks + x - 1) / x));
  }
  // Most views of one launch: its workgroups' numbers fit 32 bits, the last
  // row's padding included.  (Views of one size never come near, 2^32
  // workgroups of them would not fit the memory; a batch's grid is that of its
  // largest output for every request.)
  static int most_views(int bands, int pieces) {
    return (int)((((uint64_t)1 << 32) - kRow) / ((uint64_t)8 * ((bands + 7) / 8) * pieces));
  }
};

template <bool FOCAL, int R>
__global__ __launch_bounds__(kThreads) void k_interp_rgb(InterpRGBArgs a, InterpGrid g) {
  int X, n, band;
  g.at(X, n, band);
  if (band * R >= a.ho || X - (int)(threadIdx.x & 63) >= a.wo) return;   // (whole waves)
  interp_rgb_rows<FOCAL, R>(a, a.views[n], a.out + (size_t)n * 3 * a.ho * a.wo, X, band * R);
}

// Output rows per thread of the plain interpolation.  Small batches gain too:
// 4 views of 128 x 128 from 8 x 8 x 256 x 256 take 26 us with the decode, 32 us
// with one row per thread; 64 of 512 x 512 take 66, 112.
constexpr int kInterpRows = 4;

// Requests of several light fields and output sizes interpolated in one
// launch: a workgroup exits when its request's output is smaller.  A request's
// record carries its light field's decoded views (views unused; the camera is
// in the record).
struct InterpReq {
  InterpRGBArgs a;
  lfc_view view;
};

__global__ __launch_bounds__(kThreads) void k_interp_multi(const InterpReq *reqs, InterpGrid g) {
  int X, n, band;
  g.at(X, n, band);
  const InterpReq r = reqs[n];
  if (band * kInterpRows >= r.a.ho || X - (int)(threadIdx.x & 63) >= r.a.wo) return;   // (whole waves)
  interp_rgb_rows<false, kInterpRows>(r.a, r.view, r.a.out, X, band * kInterpRows);
}

// ---------------------------------------------------------------------------
// host-side checks and launches
// ---------------------------------------------------------------------------

using lfc::fail;

lfc_status check_device(const lfc_lf *lf, const char *who) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(LFC_E_HIP, std::string(who) + ": no current device");
  if (dev != lf->device)
    return fail(LFC_E_INVALID, std::string(who) + ": the current device is not the one the light field was opened on");
  return LFC_OK;
}

// the device buffer at p must hold at least need bytes inside one allocation
lfc_status check_buffer(const void *p, size_t need, size_t align, const char *who, const char *what) {
  if (!p) return fail(LFC_E_INVALID, std::string(who) + ": null " + what);
  if (reinterpret_cast<uintptr_t>(p) % align)
    return fail(LFC_E_INVALID, std::string(who) + ": " + what + " is not " + std::to_string(align) + "-byte aligned");
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess || !base) {
    (void)hipGetLastError();
    return fail(LFC_E_INVALID, std::string(who) + ": " + what + " is not device memory");
  }
  const size_t off = static_cast<const char *>(p) - static_cast<const char *>(base);
  if (off + need > size) return fail(LFC_E_INVALID, std::string(who) + ": " + what + " is too small");
  return LFC_OK;
}

RAArgs ra_args(const lfc_lf *lf) {
  const lfc::Geometry &g = lf->geo;
  return RAArgs{lf->d_rkv, lf->d_off, lf->d_srv, lf->d_poff, lf->d_path, lf->d_root,
                g.nb, g.nbx, g.nv(), g.nbw, g.L, g.q, lf->d_dir2};
}

lfc_status launched(const char *who) {
  const hipError_t he = hipGetLastError();
  if (he != hipSuccess) return fail(LFC_E_HIP, std::string(who) + ": launch failed: " + hipGetErrorString(he));
  return LFC_OK;
}

// LDS a workgroup may use on the current device (queried once per device).
int max_lds_bytes() {
  constexpr int kDevices = 64;
  static std::atomic<int> cached[kDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 64 * 1024;
  if (dev < kDevices)
    if (const int v = cached[dev].load(std::memory_order_relaxed)) return v;
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0) {
    (void)hipGetLastError();
    v = 64 * 1024;
  }
  if (dev < kDevices) cached[dev].store(v, std::memory_order_relaxed);
  return v;
}

// Compute units of the current device (queried once per device).
int device_cus() {
  constexpr int kDevices = 64;
  static std::atomic<int> cached[kDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
  if (dev < kDevices)
    if (const int v = cached[dev].load(std::memory_order_relaxed)) return v;
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) {
    (void)hipGetLastError();
    v = 256;
  }
  if (dev < kDevices) cached[dev].store(v, std::memory_order_relaxed);
  return v;
}

// Stream-ordered scratch from a memory pool of the library's own per device,
// which keeps up to 1 GiB of freed memory for the next call instead of
// returning it at each synchronisation (the default pool's release threshold
// is zero); the process's default pool is left as it is.
hipMemPool_t scratch_pool() {
  constexpr int kDevices = 64;
  static std::mutex mu;
  static hipMemPool_t pools[kDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!pools[dev]) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pl = nullptr;
    if (hipMemPoolCreate(&pl, &props) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    uint64_t keep = (uint64_t)1 << 30;
    if (hipMemPoolSetAttribute(pl, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) (void)hipGetLastError();
    pools[dev] = pl;
  }
  return pools[dev];
}

// LDS of the whole-field kernel: the fixed part (LUT and extents, residual
// tile, key-view rows) plus staging for the strip's groups and decode
// schedule, up to 80 KB so that two workgroups share a compute unit.
// Output larger than this (the MI355X's 256 MiB Infinity Cache) cannot stay
// cached for a consumer, and stored normally it would evict the compressed
// input; it is stored with the non-temporal hint.
constexpr uint64_t kStreamOutBytes = (uint64_t)256 << 20;

// stage_cap < 0: as much LDS staging as the strips need, up to the 80 KB
// workgroup budget; else at most stage_cap words (tests of the tiers).
template <int B>
lfc_status decode_images(const lfc_lf *lf, int16_t *out, hipStream_t s, int64_t stage_cap = -1) {
  const lfc::Geometry &g = lf->geo;
  constexpr int NBLK = 64 / B;

  // key-view rows of a strip, when they take at most 16 KB
  const int64_t key_words = (int64_t)g.n_top * NBLK * (B * B / 2) <= 4096 ? (int64_t)g.n_top * NBLK * (B * B / 2) : 0;
  if ((int64_t)3 * g.hp * g.wp >= ((int64_t)1 << 32))
    return fail(LFC_E_UNSUPPORTED, "lfc_decode_blocks: view too large for the whole-field kernel");
  const int tab_words = lf->lf_tab_words;
  const int64_t fixed = kLFHeadWords + (int64_t)lf_tile_words(lf->tile_cap, B * B) + key_words + 2 * tab_words;
  const int64_t limit = max_lds_bytes() / 4;
  if (fixed > limit)
    return fail(LFC_E_UNSUPPORTED, "lfc_decode_blocks: tree too large for the whole-field kernel; use BLOCKS layout");
  const int64_t target = std::min<int64_t>(limit, std::max<int64_t>(80 * 1024 / 4, fixed));
  int64_t cap = std::min<int64_t>(target - fixed, (int64_t)lf->max_strip_words + kStagePad);
  if (stage_cap >= 0) cap = std::min<int64_t>(cap, stage_cap);
  const size_t lds = 4 * (size_t)(fixed + cap);
  LFArgs a{lf->d_rkv, lf->d_srv, lf->d_sched, lf->d_order, lf->d_batch, out,
           g.nbx, g.L, g.q, g.wp, g.hp, g.nb, lf->n_batch, (int)cap,
           (int)(g.wp % 8 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0), g.n_top, (int)key_words,
           lf->tile_cap, tab_words, (int)((uint64_t)g.nv() * 3 * g.hp * g.wp * 2 > kStreamOutBytes)};
  dim3 grid((g.nbx + NBLK - 1) / NBLK, g.nby, 3);
  auto *kernel = cap > 0 ? (key_words ? k_decode_lf<B, true, true> : k_decode_lf<B, true, false>)
                         : (key_words ? k_decode_lf<B, false, true> : k_decode_lf<B, false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kLFThreads), lds, s, a);
  return launched("lfc_decode_blocks");
}

// Key views whose rows a workgroup of the colour decode holds in LDS: all, or
// those of one chunk (read from global memory in the gather, they would wait for
// the wave's stores: 289 views of 256 x 256 in two levels 108 -> 31 us, 64 key
// views of 128 x 128 95 -> 9 us).
int rgb_key_views(const lfc_lf *lf) { return std::min(lf->geo.n_top, lfc::rgb_key_roots(lf->geo.B)); }

// Every view (or those whose bit is set in vneed) as 8-bit RGB words
// [nv][hp][wp], inverse YCoCg-R and clamp applied to the decoded samples.
template <int B>
lfc_status decode_rgb(const lfc_lf *lf, uint32_t *out, const uint32_t *vneed, hipStream_t s, const char *who,
                      const lfc_view *views = nullptr, int nviews = 0) {
  const lfc::Geometry &g = lf->geo;
  constexpr int NBLK = 64 / B;
  if ((uint64_t)g.nv() * g.hp * g.wp >= ((uint64_t)1 << 32))
    return fail(LFC_E_UNSUPPORTED, std::string(who) + ": light field too large for 32-bit pixel indices");
  const int key_views = rgb_key_views(lf);
  // a view mask longer than the kernel's LDS copy of it: every view is decoded
  if (g.nv() > 32 * kRGBNeedWords) vneed = nullptr, views = nullptr;
  const int need_words = vneed || (views && nviews > 0) ? (g.nv() + 31) / 32 : 0;
  const size_t lds = 4 * ((size_t)rgb_head_words(need_words, lf->rgb_tab_cap, lf->rgb_run_cap) +
                          (size_t)lf_tile_words(lf->tile_cap_rgb, B * B) + (size_t)key_views * lfc::rgb_key_words(B));
  if (lds > (size_t)max_lds_bytes())
    return fail(LFC_E_UNSUPPORTED, std::string(who) + ": tree too large for the colour whole-field kernel");
  const int nsx = (g.nbx + NBLK - 1) / NBLK, nstrips = g.nby * nsx;
  // workgroups per strip: enough for several rounds of the resident
  // workgroups (about three per compute unit), at most the strips' chunk count
  int parts = std::max(1, std::min(lf->rgb_max_chunks, (3 * 3 * device_cus() + nstrips - 1) / nstrips));
  RGBArgs a{lf->d_rkv, lf->d_off, lf->d_srv, lf->d_sched_rgb, lf->d_order_rgb, lf->d_batch,
            vneed, out, g.nbx, nsx, g.L, g.q, g.wp, g.hp, g.nb, lf->n_batch, g.nv(), g.n_top, key_views,
            lf->tile_cap_rgb, parts, need_words, lf->rgb_tab_cap, lf->rgb_run_cap};
  if (!vneed && views && nviews > 0) {
    a.views = views;
    a.nviews = nviews;
    a.U = g.U;
    a.V = g.V;
  }
  const dim3 grid((unsigned)(nstrips * parts));
  hipLaunchKernelGGL(k_decode_rgb<B>, grid, dim3(kLFThreads), lds, s, a);
  return launched(who);
}

template <int B>
lfc_status decode_list(const lfc_lf *lf, const int32_t *req, int64_t n, int16_t *out, hipStream_t s, int stop = 0) {
  constexpr int RPW = 64 / request_lanes<B>();
  BlocksArgs a{ra_args(lf), req, out, lf->d_err, n, stop};
  const int64_t waves = (n + RPW - 1) / RPW;
  const int64_t blocks = (waves + kThreads / 64 - 1) / (kThreads / 64);
  if (blocks > 0x7FFFFFFF) return fail(LFC_E_INVALID, "lfc_decode_blocks: too many requests");
  if constexpr (B <= 4) {
    // By bands if the list and the tables are long (what is requested of higher
    // levels only is little).  Random lists of 131,072 to 10^6 of 17 x 17 views:
    // 0.76 to 0.94 times as fast with tables of 2 to 4 MB, 0.96 to 1.17 of 5 to 7,
    // 1.1 to 1.3 of 9 to 11, 1.1 to 1.75 from 13 MB on; shorter ones 0.9 to 1.1
    // (30,000) and 0.8 to 1.2 (60,000).  Lists sorted by block lose with any
    // table, 0.65 to 0.9 times, so the line lies where random ones gain more.
    const lfc::Geometry &g = lf->geo;
    const int64_t tables = (int64_t)lf->stream_bytes + 4 * (int64_t)lf->present + 8 * (int64_t)g.ng * g.nbw;
    const int64_t pieces = (n + 2 * kThreads - 1) / (2 * kThreads);
    if (req && stop == 0 && n >= kBandRequests && tables >= kBandBytes && 8 * pieces * kThreads < ((int64_t)1 << 32)) {
      hipLaunchKernelGGL(k_decode_banded<B>, dim3((unsigned)(8 * pieces)), dim3(kThreads), 0, s, a);
      return launched("lfc_decode_blocks");
    }
  }
  hipLaunchKernelGGL(k_decode_blocks<B>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
  return launched("lfc_decode_blocks");
}

// Tile of output pixels per workgroup, and the largest footprint (in blocks)
// any tile can need; starting from TX x TY, shrinks the tile (if allowed)
// until the footprint fits 64 KB of LDS.
struct RenderPlan {
  int TX, TY, fbx, fby;
  size_t lds;
};

bool plan_render(const lfc::Geometry &g, int wo, int ho, RenderPlan &pl, int TX = 64, int TY = 16,
                 bool shrink = true) {
  const double sxs = (double)g.W / wo, tys = (double)g.H / ho;
  for (;;) {
    // footprint span: (T-1)*scale pixels plus the 1-pixel widening on each
    // side, the interpolation neighbour and float slack, then block alignment
    // a tile never spans more than the output
    const int tw = std::min(TX, wo), th = std::min(TY, ho);
    const int fbx = ((int)std::ceil((tw - 1) * sxs) + 5 + g.B - 1) / g.B + 2;
    const int fby = ((int)std::ceil((th - 1) * tys) + 5 + g.B - 1) / g.B + 2;
    const size_t lds = 4 * ((size_t)kLutEntries / 2 + (size_t)4 * fbx * fby * (3 * g.B * g.B / 2));
    if (lds <= 64 * 1024) {
      pl = RenderPlan{TX, TY, fbx, fby, lds};
      return true;
    }
    if (!shrink) return false;
    if (TY > 2) TY /= 2;
    else if (TX > 8) TX /= 2;
    else return false;
  }
}

// The tile of up to 64 x 16 pixels for n renders together: the fewest passes of
// the workgroups over their footprints (a lane takes one channel of one block of
// one view at a time) in all, where a launch of fewer than three workgroups to
// two compute units counts as one of that many, a pass being a chain of reads.
// Against 64 x 16, its height halved until it fits: 512 x 512 of 512 x 512 16.0
// -> 13.7 us, 256 x 256 15.0 -> 8.4, four of 200 x 150 from 400 x 300 37 -> 20.
bool best_plan(const lfc::Geometry &g, int64_t n, int wo, int ho, RenderPlan &best) {
  int64_t cost = INT64_MAX;
  for (int TX = 64; TX >= 8; TX /= 2)
    for (int TY = 16; TY >= 2; TY /= 2) {
      RenderPlan pl;
      if (!plan_render(g, wo, ho, pl, TX, TY, false)) continue;
      const int64_t passes = (12 * pl.fbx * pl.fby + kRenderThreads - 1) / kRenderThreads;
      const int64_t tiles = n * ((wo + TX - 1) / TX) * ((ho + TY - 1) / TY);
      const int64_t c = passes * std::max<int64_t>(tiles, 3 * device_cus() / 2);
      if (c < cost) {
        cost = c;
        best = pl;
      }
    }
  return cost != INT64_MAX;
}

// Decoding every source view once and interpolating from the decoded planes
// pays off when the batch's footprints together cover about as many blocks as
// the light field holds: each output pixel reads four views, and the
// whole-field decode is several times cheaper per block than decoding tile
// footprints.  lfc_render_views_ex forces either path.
bool render_decoded(const lfc::Geometry &g, int32_t n, int32_t wo, int32_t ho) {
  return 20.0 * n * wo * ho >= (double)g.nv() * g.hp * g.wp;
}

// A render request resolved to one launch shape: decode-then-interpolate, or
// per-tile footprint decode with a tile plan.
struct RenderChoice {
  bool decoded;
  RenderPlan pl;
  float disp;   // focal disparity
};

// cfg NULL or path LFC_RENDER_AUTO: the library's choice (render_decoded, and
// best_plan's tile); LFC_RENDER_TILES with
// tile_w x tile_h (0: 64 x 16, shrunk to fit) or LFC_RENDER_DECODED.
lfc_status choose_render(const lfc_lf *lf, int32_t n, int32_t wo, int32_t ho, const lfc_render_config *cfg,
                         RenderChoice &rc, const char *who) {
  const lfc::Geometry &g = lf->geo;
  const int path = cfg ? cfg->path : LFC_RENDER_AUTO;
  if (path != LFC_RENDER_AUTO && path != LFC_RENDER_TILES && path != LFC_RENDER_DECODED)
    return fail(LFC_E_INVALID, std::string(who) + ": unknown render path");
  rc.disp = cfg ? cfg->disparity : 0.0f;
  if (!std::isfinite(rc.disp) || std::fabs(rc.disp) > 1.0e6f)
    return fail(LFC_E_INVALID, std::string(who) + ": disparity must be finite, |d| <= 1e6");
  // the decoded path addresses its scratch with 32-bit byte offsets
  const bool fits = (uint64_t)g.nv() * g.hp * g.wp * 4 < ((uint64_t)1 << 32);
  if (path == LFC_RENDER_DECODED && !fits)
    return fail(LFC_E_UNSUPPORTED, std::string(who) + ": the decoded views would take 4 GiB or more");
  rc.decoded = fits && (path == LFC_RENDER_AUTO ? render_decoded(g, n, wo, ho) : path == LFC_RENDER_DECODED);
  if (rc.decoded) return LFC_OK;
  int TX = 64, TY = 16;
  bool shrink = true;
  if (path == LFC_RENDER_TILES && (cfg->tile_w || cfg->tile_h)) {
    if (cfg->tile_w < 1 || cfg->tile_h < 1 || cfg->tile_w > 1024 || cfg->tile_h > 1024)
      return fail(LFC_E_INVALID, std::string(who) + ": tile_w and tile_h must be 1..1024 (or both 0)");
    TX = cfg->tile_w;
    TY = cfg->tile_h;
    shrink = false;
  }
  if (path == LFC_RENDER_AUTO ? !best_plan(g, n, wo, ho, rc.pl) : !plan_render(g, wo, ho, rc.pl, TX, TY, shrink))
    return fail(LFC_E_UNSUPPORTED, std::string(who) + (shrink ? ": output too strongly minified for the tile footprint"
                                                             : ": the tile's source footprint exceeds 64 KB of LDS"));
  return LFC_OK;
}

// Scratch of the decode-then-interpolate path: the source views as 8-bit
// RGB words.
size_t rgb_bytes(const lfc::Geometry &g) { return (size_t)g.nv() * g.hp * g.wp * sizeof(uint32_t); }
size_t decoded_bytes(const lfc::Geometry &g) { return rgb_bytes(g); }

// Whether a decoded render's output is stored with the non-temporal hint: when
// it and the decoded views do not fit the Infinity Cache together, stored
// normally it would push out the views that are still to be read and the
// compressed input of the next call (64 views of 512 x 512 from 17 x 17 x 512
// x 512: interpolation 82 us, 96 without; the next decode 122, 129).
int stream_render(uint64_t decoded, uint64_t out) { return decoded + out > kStreamOutBytes; }

// One render with a resolved choice.  The decoded path decodes into ws when
// given, else into stream-ordered scratch from the library's pool.
template <int B>
lfc_status render_with(const lfc_lf *lf, const lfc_view *views, int32_t n, int32_t wo, int32_t ho, float *out,
                       const RenderChoice &rc, void *ws, hipStream_t s) {
  const lfc::Geometry &g = lf->geo;
  if (rc.decoded) {
    void *dec = ws;
    if (!dec && lfc::scratch_alloc(&dec, decoded_bytes(g), s) != LFC_OK)
      return fail(LFC_E_NOMEM, "lfc_render_views: scratch for the decoded views");
    uint32_t *rgb = static_cast<uint32_t *>(dec);
    // the views the batch reads (found by each workgroup of the colour
    // decode from the cameras) decoded, then the interpolation
    lfc_status st = decode_rgb<B>(lf, rgb, nullptr, s, "lfc_render_views", views, n);
    if (st == LFC_OK) {
      InterpRGBArgs ia{rgb, (uint32_t)rgb_bytes(g), views, out, wo, ho, g.U, g.V, g.W, g.H, g.wp, g.hp, rc.disp,
                       (float)g.W / (float)wo, (float)g.H / (float)ho,
                       stream_render(decoded_bytes(g), (uint64_t)12 * n * wo * ho)};
      const InterpGrid gr{(wo + kThreads - 1) / kThreads, n};
      if (rc.disp != 0.0f)
        hipLaunchKernelGGL((k_interp_rgb<true, 1>), gr.grid(ho), dim3(kThreads), 0, s, ia, gr);
      else
        hipLaunchKernelGGL((k_interp_rgb<false, kInterpRows>), gr.grid((ho + kInterpRows - 1) / kInterpRows),
                           dim3(kThreads), 0, s, ia, gr);
      st = launched("lfc_render_views");
    }
    if (!ws && hipFreeAsync(dec, s) != hipSuccess && st == LFC_OK)
      st = fail(LFC_E_HIP, "lfc_render_views: scratch release");
    return st;
  }
  const RenderPlan &pl = rc.pl;
  RenderArgs a{ra_args(lf), views, out, wo, ho, g.U, g.V, g.W, g.H, pl.TX, pl.TY, pl.fbx, pl.fby, rc.disp};
  dim3 grid((wo + pl.TX - 1) / pl.TX, (ho + pl.TY - 1) / pl.TY, n);
  if (rc.disp != 0.0f)
    hipLaunchKernelGGL((k_render<B, true>), grid, dim3(kRenderThreads), pl.lds, s, a);
  else
    hipLaunchKernelGGL((k_render<B, false>), grid, dim3(kRenderThreads), pl.lds, s, a);
  return launched("lfc_render_views");
}

lfc_status render_any(const lfc_lf *lf, const lfc_view *views, int32_t n, int32_t wo, int32_t ho, float *out,
                      const RenderChoice &rc, void *ws, hipStream_t s) {
  switch (lf->geo.B) {
    case 2: return render_with<2>(lf, views, n, wo, ho, out, rc, ws, s);
    case 4: return render_with<4>(lf, views, n, wo, ho, out, rc, ws, s);
    default: return render_with<8>(lf, views, n, wo, ho, out, rc, ws, s);
  }
}

// Argument checks shared by the render entry points.
lfc_status check_render(const lfc_lf *lf, const lfc_view *d_views, int32_t n, int32_t out_w, int32_t out_h,
                        const float *d_out, const char *who) {
  if (!lf) return fail(LFC_E_INVALID, std::string(who) + ": null handle");
  if (lfc_status st = check_device(lf, who)) return st;
  if (n < 0 || n > 65535) return fail(LFC_E_INVALID, std::string(who) + ": n must be 0..65535");
  if (out_w < 1 || out_h < 1 || out_w > 16384 || out_h > 16384)
    return fail(LFC_E_INVALID, std::string(who) + ": out_w and out_h must be 1..16384");
  if (n == 0) return LFC_OK;
  if (lfc_status st = check_buffer(d_views, (size_t)n * sizeof(lfc_view), 4, who, "d_views")) return st;
  return check_buffer(d_out, (size_t)n * 3 * out_h * out_w * 4, 4, who, "d_out");
}

}  // namespace

extern "C" lfc_status lfc_decode_blocks(const lfc_lf *lf, const int32_t *d_req, int64_t n, int32_t layout,
                                        int16_t *d_out, hipStream_t s) {
  return lfc_decode_blocks_ex(lf, d_req, n, layout, d_out, nullptr, s);
}

extern "C" lfc_status lfc_decode_blocks_ex(const lfc_lf *lf, const int32_t *d_req, int64_t n, int32_t layout,
                                           int16_t *d_out, const lfc_decode_config *cfg, hipStream_t s) {
  const char *who = "lfc_decode_blocks";
  const int64_t stage_cap = cfg ? cfg->stage_cap_words : (lf ? lf->stage_cap : 0);
  if (stage_cap < -1) return fail(LFC_E_INVALID, "lfc_decode_blocks: stage_cap_words must be >= -1");
  if (!lf) return fail(LFC_E_INVALID, "lfc_decode_blocks: null handle");
  if (lfc_status st = check_device(lf, who)) return st;
  const lfc::Geometry &g = lf->geo;
  if (n < 0) return fail(LFC_E_INVALID, "lfc_decode_blocks: n < 0");
  if (layout == LFC_LAYOUT_IMAGES) {
    if (d_req) return fail(LFC_E_INVALID, "lfc_decode_blocks: the images layout decodes every block (d_req must be NULL)");
    if (n != g.nv()) return fail(LFC_E_INVALID, "lfc_decode_blocks: images layout needs n == grid_u*grid_v");
    if (lfc_status st = check_buffer(d_out, (size_t)g.nv() * 3 * g.hp * g.wp * 2, 16, who, "d_out")) return st;
    switch (g.B) {
      case 2: return decode_images<2>(lf, d_out, s, stage_cap);
      case 4: return decode_images<4>(lf, d_out, s, stage_cap);
      default: return decode_images<8>(lf, d_out, s, stage_cap);
    }
  }
  if (layout != LFC_LAYOUT_BLOCKS) return fail(LFC_E_INVALID, "lfc_decode_blocks: unknown layout");
  if (n == 0) return LFC_OK;
  if (!d_req && n != (int64_t)g.nv() * g.nb)
    return fail(LFC_E_INVALID, "lfc_decode_blocks: with d_req NULL, n must be grid_u*grid_v*n_blocks");
  if (d_req)
    if (lfc_status st = check_buffer(d_req, (size_t)n * 8, 4, who, "d_req")) return st;
  if (lfc_status st = check_buffer(d_out, (size_t)n * 3 * g.S * 2, 16, who, "d_out")) return st;
  switch (g.B) {
    case 2: return decode_list<2>(lf, d_req, n, d_out, s);
    case 4: return decode_list<4>(lf, d_req, n, d_out, s);
    default: return decode_list<8>(lf, d_req, n, d_out, s);
  }
}

extern "C" lfc_status lfc_decode_rgb(const lfc_lf *lf, uint32_t *d_out, hipStream_t s) {
  const char *who = "lfc_decode_rgb";
  if (!lf) return fail(LFC_E_INVALID, "lfc_decode_rgb: null handle");
  if (lfc_status st = check_device(lf, who)) return st;
  if (lfc_status st = check_buffer(d_out, rgb_bytes(lf->geo), 16, who, "d_out")) return st;
  switch (lf->geo.B) {
    case 2: return decode_rgb<2>(lf, d_out, nullptr, s, who);
    case 4: return decode_rgb<4>(lf, d_out, nullptr, s, who);
    default: return decode_rgb<8>(lf, d_out, nullptr, s, who);
  }
}

extern "C" lfc_status lfc_decode_progressive(const lfc_lf *lf, const int32_t *d_req, int64_t n, int32_t level,
                                             int16_t *d_out, hipStream_t s) {
  const char *who = "lfc_decode_progressive";
  if (!lf) return fail(LFC_E_INVALID, "lfc_decode_progressive: null handle");
  if (lfc_status st = check_device(lf, who)) return st;
  const lfc::Geometry &g = lf->geo;
  if (n < 0) return fail(LFC_E_INVALID, "lfc_decode_progressive: n < 0");
  if (level < 0 || level >= g.L) return fail(LFC_E_INVALID, "lfc_decode_progressive: level must be 0..levels-1");
  if (n == 0) return LFC_OK;
  if (!d_req && n != (int64_t)g.nv() * g.nb)
    return fail(LFC_E_INVALID, "lfc_decode_progressive: with d_req NULL, n must be grid_u*grid_v*n_blocks");
  if (d_req)
    if (lfc_status st = check_buffer(d_req, (size_t)n * 8, 4, who, "d_req")) return st;
  if (lfc_status st = check_buffer(d_out, (size_t)n * 3 * g.S * 2, 16, who, "d_out")) return st;
  switch (g.B) {
    case 2: return decode_list<2>(lf, d_req, n, d_out, s, level);
    case 4: return decode_list<4>(lf, d_req, n, d_out, s, level);
    default: return decode_list<8>(lf, d_req, n, d_out, s, level);
  }
}

extern "C" lfc_status lfc_render_views(const lfc_lf *lf, const lfc_view *d_views, int32_t n, int32_t out_w,
                                       int32_t out_h, float *d_out, hipStream_t s) {
  return lfc_render_views_ex(lf, d_views, n, out_w, out_h, d_out, nullptr, s);
}

extern "C" lfc_status lfc_render_views_ex(const lfc_lf *lf, const lfc_view *d_views, int32_t n, int32_t out_w,
                                          int32_t out_h, float *d_out, const lfc_render_config *cfg, hipStream_t s) {
  const char *who = "lfc_render_views";
  if (lfc_status st = check_render(lf, d_views, n, out_w, out_h, d_out, who)) return st;
  if (n == 0) return LFC_OK;
  RenderChoice rc;
  if (lfc_status st = choose_render(lf, n, out_w, out_h, cfg, rc, who)) return st;
  return render_any(lf, d_views, n, out_w, out_h, d_out, rc, nullptr, s);
}

namespace {

// Device address of `scratch` on the current device, looked up once per
// device (the first call on a device) and kept.
lfc_status noalloc_scratch(void **out, const char *who) {
  constexpr int kDevices = 64;
  static std::atomic<void *> ptrs[kDevices];
  static std::mutex mu;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return fail(LFC_E_HIP, std::string(who) + ": no current device");
  if (dev >= kDevices) return fail(LFC_E_UNSUPPORTED, std::string(who) + ": device index above 63");
  void *p = ptrs[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lock(mu);
    p = ptrs[dev].load(std::memory_order_relaxed);
    if (!p) {
      const hipError_t he = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (he != hipSuccess || !p) {
        (void)hipGetLastError();
        return fail(LFC_E_HIP, std::string(who) + ": address of the static scratch: " + hipGetErrorString(he));
      }
      ptrs[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return LFC_OK;
}

}  // namespace

extern "C" lfc_status lfc_render_views_noalloc(const lfc_lf *lf, const lfc_view *d_views, int32_t n, int32_t out_w,
                                               int32_t out_h, float *d_out, const lfc_render_config *cfg,
                                               hipStream_t s) {
  const char *who = "lfc_render_views_noalloc";
  if (lfc_status st = check_render(lf, d_views, n, out_w, out_h, d_out, who)) return st;
  if (n == 0) return LFC_OK;
  RenderChoice rc;
  if (lfc_status st = choose_render(lf, n, out_w, out_h, cfg, rc, who)) return st;
  const size_t need = decoded_bytes(lf->geo);
  if (rc.decoded && need > (size_t)LFC_NOALLOC_SCRATCH_BYTES) {
    if (cfg && cfg->path == LFC_RENDER_DECODED)
      return fail(LFC_E_RANGE, std::string(who) + ": the decoded views need " + std::to_string(need) +
                                   " bytes; the static scratch holds " + std::to_string(LFC_NOALLOC_SCRATCH_BYTES));
    // the automatic choice falls back to the tile path, which needs no scratch
    rc.decoded = false;
    if (!best_plan(lf->geo, n, out_w, out_h, rc.pl))
      return fail(LFC_E_UNSUPPORTED, std::string(who) + ": output too strongly minified for the tile footprint");
  }
  void *ws = nullptr;
  if (rc.decoded)
    if (lfc_status st = noalloc_scratch(&ws, who)) return st;
  return render_any(lf, d_views, n, out_w, out_h, d_out, rc, ws, s);
}

// Measured tuning: every candidate launch shape timed on the caller's views.
extern "C" lfc_status lfc_render_tune(const lfc_lf *lf, const lfc_view *d_views, int32_t n, int32_t out_w,
                                      int32_t out_h, float *d_out, int32_t reps, lfc_render_tuning *res,
                                      hipStream_t s) {
  const char *who = "lfc_render_tune";
  if (!res) return fail(LFC_E_INVALID, "lfc_render_tune: null result");
  if (lfc_status st = check_render(lf, d_views, n, out_w, out_h, d_out, who)) return st;
  if (n < 1 || reps < 1 || reps > 1000) return fail(LFC_E_INVALID, "lfc_render_tune: need n >= 1 and reps 1..1000");
  std::memset(res, 0, sizeof *res);
  static const int kShapes[][2] = {{32, 8}, {32, 16}, {64, 8}, {64, 16}, {64, 32}, {128, 8}, {128, 16}, {256, 8}};
  std::vector<lfc_render_config> cands;
  cands.push_back(lfc_render_config{LFC_RENDER_DECODED, 0, 0, 0.0f});
  RenderPlan pl{};   // the automatic choice's tile first, so that no choice made here is slower than it
  if (best_plan(lf->geo, n, out_w, out_h, pl)) cands.push_back(lfc_render_config{LFC_RENDER_TILES, pl.TX, pl.TY, 0.0f});
  const int auto_w = pl.TX, auto_h = pl.TY;
  for (const auto &sh : kShapes) {
    if (sh[0] == auto_w && sh[1] == auto_h) continue;
    if (plan_render(lf->geo, out_w, out_h, pl, sh[0], sh[1], false))
      cands.push_back(lfc_render_config{LFC_RENDER_TILES, sh[0], sh[1], 0.0f});
  }
  void *ws = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  lfc_status st = LFC_OK;
  if (hipMalloc(&ws, decoded_bytes(lf->geo)) != hipSuccess) {
    ws = nullptr;
    (void)hipGetLastError();      // clear the failed allocation's error
    cands.erase(cands.begin());   // no room for the decoded views: tile shapes only
  }
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) st = fail(LFC_E_HIP, "lfc_render_tune: events");
  float best = 0.0f;
  for (size_t i = 0; st == LFC_OK && i < cands.size() && res->n_tried < LFC_TUNE_MAX; i++) {
    RenderChoice rc;
    if (choose_render(lf, n, out_w, out_h, &cands[i], rc, who) != LFC_OK) continue;
    st = render_any(lf, d_views, n, out_w, out_h, d_out, rc, ws, s);   // warm-up
    if (st == LFC_OK && hipEventRecord(e0, s) != hipSuccess) st = fail(LFC_E_HIP, "lfc_render_tune: event record");
    for (int r = 0; st == LFC_OK && r < reps; r++) st = render_any(lf, d_views, n, out_w, out_h, d_out, rc, ws, s);
    float ms = 0.0f;
    if (st == LFC_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
      st = fail(LFC_E_HIP, "lfc_render_tune: timing");
    if (st != LFC_OK) break;
    const int k = res->n_tried++;
    res->cfg[k] = cands[i];
    res->ms[k] = ms / (float)reps;
    if (k == 0 || res->ms[k] < best) {
      best = res->ms[k];
      res->best = k;
    }
  }
  if (st == LFC_OK && res->n_tried == 0) st = fail(LFC_E_UNSUPPORTED, "lfc_render_tune: no launch shape fits this output");
  if (hipStreamSynchronize(s) != hipSuccess && st == LFC_OK) st = fail(LFC_E_HIP, "lfc_render_tune: synchronize");
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (ws) (void)hipFree(ws);
  return st;
}

// A render with everything fixed at creation, optionally captured in a graph.
struct lfc_render_plan {
  const lfc_lf *lf = nullptr;
  const lfc_view *views = nullptr;
  float *out = nullptr;
  int32_t n = 0, w = 0, h = 0;
  RenderChoice rc{};
  void *ws = nullptr;               // decoded views and their mask (decoded path)
  hipStream_t cap = nullptr;        // stream the graph was captured on
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

extern "C" void lfc_render_plan_destroy(lfc_render_plan *p) {
  if (!p) return;
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  if (p->cap) (void)hipStreamDestroy(p->cap);
  if (p->ws) (void)hipFree(p->ws);
  delete p;
}

extern "C" lfc_status lfc_render_plan_create(const lfc_lf *lf, const lfc_render_config *cfg, const lfc_view *d_views,
                                             int32_t n, int32_t out_w, int32_t out_h, float *d_out, int32_t graph,
                                             lfc_render_plan **out) {
  const char *who = "lfc_render_plan_create";
  if (!out) return fail(LFC_E_INVALID, "lfc_render_plan_create: null result");
  *out = nullptr;
  if (lfc_status st = check_render(lf, d_views, n, out_w, out_h, d_out, who)) return st;
  if (n < 1) return fail(LFC_E_INVALID, "lfc_render_plan_create: n must be 1..65535");
  lfc_render_plan *p = new (std::nothrow) lfc_render_plan;
  if (!p) return fail(LFC_E_NOMEM, "lfc_render_plan_create: out of host memory");
  p->lf = lf;
  p->views = d_views;
  p->out = d_out;
  p->n = n;
  p->w = out_w;
  p->h = out_h;
  lfc_status st = choose_render(lf, n, out_w, out_h, cfg, p->rc, who);
  if (st == LFC_OK && p->rc.decoded) {
    hipError_t he = hipMalloc(&p->ws, decoded_bytes(lf->geo));
    if (he != hipSuccess) {
      p->ws = nullptr;
      st = fail(he == hipErrorOutOfMemory ? LFC_E_NOMEM : LFC_E_HIP, "lfc_render_plan_create: decoded views");
    }
  }
  if (st == LFC_OK && graph) {
    (void)max_lds_bytes();   // device queries done before the capture
    (void)device_cus();
    if (hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking) != hipSuccess) {
      p->cap = nullptr;
      st = fail(LFC_E_HIP, "lfc_render_plan_create: capture stream");
    } else if (hipStreamBeginCapture(p->cap, hipStreamCaptureModeRelaxed) != hipSuccess) {
      st = fail(LFC_E_HIP, "lfc_render_plan_create: begin capture");
    } else {
      st = render_any(lf, d_views, n, out_w, out_h, d_out, p->rc, p->ws, p->cap);
      hipGraph_t g = nullptr;
      const hipError_t he = hipStreamEndCapture(p->cap, &g);
      p->graph = g;
      if (st == LFC_OK && (he != hipSuccess || !g)) st = fail(LFC_E_HIP, "lfc_render_plan_create: end capture");
      if (st == LFC_OK && hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0) != hipSuccess) {
        p->exec = nullptr;
        st = fail(LFC_E_HIP, "lfc_render_plan_create: graph instantiation");
      }
    }
  }
  if (st != LFC_OK) {
    lfc_render_plan_destroy(p);
    return st;
  }
  *out = p;
  return LFC_OK;
}

extern "C" lfc_status lfc_render_plan_launch(lfc_render_plan *p, hipStream_t s) {
  if (!p) return fail(LFC_E_INVALID, "lfc_render_plan_launch: null plan");
  if (lfc_status st = check_device(p->lf, "lfc_render_plan_launch")) return st;
  if (p->exec) {
    if (hipGraphLaunch(p->exec, s) != hipSuccess) return fail(LFC_E_HIP, "lfc_render_plan_launch: graph launch");
    return LFC_OK;
  }
  return render_any(p->lf, p->views, p->n, p->w, p->h, p->out, p->rc, p->ws, s);
}

extern "C" lfc_status lfc_render_plan_info(const lfc_render_plan *p, lfc_render_config *cfg, int32_t *graph) {
  if (!p || !cfg || !graph) return fail(LFC_E_INVALID, "lfc_render_plan_info: null argument");
  *cfg = p->rc.decoded ? lfc_render_config{LFC_RENDER_DECODED, 0, 0, p->rc.disp}
                       : lfc_render_config{LFC_RENDER_TILES, p->rc.pl.TX, p->rc.pl.TY, p->rc.disp};
  *graph = p->exec != nullptr;
  return LFC_OK;
}

namespace lfc {

lfc_status scratch_alloc(void **p, size_t bytes, hipStream_t s) {
  *p = nullptr;
  hipMemPool_t pl = scratch_pool();
  const hipError_t he = pl ? hipMallocFromPoolAsync(p, bytes, pl, s) : hipMallocAsync(p, bytes, s);
  if (he != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
    return LFC_E_NOMEM;
  }
  return LFC_OK;
}

lfc_status device_buffer(const void *p, size_t need, size_t align, const char *who, const char *what) {
  return check_buffer(p, need, align, who, what);
}

size_t render_req_bytes() { return sizeof(RenderReq); }

size_t lf_table_bytes() { return sizeof(RAArgs); }

int lf_block(const lfc_lf *lf) { return lf->geo.B; }

void lf_table_fill(const lfc_lf *lf, void *dst) {
  const RAArgs r = ra_args(lf);
  std::memcpy(dst, &r, sizeof r);
}

lfc_status decode_multi_launch(int block, const void *d_lfs, int n_lf, const int32_t *d_req, int64_t n, int16_t *out,
                               int32_t *err, hipStream_t s) {
  if (n <= 0) return LFC_OK;
  MultiArgs a{static_cast<const RAArgs *>(d_lfs), n_lf, d_req, out, err, n};
  const int rpw = 64 / (block == 2 ? request_lanes<2>() : (block == 4 ? request_lanes<4>() : request_lanes<8>()));
  const int64_t waves = (n + rpw - 1) / rpw;
  const int64_t blocks = (waves + kThreads / 64 - 1) / (kThreads / 64);
  if (blocks > 0x7FFFFFFF) return fail(LFC_E_INVALID, "lfc_batch_decode: too many requests");
  switch (block) {
    case 2: hipLaunchKernelGGL(k_decode_multi<2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_decode_multi<4>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a); break;
    default: hipLaunchKernelGGL(k_decode_multi<8>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a); break;
  }
  return launched("lfc_batch_decode");
}

int lf_device(const lfc_lf *lf) { return lf->device; }

lfc_status render_req_fill(const lfc_lf *lf, const lfc_view &v, int wo, int ho, int n, float *out, void *dst, int *block,
                           int *ntiles, size_t *lds) {
  const Geometry &g = lf->geo;
  RenderPlan pl;
  if (!best_plan(g, n, wo, ho, pl))
    return fail(LFC_E_UNSUPPORTED, "lfc_batch_render: output too strongly minified for the tile footprint");
  RenderReq r{};
  r.a = RenderArgs{ra_args(lf), nullptr, out, wo, ho, g.U, g.V, g.W, g.H, pl.TX, pl.TY, pl.fbx, pl.fby, 0.0f};
  r.view = v;
  r.ntx = (wo + pl.TX - 1) / pl.TX;
  r.ntiles = r.ntx * ((ho + pl.TY - 1) / pl.TY);
  std::memcpy(dst, &r, sizeof r);
  *block = g.B;
  *ntiles = r.ntiles;
  *lds = pl.lds;
  return LFC_OK;
}

// ---- the colour decode-then-interpolate path of a batch -------------------

namespace {

int rgb_parts(const lfc_lf *lf) {
  const lfc::Geometry &g = lf->geo;
  const int nblk = 64 / g.B, nstrips = g.nby * ((g.nbx + nblk - 1) / nblk);
  return std::max(1, std::min(lf->rgb_max_chunks, (3 * 3 * device_cus() + nstrips - 1) / nstrips));
}

}  // namespace

bool lf_rgb_batchable(const lfc_lf *lf, double out_pixels) {
  const Geometry &g = lf->geo;
  const size_t lds = 4 * ((size_t)rgb_head_words((g.nv() + 31) / 32, lf->rgb_tab_cap, lf->rgb_run_cap) +
                          (size_t)lf_tile_words(lf->tile_cap_rgb, g.B * g.B) + (size_t)rgb_key_views(lf) * lfc::rgb_key_words(g.B));
  return (uint64_t)g.nv() * g.hp * g.wp * 4 < ((uint64_t)1 << 32) && g.nv() <= 32 * kRGBNeedWords &&
         lds <= (size_t)max_lds_bytes() && 20.0 * out_pixels >= (double)g.nv() * g.hp * g.wp;
}

size_t lf_rgb_bytes(const lfc_lf *lf) { return rgb_bytes(lf->geo); }

int lf_rgb_items(const lfc_lf *lf) {
  const Geometry &g = lf->geo;
  const int nblk = 64 / g.B;
  return g.nby * ((g.nbx + nblk - 1) / nblk) * rgb_parts(lf);
}

int lf_views(const lfc_lf *lf) { return lf->geo.nv(); }

size_t rgb_args_bytes() { return sizeof(RGBArgs); }

void rgb_args_fill(const lfc_lf *lf, uint32_t *d_rgb, const uint32_t *d_mask, void *dst) {
  const Geometry &g = lf->geo;
  const int nblk = 64 / g.B;
  RGBArgs a{lf->d_rkv, lf->d_off, lf->d_srv, lf->d_sched_rgb, lf->d_order_rgb, lf->d_batch,
            d_mask, d_rgb, g.nbx, (g.nbx + nblk - 1) / nblk, g.L, g.q, g.wp, g.hp, g.nb, lf->n_batch, g.nv(),
            g.n_top, rgb_key_views(lf), lf->tile_cap_rgb, rgb_parts(lf), (g.nv() + 31) / 32, lf->rgb_tab_cap,
            lf->rgb_run_cap};
  std::memcpy(dst, &a, sizeof a);
}

size_t rgb_lds_bytes(const lfc_lf *lf) {
  const Geometry &g = lf->geo;
  return 4 * ((size_t)rgb_head_words((g.nv() + 31) / 32, lf->rgb_tab_cap, lf->rgb_run_cap) +
              (size_t)lf_tile_words(lf->tile_cap_rgb, g.B * g.B) + (size_t)rgb_key_views(lf) * lfc::rgb_key_words(g.B));
}

void need_mask_host(const lfc_lf *lf, const lfc_view &v, uint32_t *mask) {
  const Geometry &g = lf->geo;
  // the grid cell the renderers read (cell() on the device, the same float
  // clamp and floor)
  auto cell_host = [](float x, int n, int &i0, int &i1) {
    x = std::fmin(std::fmax(x, 0.0f), (float)(n - 1));
    if (n == 1) {
      i0 = i1 = 0;
      return;
    }
    int i = (int)std::floor(x);
    i = std::min(std::max(i, 0), n - 2);
    i0 = i;
    i1 = i + 1;
  };
  int iu0, iu1, jv0, jv1;
  cell_host(v.u, g.U, iu0, iu1);
  cell_host(v.v, g.V, jv0, jv1);
  for (int vi : {jv0 * g.U + iu0, jv0 * g.U + iu1, jv1 * g.U + iu0, jv1 * g.U + iu1}) mask[vi >> 5] |= 1u << (vi & 31);
}

size_t interp_req_bytes() { return sizeof(InterpReq); }

void interp_req_fill(const lfc_lf *lf, const uint32_t *d_rgb, const lfc_view &v, int wo, int ho, float *out,
                     uint64_t call_bytes, void *dst) {
  const Geometry &g = lf->geo;
  InterpReq r{};
  r.a = InterpRGBArgs{d_rgb, (uint32_t)rgb_bytes(g), nullptr, out, wo, ho, g.U, g.V, g.W, g.H, g.wp, g.hp, 0.0f,
                      (float)g.W / (float)wo, (float)g.H / (float)ho, call_bytes > kStreamOutBytes};
  r.view = v;
  std::memcpy(dst, &r, sizeof r);
}

lfc_status rgb_multi_launch(int block, const void *d_args, const int32_t *d_first, int n_lf, int n_items,
                            size_t lds, hipStream_t s) {
  if (n_items <= 0) return LFC_OK;
  RGBMultiArgs m{static_cast<const RGBArgs *>(d_args), d_first, n_lf};
  auto launch = [&](auto kern) -> lfc_status {
    hipLaunchKernelGGL(kern, dim3((unsigned)n_items), dim3(kLFThreads), lds, s, m);
    return launched("lfc_batch_render");
  };
  switch (block) {
    case 2: return launch(k_decode_rgb_multi<2>);
    case 4: return launch(k_decode_rgb_multi<4>);
    default: return launch(k_decode_rgb_multi<8>);
  }
}

lfc_status interp_multi_launch(const void *d_reqs, int n, int max_wo, int max_ho, hipStream_t s) {
  if (n <= 0) return LFC_OK;
  if (n > 65535) return fail(LFC_E_INVALID, "lfc_batch_render: at most 65535 interpolated requests per batch");
  const int pieces = (max_wo + kThreads - 1) / kThreads, bands = (max_ho + kInterpRows - 1) / kInterpRows;
  const int most = InterpGrid::most_views(bands, pieces);   // (16,352 or more)
  lfc_status st = LFC_OK;
  for (int at = 0; at < n && st == LFC_OK; at += most) {
    const InterpGrid gr{pieces, std::min(most, n - at)};
    hipLaunchKernelGGL(k_interp_multi, gr.grid(bands), dim3(kThreads), 0, s, static_cast<const InterpReq *>(d_reqs) + at, gr);
    st = launched("lfc_batch_render");
  }
  return st;
}

lfc_status render_multi_launch(int block, const void *d_reqs, int n, int max_tiles, size_t lds, hipStream_t s) {
  if (n <= 0) return LFC_OK;
  if (n > 65535) return fail(LFC_E_INVALID, "lfc_batch_render: at most 65535 requests of one block size per batch");
  const RenderReq *r = static_cast<const RenderReq *>(d_reqs);
  dim3 grid((unsigned)max_tiles, (unsigned)n);
  switch (block) {
    case 2: hipLaunchKernelGGL(k_render_multi<2>, grid, dim3(kRenderThreads), lds, s, r); break;
    case 4: hipLaunchKernelGGL(k_render_multi<4>, grid, dim3(kRenderThreads), lds, s, r); break;
    default: hipLaunchKernelGGL(k_render_multi<8>, grid, dim3(kRenderThreads), lds, s, r); break;
  }
  return launched("lfc_batch_render");
}

}  // namespace lfc
