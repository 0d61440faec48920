// CompressLFI (Alg. 1) on the GPU: the same stream, byte for byte, as the
// host encoder with the paper's global thresholds (lfc_encode_ex).
//
// Level 0 (YCoCg-R of the padded views, Sec. 4), the key-view filter of
// each level (eqs. 1-2), and, level by level from the top, the closed-loop
// residuals against the reconstructed parent (eq. 3 with the pixel and
// block-energy thresholds and the quantiser, Sec. 3.2) walk plane rows, several
// samples or one block per thread; then the groups' sizes and offsets, and
// every group's bitmap, range codes and BISE payloads (Sec. 3.3-3.4), packed by
// one wave per group.  The host writes the header around them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "encode.h"
#include "internal.h"
#include "serve.h"

namespace {

constexpr int kT = 256;

struct EncGeo {
  int U, V, W, H, wp, hp, B, S, L, q, nbx, nb, ng, n_srv, nbw;
  int lu[lfc::kMaxLevels], lv[lfc::kMaxLevels], c[lfc::kMaxLevels];
  int pix_thr, blk_thr;
};

// The smallest allowed range code that holds a largest zigzag value below
// kZMax (-1: none; no code holds more).
constexpr int kZMax = 4096;
struct RangeTab {
  int8_t code[kZMax];
};

__device__ __forceinline__ uint32_t zz(int32_t v) { return (uint16_t)(((uint32_t)v << 1) ^ (uint32_t)(v >> 31)); }

// range code k: kind (0 bits, 1 trit, 2 quint) and low-bit count m
__device__ __forceinline__ void code_km(int k, int &kind, int &m) {
  kind = k < 12 ? 0 : (k < 19 ? 1 : 2);
  m = k - (k < 12 ? -1 : (k < 19 ? 12 : 19));
}

__device__ __forceinline__ uint32_t block_bits_d(int k, int S) {
  int kind, m;
  code_km(k, kind, m);
  const uint32_t plane = kind == 1 ? (8u * S + 4u) / 5u : (kind == 2 ? (7u * S + 2u) / 3u : 0u);
  return (uint32_t)(S * m) + plane;
}

// N consecutive int16 samples, aligned to their size
template <int N>
struct alignas(2 * N) Samples {
  int16_t v[N];
};

struct __attribute__((packed)) Words3 {
  uint32_t v[3];
};

// level 0: padded YCoCg-R planes [nv][3][hp][wp], edges replicated; N samples
// of a row per thread (bound by its 9 bytes a pixel: 34 us for 9 x 9 x 625 x
// 434, 5.9 TB/s; byte loads of one pixel per thread took 54 to 74 us)
template <int N>
__global__ __launch_bounds__(kT) void k_enc_level0(const uint8_t *rgb, int16_t *lvl, EncGeo g) {
  const int per = g.wp / N, i = blockIdx.x * kT + threadIdx.x, vi = blockIdx.y;
  if (i >= per * g.hp) return;
  const int y = i / per, x = i % per * N, sy = min(y, g.H - 1);
  const uint8_t *row = rgb + ((size_t)vi * g.H + sy) * g.W * 3;
  uint8_t px[3 * N];
  if (N == 4 && x + N <= g.W) {   // (words at any byte offset)
    const Words3 w = *reinterpret_cast<const Words3 *>(row + 3 * (size_t)x);
#pragma unroll
    for (int k = 0; k < 3 * N; k++) px[k] = (uint8_t)(w.v[k / 4] >> (8 * (k % 4)));
  } else {
#pragma unroll
    for (int k = 0; k < N; k++)
#pragma unroll
      for (int c = 0; c < 3; c++) px[3 * k + c] = row[3 * (size_t)min(x + k, g.W - 1) + c];
  }
  Samples<N> o[3];
#pragma unroll
  for (int k = 0; k < N; k++) {
    const int co = px[3 * k] - px[3 * k + 2];
    const int t = px[3 * k + 2] + (co >> 1);
    const int cg = px[3 * k + 1] - t;
    o[0].v[k] = (int16_t)(t + (cg >> 1));
    o[1].v[k] = (int16_t)co;
    o[2].v[k] = (int16_t)cg;
  }
  const size_t plane = (size_t)g.hp * g.wp, at = (size_t)vi * 3 * plane + (size_t)y * g.wp + x;
#pragma unroll
  for (int c = 0; c < 3; c++) *reinterpret_cast<Samples<N> *>(lvl + at + c * plane) = o[c];
}

// level l >= 1: the binomial-weighted, rounded mean of each cluster of
// level l-1 over the members that exist (eqs. 1-2); N samples per thread.  The
// weights sum to at most 2^14, so the sums stay in 32 bits; a whole cluster's
// weights sum to a power of two and its division is a shift.  (Bound by
// reading the level below: 36 us for 81 views of 625 x 434 to 25, 4.8 TB/s; 138 us
// with one sample per thread in 64 bits.)
template <int N>
__global__ __launch_bounds__(kT) void k_enc_filter(const int16_t *below, int16_t *above, EncGeo g, int l) {
  const size_t img = (size_t)3 * g.hp * g.wp, off = ((size_t)blockIdx.x * kT + threadIdx.x) * N;
  const int node = blockIdx.y, c = g.c[l], nx = node % g.lu[l], ny = node / g.lu[l];
  if (off >= img) return;
  int pascal[8] = {1, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int i = 1; i < 8; i++)
    if (i < c)
#pragma unroll
      for (int k = 7; k >= 1; k--) pascal[k] += pascal[k - 1];
  int acc[N] = {}, wsum = 0;
#pragma unroll
  for (int j = 0; j < 8; j++)
    if (j < c && ny * c + j < g.lv[l - 1])
#pragma unroll
      for (int i = 0; i < 8; i++)
        if (i < c && nx * c + i < g.lu[l - 1]) {
          const int w = pascal[i] * pascal[j];
          const Samples<N> s =
              *reinterpret_cast<const Samples<N> *>(below + (size_t)((ny * c + j) * g.lu[l - 1] + nx * c + i) * img + off);
          wsum += w;
#pragma unroll
          for (int k = 0; k < N; k++) acc[k] += w * s.v[k];
        }
  Samples<N> o;
  const bool pow2 = (wsum & (wsum - 1)) == 0;
  const int sh = 31 - __clz(wsum);
#pragma unroll
  for (int k = 0; k < N; k++) {
    const int x = acc[k] + wsum / 2;
    o.v[k] = (int16_t)(pow2 ? x >> sh : (x >= 0 ? x / wsum : -((-x + wsum - 1) / wsum)));   // floor
  }
  *reinterpret_cast<Samples<N> *>(above + (size_t)node * img + off) = o;
}

// The children, on level l, of one (parent, channel, block): residual of each
// against the reconstructed parent, pixel threshold, block-energy threshold,
// quantiser, range code; writes the code table, the zigzag values and the
// reconstruction (rec; null on level 0, which no level reads) and, with sse,
// adds the squared error of the unpadded area to the (child, channel)'s sum.
// What bounds it: the samples read and the zigzag values written.  Lanes take
// consecutive blocks of a row of blocks, so plane rows are read whole; a
// thread keeps the parent's block for all siblings, whose serial numbers
// follow each other, so their values fill a cache line of the table.
// Measured, 9 x 9 x 625 x 434, both levels: 201 us with the squared error (one
// thread per child, channels interleaved over the lanes and a pass of its own
// for the squared error: 734 + 108).
template <int B>
__global__ __launch_bounds__(kT) void k_enc_residual(const int16_t *own_lvl, const int16_t *par_rec, int16_t *rec,
                                                     const int32_t *serial, int8_t *code_tab, uint16_t *zv,
                                                     unsigned long long *sse, int32_t *err, EncGeo g,
                                                     const RangeTab *rt, int l) {
  constexpr int S = B * B;
  typedef Samples<B> Row;
  const int b = blockIdx.x * kT + threadIdx.x, ch = blockIdx.y, parent = blockIdx.z;
  const bool live = b < g.nb;
  const int bb = live ? b : 0, bx = bb % g.nbx, by = bb / g.nbx;
  const int cp = g.c[l + 1], px = parent % g.lu[l + 1], py = parent / g.lu[l + 1];
  const int x1 = min(px * cp + cp, g.lu[l]), y1 = min(py * cp + cp, g.lv[l]);
  const size_t plane = (size_t)g.hp * g.wp, img = 3 * plane;
  const size_t base = (size_t)ch * plane + (size_t)by * B * g.wp + (size_t)bx * B;
  Row par[B];
#pragma unroll
  for (int y = 0; y < B; y++) par[y] = *reinterpret_cast<const Row *>(par_rec + (size_t)parent * img + base + (size_t)y * g.wp);
  // samples of the block inside the image (all of them but at the right and lower edges)
  const int in_x = g.W - bx * B, in_y = g.H - by * B;
  const bool inside = __all(in_x >= B && in_y >= B);
  int s = serial[py * cp * g.lu[l] + px * cp];
  // the next child's block is requested before this one's stores: a wait for
  // loads also waits for the stores issued before them
  Row next[B];
  auto request = [&](int node) {
#pragma unroll
    for (int y = 0; y < B; y++)
      next[y] = *reinterpret_cast<const Row *>(own_lvl + (size_t)node * img + base + (size_t)y * g.wp);
  };
  request(py * cp * g.lu[l] + px * cp);
  for (int ny = py * cp; ny < y1; ny++)
    for (int nx = px * cp; nx < x1; nx++, s++) {
      const int node = ny * g.lu[l] + nx;
      Row own[B];
#pragma unroll
      for (int y = 0; y < B; y++) own[y] = next[y];
      if (nx + 1 < x1) request(node + 1);
      else if (ny + 1 < y1) request((ny + 1) * g.lu[l] + px * cp);
      int32_t v[S];
      int32_t energy = 0;
#pragma unroll
      for (int i = 0; i < S; i++) {
        int32_t x = (int32_t)own[i / B].v[i % B] - (int32_t)par[i / B].v[i % B];
        if (abs(x) < g.pix_thr) x = 0;
        v[i] = x;
        energy += abs(x);
      }
      uint32_t zmax = 0, any = 0;
      if (g.q) {
#pragma unroll
        for (int i = 0; i < S; i++) {
          const int32_t mag = (abs(v[i]) + (1 << (g.q - 1))) >> g.q;
          v[i] = v[i] < 0 ? -mag : mag;
        }
      }
#pragma unroll
      for (int i = 0; i < S; i++) {
        any |= (uint32_t)v[i];
        zmax = max(zmax, zz(v[i]));
      }
      const bool keep = energy > g.blk_thr && any != 0;
      int code = -1;
      if (keep && zmax < (uint32_t)kZMax) code = rt->code[zmax];
      const bool fits = !keep || code >= 0;
      if (live) {
        const size_t key = (size_t)(3 * b + ch) * g.n_srv + s;
        if (!fits) {
          atomicOr(err, 1);
        } else {
          if (keep) {
            uint32_t z[S / 2];
#pragma unroll
            for (int i = 0; i < S / 2; i++) z[i] = zz(v[2 * i]) | zz(v[2 * i + 1]) << 16;
            uint32_t *dst = reinterpret_cast<uint32_t *>(zv + key * S);
            if constexpr (S == 4) {
              *reinterpret_cast<uint2 *>(dst) = make_uint2(z[0], z[1]);
            } else {
#pragma unroll
              for (int i = 0; i < S / 2; i += 4)
                *reinterpret_cast<uint4 *>(dst + i) = make_uint4(z[i], z[i + 1], z[i + 2], z[i + 3]);
            }
          }
          code_tab[key] = (int8_t)code;
        }
      }
      bool range = false;
      unsigned long long e = 0;
#pragma unroll
      for (int y = 0; y < B; y++) {
        Row r;
#pragma unroll
        for (int x = 0; x < B; x++) {
          const int32_t w = (int32_t)par[y].v[x] + (keep ? v[y * B + x] * (1 << g.q) : 0);
          range |= w < -32768 || w > 32767;
          r.v[x] = (int16_t)w;
          const uint32_t d = (uint32_t)abs((int32_t)r.v[x] - (int32_t)own[y].v[x]);   // below 2^16
          if (sse) e += inside || (x < in_x && y < in_y) ? __umul24(d, d) : 0u;
        }
        if (rec && live && fits) *reinterpret_cast<Row *>(rec + (size_t)node * img + base + (size_t)y * g.wp) = r;
      }
      if (range && live && fits) atomicOr(err, 2);
      if (sse) {
        if (!live) e = 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) e += __shfl_xor(e, d);
        if ((threadIdx.x & 63) == 0 && e) atomicAdd(sse + (size_t)node * 3 + ch, e);
      }
    }
}

// words of each group (bitmap, 5-bit codes, payload; 0 for an empty group),
// one group per wave at a time; with hist, also the stored blocks per code, in
// kHistCopies copies that the host adds up (one copy made the workgroups' adds
// wait for each other: 43 us against 12 for 51 k groups)
constexpr int kHistCopies = 32, kHistStride = 32;
__global__ __launch_bounds__(kT) void k_enc_group_words(const int8_t *code_tab, uint32_t *gwords, unsigned long long *hist,
                                                        EncGeo g) {
  // (copies of the histogram, so that lanes that count one code rarely meet)
  constexpr int kCopies = 8;
  __shared__ uint32_t h[lfc::kNumCodes * kCopies];
  const int lane = threadIdx.x & 63, waves = gridDim.x * (kT / 64);
  if (threadIdx.x < lfc::kNumCodes * kCopies) h[threadIdx.x] = 0;
  __syncthreads();
  for (int gi = blockIdx.x * (kT / 64) + (threadIdx.x >> 6); gi < g.ng; gi += waves) {
    const int8_t *ct = code_tab + (size_t)gi * g.n_srv;
    uint32_t present = 0, bits = 0;   // (a group's payload stays below 2^32 bits: 65535 nodes of 768 bits a level)
    for (int s = lane; s < g.n_srv; s += 64)
      if (ct[s] >= 0) {
        present++;
        bits += block_bits_d(ct[s], g.S);
        if (hist) atomicAdd(&h[ct[s] * kCopies + lane % kCopies], 1u);
      }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      present += __shfl_xor(present, d);
      bits += __shfl_xor(bits, d);
    }
    if (lane == 0) gwords[gi] = present ? (uint32_t)g.nbw + (5 * present + 31) / 32 + (bits + 31) / 32 : 0u;
  }
  __syncthreads();
  if (hist && threadIdx.x < lfc::kNumCodes) {
    unsigned long long n = 0;
    for (int k = 0; k < kCopies; k++) n += h[threadIdx.x * kCopies + k];
    if (n) atomicAdd(hist + blockIdx.x % kHistCopies * kHistStride + threadIdx.x, n);
  }
}

// exclusive prefix sum of the group sizes: offsets[0..n], and the total in 64
// bits.  Each workgroup scans `chunk` sizes after summing all those before them
// (at most kScanWgs passes over the sizes, which L2 holds; one workgroup for
// everything took 52 us for 51 k groups, this 16).
constexpr int kScanT = 1024, kScanWgs = 512;
__global__ __launch_bounds__(kScanT) void k_enc_offsets(const uint32_t *gwords, uint32_t *offsets, unsigned long long *total,
                                                        int n, int chunk) {
  __shared__ unsigned long long wsum[kScanT / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t first = (int64_t)blockIdx.x * chunk, last = min((int64_t)n, first + chunk);
  unsigned long long run = 0;
#pragma unroll 8
  for (int64_t i = t; i < first; i += kScanT) run += gwords[i];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) run += __shfl_xor(run, d);
  if (lane == 0) wsum[wave] = run;
  __syncthreads();
  run = 0;
  for (int w = 0; w < kScanT / 64; w++) run += wsum[w];
  for (int64_t base = first; base < last; base += kScanT) {
    const int64_t i = base + t;
    const uint32_t v = i < last ? gwords[i] : 0u;
    unsigned long long incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long u = __shfl_up(incl, d);
      if (lane >= d) incl += u;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned long long at = run + incl - v;
    for (int w = 0; w < kScanT / 64; w++) {
      if (w < wave) at += wsum[w];
      run += wsum[w];
    }
    if (i < last) offsets[i] = (uint32_t)at;
  }
  if (last == n && t == 0) {
    offsets[n] = (uint32_t)run;
    *total = run;
  }
}

// Packing: one wave per group, 64 of its nodes at a time.  A node's range code
// and payload have places in the group's bit stream that follow from the
// stored nodes below it (a ballot and a prefix sum over the wave); its lane
// builds the payload in a 64-bit window and puts whole words into the chunk's
// words in LDS, which the wave then writes in order.  The bit stream's last,
// incomplete word is carried into the next chunk, so every word is written
// once and the output needs no clearing.
// What bounds it: the vector operations of the bit packing.  Measured, 9 x 9 x
// 625 x 434: 59 us (one thread per group, bit by bit in global memory: 1057).
template <int S>
struct PackLds {
  static constexpr int kPayload = 64 * 12 * S / 32 + 2;   // words of 64 blocks (at most 12 bits a value) and a started one
  uint32_t payload[kPayload];
  uint32_t codes[64 * 5 / 32 + 2];
};

// One lane's part of a bit stream in LDS words (zero where nothing is put).
struct BitPut {
  uint32_t *w;      // the word that holds the next bit
  uint64_t acc;     // bits put but not yet in LDS, from that word's bit 0
  uint32_t n;       // their number
  __device__ __forceinline__ BitPut(uint32_t *words, uint32_t pos) : w(words + (pos >> 5)), acc(0), n(pos & 31u) {}
  // at most 32 bits
  __device__ __forceinline__ void put(uint32_t v, uint32_t bits) {
    acc |= (uint64_t)v << n;
    n += bits;
    if (n >= 32) {
      atomicOr(w++, (uint32_t)acc);
      acc >>= 32;
      n -= 32;
    }
  }
  __device__ __forceinline__ void flush() {
    if (n) atomicOr(w, (uint32_t)acc);
  }
};

// A block's BISE payload (digit plane, then the low-bit plane) from its
// zigzag values, two per word.
template <int S>
__device__ __forceinline__ void put_block(BitPut &out, const uint32_t (&z)[S / 2], int code) {
  int kind, m;
  code_km(code, kind, m);
  auto digits = [&](auto glen_, auto radix_, auto full_) {
    constexpr int glen = decltype(glen_)::value, radix = decltype(radix_)::value, full = decltype(full_)::value;
#pragma unroll
    for (int i0 = 0; i0 < S; i0 += glen) {
      constexpr int G = glen;
      const int k = i0 + G <= S ? G : S - i0;
      uint32_t num = 0;
#pragma unroll
      for (int r = G - 1; r >= 0; r--)
        if (r < k) num = num * radix + (((z[(i0 + r) / 2] >> (16 * ((i0 + r) & 1))) & 0xFFFFu) >> m);
      out.put(num, (uint32_t)((full * k + G - 1) / G));
    }
  };
  if (kind == 1) digits(std::integral_constant<int, 5>{}, std::integral_constant<int, 3>{}, std::integral_constant<int, 8>{});
  if (kind == 2) digits(std::integral_constant<int, 3>{}, std::integral_constant<int, 5>{}, std::integral_constant<int, 7>{});
  if (m == 0) return;
  const uint32_t mask = (1u << m) - 1u;
#pragma unroll
  for (int i = 0; i < S / 2; i++) out.put((z[i] & mask) | ((z[i] >> 16) & mask) << m, 2u * (uint32_t)m);   // (m <= 12)
}

template <int B>
__global__ __launch_bounds__(kT) void k_enc_pack(const int8_t *code_tab, const uint16_t *zv, const uint32_t *offsets,
                                                 uint32_t *off_out, uint32_t *srv, EncGeo g) {
  constexpr int S = B * B;
  __shared__ PackLds<S> lds[kT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int gi = (int)(blockIdx.y * gridDim.x + blockIdx.x) * (kT / 64) + wv;   // (at most 2^30 groups)
  if (gi >= g.ng) {
    if (gi == g.ng && lane < 2) srv[offsets[g.ng] + lane] = 0;   // the section's spare words
    if (gi == g.ng && lane == 0) off_out[gi] = offsets[gi];
    return;
  }
  const uint32_t o0 = offsets[gi];
  if (lane == 0) off_out[gi] = o0;   // (the stream's copy)
  if (o0 == offsets[gi + 1]) return;
  PackLds<S> &sm = lds[wv];
  uint32_t *w = srv + o0;
  const int8_t *ct = code_tab + (size_t)gi * g.n_srv;
  // bitmap, and the number of stored nodes
  uint32_t present = 0;
  for (int s0 = 0; s0 < g.n_srv; s0 += 64) {
    const uint64_t m = __ballot(s0 + lane < g.n_srv && ct[min(s0 + lane, g.n_srv - 1)] >= 0);
    if (lane < 2 && s0 / 32 + lane < g.nbw) w[s0 / 32 + lane] = (uint32_t)(m >> (32 * lane));
    present += (uint32_t)__popcll(m);
  }
  // the code section and the payload: next bit of each, and the started word
  uint32_t cpos = 32u * (uint32_t)g.nbw, pos = 32u * ((uint32_t)g.nbw + (5 * present + 31) / 32);
  uint32_t ccarry = 0, carry = 0;
  // the words of a chunk that are complete, to the output; the started one back
  auto write = [&](uint32_t *words, uint32_t first, uint32_t end) {
    const uint32_t n = (end >> 5) - (first >> 5);
    for (uint32_t i = lane; i < n; i += 64) w[(first >> 5) + i] = words[i];
    return words[n];
  };
  for (int s0 = 0; s0 < g.n_srv; s0 += 64) {
    const int s = s0 + lane, code = s < g.n_srv ? ct[s] : -1;
    const uint64_t mask = __ballot(code >= 0);
    if (!mask) continue;
    const uint32_t bits = code >= 0 ? block_bits_d(code, S) : 0u;
    uint32_t incl = bits;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t u = __shfl_up(incl, d);
      if (lane >= d) incl += u;
    }
    const uint32_t all = __shfl(incl, 63), count = (uint32_t)__popcll(mask);
    uint32_t z[S / 2];
    if (code >= 0) {
      const uint32_t *src = reinterpret_cast<const uint32_t *>(zv + ((size_t)gi * g.n_srv + s) * S);
      if constexpr (S == 4) {
        const uint2 v = *reinterpret_cast<const uint2 *>(src);
        z[0] = v.x, z[1] = v.y;
      } else {
#pragma unroll
        for (int i = 0; i < S / 2; i += 4) {
          const uint4 v = *reinterpret_cast<const uint4 *>(src + i);
          z[i] = v.x, z[i + 1] = v.y, z[i + 2] = v.z, z[i + 3] = v.w;
        }
      }
    }
    // the chunk's words, zero but for the started ones
    const uint32_t cw = ((cpos & 31u) + 5u * count) / 32u + 1u, pw = ((pos & 31u) + all) / 32u + 1u;
    if ((uint32_t)lane < cw) sm.codes[lane] = lane == 0 ? ccarry : 0u;
    for (uint32_t i = lane; i < pw; i += 64) sm.payload[i] = i == 0 ? carry : 0u;
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    if (code >= 0) {
      BitPut c(sm.codes, (cpos & 31u) + 5u * (uint32_t)__popcll(mask & ((1ull << lane) - 1ull)));
      c.put((uint32_t)code, 5u);
      c.flush();
      BitPut out(sm.payload, (pos & 31u) + incl - bits);
      put_block<S>(out, z, code);
      out.flush();
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    ccarry = write(sm.codes, cpos, cpos + 5u * count);
    carry = write(sm.payload, pos, pos + all);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    cpos += 5u * count;
    pos += all;
  }
  if (lane == 0 && (cpos & 31u)) w[cpos >> 5] = ccarry;
  if (lane == 1 && (pos & 31u)) w[pos >> 5] = carry;
}

// the top level as the stream stores it: [n_top][nb][3][B*B], one row of a
// block per thread
template <int B>
__global__ __launch_bounds__(kT) void k_enc_top_blocks(const int16_t *top, int16_t *dst, EncGeo g, int n_top) {
  typedef Samples<B> Row;
  const int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (r >= (int64_t)n_top * g.nb * 3 * B) return;
  const int y = (int)(r % B), ch = (int)(r / B % 3);
  const int64_t nb = r / (3 * B);
  const int b = (int)(nb % g.nb), n = (int)(nb / g.nb), bx = b % g.nbx, by = b / g.nbx;
  const size_t plane = (size_t)g.hp * g.wp;
  *reinterpret_cast<Row *>(dst + r * B) =
      *reinterpret_cast<const Row *>(top + ((size_t)n * 3 + ch) * plane + (size_t)(by * B + y) * g.wp + bx * B);
}

constexpr int kWordsWgs = 2048;   // workgroups of the group sizes (each adds its histogram once)

lfc_status launched(const char *what) {
  const hipError_t he = hipGetLastError();
  if (he != hipSuccess) return lfc::fail(LFC_E_HIP, std::string("lfc_encode_gpu: ") + what + ": " + hipGetErrorString(he));
  return LFC_OK;
}

// Device scratch of one encode, given back on every path (and on its stream, so
// after the work that uses it).
struct Scratch {
  hipStream_t s;
  void *p = nullptr;
  explicit Scratch(hipStream_t stream) : s(stream) {}
  ~Scratch() {
    if (p) (void)hipFreeAsync(p, s);
  }
  Scratch(const Scratch &) = delete;
  lfc_status alloc(size_t bytes) {
    if (lfc::scratch_alloc(&p, std::max<size_t>(bytes, 256), s) != LFC_OK)
      return lfc::fail(LFC_E_NOMEM, "lfc_encode_gpu: device memory");
    return LFC_OK;
  }
};

// Waits for the stream at the end of its scope: declared after host memory that a
// copy on it reads, so that a return before the call's own wait does not free
// that memory under the copy.
struct WaitOnReturn {
  hipStream_t s;
  bool pending = true;
  ~WaitOnReturn() {
    if (pending) (void)hipStreamSynchronize(s);
  }
};

// Parts of one allocation, 256-byte aligned.
struct Parts {
  size_t bytes = 0;
  template <typename T>
  size_t add(size_t n) {
    const size_t at = bytes;
    bytes = (at + n * sizeof(T) + 255) & ~(size_t)255;
    return at;
  }
};

lfc_status encode_gpu(const uint8_t *d_rgb, const lfc_params *p, void **stream_out, size_t *bytes_out,
                      lfc_encode_stats *stats, hipStream_t s) {
  using namespace lfc;
  if (!d_rgb || !p || (!stream_out) != (!bytes_out)) return fail(LFC_E_INVALID, "lfc_encode_gpu: null argument");
  if (stream_out) {
    *stream_out = nullptr;
    *bytes_out = 0;
  }
  Geometry geo;
  std::string why;
  if (make_geometry(*p, geo, &why) != LFC_OK) return fail(LFC_E_INVALID, "lfc_encode_gpu: " + why);
  const int nv = geo.nv(), L = geo.L, S = geo.S;
  {
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    const size_t need = (size_t)nv * geo.H * geo.W * 3;
    if (hipMemGetAddressRange(&base, &size, const_cast<uint8_t *>(d_rgb)) != hipSuccess || !base ||
        (size_t)(d_rgb - static_cast<const uint8_t *>(base)) + need > size) {
      (void)hipGetLastError();
      return fail(LFC_E_INVALID, "lfc_encode_gpu: d_rgb is not device memory of [V][U][H][W][3] bytes");
    }
  }
  // views and the nodes of a level are a grid dimension of launches below; the
  // bounds of three rows and three views to one are the entry point's own
  bool fits = 3 * geo.hp <= 65535 && nv * 3 <= 65535;
  for (int l = 0; l < L; l++) fits &= geo.lu[l] * geo.lv[l] <= 65535;
  if (!fits) return fail(LFC_E_UNSUPPORTED, "lfc_encode_gpu: light field too large for the GPU encoder's grids");
  const uint32_t mask = p->range_mask ? p->range_mask : kAllCodes;
  EncGeo g{};
  g.U = geo.U, g.V = geo.V, g.W = geo.W, g.H = geo.H, g.wp = geo.wp, g.hp = geo.hp, g.B = geo.B, g.S = S, g.L = L;
  g.q = geo.q, g.nbx = geo.nbx, g.nb = geo.nb, g.ng = geo.ng, g.n_srv = geo.n_srv, g.nbw = geo.nbw;
  for (int l = 0; l < kMaxLevels; l++) g.lu[l] = geo.lu[l], g.lv[l] = geo.lv[l], g.c[l] = geo.c[l];
  g.pix_thr = p->pix_threshold, g.blk_thr = p->blk_threshold;
  RangeTab rt;
  {
    std::pair<int, int> r[kNumCodes];   // allowed ranges by increasing number of values
    int n = 0;
    for (int k = 0; k < kNumCodes; k++)
      if ((mask >> k) & 1u) r[n++] = {k < 12 ? 2 << k : (k < 19 ? 3 << (k - 12) : 5 << (k - 19)), k};
    std::sort(r, r + n);
    for (int z = 0, i = 0; z < kZMax; z++) {
      while (i < n && r[i].first <= z) i++;
      rt.code[z] = i < n ? (int8_t)r[i].second : (int8_t)-1;
    }
  }
  TreeTables tt;
  build_tree_tables(geo, tt);
  const size_t plane = (size_t)geo.hp * geo.wp, img = 3 * plane;
  const size_t nsg = (size_t)geo.ng * geo.n_srv;
  // one scratch: the levels, the reconstructions between the top and level 0,
  // the tables; and the small results, copied to the host together: the
  // offsets' total, the stored blocks per code, the error flags, the squared
  // errors
  const size_t at_hist = 1, at_err = at_hist + kHistCopies * kHistStride, at_sse = at_err + 1,
               n_small = at_sse + (size_t)nv * 3;
  Parts parts;
  std::vector<size_t> p_lvl(L), p_rec(L), p_serial(L);
  size_t n_serial = 0;
  for (int l = 0; l < L; l++) {
    const size_t nodes = (size_t)geo.lu[l] * geo.lv[l];
    p_lvl[l] = parts.add<int16_t>(nodes * img);
    if (l > 0 && l < L - 1) p_rec[l] = parts.add<int16_t>(nodes * img);
    if (l < L - 1) p_serial[l] = n_serial, n_serial += nodes;
  }
  const size_t p_code = parts.add<int8_t>(nsg), p_zv = parts.add<uint16_t>(nsg * S), p_gw = parts.add<uint32_t>(geo.ng),
               p_off = parts.add<uint32_t>((size_t)geo.ng + 1), p_small = parts.add<unsigned long long>(n_small),
               p_host = parts.add<char>(sizeof(RangeTab) + 4 * n_serial);
  Scratch ws(s);
  if (lfc_status st = ws.alloc(parts.bytes)) return st;
  char *base = static_cast<char *>(ws.p);
  std::vector<int16_t *> lvl(L), rec(L, nullptr);
  std::vector<const int32_t *> serial(L, nullptr);
  // the host's tables in one copy: the range table, the serial numbers
  std::vector<char> host(sizeof(RangeTab) + 4 * n_serial);
  std::memcpy(host.data(), &rt, sizeof rt);
  for (int l = 0; l < L; l++) {
    lvl[l] = reinterpret_cast<int16_t *>(base + p_lvl[l]);
    if (l > 0 && l < L - 1) rec[l] = reinterpret_cast<int16_t *>(base + p_rec[l]);
    if (l < L - 1) {
      const size_t at = sizeof(RangeTab) + 4 * p_serial[l];
      std::memcpy(host.data() + at, tt.serial[l].data(), 4 * tt.serial[l].size());
      serial[l] = reinterpret_cast<const int32_t *>(base + p_host + at);
    }
  }
  WaitOnReturn tables{s};
  if (hipMemcpyAsync(base + p_host, host.data(), host.size(), hipMemcpyHostToDevice, s) != hipSuccess)
    return fail(LFC_E_HIP, "lfc_encode_gpu: copy of the tables");
  const RangeTab *d_rt = reinterpret_cast<const RangeTab *>(base + p_host);
  int8_t *code_tab = reinterpret_cast<int8_t *>(base + p_code);
  uint16_t *zv = reinterpret_cast<uint16_t *>(base + p_zv);
  uint32_t *gw = reinterpret_cast<uint32_t *>(base + p_gw), *d_off = reinterpret_cast<uint32_t *>(base + p_off);
  unsigned long long *small = reinterpret_cast<unsigned long long *>(base + p_small);
  rec[L - 1] = lvl[L - 1];   // the top level is stored losslessly
  if (hipMemsetAsync(small, 0, 8 * n_small, s) != hipSuccess ||
      hipMemsetAsync(code_tab, 0xFF, std::max<size_t>(nsg, 1), s) != hipSuccess)
    return fail(LFC_E_HIP, "lfc_encode_gpu: clearing tables");
  int32_t *err = reinterpret_cast<int32_t *>(small + at_err);

  // samples per thread of the kernels that walk plane rows: 16 bytes where the
  // padded width allows
  auto by_width = [&](auto f) {
    if (geo.wp % 8 == 0) f(std::integral_constant<int, 8>{});
    else if (geo.wp % 4 == 0) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 2>{});
  };
  auto by_block = [&](auto f) {
    if (geo.B == 8) f(std::integral_constant<int, 8>{});
    else if (geo.B == 4) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 2>{});
  };
  // Stage I: level 0, then the key views of every level above
  by_width([&](auto n) {
    constexpr int N = decltype(n)::value < 4 ? decltype(n)::value : 4;
    hipLaunchKernelGGL(k_enc_level0<N>, dim3((unsigned)((plane / N + kT - 1) / kT), nv), dim3(kT), 0, s, d_rgb, lvl[0], g);
  });
  if (lfc_status st = launched("level 0")) return st;
  for (int l = 1; l < L; l++) {
    by_width([&](auto n) {
      constexpr int N = decltype(n)::value;
      hipLaunchKernelGGL(k_enc_filter<N>, dim3((unsigned)((img / N + kT - 1) / kT), geo.lu[l] * geo.lv[l]), dim3(kT), 0, s,
                         (const int16_t *)lvl[l - 1], lvl[l], g, l);
    });
    if (lfc_status st = launched("key-view filter")) return st;
  }
  // Stage II: residual levels from the top down against the reconstruction
  for (int l = L - 2; l >= 0; l--) {
    by_block([&](auto n) {
      constexpr int B = decltype(n)::value;
      hipLaunchKernelGGL(k_enc_residual<B>, dim3((unsigned)((geo.nb + kT - 1) / kT), 3, geo.lu[l + 1] * geo.lv[l + 1]),
                         dim3(kT), 0, s, (const int16_t *)lvl[l], (const int16_t *)rec[l + 1], rec[l],
                         serial[l], code_tab, zv, stats && l == 0 ? small + at_sse : nullptr, err, g, d_rt, l);
    });
    if (lfc_status st = launched("residuals")) return st;
  }
  // Stage III: group sizes -> offsets
  if (L > 1) {
    hipLaunchKernelGGL(k_enc_group_words, dim3(std::min((geo.ng + kT / 64 - 1) / (kT / 64), kWordsWgs)), dim3(kT), 0, s,
                       (const int8_t *)code_tab, gw, stats ? small + at_hist : nullptr, g);
    if (lfc_status st = launched("group sizes")) return st;
    const int chunk = std::max(kScanT, (geo.ng + kScanWgs - 1) / kScanWgs);
    hipLaunchKernelGGL(k_enc_offsets, dim3((geo.ng + chunk - 1) / chunk), dim3(kScanT), 0, s, (const uint32_t *)gw, d_off,
                       small, geo.ng, chunk);
    if (lfc_status st = launched("group offsets")) return st;
  } else if (hipMemsetAsync(d_off, 0, 4ull * (geo.ng + 1), s) != hipSuccess) {
    return fail(LFC_E_HIP, "lfc_encode_gpu: clearing the offsets");
  }
  std::vector<unsigned long long> hs(n_small);
  if (hipMemcpyAsync(hs.data(), small, 8 * n_small, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return fail(LFC_E_HIP, "lfc_encode_gpu: synchronize");
  tables.pending = false;
  const int32_t herr = (int32_t)hs[at_err];
  if (herr & 1) return fail(LFC_E_RANGE, "lfc_encode_gpu: a residual block needs a BISE range the mask does not allow");
  if (herr & 2) return fail(LFC_E_RANGE, "lfc_encode_gpu: a reconstructed sample leaves int16");
  if (stats) {
    std::vector<double> se(hs.begin() + (ptrdiff_t)at_sse, hs.end());
    encode_stats_from_sse(se, nv, geo.W, geo.H, stats);
    stats->present_blocks = 0;
    for (int k = 0; k < kNumCodes; k++) {
      stats->code_hist[k] = 0;
      for (int c = 0; c < kHistCopies; c++) stats->code_hist[k] += hs[at_hist + c * kHistStride + k];
      stats->present_blocks += stats->code_hist[k];
    }
  }
  const uint64_t acc = hs[0];
  if (acc > 0xFFFFFFF0ull) return fail(LFC_E_RANGE, "lfc_encode_gpu: stream exceeds 2^32 words");
  const uint64_t srv_words = acc + 2;
  const uint64_t rkv_bytes = (uint64_t)geo.n_top * geo.nb * 3 * S * 2;
  const uint64_t rkv_off = kHeaderBytes, off_off = rkv_off + rkv_bytes, srv_off = off_off + 4ull * (geo.ng + 1);
  if (stats) stats->stream_bytes = srv_off + 4 * srv_words;
  if (!stream_out) return LFC_OK;
  // the whole stream is laid out on the device and copied once
  const size_t bytes = srv_off + 4 * srv_words;
  Scratch ds(s);
  if (lfc_status st = ds.alloc(bytes)) return st;
  char *stream = static_cast<char *>(ds.p);
  by_block([&](auto n) {
    constexpr int B = decltype(n)::value;
    // (one wave more than groups: it writes the last offset and the section's two
    // spare words; a grid dimension holds fewer than 2^32 threads)
    const unsigned wgs = (unsigned)((geo.ng + kT / 64) / (kT / 64)), row = std::min(wgs, 1u << 22);
    hipLaunchKernelGGL(k_enc_pack<B>, dim3(row, (wgs + row - 1) / row), dim3(kT), 0, s,
                       (const int8_t *)code_tab, (const uint16_t *)zv, (const uint32_t *)d_off,
                       reinterpret_cast<uint32_t *>(stream + off_off), reinterpret_cast<uint32_t *>(stream + srv_off), g);
    const int64_t rows = (int64_t)geo.n_top * geo.nb * 3 * B;
    hipLaunchKernelGGL(k_enc_top_blocks<B>, dim3((unsigned)((rows + kT - 1) / kT)), dim3(kT), 0, s,
                       (const int16_t *)lvl[L - 1], reinterpret_cast<int16_t *>(stream + rkv_off), g, geo.n_top);
  });
  if (lfc_status st = launched("packing")) return st;
  uint8_t *out = static_cast<uint8_t *>(stream_alloc(bytes));
  if (!out) return fail(LFC_E_NOMEM, "lfc_encode_gpu: out of host memory");
  put_stream_header(out, geo, *p, mask, rkv_off, off_off, srv_off);
  if (hipMemcpyAsync(out + kHeaderBytes, stream + kHeaderBytes, bytes - kHeaderBytes, hipMemcpyDeviceToHost, s) !=
          hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    stream_free(out);
    return fail(LFC_E_HIP, "lfc_encode_gpu: copy of the stream");
  }
  *stream_out = out;
  *bytes_out = bytes;
  return LFC_OK;
}

}  // namespace

extern "C" lfc_status lfc_encode_gpu(const uint8_t *d_rgb, const lfc_params *p, void **stream_out, size_t *bytes_out,
                                     lfc_encode_stats *stats, hipStream_t s) {
  try {
    return encode_gpu(d_rgb, p, stream_out, bytes_out, stats, s);
  } catch (const std::bad_alloc &) {
    return lfc::fail(LFC_E_NOMEM, "lfc_encode_gpu: out of host memory");
  }
}
