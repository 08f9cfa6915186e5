// FNV-1a-64 of many items at once on gfx950, staged through LDS with coalesced
// loads: one lane per item running the serial byte chain (wave_fnv_t), or many
// lanes per item (wave_fnv_par).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fnv_rules.hpp"
#include "gsys_device.hpp"

namespace gsys_k {

using namespace gsys;

// h * 0x100000001b3 mod 2^64 written as (h << 40) + h * 0x1b3.
__device__ __forceinline__ uint64_t fnv_byte(uint64_t h, uint32_t byte) {
  h ^= byte;
  return (h << 40) + h * 0x1b3ull;
}

__device__ __forceinline__ uint64_t fnv_word(uint64_t h, uint32_t w, int nbytes) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < nbytes) h = fnv_byte(h, (w >> (8 * j)) & 0xffu);
  return h;
}

__device__ __forceinline__ uint64_t fnv_word4(uint64_t h, uint32_t w) {
  h = fnv_byte(h, w & 0xffu);
  h = fnv_byte(h, (w >> 8) & 0xffu);
  h = fnv_byte(h, (w >> 16) & 0xffu);
  return fnv_byte(h, w >> 24);
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
  uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64);
  return ((uint64_t)hi << 32) | lo;
}

// Per step every row (item) of the wave contributes CH contiguous bytes:
// CH/16 lanes x 16 B per row, 1024/CH rows per load instruction, CH/16
// instructions for the 64 rows.  The next step's loads are issued before the
// current step is hashed, so the host-link round trip overlaps the FNV chain.
// Rows of a wavefront are consecutive items, so row r starts at
// row0 + r * item_bytes; each row's byte count sits in LDS next to the tile.
// The loads are global and the tile accesses LDS (not flat) instructions, so
// the LDS reads of the hashing loop never wait for the loads in flight.
template <uint32_t CH>
struct Tile {
  static constexpr uint32_t kLanesPerRow = CH / 16;
  static constexpr uint32_t kRowsPerLoad = 64 / kLanesPerRow;
  static constexpr uint32_t kLoads = 64 / kRowsPerLoad;
  static constexpr uint32_t kRowStride = CH + 16;  // pad: conflict-free 16-byte LDS reads
  static constexpr uint32_t kBytes = 64 * kRowStride + 64 * 4;  // + each row's byte count
};

// 256-byte rows for work-groups of up to 256 work-items; 128-byte rows for
// larger work-groups (fewer registers per lane are available there).  Rows of
// 256 bytes read host staging at the link's rate (57 GB/s measured on MI355X
// against 42 GB/s for 128-byte rows): each row's request covers two
// 128-byte lines.
template <uint32_t WGMAX>
constexpr uint32_t chunk_for() { return WGMAX <= 256 ? 256u : 128u; }

// All 64 lanes of the wave call this.  Lane l hashes `nbytes` bytes of the item
// at address row(l).  `tile` is this wave's LDS tile (Tile<CH>::kBytes).
template <uint32_t CH, class Row>
__device__ __forceinline__ uint64_t wave_fnv_rows(Row row, uint32_t nbytes, uint32_t item_bytes,
                                                  uint8_t* tile_generic) {
  using T = Tile<CH>;
  lptr_t<uint8_t> tile = lp(tile_generic);
  const uint32_t lane = lane_id();
  const uint32_t col = lane % T::kLanesPerRow;
  const uint32_t rsub = lane / T::kLanesPerRow;
  uint32_t maxlen = nbytes;
  for (int o = 32; o > 0; o >>= 1) maxlen = max(maxlen, (uint32_t)__shfl_xor((int)maxlen, o, 64));
  if (maxlen > item_bytes) maxlen = item_bytes;
  lptr_t<uint32_t> rlen = reinterpret_cast<lptr_t<uint32_t>>(tile + 64 * T::kRowStride);
  rlen[lane] = nbytes;
  __builtin_amdgcn_wave_barrier();
  uint64_t h = 0xcbf29ce484222325ull;
  u32x4 v[T::kLoads];
  auto load = [&](uint32_t off) {
#pragma unroll
    for (uint32_t k = 0; k < T::kLoads; ++k) {
      const uint32_t r = k * T::kRowsPerLoad + rsub;
      v[k] = u32x4{0, 0, 0, 0};
      // a row is read only where it holds bytes, inside its own item slot
      if (off < rlen[r] && off + col * 16 < item_bytes)
        v[k] = ldg16(row(r) + off + col * 16);
    }
  };
  if (maxlen) load(0);
  for (uint32_t off = 0; off < maxlen; off += CH) {
#pragma unroll
    for (uint32_t k = 0; k < T::kLoads; ++k) {
      const uint32_t r = k * T::kRowsPerLoad + rsub;
      *reinterpret_cast<lptr_t<u32x4>>(tile + r * T::kRowStride + col * 16) = v[k];
    }
    __builtin_amdgcn_wave_barrier();
    if (off + CH < maxlen) load(off + CH);  // prefetch the next step
    lptr_t<const uint8_t> mine = tile + lane * T::kRowStride;
    if (__ballot(off < nbytes && off + CH > nbytes) == 0) {
      if (off + CH <= nbytes) {
#pragma unroll 2
        for (uint32_t q = 0; q < CH / 16; ++q) {
          const u32x4 w = *reinterpret_cast<lptr_t<const u32x4>>(mine + q * 16);
          h = fnv_word4(h, w.x);
          h = fnv_word4(h, w.y);
          h = fnv_word4(h, w.z);
          h = fnv_word4(h, w.w);
        }
      }
    } else if (off < nbytes) {
      // some lanes are at their items' ends: all go on in 16-byte pieces, and
      // those take the rest of the last one byte by byte.  (With the others
      // waiting for a byte-wise loop over all that is left, lengths up to 512
      // took 60 ns a byte.)
      const uint32_t left = min(CH, nbytes - off);
      uint32_t q = 0;
      for (; q + 16 <= left; q += 16) {
        const u32x4 w = *reinterpret_cast<lptr_t<const u32x4>>(mine + q);
        h = fnv_word4(h, w.x);
        h = fnv_word4(h, w.y);
        h = fnv_word4(h, w.z);
        h = fnv_word4(h, w.w);
      }
      if (q < left) {
        const u32x4 w = *reinterpret_cast<lptr_t<const u32x4>>(mine + q);
        for (uint32_t j = 0; q + j < left; ++j)
          h = fnv_byte(h, (w[j >> 2] >> (8 * (j & 3u))) & 0xffu);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  return h;
}

// The same for items that follow each other from row0 on.
template <uint32_t CH>
__device__ __forceinline__ uint64_t wave_fnv_t(uint64_t row0, uint32_t nbytes,
                                               uint32_t item_bytes, uint8_t* tile) {
  return wave_fnv_rows<CH>([=](uint32_t r) { return row0 + (uint64_t)r * item_bytes; }, nbytes,
                           item_bytes, tile);
}

// ---------------------------------------------------------------------------
// FNV-1a-64 of one item by many lanes.
//
// h' = (h ^ b) * p is serial, but its parts are not.  Let s be the low byte of
// h and x = s ^ b; the XOR adds x - s to h, so
//   h_n = p^n h_0 + sum_i (x_i - s_i) p^(n - i)   (mod 2^64),
// a plain weighted sum once the low bytes are known, and those follow their
// own recurrence s' = 179 x mod 256 (179 = p mod 256).  Bit j of 179 x is bit
// j of x XOR a function of x's lower bits, so with the bits below j known at
// every position, bit j of all the s is a running XOR along the item: eight
// running XORs, one per bit, each a parallel prefix.
//
// A lane holds 128 consecutive bytes, four to a 32-bit word and 32 words, as
// eight bit planes of four words: bit w of plane word t is the bit of byte
// 4 w + t.  A plane's running XOR takes three XORs down the four words, a
// five-step prefix in one word and one ballot across the lanes.  The weighted
// sum goes to the matrix cores: int8 MFMAs of the x (and of the s, subtracted)
// with the eight balanced base-256 digits of the powers of p; one column sums
// 512 bytes.  Bytes past an item's end are zeros: a zero byte multiplies h by
// p, which the inverse of p undoes.
//
// Bound by vector-ALU issue: about 780 instructions and 16 MFMAs per 8 KiB step of
// a wavefront (26 cycles per byte and lane; the serial chain takes 32), but a
// 4 KiB item takes half a step instead of the chain's 61 us.  Measured: 50,000
// items of 4 KiB in HBM 106 -> 60 us (3.4 TB/s), 200 of 1 MiB 15.4 -> 0.27 ms,
// a kernel that reads 64 of 4 KiB by one list call and hashes them in one
// work-group of eight wavefronts 85 -> 42 us.

constexpr uint64_t kFnvPrime = 0x100000001b3ull;
constexpr uint64_t kFnvBasis = 0xcbf29ce484222325ull;
constexpr uint32_t kColBytes = 4 * kSegBytes;     // summed by one MFMA column
constexpr uint32_t kSegStride = kSegBytes + 16;   // in LDS: conflict-free 16-byte reads
// Wave tile: the step's bytes, then the byte counts of two groups of items.
constexpr uint32_t kParTile = 64 * kSegStride + 2 * 8 * 4;

struct FnvWeights {
  // [t * 2 + half][lane][register]: four digits of one plane per register
  uint32_t a[8][64][4];
  uint64_t col[16];    // p^(512 k)
  uint64_t seg[8];     // p^(128 * 2^k)
  uint64_t inv[24];    // p^-(2^k)
};
constexpr FnvWeights fnv_weights() {
  FnvWeights w{};
  uint64_t pw[kColBytes + 1] = {};
  pw[0] = 1;
  for (uint32_t i = 1; i <= kColBytes; ++i) pw[i] = pw[i - 1] * kFnvPrime;
  uint8_t digit[kColBytes + 1][8] = {};
  for (uint32_t i = 0; i <= kColBytes; ++i) {
    uint64_t r = pw[i];
    for (uint32_t m = 0; m < 8; ++m) {
      digit[i][m] = (uint8_t)r;
      r = (r >> 8) + ((r >> 7) & 1u);  // digits 128..255 stand for -128..-1
    }
  }
  for (uint32_t op = 0; op < 8; ++op)
    for (uint32_t lane = 0; lane < 64; ++lane)
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t m = lane & 15, g = lane >> 4, t = op >> 1, half = op & 1;
        uint32_t v = 0;
        if (m < 8)
          for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t o = g * kSegBytes + 4 * (8 * c + 4 * half + q) + t;
            v |= (uint32_t)digit[kColBytes - o][m] << (8 * c);
          }
        w.a[op][lane][q] = v;
      }
  w.col[0] = 1;
  for (uint32_t k = 1; k < 16; ++k) w.col[k] = w.col[k - 1] * pw[kColBytes];
  w.seg[0] = pw[kSegBytes];
  for (uint32_t k = 1; k < 8; ++k) w.seg[k] = w.seg[k - 1] * w.seg[k - 1];
  uint64_t iv = kFnvPrime;  // Newton: p * iv = 1 mod 2^64
  for (int k = 0; k < 6; ++k) iv *= 2 - kFnvPrime * iv;
  w.inv[0] = iv;
  for (uint32_t k = 1; k < 24; ++k) w.inv[k] = w.inv[k - 1] * w.inv[k - 1];
  return w;
}
static __device__ const FnvWeights fnv_w = fnv_weights();

typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void opaque(uint32_t& v) { asm("" : "+v"(v)); }

// Three-input operations, one instruction each (the compiler does not find
// all of them by itself).  bfi: a where m is set, b elsewhere.
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_bitop3_b32(m, a, b, 0xca);
}

// 8 x 8 bit transpose in every byte column: bit j of byte c of a[r] <-> bit r
// of byte c of a[j].  A step exchanges the fields m of one row with the fields
// ~m of the row s below; the lower row is left rotated by s, so that one
// rotation serves both rows.  Rows of a pair always have the same rotation;
// row r ends with r, which one rotation each takes out: 43 instructions, 48
// with two shifts a pair (50,000 items of 4 KiB in HBM 60.8 -> 59.2 us).
__device__ __forceinline__ uint32_t rotl(uint32_t v, uint32_t s) {
  return __builtin_amdgcn_alignbit(v, v, (32 - s) & 31);
}
__device__ __forceinline__ void transpose_bits(uint32_t (&a)[8]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t s = 1u << k, m = k == 0 ? 0x55555555u : k == 1 ? 0x33333333u : 0x0f0f0f0fu;
#pragma unroll
    for (uint32_t r = 0; r < 8; ++r)
      if (!(r & s)) {
        const uint32_t rot = r & (s - 1u);  // of both rows
        const uint32_t mr = rot ? (m << rot) | (m >> (32 - rot)) : m;
        const uint32_t lo = a[r], hi = rotl(a[r + s], s);
        a[r] = bfi(mr, lo, hi);
        a[r + s] = bfi(mr, hi, lo);
      }
  }
#pragma unroll
  for (uint32_t r = 1; r < 8; ++r) a[r] = rotl(a[r], 32 - r);
}

__device__ __forceinline__ uint32_t maj(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xe8);
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

template <int ctrl>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, ctrl, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), ctrl, 0xf, 0xf, true);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_xor64(uint64_t v, int m) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m, 64);
  const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m, 64);
  return ((uint64_t)hi << 32) | lo;
}

// The sum of the item's (x - s) p^(bytes to the end of its slot of 128 << ll
// bytes in this step), in every lane of the item.  w: the lane's 128 bytes;
// ent: low byte of the item's hash before the step; before: lanes holding
// earlier bytes of the same item; wt: the weights.
__device__ __forceinline__ uint64_t par_step(uint32_t (&w)[32], uint32_t ent, uint64_t before,
                                             const i32x4 (&wt)[8], uint64_t colw, uint32_t ll) {
  // bytes to (t, r): byte c of b[t][r] is byte t of word 8 c + r
  uint32_t b[4][8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t p0 = __builtin_amdgcn_perm(w[8 + r], w[r], 0x05010400u);
    const uint32_t p1 = __builtin_amdgcn_perm(w[8 + r], w[r], 0x07030602u);
    const uint32_t p2 = __builtin_amdgcn_perm(w[24 + r], w[16 + r], 0x05010400u);
    const uint32_t p3 = __builtin_amdgcn_perm(w[24 + r], w[16 + r], 0x07030602u);
    b[0][r] = __builtin_amdgcn_perm(p2, p0, 0x05040100u);
    b[1][r] = __builtin_amdgcn_perm(p2, p0, 0x07060302u);
    b[2][r] = __builtin_amdgcn_perm(p3, p1, 0x05040100u);
    b[3][r] = __builtin_amdgcn_perm(p3, p1, 0x07060302u);
  }
  // The scheduling barriers and opaque values keep one stage's temporaries
  // from overlapping the next one's: without them the compiler regroups the
  // XORs and interleaves the stages until the registers spill.
  uint32_t x[4][8];  // planes of b, then of x
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      opaque(b[t][r]);
      x[t][r] = b[t][r];
    }
    transpose_bits(x[t]);
#pragma unroll
    for (int r = 0; r < 8; ++r) opaque(x[t][r]);
  }
  // 179 x = y + 16 y + 128 x with y = x + 2 x: carries cy of the first sum, cz
  // of the second
  uint32_t y[4][8], cy[4], cz[4];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    uint32_t gj[4], v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (j == 0) gj[t] = 0;
      if (j == 1) gj[t] = x[t][0];
      if (j == 2 || j == 3) gj[t] = x[t][j - 1] ^ cy[t];
      if (j >= 4) gj[t] = xor3(x[t][j - 1], cy[t], y[t][j - 4]);
      if (j == 5 || j == 6) gj[t] ^= cz[t];
      if (j == 7) gj[t] = xor3(gj[t], cz[t], x[t][0]);
      v[t] = j == 0 ? (t ? x[t][j] ^ v[t - 1] : x[t][j])
                    : t ? xor3(x[t][j], gj[t], v[t - 1]) : x[t][j] ^ gj[t];
    }
    uint32_t run = v[3];
    run ^= run << 1;
    run ^= run << 2;
    run ^= run << 4;
    run ^= run << 8;
    run ^= run << 16;
    const uint64_t odd = __ballot((int32_t)run < 0) & before;
    const uint32_t par = (uint32_t)__popcll(odd) ^ (ent >> j);
    const uint32_t in = xor3(run, v[3], 0u - (par & 1u));  // bit j of s before word w
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      x[t][j] = j == 0 ? v[t] ^ in : xor3(v[t], in, gj[t]);
      if (j == 0) y[t][0] = x[t][0];
      if (j == 1) y[t][1] = x[t][1] ^ x[t][0];
      if (j >= 2 && j < 7) y[t][j] = xor3(x[t][j], x[t][j - 1], cy[t]);
      if (j >= 4 && j < 7)
        cz[t] = j >= 5 ? maj(y[t][j], y[t][j - 4], cz[t]) : y[t][j] & y[t][j - 4];
      if (j >= 1 && j < 7)
        cy[t] = j >= 2 ? maj(x[t][j], x[t][j - 1], cy[t]) : x[t][j] & x[t][j - 1];
      opaque(x[t][j]);
      if (j < 4) opaque(y[t][j]);
      if (j >= 1 && j < 7) opaque(cy[t]);
      if (j >= 4 && j < 7) opaque(cz[t]);
    }
  }
  // back to bytes, as signed numbers 128 lower (the sums cancel the offset)
  i32x4 dx = {0, 0, 0, 0}, ds = {0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    __builtin_amdgcn_sched_barrier(0);
    x[t][7] = ~x[t][7];
    transpose_bits(x[t]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      i32x4 bx, bs;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bx[q] = (int)x[t][4 * h + q];
        bs[q] = (int)(x[t][4 * h + q] ^ b[t][4 * h + q]);
      }
      const i32x4 a = wt[2 * t + h];
      dx = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bx, dx, 0, 0, 0);
      ds = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bs, ds, 0, 0, 0);
    }
  }
  // lanes 0..15 hold digits 0..3 of their column's sum, lanes 16..31 digits
  // 4..7, the others zeros
  int64_t u = 0;
#pragma unroll
  for (int i = 3; i >= 0; --i) u = (u << 8) + (int64_t)(dx[i] - ds[i]);
  uint64_t sum = (lane_id() & 16u) ? (uint64_t)u << 32 : (uint64_t)u;
  sum *= colw;
  sum += shfl_xor64(sum, 16);
  sum += shfl_xor64(sum, 32);
  sum += dpp64<0xb1>(sum);               // lane ^ 1
  if (ll > 3) sum += dpp64<0x4e>(sum);   // lane ^ 2
  if (ll > 4) sum += dpp64<0x141>(sum);  // the other four of eight
  if (ll > 5) sum += dpp64<0x140>(sum);  // the other eight of sixteen
  return sum;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// All 64 lanes of the wavefront call this.  Hashes groups of
// par_items(item_bytes) consecutive items: the first group's are from `first`
// on, and after the one at i comes next(i)'s (the same in every lane), until
// that is `cnt` or more; items from cnt on are not there.  Item i's bytes start
// at row0 + i * item_bytes and it has len_of(i) of them (at most item_bytes, a
// multiple of 16 and more than kParMinItem); len0 is the length of item first +
// lane, in the lanes below par_items.  done(i, h) is called by one lane per
// item.  `tile`: this wavefront's kParTile bytes of LDS.  The next step's bytes
// are loaded while this one is hashed, and the weights stay in registers (256
// per lane, so work-groups of up to 512 work-items).
template <class LenOf, class Next, class Done>
__device__ __forceinline__ void wave_fnv_par(uint64_t row0, uint32_t item_bytes, uint64_t first,
                                             uint32_t len0, uint64_t cnt, uint8_t* tile_generic,
                                             LenOf len_of, Next next, Done done) {
  first = uniform64(first);
  cnt = uniform64(cnt);
  row0 = uniform64(row0);
  if (first >= cnt) return;
  lptr_t<uint8_t> tile = lp(tile_generic);
  lptr_t<uint32_t> rlen = reinterpret_cast<lptr_t<uint32_t>>(tile + 64 * kSegStride);
  const uint32_t lane = lane_id();
  const uint32_t ll = par_lanes_log2(item_bytes), items = 64u >> ll;
  const uint32_t n = lane & 15u, g = lane >> 4, seg = 4 * n + g;
  // lanes with earlier bytes of the same item: the item's columns before this
  // one, then this column's earlier quarters
  const uint32_t col = n & ((16u >> (6 - ll)) - 1u);
  const uint64_t colm = (uint64_t)((1u << n) - (1u << (n - col)));
  uint64_t before = colm * 0x0001000100010001ull;
  for (uint32_t k = 0; k < 3; ++k)
    if (k < g) before |= 1ull << (16 * k + n);
  const uint64_t colw = fnv_w.col[(16u >> (6 - ll)) - 1u - col];
  const uint64_t slotw = fnv_w.seg[ll];
  const uint64_t wbase = (uint64_t)&fnv_w.a[0][lane][0];
  i32x4 wt[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) wt[k] = *gp<const i32x4>(wbase + k * sizeof fnv_w.a[0]);
  auto set_len = [&](uint32_t buf, uint64_t i0) {
    if (lane < items) rlen[8 * buf + lane] = i0 + lane < cnt ? len_of(i0 + lane) : 0u;
    __builtin_amdgcn_wave_barrier();
  };
  if (lane < items) rlen[lane] = first + lane < cnt ? len0 : 0u;
  __builtin_amdgcn_wave_barrier();
  // Load k covers 1 KiB of one item.  A lane's place in it does not depend on
  // k; the rest is the same in every lane.
  const uint32_t at = lane * 16;
  auto item_of = [&](uint32_t k) { return k >> (ll - 3); };
  auto off_of = [&](uint32_t k) { return (k & ((1u << (ll - 3)) - 1u)) * 1024u; };
  u32x4 v[8];
  // bytes of the lane's item from the vector of load k on (<= 0: none)
  auto left = [&](uint32_t k, uint32_t buf, uint32_t step) {
    return (int32_t)(rlen[8 * buf + item_of(k)] - step * kStepBytes - off_of(k) - at);
  };
  // 16 bytes at a scalar address plus a 32-bit offset of the lane (opaque, so
  // that no 64-bit address per load is kept in vector registers)
  auto fetch = [&](uint64_t base, uint32_t voff) {
    base = uniform64(base);
    asm("" : "+s"(base));
    return ldg16(base + voff);
  };
  // the step is consecutive bytes and all of them are there
  auto whole = [&](uint32_t buf, uint32_t step) {
    if (ll < 6 && item_bytes != kSegBytes << ll) return false;
    const uint32_t need = ll == 6 ? (step + 1) * kStepBytes : item_bytes;
    return __ballot(rlen[8 * buf + (lane & (items - 1u))] < need) == 0;
  };
  auto load_whole = [&](uint64_t i0, uint32_t step) {
    const uint64_t p = row0 + i0 * item_bytes + step * kStepBytes;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) v[k] = fetch(p, k * 1024 + lane * 16);
  };
  // otherwise only vectors that hold bytes of an item are read, and the bytes
  // past its end are cleared
  auto load_part = [&](uint32_t buf, uint64_t i0, uint32_t step) {
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      v[k] = u32x4{0, 0, 0, 0};
      if (left(k, buf, step) > 0)
        v[k] = fetch(row0 + (i0 + item_of(k)) * item_bytes + step * kStepBytes + off_of(k), at);
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const int32_t keep = left(k, buf, step);
      if (keep > 0 && keep < 16)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          v[k][q] = keep >= 4 * q + 4 ? v[k][q]
                    : keep <= 4 * q ? 0u : v[k][q] & ((1u << (8 * (keep - 4 * q))) - 1u);
    }
  };
  uint32_t buf = 0;
  bool have = false;  // v holds the coming step's bytes
  for (uint64_t i0 = first, i1; i0 < cnt; i0 = i1) {
    i1 = next(i0);
    const uint32_t len = rlen[8 * buf + (seg >> ll)];
    uint32_t steps = 1;
    if (ll == 6) steps = max(1u, (__builtin_amdgcn_readfirstlane(len) + kStepBytes - 1) / kStepBytes);
    const bool more = i1 < cnt;
    uint64_t h = kFnvBasis;
    for (uint32_t st = 0; st < steps; ++st) {
      if (!have) {
        if (whole(buf, st)) load_whole(i0, st);
        else load_part(buf, i0, st);
      }
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) {
        const uint32_t sg = k * 8 + (lane >> 3);
        const uint32_t slot = (sg >> 2) + 16 * (sg & 3);  // the lane that hashes it
        *reinterpret_cast<lptr_t<u32x4>>(tile + slot * kSegStride + (lane & 7u) * 16) = v[k];
      }
      __builtin_amdgcn_wave_barrier();
      const bool same = st + 1 < steps;
      if (!same && more) set_len(buf ^ 1u, i1);
      have = (same || more) && whole(same ? buf : buf ^ 1u, same ? st + 1 : 0u);
      if (have) load_whole(same ? i0 : i1, same ? st + 1 : 0u);
      uint32_t w[32];
#pragma unroll
      for (uint32_t q = 0; q < 8; ++q) {
        const u32x4 m = *reinterpret_cast<lptr_t<const u32x4>>(tile + lane * kSegStride + q * 16);
        w[4 * q] = m.x;
        w[4 * q + 1] = m.y;
        w[4 * q + 2] = m.z;
        w[4 * q + 3] = m.w;
      }
      __builtin_amdgcn_wave_barrier();
      h = h * slotw + par_step(w, (uint32_t)h & 0xffu, before, wt, colw, ll);
    }
    // undo the zero bytes after the item's end
    uint32_t pad = ((kSegBytes << ll) * steps) - len;
#pragma unroll 1
    for (uint32_t k = 0; __ballot(pad != 0); ++k, pad >>= 1)
      if (pad & 1u) h *= fnv_w.inv[k];
    const uint64_t it = i0 + (seg >> ll);
    if ((seg & ((1u << ll) - 1u)) == 0 && it < cnt) done(it, h);
    buf ^= 1u;
  }
}

// The same, a group every `stride` items.
template <class LenOf, class Done>
__device__ __forceinline__ void wave_fnv_par(uint64_t row0, uint32_t item_bytes, uint64_t first,
                                             uint64_t stride, uint64_t cnt, uint8_t* tile,
                                             LenOf len_of, Done done) {
  first = uniform64(first);
  stride = uniform64(stride);
  const uint64_t i = first + lane_id();
  const uint32_t len0 = lane_id() < par_items(item_bytes) && i < cnt ? len_of(i) : 0u;
  wave_fnv_par(
      row0, item_bytes, first, len0, cnt, tile, len_of, [=](uint64_t i) { return i + stride; }, done);
}

}  // namespace gsys_k
