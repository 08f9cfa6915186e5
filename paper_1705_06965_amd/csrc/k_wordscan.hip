// Word search over files read with GPU-issued pread calls: the wordcount case
// study of section 7.1 (search 64 strings in many files; work-group
// granularity reads).  counts[f][q] = number of tokens of file f equal to
// query q, where a token is a maximal run of bytes other than space and
// newline.
//
// Files are cut into chunks of at most chunk_max bytes.  A chunk is read with
// one pread that also fetches the byte before it (to tell whether the chunk
// starts inside a token) and OVERLAP bytes after it (to finish the last
// token); a token belongs to the chunk in which it starts.  The persistent
// form takes chunks from a device work counter and prefetches the next one.
//
// Each wavefront scans 4 KiB sub-blocks of the chunk by itself (no work-group
// barrier inside a chunk), streamed from host staging with coalesced 16-byte
// loads (the next sub-block's loads are in flight while the current one is
// scanned).  A lane turns the vectors it loaded into delimiter bits with
// byte-parallel compares and puts both in LDS; then every lane owns a 64-byte
// stretch and packs the positions of its token starts into one list of the
// wavefront, so that the lanes share the tokens evenly.  Each token's length
// comes from the delimiter bits after its start; one of at most 16 bytes is
// tested, by its first four bytes and its length, against a 2,048-bit filter
// of the queries.  What passes is appended to a list of
// the wavefront, and whenever 64 tokens are listed each lane takes one: its
// (zero-padded) 16 bytes, assembled from aligned LDS words with alignbyte,
// and its length are looked up in an LDS hash table of the queries and
// compared exactly; matches are counted in per-wavefront LDS counters and
// added to counts[file] once per chunk.
#include "gsys_device.hpp"
#include "gsys.h"
#include "kernels.hpp"

#include <fcntl.h>

#include <algorithm>

namespace gsys_ws {

using namespace gsys;

// Work-groups of 512 (eight 4 KiB sub-blocks of host staging in flight while
// the previous ones are scanned) scan the 2,000-file corpus as fast as the
// link delivers it: 4.27 ms with 64 of them and 128 chunk buffers, against
// 4.49 ms with work-groups of 1,024, whose loads slow the host pool.  (End to
// end, with a drain about 40 us longer than today's.)  A launch with few
// chunks per work-group lasts as long as its longest ones, and 1,024 scan
// those sooner.  64 work-groups of 1,024 against 512: 90 files in 91 chunks
// 0.38 against 0.44 ms, 128 0.46 against 0.51, 170 0.50 against 0.52, 800 1.93
// against 1.85; of 4 KiB each 190 0.35 either way.  By name the same holds for
// one file per work-group and pieces of at least one round of sub-blocks: 40
// files with reads of 1 MiB 0.24 against 0.28 ms, of 64 KiB 0.31 against 0.33,
// of 16 KiB 0.76 against 0.70; 100 files of 4 KiB 0.20 either way but 512
// ahead by 2%.
constexpr uint32_t kNarrow = 512, kWide = 1024;
constexpr uint32_t kFewChunks = 3;  // per work-group
// Work-groups of the search by name unless GSYS_PERSISTENT_GRID asks for
// others: more of them, polling host memory, slow the host pool.  2,000 files
// of 64 KiB with buffers for 256 work-groups: 6.45 ms with 256, 4.88 with 128,
// 4.71 with 96, 4.99 with 64; 400 files of 4 KiB 0.62, 0.77, 0.60, 0.56.
constexpr uint32_t kOpenGrid = 96;
constexpr uint32_t kSeg = 64;                 // bytes scanned per lane per sub-block
constexpr uint32_t kSB = 64 * kSeg;           // 4 KiB sub-block of a wavefront
constexpr uint32_t kOverlap = 16;             // max query length and read-ahead
constexpr uint32_t kHead = 16;                // staging bytes before chunk byte 0
constexpr uint32_t kVecs = (kHead + kSB + kOverlap) / 16;  // 16-byte vectors per sub-block
constexpr uint32_t kMaxQ = 64;
constexpr uint32_t kTab = 128;                // query hash table slots
constexpr uint32_t kFilter = 2048;            // filter bits

struct WsArgs {
  gsys_dev_ctx c;
  const gsys_chunk* chunks;
  const uint8_t* queries;   // nq x 16 bytes
  const uint32_t* qlens;
  uint32_t* counts;         // nfiles x nq
  unsigned int* work;       // device work counter (zeroed per launch)
  uint64_t staging;         // chunk buffers of `cbuf` bytes
  uint32_t cbuf;
  uint32_t n_chunks;
  uint32_t nq;
  uint32_t passes;          // persistent forms: scans of every chunk in one launch
};

// One wavefront's sub-block: its bytes (16 before the first position, 16 after
// the last, and the rest of the last token's aligned words), the delimiter
// bits of vector i in bits[i + 3] (so that a lane's 64 bits are one aligned
// word: position p is bit p + 64), and the tokens that passed the filter
// (position | length << 16).
struct __align__(16) WaveBuf {
  uint8_t buf[kVecs * 16 + 16];
  uint16_t bits[kVecs + 3 + 3];
  uint32_t list[64 + 2 * 64];
  uint16_t starts[kSB / 2];   // positions of the sub-block's token starts
};

typedef uint64_t __attribute__((may_alias)) u64_any;  // several of `bits` at once
typedef uint32_t __attribute__((may_alias)) u32_any;

template <uint32_t WG>
struct Shared {
  static constexpr uint32_t kWaves = WG / 64;
  WaveBuf wb[kWaves];
  u32x4 qw[kTab];           // query bytes per slot, zero-padded to 16
  u32x4 mask[kOverlap + 1]; // the first n bytes of 16
  uint32_t tkey[kTab];      // hash key per slot; 0 = empty
  int32_t tq[kTab];         // query index | length << 16 per slot
  uint32_t filter[kFilter / 32];
  uint32_t cnt[kWaves][kMaxQ];
  uint32_t next;
};

// Key of a token or query: its (zero-padded) 16 bytes and length mixed into
// 32 bits; never 0.  Equal strings have equal keys; a key match is confirmed
// by comparing all 16 bytes and the length.
__device__ __forceinline__ uint32_t token_key(u32x4 w, uint32_t len) {
  const uint32_t r = w.x ^ __builtin_amdgcn_alignbit(w.y, w.y, 25) ^
                     __builtin_amdgcn_alignbit(w.z, w.z, 18) ^ __builtin_amdgcn_alignbit(w.w, w.w, 11);
  const uint32_t h = (r ^ (len << 3)) * 0x9e3779b1u;
  return (h ^ (h >> 15)) | 1u;
}

// The low `keep` bytes of a word (keep <= 0: none, >= 4: all).
__device__ __forceinline__ uint32_t byte_mask(int32_t keep) {
  return keep >= 4 ? ~0u : (keep <= 0 ? 0u : (1u << (8 * keep)) - 1u);
}

// Filter bit of a string from its first four bytes (those past its length
// shifted out) and its length.
__device__ __forceinline__ uint32_t filter_bit(uint32_t w0, uint32_t len) {
  const uint32_t k = w0 << (len >= 4 ? 0u : 32 - 8 * len);
  return ((k ^ (len << 3)) * 0x9e3779b1u) >> (32 - 11);
}
static_assert(kFilter == 1u << 11, "filter_bit gives 11 bits");

// Clear the counters and build the query table and filter.  The second
// wavefront does it, so that the first can issue the first call meanwhile;
// the caller's next work-group barrier ends it.
template <uint32_t WG>
__device__ void build_table(const WsArgs& A, Shared<WG>& S) {
  if (threadIdx.x >= 128)
    for (uint32_t i = threadIdx.x - 128; i < (WG / 64) * kMaxQ; i += WG - 128) (&S.cnt[0][0])[i] = 0;
  if (threadIdx.x < 64 || threadIdx.x >= 128) return;
  const uint32_t q = threadIdx.x - 64;
  static_assert(kTab == 128 && kFilter == 64 * 32 && kMaxQ == 64, "one wavefront's shares");
  S.tkey[q] = 0;
  S.tkey[q + 64] = 0;
  S.tq[q] = -1;
  S.tq[q + 64] = -1;
  S.filter[q] = 0;
  if (q <= kOverlap)
#pragma unroll
    for (int i = 0; i < 4; ++i) S.mask[q][i] = byte_mask((int32_t)q - 4 * i);
  __builtin_amdgcn_wave_barrier();
  uint32_t len = 0, k = 0;
  u32x4 w = {0, 0, 0, 0};
  if (q < A.nq) {
    len = A.qlens[q];
    const uint32_t* qp = reinterpret_cast<const uint32_t*>(A.queries + q * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = qp[i] & byte_mask((int32_t)len - 4 * i);
    k = token_key(w, len);
    uint32_t s = k & (kTab - 1);
    while (atomicCAS(&S.tkey[s], 0u, k) != 0u) s = (s + 1) & (kTab - 1);
    S.tq[s] = (int32_t)(q | (len << 16));
    S.qw[s] = w;
    const uint32_t f = filter_bit(w.x, len);
    atomicOr(&S.filter[f >> 5], 1u << (f & 31u));
  }
  __builtin_amdgcn_wave_barrier();
  // Of equal queries the first gets the counts, whichever lane's entry a
  // lookup meets first: all of them find that entry here and the lowest index
  // goes into it.
  if (q < A.nq) {
    uint32_t s = k & (kTab - 1);
    for (;; s = (s + 1) & (kTab - 1)) {
      const u32x4 o = S.qw[s];
      if (S.tkey[s] == k && o.x == w.x && o.y == w.y && o.z == w.z && o.w == w.w &&
          (uint32_t)S.tq[s] >> 16 == (len & 0xffffu))
        break;
    }
    atomicMin(&S.tq[s], (int32_t)(q | (len << 16)));
  }
}

// The bytes of x equal to space or newline, as bits weighted by wt's bytes and
// added to acc.
__device__ __forceinline__ uint32_t delim_bits(uint32_t x, uint32_t wt, uint32_t acc) {
  const uint32_t a = x ^ 0x20202020u, b = x ^ 0x0a0a0a0au;
  // 0x80 in every byte that is not zero
  const uint32_t na = ((a & 0x7f7f7f7fu) + 0x7f7f7f7fu) | a;
  const uint32_t nb = ((b & 0x7f7f7f7fu) + 0x7f7f7f7fu) | b;
  return __builtin_amdgcn_udot4((~(na & nb) >> 7) & 0x01010101u, wt, acc, false);
}

// 16 delimiter bits of a 16-byte vector (bit j = byte j).
__device__ __forceinline__ uint32_t delim16(u32x4 v) {
  const uint32_t lo = delim_bits(v.y, 0x80402010u, delim_bits(v.x, 0x08040201u, 0));
  const uint32_t hi = delim_bits(v.w, 0x80402010u, delim_bits(v.z, 0x08040201u, 0));
  return lo | (hi << 8);
}

// Staging buffer `slot` holds one chunk: byte k of the chunk at kHead + k and
// the byte before the chunk at kHead - 1.  Issue its pread (work-group
// granularity, relaxed: a consumer call, non-blocking).
__device__ Ticket issue_chunk(const WsArgs& A, uint32_t ci, uint64_t slot) {
  const gsys_chunk ch = A.chunks[ci];
  const uint32_t lb = ch.off > 0 ? 1u : 0u;
  const uint64_t dst = A.staging + slot * A.cbuf + kHead - lb;
  Args6 a{{(uint64_t)(int64_t)ch.fd, dst, (uint64_t)ch.len + kOverlap + lb, ch.off - lb, 0, 0}};
  Ticket tk{0, 0, 0};
  call_wg<O::Relaxed, B::NonBlocking>(A.c, GSYS_NR_PREAD64, 0, a, &tk);
  return tk;
}

// This lane's vectors of the sub-block at staging byte sb0: vector i covers
// bytes sb0 + 16 i of stg, lane l has vectors l + 64 k.  Only vectors that lie
// inside the buffer (`lim` bytes from stg) and start before `data` (the end of
// the bytes the call returned) cross the host link; the rest read as spaces,
// which the scan treats as delimiters, as it does every position past the
// valid extent.
constexpr uint32_t kPerLane = (kVecs + 63) / 64;
__device__ __forceinline__ void load_sub(const uint8_t* stg, uint32_t lim, uint32_t data,
                                         uint32_t sb0, u32x4 (&v)[kPerLane]) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (uint32_t k = 0; k < kPerLane; ++k) {
    const uint32_t i = lane + k * 64;
    v[k] = u32x4{0x20202020u, 0x20202020u, 0x20202020u, 0x20202020u};
    if (i < kVecs && sb0 + i * 16 + 16 <= lim && sb0 + i * 16 < data)
      v[k] = ldg16((uint64_t)(stg + sb0 + i * 16));
  }
}

// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr 1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast 15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast 31
  return v;
}

// The first dword of the (unaligned) text at buf + pos.
__device__ __forceinline__ uint32_t text4(lptr_t<const uint8_t> buf, uint32_t pos) {
  lptr_t<const uint32_t> a = reinterpret_cast<lptr_t<const uint32_t>>(buf + (pos & ~3u));
  return __builtin_amdgcn_alignbyte(a[1], a[0], pos & 3u);
}

// Look the token at buf + pos up and count it (lanes with len == 0 hold none).
template <class Sh>
__device__ __forceinline__ void count_token(Sh& S, uint32_t wave, lptr_t<const uint8_t> buf,
                                            uint32_t pos, uint32_t len) {
  if (!len) return;
  lptr_t<const uint32_t> aw = reinterpret_cast<lptr_t<const uint32_t>>(buf + (pos & ~3u));
  const uint32_t sh = pos & 3u;
  const uint32_t a0 = aw[0], a1 = aw[1], a2 = aw[2], a3 = aw[3], a4 = aw[4];
  const u32x4 w = u32x4{__builtin_amdgcn_alignbyte(a1, a0, sh), __builtin_amdgcn_alignbyte(a2, a1, sh),
                        __builtin_amdgcn_alignbyte(a3, a2, sh), __builtin_amdgcn_alignbyte(a4, a3, sh)} &
                  S.mask[len];
  const uint32_t k = token_key(w, len);
  uint32_t t = k & (kTab - 1);
  for (uint32_t n = 0; n < kTab; ++n) {
    const uint32_t tk = S.tkey[t];
    if (!tk) break;
    if (tk == k) {
      const u32x4 q = S.qw[t];
      const int32_t tq = S.tq[t];
      if (q.x == w.x && q.y == w.y && q.z == w.z && q.w == w.w && (uint32_t)(tq >> 16) == len) {
        atomicAdd(&S.cnt[wave][tq & 0xffff], 1u);
        break;
      }
    }
    t = (t + 1) & (kTab - 1);
  }
}

// Count the tokens that start at range positions [0, own) into
// counts[file].  Range position p is staging byte stg[kHead + p]; `ext`
// bytes from position 0 on are valid (later ones count as delimiters);
// stg[kHead - 1] is the byte before position 0 when lb_ok (else position 0
// starts a token if it is not a delimiter).  `lim` bytes from stg on lie in
// the buffer.  Every work-item calls this; the counters and the table are
// ready (a barrier came before).
//
// Bound by vector-ALU issue and LDS latency, about 4 us per 32 KiB of a
// work-group.  (All lanes checking each token in full, over 32 KiB
// sub-blocks between work-group barriers, took 27 us: the last 1 MiB chunk
// of a pass then kept the launch 0.8 ms after the last read, and one file of
// 500 KiB took 0.4 ms.)
template <uint32_t WG>
__device__ void scan_range(const WsArgs& A, Shared<WG>& S, uint32_t file, const uint8_t* stg,
                           uint32_t lim, uint32_t own_total, int64_t ext, bool lb_ok) {
  constexpr uint32_t kWaves = WG / 64;
  const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
  // staging bytes that hold data: the look-behind byte and positions < ext
  const uint32_t data = (uint32_t)min<int64_t>((int64_t)lim, (int64_t)kHead + max<int64_t>(ext, 0));
  lptr_t<uint8_t> buf = lp(S.wb[wave].buf);
  lptr_t<uint16_t> bits = lp(S.wb[wave].bits);
  lptr_t<u64_any> bits64 = reinterpret_cast<lptr_t<u64_any>>(bits);
  lptr_t<const u32_any> bits32 = reinterpret_cast<lptr_t<const u32_any>>(bits);
  lptr_t<uint32_t> list = lp(S.wb[wave].list);
  lptr_t<const uint32_t> filter = lp(S.filter);
  u32x4 v[kPerLane];
  uint32_t sb0 = wave * kSB;
  if (sb0 < own_total) load_sub(stg, lim, data, sb0, v);
  for (; sb0 < own_total; sb0 += kWaves * kSB) {
#pragma unroll
    for (uint32_t k = 0; k < kPerLane; ++k) {
      const uint32_t i = lane + k * 64;
      if (i < kVecs) {
        *reinterpret_cast<lptr_t<u32x4>>(buf + i * 16) = v[k];
        bits[i + 3] = (uint16_t)delim16(v[k]);
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (sb0 + kWaves * kSB < own_total)  // in flight during the scan
      load_sub(stg, lim, data, sb0 + kWaves * kSB, v);
    const int64_t sb_ext = ext - (int64_t)sb0;       // valid positions: p < sb_ext
    const uint32_t own = min(kSB, own_total - sb0);  // tokens may start at p < own
    const uint32_t p0 = lane * kSeg;
    // delimiter bits: bit i of dlo = position p0 + i; positions past the valid
    // extent count as delimiters, in LDS too
    uint64_t dlo = bits64[lane + 1];
    if (sb_ext < kSB + kOverlap) {
      const int64_t vlen = sb_ext - (int64_t)p0;  // valid bytes from p0 on
      if (vlen < 64) {
        dlo |= vlen <= 0 ? ~0ull : (~0ull << vlen);
        bits64[lane + 1] = dlo;
      }
      if (lane == 63 && vlen < 80) bits[kVecs + 2] |= vlen <= 64 ? 0xffffu : (0xffffu << (vlen - 64));
    }
    uint32_t prev_delim = (uint32_t)(bits64[lane] >> 63);  // position p0 - 1
    if (sb0 == 0 && p0 == 0) prev_delim = lb_ok ? prev_delim : 1u;
    else if ((int64_t)p0 - 1 >= sb_ext) prev_delim = 1u;
    uint64_t starts = ~dlo & ((dlo << 1) | prev_delim);
    if (own < kSB) {
      const uint32_t own_n = own > p0 ? min(kSeg, own - p0) : 0u;
      starts &= own_n >= 64 ? ~0ull : ((1ull << own_n) - 1ull);
    }
    // the positions of all starts, packed in order (lanes hold 0 to 32 each)
    const uint32_t mine = (uint32_t)__popcll(starts);
    const uint32_t upto = wave_scan(mine);
    const uint32_t total = __builtin_amdgcn_readlane(upto, 63);
    lptr_t<uint16_t> at = lp(S.wb[wave].starts) + (upto - mine);
    while (__ballot(starts != 0)) {
      if (starts) {
        *at++ = (uint16_t)(p0 + (uint32_t)__builtin_ctzll(starts));
        starts &= starts - 1;
      }
    }
    __builtin_amdgcn_wave_barrier();
    uint32_t n = 0;  // listed tokens (the same in every lane)
    for (uint32_t i = 0; i < total; i += 128) {
      // two tokens per lane at a time: their LDS reads overlap
      bool pass[2];
      uint32_t pos[2], w0[2], w1[2], len[2], f[2], fw[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        pass[u] = i + 64 * u + lane < total;
        pos[u] = pass[u] ? lp(S.wb[wave].starts)[i + 64 * u + lane] : 0u;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t k = (pos[u] + 64) >> 5;
        w0[u] = bits32[k];
        w1[u] = bits32[k + 1];
        f[u] = text4(buf, kHead + pos[u]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        // the first delimiter after the start, 17 for more than 16 bytes
        const uint32_t win = __builtin_amdgcn_alignbit(w1[u], w0[u], pos[u] & 31u) | (1u << 17);
        len[u] = (uint32_t)__builtin_ctz(win);
        pass[u] = pass[u] && len[u] <= kOverlap;
        f[u] = filter_bit(f[u], len[u]);
        fw[u] = filter[f[u] >> 5];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        pass[u] = pass[u] && ((fw[u] >> (f[u] & 31u)) & 1u);
        const uint64_t m = __ballot(pass[u]);
        if (pass[u])
          list[n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
              (kHead + pos[u]) | (len[u] << 16);
        n += (uint32_t)__popcll(m);
      }
      while (n >= 64) {
        __builtin_amdgcn_wave_barrier();
        n -= 64;
        const uint32_t e = list[n + lane];
        count_token(S, wave, buf, e & 0xffffu, e >> 16);
        __builtin_amdgcn_wave_barrier();
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (n) {
      const uint32_t e = lane < n ? list[lane] : 0u;
      count_token(S, wave, buf, e & 0xffffu, e >> 16);
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // flush this chunk's counts
  for (uint32_t q = threadIdx.x; q < A.nq; q += blockDim.x) {
    uint32_t c = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      c += S.cnt[w][q];
      S.cnt[w][q] = 0;
    }
    if (c) atomicAdd(&A.counts[(uint64_t)file * A.nq + q], c);
  }
  __syncthreads();
}

template <uint32_t WG>
__device__ void scan_chunk(const WsArgs& A, Shared<WG>& S, uint32_t ci, uint64_t slot, int64_t ret) {
  const gsys_chunk ch = A.chunks[ci];
  const uint32_t lb = ch.off > 0 ? 1u : 0u;
  // bytes available at chunk positions >= 0 (chunk + read-ahead, EOF-bounded)
  const int64_t ext = ret > (int64_t)lb ? ret - (int64_t)lb : 0;
  const bool lb_ok = lb && ret >= 1;
  const uint8_t* stg = reinterpret_cast<const uint8_t*>(A.staging) + slot * A.cbuf;
  scan_range(A, S, ch.file, stg, A.cbuf, ch.len, ext, lb_ok);
}

// The next work item for the whole work-group.  The leading barrier closes
// whatever thread-0-only code ran before it (a weak blocking call's wait, a
// result store): without it such code joins the atomic below into one
// thread-0 region across the loop's back edge, and the compiled loop then
// lets the other work-items of thread 0's wavefront pass the barrier below
// before thread 0 has taken the item, read a stale S.next, and never leave
// the loop.
template <uint32_t WG>
__device__ __forceinline__ uint32_t grab(const WsArgs& A, Shared<WG>& S) {
  __syncthreads();
  if (threadIdx.x == 0) S.next = atomicAdd(A.work, 1u);
  __syncthreads();
  const uint32_t v = S.next;
  __syncthreads();
  return v;
}

// Persistent form: work items come from a device work counter; the pread of
// the next one is issued before the current one is scanned.  Work item w is
// chunk w mod n_chunks of pass w / n_chunks: with several passes the
// work-groups go from one pass to the next without draining, and each pass
// adds its counts.
template <uint32_t WG>
__global__ __launch_bounds__(WG) void wordscan_persistent(WsArgs A) {
  __shared__ Shared<WG> S;
  const uint32_t total = A.n_chunks * A.passes;
  uint32_t cur = grab(A, S);
  if (cur >= total) return;
  uint32_t bi = 0;
  build_table(A, S);  // the barriers of the calls below end it
  Ticket tk = issue_chunk(A, cur % A.n_chunks, (uint64_t)blockIdx.x * 2 + bi);
  for (;;) {
    const uint32_t nxt = grab(A, S);
    Ticket tkn{0, 0, 0};
    if (nxt < total)
      tkn = issue_chunk(A, nxt % A.n_chunks, (uint64_t)blockIdx.x * 2 + (bi ^ 1u));
    const int64_t r = wait_wg(A.c, tk);
    scan_chunk(A, S, cur % A.n_chunks, (uint64_t)blockIdx.x * 2 + bi, r);
    if (nxt >= total) break;
    cur = nxt;
    tk = tkn;
    bi ^= 1u;
  }
}

// Plain form: one work-group per chunk, blocking relaxed work-group call
// (the paper's wordcount setting: work-group granularity, blocking, weak).
template <uint32_t WG>
__global__ __launch_bounds__(WG) void wordscan_plain(WsArgs A) {
  __shared__ Shared<WG> S;
  build_table(A, S);
  const uint32_t ci = blockIdx.x;
  if (ci >= A.n_chunks) return;
  const gsys_chunk ch = A.chunks[ci];
  const uint32_t lb = ch.off > 0 ? 1u : 0u;
  const uint64_t dst = A.staging + (uint64_t)ci * A.cbuf + kHead - lb;
  Args6 a{{(uint64_t)(int64_t)ch.fd, dst, (uint64_t)ch.len + kOverlap + lb, ch.off - lb, 0, 0}};
  // a consumer call has no barrier before it: the table is built while the
  // first wavefront waits
  const int64_t r = call_wg<O::Relaxed, B::Blocking>(A.c, GSYS_NR_PREAD64, 0, a);
  scan_chunk(A, S, ci, ci, r);
}

// ---------------------------------------------------------------------------
// The wordcount as the case study issues it (section 7.1): each work-group
// takes a file, opens it by name, reads it front to back with read() (the
// file offset advances on the host), scans the pieces and closes the file.
// Reads are sequential, so there is no read-ahead: a piece owns the tokens
// that start before its last kOverlap bytes, and those bytes, with the byte
// before them, are carried in front of the next piece (the next read is
// already in flight into the other buffer while this piece is scanned).  A
// read shorter than asked, or of 0 bytes, ends the file (a regular file).
//
// Piece buffer layout: [0, kOpenHead) carry, data from kOpenHead on.  The
// carry's 16 bytes sit at [kOpenHead - 16, kOpenHead), the byte before them
// at kOpenHead - 17, each piece's data on a fresh 64-byte line.

constexpr uint32_t kOpenHead = 64;
// Room past the piece.  A scan reads at most the rest of the last 16-byte
// vector; callers size their buffers by the whole, which decides what is
// accepted and how many work-groups fit, so it stays.
constexpr uint32_t kOpenTail = (32u << 10) + 48;
constexpr uint32_t kCarry = kOverlap;  // deferred bytes

struct WoArgs {
  WsArgs w;             // queries, counts, staging (2 buffers of w.cbuf per group)
  uint64_t paths;       // registered host buffer: nfiles x GSYS_PATH_MAX bytes
  int64_t* file_ret;    // device: bytes read per file, or -errno
  uint64_t progress;    // host-visible: 2 x u64 per work-group, or 0
  uint32_t records;     // of them, the ones that end as kPhDone
  uint32_t nfiles;
  uint32_t chunk;       // bytes per read()
  int32_t dirfd;
};

// Where a work-group is (thread 0 only): word 0 = (file + 1) << 32 | phase,
// word 1 = piece << 32 | low 32 bits of the last call's ticket.  Written
// with system-scope stores, so the host can read it while the kernel runs.
enum : uint32_t { kPhOpen = 1, kPhRead = 2, kPhScan = 3, kPhClose = 4, kPhDone = 5 };
__device__ __forceinline__ void progress(const WoArgs& A, uint32_t f, uint32_t phase,
                                         uint32_t piece, uint64_t ticket) {
  if (!A.progress || threadIdx.x != 0) return;
  uint64_t* p = reinterpret_cast<uint64_t*>(A.progress) + 2ull * blockIdx.x;
  st_sys(p + 1, ((uint64_t)piece << 32) | (uint32_t)ticket);
  st_sys(p, ((uint64_t)(f + 1) << 32) | phase);
}

template <uint32_t WG>
__device__ void open_and_scan(const WoArgs& A, Shared<WG>& S, uint32_t f) {
  const gsys_dev_ctx& c = A.w.c;
  const uint64_t base = A.w.staging + (uint64_t)blockIdx.x * 2 * A.w.cbuf;
  progress(A, f, kPhOpen, 0, 0);
  // openat: a consumer call, blocking: every work-item needs the descriptor
  const int64_t fd = call_wg<O::Relaxed, B::Blocking>(
      c, GSYS_NR_OPENAT, 0,
      Args6{{(uint64_t)(int64_t)A.dirfd, A.paths + (uint64_t)f * GSYS_PATH_MAX,
             (uint64_t)O_RDONLY, 0, 0, 0}});
  if (fd < 0) {
    if (threadIdx.x == 0) A.file_ret[f] = fd;
    return;
  }
  auto issue = [&](uint32_t b) {
    Ticket tk{0, 0, 0};
    call_wg<O::Relaxed, B::NonBlocking>(
        c, GSYS_NR_READ, 0,
        Args6{{(uint64_t)fd, base + b * A.w.cbuf + kOpenHead, A.chunk, 0, 0, 0}}, &tk);
    return tk;
  };
  int64_t total = 0, err = 0;
  uint32_t b = 0, piece = 0;
  bool first = true;
  Ticket tk = issue(0);
  for (;;) {
    progress(A, f, kPhRead, piece, tk.t);
    const int64_t r = wait_wg(c, tk);
    if (r < 0) {
      err = r;
      break;
    }
    const bool end = (uint64_t)r < A.chunk;
    const uint64_t buf = base + b * A.w.cbuf;
    if (!end) {
      // carry this piece's last kCarry + 1 bytes in front of the next one,
      // then start reading it
      const uint64_t nb = base + (b ^ 1u) * A.w.cbuf;
      if (threadIdx.x <= kCarry)
        gp<uint8_t>(nb + kOpenHead - kCarry - 1)[threadIdx.x] =
            gp<const uint8_t>(buf + kOpenHead + (uint64_t)r - kCarry - 1)[threadIdx.x];
      tk = issue(b ^ 1u);
    }
    // the range: the carry (none for the first piece), then the data
    const uint32_t carry = first ? 0u : kCarry;
    const int64_t ext = (int64_t)carry + r;
    const uint32_t own = end ? (uint32_t)ext : (uint32_t)(ext - kCarry);
    const uint32_t p0 = kOpenHead - carry;  // buffer byte of range position 0
    progress(A, f, kPhScan, piece, tk.t);
    scan_range(A.w, S, f, reinterpret_cast<const uint8_t*>(buf + p0 - kHead),
               A.w.cbuf - (p0 - kHead), own, ext, !first);
    total += r;
    if (end) break;
    b ^= 1u;
    first = false;
    ++piece;
  }
  // close: a producer call (every work-item is done with the descriptor);
  // the designated caller records the file's result
  progress(A, f, kPhClose, piece, 0);
  const int64_t rc = call_wg<O::Relaxed, B::Blocking>(c, GSYS_NR_CLOSE, 0,
                                                      Args6{{(uint64_t)fd, 0, 0, 0, 0, 0}});
  if (threadIdx.x == 0) A.file_ret[f] = err ? err : (rc < 0 ? rc : total);
}

template <uint32_t WG>
__global__ __launch_bounds__(WG) void wordopen_persistent(WoArgs A) {
  __shared__ Shared<WG> S;
  uint32_t last = ~0u;
  uint32_t f = grab(A.w, S);
  if (f < A.nfiles) build_table(A.w, S);  // while the first openat is served
  while (f < A.nfiles) {
    open_and_scan(A, S, f);
    last = f;
    // grab() opens with a barrier: the thread-0-only result store that ends
    // open_and_scan never shares a region with the next grab's atomic
    f = grab(A.w, S);
  }
  progress(A, last, kPhDone, 0, 0);
  // the records of work-groups that were not launched
  if (A.progress && threadIdx.x == 0)
    for (uint32_t r = blockIdx.x + gridDim.x; r < A.records; r += gridDim.x) {
      uint64_t* p = reinterpret_cast<uint64_t*>(A.progress) + 2ull * r;
      st_sys(p + 1, 0);
      st_sys(p, kPhDone);
    }
}

// Clear the counts and the work counter before a scan.
__global__ void zero_counts(uint32_t* p, uint64_t n, uint32_t* work) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *work = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

}  // namespace gsys_ws

using namespace gsys_ws;

int gsys_wordscan(gsys_ctx* ctx, uint64_t chunks, uint32_t n_chunks, uint32_t chunk_max,
                  uint64_t queries, uint64_t qlens, uint32_t nq, uint64_t counts, uint32_t nfiles,
                  uint64_t staging, uint64_t staging_bytes, uint32_t form, uint32_t passes,
                  void* stream) {
  // no chunks (every file empty, or no files) only zeroes the counts
  if (!ctx || (!chunks && n_chunks) || !queries || !qlens || !counts) return -EINVAL;
  if (passes == 0 || (form == GSYS_PLAIN && passes != 1) ||
      (uint64_t)n_chunks * passes > 0xffffffffull)
    return -EINVAL;
  if (nq == 0 || nq > kMaxQ || chunk_max == 0 || chunk_max > (64u << 20)) return -EINVAL;
  const uint32_t cbuf = (chunk_max + 64 + 15) & ~15u;
  if (gsys_internal::check_host_range(ctx, staging, staging_bytes)) return -EFAULT;
  const uint64_t per_wg = 2ull * cbuf;
  hipStream_t s = (hipStream_t)stream;
  WsArgs A;
  if (int e = gsys_device_ctx(ctx, &A.c)) return e;
  A.chunks = (const gsys_chunk*)chunks;
  A.queries = (const uint8_t*)queries;
  A.qlens = (const uint32_t*)qlens;
  A.counts = (uint32_t*)counts;
  A.work = (unsigned int*)gsys_internal::kstate(ctx) + 8;
  A.staging = staging;
  A.cbuf = cbuf;
  A.n_chunks = n_chunks;
  A.nq = nq;
  A.passes = passes;
  if (form != GSYS_PLAIN && form != GSYS_PERSISTENT && form != GSYS_GRAPH) return -EINVAL;
  // zero the counts and the work counter, then scan
  uint64_t ncount = (uint64_t)nfiles * nq;
  uint32_t* counts32 = (uint32_t*)counts;
  uint32_t* work32 = (uint32_t*)A.work;
  void* z_args[] = {&counts32, &ncount, &work32};
  void* args[] = {&A};
  const dim3 z_grid((uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((ncount + 255) / 256, 4096)));
  gsys_internal::KLaunch k[2] = {{(const void*)zero_counts, z_grid, dim3(256), 0, z_args},
                                 {nullptr, dim3(1), dim3(kNarrow), 0, args}};
  if (form == GSYS_PLAIN) {
    if (n_chunks && staging_bytes < (uint64_t)cbuf * n_chunks) return -EINVAL;
    const bool wide = n_chunks <= gsys_internal::cu_count(ctx);
    k[1].kernel = wide ? (const void*)wordscan_plain<kWide> : (const void*)wordscan_plain<kNarrow>;
    k[1].block = dim3(wide ? kWide : kNarrow);
    k[1].grid = dim3(n_chunks);
  } else {
    if (n_chunks && staging_bytes < per_wg) return -EINVAL;
    const uint64_t items = (uint64_t)n_chunks * passes;
    // as many work-groups as are resident, have staging and have a chunk
    const uint64_t groups = std::min<uint64_t>(staging_bytes / per_wg, gsys_internal::cu_count(ctx));
    const bool wide = items <= kFewChunks * groups;
    const void* kp = wide ? (const void*)wordscan_persistent<kWide>
                          : (const void*)wordscan_persistent<kNarrow>;
    const uint32_t block = wide ? kWide : kNarrow;
    uint32_t grid = gsys_internal::resident_grid(ctx, kp, block, 0);
    if (!grid) return -ENODEV;
    grid = (uint32_t)std::min<uint64_t>({(uint64_t)grid, staging_bytes / per_wg, items});
    const uint32_t req = gsys_internal::persistent_grid_override(ctx);
    if (req && req < grid) grid = req;
    k[1].kernel = kp;
    k[1].block = dim3(block);
    k[1].grid = dim3(grid);
  }
  if (form == GSYS_GRAPH && n_chunks) {
    // one graph per shape: the fill and the scan, replayed with this call's
    // arguments
    const uint64_t key = gsys_internal::hash_words({0x3C5ull, z_grid.x, k[1].grid.x, k[1].block.x});
    return gsys_internal::launch_graph(ctx, key, k, 2, s);
  }
  for (uint32_t i = 0; i < 2; ++i) {
    if (i == 1 && !n_chunks) break;
    if (int e = gsys_internal::launch(ctx, k[i].kernel, k[i].grid.x, k[i].block.x, 0, k[i].args, s))
      return e;
  }
  return 0;
}

uint64_t gsys_wordcount_open_buffer_bytes(uint32_t chunk) {
  return ((uint64_t)kOpenHead + chunk + kOpenTail + 15) & ~15ull;
}

uint32_t gsys_wordcount_open_groups(gsys_ctx* ctx) {
  if (!ctx) return 0;
  const uint32_t req = gsys_internal::persistent_grid_override(ctx);
  return req ? req : kOpenGrid;
}

int gsys_wordcount_open(gsys_ctx* ctx, int dirfd, uint64_t paths, uint32_t nfiles,
                        uint64_t queries, uint64_t qlens, uint32_t nq, uint64_t counts,
                        uint64_t file_ret, uint32_t chunk, uint64_t staging,
                        uint64_t staging_bytes, uint64_t progress, uint32_t progress_groups,
                        void* stream) {
  if (!ctx) return -EINVAL;
  if (nq == 0 || nq > kMaxQ) return -EINVAL;
  if (chunk < 64 || chunk % 64 || chunk > (64u << 20)) return -EINVAL;
  if (!nfiles) return 0;  // the outputs are empty and may be null
  if (!queries || !qlens || !counts || !file_ret) return -EINVAL;
  if (gsys_internal::check_host_range(ctx, paths, (uint64_t)nfiles * GSYS_PATH_MAX)) return -EFAULT;
  // carry head + data + the room past it
  const uint32_t cbuf = (uint32_t)gsys_wordcount_open_buffer_bytes(chunk);
  const uint64_t per_wg = 2ull * cbuf;
  if (staging_bytes < per_wg) return -EINVAL;
  if (gsys_internal::check_host_range(ctx, staging, staging_bytes)) return -EFAULT;
  if (progress && (!progress_groups ||
                   gsys_internal::check_host_range(ctx, progress, 16ull * progress_groups)))
    return progress_groups ? -EFAULT : -EINVAL;
  hipStream_t s = (hipStream_t)stream;
  WoArgs A;
  if (int e = gsys_device_ctx(ctx, &A.w.c)) return e;
  A.w.chunks = nullptr;
  A.w.queries = (const uint8_t*)queries;
  A.w.qlens = (const uint32_t*)qlens;
  A.w.counts = (uint32_t*)counts;
  A.w.work = (unsigned int*)gsys_internal::kstate(ctx) + 8;
  A.w.staging = staging;
  A.w.cbuf = cbuf;
  A.w.n_chunks = 0;
  A.w.passes = 1;
  A.w.nq = nq;
  A.paths = paths;
  A.file_ret = (int64_t*)file_ret;
  A.nfiles = nfiles;
  A.chunk = chunk;
  A.dirfd = dirfd;
  const uint64_t ncount = (uint64_t)nfiles * nq;
  if (gsys_internal::no_device(ctx)) return -ENODEV;
  hipLaunchKernelGGL(zero_counts, dim3((uint32_t)std::min<uint64_t>((ncount + 255) / 256, 4096)),
                     dim3(256), 0, s, (uint32_t*)counts, ncount, (uint32_t*)A.w.work);
  if (hipGetLastError() != hipSuccess) return -ENODEV;
  uint64_t groups = std::min<uint64_t>({staging_bytes / per_wg, nfiles, gsys_internal::cu_count(ctx)});
  if (progress && progress_groups < groups) groups = progress_groups;  // one record per work-group
  A.records = (uint32_t)groups;
  groups = std::min<uint64_t>(groups, gsys_wordcount_open_groups(ctx));
  const bool wide = nfiles <= groups && chunk >= (kWide / 64) * kSB;
  const void* kp = wide ? (const void*)wordopen_persistent<kWide>
                        : (const void*)wordopen_persistent<kNarrow>;
  const uint32_t block = wide ? kWide : kNarrow;
  uint32_t grid = gsys_internal::resident_grid(ctx, kp, block, 0);
  if (!grid) return -ENODEV;
  grid = (uint32_t)std::min<uint64_t>(grid, groups);
  A.progress = progress;
  void* args[] = {&A};
  return gsys_internal::launch(ctx, kp, grid, block, 0, args, s);
}
