// Which way a checksum launch hashes its items, from sizes alone: one lane per
// item (the serial chain, wave_fnv_t) or many (wave_fnv_par).  Plain functions
// without HIP, which the kernels' geometry and the launches share.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace gsys_k {

constexpr uint32_t kSegBytes = 128;               // per lane and step
constexpr uint32_t kStepBytes = 64 * kSegBytes;   // per wavefront and step
// Items up to this size are hashed one per lane: a matrix column sums 512
// bytes of one item, so a shorter one would waste lanes, and its chain is
// short (8 us for 512 bytes).
constexpr uint32_t kParMinItem = 512;
// Threads of the widest block of a kernel variant that hashes items with many
// lanes, holding the next step's bytes and the weights in registers (256 per
// lane).
constexpr uint32_t kParBlock = 512;

// Lanes an item of more than kParMinItem bytes occupies in a step (a power of
// two, at most the wavefront) as a shift.
constexpr uint32_t par_lanes_log2(uint32_t item_bytes) {
  uint32_t k = 3;
  while (k < 6 && (kSegBytes << k) < item_bytes) ++k;
  return k;
}

// The items a wavefront takes at once.
constexpr uint32_t par_items(uint32_t item_bytes) { return 64u >> par_lanes_log2(item_bytes); }

constexpr uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// Steps of a full item.
constexpr uint64_t par_steps(uint32_t item_bytes) { return ceil_div(item_bytes, kStepBytes); }

// Threads of a work-group with helper wavefronts: few work-groups leave
// compute units idle while theirs hash, so wavefronts that make no calls, up
// to eight per compute unit, share the group's items.  A kernel of one
// work-group of 64 work-items, one list call and 64 items of 4 KiB takes 94 us
// with its one wavefront, 42 with eight.
constexpr uint32_t helped_block(uint32_t block, uint64_t grid, uint32_t cus) {
  while (block * 2 <= kParBlock && grid * block * 2 <= (uint64_t)cus * kParBlock) block *= 2;
  return block;
}

// Work-groups of `wg` items (n in all) in blocks of `block` threads, plain
// form: true if many lanes per item are ahead of the chains.
//
// After its calls a work-group hashes its items alone on its compute unit, so
// what counts is how long one does.  A chain takes 15 ns a byte, 25 with eight
// wavefronts of them; a step of many lanes 2.65 us, 3.9 with eight wavefronts.
// Work-groups of 1,024 always run the chains: 128 registers per lane are too
// few for the other (8,000 work-item preads of 4 KiB took 2.1 ms with many
// lanes, 1.0 with the chains).  And the launch as a whole moves n items over
// the link: the chains of work-groups of more than 256 read it in 128-byte
// pieces, at 42 GB/s against 57, and where items are no multiple of 256 bytes
// the 256-byte pieces of the others straddle lines (about 50).
//
// Measured with one list call per work-group, chains against many lanes:
// work-groups of 512 with items of 8,256 bytes, 512 of them 0.50 against 0.77
// ms, 2,051 0.83 against 1.06, 12,192 3.01 against 2.50; of 256 with the same
// 256 items 0.30 against 0.40, 12,192 2.43 against 2.15; of 64 with 64 items
// of 4 KiB 0.15 against 0.07; of 1,024 with 1,024 items of 64 KiB 8.6 against
// 16.6.
inline bool many_lanes(uint64_t n, uint32_t item_bytes, uint32_t wg, uint32_t block) {
  if (item_bytes <= kParMinItem || block > kParBlock) return false;
  const uint64_t cnt = std::min<uint64_t>(wg, n);
  const uint64_t chains = ceil_div(cnt, 64);  // wavefronts with items
  const double chain_us = item_bytes * (chains <= 4 ? 0.015 : 0.025);
  // helpers share the work-group's items; without any, each wavefront has its own 64
  const uint64_t waves = block > wg ? block / 64 : chains;
  const uint64_t rounds = block > wg
                              ? ceil_div(ceil_div(cnt, par_items(item_bytes)), waves)
                              : ceil_div(std::min<uint64_t>(cnt, 64), par_items(item_bytes));
  const double par_us = (double)(rounds * par_steps(item_bytes)) * (waves <= 4 ? 2.65 : 3.9);
  const double link_us = (double)n * item_bytes * (wg > 256 ? 6.3e-6 : item_bytes % 256 ? 2.4e-6 : 0);
  return par_us < chain_us + link_us;
}

// Work-items per work-group of n work-item calls asked for in work-groups of
// wg (the calls do not depend on it).  A launch that leaves compute units idle
// is spread over more and smaller work-groups, down to one step of hashing for
// each of their eight wavefronts.  With a call's launch, reads and drain,
// against one work-group per wg items: 64 items of 4 KiB 57.5 against 68.0 us,
// 300 of 64 KiB 452 against 567, 20 of 1 MiB 0.75 against 1.36 ms.  Not with
// more calls than the ring has slots: those that wait for one poll host
// memory, and from more compute units they slow the host more: 100,000 calls
// of 576 bytes in work-groups of 1,024 (98 of them, a ring of 65,536) 10.8 ms,
// spread 12.4.
constexpr uint32_t spread_group(uint64_t n, uint32_t item_bytes, uint32_t wg, uint32_t cus,
                                uint64_t slots) {
  if (item_bytes <= kParMinItem || n > slots) return wg;
  while (wg > 8 * par_items(item_bytes) && ceil_div(n, wg / 2) <= cus) wg /= 2;
  return wg;
}

// Items that are in memory already, hashed by as many work-groups as they
// fill: true if many lanes per item are ahead of the chains (where the items
// are full: short ones go to the chains either way), which need 65,536 items
// to fill the chip.  The weights are cycles per byte and lane: a step
// whose 8 KiB are all there 26, others 40 (not loaded ahead; also the bytes a
// slot leaves empty are paid for), the chain 32.  Chains against many lanes:
// 200,000 items of 640 bytes 51 against 75 us, of 4 KiB 244 against 233,
// 65,536 of 8,256 bytes 174 against 281, 20,000 of them 133 against 91, 65,536
// of 12 KiB 216 against 283, 40,000 of 16,448 bytes 262 against 243.
inline bool consume_many_lanes(uint64_t n, uint32_t item_bytes) {
  if (item_bytes <= kParMinItem) return false;
  const uint64_t slot = item_bytes > kStepBytes ? kStepBytes : kSegBytes << par_lanes_log2(item_bytes);
  const uint64_t whole = item_bytes / slot, part = item_bytes % slot ? 1 : 0;
  const double par = (double)n * slot * (double)(whole * 26 + part * 40);
  return par < 32.0 * item_bytes * (double)std::max<uint64_t>(n, 65536);
}

// Groups of a wavefront of the many-lanes kernel, which keeps a bit for each of
// at most 64.
constexpr uint32_t kConsumeRounds = 64;
constexpr uint64_t consume_rounds(uint64_t n, uint32_t item_bytes, uint32_t wg, uint32_t grid) {
  return ceil_div(n, (uint64_t)grid * (wg / 64) * par_items(item_bytes));
}

// The same with the caller's grid of work-groups of wg work-items (many lanes
// make two of 512 out of one of 1,024): what counts is how long a wavefront's
// share takes, by the wavefronts on a SIMD.  Chains against many lanes, 20,000
// items of 4 KiB: 79 work-groups of 256 66 against 89 us, 200 66 against 40,
// 313 of 64 66 against 84, 40 of 512 106 against 126; 300 of 64 KiB in 64 of
// 256 966 against 38, 20,000 of 8,256 bytes in 79 of 256 132 against 400.
inline bool consume_many_lanes(uint64_t n, uint32_t item_bytes, uint32_t wg, uint32_t grid,
                               uint32_t cus) {
  if (item_bytes <= kParMinItem || !cus ||
      consume_rounds(n, item_bytes, wg, grid) > kConsumeRounds)
    return false;
  const uint64_t waves = (uint64_t)grid * (wg / 64);
  const double chains = (double)(ceil_div(grid, cus) * wg) / 256;  // per SIMD
  const double chain_ns = chains <= 1 ? 15 : chains <= 2 ? 25 : 11.2 * chains;
  const uint32_t block = std::min(wg, kParBlock);
  const double others = (double)(ceil_div((uint64_t)grid * (wg / block), cus) * block) / 256;
  const double step_ns = others <= 1 ? 2650 : 1950 * std::max(others, 2.0);
  const double chain = (double)ceil_div(n, waves * 64) * item_bytes * chain_ns;
  const double par = (double)(ceil_div(ceil_div(n, par_items(item_bytes)), waves) *
                              par_steps(item_bytes)) * step_ns;
  return par < chain;
}

}  // namespace gsys_k
