// Per-item pread + FNV-1a-64 on gfx950: the pread microbenchmark of section 6
// (Fig. 5) issued at work-item, work-group or kernel granularity, strong or
// relaxed, blocking or non-blocking, and a persistent form that drains the
// items in one launch with double-buffered non-blocking group calls.
//
// Data path: the host pool preads each item into pinned host staging; the GPU
// reads the staging bytes once over the host link with coalesced 16-byte
// loads, transposes them through LDS and hashes them: items of more than 512
// bytes with many lanes each (wave_fnv_par), shorter ones with a lane each
// running the serial byte chain (wave_fnv_t).
#include "gsys_device.hpp"
#include "fnv_wave.hpp"
#include "gsys.h"
#include "kernels.hpp"

#include <algorithm>

namespace gsys_k {

using namespace gsys;

// Default persistent grid (work-groups); see gsys_fnv4k.  64 of them keep 128
// lists in flight, which is enough for the host pool, and fewer waiters poll
// host memory: the 262,144-item sweep took 19.7 ms with 64 or 48, 20.0 with
// 32 and 19.8 with 80 to 128.
constexpr uint32_t kPersistentGrid = 64;

struct FnvArgs {
  gsys_dev_ctx c;
  const uint64_t* offsets;
  uint64_t n_items;
  uint64_t staging;
  gsys_iodesc* lists;
  uint64_t* out_fnv;
  int64_t* out_ret;
  KState* ks;
  int32_t fd;
  uint32_t item_bytes;
  uint32_t ring;  // persistent forms: 1 = each work-group owns two batch buffers
  uint32_t lds_list;  // strong work-group cells: aggregate the list in LDS first
  uint32_t wg;     // work-items (and items) per work-group; wider blocks bring helper wavefronts
  uint32_t batch;  // persistent forms: items per list call (wg is the same)
};

// Staging address of item `item` of batch `bt` (slot = item - bt * batch).
__device__ __forceinline__ uint64_t stage_addr(const FnvArgs& A, uint64_t bt, uint32_t batch,
                                               uint64_t item) {
  if (!A.ring) return A.staging + item * A.item_bytes;
  const uint64_t buf = (uint64_t)blockIdx.x * 2 + (bt / gridDim.x) % 2;
  return A.staging + (buf * batch + (item - bt * batch)) * A.item_bytes;
}

// The group's items first .. first + cnt - 1 (from staging address row0):
// store each work-item's call result and hash the bytes.  `ret` is the result
// of item first + threadIdx.x (cnt <= A.wg <= blockDim.x).  Serial: each
// wavefront hashes its own 64 work-items' items.  Otherwise, in a block of
// A.wg work-items each wavefront takes its own work-items' items too (no
// wavefront waits for another's calls); in a wider block all wavefronts share
// the group's items after a barrier.
template <uint32_t WGMAX, bool par>
__device__ __forceinline__ void consume_items(const FnvArgs& A, uint64_t first, uint32_t cnt,
                                              int64_t ret, uint8_t* lds, uint64_t row0) {
  const uint32_t t = threadIdx.x, wave = t >> 6;
  const bool valid = t < cnt;
  const uint32_t nbytes =
      (valid && ret > 0) ? (uint32_t)min<int64_t>(ret, (int64_t)A.item_bytes) : 0u;
  if (valid) A.out_ret[first + t] = ret;
  if constexpr (!par) {
    constexpr uint32_t CH = chunk_for<WGMAX>();
    const uint64_t h = wave_fnv_t<CH>(row0 + (uint64_t)(t & ~63u) * A.item_bytes, nbytes,
                                      A.item_bytes, lds + wave * Tile<CH>::kBytes);
    if (valid) A.out_fnv[first + t] = h;
  } else {
    const uint32_t waves = blockDim.x >> 6, items = par_items(A.item_bytes);
    lptr_t<uint32_t> lens = reinterpret_cast<lptr_t<uint32_t>>(lp(lds) + waves * kParTile);
    if (t < A.wg) lens[t] = nbytes;
    const bool shared = blockDim.x > A.wg;
    uint32_t lo = 0, hi = cnt, step = waves * items;
    if (shared) {
      __syncthreads();
      lo = wave * items;
    } else {
      __builtin_amdgcn_wave_barrier();
      lo = wave * 64;
      hi = min(cnt, lo + 64);
      step = items;
    }
    wave_fnv_par(
        row0, A.item_bytes, lo, step, hi, lds + wave * kParTile,
        [&](uint64_t i) { return lens[i]; },
        [&](uint64_t i, uint64_t h) { A.out_fnv[first + i] = h; });
  }
}

// Plain form: one launch, one item per work-item, the call made at the
// granularity / ordering / blocking of the template.
template <G g, O o, B b, uint32_t WGMAX, bool par>
__global__ __launch_bounds__(WGMAX, WGMAX <= kParBlock ? 2 : 4) void fnv4k_plain(FnvArgs A) {
  extern __shared__ __align__(16) uint8_t lds[];
  const uint64_t first = (uint64_t)blockIdx.x * A.wg;
  const uint64_t item = first + threadIdx.x;
  const uint32_t cnt = (uint32_t)min<uint64_t>(A.wg, A.n_items - first);
  const bool valid = threadIdx.x < cnt;
  int64_t ret = 0;
  if constexpr (g == G::WorkItem) {
    if (valid) {
      Args6 a{{(uint64_t)(int64_t)A.fd, A.staging + item * A.item_bytes, A.item_bytes,
               A.offsets[item], 0, 0}};
      Ticket tk;
      ret = call_wi<b>(A.c, GSYS_NR_PREAD64, a, &tk);
      if constexpr (b == B::NonBlocking) ret = ret ? ret : wait_wi(A.c, tk);
    }
  } else if constexpr (g == G::WorkGroup) {
    gsys_iodesc* L = A.lists + first;
    if constexpr (o == O::Strong) {
      const gsys_iodesc d{valid ? A.offsets[item] : 0, threadIdx.x * A.item_bytes,
                          (int32_t)A.item_bytes};
      if (A.lds_list) {
        // aggregated in LDS (the transposer's tile space, unused until the
        // hash): every work-item stores its descriptor there, and after a
        // barrier the caller's wavefront copies the list to the host-visible
        // buffer with 16-byte stores; the call's barrier before releases them
        gsys_iodesc* S = reinterpret_cast<gsys_iodesc*>(lds);
        if (valid) *lp(reinterpret_cast<u32x4*>(S + threadIdx.x)) = *reinterpret_cast<const u32x4*>(&d);
        __syncthreads();
        if (threadIdx.x < 64)
          for (uint32_t i = threadIdx.x; i < cnt; i += 64)
            stg16((uint64_t)(L + i), *lp(reinterpret_cast<u32x4*>(S + i)));
      } else if (valid) {
        // every work-item writes its own descriptor straight into the host-
        // visible list (a wavefront's 64 are 1 KiB of consecutive bytes);
        // the barrier before the call makes all of them visible to the host
        L[threadIdx.x] = d;
      }
    } else {
      // relaxed consumer call: no barrier before it, so the designated
      // caller's wavefront builds the list from the offset table itself
      if (threadIdx.x < 64)
        for (uint32_t i = threadIdx.x; i < cnt; i += 64)
          L[i] = gsys_iodesc{A.offsets[first + i], i * A.item_bytes, (int32_t)A.item_bytes};
    }
    Args6 a{{(uint64_t)(int64_t)A.fd, (uint64_t)L, cnt, A.staging + first * A.item_bytes, 0, 0}};
    Ticket tk{0, 0, 0};
    int64_t r = call_wg<o, b>(A.c, GSYS_NR_PREAD64, GSYS_F_LIST, a, &tk);
    if constexpr (b == B::NonBlocking) r = wait_wg(A.c, tk);
    ret = valid ? (r < 0 ? r : (int64_t)__hip_atomic_load(&L[threadIdx.x].len_ret, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_SYSTEM))
                : 0;
  } else {
    Ticket tk{0, 0, 0};
    int64_t r = call_kernel<b>(
        A.c, A.ks, GSYS_NR_PREAD64, GSYS_F_LIST,
        [&]() {
          for (uint64_t i = threadIdx.x; i < A.n_items; i += blockDim.x)
            A.lists[i] = gsys_iodesc{A.offsets[i], (uint32_t)(i * A.item_bytes), (int32_t)A.item_bytes};
        },
        [&]() {
          return Args6{{(uint64_t)(int64_t)A.fd, (uint64_t)A.lists, A.n_items, A.staging, 0, 0}};
        },
        &tk);
    if constexpr (b == B::NonBlocking) r = r ? r : wait_kernel(A.c, tk);
    ret = valid ? (r < 0 ? r : (int64_t)__hip_atomic_load(&A.lists[item].len_ret, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_SYSTEM))
                : 0;
  }
  consume_items<WGMAX, par>(A, first, cnt, ret, lds, A.staging + first * A.item_bytes);
}

// Persistent form: a co-resident grid; work-group w handles batches w,
// w + grid, ...; each batch of A.batch items is one work-group call (relaxed
// consumer, non-blocking) whose descriptor list the caller's wavefront builds.  The
// call for the next batch is issued before waiting on the current one, so
// host servicing overlaps the GPU's consumption.
__device__ __forceinline__ Ticket issue_batch(const FnvArgs& A, uint64_t bt, uint32_t batch) {
  const uint64_t first = bt * batch;
  const uint32_t cnt = (uint32_t)min<uint64_t>(batch, A.n_items - first);
  gsys_iodesc* L = A.lists + first;
  if (threadIdx.x < 64)
    for (uint32_t i = threadIdx.x; i < cnt; i += 64)
      L[i] = gsys_iodesc{A.offsets[first + i], i * A.item_bytes, (int32_t)A.item_bytes};
  Args6 a{{(uint64_t)(int64_t)A.fd, (uint64_t)L, cnt, stage_addr(A, bt, batch, first), 0, 0}};
  Ticket tk{0, 0, 0};
  call_wg<O::Relaxed, B::NonBlocking>(A.c, GSYS_NR_PREAD64, GSYS_F_LIST, a, &tk);
  return tk;
}

template <uint32_t WGMAX, bool par>
__global__ __launch_bounds__(WGMAX, 2) void fnv4k_persistent(FnvArgs A) {
  extern __shared__ __align__(16) uint8_t lds[];
  const uint32_t batch = A.batch;
  const uint64_t nb = (A.n_items + batch - 1) / batch;
  uint64_t bt = blockIdx.x;
  if (bt >= nb) return;
  Ticket tk = issue_batch(A, bt, batch);
  while (bt < nb) {
    const uint64_t bn = bt + gridDim.x;
    Ticket tkn{0, 0, 0};
    if (bn < nb) tkn = issue_batch(A, bn, batch);
    const int64_t r = wait_wg(A.c, tk);
    const uint64_t first = bt * batch;
    const uint32_t cnt = (uint32_t)min<uint64_t>(batch, A.n_items - first);
    const int64_t ret =
        threadIdx.x < cnt
            ? (r < 0 ? r : (int64_t)__hip_atomic_load(&A.lists[first + threadIdx.x].len_ret,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM))
            : 0;
    consume_items<WGMAX, par>(A, first, cnt, ret, lds, stage_addr(A, bt, batch, first));
    // the buffer of batch bt is reused by batch bt + 2 * grid, issued in the
    // next iteration: every lane must be done reading it first
    __syncthreads();
    bt = bn;
    tk = tkn;
  }
}

// Kernel-split form: the host has already read every item (section 2,
// Fig. 1 left); a plain kernel checksums staging.  rets[i] is the byte count
// of item i (<= 0: no bytes).
template <uint32_t WGMAX, uint32_t CH>
__global__ __launch_bounds__(WGMAX, WGMAX <= 256 ? 2 : 4) void fnv4k_consume(
    uint64_t staging, const int64_t* rets, uint64_t n_items, uint32_t item_bytes,
    uint64_t* out_fnv) {
  extern __shared__ __align__(16) uint8_t lds[];
  const uint32_t wave = threadIdx.x >> 6;
  for (uint64_t first = (uint64_t)blockIdx.x * blockDim.x; first < n_items;
       first += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t item = first + threadIdx.x;
    const bool valid = item < n_items;
    const int64_t ret = valid ? rets[item] : 0;
    const uint32_t nbytes = ret > 0 ? (uint32_t)min<int64_t>(ret, (int64_t)item_bytes) : 0u;
    const uint64_t row0 = staging + (first + (threadIdx.x & ~63u)) * (uint64_t)item_bytes;
    const uint64_t h = wave_fnv_t<CH>(row0, nbytes, item_bytes, lds + wave * Tile<CH>::kBytes);
    if (valid) out_fnv[item] = h;
  }
}

// The same for items of more than 512 bytes, mostly by many lanes each.  A
// step costs the same however short its items are, so short items are hashed by
// the chains.
//
// A wavefront takes a group of par_items items per round, at the stride of the
// launch.  First it looks at the lengths of its own items, 64 at a time: one
// load, which brings the first group's lengths too, and nothing to exchange
// with others.  Chains take one lane per item, so those 64 need not follow
// each other; and since every wavefront's items come from all over the launch,
// a region of short ones leaves none idle.  (With consecutive items for each
// wavefront the steps took 3 us longer: fewer memory channels at a time.)
//
// us for slots of 4 KiB in HBM, by the chains alone, many lanes alone, and
// this: 50,000 full 71, 60.5, 60.8; lengths up to 4,096 255, 78, 79; up to
// 1,000 74, 72, 40; up to 512 39, 72, 24; up to 100 9.8, 72, 8.2; half of them
// 0 68, 65, 66.  200,000 full 246, 242, 241; up to 4,096 582, 302, 257; up to
// 512 81, 277, 44; ascending lengths 148, 300, 212.
// LDS of a wavefront, for either way.
constexpr uint32_t kConsumeTile = std::max(kParTile, Tile<128>::kBytes);

struct ConsumeArgs {
  uint64_t staging;
  const int64_t* rets;
  uint64_t n_items;
  uint64_t* out_fnv;
  uint32_t item_bytes;
};

// A reduction over the lanes (0 must be its identity).
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr 1
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast 15
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast 31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  return wave_reduce(v, [](uint32_t a, uint32_t b) { return max(a, b); });
}

// Which of the up to 64 items of a look the chains hash, as a bit per group
// (the same in every lane).  `groups` of them hold items; len is the length of
// this lane's item (0 if there is none), part the lanes whose item is not full.
// Either all, or the groups whose items have at most 512 bytes, or none.
//
// Costs in ns, with two wavefronts on a SIMD: a step of a group, half as much
// again where not all of it is there; a byte of the chains while all items
// that are not empty go on, and once some have ended.
__device__ __forceinline__ uint64_t chain_groups(uint32_t item_bytes, uint32_t groups, uint32_t len,
                                                 uint64_t part) {
  constexpr uint32_t kStep = 3900, kAll = 25, kSome = 45;
  const uint32_t ilog = 6 - par_lanes_log2(item_bytes), lane = lane_id();
  const uint32_t most = wave_max(len);
  const uint32_t least = min(~wave_max(len ? ~len : 0u), most) & ~255u;
  uint32_t steps = groups;
  if (ilog == 0 && most > kStepBytes)
    steps = wave_reduce(lane < groups ? max(1u, (len + kStepBytes - 1) / kStepBytes) : 0u,
                        [](uint32_t a, uint32_t b) { return a + b; });
  const uint32_t ragged = min(steps, (uint32_t)__popcll(part));
  if (kAll * least + kSome * (most - least) < kStep * steps + kStep / 2 * ragged) return ~0ull;
  // lanes with longer items, then groups with any
  uint64_t big = __ballot(len > kParMinItem);
  for (uint32_t k = 0; k < ilog; ++k) big |= big >> (1u << k);
  const uint64_t small = __ballot(lane < groups && !((big >> (lane << ilog)) & 1ull));
  const uint32_t top = wave_max((small >> (lane >> ilog)) & 1ull ? len : 0u);
  return kSome * top < (kStep + kStep / 2) * (uint32_t)__popcll(small) ? small : 0ull;
}

__global__ __launch_bounds__(kParBlock, 2) void fnv4k_consume_par(ConsumeArgs A) {
  extern __shared__ __align__(16) uint8_t lds[];
  const uint32_t lane = lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t ilog = 6 - par_lanes_log2(A.item_bytes), items = 1u << ilog;
  const uint64_t first = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wave) << ilog;
  const uint64_t step = ((uint64_t)gridDim.x * (blockDim.x >> 6)) << ilog;
  uint8_t* tile = lds + wave * kConsumeTile;
  auto len_of = [&](uint64_t i) {
    const int64_t r = A.rets[i];
    return r > 0 ? (uint32_t)min<int64_t>(r, (int64_t)A.item_bytes) : 0u;
  };
  auto len_or_0 = [&](uint64_t i) { return i < A.n_items ? len_of(i) : 0u; };
  auto store = [&](uint64_t i, uint64_t h) { A.out_fnv[i] = h; };
  // A look is at 64 >> ilog rounds; lane l has item l mod `items` of the
  // l >> ilog-th of them.  (The launch has at most kConsumeRounds.)
  uint64_t many = 0;  // bit j: many lanes hash the group of round j
  bool chained = false;
  uint64_t i = first + (uint64_t)(lane >> ilog) * step + (lane & (items - 1u));
  uint32_t coming = len_or_0(i);
  const uint32_t len0 = coming;  // (the first group's in the first lanes)
  uint32_t round = 0;
  for (uint64_t g0 = first; g0 < A.n_items; g0 += step << (6 - ilog), round += 64u >> ilog) {
    const uint64_t at = i;
    const bool there = at < A.n_items;
    const uint32_t len = coming;
    i += step << (6 - ilog);
    coming = len_or_0(i);
    const uint64_t part = __ballot(there && len < A.item_bytes);
    // groups that hold items: those whose first one is there
    const uint64_t has = __ballot(lane < (64u >> ilog) && g0 + lane * step < A.n_items);
    uint64_t chains = 0;
    if (__builtin_expect(part != 0, 0))
      chains = chain_groups(A.item_bytes, (uint32_t)__popcll(has), len, part);
    if (__builtin_expect(chains != 0, 0)) {
      const bool mine = there && ((chains >> (lane >> ilog)) & 1ull);
      const uint64_t g = A.staging + g0 * A.item_bytes;
      const uint64_t h = wave_fnv_rows<128>(
          [&](uint32_t r) {
            return g + ((uint64_t)(r >> ilog) * step + (r & (items - 1u))) * A.item_bytes;
          },
          mine ? len : 0u, A.item_bytes, tile);
      if (mine) store(at, h);
      chained = true;
    }
    many |= (has & ~chains) << round;
  }
  if (__builtin_expect(!chained, 1)) {
    wave_fnv_par(A.staging, A.item_bytes, first, len0, A.n_items, tile, len_of,
                 [&](uint64_t i) { return i + step; }, store);
    return;
  }
  many = uniform64(many);
  if (!many) return;
  const uint32_t skip = (uint32_t)__builtin_ctzll(many);
  const uint64_t begin = first + skip * step;
  many >>= skip;
  wave_fnv_par(
      A.staging, A.item_bytes, begin, len_or_0(begin + lane), A.n_items, tile, len_of,
      [&](uint64_t i) -> uint64_t {  // bit 0 of `many` is i's round
        many >>= 1;
        if (!many) return A.n_items;
        const uint32_t s = (uint32_t)__builtin_ctzll(many);
        many >>= s;
        return i + (s + 1) * step;
      },
      store);
}

__global__ void zero_words(unsigned long long* p, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace gsys_k

// ---------------------------------------------------------------- host side
using namespace gsys_k;

int gsys_fnv4k(gsys_ctx* ctx, int fd, uint64_t offsets, uint64_t n_items, uint32_t item_bytes,
               uint64_t staging, uint64_t staging_bytes, uint64_t lists, uint64_t out_fnv,
               uint64_t out_ret, uint32_t cell, uint32_t form, uint32_t wg_size, void* stream) {
  if (!ctx) return -EINVAL;
  if (!n_items) return 0;
  if (item_bytes == 0 || item_bytes % 64 || item_bytes > (1u << 20)) return -EINVAL;
  if (!(wg_size == 64 || wg_size == 128 || wg_size == 256 || wg_size == 512 || wg_size == 1024))
    return -EINVAL;
  if (!offsets || !out_fnv || !out_ret) return -EINVAL;
  if (n_items > (1ull << 32)) return -EINVAL;
  const uint64_t stage_bytes = n_items * (uint64_t)item_bytes;
  if (!staging_bytes) staging_bytes = stage_bytes;
  if (gsys_internal::check_host_range(ctx, staging, staging_bytes)) return -EFAULT;
  const bool persistent = form == GSYS_PERSISTENT || form == GSYS_GRAPH;
  const uint64_t batch_bytes = (uint64_t)wg_size * item_bytes;
  if (staging_bytes < stage_bytes && (!persistent || staging_bytes < 2 * batch_bytes))
    return -EINVAL;
  if (gsys_internal::check_host_range(ctx, lists, n_items * sizeof(gsys_iodesc))) return -EFAULT;

  FnvArgs A;
  if (int e = gsys_device_ctx(ctx, &A.c)) return e;
  A.offsets = (const uint64_t*)offsets;
  A.n_items = n_items;
  A.staging = staging;
  A.lists = (gsys_iodesc*)lists;
  A.out_fnv = (uint64_t*)out_fnv;
  A.out_ret = (int64_t*)out_ret;
  A.ks = (KState*)gsys_internal::kstate(ctx);
  A.fd = fd;
  A.item_bytes = item_bytes;
  A.ring = 0;
  {
    // Strong work-group cells aggregate their descriptor list in LDS before
    // one wavefront copies it out; GSYS_LDS_LISTS=0 has every work-item write
    // its own descriptor to host memory instead (measured equal, within 1%,
    // on the full sweep: the host pool, not the list, bounds these cells)
    const char* e = getenv("GSYS_LDS_LISTS");
    A.lds_list = (e && *e == '0') ? 0u : 1u;
  }
  A.wg = wg_size;
  A.batch = wg_size;
  hipStream_t s = (hipStream_t)stream;
  bool par = false;  // many lanes per item
  bool small = wg_size <= 256;  // the chain variant's block: see chunk_for
  uint32_t block = wg_size;
  auto lds_for = [&](uint32_t threads) {
    return par ? (threads / 64) * kParTile + A.wg * 4
               : (threads / 64) * (small ? Tile<256>::kBytes : Tile<128>::kBytes);
  };

  if (form == GSYS_PERSISTENT || form == GSYS_GRAPH) {
    // Lists of at most 256 items and 256 KiB, or of one larger item: one
    // service thread runs a list, so the first bytes cross the link a list's
    // service time after the start and the last list is hashed after the link
    // is done.  A launch of few items takes shorter ones still, at least 128
    // (two per work-group of the default grid) so that every service thread has
    // several, down to 64 KiB.
    // End to end (with a drain about 40 us longer than today's), 1 GiB in 4 KiB
    // items: 20.2 ms with 1 MiB lists, 20.1 with 512 KiB, 19.9 with 256 KiB,
    // 20.0 with 128 KiB; 5,003 items: 585 us with 1 MiB, 495 with 256 KiB, 485
    // with 128 KiB, 494 with 64 KiB, 554 with 32 KiB.
    A.batch = std::min(wg_size, 256u);
    while (A.batch > 1 && (uint64_t)A.batch * item_bytes > 262144) A.batch = (A.batch + 1) / 2;
    while (A.batch > 1 && n_items < 128ull * A.batch && (uint64_t)A.batch * item_bytes > 65536)
      A.batch = (A.batch + 1) / 2;
    A.wg = A.batch;
    const uint64_t nb = (n_items + A.batch - 1) / A.batch;
    // Eight wavefronts hash a list sooner, four leave the link and the pool
    // more to the others: 25,000 items of 4 KiB (391 lists) take 2.03 against
    // 2.08 ms, 60,000 (938) 4.63 either way, 262,144 19.9 either way.
    par = item_bytes > kParMinItem;
    block = par && nb <= 1024 ? kParBlock : 256;
    small = true;
    const uint32_t lds = lds_for(block);
    const void* kp = par ? (const void*)fnv4k_persistent<kParBlock, true>
                         : (const void*)fnv4k_persistent<256, false>;
    uint32_t grid = gsys_internal::resident_grid(ctx, kp, block, lds);
    if (grid == 0) return -ENODEV;
    if ((uint64_t)grid > nb) grid = (uint32_t)nb;
    const uint32_t req = gsys_internal::persistent_grid_override(ctx);
    if (req && req < grid) grid = req;
    // waiting work-groups poll host memory: no more of them than keep the
    // host pool and the link busy
    if (!req && grid > kPersistentGrid) grid = kPersistentGrid;
    if (staging_bytes < stage_bytes) {
      // staging ring: two batch buffers per resident work-group
      A.ring = 1;
      const uint64_t fit = staging_bytes / (2ull * A.batch * item_bytes);
      if ((uint64_t)grid > fit) grid = (uint32_t)fit;
    }
    void* args[] = {&A};
    if (form == GSYS_GRAPH) {
      const uint64_t key = gsys_internal::hash_words({0xF4Bull, (uint64_t)kp, grid, block, lds});
      const gsys_internal::KLaunch k{kp, dim3(grid), dim3(block), lds, args};
      return gsys_internal::launch_graph(ctx, key, &k, 1, s);
    }
    return gsys_internal::launch(ctx, kp, grid, block, lds, args, s);
  }

  const uint32_t gran = GSYS_CELL_GRAN(cell);
  const bool strong = (cell & GSYS_CELL_STRONG) != 0;
  const bool blocking = (cell & GSYS_CELL_BLOCKING) != 0;
  // Helper wavefronts share the items of the work-group after a barrier, so
  // of a work-group with several calling wavefronts none hashes before the
  // last call of all is done: more than 64 work-item calls per work-group (a
  // launch that fills the compute units) go without.  60,000 of 4 KiB in
  // work-groups of 256: 6.2 ms without, 6.9 with.
  const uint32_t cus = gsys_internal::cu_count(ctx);
  if (gran == GSYS_GRAN_WI && item_bytes > kParMinItem) {
    A.wg = spread_group(n_items, item_bytes, wg_size, cus, A.c.ring_mask + 1);
    par = A.wg <= 64 || many_lanes(n_items, item_bytes, A.wg, A.wg);
    block = A.wg > 64 ? A.wg : helped_block(64, ceil_div(n_items, A.wg), cus);
  } else if (gran != GSYS_GRAN_WI && item_bytes > kParMinItem) {
    const uint32_t helped = helped_block(wg_size, ceil_div(n_items, wg_size), cus);
    par = many_lanes(n_items, item_bytes, wg_size, helped);
    if (par) block = helped;
  }
  const uint64_t grid64 = (n_items + A.wg - 1) / A.wg;
  if (grid64 > 0x7fffffffull) return -EINVAL;
  const uint32_t grid = (uint32_t)grid64;
  const void* k = nullptr;
#define GSYS_PLAIN_K(G_, O_, B_)                                                   \
  (par     ? (const void*)fnv4k_plain<G_, O_, B_, kParBlock, true>                 \
   : small ? (const void*)fnv4k_plain<G_, O_, B_, 256, false>                      \
           : (const void*)fnv4k_plain<G_, O_, B_, 1024, false>)
  if (gran == GSYS_GRAN_WI) {
    if (!strong) return -EINVAL;  // work-item calls are implicitly strong
    k = blocking ? GSYS_PLAIN_K(G::WorkItem, O::Strong, B::Blocking)
                 : GSYS_PLAIN_K(G::WorkItem, O::Strong, B::NonBlocking);
  } else if (gran == GSYS_GRAN_WG) {
    if (strong)
      k = blocking ? GSYS_PLAIN_K(G::WorkGroup, O::Strong, B::Blocking)
                   : GSYS_PLAIN_K(G::WorkGroup, O::Strong, B::NonBlocking);
    else
      k = blocking ? GSYS_PLAIN_K(G::WorkGroup, O::Relaxed, B::Blocking)
                   : GSYS_PLAIN_K(G::WorkGroup, O::Relaxed, B::NonBlocking);
  } else if (gran == GSYS_GRAN_KERNEL) {
    if (strong) return -EINVAL;  // kernel calls are relaxed only
    if (stage_bytes > 0xffffffffull) return -EINVAL;  // descriptor offsets are 32-bit
    k = blocking ? GSYS_PLAIN_K(G::Kernel, O::Relaxed, B::Blocking)
                 : GSYS_PLAIN_K(G::Kernel, O::Relaxed, B::NonBlocking);
    // fresh per-launch state for the kernel-granularity call site
    if (gsys_internal::no_device(ctx)) return -ENODEV;
    hipLaunchKernelGGL(zero_words, dim3(1), dim3(64), 0, s, (unsigned long long*)A.ks,
                       (uint32_t)(sizeof(KState) / 8));
    if (hipGetLastError() != hipSuccess) return -ENODEV;
  } else {
    return -EINVAL;
  }
#undef GSYS_PLAIN_K
  void* args[] = {&A};
  return gsys_internal::launch(ctx, k, grid, block, lds_for(block), args, s);
}

int gsys_fnv4k_consume(gsys_ctx* ctx, uint64_t staging, uint64_t rets, uint64_t n_items,
                       uint32_t item_bytes, uint64_t out_fnv, uint32_t wg_size, uint32_t grid,
                       void* stream) {
  if (!ctx) return -EINVAL;
  if (!n_items) return 0;  // the outputs are empty and may be null
  if (!staging || !rets || !out_fnv) return -EINVAL;
  if (item_bytes == 0 || item_bytes % 64 || item_bytes > (1u << 20)) return -EINVAL;
  if (!(wg_size == 64 || wg_size == 128 || wg_size == 256 || wg_size == 512 || wg_size == 1024))
    return -EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const uint32_t cus = gsys_internal::cu_count(ctx);
  const bool many = grid ? consume_many_lanes(n_items, item_bytes, wg_size, grid, cus)
                         : consume_many_lanes(n_items, item_bytes);
  if (many) {
    // grid 0: four wavefronts per work-group, each with work, as many as run
    // at once; otherwise the caller's grid of wg_size work-items each, two
    // work-groups of 512 for one of 1,024 (whose registers are too few)
    if (gsys_internal::no_device(ctx)) return -ENODEV;
    const uint32_t block = grid ? std::min(wg_size, kParBlock) : 256;
    const uint64_t blocks = (uint64_t)grid * (wg_size / block);
    const uint32_t lds = (block / 64) * kConsumeTile;
    const void* k = (const void*)fnv4k_consume_par;
    const uint64_t nb = ceil_div(n_items, (uint64_t)(block / 64) * par_items(item_bytes));
    if (!grid) {
      grid = gsys_internal::resident_grid(ctx, k, block, lds);
      if (!grid) return -ENODEV;
      grid = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(grid, ceil_div(nb, kConsumeRounds)),
                                          0x7fffffffu);
    } else {
      grid = (uint32_t)std::min<uint64_t>(blocks, 0x7fffffffu);
    }
    if (grid > nb) grid = (uint32_t)nb;
    ConsumeArgs A{staging, (const int64_t*)rets, n_items, (uint64_t*)out_fnv, item_bytes};
    void* args[] = {&A};
    return gsys_internal::launch(ctx, k, grid, block, lds, args, s);
  }
  void* args[] = {&staging, &rets, &n_items, &item_bytes, &out_fnv};
  const uint64_t nb = (n_items + wg_size - 1) / wg_size;
  if (!grid || grid > nb) grid = (uint32_t)std::min<uint64_t>(nb, 0x7fffffffull);
  const bool small = wg_size <= 256;
  const uint32_t lds = (wg_size / 64) * (small ? Tile<256>::kBytes : Tile<128>::kBytes);
  const void* k = small ? (const void*)fnv4k_consume<256, 256> : (const void*)fnv4k_consume<1024, 128>;
  return gsys_internal::launch(ctx, k, grid, wg_size, lds, args, s);
}
