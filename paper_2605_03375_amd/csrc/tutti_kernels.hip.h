// Device code of libtutti for gfx950 (wave64).  Included once, by tutti_api.hip.
//
// Kernels
//   k_layout        one workgroup: extents of all requests by a prefix scan
//   k_sqe           submission entries from extents, four lanes per 64-byte entry
//   k_move          pack / unpack between paged blocks and objects, extents given
//   k_move_lds      the same for head-major pools with short rows and more blocks than k_move's line tiles can number
//                   (and for the measurement build): token tile transposed in LDS
//   k_layer         one layer's restore (or save) in one launch: scan + entries + unpack (or pack)
//   k_layer_lds     the same with the LDS-staged transpose
//   k_sgl_table     direct-to-block mode: the pool's mapping table, one 16-byte descriptor per block
//   k_sqe_direct    one entry per (hit block, K|V), naming the block's descriptor: no staging copy
//   k_ring_init, k_iocb_fill, k_issue_io, k_complete, k_cq_check
//                   SQ/CQ rings: IOCBs filled by the GPU, the entry-driven I/O kernel, completions
//   k_layer_ring    one layer through the rings in one launch: scan + IOCB fill + the blocks' I/O
//   k_copy, k_stream, k_scatter, k_scatter_piece   (measurement build only) plain copy, one-direction streams and
//                   copies with one side permuted at a given granularity: ceilings and floors for the above
//   k_table_validate  debugging aid: ids in range and no id twice, by all-pairs comparison (no workspace)
//   k_bitmap_clear, k_table_validate_bitmap   the same check in linear time with one bit per pool block
//
// A workgroup first puts the per-request offsets into LDS (from the extents, or by redoing the scan; a fused launch of
// one request needs neither), then walks work items with a persistent grid-stride loop, so the grid can be any size: the
// whole GPU, or a few compute units' worth when the caller sets a CU budget.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "launch_rules.h"
#include "layer_call.h"
#include "tutti.h"

namespace tutti {

constexpr uint32_t kWave = 64;
constexpr uint32_t kWgThreads = 256;         // whole-GPU launches: 8 such workgroups per CU
constexpr uint32_t kBudgetWgThreads = 1024;  // CU-budgeted launches: one 16-wave workgroup per budgeted CU

// Wavefronts per SIMD the register allocator must leave room for: the whole-GPU grids are sized for eight
// 256-thread workgroups per CU being resident at once (a kernel that needs more than 64 VGPRs would hold only
// seven, and the persistent workgroups beyond that would run after the others: a tail).  Asked for where it
// costs no scratch: 256-thread kernels with at most four 16-byte units in flight per lane.
constexpr int min_waves_per_simd(int wg_threads, int units) { return (wg_threads == 256 && units <= 4) ? 8 : 4; }

// Requests a kernel is for: one, up to 64, any number; ...Ahead: several whose slices are read behind the loads of the counts,
// under the scan (a pack's by preload_pack).
// ...Counted: a pack whose slices are read when the counts have been summed.
constexpr int kOne = 1, kFew = 2, kMany = 3, kFewAhead = 4, kManyAhead = 5, kFewCounted = 6, kManyCounted = 7;
constexpr bool counts_first(int reqs) { return reqs == kFewCounted || reqs == kManyCounted; }
constexpr bool reads_under_scan(int reqs) { return reqs == kFewAhead || reqs == kManyAhead || counts_first(reqs); }
constexpr bool any_number(int reqs) { return reqs == kMany || reqs == kManyAhead || reqs == kManyCounted; }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A wave-uniform 32-bit value moved to a scalar register.
__device__ __forceinline__ uint32_t rfl(uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(v)); }

// Wave-uniform words (counts, block ids, visiting order) are fetched through the scalar (constant) path: one s_load per
// wavefront, counted apart from the vector loads and stores in flight: it neither queues behind them nor waits for them.
typedef const __attribute__((address_space(4))) uint32_t *const_u32_ptr;
__device__ __forceinline__ const_u32_ptr as_const(const uint32_t *p) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
  return (const_u32_ptr)p;
#pragma clang diagnostic pop
}

// NT is a bit mask: bit 0 = non-temporal loads, bit 1 = non-temporal stores.
template <int NT>
__device__ __forceinline__ u32x4 ld16(const unsigned char *p) {
  if (NT & 1) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  return *reinterpret_cast<const u32x4 *>(p);
}
template <int NT>
__device__ __forceinline__ void st16(unsigned char *p, u32x4 v) {
  if (NT & 2)
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p));
  else
    *reinterpret_cast<u32x4 *>(p) = v;
}


// ------------------------------------------------------------------------------------------
// Per-request offsets in LDS.  Laid out in the dynamic LDS block as
//   u64 stage_off[R] | u64 obj_bytes[R] | u32 table_off[R+1] | u32 sqe_base[R+1]
// with the totals in the two sentinel slots.  24*R + 8 bytes.
// blk_off[r] is the number of blocks of the requests before r that the call moves: the copy loops number their
// work items by it.  When the library computed the extents itself it is the table offset (same array); a copy
// kernel that was handed extents keeps it in the sqe_base array, which it has no other use for.
// The direct-to-block mode has no use for sqe_base and keeps `wraps` there: not 0 if the requests' blocks sum to 2^32 or
// more.  table_off, which is not cut at the table's length in that mode, then starts again from 0 somewhere and is not in
// order.
// ------------------------------------------------------------------------------------------
struct ReqLds {
  uint64_t *stage_off;
  uint64_t *obj_bytes;
  uint32_t *table_off;
  uint32_t *sqe_base;
  uint32_t *blk_off;
  __device__ __forceinline__ uint32_t &wraps() const { return sqe_base[0]; }
  bool unordered;  // the same, in a register: set behind the scan for more than 64 requests
};

__device__ __forceinline__ ReqLds carve_lds(unsigned char *smem, uint32_t n_req, bool caller_extents = false) {
  ReqLds l;
  l.stage_off = reinterpret_cast<uint64_t *>(smem);
  l.obj_bytes = l.stage_off + n_req;
  l.table_off = reinterpret_cast<uint32_t *>(l.obj_bytes + n_req);
  l.sqe_base = l.table_off + n_req + 1;
  l.blk_off = caller_extents ? l.sqe_base : l.table_off;
  l.unordered = false;
  return l;
}

__host__ __device__ constexpr uint32_t req_lds_bytes(uint32_t n_req) { return 24u * n_req + 8u; }

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, uint32_t src) {
  uint32_t lo = __shfl(static_cast<uint32_t>(v), src, kWave);
  uint32_t hi = __shfl(static_cast<uint32_t>(v >> 32), src, kWave);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Inclusive prefix sums over the wavefront (all 64 lanes take part), by data-parallel-primitive moves: within rows of
// 16 lanes by shifts of 1, 2, 4 and 8, then the last lane of a row broadcast to the row (or rows) behind it.  A move
// is one VALU instruction; the same steps through __shfl_up are LDS permutes of 64+ cycles each.  Only the first `active`
// lanes' sums are right: two requests take one step instead of six, each with 64-bit adds for up to three sums (64 blocks
// of 32 KiB in 2 requests: restore 4.1 -> 3.9 us, save 4.1 -> 3.9; 512 of 4 KiB: retrieve 7.0 -> 6.7).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_0(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_or_0(uint64_t v) {
  return (static_cast<uint64_t>(dpp_or_0<CTRL, ROWS>(static_cast<uint32_t>(v >> 32))) << 32) |
         dpp_or_0<CTRL, ROWS>(static_cast<uint32_t>(v));
}
// SAT: sums that would pass 2^32 - 1 stay there (min(sum, 2^32 - 1) is associative, so any order of adding agrees).
template <bool SAT, typename S>
__device__ __forceinline__ S add_(S a, S b) {
  return SAT ? __builtin_elementwise_add_sat(a, b) : a + b;
}
template <bool SAT, typename S>
__device__ __forceinline__ S wave_scan(S v, uint32_t active = kWave) {
  if (active <= 1) return v;
  v = add_<SAT>(v, dpp_or_0<0x111, 0xf>(v));  // row_shr:1
  if (active <= 2) return v;
  v = add_<SAT>(v, dpp_or_0<0x112, 0xf>(v));  // row_shr:2
  if (active <= 4) return v;
  v = add_<SAT>(v, dpp_or_0<0x114, 0xf>(v));  // row_shr:4
  if (active <= 8) return v;
  v = add_<SAT>(v, dpp_or_0<0x118, 0xf>(v));  // row_shr:8
  if (active <= 16) return v;
  v = add_<SAT>(v, dpp_or_0<0x142, 0xa>(v));  // row_bcast:15 into rows 1 and 3
  if (active <= 32) return v;
  v = add_<SAT>(v, dpp_or_0<0x143, 0xc>(v));  // row_bcast:31 into rows 2 and 3
  return v;
}

// The wavefront's sum of a count per lane (0 in the lanes from n_req on), 2^32 - 1 if it is that or more.
__device__ __forceinline__ uint32_t sum_of_counts(uint32_t n, uint32_t n_req) {
  const uint32_t sums = wave_scan<true>(n, n_req);
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sums), static_cast<int>(n_req - 1)));
}

// The file store of the direct-to-block mode: file f at base + (f - first_file_id)*file_stride.
struct FileArgs {
  uint64_t file_stride;
  uint32_t first_file_id;
  uint32_t n_files;
};

constexpr uint64_t kNoFile = ~0ull;

struct ScanGeom {
  uint32_t block_bytes;
  uint32_t align;       // power of two
  uint32_t chunk_bytes; // multiple of align
};

// Bytes of a request's object beyond its blocks (align is a power of two, so 32 bits of the product suffice), and its
// submission entries: ceil(obj / chunk_bytes), in 32 bits where the object is that small (the 64-bit division is ten
// times the instructions).
__device__ __forceinline__ uint32_t obj_pad(const ScanGeom &g, uint32_t n) {
  return (0u - n * g.block_bytes) & (g.align - 1);
}
__device__ __forceinline__ uint64_t obj_chunks(const ScanGeom &g, uint64_t obj) {
  if (obj <= 0xffffffffull - (g.chunk_bytes - 1u))
    return (static_cast<uint32_t>(obj) + (g.chunk_bytes - 1u)) / g.chunk_bytes;
  return (obj + g.chunk_bytes - 1) / g.chunk_bytes;
}

// What the per-request staging slot holds: the offset of the K object in the staging buffer or, in the direct-to-block
// mode, the start of the request's file in the store (kNoFile if the store has no such file).
__device__ __forceinline__ uint64_t stage_slot(uint64_t stage_off, const uint32_t *file_id, uint32_t fid,
                                               const FileArgs &files) {
  if (!file_id) return stage_off;
  const uint32_t rel = fid - files.first_file_id;
  return fid >= files.first_file_id && rel < files.n_files ? static_cast<uint64_t>(rel) * files.file_stride : kNoFile;
}

// Extents of all requests, by the whole workgroup; results go to LDS and, when ext_out != nullptr, to global memory.
// Ends with a barrier.
// In the staged mode (file_id == nullptr) the requests are taken in order while the running sum of
// their blocks stays within table_len: the request that pushes it beyond, and every later one, gets no
// work items (its LDS table offset is the cut, so it owns no blocks) and TUTTI_ST_BAD_EXTENT is reported
// by the workgroup that publishes.  The published extents are the plain sums either way.
//
// Up to 64 requests: one wavefront, a request per lane (a single request needs no scan at all); n and fid: the block
// count and file id of the lane's request.
__device__ __forceinline__ void wave_scan_extents(const ScanGeom g, uint32_t n, uint32_t fid, uint32_t n_req,
                                                  uint32_t lane, ReqLds l, tutti_extent *__restrict__ ext_out,
                                                  uint64_t *__restrict__ totals_out, uint32_t table_len,
                                                  uint32_t *__restrict__ status, bool with_chunks,
                                                  const uint32_t *__restrict__ file_id, const FileArgs files) {
  const uint32_t r = lane;
  const uint64_t obj = static_cast<uint64_t>(n) * g.block_bytes + obj_pad(g, n);
  // a workgroup that only moves blocks never reads the entry bases: it skips the division
  const uint64_t chunks = with_chunks ? obj_chunks(g, obj) : 0;
  uint64_t inc_stage = 2 * obj, inc_sqe = 2 * chunks, inc_tab = n;
  inc_stage = wave_scan<false>(inc_stage, n_req);
  if (with_chunks) inc_sqe = wave_scan<false>(inc_sqe, n_req);
  inc_tab = wave_scan<false>(inc_tab, n_req);
  const bool beyond = !file_id && r < n_req && inc_tab > table_len;
  const uint64_t beyond_mask = __ballot(beyond);
  uint32_t cut_total = 0;  // blocks of the requests in front of the first that runs beyond the table
  if (beyond_mask != 0) {
    const uint32_t first = static_cast<uint32_t>(__ffsll(static_cast<long long>(beyond_mask))) - 1u;
    cut_total = static_cast<uint32_t>(shfl_u64(inc_tab - n, first));
  }
  if (r < n_req) {
    const uint64_t stage_off = inc_stage - 2 * obj;
    const uint32_t sqe_base = static_cast<uint32_t>(inc_sqe - 2 * chunks);
    const uint32_t table_off = static_cast<uint32_t>(inc_tab - n);
    l.stage_off[r] = stage_slot(stage_off, file_id, fid, files);
    l.obj_bytes[r] = obj;
    l.table_off[r] = beyond ? cut_total : table_off;
    l.sqe_base[r] = sqe_base;
    if (ext_out) {
      tutti_extent e;
      e.stage_off = stage_off;
      e.obj_bytes = obj;
      e.n_blocks = n;
      e.n_chunks = static_cast<uint32_t>(chunks);
      e.sqe_base = sqe_base;
      e.table_off = table_off;
      ext_out[r] = e;
    }
    if (r + 1 == n_req) {
      l.table_off[n_req] = beyond_mask != 0 ? cut_total : static_cast<uint32_t>(inc_tab);
      l.sqe_base[n_req] = static_cast<uint32_t>(inc_sqe);
      if (file_id) l.wraps() = inc_tab > 0xffffffffu ? 1u : 0u;
      if (totals_out) {
        totals_out[0] = inc_stage;
        totals_out[1] = inc_sqe;
      }
    }
  }
  if (n_req == 0 && lane == 0) {
    l.table_off[0] = l.sqe_base[0] = 0;
    if (totals_out) totals_out[0] = totals_out[1] = 0;
  }
  if (lane == 0 && beyond_mask != 0 && totals_out && status) atomicOr(status, TUTTI_ST_BAD_EXTENT);
}

// More than 64 requests: every thread takes a run of consecutive requests (at most TUTTI_MAX_REQ / WG), whose block
// counts it loads at once; one scan of the threads' sums per wavefront, the wavefronts' totals through LDS.  The runs
// replace 64 requests per pass on one wavefront, each pass a load, a chain of LDS permutes and a carry behind the pass
// before: a save of 512 requests of 1..4 blocks (8 KiB blocks, 42 MB of traffic) took 18.2 us that way and takes 10.6.
// All workgroups scan all requests, so the instructions count too: a workgroup that only moves blocks (EXACT = false)
// carries two 32-bit sums, blocks and padding bytes, from which the staging offset follows (2 * (blocks * block_bytes
// + padding)).  The block sums of the staged mode saturate, which is as good as exact: every offset that is used lies
// within table_len, and the host keeps 2 * table_len within 32 bits.  The others (the entry writers and the publishing
// workgroup; align > 1 MiB, where the padding of 2048 requests may need more bits; the direct-to-block mode, whose
// offsets wrap) carry 64-bit sums and the chunks.
// KEEP: the counts stay in LDS (in sqe_base, which such a workgroup has no use for) instead of being read again, because the
// bytes that `counted` requests are on their way by then, and loads arrive in order.
template <int WG, bool EXACT, bool SAT, bool KEEP, typename P, typename C>
__device__ __forceinline__ void wg_scan_extents(const ScanGeom g, const uint32_t *__restrict__ n_blocks, uint32_t n_req,
                                                ReqLds l, tutti_extent *__restrict__ ext_out,
                                                uint64_t *__restrict__ totals_out, uint32_t table_len,
                                                uint32_t *__restrict__ status, const uint32_t *__restrict__ file_id,
                                                const FileArgs files, P preload, C counted) {
  typedef typename std::conditional<EXACT, uint64_t, uint32_t>::type S;
  constexpr uint32_t kPer = TUTTI_MAX_REQ / WG, kWaves = WG / kWave;
  static_assert(3 * kWaves <= kWave, "the wavefronts' totals fit the staging-offset slots of 65 requests");
  const uint32_t lane = threadIdx.x & (kWave - 1), wave = rfl(threadIdx.x / kWave);
  const uint32_t per = (n_req + WG - 1) / WG, r0 = threadIdx.x * per;
  S blocks = 0, pads = 0, chunks = 0;
  {
    uint32_t n[kPer];  // all loads in flight together; the loops below read the counts again (from the L1 cache), which
                       // keeps these registers free for the bytes that a restore has in flight meanwhile
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) n[k] = (k < per && r0 + k < n_req) ? n_blocks[r0 + k] : 0u;
    __builtin_amdgcn_sched_barrier(0);
    preload();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      blocks = add_<SAT>(blocks, static_cast<S>(n[k]));
      pads += obj_pad(g, n[k]);
      if (KEEP && k < per && r0 + k < n_req) l.sqe_base[r0 + k] = n[k];
    }
  }
  if (EXACT) {
#pragma unroll 1
    for (uint32_t k = 0; k < per && r0 + k < n_req; ++k) {
      const uint32_t n = n_blocks[r0 + k];
      chunks += obj_chunks(g, static_cast<uint64_t>(n) * g.block_bytes + obj_pad(g, n));
    }
  }
  const S blocks_in = wave_scan<SAT>(blocks), pads_in = wave_scan<false>(pads);
  const S chunks_in = EXACT ? wave_scan<false>(chunks) : 0;
  uint64_t *part = l.stage_off;  // the slots are written behind the second barrier
  if (lane == kWave - 1) {
    part[wave] = blocks_in;
    part[kWaves + wave] = pads_in;
    if (EXACT) part[2 * kWaves + wave] = chunks_in;
  }
  __syncthreads();
  // sums in front of this thread's run: of the lanes before it (a scan result moved on by one lane, because a saturated
  // sum cannot be subtracted from) and of the wavefronts before it
  S t = dpp_or_0<0x138, 0xf>(blocks_in), t_all = 0;  // wave_shr:1
  S p = pads_in - pads, p_all = 0, c = chunks_in - chunks, c_all = 0;
#pragma unroll
  for (uint32_t w = 0; w < kWaves; ++w) {
    const S pt = static_cast<S>(part[w]), pp = static_cast<S>(part[kWaves + w]);
    const S pc = EXACT ? static_cast<S>(part[2 * kWaves + w]) : 0;
    t_all = add_<SAT>(t_all, pt);
    p_all += pp;
    c_all += pc;
    if (w < wave) {
      t = add_<SAT>(t, pt);
      p += pp;
      c += pc;
    }
  }
  if (KEEP) counted(static_cast<uint32_t>(t_all));
  __syncthreads();
  const bool cut = !file_id && t_all > table_len;  // the same in every thread
  uint32_t cut_total = 0;
  if (cut) {
    S x = t;
#pragma unroll 1
    for (uint32_t k = 0; k < per && r0 + k < n_req; ++k) {  // exactly one request starts within the table and ends beyond it
      const S next = add_<SAT>(x, static_cast<S>(KEEP ? l.sqe_base[r0 + k] : n_blocks[r0 + k]));
      if (x <= table_len && next > table_len) l.table_off[n_req] = static_cast<uint32_t>(x);
      x = next;
    }
    __syncthreads();
    cut_total = l.table_off[n_req];
  }
#pragma unroll 1
  for (uint32_t k = 0; k < per && r0 + k < n_req; ++k) {
    const uint32_t r = r0 + k, n = KEEP ? l.sqe_base[r] : n_blocks[r];
    const uint32_t pad = obj_pad(g, n);
    const uint64_t obj = static_cast<uint64_t>(n) * g.block_bytes + pad;
    const uint64_t stage_off = 2 * (static_cast<uint64_t>(t) * g.block_bytes + p);
    const S next = add_<SAT>(t, static_cast<S>(n));
    l.stage_off[r] = stage_slot(stage_off, file_id, file_id ? file_id[r] : 0u, files);
    l.obj_bytes[r] = obj;
    l.table_off[r] = cut && next > table_len ? cut_total : static_cast<uint32_t>(t);
    if (EXACT) {
      const uint64_t n_chunks = obj_chunks(g, obj);
      const uint32_t sqe_base = static_cast<uint32_t>(2 * c);
      if (!file_id) l.sqe_base[r] = sqe_base;
      if (ext_out) {
        tutti_extent e;
        e.stage_off = stage_off;
        e.obj_bytes = obj;
        e.n_blocks = n;
        e.n_chunks = static_cast<uint32_t>(n_chunks);
        e.sqe_base = sqe_base;
        e.table_off = static_cast<uint32_t>(t);
        ext_out[r] = e;
      }
      c += n_chunks;
    }
    t = next;
    p += pad;
  }
  if (threadIdx.x == 0) {
    if (!cut) l.table_off[n_req] = static_cast<uint32_t>(t_all);
    if (EXACT) {
      l.sqe_base[n_req] = static_cast<uint32_t>(2 * c_all);
      if (file_id) l.wraps() = t_all > 0xffffffffu ? 1u : 0u;
      if (totals_out) {
        totals_out[0] = 2 * (static_cast<uint64_t>(t_all) * g.block_bytes + p_all);
        totals_out[1] = 2 * c_all;
        if (cut && status) atomicOr(status, TUTTI_ST_BAD_EXTENT);
      }
    }
  }
}

// with_chunks: the workgroup writes entries or publishes (ext_out, totals_out): it needs the chunk counts as well.
// `preload` requests a first slice's bytes, so that they are on their way during the scan.  Up to 64 requests: in front
// of the loads of the counts, which return behind the scanning wavefront's slice, so that no wavefront of the workgroup
// stores before (see hold_back).  More requests: behind the scan (600 requests, 49 MB: 20.3 us against 22.0 in front of
// it); in the 64-bit scan (a few workgroups of a launch) not at all, it leaves no registers.
// REQS = kFew: the host knows of at most 64 requests.  A kernel of its own, because the other scans' arguments push the
// scalar registers over their limit, and the kernel then starts with more rounds of argument loads and spills (what that
// gives stands at few_requests).
// Kernels that read under the scan: `preload` is called behind the loads of the counts, so that the scan need not wait for it,
// and, where they count first, `counted` with the requests' blocks (2^32 - 1 if there are more) once they are summed.  In the
// 64-bit scan neither is called.
template <int WG, int REQS, typename P, typename C>
__device__ __forceinline__ void scan_extents(const ScanGeom g, const uint32_t *__restrict__ n_blocks, uint32_t n_req,
                                             ReqLds l, tutti_extent *__restrict__ ext_out,
                                             uint64_t *__restrict__ totals_out, uint32_t table_len,
                                             uint32_t *__restrict__ status, bool with_chunks,
                                             const uint32_t *__restrict__ file_id, const FileArgs files, P preload,
                                             C counted) {
  if (REQS == kFew || REQS == kFewAhead || REQS == kFewCounted || (REQS == kMany && n_req <= kWave)) {
    uint32_t n = 0, fid = 0;
    // (to sum the counts every wavefront needs them, the same few words as the one before it: the cache has them)
    const uint32_t r = REQS == kFewCounted ? threadIdx.x & (kWave - 1) : threadIdx.x;
    const auto load_counts = [&] {
      if (r < n_req) {
        n = n_blocks[r];
        if (file_id) fid = file_id[r];
      }
    };
    if (reads_under_scan(REQS)) {
      load_counts();
      __builtin_amdgcn_sched_barrier(0);
      preload();
      __builtin_amdgcn_sched_barrier(0);
    } else {
      preload();
    }
    if (counts_first(REQS)) counted(sum_of_counts(n, n_req));
    if (threadIdx.x < kWave) {
      // In here and not in front: as far as the compiler can tell every wavefront has them on their way there, behind the slice
      // that it reads ahead, and waits for all of that where their registers are used next, before it works out where its slice
      // goes.  Restores with no pause to hide that, 32 KiB blocks in 200 requests, us, in front / here: 512 blocks 13.6 / 13.0,
      // 640 16.3 / 16.0, 1024 23.7 / 23.5; of line tiles, 512 blocks, 14.1 / 13.4.
      if (!reads_under_scan(REQS)) load_counts();
      wave_scan_extents(g, n, fid, n_req, threadIdx.x, l, ext_out, totals_out, table_len, status, with_chunks, file_id,
                        files);
    }
  } else if (with_chunks || file_id || g.align > (1u << 20)) {
    wg_scan_extents<WG, true, false, false>(g, n_blocks, n_req, l, ext_out, totals_out, table_len, status, file_id, files,
                                           [] {}, [](uint32_t) {});
  } else {
    wg_scan_extents<WG, false, true, counts_first(REQS)>(g, n_blocks, n_req, l, nullptr, nullptr, table_len, status, nullptr, files,
                                           [&] {
                                             if (reads_under_scan(REQS)) preload();
                                           },
                                           counted);
    if (!reads_under_scan(REQS)) preload();
  }
  __syncthreads();
}

// Per-request offsets for the entry builders, from extents the caller already has (workgroup-wide, with
// barriers).  The entry builders number entries by sqe_base (or by twice table_off in the direct-to-block mode)
// and take a request's chunk and block counts from the differences of consecutive offsets, which is right for
// extents as tutti_obj_layout writes them for exactly these requests: offsets running from 0 without gaps, sizes
// that follow from n_blocks.  That is checked here, every request against its successor; the result is the same
// in every workgroup.  Returns false (after reporting TUTTI_ST_BAD_EXTENT once) if the extents are anything else:
// the caller then writes nothing.
template <int WG>
__device__ __forceinline__ bool lds_from_extents(const tutti_extent *__restrict__ ext, uint32_t n_req, ReqLds l,
                                                 const ScanGeom g, uint32_t *__restrict__ status) {
  // Called by workgroups of WG threads: thread t holds requests t, t + WG, ... (at most kPer of them).  The loop is
  // fully unrolled so that a thread's loads are all in flight together; a request's successor sits in the next
  // lane, and for the last lane of a wavefront in LDS once the barrier has been crossed.  Every workgroup of an
  // entry builder runs this over all requests, so its instruction count matters when there are thousands of
  // both: the host then launches few, large workgroups (entry_launch in the host code).
  constexpr uint32_t kPer = TUTTI_MAX_REQ / WG;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  bool bad = false;
  uint32_t nx_sqe[kPer], nx_tab[kPer];
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    const uint32_t r = k * WG + threadIdx.x;
    tutti_extent e;
    e.stage_off = e.obj_bytes = 0;
    e.n_blocks = e.n_chunks = e.sqe_base = e.table_off = 0;
    if (r < n_req) e = ext[r];
    uint64_t next_sqe = 0, next_tab = 0;
    if (r < n_req) {
      l.stage_off[r] = e.stage_off;
      l.obj_bytes[r] = e.obj_bytes;
      l.table_off[r] = e.table_off;
      l.sqe_base[r] = e.sqe_base;
      const uint64_t raw = static_cast<uint64_t>(e.n_blocks) * g.block_bytes;
      const uint64_t obj = (raw + (g.align - 1)) & ~static_cast<uint64_t>(g.align - 1);
      // n_chunks == ceil(obj / chunk_bytes), without the 64-bit division: c*chunk >= obj > (c-1)*chunk
      const uint32_t c = e.n_chunks;
      const bool chunks_ok = obj == 0 ? c == 0
                                      : (c >= 1 && static_cast<uint64_t>(c) * g.chunk_bytes >= obj &&
                                         static_cast<uint64_t>(c - 1) * g.chunk_bytes < obj);
      bad = bad || e.obj_bytes != obj || !chunks_ok;
      // 64-bit sums: offsets that would wrap around 32 bits are not dense either
      next_sqe = static_cast<uint64_t>(e.sqe_base) + 2ull * e.n_chunks;
      next_tab = static_cast<uint64_t>(e.table_off) + e.n_blocks;
      bad = bad || next_sqe > 0xffffffffull || next_tab > 0xffffffffull;
      if (r == 0) bad = bad || e.sqe_base != 0 || e.table_off != 0;
      if (r + 1 == n_req) {
        l.table_off[n_req] = static_cast<uint32_t>(next_tab);
        l.sqe_base[n_req] = static_cast<uint32_t>(next_sqe);
      }
    }
    nx_sqe[k] = static_cast<uint32_t>(next_sqe);
    nx_tab[k] = static_cast<uint32_t>(next_tab);
    // the successor's offsets, from the next lane (every lane takes part in the exchange)
    const uint32_t f_sqe = static_cast<uint32_t>(__shfl_down(static_cast<int>(e.sqe_base), 1, kWave));
    const uint32_t f_tab = static_cast<uint32_t>(__shfl_down(static_cast<int>(e.table_off), 1, kWave));
    if (r + 1 < n_req && lane != kWave - 1) bad = bad || f_sqe != nx_sqe[k] || f_tab != nx_tab[k];
  }
  if (n_req == 0 && threadIdx.x == 0) {
    l.table_off[0] = 0;
    l.sqe_base[0] = 0;
  }
  __syncthreads();  // publishes the LDS writes above
  if (lane == kWave - 1) {
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t r = k * WG + threadIdx.x;
      if (r + 1 < n_req) bad = bad || l.sqe_base[r + 1] != nx_sqe[k] || l.table_off[r + 1] != nx_tab[k];
    }
  }
  __shared__ uint32_t bad_waves[WG / kWave];
  const bool bad_wave = __ballot(bad) != 0;
  if (lane == 0) bad_waves[threadIdx.x / kWave] = bad_wave ? 1u : 0u;
  __syncthreads();
  bool any_bad = false;
#pragma unroll
  for (uint32_t w = 0; w < WG / kWave; ++w) any_bad = any_bad || bad_waves[w] != 0;
  if (any_bad && blockIdx.x == 0 && threadIdx.x == 0 && status) atomicOr(status, TUTTI_ST_BAD_EXTENT);
  return !any_bad;
}

// Per-request offsets for the copy kernels, from extents the caller hands in: every field is honoured as it
// stands (a gap between requests, any order in the staging buffer, a table range that does not start at 0), and
// what cannot be honoured is taken out here, once, so that the copy loop never sees it:
//   - requests are taken in order while the running sum of n_blocks stays within table_len; the request that
//     pushes it beyond and every later one get no work items (TUTTI_ST_BAD_EXTENT);
//   - a request whose stage_off or obj_bytes is not a multiple of 16 (TUTTI_ST_BAD_EXTENT), or whose two objects
//     do not fit in stage_cap (TUTTI_ST_STAGE_CAP), keeps its work items but gets a zero-sized object, so the
//     copy loop skips every block of it;
//   - blocks that would end beyond their object are skipped by the copy loop (TUTTI_ST_BAD_EXTENT).
// All threads stage the raw fields, then the first wavefront scans n_blocks (64 requests per pass) into
// blk_off[], the numbering of the work items.  Workgroup 0 reports.
template <int WG>
__device__ __forceinline__ void lds_from_caller_extents(const tutti_extent *__restrict__ ext, uint32_t n_req, ReqLds l,
                                                        uint32_t table_len, uint32_t block_bytes, uint64_t stage_cap,
                                                        uint32_t *__restrict__ status) {
  for (uint32_t r = threadIdx.x; r < n_req; r += WG) {
    const tutti_extent e = ext[r];
    l.stage_off[r] = e.stage_off;
    l.obj_bytes[r] = e.obj_bytes;
    l.table_off[r] = e.table_off;
    l.blk_off[r] = e.n_blocks;  // replaced by its exclusive prefix sum below
  }
  __syncthreads();
  if (threadIdx.x < kWave) {
    const uint32_t lane = threadIdx.x;
    uint64_t carry = 0;
    bool cut_found = false;
    uint32_t cut_total = 0, flags = 0;
    for (uint32_t base = 0; base < n_req; base += kWave) {
      const uint32_t r = base + lane;
      const uint32_t active = n_req - base < kWave ? n_req - base : kWave;
      const uint32_t n = r < n_req ? l.blk_off[r] : 0u;
      const uint64_t incl = carry + wave_scan<false>(static_cast<uint64_t>(n), active);
      const bool beyond = r < n_req && incl > table_len;
      const uint64_t beyond_mask = __ballot(beyond);
      if (!cut_found && beyond_mask != 0) {
        const uint32_t first = static_cast<uint32_t>(__ffsll(static_cast<long long>(beyond_mask))) - 1u;
        cut_total = static_cast<uint32_t>(shfl_u64(incl - n, first));
        cut_found = true;
      }
      if (r < n_req) {
        const uint64_t so = l.stage_off[r], ob = l.obj_bytes[r];
        bool dead = true;
        if (beyond)
          flags |= TUTTI_ST_BAD_EXTENT;
        else if (((so | ob) & 15u) != 0)
          flags |= TUTTI_ST_BAD_EXTENT;
        else if (so > stage_cap || ob > (stage_cap - so) / 2)
          flags |= TUTTI_ST_STAGE_CAP;
        else {
          dead = false;
          if (static_cast<uint64_t>(n) * block_bytes > ob) flags |= TUTTI_ST_BAD_EXTENT;
        }
        if (dead) {
          l.stage_off[r] = 0;
          l.obj_bytes[r] = 0;
        }
        l.blk_off[r] = beyond ? cut_total : static_cast<uint32_t>(incl - n);
      }
      carry = shfl_u64(incl, active - 1);
    }
    if (lane == 0) l.blk_off[n_req] = cut_found ? cut_total : static_cast<uint32_t>(carry);
    if (flags != 0 && blockIdx.x == 0 && status) atomicOr(status, flags);
  }
  __syncthreads();
}

// Largest r in [0, n) with a[r] <= key, for a non-decreasing a with a[0] <= key.  Empty
// requests share their offset with the next one, so the answer is never an empty request
// when key is below the total.
__device__ __forceinline__ uint32_t find_owner(const uint32_t *a, uint32_t n, uint32_t key) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (a[mid] <= key)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The same for a key that all lanes of the wavefront share (and all are active): every lane compares, a ballot counts.
// One read of LDS for up to 64 requests (FEW: there are no more) and two for more, instead of 6 to 11 that wait for each
// other.
// For offsets that may be out of order (the direct-to-block mode's, ReqLds::wraps) it makes find_owner's choice: a position
// may belong to several requests then, and the recorded contexts name that one.  Up to 64 requests need no flag for it: where
// the lanes that compare true are the first ones, without a gap, there is one place only where a search can end, and where
// they are not the same search runs over the ballot's bits.
template <bool FEW, bool DIRECT>
__device__ __forceinline__ uint32_t find_owner_of_wave(const ReqLds &l, const uint32_t *a, uint32_t n, uint32_t key) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  if (FEW) {
    const uint64_t below = __ballot(lane < n && a[lane] <= key);
    if (DIRECT && __builtin_expect((below & (below + 1)) != 0, 0)) {
      uint32_t lo = 0, hi = n;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((below >> mid & 1) != 0)
          lo = mid;
        else
          hi = mid;
      }
      return lo;
    }
    return static_cast<uint32_t>(__popcll(below)) - 1;
  }
  if (DIRECT && __builtin_expect(l.unordered, 0)) return find_owner(a, n, key);
  const uint32_t step = (n + kWave - 1) / kWave;  // at most TUTTI_MAX_REQ / 64
  uint32_t at = lane * step;
  const uint32_t first = (static_cast<uint32_t>(__popcll(__ballot(at < n && a[at] <= key))) - 1) * step;
  at = first + lane;
  return first + static_cast<uint32_t>(__popcll(__ballot(lane < step && at < n && a[at] <= key))) - 1;
}

// ------------------------------------------------------------------------------------------
// Submission entries.  Four consecutive lanes write the four 16-byte quarters of one 64-byte
// entry, so a wavefront's store covers 16 whole entries = 1 KiB of consecutive bytes.
// ------------------------------------------------------------------------------------------
struct SqeArgs {
  const uint32_t *file_id;
  tutti_sqe *sqe;
  uint32_t *status;
  uint64_t stage_addr;
  uint32_t sqe_cap;
  uint32_t chunk_bytes;
  uint32_t layer;
  uint32_t opcode;
  uint32_t sgl_id;
};

// Quarter `part` (16 bytes) of entry i, which belongs to request r whose file id is fid.
__device__ __forceinline__ u32x4 sqe_quarter(const SqeArgs &a, const ReqLds &l, uint32_t r, uint32_t i, uint32_t part,
                                             uint32_t fid) {
  const uint32_t base = l.sqe_base[r];
  const uint32_t n_chunks = (l.sqe_base[r + 1] - base) >> 1;
  const uint32_t v = i - base;
  const uint32_t kind = v >= n_chunks ? 1u : 0u;
  const uint32_t c = v - kind * n_chunks;
  const uint64_t obj = l.obj_bytes[r];
  const uint64_t in_obj = static_cast<uint64_t>(c) * a.chunk_bytes;
  u32x4 w = {0u, 0u, 0u, 0u};
  if (part == 0) {
    const uint64_t file_off = (2ull * a.layer + kind) * obj + in_obj;
    w.x = (a.opcode & 0xffu) | (kind << 8) | (a.layer << 16);
    w.y = fid;
    w.z = static_cast<uint32_t>(file_off);
    w.w = static_cast<uint32_t>(file_off >> 32);
  } else if (part == 1) {
    const uint64_t addr = a.stage_addr + l.stage_off[r] + kind * obj + in_obj;
    const uint64_t left = obj - in_obj;
    w.x = static_cast<uint32_t>(addr);
    w.y = static_cast<uint32_t>(addr >> 32);
    w.z = left < a.chunk_bytes ? static_cast<uint32_t>(left) : a.chunk_bytes;
    w.w = a.sgl_id;
  } else if (part == 2) {
    w.x = i;
    w.y = r;
    w.z = i / TUTTI_IOCB_SLOTS;
    w.w = i % TUTTI_IOCB_SLOTS;
  }
  return w;
}

// The entries of a layer are written by the `n_wgs` workgroups starting at workgroup `first_wg`, one lane per
// quarter.  A workgroup that also moves blocks splits the job: sqe_head, right after the scan, finds the owner
// of the lane's first quarter and requests its file id (the only value that comes from global memory);
// emit_sqes, after the copy loop, assembles and stores, so the load's latency is spent under the copy.
struct SqeHead {
  uint64_t q;    // the lane's first quarter
  uint32_t r;    // its request
  uint32_t fid;  // file id of that request (quarter 0 only)
  bool live;     // the lane has a first quarter
};

template <int WG>
__device__ __forceinline__ SqeHead sqe_head(const SqeArgs a, const ReqLds l, uint32_t n_req, uint32_t first_wg) {
  const uint32_t n_sqe = l.sqe_base[n_req];
  const uint32_t n_write = n_sqe < a.sqe_cap ? n_sqe : a.sqe_cap;
  SqeHead h;
  h.q = static_cast<uint64_t>(blockIdx.x - first_wg) * WG + threadIdx.x;
  h.live = h.q < 4ull * n_write;
  h.r = 0;
  h.fid = 0;
  if (h.live) {
    h.r = find_owner(l.sqe_base, n_req, static_cast<uint32_t>(h.q >> 2));
    if ((h.q & 3) == 0) h.fid = a.file_id[h.r];
  }
  return h;
}

template <int WG>
__device__ __forceinline__ void emit_sqes(const SqeArgs a, const ReqLds l, uint32_t n_req, uint32_t first_wg,
                                          uint32_t n_wgs, const SqeHead h) {
  const uint32_t n_sqe = l.sqe_base[n_req];
  const uint32_t n_write = n_sqe < a.sqe_cap ? n_sqe : a.sqe_cap;
  const uint32_t wg = blockIdx.x - first_wg;
  if (n_sqe > a.sqe_cap && wg == 0 && threadIdx.x == 0 && a.status) atomicOr(a.status, TUTTI_ST_SQE_CAP);
  if (!h.live) return;
  const uint64_t n_quarters = 4ull * n_write;
  const uint64_t stride = static_cast<uint64_t>(n_wgs) * WG;
  u32x4 *out = reinterpret_cast<u32x4 *>(a.sqe);
  const uint32_t part = static_cast<uint32_t>(h.q & 3);  // the stride is a multiple of 4: the same quarter every pass
  out[h.q] = sqe_quarter(a, l, h.r, static_cast<uint32_t>(h.q >> 2), part, h.fid);
  for (uint64_t q = h.q + stride; q < n_quarters; q += stride) {
    const uint32_t i = static_cast<uint32_t>(q >> 2);
    const uint32_t r = find_owner(l.sqe_base, n_req, i);
    out[q] = sqe_quarter(a, l, r, i, part, part == 0 ? a.file_id[r] : 0u);
  }
}

// ------------------------------------------------------------------------------------------
// Direct-to-block mode.  The mapping table holds one 16-byte descriptor per pool block; an entry
// then names the descriptor of the block it transfers instead of a staging address.
// ------------------------------------------------------------------------------------------
struct SglArgs {
  tutti_sgl *table;
  uint32_t *status;
  uint64_t k_addr;
  uint64_t v_addr;
  uint64_t block_stride;
  uint32_t num_blocks;
  uint32_t block_bytes;
  uint32_t sgl_id;
  uint32_t cap;
};

__global__ __launch_bounds__(kWgThreads) void k_sgl_table(const SglArgs a, uint32_t n_wgs) {
  const uint64_t n = 2ull * a.num_blocks;
  if (n > a.cap && blockIdx.x == 0 && threadIdx.x == 0 && a.status) atomicOr(a.status, TUTTI_ST_SQE_CAP);
  const uint64_t n_write = n < a.cap ? n : a.cap;
  const uint64_t stride = static_cast<uint64_t>(n_wgs) * kWgThreads;
  u32x4 *out = reinterpret_cast<u32x4 *>(a.table);
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kWgThreads + threadIdx.x; i < n_write; i += stride) {
    const bool v_plane = i >= a.num_blocks;
    const uint64_t b = v_plane ? i - a.num_blocks : i;
    const uint64_t addr = (v_plane ? a.v_addr : a.k_addr) + b * a.block_stride;
    u32x4 w;
    w.x = static_cast<uint32_t>(addr);
    w.y = static_cast<uint32_t>(addr >> 32);
    w.z = a.block_bytes;
    w.w = a.sgl_id;
    out[i] = w;  // a wavefront stores 64 descriptors = 1 KiB of consecutive bytes
  }
}

struct DirectArgs {
  const uint32_t *table;
  uint64_t sgl_table_addr;
  uint32_t table_len;
  uint32_t num_blocks;
  uint32_t block_bytes;
};

// Direct-mode entry i in two steps, so that the loads of the next entry can be in flight while the current one
// is assembled.  Step one: where the entry sits in its request, and the two values that come from global
// memory (the block id; the file id for the lane that writes the first quarter).
struct DirectLoc {
  uint32_t r, kind, j;
  uint32_t id;   // block id, or num_blocks when the table has no such position
  uint32_t fid;  // file id of the request (quarter 0 only)
};

__device__ __forceinline__ DirectLoc direct_locate(const SqeArgs &a, const DirectArgs &d, const ReqLds &l, uint32_t r,
                                                   uint32_t i, uint32_t part) {
  DirectLoc c;
  const uint32_t toff = l.table_off[r];
  const uint32_t n = l.table_off[r + 1] - toff;
  const uint32_t v = i - 2u * toff;
  c.r = r;
  c.kind = v >= n ? 1u : 0u;
  c.j = v - c.kind * n;
  const uint32_t tab_idx = toff + c.j;
  c.id = d.num_blocks;
  if (tab_idx < d.table_len) c.id = d.table[tab_idx];  // the four lanes of an entry read the same word
  c.fid = part == 0 ? a.file_id[r] : 0u;
  return c;
}

// Step two: quarter `part` (16 bytes) of the entry.  *bad is set for an id out of range.
__device__ __forceinline__ u32x4 direct_entry_quarter(const SqeArgs &a, const DirectArgs &d, const ReqLds &l,
                                                      const DirectLoc &c, uint32_t i, uint32_t part, bool *bad) {
  const bool ok = c.id < d.num_blocks;
  *bad = !ok;
  u32x4 w = {0u, 0u, 0u, 0u};
  if (part == 0) {
    const uint64_t file_off = (2ull * a.layer + c.kind) * l.obj_bytes[c.r] + static_cast<uint64_t>(c.j) * d.block_bytes;
    w.x = (a.opcode & 0xffu) | (c.kind << 8) | (a.layer << 16);
    w.y = c.fid;
    w.z = static_cast<uint32_t>(file_off);
    w.w = static_cast<uint32_t>(file_off >> 32);
  } else if (part == 1) {
    const uint64_t addr = ok ? d.sgl_table_addr + 16ull * (static_cast<uint64_t>(c.kind) * d.num_blocks + c.id) : 0ull;
    w.x = static_cast<uint32_t>(addr);
    w.y = static_cast<uint32_t>(addr >> 32);
    w.z = ok ? d.block_bytes : 0u;
    w.w = a.sgl_id;
  } else if (part == 2) {
    w.x = i;
    w.y = c.r;
    w.z = i / TUTTI_IOCB_SLOTS;
    w.w = i % TUTTI_IOCB_SLOTS;
  }
  return w;
}

// The request that owns block-table position `key`, found from the owner of an earlier (smaller) position:
// the offsets are non-decreasing, so walking forward gives what find_owner gives.
__device__ __forceinline__ uint32_t advance_owner(const uint32_t *table_off, uint32_t n_req, uint32_t r, uint32_t key) {
  while (r + 1 < n_req && table_off[r + 1] <= key) ++r;
  return r;
}

// Four lanes per entry, as in emit_sqes: a wavefront's store covers 16 whole entries.  The `n_wgs` workgroups
// starting at `first_wg` each take one contiguous run of entries (a whole number of 4 KiB workgroup stores), so a
// thread's consecutive entries are 64 apart and their owner is found by walking on from the previous one: one
// binary search per thread instead of one per entry.  The loop is pipelined by one entry: the table and file-id
// loads of the next entry are issued before the current one is assembled and stored; the first entry's are issued
// by direct_head, which a workgroup that also moves blocks calls before its copy loop.  `dst(i)` gives the
// address of entry i.
struct DirectHead {
  uint64_t q, end;  // the lane's first quarter and the end of its workgroup's run
  DirectLoc loc;    // that quarter's entry, located, with its loads requested
  bool live;
};

template <int WG>
__device__ __forceinline__ DirectHead direct_head(const SqeArgs a, const DirectArgs d, const ReqLds l, uint32_t n_req,
                                                  uint64_t n_write, uint32_t first_wg, uint32_t n_wgs) {
  const uint64_t n_quarters = 4ull * n_write;
  constexpr uint64_t per_pass = WG;  // quarters one workgroup writes per pass: 4 KiB for 256 threads
  const uint64_t passes = (n_quarters + per_pass * n_wgs - 1) / (per_pass * n_wgs);
  const uint64_t begin = static_cast<uint64_t>(blockIdx.x - first_wg) * passes * per_pass;
  DirectHead h;
  h.end = begin + passes * per_pass;
  if (h.end > n_quarters) h.end = n_quarters;
  h.q = begin + threadIdx.x;
  h.live = h.q < h.end;
  if (h.live) {
    const uint32_t i = static_cast<uint32_t>(h.q >> 2);
    h.loc = direct_locate(a, d, l, find_owner(l.table_off, n_req, i >> 1), i, static_cast<uint32_t>(h.q & 3));
  }
  return h;
}

template <int WG, typename Dst>
__device__ __forceinline__ void emit_direct_entries(const SqeArgs a, const DirectArgs d, const ReqLds l, uint32_t n_req,
                                                    const DirectHead h, Dst dst) {
  if (!h.live) return;
  constexpr uint64_t per_pass = WG;
  uint64_t q = h.q;
  uint32_t i = static_cast<uint32_t>(q >> 2);
  const uint32_t part = static_cast<uint32_t>(q & 3);  // per_pass is a multiple of 4: the same quarter every pass
  DirectLoc cur = h.loc;
  for (;;) {
    const uint64_t qn = q + per_pass;
    const bool more = qn < h.end;
    const uint32_t in = static_cast<uint32_t>(qn >> 2);
    DirectLoc nxt = cur;
    if (more) nxt = direct_locate(a, d, l, advance_owner(l.table_off, n_req, cur.r, in >> 1), in, part);
    bool bad = false;
    const u32x4 w = direct_entry_quarter(a, d, l, cur, i, part, &bad);
    if (bad && part == 0 && a.status) atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
    reinterpret_cast<u32x4 *>(dst(i))[part] = w;
    if (!more) break;
    q = qn;
    i = in;
    cur = nxt;
  }
}

template <int WG>
__device__ __forceinline__ void emit_direct_sqes(const SqeArgs a, const DirectArgs d, const ReqLds l, uint32_t n_req,
                                                 uint32_t n_wgs) {
  const uint64_t n_sqe = 2ull * l.table_off[n_req];
  const uint64_t n_write = n_sqe < a.sqe_cap ? n_sqe : a.sqe_cap;
  if (n_sqe > a.sqe_cap && blockIdx.x == 0 && threadIdx.x == 0 && a.status) atomicOr(a.status, TUTTI_ST_SQE_CAP);
  tutti_sqe *out = a.sqe;
  emit_direct_entries<WG>(a, d, l, n_req, direct_head<WG>(a, d, l, n_req, n_write, 0, n_wgs),
                          [out](uint32_t i) { return out + i; });
}

// ------------------------------------------------------------------------------------------
// Rings.  An SQ slot is an IOCB: 64-byte header + 2048 contexts.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kWgThreads) void k_ring_init(tutti_iocb *sq, tutti_cq_hdr *cq, uint32_t depth) {
  const uint32_t i = blockIdx.x * kWgThreads + threadIdx.x;
  if (i < depth) {
    u32x4 *h = reinterpret_cast<u32x4 *>(&sq[i].hdr);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const u32x4 first = {i, 0u, TUTTI_IOCB_FREE, 0u};
    h[0] = first;
    h[1] = zero;
    h[2] = zero;
    h[3] = zero;
    reinterpret_cast<uint32_t *>(cq + 1)[i] = 0xffffffffu;
  }
  if (i < 16) reinterpret_cast<uint32_t *>(cq)[i] = (i == 1) ? depth : 0u;
}

struct RingArgs {
  tutti_iocb *sq;
  tutti_cq_hdr *cq;
  uint32_t depth;
  uint32_t first_slot;
  uint32_t n_slots;
};

// Contexts of one layer dealt into IOCBs (see emit_direct_sqes for the entry itself), plus the headers, by the
// `n_wgs` workgroups starting at workgroup `first_wg`: iocb_head before a copy loop, emit_iocbs after it.
__device__ __forceinline__ uint64_t iocb_fill_count(const RingArgs &g, const ReqLds &l, uint32_t n_req) {
  const uint64_t n_ctx = 2ull * l.table_off[n_req];
  const uint64_t cap = static_cast<uint64_t>(g.n_slots) * TUTTI_IOCB_SLOTS;
  return n_ctx < cap ? n_ctx : cap;
}

template <int WG>
__device__ __forceinline__ DirectHead iocb_head(const RingArgs g, const SqeArgs a, const DirectArgs d, const ReqLds l,
                                                uint32_t n_req, uint32_t first_wg, uint32_t n_wgs) {
  return direct_head<WG>(a, d, l, n_req, iocb_fill_count(g, l, n_req), first_wg, n_wgs);
}

template <int WG>
__device__ __forceinline__ void emit_iocbs(const RingArgs g, const SqeArgs a, const DirectArgs d, const ReqLds l,
                                           uint32_t n_req, uint32_t first_wg, uint32_t n_wgs, const DirectHead h) {
  const uint64_t n_ctx = 2ull * l.table_off[n_req];
  const uint64_t cap = static_cast<uint64_t>(g.n_slots) * TUTTI_IOCB_SLOTS;
  const uint64_t n_fill = iocb_fill_count(g, l, n_req);
  const uint64_t tid = static_cast<uint64_t>(blockIdx.x - first_wg) * WG + threadIdx.x;
  if (n_ctx > cap && tid == 0 && a.status) atomicOr(a.status, TUTTI_ST_SQE_CAP);
  const uint64_t stride = static_cast<uint64_t>(n_wgs) * WG;
  for (uint64_t b = tid; b < g.n_slots; b += stride) {  // one thread per IOCB header
    const uint64_t lo = b * TUTTI_IOCB_SLOTS;
    uint64_t cnt = n_fill > lo ? n_fill - lo : 0;
    if (cnt > TUTTI_IOCB_SLOTS) cnt = TUTTI_IOCB_SLOTS;
    tutti_iocb_hdr *hd = &g.sq[(g.first_slot + b) % g.depth].hdr;
    hd->num_ioctx = static_cast<uint32_t>(cnt);
    hd->state = TUTTI_IOCB_FILLED;
    hd->done = 0;
    hd->layer = a.layer;
    hd->opcode = a.opcode;
  }
  const RingArgs ring = g;
  emit_direct_entries<WG>(a, d, l, n_req, h, [ring](uint32_t i) {
    return &ring.sq[(ring.first_slot + i / TUTTI_IOCB_SLOTS) % ring.depth].ioctx[i % TUTTI_IOCB_SLOTS];
  });
}

// The arguments of k_iocb_fill and k_issue_io, each once: 104 bytes, as separate records 172 and 132 (up to 112 bytes the runtime
// handles a launch faster: layer_call.h).  Trains of fills, issues and completions of 16 layers of 0.5 MiB, us a layer: reads
// 11.7 / 9.2, writes of 1.4 MiB 11.9 / 9.7; in processes whose heap happens to be in order 9.6 / 9.2, 10.2 / 9.7.
struct FillCall {
  tutti_iocb *sq;
  const uint32_t *file_id;
  uint32_t *status;
  const uint32_t *table;
  const tutti_extent *ext;
  uint64_t sgl_table_addr;
  uint32_t depth, first_slot, n_slots, layer, opcode, sgl_id, table_len, num_blocks;
  ScanGeom geom;
  uint32_t n_req, n_wgs;
};
static_assert(sizeof(FillCall) <= sizeof(LayerCall), "one of malloc's smallest chunks");

template <int WG>
__global__ __launch_bounds__(WG) void k_iocb_fill(const FillCall c) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RingArgs g{c.sq, nullptr, c.depth, c.first_slot, c.n_slots};
  const SqeArgs a{c.file_id, nullptr, c.status, 0, 0, c.geom.block_bytes, c.layer, c.opcode, c.sgl_id};
  const DirectArgs d{c.table, c.sgl_table_addr, c.table_len, c.num_blocks, c.geom.block_bytes};
  const ReqLds l = carve_lds(smem, c.n_req);
  if (!lds_from_extents<WG>(c.ext, c.n_req, l, c.geom, c.status)) return;
  emit_iocbs<WG>(g, a, d, l, c.n_req, 0, c.n_wgs, iocb_head<WG>(g, a, d, l, c.n_req, 0, c.n_wgs));
}

constexpr uint32_t kPiece = kWave * 16u;  // what one wavefront instruction of 16 bytes per lane covers: 1 KiB

constexpr int kWaitVmcnt0 = 0x0f70;  // operand of s_waitcnt: vector accesses done, the other counters as they are

// The value that lane `src` holds, in scalar registers.
__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, uint32_t src) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>(src)));
}
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, uint32_t src) {
  const uint32_t lo = readlane_u32(static_cast<uint32_t>(v), src);
  return (static_cast<uint64_t>(readlane_u32(static_cast<uint32_t>(v >> 32), src)) << 32) | lo;
}
typedef __attribute__((address_space(1))) unsigned char *global_u8_ptr;
__device__ __forceinline__ unsigned char *as_global(uint64_t address) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
  return (unsigned char *)(global_u8_ptr)address;  // a global pointer, so that the accesses are global ones
#pragma clang diagnostic pop
}

// Moves item i of a batch that the lanes have decoded: G parts of U/G KiB each, part g decoded by lane i * G + g.
// `len`: bytes of the lane's part (0 = skip it), `whole`: the lanes whose part is of full length; src(g, o), dst(g, o):
// the address o bytes into part g on either side (worked out where they are used: all at once they would not fit the
// registers).  U loads in flight, then U stores.  Where a part is short, the lanes beyond it load its first 16 bytes
// again and store nothing (src of a part to skip is any readable 16 bytes): guarded loads end in a wait each.
template <int U, int G, int NT, typename Src, typename Dst>
__device__ __forceinline__ void move_decoded(uint32_t i, uint64_t whole, uint32_t len, Src src, Dst dst) {
  constexpr uint32_t P = U / G;
  constexpr uint64_t kAll = (1ull << G) - 1;
  const uint32_t o = (threadIdx.x & (kWave - 1)) * 16u;
  u32x4 buf[U];
  if ((whole >> (i * G) & kAll) == kAll) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) buf[u] = ld16<NT>(src(u / P, o + u % P * kPiece));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) st16<NT>(dst(u / P, o + u % P * kPiece), buf[u]);
    asm volatile("; whole item");  // (the marks keep the compiler from merging the paths' last stores, which
                                   // would put a wait for all other stores in front of the merged one)
  } else {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t at = o + u % P * kPiece;
      buf[u] = ld16<NT>(src(u / P, at < readlane_u32(len, i * G + u / P) ? at : 0u));
    }
    // one wait for all loads: left to itself the compiler waits in front of each guarded store, and with that
    // for the stores before it (loads and stores share a counter)
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t at = o + u % P * kPiece;
      if (at < readlane_u32(len, i * G + u / P)) st16<NT>(dst(u / P, at), buf[u]);
    }
    asm volatile("; guarded item");
  }
}

// `v` in the lanes of `live`, the value of the first of them in the others.
__device__ __forceinline__ uint64_t or_first(uint64_t v, uint64_t live) {
  const uint64_t first = readlane_u64(v, static_cast<uint32_t>(__ffsll(static_cast<long long>(live))) - 1u);
  return (live >> (threadIdx.x & (kWave - 1)) & 1u) != 0 ? v : first;
}

struct IoArgs {
  const tutti_sgl *sgl;
  unsigned char *store_base;
  uint32_t *status;
  uint64_t sgl_table_addr;
  uint64_t file_stride;
  uint32_t n_desc;
  uint32_t first_file_id;
  uint32_t n_files;
  uint32_t max_len;
  uint32_t parts;  // per context: slices or pieces that cover max_len
};

struct IoCall {
  IoArgs io;
  tutti_iocb *sq;
  tutti_cq_hdr *cq;
  uint32_t depth, first_slot, n_slots, done_first, done_n, grid;
};
static_assert(sizeof(IoCall) <= sizeof(LayerCall), "one of malloc's smallest chunks");

// One part of one context, resolved: where its bytes come from and go to.
struct IoPart {
  uint64_t src, dst;
  uint32_t len;  // bytes of the part; 0: nothing to move (empty slot, no-op or rejected context, part beyond its length)
};

// Everything between a part's number and its two addresses: IOCB header and context, SGL descriptor, validity.
__device__ __forceinline__ IoPart io_decode(const RingArgs &g, const IoArgs &a, uint32_t ctx, uint32_t part,
                                            uint32_t part_bytes) {
  IoPart r;
  r.src = r.dst = 0;
  r.len = 0;
  const uint32_t b = ctx / TUTTI_IOCB_SLOTS, k = ctx % TUTTI_IOCB_SLOTS;
  const uint32_t slot = g.first_slot + b;  // below 2 * depth: the host checked first_slot < depth and n_slots <= depth
  const tutti_iocb *io = &g.sq[slot < g.depth ? slot : slot - g.depth];
  const u32x4 *h = reinterpret_cast<const u32x4 *>(&io->hdr);  // iocb_idx, num_ioctx, state, done
  const u32x4 *e = reinterpret_cast<const u32x4 *>(&io->ioctx[k]);
  // Contexts of one or two parts: header and context in one round trip, whether or not the context is submitted (the slot
  // holds all of them); left to itself the compiler moves the context's loads behind the header's check (128 blocks of 4
  // KiB 9.4 us instead of 9.0).  A larger context would be read once for each of its parts, also where nothing was
  // submitted (3 blocks of 128 KiB, cold, 10.1 us instead of 9.5): those wait for the header.
  const bool together = a.parts <= 2;
  u32x4 hdr, q0, q1;
  if (together) {
    hdr = h[0];
    q0 = e[0];
    q1 = e[1];
    asm volatile("" : "+v"(hdr), "+v"(q0), "+v"(q1));
  } else {
    hdr = h[0];
  }
  if (hdr.z != TUTTI_IOCB_FILLED || k >= hdr.y) return r;  // nothing submitted in this slot / position
  if (!together) {
    q0 = e[0];
    q1 = e[1];
  }
  const uint32_t opcode = q0.x & 0xffu, file_id = q0.y, len = q1.z;
  const uint64_t file_off = (static_cast<uint64_t>(q0.w) << 32) | q0.z;
  const uint64_t addr = (static_cast<uint64_t>(q1.y) << 32) | q1.x;
  if (len == 0) return r;  // a no-op context
  bool ok = (opcode == TUTTI_OP_READ || opcode == TUTTI_OP_WRITE) && addr >= a.sgl_table_addr &&
            ((addr - a.sgl_table_addr) & 15u) == 0 && len <= a.max_len && (len & 15u) == 0 && (file_off & 15u) == 0;
  const uint64_t di = ok ? (addr - a.sgl_table_addr) >> 4 : 0;
  ok = ok && di < a.n_desc;
  uint64_t blk_addr = 0;
  if (ok) {
    const u32x4 dsc = *reinterpret_cast<const u32x4 *>(&a.sgl[di]);
    blk_addr = (static_cast<uint64_t>(dsc.y) << 32) | dsc.x;
    ok = len <= dsc.z && (blk_addr & 15u) == 0;
  }
  ok = ok && file_id >= a.first_file_id && file_id - a.first_file_id < a.n_files &&
       file_off + len <= a.file_stride && file_off + len >= file_off;
  if (!ok) {
    if (part == 0 && a.status) atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
    return r;
  }
  const uint32_t in_ctx = part * part_bytes;
  if (in_ctx >= len) return r;  // the context is shorter than max_len: this part holds none of it
  const uint64_t blk = blk_addr + in_ctx;
  const uint64_t fil = reinterpret_cast<uint64_t>(a.store_base) +
                       static_cast<uint64_t>(file_id - a.first_file_id) * a.file_stride + file_off + in_ctx;
  r.src = opcode == TUTTI_OP_READ ? fil : blk;
  r.dst = opcode == TUTTI_OP_READ ? blk : fil;
  r.len = len - in_ctx < part_bytes ? len - in_ctx : part_bytes;
  return r;
}

__device__ __forceinline__ void complete_iocbs(const RingArgs g, uint32_t lane);  // defined below

// The I/O kernel: no inter-wave communication.  A context is cut into slices of U KiB or, where those do not fill
// max_len exactly, into pieces of 1 KiB; a work item is one slice or U consecutive pieces, moved by one wavefront.  A
// wavefront resolves its next 64 slices or pieces at once, one per lane: the three dependent loads behind each (header
// and context together, then the descriptor) are paid once per batch, with all lanes' loads in flight together and no
// data loads in front of them; resolved item by item they queue behind the current item's data.  On 32 compute units
// (33.5 MB to write from 32 KiB blocks) that and the 16 KiB slices took the kernel from 49 us to 42 us.  On the whole GPU a
// wavefront has one item or few, and the decode is paid in full: fill, issue and completion of 128 4 KiB blocks 9.0 us.
// Completion is published by k_complete, enqueued right behind it on the same stream: counting finished items with
// atomics on the IOCB header serialises on one address (measured: 1.5 ms per 4096-context layer instead of 55 us), and
// a kernel boundary already is the "all contexts done" event.
// `done`: IOCBs that an earlier launch on the same stream has executed; when done.n_slots is not 0 the grid has one
// workgroup more, in front, whose first wavefront completes them and leaves (see k_layer_ring).
template <int U, int WG, bool PIECES>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_issue_io(const IoCall call) {
  const RingArgs g{call.sq, call.cq, call.depth, call.first_slot, call.n_slots};
  const RingArgs done{call.sq, call.cq, call.depth, call.done_first, call.done_n};
  const IoArgs a = call.io;
  const uint32_t grid = call.grid;
  constexpr uint32_t G = PIECES ? U : 1, kBatch = kWave / G;  // parts of an item, items decoded at once
  constexpr uint32_t kPart = PIECES ? kPiece : U * kPiece;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t lead = done.n_slots != 0 ? 1u : 0u;
  if (lead && blockIdx.x == 0) {
    if (threadIdx.x < kWave) complete_iocbs(done, threadIdx.x);
    return;
  }
  const uint32_t wgs = grid - lead, wg = blockIdx.x - lead, wave = rfl(threadIdx.x / kWave);
  const uint32_t n_waves = wgs * (WG / kWave);
  const uint64_t n_parts = static_cast<uint64_t>(g.n_slots) * TUTTI_IOCB_SLOTS * a.parts;
  const uint32_t n_items = static_cast<uint32_t>((n_parts + G - 1) / G);  // the host checked this fits 32 bits

  // (as first_item: a budgeted launch deals neighbouring items to neighbouring workgroups)
  for (uint64_t it = WG == kWgThreads ? wg * (WG / kWave) + wave : wave * wgs + wg; it < n_items;
       it += kBatch * static_cast<uint64_t>(n_waves)) {
    IoPart d;
    d.src = d.dst = 0;
    d.len = 0;
    const uint64_t mine = it + static_cast<uint64_t>(lane / G) * n_waves;
    if (mine * G + lane % G < n_parts) {
      // part number / parts per context without a 64-bit division (see move_pieces)
      const uint32_t q = static_cast<uint32_t>(mine) / a.parts;
      const uint32_t rest = (static_cast<uint32_t>(mine) - q * a.parts) * G + lane % G;
      const uint32_t q2 = PIECES ? rest / a.parts : 0;
      d = io_decode(g, a, q * G + q2, rest - q2 * a.parts, kPart);
    }
    const uint64_t live = __ballot(d.len != 0), whole = __ballot(d.len == kPart);
    if (live == 0) continue;
    d.src = or_first(d.src, live);
#pragma unroll 1
    for (uint32_t i = 0; i < kBatch && live >> (i * G) != 0; ++i) {
      constexpr uint64_t kAll = (1ull << G) - 1;
      if ((live >> (i * G) & kAll) == 0) continue;
      move_decoded<U, G, 3>(
          i, whole, d.len, [&](uint32_t p, uint32_t o) { return as_global(readlane_u64(d.src, i * G + p)) + o; },
          [&](uint32_t p, uint32_t o) { return as_global(readlane_u64(d.dst, i * G + p)) + o; });
    }
  }
}

// Completion of the IOCBs an I/O kernel has executed: FILLED -> DONE, done = num_ioctx, index appended to the CQ
// in slot order.  Run by ONE wavefront (lane = its lane id) once every store of the I/O is visible to it: the
// k_complete kernel enqueued behind the I/O kernel (stream order).  Doing it inside the I/O kernel instead, by
// whichever workgroup finishes last (each workgroup releasing its stores at agent scope and counting itself in
// on a two-level tree of counters), was built and measured: 153 us per layer against 50 + 4: an agent-scope
// release writes back the XCD's whole L2, and 2048 workgroups each pay for one.  The CQ tail is only ever
// advanced here, so no read-modify-write atomics are needed within a stream.  A ring (or just its CQ) placed in pinned
// host memory can be polled by the CPU while the stream runs on: a state and its finished count are one 8-byte store, they
// and the queue entries are written through to system scope, and all have arrived (one wait) before the tail is written.
// Whoever sees a state sees its count, whoever sees the new tail the entries and states before it.  Bound by its dependent
// round trips (headers, states, tail) and, as a kernel of its own, by the launch.  There is no release: it would write back
// the XCD's L2, which in a train of layers is full of the next layer's blocks, and costs a round trip more.  Us, with one
// release in front of the states / without: retrieve of 16 blocks of 32 KiB 5.97 / 5.67, of 2048 46.3 / 46.0; a read of 50
// blocks of 4 KiB a layer, 8 layers, 68.4 / 66.2; tutti_complete_io of 200 slots 3.2 / 2.4.
__device__ __forceinline__ void complete_iocbs(const RingArgs g, uint32_t lane) {
  uint32_t *cq_entry = reinterpret_cast<uint32_t *>(g.cq + 1);
  uint32_t tail = g.cq->tail;  // every lane reads the same word
  // one lane per IOCB, 64 per pass (the host checked n_slots <= depth, so the slots are distinct): the header
  // loads of a pass are in flight together, and a ballot gives each executed IOCB its place in the queue
  for (uint32_t base = 0; base < g.n_slots; base += kWave) {
    const uint32_t b = base + lane;
    tutti_iocb_hdr *h = nullptr;
    u32x4 hdr = {0u, 0u, TUTTI_IOCB_FREE, 0u};  // iocb_idx, num_ioctx, state, done
    if (b < g.n_slots) {
      const uint32_t slot = g.first_slot + b;  // below 2 * depth, as in io_decode
      h = &g.sq[slot < g.depth ? slot : slot - g.depth].hdr;
      hdr = *reinterpret_cast<const u32x4 *>(h);
    }
    const bool live = hdr.z == TUTTI_IOCB_FILLED;
    const uint64_t mask = __ballot(live);
    const uint32_t before = static_cast<uint32_t>(__popcll(mask & ((1ull << lane) - 1ull)));
    if (live) {
      __hip_atomic_store(&cq_entry[(tail + before) % g.depth], hdr.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(reinterpret_cast<uint64_t *>(h) + 1, (static_cast<uint64_t>(hdr.y) << 32) | TUTTI_IOCB_DONE,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    tail += static_cast<uint32_t>(__popcll(mask));
  }
  // what was written through has arrived when the wavefront's stores are done (the wavefront runs in step, so lane 0's
  // store is issued after the other lanes' wait)
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  __builtin_amdgcn_wave_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (lane == 0) __hip_atomic_store(&g.cq->tail, tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kWave) void k_complete(const RingArgs g) {
  if (blockIdx.x != 0) return;
  complete_iocbs(g, threadIdx.x);
}

// wait_cqe for n slots from `slot` on (wrapping at depth): flag[i] <- 1 if IOCB (slot + i) % depth is DONE, else 0.
__global__ __launch_bounds__(kWgThreads) void k_cq_check(const tutti_iocb *sq, uint32_t depth, uint32_t slot, uint32_t n,
                                                          uint32_t *flag, uint32_t n_wgs) {
  for (uint32_t i = blockIdx.x * kWgThreads + threadIdx.x; i < n; i += n_wgs * kWgThreads) {
    const uint32_t st =
        __hip_atomic_load(&sq[(slot + i) % depth].hdr.state, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    flag[i] = st == TUTTI_IOCB_DONE ? 1u : 0u;
  }
}

template <int WG>
__global__ __launch_bounds__(WG) void k_sqe_direct(const SqeArgs a, const DirectArgs d, const ScanGeom geom,
                                                            const tutti_extent *__restrict__ ext, uint32_t n_req,
                                                            uint32_t n_wgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, n_req);
  if (!lds_from_extents<WG>(ext, n_req, l, geom, a.status)) return;
  emit_direct_sqes<WG>(a, d, l, n_req, n_wgs);
}

// ------------------------------------------------------------------------------------------
// Pack / unpack.  A work item is one slice of one (block, K|V): kSliceUnits*1 KiB, moved by one
// wavefront with 16-byte accesses per lane (1 KiB per wavefront instruction, whole cache lines
// on both sides).  Items are numbered in staging-buffer order (request, K then V, block, slice),
// so neighbouring wavefronts stream neighbouring object bytes while the pool side jumps from
// block to block as the table says.
// Blocks that are no whole number of slices are cut into pieces instead: 1 KiB, what one wavefront instruction covers
// (the last of a block may be shorter), and an item is U consecutive pieces, which may belong to different blocks.
// A block of 12.5 KiB is 13 pieces instead of four slices of which the last moves 512 of its 4096 bytes; four blocks
// of 1 KiB are one item instead of four.  (Where a launch is bound by how soon its first bytes move rather than by how many
// are on their way, such blocks are cut into equal slices all the same: cuts_blocks.)
// ------------------------------------------------------------------------------------------
struct MoveArgs {
  unsigned char *k_base;
  unsigned char *v_base;
  unsigned char *stage;
  const uint32_t *table;
  uint32_t *status;
  uint64_t block_stride;
  uint64_t stage_cap;
  uint32_t num_blocks;
  uint32_t block_bytes;
  uint32_t table_len;
  uint32_t slices_per_block;  // slices, pieces or (through LDS) tiles
  // head-major pools only: a row is the d*e bytes of one (token, head)
  uint32_t row_bytes;
  uint32_t block_tokens;
  uint32_t num_kv_heads;
  // head-major pools moved as line tiles or through LDS (T, h and the row size are powers of two there): a tile is
  // 2^tile_shift tokens x as many heads as make up 1 KiB (tile_offsets), or x all heads; through LDS slices_per_block counts
  // tiles
  uint32_t row_shift;    // log2(row_bytes)
  uint32_t head_shift;   // log2(num_kv_heads)
  uint32_t token_shift;  // log2(block_tokens)
  uint32_t tile_shift;   // log2(tokens per tile)
  uint32_t lds_pitch;    // bytes between consecutive tokens of the tile in LDS: h*row_bytes + row_bytes
  uint32_t slice_bytes;  // kCut: what a slice of a block moves
  // dense staging: blocks are whole alignment units and whole slices, so item `it` of an unpack reads the
  // staging bytes [it*slice, (it+1)*slice) whatever the extents are; items_bound = 2 * table_len * slices
  uint32_t dense;
  uint32_t items_bound;
  uint32_t chip_waves;  // whole-GPU restore: wavefronts that the chip holds (hold_back_pause); 0 = never hold back
  // workgroup -> item mapping: 0 = workgroup b starts at item 4b (neighbouring workgroups, which the
  // dispatcher deals round-robin to the 8 XCDs, take neighbouring 16 KiB); 1 = each XCD takes one
  // contiguous eighth of the copy workgroups' items
  uint32_t xcd_contiguous;
  // direct-to-block mode (the rings' one-launch layer path, DIRECT below): `stage` is the base of the file store, the
  // per-request staging offsets in LDS hold the start of each request's file in it (kNoFile if the store has no
  // such file), and the object side of (request, kind, block j) is the file offset of the context that
  // emit_iocbs records for it; only the first ctx_cap contexts were recorded and are executed
  uint32_t layer;
  uint64_t file_stride;
  uint64_t ctx_cap;
  // ordered restore: table positions in the order in which their blocks are to be visited (table_len entries);
  // unit u of the launch is (plane u / table_len, position visit[u % table_len]) instead of staging order
  const uint32_t *visit;
};


struct LayoutArgs {
  const uint32_t *n_blocks;
  tutti_extent *extents;
  uint64_t *totals;
  ScanGeom geom;
  uint32_t n_req;
};

// The workgroup index used for item numbering (see MoveArgs::xcd_contiguous).
__device__ __forceinline__ uint32_t item_wg(const MoveArgs &a, uint32_t wg, uint32_t copy_wgs) {
  const uint32_t b = wg;  // index among the copy workgroups
  if (!a.xcd_contiguous || copy_wgs < 16u) return b;
  const uint32_t per = copy_wgs / 8u;            // workgroups per XCD (the remainder keeps its own index)
  if (b >= per * 8u) return b;
  return (b % 8u) * per + b / 8u;
}

// The first item of this wavefront; its others follow n_waves apart.  Whole-GPU launches: the wavefronts of a workgroup
// take neighbouring items.  CU-budgeted launches (large workgroups): neighbouring workgroups do, so that a job of few
// items is spread over all the budgeted compute units; but slices of 8 KiB that give every wavefront an item go to
// neighbouring wavefronts (512 blocks of 8 KiB on 8 compute units, warm: save 28.5 us against 34.8, restore 30.1 against
// 32.8; with slices or pieces of 16 KiB the two orders differ by 3 % either way).
template <int WG, int U>
__device__ __forceinline__ uint32_t first_item(const MoveArgs &a, uint32_t wg, uint32_t copy_wgs) {
  const uint32_t wave = rfl(threadIdx.x / kWave);
  if (WG == kBudgetWgThreads && !(U == 8 && a.items_bound >= copy_wgs * (WG / kWave))) return wave * copy_wgs + wg;
  return item_wg(a, wg, copy_wgs) * (WG / kWave) + wave;
}

constexpr int kPack = 0;   // pool -> object
constexpr int kUnpack = 1; // object -> pool

// Offset inside a head-major block [h][T][row] of the 16 bytes that sit at canonical
// (token-major, [T][h][row]) offset o.
__device__ __forceinline__ uint32_t hnd_offset(uint32_t o, uint32_t row_bytes, uint32_t T, uint32_t h) {
  const uint32_t row = o / row_bytes;
  const uint32_t w = o - row * row_bytes;
  const uint32_t t = row / h;
  const uint32_t i = row - t * h;
  return (i * T + t) * row_bytes + w;
}

// How a lane's 16-byte units lie on one side of a copy: one behind the other, found row by row in a head-major block, or
// as line tiles (LineTile).
// kCut: token-major blocks that are no whole number of U KiB, cut into equal slices of fewer bytes (cut_slice, which has the
// figures); what a slice leaves of the U KiB that a wavefront's accesses cover, the bounds check of a buffer access drops.
constexpr int kNhd = 0, kHnd = 1, kLines = 2, kCut = 3;                     // pools
constexpr int kLinear = 0, kRows = 1, kTileObj = 2, kTilePool = 3, kShort = 4;  // sides
constexpr int pool_side(int hnd) { return hnd == kLines ? kTilePool : hnd == kHnd ? kRows : hnd == kCut ? kShort : kLinear; }
constexpr int obj_side(int hnd) { return hnd == kLines ? kTileObj : hnd == kCut ? kShort : kLinear; }
template <int HND, int U>
__device__ __forceinline__ uint32_t slice_bytes(const MoveArgs &a) {
  return HND == kCut ? a.slice_bytes : U * kPiece;
}

// Buffer accesses to the `bytes` bytes from p on (the same in every lane): beyond them a load gives zeroes and a store does
// nothing, decided by the memory pipe for each lane, with no branch and no address to clamp.
constexpr int kRawBuffer = 0x00027000;  // descriptor word 3: untyped 32-bit elements
constexpr int kNonTemporal = 2;         // cache policy of a buffer access
__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded(const unsigned char *p, uint32_t bytes) {
  const uint64_t at = reinterpret_cast<uint64_t>(p);
  const uint64_t base = static_cast<uint64_t>(rfl(static_cast<uint32_t>(at >> 32))) << 32 | rfl(static_cast<uint32_t>(at));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, static_cast<int>(bytes), kRawBuffer);
}

// The offsets in the block of a lane's 16-byte units, whose canonical offsets o, o + 1 KiB, o + 2 KiB, ... lie a piece
// apart: as they are, or (head-major) with the row and head of the first unit found by division and those of the others
// by addition.  Divided out for 16 units at a time they stand beside 64 data registers, and the kernel spills.
struct HeadWalk {
  uint32_t at, w, i;                          // offset in the block, byte in the row, head
  uint32_t row, h, dw, di, step, up, around;  // the same in every lane
  __device__ __forceinline__ HeadWalk(const MoveArgs &a, uint32_t o) : row(a.row_bytes), h(a.num_kv_heads) {
    const uint32_t r = o / row, t = r / h, rows = kPiece / row, tokens = rows / h;
    w = o - r * row;
    i = r - t * h;
    at = (i * a.block_tokens + t) * row + w;
    dw = kPiece - rows * row;
    di = rows - tokens * h;
    step = (di * a.block_tokens + tokens) * row + dw;
    up = (a.block_tokens - 1) * row;           // the next head's row instead of `row` bytes further on
    around = row - h * a.block_tokens * row;   // the next token's first head instead of head h
  }
  __device__ __forceinline__ uint32_t next() {
    const uint32_t now = at;
    at += step;
    w += dw;
    i += di;
    if (w >= row) {
      w -= row;
      i += 1;
      at += up;
    }
    if (i >= h) {  // i is below 2h: both addends are below h, plus one
      i -= h;
      at += around;
    }
    return now;
  }
};

// Loads (or stores) of a slice of U pieces that starts at offset o0 of a block, the lane's 16 bytes of each, in the
// order of the pieces and one behind the other: a store whose data was loaded behind other data waits for that too, and
// a run of stores with arithmetic in between moves less.  Under a budget of 32 compute units a save of 16 KiB slices
// took 82 us instead of 74 with the third and fourth load last; a head-major restore of 64-byte rows 53 instead of 45
// with each store behind the arithmetic for its offset.  Four pieces are left to the scheduler and to division, which
// are independent of each other (whole-GPU restore of 64 blocks of 32 KiB: 3.5 us against 3.65).
template <int U>
__device__ __forceinline__ void head_offsets(const MoveArgs &a, uint32_t o0, uint32_t (&at)[U]) {
  if (U <= 4) {
#pragma unroll
    for (int k = 0; k < U; ++k) at[k] = hnd_offset(o0 + k * kPiece, a.row_bytes, a.block_tokens, a.num_kv_heads);
  } else {
    HeadWalk w(a, o0);
#pragma unroll
    for (int k = 0; k < U; ++k) at[k] = w.next();
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Line tiles: a head-major pool whose (token, head) rows are shorter than a 128-byte line, without a detour through LDS.
// What bounds such a copy is the lines that a wavefront instruction touches in part, above all with stores: in the object's
// order it stores one row to every head.  So an instruction takes a tile of 2^tile_shift tokens by as many heads as make up
// 1 KiB, and the lanes are dealt out so that it touches whole lines on both sides: runs of 2^tile_shift rows in the block,
// of the tile's heads in the object (rows of 64 / 32 / 16 bytes: 256 and 256, 128 and 256, 128 and 128 bytes).  The tiles
// of a block are numbered in the object's order, a slice is U of them; row size, heads and tokens are powers of two.  A
// lane's place in a tile is the same for every tile; what depends on the tile is wave-uniform.
// Graph replay, us, through LDS (or, under a budget, direct where that was faster) / so, blocks of 16 KiB, 4 requests:
//   rows of 64 bytes   restore of 4096 blocks 45.8 / 43.5 (a token-major pool: 43.2), 384 6.2 / 5.5, 64 in one request 3.8 /
//                      3.5; save 49.0 / 47.7, 6.3 / 5.3, 4.0 / 3.5; on 32 compute units, 1536 blocks: restore 69 / 59, save 80 / 59
//   rows of 32 bytes   restore of 4096 45.9 / 43.7, save 49.3 / 48.0; on 32 units, 1536: 95 / 62, 111 / 63
//   rows of 16 bytes   restore of 4096 45.9 / 44.3, save 49.2 / 48.1; on 32 units, 1536: 144 / 70, 152 / 74
template <bool POOL, int U>
__device__ __forceinline__ void tile_offsets(const MoveArgs &a, uint32_t o0, uint32_t (&at)[U]) {
  const uint32_t lane = threadIdx.x & (kWave - 1), first = rfl(o0 / kPiece);
  const uint32_t rs = a.row_shift, hs = a.head_shift, ts = a.token_shift, tg = a.tile_shift, hg = 10u - rs - tg;
  // lane -> 16-byte unit of a row, token, head, the block's order
  const uint32_t w = lane & ((1u << (rs - 4)) - 1u), t = lane >> (rs - 4) & ((1u << tg) - 1u), i = lane >> (rs - 4 + tg);
  const uint32_t mine = (POOL ? (i << ts) + t : (t << hs) + i) << rs | w << 4;
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t q = first + k, heads = q & ((1u << (hs - hg)) - 1u), tokens = q >> (hs - hg);
    at[k] = mine + ((POOL ? (heads << (hg + ts)) + (tokens << tg) : (tokens << (tg + hs)) + (heads << hg)) << rs);
  }
  if (U > 4) __builtin_amdgcn_sched_barrier(0);  // a run of stores with arithmetic in between moves less
}
template <int SIDE, int U, int NT>
__device__ __forceinline__ void load_slice(const MoveArgs &a, const unsigned char *blk, uint32_t o0, u32x4 (&buf)[U]) {
  if (SIDE == kLinear) {
#pragma unroll
    for (int k = 0; k < U; ++k) buf[k] = ld16<NT>(blk + (o0 + k * kPiece));
  } else if (SIDE == kShort) {
    const uint32_t mine = (threadIdx.x & (kWave - 1)) * 16u;
    const __amdgpu_buffer_rsrc_t s = bounded(blk + (o0 - mine), a.slice_bytes);
#pragma unroll
    for (int k = 0; k < U; ++k)
      buf[k] = __builtin_amdgcn_raw_buffer_load_b128(s, static_cast<int>(mine + k * kPiece), 0, kNonTemporal);
  } else {
    uint32_t at[U];
    if (SIDE == kRows)
      head_offsets(a, o0, at);
    else
      tile_offsets<SIDE == kTilePool>(a, o0, at);
#pragma unroll
    for (int k = 0; k < U; ++k) buf[k] = ld16<NT>(blk + at[k]);
  }
}
template <int SIDE, int U, int NT>
__device__ __forceinline__ void store_slice(const MoveArgs &a, unsigned char *blk, uint32_t o0, const u32x4 (&buf)[U]) {
  if (SIDE == kLinear) {
#pragma unroll
    for (int k = 0; k < U; ++k) st16<NT>(blk + (o0 + k * kPiece), buf[k]);
  } else if (SIDE == kShort) {
    const uint32_t mine = (threadIdx.x & (kWave - 1)) * 16u;
    const __amdgpu_buffer_rsrc_t s = bounded(blk + (o0 - mine), a.slice_bytes);
#pragma unroll
    for (int k = 0; k < U; ++k)
      __builtin_amdgcn_raw_buffer_store_b128(buf[k], s, static_cast<int>(mine + k * kPiece), 0, kNonTemporal);
  } else {
    if (U > 4) __builtin_amdgcn_sched_barrier(0);  // the loads first: the offsets are worked out under them
    uint32_t at[U];
    if (SIDE == kRows)
      head_offsets(a, o0, at);
    else
      tile_offsets<SIDE == kTilePool>(a, o0, at);
#pragma unroll
    for (int k = 0; k < U; ++k) st16<NT>(blk + at[k], buf[k]);
  }
}

// Description of one slice, piece or tile: where it sits on the object side and which block-table entry names the pool
// side.  Wave-uniform, except that the pieces of an item are decoded one per lane.
struct Item {
  unsigned char *obj_ptr;  // start of the (request, kind) object; nullptr = skip the item
  unsigned char *obj_blk;  // where block j of it sits on the object side
  uint64_t obj_bytes;
  uint32_t tab_idx;        // index into the block table
  uint32_t n;              // blocks of the request
  uint32_t j;              // block within the request
  uint32_t s;              // slice within the block
  uint32_t kind;
};

// SEP: the extents came from the caller (lds_from_caller_extents): items are numbered by blk_off, the table is
// indexed by the request's own table_off, and requests that cannot be honoured already have a zero-sized object.
// ORD: the units in staging order, or all K blocks and then all V blocks, each in the order that a.visit lists or in the
// table's own, or the K and the V block of every table position in turn;
// a listed position that is not a block of a request that takes part is passed over.
// u: (block, kind) unit in staging order; s: its slice, piece or tile; `report`: this thread reports what it finds out
// of order with a unit's first part.
// OWNER: how the request is found; kPerLane: the lanes ask for units of their own, kOfFew and kOfMany: all for the same
// one, of at most 64 requests or of any number.
constexpr int kPerLane = 0, kOfFew = 1, kOfMany = 2;
constexpr int kStagingOrder = 0, kListOrder = 1, kTableOrder = 2, kPairOrder = 3;

template <bool SEP, int ORD, bool DIRECT, int OWNER>
__device__ __forceinline__ Item decode_unit(const MoveArgs &a, const ReqLds &l, uint32_t n_req, uint32_t u, uint32_t s,
                                            bool report) {
  Item d;
  d.s = s;
  report = report && s == 0 && a.status != nullptr;
  const uint32_t *off = SEP ? l.blk_off : l.table_off;
  uint32_t r, toff, end;
  uint64_t stage_off;
  const auto owner = [&](const uint32_t *of, uint32_t key) {
    return OWNER == kPerLane ? find_owner(of, n_req, key)
                             : find_owner_of_wave<OWNER == kOfFew, DIRECT>(l, of, n_req, key);
  };
  // all of a request's words are asked for together: they come out of LDS one behind the other, and a workgroup that has
  // one tile in flight waits for each (tiles of 16-byte rows on 8 compute units: 594 ns each with two waits, 550 with one)
  const auto request = [&] {
    d.obj_bytes = l.obj_bytes[r];
    stage_off = l.stage_off[r];
    toff = off[r];
    end = off[r + 1];
    __builtin_amdgcn_sched_barrier(0);
  };
  if (ORD != kStagingOrder) {
    d.kind = ORD == kPairOrder ? u & 1u : u >= a.table_len ? 1u : 0u;
    uint32_t pos = ORD == kPairOrder ? u >> 1 : u - d.kind * a.table_len;
    if (ORD == kListOrder) pos = as_const(a.visit)[rfl(pos)];  // wave-uniform index: one scalar load
    if (pos >= l.table_off[n_req]) {  // beyond the blocks of the requests that take part
      d.obj_ptr = nullptr;
      d.obj_blk = nullptr;
      d.obj_bytes = 0;
      d.tab_idx = d.n = d.j = 0;
      return d;
    }
    r = owner(l.table_off, pos);
    request();
    d.n = end - toff;
    d.j = pos - toff;
  } else {
    r = owner(off, u >> 1);
    request();
    d.n = end - toff;
    const uint32_t v = u - 2u * toff;
    d.kind = v >= d.n ? 1u : 0u;
    d.j = v - d.kind * d.n;
  }
  d.tab_idx = (SEP ? l.table_off[r] : toff) + d.j;
  if (DIRECT) {
    // same arithmetic as the context's file offset (direct_entry_quarter), then the I/O kernel's checks
    const uint64_t file_off = (2ull * a.layer + d.kind) * d.obj_bytes + static_cast<uint64_t>(d.j) * a.block_bytes;
    const uint64_t end = file_off + a.block_bytes;
    d.obj_ptr = a.stage;
    d.obj_blk = a.stage + stage_off + file_off;
    const uint32_t ctx = ORD != kStagingOrder ? 2u * toff + d.kind * d.n + d.j : u;  // the unit's place in staging order
    if (ctx >= a.ctx_cap) {
      d.obj_ptr = nullptr;  // beyond the IOCBs the caller gave: not recorded, not executed
    } else if (stage_off == kNoFile || end > a.file_stride || end < file_off) {
      if (report) atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
      d.obj_ptr = nullptr;
    }
    return d;
  }
  d.obj_ptr = a.stage + stage_off + d.kind * d.obj_bytes;
  d.obj_blk = d.obj_ptr + static_cast<uint64_t>(d.j) * a.block_bytes;
  if (!SEP && ((stage_off > a.stage_cap) | (d.obj_bytes > (a.stage_cap - stage_off) / 2))) {
    // the request's objects do not fit: skip it, report once
    // (an ordered launch reports from its first workgroup instead: its list need not name the request's first block)
    if (ORD != kListOrder && report && d.j == 0 && d.kind == 0) atomicOr(a.status, TUTTI_ST_STAGE_CAP);
    d.obj_ptr = nullptr;
  } else if ((static_cast<uint64_t>(d.j) + 1) * a.block_bytes > d.obj_bytes) {
    d.obj_ptr = nullptr;  // the block would end beyond its object (caller-made extents only)
  }
  return d;
}

template <bool SEP, int REQS, int ORD = kStagingOrder, bool DIRECT = false>
__device__ __forceinline__ Item decode_item(const MoveArgs &a, const ReqLds &l, uint32_t n_req, uint32_t it,
                                            uint32_t lane) {
  const uint32_t u = it / a.slices_per_block;
  return decode_unit<SEP, ORD, DIRECT, any_number(REQS) ? kOfMany : kOfFew>(a, l, n_req, u, it - u * a.slices_per_block,
                                                                         lane == 0);
}

// Block id of an item through the scalar (constant) path: the index is wave-uniform, so this is
// one s_load that overlaps the vector loads and stores of the item before it.
__device__ __forceinline__ uint32_t load_block_id(const MoveArgs &a, const Item &d) {
  const_u32_ptr tab = as_const(a.table);
  const uint32_t idx = __builtin_amdgcn_readfirstlane(d.tab_idx);  // uniform by construction
  const bool ok = __builtin_amdgcn_readfirstlane(d.obj_ptr != nullptr && idx < a.table_len ? 1 : 0) != 0;
  return ok ? tab[idx] : a.num_blocks;
}

// A pack's last slice of an object: zeroes behind it, up to the object's aligned size (fewer than `align` bytes).
__device__ __forceinline__ void zero_tail(const MoveArgs &a, const Item &d, uint32_t lane) {
  if (d.j + 1 == d.n && d.s + 1 == a.slices_per_block) {
    const uint64_t used = static_cast<uint64_t>(d.n) * a.block_bytes;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (uint64_t o = used + lane * 16ull; o < d.obj_bytes; o += kWave * 16ull) st16<0>(d.obj_ptr + o, zero);
  }
}

// ORD: the block need not be a whole number of slices (the others are moved as pieces then).
template <int DIR, int HND, int U, int NT, bool ORD, bool DIRECT>
__device__ __forceinline__ void move_one(const MoveArgs &a, const Item &d, uint32_t id, uint32_t lane) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  if (d.obj_ptr == nullptr) return;
  const uint32_t in_blk = d.s * slice;  // first byte of the slice inside the block
  if (id < a.num_blocks) {
    unsigned char *blk_ptr = (d.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride;
    unsigned char *obj_blk = d.obj_blk;
    const uint32_t o0 = in_blk + lane * 16u;  // this lane's first 16 bytes, canonical offset in the block
    if (!ORD || in_blk + slice <= a.block_bytes) {
      // whole slice inside the block: U independent loads in flight, then U stores
      u32x4 buf[U];
      load_slice<DIR == kPack ? pool_side(HND) : obj_side(HND), U, NT>(a, DIR == kPack ? blk_ptr : obj_blk, o0, buf);
      store_slice<DIR == kPack ? obj_side(HND) : pool_side(HND), U, NT>(a, DIR == kPack ? obj_blk : blk_ptr, o0, buf);
    } else {
      // ragged last slice of a block: one guarded 16-byte move at a time
      for (int k = 0; k < U; ++k) {
        const uint32_t o = o0 + k * (kWave * 16u);
        if (o < a.block_bytes) {
          const uint32_t po = HND ? hnd_offset(o, a.row_bytes, a.block_tokens, a.num_kv_heads) : o;
          if (DIR == kPack)
            st16<NT>(obj_blk + o, ld16<NT>(blk_ptr + po));
          else
            st16<NT>(blk_ptr + po, ld16<NT>(obj_blk + o));
        }
      }
    }
  } else if (lane == 0 && d.s == 0 && a.status) {
    atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
  }
  if (DIR == kPack && !DIRECT) zero_tail(a, d, lane);
}

// Items as slices of U KiB: cut slices are less.
template <int HND, int U>
__device__ __forceinline__ uint32_t full_slices(const MoveArgs &a, uint32_t items) {
  return HND == kCut ? items * (a.slice_bytes / 128) / (8 * U) : items;
}

// Holds the stores of a wavefront that has read ahead back (hold_back_pause).
__device__ __forceinline__ void hold_back(uint32_t pause) {
  for (uint32_t i = 0; i < pause; ++i) __builtin_amdgcn_s_sleep(8);
}

// Number of (block, kind) units of a copy.  Staged mode: the scan (or the loader of caller-made extents) has already cut
// the requests at table_len blocks.  Direct-to-block mode: one unit per recorded context.  The host checked that
// the bound (2 * table_len, or the contexts the IOCBs hold) times the slices per block fits 32 bits.
template <bool SEP, int ORD = kStagingOrder, bool DIRECT = false>
__device__ __forceinline__ uint32_t count_units(const MoveArgs &a, const ReqLds &l, uint32_t n_req) {
  if (ORD != kStagingOrder) return 2u * a.table_len;  // every listed position, for K and for V
  if (DIRECT) {
    const uint64_t units = 2ull * rfl(l.table_off[n_req]);
    return static_cast<uint32_t>(units < a.ctx_cap ? units : a.ctx_cap);
  }
  return 2u * rfl(SEP ? l.blk_off[n_req] : l.table_off[n_req]);
}

// First item of a wavefront in an unpack from dense staging: its source bytes do not depend on the extents,
// so their loads can be in flight while the workgroup is still fetching or scanning the extents.  (Slices of up to 8 KiB:
// 16 loads in flight need the registers, and such launches have many items a wavefront.)
constexpr bool reads_ahead(int units) { return units <= 8; }

template <int U>
struct Preload {
  u32x4 buf[U];
  const unsigned char *src;  // where the slice was read from (wave-uniform)
  bool valid;
};

template <int HND, int U, int NT, int WG>
__device__ __forceinline__ Preload<U> preload_first(const MoveArgs &a, uint32_t wg, uint32_t copy_wgs) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t it = first_item<WG, U>(a, wg, copy_wgs);
  const uint64_t at = static_cast<uint64_t>(it) * slice;
  // a slice of line tiles lies anywhere in its block (a power of two, and dense staging has no gap between blocks)
  const uint32_t in_blk = HND == kLines ? static_cast<uint32_t>(at) & (a.block_bytes - 1) : 0u;
  Preload<U> p;
  p.valid = a.dense != 0 && it < a.items_bound && at - in_blk + (HND == kLines ? a.block_bytes : slice) <= a.stage_cap;
  p.src = a.stage + at;
  if (p.valid) {
    load_slice<obj_side(HND), U, NT>(a, p.src - in_blk, in_blk + lane * 16u, p.buf);
  }
  return p;
}

// A pack in table order (reads_under_scan): the launch gives every wavefront one item at most, so the order does not matter to
// the memory, and where an item's bytes sit follows from the table alone: they are read while the requests are being scanned,
// instead of behind the scan, the owner and the block id: small saves are bound by that chain of dependent loads.  In a table
// longer than the requests' blocks some are read for nothing; where pack_at_once says no they are therefore read when the sum of
// the counts has said that the position is one of the requests' (and K and V of a position side by side: what there is to do
// then lies in the first workgroups).  The item's block id is asked for behind the counts: in front of them saves of 72 to 150
// blocks took 0.3 us longer.
// Graph replay, 32 KiB blocks, us, in staging order / read at once whatever the table's length / so: 64 blocks in 30 requests
// 5.4 / 3.8 / 3.8, with a table of 384 blocks 5.2 / 6.7 / 4.5; 150 in 8 6.2 / 5.1 / 5.1, table of 384 6.6 / 8.1 / 5.9; 2 in 2, table of
// 384 3.7 / 6.1 / 3.7; 128 in 128 6.9 / 5.4 / 5.4; 300 in 200 10.4 / 8.0 / 8.2; 1280 of 8 KiB in 512 11.0 / 9.7 / 9.7.  (Of more than
// 64 requests, the first quarter of the chip's items read at once and the others counted: waits on both in one kernel made the
// short tables 0.3 us slower.)  With several items a wavefront, reading all K blocks first loses (1000 blocks in 8 requests
// 24.3 / 25.5).
constexpr int pack_order(int reqs) { return counts_first(reqs) ? kPairOrder : kTableOrder; }

template <int U, int WG, int REQS>
struct PackItem {
  uint32_t kind, pos, part;  // pos: in the table
  uint32_t id;               // num_blocks: no such item
  PackItem() = default;
  __device__ __forceinline__ PackItem(const MoveArgs &a, uint32_t wg, uint32_t copy_wgs)
      : kind(0), pos(0), part(0), id(a.num_blocks) {
    const uint32_t it = first_item<WG, U>(a, wg, copy_wgs);
    if (wg < copy_wgs && it < a.items_bound) {
      const uint32_t u = it / a.slices_per_block;
      part = it - u * a.slices_per_block;
      kind = pack_order(REQS) == kPairOrder ? u & 1u : u >= a.table_len ? 1u : 0u;
      pos = pack_order(REQS) == kPairOrder ? u >> 1 : u - kind * a.table_len;
      id = as_const(a.table)[pos];
    }
  }
};

template <int HND, int U, int NT, int WG, int REQS>
__device__ __forceinline__ Preload<U> preload_pack(const MoveArgs &a, const PackItem<U, WG, REQS> &f) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  const uint32_t lane = threadIdx.x & (kWave - 1);
  Preload<U> p;
  p.valid = f.id < a.num_blocks;
  // every path issues the loads (of some block for want of another, not the same one from all XCDs): the wait for the counts,
  // asked for in front of them, would otherwise be one for both
  const uint32_t spare = blockIdx.x < a.num_blocks ? blockIdx.x : 0u;
  p.src = (f.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(p.valid ? f.id : spare) * a.block_stride;
  load_slice<pool_side(HND), U, NT>(a, p.src, f.part * slice + lane * 16u, p.buf);
  return p;
}

// The pack of a ring call whose offsets are out of order (ReqLds::wraps), instead of store_pack: table order is not the
// contexts' order then.  A block at a time: such counts are a caller's mistake, and the code has to be small rather than fast
// (as a second whole copy loop in the kernel it cost ordinary calls 0.2 us).
__device__ __forceinline__ void pack_unordered(const MoveArgs &a, const ReqLds &l, uint32_t n_req, uint32_t first_wave,
                                               uint32_t n_waves) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t units = count_units<false, kStagingOrder, true>(a, l, n_req);
#pragma unroll 1
  for (uint32_t u = first_wave; u < units; u += n_waves) {
    const Item d = decode_unit<false, kStagingOrder, true, kPerLane>(a, l, n_req, u, 0, lane == 0);
    const uint32_t id = load_block_id(a, d);
    if (d.obj_ptr == nullptr) continue;
    if (id < a.num_blocks) {
      const unsigned char *blk = (d.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride;
#pragma unroll 1
      for (uint32_t o = lane * 16u; o < a.block_bytes; o += kPiece) st16<3>(d.obj_blk + o, ld16<3>(blk + o));
    } else if (lane == 0 && a.status) {
      atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
    }
  }
}

// What is left of it once the requests are known.
template <int HND, int U, int NT, int WG, int REQS, bool DIRECT>
__device__ __forceinline__ void store_pack(const MoveArgs &a, const ReqLds &l, uint32_t n_req, uint32_t wg,
                                           uint32_t copy_wgs, const Preload<U> &pre) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t it = first_item<WG, U>(a, wg, copy_wgs);
  if (it >= a.items_bound) return;
  const Item d = decode_item<false, REQS, pack_order(REQS), DIRECT>(a, l, n_req, it, lane);
  if (d.obj_ptr == nullptr) return;
  if (pre.valid)
    store_slice<obj_side(HND), U, NT>(a, d.obj_blk, d.s * slice + lane * 16u, pre.buf);
  else if (lane == 0 && d.s == 0 && a.status)
    atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
  if (!DIRECT) zero_tail(a, d, lane);
}

// Stores of an unpack item whose slice was preloaded (whole slices only: dense staging).
template <int HND, int U, int NT>
__device__ __forceinline__ void store_preloaded(const MoveArgs &a, const Item &d, uint32_t id, uint32_t lane,
                                                const Preload<U> &p) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  if (d.obj_ptr == nullptr) return;
  if (id < a.num_blocks) {
    unsigned char *blk_ptr = (d.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride;
    store_slice<pool_side(HND), U, NT>(a, blk_ptr, d.s * slice + lane * 16u, p.buf);
  } else if (lane == 0 && d.s == 0 && a.status) {
    atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
  }
}

// The copy loop of the `copy_wgs` copy workgroups of the grid; `wg` is this workgroup's index among them (the
// grid may hold other workgroups with other work).
// Software-pipelined by one item: the next item is decoded and its block id requested before the
// current item's loads and stores are issued.
template <int DIR, int HND, int U, int NT, int WG, int REQS, bool SEP, int ORD, bool DIRECT>
__device__ __forceinline__ void move_items(const MoveArgs a, const ReqLds l, uint32_t n_req, uint32_t wg,
                                           uint32_t copy_wgs, const Preload<U> &pre) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t n_waves = copy_wgs * (WG / kWave);
  const uint32_t n_items = count_units<SEP, ORD, DIRECT>(a, l, n_req) * a.slices_per_block;

  uint32_t it = first_item<WG, U>(a, wg, copy_wgs);
  if (it >= n_items) return;
  Item cur = decode_item<SEP, REQS, ORD, DIRECT>(a, l, n_req, it, lane);
  uint32_t id = load_block_id(a, cur);
  uint32_t ahead = DIR == kUnpack && pre.valid ? 1u : 0u;  // the item at hand has been read ahead
  for (;;) {
    const uint32_t nit = it + n_waves;
    const bool more = nit < n_items;
    Item nxt = cur;
    uint32_t nid = a.num_blocks;
    if (more) {
      nxt = decode_item<SEP, REQS, ORD, DIRECT>(a, l, n_req, nit, lane);
      nid = load_block_id(a, nxt);
    }
    // the preloaded bytes were read where the item's slice sits when the extents are the library's own; extents
    // from the caller (and the files of the direct-to-block mode) may put it elsewhere: then the slice is loaded
    // from where they say
    const bool preloaded = DIR == kUnpack && ahead != 0 &&
                           ((!SEP && ORD == kStagingOrder && !DIRECT) ||
                            cur.obj_blk + static_cast<uint64_t>(cur.s) * slice == pre.src);
    if (preloaded)
      store_preloaded<HND, U, NT>(a, cur, id, lane, pre);
    else
      move_one<DIR, HND, U, NT, ORD == kListOrder, DIRECT>(a, cur, id, lane);
    if (!more) break;
    if (DIR == kUnpack) {
      ahead = 0;
      asm volatile("" : "+s"(ahead));  // left to itself the compiler takes the first item out of the loop, and the loop
    }                                  // then starts with a wait for that item's stores
    cur = nxt;
    id = nid;
    it = nit;
  }
}

// ------------------------------------------------------------------------------------------
// One request (the whole prefix of one prompt, the common call).  Everything an item needs follows from the block count,
// one scalar load away: there is no scan, nothing goes through LDS, no wavefront waits for another one, and the
// arguments fit the scalar registers.  Through the general path the first store of a wavefront stands behind the scan, a
// barrier, a binary search in LDS and a dozen reloads of spilled arguments.  Kernel time in us, general path / this one:
// restore of 256 KiB 3.7 / 2.7, of 4 MiB (1K tokens) 4.8 / 4.1; save of 24 MiB 11.4 / 10.7, of 128 MiB (32K tokens)
// 46.9 / 45.6, of 512 MiB 185.6 / 183.4.  A restore that fills half the chip or more takes the general path: its stores
// would start among the other wavefronts' first loads (hold_back), 32K tokens 43.8 / 44.9.
// ------------------------------------------------------------------------------------------
struct OneReq {
  unsigned char *base;  // the staging buffer, or the request's file
  uint64_t lo;          // where the K object starts in it; the V object follows obj_bytes later
  uint64_t obj_bytes;
  uint64_t room;        // size of the file (0: the store has no such file)
  uint32_t n;           // blocks to move (0: the request is skipped)
  uint32_t units;       // (block, kind) units to move
};

// The request's extent: published by workgroup 0, put into LDS by the workgroups that write entries (which alone pass
// the barrier).  Staged: a request whose blocks run beyond the table, or whose objects do not fit, is skipped and
// reported.  Direct-to-block mode (file_id != nullptr): a block beyond the file, or every block if the store has no
// such file, is skipped and reported by the loop.
__device__ __forceinline__ OneReq one_request(const MoveArgs &m, const LayoutArgs &a, const ReqLds &l, bool publish,
                                              bool entries, const uint32_t *file_id, const FileArgs f) {
  OneReq q;
  const uint32_t n = as_const(a.n_blocks)[0];
  const uint64_t obj = static_cast<uint64_t>(n) * a.geom.block_bytes + obj_pad(a.geom, n);
  const bool cut = !file_id && n > m.table_len;
  uint64_t at = 0;
  q.base = m.stage;
  q.lo = 0;
  q.obj_bytes = obj;
  q.room = m.stage_cap;
  q.n = cut ? 0 : n;
  q.units = 2u * q.n;
  uint32_t flags = 0;
  if (file_id) {
    const uint32_t fid = as_const(file_id)[0], rel = fid - f.first_file_id;
    const bool has_file = fid >= f.first_file_id && rel < f.n_files;
    at = has_file ? static_cast<uint64_t>(rel) * f.file_stride : kNoFile;
    if (has_file) q.base += at;
    q.lo = 2ull * m.layer * obj;
    q.room = has_file ? f.file_stride : 0;
    q.units = static_cast<uint32_t>(2ull * n < m.ctx_cap ? 2ull * n : m.ctx_cap);
  } else {
    if (cut) flags |= TUTTI_ST_BAD_EXTENT;
    if (!cut && n != 0 && obj > m.stage_cap / 2) {
      flags |= TUTTI_ST_STAGE_CAP;
      q.n = q.units = 0;
    }
  }
  if (entries) {
    if (threadIdx.x == 0) {
      const uint32_t chunks = static_cast<uint32_t>(obj_chunks(a.geom, obj));
      l.stage_off[0] = at;
      l.obj_bytes[0] = obj;
      l.table_off[0] = l.sqe_base[0] = 0;
      l.table_off[1] = cut ? 0u : n;
      l.sqe_base[1] = 2u * chunks;
      if (publish) {
        tutti_extent e;
        e.stage_off = 0;
        e.obj_bytes = obj;
        e.n_blocks = n;
        e.n_chunks = chunks;
        e.sqe_base = 0;
        e.table_off = 0;
        a.extents[0] = e;
        a.totals[0] = 2 * obj;
        a.totals[1] = 2 * obj_chunks(a.geom, obj);
        if (flags != 0 && m.status) atomicOr(m.status, flags);
      }
    }
    __syncthreads();
  }
  return q;
}

// The copy loop of one request whose blocks are a whole number of slices; the next item's block id is requested before
// the current item's loads and stores are issued.  `pause`: how long the first item's stores are held back.
template <int DIR, int HND, int U, int NT, int WG, bool DIRECT>
__device__ __forceinline__ void move_request(const MoveArgs &a, const OneReq &q, uint32_t wg, uint32_t copy_wgs,
                                             const Preload<U> &pre, uint32_t pause) {
  const uint32_t slice = slice_bytes<HND, U>(a);
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t n_waves = copy_wgs * (WG / kWave);
  const uint32_t S = a.slices_per_block;
  const uint32_t n_items = q.units * S;
  const const_u32_ptr table = as_const(a.table);
  uint32_t it = first_item<WG, U>(a, wg, copy_wgs);
  if (it >= n_items) return;
  uint32_t u = it / S;
  uint32_t j = u >= q.n ? u - q.n : u;
  uint32_t id = j < a.table_len ? table[j] : a.num_blocks;
  bool first = DIR == kPack || pre.valid;
  for (;;) {
    const uint32_t kind = u >= q.n ? 1u : 0u, part = it - u * S;
    const uint32_t nit = it + n_waves;
    const bool more = nit < n_items && nit > it;
    uint32_t nu = u, nj = j, nid = a.num_blocks;
    if (more) {
      nu = nit / S;
      nj = nu >= q.n ? nu - q.n : nu;
      if (nj < a.table_len) nid = table[nj];
    }
    const uint64_t at = q.lo + kind * q.obj_bytes + static_cast<uint64_t>(j) * a.block_bytes;
    const bool fits = !DIRECT || (at + a.block_bytes >= at && at + a.block_bytes <= q.room);
    if (fits && id < a.num_blocks) {
      unsigned char *blk = (kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride;
      unsigned char *obj = q.base + at;
      const uint32_t o0 = part * slice + lane * 16u;
      if (DIR == kUnpack && first) {
        hold_back(pause);
        store_slice<pool_side(HND), U, NT>(a, blk, o0, pre.buf);
      } else {
        u32x4 buf[U];
        load_slice<DIR == kPack ? pool_side(HND) : obj_side(HND), U, NT>(a, DIR == kPack ? blk : obj, o0, buf);
        if (DIR == kPack && !DIRECT && first) {
          __builtin_amdgcn_sched_barrier(0);
          hold_back(pause);
          __builtin_amdgcn_sched_barrier(0);
        }
        store_slice<DIR == kPack ? obj_side(HND) : pool_side(HND), U, NT>(a, DIR == kPack ? obj : blk, o0, buf);
      }
    } else if (lane == 0 && part == 0 && a.status) {
      atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
    }
    if (DIR == kPack && !DIRECT && j + 1 == q.n && part + 1 == S) {  // zero the object's tail up to its aligned size
      const u32x4 zero = {0u, 0u, 0u, 0u};
      for (uint64_t o = static_cast<uint64_t>(q.n) * a.block_bytes + lane * 16ull; o < q.obj_bytes; o += kPiece)
        st16<0>(q.base + kind * q.obj_bytes + o, zero);
    }
    if (!more) break;
    first = false;
    it = nit;
    u = nu;
    j = nj;
    id = nid;
  }
}

// The copy loop for blocks that are no whole number of slices.  A wavefront decodes its next 64 pieces at once, one per
// lane (owner by binary search, block id, both addresses), so that the table loads of 64/U items are in flight together
// and an item costs a few lane reads; then it moves them item by item.
template <int DIR, int HND, int U, int NT, int WG, bool SEP, bool DIRECT>
__device__ __forceinline__ void move_pieces(const MoveArgs a, const ReqLds l, uint32_t n_req, uint32_t wg,
                                            uint32_t copy_wgs) {
  constexpr uint32_t kBatch = kWave / U;  // items decoded at once
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t n_waves = copy_wgs * (WG / kWave);
  const uint32_t ppb = a.slices_per_block;
  const uint64_t n_pieces = static_cast<uint64_t>(count_units<SEP, kStagingOrder, DIRECT>(a, l, n_req)) * ppb;
  const uint32_t n_items = static_cast<uint32_t>((n_pieces + U - 1) / U);
  const uint32_t in_piece = lane * 16u;

  for (uint64_t it = first_item<WG, U>(a, wg, copy_wgs); it < n_items;
       it += kBatch * static_cast<uint64_t>(n_waves)) {
    // ---- decode: lane -> piece lane % U of item it + (lane / U) * n_waves
    uint64_t obj = 0, blk = 0;        // where the piece sits on the two sides (head-major: blk = its block)
    uint32_t off = 0, len = 0;        // its offset in the block, its bytes (0: skip it)
    uint64_t tail = 0, tail_at = 0;   // pack: padding behind it
    const uint64_t mine = it + static_cast<uint64_t>(lane / U) * n_waves;
    if (mine * U + lane % U < n_pieces) {
      // unit = piece / ppb without a 64-bit division: item = q * ppb + rem, piece = q * ppb * U + (rem * U + lane % U)
      const uint32_t q = static_cast<uint32_t>(mine) / ppb;
      const uint32_t rest = (static_cast<uint32_t>(mine) - q * ppb) * U + lane % U;
      const uint32_t q2 = rest / ppb;
      const Item d = decode_unit<SEP, kStagingOrder, DIRECT, kPerLane>(a, l, n_req, q * U + q2, rest - q2 * ppb, true);
      if (d.obj_ptr != nullptr) {
        const uint32_t id = d.tab_idx < a.table_len ? a.table[d.tab_idx] : a.num_blocks;
        off = d.s * kPiece;
        const uint32_t bytes = a.block_bytes - off < kPiece ? a.block_bytes - off : kPiece;
        obj = reinterpret_cast<uint64_t>(d.obj_blk) + off;
        if (DIR == kPack && !DIRECT && d.j + 1 == d.n && d.s + 1 == ppb) {
          tail = d.obj_bytes - static_cast<uint64_t>(d.n) * a.block_bytes;
          tail_at = obj + bytes;
        }
        if (id < a.num_blocks) {
          len = bytes;
          blk = reinterpret_cast<uint64_t>(d.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride +
                (HND ? 0u : off);
        } else if (d.s == 0 && a.status) {
          atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
        }
      }
    }
    if (DIR == kPack) {  // zero the objects' tails up to their aligned sizes (fewer than `align` bytes each)
      for (uint64_t m = __ballot(tail != 0); m != 0; m &= m - 1) {
        const uint32_t src = static_cast<uint32_t>(__ffsll(static_cast<long long>(m))) - 1u;
        const uint64_t n = readlane_u64(tail, src);
        unsigned char *end = as_global(readlane_u64(tail_at, src));
        const u32x4 zero = {0u, 0u, 0u, 0u};
        for (uint64_t o = in_piece; o < n; o += kPiece) st16<0>(end + o, zero);
      }
    }
    const uint64_t live = __ballot(len != 0), whole = __ballot(len == kPiece);
    if (live == 0) continue;
    if (len == 0) off = 0;
    if (DIR == kPack)
      blk = or_first(blk, live);
    else
      obj = or_first(obj, live);
    // ---- move
#pragma unroll 1
    for (uint32_t i = 0; i < kBatch && live >> (i * U) != 0; ++i) {
      if ((live >> (i * U) & ((1ull << U) - 1)) == 0) continue;
      const auto obj_at = [&](uint32_t k, uint32_t o) { return as_global(readlane_u64(obj, i * U + k)) + o; };
      const auto blk_at = [&](uint32_t k, uint32_t o) {
        return as_global(readlane_u64(blk, i * U + k)) +
               (HND ? hnd_offset(readlane_u32(off, i * U + k) + o, a.row_bytes, a.block_tokens, a.num_kv_heads) : o);
      };
      if (DIR == kPack)
        move_decoded<U, U, NT>(i, whole, len, blk_at, obj_at);
      else
        move_decoded<U, U, NT>(i, whole, len, obj_at, blk_at);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Head-major pools with short rows.  A block is stored [h][T][row]; the object wants [T][h][row].
// Moving 16 bytes per lane straight between the two orders touches the pool in row-sized pieces,
// which is fine while a row fills whole 128-byte lines and poor below that (partial-line writes).
// Line tiles (tile_offsets) are the faster way round that; this one stays for tables with more blocks than they can number
// and for the measurement build.
// Here a workgroup stages one tile (2^tile_shift tokens x all heads) in LDS instead: the object
// side is read or written as one contiguous run, the pool side as h runs of tile_tokens*row bytes,
// and the transpose happens in LDS.  Tokens are padded by one row in LDS so that the lanes of a
// wavefront, which walk the rows of one head, fall on different banks.
// PT = 16-byte units per thread per tile (tile bytes = PT * 16 * workgroup size).
// ------------------------------------------------------------------------------------------
// Shifts and masks of the tile geometry.
struct TileGeom {
  uint32_t rs, gs, hr;               // log2 bytes of a row, of one token across all heads, of one head's run in the tile
  uint32_t g_mask, hr_mask, r_mask;
};

// The tile of an item on both sides: global loads of its PT 16-byte units per thread (object order for an
// unpack, pool order for a pack), and where they go afterwards.
template <int DIR, int PT, int WG>
struct TileMove {
  static __device__ __forceinline__ unsigned char *obj_tile(const MoveArgs &a, const TileGeom &g, const Item &d) {
    const uint32_t t0 = d.s << a.tile_shift;
    return d.obj_ptr + static_cast<uint64_t>(d.j) * a.block_bytes + (static_cast<uint64_t>(t0) << g.gs);
  }
  static __device__ __forceinline__ unsigned char *blk(const MoveArgs &a, const Item &d, uint32_t id) {
    return (d.kind ? a.v_base : a.k_base) + static_cast<uint64_t>(id) * a.block_stride;
  }
  // byte offset inside the block of pool-order position p of the tile that starts at token t0
  static __device__ __forceinline__ uint32_t pool_off(const MoveArgs &a, const TileGeom &g, uint32_t t0, uint32_t p) {
    const uint32_t i = p >> g.hr, t = (p & g.hr_mask) >> g.rs, w = p & g.r_mask;
    return (((i << a.token_shift) + t0 + t) << g.rs) + w;
  }
  // LDS offset of object-order position o, and of pool-order position p
  static __device__ __forceinline__ uint32_t lds_obj(const MoveArgs &a, const TileGeom &g, uint32_t o) {
    return (o >> g.gs) * a.lds_pitch + (o & g.g_mask);
  }
  static __device__ __forceinline__ uint32_t lds_pool(const MoveArgs &a, const TileGeom &g, uint32_t p) {
    const uint32_t i = p >> g.hr, t = (p & g.hr_mask) >> g.rs, w = p & g.r_mask;
    return t * a.lds_pitch + (i << g.rs) + w;
  }
  static __device__ __forceinline__ void load(const MoveArgs &a, const TileGeom &g, const Item &d, uint32_t id,
                                              uint32_t tid, u32x4 (&v)[PT]) {
    const uint32_t t0 = d.s << a.tile_shift;
    const unsigned char *src = DIR == kUnpack ? obj_tile(a, g, d) : blk(a, d, id);
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const uint32_t q = (k * WG + tid) * 16u;
      v[k] = ld16<1>(src + (DIR == kUnpack ? q : pool_off(a, g, t0, q)));
    }
  }
  static __device__ __forceinline__ void to_lds(const MoveArgs &a, const TileGeom &g, uint32_t tid, unsigned char *tile,
                                                const u32x4 (&v)[PT]) {
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const uint32_t q = (k * WG + tid) * 16u;
      *reinterpret_cast<u32x4 *>(tile + (DIR == kUnpack ? lds_obj(a, g, q) : lds_pool(a, g, q))) = v[k];
    }
  }
  static __device__ __forceinline__ void from_lds_and_store(const MoveArgs &a, const TileGeom &g, const Item &d,
                                                            uint32_t id, uint32_t tid, const unsigned char *tile) {
    const uint32_t t0 = d.s << a.tile_shift;
    unsigned char *dst = DIR == kUnpack ? blk(a, d, id) : obj_tile(a, g, d);
    u32x4 w[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const uint32_t q = (k * WG + tid) * 16u;
      w[k] = *reinterpret_cast<const u32x4 *>(tile + (DIR == kUnpack ? lds_pool(a, g, q) : lds_obj(a, g, q)));
    }
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const uint32_t q = (k * WG + tid) * 16u;
      st16<2>(dst + (DIR == kUnpack ? pool_off(a, g, t0, q) : q), w[k]);
    }
  }
};

// One tile per workgroup and iteration.  Not pipelined across tiles: holding the next tile's loads in
// registers cost the eighth resident workgroup per CU (more than 64 VGPRs) and bought 0.3 us; the eight
// workgroups of a CU cover each other's latency instead.
template <int DIR, int PT, int WG, int REQS, bool SEP>
__device__ __forceinline__ void move_items_hnd_lds(const MoveArgs a, const ReqLds l, uint32_t n_req, uint32_t wg,
                                                   uint32_t copy_wgs, unsigned char *tile) {
  typedef TileMove<DIR, PT, WG> TM;
  const uint32_t tid = threadIdx.x;
  const uint32_t n_items = count_units<SEP>(a, l, n_req) * a.slices_per_block;
  TileGeom g;
  g.rs = a.row_shift;
  g.gs = a.row_shift + a.head_shift;
  g.hr = a.tile_shift + a.row_shift;
  g.g_mask = (1u << g.gs) - 1u;
  g.hr_mask = (1u << g.hr) - 1u;
  g.r_mask = (1u << g.rs) - 1u;

  for (uint32_t it = wg; it < n_items; it += copy_wgs) {
    const Item d = decode_item<SEP, REQS>(a, l, n_req, it, tid);  // workgroup-uniform; thread 0 reports
    const uint32_t id = load_block_id(a, d);
    if (d.obj_ptr != nullptr && id < a.num_blocks) {
      u32x4 v[PT];
      TM::load(a, g, d, id, tid, v);
      TM::to_lds(a, g, tid, tile, v);
      __syncthreads();
      TM::from_lds_and_store(a, g, d, id, tid, tile);
      __syncthreads();  // the tile is free again
    } else if (d.obj_ptr != nullptr && tid == 0 && d.s == 0 && a.status) {
      atomicOr(a.status, TUTTI_ST_BAD_BLOCK);
    }
    if (DIR == kPack && d.obj_ptr != nullptr && d.j + 1 == d.n && d.s + 1 == a.slices_per_block) {
      const uint64_t used = static_cast<uint64_t>(d.n) * a.block_bytes;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      for (uint64_t o = used + tid * 16ull; o < d.obj_bytes; o += WG * 16ull) st16<0>(d.obj_ptr + o, zero);
    }
  }
}

__host__ __device__ constexpr uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }

__global__ __launch_bounds__(kWgThreads) void k_layout(const LayoutArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, a.n_req);
  scan_extents<kWgThreads, kMany>(a.geom, a.n_blocks, a.n_req, l, a.extents, a.totals, 0xffffffffu, nullptr, true, nullptr,
                           FileArgs{0, 0, 0}, [] {}, [](uint32_t) {});
}

template <int WG>
__global__ __launch_bounds__(WG) void k_sqe(const SqeArgs a, const ScanGeom g,
                                                     const tutti_extent *__restrict__ ext, uint32_t n_req, uint32_t n_wgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, n_req);
  if (!lds_from_extents<WG>(ext, n_req, l, g, a.status)) return;
  emit_sqes<WG>(a, l, n_req, 0, n_wgs, sqe_head<WG>(a, l, n_req, 0));
}

// PIECES: the blocks are no whole number of slices (here and below).
template <int DIR, int HND, int U, int NT, int WG, bool PIECES = false>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_move(const MoveArgs a, const tutti_extent *__restrict__ ext,
                                                      uint32_t n_req, uint32_t n_wgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, n_req, true);
  Preload<U> pre;
  pre.valid = false;
  if (DIR == kUnpack && !PIECES && reads_ahead(U)) pre = preload_first<HND, U, NT, WG>(a, blockIdx.x, n_wgs);
  lds_from_caller_extents<WG>(ext, n_req, l, a.table_len, a.block_bytes, a.stage_cap, a.status);
  if (PIECES)
    move_pieces<DIR, HND, U, NT, WG, true, false>(a, l, n_req, blockIdx.x, n_wgs);
  else
    move_items<DIR, HND, U, NT, WG, kMany, true, kStagingOrder, false>(a, l, n_req, blockIdx.x, n_wgs, pre);
}

template <int DIR, int PT, int WG>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, PT)) void k_move_lds(const MoveArgs a, const tutti_extent *__restrict__ ext,
                                                  uint32_t n_req, uint32_t n_wgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, n_req, true);
  lds_from_caller_extents<WG>(ext, n_req, l, a.table_len, a.block_bytes, a.stage_cap, a.status);
  move_items_hnd_lds<DIR, PT, WG, kMany, true>(a, l, n_req, blockIdx.x, n_wgs, smem + align16(req_lds_bytes(n_req)));
}

// One layer's restore (DIR = kUnpack) or save (DIR = kPack) in one launch: every workgroup redoes the
// (tiny) scan into its own LDS, with its first wavefront up to 64 requests, as a whole for more, and not at all for one
// (move_request).  The workgroups [copy_first, copy_first + copy_wgs)
// move the blocks; the first `sqe_wgs` workgroups of the grid also (or only) write the entries, one quarter per
// lane, and workgroup 0 publishes extents and totals.  The copy workgroups are persistent and split the items
// evenly, so the kernel ends when its slowest workgroup does: a workgroup with extra work in front of or behind
// its share, or one that has to wait for a free slot because the grid is larger than what the chip holds at
// once, adds that work's latency to the whole kernel (measured: 2.4 us of 53 with the entry writers as extra
// workgroups behind a full grid).  So the entries ride along: an entry-writing workgroup finds its quarter's
// request and asks for the file id right after the scan, runs its share of the copy, and only then assembles
// and stores the entry; with enough entries every workgroup of the grid takes one pass of them.  A small launch leaves places
// free and hides nothing behind its few items: there the entry writers are workgroups of their own (entries_apart).
struct Roles {
  uint32_t sqe_wgs;     // workgroups [0, sqe_wgs) write entries
  uint32_t copy_first;  // workgroups [copy_first, copy_first + copy_wgs) move blocks (the grid may be larger when
  uint32_t copy_wgs;    // there are more passes of entries than copy workgroups); 0, or beyond the entry writers
};

// The arguments that the way to the first load needs, asked for together: left to itself the compiler loads each where it
// is used, five or six waits one behind the other.
__device__ __forceinline__ void args_at_hand(const MoveArgs &m, const LayoutArgs &a, const Roles &w) {
  asm volatile("" ::"s"(m.k_base), "s"(m.v_base), "s"(m.table), "s"(m.block_stride), "s"(m.num_blocks), "s"(m.table_len),
               "s"(m.slices_per_block), "s"(m.items_bound), "s"(m.xcd_contiguous), "s"(a.n_blocks), "s"(a.n_req),
               "s"(w.sqe_wgs), "s"(w.copy_first), "s"(w.copy_wgs));
}

// The words of a LayerCall behind the first ones, which are arguments of their own.
typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
struct LateWords {
  uint64_t w[kLayerCallWords - kEarlyWords];
};
struct OrderedLateWords {
  LateWords late;
  const uint32_t *visit;
};
// Where k_layer's arguments lie: fields_again and word_in_lane read them as one run of words.  An ordered restore hands over 8
// bytes more than malloc's smallest chunks hold (layer_call.h): of the ordinary fields only the gaps are left, and those are full.
template <typename Rest>
struct LayerArguments {
  u64x4 w0;
  u64x2 w4;
  uint64_t w6;
  Rest rest;
};
static_assert(offsetof(LayerArguments<LateWords>, w0) == 0 && offsetof(LayerArguments<LateWords>, w4) == 4 * sizeof(uint64_t) &&
                  offsetof(LayerArguments<LateWords>, w6) == 6 * sizeof(uint64_t) &&
                  offsetof(LayerArguments<LateWords>, rest) == kEarlyWords * sizeof(uint64_t) &&
                  offsetof(LayerArguments<OrderedLateWords>, rest) == kEarlyWords * sizeof(uint64_t) &&
                  offsetof(OrderedLateWords, late) == 0,
              "a LayerCall's words, one behind the other");
static_assert(offsetof(LayerArguments<LateWords>, rest) + sizeof(LateWords) == sizeof(LayerCall) &&
                  offsetof(LayerArguments<OrderedLateWords>, rest) + sizeof(OrderedLateWords) == sizeof(LayerCall) + 8,
              "what the runtime copies");

template <int DIR>
__device__ __forceinline__ SqeArgs entry_args(const LayerFields &f) {
  SqeArgs q;
  q.file_id = reinterpret_cast<const uint32_t *>(as_global(f.file_id));
  q.sqe = reinterpret_cast<tutti_sqe *>(as_global(f.sqe));
  q.status = reinterpret_cast<uint32_t *>(as_global(f.status));
  q.stage_addr = f.stage_addr;
  q.sqe_cap = f.sqe_cap;
  q.chunk_bytes = f.chunk_bytes;
  q.layer = f.layer;
  q.opcode = DIR == kUnpack ? TUTTI_OP_READ : TUTTI_OP_WRITE;
  q.sgl_id = f.sgl_id;
  return q;
}

typedef const __attribute__((address_space(4))) uint64_t *const_u64_ptr;
__device__ __forceinline__ const_u64_ptr call_words() {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
  const_u64_ptr p = (const_u64_ptr)__builtin_amdgcn_kernarg_segment_ptr();
#pragma clang diagnostic pop
  asm volatile("" : "+s"(p));
  return p;
}

// The arguments once more, from memory: what is read again where it is used holds no scalar registers until then.
__device__ __forceinline__ LayerFields fields_again() {
  const const_u64_ptr p = call_words();
  LayerCall c;
#pragma unroll
  for (uint32_t i = 0; i < kLayerCallWords; ++i) c.w[i] = p[i];
  return unpack(c);
}

// The same for use behind the copy, when they would have to come from HBM again at the very end of the kernel: a word in each
// lane, asked for in front of it.
__device__ __forceinline__ uint64_t word_in_lane() {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  return call_words()[lane < kLayerCallWords ? lane : 0u];
}
__device__ __forceinline__ LayerFields fields_of_lanes(uint64_t word) {
  LayerCall c;
#pragma unroll
  for (uint32_t i = 0; i < kLayerCallWords; ++i) c.w[i] = readlane_u64(word, i);
  return unpack(c);
}

// A fused launch's arguments as the device code reads them.
template <int DIR, int HND, int U, bool PIECES>
__device__ __forceinline__ void take_apart(const LayerFields &f, const uint32_t *visit, MoveArgs &m, SqeArgs &q,
                                           LayoutArgs &a, Roles &w) {
  m.k_base = as_global(f.k_base);
  m.v_base = as_global(f.v_base);
  m.stage = as_global(f.stage);
  m.table = reinterpret_cast<const uint32_t *>(as_global(f.table));
  m.status = reinterpret_cast<uint32_t *>(as_global(f.status));
  m.block_stride = f.block_stride;
  m.stage_cap = f.stage_cap;
  m.num_blocks = f.num_blocks;
  m.block_bytes = f.block_bytes;
  m.table_len = f.table_len;
  asm("" : "+s"(m.table_len));  // that it has 31 bits makes the compiler write the scan out twice (1900 / 2860 instructions)
  const auto covered_by = [&](uint32_t bytes) { return (f.block_bytes / 16 + (bytes / 16 - 1)) / (bytes / 16); };
  const uint32_t slices = HND == kCut ? f.size_b : covered_by(U * kPiece);
  m.slices_per_block = PIECES ? covered_by(kPiece) : slices;
  m.items_bound = 2u * m.table_len * slices;
  m.slice_bytes = HND == kCut ? 128u * f.size_a : 0u;
  m.row_bytes = m.block_tokens = m.num_kv_heads = 0;
  m.row_shift = m.head_shift = m.token_shift = m.tile_shift = m.lds_pitch = 0;
  if (HND == kHnd || HND == kLines) {
    const BlockSizes b = get_sizes(f, HND == kLines);
    m.row_bytes = rfl(b.row_bytes);
    m.block_tokens = rfl(b.tokens);
    m.num_kv_heads = rfl(b.heads);
    if (HND == kLines) {
      m.row_shift = log2_of(m.row_bytes);
      m.head_shift = log2_of(m.num_kv_heads);
      m.token_shift = log2_of(m.block_tokens);
      m.tile_shift = line_tile_shift(m.row_shift, m.head_shift, m.token_shift);
    }
  }
  m.dense = f.dense;
  m.chip_waves = f.chip_waves;
#ifdef TUTTI_BENCH_BUILD
  m.xcd_contiguous = f.xcd_contiguous;
#else
  m.xcd_contiguous = 0;
#endif
  m.layer = 0;
  m.file_stride = m.ctx_cap = 0;
  m.visit = visit;
  q = entry_args<DIR>(f);
  a.n_blocks = reinterpret_cast<const uint32_t *>(as_global(f.n_blocks));
  a.extents = reinterpret_cast<tutti_extent *>(as_global(f.extents));
  a.totals = reinterpret_cast<uint64_t *>(as_global(f.totals));
  a.geom = ScanGeom{f.block_bytes, f.align, f.chunk_bytes};
  a.n_req = f.n_req;
  w.sqe_wgs = f.sqe_wgs;
  w.copy_first = f.copy_first;
  w.copy_wgs = f.copy_wgs;
}

// Holds the late words' registers until here: the loads that bring them are on their way from the start, and a register that
// is put to another use meanwhile would make that use wait for them.
__device__ __forceinline__ void late_words_at_hand(const LayerCall &c) {
  asm volatile("" ::"s"(c.w[7]), "s"(c.w[8]), "s"(c.w[9]), "s"(c.w[10]), "s"(c.w[11]), "s"(c.w[12]), "s"(c.w[13]));
}

// The same for all of them, in front of everything else: one wait.
__device__ __forceinline__ void words_at_hand(const LayerCall &c) {
  asm volatile("" ::"s"(c.w[0]), "s"(c.w[1]), "s"(c.w[2]), "s"(c.w[3]), "s"(c.w[4]), "s"(c.w[5]), "s"(c.w[6]));
  late_words_at_hand(c);
}

// ORD (restore only): the blocks are visited in the order `visit` lists instead of staging order; the first slices
// cannot be preloaded then (where they sit depends on the list).
template <int DIR, int HND, int U, int NT, int WG, int REQS, bool ORD, bool PIECES>
__device__ __forceinline__ void run_layer(const LayerCall &c, const uint32_t *visit) {
  extern __shared__ __align__(16) unsigned char smem[];
  MoveArgs m;
  SqeArgs q;
  LayoutArgs a;
  Roles w;
  take_apart<DIR, HND, U, PIECES>(unpack(c), visit, m, q, a, w);
  const ReqLds l = carve_lds(smem, a.n_req);
  const uint32_t wg = blockIdx.x - w.copy_first;  // wraps for the workgroups in front of the copy ones
  const bool copies = wg < w.copy_wgs;
  Preload<U> pre;
  pre.valid = false;
  const bool publish = blockIdx.x == 0;  // also an entry-writing workgroup: there is at least one
  if constexpr (REQS == kOne) {
    if (DIR == kUnpack && reads_ahead(U) && copies) pre = preload_first<HND, U, NT, WG>(m, wg, w.copy_wgs);
    if (DIR == kUnpack) late_words_at_hand(c);
    const bool entries = blockIdx.x < w.sqe_wgs;
    const OneReq one = one_request(m, a, l, publish, entries, nullptr, FileArgs{0, 0, 0});
    if (DIR == kPack) late_words_at_hand(c);
    SqeHead one_head;
    one_head.live = false;
    uint64_t word = 0;
    if (entries) {
      one_head = sqe_head<WG>(q, l, 1, 0);
      word = word_in_lane();
    }
    if (copies) {
      const uint32_t items = full_slices<HND, U>(m, one.units * m.slices_per_block);
      const uint32_t pause = HND == kHnd || (DIR == kUnpack && HND == kCut) ? 0u
                             : DIR == kPack ? one_save_pause(items, m.chip_waves, true) : one_restore_pause(items, m.chip_waves);
      move_request<DIR, HND, U, NT, WG, false>(m, one, wg, w.copy_wgs, pre, pause);
    }
    if (entries) emit_sqes<WG>(entry_args<DIR>(fields_of_lanes(word)), l, 1, 0, w.sqe_wgs, one_head);
    return;
  }
  PackItem<U, WG, REQS> first;
  scan_extents<WG, REQS>(
      a.geom, a.n_blocks, a.n_req, l, publish ? a.extents : nullptr, publish ? a.totals : nullptr, m.table_len, m.status,
      blockIdx.x < w.sqe_wgs, nullptr, FileArgs{0, 0, 0}, [&] {
        if (DIR == kPack && reads_under_scan(REQS)) {
          first = PackItem<U, WG, REQS>(m, wg, w.copy_wgs);
          late_words_at_hand(c);
          if (!counts_first(REQS)) pre = preload_pack<HND, U, NT>(m, first);
        } else if (DIR == kUnpack && !ORD && !PIECES && reads_ahead(U) && copies) {
          pre = preload_first<HND, U, NT, WG>(m, wg, w.copy_wgs);
        }
        if (DIR == kUnpack && !ORD && !PIECES && reads_ahead(U)) late_words_at_hand(c);
      },
      [&](uint32_t blocks) {
        if (DIR == kPack && first.pos < blocks) pre = preload_pack<HND, U, NT>(m, first);
      });
  if (REQS == kFew && DIR == kUnpack && pre.valid)
    hold_back(hold_back_pause(full_slices<HND, U>(m, count_units<false>(m, l, a.n_req) * m.slices_per_block), m.chip_waves,
                              a.n_req, false));
  SqeHead head;
  head.live = false;
  // the scan of many requests needs most scalar registers for itself
  if (any_number(REQS)) take_apart<DIR, HND, U, PIECES>(fields_again(), visit, m, q, a, w);
  uint64_t word = 0;
  if (blockIdx.x < w.sqe_wgs) {
    head = sqe_head<WG>(q, l, a.n_req, 0);
    word = word_in_lane();
  }
  if (ORD && wg == 0 && m.status) {
    // requests whose objects do not fit the staging buffer are skipped by every item: report them here, once
    for (uint32_t r = threadIdx.x; r < a.n_req; r += WG)
      if (l.table_off[r + 1] > l.table_off[r] &&
          (l.stage_off[r] > m.stage_cap || l.obj_bytes[r] > (m.stage_cap - l.stage_off[r]) / 2))
        atomicOr(m.status, TUTTI_ST_STAGE_CAP);
  }
  if (copies) {
    if (DIR == kPack && (REQS == kManyAhead || ((REQS == kFewAhead || REQS == kFewCounted) && HND != kHnd))) {
      const uint32_t items = full_slices<HND, U>(m, count_units<false>(m, l, a.n_req) * m.slices_per_block);
      hold_back(REQS == kManyAhead ? pack_pause(items, m.chip_waves) : few_save_pause(items, m.chip_waves, a.n_req, HND == kLines));
    }
    if (DIR == kPack && reads_under_scan(REQS))
      store_pack<HND, U, NT, WG, REQS, false>(m, l, a.n_req, wg, w.copy_wgs, pre);
    else if (PIECES)
      move_pieces<DIR, HND, U, NT, WG, false, false>(m, l, a.n_req, wg, w.copy_wgs);
    else
      move_items<DIR, HND, U, NT, WG, REQS, false, ORD ? kListOrder : kStagingOrder, false>(m, l, a.n_req, wg, w.copy_wgs, pre);
  }
  if (blockIdx.x < w.sqe_wgs) emit_sqes<WG>(entry_args<DIR>(fields_of_lanes(word)), l, a.n_req, 0, w.sqe_wgs, head);
}

// One request's kernels take the words in one argument, which is read from memory, all of it behind one wait: there it is the launch
// on the host that a train waits for, and a kernel of four arguments takes longer to launch.  Calls from Python, us, least of 12
// trains in each of three processes, the four arguments below / so: restore of 256 KiB 3.22 to 3.31 / 3.06 to 3.20, 32 layers of
// 4 MiB 104 to 107 / 96 to 104 (with every kernel's words in one argument 3.05 to 3.13 and 95 to 101, but then those of 8 requests
// take 127 instead of 120, 32 layers of 16 MiB in 8 requests 221 instead of 205).
template <int DIR, int HND, int U, int NT, int WG>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_layer(const LayerCall c) {
  words_at_hand(c);
  run_layer<DIR, HND, U, NT, WG, kOne, false, false>(c, nullptr);
}

// The early words are arguments by themselves because such are in registers when a wavefront starts (-amdgpu-kernarg-preload-count);
// the members of a struct are read from memory.  Graph replay of a copy kernel of four arguments, us, read / in registers:
// 4 KiB 2.48 / 2.40, 64 KiB 3.74 / 3.60, 256 KiB 6.9 / 6.7.  Calls with the words from memory / so: save of 1280 blocks in 512
// requests 8.07 / 7.93, restore of 128 MiB 44.0 / 43.8.
template <int DIR, int HND, int U, int NT, int WG, int REQS, bool ORD = false, bool PIECES = false>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_layer(
    const u64x4 w0, const u64x2 w4, uint64_t w6, const typename std::conditional<ORD, OrderedLateWords, LateWords>::type rest) {
  LayerCall c{{w0.x, w0.y, w0.z, w0.w, w4.x, w4.y, w6}};
  const uint32_t *visit = nullptr;
  const LateWords *late;
  if constexpr (ORD) {
    late = &rest.late;
    visit = rest.visit;
  } else {
    late = &rest;
  }
#pragma unroll
  for (uint32_t i = kEarlyWords; i < kLayerCallWords; ++i) c.w[i] = late->w[i - kEarlyWords];
  run_layer<DIR, HND, U, NT, WG, REQS, ORD, PIECES>(c, visit);
}

template <typename Rest>
using LayerKernel = void (*)(u64x4, u64x2, uint64_t, Rest);  // parameters in the order of LayerArguments' members
static_assert(std::is_same_v<decltype(&k_layer<kPack, kNhd, 4, 3, kWgThreads>), void (*)(LayerCall)> &&
                  std::is_same_v<decltype(&k_layer<kPack, kNhd, 4, 3, kWgThreads, kFew>), LayerKernel<LateWords>> &&
                  std::is_same_v<decltype(&k_layer<kUnpack, kNhd, 4, 3, kWgThreads, kMany, true>), LayerKernel<OrderedLateWords>>,
              "LayerArguments mirrors k_layer");

// First item of a wavefront in a retrieve of ONE request: its file bytes sit at
//   file start + 2*layer*obj_bytes + item*slice        (obj_bytes = n_blocks*block_bytes: blocks are whole
// alignment units in this mode), which takes two words from memory, the block count and the file id, and no scan.
// Every wavefront fetches them itself through the scalar path and has its loads in flight while the workgroup's
// first wavefront scans and the barrier is crossed; move_items checks the address against the decoded one.
template <int U, int WG>
__device__ __forceinline__ Preload<U> preload_first_direct(const MoveArgs &m, const uint32_t *n_blocks,
                                                           const uint32_t *file_id, const FileArgs f, uint32_t wg,
                                                           uint32_t copy_wgs) {
  constexpr uint32_t kSlice = kWave * 16u * U;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t it = first_item<WG, U>(m, wg, copy_wgs);
  Preload<U> p;
  p.valid = false;
  if (m.block_bytes % kSlice != 0) return p;
  const uint32_t n = rfl(n_blocks[0]), fid = rfl(file_id[0]);
  const uint32_t rel = fid - f.first_file_id;
  const uint64_t obj = static_cast<uint64_t>(n) * m.block_bytes;
  const uint64_t units = 2ull * (n < m.table_len ? n : m.table_len);
  const uint64_t lo = 2ull * m.layer * obj;  // file offset of the layer's K object
  // inside the table, inside the recorded contexts, inside the file (K and V objects of the layer: 2*obj bytes)
  if (fid < f.first_file_id || rel >= f.n_files || it >= units * m.slices_per_block ||
      it / m.slices_per_block >= m.ctx_cap || obj == 0 || lo / obj != 2ull * m.layer || lo + 2 * obj < lo ||
      lo + 2 * obj > f.file_stride)
    return p;
  p.valid = true;
  p.src = m.stage + static_cast<uint64_t>(rel) * f.file_stride + lo + static_cast<uint64_t>(it) * kSlice;
  const unsigned char *src = p.src + lane * 16u;
#pragma unroll
  for (int k = 0; k < U; ++k) p.buf[k] = ld16<3>(src + k * (kWave * 16u));
  return p;
}

// The arguments of k_layer_ring, each once: 192 bytes, and few enough that the kernels of many requests spill half as many scalar
// registers (as eight records that repeated each other they were 372; they do not fit a LayerCall's 112).  As records / so, us:
// retrieve of 64 blocks of 32 KiB 7.5 / 7.2, of 512 in one request 14.7 / 13.4, in 40 16.5 / 16.1, in 200 18.9 / 18.0; store of 512
// in one request 15.6 / 14.7, in 200 18.9 / 18.2; trains of 16 layers of 129 blocks, retrieve 106.5 / 102.5, store 98.1 / 89.3.
struct RingCall {
  uint64_t k_base, v_base, stage, table, n_blocks, file_id, status, extents, totals, sq, cq;  // addresses
  uint64_t block_stride, file_stride, sgl_table_addr;
  uint32_t num_blocks, block_bytes, table_len, chip_waves, n_req, align, chunk_bytes, layer, sgl_id, first_file_id, n_files;
  uint32_t depth, first_slot, n_slots, done_first, done_n, sqe_wgs, copy_first, copy_wgs, xcd_contiguous;
};
constexpr uint32_t kRingCallWords = sizeof(RingCall) / sizeof(uint64_t);
static_assert(sizeof(RingCall) == 24 * sizeof(uint64_t), "whole words");

struct RingParts {
  MoveArgs m;
  SqeArgs q;
  DirectArgs d;
  RingArgs g, done;
  FileArgs f;
  LayoutArgs a;
  Roles w;
};
template <int DIR, int U, bool PIECES>
__device__ __forceinline__ RingParts take_apart(const RingCall &c) {
  const auto words = [](uint64_t address) { return reinterpret_cast<uint32_t *>(as_global(address)); };
  const auto covered_by = [&](uint32_t bytes) { return (c.block_bytes / 16 + (bytes / 16 - 1)) / (bytes / 16); };
  RingParts p;
  p.m = MoveArgs{};
  p.m.k_base = as_global(c.k_base);
  p.m.v_base = as_global(c.v_base);
  p.m.stage = as_global(c.stage);
  p.m.table = words(c.table);
  p.m.status = words(c.status);
  p.m.block_stride = c.block_stride;
  p.m.num_blocks = c.num_blocks;
  p.m.block_bytes = c.block_bytes;
  p.m.table_len = c.table_len;
  p.m.slices_per_block = covered_by(PIECES ? kPiece : U * kPiece);
  p.m.items_bound = 2u * c.table_len * covered_by(U * kPiece);
  p.m.chip_waves = c.chip_waves;
#ifdef TUTTI_BENCH_BUILD
  p.m.xcd_contiguous = c.xcd_contiguous;
#endif
  p.m.layer = c.layer;
  p.m.file_stride = c.file_stride;
  p.m.ctx_cap = static_cast<uint64_t>(c.n_slots) * TUTTI_IOCB_SLOTS;
  p.q = SqeArgs{words(c.file_id), nullptr, p.m.status, 0, 0, c.block_bytes, c.layer,
                static_cast<uint32_t>(DIR == kUnpack ? TUTTI_OP_READ : TUTTI_OP_WRITE), c.sgl_id};
  p.d = DirectArgs{p.m.table, c.sgl_table_addr, c.table_len, c.num_blocks, c.block_bytes};
  p.g = RingArgs{reinterpret_cast<tutti_iocb *>(as_global(c.sq)), reinterpret_cast<tutti_cq_hdr *>(as_global(c.cq)), c.depth,
                 c.first_slot, c.n_slots};
  p.done = RingArgs{p.g.sq, p.g.cq, c.depth, c.done_first, c.done_n};
  p.f = FileArgs{c.file_stride, c.first_file_id, c.n_files};
  p.a = LayoutArgs{words(c.n_blocks), reinterpret_cast<tutti_extent *>(as_global(c.extents)),
                   reinterpret_cast<uint64_t *>(as_global(c.totals)), ScanGeom{c.block_bytes, c.align, c.chunk_bytes}, c.n_req};
  p.w = Roles{c.sqe_wgs, c.copy_first, c.copy_wgs};
  return p;
}
// Read from memory once more, as in fields_again.
__device__ __forceinline__ RingCall ring_call_again() {
  const const_u64_ptr p = call_words();
  uint64_t w[kRingCallWords];
#pragma unroll
  for (uint32_t i = 0; i < kRingCallWords; ++i) w[i] = p[i];
  RingCall c;
  __builtin_memcpy(&c, w, sizeof(c));
  return c;
}

// retrieve_layer / store_layer through the rings in one launch (direct-to-block mode): the scan puts the start
// of every request's file in the store where the staging offsets would be, then the first `sqe_wgs`
// workgroups record the layer's contexts in the IOCBs while the copy workgroups move the very same blocks,
// each item deriving its file offset and block from the extents and the table exactly as its context does.
// Blocks go to the file as they sit in the pool (a descriptor names raw bytes), so there is no head-major case.
// The completion of these IOCBs is a kernel boundary away: the host enqueues k_complete behind this kernel, or the
// next layer's launch carries it along (`done`: the IOCBs an earlier launch on the same stream has executed; when
// done.n_slots is not 0 the grid has one workgroup more, in front, whose first wavefront completes them and leaves,
// so a train of layers pays for no kernel boundary between a layer's data and the next layer's).
template <int DIR, int U, int WG, int REQS, bool PIECES = false>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_layer_ring(const RingCall call) {
  extern __shared__ __align__(16) unsigned char smem[];
  RingParts parts = take_apart<DIR, U, PIECES>(call);
  MoveArgs &m = parts.m;
  SqeArgs &q = parts.q;
  DirectArgs &d = parts.d;
  RingArgs &g = parts.g, &done = parts.done;
  FileArgs &f = parts.f;
  LayoutArgs &a = parts.a;
  Roles &w = parts.w;
  const uint32_t lead = done.n_slots != 0 ? 1u : 0u;
  if (lead && blockIdx.x == 0) {  // the whole workgroup takes this branch: no barrier is left waiting
    if (threadIdx.x < kWave) complete_iocbs(done, threadIdx.x);
    return;
  }
  const uint32_t bx = blockIdx.x - lead;
  ReqLds l = carve_lds(smem, a.n_req);
  const bool copies = bx - w.copy_first < w.copy_wgs;
  Preload<U> pre;
  pre.valid = false;
  const bool publish = bx == 0;
  if constexpr (REQS == kOne) {
    if (DIR == kUnpack && reads_ahead(U) && copies)
      pre = preload_first_direct<U, WG>(m, a.n_blocks, q.file_id, f, bx - w.copy_first, w.copy_wgs);
    const bool entries = bx < w.sqe_wgs;
    const OneReq one = one_request(m, a, l, publish, entries, q.file_id, f);
    DirectHead one_head;
    one_head.live = false;
    if (entries) one_head = iocb_head<WG>(g, q, d, l, 1, lead, w.sqe_wgs);
    if (copies) move_request<DIR, kNhd, U, 3, WG, true>(m, one, bx - w.copy_first, w.copy_wgs, pre, 0);
    if (entries) emit_iocbs<WG>(g, q, d, l, 1, lead, w.sqe_wgs, one_head);
    return;
  }
  // chunk counts only matter for the published extents; the LDS copy gets file starts instead of staging offsets
  if (reads_under_scan(REQS)) args_at_hand(m, a, w);
  PackItem<U, WG, REQS> first;
  scan_extents<WG, REQS>(
      a.geom, a.n_blocks, a.n_req, l, publish ? a.extents : nullptr, publish ? a.totals : nullptr, 0xffffffffu, nullptr,
      publish, q.file_id, f, [&] {
        if (DIR == kPack && reads_under_scan(REQS)) {
          first = PackItem<U, WG, REQS>(m, bx - w.copy_first, w.copy_wgs);
          if (!counts_first(REQS)) pre = preload_pack<kNhd, U, 3>(m, first);
        } else if (DIR == kUnpack && !PIECES && reads_ahead(U) && copies && a.n_req == 1) {
          pre = preload_first_direct<U, WG>(m, a.n_blocks, q.file_id, f, bx - w.copy_first, w.copy_wgs);
        }
      },
      [&](uint32_t blocks) {
        if (DIR == kPack && first.pos < blocks) pre = preload_pack<kNhd, U, 3>(m, first);
      });
  if (REQS == kFew && DIR == kUnpack && pre.valid)
    hold_back(hold_back_pause(count_units<false, kStagingOrder, true>(m, l, a.n_req) * m.slices_per_block, m.chip_waves, 1, true));
  if (any_number(REQS)) {
    l.unordered = rfl(l.wraps()) != 0;
    parts = take_apart<DIR, U, PIECES>(ring_call_again());  // the scan of many requests needs most scalar registers for itself
  }
  DirectHead head;
  head.live = false;
  if (bx < w.sqe_wgs) head = iocb_head<WG>(g, q, d, l, a.n_req, lead, w.sqe_wgs);
  if (copies) {
    if (reads_under_scan(REQS) && __builtin_expect(rfl(l.wraps()) != 0, 0))
      pack_unordered(m, l, a.n_req, (bx - w.copy_first) * (WG / kWave) + rfl(threadIdx.x / kWave), w.copy_wgs * (WG / kWave));
    else if (reads_under_scan(REQS))
      store_pack<kNhd, U, 3, WG, REQS, true>(m, l, a.n_req, bx - w.copy_first, w.copy_wgs, pre);
    else if (PIECES)
      move_pieces<DIR, kNhd, U, 3, WG, false, true>(m, l, a.n_req, bx - w.copy_first, w.copy_wgs);
    else
      move_items<DIR, kNhd, U, 3, WG, REQS, false, kStagingOrder, true>(m, l, a.n_req, bx - w.copy_first, w.copy_wgs, pre);
  }
  if (bx < w.sqe_wgs) emit_iocbs<WG>(g, q, d, l, a.n_req, lead, w.sqe_wgs, head);
}

template <int DIR, int PT, int WG, int REQS>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, PT)) void k_layer_lds(const MoveArgs m, const SqeArgs q, const LayoutArgs a, const Roles w) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ReqLds l = carve_lds(smem, a.n_req);
  const bool publish = blockIdx.x == 0;  // also an entry-writing workgroup: there is at least one
  scan_extents<WG, REQS>(a.geom, a.n_blocks, a.n_req, l, publish ? a.extents : nullptr, publish ? a.totals : nullptr,
                   m.table_len, m.status, blockIdx.x < w.sqe_wgs, nullptr, FileArgs{0, 0, 0}, [] {}, [](uint32_t) {});
  SqeHead head;
  head.live = false;
  if (blockIdx.x < w.sqe_wgs) head = sqe_head<WG>(q, l, a.n_req, 0);
  if (blockIdx.x - w.copy_first < w.copy_wgs)
    move_items_hnd_lds<DIR, PT, WG, REQS, false>(m, l, a.n_req, blockIdx.x - w.copy_first, w.copy_wgs,
                                    smem + align16(req_lds_bytes(a.n_req)));
  if (blockIdx.x < w.sqe_wgs) emit_sqes<WG>(q, l, a.n_req, 0, w.sqe_wgs, head);
}

// The preconditions of an unpack on its table, checked without any workspace: every id below num_blocks, no id
// twice.  All pairs: workgroup b takes the 256 table positions [256b, 256b + 256) as rows (one per thread), walks
// the column tiles from its own onwards through LDS and compares each row with the later positions of the tile,
// four ids per LDS read.  O(table_len^2) comparisons: a debugging aid (a 40,000-entry table takes microseconds, a
// million entries tens of milliseconds), not part of the per-layer path.
__global__ __launch_bounds__(kWgThreads) void k_table_validate(const uint32_t *__restrict__ table, uint32_t n,
                                                                uint32_t num_blocks, uint32_t *__restrict__ status) {
  __shared__ __align__(16) uint32_t tile[kWgThreads];
  const uint32_t n_tiles = (n + kWgThreads - 1) / kWgThreads;
  uint32_t found = 0;
  for (uint32_t b = blockIdx.x; b < n_tiles; b += gridDim.x) {
    const uint32_t i = b * kWgThreads + threadIdx.x;
    const uint32_t id = i < n ? table[i] : 0xffffffffu;
    const bool valid = id < num_blocks;
    if (i < n && !valid) found |= TUTTI_ST_BAD_BLOCK;
    for (uint32_t c = b; c < n_tiles; ++c) {
      const uint32_t j0 = c * kWgThreads;
      const uint32_t j = j0 + threadIdx.x;
      __syncthreads();  // the previous tile has been read by everyone
      tile[threadIdx.x] = j < n ? table[j] : 0xffffffffu;  // an id no valid row can equal
      __syncthreads();
      if (valid) {
        // positions after i only: in the row's own tile start behind it (rounded down to a group of four,
        // with the row's own and earlier positions masked out), in later tiles take everything
        const uint32_t first = c == b ? (threadIdx.x + 1) : 0;
        for (uint32_t k = first & ~3u; k < kWgThreads; k += 4) {
          const u32x4 t = *reinterpret_cast<const u32x4 *>(&tile[k]);
          const bool e0 = t.x == id && k + 0 >= first, e1 = t.y == id && k + 1 >= first;
          const bool e2 = t.z == id && k + 2 >= first, e3 = t.w == id && k + 3 >= first;
          if (e0 || e1 || e2 || e3) found |= TUTTI_ST_DUP_BLOCK;
        }
      }
    }
  }
  if (found && status) atomicOr(status, found);
}

// The same two preconditions in time linear in the table, with one bit per pool block in memory that the caller
// lends (or that the library keeps): a thread sets the bit of its id with an atomic OR and has found a duplicate
// when the bit was already set.  The bits a call uses are cleared by a kernel in front of it (a fill kernel, not
// a memset node, so that the pair can be captured in a graph).
__global__ __launch_bounds__(kWgThreads) void k_bitmap_clear(uint32_t *__restrict__ bits, uint32_t n_words) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += gridDim.x * blockDim.x) bits[i] = 0u;
}

__global__ __launch_bounds__(kWgThreads) void k_table_validate_bitmap(const uint32_t *__restrict__ table, uint32_t n,
                                                                       uint32_t num_blocks, uint32_t *__restrict__ bits,
                                                                       uint32_t *__restrict__ status) {
  uint32_t found = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t id = table[i];
    if (id >= num_blocks) {
      found |= TUTTI_ST_BAD_BLOCK;
    } else {
      const uint32_t bit = 1u << (id & 31u);
      if (atomicOr(&bits[id >> 5], bit) & bit) found |= TUTTI_ST_DUP_BLOCK;
    }
  }
  // one atomic per wavefront that found something
  const uint32_t lane = threadIdx.x & (kWave - 1);
  uint32_t any = found;
#pragma unroll
  for (uint32_t d = kWave / 2; d >= 1; d >>= 1) any |= __shfl_xor(any, d, kWave);
  if (lane == 0 && any && status) atomicOr(status, any);
}

// The visiting order of a table by ascending block id, from the bitmap of its ids: the rank of an id is the number
// of set bits below it.  k_bitmap_prefix (ONE workgroup) turns the per-word bit counts into exclusive prefix sums;
// k_table_rank then places every table position at its id's rank.  If the check that set the bits found an id out
// of range or twice (flags != 0) the ranks are not a permutation and the identity order is written instead.
constexpr uint32_t kPrefixThreads = 1024;

__global__ __launch_bounds__(kPrefixThreads) void k_bitmap_prefix(const uint32_t *__restrict__ bits, uint32_t n_words,
                                                                   uint32_t *__restrict__ prefix) {
  __shared__ uint32_t part[kPrefixThreads];
  const uint32_t t = threadIdx.x;
  const uint32_t per = (n_words + kPrefixThreads - 1) / kPrefixThreads;  // consecutive words per thread
  const uint32_t lo = t * per < n_words ? t * per : n_words;
  const uint32_t hi = lo + per < n_words ? lo + per : n_words;
  uint32_t sum = 0;
  for (uint32_t i = lo; i < hi; ++i) sum += static_cast<uint32_t>(__popc(bits[i]));
  part[t] = sum;
  __syncthreads();
  for (uint32_t d = 1; d < kPrefixThreads; d <<= 1) {  // inclusive scan of the per-thread sums
    const uint32_t v = t >= d ? part[t - d] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  uint32_t run = part[t] - sum;  // bits in front of this thread's words
  for (uint32_t i = lo; i < hi; ++i) {
    prefix[i] = run;
    run += static_cast<uint32_t>(__popc(bits[i]));
  }
}

__global__ __launch_bounds__(kWgThreads) void k_table_rank(const uint32_t *__restrict__ table, uint32_t n,
                                                            const uint32_t *__restrict__ bits,
                                                            const uint32_t *__restrict__ prefix,
                                                            const uint32_t *__restrict__ flags, uint32_t *__restrict__ visit,
                                                            uint32_t *__restrict__ status) {
  const uint32_t found = flags[0];  // what the check in front of this kernel found
  if (found && status && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(status, found);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    if (found) {
      visit[i] = i;
    } else {
      const uint32_t id = table[i];
      const uint32_t below = bits[id >> 5] & ((1u << (id & 31u)) - 1u);
      visit[prefix[id >> 5] + static_cast<uint32_t>(__popc(below))] = i;
    }
  }
}

#ifdef TUTTI_BENCH_BUILD
// ---- measurement kernels (libtutti_bench.so only)

// Plain contiguous copy with the access shape of move_items: the ceiling pack / unpack can reach.
template <int U, int NT, int WG>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_copy(unsigned char *__restrict__ dst,
                                                      const unsigned char *__restrict__ src, uint64_t bytes) {
  constexpr uint64_t kSlice = kWave * 16ull * U;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint64_t n_waves = static_cast<uint64_t>(gridDim.x) * (blockDim.x / kWave);
  const uint64_t n_items = (bytes + kSlice - 1) / kSlice;
  for (uint64_t it = static_cast<uint64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave; it < n_items;
       it += n_waves) {
    const uint64_t o0 = it * kSlice + lane * 16ull;
    if ((it + 1) * kSlice <= bytes) {
      u32x4 buf[U];
#pragma unroll
      for (int k = 0; k < U; ++k) buf[k] = ld16<NT>(src + o0 + k * (kWave * 16ull));
      if (U > 4) __builtin_amdgcn_sched_barrier(0);  // one run of loads, one of stores, as in load_slice and store_slice
#pragma unroll
      for (int k = 0; k < U; ++k) st16<NT>(dst + o0 + k * (kWave * 16ull), buf[k]);
    } else {
      for (int k = 0; k < U; ++k) {
        const uint64_t o = o0 + k * (kWave * 16ull);
        if (o < bytes) st16<NT>(dst + o, ld16<NT>(src + o));
      }
    }
  }
}

// One direction only, same access shape: READ xors every 16-byte unit into four words per wavefront, added to
// one of TUTTI_STREAM_SLOTS slots at the end, FILL writes unit i as {lo(i), hi(i), ~lo(i), tag}.  What a CU, or the chip, can read or
// write when it does nothing else.
constexpr uint32_t kFillTag = 0x54555454u;

template <int WRITE, int U, int WG>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_stream(unsigned char *__restrict__ buf, uint64_t bytes, uint32_t *__restrict__ xor4) {
  constexpr uint64_t kSlice = kWave * 16ull * U;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint64_t n_waves = static_cast<uint64_t>(gridDim.x) * (blockDim.x / kWave);
  const uint64_t n_items = (bytes + kSlice - 1) / kSlice;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (uint64_t it = static_cast<uint64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave; it < n_items;
       it += n_waves) {
    const uint64_t o0 = it * kSlice + lane * 16ull;
    const bool whole = (it + 1) * kSlice <= bytes;
    if (WRITE) {
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint64_t o = o0 + k * (kWave * 16ull);
        const uint64_t unit = o >> 4;
        const u32x4 v = {static_cast<uint32_t>(unit), static_cast<uint32_t>(unit >> 32), ~static_cast<uint32_t>(unit),
                         kFillTag};
        if (whole || o < bytes) st16<3>(buf + o, v);
      }
    } else if (whole) {
      u32x4 v[U];
#pragma unroll
      for (int k = 0; k < U; ++k) v[k] = ld16<3>(buf + o0 + k * (kWave * 16ull));
#pragma unroll
      for (int k = 0; k < U; ++k) acc ^= v[k];
    } else {
      for (int k = 0; k < U; ++k) {
        const uint64_t o = o0 + k * (kWave * 16ull);
        if (o < bytes) acc ^= ld16<3>(buf + o);
      }
    }
  }
  if (!WRITE) {
#pragma unroll
    for (uint32_t d = kWave / 2; d >= 1; d >>= 1) {
      acc.x ^= __shfl_xor(acc.x, d, kWave);
      acc.y ^= __shfl_xor(acc.y, d, kWave);
      acc.z ^= __shfl_xor(acc.z, d, kWave);
      acc.w ^= __shfl_xor(acc.w, d, kWave);
    }
    if (lane == 0) {
      // one slot per wavefront (modulo the slot count): atomics on one address from every wavefront of the chip
      // would take longer than the reads themselves
      const uint32_t w = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
      uint32_t *slot = xor4 + 4u * (w % TUTTI_STREAM_SLOTS);
      atomicXor(&slot[0], acc.x);
      atomicXor(&slot[1], acc.y);
      atomicXor(&slot[2], acc.z);
      atomicXor(&slot[3], acc.w);
    }
  }
}

// The copy with one side permuted at `gran` bytes: the memory system's own cost of the scatter.
template <int U, int WG>
__global__ __launch_bounds__(WG, min_waves_per_simd(WG, U)) void k_scatter(unsigned char *__restrict__ scattered, uint64_t span_bytes,
                                                 unsigned char *__restrict__ contig, uint64_t bytes,
                                                 const uint32_t *__restrict__ perm, uint32_t gran, uint32_t to_scattered) {
  constexpr uint32_t kSlice = kWave * 16u * U;  // gran is a multiple of 4096 and of kSlice (host-checked)
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave_in_wg = rfl(threadIdx.x / kWave);
  const uint64_t n_waves = static_cast<uint64_t>(gridDim.x) * (blockDim.x / kWave);
  const uint32_t per = gran / kSlice;
  const uint64_t n_items = bytes / kSlice;
  for (uint64_t it = static_cast<uint64_t>(blockIdx.x) * (blockDim.x / kWave) + wave_in_wg; it < n_items; it += n_waves) {
    const uint64_t piece = it / per;
    const uint32_t s = static_cast<uint32_t>(it - piece * per);
    const uint64_t so = static_cast<uint64_t>(rfl(perm[piece])) * gran;
    if (so + gran > span_bytes) continue;
    unsigned char *sp = scattered + so + s * kSlice + lane * 16u;
    unsigned char *cp = contig + it * kSlice + lane * 16u;
    const unsigned char *src = to_scattered ? cp : sp;
    unsigned char *dst = to_scattered ? sp : cp;
    u32x4 buf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) buf[u] = ld16<3>(src + u * (kWave * 16u));
#pragma unroll
    for (int u = 0; u < U; ++u) st16<3>(dst + u * (kWave * 16u), buf[u]);
  }
}

// The same scattered copy with the work dealt differently: a whole piece per wavefront (PER_WG = false) or per
// workgroup (true), walked in 4 KiB steps, with any of the four cache policies.  Whether another way of dealing
// out the same bytes would suit the memory system better than the product's wavefront-per-4-KiB.
template <bool PER_WG, int NT>
__global__ __launch_bounds__(kWgThreads, 8) void k_scatter_piece(unsigned char *__restrict__ scattered, uint64_t span_bytes,
                                                                  unsigned char *__restrict__ contig, uint64_t bytes,
                                                                  const uint32_t *__restrict__ perm, uint32_t gran,
                                                                  uint32_t to_scattered) {
  constexpr uint32_t kStep = kWave * 16u * 4u;  // 4 KiB per wavefront and step; gran is a multiple of it
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave_in_wg = rfl(threadIdx.x / kWave);
  const uint32_t waves = blockDim.x / kWave;
  const uint64_t n_pieces = bytes / gran;
  const uint64_t first = PER_WG ? blockIdx.x : static_cast<uint64_t>(blockIdx.x) * waves + wave_in_wg;
  const uint64_t stride = PER_WG ? gridDim.x : static_cast<uint64_t>(gridDim.x) * waves;
  for (uint64_t piece = first; piece < n_pieces; piece += stride) {
    const uint64_t so = static_cast<uint64_t>(rfl(perm[piece])) * gran;
    if (so + gran > span_bytes) continue;
    for (uint32_t off = PER_WG ? wave_in_wg * kStep : 0u; off < gran; off += PER_WG ? waves * kStep : kStep) {
      unsigned char *sp = scattered + so + off + lane * 16u;
      unsigned char *cp = contig + piece * gran + off + lane * 16u;
      const unsigned char *src = to_scattered ? cp : sp;
      unsigned char *dst = to_scattered ? sp : cp;
      u32x4 buf[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) buf[u] = ld16<NT>(src + u * (kWave * 16u));
#pragma unroll
      for (int u = 0; u < 4; ++u) st16<NT>(dst + u * (kWave * 16u), buf[u]);
    }
  }
}

#endif  // TUTTI_BENCH_BUILD

}  // namespace tutti
