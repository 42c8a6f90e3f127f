// The arguments of a fused launch in 112 bytes.  Plain C++, so that it can be tested without a GPU.
#pragma once

#include <stdint.h>

namespace tutti {

// The runtime copies the arguments of every launch into memory from malloc, which it gives back when the kernel has
// ended.  Up to 112 bytes that is one of malloc's smallest chunks, kept in lists of their own size; a larger one is
// merged with its neighbours and cut out again.  A train of launches of an otherwise empty kernel, us each, by bytes of
// arguments (the first train after a start takes 2.5 to 2.8 with any):
//   32  2.64   64  2.80   96  2.85   104  2.88   112  2.88   120  3.45   128  3.6   160  3.65   264  3.7   384  3.8
// So a fused launch hands over bit fields (its arguments as separate words are 260 bytes), and the kernel takes them apart
// with some thirty scalar instructions.  Calls from Python, us, words / fields: restore of 256 KiB 4.2 / 3.4, a train of 32 of
// 4 MiB 131 / 113 and 139 / 116; the kernels by themselves (graph replay of 60 kinds of call) take the same time within 0.2 %;
// the smallest 0.03 us more, and small ones on 32 compute units whose blocks are moved as pieces 0.05 to 0.2 (8 blocks of one request,
// token-major of 12.5 KiB 5.4 / 5.5, head-major of 10 and 30 KiB 5.7 / 5.9; 256 blocks the same).  An ordered restore hands over 120
// bytes (OrderedLateWords).
//
// What a field leaves out is what it cannot hold: addresses lie below 2^47 (the host checks the ones that are used), planes,
// staging, entries, strides and block sizes are multiples of 16, a chunk is a multiple of the alignment, which is a power of two.
constexpr uint32_t kLayerCallWords = 14, kEarlyWords = 7;
struct LayerCall {
  uint64_t w[kLayerCallWords];
};
static_assert(sizeof(LayerCall) <= 112, "one of malloc's smallest chunks");

struct LayerFields {
  uint64_t k_base, v_base, stage, sqe;                             // addresses, multiples of 16
  uint64_t table, n_blocks, extents, totals, file_id, status;      // addresses
  uint64_t block_stride;                                           // multiple of 16; taken as signed
  uint64_t stage_cap;                                              // rounded down to 16; 2^47 - 16 where it is more
  uint64_t stage_addr;                                             // multiple of 16
  uint32_t num_blocks, table_len, block_bytes, chunk_bytes, sqe_cap, sgl_id, layer, n_req, align;
  uint32_t sqe_wgs, copy_wgs, copy_first;                          // workgroups, at most kMostWgs + 7 each
  uint32_t chip_waves;                                             // rounded down to 128; 127 * 128 where it is more
  uint32_t dense, xcd_contiguous;                                  // 0 or 1
  uint32_t size_a, size_b, left_out;                               // of a block (BlockSizes), or of its slices
};

// Tokens, heads and row size of a head-major block: two of them, in 14 bits each, and which one is left out, the block having
// the size that it has.  With the row in units of 16 bytes the three make up at most 2^28, so no two are above 2^14.
struct BlockSizes {
  uint32_t tokens, heads, row_bytes;
};
constexpr uint32_t kMostSize = 1u << 14;
constexpr void put_sizes(LayerFields &f, BlockSizes s) {
  const uint32_t row = s.row_bytes / 16;
  f.left_out = s.tokens <= kMostSize && row <= kMostSize ? 0u : s.heads <= kMostSize && row <= kMostSize ? 1u : 2u;
  f.size_a = f.left_out == 1 ? s.heads : s.tokens;
  f.size_b = f.left_out == 2 ? s.heads : row;
}
constexpr uint32_t log2_of(uint32_t power) { return 31u - static_cast<uint32_t>(__builtin_clz(power)); }
// `powers`: all three are powers of two.
constexpr BlockSizes get_sizes(const LayerFields &f, bool powers) {
  const uint32_t units = f.block_bytes / 16;
  const uint32_t third = powers ? units >> (log2_of(f.size_a) + log2_of(f.size_b)) : units / (f.size_a * f.size_b);
  return BlockSizes{f.left_out == 1 ? third : f.size_a, f.left_out == 0 ? third : f.left_out == 1 ? f.size_a : f.size_b,
                    16 * (f.left_out == 2 ? third : f.size_b)};
}

namespace layer_call {
struct Bits {
  uint32_t at, n;
};
// The first words, kEarlyWords of them, are in scalar registers when a wavefront of several requests' kernels starts (k_layer): they hold what the way to the
// first load of a restore needs, and most of a save's.  Each field there is one piece of one word.
constexpr Bits kCopyWgs{0, 12}, kCopyFirst{12, 12}, kSqeWgs{24, 12}, kChip{36, 7}, kXcd{43, 1}, kAlign{44, 5}, kDense{49, 1},
    kLeftOut{50, 2}, kLayerLow{52, 12};
constexpr Bits kBlockBytes{64, 28}, kSizeA{92, 14}, kSizeB{106, 14}, kLayerHigh{120, 4};
constexpr Bits kNumBlocks{128, 32}, kTableLen{160, 31};
constexpr Bits kStage{192, 44}, kReqs{236, 12};
constexpr Bits kNBlocks{256, 47}, kTable{320, 47}, kStageCap{384, 43};
constexpr Bits kKBase{448, 44}, kVBase{512, 44}, kStride{576, 44};
constexpr Bits kStageAddr{640, 60}, kSqeCap{704, 32}, kSglId{736, 32}, kExtents{768, 47}, kTotals{832, 47};

// What those leave free, one gap behind the other, holds the fields that only the entry writers and the error paths read.
constexpr uint32_t kGaps = 11;
constexpr Bits gap(uint32_t i) {
  switch (i) {
    case 0: return Bits{303, 17};  // behind n_blocks
    case 1: return Bits{367, 17};  // table
    case 2: return Bits{427, 21};  // stage_cap
    case 3: return Bits{492, 20};  // k_base
    case 4: return Bits{556, 20};  // v_base
    case 5: return Bits{620, 20};  // block_stride
    case 6: return Bits{815, 17};  // extents
    case 7: return Bits{879, 17};  // totals
    case 8: return Bits{248, 8};   // n_req
    case 9: return Bits{124, 4};   // the layer's upper bits
    default: return Bits{700, 4};  // stage_addr
  }
}
constexpr Bits kFileId{0, 47}, kStatus{47, 47}, kSqe{94, 43}, kChunk{137, 28};  // `at` counts through the gaps
constexpr uint32_t gap_bits(uint32_t i = 0) { return i == kGaps ? 0 : gap(i).n + gap_bits(i + 1); }
static_assert(gap_bits() == kChunk.at + kChunk.n, "the last field ends the last gap");

constexpr uint64_t kBelow(uint32_t n) { return n == 64 ? ~0ull : (1ull << n) - 1; }
constexpr uint64_t get(const LayerCall &c, Bits f) {
  const uint32_t i = f.at / 64, s = f.at % 64;
  uint64_t v = c.w[i] >> s;
  if (s + f.n > 64) v |= c.w[i + 1] << (64 - s);
  return v & kBelow(f.n);
}
constexpr uint32_t get32(const LayerCall &c, Bits f) { return static_cast<uint32_t>(get(c, f)); }
constexpr void put(LayerCall &c, Bits f, uint64_t v) {
  const uint32_t i = f.at / 64, s = f.at % 64;
  v &= kBelow(f.n);
  c.w[i] |= v << s;
  if (s + f.n > 64) c.w[i + 1] |= v >> (64 - s);
}

// The same for a field in the gaps: the part of it that lies in gap `i`, which starts at `pos`, and in those behind.
constexpr Bits part_in(Bits f, uint32_t i, uint32_t pos) {
  const uint32_t lo = f.at > pos ? f.at : pos, end = f.at + f.n, gap_end = pos + gap(i).n, hi = end < gap_end ? end : gap_end;
  return lo < hi ? Bits{lo, hi - lo} : Bits{0, 0};
}
constexpr uint64_t get_from_gaps(const LayerCall &c, Bits f, uint32_t i = 0, uint32_t pos = 0) {
  if (i == kGaps) return 0;
  const Bits p = part_in(f, i, pos);
  const uint64_t here = p.n == 0 ? 0 : get(c, Bits{gap(i).at + p.at - pos, p.n}) << (p.at - f.at);
  return here | get_from_gaps(c, f, i + 1, pos + gap(i).n);
}
constexpr void put_into_gaps(LayerCall &c, Bits f, uint64_t v, uint32_t i = 0, uint32_t pos = 0) {
  if (i == kGaps) return;
  const Bits p = part_in(f, i, pos);
  if (p.n != 0) put(c, Bits{gap(i).at + p.at - pos, p.n}, v >> (p.at - f.at));
  put_into_gaps(c, f, v, i + 1, pos + gap(i).n);
}
}  // namespace layer_call

constexpr uint64_t kAddressEnd = 1ull << 47;  // user addresses, of the host and of the GPU alike, lie below
constexpr uint32_t kMostWgs = 4088;           // workgroups of a launch that the fields hold

// The blocks of a pool that memory can be at.  With a stride that the field does not hold that is block 0 alone: the others count
// as ids that the pool has not got (a bad id is skipped and reported), instead of lying where the stride's low bits say.
struct PoolBlocks {
  uint64_t stride;
  uint32_t n;
};
constexpr PoolBlocks blocks_in_memory(uint64_t stride, uint32_t n) {
  const bool held = stride + kAddressEnd < 2 * kAddressEnd;  // as a signed number from -2^47 on and below 2^47
  return PoolBlocks{held ? stride : 0, held || n == 0 ? n : 1};
}

constexpr LayerCall pack(const LayerFields &f) {
  using namespace layer_call;
  LayerCall c{};
  put(c, kKBase, f.k_base >> 4);
  put(c, kVBase, f.v_base >> 4);
  put(c, kStage, f.stage >> 4);
  put_into_gaps(c, kSqe, f.sqe >> 4);
  put(c, kTable, f.table);
  put(c, kNBlocks, f.n_blocks);
  put(c, kExtents, f.extents);
  put(c, kTotals, f.totals);
  put_into_gaps(c, kFileId, f.file_id);
  put_into_gaps(c, kStatus, f.status);
  put(c, kStride, f.block_stride >> 4);
  put(c, kStageCap, (f.stage_cap < kAddressEnd ? f.stage_cap : kAddressEnd - 16) >> 4);
  put(c, kStageAddr, f.stage_addr >> 4);
  put(c, kNumBlocks, f.num_blocks);
  put(c, kTableLen, f.table_len);
  put(c, kBlockBytes, f.block_bytes >> 4);
  put_into_gaps(c, kChunk, f.chunk_bytes >> 4);
  put(c, kSqeCap, f.sqe_cap);
  put(c, kSglId, f.sgl_id);
  put(c, kLayerLow, f.layer);
  put(c, kLayerHigh, f.layer >> 12);
  put(c, kReqs, f.n_req);
  put(c, kAlign, log2_of(f.align));
  put(c, kSqeWgs, f.sqe_wgs);
  put(c, kCopyWgs, f.copy_wgs);
  put(c, kCopyFirst, f.copy_first);
  put(c, kChip, f.chip_waves / 128 < 127 ? f.chip_waves / 128 : 127);
  put(c, kDense, f.dense);
  put(c, kXcd, f.xcd_contiguous);
  put(c, kSizeA, f.size_a - 1);
  put(c, kSizeB, f.size_b - 1);
  put(c, kLeftOut, f.left_out);
  return c;
}

constexpr LayerFields unpack(const LayerCall &c) {
  using namespace layer_call;
  LayerFields f{};
  f.k_base = get(c, kKBase) << 4;
  f.v_base = get(c, kVBase) << 4;
  f.stage = get(c, kStage) << 4;
  f.sqe = get_from_gaps(c, kSqe) << 4;
  f.table = get(c, kTable);
  f.n_blocks = get(c, kNBlocks);
  f.extents = get(c, kExtents);
  f.totals = get(c, kTotals);
  f.file_id = get_from_gaps(c, kFileId);
  f.status = get_from_gaps(c, kStatus);
  f.block_stride = static_cast<uint64_t>(static_cast<int64_t>(get(c, kStride) << 20) >> 16);
  f.stage_cap = get(c, kStageCap) << 4;
  f.stage_addr = get(c, kStageAddr) << 4;
  f.num_blocks = get32(c, kNumBlocks);
  f.table_len = get32(c, kTableLen);
  f.block_bytes = get32(c, kBlockBytes) << 4;
  f.chunk_bytes = static_cast<uint32_t>(get_from_gaps(c, kChunk)) << 4;
  f.sqe_cap = get32(c, kSqeCap);
  f.sgl_id = get32(c, kSglId);
  f.layer = get32(c, kLayerHigh) << 12 | get32(c, kLayerLow);
  f.n_req = get32(c, kReqs);
  f.align = 1u << get32(c, kAlign);
  f.sqe_wgs = get32(c, kSqeWgs);
  f.copy_wgs = get32(c, kCopyWgs);
  f.copy_first = get32(c, kCopyFirst);
  f.chip_waves = 128 * get32(c, kChip);
  f.dense = get32(c, kDense);
  f.xcd_contiguous = get32(c, kXcd);
  f.size_a = get32(c, kSizeA) + 1;
  f.size_b = get32(c, kSizeB) + 1;
  f.left_out = get32(c, kLeftOut);
  return f;
}

}  // namespace tutti
