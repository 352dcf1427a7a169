// decode.hip -- routed decode over an INT8 key/value cache (TileMix, arXiv 2608.17336,
// Appendix C "Additional Execution Interfaces").
//
// One new query token per (sequence, query head) attends to the L_k cached keys.  Cached K8
// (with its FP16 block scales) feeds the INT8 score path, the FP16 key cache the FP16 path;
// the routing bit of the key's tile group chooses (Sections 4.2, 4.3).  Cached V8 is widened
// to float on chip and its block scale is folded into the probability before the P.V
// product.  Decode reads every cached byte once and does O(1) work per byte, so it is bound
// by HBM bandwidth; a split-K layout spreads each (sequence, KV head) stream over many
// workgroups.
//
//   decode_partial_kernel<D>: workgroup (chunk of keys, KV head, sequence), 8 waves.  The grid
//     is sized for one 8-wave workgroup per CU (256 on an MI355X): each wave streams about the same
//     number of 64-key tiles (tile t of the chunk goes to wave t % 8, so the eight waves read
//     neighbouring tiles at a time) and keeps its own online-softmax state (max,
//     normalizer, output) in registers across them; the group's query heads (G <= 16) sit on
//     the columns of 16x16 matrix-core tiles (padding columns carry no weight).  Per tile the
//     wave issues the key rows on the routed path and the value rows together, scores the tile
//     (v_mfma_i32_16x16x64_i8 on K8 rows, v_mfma_f32_16x16x32_f16 on FP16 key rows), and adds
//     V^T (P dV)^T on v_mfma_f32_16x16x32_f16 with P in registers.  The group's query rows are
//     quantized on chip once per workgroup (the lone decode row is a whole 128-row
//     quantization block), while the first tile is on its way.  At the end the waves' states are
//     merged through LDS with the
//     log-sum-exp rule; the workgroup writes (max, normalizer, unnormalized output) per
//     (sequence, query head, chunk).
//   decode_combine_kernel: merges the chunks of one (sequence, query head) with the
//     log-sum-exp rule and writes O in FP16.
// A ragged batch (per-sequence cache lengths in a padded cache) runs the same kernels.  Its chunks
// are cut on the device, from the lengths themselves, so that every workgroup streams about the
// same number of tiles whatever the lengths (by every wave, or for more than 64 sequences by a
// kernel before the others); a sequence with no key gets O = 0.
#include "tilemix_device.h"
#include "tilemix_internal.h"

#include <algorithm>
#include <type_traits>

namespace tilemix {

namespace {

// Waves per workgroup.  With 8, one workgroup fills a CU, and fewer partial results are written: the
// choice for one sequence and for sequences of one length.  Chunks that are cut by several lengths
// differ: with 4, two workgroups share a CU, and the start and end of one overlap the streaming of
// the other.
constexpr int kDecWavesEven = 8, kDecWavesRagged = 4;
constexpr int kDecHeads = 16;                       // query heads per KV head on the MFMA columns
constexpr int kDecResident = 2048;                  // waves of the partial kernel resident at once
// Waves that share the tiles of a ragged batch: more than run at once, since its chunks differ (a
// sequence's last one is shorter).  Only where the lengths are alike and a chunk is short is it as many as
// run at once, provided that its workgroups are no more than run at once either: one round, where 3072
// waves would take two of three quarters.  us a call, half of the tiles on each route, 32 / 8
// heads, d = 128, 2048 / 3072 waves:
//   32 sequences of 64 to 8192 keys     81.3 / 78.1    16 x 4096 keys                 30.7 / 32.6
//   48 of 2004 to 4096                  92.0 / 80.5    16 x 16000, 16 / 4 heads       55.6 / 63.2
//   48 of 3501 to 4096 (768 workgroups) 104  / 91      8 of 14165 to 16384, 64 heads  56.3 / 61.3
//   4 x 65536, 64 heads (16 tiles)      131  / 125     4 x 57000, 64 heads (14 tiles) 111 / 115
// and with 8 waves, one sequence of 65536, 64 heads     32.0 / 38.0
constexpr int kDecRaggedWaves = 3072;
constexpr int kDecOneRoundTiles = 14;               // most key tiles per wave of a short chunk
constexpr int kCombineThreads = 256;

// Eight int8 codes (one per byte of v) widened to FP16, exactly: with the sign bit flipped a
// byte b reads as 1024 + 128 + b in the FP16 pattern 0x64xx, and 1152 is then subtracted.
__device__ __forceinline__ half8 i8x8_to_half8(uint32_t w0, uint32_t w1) {
  const half2v bias = {(_Float16)-1152.0f, (_Float16)-1152.0f};
  half8 out;
  const uint32_t w[2] = {w0 ^ 0x80808080u, w1 ^ 0x80808080u};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    // bytes 0,1 -> halves 0x64b0, 0x64b1; bytes 2,3 -> 0x64b2, 0x64b3
    const uint32_t p01 = __builtin_amdgcn_perm(0x64646464u, w[i], 0x07010700u);
    const uint32_t p23 = __builtin_amdgcn_perm(0x64646464u, w[i], 0x07030702u);
    const half2v h01 = __builtin_bit_cast(half2v, p01) + bias;
    const half2v h23 = __builtin_bit_cast(half2v, p23) + bias;
    out[4 * i + 0] = h01[0]; out[4 * i + 1] = h01[1];
    out[4 * i + 2] = h23[0]; out[4 * i + 3] = h23[1];
  }
  return out;
}

// Key tiles of sequence b of a ragged batch.
__device__ __forceinline__ int ragged_keys(const DecodeArgs& a, int b) {
  return min(max(a.seqlens[b], 0), a.Lk);
}
__device__ __forceinline__ int ragged_tiles(const DecodeArgs& a, int b) {
  return b < a.B ? (ragged_keys(a, b) + kBlockN - 1) / kBlockN : 0;
}

// Chunks of a ragged batch: all hold `tiles` key tiles (a sequence's last one maybe fewer), the same
// number for every wave and the fewest for which the KV heads' chunks fit kDecRaggedWaves, up to one
// more per sequence and head.  Chunk slots are numbered sequence after sequence.
// With an equal share of the capacity per workgroup instead, the longest sequence decides: 32 sequences
// of 395 to 8192 keys, 32 / 8 heads, d = 128, all INT8, take 74.9 us; cut by length 60.1.
// total: key tiles of the batch; some: its sequences with any; longest: the most of one; chunks_of(tiles):
// the chunks of all sequences at so many tiles a chunk.  Alike: within 20% of the longest in the mean.
// One sequence has chunks of one size, whatever its length: one round.
template <typename F>
__device__ __forceinline__ int ragged_chunk_tiles(const DecodeArgs& a, int total, int some, int longest, F&& chunks_of) {
  const int share = total * a.Hk;   // (B H_k <= 65535 and 4096 tiles each: these fit 31 bits)
  const int one_round = (share + kDecResident - 1) / kDecResident;
  if (a.B == 1) return a.waves * max(1, one_round);
  if (5 * total >= 4 * some * longest && one_round <= kDecOneRoundTiles) {
    const int tiles = a.waves * max(1, one_round);
    if (chunks_of(tiles) * a.Hk <= kDecResident / a.waves) return tiles;
  }
  return a.waves * max(1, (share + kDecRaggedWaves - 1) / kDecRaggedWaves);
}
// ceil(t / tiles) for t <= 4096, inv = 1 / tiles: the quotient's distance from the next whole number,
// at least 1 / (2 tiles), is far above its rounding error.
__device__ __forceinline__ int ragged_chunks_of(int t, int tiles, float inv) {
  return (int)(((float)(t + tiles - 1) + 0.5f) * inv);
}
// Of up to 64 sequences, t: the tiles of the lane's.
__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_scan(x), kWave - 1); }
__device__ __forceinline__ int ragged_chunk_tiles(const DecodeArgs& a, int t) {
  if (a.B == 1) return ragged_chunk_tiles(a, __builtin_amdgcn_readfirstlane(t), 1, 0, [](int) { return 0; });
  const int longest = __builtin_amdgcn_readfirstlane((int)wave_max((float)t));
  return ragged_chunk_tiles(a, wave_sum(t), __popcll(__ballot(t > 0)), longest,
                            [&](int tiles) { return wave_sum(ragged_chunks_of(t, tiles, 1.0f / (float)tiles)); });
}

// A batch of up to kCutInWave sequences is cut by every wave for itself, one length a lane.  For more, the
// walk over the lengths would delay every workgroup; one workgroup then writes the cut down before the
// others start: {tiles, slots in use}, the first slot of every sequence and one past the last, and
// {sequence, chunk} of every slot in use.  1024 sequences of up to 256 keys, 32 / 8 heads, d = 128: 336 us
// with the walk in every wave, 217 with an equal share of the capacity for each workgroup, 128 so; 256
// sequences of up to 1024 keys 95.8, 95.7, 79.3; 100 sequences, one of them long: 15.1, 97.7, 16.4.
constexpr int kCutInWave = kWave;
__host__ __device__ constexpr size_t cut_first_at() { return 2; }
__host__ __device__ constexpr size_t cut_slots_at(int batch) { return (cut_first_at() + batch + 1 + 1) & ~(size_t)1; }

// The chunk of a workgroup.  Ids run over the slots in use (a multiple of kSlotsPad, so that a slot's
// workgroups of all KV heads are on one XCD: at d = 64 two heads' K8 rows share a cache line) of one head
// after another.  The workgroups beyond, which only the device can tell, are the last: in between
// they would leave CUs without work (4 x 65536 keys, all INT8, 64 / 8 heads, d = 64: 70.5 us with the
// unused slots of every head in between, 50.9 so).
constexpr int kSlotsPad = 8;
struct RaggedChunk {
  int tiles, hk, slot, b, chunk;   // b = -1: no chunk
  __device__ __forceinline__ bool place(const DecodeArgs& a, int id, int used) {
    const int padded = (used + kSlotsPad - 1) / kSlotsPad * kSlotsPad;
    hk = padded ? id / padded : a.Hk;
    slot = id - hk * padded;
    return hk < a.Hk && slot < used;
  }
  __device__ __forceinline__ RaggedChunk(const DecodeArgs& a, int id, int lane) : tiles(0), b(-1), chunk(0) {
    if (a.cut) {
      if (!place(a, id, a.cut[1])) return;
      tiles = a.cut[0];
      const int2 e = reinterpret_cast<const int2*>(a.cut + cut_slots_at(a.B))[slot];
      b = __builtin_amdgcn_readfirstlane(e.x);
      chunk = __builtin_amdgcn_readfirstlane(e.y);
      return;
    }
    const int t = ragged_tiles(a, lane);
    tiles = ragged_chunk_tiles(a, t);
    const int n = ragged_chunks_of(t, tiles, 1.0f / (float)tiles), end = wave_scan(n);
    if (!place(a, id, __builtin_amdgcn_readlane(end, kWave - 1))) return;
    const uint64_t hit = __ballot(slot >= end - n && slot < end);
    if (hit) {
      b = __builtin_ctzll(hit);
      chunk = slot - (__builtin_amdgcn_readlane(end, b) - __builtin_amdgcn_readlane(n, b));
    }
  }
};

struct RaggedSequence {
  int first, count;   // its slots
  __device__ __forceinline__ RaggedSequence(const DecodeArgs& a, int seq, int lane) {
    if (a.cut) {
      first = a.cut[cut_first_at() + seq];
      count = a.cut[cut_first_at() + seq + 1] - first;
      return;
    }
    const int t = ragged_tiles(a, lane);
    const int tiles = ragged_chunk_tiles(a, t);
    const int n = ragged_chunks_of(t, tiles, 1.0f / (float)tiles);
    first = __builtin_amdgcn_readlane(wave_scan(n) - n, seq);
    count = __builtin_amdgcn_readlane(n, seq);
  }
};

// The cut of a batch of many sequences, by one workgroup.
constexpr int kCutThreads = 1024, kCutWaves = kCutThreads / kWave;
__global__ __launch_bounds__(kCutThreads) void ragged_cut_kernel(DecodeArgs a) {
  __shared__ int sum[kCutWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  // Sums of v over the waves before this one and over all of them.
  auto across = [&](int v, int& before) {
    __syncthreads();
    if (lane == kWave - 1) sum[wave] = v;
    __syncthreads();
    int all = 0;
    before = 0;
#pragma unroll
    for (int w = 0; w < kCutWaves; ++w) {
      if (w == wave) before = all;
      all += sum[w];
    }
    return all;
  };
  __shared__ float longest[kCutWaves];
  int mine = 0, some = 0, most = 0, before;
#pragma unroll 4
  for (int b = tid; b < a.B; b += kCutThreads) {
    const int t = ragged_tiles(a, b);
    mine += t;
    some += t > 0 ? 1 : 0;
    most = max(most, t);
  }
  const float wave_most = wave_max((float)most);
  if (lane == 0) longest[wave] = wave_most;
  const int total = across(wave_scan(mine), before);   // (its barriers are the ones for longest, too)
  float all_most = 0.0f;
#pragma unroll
  for (int w = 0; w < kCutWaves; ++w) all_most = fmaxf(all_most, longest[w]);
  const int tiles = ragged_chunk_tiles(a, total, across(wave_scan(some), before), (int)all_most, [&](int tiles) {
    int chunks = 0;
#pragma unroll 4
    for (int b = tid; b < a.B; b += kCutThreads) chunks += ragged_chunks_of(ragged_tiles(a, b), tiles, 1.0f / (float)tiles);
    return across(wave_scan(chunks), before);
  });
  const float inv = 1.0f / (float)tiles;
  int* first = a.cut + cut_first_at();
  int2* slots = reinterpret_cast<int2*>(a.cut + cut_slots_at(a.B));
  int base = 0;
  for (int b0 = 0; b0 < a.B; b0 += kCutThreads) {
    const int b = b0 + tid, n = ragged_chunks_of(ragged_tiles(a, b), tiles, inv), end = wave_scan(n);
    const int all = across(end, before), at = base + before + end - n;
    if (b < a.B) first[b] = at;
    for (int i = 0; i < n; ++i) slots[at + i] = make_int2(b, i);
    base += all;
  }
  if (tid == 0) {
    a.cut[0] = tiles;
    a.cut[1] = base;
    first[a.B] = base;
  }
}

// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float quad_rows_max(float x) {
  const int v = __builtin_bit_cast(int, x);
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return pair_max(fmaxf(__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1])));
}

// Workgroup = (chunk of chunk_tiles key tiles, KV head, sequence), or with `balanced` a slot and KV
// head of the ragged batch, as RaggedChunk places them.
//
// Scores are computed transposed, S^T = K Q^T, with keys on the 16 rows and the group's query
// heads on the 16 columns of each tile product.  Score block blk (= 2 * st + h) of a tile puts
// key 16 * (i / 4) + 4 * blk + i % 4 on row i, so that lane (head, lq) receives the keys
// 16 * lq + 8 * st + 4 * h + r (r < 4): for each st these are the eight keys 16 * lq + 8 * st + e
// that the B operand of P.V step st needs in lane (head, lq), slot e.  P therefore never
// leaves the registers, and the V^T operand of step st is bytes [16 * lq + 8 * st, + 8) of a
// channel row of the transposed value tile: one 16-byte load per lane covers both steps.
// Registers (about 180 per lane: key rows, value rows, output, scores) allow two waves per
// SIMD, so one 8-wave workgroup fills a CU.
template <int D, int kDecWaves>
__global__ __launch_bounds__(kDecWaves * kWave) __attribute__((amdgpu_waves_per_eu(2)))
void decode_partial_kernel(DecodeArgs a) {
  constexpr int kDecThreads = kDecWaves * kWave;
  constexpr int kCB = D / 16;      // 16-channel blocks of the output
  constexpr int kS16 = D / 32;     // FP16 score products per 16-key block
  constexpr int kS8 = D / 64;      // INT8 score products per 16-key block
  constexpr int kQ16 = D + 8, kQ8 = D + 16, kOS = D + 4;   // padded LDS row lengths
  int hk = blockIdx.y;
  const int G = a.Hq / a.Hk;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  int b = blockIdx.z, chunk = blockIdx.x, chunk_tiles = a.chunk_tiles;
  // The partial results of head hq go to row part_row + hq * chunks.
  size_t part_row = (size_t)b * a.Hq * a.chunks + chunk;
  if (a.balanced) {
    const RaggedChunk r(a, blockIdx.x, lane);
    if (r.b < 0) return;
    hk = r.hk;
    b = r.b;
    chunk = r.chunk;
    chunk_tiles = r.tiles;
    part_row = r.slot;
  }
  // Keys of this sequence: all L_k cached ones, or its own length in a ragged batch.  A chunk
  // past the end has nothing to contribute and is not merged.
  const int Lkb = a.seqlens ? ragged_keys(a, b) : a.Lk;
  const int tile0 = chunk * chunk_tiles;   // first key tile of the chunk
  if (tile0 * kBlockN >= Lkb) return;
  const int tile_end = min(tile0 + chunk_tiles, (Lkb + kBlockN - 1) / kBlockN);
  __shared__ __align__(16) _Float16 q16[kDecHeads][kQ16];
  __shared__ __align__(16) int8_t q8[kDecHeads][kQ8];
  __shared__ float cq[kDecHeads];                         // scale * log2(e) * dQ per head
  __shared__ float red_m[kDecWaves][kDecHeads], red_z[kDecWaves][kDecHeads];
  __shared__ __align__(16) float osum[kDecWaves][kDecHeads][kOS];

  // 1. This (sequence, KV head)'s routing row (Section 4.2): lane w holds word w, so a tile's bit
  //    is a lane read plus a shift; and the group's query rows.
  const uint64_t my_word =
      (!a.force_fp16 && lane < a.W) ? a.route[((size_t)(a.route_per_batch ? b : 0) * a.Hk + hk) * a.W + lane] : 0ull;
  constexpr int kHeadsPerWave = kDecHeads / kDecWaves;
  _Float16 qx[kHeadsPerWave][D / 64];
#pragma unroll
  for (int i = 0; i < kHeadsPerWave; ++i) {
    const int g = wave + kDecWaves * i;
#pragma unroll
    for (int e = 0; e < D / 64; ++e)
      qx[i][e] = a.Q[((size_t)b * a.Hq + hk * G + min(g, G - 1)) * D + lane + 64 * e];
  }
  const uint32_t word_lo = (uint32_t)my_word, word_hi = (uint32_t)(my_word >> 32);
  auto route_of = [&](int n) -> bool {
    const int gj = (int)a.div_g.quot(n), w = gj >> 6, bit = gj & 63;
    const uint32_t h = bit < 32 ? __builtin_amdgcn_readlane(word_lo, w) : __builtin_amdgcn_readlane(word_hi, w);
    return (h >> (bit & 31)) & 1u;
  };

  // One key tile in registers: the key rows on the routed path, the value rows and the scales.  K8
  // and FP16 key rows differ only in their row length (D or 2 D bytes): lane lq reads bytes
  // 16 * lq + 64 * s of the row for product s of a 16-key block.  Both have kS8 products in the
  // first half of the registers; only FP16 rows have the second.
  // The halves of an FP16 tile are the first and the second half of each row's bytes.  At d = 64 that
  // would cut each 128-byte line of the cache in two that are requested at different times; there
  // the halves are score blocks 0, 1 and 2, 3 with whole rows: 32 x 8192 keys, 64 / 8 heads 93.6 ->
  // 84.0 us, 4 x 65536 keys 92.3 -> 87.4 (all FP16).  At d = 128, where a half is a line, it measured
  // 0 to 1% slower.
  constexpr bool kHalvesByKey = D == 64;
  auto kr16 = [](int blk, int s) {   // register of product s of block blk on the FP16 route
    return kHalvesByKey ? blk * kS16 + s : blk * kS8 + s % kS8 + 4 * kS8 * (s / kS8);
  };
  uint4 kr[4 * kS16], vr[kCB];
  uint16_t dk_bits = 0, dv_bits = 0;
  // Addresses: a uniform tile base and the lane's 32-bit offset in the tile.  In a wave without a tile
  // every lane's offset is 0, so that the tile it requests all the same (below) costs it a few cache
  // lines: with the whole rows, a cache of 100 keys (2 tiles for 8 waves) took 9.1 us instead of 8.2.
  const bool idle = tile0 + wave >= tile_end;
  const uint32_t row8 = idle ? 0u : (uint32_t)(a.Hk * D);       // bytes between K8 rows
  const uint32_t lane16 = idle ? 0u : 16 * lq;
  const uint32_t lane_key = 16 * (l16 >> 2) + (l16 & 3);        // key of block 0 in the tile
  const uint32_t v_off = idle ? 0u : (uint32_t)(l16 * kBlockN + 16 * lq);
  auto load_keys = [&](int n, bool int8, auto second) {
    const int sh = int8 ? 0 : 1;
    const size_t row0 = (size_t)b * a.Lk + (size_t)n * kBlockN;
    const char* base = (int8 ? reinterpret_cast<const char*>(a.K8) : reinterpret_cast<const char*>(a.K)) +
                       ((row0 * a.Hk + hk) * D << sh);
    const uint32_t last = (uint32_t)(Lkb - 1 - n * kBlockN);    // keys past the length are masked below
    constexpr int kHalf = decltype(second)::value ? 1 : 0;
#pragma unroll
    for (int i = 0; i < 4 * kS8; ++i) {
      int blk = i / kS8, s = i % kS8 + kS8 * kHalf;
      if constexpr (kHalvesByKey) {
        if (!int8) {   // (scalar selects)
          blk = i / kS16 + 2 * kHalf;
          s = i % kS16;
        }
      }
      const uint32_t off = (min(lane_key + 4 * blk, last) * row8 << sh) + lane16;
      kr[i + 4 * kS8 * kHalf] = ld_global_16(base + 64 * s + off);
    }
  };
  auto load_values = [&](int n) {
    const int8_t* vt = a.V8 + (((size_t)b * a.Hk + hk) * a.nKB + n) * (size_t)(D * kBlockN);
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) vr[cb] = ld_global_16(vt + v_off + cb * 16 * kBlockN);
  };
  auto load_scales = [&](int n) {
    const size_t si = ((size_t)b * a.nKB + n) * a.Hk + hk;
    dk_bits = a.dK[si];
    dv_bits = a.dV[si];
  };
  using First = std::integral_constant<bool, false>;
  using Second = std::integral_constant<bool, true>;
  // Rows of a tile are requested in the order keys (first half, second half), scales, values, here
  // and in the loop: loads complete in order, and a wait then counts the same younger loads
  // whichever way it was reached.  For that a wave without a tile requests one, too.
  int n = tile0 + wave;
  bool int8 = route_of(min(n, tile_end - 1));
  {
    const int first = min(n, tile_end - 1);
    load_keys(first, int8, First{});
    if (!int8) load_keys(first, int8, Second{});
    load_scales(first);
    load_values(first);
  }

  // 2. FP16 copy, INT8 codes and FP16-stored scale of the query rows (Appendix C
  //    quantization; the lone decode row forms its own 128-row block).  Rows past G are 0.
#pragma unroll
  for (int i = 0; i < kHeadsPerWave; ++i) {
    const int g = wave + kDecWaves * i;
    if (g < G) {
#pragma unroll
      for (int e = 0; e < D / 64; ++e) q16[g][lane + 64 * e] = qx[i][e];
      float amax = 0.0f;
#pragma unroll
      for (int e = 0; e < D / 64; ++e) amax = fmaxf(amax, fabsf((float)qx[i][e]));
      const BlockScale bs(wave_max(amax));
#pragma unroll
      for (int e = 0; e < D / 64; ++e) q8[g][lane + 64 * e] = (int8_t)bs.word((float)qx[i][e]);
      if (lane == 0) cq[g] = a.scale_log2e * half_bits_to_float(bs.bits);
    } else {
#pragma unroll
      for (int e = 0; e < D / 64; ++e) {
        q16[g][lane + 64 * e] = (_Float16)0.0f;
        q8[g][lane + 64 * e] = 0;
      }
      if (lane == 0) cq[g] = 0.0f;
    }
  }
  __syncthreads();

  // 3. The wave's tiles tile0 + wave, tile0 + wave + 8, ...: scores in log2 units; the running
  //    max, normalizer and output of the wave are rescaled when the max grows (Section 3.1);
  //    P = 2^(s - m) with the V block scale folded in is the FP16 B operand of the P.V products.
  const bool head_ok = l16 < G;   // columns past G are padding
  const float ninf = -__builtin_huge_valf();
  float m_w = ninf, z_w = 0.0f;   // z_w: this lane's share of the normalizer
  f32x4 acc[kCB];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) acc[cb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // A tile's key registers are free once its scores are formed and its value registers after
  // P.V: the next tile's rows are requested there, so that a wave has loads in flight while it
  // computes.  The second half of FP16 key rows waits until P.V has its operands, so that the
  // number of younger loads does not depend on the route where the values are waited for.
  // The last tile, after which nothing is requested, is a copy of the body of its own.
  auto tile_step = [&](auto more) {
    constexpr bool kMore = decltype(more)::value;
    const int next = n + kDecWaves;
    bool next_int8 = false;
    if constexpr (kMore) next_int8 = route_of(next);
    const uint16_t dk_cur = dk_bits, dv_cur = dv_bits;
    // Raw scores (exact INT32 products or FP32 dot products) and the factor f that turns them into
    // log2-domain scaled ones.  Columns past G hold the scores of zero query rows and are never
    // written out.
    float sc[4][4], f;
    if (int8) {
      i32x4 c[4];
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) c[blk] = i32x4{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < kS8; ++s) {   // one query operand slice live at a time
        const i32x4 qb = *reinterpret_cast<const i32x4*>(&q8[l16][64 * s + 16 * lq]);
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
          c[blk] = __builtin_amdgcn_mfma_i32_16x16x64_i8(as_i32x4(kr[blk * kS8 + s]), qb, c[blk], 0, 0, 0);
      }
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[blk][r] = (float)c[blk][r];
      f = cq[l16] * half_bits_to_float(dk_cur);
    } else {
      f32x4 c[4];
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) c[blk] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < kS16; ++s) {
        const half8 qb = *reinterpret_cast<const half8*>(&q16[l16][32 * s + 8 * lq]);
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
          c[blk] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(kr[kr16(blk, s)]), qb, c[blk], 0, 0, 0);
      }
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[blk][r] = c[blk][r];
      f = a.scale_log2e;
    }
    if constexpr (kMore) load_keys(next, next_int8, First{});
    const float dv = half_bits_to_float(dv_cur);
    // Scores are scaled and rounded once, before the max and the exp see them: with an FMA in the exp,
    // 2^(f sc - m) would be taken against the max's own rounding, which overflows P once that exceeds
    // 16 (scores from about 2^28 on).
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i >> 2][i & 3] *= f;
    // Only a sequence's last tile has keys past the length (the others' limit is above every key).
    const int lim = Lkb - n * kBlockN - 16 * lq;
    const bool masked = (n + 1) * kBlockN > Lkb;
    if (masked) {
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[blk][r] = 4 * blk + r < lim ? sc[blk][r] : ninf;
    }
    float mt = sc[0][0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mt = fmaxf(mt, sc[i >> 2][i & 3]);
    const float m_new = fmaxf(m_w, quad_rows_max(mt));
    if (__any(m_new > m_w)) {
      const float alpha = m_w == ninf ? 0.0f : __builtin_amdgcn_exp2f(m_w - m_new);
      z_w *= alpha;
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) acc[cb] *= alpha;
      m_w = m_new;
    }
    const float msub = m_w == ninf ? 0.0f : m_w;   // no finite score so far: P = 0, not a NaN
    half8 pb[2];
#pragma unroll
    for (int blk = 0; blk < 4; ++blk)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = __builtin_amdgcn_exp2f(sc[blk][r] - msub);
        z_w += p;
        pb[blk >> 1][4 * (blk & 1) + r] = (_Float16)(p * dv);
      }
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) {
      acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(i8x8_to_half8(vr[cb].x, vr[cb].y), pb[0], acc[cb], 0, 0, 0);
      acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(i8x8_to_half8(vr[cb].z, vr[cb].w), pb[1], acc[cb], 0, 0, 0);
    }
    if constexpr (kMore) {
      if (!next_int8) load_keys(next, next_int8, Second{});
      load_scales(next);
      load_values(next);
    }
    n = next;
    int8 = next_int8;
  };
  while (n + kDecWaves < tile_end) {
    asm volatile("" ::: "memory");   // keep the LDS operand reads inside the loop
    tile_step(std::integral_constant<bool, true>{});
  }
  if (n < tile_end) tile_step(std::integral_constant<bool, false>{});
  // 4. Merge of the waves (log-sum-exp rule through LDS), then (max, normalizer,
  //    unnormalized output) of the chunk per head.
  z_w += __shfl_xor(z_w, 16, kWave);
  z_w += __shfl_xor(z_w, 32, kWave);
  if (lq == 0) red_m[wave][l16] = m_w;
  __syncthreads();
  float mc = red_m[0][l16];
#pragma unroll
  for (int w = 1; w < kDecWaves; ++w) mc = fmaxf(mc, red_m[w][l16]);
  const float fw = m_w == ninf ? 0.0f : __builtin_amdgcn_exp2f(m_w - mc);
  if (lq == 0) red_z[wave][l16] = z_w * fw;
  if (head_ok) {
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb)
      *reinterpret_cast<f32x4*>(&osum[wave][l16][16 * cb + 4 * lq]) = acc[cb] * fw;
  }
  __syncthreads();
  for (int o = tid; o < G * D; o += kDecThreads) {
    const int g = o / D, c = o % D;
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) sum += osum[w][g][c];
    a.part_o[(part_row + (size_t)(hk * G + g) * a.chunks) * D + c] = sum;
  }
  if (tid < G) {
    float zz = 0.0f, mm = red_m[0][tid];
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      zz += red_z[w][tid];
      mm = fmaxf(mm, red_m[w][tid]);
    }
    const size_t o = part_row + (size_t)(hk * G + tid) * a.chunks;
    a.part_m[o] = mm;
    a.part_z[o] = zz;
  }
}

// One workgroup per (sequence, query head).  Thread (part, c4) owns channels 4*c4 .. 4*c4+3
// and the chunks part, part + kRows, ...; it keeps a running (max, normalizer, output) merged
// with the log-sum-exp rule, loading kUnroll chunks ahead.  The parts are merged in LDS.
template <int D>
__global__ __launch_bounds__(kCombineThreads) void decode_combine_kernel(DecodeArgs a) {
  constexpr int kLanes = D / 4;                     // float4 lanes per chunk row
  constexpr int kRows = kCombineThreads / kLanes;   // chunk rows per pass
  constexpr int kUnroll = 8;
  const int bh = blockIdx.x;   // b * Hq + hq
  const int tid = threadIdx.x, c4 = tid % kLanes, part = tid / kLanes;
  // The chunks that hold keys of this sequence, and the first one's partial results.
  int chunks = a.chunks;
  size_t row = (size_t)bh * a.chunks;
  if (a.balanced) {
    const int b = bh / a.Hq;
    const RaggedSequence r(a, b, tid & (kWave - 1));
    chunks = r.count;
    row = (size_t)(bh - b * a.Hq) * a.chunks + r.first;
  } else if (a.seqlens) {
    const int len = ragged_keys(a, bh / a.Hq);
    chunks = min(chunks, ((len + kBlockN - 1) / kBlockN + a.chunk_tiles - 1) / a.chunk_tiles);
  }
  __shared__ float sm[kRows], sz[kRows];
  __shared__ f32x4 so[kRows][kLanes];
  const float* pm = a.part_m + row;
  const float* pz = a.part_z + row;
  const f32x4* po = reinterpret_cast<const f32x4*>(a.part_o + row * D) + c4;
  const float ninf = -__builtin_huge_valf();
  float m = ninf, z = 0.0f;
  f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int i0 = part; i0 < chunks; i0 += kRows * kUnroll) {
    float mi[kUnroll], zi[kUnroll];
    f32x4 oi[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int i = i0 + u * kRows;
      const bool ok = i < chunks;
      mi[u] = ok ? pm[i] : ninf;
      zi[u] = ok ? pz[i] : 0.0f;
      oi[u] = ok ? po[(size_t)i * kLanes] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    float mn = m;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) mn = fmaxf(mn, mi[u]);
    if (mn == ninf) continue;
    const float f = m == ninf ? 0.0f : __builtin_amdgcn_exp2f(m - mn);
    z *= f;
    o *= f;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const float fu = mi[u] == ninf ? 0.0f : __builtin_amdgcn_exp2f(mi[u] - mn);
      z += zi[u] * fu;
      o += oi[u] * fu;
    }
    m = mn;
  }
  if (c4 == 0) {
    sm[part] = m;
    sz[part] = z;
  }
  so[part][c4] = o;
  __syncthreads();
  if (tid < kLanes) {
    float mm = sm[0];
#pragma unroll
    for (int p = 1; p < kRows; ++p) mm = fmaxf(mm, sm[p]);
    float zz = 0.0f;
    f32x4 oo = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int p = 0; p < kRows; ++p) {
      const float fp = sm[p] == ninf ? 0.0f : __builtin_amdgcn_exp2f(sm[p] - mm);
      zz += sz[p] * fp;
      oo += so[p][tid] * fp;
    }
    const float inv = zz > 0.0f ? 1.0f / zz : 0.0f;
    half4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = (_Float16)(oo[r] * inv);
    *reinterpret_cast<half4*>(a.O + (size_t)bh * D + 4 * tid) = h;
  }
}

template <int D>
hipError_t launch_decode_t(const DecodeArgs& a, hipStream_t stream) {
  if (a.Hq / a.Hk > kDecHeads) return hipErrorInvalidValue;
  if (a.cut) hipLaunchKernelGGL(ragged_cut_kernel, dim3(1), dim3(kCutThreads), 0, stream, a);
  const dim3 grid = a.balanced ? dim3((a.chunks + kSlotsPad - 1) / kSlotsPad * kSlotsPad * a.Hk) : dim3(a.chunks, a.Hk, a.B);
  if (a.waves == kDecWavesEven)
    hipLaunchKernelGGL((decode_partial_kernel<D, kDecWavesEven>), grid, dim3(kDecWavesEven * kWave), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_partial_kernel<D, kDecWavesRagged>), grid, dim3(kDecWavesRagged * kWave), 0,
                       stream, a);
  hipLaunchKernelGGL(decode_combine_kernel<D>, dim3(a.B * a.Hq), dim3(kCombineThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(DecodeArgs a, int d, hipStream_t stream) {
  a.div_g = FastDiv(a.g);
  if (d == 128) return launch_decode_t<128>(a, stream);
  if (d == 64) return launch_decode_t<64>(a, stream);
  return hipErrorInvalidValue;
}

DecodePlan plan_decode(const tilemix_params& p, DecodeCut cut) {
  const long long nKB = (p.len_k + kBlockN - 1) / kBlockN;
  DecodePlan pl{};
  if (cut == DecodeCut::kByLength) {   // one round of workgroups and a rest per sequence
    pl.waves = p.batch > 1 ? kDecWavesRagged : kDecWavesEven;
    const long long round = (p.batch > 1 ? kDecRaggedWaves : kDecResident) / pl.waves;
    const long long most = (long long)p.batch * ((nKB + pl.waves - 1) / pl.waves);
    pl.chunks = (int)std::min<long long>((round + p.heads_kv - 1) / p.heads_kv + p.batch, most);
    pl.rows = (size_t)p.heads_q * pl.chunks;
    if (p.batch > kCutInWave) pl.cut_bytes = (cut_slots_at(p.batch) + 2 * (size_t)pl.chunks) * sizeof(int);
    return pl;
  }
  // The grid holds about one round of workgroups, however long the cache.
  const long long tiles = (long long)p.batch * p.heads_kv * nKB;
  pl.waves = kDecWavesEven;
  pl.chunk_tiles = (int)(pl.waves * std::max<long long>(1, (tiles + kDecResident - 1) / kDecResident));
  pl.chunks = (int)((nKB + pl.chunk_tiles - 1) / pl.chunk_tiles);
  pl.rows = (size_t)p.batch * p.heads_q * pl.chunks;
  return pl;
}

}  // namespace tilemix
