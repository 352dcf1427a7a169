// prepare.hip -- operand preparation for the routed attention and decode kernels
// (bandwidth-bound).
//
// quantize_rows_kernel, kv_operands_kernel (key part): the quantize-once pass of Appendix C
//   ("Blockwise INT8 Quantization", "Quantization Granularity", "Quantize-Once Execution"):
//   for every (sequence, head, block of 128 query / 64 key tokens) the FP32 absmax, the
//   FP32 scale absmax/127, the codes round-half-even(x / scale) clamped to [-127, 127]
//   and the FP16 scale.  One workgroup per block; the block is read once into
//   registers, reduced, then converted and written.
//
// kv_operands_kernel (value part): V per 64-key tile with the channels as rows, so that a P.V
//   matrix-core step reads its A operand (V^T) as contiguous 16-byte runs:
//   - prefill: FP16 [d][64].  Within each run of 16 keys the order is (0-3, 8-11 | 4-7, 12-15):
//     this is the key order in which the score accumulator hands P to the P.V step (accumulator
//     rows 8*(r/4) + 4*(lane/32) + r%4), so P never leaves registers;
//   - decode cache: the INT8 codes of the tile (64-key blocks, as for K) as [d][64] in key order.
//   Keys past L are zero.
#include "tilemix_device.h"
#include "tilemix_internal.h"

namespace tilemix {

namespace {

// Threads that take one 64-row block: every thread holds four 16-byte chunks (8 channels of 4 rows),
// whatever d.
template <int D>
constexpr int kTileThreads = 2 * D;
constexpr int kRowsThreads = 256;

// Maximum of v over the kThreads threads that share red; tid counts them.
template <int kThreads>
__device__ __forceinline__ float block_max(float v, int tid, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
  const int wave = tid / kWave;
  if ((tid & (kWave - 1)) == 0) red[wave] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < kThreads / kWave; ++w) r = fmaxf(r, red[w]);
  return r;
}

// Running packed maximum and minimum of FP16 values (a NaN is passed over, as by fmaxf); the
// absmax is the larger of the maximum and the negated minimum.
struct AbsMax {
  half2v hi = {(_Float16)0.0f, (_Float16)0.0f}, lo = {(_Float16)0.0f, (_Float16)0.0f};
  __device__ __forceinline__ void add(uint4 v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const half2v x = __builtin_bit_cast(half2v, w[i]);
      hi = __builtin_elementwise_max(hi, x);
      lo = __builtin_elementwise_min(lo, x);
    }
  }
  __device__ __forceinline__ float get() const {
    return fmaxf(fmaxf((float)hi[0], (float)hi[1]), -fminf((float)lo[0], (float)lo[1]));
  }
};

// Codes of BLK rows starting at row0 of a [.., H, D] tensor, read and written row by row by kThreads
// threads.
template <int D, int BLK, int kThreads>
__device__ __forceinline__ void quantize_rows(const _Float16* __restrict__ X, int8_t* __restrict__ X8,
                                              uint16_t* __restrict__ scale, size_t row0, int rows, int H,
                                              int h, int tid, float* red) {
  constexpr int kChunksPerRow = D / 8;                          // 16-byte chunks of 8 halfs
  constexpr int kPer = BLK * kChunksPerRow / kThreads;          // chunks per thread
  static_assert(kPer * kThreads == BLK * kChunksPerRow, "block split");
  uint4 v[kPer];
  AbsMax am;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int c = tid + kThreads * i;
    const int row = c / kChunksPerRow, ch = c % kChunksPerRow;
    v[i] = row < rows ? ld_global_16(X + ((row0 + row) * H + h) * D + ch * 8) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) am.add(v[i]);
  const BlockScale sc(block_max<kThreads>(am.get(), tid, red));
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int c = tid + kThreads * i;
    const int row = c / kChunksPerRow, ch = c % kChunksPerRow;
    if (row >= rows) continue;
    uint32_t w[8];
    sc.words(v[i], w);
    *reinterpret_cast<uint2*>(X8 + ((row0 + row) * H + h) * D + ch * 8) =
        make_uint2(pack4(w[0], w[1], w[2], w[3]), pack4(w[4], w[5], w[6], w[7]));
  }
  if (tid == 0) *scale = sc.bits;
}

// Query blocks of the stand-alone quantization pass.
template <int D>
__global__ __launch_bounds__(kRowsThreads) void quantize_rows_kernel(
    const _Float16* __restrict__ X, int8_t* __restrict__ X8, uint16_t* __restrict__ dX, int L, int H,
    int nblk) {
  __shared__ float red[kRowsThreads / kWave];
  const int r = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int row0 = r * kQuantBlockQ;
  quantize_rows<D, kQuantBlockQ, kRowsThreads>(X, X8, dX + ((size_t)b * nblk + r) * H + h,
                                               (size_t)b * L + row0, min(kQuantBlockQ, L - row0), H, h, threadIdx.x, red);
}

// One workgroup per 64-key block, operand and group of kHeads adjacent heads.  KEYS: the block's K codes
// and scale.  VALUES: its transposed V tile in FP16 (kValuesFp16, prefill) or as INT8 codes and scale
// (kValuesInt8, the decode cache).  With both operands, workgroup 2 i takes the keys and 2 i + 1
// the values of head group i, so that one launch streams K and V; heads vary fastest, which keeps the
// concurrently read rows of [.., H, D] contiguous.
// Two heads: at d = 64 their K8 rows are one 128-byte line, which two workgroups on different XCDs would
// each write in part.  8 x 8192 tokens, 28 heads, both operands for prefill: 182 us with one head (K
// and V in launches of their own took 160), 154 with two; 4 x 65536, 8 heads 209 (197), 174.
//
// Tile n of KV head h of sequence b lands at tile index (b H + h) nblk + n for one common length,
// or h * (all key tiles of the batch) + (first key tile of b) + n for a variable-length batch.
//
// Transposing: thread (quad kq, chunk ch) holds channels 8 ch .. 8 ch + 7 of keys 4 kq .. 4 kq + 3
// and writes each channel's four keys as one 8-byte (FP16) or 4-byte (INT8) unit into LDS.
// Channel 8 ch + e sits in LDS row (D / 8) e + ch, with its 16-byte granules XOR-swizzled by ch,
// so that the lanes of one write spread over the banks instead of meeting in one row's.
//
// Bound: HBM (2 + 1 bytes per key element, 2 + 2 or 2 + 1 per value element).  Two kernels with
// an IEEE division per code and byte-wise transposing writes were bound by the vector units
// instead: the cache of 2 x 16384 tokens, 8 heads of d = 128 (201 MB) took 27.5 us for K and
// 39.4 us for V; this one takes 38.2 us per call, 5.26 TB/s, where a plain copy reaches 5.1.
// For prefill, one launch saves 4 us at 2 x 9777 tokens and 4 heads.
constexpr int kValuesNone = 0, kValuesFp16 = 1, kValuesInt8 = 2;

template <int D, bool KEYS, int VALUES, int kHeads>
__global__ __launch_bounds__(kTileThreads<D> * kHeads) void kv_operands_kernel(KvOperandArgs a) {
  constexpr int kThreads = kTileThreads<D>;
  constexpr int kParts = (KEYS ? 1 : 0) + (VALUES != kValuesNone ? 1 : 0);
  constexpr int kCh = D / 8;                                     // 16-byte chunks per row
  constexpr int kUnit = VALUES == kValuesInt8 ? 4 : 8;           // bytes of four keys of a channel
  constexpr int kRow = 16 * kUnit;                               // bytes of a channel row (64 keys)
  constexpr int kGr = kRow / 16;                                 // 16-byte granules of it
  __shared__ float reds[kHeads][kThreads / kWave];
  __shared__ __align__(16) char tiles[kHeads][VALUES != kValuesNone ? D * kRow : 16];

  const int sub = threadIdx.x / kThreads, tid = threadIdx.x % kThreads;
  const int h = blockIdx.x / kParts * kHeads + sub, n = blockIdx.y, b = blockIdx.z;
  float* red = reds[sub];
  char* tile = tiles[sub];
  const bool keys = KEYS && (kParts == 1 || blockIdx.x % kParts == 0);
  long long start = (long long)b * a.L, blk0 = (long long)b * a.nblk;
  long long tile_id = ((long long)b * a.H + h) * a.nblk + n;
  int len = a.L;
  if (a.seqs) {
    const int* e = a.seqs + kSeqFields * b;
    start = e[kSeqKStart];
    len = e[kSeqKLen];
    blk0 = e[kSeqKBlk];
    tile_id = (long long)h * a.seqs[kSeqFields * a.batch + kSeqKTile] + e[kSeqKTile] + n;
  }
  const int key0 = n * kBlockN;
  if (key0 >= len) return;   // past the end of a shorter sequence
  const int rows = min(kBlockN, len - key0);
  const size_t scale_id = (size_t)(blk0 + n) * a.H + h;
  if constexpr (KEYS) {
    if (keys) {
      quantize_rows<D, kBlockN, kThreads>(a.K, a.K8, a.dK + scale_id, (size_t)(start + key0), rows, a.H, h, tid, red);
      return;
    }
  }
  if constexpr (VALUES != kValuesNone) {
    const int kq = tid / kCh, ch = tid % kCh;
    uint4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * kq + i;
      v[i] = row < rows ? ld_global_16(a.V + ((size_t)(start + key0 + row) * a.H + h) * D + ch * 8)
                        : make_uint4(0, 0, 0, 0);
    }
    // LDS address of granule g of channel 8 c8 + e.
    auto at = [](int c8, int e, int g) {
      const int swz = VALUES == kValuesInt8 ? (c8 >> 2) & 3 : (c8 >> 1) & 7;
      return (e * kCh + c8) * kRow + 16 * (g ^ swz);
    };
    if constexpr (VALUES == kValuesInt8) {
      AbsMax am;
#pragma unroll
      for (int i = 0; i < 4; ++i) am.add(v[i]);
      const BlockScale sc(block_max<kThreads>(am.get(), tid, red));
      uint32_t w[4][8];
#pragma unroll
      for (int i = 0; i < 4; ++i) sc.words(v[i], w[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        *reinterpret_cast<uint32_t*>(tile + at(ch, e, kq >> 2) + 4 * (kq & 3)) =
            pack4(w[0][e], w[1][e], w[2][e], w[3][e]);
      if (tid == 0) a.dV[scale_id] = sc.bits;
    } else {
      // Key quad j of a 16-key run goes to place 0, 2, 1, 3 of it.
      const int place = 2 * (kq & 1) + ((kq >> 1) & 1);
      const int g = 2 * (kq >> 2) + (place >> 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint32_t x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = e < 2 ? v[i].x : e < 4 ? v[i].y : e < 6 ? v[i].z : v[i].w;
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;   // the odd / even half of both
        *reinterpret_cast<uint2*>(tile + at(ch, e, g) + 8 * (place & 1)) =
            make_uint2(__builtin_amdgcn_perm(x[1], x[0], sel), __builtin_amdgcn_perm(x[3], x[2], sel));
      }
    }
    __syncthreads();
    char* out = static_cast<char*>(a.Vout) + (size_t)tile_id * (size_t)(D * kRow);
#pragma unroll
    for (int i = 0; i < D * kGr / kThreads; ++i) {
      const int k = tid + kThreads * i, c = k / kGr, g = k % kGr;
      *reinterpret_cast<uint4*>(out + (size_t)k * 16) =
          *reinterpret_cast<const uint4*>(tile + at(c / 8, c % 8, g));
    }
  }
}

}  // namespace

namespace {

// Sequence table of a variable-length batch, built on the device from cu_seqlens so that the
// host never reads them: for each sequence its rows in the packed Q and K (clamped to the
// tensors, the maximum lengths and after the previous sequence, so that a malformed table
// stays in bounds) and the running totals of scale blocks, query-tile rows and key tiles;
// row B holds the totals.  Once a sequence's query-tile rows would run past the route_rows
// routing rows the caller passed, it and every later sequence are treated as empty (no query
// rows).  One thread walks the batch, out of LDS: the other threads fetch the prefix sums
// kSeqChunk at a time, so that the walk waits for one memory latency per chunk and not per
// sequence.
constexpr int kSeqThreads = 256, kSeqChunk = 1024;
__global__ __launch_bounds__(kSeqThreads) void seq_table_kernel(
    const int* __restrict__ cu_q, const int* __restrict__ cu_k, int batch, int total_q, int total_k,
    int max_q, int max_k, int block_m, int route_rows, int* __restrict__ seqs) {
  __shared__ int cq[kSeqChunk + 1], ck[kSeqChunk + 1];
  int q_end = 0, k_end = 0, qblk = 0, kblk = 0, qtile = 0, ktile = 0;
  bool fits = true;
  for (int b0 = 0; b0 < batch; b0 += kSeqChunk) {
    const int count = min(kSeqChunk, batch - b0);
    __syncthreads();
    for (int i = threadIdx.x; i <= count; i += kSeqThreads) {
      cq[i] = cu_q[b0 + i];
      ck[i] = cu_k[b0 + i];
    }
    __syncthreads();
    if (threadIdx.x != 0) continue;
    for (int i = 0; i < count; ++i) {
      const int qs = min(max(cq[i], q_end), total_q);
      const int qe = min(max(cq[i + 1], qs), total_q);
      const int ks = min(max(ck[i], k_end), total_k);
      const int ke = min(max(ck[i + 1], ks), total_k);
      int ql = min(qe - qs, max_q);
      const int kl = min(ke - ks, max_k);
      fits = fits && qtile + (ql + block_m - 1) / block_m <= route_rows;
      if (!fits) ql = 0;
      int* e = seqs + kSeqFields * (b0 + i);
      e[kSeqQStart] = qs; e[kSeqQLen] = ql; e[kSeqKStart] = ks; e[kSeqKLen] = kl;
      e[kSeqQBlk] = qblk; e[kSeqKBlk] = kblk; e[kSeqQTile] = qtile; e[kSeqKTile] = ktile;
      qblk += (ql + kQuantBlockQ - 1) / kQuantBlockQ;
      kblk += (kl + kQuantBlockK - 1) / kQuantBlockK;
      qtile += (ql + block_m - 1) / block_m;
      ktile += (kl + kBlockN - 1) / kBlockN;
      q_end = qs + ql;
      k_end = ks + kl;
    }
  }
  if (threadIdx.x != 0) return;
  int* e = seqs + kSeqFields * batch;
  e[kSeqQStart] = q_end; e[kSeqQLen] = 0; e[kSeqKStart] = k_end; e[kSeqKLen] = 0;
  e[kSeqQBlk] = qblk; e[kSeqKBlk] = kblk; e[kSeqQTile] = qtile; e[kSeqKTile] = ktile;
}

}  // namespace

hipError_t launch_seq_table(const int* cu_q, const int* cu_k, int batch, int total_q, int total_k,
                            int max_q, int max_k, int block_m, int route_rows, int* seqs,
                            hipStream_t stream) {
  hipLaunchKernelGGL(seq_table_kernel, dim3(1), dim3(kSeqThreads), 0, stream, cu_q, cu_k, batch, total_q,
                     total_k, max_q, max_k, block_m, route_rows, seqs);
  return hipGetLastError();
}

hipError_t launch_quantize_q(const _Float16* Q, int8_t* Q8, uint16_t* dQ, int B, int L, int H, int d,
                             hipStream_t stream) {
  const int nblk = (L + kQuantBlockQ - 1) / kQuantBlockQ;
  const dim3 grid(nblk, H, B), block(kRowsThreads);
  if (d == 128)
    hipLaunchKernelGGL(quantize_rows_kernel<128>, grid, block, 0, stream, Q, Q8, dQ, L, H, nblk);
  else if (d == 64)
    hipLaunchKernelGGL(quantize_rows_kernel<64>, grid, block, 0, stream, Q, Q8, dQ, L, H, nblk);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {

template <int D, bool KEYS, int VALUES, int HEADS = 1>
hipError_t launch_kv_t(const KvOperandArgs& a, hipStream_t stream) {
  constexpr int kParts = (KEYS ? 1 : 0) + (VALUES != kValuesNone ? 1 : 0);
  hipLaunchKernelGGL((kv_operands_kernel<D, KEYS, VALUES, HEADS>), dim3(a.H / HEADS * kParts, a.nblk, a.batch),
                     dim3(kTileThreads<D> * HEADS), 0, stream, a);
  return hipGetLastError();
}

template <int D>
hipError_t launch_kv_d(const KvOperandArgs& a, hipStream_t stream) {
  if (a.V && a.dV) return a.K ? launch_kv_t<D, true, kValuesInt8>(a, stream) : hipErrorInvalidValue;
  if (a.V && a.K) {
    // Two heads where the write traffic fills the memory; below that one is ahead (1000 tokens, 8 heads: 3.0
    // against 3.1 us; 4096 tokens, 8 heads, 512 blocks: 3.8 either way).
    if constexpr (D == 64) {
      if (a.H % 2 == 0 && (long long)a.H * a.nblk * a.batch >= 512) return launch_kv_t<D, true, kValuesFp16, 2>(a, stream);
    }
    return launch_kv_t<D, true, kValuesFp16>(a, stream);
  }
  if (a.V) return launch_kv_t<D, false, kValuesFp16>(a, stream);
  return a.K ? launch_kv_t<D, true, kValuesNone>(a, stream) : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_kv_operands(KvOperandArgs a, int d, hipStream_t stream) {
  a.nblk = (a.L + kBlockN - 1) / kBlockN;
  if (d == 128) return launch_kv_d<128>(a, stream);
  if (d == 64) return launch_kv_d<64>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace tilemix
