// HIP kernels of the two rollback strategies of arXiv 2510.22876, Section 2
// ("Family A: contiguous layout", "Family B: variable-length layout"), on
// MI355X (gfx950, wave64).
//
//   rollback_kernel     Family A: one workgroup truncates every row to the
//                       batch-minimum accepted count m and applies Eq. (1) /
//                       Eq. (2) with a_i = m + 1 (all offsets equal: the cache
//                       realignment that follows moves nothing in place).
//   varlen_offsets      Family B: one workgroup computes each sequence's kept
//                       length (its rows minus its rejected window entries)
//                       and their running sum, the new cumulative offsets.
//   varlen_compact      Family B: the flat [T][H][D] cache of every (layer,
//                       K/V) is compacted into a second buffer, in the
//                       split-piece layout of the other out-of-place copies
//                       laid over the whole output; extra workgroups write the
//                       position ids (I2: each row's index in its sequence).
#include "posmask.h"
#include "span_copy.h"
#include "specdec_internal.h"

namespace specdec {
namespace {

constexpr uint32_t kBadPadIn = 0x1u, kBadAccept = 0x2u, kBadWidth = 0x4u;
constexpr int kOneBlock = 1024;

__device__ __forceinline__ int32_t block_min_i32(int32_t v, int32_t* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int32_t o = __shfl_xor(v, off);
    v = o < v ? o : v;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  int32_t m = red[0];
#pragma unroll
  for (int q = 1; q < kOneBlock / 64; ++q) m = red[q] < m ? red[q] : m;
  return m;
}

__device__ __forceinline__ int32_t block_max_i32(int32_t v, int32_t* red) {
  return -block_min_i32(-v, red);
}

struct RollbackArgs {
  const int32_t* tokens;
  const int32_t* n_acc_in;
  const int32_t* pad_in;
  int32_t B, k, W_in;
  int32_t* n_acc_out;   // may equal n_acc_in
  int32_t* bonus_out;
  int32_t* pad_out;     // may equal pad_in
  int32_t* w_new;
  uint32_t* dev_status;
};

__global__ __launch_bounds__(kOneBlock) void rollback_kernel(RollbackArgs a) {
  __shared__ int32_t red[kOneBlock / 64];
  const int32_t L = a.W_in - (a.k + 1);
  // every input is read before any output is written (outputs may alias them)
  int32_t m = a.k;
  for (int i = threadIdx.x; i < a.B; i += kOneBlock) {
    const int32_t p = a.pad_in[i], n = a.n_acc_in[i];
    uint32_t err = 0u;
    if (p < 0 || p > L) err |= kBadPadIn;
    if (n < 0 || n > a.k) err |= kBadAccept;
    if (err) {
      if (a.dev_status) atomicOr(a.dev_status, err);
    } else {
      m = n < m ? n : m;
    }
  }
  m = block_min_i32(m, red);
  int32_t w = 0;
  for (int i = threadIdx.x; i < a.B; i += kOneBlock) {
    const int32_t p = a.pad_in[i], n = a.n_acc_in[i];
    if (p >= 0 && p <= L && n >= 0 && n <= a.k) {
      const int32_t len = (L - p) + m + 1;               // Eq. (1) with a_i = m + 1
      w = len > w ? len : w;
    }
  }
  w = block_max_i32(w, red);
  // each thread writes only the rows it reads here, after the block-wide
  // reductions: outputs may alias the inputs
  for (int i = threadIdx.x; i < a.B; i += kOneBlock) {
    const int32_t p = a.pad_in[i], n = a.n_acc_in[i];
    const bool ok = p >= 0 && p <= L && n >= 0 && n <= a.k;
    a.bonus_out[i] = ok ? a.tokens[static_cast<int64_t>(i) * (a.k + 1) + m] : -1;
    // Eq. (2): delta = (w - L) - (m + 1), the same for every row
    a.pad_out[i] = ok ? p + ((w - L) - (m + 1)) : -1;
    a.n_acc_out[i] = ok ? m : n;
  }
  if (threadIdx.x == 0) a.w_new[0] = w;
}

// ---- Family B ------------------------------------------------------------------

constexpr int kTpb = 64;
constexpr int kPieces = 2;
constexpr int kSplit = 512;
constexpr int kNt = 3;

struct VarlenArgs {
  const u32x4* src;
  u32x4* dst;
  int64_t src_slab_vecs, dst_slab_vecs;  // T_cap * H * D / 8 per (layer, K/V)
  int64_t row_vecs;                      // H * D / 8: one token row of the flat buffer
  int32_t row_shift;                     // its logarithm when it is a power of two, else -1
  int64_t src_T, dst_T;
  const int32_t* cu_in;
  const int32_t* n_acc;
  int32_t* cu_out;
  int64_t* pos;
  int32_t B, k, max_len;
  uint32_t* dev_status;
  int64_t rows_cap;       // rows that the kept sequences can have in all (below 2^31)
  uint32_t chunks;        // workgroups per (layer, K/V) slab
  uint32_t block_base;    // compaction workgroups of earlier launches
  uint32_t pos_blocks;    // position-id workgroups (first launch only)
};

// Kept lengths and their running sum (one workgroup, B in stripes of 1024).
// Sequences of a nondecreasing cu_in are disjoint, so their rows fit rows_cap.
// Offsets that fall make sequences overlap; the sum (saturating, it can pass
// 2^32) then stops at rows_cap, so that the offsets never fall and every output row
// below cu_out[B] lies in the sequence that a search in them finds.
__global__ __launch_bounds__(kOneBlock) void varlen_offsets_kernel(VarlenArgs a) {
  __shared__ uint32_t wsum[kOneBlock / 64];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) {
    carry = 0;
    a.cu_out[0] = 0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i0 = 0; i0 < a.B; i0 += kOneBlock) {
    const int i = i0 + threadIdx.x;
    int32_t keep = 0;
    if (i < a.B) {
      const int64_t b = a.cu_in[i], e = a.cu_in[i + 1];
      const int32_t n = a.n_acc[i];
      uint32_t err = 0u;
      if (b < 0 || e < b || e > a.src_T || e - b < a.k + 1 || e - b > a.max_len) err |= kBadWidth;
      if (n < 0 || n > a.k) err |= kBadAccept;
      if (err) {
        if (a.dev_status) atomicOr(a.dev_status, err);
      } else {
        keep = static_cast<int32_t>(e - b) - (a.k - n);
      }
    }
    // inclusive scan of keep over the stripe
    uint32_t v = static_cast<uint32_t>(keep);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = __shfl_up(v, off);
      if (lane >= off) v = __builtin_elementwise_add_sat(v, o);
    }
    if (lane == 63) wsum[wave] = v;
    __syncthreads();
    uint32_t end = carry;
#pragma unroll
    for (int q = 0; q < kOneBlock / 64; ++q) end = __builtin_elementwise_add_sat(end, q < wave ? wsum[q] : 0u);
    end = __builtin_elementwise_add_sat(end, v);
    if (i < a.B) {
      const uint32_t most = static_cast<uint32_t>(a.rows_cap);
      a.cu_out[i + 1] = static_cast<int32_t>(end < most ? end : most);
      if (keep > 0 && end > most && a.dev_status) atomicOr(a.dev_status, kBadWidth);
    }
    __syncthreads();
    if (threadIdx.x == kOneBlock - 1) carry = end;
    __syncthreads();
  }
}

// The sequence whose kept rows hold output row r < cu_out[B]: the first one in
// [lo, B) that ends beyond r.  `Load` reads cu_out (scalar loads for a
// wave-uniform r).  A workgroup moves 2 KB, about 700 cycles of its SIMD's
// time at full bandwidth, so the steps are few and 32-bit: comparing in vectors
// (64-bit products) took 1062 us instead of 1045 over 6.95 GB, and a search that
// probes seven offsets a round, for fewer dependent loads, 948 instead of 905
// over 6.0 GB.
template <typename Load>
__device__ __forceinline__ int sequence_of(int32_t r, int lo, int B, Load cu_out) {
  int hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cu_out(mid + 1) > r) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// The output of a (layer, K/V) slab is one run of cu_out[B] rows, so it is
// tiled as such, whatever the lengths: workgroups are laid over the rows that
// the slab can hold (at most T, and at most B * max_len), in the split-piece
// layout tiled from the slab's 16 KB boundary, and each finds its sequence by
// a search in the offsets (scalar loads).  Tiling each sequence to the
// longest one's length instead left 70% of the workgroups of a ragged batch
// (32 sequences, lengths log-uniform in 64..4096) without work, and the
// dispatch of empty workgroups bounded the kernel: 1510 us a call, against
// 1045 with this tiling (6.95 GB; 8 sequences of U[128, 1024], 6.0 GB: 917 and
// 905).  The search costs a few dependent loads, and a piece in which a
// sequence begins more of them, unless it is the next one, which is tried
// first: 64 sequences of 64-byte rows (125 MB in all) take 24.3 us instead of 24.0
// with each sequence tiled for itself (26.1 with a search for every lane
// beyond the first sequence), 256 sequences of 10..100 256-byte rows (518 MB)
// 82 instead of 90 (86).
__global__ __launch_bounds__(kTpb) void varlen_compact_kernel(VarlenArgs a) {
  const uint32_t b = blockIdx.x;
  auto cu_scalar = [&](int i) { return load_invariant(a.cu_out + i); };
  auto cu_lane = [&](int i) { return a.cu_out[i]; };
  auto row_of = [&](int64_t u) {
    return static_cast<int32_t>(a.row_shift >= 0 ? u >> a.row_shift : u / a.row_vecs);
  };
  const int64_t rows = cu_scalar(a.B);   // in all, at most rows_cap
  if (b < a.pos_blocks) {
    // position ids of the kept rows: 4*kTpb rows per workgroup
    const int64_t r0 = static_cast<int64_t>(b) * (4 * kTpb);
    if (r0 >= rows) return;
    const int first = sequence_of(static_cast<int32_t>(r0), 0, a.B, cu_scalar);
    const int64_t start = cu_scalar(first), end = cu_scalar(first + 1);
    const int64_t next_end = cu_scalar(first + 2 < a.B ? first + 2 : a.B);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t r = r0 + q * kTpb + threadIdx.x;
      if (r >= rows) break;
      int64_t of = r < end ? start : end;   // the first row of r's sequence
      if (r >= next_end) of = cu_lane(sequence_of(static_cast<int32_t>(r), first, a.B, cu_lane));
      a.pos[r] = r - of;
    }
    return;
  }
  const uint32_t g = a.block_base + (b - a.pos_blocks);
  const uint32_t lk = g / a.chunks;
  const uint32_t sub = g - lk * a.chunks;
  const int64_t total = rows * a.row_vecs;
  u32x4* d = a.dst + static_cast<int64_t>(lk) * a.dst_slab_vecs;
  const u32x4* s = a.src + static_cast<int64_t>(lk) * a.src_slab_vecs;
  const int64_t base = split_base<kPieces, kTpb, kSplit>(sub) - split_misalign<kPieces, kSplit>(d);
  if (base >= total) return;
  const int t = threadIdx.x;
  u32x4 v[kPieces] = {};
  int seq = 0;
  int64_t end = 0, move = 0;   // the sequence's end in the output, and how far its rows come from (vectors)
#pragma unroll
  for (int j = 0; j < kPieces; ++j) {
    const int64_t p0 = base + static_cast<int64_t>(j) * kSplit;   // the piece's first vector (wave-uniform)
    const int64_t first = p0 > 0 ? p0 : 0;
    if (first >= total) break;
    if (first >= end) {
      seq = sequence_of(row_of(first), seq, a.B, cu_scalar);
      end = static_cast<int64_t>(cu_scalar(seq + 1)) * a.row_vecs;
      move = (static_cast<int64_t>(load_invariant(a.cu_in + seq)) - cu_scalar(seq)) * a.row_vecs;
    }
    const int64_t last = end < total ? end : total;
    int64_t si = p0 + t;
    int64_t next_end = 0, next_move = 0;
    if (last < total && p0 + kTpb > last) {   // the next sequence's rows begin inside the piece
      next_end = static_cast<int64_t>(cu_scalar(seq + 2)) * a.row_vecs;
      next_move = (static_cast<int64_t>(load_invariant(a.cu_in + seq + 1)) - cu_scalar(seq + 1)) * a.row_vecs;
    }
    if (si >= last && si < next_end) {
      si += next_move;
    } else if (si >= last && si < total) {    // and those of later ones
      const int q = sequence_of(row_of(si), seq, a.B, cu_lane);
      si += (static_cast<int64_t>(a.cu_in[q]) - cu_lane(q)) * a.row_vecs;
    } else {                          // lanes outside the slab read a vector that is there, and store nothing
      si = (si < first ? first : (si >= last ? last - 1 : si)) + move;
    }
    v[j] = ld16<(kNt & 1) != 0>(s + si);
  }
#pragma unroll
  for (int j = 0; j < kPieces; ++j) asm volatile("" ::"v"(v[j].x), "v"(v[j].y), "v"(v[j].z), "v"(v[j].w));
#pragma unroll
  for (int j = 0; j < kPieces; ++j) {
    const int64_t p0 = base + static_cast<int64_t>(j) * kSplit;
    const int64_t u = p0 + t;
    if (u >= 0 && u < total) st16_at<(kNt & 2) != 0>(d + p0, t, v[j]);
  }
}

}  // namespace

hipError_t launch_rollback(const RollbackLaunch& p, hipStream_t stream) {
  RollbackArgs a{p.tokens, p.n_acc_in, p.pad_in, p.B, p.k, p.W_in, p.n_acc_out, p.bonus_out, p.pad_out, p.w_new,
                 p.dev_status};
  hipLaunchKernelGGL(rollback_kernel, dim3(1), dim3(kOneBlock), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_varlen_rollback(const VarlenLaunch& p, hipStream_t stream) {
  VarlenArgs a{};
  a.src = static_cast<const u32x4*>(p.src);
  a.dst = static_cast<u32x4*>(p.dst);
  a.row_vecs = static_cast<int64_t>(p.H) * p.D / 8;
  a.row_shift = (a.row_vecs & (a.row_vecs - 1)) == 0 ? __builtin_ctzll(static_cast<uint64_t>(a.row_vecs)) : -1;
  a.src_slab_vecs = p.src_T * a.row_vecs;
  a.dst_slab_vecs = p.dst_T * a.row_vecs;
  a.src_T = p.src_T;
  a.dst_T = p.dst_T;
  a.cu_in = p.cu_in;
  a.n_acc = p.n_acc;
  a.cu_out = p.cu_out;
  a.pos = p.pos;
  a.B = p.B;
  a.k = p.k;
  a.max_len = p.max_len;
  a.dev_status = p.dev_status;
  a.rows_cap = static_cast<int64_t>(p.max_len) * p.B < p.src_T ? static_cast<int64_t>(p.max_len) * p.B : p.src_T;
  if (a.rows_cap > INT32_MAX) a.rows_cap = INT32_MAX;   // cu_in names no row beyond
  hipLaunchKernelGGL(varlen_offsets_kernel, dim3(1), dim3(kOneBlock), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t pos_blocks = p.pos ? (a.rows_cap + 4 * kTpb - 1) / (4 * kTpb) : 0;
  // a slab may start anywhere: room for the extra group of the aligned tiling
  const int64_t chunks = split_blocks<kPieces, kTpb, kSplit>(a.rows_cap * a.row_vecs, true);
  const int64_t blocks = static_cast<int64_t>(p.L) * 2 * chunks;
  const int64_t most = max_launch_items() / kTpb;
  if (most <= pos_blocks || blocks > 0xFFFFFFFFLL) return hipErrorInvalidConfiguration;
  a.chunks = static_cast<uint32_t>(chunks);
  a.pos_blocks = static_cast<uint32_t>(pos_blocks);
  for (int64_t g = 0; g < blocks || a.pos_blocks > 0;) {
    const int64_t room = most - a.pos_blocks;
    const int64_t n = blocks - g < room ? blocks - g : room;
    a.block_base = static_cast<uint32_t>(g);
    hipLaunchKernelGGL(varlen_compact_kernel, dim3(static_cast<uint32_t>(n + a.pos_blocks)), dim3(kTpb), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    g += n;
    a.pos_blocks = 0;
  }
  return hipSuccess;
}

}  // namespace specdec
