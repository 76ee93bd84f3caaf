// HIP kernels for one greedy verify + KV realign step (EqSpec, arXiv 2510.22876)
// on MI355X (gfx950, wave64).
//
//   verify_partial     vocab-wide argmax of every logit row (Algorithm 3), split
//                      over workgroups per row; each workgroup stores its
//                      packed (key, index) maximum in its own workspace slot.
//   verify_finalize    one workgroup: reduces the slots of each row, then the
//                      prefix-match scan, the bonus token and the new width /
//                      paddings (Eq. (1), Eq. (2)).  Two launches instead of a
//                      last-workgroup-done counter: a device-scope fence and
//                      atomic per workgroup costs more than a kernel boundary.
//   realign_oop        out-of-place unpad-append-repad of the bf16 KV cache:
//                      64-thread workgroups, two 1 KB pieces of a (layer,
//                      K/V, row, head) span each, 128-bit loads and stores.
//   realign_inplace    in-place variant for long spans: one workgroup walks a
//                      whole span in the direction of its shift, a barrier
//                      between the reads and the writes of each chunk.
//   realign_chunk,     in-place variant for short spans and for few long ones:
//   realign_strips     a workgroup per chunk of a span, all at once, then the
//                      few vectors that cross from a chunk to the next.
//   small_step         a small step's merge of the scan and its realignment, in
//                      one launch.
//   posmask blocks     position ids / mask of invariant I2, appended to either
//                      realign grid (or launched alone).
//
// Everything here is bandwidth-bound data movement plus integer compares: no
// matrix cores.
#include <cstdlib>

#include "posmask.h"
#include "span_copy.h"
#include "specdec_internal.h"

namespace specdec {
namespace {

constexpr uint32_t kBadPadIn = 0x1u, kBadAccept = 0x2u, kBadWidth = 0x4u, kBadPadOut = 0x8u;
constexpr int kWaves = kThreads / 64;
constexpr int kPmColsPerBlock = 4 * kThreads;

// ---------------------------------------------------------------------------
// argmax keys
//
// A logit is mapped to an unsigned key whose integer order is the order of
// the values: -0.0 and +0.0 share a key, every NaN gets the largest key (a NaN
// ranks above every number).  Within a thread elements are visited in
// increasing index order and only a strictly larger key replaces the best,
// so the lowest index wins among equal keys; across threads the pair is
// packed as (key << 32) | ~index, whose maximum again prefers the lowest
// index.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t key_f32(uint32_t u) {
  const uint32_t mag = u & 0x7FFFFFFFu;
  if (mag > 0x7F800000u) return 0xFFFFFFFFu;
  if (mag == 0u) return 0x80000000u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// 16-bit logits: a positive h maps to h | 0x8000, a negative one to
// (h ^ 0xFFFF) + 1 (so -0.0 lands on +0.0's key 0x8000), a NaN to 0xFFFF.
template <uint32_t kNanMag>  // 0x7F80 for bf16, 0x7C00 for f16
__device__ __forceinline__ uint32_t key_16(uint32_t h) {
  if ((h & 0x7FFFu) > kNanMag) return 0xFFFFu;
  return (h & 0x8000u) ? ((h ^ 0xFFFFu) + 1u) : (h | 0x8000u);
}

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// The keys of both halves of a word with packed 16-bit operations, exact
// except for NaNs (which land outside the keys of -inf..+inf).
__device__ __forceinline__ u16x2 keys2(uint32_t w) {
  const s16x2 sign = __builtin_bit_cast(s16x2, w) >> (s16x2){15, 15};   // 0xFFFF on negative halves
  const uint32_t m = __builtin_bit_cast(uint32_t, sign);
  return __builtin_bit_cast(u16x2, w ^ (m | 0x80008000u)) + __builtin_bit_cast(u16x2, m & 0x00010001u);
}

struct Best {
  uint32_t key = 0u;
  int32_t idx = 0;
  __device__ __forceinline__ void take(uint32_t k, int32_t i) {
    if (k > key) {
      key = k;
      idx = i;
    }
  }
};

template <int DT>
struct Logit;

template <>
struct Logit<0> {  // f32
  static constexpr int kBytes = 4;
  __device__ static uint32_t key_at(const char* row, int64_t i) {
    return key_f32(*reinterpret_cast<const uint32_t*>(row + 4 * i));
  }
  __device__ static void take_vec(Best& b, const uint4& q, int32_t e) {
    b.take(key_f32(q.x), e);
    b.take(key_f32(q.y), e + 1);
    b.take(key_f32(q.z), e + 2);
    b.take(key_f32(q.w), e + 3);
  }
};

template <uint32_t kNanMag>
struct Logit16 {
  static constexpr int kBytes = 2;
  __device__ static uint32_t key_at(const char* row, int64_t i) {
    return key_16<kNanMag>(*reinterpret_cast<const uint16_t*>(row + 2 * i));
  }
  static constexpr uint32_t kPosInf = kNanMag | 0x8000u;                  // key of +inf
  static constexpr uint32_t kNegInf = ((kNanMag | 0x8000u) ^ 0xFFFFu) + 1u;  // key of -inf
  // Largest key of a 16-byte vector of 8 logits (0xFFFF if it holds a NaN).
  __device__ static uint32_t vec_key(const uint4& q) {
    const u16x2 a = keys2(q.x), b = keys2(q.y), c = keys2(q.z), d = keys2(q.w);
    const u16x2 hi = __builtin_elementwise_max(__builtin_elementwise_max(a, b), __builtin_elementwise_max(c, d));
    const u16x2 lo = __builtin_elementwise_min(__builtin_elementwise_min(a, b), __builtin_elementwise_min(c, d));
    const uint32_t vmax = hi.x > hi.y ? hi.x : hi.y;
    const uint32_t vmin = lo.x < lo.y ? lo.x : lo.y;
    return (vmax > kPosInf || vmin < kNegInf) ? 0xFFFFu : vmax;
  }
  // The lowest element of vector q (first element index e) whose key is k.
  __device__ static void take_in_vec(Best& b, const uint4& q, uint32_t k, int32_t e) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    int32_t at = e + 7;
#pragma unroll
    for (int j = 7; j >= 0; --j) {
      const uint32_t h = (w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
      if (key_16<kNanMag>(h) == k) at = e + j;
    }
    b.take(k, at);
  }
};
template <>
struct Logit<1> : Logit16<0x7F80u> {};  // bf16
template <>
struct Logit<2> : Logit16<0x7C00u> {};  // f16

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor(v, off);
    v = o > v ? o : v;
  }
  return v;
}

__device__ __forceinline__ int32_t wave_max_i32(int32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int32_t o = __shfl_xor(v, off);
    v = o > v ? o : v;
  }
  return v;
}

struct VerifyArgs {
  const char* logits;
  const int32_t* draft;
  const int32_t* pad_in;
  int32_t B, k, V, W_in;
  int32_t* tokens;
  int32_t* n_acc;
  int32_t* bonus;
  int32_t* pad_out;
  int32_t* w_new;
  unsigned long long* partial;  // [B*(k+1)][chunks] packed maxima
  uint32_t* dev_status;
  int64_t chunk_elems;
  int32_t chunks;               // workgroups per logit row
  int32_t* order;               // in-place realignment order table (NULL: not written)
  int32_t* order_group;         // the rows that the walk takes at a time
  int32_t order_even_len;
  int32_t order_by_row;         // 2: rows one at a time; 1: where their lengths are uneven; 0: never
};

// Tunables of the vocabulary scan (compile-time; chosen by sweeping on
// MI355X with the logits read from HBM):
//   SPECDEC_VERIFY_UNROLL     16-byte loads per thread in flight per iteration
//   SPECDEC_VERIFY_TARGET     workgroups the scan aims for in total
//   SPECDEC_VERIFY_MIN_CHUNK / SPECDEC_VERIFY_MAX_CHUNK  logits per workgroup
#ifndef SPECDEC_VERIFY_UNROLL
#define SPECDEC_VERIFY_UNROLL 4
#endif
#ifndef SPECDEC_VERIFY_TARGET
#define SPECDEC_VERIFY_TARGET 2048
#endif
#ifndef SPECDEC_VERIFY_MIN_CHUNK
#define SPECDEC_VERIFY_MIN_CHUNK 2048
#endif
#ifndef SPECDEC_VERIFY_MAX_CHUNK
#define SPECDEC_VERIFY_MAX_CHUNK 16384
#endif
// Scan logit elements [beg, end) of one row; 16-byte vectors over the aligned
// interior, single elements for the unaligned head and the tail.
template <int DT, int kTpb = kThreads, int kUnroll = SPECDEC_VERIFY_UNROLL>
__device__ __forceinline__ void scan_range(const char* row, int64_t beg, int64_t end, Best& b) {
  using T = Logit<DT>;
  constexpr int kPerVec = 16 / T::kBytes;
  const int tid = threadIdx.x;
  const uintptr_t addr = reinterpret_cast<uintptr_t>(row) + static_cast<uintptr_t>(beg) * T::kBytes;
  int64_t head = static_cast<int64_t>((16u - (addr & 15u)) & 15u) / T::kBytes;
  if (head > end - beg) head = end - beg;
  const int64_t a0 = beg + head;
  const int64_t nvec = (end - a0) / kPerVec;
  const int64_t a1 = a0 + nvec * kPerVec;
  if (tid < head) b.take(T::key_at(row, beg + tid), static_cast<int32_t>(beg + tid));
  const uint4* vp = reinterpret_cast<const uint4*>(row + a0 * T::kBytes);
  if constexpr (T::kBytes == 2) {
    // per vector only its largest key; the first vector (lowest index) holding
    // this thread's largest key is kept in registers and searched at the end
    uint32_t vk = 0u;
    int32_t ve = -1;
    uint4 vq = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t v0 = 0; v0 < nvec; v0 += kTpb * kUnroll) {
      uint4 q[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t v = v0 + u * kTpb + tid;
        q[u] = v < nvec ? vp[v] : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t v = v0 + u * kTpb + tid;
        const uint32_t k = T::vec_key(q[u]);
        if (v < nvec && k > vk) {
          vk = k;
          ve = static_cast<int32_t>(a0 + v * kPerVec);
          vq = q[u];
        }
      }
    }
    if (ve >= 0) T::take_in_vec(b, vq, vk, ve);
  } else {
    for (int64_t v0 = 0; v0 < nvec; v0 += kTpb * kUnroll) {
      uint4 q[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t v = v0 + u * kTpb + tid;
        q[u] = v < nvec ? vp[v] : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t v = v0 + u * kTpb + tid;
        if (v < nvec) T::take_vec(b, q[u], static_cast<int32_t>(a0 + v * kPerVec));
      }
    }
  }
  if (tid < end - a1) b.take(T::key_at(row, a1 + tid), static_cast<int32_t>(a1 + tid));
}

template <int DT>
__global__ __launch_bounds__(kThreads) void verify_partial_kernel(VerifyArgs a) {
  __shared__ unsigned long long wkey[kWaves];
  const int64_t row = blockIdx.x / a.chunks;
  const int64_t chunk = blockIdx.x - row * a.chunks;
  const int64_t beg = chunk * a.chunk_elems;
  int64_t end = beg + a.chunk_elems;
  if (end > a.V) end = a.V;
  const char* rowp = a.logits + row * static_cast<int64_t>(a.V) * Logit<DT>::kBytes;

  Best b;
  scan_range<DT>(rowp, beg, end, b);
  unsigned long long key =
      (static_cast<unsigned long long>(b.key) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(b.idx));
  key = wave_max_u64(key);
  if ((threadIdx.x & 63) == 0) wkey[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long k2 = wkey[0];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) k2 = wkey[q] > k2 ? wkey[q] : k2;
    a.partial[blockIdx.x] = k2;
  }
}

constexpr int kFinalizeThreads = 1024;

// Geometry of row i after verification: ok (pad_in in range), the new length
// and padding; the row moves when its padding changes.
struct RowMove {
  bool ok, moves;
  int32_t p, po, len;
};
__device__ __forceinline__ RowMove row_move(const VerifyArgs& a, int i, int32_t w) {
  const int32_t L = a.W_in - (a.k + 1);
  RowMove m;
  m.p = a.pad_in[i];
  m.ok = m.p >= 0 && m.p <= L;
  m.len = (L - m.p) + a.n_acc[i] + 1;
  m.po = w - m.len;
  m.moves = m.ok && m.po != m.p;
  return m;
}

// The in-place realignment order (one workgroup of kFinalizeThreads, after
// the paddings): moving rows in classes of equal length range, longest first,
// then the rows with nothing to move; each class in increasing row order (a
// stable partition: per chunk of rows a ballot per class, then prefixes over
// the waves).  The in-place walk takes the spans of the longest rows first, so
// that the longest walks do not start last.  It takes them one at a time (in
// 7 classes) or, for a cache of many spans or even lengths, 32 (in 2): see
// inplace_plan.
__device__ void write_inplace_order(const VerifyArgs& a, int32_t w) {
  constexpr int kW = kFinalizeThreads / 64;
  constexpr int kCls = kMaxOrderClasses;
  __shared__ int32_t s_lo[kW], s_hi[kW], s_movers[kW];
  __shared__ int32_t s_cnt[kCls], s_start[kCls], s_carry[kCls];
  __shared__ int32_t s_wave[kCls][kW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int32_t lo = 0x7FFFFFFF, hi = 0, movers = 0;
  for (int i = tid; i < a.B; i += kFinalizeThreads) {
    const RowMove m = row_move(a, i, w);
    if (m.moves) {
      lo = m.len < lo ? m.len : lo;
      hi = m.len > hi ? m.len : hi;
      movers = 1;
    }
  }
  movers = __popcll(__ballot(movers != 0));   // of this wave, at least
  hi = wave_max_i32(hi);
  lo = -wave_max_i32(-lo);
  if (lane == 0) {
    s_hi[wv] = hi;
    s_lo[wv] = lo;
    s_movers[wv] = movers;
  }
  if (tid < kCls) {
    s_cnt[tid] = 0;
    s_carry[tid] = 0;
  }
  __syncthreads();
  hi = s_hi[0];
  lo = s_lo[0];
  movers = s_movers[0];
#pragma unroll
  for (int q = 1; q < kW; ++q) {
    movers += s_movers[q];
    hi = s_hi[q] > hi ? s_hi[q] : hi;
    lo = s_lo[q] < lo ? s_lo[q] : lo;
  }
  const int64_t range = static_cast<int64_t>(hi) - lo + 1;
  // even: at least five rows, of lengths within a quarter of the longest
  const bool by_row = a.order_by_row == 2 ||
                      (a.order_by_row == 1 && (movers < 5 || lo < hi - hi / 4 || hi < a.order_even_len));
  const int moving = by_row ? kCls - 1 : 2;    // the class after them: rows with nothing to move
  if (tid == 0) *a.order_group = by_row ? 1 : 32;
  auto cls = [&](const RowMove& m) {
    if (!m.moves) return moving;
    const int64_t c = (static_cast<int64_t>(hi) - m.len) * moving / range;
    return static_cast<int>(c < moving ? c : moving - 1);
  };
  for (int i = tid; i < a.B; i += kFinalizeThreads) atomicAdd(&s_cnt[cls(row_move(a, i, w))], 1);
  __syncthreads();
  if (tid == 0) {
    int32_t acc = 0;
    for (int c = 0; c < kCls; ++c) {
      s_start[c] = acc;
      acc += s_cnt[c];
    }
  }
  __syncthreads();
  for (int base = 0; base < a.B; base += kFinalizeThreads) {
    const int i = base + tid;
    RowMove m{};
    int c = kCls;   // past the end of the batch
    if (i < a.B) {
      m = row_move(a, i, w);
      c = cls(m);
    }
    int rank = 0;
#pragma unroll
    for (int cc = 0; cc < kCls; ++cc) {
      const unsigned long long bits = __ballot(c == cc);
      if (lane == 0) s_wave[cc][wv] = __popcll(bits);
      if (c == cc) rank = __popcll(bits & ((1ull << lane) - 1ull));
    }
    __syncthreads();
    if (c < kCls) {
      int32_t pos = s_start[c] + s_carry[c] + rank;
      for (int q = 0; q < wv; ++q) pos += s_wave[c][q];
      int32_t* e = a.order + 4 * static_cast<int64_t>(pos);   // four words (the workspace is 8-byte aligned)
      e[0] = i;
      e[1] = m.p;
      e[2] = m.moves ? m.po : m.p;   // nothing to move: equal paddings
      e[3] = m.len;
    }
    __syncthreads();
    if (tid < kCls) {
      int32_t add = 0;
      for (int q = 0; q < kW; ++q) add += s_wave[tid][q];
      s_carry[tid] += add;
    }
    __syncthreads();
  }
}

// One workgroup of kFinalizeThreads: row maxima, then per sequence the
// prefix-match scan, the bonus token and its new length; then the width and
// the paddings.

__global__ __launch_bounds__(kFinalizeThreads) void verify_finalize_kernel(VerifyArgs a) {
  __shared__ int32_t wmax[kFinalizeThreads / 64];
  const int32_t L = a.W_in - (a.k + 1);
  const int kp1 = a.k + 1;
  const int64_t rows = static_cast<int64_t>(a.B) * kp1;
  // row maxima -> predicted tokens
  for (int64_t r = threadIdx.x; r < rows; r += kFinalizeThreads) {
    const unsigned long long* p = a.partial + r * a.chunks;
    unsigned long long m = p[0];
    for (int c = 1; c < a.chunks; ++c) m = p[c] > m ? p[c] : m;
    a.tokens[r] = static_cast<int32_t>(~static_cast<uint32_t>(m & 0xFFFFFFFFull));
  }
  __syncthreads();  // tokens written by this workgroup are visible to it
  int32_t local = 0;
  for (int i = threadIdx.x; i < a.B; i += kFinalizeThreads) {
    const int32_t p = a.pad_in[i];
    const bool ok = p >= 0 && p <= L;
    const int32_t* tok = a.tokens + static_cast<int64_t>(i) * kp1;
    const int32_t* dr = a.draft + static_cast<int64_t>(i) * a.k;
    int32_t nacc = a.k;
    for (int r = 0; r < a.k; ++r)
      if (dr[r] != tok[r]) {
        nacc = r;
        break;
      }
    a.n_acc[i] = nacc;
    if (a.bonus) a.bonus[i] = tok[nacc];
    if (ok) {
      const int32_t len = (L - p) + nacc + 1;
      local = len > local ? len : local;
    } else if (a.dev_status) {
      atomicOr(a.dev_status, kBadPadIn);
    }
  }
  local = wave_max_i32(local);
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = local;
  __syncthreads();
  int32_t w = wmax[0];
#pragma unroll
  for (int q = 1; q < kFinalizeThreads / 64; ++q) w = wmax[q] > w ? wmax[q] : w;
  for (int i = threadIdx.x; i < a.B; i += kFinalizeThreads) {
    const int32_t p = a.pad_in[i];
    const bool ok = p >= 0 && p <= L;
    a.pad_out[i] = ok ? w - ((L - p) + a.n_acc[i] + 1) : -1;
  }
  if (threadIdx.x == 0) a.w_new[0] = w;
  if (a.order) write_inplace_order(a, w);
}

// One launch of greedy verification for batches whose logit rows are short
// enough for one workgroup each (used where the library owns the scratch and
// so knows its counters start at zero).  Every workgroup scans one whole row
// and writes its prediction; the last row of a sequence to finish (an
// agent-scope acquire-release count per sequence) does that sequence's
// prefix-match scan, bonus token and new length; the last sequence to finish
// (one more count) computes the width and the paddings.  A release fence
// costs a serialized L2 write-back on this GPU (about 19 ns each, measured),
// so the design keeps one count per row and one per sequence, never one per
// chunk of a row.  No workgroup waits for another: each one counts and either
// exits or, being last, carries on.
struct FusedVerifyArgs {
  VerifyArgs v;
  uint32_t* seq_count;    // [B], zero on entry
  uint32_t* batch_count;  // [1], zero on entry
  int32_t* lens;          // [B] new lengths (0 for a row with a bad pad_in)
};

constexpr int kFusedThreads = 1024, kFusedUnroll = 8, kFusedWaves = kFusedThreads / 64;
static_assert(kFusedThreads * kFusedUnroll * 16 >= 128 * 1024, "a fused row is one iteration of loads");

template <int DT>
__global__ __launch_bounds__(kFusedThreads) void verify_fused_kernel(FusedVerifyArgs f) {
  const VerifyArgs& a = f.v;
  __shared__ unsigned long long wkey[kFusedWaves];
  __shared__ int32_t wmax[kFusedWaves];
  __shared__ int seq_last, batch_last;   // one flag per stage: no wave reads a flag another stage rewrites
  const int64_t row = blockIdx.x;
  const int kp1 = a.k + 1;
  const int i = static_cast<int>(row / kp1);
  Best b;
  scan_range<DT, kFusedThreads, kFusedUnroll>(a.logits + row * static_cast<int64_t>(a.V) * Logit<DT>::kBytes, 0,
                                              a.V, b);
  unsigned long long key =
      (static_cast<unsigned long long>(b.key) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(b.idx));
  key = wave_max_u64(key);
  if ((threadIdx.x & 63) == 0) wkey[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long k2 = wkey[0];
#pragma unroll
    for (int q = 1; q < kFusedWaves; ++q) k2 = wkey[q] > k2 ? wkey[q] : k2;
    a.tokens[row] = static_cast<int32_t>(~static_cast<uint32_t>(k2 & 0xFFFFFFFFull));
    const uint32_t before = __hip_atomic_fetch_add(f.seq_count + i, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    seq_last = before == static_cast<uint32_t>(a.k);
  }
  __syncthreads();
  if (!seq_last) return;
  // the sequence's k+1 predictions are all written: wave 0 makes them visible
  // to itself and loads them, and the drafts, at once (one lane per slot)
  if (threadIdx.x < 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const int lane = static_cast<int>(threadIdx.x);
    const int32_t L = a.W_in - kp1;
    const int32_t* tok = a.tokens + static_cast<int64_t>(i) * kp1;
    const int32_t* dr = a.draft + static_cast<int64_t>(i) * a.k;
    const int32_t t = lane <= a.k ? tok[lane] : 0;
    const int32_t d = lane < a.k ? dr[lane] : 0;
    const int32_t t_last = tok[a.k];                       // the prediction after the last draft (lane 64 for k = 64)
    const unsigned long long miss = __ballot(lane < a.k && d != t);
    const int32_t nacc = miss ? static_cast<int32_t>(__builtin_ctzll(miss)) : a.k;
    const int32_t bon = __shfl(t, nacc < 64 ? nacc : 0);
    if (lane == 0) {
      const int32_t p = a.pad_in[i];
      a.n_acc[i] = nacc;
      if (a.bonus) a.bonus[i] = nacc < 64 ? bon : t_last;
      const bool ok = p >= 0 && p <= L;
      f.lens[i] = ok ? (L - p) + nacc + 1 : 0;           // 0: left out of the width, padding -1
      if (!ok && a.dev_status) atomicOr(a.dev_status, kBadPadIn);
      const uint32_t before = __hip_atomic_fetch_add(f.batch_count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      batch_last = before == static_cast<uint32_t>(a.B - 1);
    }
  }
  __syncthreads();
  if (!batch_last) return;
  // every sequence's length is written; each wave makes them visible to
  // itself, and one load of each length gives both the width and the padding
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  constexpr int kPer = kMaxFusedVerifyRows / kFusedThreads;   // sequences per thread at most (B <= rows)
  int32_t len[kPer];
  int32_t local = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int q = static_cast<int>(threadIdx.x) + j * kFusedThreads;
    len[j] = q < a.B ? f.lens[q] : 0;
    local = len[j] > local ? len[j] : local;
  }
  local = wave_max_i32(local);
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = local;
  __syncthreads();
  int32_t w = wmax[0];
#pragma unroll
  for (int q = 1; q < kFusedWaves; ++q) w = wmax[q] > w ? wmax[q] : w;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int q = static_cast<int>(threadIdx.x) + j * kFusedThreads;
    if (q < a.B) a.pad_out[q] = len[j] > 0 ? w - len[j] : -1;
  }
  if (threadIdx.x == 0) a.w_new[0] = w;
}

// ---------------------------------------------------------------------------
// realign
//
// Tunables (compile-time; the defaults were chosen by sweeping on MI355X):
//   *_VEC  16-byte vectors per lane per chunk (out of place: pieces per
//          workgroup)
//   *_TPB  threads per workgroup (a multiple of 64)
//   *_NT   nontemporal hints (the cache is streamed once): bit 0 on loads,
//          bit 1 on stores
// Small, in-order workgroups keep the set of DRAM rows touched at any moment
// compact; spreading a workgroup's pieces apart keeps that pattern while
// halving the number of workgroups, which matters where a workgroup only
// stores (padding) and the dispatch rate would otherwise bound the kernel.
// ---------------------------------------------------------------------------
#ifndef SPECDEC_OOP_VEC
#define SPECDEC_OOP_VEC 2
#endif
#ifndef SPECDEC_OOP_TPB
#define SPECDEC_OOP_TPB 64
#endif
#ifndef SPECDEC_OOP_NT
#define SPECDEC_OOP_NT 3
#endif
#ifndef SPECDEC_INPLACE_VEC
#define SPECDEC_INPLACE_VEC 32
#endif
#ifndef SPECDEC_INPLACE_TPB
#define SPECDEC_INPLACE_TPB 256
#endif
#ifndef SPECDEC_INPLACE_NT
#define SPECDEC_INPLACE_NT 3
#endif

constexpr int kOopVec = SPECDEC_OOP_VEC, kOopTpb = SPECDEC_OOP_TPB, kOopNt = SPECDEC_OOP_NT;
constexpr int kInVec = SPECDEC_INPLACE_VEC, kInTpb = SPECDEC_INPLACE_TPB, kInNt = SPECDEC_INPLACE_NT;
static_assert(kOopTpb % 64 == 0 && kInTpb % 64 == 0, "workgroups are whole wavefronts");
constexpr int kCus = 256;        // compute units of the GPU
constexpr int kSmallTpb = 256;   // threads of a small step's merged launch
// A small step: workgroups that move the cache, and bytes that they merge in
// all (out of place, in place).  Steps in us, three launches / two: 1024
// workgroups of 3 KB, in place 20.0 / 15.9; 2048 of 24 KB 33.2 / 32.9; 4096 of
// 12 KB 55.8 / 55.2; 8192 of 3 KB 97.7 / 94.4, of 14 KB 45.2 / 54.3.  Out of
// place 2560 of 6 KB 15.7 / 14.9, 3072 of 6 KB 15.3 / 15.7, 5120 of 1.5 KB 19.0 /
// 17.5, 6144 of 0.8 KB 21.2 / 20.4.
constexpr int64_t kSmallMaxBlocks = 8192, kSmallMaxMergedOop = 16 << 20, kSmallMaxMergedInPlace = 52 << 20;

struct RealignArgs {
  const u32x4* src;
  u32x4* dst;
  int64_t src_span_vecs, dst_span_vecs;  // cap * D / 8
  int32_t vpc;                           // 16-byte vectors per column: D / 8
  int32_t B, H, k, W_in;
  const int32_t* pad_in;
  const int32_t* n_acc;
  const int32_t* w_new;
  uint32_t* dev_status;
  uint32_t chunks;                       // workgroups per span (out of place)
  uint32_t misaligned;                   // out of place: spans tiled from the group boundary below them
  uint32_t realign_blocks;               // realign workgroups in this launch
  uint32_t span_base;                    // first span of this launch
  uint32_t nspans;                       // L * 2 * B * H
  // workgroups before the realign ones: position ids / mask, then the token row
  uint32_t extra_blocks;
  uint32_t pm_blocks;
  int64_t* pos;
  uint8_t* mask;
  const int32_t* pad_out;
  int64_t pm_cap;
  uint32_t pm_col_blocks;
  const int32_t* s_in;                   // token row S [B][s_in_stride]
  int32_t* s_out;                        // [B][s_out_stride]; == s_in: in place
  int64_t s_in_stride, s_out_stride;
  const int32_t* tokens;                 // [B][k+1] predictions from verification
  int32_t pad_id;
  uint32_t tok_col_blocks;               // workgroups per token row (1 in place)
  uint32_t tok_blocks;                   // token-row workgroups in all
  uint32_t* clear_words;                 // one more workgroup zeroes these (NULL: none)
  uint32_t clear_count;
  const int32_t* order;                  // in place: verification's order table (NULL: the cache's order)
  const int32_t* order_group;            // with the table, and row_group 0: rows taken together
  uint32_t span_rows;                    // spans per row: L * 2 * H
  uint32_t row_group;                    // ordered rows taken together, slab by slab (0: as order_group says)
  int32_t len_half, len_quarter;         // longest rows whose spans fit half / a quarter of a walk's chunk
  uint32_t slots;                        // in place by chunks, and in a small step: spans * chunks
};

struct RowGeom {
  int32_t pad_in, pad_out, len, w;
};

// Geometry of a row with padding p, n accepted drafts and the new width w;
// returns the error bits (0 = valid).
__device__ __forceinline__ uint32_t geometry_of(const RealignArgs& a, int32_t w, int32_t p, int32_t n, RowGeom& g) {
  const int32_t L = a.W_in - (a.k + 1);
  uint32_t err = 0u;
  if (p < 0 || p > L) err |= kBadPadIn;
  if (n < 0 || n > a.k) err |= kBadAccept;
  if (err) return err;
  const int32_t len = (L - p) + n + 1;
  if (w < 1 || w > a.W_in || len > w) return kBadWidth;
  g.pad_in = p;
  g.pad_out = w - len;
  g.len = len;
  g.w = w;
  return 0u;
}

__device__ __forceinline__ uint32_t row_geometry(const RealignArgs& a, int row, RowGeom& g) {
  return geometry_of(a, load_invariant(a.w_new), load_invariant(a.pad_in + row), load_invariant(a.n_acc + row), g);
}

// Position ids and mask for 4*kTpb columns (the cb-th) of one row with new
// padding po, in a batch of new width w.
template <int kTpb>
__device__ __forceinline__ void posmask_row(uint32_t row, uint32_t cb, int64_t* pos, uint8_t* mask, int32_t po, int32_t w,
                                            int32_t k, int64_t pm_cap, uint32_t* dev_status) {
  const int64_t width = static_cast<int64_t>(w) + k + 1;
  if (w < 0 || po < 0 || po > w || width > pm_cap) {
    if (cb == 0 && threadIdx.x == 0 && dev_status) atomicOr(dev_status, kBadPadOut);
    return;
  }
  posmask_cols<kTpb>(cb, pos + static_cast<int64_t>(row) * pm_cap, mask + static_cast<int64_t>(row) * pm_cap, po,
                     width);
}

template <int kTpb>
__device__ void posmask_block(uint32_t blk, int64_t* pos, uint8_t* mask, const int32_t* pad_out,
                              const int32_t* w_new, int32_t k, int64_t pm_cap, uint32_t col_blocks,
                              uint32_t* dev_status) {
  const uint32_t row = blk / col_blocks;
  posmask_row<kTpb>(row, blk - row * col_blocks, pos, mask, load_invariant(pad_out + row), load_invariant(w_new), k,
                    pm_cap, dev_status);
}

// Token row S of one sequence (Alg. 1, phase 3): the c_i + 1 tokens of the
// row (its cached tokens and the pending token) move from column pad_in to
// pad_out, the accepted drafts and the bonus token (the predictions
// tokens[0..n_acc]) follow them, and columns [0, pad_out) hold pad_id; the
// new row is L' + 1 wide.  Out of place a workgroup writes 4*kTpb columns of
// one row; in place one workgroup walks the whole row in the direction of its
// shift and writes the padding and the appended tokens after a barrier.
// (w, p, n: the new width, the row's padding and accepted count; tk: its
// predictions.)
template <int kTpb>
__device__ void token_row(const RealignArgs& a, uint32_t row, uint32_t cb, int32_t w, int32_t p, int32_t n,
                          const int32_t* tk) {
  RowGeom g;
  const uint32_t err = geometry_of(a, w, p, n, g);
  if (err) {
    if (cb == 0 && threadIdx.x == 0 && a.dev_status) atomicOr(a.dev_status, err);
    return;
  }
  const int32_t c = a.W_in - (a.k + 1) - p;
  const int64_t po = g.pad_out;                                 // new padding
  const int64_t keep_end = po + c + 1;                          // end of the moved tokens
  const int64_t width = static_cast<int64_t>(w) + 1;
  const int32_t* src = a.s_in + static_cast<int64_t>(row) * a.s_in_stride;
  int32_t* dst = a.s_out + static_cast<int64_t>(row) * a.s_out_stride;
  if (a.s_in != a.s_out) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t j = static_cast<int64_t>(cb) * (4 * kTpb) + q * kTpb + threadIdx.x;
      if (j < width) {
        int32_t v;
        if (j < po) v = a.pad_id;
        else if (j < keep_end) v = src[j - po + p];
        else v = tk[j - keep_end];
        dst[j] = v;
      }
    }
    return;
  }
  // in place
  const int64_t nt = c + 1;
  const int64_t shift = po - p;
  constexpr int64_t kChunk = 4 * kTpb;
  if (shift != 0) {
    for (int64_t it = 0; it < nt; it += kChunk) {
      // right shifts walk from the top, left shifts from the bottom
      const int64_t lo = shift > 0 ? nt - it - kChunk : it;
      int32_t v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int64_t u = lo + q * kTpb + threadIdx.x;
        u = u < 0 ? 0 : (u >= nt ? nt - 1 : u);
        v[q] = dst[p + u];
      }
      asm volatile("" ::"v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t u = lo + q * kTpb + threadIdx.x;
        if (u >= 0 && u < nt) dst[po + u] = v[q];
      }
    }
    __syncthreads();
  }
  for (int64_t j = threadIdx.x; j < po; j += kTpb) dst[j] = a.pad_id;
  for (int64_t j = keep_end + threadIdx.x; j < width; j += kTpb) dst[j] = tk[j - keep_end];
}

template <int kTpb>
__device__ void token_block(const RealignArgs& a, uint32_t blk) {
  const uint32_t row = blk / a.tok_col_blocks;
  token_row<kTpb>(a, row, blk - row * a.tok_col_blocks, load_invariant(a.w_new), load_invariant(a.pad_in + row),
                  load_invariant(a.n_acc + row), a.tokens + static_cast<int64_t>(row) * (a.k + 1));
}

template <int kTpb>
__device__ __forceinline__ void extra_block(const RealignArgs& a, uint32_t b) {
  if (b < a.pm_blocks)
    posmask_block<kTpb>(b, a.pos, a.mask, a.pad_out, a.w_new, a.k, a.pm_cap, a.pm_col_blocks, a.dev_status);
  else if (b - a.pm_blocks < a.tok_blocks)
    token_block<kTpb>(a, b - a.pm_blocks);
  else   // the completion counts of the one-launch verification that ran before
    for (uint32_t q = threadIdx.x; q < a.clear_count; q += kTpb) a.clear_words[q] = 0u;
}

// Out of place: the output of a span is cut into groups of kPieces*kSplit
// vectors, each covered by kSplit/kTpb workgroups; every workgroup moves
// kPieces pieces of one wave-width (see split_pieces).
template <int kPieces, int kTpb, int kSplit, int kNt>
__global__ __launch_bounds__(kTpb) void realign_oop_kernel(RealignArgs a) {
  if (blockIdx.x < a.extra_blocks) {
    extra_block<kTpb>(a, blockIdx.x);
    return;
  }
  const uint32_t b = blockIdx.x - a.extra_blocks;
  const uint32_t rel = b / a.chunks;
  const uint32_t sub = b - rel * a.chunks;            // workgroup within the span
  const uint32_t span = a.span_base + rel;
  const int row = static_cast<int>((span / static_cast<uint32_t>(a.H)) % static_cast<uint32_t>(a.B));
  RowGeom g;
  const uint32_t err = row_geometry(a, row, g);
  if (err) {
    if (sub == 0 && span == static_cast<uint32_t>(row) * a.H && threadIdx.x == 0 && a.dev_status)
      atomicOr(a.dev_status, err);
    return;
  }
  u32x4* dspan = a.dst + static_cast<int64_t>(span) * a.dst_span_vecs;
  const int64_t mis = a.misaligned ? split_misalign<kPieces, kSplit>(dspan) : 0;
  const int64_t base = split_base<kPieces, kTpb, kSplit>(sub) - mis;
  const int64_t vpc = a.vpc;
  const int64_t total = static_cast<int64_t>(g.w) * vpc;        // output vectors of the span
  if (base >= total) return;
  const int64_t zero_end = static_cast<int64_t>(g.pad_out) * vpc;
  const int64_t shift = static_cast<int64_t>(g.pad_out - g.pad_in) * vpc;
  split_pieces<kPieces, kTpb, kSplit, kNt>(a.src + static_cast<int64_t>(span) * a.src_span_vecs, dspan, base, total,
                                           zero_end, shift);
}

// Register values of the current thread are live; forces the compiler to
// wait for the loads that produce them before this point.
__device__ __forceinline__ void hold(const u32x4& v) {
  asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
}

// Loads the part that wave `wave` of those on the span has of the chunk from
// `lo` on, 64*kVec vectors each (clipped to [0, n); indices outside are
// clamped, their values unused), of one row's kept vectors, which start at
// `from` within the span.  A wave that is outside as a whole loads nothing
// (ragged rows of 5..124 KB: 511 us a step with its loads, 425 without).
template <int kVec, int kNt>
__device__ __forceinline__ void load_chunk(const u32x4* base, int64_t from, int64_t lo, int64_t n, int wave, u32x4 (&v)[kVec]) {
  const int64_t w0 = lo + static_cast<int64_t>(wave) * (64 * kVec);   // the wave's first vector
  if (w0 >= n || w0 + 64 * kVec <= 0) return;   // the whole wave is outside
  const int64_t t0 = w0 + (threadIdx.x & 63);
#pragma unroll
  for (int j = 0; j < kVec; ++j) {
    int64_t u = t0 + j * 64;
    u = u < 0 ? 0 : (u >= n ? n - 1 : u);
    v[j] = ld16<(kNt & 1) != 0>(base + (from + u));
  }
}

template <int kVec, int kNt>
__device__ __forceinline__ void store_chunk(u32x4* base, int64_t to, int64_t lo, int64_t n, int wave, const u32x4 (&v)[kVec]) {
  const int64_t w0 = lo + static_cast<int64_t>(wave) * (64 * kVec);   // the wave's first vector
  const int lane = static_cast<int>(threadIdx.x & 63);
  u32x4* wb = base + (to + w0);
#pragma unroll
  for (int j = 0; j < kVec; ++j) {
    const int64_t u = w0 + lane + j * 64;
    if (u >= 0 && u < n) st16_at<(kNt & 2) != 0>(wb, static_cast<uint32_t>(lane + j * 64), v[j]);
  }
}

// Workgroup barrier that orders nothing but execution: the values this
// thread loaded are already in its registers (hold), so no other thread's
// later store can change them; loads issued after the barrier's program point
// stay in flight across it.
__device__ __forceinline__ void exec_barrier() { asm volatile("s_barrier" ::: "memory"); }

// The moving rows of a batch of at most 64, put in order by each wave for
// itself, one lane a row, where verification writes no order table (a
// realignment alone).  Rows of unequal lengths go longest first, all spans of
// one row and then the next row's, so that no long walk starts last; where half
// of them reach half of the longest and the spans are many, slab by slab, as
// neighbouring workgroups on neighbouring spans matter more then.  Rows within
// a quarter of the longest keep the cache's order: of up to 2048 spans with the
// rows that stay in their places (1024 spans of 16 rows 246 us, as in the
// cache's order without a look at the rows; 259 with them left out), beyond
// that without them, row_group at a time (4096 spans 1013 -> 997).  Spans
// of uneven rows that fit half or a quarter of a chunk go two or four to a
// workgroup (6144 spans of 5 to 232 KB 155 -> 137 us).  What a workgroup spends
// here counts: it has the CU to itself, and with the longest, the shortest and
// the sum of the lengths kept along in the loop those took 152.
struct OrderedRows {
  RowGeom row;      // lane i: row i
  bool moves;
  int rank;         // its place among the rows that move
  int count;        // of them
  bool even;
  bool together;    // uneven: slab by slab
  // `flag`: this wave reports the rows that it finds out of range
  __device__ __forceinline__ OrderedRows(const RealignArgs& a, bool flag) {
    const int lane = static_cast<int>(threadIdx.x & 63);
    const int32_t w = load_invariant(a.w_new);
    uint32_t err = 0u;
    moves = false;
    row = RowGeom{0, 0, 0, 0};
    if (lane < a.B) {
      err = geometry_of(a, w, a.pad_in[lane], a.n_acc[lane], row);
      moves = err == 0u && row.pad_out != row.pad_in;
    }
    if (flag && err && a.dev_status) atomicOr(a.dev_status, err);
    const unsigned long long movers = __ballot(moves);
    count = __popcll(movers);
    // one key a row: its length (at most 2^24), then its index; 0 for a row that stays
    const uint32_t key = moves ? static_cast<uint32_t>(row.len) << 6 | static_cast<uint32_t>(63 - lane) : 0u;
    rank = 0;
    for (int j = 0; j < a.B; j += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) rank += __builtin_amdgcn_readlane(key, j + u) > key ? 1 : 0;
    even = together = false;
    if (count == 0 || a.row_group == 1u) return;
    auto length_at = [&](int r) { return __builtin_amdgcn_readlane(key, __builtin_ctzll(__ballot(moves && rank == r))) >> 6; };
    const uint32_t longest = length_at(0);
    even = length_at(count - 1) >= longest - longest / 4;
    together = a.nspans > 2048u && 2u * length_at(count / 2) >= longest;
    if (even) rank = __popcll(movers & ((1ull << lane) - 1ull));
  }
  // The lin-th workgroup has the spans j .. j + share - 1 (in the cache's
  // order) of row row_u with geometry g; false past the last.
  __device__ __forceinline__ bool find(const RealignArgs& a, uint32_t lin, uint32_t& j, uint32_t& share, uint32_t& row_u,
                                       RowGeom& g) const {
    const uint32_t S = a.span_rows;
    uint32_t n = static_cast<uint32_t>(count), r;
    share = 1u;
    if (even && a.nspans <= 2048u) {
      const uint32_t H = static_cast<uint32_t>(a.H);
      const uint32_t slab_row = lin / H;
      const uint32_t slab = slab_row / static_cast<uint32_t>(a.B);
      row_u = slab_row - slab * static_cast<uint32_t>(a.B);
      j = slab * H + (lin - slab_row * H);
      geometry_at(static_cast<int>(row_u), g);
      return __builtin_amdgcn_readlane(moves ? 1 : 0, static_cast<int>(row_u)) != 0;
    }
    if (even) {
      if (lin >= n * S) return false;
      const uint32_t H = static_cast<uint32_t>(a.H), R = a.row_group < n ? a.row_group : n;
      const uint32_t gi = lin / (R * S);
      const uint32_t rem = lin - gi * (R * S);
      const uint32_t rows_here = n - gi * R < R ? n - gi * R : R;
      const uint32_t slab = rem / (rows_here * H);
      const uint32_t rr = rem - slab * rows_here * H;
      r = rr / H;
      j = slab * H + (rr - r * H);
      r += gi * R;
    } else {
      uint32_t first = 0u, units = S;   // of the rows with this share: the first one's rank, workgroups a row
      n = __popcll(__ballot(moves && row.len > a.len_half));
      if (lin >= n * units) {
        lin -= n * units;
        first = n;
        share = 2u;
        units = (S + 1u) / 2u;
        n = __popcll(__ballot(moves && row.len > a.len_quarter)) - first;
        if (lin >= n * units) {
          lin -= n * units;
          first += n;
          share = 4u;
          units = (S + 3u) / 4u;
          n = static_cast<uint32_t>(count) - first;
          if (lin >= n * units) return false;
        }
      }
      // together: slab by slab where a slab's heads share out evenly
      const uint32_t H = static_cast<uint32_t>(a.H);
      uint32_t u;
      if (together) {
        const uint32_t hu = H % share == 0u ? H / share : 1u;
        const uint32_t block = lin / (n * hu);
        const uint32_t rem = lin - block * (n * hu);
        r = rem / hu;
        u = block * hu + (rem - r * hu);
      } else {
        r = lin / units;
        u = lin - r * units;
      }
      r += first;
      j = u * share;
    }
    const int i = __builtin_ctzll(__ballot(moves && rank == static_cast<int>(r)));
    row_u = static_cast<uint32_t>(i);
    geometry_at(i, g);
    return true;
  }
  __device__ __forceinline__ void geometry_at(int i, RowGeom& g) const {
    g.pad_in = __builtin_amdgcn_readlane(row.pad_in, i);
    g.pad_out = __builtin_amdgcn_readlane(row.pad_out, i);
    g.len = __builtin_amdgcn_readlane(row.len, i);
    g.w = __builtin_amdgcn_readlane(row.w, i);
  }
};

// In place: one workgroup per span moves the row's kept vectors [from, from+n)
// to [to, to+n) in chunks of kTpb*kVec, walking from the top for a shift to
// higher addresses and from the bottom for a shift to lower ones.  The next
// chunk's source never meets the current chunk's destination, so its loads
// are issued before the current chunk is stored; a barrier after the current
// chunk's loads have landed keeps every read of a chunk ahead of every write
// to it.
// With kSorted the rows are ordered here (OrderedRows), and short ones have two
// or four spans on a workgroup, so many waves each.
template <int kVec, int kTpb, int kNt, bool kSorted>
__global__ __launch_bounds__(kTpb) void realign_inplace_kernel(RealignArgs a) {
  if (blockIdx.x < a.extra_blocks) {
    extra_block<kTpb>(a, blockIdx.x);
    return;
  }
  // Workgroups are dispatched round-robin over the 8 XCDs, and only the rows
  // whose padding changes do any work.  In the cache's own order a row's H
  // spans sit on H consecutive workgroups: with H = 4 and every other row
  // moving, all the work would land on half the XCDs.  So workgroups take
  // the spans in groups of 8 consecutive spans (memory locality as in the
  // cache's order), with the group's spans rotated over the XCDs by the
  // group index: any periodic pattern of moving rows spreads over all XCDs.
  const uint32_t rel = a.span_base + (blockIdx.x - a.extra_blocks);
  const uint32_t grp = rel >> 3;
  const uint32_t lin =
      static_cast<uint64_t>(grp) * 8u + 8u <= a.nspans ? (grp << 3) + ((rel + grp) & 7u) : rel;
  constexpr int kWavesHere = kTpb / 64;
  static_assert(kWavesHere == 4, "four waves share out");
  uint32_t span;
  RowGeom g;
  int waves = kWavesHere, wave = wave_index();   // on the span, and this one's place among them
  bool idle = false;                             // a wave without a span
  if constexpr (kSorted) {
    const OrderedRows rows(a, rel == 0u && threadIdx.x < 64);
    uint32_t j, share, row_u;
    if (!rows.find(a, lin, j, share, row_u, g)) return;
    waves = kWavesHere / static_cast<int>(share);
    j += static_cast<uint32_t>(wave_index() / waves);
    wave = wave_index() % waves;
    idle = j >= a.span_rows;
    const uint32_t slab = j / static_cast<uint32_t>(a.H);
    span = (slab * static_cast<uint32_t>(a.B) + row_u) * static_cast<uint32_t>(a.H) + (j - slab * static_cast<uint32_t>(a.H));
  } else if (a.order) {
    // the rows in the order verification wrote (longest moving rows first),
    // row_group rows at a time, each group slab by slab in the cache's
    // order: the index alone gives (group, slab, row, head), and one load the
    // row's geometry.  Where verification chose the group, the entry for rows
    // one at a time is loaded along with the choice.
    const uint32_t B = static_cast<uint32_t>(a.B), H = static_cast<uint32_t>(a.H);
    const uint32_t group = a.row_group ? a.row_group : static_cast<uint32_t>(load_invariant(a.order_group));
    uint32_t at = lin / a.span_rows, row_u = 0u;
    uint32_t slab = (lin - at * a.span_rows) / H, h = (lin - at * a.span_rows) - slab * H;
    auto entry = [&] {
      const int32_t* info = a.order + 4 * static_cast<int64_t>(at);
      row_u = static_cast<uint32_t>(load_invariant(info));
      g.pad_in = load_invariant(info + 1);
      g.pad_out = load_invariant(info + 2);
      g.len = load_invariant(info + 3);
    };
    if (a.row_group <= 1u) entry();
    if (group > 1u) {
      // R <= B, so a group's spans (R * span_rows <= nspans) fit 32 bits
      const uint32_t R = group < B ? group : B;
      const uint32_t grp_spans = R * a.span_rows;
      const uint32_t gi = lin / grp_spans;
      const uint32_t rem = lin - gi * grp_spans;
      const uint32_t rows_here = B - gi * R < R ? B - gi * R : R;
      slab = rem / (rows_here * H);
      const uint32_t rr = rem - slab * rows_here * H;
      at = gi * R + rr / H;
      h = rr - (rr / H) * H;
      entry();
    }
    span = (slab * B + row_u) * H + h;
  } else {
    span = lin;
    const uint32_t row_u = (span / static_cast<uint32_t>(a.H)) % static_cast<uint32_t>(a.B);
    const int row = static_cast<int>(row_u);
    const uint32_t err = row_geometry(a, row, g);
    if (err) {
      if (span == row_u * static_cast<uint32_t>(a.H) && threadIdx.x == 0 && a.dev_status) atomicOr(a.dev_status, err);
      return;
    }
  }
  const int32_t s = g.pad_out - g.pad_in;
  if (s == 0) return;  // no shift: the row is already in place (uniform acceptance)
  const int64_t vpc = a.vpc;
  u32x4* base = a.dst + static_cast<int64_t>(span) * a.dst_span_vecs;
  const int64_t n = idle ? 0 : static_cast<int64_t>(g.len) * vpc;
  const int64_t from = static_cast<int64_t>(g.pad_in) * vpc;
  const int64_t to = static_cast<int64_t>(g.pad_out) * vpc;
  const int64_t chunk = static_cast<int64_t>(waves) * (64 * kVec);
  const int64_t nchunks = waves < kWavesHere ? 1 : (n + chunk - 1) / chunk;   // the same in all waves of the workgroup
  // chunk c starts at lo(c): from the top for s > 0, from the bottom for s < 0
  auto lo_of = [&](int64_t c) { return s > 0 ? n - (c + 1) * chunk : c * chunk; };
  u32x4 cur[kVec], nxt[kVec];
  load_chunk<kVec, kNt>(base, from, lo_of(0), n, wave, cur);
  for (int64_t c = 0; c < nchunks; ++c) {
    const bool more = c + 1 < nchunks;
    if (more) load_chunk<kVec, kNt>(base, from, lo_of(c + 1), n, wave, nxt);
#pragma unroll
    for (int j = 0; j < kVec; ++j) hold(cur[j]);
    exec_barrier();  // every thread's loads of chunk c have landed
    store_chunk<kVec, kNt>(base, to, lo_of(c), n, wave, cur);
    if (more) {
#pragma unroll
      for (int j = 0; j < kVec; ++j) cur[j] = nxt[j];
    }
  }
  if (s > 0 && !idle) {
    // the vacated columns [pad_in, pad_out) become padding; every read of
    // them landed before the last barrier
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int64_t u0 = 0; u0 < to - from; u0 += waves * 64) {
      const int64_t w0 = u0 + static_cast<int64_t>(wave) * 64;
      const int lane = static_cast<int>(threadIdx.x & 63);
      if (w0 + lane < to - from) st16_at<(kNt & 2) != 0>(base + (from + w0), static_cast<uint32_t>(lane), zero);
    }
  }
  // columns [0, pad_out) already hold padding (+0.0) for a shift to lower addresses
}

// The first `count` vectors from `at` become padding.
template <int kTpb, int kNt>
__device__ __forceinline__ void zero_vectors(u32x4* at, int64_t count) {
  const u32x4 zero = {0u, 0u, 0u, 0u};
  const int lane = static_cast<int>(threadIdx.x & 63);
  for (int64_t u0 = static_cast<int64_t>(wave_index()) * 64; u0 < count; u0 += kTpb)
    if (u0 + lane < count) st16_at<(kNt & 2) != 0>(at + u0, static_cast<uint32_t>(lane), zero);
}

// Moves the vectors [0, n) at `at` by `shift` with one workgroup, chunk after
// chunk in the direction of the shift; with kAhead the next chunk's loads are
// issued before this one's stores, as in realign_inplace_kernel.
template <int kVec, int kTpb, int kNt, bool kAhead>
__device__ void walk_span(u32x4* at, int64_t n, int64_t shift) {
  constexpr int64_t kChunk = static_cast<int64_t>(kTpb) * kVec;
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  const int wave = wave_index();
  auto lo_of = [&](int64_t c) { return shift > 0 ? n - (c + 1) * kChunk : c * kChunk; };
  u32x4 cur[kVec], nxt[kAhead ? kVec : 1];
  if constexpr (kAhead) load_chunk<kVec, kNt>(at, 0, lo_of(0), n, wave, cur);
  for (int64_t c = 0; c < nchunks; ++c) {
    const bool more = c + 1 < nchunks;
    if constexpr (!kAhead) load_chunk<kVec, kNt>(at, 0, lo_of(c), n, wave, cur);
    else if (more) load_chunk<kVec, kNt>(at, 0, lo_of(c + 1), n, wave, nxt);
#pragma unroll
    for (int j = 0; j < kVec; ++j) hold(cur[j]);
    exec_barrier();   // every thread's loads of chunk c have landed, and no later chunk's source meets its place
    store_chunk<kVec, kNt>(at, shift, lo_of(c), n, wave, cur);
    if constexpr (kAhead)
      if (more) {
#pragma unroll
        for (int j = 0; j < kVec; ++j) cur[j] = nxt[j];
      }
  }
  if (shift > 0) zero_vectors<kTpb, kNt>(at, shift);
}

// A row's kept vectors [0, n) cut into chunks of whole 64-vector units, as even
// as they come, each of at most `most` vectors.
struct Chunks {
  int64_t n, per, more;   // per units in a chunk, one more in the first `more`
  int64_t count;
  __device__ __forceinline__ Chunks(int64_t n_, int64_t most) : n(n_) {
    const int64_t units = (n + 63) >> 6;
    count = (n + most - 1) / most;
    per = units / count;
    more = units - per * count;
  }
  __device__ __forceinline__ int64_t lo(int64_t c) const {
    const int64_t at = (c * per + (c < more ? c : more)) << 6;
    return at < n ? at : n;
  }
  // the shortest chunk (the last one's last unit may be ragged)
  __device__ __forceinline__ int64_t shortest() const { return n - lo(count - 1); }
};

// Workgroups start round-robin over the 8 XCDs, and which of the slots hold
// work repeats along the grid (the rows that move, the chunks that a row has):
// with 16 chunks a span, the first chunks of all spans would be one XCD's.
// Slots are taken in groups of 8 neighbours, each group rotated over the XCDs
// by the octal digit sum of its index, so that no power-of-two period meets
// one XCD only.  (64 rows of 128..4096 columns, 16 chunks a span: 2140 us in
// the grid's own order, 1225 so.)
__device__ __forceinline__ uint32_t spread(uint32_t i, uint32_t slots) {
  const uint32_t g = i >> 3;
  const uint32_t r = g + (g >> 3) + (g >> 6) + (g >> 9) + (g >> 12) + (g >> 15) + (g >> 18);
  return (i | 7u) < slots ? (g << 3) | ((i + r) & 7u) : i;
}

// In place, a chunk per workgroup, in two launches.  A span that fits one
// chunk is loaded whole into registers and stored at its new place.  A longer
// one is cut into chunks that move at the same time: each is loaded whole and
// *rotated* by the shift d within its own bounds, so that no workgroup writes
// what another reads.  All but d vectors of a chunk then lie where they
// belong; the d that belong to the neighbour chunk lie in the place that the
// shift vacated (its first d vectors for a shift to higher addresses, its
// last d for one to lower), and realign_strips_kernel hands them over.  Where
// a chunk is shorter than 2 d (a shift of many columns), one workgroup of the
// second launch walks the span instead.
template <int kVec, int kTpb, int kNt, bool kMany>
__device__ __forceinline__ void move_chunk(const RealignArgs& a, uint32_t span, int c, const RowGeom& geo) {
  constexpr int kChunk = kTpb * kVec;
  const int64_t vpc = a.vpc;
  const int64_t shift = static_cast<int64_t>(geo.pad_out - geo.pad_in) * vpc;
  if (shift == 0) return;
  const int64_t n = static_cast<int64_t>(geo.len) * vpc;
  u32x4* at = a.dst + static_cast<int64_t>(span) * a.dst_span_vecs + static_cast<int64_t>(geo.pad_in) * vpc;
  const int lane = static_cast<int>(threadIdx.x & 63);
  const int wv = wave_index();
  int64_t lo = 0;
  int len = static_cast<int>(n < kChunk ? n : kChunk);
  bool first = true, last = true;   // no chunk below / above: its vectors leave it for a place no chunk holds
  if constexpr (kMany) {
    if (n > kChunk) {
      const Chunks ch(n, kChunk);
      if (c >= ch.count) return;
      const int64_t d = shift < 0 ? -shift : shift;
      if (ch.shortest() < 2 * d) return;   // left to the launch that follows
      lo = ch.lo(c);
      len = static_cast<int>(ch.lo(c + 1) - lo);
      first = c == 0;
      last = c == ch.count - 1;
    } else if (c > 0) {
      return;
    }
  }
  const int w0 = wv * (64 * kVec);   // the wave's first vector of the chunk
  const u32x4* s = at + lo + w0;
  // indices past the chunk are clamped, their values unused: a branch per load
  // made the compiler write out a path for every count (227 registers, not 60)
  u32x4 v[kVec] = {};
  if (w0 < len) {
    const int end = len - 1 - w0;
#pragma unroll
    for (int j = 0; j < kVec; ++j) v[j] = ld16<(kNt & 1) != 0>(s + (j * 64 + lane < end ? j * 64 + lane : end));
  }
#pragma unroll
  for (int j = 0; j < kVec; ++j) hold(v[j]);
  exec_barrier();   // every thread's loads have landed
  const bool alone = first && last;
  if (alone || n <= kChunk) {
    u32x4* d = at + (lo + w0 + shift);
#pragma unroll
    for (int j = 0; j < kVec; ++j)
      if (w0 + j * 64 + lane < len) st16_at<(kNt & 2) != 0>(d, static_cast<uint32_t>(j * 64 + lane), v[j]);
    if (shift > 0) zero_vectors<kTpb, kNt>(at, shift);
  } else {
    const int d = static_cast<int>(shift);
    u32x4* base = at + (lo - (first && d < 0 ? -d : 0));
    const int off = first && d < 0 ? -d : 0;
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
      const int e = w0 + j * 64 + lane;
      if (e < len) {
        int to = e + d;
        if (to >= len && !last) to -= len;
        if (to < 0 && !first) to += len;
        st16_at<(kNt & 2) != 0>(base, static_cast<uint32_t>(to + off), v[j]);
      }
    }
  }
}

template <int kVec, int kTpb, int kNt, bool kMany>
__global__ __launch_bounds__(kTpb) void realign_chunk_kernel(RealignArgs a) {
  if (blockIdx.x < a.extra_blocks) {
    extra_block<kTpb>(a, blockIdx.x);
    return;
  }
  const uint32_t g = spread(a.span_base + (blockIdx.x - a.extra_blocks), a.slots);   // span * chunks + chunk
  const uint32_t span = kMany ? g / a.chunks : g;
  const int c = kMany ? static_cast<int>(g - span * a.chunks) : 0;
  const uint32_t row = (span / static_cast<uint32_t>(a.H)) % static_cast<uint32_t>(a.B);
  RowGeom geo;
  const uint32_t err = row_geometry(a, static_cast<int>(row), geo);
  if (err) {
    if (c == 0 && span == row * static_cast<uint32_t>(a.H) && threadIdx.x == 0 && a.dev_status)
      atomicOr(a.dev_status, err);
    return;
  }
  move_chunk<kVec, kTpb, kNt, kMany>(a, span, c, geo);
}

// Hands the strips that realign_chunk_kernel parked over to the neighbour
// chunks, one workgroup per span.  For a shift to higher addresses, strip c
// (the first d vectors of chunk c) goes to the first d vectors of chunk c+1,
// and those of chunk 0 become padding; for one to lower addresses, strip c
// (the last d of chunk c) goes to the last d of chunk c-1, and the end of the
// row, which no column of the new row holds, is left as the walk leaves it:
// with the vectors that moved away from there.  A batch of strips is loaded
// before any is stored; a strip's place holds the strip that was loaded
// before it.
//
// A span whose shift is too long for that is walked here.  kWalk is the walk of
// few spans, 128 KB a turn with the next turn's loads ahead, which takes a CU's
// registers for one workgroup; without it, for the many spans whose strips
// want several workgroups on a CU, 64 KB a turn.  (128 spans of 1 MB moved 200
// columns left, us a step: 98 with 16 KB a turn on the chunks' own launch, 62
// so, 54 with realign_inplace_kernel.)
template <int kTpb, int kNt, bool kWalk>
__global__ __launch_bounds__(kTpb) void realign_strips_kernel(RealignArgs a, int most) {
  constexpr int kVec = 4;
  const uint32_t span = a.span_base + blockIdx.x;
  const uint32_t row = (span / static_cast<uint32_t>(a.H)) % static_cast<uint32_t>(a.B);
  RowGeom geo;
  if (row_geometry(a, static_cast<int>(row), geo)) return;
  const int64_t vpc = a.vpc;
  const int64_t shift = static_cast<int64_t>(geo.pad_out - geo.pad_in) * vpc;
  const int64_t n = static_cast<int64_t>(geo.len) * vpc;
  if (shift == 0 || n <= most) return;
  u32x4* at = a.dst + static_cast<int64_t>(span) * a.dst_span_vecs + static_cast<int64_t>(geo.pad_in) * vpc;
  const Chunks ch(n, most);
  const int64_t d64 = shift < 0 ? -shift : shift;
  if (ch.shortest() < 2 * d64) {
    walk_span<kWalk ? 32 : 16, kTpb, kNt, kWalk>(at, n, shift);
    return;
  }
  const uint32_t d = static_cast<uint32_t>(d64);
  // strips to hand over: count - 1, and to lower addresses the row's end
  const int64_t strips = ch.count - 1 + (shift < 0 ? 1 : 0);
  const int64_t total = strips * d64;
  for (int64_t t0 = 0; t0 < total; t0 += kTpb * kVec) {
    u32x4 v[kVec];
    int64_t to[kVec];
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
      const int64_t t = t0 + j * kTpb + threadIdx.x;
      to[j] = -1;
      if (t < total) {
        const int64_t i = t / d;
        const int64_t e = t - i * d64;
        int64_t from;
        if (shift > 0) {
          const int64_t c = ch.count - 2 - i;
          from = ch.lo(c) + e;
          to[j] = ch.lo(c + 1) + e;
        } else {
          from = (i < ch.count - 1 ? ch.lo(i + 2) - d64 : n - 2 * d64) + e;
          to[j] = ch.lo(i + 1) - d64 + e;
        }
        v[j] = ld16<(kNt & 1) != 0>(at + from);
      }
    }
#pragma unroll
    for (int j = 0; j < kVec; ++j) hold(v[j]);
    exec_barrier();
#pragma unroll
    for (int j = 0; j < kVec; ++j)
      if (to[j] >= 0) st16_at<(kNt & 2) != 0>(at + to[j], 0u, v[j]);
  }
  if (shift > 0) zero_vectors<kTpb, kNt>(at, shift);
}

// ---------------------------------------------------------------------------
// Small steps: after the vocabulary scan, one launch that merges it and
// realigns.  Every workgroup merges the partial maxima for itself (a few KB:
// at most kSmallRows logit rows) and goes on with its share of the
// realignment, so that the merge is not a launch of its own; workgroup 0 also
// stores the verification's outputs.  A launch costs such a step more than
// the repeated merge: the tiny step takes 9.1 us instead of 12.4, two rows of 64
// to 200 columns on one KV head in place 10.4 instead of 20.1.
// ---------------------------------------------------------------------------
constexpr int kSmallRows = kSmallTpb;

struct SmallOutcome {
  int32_t tok[kSmallRows];    // predictions [B][k+1]
  int32_t n_acc[kSmallRows], pad_in[kSmallRows], pad_out[kSmallRows];
  int32_t wmax[kSmallTpb / 64];
  int32_t w;
};

// `lanes` threads to a logit row: a power of two, at most 64, rows * lanes <= kSmallTpb.
__device__ void small_merge(const VerifyArgs& a, int lanes, SmallOutcome& s) {
  const int t = threadIdx.x, kp1 = a.k + 1, rows = a.B * kp1;
  const int row = t / lanes, q = t & (lanes - 1);
  const int i = row / kp1, r = row - i * kp1;
  const bool leads = row < rows && q == 0;
  const int32_t drafted = leads && r < a.k ? a.draft[i * a.k + r] : 0;
  const int32_t p = t < a.B ? a.pad_in[t] : 0;
  unsigned long long m = 0u;
  if (row < rows)
    for (int c = q; c < a.chunks; c += lanes) {
      const unsigned long long v = a.partial[static_cast<int64_t>(row) * a.chunks + c];
      m = v > m ? v : m;
    }
  for (int off = lanes >> 1; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(m, off);
    m = o > m ? o : m;
  }
  if (t < a.B) {
    s.n_acc[t] = a.k;
    s.pad_in[t] = p;
  }
  __syncthreads();
  if (leads) {
    const int32_t tok = static_cast<int32_t>(~static_cast<uint32_t>(m & 0xFFFFFFFFull));
    s.tok[row] = tok;
    if (r < a.k && drafted != tok) atomicMin(&s.n_acc[i], r);   // the first mismatch
  }
  __syncthreads();
  const int32_t L = a.W_in - kp1;
  const int32_t len = t < a.B && p >= 0 && p <= L ? (L - p) + s.n_acc[t] + 1 : 0;
  const int32_t most = wave_max_i32(len);
  if ((t & 63) == 0) s.wmax[t >> 6] = most;
  __syncthreads();
  int32_t w = s.wmax[0];
#pragma unroll
  for (int v = 1; v < kSmallTpb / 64; ++v) w = s.wmax[v] > w ? s.wmax[v] : w;
  const int32_t po = len > 0 ? w - len : -1;
  if (t < a.B) s.pad_out[t] = po;
  if (t == 0) s.w = w;
  __syncthreads();
  if (blockIdx.x == 0) {
    if (t < rows) a.tokens[t] = s.tok[t];
    if (t < a.B) {
      const int32_t n = s.n_acc[t];
      a.n_acc[t] = n;
      a.pad_out[t] = po;
      if (a.bonus) a.bonus[t] = s.tok[t * kp1 + n];
      if (len == 0 && a.dev_status) atomicOr(a.dev_status, kBadPadIn);
    }
    if (t == 0) a.w_new[0] = w;
  }
}

template <bool kInPlace, int kVec>
__global__ __launch_bounds__(kSmallTpb) void small_step_kernel(VerifyArgs v, RealignArgs a, int lanes) {
  __shared__ SmallOutcome s;
  small_merge(v, lanes, s);
  uint32_t b = blockIdx.x;
  if (b < a.pm_blocks) {
    const uint32_t row = b / a.pm_col_blocks;
    posmask_row<kSmallTpb>(row, b - row * a.pm_col_blocks, a.pos, a.mask, s.pad_out[row], s.w, a.k, a.pm_cap, a.dev_status);
    return;
  }
  b -= a.pm_blocks;
  if (b < a.tok_blocks) {
    const uint32_t row = b / a.tok_col_blocks;
    token_row<kSmallTpb>(a, row, b - row * a.tok_col_blocks, s.w, s.pad_in[row], s.n_acc[row], s.tok + row * (a.k + 1));
    return;
  }
  b = spread(b - a.tok_blocks, a.slots);
  const uint32_t span = b / a.chunks, sub = b - span * a.chunks;
  const uint32_t row = (span / static_cast<uint32_t>(a.H)) % static_cast<uint32_t>(a.B);
  RowGeom g;
  if (geometry_of(a, s.w, s.pad_in[row], s.n_acc[row], g)) return;   // a bad padding: flagged by workgroup 0
  if constexpr (kInPlace) {
    move_chunk<kVec, kSmallTpb, kInNt, false>(a, span, 0, g);
  } else {
    // pieces of a whole workgroup, one after the other
    const int64_t total = static_cast<int64_t>(g.w) * a.vpc;
    const int64_t base = static_cast<int64_t>(sub) * (kVec * kSmallTpb);
    if (base >= total) return;
    split_pieces<kVec, kSmallTpb, kSmallTpb, kOopNt>(a.src + static_cast<int64_t>(span) * a.src_span_vecs,
                                                     a.dst + static_cast<int64_t>(span) * a.dst_span_vecs, base, total,
                                                     static_cast<int64_t>(g.pad_out) * a.vpc,
                                                     static_cast<int64_t>(g.pad_out - g.pad_in) * a.vpc);
  }
}

__global__ __launch_bounds__(kThreads) void posmask_kernel(int64_t* pos, uint8_t* mask,
                                                           const int32_t* pad_out, const int32_t* w_new,
                                                           int32_t k, int64_t pm_cap, uint32_t col_blocks,
                                                           uint32_t* dev_status) {
  posmask_block<kThreads>(blockIdx.x, pos, mask, pad_out, w_new, k, pm_cap, col_blocks, dev_status);
}

__global__ __launch_bounds__(kThreads) void tokens_kernel(RealignArgs a) {
  token_block<kThreads>(a, blockIdx.x);
}

__global__ __launch_bounds__(kThreads) void zero_kernel(uint4* p16, int64_t n16, uint8_t* tail, int64_t ntail) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i < n16) p16[i] = make_uint4(0u, 0u, 0u, 0u);
  if (i < ntail) tail[i] = 0;
}


}  // namespace

int64_t max_launch_items() {
  int64_t max_items = 0xFFFFFFFFLL;
  if (const char* env = std::getenv("SPECDEC_MAX_LAUNCH_ITEMS")) {
    const long long v = std::atoll(env);
    if (v > 0 && v < max_items) max_items = v;
  }
  return max_items;
}

int64_t verify_chunk_elems(int64_t rows, int64_t V) {
  // about SPECDEC_VERIFY_TARGET workgroups in total, each scanning
  // SPECDEC_VERIFY_MIN_CHUNK..SPECDEC_VERIFY_MAX_CHUNK elements (a multiple
  // of the minimum), and at most kMaxVerifyChunks workgroups per row
  constexpr int64_t kTarget = SPECDEC_VERIFY_TARGET, kMin = SPECDEC_VERIFY_MIN_CHUNK, kMax = SPECDEC_VERIFY_MAX_CHUNK;
  static_assert(kMin % 8 == 0 && kMax % kMin == 0, "chunks are whole 16-byte vectors");
  const int64_t per = (rows * V + kTarget - 1) / kTarget;
  int64_t c = ((per + kMin - 1) / kMin) * kMin;
  if (c < kMin) c = kMin;
  if (c > kMax) c = kMax;
  int64_t min_c = (V + kMaxVerifyChunks - 1) / kMaxVerifyChunks;
  min_c = ((min_c + 7) / 8) * 8;
  if (c < min_c) c = min_c;
  if (c > V) c = V;
  return c;
}

int64_t verify_chunks(int64_t rows, int64_t V) {
  const int64_t c = verify_chunk_elems(rows, V);
  return (V + c - 1) / c;
}

static VerifyArgs verify_args(const VerifyLaunch& p) {
  VerifyArgs a;
  a.logits = static_cast<const char*>(p.logits);
  a.draft = p.draft;
  a.pad_in = p.pad_in;
  a.B = p.B;
  a.k = p.k;
  a.V = p.V;
  a.W_in = p.W_in;
  a.tokens = p.tokens;
  a.n_acc = p.n_acc;
  a.bonus = p.bonus;
  a.pad_out = p.pad_out;
  a.w_new = p.w_new;
  a.partial = reinterpret_cast<unsigned long long*>(static_cast<char*>(p.workspace) + kWsHeaderBytes);
  a.dev_status = p.dev_status;
  const int64_t rows = static_cast<int64_t>(p.B) * (p.k + 1);
  a.chunk_elems = verify_chunk_elems(rows, p.V);
  a.chunks = static_cast<int32_t>((p.V + a.chunk_elems - 1) / a.chunk_elems);
  a.order = p.write_order ? reinterpret_cast<int32_t*>(static_cast<char*>(p.workspace) + order_offset(p.B, p.k, p.V))
                          : nullptr;
  a.order_group = reinterpret_cast<int32_t*>(static_cast<char*>(p.workspace) + kOrderGroupOffset);
  a.order_by_row = p.order_by_row;
  a.order_even_len = p.order_even_len;
  return a;
}

int64_t order_offset(int64_t B, int64_t k, int64_t V) {
  const int64_t rows = B * (k + 1);
  return static_cast<int64_t>(kWsHeaderBytes) + ((rows * verify_chunks(rows, V) * 8 + 15) / 16) * 16;
}

int64_t order_bytes(int64_t B) { return 16 * B; }

hipError_t launch_verify_scan(const VerifyLaunch& p, hipStream_t stream) {
  const VerifyArgs a = verify_args(p);
  const int64_t blocks = static_cast<int64_t>(p.B) * (p.k + 1) * a.chunks;
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kThreads);
  switch (p.dtype) {
    case 0: hipLaunchKernelGGL(verify_partial_kernel<0>, grid, block, 0, stream, a); break;
    case 1: hipLaunchKernelGGL(verify_partial_kernel<1>, grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL(verify_partial_kernel<2>, grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_verify_finalize(const VerifyLaunch& p, hipStream_t stream) {
  const VerifyArgs a = verify_args(p);
  hipLaunchKernelGGL(verify_finalize_kernel, dim3(1), dim3(kFinalizeThreads), 0, stream, a);
  return hipGetLastError();
}

bool verify_fused_fits(int64_t B, int64_t k, int64_t V, int dtype) {
  const int64_t eb = dtype == 0 ? 4 : 2;
  return B >= 1 && B * (k + 1) <= kMaxFusedVerifyRows && V * eb <= kMaxFusedVerifyRowBytes;
}

hipError_t launch_verify_fused(const VerifyLaunch& p, uint32_t* counts, hipStream_t stream) {
  FusedVerifyArgs f;
  f.v = verify_args(p);
  // the counts first (cleared after the call), the lengths above every count
  // a batch of any size uses, so that no call's lengths land in another's counts
  f.batch_count = counts;
  f.seq_count = counts + 1;
  f.lens = reinterpret_cast<int32_t*>(counts + 1 + kMaxFusedVerifyRows);
  const dim3 grid(static_cast<uint32_t>(static_cast<int64_t>(p.B) * (p.k + 1))), block(kFusedThreads);
  switch (p.dtype) {
    case 0: hipLaunchKernelGGL(verify_fused_kernel<0>, grid, block, 0, stream, f); break;
    case 1: hipLaunchKernelGGL(verify_fused_kernel<1>, grid, block, 0, stream, f); break;
    default: hipLaunchKernelGGL(verify_fused_kernel<2>, grid, block, 0, stream, f); break;
  }
  return hipGetLastError();
}

hipError_t launch_verify(const VerifyLaunch& p, hipStream_t stream) {
  const hipError_t e = launch_verify_scan(p, stream);
  if (e != hipSuccess) return e;
  return launch_verify_finalize(p, stream);
}

static void fill_token_args(RealignArgs& a, const RealignLaunch& p, int tpb) {
  a.s_in = p.s_in;
  a.s_out = p.s_out;
  a.s_in_stride = p.s_in_stride;
  a.s_out_stride = p.s_out_stride;
  a.tokens = p.tokens;
  a.pad_id = p.pad_id;
  a.tok_col_blocks = 0;
  a.clear_words = p.clear_words;
  a.clear_count = p.clear_words ? p.clear_count : 0u;
  if (p.s_in) {
    const int64_t width = static_cast<int64_t>(p.W_in) + 1;   // L' + 1 <= W_in + 1
    a.tok_col_blocks = p.s_in == p.s_out ? 1u : static_cast<uint32_t>((width + 4 * tpb - 1) / (4 * tpb));
  }
}

// The in-place plan, by the longest span a row can have and the number of
// spans (the host does not know the rows' lengths).  us, one box a line; walk 32
// / walk 1: the walk with the order table, 32 rows at a time in 2 length
// classes / a row at a time in 7, so that the long rows of all layers come
// first; chunks: of 64 KB up to 1536 spans, else of 128 KB, at most two
// workgroups a CU (through LDS they do not use: more in flight spreads the
// DRAM traffic and costs up to 15%) unless noted.
//   steps, spans of one chunk: to 22 KB, walk 32 237, chunks 77 (no limit to two); to
//     60 KB, ragged 580 / 138 (no limit), even 288 / 243; 5..124 KB, ragged 605 /
//     358, even ones of 77..124 KB 451 / 466, 65536 of 100..128 KB 1987 / 2105: one
//     workgroup a CU takes 441 and 1978, but 476 for the ragged ones
//   steps, longer, walk 32 / walk 1 / chunks, ragged (log-uniform from 16 KB) and
//     even ones to 1 MB: 256 spans 15.7 / 13.7 / 19.1 and 71 / 70 / 71; 512 50 / 40 / 61
//     and 116 / 128 / 118; 1024 112 / 88 / 114 and 270 / 287 / 273; 2048 249 / 165 / 203
//     and 521 / 538 / 535; 4096 436 / 285 / 333 and 1034 / 1044 / 1020; 8192 586 / 556 /
//     640 and 2032 / 2065 / 2050
//   128 spans, the longer of two rows staying: the other one of 1 MB 48 / 48 / 37, of 0.1
//     MB (1 MB possible) 24 / 24 / 28, both possible to 0.3 MB 23 / 23 / 20 and 15 /
//     14 / 17
// One row at a time, neighbouring workgroups move distant spans; 32 at a time,
// the last layers' long rows start last.  So the walk's table says which,
// where the spans are at most 8192 (beyond, there are enough to hide the last
// round: 16384 to 0.9 MB 790 / 819 / 855): 32 where at least five rows move and
// their lengths are long and within a quarter of each other (shorter even
// ones, 4480 of 320 KB: 288 / 253).  Chunks are for 128 spans at most, half the
// CUs' number.  Without a table (`ordered` false: a realignment alone, a
// sampled step) the walk orders up to 64 rows itself; realignments, cache's
// order / chunks / so: 256 spans 7.7 / 12.9 / 7.1 and 64 / 65 / 63; 512 44 / 54 / 33 and
// 109 / 111 / 109; 1024 106 / 124 / 80 and 266 / 268 / 266 (even ones keep the
// cache's order up to 2048); 4096 572 / 282 / 285 and 1064 / 1080 / 1036; 8192 679 / 554
// / 558 and 2103 / 2176 / 2063.  More rows than that
// go by chunks.  A single row stays where it is in a decoding loop (its
// padding is 0), so one launch that finds nothing to do is the better one
// (13.3 us a step, 16.3 with the strips).
InplacePlan inplace_plan(int64_t L, int64_t B, int64_t H, int64_t D, int64_t W_in, bool ordered) {
  InplacePlan plan;
  const int64_t longest = W_in * (D / 8);   // a row holds at most W_in columns
  const int64_t nspans = L * 2 * B * H;
  if (longest <= 16 * 256) {
    plan.vec = longest <= 4 * 256 ? 4 : (longest <= 8 * 256 ? 8 : 16);
    plan.tpb = longest <= 4 * 64 ? 64 : 256;
    plan.chunks = 1;
    return plan;
  }
  const bool few = nspans <= kCus / 2 && longest >= 32 * 1024;
  if (longest > 32 * 256 && (B == 1 || nspans > 8192 || (!few && (ordered || B <= 64)))) {   // the walk
    plan.table = ordered && B > 1;
    plan.sorted = !plan.table && B > 1 && nspans <= 8192;
    plan.even_len = static_cast<int>(32 * 1024 / (D / 8));
    plan.by_row = nspans > 8192 ? 0 : nspans > 384 ? 1 : 2;
    return plan;
  }
  InplacePlan walk = plan;
  walk.table = ordered;
  plan.vec = longest > 32 * 256 && nspans <= 1536 ? 16 : 32;
  plan.tpb = 256;
  plan.chunks = (longest + plan.vec * plan.tpb - 1) / (plan.vec * plan.tpb);
  plan.lds = 64 * 1024;
  return nspans * plan.chunks <= 0x7FFFFFFF ? plan : walk;
}

template <int kVec, int kTpb, bool kMany>
static void launch_chunks(const RealignArgs& a, dim3 grid, int lds, hipStream_t stream) {
  hipLaunchKernelGGL((realign_chunk_kernel<kVec, kTpb, kInNt, kMany>), grid, dim3(kTpb), lds, stream, a);
}

hipError_t launch_realign(const RealignLaunch& p, hipStream_t stream) {
  RealignArgs a{};
  a.src = static_cast<const u32x4*>(p.src);
  a.dst = static_cast<u32x4*>(p.dst);
  a.vpc = p.D / 8;
  a.src_span_vecs = p.src_cap * a.vpc;
  a.dst_span_vecs = p.dst_cap * a.vpc;
  a.B = p.B;
  a.H = p.H;
  a.k = p.k;
  a.W_in = p.W_in;
  a.pad_in = p.pad_in;
  a.n_acc = p.n_acc;
  a.w_new = p.w_new;
  a.dev_status = p.dev_status;
  const int64_t nspans = static_cast<int64_t>(p.L) * 2 * p.B * p.H;
  a.nspans = static_cast<uint32_t>(nspans);
  a.pos = p.pos;
  a.mask = p.mask;
  a.pad_out = p.pad_out;
  a.pm_cap = p.pm_cap;
  const InplacePlan& plan = p.plan;
  if (p.in_place && plan.table != (p.order != nullptr)) return hipErrorInvalidValue;   // a table unread, or missing
  a.order = p.in_place ? p.order : nullptr;
  a.order_group = p.order_group;
  a.row_group = plan.by_row == 0 ? 32u : plan.by_row == 2 ? 1u : plan.table ? 0u : 32u;
  a.len_half = kInTpb * kInVec / 2 / a.vpc;
  a.len_quarter = kInTpb * kInVec / 4 / a.vpc;
  a.span_rows = static_cast<uint32_t>(static_cast<int64_t>(p.L) * 2 * p.H);
  const bool by_chunk = p.in_place && plan.chunks > 0;
  const int tpb = by_chunk ? plan.tpb : (p.in_place ? kInTpb : kOopTpb);
  int64_t pm_blocks = 0;
  a.pm_col_blocks = 1;
  if (p.pos) {
    const int64_t bound = static_cast<int64_t>(p.W_in) + p.k + 1;
    a.pm_col_blocks = static_cast<uint32_t>((bound + 4 * tpb - 1) / (4 * tpb));
    pm_blocks = static_cast<int64_t>(a.pm_col_blocks) * p.B;
  }
  fill_token_args(a, p, tpb);
  const int64_t tok_blocks = static_cast<int64_t>(a.tok_col_blocks) * p.B;
  a.tok_blocks = static_cast<uint32_t>(tok_blocks);
  const int64_t extra = pm_blocks + tok_blocks + (a.clear_words ? 1 : 0);
  const int64_t row_vecs = static_cast<int64_t>(p.W_in) * a.vpc;   // a span's output is at most this long
  const int split = split_distance(row_vecs, true);
  a.misaligned = !p.in_place && !split_spans_aligned(kOopVec, split, p.dst, a.dst_span_vecs);
  const int64_t chunks = by_chunk ? plan.chunks : p.in_place ? 1 : split_blocks(kOopVec, kOopTpb, split, row_vecs,
                                                                                      a.misaligned != 0);
  a.chunks = static_cast<uint32_t>(chunks);
  // one dispatch holds fewer than 2^32 work-items: split the spans over
  // several launches when the cache is larger than that
  const int64_t max_blocks = (max_launch_items() / tpb) - extra;
  if (by_chunk) {
    // (the chunks of a span may fall into several launches)
    if (max_blocks < 1) return hipErrorInvalidConfiguration;
    const int64_t slots = nspans * chunks;
    a.slots = static_cast<uint32_t>(slots);
    a.extra_blocks = static_cast<uint32_t>(extra);
    a.pm_blocks = static_cast<uint32_t>(pm_blocks);
    for (int64_t g = 0; g < slots || a.extra_blocks > 0;) {
      const int64_t n = slots - g < max_blocks ? slots - g : max_blocks;
      a.span_base = static_cast<uint32_t>(g);
      const dim3 grid(static_cast<uint32_t>(n + a.extra_blocks));
      if (chunks > 1) {
        if (plan.vec == 16) launch_chunks<16, 256, true>(a, grid, plan.lds, stream);
        else launch_chunks<32, 256, true>(a, grid, plan.lds, stream);
      } else if (plan.tpb == 64) {
        launch_chunks<4, 64, false>(a, grid, plan.lds, stream);
      } else {
        switch (plan.vec) {
          case 4: launch_chunks<4, 256, false>(a, grid, plan.lds, stream); break;
          case 8: launch_chunks<8, 256, false>(a, grid, plan.lds, stream); break;
          case 16: launch_chunks<16, 256, false>(a, grid, plan.lds, stream); break;
          default: launch_chunks<32, 256, false>(a, grid, plan.lds, stream); break;
        }
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      g += n;
      a.extra_blocks = 0;
    }
    if (chunks > 1)
      for (int64_t s0 = 0; s0 < nspans;) {
        const int64_t most = max_launch_items() / kInTpb;
        const int64_t n = nspans - s0 < most ? nspans - s0 : most;
        a.span_base = static_cast<uint32_t>(s0);
        const dim3 grid(static_cast<uint32_t>(n)), block(kInTpb);
        const int most_vecs = plan.vec * plan.tpb;
        if (nspans <= kCus)
          hipLaunchKernelGGL((realign_strips_kernel<kInTpb, kInNt, true>), grid, block, 0, stream, a, most_vecs);
        else
          hipLaunchKernelGGL((realign_strips_kernel<kInTpb, kInNt, false>), grid, block, 0, stream, a, most_vecs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        s0 += n;
      }
    return hipSuccess;
  }
  const int64_t spans_per_launch = max_blocks / chunks;
  if (spans_per_launch < 1) return hipErrorInvalidConfiguration;
  const dim3 block(tpb);
  for (int64_t s0 = 0; s0 < nspans || (nspans == 0 && s0 == 0); s0 += spans_per_launch) {
    const int64_t ns = nspans - s0 < spans_per_launch ? nspans - s0 : spans_per_launch;
    const bool first = s0 == 0;
    a.span_base = static_cast<uint32_t>(s0);
    a.realign_blocks = static_cast<uint32_t>(ns * chunks);
    a.extra_blocks = first ? static_cast<uint32_t>(extra) : 0u;
    a.pm_blocks = first ? static_cast<uint32_t>(pm_blocks) : 0u;
    const int64_t blocks = ns * chunks + (first ? extra : 0);
    if (blocks == 0) break;
    const dim3 grid(static_cast<uint32_t>(blocks));
    if (p.in_place && plan.sorted)
      hipLaunchKernelGGL((realign_inplace_kernel<kInVec, kInTpb, kInNt, true>), grid, block, 0, stream, a);
    else if (p.in_place)
      hipLaunchKernelGGL((realign_inplace_kernel<kInVec, kInTpb, kInNt, false>), grid, block, 0, stream, a);
    else if (split == 64)
      hipLaunchKernelGGL((realign_oop_kernel<kOopVec, kOopTpb, 64, kOopNt>), grid, block, 0, stream, a);
    else if (split == 512)
      hipLaunchKernelGGL((realign_oop_kernel<kOopVec, kOopTpb, 512, kOopNt>), grid, block, 0, stream, a);
    else
      hipLaunchKernelGGL((realign_oop_kernel<kOopVec, kOopTpb, 1024, kOopNt>), grid, block, 0, stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (nspans == 0) break;
  }
  return hipSuccess;
}

// Threads to a logit row in the small step's merge, or 0 where the step is
// not a small one.
static int small_step_lanes(const VerifyLaunch& v) {
  const int64_t rows = static_cast<int64_t>(v.B) * (v.k + 1);
  if (rows > kSmallRows || rows < 1) return 0;
  int lanes = 1;
  while (lanes < 64 && rows * lanes * 2 <= kSmallTpb) lanes *= 2;
  return lanes;
}

// Vectors a thread of the merged launch moves, and workgroups per span.
static void small_step_share(const RealignLaunch& p, int* vec, int64_t* blocks) {
  const int64_t longest = static_cast<int64_t>(p.W_in) * (p.D / 8);
  if (p.in_place) {
    *vec = longest <= 4 * kSmallTpb ? 4 : 16;
    *blocks = 1;
  } else {
    *vec = 2;
    *blocks = (longest + 2 * kSmallTpb - 1) / (2 * kSmallTpb);
  }
}

bool small_step_fits(const VerifyLaunch& v, const RealignLaunch& p) {
  const int64_t nspans = static_cast<int64_t>(p.L) * 2 * p.B * p.H;
  if (!small_step_lanes(v) || nspans < 1 || p.clear_words || !p.pos) return false;
  const int64_t longest = static_cast<int64_t>(p.W_in) * (p.D / 8);
  if (p.in_place && longest > 16 * kSmallTpb) return false;
  int vec;
  int64_t blocks;
  small_step_share(p, &vec, &blocks);
  blocks *= nspans;
  const int64_t rows = static_cast<int64_t>(v.B) * (v.k + 1);
  const int64_t merged = rows * verify_chunks(rows, v.V) * 8;   // bytes each workgroup merges
  const int64_t cols = static_cast<int64_t>(p.W_in) + p.k + 1;
  const int64_t extra = 2 * p.B * ((cols + 4 * kSmallTpb - 1) / (4 * kSmallTpb));
  return blocks <= kSmallMaxBlocks && blocks * merged <= (p.in_place ? kSmallMaxMergedInPlace : kSmallMaxMergedOop) && (blocks + extra) * kSmallTpb <= max_launch_items();
}

hipError_t launch_small_step(const VerifyLaunch& v, const RealignLaunch& p, hipStream_t stream) {
  RealignArgs a{};
  a.src = static_cast<const u32x4*>(p.src);
  a.dst = static_cast<u32x4*>(p.dst);
  a.vpc = p.D / 8;
  a.src_span_vecs = p.src_cap * a.vpc;
  a.dst_span_vecs = p.dst_cap * a.vpc;
  a.B = p.B;
  a.H = p.H;
  a.k = p.k;
  a.W_in = p.W_in;
  a.dev_status = p.dev_status;
  a.pos = p.pos;
  a.mask = p.mask;
  a.pm_cap = p.pm_cap;
  const int64_t cols = static_cast<int64_t>(p.W_in) + p.k + 1;
  a.pm_col_blocks = static_cast<uint32_t>((cols + 4 * kSmallTpb - 1) / (4 * kSmallTpb));
  a.pm_blocks = a.pm_col_blocks * static_cast<uint32_t>(p.B);
  fill_token_args(a, p, kSmallTpb);
  a.tok_blocks = a.tok_col_blocks * static_cast<uint32_t>(p.B);
  int vec;
  int64_t blocks;
  small_step_share(p, &vec, &blocks);
  a.chunks = static_cast<uint32_t>(blocks);
  a.slots = static_cast<uint32_t>(static_cast<int64_t>(p.L) * 2 * p.B * p.H * blocks);
  const dim3 grid(a.slots + a.pm_blocks + a.tok_blocks), block(kSmallTpb);
  const VerifyArgs va = verify_args(v);
  const int lanes = small_step_lanes(v);
  if (!p.in_place) hipLaunchKernelGGL((small_step_kernel<false, 2>), grid, block, 0, stream, va, a, lanes);
  else if (vec == 4) hipLaunchKernelGGL((small_step_kernel<true, 4>), grid, block, 0, stream, va, a, lanes);
  else hipLaunchKernelGGL((small_step_kernel<true, 16>), grid, block, 0, stream, va, a, lanes);
  return hipGetLastError();
}

hipError_t launch_tokens(const RealignLaunch& p, hipStream_t stream) {
  RealignArgs a{};
  a.B = p.B;
  a.k = p.k;
  a.W_in = p.W_in;
  a.pad_in = p.pad_in;
  a.n_acc = p.n_acc;
  a.w_new = p.w_new;
  a.dev_status = p.dev_status;
  fill_token_args(a, p, kThreads);
  const int64_t blocks = static_cast<int64_t>(a.tok_col_blocks) * p.B;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(tokens_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}


hipError_t launch_posmask(const PosmaskLaunch& p, hipStream_t stream) {
  const int64_t col_blocks = (p.col_bound + kPmColsPerBlock - 1) / kPmColsPerBlock;
  const int64_t blocks = col_blocks * p.B;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(posmask_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(kThreads), 0, stream, p.pos,
                     p.mask, p.pad_out, p.w_new, p.k, p.pm_cap, static_cast<uint32_t>(col_blocks), p.dev_status);
  return hipGetLastError();
}

hipError_t launch_zero(void* ptr, size_t bytes, hipStream_t stream) {
  const uintptr_t base = reinterpret_cast<uintptr_t>(ptr);
  // 16-byte stores over the aligned body, byte stores for the rest (the
  // workspace is 8-byte aligned; the rare unaligned prefix is byte-cleared)
  if ((base & 15u) != 0u || bytes < 16) {
    const int64_t n = static_cast<int64_t>(bytes);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3(static_cast<uint32_t>((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       stream, static_cast<uint4*>(nullptr), int64_t{0}, static_cast<uint8_t*>(ptr), n);
    return hipGetLastError();
  }
  const int64_t n16 = static_cast<int64_t>(bytes / 16);
  const int64_t ntail = static_cast<int64_t>(bytes % 16);
  const int64_t n = n16 > ntail ? n16 : ntail;
  hipLaunchKernelGGL(zero_kernel, dim3(static_cast<uint32_t>((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     stream, static_cast<uint4*>(ptr), n16, static_cast<uint8_t*>(ptr) + n16 * 16, ntail);
  return hipGetLastError();
}

}  // namespace specdec
