// Paged attention on gfx950 matrix cores for every layout except bf16 with head size 128: bf16 of any head size
// that is a multiple of 8 and fp32 of any that is a multiple of 4, up to 256.  The decode kernel here also serves
// small batches of that layout (small_decode), and decode_short_kernel those whose contexts it takes whole (decode_short) or cuts itself (decode_sliced).
//
// Eq. 2 of Section 2.1 over the paged cache, as the kernels for (bf16, 128) evaluate it, with the arithmetic of
// the plain kernels: scores, weights and sums are fp32.
//   scores  S^T[key][row] = K . Q^T      fp32: v_mfma_f32_16x16x4_f32;  bf16: v_mfma_f32_16x16x32_bf16
//   values  O^T[d][row]  += V^T . P^T    fp32: v_mfma_f32_16x16x4_f32;  bf16: v_mfma_f32_16x16x16_bf16, three times: the
//           weight as a bf16 number, the bf16 number nearest to what that left over, and again: 24 bits, as fp32 holds
//           (small (bf16, 128) decode batches: see Block)
// A cache block is in operand layout already (see attn_decode_mfma.hip): lane (col, quad) reads the 16-byte units
// (4 j + quad, token col) of K, whose elements are the K dimension of a step (the order inside a step does not
// matter as long as Q has the same), and row 16 dt + col, tokens 4 quad .. + 3 of V.  No LDS staging, no
// transposition; the scores' accumulator layout is the weights' operand layout.  Head sizes that do not fill the
// last step read zeros there: the loads go through a descriptor that ends with the block.
//
// Rows that share a K/V head share its loads: the 16 columns of a product are the query heads of the group
// (decode), or (position, query head of the group) pairs of a prompt (prefill), position-major.
//
// What bounds them: such batches are small (tens of MB of K/V at most), so a step is latency: launches, the chain
// length -> block ids -> blocks, and the walk of the blocks.  Hence decode is one
// launch (instead of three): eight wavefronts (four for large heads and for batches of more than one workgroup per CU) per
// (sequence, K/V head) and slice of the context, slices as short as a merge allows, the step's append inside.
// Measured beside the plain kernels (one wavefront per query row, a scalar product per lane): a prompt batch of 4 x
// 50..600 tokens and 8 decode steps, bf16, head size 64, 32/8 heads: 398 -> 65 us (prefill kernel 243 -> 11 us, a
// decode step's kernels 21.8 -> 5.6 us); 4 x 37..700 tokens in fp32, 4/2 heads: 195 -> 68 us (55 -> 8 us, 19.1 -> 7.1 us).
// Not gained: a prompt of 8 tokens or fewer with nothing cached (a graph of such calls: 0.2 to 0.9 us more than the plain
// kernel's 3 to 8); with 40 to 100 tokens cached, which the host cannot see, the plain kernel takes up to six times as long.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "decode_slices.h"

namespace eco {

constexpr int kRsrc32 = 0x00020000;  // buffer descriptor: untyped 32-bit data, no swizzle, no stride
constexpr int kNonTemporal = 2;      // cache policy: do not keep the lines
constexpr float kRaise = 8.f;        // the exponent offset is raised when a score exceeds it by more (log2 units)

// Operands of one cache block for head sizes up to 32 KS, and the two products.  AUX: cache policy of the loads.  FULL:
// weights have all bits of fp32; false is for (bf16, 128) alone, whose other kernels hold weights in 8 bits and flush those
// below 2^-126: two parts (16 bits) and the bare exponent instruction there (one sequence of 777 tokens, 16 layers: 148 us,
// with three parts and exp2f 157, when the launch took 8 us).
template <typename E, int KS, int AUX = 0, bool FULL = true>
struct Block {
  static constexpr bool kF32 = std::is_same<E, float>::value;
  static constexpr int X = Elem<E>::X;
  static constexpr int NK = kF32 ? 2 * KS : KS;  // 16-byte loads of K (and of a query row) per lane
  static constexpr int NV = 2 * KS;              // 16-row tiles of V^T
  typedef typename std::conditional<kF32, f32x4, s16x4>::type VFrag;
  u32x4 k[NK];
  VFrag v[NV];

  // `bytes`: size of one (block, head) piece of the pool
  __device__ __forceinline__ void load(const char* kbase, const char* vbase, int bytes, int lane, int col, int quad) {
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kbase), 0, bytes, kRsrc32);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vbase), 0, bytes, kRsrc32);
#pragma unroll
    for (int j = 0; j < NK; ++j)
      k[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, lane * 16 + j * 1024, 0, AUX));
#pragma unroll
    for (int dt = 0; dt < NV; ++dt) {
      if constexpr (kF32)
        v[dt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, col * 64 + quad * 16 + dt * 1024, 0, AUX));
      else
        v[dt] = __builtin_bit_cast(s16x4, __builtin_amdgcn_raw_buffer_load_b64(rv, col * 32 + quad * 8 + dt * 512, 0, AUX));
    }
  }
  // slots >= n hold no token: their V entries (stale bits, possibly NaN) must not meet their zero weights
  __device__ __forceinline__ void clear_tail(int n, int quad) {
#pragma unroll
    for (int dt = 0; dt < NV; ++dt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * quad + e >= n) v[dt][e] = 0;
  }
  // the token in `slot` comes from a K row and a V row (D elements each) instead of the cache
  __device__ __forceinline__ void put_token(const E* krow, const E* vrow, int slot, int D, int col, int quad) {
    if (col == slot) {
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const int d = (4 * j + quad) * X;
        if (d < D) k[j] = *reinterpret_cast<const u32x4*>(krow + d);
      }
    }
    if (quad == (slot >> 2)) {
#pragma unroll
      for (int dt = 0; dt < NV; ++dt) {
        const int d = dt * 16 + col;
        if (d < D) {
          const E x = vrow[d];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (e == (slot & 3)) {
              if constexpr (kF32) v[dt][e] = x;
              else v[dt][e] = (short)x;
            }
        }
      }
    }
  }
  // S^T[key 4 quad + i][row col]
  __device__ __forceinline__ f32x4 scores(const u32x4 (&q)[NK]) const {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kF32) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};  // (two chains: a dependent matrix instruction cannot issue back to back)
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const f32x4 a = __builtin_bit_cast(f32x4, k[j]), b = __builtin_bit_cast(f32x4, q[j]);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], s, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], t, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], s, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], t, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] += t[i];
    } else {
#pragma unroll
      for (int j = 0; j < NK; ++j)
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[j]), __builtin_bit_cast(bf16x8, q[j]), s, 0, 0, 0);
    }
    return s;
  }
  // O^T[d][row] += V^T P^T for the weights p of keys 4 quad .. + 3
  __device__ __forceinline__ void values(const f32x4& p, f32x4 (&acc)[NV]) const {
    if constexpr (kF32) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int dt = 0; dt < NV; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[dt][e], p[e], acc[dt], 0, 0, 0);
    } else {
      f32x4 left = p;
#pragma unroll
      for (int n = 0; n < (FULL ? 3 : 2); ++n) {
        const bf16x4 part = __builtin_convertvector(left, bf16x4);
        left -= __builtin_convertvector(part, f32x4);
        const s16x4 bits = __builtin_bit_cast(s16x4, part);
#pragma unroll
        for (int dt = 0; dt < NV; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[dt], bits, acc[dt], 0, 0, 0);
      }
    }
  }
};

// v / l to the last bit, for l >= 1: one reciprocal, and each quotient put right by its remainder (four divisions of their own are 40 instructions, this 26).
__device__ __forceinline__ f32x4 divided(const f32x4& v, float l) {
  const float inv = 1.f / l;
  f32x4 q;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float near = v[e] * inv;
    q[e] = __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-near, l, v[e]), inv, near), l, v[e]);  // (infinities, NaNs and zeros as a division has them)
  }
  return q;
}
__device__ __forceinline__ void store4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store4(uint16_t* p, const f32x4& v) {
  *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

// Online softmax of one row (a column of the products; its keys are spread over the four 16-lane groups).
// `m`: exponent offset, -inf until the row has seen a key; `l`: this lane's share of the sum of weights.  The
// offset is raised only when a score exceeds it by more than 2^kRaise, so the rescaling leaves the loop; weights
// are fp32, which holds 2^8 as exactly as 1.
template <bool FULL, int NV>
__device__ __forceinline__ f32x4 softmax_step(const f32x4& s, float& m, float& l, f32x4 (&acc)[NV]) {
  float bm = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  if (__any(bm > m + kRaise)) {
    bm = fmaxf(bm, __shfl_xor(bm, 16));
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    const float m_new = bm > m + kRaise ? bm : m;
    const float alpha = m == -INFINITY ? 0.f : exp2f(m - m_new);
    l *= alpha;
#pragma unroll
    for (int dt = 0; dt < NV; ++dt) acc[dt] *= alpha;
    m = m_new;
  }
  const float mu = m == -INFINITY ? 0.f : m;  // (a row all of whose keys so far are masked)
  f32x4 p;
#pragma unroll
  for (int i = 0; i < 4; ++i) p[i] = s[i] - mu;
  // The bare instruction flushes weights below 2^-126, which large values can still make count: where there are any (or masked keys), exp2f.
  if (FULL && __any(fminf(fminf(p[0], p[1]), fminf(p[2], p[3])) < -126.f)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = exp2f(p[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(p[i]);
  }
  l += (p[0] + p[1]) + (p[2] + p[3]);
  return p;
}

// Values all lanes have, as scalars, and a lane's own, that are known from here on only: what follows from them is worked out behind this
// point.  Otherwise it may stand in front of the branch that leads here, or (a scalar base and the lanes' offsets) be added up per lane and access.
template <typename T>
__device__ __forceinline__ T* scalar_here(T* p) {
  const uint64_t u = (uint64_t)p;
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  asm volatile("" : "+s"(lo), "+s"(hi));
  return (T*)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int scalar_here(int x) {
  int y = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(y));
  return y;
}
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// One row over keys [t0, t1), one wavefront, key after key: what a row falls back to when its sums are not finite
// although its weights are.  Either a V element that is infinite or not a number met the zero weight of a
// masked key, or the zero remainder of a bf16 weight, in the products above; here it meets only the rows that see
// it.  Or values within a factor of 2^kRaise of the largest fp32 overflowed under weights above 1; here weights are
// taken relative to the largest score so far and do not exceed 1.  Lane owns elements lane + 64 r.
__device__ __forceinline__ bool not_finite(float x) { return !(fabsf(x) < INFINITY); }
template <typename E>
__device__ __forceinline__ void attend_row(const E* __restrict__ qrow, const E* __restrict__ k_cache, const E* __restrict__ v_cache,
                                        const int32_t* __restrict__ bt_row, int g, int Hkv, int D, int t0, int t1, float scale_log2e,
                                        float& m, float& l, float (&o)[4]) {
  constexpr int X = Elem<E>::X;
  const int lane = here((int)threadIdx.x & 63);
  m = -INFINITY;
  l = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = 0.f;
  for (int t = t0; t < t1; ++t) {
    const int64_t blk = bt_row[t >> 4];
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int d = lane + 64 * r;
      if (d < D) s += Elem<E>::load(qrow + d) * Elem<E>::load(k_cache + k_index<X>(blk, g, t & 15, d, Hkv, D));
    }
    s = wave_sum(s) * scale_log2e;
    const float m_new = fmaxf(m, s), mu = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = m == -INFINITY ? 0.f : exp2f(m - mu), p = exp2f(s - mu);
    l = l * alpha + p;
    m = m_new;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int d = lane + 64 * r;
      if (d < D) o[r] = o[r] * alpha + p * Elem<E>::load(v_cache + v_index(blk, g, t & 15, d, Hkv, D));
    }
  }
}

// Partial states, from the workgroup of one slice to the one that merges them, within a launch and possibly between XCDs: past the
// caches that XCDs do not share, and word by word.  A word holds the complement of the value's bits and is zero while it holds none, so a reader
// sees by itself whether what it asked for has arrived, and nobody waits for a store to be acknowledged before it is announced.  (The one value
// whose complement is zero, a NaN, is stored as its neighbour.)  Who reads a state clears it: the words are zero between launches.
// That is for a few states of short slices.  Long ones end at very different times, and many take long to clear: those lie elsewhere, and who has stored his, and has had the
// stores acknowledged, is counted; the last one finds all of them and leaves the words as they are.  (Clearing is a store of one CU's for each state it reads: us per
// call with it, 8 on 1, 1 x 150000 tokens 36.5, 30.9 so; 16 on 1, 1 x 60000 32.7, 25.8.)  Nobody waits for such a slice, however long it takes rows again (see attend_row).
__device__ __forceinline__ uint32_t part_bits(float v) { return max(~__float_as_uint(v), 1u); }
__device__ __forceinline__ float part_value(uint32_t bits) { return __uint_as_float(~bits); }
// (The instructions of relaxed atomics of agent scope, as buffer accesses: a scalar base and 32 bits of offset per lane, and nothing is read behind
// the range.)
constexpr int kAuxAgent = 16;  // sc1
__device__ __forceinline__ u32x4 part_bits(const f32x4& v) { return u32x4{part_bits(v[0]), part_bits(v[1]), part_bits(v[2]), part_bits(v[3])}; }
__device__ __forceinline__ void store_part(__amdgpu_buffer_rsrc_t r, int byte, const u32x2& w) { __builtin_amdgcn_raw_buffer_store_b64(w, r, byte, 0, kAuxAgent); }
__device__ __forceinline__ void store_part(__amdgpu_buffer_rsrc_t r, int byte, const u32x4& w) { __builtin_amdgcn_raw_buffer_store_b128(w, r, byte, 0, kAuxAgent); }
constexpr int part_words(int D) { return D + 4; }  // of a state: the unnormalised head vector, its maximum, its sum, and two that keep 16 bytes aligned
// A merging wavefront asks again at most so often (half a second).  The slices it waits for run already, wait for nothing themselves and are short: microseconds from their
// end, milliseconds where rows are taken again.  So it never gives up, but for calls that overlap on one workspace, which they may not: they end with NaN then.
constexpr int kMostPolls = 1 << 19;

// Over the two halves, or (N 4) the four 16-lane groups, of a wavefront, lane by lane.
template <int N, typename F>
__device__ __forceinline__ float of_groups(float v, F f) {
  if constexpr (N == 4) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  }
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int N>
__device__ __forceinline__ float max_of_groups(float v) {
  return of_groups<N>(v, [](float a, float b) { return fmaxf(a, b); });
}
template <int N>
__device__ __forceinline__ float sum_of_groups(float v) {
  return of_groups<N>(v, [](float a, float b) { return a + b; });
}

// Balanced slices: lane b holds the number of blocks of sequence b; every K/V head has `slots` workgroups.  Whole contexts,
// or slices of whole rounds of the W wavefronts, as short as all sequences' slices fit the workgroups and a merge stays short
// (least_slice).  Returns the slice in blocks; `end`: inclusive prefix sums of the sequences' numbers of slices, `n`.
// (A trial is one scan; with all lanes as candidates and a loop over the sequences, 16 of them took 0.3 us longer.)
__device__ __forceinline__ int balanced_slice_blocks(int nb, int Hkv, int slots, int W, int& n, int& end) {
  const int longest = lanes_max(nb), sum = __builtin_amdgcn_readlane(lanes_prefix_sum(nb), 63);
  int st = first_balanced_slice(longest, sum, Hkv, slots, W);
  for (;;) {
    n = balanced_slices_of(nb, st);
    end = lanes_prefix_sum(n);
    if (st >= longest || __builtin_amdgcn_readlane(end, 63) <= slots) return st;
    st = next_balanced_slice(st, W);
  }
}

// Which slice a workgroup of the decode kernel computes: slice `sp` (-1: none) of sequence b, L tokens in slices of `tokens`, `most`
// at most.
struct SliceOf {
  int b, sp, L, tokens, most;
};
template <bool BALANCED>
__device__ __forceinline__ SliceOf slice_of_workgroup(const int32_t* __restrict__ ctx_len, int B, int Hkv, int split_tokens, int W) {
  if constexpr (BALANCED) {
    const int x = blockIdx.y;
    const int lane = threadIdx.x & 63, len = lane < B ? ctx_len[lane] : 0, nb = (len + 15) >> 4;
    int n, end;
    const int st = balanced_slice_blocks(nb, Hkv, gridDim.y, W, n, end);
    if (x >= __builtin_amdgcn_readlane(end, 63)) return {0, -1, 0, 16, 1};
    const int b = __popcll(__ballot(end - n <= x)) - 1;  // (lanes behind B have no slices: their first is behind the last)
    return {b, x - __builtin_amdgcn_readlane(end - n, b), __builtin_amdgcn_readlane(len, b), st * 16, __builtin_amdgcn_readlane(n, b)};
  } else {
    // (the constant address space: a scalar load)
    return {(int)blockIdx.z, (int)blockIdx.x, ((const __attribute__((address_space(4))) int32_t*)(uintptr_t)ctx_len)[blockIdx.z], split_tokens, (int)gridDim.x};
  }
}

// A row's partial states, one wavefront:
//   M = max_k m_k;  l = sum_k l_k 2^(m_k - M);  o = sum_k acc_k 2^(m_k - M) / l,  in the order of the slices, whichever merges
// (the division is the caller's), with weights below the smallest normal number, which the bare exponent flushes: whole states weigh that little beside
// another one, and large values make them count (the bare instruction: 1 x 777 tokens, 40 on 8, 6.81 us a call, 6.89 so).  `first`: the state of slice 0, the next ones slice_bytes further on each; slice `own` (-1: none) is in M, total and o.
// The states of eight slices are asked for at once, those of the next eight while they are added up, and, unless they are COUNTED and there, all again until they have
// arrived: every slice has started, and none waits for another.  Each group of lanes takes every NG-th slice.  (Slices whose scores are all
// -inf weigh nothing: their m is -inf, their sums are zero.)  Lane l has elements 4 (l % LG) of every 128.
constexpr int lane_groups(int KS) { return KS <= 2 ? 4 : 2; }
template <int KS, bool FULL, bool COUNTED>
__device__ __forceinline__ void merge_slices(uint32_t* first, int slice_bytes, int row_bytes, int D, int n_split, int own_slice, float& M, float& total,
                                             f32x4 (&o)[(KS + 3) / 4]) {
  constexpr int NC = (KS + 3) / 4, NG = lane_groups(KS), LG = 64 / NG, kAtOnce = 8 / NG;  // (per group of lanes)
  const int lane = threadIdx.x & 63, grp = lane / LG, el = (lane % LG) * 4;
  slice_bytes = scalar_here(slice_bytes);
  float m2 = -INFINITY, l2 = 0.f;
  f32x4 o2[NC];
  int at_o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    o2[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    at_o[c] = (FULL ? min(el + 128 * c, D - 4) : el + 128 * c) * 4 + grp * slice_bytes;
  }
  const int at_ml = D * 4 + grp * slice_bytes;
  struct Group {
    u32x2 ml[kAtOnce];
    u32x4 o[kAtOnce][NC];
  };
  auto range = [&](int base) {  // of the slices from `base` on, up to eight
    const int more = min(n_split - base, NG * kAtOnce);
    return __builtin_amdgcn_make_buffer_rsrc(scalar_here(reinterpret_cast<char*>(first) + (int64_t)base * slice_bytes), 0,
                                             more > 0 ? (more - 1) * slice_bytes + row_bytes : 0, kRsrc32);
  };
  auto ask = [&](__amdgpu_buffer_rsrc_t from, Group& x) {  // (behind the last slice: out of range, zeros)
    asm volatile("" ::: "memory");  // (memory has changed: without this the loads of a poll are taken for the same as before, and its loop for none)
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      x.ml[j] = __builtin_amdgcn_raw_buffer_load_b64(from, at_ml + NG * j * slice_bytes, 0, kAuxAgent);
#pragma unroll
      for (int c = 0; c < NC; ++c) x.o[j][c] = __builtin_amdgcn_raw_buffer_load_b128(from, at_o[c] + NG * j * slice_bytes, 0, kAuxAgent);
    }
  };
  Group now, then;
  int polls = 0;
  __amdgpu_buffer_rsrc_t from = range(0);
  ask(from, now);
  for (int base = 0; base < n_split; base += NG * kAtOnce) {
    const int more = n_split - base - grp, own = own_slice - base - grp;  // (slice NG j of this group of lanes: there, if NG j < more, this workgroup's, if NG j = own)
    const __amdgpu_buffer_rsrc_t next = range(base + NG * kAtOnce);
    ask(next, then);
    auto missing = [&]() {
      bool any = false;
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        uint32_t least = min(now.ml[j][0], now.ml[j][1]);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) least = min(least, now.o[j][c][e]);
        any |= (least == 0) & (NG * j < more) & (NG * j != own);
      }
      return __any(any);
    };
    if (!COUNTED && missing()) {  // (apart from the first look, which then waits for these slices alone)
      asm volatile("" ::: "memory");
      do {
        // who waits for long keeps out of the others' way: 0.4 us between looks, at the sums alone
        for (bool wait = polls > 1; wait && polls < kMostPolls; ++polls) {
          __builtin_amdgcn_s_sleep(16);
          asm volatile("" ::: "memory");
          bool any = false;
#pragma unroll
          for (int j = 0; j < kAtOnce; ++j)
            any |= (__builtin_amdgcn_raw_buffer_load_b32(from, at_ml + 4 + NG * j * slice_bytes, 0, kAuxAgent) == 0) & (NG * j < more) & (NG * j != own);
          wait = __any(any);
        }
        ask(from, now);
      } while (missing() && ++polls < kMostPolls);
    }
    float m_new = m2, x[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {  // (behind the last slice: nothing, of no weight)
      x[j] = NG * j == own ? M : NG * j < more ? part_value(now.ml[j][0]) : -INFINITY;
      m_new = fmaxf(m_new, x[j]);
    }
#pragma unroll
    for (int j = 0; j < kAtOnce && !COUNTED; ++j) {  // (this workgroup's own words are zero already)
#pragma unroll
      for (int c = 0; c < NC; ++c) store_part(from, at_o[c] + NG * j * slice_bytes, u32x4{0u, 0u, 0u, 0u});
      store_part(from, at_ml + NG * j * slice_bytes, u32x2{0u, 0u});
    }
    const float mu = m_new == -INFINITY ? 0.f : m_new;
    if (base > 0) {
      const float old = m2 == -INFINITY ? 0.f : exp2f(m2 - mu);
      l2 *= old;
#pragma unroll
      for (int c = 0; c < NC; ++c) o2[c] *= old;
    }
    m2 = m_new;
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const float wk = exp2f(x[j] - mu);
      l2 += (NG * j == own ? total : NG * j < more ? part_value(now.ml[j][1]) : 0.f) * wk;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o2[c][e] += (NG * j == own ? o[c][e] : NG * j < more ? part_value(now.o[j][c][e]) : 0.f) * wk;
    }
    from = next;
    now = then;
  }
  M = max_of_groups<NG>(m2);
  const float mine_weighs = m2 == -INFINITY ? 0.f : exp2f(m2 - M);
  total = sum_of_groups<NG>(l2 * (m2 == -INFINITY ? 1.f : mine_weighs));
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[c][e] = sum_of_groups<NG>(o2[c][e] * mine_weighs);
}

// Decode: grid (splits, Hkv, B), or (Hkv, slices of all sequences) with balanced slices, W wavefronts; the blocks of a slice of `split_tokens` tokens of one (sequence, K/V
// head) go to the wavefronts in turn, whose states are combined through LDS.  With one slice the result is final,
// otherwise it is a partial state, and one workgroup of the (sequence, K/V head) merges them (`counters`, one per (sequence, K/V head), and `parts`, a few short slices'
// states: zero before and after; `states`: the others').  With k_new given the wavefront that has the last block takes the newest token (position ctx_len - 1) from the new rows and stores it into the cache.
// What such a launch is made of (1 x 777 tokens, 40 query heads on 8, 8.4 us a call, time stamps): 0.4 us to the length, 0.5 to the block ids, 1.4 to the blocks,
// 1.6 for the states through LDS (three barriers, divisions, the code of a row taken again in front of them), 0.2 and 0.35 for stores acknowledged and the count,
// 1.2 for the maxima, 1.4 for the states and the result.  Now 6.8 us: one barrier, whole rows per wavefront, 16 bytes per lane; the count asked for behind the
// first blocks; states that say by themselves when they have arrived; arguments fetched at once, query rows while the ids are on their way.  The same steps elsewhere, us
// (in graphs of several layers, both on one device; 1 x 777 8.5 / 6.9 there): 64 on 8, 16 x 20..2000 18.6 / 17.4, 40 on 8, 1 x 2000 9.7 / 8.0, 8 x 1000 13.7 / 12.0, 52 on 52, 1 x 700
// 10.7 / 9.3, 32 on 8, 1 x 16000 20.6 / 18.5, fp32, 64, 2 K/V heads, 1 x 700 7.5 / 6.0, fp32, 128, 3, 4 x 400 9.7 / 8.4, bf16, 256, 1, 1 x 800 13.9 / 10.7, bf16, 64, 8, 4 x 50..600
// 7.4 / 7.3; with long slices, counted, 8 on 1, 1 x 60000 (53 slices) 23.1 / 21.0, bf16, 256, 1, 1 x 40000 48 / 30.
template <typename E, int KS, int W, int AUX = 0, bool FULL = true, bool BALANCED = false>
__global__ __launch_bounds__(W * 64) void decode_any_kernel(
    const E* __restrict__ q, int q_row_stride, const E* __restrict__ k_new, const E* __restrict__ v_new, int new_row_stride,
    E* k_cache, E* v_cache, const int32_t* __restrict__ block_table, int bt_stride, const int32_t* __restrict__ ctx_len,
    E* __restrict__ out, float* __restrict__ lse, uint32_t* parts, uint32_t* states, uint32_t* counters, int split_tokens, int Hq,
    int Hkv, int G, int head_size, float scale_log2e, int B) {
  typedef Block<E, KS, AUX, FULL> Blk;
  constexpr int X = Elem<E>::X, NK = Blk::NK, NV = Blk::NV;
  // Where a wavefront has a row: NG groups of lanes share the states, and a lane has four elements of every 128 (or of 64).
  constexpr int NC = (KS + 3) / 4, NG = lane_groups(KS), LG = 64 / NG;
  __shared__ __attribute__((aligned(16))) E s_new[2][256];
  __shared__ __attribute__((aligned(16))) float2 s_ml[16][W];
  __shared__ __attribute__((aligned(16))) float s_acc[W][16][32 * KS + 4];
  __shared__ int s_order;
  const int g = BALANCED ? blockIdx.x : blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, quad = lane >> 4;
  const int D = FULL ? head_size : 128;
  // All arguments at once; fetched where they are wanted, they come in several round trips (us a call: 40 on 8, 1 x 2000 tokens 8.33 / 8.17, 52 on 52, 1 x 700
  // 8.82 / 8.51, fp32, 128, 4 x 400 8.81 / 8.56, bf16, 64, 4 x 600 7.80 / 7.58; balanced 17.33 / 17.45).
  asm volatile("" ::"s"(q), "s"(q_row_stride), "s"(k_new), "s"(v_new), "s"(new_row_stride), "s"(k_cache), "s"(v_cache), "s"(block_table), "s"(bt_stride),
               "s"(ctx_len), "s"(split_tokens), "s"(Hkv), "s"(G), "s"(head_size));
  const SliceOf at = slice_of_workgroup<BALANCED>(ctx_len, B, Hkv, split_tokens, W);
  if (BALANCED && at.sp < 0) return;
  const int b = at.b, sp = at.sp, L = at.L;
  const int32_t* const bt_row = block_table + (size_t)b * bt_stride;
  const Slice slice = decode_slice(L, at.tokens, at.most, sp);
  const int t0 = slice.t0, t1 = slice.t1;
  if (t1 <= t0) return;
  const WaveBlocks blocks = wave_blocks(t0, t1, wave, W);  // this wavefront's
  const int n = blocks.n;
  // (the block ids wait for the length: entries behind the sequence's last block are not read)
  int ids = lane < n ? bt_row[blocks.first + W * lane] : 0;
  // While the ids are on their way: the query rows (columns behind the group's heads have the last one's and are not used) and, for the wavefront
  // that has the block of the newest token, the new rows, element lane + 64 i.
  u32x4 qf[NK];
#pragma unroll
  for (int j = 0; j < NK; ++j) {
    const int d = (4 * j + quad) * X;
    qf[j] = *reinterpret_cast<const u32x4*>(q + (size_t)b * q_row_stride + (size_t)(g * G + min(col, G - 1)) * D + (FULL ? min(d, D - X) : d));
    if (FULL && d >= D) qf[j] = u32x4{0u, 0u, 0u, 0u};
  }
  const bool newest = k_new != nullptr && t1 == L && n > 0 && blocks.first + W * (n - 1) == (L - 1) >> 4;
  constexpr int NN = (KS + 1) / 2;
  typedef typename std::conditional<Blk::kF32, float, uint32_t>::type Word;  // (two elements of 16 bits to a register would be put together here, and waited for)
  Word kn[NN], vn[NN];
  if (newest) {
#pragma unroll
    for (int i = 0; i < NN; ++i) {
      const int d = FULL ? min(lane + 64 * i, D - 1) : lane + 64 * i;
      kn[i] = k_new[(size_t)b * new_row_stride + (size_t)g * D + d];
      vn[i] = v_new[(size_t)b * new_row_stride + (size_t)g * D + d];
    }
  }
  // (a scalar copy of its own: the merge below takes D into vector registers, and the blocks' addresses with it, were it the
  // same value - every load then goes through a loop over its descriptors, 1 us per call)
  int d_scalar = D;
  if constexpr (FULL) asm("" : "+s"(d_scalar));
  const size_t piece = (size_t)16 * d_scalar * sizeof(E);
  const char* const kc = reinterpret_cast<const char*>(k_cache);
  const char* const vc = reinterpret_cast<const char*>(v_cache);

  // The blocks are walked in windows of the 64 ids a register holds, two blocks in flight.  Most slices are at most 1024 W tokens
  // and take one window; more are for one very long context (its balanced slices: 52 on 52, 1 x 40000 tokens, 4450 and four wavefronts) and for one
  // longer than the caller's max_ctx_len, which the persistent kernel never minded and whose last slice takes the rest here.  A wavefront's last block comes first in its window: it may be the slice's last one, and what that needs
  // (the newest token, the slots behind the end) then stands once, in front of the loop - a short context is latency
  // from the first instruction on, and code that runs once costs its fetch.
  Blk f[2];
  int base = 0, nw = min(64, n);
  auto fetch = [&](Blk& fr, int i) {
    const int at = base + 64 < n ? i : i == 0 ? nw - 1 : i - 1;
    const size_t off = ((size_t)__builtin_amdgcn_readlane(ids, max(min(at, nw - 1), 0)) * Hkv + g) * piece;
    fr.load(kc + off, vc + off, (int)piece, lane, col, quad);
  };
  f32x4 acc[NV];
#pragma unroll
  for (int dt = 0; dt < NV; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  auto work = [&](const Blk& fr, int tail) {
    f32x4 s = fr.scores(qf) * scale_log2e;
    if (tail < 16) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * quad + e >= tail) s[e] = -INFINITY;
    }
    const f32x4 p = softmax_step<FULL>(s, m, l, acc);
    fr.values(p, acc);
  };
  if (n > 0) fetch(f[0], 0);
  if (n > 1) fetch(f[1], 1);
  // Which of the slices starts last merges them all (see the end).  Asked here, behind the first blocks, the answer is there before it is wanted.  Slices of
  // more than four rounds end at so many times that who waits for them is in their way: there it is the one that is done last (1 x 75000 tokens, 62.3 us; waiting 65.2).
  const int n_split = slice.n;
  // So it is where there are many states: those of the others are cleared by one CU (16 on 1, 17 x 100..6425 tokens 18.2 us, 15.6 so, 1 x 3000 11.8, 11.3; 8 on 1, 1 x 8000, 128 states,
  // 10.0, 9.9; fewer lose: 5 on 1, 4 x 130..1300, 55 states, 6.9, 7.2).
  const bool early = at.tokens <= kShortRounds * 16 * W && n_split * G <= 96;  // (the same for all slices of a context)
  auto arrive = [&]() { return (int)atomicInc(counters + (size_t)b * Hkv + g, (unsigned)n_split - 1); };  // (the last one wraps it to zero)
  int order = 0, newest_blk = 0;
  if (n_split > 1 && early && tid == 0) order = arrive();
  if (newest) {
#pragma unroll
    for (int i = 0; i < NN; ++i)
      if (lane + 64 * i < 32 * KS) {
        s_new[0][lane + 64 * i] = (E)kn[i];
        s_new[1][lane + 64 * i] = (E)vn[i];
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  while (base < n) {
    int tail = 16;
    const int last = blocks.first + W * (n - 1);
    if (base + 64 >= n && last == (t1 - 1) >> 4) {  // f[0] is the slice's last block
      tail = t1 - (last << 4);
      // (Where the lane stands is worked out here: kept from in front of the loop, with all that follows from it, it took the
      // registers of the blocks.  fp32, 256, spilled them, and its first and last blocks went through scratch memory: 50
      // tokens 12.2 us, 10.6 without; bf16, 128, kept 16 scalars in vector registers: 2000 tokens 10.8 and 10.7.  Heads of up to 96
      // elements have registers enough, and lose 0.06.)
      int at_lane = lane;
      if constexpr (KS > 3) asm volatile("" : "+v"(at_lane));
      if (newest) {
        f[0].put_token(s_new[0], s_new[1], tail - 1, D, at_lane & 15, at_lane >> 4);
        newest_blk = __builtin_amdgcn_readlane(ids, nw - 1);
      }
      if (tail < 16) f[0].clear_tail(tail, at_lane >> 4);
    }
    // Only blocks that exist are asked for: a load of nothing still takes its turn in the address unit, and three such
    // blocks (36 loads) per wavefront were 1 us of a context of 100 tokens.  Inside the loop every path issues the same
    // loads, so its waits are exact.
    work(f[0], tail);
    int i = 1;
    for (; i + 2 < nw; i += 2) {
      fetch(f[0], i + 1);
      work(f[1], 16);
      fetch(f[1], i + 2);
      work(f[0], 16);
    }
    if (i < nw) {
      if (i + 1 < nw) fetch(f[0], i + 1);
      work(f[1], 16);
      if (i + 1 < nw) work(f[0], 16);
    }
    base += 64;
    if (base < n) {
      nw = min(64, n - base);
      ids = lane < nw ? bt_row[blocks.first + W * (base + lane)] : 0;
      fetch(f[0], 0);
      if (nw > 1) fetch(f[1], 1);
    }
  }
  // The wavefronts' states through LDS, one barrier; then a wavefront has whole rows (heads h = wave + W k of the group), each group of lanes
  // the states of its share of the wavefronts:   M = max_w m_w;  total = sum_w l_w 2^(m_w - M);  o = sum_w acc_w 2^(m_w - M)  (weights as in merge_slices).
  l = sum_of_groups<4>(l);
  if (quad == 0) s_ml[col][wave] = float2{m, l};
#pragma unroll
  for (int dt = 0; dt < NV; ++dt)
    if (col < G) *reinterpret_cast<f32x4*>(&s_acc[wave][col][dt * 16 + 4 * quad]) = acc[dt];
  if (newest) {  // (nobody else in this launch needs the slot)
    const size_t off = ((size_t)newest_blk * Hkv + g) * piece;
    const int slot = (L - 1) & 15, units = D / X;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(scalar_here(const_cast<char*>(kc) + off), 0, (int)piece, kRsrc32);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(scalar_here(const_cast<char*>(vc) + off), 0, (int)piece, kRsrc32);
    if (lane < units) __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(&s_new[0][lane * X]), rk, (lane * 16 + slot) * 16, 0, 0);
#pragma unroll
    for (int i = 0; i < NN; ++i) {
      const int d = lane + 64 * i, at_d = (d * 16 + slot) * (int)sizeof(E);
      if (d >= D) continue;
      if constexpr (Blk::kF32) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s_new[1][d]), rv, at_d, 0, 0);
      else __builtin_amdgcn_raw_buffer_store_b16(s_new[1][d], rv, at_d, 0, 0);
    }
  }
  if (tid == 0) s_order = order;
  __syncthreads();
  const bool merges = (early || n_split == 1) && __builtin_amdgcn_readfirstlane(s_order) == n_split - 1;  // (one slice: it is the last one, and there is nothing to merge)
  // Partial states: [B][Hq][slices], or (balanced) [slices of all sequences][Hq].  slot0: of this slice and the group's first head.
  const int row_words = part_words(d_scalar), grp = lane / LG, el = (lane % LG) * 4;
  const size_t slot0 = BALANCED ? (size_t)blockIdx.y * Hq + (size_t)g * G : ((size_t)b * Hq + (size_t)g * G) * gridDim.x + sp;
  const size_t slot_step = BALANCED ? 1 : gridDim.x, slice_words = (size_t)(BALANCED ? Hq : 1) * row_words;
  auto to_out = [&](int h, float M, float total, const f32x4 (&o)[NC]) {
    const size_t row = (size_t)b * Hq + g * G + h;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (grp == 0 && (!FULL || el + 128 * c < D)) store4(out + row * D + el + 128 * c, divided(o[c], total));
    if (lse && lane == 0) lse[row] = (M + log2f(total)) * kLn2;
  };
  // Whole contexts: two rows of a wavefront at once, a half each with half the groups of lanes, and nothing behind it that a merge or a second walk needs (the loop below takes a row after
  // the other, and its code is fetched around theirs).  Us per call, the loop / so: bf16, 32, 16 on 1, 7 x 60 tokens 4.64 / 4.05, 16 on 2 4.15 / 4.09; 64, 16 on 1 5.22 / 4.57, 8 on 2 4.42 / 4.27,
  // 32 on 8, 4 x 50..600 7.22 / 7.05; fp32, 64, 16 on 1 6.28 / 5.50, 128, 8.51 / 7.94; bf16, 128, 16 on 1, 9 x 400 7.73 / 7.21.
  if constexpr (KS <= 4) {
    if (n_split == 1 && G <= 2 * W) {
      constexpr int NH = NG / 2;
      const int h = wave + W * (lane >> 5), hr = min(h, G - 1), of = (grp % NH) * (W / NH);
      auto both = [](float v, auto f) {
        if constexpr (NH == 1) return v;
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return f(__uint_as_float(a[0]), __uint_as_float(a[1]));
      };
      auto add = [](float a, float b) { return a + b; };
      float2 ml[W / NH];
      float M = -INFINITY, total = 0.f, zero = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < W / NH; ++w) {
        ml[w] = s_ml[hr][of + w];
        M = fmaxf(M, ml[w].x);
      }
      M = both(M, [](float a, float b) { return fmaxf(a, b); });
#pragma unroll
      for (int w = 0; w < W / NH; ++w) {
        const float wk = ml[w].x == -INFINITY ? 0.f : exp2f(ml[w].x - M);
        total += ml[w].y * (ml[w].x == -INFINITY ? 1.f : wk);
        o += *reinterpret_cast<const f32x4*>(&s_acc[of + w][hr][KS == 2 || KS == 4 ? el : min(el, 32 * KS - 4)]) * wk;
      }
      total = both(total, add);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = both(o[e], add);
        zero = __builtin_fmaf(o[e], 0.f, zero);
      }
      if (!__any(zero != zero && total == total)) {  // (otherwise as below)
        const size_t row = (size_t)b * Hq + g * G + h;
        if (h < G && grp % NH == 0 && (!FULL || el < D)) store4(out + row * D + el, divided(o, total));
        if (lse && h < G && (lane & 31) == 0) lse[row] = (M + log2f(total)) * kLn2;
        return;
      }
    }
  }
#pragma unroll 1
  for (int h = wave; h < G; h += W) {
    float2 ml[W / NG];
#pragma unroll
    for (int w = 0; w < W / NG; ++w) ml[w] = s_ml[h][grp * (W / NG) + w];
    float M = ml[0].x, total = 0.f;
#pragma unroll
    for (int w = 1; w < W / NG; ++w) M = fmaxf(M, ml[w].x);
    M = max_of_groups<NG>(M);
    f32x4 o[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W / NG; ++w) {
      const float wk = ml[w].x == -INFINITY ? 0.f : exp2f(ml[w].x - M);
      total += ml[w].y * (ml[w].x == -INFINITY ? 1.f : wk);
#pragma unroll
      for (int c = 0; c < NC; ++c)  // (lanes behind the last element have that one's four)
        o[c] += *reinterpret_cast<const f32x4*>(&s_acc[grp * (W / NG) + w][h][KS == 2 || KS % 4 == 0 ? el + 128 * c : min(el + 128 * c, 32 * KS - 4)]) * wk;
    }
    total = sum_of_groups<NG>(total);
    float zero = 0.f;  // (not a number if an element is not finite)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[c][e] = sum_of_groups<NG>(o[c][e]);
        zero = __builtin_fmaf(o[c][e], 0.f, zero);
      }
    if (__builtin_expect(__any(zero != zero && total == total), 0)) {  // (see attend_row)
      float r[4];
      attend_row<E>(scalar_here(q + (size_t)b * q_row_stride) + (size_t)(scalar_here(g) * G + h) * D, scalar_here(k_cache), scalar_here(v_cache), scalar_here(bt_row),
                    scalar_here(g), scalar_here(Hkv), scalar_here(D), scalar_here(t0), scalar_here(t1), scale_log2e, M, total, r);
      const int ln = here(lane);
#pragma unroll
      for (int k = 0; k < (KS + 1) / 2; ++k)
        if (ln + 64 * k < 32 * KS) s_acc[0][h][ln + 64 * k] = r[k];  // (nobody else reads this row)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int c = 0; c < NC; ++c)
        o[c] = *reinterpret_cast<const f32x4*>(&s_acc[0][h][min((ln % LG) * 4 + 128 * c, 32 * KS - 4)]);
    }
    uint32_t* const mine = (early ? parts : states) + (slot0 + h * slot_step) * row_words;
    if (!merges) {
      const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(scalar_here(mine), 0, row_words * 4, kRsrc32);
      if (grp == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (!FULL || el + 128 * c < D) store_part(to, (el + 128 * c) * 4, part_bits(o[c]));
      } else {
        store_part(to, D * 4, u32x2{part_bits(M), part_bits(total)});
      }
      continue;
    }
    if (n_split > 1) merge_slices<KS, FULL, false>(mine - (int64_t)sp * (int64_t)slice_words, (int)slice_words * 4, row_words * 4, D, n_split, sp, M, total, o);
    to_out(h, M, total, o);
  }
  if (early || n_split == 1) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (this wavefront's states are where every XCD finds them)
  __syncthreads();
  if (tid == 0) s_order = arrive();
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(s_order) != n_split - 1) return;
#pragma unroll 1
  for (int h = wave; h < G; h += W) {
    float M = 0.f, total = 0.f;
    f32x4 o[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    merge_slices<KS, FULL, true>(states + (slot0 + h * slot_step) * row_words - (int64_t)sp * (int64_t)slice_words, (int)slice_words * 4, row_words * 4, D, n_split, -1, M, total, o);
    to_out(h, M, total, o);
  }
}

// Decode of (bf16, 128), whole contexts (decode_short in decode_slices.h has the line, and the number of wavefronts) or, kSliced, the longer ones
// cut (decode_sliced): the W wavefronts of a workgroup walk the blocks of one (sequence, K/V head) in turn; no numbering, and but for what is
// cut nothing shared between workgroups, whom the hardware hands out.  The wavefront that has the last block takes it last.  With k_new given it puts the
// newest token into the block's registers and writes the block's V whole, and of its K whole lines, back (see there).
// Small batches are round trips; large ones are bound by memory and by what still runs when the rest is done.  Hence kLongest, for batches of more
// workgroups than run at once: grid (K/V heads, groups of up to 64 sequences, rank), and the workgroup takes the sequence of its rank in its group, by
// length (in 16 classes of 2^shift tokens), longest first.  A wavefront finds it among its lanes' 64 lengths with four ballots (0.2 to 1 us
// of a launch, which is why a batch that starts all at once, or has little to gain, does without: the grid is (K/V heads, B) then).
// us per call with the append, in the order of the batch / longest first: 40 query heads on 8, 1024 x ~103 tokens up to 800, one
// wavefront 124 / 100, 2 wavefronts 116 / 102, 4 117 / 110; 512 x 20..600 133 / 121; 8 on 1, 1024 x 8..600 39 / 34; 32 on 8, 152 x ~412 up to 1391 62 / 51 (persistent 65).
// What the persistent kernel spends on such batches: 1.2 us of a wavefront on a piece, a start-up of 7 us, and a second launch for the V columns.
// us per call, the kernels that had these batches / without order: 40 on 8, 819 x 193 159 / 146, 139 x ~46 20.7 / 13.1, 112 x
// 8 13.9 / 6.4; 32 on 8, 375 x ~18 28.6 / 15.3, 112 x 866 82.8 / 69.4; 52 on 52, 628 x 49..99 380 / 332, 23 x 63 21.3 / 13.1; 8 on 1, 1 x 180
// 6.5 / 5.1, 1 x 14 5.6 / 3.6.  Of that, whole V blocks instead of columns: 375 x ~18 19.4 -> 15.3 (one wavefront, decode_any_kernel before).  Tried:
// the last block read with the non-temporal hint or without, all of the block's K written back (4% worse than 16 bytes a unit), eight and
// sixteen wavefronts (one CU takes in 24 bytes a clock, however many ask: 1 x 777 tokens 10.2, 10.1, 10.9 with 4, 8, 16), fewer workgroups
// on a CU at a time (1024 x ~103: 118 with six, 124 with four, 160 with two).
// kSliced: bound by memory (reads at 6.0 to 6.4 TB/s, of the 7.0 that plain reads reach), and the order sees to it that the end is even whatever the
// lengths, which the host does not know: grid (K/V heads, rank).  Every wavefront reads all lengths (at most 256, four per lane), and their sum
// gives the slice with which no more than `max_full` whole ones come of a K/V head.  Those are handed out first, then what is left of the contexts, longest first; a
// workgroup without a rank ends (ranked in each group of 64 sequences, up to 3000 of them stood at the end of a launch: 16 on 1, 238 x 1140..11406 tokens 63.8 us, 56.3 so).  Of a context that is cut, the workgroup that is done last adds the states up (merge_slices): one that waited for
// the others while they walk slows them (long slices). `states` has max_full slots of whole slices and as many of the rest per K/V head.  A slice below 24 blocks
// costs more in states than it evens out.  us per layer, persistent kernel and its merge / here, two layers: 40 on 8, 128 x 512..4096 215 / 202, 52 on 52, 24 x 300..3000 193 / 187,
// 64 on 8, 256 x 1024..4096 463 / 458 (within the noise of either); other batches at decode_sliced.
enum class Order { kBatch, kLongest, kSliced };
template <int W, Order ORDER>
__global__ __launch_bounds__(W * 64, 3) void decode_short_kernel(
    const uint16_t* __restrict__ q, int q_row_stride, const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int new_row_stride,
    uint16_t* k_cache, uint16_t* v_cache, const int32_t* __restrict__ block_table, int bt_stride, const int32_t* __restrict__ ctx_len,
    uint16_t* __restrict__ out, float* __restrict__ lse, int Hq, int Hkv, int G, float scale_log2e, int B,
    int per_group, int shift, int stream, uint32_t* states, uint32_t* counters, int max_full) {
  typedef Block<uint16_t, 4, kNonTemporal, false> Blk;
  constexpr int D = 128, kPiece = 16 * D * 2;
  static_assert(W <= 8, "a wavefront adds up whole tiles");
  __shared__ __attribute__((aligned(16))) uint16_t s_new[256];   // the newest token's K row, then its V row
  __shared__ __attribute__((aligned(16))) char s_out[16 * 256];  // output rows: chunk c of row r at 256 r + 16 (c ^ r)
  __shared__ __attribute__((aligned(16))) f32x4 s_acc[W > 1 ? W : 1][W > 1 ? 8 : 1][64];
  __shared__ float s_m[W][16], s_l[W][16];
  __shared__ int s_bad, s_order;
  const int g = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int col = lane & 15, quad = lane >> 4;
  int b = blockIdx.y, L, n_split = 1, slice_no = 0, slot = 0, blk0 = 0, blk1 = 0;  // (sliced: the slices of the context, this one, its slot and its blocks)
  // the lane of rank r, by a class of 0 to 15, largest first, among lanes 0 .. have - 1
  auto select = [&](int key, int have, int r) {
    // `left`: the lanes among which the one of rank r still is; a bit of the key at a time, those that have it come first
    unsigned long long left = ~0ull >> (64 - have);
#pragma unroll
    for (int bit = 8; bit > 0; bit >>= 1) {
      const unsigned long long ones = __ballot((key & bit) != 0) & left;
      const int n_ones = __popcll(ones);
      left = r < n_ones ? ones : left & ~ones;
      r = r < n_ones ? r : r - n_ones;
    }
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(left >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)left, 0u));
    return (int)__builtin_ctzll(__ballot((left >> lane & 1) != 0 && before == r));
  };
  if constexpr (ORDER == Order::kLongest) {
    const int first = b * per_group, have = min(per_group, B - first), r = blockIdx.z;
    if (r >= have) return;
    const int len = lane < have ? ctx_len[first + lane] : 0, at = select(min(len >> shift, 15), have, r);
    b = first + at;
    L = __builtin_amdgcn_readlane(len, at);
  } else if constexpr (ORDER == Order::kSliced) {
    // Lane l has the sequences l groups + j, j < groups; group j, whose rests are ranked among themselves, the j-th of all lanes: much the same lengths where a
    // batch is sorted.
    const int groups = (B + 63) >> 6;
    int len[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = lane * groups + j;
      len[j] = j < groups && s < B ? ctx_len[s] : 0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) sum += (len[j] + 15) >> 4;
    const SlicedContexts cut = sliced_contexts(__builtin_amdgcn_readlane(lanes_prefix_sum(sum), 63), max_full, W);
    // whole slices, and (from bit 16 on) the contexts that are cut, of this lane's sequences and of those before them
    int full[4], own = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      full[j] = cut.full((len[j] + 15) >> 4);
      own += full[j] + (full[j] > 0 ? 1 << 16 : 0);
    }
    const int upto = lanes_prefix_sum(own), n_full = __builtin_amdgcn_readlane(upto, 63) & 0xffff;
    int r = blockIdx.y, at, group = 0;
    const bool whole = r < n_full;
    if (whole) {
      at = __builtin_ctzll(__ballot((upto & 0xffff) > r));
      slice_no = r - (__builtin_amdgcn_readlane(upto - own, at) & 0xffff);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int f = __builtin_amdgcn_readlane(full[j], at);
        if (group == j && slice_no >= f) {
          slice_no -= f;
          group = j + 1;
        }
      }
    } else {
      r -= n_full;
      if (r >= B) return;
      group = r % groups;
    }
    int mine = len[0], mine_full = full[0], before = 0;  // (of this group's sequence; whole slices and cuts in the lane's earlier groups)
#pragma unroll
    for (int j = 1; j < 4; ++j) {
      before += j <= group ? full[j - 1] + (full[j - 1] > 0 ? 1 << 16 : 0) : 0;
      mine = j == group ? len[j] : mine;
      mine_full = j == group ? full[j] : mine_full;
    }
    if (!whole) {
      at = select(cut.size_class(((mine + 15) >> 4) - mine_full * cut.blocks), (B - group + groups - 1) / groups, r / groups);
      slice_no = __builtin_amdgcn_readlane(mine_full, at);
    }
    b = at * groups + group;
    L = __builtin_amdgcn_readlane(mine, at);
    n_split = __builtin_amdgcn_readlane(mine_full, at) + 1;
    blk0 = slice_no * cut.blocks;
    blk1 = slice_no < n_split - 1 ? blk0 + cut.blocks : (L + 15) >> 4;
    const int first = __builtin_amdgcn_readlane(upto - own + before, at);  // (a slot for each whole slice, and one for the rest of each context that is cut)
    slot = (first & 0xffff) + (first >> 16) + slice_no;
  } else {
    L = __builtin_amdgcn_readfirstlane(ctx_len[b]);
  }
  const int32_t* const bt_row = block_table + (size_t)b * bt_stride;
  const bool fused = k_new != nullptr;
  u32x2 row = {0u, 0u};  // 8 bytes per lane of (K row, V row)
  if (fused) row = *reinterpret_cast<const u32x2*>((lane < 32 ? k_new : v_new) + (size_t)b * new_row_stride + (size_t)g * D + (lane & 31) * 4);
  u32x4 qf[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    qf[j] = col < G ? *reinterpret_cast<const u32x4*>(q + (size_t)b * q_row_stride + (size_t)(g * G + col) * D + (4 * j + quad) * 8) : z;
  }
  if (L <= 0) return;  // (no output for an empty sequence)
  if (ORDER != Order::kSliced) blk1 = (L + 15) >> 4;
  const int nb = blk1 - blk0, n = (nb - wave + W - 1) / W;  // this wavefront's blocks: blk0 + wave + W i, i < n
  const bool ends = ORDER != Order::kSliced || blk1 == (L + 15) >> 4, has_last = ends && wave + W * (n - 1) == nb - 1;
  const char* const kc = reinterpret_cast<const char*>(k_cache) + (size_t)g * kPiece;
  const char* const vc = reinterpret_cast<const char*>(v_cache) + (size_t)g * kPiece;
  const size_t blk_stride = (size_t)Hkv * kPiece;
  f32x4 acc[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  auto work = [&](const Blk& f, int tail) {
    f32x4 s = f.scores(qf) * scale_log2e;
    if (tail < 16) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * quad + e >= tail) s[e] = -INFINITY;
    }
    const f32x4 p = softmax_step<false>(s, m, l, acc);
    f.values(p, acc);
  };
  Blk f0;
  for (int base = 0; base < n; base += 64) {  // (the 64 ids that a register holds: 1024 W tokens)
    const int nw = min(64, n - base);
    const int ids = lane < nw ? bt_row[blk0 + wave + W * (base + lane)] : 0;
    if (base == 0 && has_last && fused) {  // (kept in LDS: it was asked for before the ids, and registers are short)
      *reinterpret_cast<u32x2*>(s_new + lane * 4) = row;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    auto fetch = [&](Blk& f, int i) {
      const size_t off = (size_t)__builtin_amdgcn_readlane(ids, i) * blk_stride;
      f.load(kc + off, vc + off, kPiece, lane, col, quad);
    };
    // Two blocks in flight, and no branch around a load inside the loop: its waits are exact.  An even number of blocks begins with
    // one of the other parity, so that the last block always lies in f0 and what it needs stands once.
    Blk f1;
    int i = 0;
    if (nw & 1) {
      fetch(f0, 0);
      if (nw > 1) fetch(f1, 1);
    } else {
      fetch(f1, 0);
      fetch(f0, 1);
      work(f1, 16);
      i = 1;
      if (nw > 2) fetch(f1, 2);
    }
    for (; i + 4 < nw; i += 2) {
      work(f0, 16);
      fetch(f0, i + 2);
      work(f1, 16);
      fetch(f1, i + 3);
    }
    if (i + 2 < nw) {
      work(f0, 16);
      fetch(f0, i + 2);
      work(f1, 16);
    }
    int tail = 16;
    if (base + 64 >= n && has_last) {  // f0 is the sequence's last block
      tail = L - 16 * (blk1 - 1);
      if (fused) {
        f0.put_token(s_new, s_new + D, tail - 1, D, col, quad);
        // A token is 16 places of 16 bytes of K and 128 places of two bytes of V, and the memory reads and writes 64 bytes at a time.  The
        // block is in the registers: the V block, and the four tokens of K that share the newest one's 64 bytes, go back whole, and nothing is read
        // for it (52 on 52, 320 x 49..99: 151 us with K's 16 bytes alone, 146).  Nobody else in the launch reads or writes this
        // piece; slots behind the end keep what they hold.
        const size_t off = (size_t)__builtin_amdgcn_readlane(ids, nw - 1) * blk_stride;
        char* const kd = const_cast<char*>(kc) + off;
        char* const vd = const_cast<char*>(vc) + off;
        int ln = lane;
        asm volatile("" : "+v"(ln));  // (where the lane writes is worked out here, not kept through the walk)
        const bool of_k = ((ln & 15) >> 2) == (tail - 1) >> 2;
        // (nothing follows in this wavefront that waits for the stores)
        if (stream) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (of_k) __builtin_nontemporal_store(f0.k[j], reinterpret_cast<u32x4*>(kd + ln * 16 + j * 1024));
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) __builtin_nontemporal_store(f0.v[dt], reinterpret_cast<s16x4*>(vd + (ln & 15) * 32 + (ln >> 4) * 8 + dt * 512));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (of_k) *reinterpret_cast<u32x4*>(kd + ln * 16 + j * 1024) = f0.k[j];
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<s16x4*>(vd + (ln & 15) * 32 + (ln >> 4) * 8 + dt * 512) = f0.v[dt];
        }
      }
      if (tail < 16) f0.clear_tail(tail, quad);
    }
    work(f0, tail);
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  // Lanes (col = head, quad) hold o[16 dt + 4 quad ..].  Through LDS into whole rows; with several wavefronts each adds up the states of
  // 8 / W tiles:   M = max_w m_w;  l = sum_w l_w 2^(m_w - M);  o = sum_w o_w 2^(m_w - M) / l.
  float zero = 0.f;  // (not a number if an element is not finite)
  auto to_rows = [&](const f32x4& v, int dt, float inv) {
#pragma unroll
    for (int e = 0; e < 4; ++e) zero = __builtin_fmaf(v[e], 0.f, zero);
    const u32x2 w = {pack_bf16x2(v[0] * inv, v[1] * inv), pack_bf16x2(v[2] * inv, v[3] * inv)};
    *reinterpret_cast<u32x2*>(s_out + col * 256 + ((2 * dt + (quad >> 1)) ^ col) * 16 + (quad & 1) * 8) = w;
  };
  bool bad;
  if constexpr (W > 1) {
    constexpr int kOwn = 8 / W;  // tiles of a wavefront
    if (quad == 0) {
      s_m[wave][col] = m;
      s_l[wave][col] = l;
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) s_acc[wave][dt][lane] = acc[dt];
    if (tid == 0) s_bad = 0;
    __syncthreads();
    float M = s_m[0][col];
#pragma unroll
    for (int w = 1; w < W; ++w) M = fmaxf(M, s_m[w][col]);
    float total = 0.f;
    f32x4 sum[kOwn];
#pragma unroll
    for (int t = 0; t < kOwn; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int dt0 = wave * kOwn;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float mw = s_m[w][col], wk = mw == -INFINITY ? 0.f : ORDER == Order::kSliced ? exp2f(mw - M) : __builtin_amdgcn_exp2f(mw - M);
      total += s_l[w][col] * (mw == -INFINITY ? 1.f : wk);
#pragma unroll
      for (int t = 0; t < kOwn; ++t) sum[t] += s_acc[w][dt0 + t][lane] * wk;
    }
    if (ORDER == Order::kSliced && n_split > 1) {
#pragma unroll
      for (int t = 0; t < kOwn; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) zero = __builtin_fmaf(sum[t][e], 0.f, zero);
      if (zero != zero && col < G && total == total) s_bad = 1;
      __syncthreads();
      const int row_words = part_words(D);
      uint32_t* const first = states + ((size_t)(slot - slice_no) * Hq + (size_t)g * G) * row_words;  // (slice 0, the group's first head)
      const int slice_bytes = Hq * row_words * 4;
      const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(scalar_here(reinterpret_cast<char*>(first) + (size_t)slice_no * slice_bytes), 0, G * row_words * 4, kRsrc32);
      if (!s_bad) {
        if (col < G) {
#pragma unroll
          for (int t = 0; t < kOwn; ++t) store_part(to, (col * row_words + (dt0 + t) * 16 + 4 * quad) * 4, part_bits(sum[t]));
          if (wave == 0 && quad == 0) store_part(to, (col * row_words + D) * 4, u32x2{part_bits(M), part_bits(total)});
        }
      } else {  // (see attend_row)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // (the newest token is in the cache)
        for (int h = wave; h < G; h += W) {
          float rm, rl, o[4];
          attend_row<uint16_t>(q + (size_t)b * q_row_stride + (size_t)(g * G + h) * D, k_cache, v_cache, bt_row, g, Hkv, D, 16 * blk0, min(L, 16 * blk1), scale_log2e, rm, rl, o);
#pragma unroll
          for (int r = 0; r < 2; ++r) __builtin_amdgcn_raw_buffer_store_b32(part_bits(o[r]), to, (h * row_words + lane + 64 * r) * 4, 0, kAuxAgent);
          if (lane == 0) store_part(to, (h * row_words + D) * 4, u32x2{part_bits(rm), part_bits(rl)});
        }
      }
      // The slice that is done last merges them all (the last one wraps the count to zero).
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (this wavefront's states are where every XCD finds them)
      __syncthreads();
      if (tid == 0) s_order = (int)atomicInc(counters + (size_t)(slot - slice_no) * Hkv + g, (unsigned)n_split - 1);
      __syncthreads();
      if (s_order != n_split - 1) return;
      for (int h = wave; h < G; h += W) {
        float rm = 0.f, rl = 0.f;
        f32x4 o[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
        merge_slices<4, false, true>(first + h * row_words, slice_bytes, row_words * 4, D, n_split, -1, rm, rl, o);
        const size_t row = (size_t)b * Hq + (size_t)g * G + h;
        if (lane < 32) store4(out + row * D + lane * 4, o[0] * (1.f / rl));
        if (lse && lane == 0) lse[row] = (rm + log2f(rl)) * kLn2;
      }
      return;
    }
    const float inv = 1.f / total;
#pragma unroll
    for (int t = 0; t < kOwn; ++t) to_rows(sum[t], dt0 + t, inv);
    if (zero != zero && col < G && total == total) s_bad = 1;
    m = M;
    l = total;
    __syncthreads();
    bad = s_bad != 0;
  } else {
    const float inv = 1.f / l;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) to_rows(acc[dt], dt, inv);
    bad = __any(zero != zero && col < G && l == l);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  const size_t row0 = (size_t)b * Hq + (size_t)g * G;
  for (int r = wave * 4 + quad; r < G; r += 4 * W)
    *reinterpret_cast<u32x4*>(out + (row0 + r) * D + col * 8) = *reinterpret_cast<const u32x4*>(s_out + r * 256 + (col ^ r) * 16);
  if (lse && wave == 0 && lane < G) lse[row0 + lane] = (m + log2f(l)) * kLn2;
  if (bad) {  // (see attend_row)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // (the newest token is in the cache)
    for (int h = wave; h < G; h += W) {
      float rm, rl, o[4];
      attend_row<uint16_t>(q + (size_t)b * q_row_stride + (size_t)(g * G + h) * D, k_cache, v_cache, bt_row, g, Hkv, D, 0, L, scale_log2e, rm, rl, o);
#pragma unroll
      for (int r = 0; r < 2; ++r) Elem<uint16_t>::store(out + (row0 + h) * D + lane + 64 * r, o[r] / rl);
    }
  }
}

// Prefill.  The rows of one (sequence, K/V head) are (position, query head of the group) pairs, position-major:
// row r = position r / G, head r % G, so the 16 columns of a product cover few positions and the causal bound cuts
// close.  Two ways to share the work in a workgroup of four wavefronts:
//   kSplitKeys false: 4 x 16 NC consecutive rows, 16 NC per wavefront, each walking the key blocks up to its own diagonal
//     by itself (the four read the same blocks at about the same time: the caches serve three of them);
//   kSplitKeys true: 16 rows, every fourth key block per wavefront, the four states combined through LDS.  A batch that
//     does not fill the chip is bound by one wavefront's walk (0.4 to 0.9 us per block), which this cuts to a quarter.
// Sequence b's tiles are numbered from cu_q[b] G / R + b (R rows per tile): consecutive sequences are then at least
// ceil(S G / R) numbers apart, so no prefix sum over the batch is needed (find_sequence).  Later tiles of a sequence
// are longer and go first.
template <typename E, int KS, int NC, bool kSplitKeys>
__global__ __launch_bounds__(256) void prefill_any_kernel(
    const E* __restrict__ q, int q_row_stride, const E* __restrict__ k_cache, const E* __restrict__ v_cache,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ ctx_before, const int32_t* __restrict__ block_table, int bt_stride,
    E* __restrict__ out, float* __restrict__ lse, int B, int Hq, int Hkv, int G, Divisor div_g, int D, float scale_log2e) {
  typedef Block<E, KS> Blk;
  constexpr int X = Elem<E>::X, NK = Blk::NK, NV = Blk::NV, R = (kSplitKeys ? 1 : 4) * 16 * NC;
  constexpr int kRow = KS * 32 + 4;
  static_assert(!kSplitKeys || NC == 1, "one set of rows per workgroup");
  __shared__ float s_m[4][16], s_l[4][16], s_tot[2][16];
  __shared__ __attribute__((aligned(16))) float s_acc[kSplitKeys ? 4 : 1][16][kSplitKeys ? kRow : 4];
  __shared__ int s_bad;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 15, quad = lane >> 4, g = blockIdx.y;
  const int tile_no = (int)(gridDim.x - 1 - blockIdx.x);
  auto first_tile = [&](int cu, int b) { return (long long)cu * G / R + b; };
  const SeqOf seq = find_sequence(cu_q, ctx_before, B, tile_no, first_tile);
  const int b = seq.b, tok0 = seq.tok0, S = seq.S, cb = seq.cb;
  const int n_rows = S * G;
  const long long tile_r0 = (tile_no - first_tile(tok0, b)) * R + (kSplitKeys ? 0 : wave * (16 * NC));
  if (tile_r0 >= n_rows) return;
  const int r0 = (int)tile_r0;
  const int32_t* const bt_row = block_table + (size_t)b * bt_stride;
  const size_t piece = (size_t)16 * D * sizeof(E);
  const int L = cb + S;

  int pos[NC], head[NC];
  bool ok[NC];
  u32x4 qf[NC][NK];
  f32x4 acc[NC][NV];
  float m[NC], l[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int r = r0 + c * 16 + col;
    ok[c] = r < n_rows;
    pos[c] = ok[c] ? fast_div(r, div_g) : 0;
    head[c] = ok[c] ? r - pos[c] * G : 0;
    const E* qrow = q + (size_t)(tok0 + pos[c]) * q_row_stride + (size_t)(g * G + head[c]) * D;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const int d = (4 * j + quad) * X;
      const u32x4 z = {0u, 0u, 0u, 0u};
      qf[c][j] = ok[c] && d < D ? *reinterpret_cast<const u32x4*>(qrow + d) : z;
    }
#pragma unroll
    for (int dt = 0; dt < NV; ++dt) acc[c][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[c] = -INFINITY;
    l[c] = 0.f;
  }
  // keys every row of the wavefront sees, and those at least one of them sees (rows that do not exist: as row 0)
  const int all_see = cb + fast_div(r0, div_g) + 1, some_see = cb + fast_div(min(n_rows, r0 + 16 * NC) - 1, div_g) + 1;
  // this wavefront's key blocks: blk0 + step i, i < n
  const int n_all = (some_see + 15) >> 4, blk0 = kSplitKeys ? wave : 0, step = kSplitKeys ? 4 : 1;
  const int n = kSplitKeys ? (n_all - wave + 3) >> 2 : n_all;
  const char* const kc = reinterpret_cast<const char*>(k_cache);
  const char* const vc = reinterpret_cast<const char*>(v_cache);

  int ids = lane < n ? bt_row[blk0 + step * lane] : 0;
  for (int base = 0; base < n; base += 64) {
    const int nw = min(64, n - base);
    const int my = ids;
    if (base + 64 + lane < n) ids = bt_row[blk0 + step * (base + 64 + lane)];
    Blk f[2];
    auto fetch = [&](Blk& fr, int i) {
      const size_t off = ((size_t)__builtin_amdgcn_readlane(my, min(i, nw - 1)) * Hkv + g) * piece;
      fr.load(kc + off, vc + off, (int)piece, lane, col, quad);
    };
    auto work = [&](Blk& fr, int i) {
      const int first = (blk0 + step * (base + i)) << 4;
      f32x4 s[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) s[c] = fr.scores(qf[c]) * scale_log2e;
      if (first + 16 > all_see) {
        asm volatile("" ::: "memory");  // (a real branch: the blocks at the diagonal only)
        if (first + 16 > L) fr.clear_tail(L - first, quad);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (first + 4 * quad + e > cb + pos[c]) s[c][e] = -INFINITY;
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const f32x4 p = softmax_step<true>(s[c], m[c], l[c], acc[c]);
        fr.values(p, acc[c]);
      }
    };
    fetch(f[0], 0);
    int i = 0;
    for (; i + 2 < nw; i += 2) {
      fetch(f[1], i + 1);
      work(f[0], i);
      fetch(f[0], i + 2);
      work(f[1], i + 1);
    }
    // The last one or two: only blocks that exist are asked for, and the loop above has no branch around a block, so its
    // waits are exact (with a branch, and loads of nothing behind the end: fp32, 4 x 350 tokens 13.1 against 11.3 us; bf16,
    // head size 80, 60 x 500 125 against 91; 256, 64 x 100 47 against 33).
    if (i + 1 < nw) fetch(f[1], i + 1);
    work(f[0], i);
    if (i + 1 < nw) work(f[1], i + 1);
  }

  auto redo_row = [&](int r) {
    const int p = fast_div(r, div_g), h = r - p * G;
    float rm, rl, o[4];
    attend_row<E>(q + (size_t)(tok0 + p) * q_row_stride + (size_t)(g * G + h) * D, k_cache, v_cache, bt_row, g, Hkv, D, 0, cb + p + 1,
                  scale_log2e, rm, rl, o);
    for (int k = 0; k < 4; ++k) {
      const int d = lane + 64 * k;
      if (d < D) Elem<E>::store(out + ((size_t)(tok0 + p) * Hq + g * G + h) * D + d, o[k] / rl);
    }
  };
  if constexpr (kSplitKeys) {
    l[0] += __shfl_xor(l[0], 16);
    l[0] += __shfl_xor(l[0], 32);
    if (quad == 0) {
      s_m[wave][col] = m[0];
      s_l[wave][col] = l[0];
    }
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    const float M = fmaxf(fmaxf(s_m[0][col], s_m[1][col]), fmaxf(s_m[2][col], s_m[3][col]));
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) total += s_m[w][col] == -INFINITY ? s_l[w][col] : s_l[w][col] * __builtin_amdgcn_exp2f(s_m[w][col] - M);
    const float mine = m[0] == -INFINITY ? 0.f : exp2f(m[0] - M);
    if (threadIdx.x < 16) {
      s_tot[0][col] = M;
      s_tot[1][col] = total;
    }
#pragma unroll
    for (int dt = 0; dt < NV; ++dt) *reinterpret_cast<f32x4*>(&s_acc[wave][col][dt * 16 + 4 * quad]) = acc[0][dt] * mine;
    __syncthreads();
    // sixteen threads per row, four elements each
    const int rr = (int)threadIdx.x >> 4, r = r0 + rr;
    if (r < n_rows) {
      const int p = fast_div(r, div_g), h = r - p * G;
      const size_t row = (size_t)(tok0 + p) * Hq + (size_t)g * G + h;
      const float sum = s_tot[1][rr], inv = 1.f / sum;
      bool bad = false;
#pragma unroll
      for (int d0 = 0; d0 < KS * 32; d0 += 64) {
        const int d = d0 + ((int)threadIdx.x & 15) * 4;
        if (d >= D) continue;
        f32x4 o = *reinterpret_cast<const f32x4*>(&s_acc[0][rr][d]);
#pragma unroll
        for (int w = 1; w < 4; ++w) o += *reinterpret_cast<const f32x4*>(&s_acc[w][rr][d]);
#pragma unroll
        for (int e = 0; e < 4; ++e) bad = bad || not_finite(o[e]);
        store4(out + row * D + d, o * inv);
      }
      if (bad && sum == sum) atomicOr(&s_bad, 1 << rr);
      if (lse && ((int)threadIdx.x & 15) == 0) lse[row] = (s_tot[0][rr] + log2f(sum)) * kLn2;
    }
    __syncthreads();
    for (int c = wave; c < 16; c += 4)  // (see attend_row)
      if (s_bad >> c & 1) redo_row(r0 + c);
  } else {
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    l[c] += __shfl_xor(l[c], 16);
    l[c] += __shfl_xor(l[c], 32);
    const float inv = 1.f / l[c];
    const size_t row = (size_t)(tok0 + pos[c]) * Hq + (size_t)g * G + head[c];
    bool bad = false;
    if (ok[c]) {
#pragma unroll
      for (int dt = 0; dt < NV; ++dt) {
        const int d = dt * 16 + 4 * quad;
        if (d < D) {
          const f32x4 o = acc[c][dt];
          store4(out + row * D + d, o * inv);
#pragma unroll
          for (int e = 0; e < 4; ++e) bad = bad || not_finite(o[e]);
        }
      }
      if (lse && quad == 0) lse[row] = (m[c] + log2f(l[c])) * kLn2;
    }
    unsigned long long redo = __ballot(bad && l[c] == l[c]);
    redo = (redo | redo >> 16 | redo >> 32 | redo >> 48) & 0xffffu;  // rows whose result is to be taken again (see attend_row)
    while (redo) {
      const int rc = __ffsll(redo) - 1;
      redo &= redo - 1;
      redo_row(r0 + c * 16 + rc);
    }
  }
  }
}

namespace {

// Calls f(std::integral_constant<int, KS>) for the smallest instantiated KS with 32 KS >= D.
template <typename F>
void for_head_size(int D, F f) {
  if (D <= 32) f(std::integral_constant<int, 1>());
  else if (D <= 64) f(std::integral_constant<int, 2>());
  else if (D <= 96) f(std::integral_constant<int, 3>());
  else if (D <= 128) f(std::integral_constant<int, 4>());
  else if (D <= 192) f(std::integral_constant<int, 6>());
  else f(std::integral_constant<int, 8>());
}

template <typename E>
void launch_prefill_typed(const AttnArgs& a, const int32_t* cu_q, const int32_t* ctx_before, int32_t T, hipStream_t s) {
  const int G = a.Hq / a.Hkv;
  for_head_size(a.D, [&](auto ks) {
    constexpr int KS = decltype(ks)::value, NC = KS <= 4 ? 2 : 1;  // two sets of 16 rows while their state fits the registers
    auto launch = [&](auto kernel, int rows) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)((int64_t)T * G / rows + a.B), (unsigned)a.Hkv), dim3(256), 0, s, (const E*)a.q,
                         a.q_row_stride, (const E*)a.k_cache, (const E*)a.v_cache, cu_q, ctx_before, a.block_table, a.bt_stride,
                         (E*)a.out, a.lse, a.B, a.Hq, a.Hkv, G, make_divisor((uint32_t)G), a.D, a.scale_log2e);
    };
    // Batches too small to fill the chip share the keys of 16 rows out instead of the rows, unless the prompts are so short
    // that there is little to share.  The line (rows x head size, against 5 Mi, or in proportion for prompts below 256
    // tokens on average) lies between what gains and what loses by it (us, rows shared / keys shared): fp32, 64, 4 heads:
    // 4 x 350 tokens 33 / 11, 16 x 100 13 / 7; fp32, 128, 6 heads: 8 x 300 50 / 36, 32 x 300 96 / 120; bf16, 64, 32 heads:
    // 4 x 330 23 / 18, 4 x 600 44 / 39, 8 x 600 70 / 70, 16 x 100 11 / 16, 100 x 20 12 / 21; bf16, 256, 8 heads: 4 x 300 21 / 20,
    // 40 x 16 7 / 11, 64 x 100 34 / 75.  It is good to a factor of two: head sizes of 128 in fp32 and of 256 meet at half of
    // it (bf16, 256, 8 x 300, keys shared: 38 where rows would take 29), few long prompts at 1.2 times it (bf16, 64, 1 x
    // 3000, rows shared: 207 where keys would take 152).
    const int64_t line = std::min<int64_t>((int64_t)5 << 20, ((int64_t)5 << 12) * T / a.B);
    if ((int64_t)T * a.Hq * (32 * KS) <= line) launch(prefill_any_kernel<E, KS, 1, true>, 16);
    else launch(prefill_any_kernel<E, KS, NC, false>, 64 * NC);
  });
}

template <typename E>
void launch_decode_typed(const AttnArgs& a, const int32_t* ctx_len, int32_t split_tokens, int32_t n_split_max, uint32_t* parts,
                         uint32_t* states, uint32_t* counters, bool many, hipStream_t s) {
  const bool balanced = split_tokens == 0;
  auto launch = [&](auto kernel, int W) {
    hipLaunchKernelGGL(kernel, balanced ? dim3((unsigned)a.Hkv, (unsigned)n_split_max) : dim3((unsigned)n_split_max, (unsigned)a.Hkv, (unsigned)a.B), dim3(W * 64), 0, s,
                       (const E*)a.q, a.q_row_stride, (const E*)a.k_new, (const E*)a.v_new, a.new_row_stride,
                       (E*)const_cast<void*>(a.k_cache), (E*)const_cast<void*>(a.v_cache), a.block_table, a.bt_stride, ctx_len,
                       (E*)a.out, a.lse, parts, states, counters, split_tokens, a.Hq, a.Hkv, a.Hq / a.Hkv, a.D, a.scale_log2e, a.B);
  };
  for_head_size(a.D, [&](auto ks) {
    constexpr int KS = decltype(ks)::value, W = decode_wavefronts(32 * KS, sizeof(E));
    if constexpr (KS == 4 && sizeof(E) == 2) {
      if (a.D == 128 && balanced)
        // (non-temporal: a batch of several long contexts comes from memory, layer after layer: 16 x 20..2000 tokens 15.7 us without the
        // hint and 14.5 with it, 16 x 2000 30.5 and 27.8, 9 x 1196..9574 32.2 and 29.0; a single one may still be in the last-level cache)
        return many ? launch(decode_any_kernel<E, KS, 4, kNonTemporal, false, true>, 4) : launch(decode_any_kernel<E, KS, W, kNonTemporal, false, true>, W);
      if (a.D == 128) return launch(decode_any_kernel<E, KS, W, 0, false>, W);
      if (many) return launch(decode_any_kernel<E, KS, 4, kNonTemporal>, 4);
    }
    launch(decode_any_kernel<E, KS, W>, W);
  });
}

}  // namespace

hipError_t launch_prefill_any(const AttnArgs& a, const int32_t* cu_q, const int32_t* ctx_before, int32_t T, hipStream_t s) {
  if (a.dtype == ECOSERVE_BF16) launch_prefill_typed<uint16_t>(a, cu_q, ctx_before, T, s);
  else launch_prefill_typed<float>(a, cu_q, ctx_before, T, s);
  return hipGetLastError();
}

namespace {

template <int W, Order ORDER>
hipError_t launch_whole(const AttnArgs& a, const int32_t* ctx_len, int32_t max_ctx_len, bool stream, uint32_t* states, uint32_t* counters, int32_t max_full, hipStream_t s) {
  // groups of equal size, at most one sequence per lane; length classes: the largest holds max_ctx_len and what lies above it
  const int groups = (a.B + 63) / 64, per_group = (a.B + groups - 1) / groups;
  int shift = 4;
  while (max_ctx_len >> shift > 15) ++shift;
  const dim3 grid = ORDER == Order::kLongest ? dim3((unsigned)a.Hkv, (unsigned)groups, (unsigned)per_group) : dim3((unsigned)a.Hkv, (unsigned)(a.B + max_full));
  hipLaunchKernelGGL((decode_short_kernel<W, ORDER>), grid, dim3(W * 64), 0, s, (const uint16_t*)a.q, a.q_row_stride, (const uint16_t*)a.k_new, (const uint16_t*)a.v_new,
                     a.new_row_stride, (uint16_t*)const_cast<void*>(a.k_cache), (uint16_t*)const_cast<void*>(a.v_cache), a.block_table, a.bt_stride, ctx_len,
                     (uint16_t*)a.out, a.lse, a.Hq, a.Hkv, a.Hq / a.Hkv, a.scale_log2e, a.B, per_group, shift, stream ? 1 : 0, states, counters, max_full);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_short(const AttnArgs& a, const int32_t* ctx_len, int32_t waves, int32_t max_ctx_len, int32_t num_cu, hipStream_t s) {
  const int64_t pairs = (int64_t)a.B * a.Hkv;
  const bool stream = decode_short_stream(pairs, max_ctx_len);
  auto of = [&](auto w) {
    constexpr int W = decltype(w)::value;
    return decode_short_ordered(pairs, max_ctx_len, num_cu) ? launch_whole<W, Order::kLongest>(a, ctx_len, max_ctx_len, stream, nullptr, nullptr, 0, s)
                                                            : launch_whole<W, Order::kBatch>(a, ctx_len, max_ctx_len, stream, nullptr, nullptr, 0, s);
  };
  return waves == 1 ? of(std::integral_constant<int, 1>()) : waves == 2 ? of(std::integral_constant<int, 2>()) : waves == 4 ? of(std::integral_constant<int, 4>())
                                                                                                                  : hipErrorInvalidValue;
}

hipError_t launch_decode_sliced(const AttnArgs& a, const int32_t* ctx_len, int32_t max_ctx_len, uint32_t* states, uint32_t* counters, int32_t num_cu, hipStream_t s) {
  if (a.B > kSlicedMostSequences) return hipErrorInvalidValue;
  return launch_whole<4, Order::kSliced>(a, ctx_len, max_ctx_len, decode_short_stream((int64_t)a.B * a.Hkv, max_ctx_len), states, counters, sliced_most_full(a.B, a.Hkv, num_cu), s);
}

hipError_t launch_decode_any(const AttnArgs& a, const int32_t* ctx_len, int32_t split_tokens, int32_t n_split_max, uint32_t* parts,
                             uint32_t* states, uint32_t* counters, int32_t num_cu, hipStream_t s) {
  const bool many = (int64_t)(split_tokens ? a.B : 1) * a.Hkv * n_split_max > num_cu;
  if (a.dtype == ECOSERVE_BF16) launch_decode_typed<uint16_t>(a, ctx_len, split_tokens, n_split_max, parts, states, counters, many, s);
  else launch_decode_typed<float>(a, ctx_len, split_tokens, n_split_max, parts, states, counters, many, s);
  return hipGetLastError();
}

}  // namespace eco
