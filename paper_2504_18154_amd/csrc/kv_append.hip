// KV-cache append: scatter new K/V rows into the paged pools through the block table.
//
// Section 2.1 of the paper (key/value embeddings of processed tokens are saved and
// reused) and Section 5 (fixed-size cache blocks).  New token i of sequence b goes to
// absolute position p = ctx_before[b] + i: block block_table[b][p / 16], slot p % 16.
// Pure integer indexing and byte copies, so the result is bit-exact.
//
// Source rows are [Hkv][D] per token, consecutive tokens `new_row_stride` elements apart (Hkv * D for a
// packed [T][Hkv][D] array, more when K and V sit inside a wider row such as a fused projection output,
// Eq. 1); destination is the library's block layout
//   K: [blk][Hkv][D/x][16 slots][x]   (x = elements per 16 bytes)
//   V: [blk][Hkv][D][16 slots]
// One workgroup fills one destination block for one, two or four adjacent K/V heads: up to 16 token
// rows in, per head one contiguous K piece and one contiguous V piece out (4 KiB each for
// bf16, D = 128).  Several heads per workgroup keep more loads in flight per thread and
// spread the cost of finding the block over more bytes; a small call ends sooner with one (append_heads.h has the line).
// K units keep their 16 bytes and only change place, so they are copied directly with the
// writes running along the destination.  V needs a transposition (16 slots of one element
// become contiguous): the token rows are staged in LDS with coalesced reads and written
// back as 16-byte units along the destination.  Blocks that are only partly addressed
// (the first block of an append that continues a sequence, the last block) write only the
// addressed slots, element by element where a 16-byte unit is not completely new.
//
// The destination blocks of the whole batch are numbered sequence after sequence, those of
// sequence b from cu_q[b] / 16 + 2 b: S new tokens touch at most S / 16 + 2 blocks, so the
// numbers of consecutive sequences do not meet, and a workgroup finds its (sequence, block)
// with a search over cu_q (find_sequence) where a prefix sum over the batch used to cost two
// barriers and a trip through LDS in front of everything else (one prompt of 93 tokens: 6.7 ->
// 5.4 us; the tables of the whole batch also no longer take the LDS of a workgroup).
// A call that brings at most one token per sequence (the decode step) takes a leaner kernel:
// one wavefront per (sequence, K/V head), no numbering, no staging.
#include <type_traits>

#include "append_heads.h"
#include "common.h"

namespace eco {

static_assert(kAppendThreads == 16 * kAppendAtOnceBytes / 16, "one unit of K and one of V per thread");

template <typename E, int HPW, bool kAtOnce>
__global__ __launch_bounds__(kAppendThreads) void kv_append_kernel(E* __restrict__ k_cache, E* __restrict__ v_cache,
                                                                    const E* __restrict__ k_new,
                                                                    const E* __restrict__ v_new, int new_row_stride,
                                                                    const int32_t* __restrict__ cu_q,
                                                                    const int32_t* __restrict__ ctx_before,
                                                                    const int32_t* __restrict__ block_table,
                                                                    int bt_stride, int B, int Hkv, int D) {
  constexpr int X = Elem<E>::X;
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  // HPW staged V tiles of 16 rows of D + X elements (padded rows), sized by the launch (append_lds_bytes)
  extern __shared__ __attribute__((aligned(16))) char staged[];
  const int vrow = D + X;
  E* vt = reinterpret_cast<E*>(staged);
  auto first_unit = [](int cu, int b) { return (cu >> 4) + 2 * b; };
  const SeqOf seq = find_sequence(cu_q, ctx_before, B, blockIdx.x, first_unit);
  const int b = seq.b, tok0 = seq.tok0, S = seq.S, cb = seq.cb;
  const int nth = (int)blockIdx.x - first_unit(tok0, b);  // destination block number within the sequence
  if (S <= 0 || nth > ((cb + S - 1) >> 4) - (cb >> 4)) return;
  const int g0 = blockIdx.y * HPW, tid = threadIdx.x;
  const int j = (cb >> 4) + nth;                            // logical block of the sequence
  const int lo = max(0, cb - (j << 4));               // addressed slots [lo, hi) of this block
  const int hi = min(16, cb + S - (j << 4));
  const int t_slot0 = tok0 + (j << 4) - cb;           // packed token index of slot 0 (may be < tok0)
  const int64_t blk = block_table[(size_t)b * bt_stride + j];
  const int upr = D / X;                              // 16-byte units per head row

  E* kdst = k_cache + ((size_t)blk * Hkv + g0) * 16 * D;
  if constexpr (kAtOnce) {
    // one unit of K and one of V per thread and head (16 D / X <= threads), all asked for before the first use
    const int kslot = tid & 15, kc = tid >> 4, vslot = tid / upr, vc = tid % upr;
    const bool kin = tid < 16 * upr && kslot >= lo && kslot < hi, vin = tid < 16 * upr && vslot >= lo && vslot < hi;
    u4 kval[HPW], vval[HPW];
    const E* const ksrc = k_new + (size_t)(t_slot0 + kslot) * new_row_stride + g0 * D + kc * X;
    const E* const vsrc = v_new + (size_t)(t_slot0 + vslot) * new_row_stride + g0 * D + vc * X;
#pragma unroll
    for (int h = 0; h < HPW; ++h) vval[h] = vin ? *reinterpret_cast<const u4*>(vsrc + (size_t)h * D) : u4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int h = 0; h < HPW; ++h) kval[h] = kin ? *reinterpret_cast<const u4*>(ksrc + (size_t)h * D) : u4{0u, 0u, 0u, 0u};
    if (vin)
#pragma unroll
      for (int h = 0; h < HPW; ++h) *reinterpret_cast<u4*>(vt + ((size_t)h * 16 + vslot) * vrow + vc * X) = vval[h];
    if (kin)
#pragma unroll
      for (int h = 0; h < HPW; ++h) *reinterpret_cast<u4*>(kdst + ((size_t)h * 16 * D) + (size_t)tid * X) = kval[h];
  } else {
  // The HPW heads of one token are adjacent in the source, so each pass below issues HPW
  // independent 16-byte loads per thread before the first use.
  // K: unit (c, slot) -> destination [c][slot][X]; threads run along the destination
  for (int u = tid; u < 16 * upr; u += kAppendThreads) {
    const int slot = u & 15, c = u >> 4;
    if (slot >= lo && slot < hi) {
      const E* src = k_new + (size_t)(t_slot0 + slot) * new_row_stride + g0 * D + c * X;
      u4 val[HPW];
#pragma unroll
      for (int h = 0; h < HPW; ++h) val[h] = *reinterpret_cast<const u4*>(src + (size_t)h * D);
#pragma unroll
      for (int h = 0; h < HPW; ++h) *reinterpret_cast<u4*>(kdst + ((size_t)h * 16 * D) + (size_t)u * X) = val[h];
    }
  }
  // V: stage rows (threads run along the source rows) ...
  for (int u = tid; u < 16 * upr; u += kAppendThreads) {
    const int slot = u / upr, c = u % upr;
    if (slot >= lo && slot < hi) {
      const E* src = v_new + (size_t)(t_slot0 + slot) * new_row_stride + g0 * D + c * X;
      u4 val[HPW];
#pragma unroll
      for (int h = 0; h < HPW; ++h) val[h] = *reinterpret_cast<const u4*>(src + (size_t)h * D);
#pragma unroll
      for (int h = 0; h < HPW; ++h) *reinterpret_cast<u4*>(vt + ((size_t)h * 16 + slot) * vrow + c * X) = val[h];
    }
  }
  }
  __syncthreads();
  // ... and write [d][16 slots] in 16-byte units of X slots (threads run along the destination)
  E* vdst = v_cache + ((size_t)blk * Hkv + g0) * D * 16;
  constexpr int kGroups = 16 / X;  // 16-byte units per element row
  for (int u = tid; u < HPW * D * kGroups; u += kAppendThreads) {
    const int h = u / (D * kGroups), r = u % (D * kGroups);
    const int d = r / kGroups, s0 = (r % kGroups) * X;
    const E* col = vt + (size_t)h * 16 * vrow + d;
    E* dst = vdst + ((size_t)h * D + d) * 16;
    if (s0 >= lo && s0 + X <= hi) {
      E tmp[X];
#pragma unroll
      for (int e = 0; e < X; ++e) tmp[e] = col[(s0 + e) * vrow];
      *reinterpret_cast<u4*>(dst + s0) = *reinterpret_cast<const u4*>(tmp);
    } else {
#pragma unroll
      for (int e = 0; e < X; ++e)
        if (s0 + e >= lo && s0 + e < hi) dst[s0 + e] = col[(s0 + e) * vrow];
    }
  }
}

// At most one new token per sequence (the decode step): one wavefront per (sequence, K/V head)
// copies the token's K row as 16-byte units and scatters its V row into the slot's column.  Launch latency and two round
// trips bound it (16 sequences, 8 K/V heads, bf16, 128: 2.94 us with the rows and stores of K and V one after the
// other, 2.47 now), and from a thousand pairs on the V columns, 128 sectors that the memory reads and writes for two bytes.
template <typename E>
__global__ __launch_bounds__(kAppendThreads) void kv_append_one_kernel(E* __restrict__ k_cache, E* __restrict__ v_cache,
                                                                        const E* __restrict__ k_new,
                                                                        const E* __restrict__ v_new, int new_row_stride,
                                                                        const int32_t* __restrict__ cu_q,
                                                                        const int32_t* __restrict__ ctx_before,
                                                                        const int32_t* __restrict__ block_table,
                                                                        int bt_stride, int B, int Hkv, int D,
                                                                        int pos_bias) {
  constexpr int X = Elem<E>::X, kPer = 256 / 64;  // V elements per lane of the largest head
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const int pair = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (pair >= B * Hkv) return;
  const int b = pair / Hkv, g = pair % Hkv;
  // cu_q == NULL: exactly one token per sequence, token b belongs to sequence b
  const int p = ctx_before[b] + pos_bias, tok = cu_q ? cu_q[b] : b, end = cu_q ? cu_q[b + 1] : b + 1;
  if (end - tok <= 0 || p < 0) return;  // (p: pos_bias -1 on an empty sequence: nothing to store)
  // the token's rows are asked for before the block that they go to: neither waits for the other
  const E* const ksrc = k_new + (size_t)tok * new_row_stride + g * D;
  const E* const vsrc = v_new + (size_t)tok * new_row_stride + g * D;
  u4 kval = {0u, 0u, 0u, 0u};
  E vval[kPer];
  if (lane < D / X) kval = *reinterpret_cast<const u4*>(ksrc + lane * X);
#pragma unroll
  for (int r = 0; r < kPer; ++r) vval[r] = lane + 64 * r < D ? vsrc[lane + 64 * r] : E(0);
  const int64_t blk = block_table[(size_t)b * bt_stride + (p >> 4)];
  // K: unit c of the row to [c][slot][X elements], V: element d to [d][slot]
  const int slot = p & 15;
  E* const kdst = k_cache + ((size_t)blk * Hkv + g) * 16 * D + (size_t)slot * X;
  E* const vdst = v_cache + ((size_t)blk * Hkv + g) * D * 16 + slot;
  if (lane < D / X) *reinterpret_cast<u4*>(kdst + (size_t)lane * 16 * X) = kval;
#pragma unroll
  for (int r = 0; r < kPer; ++r)
    if (lane + 64 * r < D) vdst[(size_t)(lane + 64 * r) * 16] = vval[r];
}

// Dynamic LDS of the tiled kernel: HPW staged V tiles.
template <typename E>
static size_t append_lds_bytes(int D, int hpw) {
  return (size_t)hpw * 16 * (D + Elem<E>::X) * sizeof(E);
}

template <typename E, int HPW, bool kAtOnce>
static void launch_tiled(const ecoserve_layout& L, void* k_cache, void* v_cache, const void* k_new, const void* v_new,
                         int32_t new_row_stride, const int32_t* cu_q, const int32_t* ctx_before, const int32_t* block_table,
                         int32_t bt_stride, int32_t B, int32_t T, hipStream_t s) {
  const int64_t max_units = (int64_t)T / 16 + 2 * (int64_t)B;  // (the numbering of the kernel, up to sequence B)
  const dim3 grid((unsigned)max_units, (unsigned)(L.num_kv_heads / HPW));
  // (above 64 KiB - fp32 with large heads - the kernel's limit was raised when the context was created)
  const size_t lds = append_lds_bytes<E>(L.head_dim, HPW);
  hipLaunchKernelGGL((kv_append_kernel<E, HPW, kAtOnce>), grid, dim3(kAppendThreads), lds, s, (E*)k_cache, (E*)v_cache,
                     (const E*)k_new, (const E*)v_new, new_row_stride, cu_q, ctx_before, block_table, bt_stride, B,
                     L.num_kv_heads, L.head_dim);
}

template <typename E>
static void launch_typed(const ecoserve_layout& L, void* k_cache, void* v_cache, const void* k_new, const void* v_new,
                         int32_t new_row_stride, const int32_t* cu_q, const int32_t* ctx_before, const int32_t* block_table,
                         int32_t bt_stride, int32_t B, int32_t T, int32_t max_new_len, int32_t pos_bias, int num_cu,
                         hipStream_t s) {
  if (max_new_len <= 1) {
    // (one wavefront per workgroup spreads a small batch over more CUs: 16 sequences, 8 K/V heads 2.47 us, 2.70 with four;
    // from two per CU on four are as good or better: 256 sequences 5.83 and 5.64)
    const int64_t pairs = (int64_t)B * L.num_kv_heads;
    const int per_wg = pairs <= 2 * num_cu ? 1 : kAppendThreads / 64;
    const dim3 grid((unsigned)((pairs + per_wg - 1) / per_wg));
    hipLaunchKernelGGL((kv_append_one_kernel<E>), grid, dim3(per_wg * 64), 0, s, (E*)k_cache, (E*)v_cache,
                       (const E*)k_new, (const E*)v_new, new_row_stride, cu_q, ctx_before, block_table, bt_stride, B,
                       L.num_kv_heads, L.head_dim, pos_bias);
    return;
  }
  const AppendHeads by = append_heads(T, B, L.num_kv_heads, (int64_t)L.head_dim * sizeof(E), num_cu);
  auto launch = [&](auto hpw, auto at_once) {
    launch_tiled<E, decltype(hpw)::value, decltype(at_once)::value>(L, k_cache, v_cache, k_new, v_new, new_row_stride, cu_q, ctx_before, block_table,
                                                                    bt_stride, B, T, s);
  };
  typedef std::integral_constant<int, 1> One;
  if (by.heads == 4) launch(std::integral_constant<int, 4>(), std::false_type());
  else if (by.heads == 2) launch(std::integral_constant<int, 2>(), std::false_type());
  else if (by.at_once) launch(One(), std::true_type());
  else launch(One(), std::false_type());
}

template <typename E, int HPW>
static hipError_t raise_lds_limit(const ecoserve_ctx* ctx) {
  const size_t lds = append_lds_bytes<E>(ctx->lay.head_dim, HPW);
  if (lds <= 60 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&kv_append_kernel<E, HPW, false>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

hipError_t prepare_kv_append(const ecoserve_ctx* ctx) {
  const int hkv = ctx->lay.num_kv_heads;
  if (ctx->lay.dtype == ECOSERVE_BF16)
    return hkv % 4 == 0 ? raise_lds_limit<uint16_t, 4>(ctx) : hkv % 2 == 0 ? raise_lds_limit<uint16_t, 2>(ctx)
                                                                          : raise_lds_limit<uint16_t, 1>(ctx);
  return hkv % 4 == 0 ? raise_lds_limit<float, 4>(ctx) : hkv % 2 == 0 ? raise_lds_limit<float, 2>(ctx)
                                                                      : raise_lds_limit<float, 1>(ctx);
}

hipError_t launch_kv_append(const ecoserve_ctx* ctx, void* k_cache, void* v_cache, const void* k_new,
                            const void* v_new, int32_t new_row_stride, const int32_t* cu_q,
                            const int32_t* ctx_before, const int32_t* block_table, int32_t bt_stride, int32_t B,
                            int32_t T, int32_t max_new_len, int32_t pos_bias, hipStream_t s) {
  const ecoserve_layout& L = ctx->lay;
  if (L.dtype == ECOSERVE_BF16)
    launch_typed<uint16_t>(L, k_cache, v_cache, k_new, v_new, new_row_stride, cu_q, ctx_before, block_table, bt_stride, B, T,
                           max_new_len, pos_bias, ctx->num_cu, s);
  else
    launch_typed<float>(L, k_cache, v_cache, k_new, v_new, new_row_stride, cu_q, ctx_before, block_table, bt_stride, B, T,
                        max_new_len, pos_bias, ctx->num_cu, s);
  return hipGetLastError();
}

}  // namespace eco
