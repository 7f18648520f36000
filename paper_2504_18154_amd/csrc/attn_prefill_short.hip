// Causal prefill attention over the paged cache for batches behind short contexts, bf16, head size 128, on gfx950 matrix cores.
//
// Eq. 2 of Section 2.1, the same arithmetic per row as attn_prefill_mfma.hip (weights rounded to bf16, the row sum from the
// rounded weights, the exponent offset raised only when a score exceeds it by more than 2^8).
//
// What bounds such a batch is not arithmetic but what stands around it: a list of tiles to be made first, a workgroup's change
// from one tile of two or three key steps to the next, barriers, copies through LDS.  Here a wavefront takes 32 or 64 rows ((position,
// query head of the group) pairs of one sequence and K/V head, as there), finds its sequence by itself (find_sequence), and reads K and V
// straight into the operand layout of v_mfma_f32_32x32x16_bf16: the cache layouts are such that a lane's 16 bytes are
// consecutive in a block.  No plan, no queue, no barrier: the hardware hands out the wavefronts, longest first.
//   K, 32 keys x 16 d per product: lane (col, half) reads unit 2 t + half of its token of the two blocks;
//   V, 32 d x 16 keys: lane (col, half) reads octet `half` of row 32 dt + col.
// Rows of S^T are assigned to keys with bits 2 and 3 swapped, so a lane's accumulator registers are the second product's operand.
// A step is a group of 32 keys (two cache blocks); each operand's registers are asked for again as soon as its products have
// read them.  Query and output rows pass through LDS (8 KiB per 32 rows): along memory they move as whole rows, four per instruction.  Read
// and written by the lanes that hold them (32 bytes of 32 rows per instruction) they kept the address unit busy for as long as
// all of K and V (40 query heads on 8, 446 x 80 tokens behind 50..100, 32 rows: 331 -> 306 us; 52 on 52, 79 x 4..155 77 -> 71), and as
// registers the query rows would leave no room for 64 rows at two wavefronts per SIMD.
//   NC: sets of 32 rows per wavefront.  64 rows share the operands of K and V: half the reads of the first-level cache, whose address
//     unit, three quarters busy with 32 rows, bounds the larger batches (446 x 80: 306 -> 251 us, 22 x 431 171 -> 138); 32 rows
//     end sooner where there are few (93 tokens 5.8, with 64 rows 7.9).
//   kWaves 4: the four wavefronts of a workgroup take every fourth group of the same 32 rows and their states are combined
//     through LDS: where there are too few rows to fill the chip a walk is the whole time (93 tokens 4.8 us, 256 6.7; 11.1 each by itself).
// Against the persistent kernel with its list made (prefill_short.h has the line between them): 93 tokens 8.4 -> 4.8, 446 x 80 334 -> 251,
// 52 heads, 128 x 22 114 -> 55 us.  Tried: wavefronts that stay and prefetch their next tile (446 x 80 with 32 rows 331 -> 367: the
// address unit, not the latency, is what they wait for), two chains of score products (no difference with two wavefronts per
// SIMD), weights of one set under the products of the other throughout (spills).
#include "common.h"
#include "prefill_short.h"

namespace eco {

namespace {

constexpr float kRaiseBy = 8.f;  // lazy rescaling, log2 units
typedef const void __attribute__((address_space(1)))* gptr_t;
typedef void __attribute__((address_space(3)))* lptr_t;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float over_halves(float v, bool max) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
  return max ? fmaxf(a, b) : a + b;
}

template <int NC, int kWaves>
__global__ __launch_bounds__(kWaves * 64, kWaves > 1 || NC > 1 ? 2 : 3) void prefill_short_kernel(
    const uint16_t* __restrict__ q, int q_row_stride, const char* __restrict__ k_cache, const char* __restrict__ v_cache,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ ctx_before, const int32_t* __restrict__ block_table, int bt_stride,
    uint16_t* __restrict__ out, float* __restrict__ lse, int B, int n_tiles, int Hq, int Hkv, int G, Divisor div_g, Divisor div_hkv,
    float scale_log2e) {
  constexpr bool kSplit = kWaves > 1;
  constexpr int kRows = 32 * NC;
  static_assert(!kSplit || NC == 1, "one set of rows per workgroup");
  __shared__ __attribute__((aligned(16))) char s_rows[kRows * 256];  // the tile's query rows, then (kWaves 1) its output rows
  __shared__ float s_m[kSplit ? kWaves : 1][32], s_l[kSplit ? kWaves : 1][32];
  __shared__ __attribute__((aligned(16))) float s_o[kSplit ? kWaves : 1][kSplit ? 4 : 1][kSplit ? 4 : 1][kSplit ? 256 : 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = kSplit ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int col = lane & 31, half = lane >> 5;
  const float c = scale_log2e;

  // Unit w is K/V head w % Hkv of tile n_tiles - 1 - w / Hkv: later tiles of a sequence are longer and go first.  Workgroups go to the
  // XCDs in turn.  With eight K/V heads, unit for workgroup, a head stays with one XCD, whose cache then holds what its tiles share; with fewer
  // than eight an XCD takes eight units in a row out of 64, the tiles of a sequence or two (us in turn / in a row: 8 on 1, 250 x 25 tokens behind
  // 43..86 19.5 / 15.2, 366 x 15 behind up to 113 14.9 / 11.8, 5 on 1, 414 x 26 13.0 / 10.4, 76 x 24 behind ~260, keys shared, 12.0 / 9.6; 223 batches
  // of 8 on 1 and 5 on 1: 32 rows 0.94 of the time, 64 rows and keys shared 0.965, the worst 1.08 of 4 us).
  int w = blockIdx.x;
  if (Hkv < 8 && w < (int)(gridDim.x & ~63u)) w = (w & ~63) | (w & 7) << 3 | (w >> 3 & 7);
  const int unit = fast_div(w, div_hkv), tile_no = n_tiles - 1 - unit, g = w - unit * Hkv;
  auto first_tile = [&](int cu, int b) { return (long long)cu * G / kRows + b; };
  const SeqOf seq = find_sequence(cu_q, ctx_before, B, tile_no, first_tile);
  const int tok0 = seq.tok0, cb = seq.cb, L = cb + seq.S, n_rows = seq.S * G;
  const long long tile_r0 = (tile_no - first_tile(tok0, seq.b)) * kRows;
  if (tile_r0 >= n_rows) return;
  const int r0 = __builtin_amdgcn_readfirstlane((int)tile_r0);
  // groups of 32 keys up to the last key that one of the rows sees; this wavefront's: grp0 + kWaves i, i < n
  const int n_groups = __builtin_amdgcn_readfirstlane((cb + fast_div(min(n_rows, r0 + kRows) - 1, div_g) + 32) >> 5);
  const int grp0 = kSplit ? wave : 0, n = kSplit ? (n_groups - wave + kWaves - 1) / kWaves : n_groups;
  const int32_t* const bt_row = block_table + (size_t)seq.b * bt_stride;
  // lane l has the id of block l & 1 of group l / 2 (none behind the sequence's last): at most 32 groups (kShortMostKeys)
  const int ids = (lane >> 1) < n ? bt_row[min(2 * (grp0 + kWaves * (lane >> 1)) + (lane & 1), ((L + 15) >> 4) - 1)] : 0;

  // Rows in LDS: the 16-byte chunk k of row r lies at 256 r + 16 (k ^ (r & 15)): whole rows come and go along memory, four per
  // instruction, and 16 lanes that want chunk k of 16 rows find them in different banks.  Of the query rows, those that do not
  // exist are copies of the last.
#pragma unroll
  for (int i = grp0; i < 8 * NC; i += kWaves) {
    const int r = 4 * i + (lane >> 4), row = min(r0 + r, n_rows - 1), pos = fast_div(row, div_g);
    const uint16_t* const src = q + (size_t)(tok0 + pos) * q_row_stride + (g * G + row - pos * G) * 128 + ((lane ^ r) & 15) * 8;
    __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(s_rows + i * 1024), 16, 0, 0);
  }
  // (chunk k + half of row col is 16 k away in its exclusive or; worked out where it is wanted: kept, the addresses take the
  // registers of the operands)
  auto row_chunks = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return (ln & 31) * 256 + (((ln >> 5) ^ ln) & 15) * 16;
  };
  // position and head of this lane's row of set x
  auto map_row = [&](int x, int& pos, int& head) {
    const int row = min(r0 + 32 * x + col, n_rows - 1);
    pos = fast_div(row, div_g);
    head = row - pos * G;
  };

  const size_t blk_stride = (size_t)Hkv * 4096, head_off = (size_t)g * 4096;
  bf16x8 kf[8], vf[2][4];
  auto load_k = [&](int i) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // (lane offsets are worked out here: kept, they cost the operands' registers)
    const int id0 = __builtin_amdgcn_readlane(ids, 2 * i), id1 = __builtin_amdgcn_readlane(ids, 2 * i + 1);
    const int token = (ln & 3) | (ln & 4) << 1 | (ln & 8) >> 1;  // this lane's row of K: key (lane & 16) + token
    const char* const p = k_cache + head_off + (size_t)(ln & 16 ? id1 : id0) * blk_stride + ((ln >> 5) * 256 + token * 16);
#pragma unroll
    for (int t = 0; t < 8; ++t) kf[t] = *reinterpret_cast<const bf16x8*>(p + t * 512);
  };
  auto load_v = [&](int i) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int off = (ln & 31) * 32 + (ln >> 5) * 16;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const char* const p = v_cache + (size_t)__builtin_amdgcn_readlane(ids, 2 * i + u) * blk_stride + head_off;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) vf[u][dt] = *reinterpret_cast<const bf16x8*>(p + off + dt * 1024);
    }
  };

  f32x16 o[NC][4];
  float m[NC], l[NC];
#pragma unroll
  for (int x = 0; x < NC; ++x) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[x][dt][i] = 0.f;
    m[x] = -INFINITY;
    l[x] = 0.f;
  }
  // register 8 u + e of the scores: key 16 u + 8 half + e of the group.  Those that a row does not see:
  auto mask = [&](f32x16& s, int x, int first) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int bound = cb + fast_div(min(r0 + 32 * x + (ln & 31), n_rows - 1), div_g) - first - (ln >> 5) * 8;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if ((e >> 3) * 16 + (e & 7) > bound) s[e] = -INFINITY;
  };
  // the exponent offset follows the maximum
  auto offset = [&](const f32x16& s, int x) {
    float bm = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
    for (int e = 3; e < 15; e += 2) bm = fmaxf(fmaxf(bm, s[e]), s[e + 1]);
    bm = over_halves(fmaxf(bm, s[15]), true);
    if (__any((bm - m[x]) * c > kRaiseBy)) {
      const float m_new = fmaxf(m[x], bm);
      if (__any(m[x] != -INFINITY)) {  // (not a tile's first group)
        const float alpha = m[x] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[x] - m_new) * c);
        l[x] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[x][dt] *= alpha;
      }
      m[x] = m_new;
    }
  };
  auto weights = [&](const f32x16& s, bf16x8 (&p)[2], int x) {
    const float mc = m[x] == -INFINITY ? 0.f : m[x] * c;  // (a row whose scores so far are all minus infinity)
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 a = {(__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * u + e], c, -mc)),
                          (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * u + e + 1], c, -mc))};
        l[x] = __builtin_amdgcn_fdot2_f32_bf16(a, ones, l[x], false);
        p[u][e] = a[0];
        p[u][e + 1] = a[1];
      }
  };
  // stale values behind the end of the sequence must not meet their zero weights
  auto clear_tail = [&](int first) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int left = L - first - (ln >> 5) * 8;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      u32x4 keep;
#pragma unroll
      for (int e = 0; e < 4; ++e) keep[e] = 16 * u + 2 * e + 1 < left ? 0xffffffffu : 16 * u + 2 * e < left ? 0xffffu : 0u;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        vf[u][dt] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[u][dt]) & keep);
        // (whole from here on, and not joined with the other path element by element.  In all three instances the registers that are cleared are
        // those that the products read, and nothing writes to them between)
        asm volatile("" : "+v"(vf[u][dt]));
      }
    }
  };

  if (!kSplit || n > 0) {
    load_k(0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the query rows are in LDS
  if constexpr (kSplit) __syncthreads();
  if (!kSplit || n > 0) {
    int i = 0;
#pragma clang loop unroll(disable)
    for (;;) {
      const int first = (grp0 + kWaves * i) << 5;
      const bool more = i + 1 < n;
      f32x16 s[NC];
      bf16x8 p[NC][2];
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int x = 0; x < NC; ++x) s[x][i] = 0.f;
      const int at = row_chunks();
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int x = 0; x < NC; ++x)
          s[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j], *reinterpret_cast<const bf16x8*>(s_rows + x * 8192 + (at ^ (32 * j))), s[x], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * NC, 0);  // (query rows are read two products ahead)
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, NC, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, NC, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * NC, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (more) load_k(i + 1);
      if (first + 32 > cb + fast_div(r0, div_g) + 1) {  // (keys that not every row sees, or that do not exist)
        asm volatile("" ::: "memory");  // (a real branch)
#pragma unroll
        for (int x = 0; x < NC; ++x) mask(s[x], x, first);
        if (first + 32 > L) clear_tail(first);
      }
#pragma unroll
      for (int x = 0; x < NC; ++x) offset(s[x], x);
      weights(s[0], p[0], 0);
#pragma unroll
      for (int x = 0; x < NC; ++x) {
        __builtin_amdgcn_sched_barrier(0);
        if (x + 1 < NC) weights(s[x + 1], p[x + 1], x + 1);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) o[x][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][dt], p[x][u], o[x][dt], 0, 0, 0);
        if (x + 1 < NC)
#pragma unroll
          for (int k = 0; k < 8; ++k) {  // a product, then the vector instructions of two weights of the next set
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x402, 6, 0);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (!more) break;
      load_v(++i);
    }
  }
#pragma unroll
  for (int x = 0; x < NC; ++x) l[x] = over_halves(l[x], false);

  // Registers 4 i4 .. + 3 of o[][dt] hold d = 32 dt + 8 i4 + 4 half + (0..3): the two lanes of a row exchange halves, and chunk
  // 4 dt + 2 p + half of the row is complete (as in attn_prefill_mfma.hip).
  auto pack_chunk = [&](const f32x16& v, int p, float inv) {
    auto pack = [&](float a, float b) { return pack_bf16x2(a * inv, b * inv); };
    const auto a = __builtin_amdgcn_permlane32_swap(pack(v[8 * p + 0], v[8 * p + 1]), pack(v[8 * p + 4], v[8 * p + 5]), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(pack(v[8 * p + 2], v[8 * p + 3]), pack(v[8 * p + 6], v[8 * p + 7]), false, false);
    return u32x4{a[0], b[0], a[1], b[1]};
  };
  if constexpr (!kSplit) {
    const int at = row_chunks();
#pragma unroll
    for (int x = 0; x < NC; ++x) {
      const float inv = 1.f / l[x];
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int p = 0; p < 2; ++p) *reinterpret_cast<u32x4*>(s_rows + x * 8192 + (at ^ (64 * dt + 32 * p))) = pack_chunk(o[x][dt], p, inv);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int ln = lane;
    asm volatile("" : "+v"(ln));  // (not the addresses of the query rows, kept)
    u32x4 rows[8 * NC];
#pragma unroll
    for (int i = 0; i < 8 * NC; ++i) rows[i] = *reinterpret_cast<const u32x4*>(s_rows + i * 1024 + ln * 16);
#pragma unroll
    for (int i = 0; i < 8 * NC; ++i) {
      const int r = 4 * i + (ln >> 4), row = r0 + r, pos = fast_div(row, div_g);
      if (row < n_rows)
        *reinterpret_cast<u32x4*>(out + ((size_t)(tok0 + pos) * Hq + g * G + row - pos * G) * 128 + ((ln ^ r) & 15) * 8) = rows[i];
    }
    if (lse && half == 0)
#pragma unroll
      for (int x = 0; x < NC; ++x)
        if (r0 + 32 * x + col < n_rows) {
          int pos, head;
          map_row(x, pos, head);
          lse[(size_t)(tok0 + pos) * Hq + g * G + head] = (m[x] * c + log2f(l[x])) * kLn2;
        }
  } else {
    //   M = max_w m_w;  l = sum_w l_w 2^(m_w - M);  o = sum_w o_w 2^(m_w - M) / l:  wavefront dt takes d 32 dt .. + 31
    if (half == 0) {
      s_m[wave][col] = m[0];
      s_l[wave][col] = l[0];
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      if (dt != wave)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          *reinterpret_cast<f32x4*>(&s_o[wave][dt][p][lane * 4]) =
              f32x4{o[0][dt][4 * p], o[0][dt][4 * p + 1], o[0][dt][4 * p + 2], o[0][dt][4 * p + 3]};
    __syncthreads();
    float M = s_m[0][col];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w][col]);
    float total = 0.f, wk[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      wk[w] = s_m[w][col] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s_m[w][col] - M) * c);
      total += s_l[w][col] * wk[w];
    }
    f32x16 v;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      if (dt == wave) v = o[0][dt] * wk[dt];
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
      if (w != wave)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const f32x4 y = *reinterpret_cast<const f32x4*>(&s_o[w][wave][p][lane * 4]);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * p + e] += y[e] * wk[w];
        }
    int pos, head;
    map_row(0, pos, head);
    const bool ok = r0 + col < n_rows;
    const size_t row = (size_t)(tok0 + pos) * Hq + g * G + head;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const u32x4 w = pack_chunk(v, p, 1.f / total);
      if (ok) *reinterpret_cast<u32x4*>(out + row * 128 + (4 * wave + 2 * p + half) * 8) = w;
    }
    if (lse && wave == 0 && half == 0 && ok) lse[row] = (M * c + log2f(total)) * kLn2;
  }
}

}  // namespace

hipError_t launch_prefill_short(const AttnArgs& a, const int32_t* cu_q, const int32_t* ctx_before, int32_t T, PrefillShort how, hipStream_t s) {
  const int G = a.Hq / a.Hkv;
  auto launch = [&](auto kernel, int rows, int waves) {
    const int64_t n_tiles = (int64_t)T * G / rows + a.B, units = n_tiles * a.Hkv;
    if (units > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, dim3((unsigned)units), dim3(waves * 64), 0, s, (const uint16_t*)a.q, a.q_row_stride, (const char*)a.k_cache,
                       (const char*)a.v_cache, cu_q, ctx_before, a.block_table, a.bt_stride, (uint16_t*)a.out, a.lse, a.B, (int)n_tiles, a.Hq, a.Hkv, G,
                       make_divisor((uint32_t)G), make_divisor((uint32_t)a.Hkv), a.scale_log2e);
    return hipGetLastError();
  };
  if (how == PrefillShort::kRows64) return launch(prefill_short_kernel<2, 1>, 64, 1);
  if (how == PrefillShort::kRows32) return launch(prefill_short_kernel<1, 1>, 32, 1);
  return launch(prefill_short_kernel<1, 4>, 32, 4);
}

}  // namespace eco
