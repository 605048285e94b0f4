// Attention of a short tail (a token or a line of dialogue) over the surviving + new KV:
// the same function as attention.hip, for launches whose packed query rows are few.
//
// Such a call reads the whole cache for a few rows, so it is bound by HBM, and by latency
// when the cache is short: what counts is how early and how widely the cache is requested.
// A workgroup takes 32 packed rows (t * G + h mod G) of one KV head and one split of the
// key range; its four waves (one per SIMD) take 32-key units of the split in turn, each
// alone: no barrier until the end. K and V units come by LDS DMA, whole cache lines at a
// time, into the wave's own K and V stages; K of the next unit is requested as soon as
// the scores of this one are formed, V as soon as its products are issued. V is read as
// it lies in the cache (bf16 rows) and transposed on the way into the MFMA operands by
// ds_read_b64_tr_b16: no V^T tile is packed or read, and without a V^T copy the call packs
// nothing at all.
//
// S^T = K Q^T on v_mfma_f32_32x32x16_bf16 as in attention.hip (a lane holds 16 keys of one
// query). P V runs on the bf16 MFMA too, with V's own bits: P is split into two bf16
// terms (16 significant bits, more than the f16 P of the long kernel), each multiplied by
// V and summed in fp32. The waves' results are merged through LDS, and the splits by
// k_attn_merge.
//
// Measured (16/2 heads of 256): one token over 32,768 rows 18.0 us (67 MB, 3.7 TB/s; the long
// kernel 24.2 us), the whole call 27.1 us with its RoPE and merge launches (33.7); 24
// tokens over 11,907 rows 22.3 us (28.5), the call 29.8 us without a V^T copy (41.4). K
// straight from global memory into operands (32 rows x 32 bytes per load) took 24.6 us for
// the latter; a copy through registers spilled.
//
// A row of D dims lies in LDS as D / 8 chunks of 16 bytes, permuted within the row so that
// the rows read together fall into different banks: chunk c of K row r at c ^ (r mod 16)
// (an operand read takes one chunk of 32 rows), of V row r at c ^ 2 (r mod 8) (a
// transposing read takes 4 rows x 16 dims per 16 lanes); less where a row has fewer chunks.
#include "attention_tile.h"

namespace tu {

namespace {

constexpr int kThreads = 256;          // 4 waves, each with units of its own
constexpr int kWaves = kThreads / 64;
constexpr int kRows = kShortRows;      // packed query rows of a workgroup
constexpr int kUnit = kShortKeys;

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// This wave's LDS reads have returned (their stage may be written again).
__device__ __forceinline__ void lds_reads_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
  asm volatile("" ::: "memory");
}

template <int B>
struct IntC {
  static constexpr int value = B;
};

// F32: contexts of the launch may have fp32 partial outputs (an instance of its own: the choice
// lengthens the kernel of 24 tokens over 11,907 rows by 0.4 us).
template <int D, bool F32>
__global__ __launch_bounds__(kThreads, D == 256 ? 1 : 2) void k_attn_short(AttnArgs a, CallStatus status) {
  constexpr int NS = D / 16;                 // 16-dim steps of S^T = K Q^T
  constexpr int NDB = D / 32;                // 32-dim blocks of O^T
  constexpr int RC = D / 8;                  // 16-byte chunks per V row
  constexpr int NL = RC / 2;                 // loads of a wave per K or V unit (32 x RC chunks)
  constexpr int LR = 64 / RC;                // rows per load
  constexpr int KSWZ = RC < 16 ? RC - 1 : 15;
  constexpr int VSWZ = RC / 2 < 8 ? RC / 2 - 1 : 7;
  constexpr int kStage = kUnit * D * 2;      // bytes of a unit
  // Two arrays, so that the compiler sees that the DMA into one does not alias the reads of
  // the other; the merge at the end reuses both.
  __shared__ __attribute__((aligned(16))) char g_k[kWaves * kStage];
  __shared__ __attribute__((aligned(16))) char g_v[kWaves * kStage];
  __shared__ float g_ml[kWaves][kRows][2];

  const int item = xcd_remap(blockIdx.x, gridDim.x);
  if (item >= a.total_items) return;
  int si = 0;
  while (si + 1 < a.n_seq && a.seq[si + 1].item_begin <= item) ++si;
  const AttnSeq& S = a.seq[si];
  int local = item - S.item_begin;
  const int tile = __builtin_amdgcn_readfirstlane(local % S.n_tiles);
  local /= S.n_tiles;
  const int split = __builtin_amdgcn_readfirstlane(local % S.n_splits);
  const int hkv = __builtin_amdgcn_readfirstlane(local / S.n_splits);

  const int Hq = a.n_q_heads, Hkv = a.n_kv_heads, G = Hq / Hkv;
  const int T = S.T, L_keep = S.L_keep;
  const int rows_total = T * G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hl = lane >> 5;     // half of the wave
  const int col = lane & 31;    // query column of this lane

  const int r = tile * kRows + col;
  const bool row_ok = r < rows_total;
  const int t = row_ok ? r / G : T - 1;
  const int qh = hkv * G + (row_ok ? r - (r / G) * G : 0);
  const int my_limit = L_keep + t;           // last key this query may see
  const int t_hi = (min(rows_total, (tile + 1) * kRows) - 1) / G;
  const int t_lo = __builtin_amdgcn_readfirstlane((tile * kRows) / G);
  const int n_units = (L_keep + t_hi + kUnit) / kUnit;          // units of keys 0 .. L_keep + t_hi
  const int ups = __builtin_amdgcn_readfirstlane((n_units + S.n_splits - 1) / S.n_splits);
  const int u_end = __builtin_amdgcn_readfirstlane(min(n_units, (split + 1) * ups));
  const int n_valid = L_keep + T;            // cache rows holding data
  const long rs = (long)Hkv * D;             // elements per cache row
  const bf16_t* kbase = S.k_cache + (long)hkv * D;
  const bf16_t* vbase = S.v_cache + (long)hkv * D;

  // ---- unit -> this wave's K or V stage. LDS chunk i * 64 + lane is written by load i of
  // the lane: row i * LR + lane / RC. The buffer resource ends at the cache's data: rows past
  // it are written as zeros. Units past the split's end are requested all the same, with
  // zero bytes: the loads in flight are then the same number at every step, which the waits
  // rely on.
  auto load = [&](char* dst, const bf16_t* head, auto swz, int u) __attribute__((always_inline)) {
    constexpr int SWZ = decltype(swz)::value;
    constexpr int MUL = SWZ == KSWZ ? 1 : 2;
    const int key0 = u * kUnit;
    const int bytes = u < u_end ? min(n_valid - key0, kUnit) * (int)rs * 2 - ((int)rs - D) * 2 : 0;
    const bf16_t* base = head + (long)key0 * rs;
    const int row0 = lane / RC, c = lane % RC;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = i * LR + row0;
      dma16(base, bytes, (uint32_t)(row * (int)rs * 2 + (c ^ (MUL * (row & SWZ))) * 16), 0, dst + i * 64 * 16);
    }
  };
  char* const my_k = g_k + wave * kStage;
  char* const my_v = g_v + wave * kStage;
  auto load_k = [&](int u) __attribute__((always_inline)) { load(my_k, kbase, IntC<KSWZ>{}, u); };
  auto load_v = [&](int u) __attribute__((always_inline)) { load(my_v, vbase, IntC<VSWZ>{}, u); };

  bf16x8 qf[NS];
  {
    const bf16_t* qrow = S.q_hat + ((long)t * Hq + qh) * D + 8 * hl;   // rows past the last repeat one (dropped)
#pragma unroll
    for (int s = 0; s < NS; ++s) qf[s] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + 16 * s));
  }

  f32x16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  float m_run = -__builtin_inff();   // lazily moved reference max (log2 units), as in attention.hip
  float l_run = 0.f;
  const float c2 = a.scale_log2;
  u16x2 big = {0, 0};                // largest |bf16| bits of V met

  // ---- transposing reads of V: lane group g reads keys 4 (g >> 1) + 0 .. 3 (+ 16 u + 8
  // part) at dims 32 db + 16 (g & 1) .. + 15; lane i of it gets dim i of the 16
  // K operand reads: key row col, chunk 2 s + hl
  const char* const krow = my_k + col * D * 2;
  uint32_t vaddr[NDB];
  {
    const int i = lane & 15, g = lane >> 4;
    const int row = 4 * (g >> 1) + (i >> 2);
    const int c0 = 2 * (g & 1) + ((i & 3) >> 1);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      vaddr[db] = (uint32_t)(row * D * 2 + (((4 * db + c0) ^ (2 * (row & VSWZ))) * 16) + (i & 1) * 8);
  }

  auto step = [&](int u, bool first) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(vm_wait(NL));   // K(u) has landed; V(u) may be in flight
    asm volatile("" ::: "memory");
    f32x16 sacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bf16x8 ka = __builtin_bit_cast(bf16x8, *(const u32x4*)(krow + (((2 * s + hl) ^ (col & KSWZ)) * 16)));
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[s], sacc, 0, 0, 0);
    }
    lds_reads_done();
    load_k(u + kWaves);
    const int kb0 = u * kUnit;
    if (kb0 + kUnit - 1 > L_keep + t_lo) {   // crosses the tail diagonal (uniform)
      const int room = my_limit - kb0 - 4 * hl;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + (e & 3) > room) sacc[e] = -__builtin_inff();
    }
    float mx = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sacc[e]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, mx),
                                                     __builtin_bit_cast(uint32_t, mx), false, false);
    mx = fmaxf(__builtin_bit_cast(float, (uint32_t)sw[0]), __builtin_bit_cast(float, (uint32_t)sw[1])) * c2;
    if (first) {
      m_run = mx;
    } else if (__any(mx > m_run + kTau)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_new == -__builtin_inff() ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db) scale_acc(o[db], alpha);
    }
    const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;
    bf16x8 ph[2], pl[2];
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e], c2, -m_use));
      ps[e & 3] += p;
      const __bf16 hi = (__bf16)p;
      ph[e >> 3][e & 7] = hi;
      pl[e >> 3][e & 7] = (__bf16)(p - (float)hi);
    }
    l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
    __builtin_amdgcn_s_waitcnt(vm_wait(NL));   // V(u) has landed; K(u + kWaves) may be in flight
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 va[NDB];
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const s16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(my_v + vaddr[db] + (16 * ks) * D * 2));
        const s16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(my_v + vaddr[db] + (16 * ks + 8) * D * 2));
        const u32x2 w0 = __builtin_bit_cast(u32x2, x0), w1 = __builtin_bit_cast(u32x2, x1);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          big = __builtin_elementwise_max(big, __builtin_bit_cast(u16x2, w0[e] & 0x7FFF7FFFu));
          big = __builtin_elementwise_max(big, __builtin_bit_cast(u16x2, w1[e] & 0x7FFF7FFFu));
        }
        va[db] = __builtin_bit_cast(bf16x8, u32x4{w0[0], w0[1], w1[0], w1[1]});
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], ph[ks], o[db], 0, 0, 0);
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], pl[ks], o[db], 0, 0, 0);
    }
    lds_reads_done();
    load_v(u + kWaves);
  };

  {
    const int u0 = split * ups + wave;
    if (u0 < u_end) {
      load_k(u0);
      load_v(u0);
      for (int u = u0; u < u_end; u += kWaves) step(u, u == u0);
      __builtin_amdgcn_s_waitcnt(vm_wait(0));   // the stages are rewritten below
    }
  }
  if (S.check_range && max((int)big[0], (int)big[1]) >= 0x4780) status_raise(status, kFaultRange);   // 0x4780: bf16 bits of 2^16

  // ---- merge of the four waves: each scales its O to the common reference and the total
  // sum and writes it (fp32) over the dead V stages; the rows are then added up
  const auto lsw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, l_run),
                                                    __builtin_bit_cast(uint32_t, l_run), false, false);
  const float l_tot = __builtin_bit_cast(float, (uint32_t)lsw[0]) + __builtin_bit_cast(float, (uint32_t)lsw[1]);
  if (hl == 0) {
    g_ml[wave][col][0] = m_run;
    g_ml[wave][col][1] = l_tot;
  }
  __syncthreads();
  float M = -__builtin_inff(), L = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, g_ml[w][col][0]);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float mw = g_ml[w][col][0];
    L += mw == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(mw - M) * g_ml[w][col][1];
  }
  const float f = m_run == -__builtin_inff() || !(L > 0.f) ? 0.f : __builtin_amdgcn_exp2f(m_run - M) / L;
  // chunk c (4 dims) of query row col of wave w at chunk c ^ (col mod 16) of the row
  auto wave_o = [&](int w) __attribute__((always_inline)) {
    return (float*)((w & 2 ? g_v : g_k) + (w & 1) * (kRows * D * 4));
  };
  {
    float* mine = wave_o(wave) + col * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = (8 * db + 2 * i + hl) ^ (col & 15);
        *(f32x4*)(mine + 4 * c) = f32x4{o[db][4 * i] * f, o[db][4 * i + 1] * f, o[db][4 * i + 2] * f, o[db][4 * i + 3] * f};
      }
  }
  __syncthreads();
  const int n_rows = min(kRows, rows_total - tile * kRows);
  const int h0 = hkv * G;
  for (int e = tid; e < n_rows * (D / 4); e += kThreads) {
    const int rr = e / (D / 4), c = e - rr * (D / 4);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += *(const f32x4*)(wave_o(w) + rr * D + 4 * (c ^ (rr & 15)));
    const int row = tile * kRows + rr, tt = row / G;
    const long at = (long)tt * Hq + h0 + (row - tt * G);
    if (S.n_splits == 1) {
      *(f32x4*)(S.out + at * D + 4 * c) = sum;
    } else if (F32 && S.part_f32) {
      *(f32x4*)((float*)S.part_o + ((long)split * T * Hq + at) * D + 4 * c) = sum;
    } else {
      const f16x4 hv = {(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
      *(f16x4*)((_Float16*)S.part_o + ((long)split * T * Hq + at) * D + 4 * c) = hv;
    }
  }
  if (S.n_splits > 1 && wave == 0 && hl == 0 && row_ok) {
    const long prow = (long)split * T * Hq + (long)t * Hq + qh;
    S.part_ml[prow * 2] = L > 0.f ? M : -__builtin_inff();
    S.part_ml[prow * 2 + 1] = L;
  }
}

}  // namespace

static_assert(sizeof(AttnArgs) + sizeof(CallStatus) <= kMaxKernargBytes, "short attention launch record");

hipError_t launch_attention_short(const AttnArgs& a, const CallStatus& status, int head_dim, hipStream_t s) {
  if (a.total_items <= 0) return hipSuccess;
  const int blocks = (a.total_items + kXcds - 1) / kXcds * kXcds;   // a whole number per die (xcd_remap)
  bool f32 = false;
  for (int i = 0; i < a.n_seq; ++i) f32 = f32 || (a.seq[i].n_splits > 1 && a.seq[i].part_f32);
  const auto run = [&](auto f16_only, auto any) {
    if (f32) hipLaunchKernelGGL(any, dim3(blocks), dim3(kThreads), 0, s, a, status);
    else hipLaunchKernelGGL(f16_only, dim3(blocks), dim3(kThreads), 0, s, a, status);
    return hipGetLastError();
  };
  switch (head_dim) {
    case 256: return run(k_attn_short<256, false>, k_attn_short<256, true>);
    case 128: return run(k_attn_short<128, false>, k_attn_short<128, true>);
    case 64: return run(k_attn_short<64, false>, k_attn_short<64, true>);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tu
