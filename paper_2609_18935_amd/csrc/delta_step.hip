// Gated delta rule of a few tokens (a character speaking, a line of dialogue): the
// recurrence itself, token by token in fp32, in one launch without a workspace.
//
//     u_t = beta_t (v_t - g_t S k_t),   S <- g_t S + u_t k_t^T,   o_t = scale S q_t
//
// The chunked form of delta.hip spends two launches and a chunk's whole inverse on any
// tail (10.1 + 5.7 us for one token); here one token costs the read and write of the
// state plus two dot products per row. Rows of S are independent: a workgroup takes 16 rows
// of one value head, 16 lanes a row, each lane DK / 16 columns in registers from the first
// token to the last, so 32 heads of 128 rows fill the 256 CUs. k, q, v and the gates of all
// tokens are staged in LDS first; a row's dot products are summed over its 16 lanes by DPP
// rotations. Serial over tokens (about 0.2 us each): for at most kStepTokens of them.
//
// Nothing is rounded to f16 here; q, k, v, u or S of magnitude 2^16 or more are reported
// all the same, as by the chunked form.
#include "common.h"

namespace tu {

namespace {

constexpr int kThreads = 256;
constexpr int kRows = kStepRows;
constexpr int kLanes = kThreads / kRows;   // lanes of a row: one DPP row
static_assert(kLanes == 16, "a state row is one DPP row");
constexpr float kF16Max = 65504.f;

template <int ROT>
__device__ __forceinline__ float add_rotated(float x) {   // x + the value ROT lanes on in the row of 16
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + ROT, 0xf, 0xf,
                                                                   true));
}

// Sum over the 16 lanes of a row, the same bits in each of them.
__device__ __forceinline__ float row_sum(float x) {
  return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(x))));
}

template <int N>
__device__ __forceinline__ void load_bf16(const bf16_t* p, float (&f)[N]) {   // N = 4 or 8, from LDS
  uint32_t w[N / 2];
  if constexpr (N == 8) {
    const u32x4 x = *(const u32x4*)p;
    w[0] = x[0], w[1] = x[1], w[2] = x[2], w[3] = x[3];
  } else {
    const u32x2 x = *(const u32x2*)p;
    w[0] = x[0], w[1] = x[1];
  }
#pragma unroll
  for (int e = 0; e < N / 2; ++e) {
    f[2 * e] = __uint_as_float(w[e] << 16);
    f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
  }
}

template <int DK>
__global__ __launch_bounds__(kThreads) void k_delta_step(DeltaArgs a) {
  constexpr int NC = DK / kLanes;      // columns of a lane
  constexpr int NSL = DK / kRows;      // workgroups of a head
  constexpr int V8 = DK / 8;           // 16-byte vectors of a q or k row
  __shared__ __attribute__((aligned(16))) bf16_t s_k[kStepTokens * DK];
  __shared__ __attribute__((aligned(16))) bf16_t s_q[kStepTokens * DK];
  __shared__ __attribute__((aligned(16))) bf16_t s_v[kStepTokens * kRows];
  __shared__ float s_bg[kStepTokens][2];
  // (context, key head, value head of its group, rows): the workgroups of one key head
  // share a die's L2
  const int Hv = a.n_v_heads, Hk = a.n_k_heads, G = Hv / Hk;
  const int item = xcd_remap(blockIdx.x, gridDim.x);
  const int si = item / (Hv * NSL);
  if (si >= a.n_seq) return;
  const int rem = item - si * Hv * NSL;
  const int h = rem / NSL, kh = h / G;
  const int i0 = (rem - h * NSL) * kRows;
  const DeltaSeq S = a.seq[si];
  const int T = S.T;
  const int tid = threadIdx.x, row = tid / kLanes, l = tid % kLanes;
  status_mark(a.status);

  float* sp = S.state + ((long)h * DK + i0 + row) * DK + NC * l;
  float st[NC];
#pragma unroll
  for (int c = 0; c < NC; c += 4) {
    const f32x4 x = *(const f32x4*)(sp + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) st[c + e] = x[e];
  }
  // largest |bf16| of q, k, v staged by this thread (two per word); fmaxf passes over NaN, which
  // is no overflow, as the chunked form does
  float big = 0.f;
  auto seen = [&](u32x4 w) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      big = fmaxf(big, fmaxf(fabsf(__uint_as_float(w[e] << 16)), fabsf(__uint_as_float(w[e] & 0xFFFF0000u))));
  };
  for (int e = tid; e < T * V8; e += kThreads) {
    const int t = e / V8, c = (e - t * V8) * 8;
    const long off = ((long)t * Hk + kh) * DK + c;
    const u32x4 kw = *(const u32x4*)(S.k + off), qw = *(const u32x4*)(S.q + off);
    seen(kw);
    seen(qw);
    *(u32x4*)(s_k + t * DK + c) = kw;
    *(u32x4*)(s_q + t * DK + c) = qw;
  }
  for (int e = tid; e < T * (kRows / 8); e += kThreads) {
    const int t = e / (kRows / 8), c = (e - t * (kRows / 8)) * 8;
    const u32x4 vw = *(const u32x4*)(S.v + ((long)t * Hv + h) * DK + i0 + c);
    seen(vw);
    *(u32x4*)(s_v + t * kRows + c) = vw;
  }
  for (int t = tid; t < T; t += kThreads) {
    s_bg[t][0] = S.beta[(long)t * Hv + h];
    s_bg[t][1] = fmaxf(S.g[(long)t * Hv + h], 0x1p-100f);   // as the chunked form holds log2 g
  }
  __syncthreads();

#pragma unroll
  for (int c = 0; c < NC; ++c) big = fmaxf(big, fabsf(st[c]));
  float* out = S.out + (long)h * DK + i0 + row;
  float kf[NC], qf[NC];
  load_bf16<NC>(s_k + NC * l, kf);
  load_bf16<NC>(s_q + NC * l, qf);
  float vt = bf16_to_f32(s_v[row]), beta = s_bg[0][0], g = s_bg[0][1];
  for (int t = 0; t < T; ++t) {
    // the next token's operands, read while this one's sums are formed
    const int n = min(t + 1, T - 1);
    float kn[NC], qn[NC];
    load_bf16<NC>(s_k + n * DK + NC * l, kn);
    load_bf16<NC>(s_q + n * DK + NC * l, qn);
    const float vn = bf16_to_f32(s_v[n * kRows + row]), bn = s_bg[n][0], gn = s_bg[n][1];
    float d0 = 0.f, d1 = 0.f;
#pragma unroll
    for (int c = 0; c < NC; c += 2) {
      st[c] *= g;
      st[c + 1] *= g;
      d0 = __builtin_fmaf(st[c], kf[c], d0);
      d1 = __builtin_fmaf(st[c + 1], kf[c + 1], d1);
    }
    const float u = beta * (vt - row_sum(d0 + d1));
    big = fmaxf(big, fabsf(u));
    float o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int c = 0; c < NC; c += 2) {
      st[c] = __builtin_fmaf(u, kf[c], st[c]);
      st[c + 1] = __builtin_fmaf(u, kf[c + 1], st[c + 1]);
      o0 = __builtin_fmaf(st[c], qf[c], o0);
      o1 = __builtin_fmaf(st[c + 1], qf[c + 1], o1);
    }
    const float o = row_sum(o0 + o1);
    if (l == 0) out[(long)t * Hv * DK] = a.scale * o;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      kf[c] = kn[c];
      qf[c] = qn[c];
    }
    vt = vn;
    beta = bn;
    g = gn;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) big = fmaxf(big, fabsf(st[c]));
#pragma unroll
  for (int c = 0; c < NC; c += 4) *(f32x4*)(sp + c) = f32x4{st[c], st[c + 1], st[c + 2], st[c + 3]};
  if (big > kF16Max) status_raise(a.status, kFaultRange);
}

}  // namespace

hipError_t launch_delta_step(const DeltaArgs& a, int d, hipStream_t s) {
  const int blocks = (a.n_seq * a.n_v_heads * (d / kRows) + 7) & ~7;   // xcd_remap wants a multiple of 8
  if (blocks <= 0) return hipSuccess;
  if (d == 128)
    hipLaunchKernelGGL(k_delta_step<128>, dim3(blocks), dim3(kThreads), 0, s, a);
  else if (d == 64)
    hipLaunchKernelGGL(k_delta_step<64>, dim3(blocks), dim3(kThreads), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace tu
