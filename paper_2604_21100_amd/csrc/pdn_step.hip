// The forward over a few tokens (decoding) as the token recurrence itself:
//   A_t  = exp(gP_t) A_{t-1} + betaP_t k_t^2       kt_t = write key of A_t, k_t
//   e_t  = beta_t (v_t - (alpha_t S_{t-1}) k_t)    S_t  = alpha_t S_{t-1} + kt_t e_t
//   o_t  = scale S_t q_t = scale ((alpha_t S_{t-1}) q_t + (kt_t . q_t) e_t)
// One launch, fp32 throughout, no workspace.  A workgroup holds one head's 32
// value columns of S^T in registers (d_k / 32 rows x 4 columns a thread);
// both products with S go through one reduction, so a token costs two
// barriers (three where the write key needs a row sum first).
//
// What bounds it: at one token, reading and writing the state, 128 KB a head
// at d = 128 (16 sequences of 16 heads: 34 MB, 6.6 us at the copy rate; the
// kernel takes 8.0 us and the call 11.3, host included, against 41 through the
// chunk kernels, which spend four dependent launches and a 64-token chunk's work
// on it).  With more tokens, the two barriers and the reduction of each, 1.2 us.
#include "pdn_device.hpp"
#include "pdn_internal.hpp"

namespace pdn {

namespace {

constexpr int kStepCols = 32;

// sum over the wave, in every lane
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

template <typename T, int DK, int GATE, int PREC>
__global__ __launch_bounds__(256) void step_tokens(FwdArgs a) {
  constexpr int R = DK / 32;         // state rows a thread holds
  constexpr int KW = DK / 64;        // waves with key channels
  constexpr bool ROWSUM = PREC == kDiagSM || PREC == kSquash;   // (squash: only with a normalisation)
  // (two buffers: a token's writes do not wait for the previous one's reads)
  __shared__ __attribute__((aligned(16))) float sK[2][DK], sQ[2][DK], sKt[2][DK], sLam[2][GATE == kGateChannel ? DK : 4];
  __shared__ __attribute__((aligned(16))) float sRed[2][4][2][kStepCols];
  __shared__ float sDot[2][KW], sSum[2][KW];
  const int nslab = a.dv / kStepCols;
  const int64_t bh = blockIdx.x / nslab, b = bh / a.H, h = bh % a.H;
  const int v0 = static_cast<int>(blockIdx.x % nslab) * kStepCols;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, cg = tid & 7, r0 = (tid >> 3) * R;
  const bool key = tid < DK;
  const int c = tid % DK;
  const int64_t HK = a.H * static_cast<int64_t>(DK), HV = a.H * static_cast<int64_t>(a.dv);
  const T* kp = static_cast<const T*>(a.k) + (b * a.T * a.H + h) * DK + c;
  const T* qp = static_cast<const T*>(a.q) + (b * a.T * a.H + h) * DK + c;
  const T* xp = PREC == kExternal ? static_cast<const T*>(a.ktilde) + (b * a.T * a.H + h) * DK + c : nullptr;
  const T* vp = static_cast<const T*>(a.v) + (b * a.T * a.H + h) * a.dv + v0 + 4 * cg;
  T* op = static_cast<T*>(a.o) + (b * a.T * a.H + h) * a.dv + v0 + 4 * cg;
  using V4 = typename Vec4<T>::type;
  // ---- the first token's inputs, then the state
  float kv = to_f(kp[0]), qv = to_f(qp[0]), xv = PREC == kExternal ? to_f(xp[0]) : 0.f;
  V4 vv = *reinterpret_cast<const V4*>(vp);
  const int64_t s0 = b * a.T * a.H + h;
  float be = a.beta[s0], gg = 0.f, bp = 0.f, gp = 0.f;
  auto scalars = [&](int64_t si) {
    if (GATE == kGateScalar) gg = a.g[si];
    if (GATE == kGateChannel) gg = a.g[si * DK + c];
    if (has_gram(PREC)) {
      bp = a.beta_p[si];
      gp = a.g_p ? a.g_p[si] : 0.f;
    }
  };
  scalars(s0);
  floatx4 st[R];
#pragma unroll
  for (int j = 0; j < R; ++j)
    st[j] = a.S0 ? *reinterpret_cast<const floatx4*>(a.S0 + (bh * DK + r0 + j) * a.dv + v0 + 4 * cg)
                 : floatx4{0.f, 0.f, 0.f, 0.f};
  // training (one chunk: the calls taken here are shorter): the chunk-start
  // state and the E rows, which are the tokens' e, the padded ones zero
  // (saved_idx: bf16 in slabs of 32 columns)
  constexpr bool SLAB = sizeof(T) == 2;
  T* er = nullptr;
  const int64_t se = SLAB ? kStepCols : a.dv;
  if (a.Hs) {
    T* hs = static_cast<T*>(a.Hs) + bh * DK * a.dv + (SLAB ? v0 * DK : v0) + 4 * cg;
#pragma unroll
    for (int j = 0; j < R; ++j) st4<T>(hs + (r0 + j) * se, st[j][0], st[j][1], st[j][2], st[j][3]);
    er = static_cast<T*>(a.Er) + bh * a.chunk * a.dv + (SLAB ? v0 * a.chunk : v0) + 4 * cg;
    for (int r = static_cast<int>(a.T) + (tid >> 3); r < a.chunk; r += 32) st4<T>(er + r * se, 0.f, 0.f, 0.f, 0.f);
  }
  float A = has_gram(PREC) && a.A0 ? a.A0[bh * DK + c] : 0.f;
  const float mu = PREC == kSquash ? fast_exp(a.log_a_scale[h]) : 0.f;
  for (int64_t t = 0; t < a.T; ++t) {
    const int u = static_cast<int>(t & 1);
    // ---- write key (and, for ATQ, the query) of this thread's channel
    float kt = PREC == kExternal ? xv : kv, q = qv, alpha = 1.f;
    if (GATE != kGateNone) alpha = fast_exp(gg);
    const float Ap = A;
    if (has_gram(PREC)) A = fast_exp(gp) * A + bp * kv * kv;
    if (PREC == kSquash) kt = squash_gain(A, mu, a.lnx) * kv;
    if (PREC == kDiagSM) kt = kv / (Ap + a.ridge);
    if (PREC == kATQ) q = qv / (A + a.ridge);
    if (ROWSUM && (PREC == kDiagSM || a.knorm != kKnormNone)) {
      const float m = wave_sum(key ? kv * kt : 0.f);
      if (key && l == 0) sSum[u][w] = m;
      __syncthreads();
      const float sum = KW == 2 ? sSum[u][0] + sSum[u][KW - 1] : sSum[u][0];
      if (PREC == kDiagSM) kt = kt / (1.f + sum);
      else if (a.knorm == kKnormM) kt = kt * (1.f / sum);
      else if (a.knorm == kKnorm1pm) kt = kt * (1.f / (1.f + sum));
      else kt = kt * (be / ((GATE == kGateScalar ? alpha : 1.f) + be * sum));
    }
    const float dot = wave_sum(key ? kt * q : 0.f);
    if (key) {
      sK[u][c] = kv;
      sQ[u][c] = q;
      sKt[u][c] = kt;
      if (GATE == kGateChannel) sLam[u][c] = alpha;
      if (l == 0) sDot[u][w] = dot;
    }
    const V4 v4 = vv;
    const float bt = be;
    if (t + 1 < a.T) {   // the next token's inputs
      kp += HK;
      qp += HK;
      vp += HV;
      kv = to_f(*kp);
      qv = to_f(*qp);
      if (PREC == kExternal) xv = to_f(*(xp += HK));
      vv = *reinterpret_cast<const V4*>(vp);
      be = a.beta[s0 + (t + 1) * a.H];
      scalars(s0 + (t + 1) * a.H);
    }
    __syncthreads();
    // ---- (alpha S) k and (alpha S) q over this thread's rows, then the block
    floatx4 y = {0.f, 0.f, 0.f, 0.f}, z = y;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (GATE == kGateScalar) st[j] *= alpha;
      if (GATE == kGateChannel) st[j] *= sLam[u][r0 + j];
      if (PREC != kATQ) y += st[j] * sK[u][r0 + j];
      z += st[j] * sQ[u][r0 + j];
    }
#pragma unroll
    for (int off = 8; off < 64; off <<= 1)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (PREC != kATQ) y[i] += __shfl_xor(y[i], off, 64);
        z[i] += __shfl_xor(z[i], off, 64);
      }
    if (l < 8) {
      *reinterpret_cast<floatx4*>(&sRed[u][w][0][4 * cg]) = y;
      *reinterpret_cast<floatx4*>(&sRed[u][w][1][4 * cg]) = z;
    }
    __syncthreads();
    floatx4 e, o = {0.f, 0.f, 0.f, 0.f};
    y = o;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      if (PREC != kATQ) y += *reinterpret_cast<const floatx4*>(&sRed[u][q4][0][4 * cg]);
      o += *reinterpret_cast<const floatx4*>(&sRed[u][q4][1][4 * cg]);
    }
    const float kq = KW == 2 ? sDot[u][0] + sDot[u][KW - 1] : sDot[u][0];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[i] = bt * (to_f(v4[i]) - y[i]);
      o[i] = a.scale * (o[i] + kq * e[i]);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) st[j] += sKt[u][r0 + j] * e;
    if (tid < 8 && a.o) st4<T>(op, o[0], o[1], o[2], o[3]);
    if (tid >> 3 == 8 && er) st4<T>(er + t * se, e[0], e[1], e[2], e[3]);
    op += HV;
  }
  if (a.S_T)
#pragma unroll
    for (int j = 0; j < R; ++j) *reinterpret_cast<floatx4*>(a.S_T + (bh * DK + r0 + j) * a.dv + v0 + 4 * cg) = st[j];
  if (has_gram(PREC) && a.A_T && v0 == 0 && key) a.A_T[bh * DK + c] = A;
}

template <typename T, int DK, int GATE>
hipError_t launch_prec(const FwdArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.BH * (a.dv / kStepCols)));
  switch (a.precond) {
    case kSquash: hipLaunchKernelGGL((step_tokens<T, DK, GATE, kSquash>), grid, dim3(256), 0, s, a); break;
    case kIdentity: hipLaunchKernelGGL((step_tokens<T, DK, GATE, kIdentity>), grid, dim3(256), 0, s, a); break;
    case kExternal: hipLaunchKernelGGL((step_tokens<T, DK, GATE, kExternal>), grid, dim3(256), 0, s, a); break;
    case kDiagSM: hipLaunchKernelGGL((step_tokens<T, DK, GATE, kDiagSM>), grid, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((step_tokens<T, DK, GATE, kATQ>), grid, dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

template <typename T, int DK>
hipError_t launch_gate(const FwdArgs& a, hipStream_t s) {
  switch (a.gate) {
    case kGateNone: return launch_prec<T, DK, kGateNone>(a, s);
    case kGateScalar: return launch_prec<T, DK, kGateScalar>(a, s);
    default: return launch_prec<T, DK, kGateChannel>(a, s);
  }
}

}  // namespace

hipError_t launch_step_tokens(const FwdArgs& a, int io_bf16, hipStream_t s) {
  if (io_bf16) return a.dk == 64 ? launch_gate<bf16, 64>(a, s) : launch_gate<bf16, 128>(a, s);
  return a.dk == 64 ? launch_gate<float, 64>(a, s) : launch_gate<float, 128>(a, s);
}

}  // namespace pdn
