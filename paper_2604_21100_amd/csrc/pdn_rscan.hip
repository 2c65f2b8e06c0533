// The bf16 reverse state-adjoint scan for gfx950: per (head, 32 value
// columns), sequential over chunks from the last.  With dS'^T the adjoint
// entering a chunk from the right, M = (I + At)^{-1}, w_t = exp(G_{C-1} - G_t):
//   dE = scale P^T dO + Diag(w) Kt dS'^T     Z = M^T dE     dV = Diag(beta) Z
//   dS^T = lam_C dS'^T + Q^T (scale Diag(lam) dO) - K^T (Diag(lam beta) Z)
// and it leaves dS'^T, Z and dV for the kernels after it.
//
// Built like the forward scan (pdn_scan.hip): two chain waves each own 16
// columns, so dE, Z and dS pass from product to product inside the wave; two
// loader waves bring the operand tiles of the chunk before into LDS; the
// output waves store the rows of the step's first half in its second and of
// its second half in the next step's first (two barriers a step).  Every
// operand comes as the rows the forward already has (q, k, the write keys, M,
// P): the transposed products take them through the transposing LDS read, so
// nothing is stored twice for this scan.  Five tiles leave LDS room for two
// stages; the tiles of a half step are refilled as soon as the half ends, a
// step and a half ahead of use.  (A scan that
// reads them transposed from memory needs P^T, M^T and both decayed
// transposes written for it: 200 MB more in the case below.)
//
// What bounds it (B = 4, T = 4096, H = 16, d = 128, scalar gate): a step's
// memory side, 608 MB by the counters in 170 us, 3.6 TB/s of the 5.1 a large
// copy reaches (225 us with the rows of a chunk split over four waves); k2,
// which writes no transposes for it, went from 146 to 106 us in the same step
// (79 since the forward scan forms P).  On 16 heads of 32768 tokens, first pass,
// 500 -> 320 us.
#include "pdn_tile.hpp"

namespace pdn {

namespace {

template <int DK, int GATE, int C>
struct RevLds {
  static constexpr int KK = DK / 32, SB = C / 32;
  static constexpr int kK = C * DK * 2, kM = C * C * 2, kV = C * kCols * 2;
  static constexpr int oT = 0, oM = oT + kK, oP = oM + kM, oD = oP + kM, oQ = oD + kV, oK = oQ + kK, oG = oK + kK;
  static constexpr int kStage = oG + (GATE == kGateChannel ? 1024 : 0);   // (one DMA unit for the gate row)
  static constexpr int kS = 2 * KK * 1024, kE = 2 * SB * 1024;
  static constexpr int oS = 2 * kStage, oZ = oS + kS, oX = oZ + kE, kTotal = oX + kE;
  static_assert(kTotal <= 160 * 1024, "LDS of one compute unit");
};

// ---------------------------------------------------------------- chain
// First half of a step on a chain wave: dE, Z and dV; bD gets the chunk's dO
// fragments, bX those of -Diag(lam) dV, gam lam_C (the second half may not
// read this half's tiles: they are being refilled).
template <int DK, int GATE, int C, bool WR>
__device__ __forceinline__ void rev_first(lds_char* sm, const lds_char* sg, int w, int l, float scale,
                                          const bf16x8 (&bS)[DK / 32], bf16x8 (&bD)[C / 32], bf16x8 (&bX)[C / 32],
                                          float& gam) {
  using L = RevLds<DK, GATE, C>;
  constexpr int KK = L::KK, SB = L::SB;
  constexpr int RK = DK * 2, RM = C * 2, RV = kCols * 2;   // row bytes
  const int m = l & 15, g = l >> 4;
  const int r0 = 8 * (m >> 2) + (m & 3);   // left-operand row of this lane, then + 4 u + 32 s
  bf16x8 fd[SB], fp[SB][2][SB], fk[KK][SB][2];
  floatx4 ww[SB][2];
#pragma unroll
  for (int s = 0; s < SB; ++s)
    fd[s] = lds_frag_t(sg + L::oD + tile_off<4>(8 * g + (m >> 2), m & 3) + w * 8 + s * 32 * RV, 4 * RV);
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = s; k < SB; ++k)
        fp[s][u][k] = lds_frag_t(sg + L::oP + tile_off<C / 8>(8 * g + (m >> 2), 4 * s + (m & 3)) + u * 8 + k * 32 * RM,
                                 4 * RM);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        fk[kk][s][u] = lds_frag(sg + L::oT + tile_off<DK / 8>(r0, 4 * kk + g) + s * 32 * RK + u * 4 * RK);
  reads_done();
  floatx4 aP[SB][2], aK[SB][2];
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      aP[s][u] = floatx4{0.f, 0.f, 0.f, 0.f};
      aK[s][u] = aP[s][u];
#pragma unroll
      for (int k = s; k < SB; ++k) aP[s][u] = mfma(fp[s][u][k], fd[k], aP[s][u]);
    }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u) aK[s][u] = mfma(fk[kk][s][u], bS[kk], aK[s][u]);
  // M^T (its upper triangle; at C = 32 the scalars' block is part of a
  // fragment and is cleared there) and the scalars
  bf16x8 fm[SB][2][SB];
  floatx4 be[SB][2], la[SB][2];
  if (GATE == kGateScalar) gam = lds_f4(sg + L::oM + scal_off<C>(0, C / 4 - 1))[3];
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      be[s][u] = lds_f4(sg + L::oM + scal_off<C>(2, 8 * s + 2 * g + u));
      if (GATE == kGateScalar) {
        la[s][u] = lds_f4(sg + L::oM + scal_off<C>(0, 8 * s + 2 * g + u));
        ww[s][u] = lds_f4(sg + L::oM + scal_off<C>(1, 8 * s + 2 * g + u));
      }
#pragma unroll
      for (int k = s; k < SB; ++k)
        fm[s][u][k] = lds_frag_t(sg + L::oM + tile_off<C / 8>(8 * g + (m >> 2), 4 * s + (m & 3)) + u * 8 + k * 32 * RM,
                                 4 * RM);
    }
  reads_done();
  if (C == 32 && m >= 8 && g < 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) fm[0][u][0] = bf16x8{};
  }
  // dE enters M^T as the sum of two io values, so its rounding does not reach
  // Z (and through it the write-key gradient, which the preconditioner's
  // adjoint divides by A): a few MFMA in a step that waits for memory
  bf16x8 bE[SB], bL[SB];
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    floatx4 e[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (GATE == kGateScalar) aK[s][u] *= ww[s][u];
      e[u] = scale * aP[s][u] + aK[s][u];
    }
    bE[s] = pack8(e[0], e[1]);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) e[u][i] -= static_cast<float>(bE[s][4 * u + i]);
    bL[s] = pack8(e[0], e[1]);
  }
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    floatx4 z[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      z[u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = s; k < SB; ++k) {
        z[u] = mfma(fm[s][u][k], bL[k], z[u]);
        z[u] = mfma(fm[s][u][k], bE[k], z[u]);
      }
    }
    if (WR) lds_put(sm + L::oZ + (w * SB + s) * 1024 + l * 16, pack8(z[0], z[1]));
    z[0] *= be[s][0];
    z[1] *= be[s][1];
    if (WR) lds_put(sm + L::oX + (w * SB + s) * 1024 + l * 16, pack8(z[0], z[1]));
    if (GATE == kGateScalar) bX[s] = pack8(-(la[s][0] * z[0]), -(la[s][1] * z[1]));
    else bX[s] = pack8(-z[0], -z[1]);
    // scale Diag(lam) dO
    floatx4 d[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d[u][i] = scale * static_cast<float>(fd[s][4 * u + i]);
        if (GATE == kGateScalar) d[u][i] *= la[s][u][i];
      }
    bD[s] = pack8(d[0], d[1]);
  }
}

// Second half: dS^T, and its io copy for the next chunk and the stores
template <int DK, int GATE, int C, bool WR>
__device__ __forceinline__ void rev_second(lds_char* sm, const lds_char* sg, int w, int l, floatx4 (&st)[DK / 32][2],
                                           bf16x8 (&bS)[DK / 32], const bf16x8 (&bD)[C / 32],
                                           const bf16x8 (&bX)[C / 32], float gam) {
  using L = RevLds<DK, GATE, C>;
  constexpr int KK = L::KK, SB = L::SB;
  constexpr int RK = DK * 2;
  const int m = l & 15, g = l >> 4;
  bf16x8 fq[KK][2][SB], fk[KK][2][SB];
  floatx4 gc[KK][2];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int o = tile_off<DK / 8>(8 * g + (m >> 2), 4 * kk + (m & 3)) + u * 8;
#pragma unroll
      for (int s = 0; s < SB; ++s) fq[kk][u][s] = lds_frag_t(sg + L::oQ + o + s * 32 * RK, 4 * RK);
    }
  reads_done();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int o = tile_off<DK / 8>(8 * g + (m >> 2), 4 * kk + (m & 3)) + u * 8;
      if (GATE == kGateChannel) gc[kk][u] = lds_f4(sg + L::oG + (32 * kk + 8 * g + 4 * u) * 4);
#pragma unroll
      for (int s = 0; s < SB; ++s) fk[kk][u][s] = lds_frag_t(sg + L::oK + o + s * 32 * RK, 4 * RK);
    }
  reads_done();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (GATE == kGateScalar) st[kk][u] *= gam;
      if (GATE == kGateChannel) st[kk][u] *= gc[kk][u];
    }
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int u = 0; u < 2; ++u) st[kk][u] = mfma(fq[kk][u][s], bD[s], st[kk][u]);
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int u = 0; u < 2; ++u) st[kk][u] = mfma(fk[kk][u][s], bX[s], st[kk][u]);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    bS[kk] = pack8(st[kk][0], st[kk][1]);
    if (WR) lds_put(sm + L::oS + (w * KK + kk) * 1024 + l * 16, bS[kk]);
  }
}

// ---------------------------------------------------------------- loaders
// A loader wave's half of a chunk's tiles, in the two groups the step's
// halves read: (write keys, M, P, dO), then (q, k) and the gate row.
template <int DK, int GATE, int C>
struct RevLoader {
  using L = RevLds<DK, GATE, C>;
  static constexpr bool CH = GATE == kGateChannel;
  static constexpr int NK = L::kK / 1024 / kLoaders, NM = L::kM / 1024 / kLoaders, NV = L::kV / 1024 / kLoaders;
  static constexpr int kFirst = NK + 2 * NM + NV, kSecond = 2 * NK + (CH ? 1 : 0);   // loads of a group
  uint32_t vk[NK], vt[NK], vm[NM], vv[NV], vg;
  const char *k, *q, *d, *m, *p, *t, *g;   // the next chunk's k, q, dO, M, P, write keys, gate row
  uint32_t hd, hv;
  int64_t heads, tok1, tok2;   // (tokens to the sequence end from each group's next chunk)
  int n1, n2;                  // chunks left in each group
  bool probe;

  __device__ __forceinline__ RevLoader(const BwdArgs& ba, const RunCtx& x, int lw, int l) {
    const FwdArgs& a = ba.f;
    const int64_t top = x.c1 - 1, t0 = top * C, ci = a.ci(x.bh, top);
    const int64_t tok = ((x.b * a.T + t0) * a.H + x.h) * 2, rows = ci * (C * DK * 2);
    auto at = [](const void* b, int64_t off) { return static_cast<const char*>(b) + off; };
    // per-channel gate: the decayed key and query rows
    k = CH ? at(a.KL, rows) : at(a.k, tok * DK);
    q = CH ? at(a.QL, rows) : at(a.q, tok * DK);
    d = at(ba.dO, tok * a.dv + x.v0 * 2);
    m = at(a.Tm, ci * (C * C * 2));
    p = at(a.Pm, ci * (C * C * 2));
    t = at(a.Kd, rows);
    g = CH ? at(a.G, ci * (DK * 4)) : nullptr;
    hd = static_cast<uint32_t>(a.H * DK * 2);
    hv = static_cast<uint32_t>(a.H * a.dv * 2);
    const int nrow = static_cast<int>(min<int64_t>(C, a.T));
    heads = a.BH;
    tok1 = tok2 = a.T - t0;
    n1 = n2 = x.c1 - x.c0;
    probe = x.probe;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      vk[j] = unit_src<DK / 8>(lw * NK + j, l, CH ? DK * 2 : hd, CH ? C : nrow);
      vt[j] = unit_src<DK / 8>(lw * NK + j, l, DK * 2);
    }
#pragma unroll
    for (int j = 0; j < NM; ++j) vm[j] = unit_src<C / 8>(lw * NM + j, l, C * 2);
#pragma unroll
    for (int j = 0; j < NV; ++j) vv[j] = unit_src<kCols / 8>(lw * NV + j, l, hv, nrow);
    vg = 16 * l;
  }
  // (past the run: empty ranges, no traffic; rows past the sequence end are
  // past the range and arrive as zeros)
  __device__ __forceinline__ void first(int lw, lds_char* sg) {
    const int n = n1 > 0 ? static_cast<int>(min<int64_t>(C, tok1)) : 0;
    const auto rd = buf_rsrc(d, n && !probe ? (n - 1) * hv + kCols * 2 : 0);
    const auto rp = buf_rsrc(p, n ? L::kM : 0), rt = buf_rsrc(t, n ? L::kK : 0), rm = buf_rsrc(m, n ? L::kM : 0);
#pragma unroll
    for (int j = 0; j < NV; ++j) unit_copy(rd, vv[j], sg + L::oD + (lw * NV + j) * 1024);
#pragma unroll
    for (int j = 0; j < NM; ++j) unit_copy(rp, vm[j], sg + L::oP + (lw * NM + j) * 1024);
#pragma unroll
    for (int j = 0; j < NK; ++j) unit_copy(rt, vt[j], sg + L::oT + (lw * NK + j) * 1024);
#pragma unroll
    for (int j = 0; j < NM; ++j) unit_copy(rm, vm[j], sg + L::oM + (lw * NM + j) * 1024);
    d -= C * static_cast<int64_t>(hv);
    p -= heads * L::kM;
    t -= heads * L::kK;
    m -= heads * L::kM;
    tok1 += C;
    --n1;
  }
  __device__ __forceinline__ void second(int lw, lds_char* sg) {
    const int n = n2 > 0 ? static_cast<int>(min<int64_t>(C, tok2)) : 0;
    const uint32_t bytes = CH ? (n ? L::kK : 0) : n ? (n - 1) * hd + DK * 2 : 0;
    const auto rq = buf_rsrc(q, bytes), rk = buf_rsrc(k, bytes);
#pragma unroll
    for (int j = 0; j < NK; ++j) unit_copy(rq, vk[j], sg + L::oQ + (lw * NK + j) * 1024);
#pragma unroll
    for (int j = 0; j < NK; ++j) unit_copy(rk, vk[j], sg + L::oK + (lw * NK + j) * 1024);
    if (CH) unit_copy(buf_rsrc(g, n ? DK * 4 : 0), vg, sg + L::oG);
    const int64_t step = CH ? heads * L::kK : C * static_cast<int64_t>(hd);
    q -= step;
    k -= step;
    if (CH) g -= heads * (DK * 4);
    tok2 += C;
    --n2;
  }
};

template <int DK, int GATE, int C, bool WR>
__device__ __forceinline__ void rev_run(const BwdArgs& ba, const RunCtx& x, int seg, int pv0, lds_char* sm) {
  using L = RevLds<DK, GATE, C>;
  constexpr int KK = L::KK, SB = L::SB;
  const FwdArgs& a = ba.f;
  const int S = a.seg_cnt;
  const int l = threadIdx.x & 63, m = l & 15, g = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cnt = x.c1 - x.c0;
  const int64_t BHDK = a.BH * static_cast<int64_t>(DK);
  if (w < 2) {
    const int v = 8 * (m >> 2) + 4 * w + (m & 3);   // this lane's column
    floatx4 st[KK][2];
    bf16x8 bS[KK], bD[SB], bX[SB];
    const float* src = nullptr;   // middle segments' local runs start from zero
    if (a.seg_phase == 0 || (a.seg_phase == 1 && seg == S - 1)) src = ba.dS_T ? ba.dS_T + x.bh * DK * a.dv : nullptr;
    else if (a.seg_phase == 3) src = a.seg_start + (seg * BHDK + x.bh * DK) * a.dv;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = 32 * kk + 8 * g + 4 * u + i;
          st[kk][u][i] = src ? src[static_cast<int64_t>(c) * a.dv + x.v0 + v] : (x.probe && c == pv0 + v) ? 1.f : 0.f;
        }
      bS[kk] = pack8(st[kk][0], st[kk][1]);
      if (WR) lds_put(sm + L::oS + (w * KK + kk) * 1024 + l * 16, bS[kk]);
    }
    lds_sync();   // the top chunk's first group is in
    const lds_char* sg = sm;
    float gam = 1.f;
    for (int j = 0; j < cnt; ++j) {
      rev_first<DK, GATE, C, WR>(sm, sg, w, l, a.scale, bS, bD, bX, gam);
      lds_sync();
      rev_second<DK, GATE, C, WR>(sm, sg, w, l, st, bS, bD, bX, gam);
      lds_sync();
      sg = sg == sm ? sm + L::kStage : sm;
    }
    // the end state: dS0 after chunk 0; phase 1: the last segment's exact
    // end, a middle segment's local end or its transition
    float* dst = nullptr;
    int64_t ld = a.dv;
    int col = x.v0 + v;
    if (a.seg_phase == 1) {
      if (x.probe) {
        dst = a.seg_phi + (seg * BHDK + x.bh * DK) * DK;
        ld = DK;
        col = pv0 + v;
      } else {
        dst = a.seg_end + (seg * BHDK + x.bh * DK) * a.dv;
      }
    } else if (x.c0 == 0 && ba.dS0) {
      dst = ba.dS0 + x.bh * DK * a.dv;
    }
    if (dst) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) dst[(32 * kk + 8 * g + 4 * u + i) * ld + col] = st[kk][u][i];
    }
  } else if (w < 4 || w >= 4 + kLoaders) {
    // ---- stores: the entering adjoint in a step's first half, Z and dV in
    // its second (rows of 32 columns, 64 bytes a row)
    const int ow = w < 4 ? w - 2 : w - 4, hh = ow & 1, f0 = ow >> 1;
    constexpr int NP = C / 32;   // pairs of output waves
    const int r0 = 8 * (m >> 2) + 4 * hh + (m & 3);
    const int64_t top = x.c1 - 1, ci = a.ci(x.bh, top);
    char* hs = static_cast<char*>(ba.dHs) + (ci * DK * a.dv + x.v0 * DK) * 2;   // (slabs of 32 columns: saved_idx)
    char* zr = static_cast<char*>(ba.Zr) + (ci * C * a.dv + x.v0 * C) * 2;
    char* dv = static_cast<char*>(ba.dv) + (((x.b * a.T + top * C) * a.H + x.h) * a.dv + x.v0) * 2;
    const uint32_t hv = static_cast<uint32_t>(a.H * a.dv * 2);
    const uint32_t os = (r0 * kCols + 8 * g) * 2, ox = row_off(32 * f0 + r0, hv, 16 * g, static_cast<int>(min<int64_t>(C, a.T)));
    int64_t left = a.T - top * C;
    lds_sync();
    for (int j = 0; j < cnt; ++j) {
      if (WR) {
#pragma unroll
        for (int u = 0; u < KK / NP; ++u) {
          const int f = u * NP + f0;
          *reinterpret_cast<bf16x8*>(hs + os + 64 * f * kCols) = frag_major_row<KK>(sm + L::oS, f, hh, l);
        }
      }
      lds_sync();
      if (WR) {
        *reinterpret_cast<bf16x8*>(zr + os + 64 * f0 * kCols) = frag_major_row<SB>(sm + L::oZ, f0, hh, l);
        // the chunk's dv rows as a buffer ending with its last valid row
        buf_put16(buf_rsrc(dv, (static_cast<int>(min<int64_t>(C, left)) - 1) * hv + kCols * 2), ox,
                  frag_major_row<SB>(sm + L::oX, f0, hh, l));
        hs -= a.BH * (DK * 2) * static_cast<int64_t>(a.dv);
        zr -= a.BH * (C * 2) * static_cast<int64_t>(a.dv);
        dv -= C * static_cast<int64_t>(hv);
        left += C;
      }
      lds_sync();
    }
  } else {
    // ---- loaders: chunk top - j uses stage j mod 2.  Before a half step's
    // barrier its group has arrived, which leaves the two groups issued after
    // it in flight; after it the stage's just-read group takes chunk j + 2.
    using F = RevLoader<DK, GATE, C>;
    const int lw = w - 4;
    F f(ba, x, lw, l);
    f.first(lw, sm);
    f.second(lw, sm);
    f.first(lw, sm + L::kStage);
    wait_loads<F::kFirst + F::kSecond>();
    lds_sync();
    lds_char* sg = sm;
    for (int j = 0; j < cnt; ++j) {
      lds_char* other = sg == sm ? sm + L::kStage : sm;
      f.second(lw, other);   // chunk j + 1's
      wait_loads<F::kFirst + F::kSecond>();
      lds_sync();            // first half done, second group of chunk j in
      f.first(lw, sg);       // chunk j + 2's
      wait_loads<F::kFirst + F::kSecond>();
      lds_sync();            // step done, first group of chunk j + 1 in
      sg = other;
    }
  }
}

template <int DK, int GATE, int C>
__global__ __launch_bounds__(scan_threads(C), 2) void rev_scan(BwdArgs ba) {
  using L = RevLds<DK, GATE, C>;
  __shared__ __attribute__((aligned(1024))) char smem[L::kTotal];
  lds_char* sm = (lds_char*)smem;
  const FwdArgs& a = ba.f;
  // workgroup -> (head, role, slab) as in the forward scan, mirrored: phase
  // 1 runs the last segment from dS_T beside the middle segments' local
  // runs (from zero) and transitions (from the identity, dO zeroed); phase
  // 3 runs segments 0 .. S - 2 from their composed starts
  const int nslab = a.dv / kCols, npslab = DK / kCols;
  const int S = a.seg_cnt;
  const int nrole = a.seg_phase == 0 ? nslab
                  : a.seg_phase == 1 ? nslab + (S - 2) * (nslab + npslab)
                                     : (S - 1) * nslab;
  int role;
  RunCtx x;
  x.bh = scan_head(nrole, &role);
  if (x.bh >= a.BH) return;
  x.b = x.bh / a.H;
  x.h = x.bh % a.H;
  int seg = S - 1, slab = role;
  x.probe = false;
  if (a.seg_phase == 1 && role >= nslab) {
    const int r = role - nslab;
    seg = 1 + r / (nslab + npslab);
    slab = r % (nslab + npslab);
    x.probe = slab >= nslab;
  } else if (a.seg_phase == 3) {
    seg = role / nslab;
    slab = role % nslab;
  }
  x.c0 = a.seg_phase == 0 ? 0 : seg * a.seg_len;
  x.c1 = a.seg_phase == 0 ? a.NT : min(a.NT, x.c0 + a.seg_len);
  x.v0 = x.probe ? 0 : slab * kCols;
  const int pv0 = x.probe ? (slab - nslab) * kCols : 0;
  // middle segments of the first pass need only their end states
  if (a.seg_phase == 1 && seg < S - 1) rev_run<DK, GATE, C, false>(ba, x, seg, pv0, sm);
  else rev_run<DK, GATE, C, true>(ba, x, seg, pv0, sm);
}

template <int DK, int GATE, int C>
hipError_t launch_typed(const BwdArgs& ba, hipStream_t s) {
  BwdArgs b = ba;
  FwdArgs& a = b.f;
  const int nslab = a.dv / kCols, npslab = DK / kCols;
  auto launch = [&](int phase, int nrole) {
    a.seg_phase = phase;
    hipLaunchKernelGGL((rev_scan<DK, GATE, C>), scan_grid(a.BH, nrole), dim3(scan_threads(C)), 0, s, b);
    return hipGetLastError();
  };
  if (a.seg_cnt < 3) return launch(0, nslab);
  // split: the last segment beside the middle segments' local runs and
  // transitions, the composed starts, then segments 0 .. S - 2
  const int S = a.seg_cnt;
  hipError_t e = launch(1, nslab + (S - 2) * (nslab + npslab));
  if (e != hipSuccess) return e;
  if ((e = launch_seg_compose(a, true, s)) != hipSuccess) return e;
  return launch(3, (S - 1) * nslab);
}

template <int DK, int C>
hipError_t launch_gate(const BwdArgs& b, hipStream_t s) {
  switch (b.f.gate) {
    case kGateNone: return launch_typed<DK, kGateNone, C>(b, s);
    case kGateScalar: return launch_typed<DK, kGateScalar, C>(b, s);
    default: return launch_typed<DK, kGateChannel, C>(b, s);
  }
}

}  // namespace

hipError_t launch_rev_scan_bf16(const BwdArgs& b, hipStream_t s) {
  if (b.f.chunk == 32) return b.f.dk == 64 ? launch_gate<64, 32>(b, s) : launch_gate<128, 32>(b, s);
  return b.f.dk == 64 ? launch_gate<64, 64>(b, s) : launch_gate<128, 64>(b, s);
}

}  // namespace pdn
