// The bf16 state scan of the chunkwise preconditioned delta rule for gfx950:
// per (head, 32 value columns), sequential over chunks (Eq.
// chunkwise_atk_form, decayed forms of App. D), with S^T the chunk-start
// state, M = (I + At)^{-1} and w_t = exp(G_{C-1} - G_t):
//   X = Diag(beta) (V - Diag(lam) K S^T)      E = M X
//   O = scale [ Diag(lam) Q S^T + P E ]       S'^T = lam_C S^T + Kt^T Diag(w) E
//
// The waves of a workgroup have three roles.  Two chain waves each own 16 of
// the 32 columns for the whole run, so X, E and S pass from one product to
// the next inside the wave, straight from accumulator to operand registers
// (the row order of the left operands is chosen so that an accumulator's rows
// are the next product's contraction order): a chunk costs one barrier, not
// three exchanges through LDS.  Two loader waves bring the operand tiles of
// the chunks ahead from memory straight into LDS, row-major; a tile serves
// products over its rows and, through the transposing LDS read, over its
// columns.  The output waves form and store the output (and the rows kept for
// the backward) of the chunk before, from the S and E fragments the chain
// leaves in LDS.
//
// What bounds it (one launch at B = 4, T = 4096, H = 16, d = 128, scalar gate,
// C = 64; 256 workgroups of 64 steps, P formed here): a step's memory side.  It
// reads q, k, v, the write keys and M once (the four workgroups of a head share
// an XCD's L2) and writes o, 374 MB by the counters in 111 us, 3.4 TB/s of the
// 5.1 a large copy reaches; keeping the backward's rows too, 600 MB in 181 us,
// 3.3 TB/s.  With P read instead of formed, 122 us: a step 1.9 us, and with one
// role running alone 1.0 us (chain: 38 MFMA in a row of dependent products),
// 1.0 us (loads) and 1.1 us (output).  The form before this one, a chunk's rows
// split over four waves with three exchanges through LDS a step, took 163 us
// (240 keeping rows).  On 16 heads of 32768 tokens (192 workgroups of 171 steps
// in the first pass, P read) 374 -> 269 us.
#include "pdn_tile.hpp"

namespace pdn {

namespace {

constexpr int kStages = 3;     // LDS stages of operand tiles

// LDS of the forward scan: stages of operand tiles, two buffers of state and
// E fragments
template <int DK, int GATE, int C>
struct FwdLds {
  static constexpr int KK = DK / 32, SB = C / 32;
  static constexpr int kK = C * DK * 2, kM = C * C * 2, kV = C * kCols * 2;
  static constexpr int oK = 0, oM = oK + kK, oKt = oM + kM, oV = oKt + kK, oG = oV + kV;
  static constexpr int kStage = oG + (GATE == kGateChannel ? 1024 : 0);   // (one DMA unit for the gate row)
  static constexpr int kS = 2 * KK * 1024, kE = 2 * SB * 1024;
  static constexpr int oS = kStages * kStage, oE = oS + 2 * kS;
  static constexpr int kTotal = oE + 2 * kE;
  static_assert(kTotal <= 160 * 1024, "LDS of one compute unit");
};

// ---------------------------------------------------------------- chain
// One chunk on a chain wave.  st[kk][u][i] holds S^T row 32 kk + 8 g + 4 u + i
// at this lane's column; bS its io copy as right-operand fragments.
template <int DK, int GATE, int C, bool LA, bool KEEP>
__device__ __forceinline__ void chain_step(lds_char* sm, lds_char* sg, int par, int w, int l, floatx4 (&st)[DK / 32][2],
                                           bf16x8 (&bS)[DK / 32]) {
  using L = FwdLds<DK, GATE, C>;
  constexpr int KK = L::KK, SB = L::SB;
  constexpr int RK = DK * 2, RM = C * 2, RV = kCols * 2;   // row bytes
  const int m = l & 15, g = l >> 4;
  // left-operand row of this lane: 8 (m >> 2) + (m & 3), then + 4 u + 32 s
  const int r0 = 8 * (m >> 2) + (m & 3);
  bf16x8 fk[KK][SB][2], vv[SB];
  floatx4 be[SB][2], la[SB][2];
  if (!LA) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const lds_char* p = sg + L::oK + tile_off<DK / 8>(r0, 4 * kk + g);
#pragma unroll
      for (int s = 0; s < SB; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u) fk[kk][s][u] = lds_frag(p + s * 32 * RK + u * 4 * RK);
    }
  }
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    vv[s] = lds_frag_t(sg + L::oV + tile_off<4>(8 * g + (m >> 2), m & 3) + w * 8 + s * 32 * RV, 4 * RV);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      be[s][u] = lds_f4(sg + L::oM + scal_off<C>(2, 8 * s + 2 * g + u));
      if (GATE == kGateScalar && !LA) la[s][u] = lds_f4(sg + L::oM + scal_off<C>(0, 8 * s + 2 * g + u));
    }
  }
  if (KEEP) {
    lds_char* s = sm + L::oS + par * L::kS + w * (KK * 1024) + l * 16;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) lds_put(s + kk * 1024, bS[kk]);
  }
  reads_done();
  floatx4 aX[SB][2];
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) aX[s][u] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (!LA) {   // linear attention: E = Diag(beta) V
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int s = 0; s < SB; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u) aX[s][u] = mfma(fk[kk][s][u], bS[kk], aX[s][u]);
  }
  // the next products' operands: M, w, and the write keys transposed
  bf16x8 fm[SB][2][SB], ft[KK][2][SB];
  floatx4 ww[SB][2], gc[KK][2];
  float gam = 1.f;
  if (!LA) {
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k <= s; ++k)
          fm[s][u][k] = lds_frag(sg + L::oM + tile_off<C / 8>(r0, 4 * k + g) + s * 32 * RM + u * 4 * RM);
  }
  if (GATE == kGateScalar) {
    gam = lds_f4(sg + L::oM + scal_off<C>(0, C / 4 - 1))[3];
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u) ww[s][u] = lds_f4(sg + L::oM + scal_off<C>(1, 8 * s + 2 * g + u));
  }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (GATE == kGateChannel) gc[kk][u] = lds_f4(sg + L::oG + (32 * kk + 8 * g + 4 * u) * 4);
      const lds_char* p = sg + L::oKt + tile_off<DK / 8>(8 * g + (m >> 2), 4 * kk + (m & 3)) + u * 8;
#pragma unroll
      for (int s = 0; s < SB; ++s) ft[kk][u][s] = lds_frag_t(p + s * 32 * RK, 4 * RK);
    }
  reads_done();
  // X = Diag(beta) (V - Diag(lam) K S^T), rows 32 s + 8 g + 4 u + i
  bf16x8 bX[SB];
  floatx4 aE[SB][2];
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    floatx4 x[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = static_cast<float>(vv[s][4 * u + i]);
        x[u][i] = be[s][u][i] *
                  (LA ? v : GATE == kGateScalar ? fmaf(-la[s][u][i], aX[s][u][i], v) : v - aX[s][u][i]);
      }
    if (LA) {
      aE[s][0] = x[0];
      aE[s][1] = x[1];
    } else {
      bX[s] = pack8(x[0], x[1]);
    }
  }
  // E = M X (M lower triangular: blocks on and below the diagonal; at C = 32
  // the scalars' block is part of a fragment and is cleared there)
  if (!LA) {
    if (C == 32 && m < 8 && g >= 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) fm[0][u][0] = bf16x8{};
    }
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        aE[s][u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k <= s; ++k) aE[s][u] = mfma(fm[s][u][k], bX[k], aE[s][u]);
      }
  }
  // Diag(w) E for the state, E for the output
  bf16x8 bW[SB];
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    if (KEEP || GATE != kGateScalar) {
      bW[s] = pack8(aE[s][0], aE[s][1]);
      if (KEEP) lds_put(sm + L::oE + par * L::kE + (w * SB + s) * 1024 + l * 16, bW[s]);
    }
    if (GATE == kGateScalar) bW[s] = pack8(aE[s][0] * ww[s][0], aE[s][1] * ww[s][1]);
  }
  // S'^T = Diag(lam_C) S^T + Kt^T (Diag(w) E)
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
      for (int u = 0; u < 2; ++u) st[kk][u] = mfma(ft[kk][u][s], bW[s], st[kk][u]);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) bS[kk] = pack8(st[kk][0], st[kk][1]);
}

// ---------------------------------------------------------------- loaders
// Addresses of a run's next chunk (wave-uniform), advanced a chunk at a time
struct ChunkCursor {
  const char *k, *q, *v, *m, *p, *t, *g;   // key, query, value, M, P, write-key rows, gate row
  uint32_t hd, hv;   // token row strides of k (q) and v, bytes
  int64_t heads;     // chunk to chunk step of the per-chunk tensors, in chunks
  int64_t tokens;    // tokens from the chunk's first to the sequence end
  int chunks;        // chunks left in the run
  bool probe;
  template <int DK, int GATE, int C, bool LA>
  __device__ __forceinline__ void start(const FwdArgs& a, const RunCtx& x) {
    constexpr bool CH = GATE == kGateChannel;
    const int64_t t0 = static_cast<int64_t>(x.c0) * C, ci = a.ci(x.bh, x.c0);
    const int64_t tok = ((x.b * a.T + t0) * a.H + x.h) * 2, rows = ci * (C * DK * 2);
    hd = static_cast<uint32_t>(a.H * DK * 2);
    hv = static_cast<uint32_t>(a.H * a.dv * 2);
    auto at = [](const void* p, int64_t off) { return static_cast<const char*>(p) + off; };
    // per-channel gate: the decayed key and query rows the prep kernel left;
    // linear attention: the preconditioned query rows
    k = CH ? at(a.KL, rows) : at(a.k, tok * DK);
    q = CH ? at(a.QL, rows) : LA ? at(a.Qt, rows) : at(a.q, tok * DK);
    v = at(a.v, tok * a.dv + x.v0 * 2);
    m = at(a.Tm, ci * (C * C * 2));
    p = at(a.Pm, ci * (C * C * 2));
    t = at(a.Kd, rows);
    g = CH ? at(a.G, ci * (DK * 4)) : nullptr;
    heads = a.BH;
    tokens = a.T - t0;
    chunks = x.c1 - x.c0;
    probe = x.probe;
  }
  // valid rows of the chunk, 0 past the run
  template <int C>
  __device__ __forceinline__ int rows() const {
    return chunks > 0 ? static_cast<int>(min<int64_t>(C, tokens)) : 0;
  }
  template <int C>
  __device__ __forceinline__ void next() {
    tokens -= C;
    chunks -= 1;
  }
};

// A loader wave moves half of a chunk's operand tiles from memory straight
// into an LDS stage, 1 KB (64 lanes of 16 bytes) an instruction; the XOR
// order of the tiles is in the lanes' source addresses.  Rows past the
// sequence end are past the buffer's range and arrive as zeros.
template <int DK, int GATE, int C, bool LA>
struct FwdLoader {
  using L = FwdLds<DK, GATE, C>;
  static constexpr bool CH = GATE == kGateChannel;
  static constexpr int NK = L::kK / 1024 / kLoaders, NV = L::kV / 1024 / kLoaders;
  // (linear attention: M is the identity; its first unit holds the scalars)
  static constexpr int NM = LA ? 1 : L::kM / 1024 / kLoaders;
  static constexpr int kLoads = (LA ? NK : 2 * NK) + NM + NV + (CH ? 1 : 0);   // per chunk
  uint32_t vk[LA ? 1 : NK], vt[NK], vm[NM], vv[NV], vg;

  __device__ __forceinline__ FwdLoader(const FwdArgs& a, int lw, int l) {
    const uint32_t hd = static_cast<uint32_t>(a.H) * DK * 2u, hv = static_cast<uint32_t>(a.H) * a.dv * 2u;
    const int nrow = static_cast<int>(min<int64_t>(C, a.T));
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      if (!LA) vk[j] = unit_src<DK / 8>(lw * NK + j, l, CH ? DK * 2u : hd, CH ? C : nrow);
      vt[j] = unit_src<DK / 8>(lw * NK + j, l, DK * 2u);
    }
#pragma unroll
    for (int j = 0; j < NM; ++j) vm[j] = unit_src<C / 8>(lw * NM + j, l, C * 2u);
#pragma unroll
    for (int j = 0; j < NV; ++j) vv[j] = unit_src<kCols / 8>(lw * NV + j, l, hv, nrow);
    vg = 16u * l;
  }
  // the next chunk into the stage at sg (past the run: empty ranges, no
  // traffic)
  __device__ __forceinline__ void issue(ChunkCursor& c, int lw, lds_char* sg) const {
    const int n = c.rows<C>();
    if (!LA) {
      const auto rk = buf_rsrc(c.k, CH ? (n ? L::kK : 0) : n ? (n - 1) * c.hd + DK * 2 : 0);
#pragma unroll
      for (int j = 0; j < NK; ++j) unit_copy(rk, vk[j], sg + L::oK + (lw * NK + j) * 1024);
    }
    const auto rv = buf_rsrc(c.v, n && !c.probe ? (n - 1) * c.hv + kCols * 2 : 0);
#pragma unroll
    for (int j = 0; j < NV; ++j) unit_copy(rv, vv[j], sg + L::oV + (lw * NV + j) * 1024);
    const auto rm = buf_rsrc(c.m, n ? L::kM : 0);
#pragma unroll
    for (int j = 0; j < NM; ++j) unit_copy(rm, vm[j], sg + L::oM + (lw * NM + j) * 1024);
    const auto rt = buf_rsrc(c.t, n ? L::kK : 0);
#pragma unroll
    for (int j = 0; j < NK; ++j) unit_copy(rt, vt[j], sg + L::oKt + (lw * NK + j) * 1024);
    if (CH) unit_copy(buf_rsrc(c.g, n ? DK * 4 : 0), vg, sg + L::oG);
    c.k += CH ? c.heads * L::kK : C * static_cast<int64_t>(c.hd);
    c.v += C * static_cast<int64_t>(c.hv);
    c.m += c.heads * L::kM;
    c.t += c.heads * L::kK;
    if (CH) c.g += c.heads * (DK * 4);
    c.next<C>();
  }
};

// An output wave's query and P rows (row tile ow of the chunk).  As loaded, a
// fragment pair (two 64-byte halves of a row's 128 bytes) comes as two rows'
// whole lines, lanes m even / odd taking the halves of row m & ~1 in the
// first and of row m | 1 in the second, and is put in order where it is first
// used (take_pair).  The memory path's cost goes by the lines an instruction
// touches: 8 this way, 16 with a fragment's own lanes.
// PSCAN: P is formed here from the query rows and the stage's write keys
// (scan_forms_p), else it is read.
template <int DK, int GATE, int C, bool LA>
struct OutRows {
  bf16x8 q[DK / 32], p[C / 32];
  float g;   // scalar gate: G_r of this lane's row
};

// a, b: the pair as loaded -> the fragments of row m's first and second half
__device__ __forceinline__ void take_pair(bf16x8& a, bf16x8& b, bool odd) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  i32x4 x = __builtin_bit_cast(i32x4, a), y = __builtin_bit_cast(i32x4, b);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int xn = __builtin_amdgcn_mov_dpp(x[i], 0xB1, 0xf, 0xf, true);   // lane m ^ 1
    const int yn = __builtin_amdgcn_mov_dpp(y[i], 0xB1, 0xf, 0xf, true);
    x[i] = odd ? yn : x[i];
    y[i] = odd ? y[i] : xn;
  }
  a = __builtin_bit_cast(bf16x8, x);
  b = __builtin_bit_cast(bf16x8, y);
}

__device__ __forceinline__ bf16x8 buf_get16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, 0));
}

// lane offsets of an output wave's loads and stores
template <int DK, int GATE, int C, bool LA>
struct OutLanes {
  static constexpr bool WS = GATE == kGateChannel || LA;
  uint32_t q, q1, p, g, o;   // q, q1: the pair's two query rows
  bool odd;
  __device__ __forceinline__ OutLanes(const ChunkCursor& c, int ow, int l, int rows) {
    const int m = l & 15, lg = l >> 4, r = 16 * ow + m;
    odd = m & 1;
    const uint32_t qrow = WS ? DK * 2 : c.hd, qc = 64 * (m & 1) + 16 * lg;
    q = row_off(r & ~1, qrow, qc, WS ? C : rows);
    q1 = row_off(r | 1, qrow, qc, WS ? C : rows);
    p = C == 64 ? (r & ~1) * (C * 2) + 64 * (m & 1) + 16 * lg : r * (C * 2) + 16 * lg;
    g = (12 + r / (C / 4)) * (2 * C) + C + (r % (C / 4)) * 4;   // G_r, among the scalars in M
    o = row_off(r, c.hv, 16 * lg, rows);
  }
};

// the next chunk's rows (rows past the sequence end are zero; past the run:
// empty ranges, no traffic)
template <bool PSCAN, int DK, int GATE, int C, bool LA>
__device__ __forceinline__ void out_load(OutRows<DK, GATE, C, LA>& f, ChunkCursor& c, const OutLanes<DK, GATE, C, LA>& o) {
  constexpr int KK = DK / 32, SB = C / 32;
  constexpr bool WS = OutLanes<DK, GATE, C, LA>::WS;
  const int n = c.rows<C>();
  const auto rq = buf_rsrc(c.q, !n ? 0 : WS ? C * DK * 2 : (n - 1) * c.hd + DK * 2);
  const auto rp = buf_rsrc(c.p, n ? C * C * 2 : 0);
  const auto rm = buf_rsrc(c.m, n ? C * C * 2 : 0);
#pragma unroll
  for (int kk = 0; kk < KK; kk += 2) {
    f.q[kk] = buf_get16(rq, o.q + 64 * kk);
    f.q[kk + 1] = buf_get16(rq, o.q1 + 64 * kk);
  }
  if (!PSCAN)
#pragma unroll
    for (int s = 0; s < SB; ++s) f.p[s] = buf_get16(rp, o.p + s * (C * 2));
  if (GATE == kGateScalar)
    f.g = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, static_cast<int>(o.g), 0, 0));
  c.q += WS ? c.heads * (C * DK * 2) : C * static_cast<int64_t>(c.hd);
  c.p += c.heads * (C * C * 2);
  c.m += c.heads * (C * C * 2);
  c.next<C>();
}

// P of this wave's rows from the write keys of the stage at sg: P^T tiles
// (rows t = 32 s + 8 (m >> 2) + 4 u + (m & 3)) whose accumulators are the right
// operand of P E.  ps: where the chunk's P goes for the backward, or null.
template <int DK, int GATE, int C, bool LA>
__device__ __forceinline__ void form_p(OutRows<DK, GATE, C, LA>& f, const OutLanes<DK, GATE, C, LA>& o, const lds_char* sg,
                                       int ow, int l, char* ps) {
  using L = FwdLds<DK, GATE, C>;
  constexpr int KK = DK / 32, SB = C / 32, RK = DK * 2;
  const int m = l & 15, g = l >> 4, r = 16 * ow + m;
#pragma unroll
  for (int kk = 0; kk < KK; kk += 2) take_pair(f.q[kk], f.q[kk + 1], o.odd);
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    if (2 * s <= ow) {   // (the block right of the diagonal is zero)
      bf16x8 fk[KK][2];
      floatx4 gt[2];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          fk[kk][u] = lds_frag(sg + L::oKt + tile_off<DK / 8>(8 * (m >> 2) + (m & 3), 4 * kk + g) + (32 * s + 4 * u) * RK);
      if (GATE == kGateScalar)
#pragma unroll
        for (int u = 0; u < 2; ++u) gt[u] = lds_f4(sg + L::oM + scal_off<C>(3, 8 * s + 2 * g + u));
      reads_done();
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u] = mfma(fk[kk][u], f.q[kk], acc[u]);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = 32 * s + 8 * g + 4 * u + i;
          const float fac = GATE == kGateScalar ? fast_exp(f.g - gt[u][i]) : 1.f;
          acc[u][i] = r >= t ? acc[u][i] * fac : 0.f;
        }
    }
    f.p[s] = pack8(acc[0], acc[1]);
    // (the reverse scan does not read the block right of the diagonal)
    if (ps && 2 * s <= ow) *reinterpret_cast<bf16x8*>(ps + r * (C * 2) + 64 * s + 16 * g) = f.p[s];
  }
}

// O rows of the chunk at ob (n valid rows) from the S and E fragments of its
// step, transposed products (rows are value columns), so a lane holds eight
// adjacent columns of a row.
template <bool PSCAN, int DK, int GATE, int C, bool LA>
__device__ __forceinline__ void out_store(OutRows<DK, GATE, C, LA>& f, const OutLanes<DK, GATE, C, LA>& o, char* ob, int n,
                                          uint32_t hv, float scale, const lds_char* sS, const lds_char* sE, int l) {
  constexpr int KK = DK / 32, SB = C / 32;
  bf16x8 fs[2][KK], fe[2][SB];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) fs[v][kk] = lds_frag(sS + (v * KK + kk) * 1024 + l * 16);
#pragma unroll
    for (int s = 0; s < SB; ++s) fe[v][s] = lds_frag(sE + (v * SB + s) * 1024 + l * 16);
  }
  reads_done();
  if (!PSCAN) {
#pragma unroll
    for (int kk = 0; kk < KK; kk += 2) take_pair(f.q[kk], f.q[kk + 1], o.odd);
    if (SB == 2) take_pair(f.p[0], f.p[SB - 1], o.odd);
  }
  floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[v] = mfma(fs[v][kk], f.q[kk], acc[v]);
  if (GATE == kGateScalar) {
    const float lam = fast_exp(f.g);
    acc[0] *= lam;
    acc[1] *= lam;
  }
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[v] = mfma(fe[v][s], f.p[s], acc[v]);
  // the chunk's output rows as a buffer ending with its last valid row
  const auto rs = buf_rsrc(ob, (n - 1) * hv + kCols * 2);
  buf_put16(rs, o.o, pack8(scale * acc[0], scale * acc[1]));
}

// The rows the backward reads: the chunk-start state S^T [dk][dv] and E rows
template <int DK, int C>
__device__ __forceinline__ void keep_store(const FwdArgs& a, int i, const RunCtx& x, const lds_char* sS,
                                           const lds_char* sE, int ow, int l) {
  constexpr int NP = C / 32;   // pairs of output waves
  const int m = l & 15, g = l >> 4, hh = ow & 1;
  // (slabs of 32 columns: saved_idx)
  bf16* hs = static_cast<bf16*>(a.Hs) + a.ci(x.bh, i) * (DK * static_cast<int64_t>(a.dv)) + x.v0 * DK;
  bf16* er = static_cast<bf16*>(a.Er) + a.ci(x.bh, i) * (C * static_cast<int64_t>(a.dv)) + x.v0 * C;
  const int r0 = 8 * (m >> 2) + 4 * hh + (m & 3);
#pragma unroll
  for (int u = 0; u < DK / 32 / NP; ++u) {
    const int f = u * NP + (ow >> 1);
    *reinterpret_cast<bf16x8*>(hs + (32 * f + r0) * kCols + 8 * g) = frag_major_row<DK / 32>(sS, f, hh, l);
  }
  const int f = ow >> 1;
  *reinterpret_cast<bf16x8*>(er + (32 * f + r0) * kCols + 8 * g) = frag_major_row<C / 32>(sE, f, hh, l);
}

template <int DK, int GATE, bool SAVE, bool OUT, bool LA, int C, bool PSCAN>
__device__ __forceinline__ void fwd_run(const FwdArgs& a, const RunCtx& x, int seg, int pv0, lds_char* sm) {
  using L = FwdLds<DK, GATE, C>;
  constexpr int KK = L::KK;
  constexpr bool KEEP = SAVE || OUT;
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cnt = x.c1 - x.c0;
  const int64_t BHDK = a.BH * static_cast<int64_t>(DK);
  if (w < 2) {
    // ---- chain: columns v of this wave
    const int m = l & 15, g = l >> 4;
    const int v = 8 * (m >> 2) + 4 * w + (m & 3);
    floatx4 st[KK][2];
    bf16x8 bS[KK];
    const float* src = nullptr;   // middle segments' local runs start from zero
    if (a.seg_phase == 0 || (a.seg_phase == 1 && seg == 0)) src = a.S0 ? a.S0 + x.bh * DK * a.dv : nullptr;
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
    }
    lds_sync();   // the first chunk's tiles are in
    lds_char* sg = sm;
    int j = 0;
    auto step = [&](int par) {
      chain_step<DK, GATE, C, LA, KEEP>(sm, sg, par, w, l, st, bS);
      sg = sg == sm + 2 * L::kStage ? sm : sg + L::kStage;
      lds_sync();
    };
    for (; j + 1 < cnt; j += 2) {
      step(0);
      step(1);
    }
    if (j < cnt) step(0);
    // the end state: S_T after the sequence's last chunk; phase 1: segment
    // 0's exact end, a middle segment's local end or its transition
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
    } else if (x.c1 == a.NT && a.S_T) {
      dst = a.S_T + x.bh * DK * a.dv;
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
    // ---- output: the step after a chunk's, from the fragments its step left
    const int ow = w < 4 ? w - 2 : w - 4;
    ChunkCursor c;
    c.start<DK, GATE, C, LA>(a, x);
    const OutLanes<DK, GATE, C, LA> lanes(c, ow, l, static_cast<int>(min<int64_t>(C, a.T)));
    char* ob = static_cast<char*>(a.o) + ((x.b * a.T + static_cast<int64_t>(x.c0) * C) * a.H + x.h) * a.dv * 2 + x.v0 * 2;
    int64_t left = c.tokens;
    constexpr bool ROWS = OUT || (SAVE && PSCAN);   // the query rows are needed
    char* ps = SAVE && PSCAN ? static_cast<char*>(a.Pm) + a.ci(x.bh, x.c0) * (C * C * 2) : nullptr;
    OutRows<DK, GATE, C, LA> q[4];
    if (ROWS) {
      out_load<PSCAN, DK, GATE, C, LA>(q[0], c, lanes);
      out_load<PSCAN, DK, GATE, C, LA>(q[1], c, lanes);
    }
    const lds_char* sg = sm;   // the step's stage
    // step j: load chunk j + 2's rows, form P of chunk j (its write keys are
    // in the step's stage)
    auto begin = [&](OutRows<DK, GATE, C, LA>& next, OutRows<DK, GATE, C, LA>& f) {
      if (ROWS) out_load<PSCAN, DK, GATE, C, LA>(next, c, lanes);
      if (ROWS && PSCAN) {
        form_p<DK, GATE, C, LA>(f, lanes, sg, ow, l, ps);
        if (SAVE) ps += a.BH * (C * C * 2);
      }
      sg = sg == sm + 2 * L::kStage ? sm : sg + L::kStage;
    };
    // chunk c0 + j, a step after its own
    auto finish = [&](OutRows<DK, GATE, C, LA>& f, int j) {
      const lds_char* sS = sm + L::oS + (j & 1) * L::kS;
      const lds_char* sE = sm + L::oE + (j & 1) * L::kE;
      if (OUT) {
        out_store<PSCAN, DK, GATE, C, LA>(f, lanes, ob, static_cast<int>(min<int64_t>(C, left)), c.hv, a.scale, sS, sE, l);
        ob += C * static_cast<int64_t>(c.hv);
        left -= C;
      }
      if (SAVE) keep_store<DK, C>(a, x.c0 + j, x, sS, sE, ow, l);
    };
    lds_sync();   // the first chunk's tiles are in
    begin(q[2], q[0]);
    lds_sync();   // step 0
    // step j (chunk j's rows in set j mod 4): as above, and chunk j - 1's output
    int j = 1;
    for (; j + 3 < cnt; j += 4) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        begin(q[(d + 3) % 4], q[(d + 1) % 4]);
        if (KEEP) finish(q[d], j + d - 1);
        lds_sync();
      }
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (j + d < cnt) {
        begin(q[(d + 3) % 4], q[(d + 1) % 4]);
        if (KEEP) finish(q[d], j + d - 1);
        lds_sync();
      } else if (j + d == cnt) {
        if (KEEP) finish(q[d], j + d - 1);
      }
    }
  } else {
    // ---- loaders: chunk c0 + j goes to stage j mod 3, issued two steps
    // before its own, so a step's loads have two steps to arrive
    using F = FwdLoader<DK, GATE, C, LA>;
    const int lw = w - 4;
    const F f(a, lw, l);
    ChunkCursor c;
    c.start<DK, GATE, C, LA>(a, x);
    f.issue(c, lw, sm);
    f.issue(c, lw, sm + L::kStage);
    wait_loads<F::kLoads>();
    lds_sync();
    lds_char* sg = sm + 2 * L::kStage;
    for (int j = 0; j < cnt; ++j) {
      f.issue(c, lw, sg);
      sg = sg == sm + 2 * L::kStage ? sm : sg + L::kStage;
      wait_loads<F::kLoads>();   // the next step's chunk is in
      lds_sync();
    }
  }
}

template <int DK, int GATE, bool SAVE, bool OUT, bool LA, int C, bool PSCAN>
__global__ __launch_bounds__(scan_threads(C), 2) void fwd_scan(FwdArgs a) {
  using L = FwdLds<DK, GATE, C>;
  __shared__ __attribute__((aligned(1024))) char smem[L::kTotal];
  lds_char* sm = (lds_char*)smem;
  // workgroup -> (head, role, slab); the slabs of one head share an XCD
  // (and its L2).  Roles per head: phase 0, the value slabs of the whole
  // sequence; phase 1, segment 0's value slabs, then per middle segment its
  // value slabs (local, from zero) and d_k / 32 transition slabs; phase 3,
  // the value slabs of segments 1 .. S - 1.
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
  int seg = 0, slab = role;
  x.probe = false;
  if (a.seg_phase == 1 && role >= nslab) {
    const int r = role - nslab;
    seg = 1 + r / (nslab + npslab);
    slab = r % (nslab + npslab);
    x.probe = slab >= nslab;
  } else if (a.seg_phase == 3) {
    seg = 1 + role / nslab;
    slab = role % nslab;
  }
  x.c0 = a.seg_phase == 0 ? 0 : seg * a.seg_len;
  x.c1 = a.seg_phase == 0 ? a.NT : min(a.NT, x.c0 + a.seg_len);
  // a transition slab reads (and zeroes) value slab 0; its own columns are
  // pv0 .. pv0 + 31 of the d_k x d_k transition
  x.v0 = x.probe ? 0 : slab * kCols;
  const int pv0 = x.probe ? (slab - nslab) * kCols : 0;
  // middle segments of the first pass need only their end states
  if constexpr (!PSCAN) {
    if (a.seg_phase == 1 && seg > 0) {
      fwd_run<DK, GATE, false, false, LA, C, false>(a, x, seg, pv0, sm);
      return;
    }
  }
  fwd_run<DK, GATE, SAVE, OUT, LA, C, PSCAN>(a, x, seg, pv0, sm);
}

template <int DK, int GATE, bool SAVE, bool OUT, bool LA, int C, bool PSCAN>
hipError_t launch_typed(const FwdArgs& a0, hipStream_t s) {
  FwdArgs a = a0;
  const int nslab = a.dv / kCols;
  const auto launch = [&](int phase, int nrole) {
    a.seg_phase = phase;
    hipLaunchKernelGGL((fwd_scan<DK, GATE, SAVE, OUT, LA, C, PSCAN>), scan_grid(a.BH, nrole), dim3(scan_threads(C)), 0,
                       s, a);
    return hipGetLastError();
  };
  if (a.seg_cnt < 3) return launch(0, nslab);
  if constexpr (PSCAN) {
    return hipErrorInvalidValue;   // (scan_forms_p: never a split scan)
  } else {
    const int S = a.seg_cnt;
    hipError_t e = launch(1, nslab + (S - 2) * (nslab + DK / kCols));
    if (e != hipSuccess) return e;
    if ((e = launch_seg_compose(a, false, s)) != hipSuccess) return e;
    return launch(3, (S - 1) * nslab);
  }
}

template <int DK, int GATE, int C, bool PSCAN>
hipError_t launch_save(const FwdArgs& a, bool save, bool out, hipStream_t s) {
  if (save)
    return out ? launch_typed<DK, GATE, true, true, false, C, PSCAN>(a, s)
               : launch_typed<DK, GATE, true, false, false, C, PSCAN>(a, s);
  return launch_typed<DK, GATE, false, true, false, C, PSCAN>(a, s);
}

template <int DK, int GATE, int C>
hipError_t launch_mode(const FwdArgs& a, bool save, bool out, hipStream_t s) {
  if (a.precond == kATQ) return launch_typed<DK, GATE, false, true, true, C, false>(a, s);
  if constexpr (GATE != kGateChannel) {
    if (a.forms_p) return launch_save<DK, GATE, C, true>(a, save, out, s);
  }
  return launch_save<DK, GATE, C, false>(a, save, out, s);
}

template <int DK, int C>
hipError_t launch_gate(const FwdArgs& a, bool save, bool out, hipStream_t s) {
  switch (a.gate) {
    case kGateNone: return launch_mode<DK, kGateNone, C>(a, save, out, s);
    case kGateScalar: return launch_mode<DK, kGateScalar, C>(a, save, out, s);
    default: return launch_mode<DK, kGateChannel, C>(a, save, out, s);
  }
}

}  // namespace

hipError_t launch_fwd_scan_bf16(const FwdArgs& a, bool save, bool out, hipStream_t s) {
  if (a.chunk == 32) return a.dk == 64 ? launch_gate<64, 32>(a, save, out, s) : launch_gate<128, 32>(a, save, out, s);
  return a.dk == 64 ? launch_gate<64, 64>(a, save, out, s) : launch_gate<128, 64>(a, save, out, s);
}

}  // namespace pdn
