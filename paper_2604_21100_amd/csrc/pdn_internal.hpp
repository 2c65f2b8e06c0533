// Host/device shared parameter blocks and launchers (internal to libpdn).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pdn {

// chunk lengths C the kernels are built for
constexpr bool chunk_supported(int c) { return c == 32 || c == 64; }

enum GateKind { kGateNone = 0, kGateScalar = 1, kGateChannel = 2 };
enum PrecondKind { kSquash = 0, kIdentity = 1, kExternal = 2, kDiagSM = 3, kATQ = 4 };
enum KnormKind { kKnormNone = 0, kKnormM = 1, kKnorm1pm = 2, kKnormBeta = 3 };

// the write key (or, for ATQ, the query) comes from the diagonal Gram
// recurrence A_t = exp(gP_t) A_{t-1} + betaP_t k_t^2
constexpr bool has_gram(int precond) {
  return precond == kSquash || precond == kDiagSM || precond == kATQ;
}

// Everything the forward kernels read or write.  Per-token tensors use the
// ABI layout [B, T, H, d]; workspace tensors are head-major and padded to
// whole chunks (T_pad = NT * C rows).
struct FwdArgs {
  int64_t B, T, H, BH;
  int chunk;     // chunk length C (32 or 64)
  int NT;        // number of chunks, ceil(T / C)
  int64_t Tpad;  // NT * C
  int dk, dv;
  int gate, precond;
  float lnx;     // log(x)
  float scale;
  float ridge;   // DIAG_SM / ATQ: lambda added to A before the inverse
  int knorm;     // SQUASH write-key normalisation (pdn_knorm)
  // inputs
  const void* q;
  const void* k;
  const void* v;
  const void* ktilde;
  const float* beta;
  const float* g;
  const float* beta_p;
  const float* g_p;
  const float* log_a_scale;
  const float* A0;
  const float* S0;
  // outputs
  void* o;
  float* S_T;
  float* A_T;
  // workspace
  float* sumL;    // [BH, NT, dk]   in-chunk decayed sum of betaP k^2
  float* sumD;    // [BH, NT]       in-chunk sum of gP (log of the decay)
  float* Abound;  // [BH, NT+1, dk] preconditioner state before each chunk
  void* KtG;      // fp32: [BH, NT, dk, C] (Kt * Gamma)^T per chunk
  bool forms_p;   // bf16: the scan forms P (scan_forms_p)
  void* Kd;       // bf16: [BH, Tpad, dk] write-key rows (per-channel gate: w_r o Kt rows)
  void* Tm;       // [BH, NT, C, C]  fp32: T = M Diag(beta); bf16: M = (I + At)^{-1}
  void* Pm;       // [BH, NT, C, C]  causal (Q*Lam)(Kt/Lam)^T, io dtype
  float* G;       // scalar gate: [BH, Tpad] in-chunk log-decay prefix; per-channel
                  // gate: [BH, NT, dk], its chunk-end row only (bf16: its exponential)
  void* Qt;       // [BH, Tpad, dk] io   ATQ: preconditioned query rows q / (A + ridge)
  void* QL;       // [BH, Tpad, dk] io   per-channel gate: Lam o (the query the scan reads)
  void* KL;       // [BH, Tpad, dk] io   per-channel gate: Lam o K
  // backward only (NULL in the forward): forward intermediates kept for the
  // adjoint kernels.  lam_r = exp(G_r), w_r = exp(G_{C-1} - G_r).
  // (per-chunk tensors are indexed by ci(); bf16 Hs, Er, dHs, Zr, dKt, dKm: saved_idx)
  void* Hs;       // [BH, NT, dk, dv] io  chunk-start states S^T
  void* Er;       // [BH, Tpad, dv] io    E = T X rows
  // (fp32 only, the transposed operands its reverse scan reads:)
  void* PtT;      // [BH, NT, C, C] io    P^T
  void* MtT;      // [BH, NT, C, C] io    M^T, M = (I + At)^{-1} (T = M Diag(beta))
  void* Ktr;      // [BH, Tpad, dk] io    write key rows (bf16 without the per-channel gate: Kd)
  void* Kw;       // [BH, Tpad, dk] io    w_r o write key rows (fp32 with the per-channel gate only; bf16: Kd)
  void* QlT;      // [BH, NT, dk, C] io   (Diag(lam) Q)^T per chunk
  void* KnT;      // [BH, NT, dk, C] io   -(Diag(lam) K)^T per chunk
  // sequence split of the state scan (see scan_split): seg_phase 0 = one
  // pass over all chunks from S0; 1 = segment 0 from S0 next to the local
  // scans (from zero) and transitions (from the identity, no values) of the
  // middle segments; 3 = segments 1 .. seg_cnt - 1 from seg_start
  int seg_phase, seg_len, seg_cnt;
  float* seg_end;    // [S, BH, dk, dv] phase-1 end states (segment 0: exact; others: local)
  float* seg_phi;    // [S, BH, dk, dk] segment transitions, S_end^T = Phi S_start^T + local
  float* seg_start;  // [S, BH, dk, dv] exact start states of segments 1 .. S - 1
  // index of head bh's chunk i in the per-chunk workspace tensors
  __host__ __device__ int64_t ci(int64_t bh, int64_t i) const { return i * BH + bh; }
};

// Sequence split of the state scan.  A scan workgroup holds one head's
// 32-column state slab (one per compute unit); with few heads most of the
// chip idles through the sequential chunk loop.  The chunks are then cut
// into S segments of L: segment 0 runs from S0 while each middle segment
// runs from zero (its local end state) and, on d_k / 32 more workgroups,
// from the identity with the values zeroed (its d_k x d_k transition); a
// short sequential pass composes the exact start of every segment, and
// segments 1 .. S - 1 run again from it.  The critical path drops from NT
// steps to about 2 NT / S; S is the largest count whose first pass still
// fits one workgroup per compute unit of the target device, with at least
// kSegMinChunks chunks per segment.
//
// kSegMinChunks was set for scans of 2.5 to 3 us a step and still fits the fp32
// ones; a bf16 step now takes 1.0 to 1.6 us while the split costs two more
// launches and a composition of 5 to 7 us, so short bf16 runs would be faster
// unsplit.  Forward, us, split against unsplit at 12, 32 and 64 chunks (d = 128,
// scalar gate):
//   C = 64   1 head 43 : 35  70 : 53  123 : 83    8 heads 46 : 36  63 : 56  78 : 88    16 heads 49 : 38  65 : 60  98 : 102
//   C = 32   1 head 35 : 27  58 : 37  105 : 57    8 heads 36 : 28  49 : 39  60 : 61    16 heads 38 : 27  48 : 42  64 : 64
// (S, and with it the workspace, goes by the problem's sizes alone.)
constexpr int kScanCUs = 256;       // compute units of MI355X
constexpr int kSegMinChunks = 4;
constexpr int kSegMax = 16;
struct ScanSplit {
  int S, L;   // segments (1: no split) and chunks per segment
};
inline ScanSplit scan_split(int64_t BH, int NT, int dk, int dv) {
  const int64_t ns = dv / 32, np = dk / 32;
  ScanSplit r{1, NT};
  for (int s = 3; s <= kSegMax; ++s) {
    if (BH * (ns + (s - 2) * (ns + np)) > kScanCUs) break;
    const int L = (NT + s - 1) / s;
    if (L < kSegMinChunks) break;
    r.S = (NT + L - 1) / L;
    r.L = L;
  }
  if (r.S < 3) r = ScanSplit{1, NT};
  return r;
}

// Whether the bf16 state scan forms P itself from the query rows and write
// keys it holds, rather than the chunk preparation writing it (which then must
// read the queries): 100 to 133 MB less traffic at the 1B layer, for 48 more
// MFMA and 48 KB more LDS reads a chunk in each of a head's scan workgroups
// (C = 64, d = 128).  Worth it where that traffic leaves the last-level cache
// (256 MB): many heads and long runs.  Forward / training step, us, P written
// against formed, at 16, 32 and 64 chunks:
//   C = 64, 64 heads of 128, scalar gate  61 : 61 / 210 : 204   97 : 100 / 411 : 408   231 : 199 / 764 : 753
//   C = 64, 64 heads of 128, no gate      60 : 55 / 202 : 194   95 :  92 / 399 : 396   225 : 192 / 748 : 739
//   C = 64, 64 heads of 64 x 128, scalar  47 : 49 / 139 : 139   76 :  77 / 281 : 288   162 : 144 / 540 : 537
//   C = 64, 128 heads of 64, scalar       68 : 63 / 201 : 202  119 : 106 / 397 : 390   266 : 224 / 741 : 727
//   C = 32, 64 heads of 128, scalar       36 : 39 / 124 : 128   54 :  58 / 239 : 245    89 :  94 / 457 : 458
//   C = 32, 128 heads of 128, scalar      57 : 60 / 242 : 245   91 :  96 / 465 : 462   191 : 182 / 849 : 841
//   C = 32, 256 heads of 64, scalar       56 : 55 / 203 : 201   93 :  92 / 389 : 383   212 : 192 / 716 : 708
// So the line is too low by up to 8 % for a forward of 64 heads in chunks of 32
// (the present scans with P formed are still 1.5 times as fast there as the ones
// it came with), and too high by up to 10 % for heads of 64 in chunks of 64.
// (The per-channel gate's P has its decay inside the contraction, and linear
// attention's preparation rewrites the queries anyway.  A scan of as many
// slabs as compute units is never split: scan_split's first pass holds them all.)
inline bool scan_forms_p(int64_t BH, int NT, int dv, int gate, int precond) {
  return gate != kGateChannel && precond != kATQ && BH * (dv / 32) >= kScanCUs && NT >= 32;
}

// Backward-only arguments and workspace (the forward recompute uses f).
struct BwdArgs {
  FwdArgs f;
  const void* dO;       // [B, T, H, dv] io
  const float* dS_T;    // [B, H, dk, dv] or NULL
  // outputs
  void* dq;
  void* dk;
  void* dv;
  float* dbeta;
  float* dg;
  float* dS0;
  float* dbeta_p;
  float* dg_p;
  float* dlog_a_scale;
  float* dA0;
  void* dktilde;
  // workspace
  void* dHs;      // [BH, NT, dk, dv] io  state adjoint entering each chunk from the right
  void* Zr;       // [BH, Tpad, dv] io    Z = M^T dE rows (dX = dV = Diag(beta) Z)
  void* dKt;      // [BH, Tpad, dk] io    gradient of the write key
  void* dKm;      // [BH, Tpad, dk] io    gradient of the read key (main recurrence)
  float* pcL;     // [BH, NT, dk]         preconditioner: in-chunk adjoint at chunk start
  float* pcS;     // [BH, NT, C/16, dk]   preconditioner: per 16-token segment, the in-segment adjoint it sends left
  float* pcA;     // [BH, NT, C/16, dk]   preconditioner: per 16-token segment, the state before it
  float* pcC;     // [BH, NT + 1, dk]     preconditioner: adjoint carried into each chunk
  float* pcMu;    // [BH, NT]             preconditioner: partial d mu
};

// The reverse state-adjoint scan of bf16 problems (pdn_rscan.hip).
hipError_t launch_rev_scan_bf16(const BwdArgs& b, hipStream_t s);

// The composition pass of a split scan (seg_compose): the exact segment
// starts from the first pass's end states and transitions, forward or (rev)
// for the reverse state-adjoint scan.
hipError_t launch_seg_compose(const FwdArgs& a, bool rev, hipStream_t s);

// The state scan of bf16 problems (pdn_scan.hip): save leaves the chunk-start
// states and E rows for the backward, out forms the output.
hipError_t launch_fwd_scan_bf16(const FwdArgs& a, bool save, bool out, hipStream_t s);

// The forward over at most kStepTokens tokens as the token recurrence
// (pdn_step.hip): for inference one launch that uses no workspace; training and
// the backward's recompute launch it in the state scan's place (with Hs set it
// leaves the rows the backward reads), so every forward returns the same.
//
// A token costs it about 1.2 us of latency while its slabs of 32 columns find a
// compute unit each, and time in proportion to them past about 1024; the chunk
// kernels take the same time for any T up to a chunk.  Forward with states,
// us, recurrence at T = 8 against the chunk kernels:
//   C = 64, d = 128, scalar gate   4 heads 13 / 23   256 23 / 42   1024 71 / 110
//   fp32, d = 128, C = 64          256 heads 24 / 83   1024 71 / 305
//   fp32, d = 64, C = 32, no gate, identity          256 13 / 21   1024 34 / 67
// In bf16 at C = 32 a chunk is little work, and many heads' chunks cost less
// than eight tokens (T = 8, 6, 4 against the chunk kernels):
//   64 x 64, identity    64 heads 12 11 11 / 14   256 14 12 11 / 14   1024 35 27 20 / 24
//   64 x 128, identity   64 heads 12 12 12 / 14   256 21 16 12 / 15   1024 62 47 34 / 35
//   128 x 128, identity  64 heads 13 12 12 / 14   256 23 18 14 / 20   1024 68 52 38 / 52
//   64 x 64, squash      64 heads 12 11 11 / 19   256 15 12 11 / 20   1024 36 28 20 / 35
//   64 x 128, squash     64 heads 13 12 12 / 19   256 21 17 12 / 23   1024 64 48 35 / 46
//   128 x 128, squash    64 heads 13 11 12 / 18   256 24 19 14 / 28   1024 69 53 39 / 66
// The lines are the inference forward's; a training step of 7 or 8 tokens pays
// for the recurrence in one scan step's place up to 3 us of 50 to 80 (256 heads
// of 64 x 128, squash, C = 32, T = 8: 74 against 70; fp32, 4 heads of 64: 79
// against 77).
constexpr int kStepTokens = 8;
inline bool step_form(const FwdArgs& a, bool io_bf16) {
  int most = kStepTokens;
  if (io_bf16 && a.chunk == 32) {
    const int64_t slabs = a.BH * (a.dv / 32);
    if (!has_gram(a.precond) && slabs > 512) most = a.dk == 64 ? 4 : 6;
    if (has_gram(a.precond) && a.dk == 64 && slabs > 1024) most = 6;
  }
  return a.T <= most;
}
hipError_t launch_step_tokens(const FwdArgs& a, int io_bf16, hipStream_t s);

struct WsLayout {
  size_t sumL, sumD, Abound, KtG, Tm, Pm, G, Qt, QL, KL, seg_end, seg_phi, seg_start, total;
  ScanSplit split;
};

WsLayout fwd_ws_layout(int64_t BH, int NT, int dk, int dv, int esz, int gate, int precond, int C);

struct BwdWsLayout {
  WsLayout f;
  size_t Hs, Er, PtT, MtT, Ktr, Kw, QlT, KnT;
  size_t dHs, Zr, dKt, dKm, pcL, pcS, pcA, pcC, pcMu, total;
};

BwdWsLayout bwd_ws_layout(int64_t BH, int NT, int dk, int dv, int esz, int gate, int precond, int C);

// ev: NULL or 8 events recorded at the stage boundaries (see
// pdn_chunk_bwd_events).  recompute = false: the forward intermediates are
// already in the workspace (left there by the training forward).
hipError_t launch_backward(const BwdArgs& a, int io_bf16, hipStream_t stream,
                           hipEvent_t const* ev = nullptr, bool recompute = true);

// Fixed scratch of pdn_chunk_fwd_noalloc (PDN_NOALLOC_SCRATCH_BYTES): a
// static device array in pdn_fwd.hip, one copy per device.
constexpr size_t kNoallocScratchBytes = static_cast<size_t>(64) << 20;
constexpr int kNoallocMaxDevices = 64;

// Device address of the current device's scratch array, looked up with
// hipGetSymbolAddress on the first call made with that device current and
// cached per device (thread-safe).  Fails for device ids >= 64.
hipError_t noalloc_scratch(void** ptr);

// ev: NULL or 4 events recorded at the stage boundaries (see
// pdn_chunk_fwd_events).  train: also leave the backward's intermediates in
// the workspace (a's backward fields set).
hipError_t launch_forward(const FwdArgs& a, int io_bf16, hipStream_t stream,
                          hipEvent_t const* ev = nullptr, bool train = false);

}  // namespace pdn
