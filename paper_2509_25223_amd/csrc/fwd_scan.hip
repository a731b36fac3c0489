// Forward state-passing scan of RLA / RDN: one 256-thread workgroup per
// (sequence, head, value block of BV columns).  Value columns evolve
// independently (the clip is elementwise and every state update acts on rows
// of the paper's d_v x d_k states), so value blocks need no communication.
//
// The workgroup walks the sequence chunk by chunk.  S and R (d_k x BV fp32,
// stored transposed like the ABI) stay in MFMA accumulators for the whole
// sequence.  Per chunk, with the prep kernel's gate sums and matrices (its
// MG, MP, MR are multiplied by T^S, T^S, T^R already, so that U = T^S Y and
// what depends on it come out of Y together; RLA: T = I):
//   KS = K S0, QS = Q S0, KR = K R0, QR = Q R0                 (MFMA)
//   RDN: Y = diag(b) (V - e^{g} KS)     RLA: Y = diag(b) V;    U = T^S Y
//   p   = e^{g_{t-1}} KS + MG T^S Y     = S_{t-1} k_t         (Sec. 3.4)
//   r   = clip(V - p)                   fused, never written to HBM
//   b_t = e^{g} QS + MP T^S Y           = aS_t S_{t-1} q_t
//   RDN: YR = diag(gamma) (r - e^{h} KR)   RLA: YR = diag(gamma) r;   UR = T^R YR
//   c_t = e^{h} QR + MR T^R YR          = R_t q_t
//   o   = b + diag(gamma) c
//   S  <- e^{g_C} S + K^T diag(e^{g_C - g}) U,  R likewise with (h, UR)
// Variants: decayed residual p = e^{g} KS + MG U (= aS_t S_{t-1} k_t, MG with
// e^{g_t - g_s}); ungated output b = e^{g_{t-1}} QS + MP U (= S_{t-1} q_t, MP
// with e^{g_{t-1} - g_s}) and o = b + c; log-cosh residual r = c tanh(x / c).
//
// Operand precision (bf16 inputs; fp32 inputs use fp32 MFMA throughout):
//   K, Q x state: bf16 K/Q fragments (exact inputs, loaded from HBM straight
//     into registers) times the state split as bf16 hi + bf16 lo (~16-bit
//     mantissa, fp32 range): two MFMAs per step.  When q, k are the fp16 rows
//     of the in-operator normalisation (qk_f16, variant instance), each row
//     is split as bf16 hi + bf16 lo too (exact: 11 = 8 + 3 bits) and a third
//     MFMA adds lo x state-hi.
//   everything else: fp16 operands (intermediates bounded by the data, clip
//     and gates), fp32 accumulation.
// With `CKPT` the chunk-start states, the clip mask |x| <= c and the blocks
// U, UR and r (token-major in 32-column pieces, mm type) are stored for the backward pass.
#include <type_traits>

#include "kernels.hpp"

namespace rla {

namespace {

template <typename IN, int DK, int BV, bool RDN>
struct FwdLayout {
  static constexpr bool kBF = sizeof(IN) == 2;
  typedef typename std::conditional<kBF, f16, float>::type XT;
  typedef Tile<XT, kChunk> TT;   // token tiles: per-token blocks [BV][64]
  // K for the state update's K^T operand: bf16 inputs keep K row-major [64][DK]
  // (16-byte stores at the commit, transpose reads at the update); fp32
  // inputs store K^T [DK][64]
  typedef typename std::conditional<kBF, TrTile<XT, DK>, TT>::type TK;
  typedef Tile<IN, DK> TSC;      // state copies [BV][DK]
  // matrix slots (swizzled 64 x 64 tiles filled by LDS-DMA); with bf16 inputs
  // T^R and MR are double-buffered so the next chunk's copies land early
  static constexpr bool kDB = kBF;
  static constexpr int kNumSlots = RDN ? (kDB ? 7 : 5) : (kDB ? 4 : 3);
  static constexpr int kNumCopies = kBF ? 4 : 2;
  static constexpr int kKT = 0;
  static constexpr int kCopies = kKT + (kBF ? kChunk * TK::kRowB : DK * TT::kRowB);
  static constexpr int kCopyBytes = BV * TSC::kRowB;
  static constexpr int kMats = kCopies + kNumCopies * kCopyBytes;
  static constexpr int kBufs = kMats + kNumSlots * Swz<XT>::kBytes;
  static constexpr int kBufBytes = BV * TT::kRowB;
  static constexpr int kVc = kBufs + 6 * kBufBytes;
  static constexpr int kVBytes = kChunk * BV * (int)sizeof(IN);
  static constexpr int kGraw = kVc + kVBytes;
  static constexpr int kGates = kGraw + kGateBlock * 4;
  // output staging, so that o, the clip mask and r leave in 16-byte stores:
  // r value-major (token tile), mask value-major [BV][kMstLd] bytes, o
  // token-major [64][BV + 4] fp32
  static constexpr int kRst = kGates + 10 * kChunk * 4;
  static constexpr int kMst = kRst + kBufBytes;
  static constexpr int kLdO = BV + 4;
  static constexpr int kMstLd = kChunk + 16;
  static constexpr int kOst = kMst + BV * kMstLd;
  static constexpr int kBytes = kOst + kChunk * kLdO * 4;
  static_assert(kVBytes == 4 * 1024, "V block = one DMA instruction per wave");
  static_assert(kBytes <= 160 * 1024, "forward scan LDS");
  // slot of each matrix (RDN: TS MG MP TR[2] MR[2]; RLA: MG MP MR[2])
  __device__ static constexpr int slot(int mat, int buf) {
    if (RDN) {
      if (mat == kMatTS) return 0;
      if (mat == kMatMG) return 1;
      if (mat == kMatMP) return 2;
      if (mat == kMatTR) return kDB ? 3 + buf : 3;
      return kDB ? 5 + buf : 4;   // MR
    }
    if (mat == kMatMG) return 0;
    if (mat == kMatMP) return 1;
    return kDB ? 2 + buf : 2;     // MR
  }
};

// Writes this lane's 4 accumulator rows of a state tile into the transposed
// state copies (tile rows r0 + column, columns c0 + row): hi (and, for bf16,
// the residual lo).
template <class TL, typename IN>
__device__ __forceinline__ void store_state_copy(IN* hi, IN* lo, int r0, int c0, floatx4 v) {
  // r0, c0 multiples of 16
  const int o = TL::off_split(r0, acc_col(), acc_row(0) * (int)sizeof(IN), c0 * (int)sizeof(IN));
  if constexpr (sizeof(IN) == 2) {   // 8-byte stores of 4 consecutive rows
    uint2 h2, l2;
    bf16_split2(v[0], v[1], h2.x, l2.x);
    bf16_split2(v[2], v[3], h2.y, l2.y);
    *reinterpret_cast<uint2*>(reinterpret_cast<char*>(hi) + o) = h2;
    *reinterpret_cast<uint2*>(reinterpret_cast<char*>(lo) + o) = l2;
  } else {
    *reinterpret_cast<floatx4*>(reinterpret_cast<char*>(hi) + o) = v;
  }
}

// VAR: an instance that reads the variant flags and qk_f16 (the default
// instance compiles them away, so the boxed operator keeps its register budget)
template <typename IN, int DK, int BV, bool RDN, bool WRITE_O, bool CKPT, typename OT, bool VAR>
__global__ __launch_bounds__(kThreads) void fwd_scan_kernel(OpParams p) {
  typedef FwdLayout<IN, DK, BV, RDN> L;
  typedef typename L::XT XT;
  typedef Mfma<IN> MI;
  typedef typename L::TT TT;
  typedef typename L::TK TK;
  constexpr bool BF = L::kBF;
  constexpr int JT = BV / 16;        // value tiles per block
  constexpr int IT = DK / 64;        // state row tiles per wave
  constexpr int KS_STEPS = DK / MI::kStep;
  // store instructions per wave of the two checkpointed states (save_state_f16:
  // one row store and one scale store per 16-row tile; fp32: one per row)
  constexpr int kCkptStores = 2 * (BF ? 2 * IT : 4 * IT * JT);
  extern __shared__ __align__(16) unsigned char smem[];
  XT* KT = reinterpret_cast<XT*>(smem + L::kKT);
  IN* Shi = reinterpret_cast<IN*>(smem + L::kCopies);
  IN* Rhi = reinterpret_cast<IN*>(smem + L::kCopies + 1 * L::kCopyBytes);
  IN* Slo = reinterpret_cast<IN*>(smem + L::kCopies + 2 * L::kCopyBytes);   // bf16 only
  IN* Rlo = reinterpret_cast<IN*>(smem + L::kCopies + 3 * L::kCopyBytes);   // bf16 only
  auto mat = [&](int m, int buf) {
    return reinterpret_cast<XT*>(smem + L::kMats + L::slot(m, buf) * Swz<XT>::kBytes);
  };
  XT* Yt = reinterpret_cast<XT*>(smem + L::kBufs);
  XT* YRt = reinterpret_cast<XT*>(smem + L::kBufs + 1 * L::kBufBytes);
  XT* DUt = reinterpret_cast<XT*>(smem + L::kBufs + 2 * L::kBufBytes);
  XT* DURt = reinterpret_cast<XT*>(smem + L::kBufs + 3 * L::kBufBytes);
  // U, UR for the saved blocks (RLA: Y, YR themselves)
  XT* Ut = RDN ? reinterpret_cast<XT*>(smem + L::kBufs + 4 * L::kBufBytes) : Yt;
  XT* URt = RDN ? reinterpret_cast<XT*>(smem + L::kBufs + 5 * L::kBufBytes) : YRt;
  IN* Vc = reinterpret_cast<IN*>(smem + L::kVc);
  float* graw = reinterpret_cast<float*>(smem + L::kGraw);   // prep's gate block
  float* gbt = reinterpret_cast<float*>(smem + L::kGates);   // beta
  float* ggm = gbt + kChunk;        // gamma
  float* egs = ggm + kChunk;        // e^{g_t}
  float* egsp = egs + kChunk;       // e^{g_{t-1}}
  float* egr = egsp + kChunk;       // e^{h_t}
  float* dls = egr + kChunk;        // e^{g_C - g_t}
  float* dlr = dls + kChunk;        // e^{h_C - h_t}
  float* edge = dlr + kChunk;       // [0] = e^{g_C}, [1] = e^{h_C}
  // output weight of c: gamma (ungated: 1); the default instance reads gamma
  float* gout = VAR ? edge + kChunk : ggm;
  // per-token factors of S0 in the residual's and the base read-out's terms
  const int vf = VAR ? p.vflags : 0;
  const bool qk16 = VAR && BF && p.qk_f16;   // q, k rows are fp16
  const float* ekp = (vf & kVarDecayed) ? egs : egsp;
  const float* eqb = (vf & kVarUngated) ? egsp : egs;
  const bool tanh_resid = (vf & kVarTanh) != 0;
  XT* Rst = reinterpret_cast<XT*>(smem + L::kRst);            // r (saving mode)
  uint8_t* Mst = reinterpret_cast<uint8_t*>(smem + L::kMst);  // clip mask (saving mode)
  float* Ost = reinterpret_cast<float*>(smem + L::kOst);      // o

  const int H = p.H, DV = p.DV, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  // XCD-aware block mapping: the value blocks of one (sequence, head) pair get
  // block ids that are congruent mod 8, so they share one XCD's L2.
  const int nvb = DV / BV;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int pair = (slot / nvb) * 8 + xcd, vb = slot % nvb;
  if (pair >= p.st.nseq * H) return;
  const int n = seq_order(p.st, pair / H), h = pair % H;
  const SeqInfo si = seq_info(p.st, n);
  const int nch = (si.len + kChunk - 1) / kChunk;
  const int j0 = vb * BV;
  const float clip = p.clip;
  const int64_t state_off = ((int64_t)n * H + h) * DK * DV;

  // ---- initial states into accumulators (wave w: rows [w*DK/4, (w+1)*DK/4)) ----
  floatx4 Sacc[IT][JT], Racc[IT][JT];
  load_acc_state<IT, JT>(Sacc, p.S0, state_off + j0, DV, w * (DK / 4));
  load_acc_state<IT, JT>(Racc, p.R0, state_off + j0, DV, w * (DK / 4));
  auto write_state_copies = [&]() {
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        store_state_copy<typename L::TSC>(Shi, Slo, jt * 16, w * (DK / 4) + it * 16, Sacc[it][jt]);
        store_state_copy<typename L::TSC>(Rhi, Rlo, jt * 16, w * (DK / 4) + it * 16, Racc[it][jt]);
      }
  };
  write_state_copies();

  const IN* qg = reinterpret_cast<const IN*>(p.q);
  const IN* kg = reinterpret_cast<const IN*>(p.k);
  const IN* vg = reinterpret_cast<const IN*>(p.v);
  OT* og = reinterpret_cast<OT*>(p.o);
  const XT* matg = reinterpret_cast<const XT*>(p.mat_ws);
  XT* fblk = reinterpret_cast<XT*>(p.fwd_blk);   // CKPT: U, UR, r blocks

  // ---- staging of chunk c+1 while chunk c computes ----
  //   K, Q fragments: register prefetch (issued after P1, when chunk c's are dead)
  //   V block, gate block, T^R, MR: LDS-DMA after P1 (V, gates dead; T^R/MR
  //     double-buffered); T^S, MG, MP: LDS-DMA after P2 (their last use)
  // Completion: every wave waits for its vector memory operations and the
  // whole workgroup passes a barrier at the end of chunk c.
  typename MI::frag Kn[KS_STEPS], Qn[KS_STEPS];
  auto chunk_len = [&](int c) { return min(kChunk, si.len - c * kChunk); };
  auto mat_src = [&](int c, int m) {
    return matg + ((int64_t)(si.chunk0 + c) * H + h) * kNumMats * kMatElems + m * kMatElems;
  };
  const MatDma<XT> mdo;   // this lane's matrix DMA offsets
  auto issue_regs = [&](int c) {
    const int64_t tok = si.start + (int64_t)c * kChunk;
    // rows past the chunk's end: its last row (no branch)
    const int t = min(16 * w + (lane & 15), chunk_len(c) - 1);
    const int64_t roff = ((tok + t) * H + h) * (int64_t)DK;
    load_rowfrags<IN, DK>(Kn, kg + roff);
    load_rowfrags<IN, DK>(Qn, qg + roff);
  };
  auto issue_early = [&](int c) {   // V, gates, T^R, MR
    const int64_t tok = si.start + (int64_t)c * kChunk;
    const int len = chunk_len(c);
    {   // V block: wave w moves rows 16w..16w+15 (64 bytes each)
      constexpr int kChunksPerRow = BV * (int)sizeof(IN) / 16;
      const int P = w * 64 + lane, t = P / kChunksPerRow, cc = P % kChunksPerRow;
      const int ts = t < len ? t : len - 1;   // padding rows: any valid row (multiplied by 0)
      const IN* src = vg + ((tok + ts) * H + h) * (int64_t)DV + j0 + cc * (16 / (int)sizeof(IN));
      dma16(src, reinterpret_cast<char*>(Vc) + w * 1024);
    }
    if (w == 0)
      dma_linear_wave(p.gate_ws + ((int64_t)(si.chunk0 + c) * H + h) * kGateBlock, graw,
                      kGateBlock * 4);
    if constexpr (L::kDB) {
      if constexpr (RDN) dma_mat64<XT>(mat_src(c, kMatTR), mat(kMatTR, c & 1), mdo);
      dma_mat64<XT>(mat_src(c, kMatMR), mat(kMatMR, c & 1), mdo);
    }
  };
  auto issue_late = [&](int c) {    // T^S, MG, MP (single-buffered: T^R, RLA: MR)
    if constexpr (RDN) dma_mat64<XT>(mat_src(c, kMatTS), mat(kMatTS, 0), mdo);
    dma_mat64<XT>(mat_src(c, kMatMG), mat(kMatMG, 0), mdo);
    dma_mat64<XT>(mat_src(c, kMatMP), mat(kMatMP, 0), mdo);
    if constexpr (!L::kDB) {
      constexpr int kLast = RDN ? kMatTR : kMatMR;
      dma_mat64<XT>(mat_src(c, kLast), mat(kLast, 0), mdo);
    }
  };
  // RDN, single-buffered MR: after P3 (its fragments are in registers)
  constexpr bool kTail = RDN && !L::kDB;
  auto issue_tail = [&](int c) {
    if constexpr (kTail) dma_mat64<XT>(mat_src(c, kMatMR), mat(kMatMR, 0), mdo);
  };
  if (nch > 0) {
    issue_regs(0);
    issue_early(0);
    issue_late(0);
    issue_tail(0);
    wait_vmem();
  }
  barrier_lds();

  for (int c = 0; c < nch; ++c) {
    const int gc = si.chunk0 + c;
    const int64_t tok = si.start + (int64_t)c * kChunk;
    const int len = chunk_len(c);
    const int buf = c & 1;

    // ---- commit: K, Q fragments from the prefetch registers, K^T (XT) and
    //      the gate-derived vectors into LDS ----
    typename MI::frag Kf[KS_STEPS], Qf[KS_STEPS];
    typename MI::frag Klo[VAR ? KS_STEPS : 1], Qlo[VAR ? KS_STEPS : 1];   // fp16 rows: bf16 residuals
    {
      const int t = 16 * w + (lane & 15);
#pragma unroll
      for (int s2 = 0; s2 < KS_STEPS; ++s2) {
        // rows past the end need no zeroing (their beta, gamma are 0, so every
        // product with them is multiplied by 0 or not stored); RDN does it all
        // the same, as its loop is scheduled better with it (4096 tokens, 16
        // heads, 128 x 128, ungated output: RDN 313 us, 315 without; RLA 275, 269 without)
        Kf[s2] = Kn[s2];
        Qf[s2] = Qn[s2];
        if constexpr (RDN) {
          Kf[s2] = __builtin_bit_cast(typename MI::frag, keep_if(__builtin_bit_cast(uint4, Kn[s2]), t < len));
          Qf[s2] = __builtin_bit_cast(typename MI::frag, keep_if(__builtin_bit_cast(uint4, Qn[s2]), t < len));
        }
        if constexpr (BF) {   // row t, 8 columns: one 16-byte store
          const u16x8 kv = __builtin_bit_cast(u16x8, Kf[s2]);
          f16x8 kh;
          if constexpr (VAR) {
            if (qk16) {   // fp16 rows: K^T as is; hi + lo bf16 fragments for the state products
              kh = __builtin_bit_cast(f16x8, kv);
              const f16x8 qh = __builtin_bit_cast(f16x8, Qf[s2]);
              u16x8 khi, klo, qhi, qlo;
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float kx = (float)kh[e], qx = (float)qh[e];
                khi[e] = f2bf(kx);
                klo[e] = f2bf(kx - bf2f(khi[e]));
                qhi[e] = f2bf(qx);
                qlo[e] = f2bf(qx - bf2f(qhi[e]));
              }
              Kf[s2] = __builtin_bit_cast(typename MI::frag, khi);
              Klo[s2] = __builtin_bit_cast(typename MI::frag, klo);
              Qf[s2] = __builtin_bit_cast(typename MI::frag, qhi);
              Qlo[s2] = __builtin_bit_cast(typename MI::frag, qlo);
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) kh[e] = (f16)bf2f(kv[e]);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) kh[e] = (f16)bf2f(kv[e]);
          }
          *reinterpret_cast<f16x8*>(TK::ptr(KT, t, s2 * 32 + (lane >> 4) * 8)) = kh;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) *TT::ptr(KT, s2 * 16 + (lane >> 4) * 4 + e, t) = Kf[s2][e];
        }
      }
      // gate vectors (lane = token), shared out over the four waves by a
      // wave-uniform index; the chunk-edge factors are stored by every lane
      // of their wave to one address
      const int tt = lane, wu = __builtin_amdgcn_readfirstlane(w);
      if (wu == 0) {
        egs[tt] = __expf(graw[tt]);
        egsp[tt] = tt > 0 ? __expf(graw[max(tt - 1, 0)]) : 1.f;
      } else if (wu == 1) {
        const float gr = graw[64 + tt], grl = graw[64 + kChunk - 1];
        egr[tt] = __expf(gr);
        dlr[tt] = __expf(grl - gr);
        edge[1] = __expf(grl);
      } else if (wu == 2) {
        const float gs = graw[tt], gsl = graw[kChunk - 1];
        dls[tt] = __expf(gsl - gs);
        edge[0] = __expf(gsl);
      } else {
        gbt[tt] = graw[128 + tt];
        ggm[tt] = graw[192 + tt];
        if constexpr (VAR) gout[tt] = (vf & kVarUngated) ? 1.f : graw[192 + tt];
      }
    }
    barrier_lds();

    // ---- P1: KS, QS, KR, QR for rows 16w..16w+15 ----
    floatx4 KS[JT], QS[JT], KR[JT], QR[JT];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      KS[jt] = zero4(); QS[jt] = zero4(); KR[jt] = zero4(); QR[jt] = zero4();
      typedef typename L::TSC TSC;
      mma_rega_tile<IN, DK, TSC>(KS[jt], Kf, Shi, jt * 16);
      mma_rega_tile<IN, DK, TSC>(QS[jt], Qf, Shi, jt * 16);
      mma_rega_tile<IN, DK, TSC>(KR[jt], Kf, Rhi, jt * 16);
      mma_rega_tile<IN, DK, TSC>(QR[jt], Qf, Rhi, jt * 16);
      if constexpr (BF) {
        mma_rega_tile<IN, DK, TSC>(KS[jt], Kf, Slo, jt * 16);
        mma_rega_tile<IN, DK, TSC>(QS[jt], Qf, Slo, jt * 16);
        mma_rega_tile<IN, DK, TSC>(KR[jt], Kf, Rlo, jt * 16);
        mma_rega_tile<IN, DK, TSC>(QR[jt], Qf, Rlo, jt * 16);
        if constexpr (VAR) {
          if (qk16) {
            mma_rega_tile<IN, DK, TSC>(KS[jt], Klo, Shi, jt * 16);
            mma_rega_tile<IN, DK, TSC>(QS[jt], Qlo, Shi, jt * 16);
            mma_rega_tile<IN, DK, TSC>(KR[jt], Klo, Rhi, jt * 16);
            mma_rega_tile<IN, DK, TSC>(QR[jt], Qlo, Rhi, jt * 16);
          }
        }
      }
    }
    float vloc[JT][4];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      floatx4 y;
      if constexpr (BF) {   // V at this lane's accumulator positions: one transpose read
        const u16x4 v4 = acc_tile_tr<PadRows<IN, BV, 0>>(Vc, 16 * w, jt * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) vloc[jt][r] = bf2f(v4[r]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = 16 * w + acc_row(r);
        if constexpr (!BF) vloc[jt][r] = to_f<IN>(Vc[t * BV + jt * 16 + acc_col()]);
        y[r] = RDN ? gbt[t] * __builtin_fmaf(-egs[t], KS[jt][r], vloc[jt][r]) : gbt[t] * vloc[jt][r];
      }
      if constexpr (RDN) {
        store_acc_tile<TT>(Yt, jt * 16, 16 * w, y);
      } else {   // both stores after the last read: a read behind a store waits on its own
        floatx4 du;
#pragma unroll
        for (int r = 0; r < 4; ++r) du[r] = dls[16 * w + acc_row(r)] * y[r];
        store_acc_tile<TT>(Yt, jt * 16, 16 * w, y);
        store_acc_tile<TT>(DUt, jt * 16, 16 * w, du);
      }
    }
    // matrix fragments are loaded ahead of the barriers that precede their
    // products (each matrix landed in an earlier chunk)
    MatFrags<XT> aTS, aMG, aMP;
    if constexpr (RDN) aTS = swz_rows_frags<XT>(mat(kMatTS, 0), 16 * w);
    aMG = swz_rows_frags<XT>(mat(kMatMG, 0), 16 * w);
    aMP = swz_rows_frags<XT>(mat(kMatMP, 0), 16 * w);
    barrier_lds();
    if (c + 1 < nch) {
      issue_regs(c + 1);
      issue_early(c + 1);
    }

    // ---- P2: U = T^S Y; residual, clip, base read-out ----
    // (explicit fmas: every instantiation, saving or not, rounds alike)
    floatx4 base[JT];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      floatx4 mgu = zero4(), mpu = zero4();
      mma_frags<XT>(mgu, aMG, Yt, jt * 16);
      mma_frags<XT>(mpu, aMP, Yt, jt * 16);
      if constexpr (RDN) {
        floatx4 u = zero4(), du;
        mma_frags<XT>(u, aTS, Yt, jt * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) du[r] = dls[16 * w + acc_row(r)] * u[r];
        if constexpr (CKPT) store_acc_tile<TT>(Ut, jt * 16, 16 * w, u);
        store_acc_tile<TT>(DUt, jt * 16, 16 * w, du);
      }
      floatx4 y, rv, xv;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = 16 * w + acc_row(r);
        const float x = __builtin_fmaf(-ekp[t], KS[jt][r], vloc[jt][r]) - mgu[r];
        xv[r] = x;
        const float rr = tanh_resid ? resid_tanh(x, clip)
                                    : (clip < 0.f ? x : fminf(fmaxf(x, -clip), clip));
        rv[r] = rr;
        base[jt][r] = __builtin_fmaf(eqb[t], QS[jt][r], mpu[r]);
        y[r] = RDN ? ggm[t] * __builtin_fmaf(-egr[t], KR[jt][r], rr) : ggm[t] * rr;
      }
      if constexpr (RDN) {
        store_acc_tile<TT>(YRt, jt * 16, 16 * w, y);
      } else {
        floatx4 du;
#pragma unroll
        for (int r = 0; r < 4; ++r) du[r] = dlr[16 * w + acc_row(r)] * y[r];
        store_acc_tile<TT>(YRt, jt * 16, 16 * w, y);
        store_acc_tile<TT>(DURt, jt * 16, 16 * w, du);
      }
      if constexpr (CKPT) {
        store_acc_tile<TT>(Rst, jt * 16, 16 * w, rv);
        *reinterpret_cast<uint32_t*>(Mst + (jt * 16 + acc_col()) * L::kMstLd + 16 * w + acc_row(0)) = mask_word(xv, clip);
      }
    }
    MatFrags<XT> aTR, aMR;   // landed in the previous chunk
    if constexpr (RDN) aTR = swz_rows_frags<XT>(mat(kMatTR, buf), 16 * w);
    else aMR = swz_rows_frags<XT>(mat(kMatMR, buf), 16 * w);
    barrier_lds();
    if (c + 1 < nch) issue_late(c + 1);
    // chunk-start states for the gradient kernel, straight from the
    // accumulators (bf16 inputs: fp16 scaled per (16 rows, 32 columns)),
    // stored after the chunk's last prefetch (fp32 RDN: but for MR).  They stay
    // in flight past the chunk's end, whose wait leaves that many operations.
    if constexpr (CKPT) {
      const int64_t off = ((int64_t)gc * H + h) * DK * DV + j0;
      if constexpr (BF) {   // blocked [DV / 32][DK][32]: each wave store is 1 KiB contiguous
        const int64_t ob = ((int64_t)gc * H + h) * DK * DV + (int64_t)j0 * DK;
        const int64_t so = ((int64_t)gc * H + h) * (DK / 16) * (DV / 32) + j0 / 32;
        save_state_f16<IT>(Sacc, reinterpret_cast<f16*>(p.ck_S) + ob, 32, p.ck_S_sc + so, DV / 32, w * (DK / 4));
        save_state_f16<IT>(Racc, reinterpret_cast<f16*>(p.ck_R) + ob, 32, p.ck_R_sc + so, DV / 32, w * (DK / 4));
      } else {
        save_state_f32<IT, JT>(Sacc, reinterpret_cast<float*>(p.ck_S) + off, DV, w * (DK / 4));
        save_state_f32<IT, JT>(Racc, reinterpret_cast<float*>(p.ck_R) + off, DV, w * (DK / 4));
      }
    }

    if constexpr (RDN) {   // ---- P3: UR = T^R YR ----
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        floatx4 u = zero4();
        mma_frags<XT>(u, aTR, YRt, jt * 16);
        floatx4 du;
#pragma unroll
        for (int r = 0; r < 4; ++r) du[r] = dlr[16 * w + acc_row(r)] * u[r];
        if constexpr (CKPT) store_acc_tile<TT>(URt, jt * 16, 16 * w, u);
        store_acc_tile<TT>(DURt, jt * 16, 16 * w, du);
      }
      aMR = swz_rows_frags<XT>(mat(kMatMR, buf), 16 * w);
      barrier_lds();
      if (c + 1 < nch) issue_tail(c + 1);
    }

    // ---- P4: correction read-out; o staged, stored after the end barrier ----
    if constexpr (WRITE_O) {
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        floatx4 mru = zero4();
        mma_frags<XT>(mru, aMR, YRt, jt * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int t = 16 * w + acc_row(r);
          Ost[t * L::kLdO + jt * 16 + acc_col()] =
              __builtin_fmaf(gout[t], __builtin_fmaf(egr[t], QR[jt][r], mru[r]), base[jt][r]);
        }
      }
    }

    // ---- state update: S <- e^{g_C} S + K^T DU, R <- e^{h_C} R + K^T DUR ----
    // (bf16 inputs: the K^T fragments from transpose reads issued as inline
    // assembly, which leaves the next chunk's DMA and the checkpoint stores
    // in flight; the builtin would drain them first)
    const float eS = edge[0], eR = edge[1];
    if constexpr (BF) {
      typedef Mfma<XT> MX;
      constexpr int NF = IT * (kChunk / MX::kStep);
      int fr0[NF], fk0[NF];
#pragma unroll
      for (int n = 0; n < NF; ++n) {
        fr0[n] = w * (DK / 4) + (n / (kChunk / MX::kStep)) * 16;
        fk0[n] = (n % (kChunk / MX::kStep)) * MX::kStep;
      }
      typename MX::frag kt[NF];
      frags_tr_sync<TK, XT, NF>(KT, fr0, fk0, kt);
#pragma unroll
      for (int it = 0; it < IT; ++it)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          Sacc[it][jt] *= eS;
          Racc[it][jt] *= eR;
#pragma unroll
          for (int ks = 0; ks < kChunk / MX::kStep; ++ks) {
            const int n = it * (kChunk / MX::kStep) + ks;
            Sacc[it][jt] = MX::mma(kt[n], TT::template frag<MX>(DUt, jt * 16, ks * MX::kStep), Sacc[it][jt]);
            Racc[it][jt] = MX::mma(kt[n], TT::template frag<MX>(DURt, jt * 16, ks * MX::kStep), Racc[it][jt]);
          }
        }
    } else {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int i0 = w * (DK / 4) + it * 16;
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          Sacc[it][jt] *= eS;
          Racc[it][jt] *= eR;
          mma_tiles<XT, kChunk, TK, TT>(Sacc[it][jt], KT, i0, DUt, jt * 16);
          mma_tiles<XT, kChunk, TK, TT>(Racc[it][jt], KT, i0, DURt, jt * 16);
        }
      }
    }
    // the next chunk's DMA data must have landed before anyone reads it; the
    // checkpoint stores, issued after it (but for a single-buffered MR), may
    // still be in flight
    wait_vmem_but<CKPT && !kTail ? kCkptStores : 0>();
    barrier_lds();
    // ---- this chunk's staged outputs, in 16-byte stores (the buffers are
    //      next written after the coming chunk's first barrier) ----
    if constexpr (WRITE_O) {
      constexpr int kVE = 16 / (int)sizeof(OT);
      constexpr int kVPR = BV / kVE;
      static_assert((kChunk * kVPR) % kThreads == 0, "whole o vectors per thread");
#pragma unroll
      for (int u = 0; u < kChunk * kVPR / kThreads; ++u) {
        const int e = tid + u * kThreads, t = e / kVPR, v = e % kVPR;
        if (t < len) {
          OT* dst = og + ((tok + t) * H + h) * (int64_t)DV + j0 + v * kVE;
          const float* src = Ost + t * L::kLdO + v * kVE;
          if constexpr (sizeof(OT) == 4) {
            *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(src);
          } else {
            u16x8 ov;
#pragma unroll
            for (int k = 0; k < 8; ++k) ov[k] = f2bf(src[k]);
            *reinterpret_cast<u16x8*>(dst) = ov;
          }
        }
      }
    }
    if constexpr (CKPT) {
      // clip mask columns, 16 bytes per thread
      if (tid < BV * kChunk / 16)
        *reinterpret_cast<uint4*>(p.ck_mask + mask_off(gc, h, H, DV) + (j0 + (tid >> 2)) * kChunk + (tid & 3) * 16) =
            *reinterpret_cast<const uint4*>(Mst + (tid >> 2) * L::kMstLd + (tid & 3) * 16);
      // U, UR, r rows (value-major in LDS): rows past the end are zero
      constexpr int kVE = 16 / (int)sizeof(XT);
      constexpr int kVPR = BV / kVE;
      static_assert(kChunk * kVPR == kThreads, "one block vector per thread");
      const int t = lane, v = w;   // lanes read consecutive tokens: no bank conflicts
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const XT* srcb = b == 0 ? Ut : b == 1 ? URt : Rst;
        uint4 x;
        if constexpr (BF) {   // two transpose reads per 16-byte row piece
          x = keep_if(tile_token_vec8<TT>(srcb, v * kVE), t < len);
        } else {
          XT vals[kVE];
#pragma unroll
          for (int k = 0; k < kVE; ++k) vals[k] = t < len ? TT::at(srcb, v * kVE + k, t) : from_f<XT>(0.f);
          x = *reinterpret_cast<const uint4*>(vals);
        }
        *reinterpret_cast<uint4*>(fblk + blk_off(gc, h, H, b, DV) + blk_el(t, j0 + v * kVE)) = x;
      }
    }
    write_state_copies();
  }

  if (p.S_fin) save_state_f32<IT, JT>(Sacc, p.S_fin + state_off + j0, DV, w * (DK / 4));
  if (p.R_fin) save_state_f32<IT, JT>(Racc, p.R_fin + state_off + j0, DV, w * (DK / 4));
}

// ---------------------------------------------------------------------------
// Wave-specialised forward scan: bf16 inputs, 32 or 16 value columns, the boxed
// operator (no variant flags); Q16: q, k are the fp16 rows of the in-operator
// normalisation.  Eight waves per workgroup in two
// groups of four that pass the same barriers in the same order:
//   chain waves (0-3): hold S and R (rows 32 w' .. 32 w' + 31) in their
//     accumulators and do every product of the chunk (the algebra of
//     fwd_scan_kernel), loading only their own K and Q rows and storing
//     nothing to HBM: o goes to LDS;
//   side waves (4-7): all other HBM traffic — the chunk-start checkpoints
//     (from the chain's stage), the U, U^R, r blocks, the clip mask and o, and the staging of the next chunk (LDS-DMA of V and the
//     matrices, the gate values) — so it overlaps the chain instead of
//     stalling it.
// Per chunk (phase: chain waves | side waves):
//   1: K^T commit; KS, KR, QS, QR;               | DMA of the next V; the
//      Y = diag(b)(V - e^g KS)                      previous o, r rows and mask; S
//                                                   checkpoint
//   2: U = T^S Y; p, r = clip(V - p), mask, Y^R;  | the previous U^R rows
//      base = e^g QS + MP T^S Y; next K, Q rows     and gate vectors; DMA of the
//                                                   gates after the next
//   3: U^R = T^R Y^R; o = base + diag(gamma) c;   | DMA of the next T^S, MG, MP; R
//      S update, its copies                         checkpoint; U rows
//   4: R update, its copies                       | DMA of the next T^R, MR
// RLA (U = Y, U^R = Y^R) has no barrier between phases 3 and 4 and refills
// all its matrices in phase 3.  Within a phase the chain issues what it reads
// from LDS first and its products in the order in which the next phase waits
// for them; everything else fills their latencies.  A matrix is read into
// registers at the start of the phase that multiplies by it and refilled in
// the next, and its copy is waited for just before that phase in the next
// chunk: the memory operations are spread over the chunk (all of a chunk's
// traffic, 100 KiB, goes through one CU's path; in bursts it stalls both roles)
// and each has most of a chunk to land.
// A chunk is bound by the serial chain (one workgroup per CU), about 6600
// cycles, and when it saves for the backward pass on every CU by the chain and
// the side waves about alike, about 8100.  With U, p and base from Y in one
// phase instead of two (128 x 128, 16 heads): 1 x 16384 tokens, 64 workgroups,
// 824 -> 656 us; saving, 4 x 4096 tokens, 256 workgroups, 287 -> 267 us;
// normalised rows, saving, 16000 tokens packed, 414 -> 344 us.
// BV = 16 (not saving; a saved checkpoint's scales are per 32 columns): half
// the columns per workgroup, for grids that leave CUs idle (the line: below, at
// launch_fwd_t); a chunk is about 4800 cycles (1 x 16384 tokens: 64 -> 128 workgroups, 651 -> 522 us, with the
// gate vectors formed in phase 2).  Columns do not meet in any product, so the
// bits are those of 32 columns.
// V is double-buffered.  The precision scheme and the arithmetic are those of
// fwd_scan_kernel, except that the split-state products sum the hi and lo terms
// per k-step.  Q16 rows are split as bf16 hi + lo in the chain's registers (a
// third MFMA adds lo x state-hi).
// The chunk-start checkpoints come from the fp32 accumulators through a stage in
// LDS: at d_k = 128 the chain stores the fp32 state beside its split copies and the
// side waves scale and convert it; at d_k = 64 (one 16-row tile of a state per wave)
// the chain does.  Saving forward scan, 16 heads, against forming them from the split
// copies (16 bits of the state): 128 x 128, packed 16000 normalised rows 340 -> 343 us,
// 4 x 4096 tokens 268 -> 269; 64 x 64, 4 x 4096 tokens 152 -> 153, RLA 155 -> 140 (the
// fp32 stage: 156, 155; converting in the chain at 128: 353, 269).  The split copies'
// 16 bits made the error of the decay parameters' gradients, sums over every token,
// 1 % larger (RLA, normalised rows, 64 x 64; 24 inputs); from fp32 it is what it was.
// ---------------------------------------------------------------------------
template <typename IN, int DK, int BV, bool RDN, bool CKPT>
struct FwdWsLayout {
  typedef f16 XT;
  typedef Tile<XT, kChunk> TT;
  typedef TrTile<XT, DK> TK;
  typedef Tile<IN, DK> TSC;
  static constexpr int kNumSlots = RDN ? 5 : 3;
  static constexpr int kKT = 0;
  static constexpr int kCopies = kKT + kChunk * TK::kRowB;
  static constexpr int kCopyBytes = BV * TSC::kRowB;
  static constexpr int kMats = kCopies + 4 * kCopyBytes;
  static constexpr int kBufs = kMats + kNumSlots * kPkBytes;   // matrices as their ten lower blocks
  static constexpr int kBufBytes = BV * TT::kRowB;
  static constexpr int kVBytes = kChunk * BV * (int)sizeof(IN);
  static constexpr int kVc = kBufs + (CKPT ? 6 : 4) * kBufBytes;   // two V blocks (chunk parity)
  static constexpr int kGateVec = 8 * kChunk;         // floats per chunk's gate vectors
  static constexpr int kGates = kVc + 2 * kVBytes;    // two sets (chunk parity)
  static constexpr int kRst = kGates + 2 * kGateVec * 4;
  static constexpr int kMst = kRst + (CKPT ? kBufBytes : 0);
  static constexpr int kMstLd = kChunk + 16;            // clip mask, value-major [BV][kMstLd] bytes
  static constexpr int kGraw = kMst + (CKPT ? BV * kMstLd : 0);   // the gate block (one side wave's DMA)
  static constexpr int kZero = kGraw + kGateBlock * 4;   // 16 zero bytes (blocks above the diagonal)
  // o of a chunk in fp32, column-major [BV][kOstLd] (the pad keeps the side's
  // 4-byte gathers of one token's 4 columns in distinct banks)
  static constexpr int kOstLd = kChunk + 4;
  static constexpr int kOst = kZero + 16;
  // S, R for the checkpoints: in fp32, column-major [BV][kCkLd] (padded like
  // o's), or (kPack) in fp16, each 16-row tile divided by its power of two
  // ([BV][DK] padded rows), with the tile scales [2][DK / 16] behind
  static constexpr bool kPack = DK == 64;
  typedef PadRows<XT, DK, 8> TCK;
  static constexpr int kCkLd = DK + 4;
  static constexpr int kCk = kOst + BV * kOstLd * 4;
  static constexpr int kCkBytes = !CKPT ? 0 : kPack ? BV * TCK::kRowB : BV * kCkLd * 4;
  static constexpr int kCkSc = kCk + 2 * kCkBytes;
  static constexpr int kBytes = kCkSc + (CKPT && kPack ? 2 * (DK / 16) * 4 : 0);
  static_assert(sizeof(IN) == 2 && (BV == 32 || (BV == 16 && !CKPT)), "bf16; saved blocks have 32 columns");
  static_assert(kBytes <= (BV == 16 ? 80 : 160) * 1024, "forward scan LDS: one or two workgroups per CU");
  // RDN: T^S, MG, MP, T^R, MR; RLA: MG, MP, MR
  __device__ static constexpr int slot(int mat) {
    if (!RDN) return mat == kMatMG ? 0 : mat == kMatMP ? 1 : 2;
    return mat == kMatTS ? 0 : mat == kMatMG ? 1 : mat == kMatMP ? 2 : mat == kMatTR ? 3 : 4;
  }
};

template <typename IN, int DK, int BV, bool RDN, bool WRITE_O, bool CKPT, bool Q16>
__global__ __launch_bounds__(2 * kThreads, 2) void fwd_scan_ws_kernel(OpParams p) {
  typedef FwdWsLayout<IN, DK, BV, RDN, CKPT> L;
  typedef typename L::XT XT;
  typedef Mfma<IN> MI;
  typedef typename L::TT TT;
  typedef typename L::TK TK;
  typedef typename L::TSC TSC;
  constexpr int JT = BV / 16;          // value tiles per block
  constexpr int IT = DK / 64;          // state row tiles per wave
  constexpr int KS_STEPS = DK / MI::kStep;
  extern __shared__ __align__(16) unsigned char smem[];
  XT* KT = reinterpret_cast<XT*>(smem + L::kKT);
  IN* Shi = reinterpret_cast<IN*>(smem + L::kCopies);
  IN* Rhi = reinterpret_cast<IN*>(smem + L::kCopies + 1 * L::kCopyBytes);
  IN* Slo = reinterpret_cast<IN*>(smem + L::kCopies + 2 * L::kCopyBytes);
  IN* Rlo = reinterpret_cast<IN*>(smem + L::kCopies + 3 * L::kCopyBytes);
  auto mat = [&](int m) { return reinterpret_cast<XT*>(smem + L::kMats + L::slot(m) * kPkBytes); };
  const XT* zero16 = reinterpret_cast<const XT*>(smem + L::kZero);
  XT* Yt = reinterpret_cast<XT*>(smem + L::kBufs);
  XT* YRt = reinterpret_cast<XT*>(smem + L::kBufs + 1 * L::kBufBytes);
  XT* DUt = reinterpret_cast<XT*>(smem + L::kBufs + 2 * L::kBufBytes);
  XT* DURt = reinterpret_cast<XT*>(smem + L::kBufs + 3 * L::kBufBytes);
  // U, UR for the saved blocks (RLA: Y, YR themselves)
  XT* Ut = RDN ? reinterpret_cast<XT*>(smem + L::kBufs + 4 * L::kBufBytes) : Yt;
  XT* URt = RDN ? reinterpret_cast<XT*>(smem + L::kBufs + 5 * L::kBufBytes) : YRt;
  auto vblk = [&](int c) { return reinterpret_cast<IN*>(smem + L::kVc + (c & 1) * L::kVBytes); };
  float* gates = reinterpret_cast<float*>(smem + L::kGates);
  XT* Rst = reinterpret_cast<XT*>(smem + L::kRst);            // r (saving mode)
  uint8_t* Mst = reinterpret_cast<uint8_t*>(smem + L::kMst);  // clip mask (saving mode)
  float* graw = reinterpret_cast<float*>(smem + L::kGraw);     // prep's gate block
  auto ckst = [&](int st) { return reinterpret_cast<float*>(smem + L::kCk + st * L::kCkBytes); };   // saving mode
  float* ckscl = reinterpret_cast<float*>(smem + L::kCkSc);

  const int H = p.H, DV = p.DV, tid = threadIdx.x, lane = tid & 63;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool chain = wu < kWaves;      // wave-uniform role
  const int ww = wu & (kWaves - 1);    // index within the role's four waves
  // XCD-aware block mapping (as fwd_scan_kernel)
  const int nvb = DV / BV;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int pair = (slot / nvb) * 8 + xcd, vb = slot % nvb;
  if (pair >= p.st.nseq * H) return;
  const int n = seq_order(p.st, pair / H), h = pair % H;
  const SeqInfo si = seq_info(p.st, n);
  const int nch = (si.len + kChunk - 1) / kChunk;
  const int j0 = vb * BV;
  const float clip = p.clip;
  const int64_t state_off = ((int64_t)n * H + h) * DK * DV;

  const IN* qg = reinterpret_cast<const IN*>(p.q);
  const IN* kg = reinterpret_cast<const IN*>(p.k);
  const IN* vg = reinterpret_cast<const IN*>(p.v);
  const XT* matg = reinterpret_cast<const XT*>(p.mat_ws);
  XT* fblk = reinterpret_cast<XT*>(p.fwd_blk);   // CKPT: U, UR, r blocks
  auto chunk_len = [&](int c) { return min(kChunk, si.len - c * kChunk); };
  auto mat_src = [&](int c, int m) {
    return matg + ((int64_t)(si.chunk0 + c) * H + h) * kNumMats * kMatElems + m * kMatElems;
  };
  // gate vectors of chunk c: beta, gamma, e^{g_t}, e^{g_{t-1}}, e^{h_t},
  // e^{g_C - g_t}, e^{h_C - h_t}, then [e^{g_C}, e^{h_C}]
  auto gvec = [&](int c, int k) { return gates + (c & 1) * L::kGateVec + k * kChunk; };

  // One loop body, instantiated once per role (std::true_type: chain
  // waves): both roles pass the same barriers in the same order by
  // construction, and each instance gets its own registers.
  auto run = [&](auto role) {
  constexpr bool CH = decltype(role)::value;
  floatx4 Sacc[IT][JT], Racc[IT][JT];  // chain: the states
  typename MI::frag Kn[KS_STEPS], Qn[KS_STEPS];   // chain: next chunk's K, Q rows 16 ww + (lane & 15)
  if constexpr (CH) {
    load_acc_state<IT, JT>(Sacc, p.S0, state_off + j0, DV, ww * (DK / 4));
    load_acc_state<IT, JT>(Racc, p.R0, state_off + j0, DV, ww * (DK / 4));
  }
  // chain: state X's (st: 0 = S, 1 = R) split copies and, saving without
  // kPack, its fp32 stage (tile by tile with the copies: behind them all it took
  // 199 us instead of 193, RLA 1 x 4096 tokens, 16 heads, 128 x 128)
  auto write_state_copies = [&](const floatx4 (&acc)[IT][JT], int st) {
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        store_state_copy<TSC>(st ? Rhi : Shi, st ? Rlo : Slo, jt * 16, ww * (DK / 4) + it * 16, acc[it][jt]);
        if constexpr (CKPT && !L::kPack)   // this lane's 4 rows of its column, one store
          *reinterpret_cast<floatx4*>(ckst(st) + (jt * 16 + acc_col()) * L::kCkLd + ww * (DK / 4) + it * 16 + acc_row(0)) =
              acc[it][jt];
      }
  };
  // chain, saving with kPack: state X into its fp16 stage
  auto stage_ckpt = [&](const floatx4 (&acc)[IT][JT], int st) {
    if constexpr (CKPT && L::kPack) {
      uint32_t m[IT];
      state_tile_absmax<IT>(acc, m);
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int ex = pow2_scale_exp(m[it]);
        const float f = exp2_int(-ex);
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
          store_acc_tile<typename L::TCK>(ckst(st), jt * 16, ww * (DK / 4) + 16 * it, acc[it][jt] * f);
        ckscl[st * (DK / 16) + ww * IT + it] = exp2_int(ex);   // every lane: the wave-uniform value
      }
    }
  };
  // Global addresses are a chunk's uniform base plus a 32-bit lane offset
  // that does not change from chunk to chunk, so the memory instructions take
  // a scalar base and the lane part is formed once.
  auto issue_rows = [&](typename MI::frag (&dst)[KS_STEPS], const IN* src, int c) {
    const int64_t tok = si.start + (int64_t)c * kChunk;
    // padding rows: the last row (their beta, gamma are 0, so every product
    // with them is multiplied by 0 or not stored)
    const int t = min(16 * ww + (lane & 15), chunk_len(c) - 1);
    const IN* base = src + (tok * H + h) * (int64_t)DK;
    const uint32_t o = (uint32_t)(t * H * DK + (lane >> 4) * 8);
#pragma unroll
    for (int s2 = 0; s2 < KS_STEPS; ++s2)
      dst[s2] = __builtin_bit_cast(typename MI::frag, *reinterpret_cast<const u16x8*>(base + o + s2 * 32));
  };
  // side wave 0 moves chunk c's gate block (g, h, beta, gamma) into LDS with
  // one DMA instruction and, after its wait, forms every gate vector
  auto issue_gates = [&](int c) {
    if (ww != 0) return;
    RLA_NOTE("copy gates");
    dma_linear_wave(p.gate_ws + ((int64_t)(si.chunk0 + c) * H + h) * kGateBlock, graw, kGateBlock * 4);
  };
  auto write_gates = [&](int c) {
    if (ww != 0) return;
    RLA_NOTE("await gates");
    write_gate_vectors(graw, gvec(c, 0));
  };
  // side waves: the five DMA instructions of the g-th matrix of a group are
  // dealt round-robin over the four side waves (the group's instruction k
  // to wave k mod 4): a wave issues at least 2 of a group of two, 3 of three
  auto dma_mat = [&](int c, int m, int g) {
    dma_mat_packed<false>(mat_src(c, m), mat(m), ((ww - 5 * g) % 4 + 4) % 4, kWaves);
  };
  auto issue_v = [&](int c) {   // V of chunk c (double-buffered)
    RLA_NOTE("copy V");
    const int64_t tok = si.start + (int64_t)c * kChunk;
    const int len = chunk_len(c);
    constexpr int kChunksPerRow = BV * (int)sizeof(IN) / 16;
    if (ww >= L::kVBytes / 1024) return;    // one instruction per wave
    const int P = ww * 64 + lane, t = P / kChunksPerRow, cc = P % kChunksPerRow;
    const int ts = t < len ? t : len - 1;   // padding rows: any valid row (multiplied by 0)
    dma16(vg + (tok * H + h) * (int64_t)DV + j0 + (uint32_t)(ts * H * DV + cc * (16 / (int)sizeof(IN))),
          reinterpret_cast<char*>(vblk(c)) + ww * 1024);
  };
  auto issue_s_mats = [&](int c) {   // T^S, MG, MP (RLA: MG, MP, MR)
    RLA_NOTE("copy S matrices");
    dma_mat(c, RDN ? (int)kMatTS : (int)kMatMR, 0);
    dma_mat(c, kMatMG, 1);
    dma_mat(c, kMatMP, 2);
  };
  auto issue_r_mats = [&](int c) {   // T^R, MR
    if constexpr (RDN) {
      RLA_NOTE("copy R matrices");
      dma_mat(c, kMatTR, 0);
      dma_mat(c, kMatMR, 1);
    }
  };
  // The side's waits leave its newest memory operations in flight, so the
  // order in which it issues groups of them is pinned (RLA_NOTE).
  constexpr int kCk = CKPT ? IT + 1 : 0;   // stores of one checkpoint
  constexpr int kBl = CKPT ? 1 : 0;        // store of one block
  // side waves: tokens 16 ww .. 16 ww + 15 of a token-major block, one
  // 64-byte segment per token (lane (g, i): token 16 ww + i, values 8 g ..
  // 8 g + 7); rows past the end are zero
  auto store_block = [&](int c, int b, const XT* src) {
    const int64_t gc = si.chunk0 + c;
    const int t = 16 * ww + (lane & 15);
    const uint4 x = keep_if(tile_token_rows16_sync<TT>(src, 16 * ww), t < chunk_len(c));
    store_stream16(fblk + blk_off(gc, h, H, b, DV) + j0 * kChunk + (uint32_t)(t * 32 + 8 * (lane >> 4)), x);
  };
  // side waves: chunk c's r rows and clip mask columns (waves 2, 3; one
  // 16-byte piece per lane)
  auto store_resid = [&](int c) {
    store_block(c, 2, Rst);
    if (ww >= 2) {
      const int e = (ww - 2) * 64 + lane;
      *reinterpret_cast<uint4*>(p.ck_mask + mask_off(si.chunk0 + c, h, H, DV) + j0 * kChunk + (uint32_t)(e * 16)) =
          lds_read16_sync(Mst + (e >> 2) * L::kMstLd + (e & 3) * 16);
    }
  };
  // side waves: chunk-start state X from its stage, rows ww DK / 4 .., fp16
  // blocked [DV / 32][DK][32] with one power-of-two scale per 16-row tile.
  // Transpose reads (fp32: eight reads) give lane (g, i) state row t0 + i at
  // columns 8 g .. 8 g + 7, so one 16-row tile is one 1 KiB store; the wave's
  // tile scales leave in one store (lane l writes tile l's)
  auto store_ckpt = [&](int c, int st) {
    const int64_t gc = si.chunk0 + c;
    f16* dst = reinterpret_cast<f16*>(st ? p.ck_R : p.ck_S) + ((int64_t)gc * H + h) * DK * DV + (int64_t)j0 * DK;
    auto put = [&](int it, uint4 v) {
      store_stream16(dst + (uint32_t)((ww * (DK / 4) + 16 * it + (lane & 15)) * 32 + 8 * (lane >> 4)), v);
    };
    float sc[IT];
    if constexpr (L::kPack) {
      uint4 v[IT];
      float* src[IT];
      int t0[IT], idx[IT];
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        src[it] = ckst(st);
        t0[it] = ww * (DK / 4) + 16 * it;
        idx[it] = st * (DK / 16) + ww * IT + it;
      }
      tile_token_rows16_sync<typename L::TCK>(src, t0, v);
      lds_read_f32_sync<IT>(ckscl, idx, sc);
#pragma unroll
      for (int it = 0; it < IT; ++it) put(it, v[it]);
    } else {
      float x[8 * IT];
      int idx[8 * IT];
#pragma unroll
      for (int k = 0; k < 8 * IT; ++k)
        idx[k] = (8 * (lane >> 4) + (k & 7)) * L::kCkLd + ww * (DK / 4) + 16 * (k >> 3) + (lane & 15);
      lds_read_f32_sync<8 * IT>(ckst(st), idx, x);
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        uint32_t m = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) m = max(m, __float_as_uint(x[8 * it + e]) & 0x7FFFFFFFu);
        const int ex = pow2_scale_exp(wave_absmax_bits(m));
        const float f = exp2_int(-ex);
        uint32_t u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = cvt_pk_f16(x[8 * it + 2 * e] * f, x[8 * it + 2 * e + 1] * f);
        put(it, uint4{u[0], u[1], u[2], u[3]});
        sc[it] = exp2_int(ex);
      }
    }
    static_assert(IT <= 2, "one or two tiles per wave");
    const int64_t so = ((int64_t)gc * H + h) * (DK / 16) * (DV / 32) + j0 / 32;
    if (lane < IT)   // one lane per tile scale
      (st ? p.ck_R_sc : p.ck_S_sc)[so + (int64_t)(ww * IT + lane) * (DV / 32)] = lane ? sc[IT - 1] : sc[0];
  };

  typedef Mfma<XT> MX;
  constexpr int XS = kChunk / MX::kStep;   // k-steps over the chunk's tokens
  // the fragments of a token tile's JT column blocks
  auto tok_frags = [&](const XT* tile, typename MX::frag (&f)[JT][XS]) {
#pragma unroll
    for (int ks = 0; ks < XS; ++ks)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) f[jt][ks] = TT::template frag<MX>(tile, jt * 16, ks * MX::kStep);
  };
  // acc[jt] += a * tile, the column blocks' chains interleaved
  auto mma_tok = [&](floatx4 (&acc)[JT], const MatFrags<XT>& a, const typename MX::frag (&f)[JT][XS]) {
#pragma unroll
    for (int ks = 0; ks < XS; ++ks)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) acc[jt] = MX::mma(a.f[ks], f[jt][ks], acc[jt]);
  };
  // X <- e X + K^T dX (the chunk's decayed corrections)
  auto update_state = [&](floatx4 (&acc)[IT][JT], float e, const typename MX::frag (&kt)[IT * XS],
                          const typename MX::frag (&f)[JT][XS]) {
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) acc[it][jt] *= e;
#pragma unroll
    for (int ks = 0; ks < XS; ++ks)
#pragma unroll
      for (int it = 0; it < IT; ++it)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) acc[it][jt] = MX::mma(kt[it * XS + ks], f[jt][ks], acc[it][jt]);
  };

  // o from the column-major stage: four 4-byte reads give a lane 4 columns of
  // one token (bf16: eight reads, 8 columns)
  float* ost = reinterpret_cast<float*>(smem + L::kOst);
  auto store_o = [&](int c) {   // side waves: chunk c's o rows 16 ww .. 16 ww + 15
    const int64_t tok = si.start + (int64_t)c * kChunk;
    const int len = chunk_len(c);
    const int64_t ob = (tok * H + h) * (int64_t)DV + j0;
    const int t = 16 * ww + (lane >> 2);
    if (p.out_bf16) {
      const int col = BV / 4 * (lane & 3);
      u16* dst = reinterpret_cast<u16*>(p.o) + ob + (uint32_t)(t * H * DV + col);
      const uint4 a = lds_read4x1_sync(ost + col * L::kOstLd + t, L::kOstLd * 4);
      if constexpr (BV == 32) {
        const uint4 b = lds_read4x1_sync(ost + (col + 4) * L::kOstLd + t, L::kOstLd * 4);
        const uint4 v = {cvt_pk_bf16(a.x, a.y), cvt_pk_bf16(a.z, a.w), cvt_pk_bf16(b.x, b.y), cvt_pk_bf16(b.z, b.w)};
        if (t < len) *reinterpret_cast<uint4*>(dst) = v;
      } else {
        const uint2 v = {cvt_pk_bf16(a.x, a.y), cvt_pk_bf16(a.z, a.w)};
        if (t < len) *reinterpret_cast<uint2*>(dst) = v;
      }
    } else {
      const int col = 4 * (lane & 3);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const uint4 v = lds_read4x1_sync(ost + (jt * 16 + col) * L::kOstLd + t, L::kOstLd * 4);
        if (t < len)
          *reinterpret_cast<uint4*>(reinterpret_cast<float*>(p.o) + ob + jt * 16 + (uint32_t)(t * H * DV + col)) = v;
      }
    }
  };

  // ---- prologue: chunk 0's staging and the initial state copies ----
  if (threadIdx.x == 0) *reinterpret_cast<uint4*>(smem + L::kZero) = uint4{0, 0, 0, 0};
  if (nch > 0) {
    if constexpr (CH) {
      issue_rows(Kn, kg, 0);
      issue_rows(Qn, qg, 0);
    } else {
      RLA_NOTE("side waves");
      issue_gates(0);
      issue_v(0);
      issue_s_mats(0);
      issue_r_mats(0);
      wait_vmem();
      write_gates(0);
      if (nch > 1) issue_gates(1);
    }
  }
  if constexpr (CH) {
    write_state_copies(Sacc, 0);
    write_state_copies(Racc, 1);
    if constexpr (RDN) stage_ckpt(Sacc, 0);
  }
  barrier_lds();

  floatx4 KS[JT], KR[JT], QS[JT], QR[JT], vloc[JT], base[JT];
  MatFrags<XT> aTS, aMG, aMP, aTR, aMR;
  typename MX::frag kt[IT * XS];   // this wave's state rows of K^T
  for (int c = 0; c < nch; ++c) {
    const bool more = c + 1 < nch;
    // this lane's four tokens of gate vector k
    auto gate4 = [&](int k) { return *reinterpret_cast<const floatx4*>(gvec(c, k) + 16 * ww + acc_row(0)); };
    floatx4 gbt, ggm, egs, egsp, egr, dls, dlr;
    float eS, eR;

    // ======== phase 1: KS, KR, QS, QR; Y = diag(b) (V - e^g KS) (RLA: diag(b) V) ========
    if constexpr (CH) {
      // fragments of the state copies, one k-step ahead of their products
      typename MI::frag f[2][4][JT];
      auto load_states = [&](int s2) {
        const IN* src[4] = {Shi, Rhi, Slo, Rlo};
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int jt = 0; jt < JT; ++jt) f[s2 & 1][x][jt] = TSC::template frag<MI>(src[x], jt * 16, s2 * MI::kStep);
      };
      load_states(0);
      sched_fence();
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) KS[jt] = KR[jt] = QS[jt] = QR[jt] = zero4();
#pragma unroll
      for (int s2 = 0; s2 < KS_STEPS; ++s2) {
        if (s2 + 1 < KS_STEPS) load_states(s2 + 1);
        else {   // what the end of the phase and the next one need
          gbt = gate4(0);
          egs = gate4(2);
#pragma unroll
          for (int jt = 0; jt < JT; ++jt) {
            const u16x4 v4 = acc_tile_tr<PadRows<IN, BV, 0>>(vblk(c), 16 * ww, jt * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) vloc[jt][r] = bf2f(v4[r]);
          }
          if constexpr (!RDN) dls = gate4(5);
        }
        sched_fence();
        // K^T commit: row 16 ww + (lane & 15), 8 columns per store
        typename MI::frag kf = Kn[s2], qf = Qn[s2], kl, ql;
        f16x8 kh;
        if constexpr (Q16) {
          kh = __builtin_bit_cast(f16x8, Kn[s2]);
          f16_split8(kh, kf, kl);
          f16_split8(__builtin_bit_cast(f16x8, Qn[s2]), qf, ql);
        } else {
          const u16x8 kv = __builtin_bit_cast(u16x8, kf);
#pragma unroll
          for (int e = 0; e < 8; ++e) kh[e] = (f16)bf2f(kv[e]);
        }
        auto& fs = f[s2 & 1];
        // eight independent chains (value tile x state x K/Q), each adding
        // the hi and the lo product of every k-step (Q16: also the rows'
        // residual times hi)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int jt = 0; jt < JT; ++jt) {
            floatx4& k = (x & 1) ? KR[jt] : KS[jt];
            floatx4& q = (x & 1) ? QR[jt] : QS[jt];
            k = MI::mma(kf, fs[x][jt], k);
            if constexpr (WRITE_O) q = MI::mma(qf, fs[x][jt], q);
          }
        if constexpr (Q16) {
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) {
              floatx4& k = (x & 1) ? KR[jt] : KS[jt];
              floatx4& q = (x & 1) ? QR[jt] : QS[jt];
              k = MI::mma(kl, fs[x][jt], k);
              if constexpr (WRITE_O) q = MI::mma(ql, fs[x][jt], q);
            }
        }
        *reinterpret_cast<f16x8*>(TK::ptr(KT, 16 * ww + (lane & 15), s2 * 32 + (lane >> 4) * 8)) = kh;
      }
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        floatx4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y[r] = RDN ? gbt[r] * __builtin_fmaf(-egs[r], KS[jt][r], vloc[jt][r]) : gbt[r] * vloc[jt][r];
        store_acc_tile<TT>(Yt, jt * 16, 16 * ww, y);
        if constexpr (!RDN) store_acc_tile<TT>(DUt, jt * 16, 16 * ww, dls * y);
      }
      sched_fence();
      ggm = gate4(1);
      egsp = gate4(3);
      egr = gate4(4);
      if constexpr (RDN) dls = gate4(5);
      dlr = gate4(6);
      eS = gvec(c, 7)[0];
      eR = gvec(c, 7)[1];
      if constexpr (!RDN) stage_ckpt(Sacc, 0);
      stage_ckpt(Racc, 1);
    } else {
      if (more) issue_v(c + 1);
      if (c > 0) {
        RLA_NOTE("store o, r");   // of a whole chunk: every row of o is there
        if constexpr (WRITE_O) store_o(c - 1);
        if constexpr (CKPT) store_resid(c - 1);
      }
      if constexpr (CKPT && RDN) store_ckpt(c, 0);   // chunk-start S
      // this chunk's T^S, MG, MP (from phase 3); since then: RDN T^R, MR, the
      // R checkpoint, U and what is above; RLA U, U^R and what is above (the
      // previous chunk's o and r; chunk 0 waited for everything)
      wait_vmem_but<RDN ? 2 + 2 * kCk + kBl : CKPT ? 3 : 1>();
      RLA_NOTE("await S matrices");
    }
    barrier_lds();

    // ======== phase 2: U; residual, clip, Y^R (explicit fmas as fwd_scan_kernel); base read-out ========
    if constexpr (CH) {
      typename MX::frag fy[JT][XS];
      tok_frags(Yt, fy);
      aMG = packed_rows_frags(mat(kMatMG), ww, zero16);
      if constexpr (RDN) aTS = packed_rows_frags(mat(kMatTS), ww, zero16);
      if constexpr (WRITE_O) aMP = packed_rows_frags(mat(kMatMP), ww, zero16);
      if constexpr (WRITE_O && !RDN) aMR = packed_rows_frags(mat(kMatMR), ww, zero16);
      sched_fence();
      if (more) {   // the next K, Q rows, while the side waves issue little
        issue_rows(Kn, kg, c + 1);
        issue_rows(Qn, qg, c + 1);
      }
      floatx4 pre[JT], mgu[JT], u[JT];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) pre[jt][r] = __builtin_fmaf(-egsp[r], KS[jt][r], vloc[jt][r]);
        mgu[jt] = u[jt] = base[jt] = zero4();
      }
      sched_fence();
      mma_tok(mgu, aMG, fy);
      if constexpr (RDN) mma_tok(u, aTS, fy);
      if constexpr (WRITE_O) mma_tok(base, aMP, fy);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const floatx4 x = pre[jt] - mgu[jt];
        floatx4 y, rv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float rr = clip < 0.f ? x[r] : fminf(fmaxf(x[r], -clip), clip);
          rv[r] = rr;
          y[r] = RDN ? ggm[r] * __builtin_fmaf(-egr[r], KR[jt][r], rr) : ggm[r] * rr;
        }
        store_acc_tile<TT>(YRt, jt * 16, 16 * ww, y);
        if constexpr (!RDN) store_acc_tile<TT>(DURt, jt * 16, 16 * ww, dlr * y);
        if constexpr (CKPT) {
          store_acc_tile<TT>(Rst, jt * 16, 16 * ww, rv);
          *reinterpret_cast<uint32_t*>(Mst + (jt * 16 + acc_col()) * L::kMstLd + 16 * ww + acc_row(0)) = mask_word(x, clip);
        }
      }
      if constexpr (RDN) {
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          store_acc_tile<TT>(DUt, jt * 16, 16 * ww, dls * u[jt]);
          if constexpr (CKPT) store_acc_tile<TT>(Ut, jt * 16, 16 * ww, u[jt]);
        }
      }
      if constexpr (WRITE_O) {
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
          for (int r = 0; r < 4; ++r) base[jt][r] = __builtin_fmaf(egs[r], QS[jt][r], base[jt][r]);
      }
      int fr0[IT * XS], fk0[IT * XS];
#pragma unroll
      for (int x = 0; x < IT * XS; ++x) {
        fr0[x] = ww * (DK / 4) + (x / XS) * 16;
        fk0[x] = (x % XS) * MX::kStep;
      }
      frags_tr_sync<TK, XT, IT * XS>(KT, fr0, fk0, kt);
    } else {
      if constexpr (CKPT) {
        if constexpr (RDN) {
          if (c > 0) {
            RLA_NOTE("store U^R");
            store_block(c - 1, 1, URt);
          }
        } else {
          store_ckpt(c, 0);
          store_ckpt(c, 1);
        }
      }
      // this chunk's T^R, MR (from phase 4); since then the S checkpoint or,
      // not saving, the previous chunk's o
      if constexpr (RDN) {
        wait_vmem_but<CKPT ? kCk + kBl : 1>();
        RLA_NOTE("await R matrices");
      }
      // the next gates: their copy, issued here a chunk ago, has landed (phase
      // 1 waited for what phase 3 issued after it; in chunk 0 for nothing)
      if (more && ww == 0) {
        if (c == 0) {
          RLA_NOTE("first chunk");
          wait_vmem();
        }
        write_gates(c + 1);
        if (c + 2 < nch) issue_gates(c + 2);
      }
    }
    barrier_lds();

    // ======== phase 3: U^R = T^R Y^R; o = base + diag(gamma) (e^h QR + MR T^R Y^R); S update ========
    if constexpr (CH) {
      typename MX::frag fy[JT][XS], fd[JT][XS];
      tok_frags(YRt, fy);
      if constexpr (RDN) aTR = packed_rows_frags(mat(kMatTR), ww, zero16);
      if constexpr (WRITE_O && RDN) aMR = packed_rows_frags(mat(kMatMR), ww, zero16);
      tok_frags(DUt, fd);
      sched_fence();
      floatx4 u[JT], mru[JT];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) u[jt] = mru[jt] = zero4();
      if constexpr (RDN) mma_tok(u, aTR, fy);
      if constexpr (WRITE_O) mma_tok(mru, aMR, fy);
      update_state(Sacc, eS, kt, fd);
      if constexpr (RDN) {
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          store_acc_tile<TT>(DURt, jt * 16, 16 * ww, dlr * u[jt]);
          if constexpr (CKPT) store_acc_tile<TT>(URt, jt * 16, 16 * ww, u[jt]);
        }
      }
      if constexpr (WRITE_O) {
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          floatx4 ov;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            ov[r] = __builtin_fmaf(ggm[r], __builtin_fmaf(egr[r], QR[jt][r], mru[jt][r]), base[jt][r]);
          // this lane's 4 tokens of its column, one store
          *reinterpret_cast<floatx4*>(ost + (jt * 16 + acc_col()) * L::kOstLd + 16 * ww + acc_row(0)) = ov;
        }
      }
      write_state_copies(Sacc, 0);
    } else {
      if (more) issue_s_mats(c + 1);   // in the chain's registers since phase 2
      if constexpr (CKPT) {
        RLA_NOTE("store R, U");
        if constexpr (RDN) store_ckpt(c, 1);   // chunk-start R (rewritten in phase 4)
        store_block(c, 0, Ut);
        if constexpr (!RDN) store_block(c, 1, URt);
      }
    }
    if constexpr (RDN) barrier_lds();

    // ======== phase 4: R update ========
    if constexpr (CH) {
      typename MX::frag fd[JT][XS];
      tok_frags(DURt, fd);
      if constexpr (RDN) stage_ckpt(Sacc, 0);   // the next chunk's (RLA: in its phase 1)
      update_state(Racc, eR, kt, fd);
      write_state_copies(Racc, 1);
    } else {
      if (more) {
        issue_r_mats(c + 1);   // in the chain's registers since phase 3
        // the next V (from phase 1); since then at least a checkpoint or two,
        // the matrices, U
        wait_vmem_but<RDN ? 2 * kCk + kBl + 5 : 2 * kCk + 2 * kBl + 3>();
        RLA_NOTE("await V");
      }
    }
    barrier_lds();
  }

  if constexpr (!CH) {
    if (nch > 0) {
      RLA_NOTE("end");
      if constexpr (WRITE_O) store_o(nch - 1);
      if constexpr (CKPT) {
        store_resid(nch - 1);
        if constexpr (RDN) store_block(nch - 1, 1, URt);
      }
    }
  }
  if constexpr (CH) {
    if (p.S_fin) save_state_f32<IT, JT>(Sacc, p.S_fin + state_off + j0, DV, ww * (DK / 4));
    if (p.R_fin) save_state_f32<IT, JT>(Racc, p.R_fin + state_off + j0, DV, ww * (DK / 4));
  }
  };
  if (chain) run(std::true_type{});
  else run(std::false_type{});
}

template <typename K>
hipError_t launch_fwd_kernel(K kern, const OpParams& p, int BV, int threads, int lds, hipStream_t stream) {
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (err != hipSuccess) return err;
  const int nvb = p.DV / BV;
  const int npairs = p.st.nseq * p.H;
  const int grid = ((npairs + 7) / 8) * 8 * nvb;
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, stream, p);
  return hipGetLastError();
}

// The operator's variants (log-cosh residual, ungated output, decayed
// residual) on the four-wave kernel; the boxed operator, with plain or
// normalised rows, on the wave-specialised one (packed prefill of 20011
// tokens from raw projections, H = 16, d = 128: 482 us with the four-wave
// kernel, 397 us here, 274 since in fewer phases).  fp32 inputs always take the
// four-wave kernel.
// Not saving, 16 columns per workgroup up to one workgroup per CU.  Both sides,
// 1024 tokens, 4 heads, time of 16 columns over time of 32 by the number of 16-column
// workgroups (plain and normalised rows alike):
//                    64 .. 256    320 .. 512   640, 768     1024
//   RDN, d_k = 128   0.79 - 0.88  1.23 - 1.33  1.08 - 1.12  1.26 - 1.31
//   RDN, d_k = 64    0.83 - 0.88  1.18 - 1.31  1.05 - 1.08  1.20 - 1.26
//   RLA, d_k = 128   0.82 - 0.90  1.32 - 1.46  1.15 - 1.20  1.36 - 1.44
//   RLA, d_k = 64    0.81 - 0.88  1.05 - 1.08  0.94 - 0.95  1.07 - 1.08
// Three of the instances take 129 to 166 registers, so past 256 their workgroups
// run in turns, one per CU; RLA at d_k = 64 (122) fits two per CU, which then share it
// at a little less than the speed of one 32-column workgroup.
constexpr int kCUs = 256;
template <typename IN, int DK, int BV, bool RDN, bool WRITE_O, bool CKPT>
hipError_t launch_fwd_t(const OpParams& p, hipStream_t s) {
  typedef FwdLayout<IN, DK, BV, RDN> L;
  if constexpr (sizeof(IN) == 2) {
    if (!(p.vflags & kVarOperator)) {
      if constexpr (!CKPT) {
        if (p.st.nseq * p.H * (p.DV / 16) <= kCUs) {
          auto kern = p.qk_f16 ? fwd_scan_ws_kernel<IN, DK, 16, RDN, WRITE_O, CKPT, true>
                               : fwd_scan_ws_kernel<IN, DK, 16, RDN, WRITE_O, CKPT, false>;
          return launch_fwd_kernel(kern, p, 16, 2 * kThreads, FwdWsLayout<IN, DK, 16, RDN, CKPT>::kBytes, s);
        }
      }
      auto kern = p.qk_f16 ? fwd_scan_ws_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, true>
                           : fwd_scan_ws_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, false>;
      return launch_fwd_kernel(kern, p, BV, 2 * kThreads, FwdWsLayout<IN, DK, BV, RDN, CKPT>::kBytes, s);
    }
    auto kern = p.out_bf16 ? fwd_scan_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, u16, true>
                           : fwd_scan_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, float, true>;
    return launch_fwd_kernel(kern, p, BV, kThreads, L::kBytes, s);
  } else {
    auto kern = (p.vflags & kVarOperator) ? fwd_scan_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, float, true>
                                          : fwd_scan_kernel<IN, DK, BV, RDN, WRITE_O, CKPT, float, false>;
    return launch_fwd_kernel(kern, p, BV, kThreads, L::kBytes, s);
  }
}

template <typename IN, int DK, int BV>
hipError_t launch_fwd_dk(const OpParams& p, bool write_o, bool ckpt, hipStream_t s) {
  if (p.rdn) {
    if (ckpt) return write_o ? launch_fwd_t<IN, DK, BV, true, true, true>(p, s) : launch_fwd_t<IN, DK, BV, true, false, true>(p, s);
    return launch_fwd_t<IN, DK, BV, true, true, false>(p, s);
  }
  if (ckpt) return write_o ? launch_fwd_t<IN, DK, BV, false, true, true>(p, s) : launch_fwd_t<IN, DK, BV, false, false, true>(p, s);
  return launch_fwd_t<IN, DK, BV, false, true, false>(p, s);
}

}  // namespace

hipError_t launch_fwd_scan(const OpParams& p, bool bf16, bool write_o, bool ckpt,
                           hipStream_t stream) {
  if (!bf16) return launch_fwd_dk<float, 64, 16>(p, write_o, ckpt, stream);
  if (p.DK == 128) return launch_fwd_dk<u16, 128, 32>(p, write_o, ckpt, stream);
  return launch_fwd_dk<u16, 64, 32>(p, write_o, ckpt, stream);
}

}  // namespace rla
