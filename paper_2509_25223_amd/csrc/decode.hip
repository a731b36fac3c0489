// Recurrent (decoding) step of RLA / RDN: the token recurrence of Sec. 3.4
// run directly, 256-thread workgroups over (sequence, head, value block),
// advancing S and R by T tokens (T is small in decoding; the chunked path
// serves long T).
//
// The states (d_k x d_v fp32, stored transposed like the ABI: element (i, j)
// is the paper's S[j][i]) are read once into registers, updated token by
// token and written once, so a step moves 2 x 2 x d_k x d_v x 4 bytes per
// (sequence, head) plus the token vectors: it is bound by HBM bandwidth.
//
// Value columns evolve independently (every column sum runs over the key
// index), so each (sequence, head) is split over DV / BV workgroups of BV
// columns.  The states are touched once per step, so they are loaded and
// stored non-temporally (measured 8% faster than cached accesses).
// Thread layout: thread (rg, cg) owns columns 4cg..4cg+3 of the block on rows
// i = ii * RG + rg (ii < RPT), as float4 registers, so the lanes of a wave
// load adjacent row segments (coalesced 16-byte accesses).
//
// Per token, with k = k_t, q = q_t and four column sums over the key index
//   Sk = S^T k, Sq = S^T q, Rk = R^T k, Rq = R^T q     (S, R: the old states)
//   x = v - Sk,  r = clip(x)                            (Sec. 3.1, 3.3)
//   RDN: a = v - aS Sk,  b = r - aR Rk                  RLA: a = v,  b = r
//   S <- aS S + beta k a^T,   R <- aR R + gamma k b^T
//   o = aS Sq + gamma (aR Rq + gamma (k.q) b)           (= aS S_{t-1} q + gamma R_t q)
// which is the boxed update S_t = aS S_{t-1}(I - beta k k^T) + beta v k^T
// (RDN) or aS S_{t-1} + beta v k^T (RLA), and likewise for R with (aR, gamma,
// r), written in the transposed storage.  Variants: x = v - aS Sk (decayed
// residual), r = c tanh(x / c) (log-cosh residual), o = Sq + R_t q (ungated).
// Pre-processing: q, k rows through SiLU and x / max(||x||, 1e-12); gates from
// pre-activations (aS, aR = exp(-a_h softplus(z + b_h)), beta, gamma = sigmoid).
#include "kernels.hpp"

namespace rla {

namespace {

// value columns per workgroup (32, 64 and 128 measured within 1% of each
// other at 256 sequences x 16 heads; 64 was the fastest)
constexpr int kDecodeBV = 64;

// Tokens staged at a time when a call has several.  All their vectors are
// loaded, normalised and their k . q formed at once, the waves sharing the
// rows, before and while the states arrive; a token is then two barriers.
// Loading token by token cost a round trip to memory and four barriers each
// (48 sequences of 5 raw tokens, 16 heads, 128 x 128: 55.5 -> 45.5 us).
constexpr int kDecodeGroup = 8;

// G: tokens staged at a time (1 for single-token calls)
template <typename IN, typename OT, int DK, int BV, bool RDN, int G>
__global__ __launch_bounds__(kThreads) void decode_kernel(OpParams p) {
  constexpr int CG = BV / 4;           // float4 column groups
  constexpr int RG = kThreads / CG;    // row groups
  constexpr int RPT = DK / RG;         // rows per thread
  constexpr int GPW = 64 / CG;         // row groups per wave
  static_assert(RPT * RG == DK && GPW * CG == 64, "decode thread layout");
  __shared__ float sq[G][DK], sk[G][DK], sv[G][BV], sg[G][4], skq[G];
  __shared__ float red[kWaves][4][BV];   // per-wave partial Sk, Sq, Rk, Rq
  __shared__ float coef[2][BV];          // a, b

  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int cg = tid % CG, rg = tid / CG;
  const int H = p.H, DV = p.DV, T = (int)p.st.dense_T;
  const int nvb = DV / BV;
  const int pair = blockIdx.x / nvb, j0 = (blockIdx.x % nvb) * BV;
  const int n = pair / H, h = pair % H;
  // a state's uniform base plus a 32-bit lane offset (scalar-base accesses)
  const int64_t sbase = (int64_t)pair * DK * DV;
  const uint32_t soff = (uint32_t)(rg * DV + j0 + 4 * cg);
  const float clip = p.clip;

  const IN* qg = reinterpret_cast<const IN*>(p.q);
  const IN* kg = reinterpret_cast<const IN*>(p.k);
  const IN* vg = reinterpret_cast<const IN*>(p.v);
  OT* og = reinterpret_cast<OT*>(p.o);

  // a group's vectors and gates (past its end: its last token)
  constexpr int kK = (G * DK + kThreads - 1) / kThreads, kV = (G * BV + kThreads - 1) / kThreads;
  IN qv[kK], kv[kK], vv[kV];
  float gv = 0.f;
  auto load_group = [&](int t0) {
    const int ng = G == 1 ? 1 : min(G, T - t0);
    const int64_t tok0 = (int64_t)n * T + t0;
#pragma unroll
    for (int u = 0; u < kK; ++u) {
      const int e = tid + u * kThreads, t = G == 1 ? 0 : min(e / DK, ng - 1);
      const int64_t o = ((tok0 + t) * H + h) * DK + e % DK;
      qv[u] = qg[o];
      kv[u] = kg[o];
    }
#pragma unroll
    for (int u = 0; u < kV; ++u) {
      const int e = tid + u * kThreads, t = G == 1 ? 0 : min(e / BV, ng - 1);
      vv[u] = vg[((tok0 + t) * H + h) * DV + j0 + e % BV];
    }
    const int k = tid & 3;
    const float* gp = k == 0 ? p.alpha_s : k == 1 ? p.beta : k == 2 ? p.alpha_r : p.gamma;
    gv = gp[(tok0 + min(tid >> 2, ng - 1)) * H + h];
  };
  if (T > 0) load_group(0);
  floatx4 S[RPT], R[RPT];
#pragma unroll
  for (int ii = 0; ii < RPT; ++ii) {
    const uint32_t o = soff + (uint32_t)(ii * RG * DV);
    S[ii] = p.S0 ? __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p.S0 + sbase + o)) : zero4();
    R[ii] = p.R0 ? __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p.R0 + sbase + o)) : zero4();
  }

  for (int t0 = 0; t0 < T; t0 += G) {
    const int ng = G == 1 ? 1 : min(G, T - t0);
    const int64_t tok0 = (int64_t)n * T + t0;
    if (t0 > 0) {
      load_group(t0);
      __syncthreads();   // the previous group's vectors are read
    }
#pragma unroll
    for (int u = 0; u < kK; ++u) {
      const int e = tid + u * kThreads;
      if (e < G * DK) {
        (&sq[0][0])[e] = to_f<IN>(qv[u]);
        (&sk[0][0])[e] = to_f<IN>(kv[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < kV; ++u) {
      const int e = tid + u * kThreads;
      if (e < G * BV) (&sv[0][0])[e] = to_f<IN>(vv[u]);
    }
    if (tid < 4 * G) {
      float x = gv;
      if (p.vflags & kVarGatePreact)
        x = (tid & 1) ? sigmoid_f(x) : __expf(-p.decay_param[h] * softplus_f(x + p.decay_param[H + h]));
      (&sg[0][0])[tid] = x;
    }
    __syncthreads();
    if (p.vflags & kVarQkNorm) {   // row r: q (even) or k (odd) of token r / 2
      for (int r = w; r < 2 * ng; r += kWaves) {
        float* x = (r & 1) ? sk[r >> 1] : sq[r >> 1];
        float y[DK / 64], ss = 0.f;
#pragma unroll
        for (int e = 0; e < DK / 64; ++e) {
          const float v = x[lane + 64 * e];
          y[e] = v / (1.f + __expf(-v));
          ss = __builtin_fmaf(y[e], y[e], ss);
        }
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) ss += __shfl_xor(ss, m);
        const float inv = 1.f / fmaxf(sqrtf(ss), 1e-12f);
#pragma unroll
        for (int e = 0; e < DK / 64; ++e) x[lane + 64 * e] = y[e] * inv;
      }
      __syncthreads();
    }
    for (int t = w; t < ng; t += kWaves) {   // k . q over the key index
      float kq = 0.f;
#pragma unroll
      for (int i = lane; i < DK; i += 64) kq = __builtin_fmaf(sk[t][i], sq[t][i], kq);
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) kq += __shfl_xor(kq, m);
      if (lane == 0) skq[t] = kq;
    }

    for (int b = 0; b < ng; ++b) {
      const int64_t tok = tok0 + b;
      // ---- column sums over this thread's rows, then over the wave's row groups ----
      floatx4 pSk = zero4(), pSq = zero4(), pRk = zero4(), pRq = zero4();
#pragma unroll
      for (int ii = 0; ii < RPT; ++ii) {
        const int i = ii * RG + rg;
        const float ki = sk[b][i], qi = sq[b][i];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          pSk[c] = __builtin_fmaf(ki, S[ii][c], pSk[c]);
          pSq[c] = __builtin_fmaf(qi, S[ii][c], pSq[c]);
          pRk[c] = __builtin_fmaf(ki, R[ii][c], pRk[c]);
          pRq[c] = __builtin_fmaf(qi, R[ii][c], pRq[c]);
        }
      }
#pragma unroll
      for (int m = CG; m < 64; m <<= 1)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          pSk[c] += __shfl_xor(pSk[c], m);
          pSq[c] += __shfl_xor(pSq[c], m);
          pRk[c] += __shfl_xor(pRk[c], m);
          pRq[c] += __shfl_xor(pRq[c], m);
        }
      if (lane < CG) {
        *reinterpret_cast<floatx4*>(&red[w][0][4 * cg]) = pSk;
        *reinterpret_cast<floatx4*>(&red[w][1][4 * cg]) = pSq;
        *reinterpret_cast<floatx4*>(&red[w][2][4 * cg]) = pRk;
        *reinterpret_cast<floatx4*>(&red[w][3][4 * cg]) = pRq;
      }
      __syncthreads();

      // ---- per value column: residual, clip, update coefficients, output ----
      if (tid < BV) {
        const int j = tid;
        float Sk = 0.f, Sq = 0.f, Rk = 0.f, Rq = 0.f;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
          Sk += red[ww][0][j];
          Sq += red[ww][1][j];
          Rk += red[ww][2][j];
          Rq += red[ww][3][j];
        }
        const float aS = sg[b][0], aR = sg[b][2], gm = sg[b][3];
        const float vj = sv[b][j];
        const float x = (p.vflags & kVarDecayed) ? __builtin_fmaf(-aS, Sk, vj) : vj - Sk;
        const float r = (p.vflags & kVarTanh) ? resid_tanh(x, clip)
                                              : (clip < 0.f ? x : fminf(fmaxf(x, -clip), clip));
        const float ca = RDN ? __builtin_fmaf(-aS, Sk, vj) : vj;
        const float cb = RDN ? __builtin_fmaf(-aR, Rk, r) : r;
        coef[0][j] = ca;
        coef[1][j] = cb;
        const float rq = __builtin_fmaf(gm * skq[b], cb, aR * Rq);   // R_t q
        const bool ung = (p.vflags & kVarUngated) != 0;
        const float oj = __builtin_fmaf(ung ? 1.f : gm, rq, ung ? Sq : aS * Sq);
        const int64_t oo = (tok * H + h) * DV + j0 + j;
        if constexpr (sizeof(OT) == 4) og[oo] = oj;
        else og[oo] = f2bf(oj);
      }
      __syncthreads();

      // ---- state updates ----
      {
        const float aS = sg[b][0], bt = sg[b][1], aR = sg[b][2], gm = sg[b][3];
        const floatx4 ca = *reinterpret_cast<const floatx4*>(&coef[0][4 * cg]);
        const floatx4 cb = *reinterpret_cast<const floatx4*>(&coef[1][4 * cg]);
#pragma unroll
        for (int ii = 0; ii < RPT; ++ii) {
          const float ki = sk[b][ii * RG + rg];
          const float bk = bt * ki, gk = gm * ki;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            S[ii][c] = __builtin_fmaf(bk, ca[c], aS * S[ii][c]);
            R[ii][c] = __builtin_fmaf(gk, cb[c], aR * R[ii][c]);
          }
        }
      }
    }
  }

#pragma unroll
  for (int ii = 0; ii < RPT; ++ii) {
    const uint32_t o = soff + (uint32_t)(ii * RG * DV);
    __builtin_nontemporal_store(S[ii], reinterpret_cast<floatx4*>(p.S_fin + sbase + o));
    __builtin_nontemporal_store(R[ii], reinterpret_cast<floatx4*>(p.R_fin + sbase + o));
  }
}

template <typename IN, typename OT, int DK>
hipError_t launch_decode_t(const OpParams& p, hipStream_t stream) {
  constexpr int BV = kDecodeBV, G = kDecodeGroup;   // d_v in {64, 128} is a multiple of BV
  const int64_t grid = (int64_t)p.st.nseq * p.H * (p.DV / BV);
  if (grid == 0) return hipSuccess;
  auto kern = p.st.dense_T == 1
                  ? (p.rdn ? decode_kernel<IN, OT, DK, BV, true, 1> : decode_kernel<IN, OT, DK, BV, false, 1>)
                  : (p.rdn ? decode_kernel<IN, OT, DK, BV, true, G> : decode_kernel<IN, OT, DK, BV, false, G>);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

template <typename IN, typename OT>
hipError_t launch_decode_in(const OpParams& p, hipStream_t stream) {
  if (p.DK == 128) return launch_decode_t<IN, OT, 128>(p, stream);
  return launch_decode_t<IN, OT, 64>(p, stream);
}

}  // namespace

hipError_t launch_decode(const OpParams& p, bool bf16, hipStream_t stream) {
  if (bf16) {
    if (p.out_bf16) return launch_decode_in<u16, u16>(p, stream);
    return launch_decode_in<u16, float>(p, stream);
  }
  return launch_decode_in<float, float>(p, stream);
}

}  // namespace rla
