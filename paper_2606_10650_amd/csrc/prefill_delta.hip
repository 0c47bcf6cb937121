// Prefill in the Gated DeltaNet form of the layer (Sec. 2.2, eq. delta_rule_rnn,
// with the decisions and merges of Sec. 3.1-3.2).
//
// With every state decayed by alpha_t = exp(g_t) first, a token that joins the
// newest state S takes the delta rule
//   S <- (I - beta_t k_t k_t^T) alpha_t S + beta_t k_t v_t^T
//      = alpha_t S + k_t u_t^T,   u_t = beta_t (v_t - (alpha_t S)^T k_t),
// and a token that opens a state starts it at beta_t k_t v_t^T, i.e. u_t =
// beta_t v_t.  So every state is the same decayed sum of rank-one terms k_s
// u_s^T over its tokens as the gated form with v_s replaced by u_s, and once the
// pseudo-values u_s are known the chunked update and readout stages apply
// unchanged.  The pseudo-values depend on the newest state before each token,
// which depends on every earlier decision, so a scan makes both: one 8-wave
// workgroup per head, sequential over chunks of 64 tokens, the newest state in
// registers (wave w: columns 16 w .. 16 w + 15, 16 x 16 MFMA tiles).
//
// Within a chunk y_t = (alpha S)^T k_t is linear in the values since the state
// began, with coefficients that do not depend on where it began:
//   y_t = A_t S_0^T k_t + sum_{r<t} W[t][r] beta_r (v_r - A_r S_0^T k_r),
//   W[t][r] = M[t][r] - sum_{r<s<t} M[t][s] beta_s W[s][r],
//   M[t][s] = exp(G_t - G_s) k_t . k_s,
// for the state S_0 before the chunk, and the same sum over r >= p with S_0 = 0
// for a state that begins at token p of the chunk.  So a chunk costs the Gram
// products, one triangular solve for W (16 x 16 diagonal blocks by
// substitution, the blocks below by MFMAs) and the products for y; the
// scores need y . v and |y|^2, explicit for S_0 and, once a boundary falls in
// the chunk, from tables over the starts p (suffix sums of W beta (.) V V^T and
// of its quadratic form).  The decisions are the gated scan's (scan_decide.h).
// Products that carry float32 values run as bfloat16 MFMAs over three-term
// splits (16-bit inputs) or as float32 MFMAs.
//
// The 64 x 64 part (Gram sums, decays, the solve, the sums over starts and the
// recurrence of |S|^2) is float64: the solve amplifies the rounding of M where
// keys repeat, and |S|^2 is a sum of terms of both signs.  In float32 the scores
// were off by up to 2e-6 where a float32 token by token scan is off by 5e-7
// (beta near 2: 4e-6, the states 3e-6), now by 4e-7 and the states by 2e-7
// (7e-7, 8e-7); a chunk of 48 heads of 128 x 128 takes 29 us, in float32 26.7.
//
// Bound: latency, as the gated scan: a chain of phases between barriers, 29 us a
// chunk at d = 128 with a state per 30 tokens (48 heads x 2048 tokens: 0.93 ms
// without the readout), 27 with one per 96 (8 x 16 heads x 4k tokens).  Taking the
// tokens one by one, as chunks with non-finite inputs, expanding steps or erased
// states still are, costs one barrier, a reduction and a score per token, 1.5 us
// (48 heads x 2048 tokens 3.12 ms; 3.77 with two full barriers and the norms of k
// and v formed per token).
//
// The call then runs the chunked update and readout stages of the gated form
// over (q, k, u, lambda), on the gated prefill's schedule: with the scan in
// segments on a second stream, overlapped with the update and readout of the
// segments already scanned, unless the caller asks for serial stages.  For
// 16-bit inputs the update takes u in float32 (it stages every value as three
// bfloat16 terms, so the states stay float32 exact) and the readout a bfloat16
// copy of u (for its in-chunk part, which rounds values to bfloat16 in the
// gated form too); float32 inputs run the float32 stages on u.
#include <type_traits>

#include "scan_decide.h"

namespace dla {

template <int DK, int DV, typename Tin>
struct DeltaP {
  static constexpr int E = (int)sizeof(Tin);
  static constexpr int EPP = 16 / E;                   // elements per 16 bytes
  static constexpr int K16 = SL * DK * E / 16 / STHR;  // 16-byte K pieces per thread
  static constexpr int V16 = SL * DV * E / 16 / STHR;
  static constexpr int NI = DK / 16;                   // 16-row tiles of the state per wave
  static constexpr int NW = DV / 16;                   // waves that hold state columns
  static_assert(NW <= SWAVE, "state columns");
  // LDS row strides (elements): padded by 16 bytes, so that lanes reading
  // consecutive rows hit distinct banks
  static constexpr int KRS = DK + EPP;  // sK [SL][KRS]
  static constexpr int VRS = DV + EPP;  // sV [SL][VRS]
  static constexpr int TRS = SL + EPP;  // sKt [DK][TRS], sVt [DV][TRS] (transposed, 16-bit inputs)
  static constexpr bool TRANS = E == 2;
  static constexpr int RRS = SL + 1;    // sR, sQ [SL][RRS]
  // sM, sVV, sW: float64, the 10 16 x 16 tiles on and below the diagonal
  static constexpr int MRS = 16 + 1;    // row stride of a tile
  static constexpr int MTS = 16 * MRS;  // tile
  static constexpr size_t MAT = 10 * (size_t)MTS * 8;
  static constexpr size_t cmax(size_t a, size_t b) { return a > b ? a : b; }
  static constexpr size_t K_BYTES = (size_t)SL * KRS * E;
  // sV, dead once the Gram products and the carry are formed; then sQ
  static constexpr size_t V_BYTES = cmax((size_t)SL * VRS * E, (size_t)SL * RRS * 4);
  static constexpr size_t T_BYTES = TRANS ? (size_t)(DK + DV) * TRS * E : 0;
  static_assert(MAT >= (size_t)SL * RRS * 4 + SWAVE * SL * 8 && MAT >= RowTables::BYTES, "aliases of sM and sVV");
  static_assert(K_BYTES % 16 == 0 && V_BYTES % 16 == 0 && T_BYTES % 16 == 0 && MAT % 16 == 0,
                "alignment");
  static size_t smem_bytes(int C) {
    size_t off = K_BYTES + V_BYTES + T_BYTES;
    off += 3 * MAT;                       // sM (then sR), sVV (then the row tables), sW
    off += 2 * (size_t)SWAVE * SL * 4;    // sPc, sPq
    off += (size_t)SL * 8 * 4;            // sG, sAl2, sKK, sV2
    off += (size_t)SL * 4 * 5;            // float rows, boundary overrides
    off += 64 + 128;                      // sRed, sMisc
    if (C > 64) off += (size_t)C * (8 + 4 + 4);
    return round_up(off, 16);
  }
};

// Whether a 16-byte piece of inputs holds an infinity or a NaN.
__device__ __forceinline__ bool piece_bad(const u32x4& v, bf16_t) {
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    bad |= (v[i] & 0x7F80u) == 0x7F80u || (v[i] & 0x7F800000u) == 0x7F800000u;
  return bad;
}
__device__ __forceinline__ bool piece_bad(const u32x4& v, float) {
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) bad |= (v[i] & 0x7F800000u) == 0x7F800000u;
  return bad;
}
__device__ __forceinline__ bool is_bad(float x) {
  return (__float_as_uint(x) & 0x7F800000u) == 0x7F800000u;
}

// exp(x) for a sum of gates x <= 0: n ln 2 taken off, a Taylor polynomial of
// degree 9 on |r| <= ln 2 / 2 (remainder r^10 / 10! < 1e-11), scaled by 2^n.
__device__ __forceinline__ double exp_gate(double x) {
  x = x > -800.0 ? x : -800.0;  // (0 in float64)
  const double n = __builtin_rint(x * 1.4426950408889634);
  const double r = __builtin_fma(n, -0.6931471805599453, x);
  double p = 1.0 / 362880.0;
  p = __builtin_fma(p, r, 1.0 / 40320.0);
  p = __builtin_fma(p, r, 1.0 / 5040.0);
  p = __builtin_fma(p, r, 1.0 / 720.0);
  p = __builtin_fma(p, r, 1.0 / 120.0);
  p = __builtin_fma(p, r, 1.0 / 24.0);
  p = __builtin_fma(p, r, 1.0 / 6.0);
  p = __builtin_fma(p, r, 0.5);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  return __builtin_ldexp(p, (int)n);
}

// A workgroup barrier that orders LDS accesses only: stores to global memory stay
// in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// NR: see the gated scan.
template <int DK, int DV, typename Tin, int NR>
__global__ __launch_bounds__(STHR) void prefill_delta_scan_kernel(PrefillArgs a, PrefillWS w,
                                                                  int tb, int te,
                                                                  const float* __restrict__ beta,
                                                                  float* __restrict__ U,
                                                                  bf16_t* __restrict__ U16) {
  if (!cache_matches(a.cache, a.desc)) return;  // refused call (see the prep kernel)
  using P = DeltaP<DK, DV, Tin>;
  using FT = typename Frag<Tin>::T;
  // float32 operands next to the inputs' type: three bfloat16 terms, or float32
  using XT = typename std::conditional<P::E == 2, Split3, f32x8>::type;
  constexpr int D = DK * DV;
  constexpr int NI = P::NI, NW = P::NW;
  constexpr int KRS = P::KRS, VRS = P::VRS, TRS = P::TRS, RRS = P::RRS;
  constexpr int MRS = P::MRS, MTS = P::MTS;
  constexpr int K16 = P::K16, V16 = P::V16;
  const int h = blockIdx.x;
  int tid = threadIdx.x;
  int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int c16 = lane & 15;
  int q4 = lane >> 4;
  // The addresses of a phase derive from lane, c16 and q4.  Made opaque before
  // each phase, they are formed there: hoisted out of the chunk loop, as the
  // compiler otherwise does, they take some 270 registers more than there are.
  auto fresh_lane = [&]() __attribute__((always_inline)) {
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    c16 = lane & 15;
    q4 = lane >> 4;
  };
  const int C = a.desc.C;
  const int T = a.T;
  const size_t tok0 = (size_t)h * T;
  const bool own = wv < NW;       // the wave holds state columns 16 wv .. 16 wv + 15
  const int col = 16 * wv + (tid & 15);  // the lane's state column

  extern __shared__ __align__(16) char smem[];
  Tin* sK = reinterpret_cast<Tin*>(smem);
  Tin* sV = reinterpret_cast<Tin*>(smem + P::K_BYTES);
  float* sQ = reinterpret_cast<float*>(smem + P::K_BYTES);                // (alias of sV)
  Tin* sKt = reinterpret_cast<Tin*>(smem + P::K_BYTES + P::V_BYTES);
  Tin* sVt = sKt + DK * TRS;
  double* sM = reinterpret_cast<double*>(smem + P::K_BYTES + P::V_BYTES + P::T_BYTES);
  float* sR = reinterpret_cast<float*>(sM);  // R[p][t] at [t RRS + p] (once M is no longer read)
  double* sVV = sM + 10 * MTS;
  const RowTables rows(reinterpret_cast<char*>(sVV));  // (once the tables for R and Q are built)
  double* sW = sVV + 10 * MTS;
  double* sG = sW + 10 * MTS;     // G_t - G(chunk start)
  double* sAl2 = sG + SL;         // alpha_t^2
  double* sKK = sAl2 + SL;        // |k_t|^2
  double* sV2 = sKK + SL;         // |v_t|^2
  double* sRed = sV2 + SL;        // [8] the waves' shares of |S|^2
  float* sPc = reinterpret_cast<float*>(sRed + 8);  // [SWAVE][SL] the waves' shares of y . v
  float* sPq = sPc + SWAVE * SL;  //                              |y|^2
  float* sA = sPq + SWAVE * SL;   // exp(sG[t])
  float* sAl = sA + SL;           // alpha_t
  float* sDe = sAl + SL;          // exp(G_end - G_t)
  float* sBeta = sDe + SL;        // beta_t (0 past the chunk's end)
  int32_t* sBo = reinterpret_cast<int32_t*>(sBeta + SL);  // boundary overrides
  int32_t* sMisc = sBo + SL;
  // sMisc: 0, 1 boundary mask; 2 start of the rows left (-1: none); 3 go on with
  // the row tables; 4, 5 non-finite inputs of an even, an odd chunk; 6 tokens that
  // the rows decided
  __shared__ double sGlast[1];

  Meta M = meta_at(a.cache + a.meta_offset + (size_t)h * a.meta_stride, C);
  InitView iv = init_at(w, h, C);
  ScarryView sv = scarry_at(w, h, C);
  const int m0 = min(max(*iv.m0, 0), C);
  using States = typename std::conditional<NR == 0, StatesInLds, StatesInRegs<NR>>::type;
  ChunkDecider<States> dec;
  dec.st.C = C;
  if constexpr (NR == 0) {
    dec.st.I = reinterpret_cast<double*>(sMisc + 32);  // [C]
    dec.st.n = reinterpret_cast<int32_t*>(dec.st.I + C);
    dec.st.ld = dec.st.n + C;
  }
  dec.m = 0;
  dec.B = 0;
  if (wv == 0) {
    if (tb == 0)
      dec.st.load(M.ibar, M.n, nullptr, m0);
    else
      dec.st.load(sv.ibar, sv.n, sv.lead, m0);
    dec.m = __builtin_amdgcn_readfirstlane(tb == 0 ? m0 : min(max(*sv.m, 0), C));
  }

  // newest state at the start of the call, true (decayed) values: S[i][r] is row
  // 16 i + 4 q4 + r of column col
  f32x4 S[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) S[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const double G0 = *M.G;
  if (own) {
    if (tb > 0) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) S[i][r] = sv.S[(((size_t)wv * NI + i) * 4 + r) * 64 + lane];
    } else if (m0 > 0) {
      const float* src =
          a.desc.state_dtype == DLA_BF16
              ? reinterpret_cast<const float*>(a.cache + a.open_offset) + (size_t)h * D
              : reinterpret_cast<const float*>(a.cache + a.states_offset) +
                    ((size_t)h * C + min(max(M.perm[m0 - 1], 0), C - 1)) * D;
      const float f = (float)exp(G0 - M.F[m0 - 1]);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) S[i][r] = f * src[(size_t)(16 * i + 4 * q4 + r) * DV + col];
    }
  }
  // |S|^2: the waves' shares in sRed, added where they are read (a chunk's
  // barriers lie between)
  auto norm_share = [&]() __attribute__((always_inline)) {
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) x += S[i][r] * S[i][r];
    x = wave_total_dpp(x);
    if (lane == 0) sRed[wv] = (double)x;
  };
  auto norm2 = [&]() __attribute__((always_inline)) -> double {
    double b = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) b += sRed[i];
    return b;
  };
  norm_share();
  // the first row of W's diagonal blocks stays zero
  for (int i = tid; i < 10 * MTS; i += STHR) sW[i] = 0.0;
  if (tid < 2) sMisc[4 + tid] = 0;

  const Tin* Kin = static_cast<const Tin*>(a.k) + tok0 * DK;
  const Tin* Vin = static_cast<const Tin*>(a.v) + tok0 * DV;
  const double* Gtok = w.Gtok + tok0;
  const float* gate = a.g + tok0;
  const float* bt = beta + tok0;
  int32_t* death = w.death + tok0;
  float* Uh = U + tok0 * DV;
  bf16_t* U16h = U16 ? U16 + tok0 * DV : nullptr;  // bfloat16 copy (16-bit inputs)
  // next chunk's tokens in registers (see the gated scan)
  u32x4 pk[K16], pv[V16];
  double gpre = 0.0;
  float fpre = 0.f, bepre = 0.f;
  int bpre = -1, mpre = -1;
  auto prefetch = [&](int c0n) __attribute__((always_inline)) {
    const int nr = min(SL, T - c0n);
#pragma unroll
    for (int u = 0; u < K16; ++u) {
      const int pi = tid + STHR * u;
      pk[u] = reinterpret_cast<const u32x4*>(Kin + (size_t)(c0n + min(pi % SL, nr - 1)) * DK)[pi / SL];
    }
#pragma unroll
    for (int u = 0; u < V16; ++u) {
      const int pi = tid + STHR * u;
      pv[u] = reinterpret_cast<const u32x4*>(Vin + (size_t)(c0n + min(pi % SL, nr - 1)) * DV)[pi / SL];
    }
    if (tid < SL) {
      const int t = min(tid, nr - 1);
      gpre = Gtok[c0n + t];
      fpre = gate[c0n + t];
      bepre = bt[c0n + t];
      bpre = (a.b_ovr && tid < nr) ? a.b_ovr[tok0 + c0n + tid] : (int8_t)-1;
      mpre = (a.m_ovr && tid < nr) ? a.m_ovr[tok0 + c0n + tid] : -1;
    }
  };
  prefetch(tb);
  int hold = 0, wait = 0;  // chunks to go token by token
  double Gprev = tb > 0 ? Gtok[tb - 1] : G0;

  for (int c0 = tb; c0 < te; c0 += SL) {
    const int nrow = min(SL, T - c0);
    int32_t* sBad = sMisc + 4 + ((c0 / SL) & 1);
    // ------------------------------------------------ stage the chunk
    fresh_lane();
    __syncthreads();  // the chunk before is done with the tables
    bool bad = false;
    float kpart = 0.f;  // the wave's share of |k|^2 of token lane
#pragma unroll
    for (int u = 0; u < K16; ++u) {
      const int pi = tid + STHR * u;
      const int r = pi % SL, pc = pi / SL;
      const u32x4 z = {0u, 0u, 0u, 0u};
      const u32x4 val = (r < nrow) ? pk[u] : z;
      bad |= piece_bad(val, Tin{});
#pragma unroll
      for (int e = 0; e < P::EPP; ++e) {
        const float x = to_f32(piece_elem<Tin>(val, e));
        kpart += x * x;
      }
      *reinterpret_cast<u32x4*>(sK + r * KRS + pc * P::EPP) = val;
      if constexpr (P::TRANS) put_transposed<TRS>(sKt, pc, r, val);
    }
#pragma unroll
    for (int u = 0; u < V16; ++u) {
      const int pi = tid + STHR * u;
      const int r = pi % SL, pc = pi / SL;
      const u32x4 z = {0u, 0u, 0u, 0u};
      const u32x4 val = (r < nrow) ? pv[u] : z;
      bad |= piece_bad(val, Tin{});
      *reinterpret_cast<u32x4*>(sV + r * VRS + pc * P::EPP) = val;
      if constexpr (P::TRANS) put_transposed<TRS>(sVt, pc, r, val);
    }
    if (tid < SL) {
      const int t = tid;
      const double Glast = __shfl(gpre, nrow - 1, 64);
      // Decays across tokens come from float64 differences of G, a token's own
      // from its gate: after a steep gate (a reset), float32 offsets from the
      // chunk start would round the later tokens' decays to that gate's ulp.
      const double gd = gpre - Gprev;
      const float be = t < nrow ? bepre : 0.f;
      sG[t] = gd;
      sA[t] = (float)exp_gate(gd);
      sAl[t] = (t < nrow) ? __expf(fpre) : 0.f;
      sBeta[t] = be;
      sBo[t] = bpre;
      // (a positive gate expands the state: token by token too)
      bad |= !(fpre <= 0.f) || is_bad((float)gd) || is_bad(be);
      if (t == 0) sGlast[0] = Glast;
    }
    sPq[wv * SL + lane] = kpart;
    if (__ballot(bad) && lane == 0) *sBad = 1;
    __syncthreads();
    const double Gnext = sGlast[0];  // G after the chunk's last token
    const double b0 = norm2();       // |S|^2
    // Token by token when an input of the chunk or the state is not finite, or
    // when a token's step is not a contraction (beta |k|^2 outside [0, 2]): the
    // tables range over starts that the boundaries may exclude, and only
    // contractions bound them.  And from a token whose step erases the state, so
    // that |S|^2 is lost in the rounding of its terms (score_row).
    float kk = 0.f;
#pragma unroll
    for (int i = 0; i < SWAVE; ++i) kk += sPq[i * SL + lane];
    const float bk = sBeta[lane] * kk;
    const bool outside =  // (workgroup-uniform)
        *sBad != 0 || is_bad((float)b0) || __ballot(!(bk >= 0.f && bk <= 2.f)) != 0;
    if (tid == 0) sMisc[4 + (((c0 / SL) & 1) ^ 1)] = 0;
    const int mforce = mpre;  // merge override of the lane's token (wave 0)
    fresh_lane();
    if (c0 + SL < te) prefetch(c0 + SL);

    auto open_at = [&](int ts, float Is) __attribute__((always_inline)) {
      dec.open(ts, Is, mforce, c0, C, T, &reinterpret_cast<CacheHeader*>(a.cache)->flags,
               [&](int ld, int tk) { (ld >= 0 ? death[ld] : iv.death0[ld + m0]) = tk; });
    };
    bool dense = false;
    if (wv == 0) {
      dense = dec.dense();
      dec.p = -1;
      dec.tn = nrow;
      dec.B = 0;
      dec.mo = -1;
      dec.dc = -1;
      dec.io = 0.f;
    }

    // After a chunk that lost a token the next ones go token by token from their
    // start, without the tables: 1, then 3 chunks, then 7.  (Counted anew at every
    // readout chunk, so that results do not depend on the call's segments.)
    if (c0 % chunk_len(P::E) == 0) hold = wait = 0;
    const bool waits = wait > 0;
    if (waits) --wait;
    int tn = 0;  // tokens taken together; the others follow one by one
    const bool serial = outside || waits;  // (workgroup-uniform)
    bool together = !serial;
    f32x4 X[4];   // X[i][r]: token 16 i + 4 q4 + r, column col
    f32x4 Vr[4];  // the values in the same layout
    if (together) {
      fresh_lane();
      // ------------------------------------ Gram products, and the carry S^T k
#pragma unroll
      for (int i = 0; i < 4; ++i) X[i] = Vr[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      // the 10 + 10 lower 16 x 16 tiles of K K^T and V V^T, dealt to the waves
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int ti = wv + SWAVE * u;
        if (ti >= 20) break;
        const bool isv = ti >= 10;
        const int x = isv ? ti - 10 : ti;
        const int tr = x < 1 ? 0 : (x < 3 ? 1 : (x < 6 ? 2 : 3));
        const int tc = x - tr * (tr + 1) / 2;
        f64x4 g = {0.0, 0.0, 0.0, 0.0};
        if (!isv) {
          const Tin* pa = sK + (16 * tr + c16) * KRS + 8 * q4;
          const Tin* pb = sK + (16 * tc + c16) * KRS + 8 * q4;
#pragma unroll
          for (int ks = 0; ks < DK / 32; ++ks)
            gram16(g, Frag<Tin>::load(pa + 32 * ks), Frag<Tin>::load(pb + 32 * ks));
        } else {
          const Tin* pa = sV + (16 * tr + c16) * VRS + 8 * q4;
          const Tin* pb = sV + (16 * tc + c16) * VRS + 8 * q4;
#pragma unroll
          for (int ks = 0; ks < DV / 32; ++ks)
            gram16(g, Frag<Tin>::load(pa + 32 * ks), Frag<Tin>::load(pb + 32 * ks));
        }
        const int s = 16 * tc + c16;
        const double gs = sG[s];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = gram_row<Tin>(r, q4), t = 16 * tr + row;
          const int at = x * MTS + row * MRS + c16;
          if (isv)
            sVV[at] = g[r];
          else
            sM[at] = s < t ? exp_gate(sG[t] - gs) * g[r] : 0.0;
          if (s == t) (isv ? sV2 : sKK)[t] = g[r];
        }
      }
      fresh_lane();
      if (own) {
#pragma unroll
        for (int kk = 0; kk < DK / 32; ++kk) {
          f32x8 sx;
#pragma unroll
          for (int e = 0; e < 8; ++e) sx[e] = S[2 * kk + (e >> 2)][e & 3];
          const XT sb(sx);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const Tin* kr = sK + (16 * i + c16) * KRS + 32 * kk + 4 * q4;
            const FT ka = load_4x2<Tin>(kr, kr + 16);
            f32x4 z = {0.f, 0.f, 0.f, 0.f};  // (short sums, added at the end)
            if constexpr (P::E == 2)
              mma16_split(z, ka, sb);
            else
              mma16(z, ka, sb);
            X[i] += z;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 at = *reinterpret_cast<const float4*>(sA + 16 * i + 4 * q4);
          X[i] *= f32x4{at.x, at.y, at.z, at.w};
          if constexpr (P::TRANS) {
            float x[4];
            load4f(sVt + col * TRS + 16 * i + 4 * q4, x);
            Vr[i] = f32x4{x[0], x[1], x[2], x[3]};
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) Vr[i][r] = sV[(16 * i + 4 * q4 + r) * VRS + col];
          }
        }
      }
      __syncthreads();
      // (a value whose square overflows float32 would spoil the sums of others)
      together = __ballot(is_bad((float)sV2[lane])) == 0;  // (workgroup-uniform)
    }
    if (together) {
      fresh_lane();
      // ---------------------------------- W: y_t = sum_{r<t} W[t][r] beta_r v_r
      // W[t][r] = M[t][r] - sum_{r<s<t} M[t][s] beta_s W[s][r]: within the 16 x 16
      // diagonal blocks by substitution (wave 0, lane = block and column r) ...
      if (wv == 0) {
        const double* Mb = sM + q4 * (q4 + 3) / 2 * MTS;
        double* Wb = sW + q4 * (q4 + 3) / 2 * MTS;
        double bw[16];  // beta_s W[s][r]
        float be[16];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const float4 b = *reinterpret_cast<const float4*>(sBeta + 16 * q4 + 4 * s4);
          be[4 * s4] = b.x; be[4 * s4 + 1] = b.y; be[4 * s4 + 2] = b.z; be[4 * s4 + 3] = b.w;
        }
        bw[0] = 0.0;
#pragma unroll
        for (int t = 1; t < 16; ++t) {
          double x0 = Mb[t * MRS + c16], x1 = 0.0;
#pragma unroll
          for (int s = 1; s < t; ++s) (s & 1 ? x0 : x1) -= Mb[t * MRS + s] * bw[s];
          const double wt = c16 < t ? x0 + x1 : 0.0;
          Wb[t * MRS + c16] = wt;
          bw[t] = (double)be[t] * wt;
        }
      } else if (wv == 1) {  // (beside it)
        sAl2[lane] = lane < nrow ? exp_gate(2.0 * (sG[lane] - (lane ? sG[lane - 1] : 0.0))) : 0.0;
      } else if (wv == 2) {
        sDe[lane] = lane < nrow ? (float)exp_gate(sG[nrow - 1] - sG[lane]) : 0.f;
      }
      __syncthreads();
      fresh_lane();
      // ... then the blocks below the diagonal, I rows and J columns of a pair of
      // neighbouring blocks: P = M_IJ (1 - beta W)_JJ, W_IJ = (1 - W_II beta) P
      auto tile = [&](int bi, int bj) __attribute__((always_inline)) -> int {
        return (bi * (bi + 1) / 2 + bj) * MTS;
      };
      auto row4 = [&](const double* m, int bi, int bj) __attribute__((always_inline)) -> f64x4 {
        const double* x = m + tile(bi, bj) + c16 * MRS + q4;
        return f64x4{x[0], x[4], x[8], x[12]};
      };
      auto tile4 = [&](const double* m, int bi, int bj) __attribute__((always_inline)) -> f64x4 {
        const double* x = m + tile(bi, bj) + q4 * MRS + c16;
        return f64x4{x[0], x[4 * MRS], x[8 * MRS], x[12 * MRS]};
      };
      auto beta4 = [&](int b) __attribute__((always_inline)) -> f64x4 {
        const float* x = sBeta + 16 * b + q4;
        return f64x4{(double)x[0], (double)x[4], (double)x[8], (double)x[12]};
      };
      auto put4 = [&](int bi, int bj, const f64x4& x) __attribute__((always_inline)) {
        double* y = sW + tile(bi, bj) + q4 * MRS + c16;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[4 * r * MRS] = x[r];
      };
      constexpr f64x4 zero4 = {0.0, 0.0, 0.0, 0.0};
      if (wv < 2) {
        const int J = 2 * wv, I = J + 1;
        f64x4 pq = zero4, wq = zero4;
        mma16(pq, row4(sM, I, J), beta4(J) * tile4(sW, J, J));
        pq = tile4(sM, I, J) - pq;
        mma16(wq, row4(sW, I, I), beta4(I) * pq);
        put4(I, J, pq - wq);
      }
      __syncthreads();
      // the 32 x 32 blocks: wave 2 ti + tj takes rows 16 (2 + ti) .. and columns 16
      // tj .., the halves' P through the bytes of sPc and sPq
      double* sP0 = reinterpret_cast<double*>(sPc);
      f64x4 pw = zero4;
      if (wv < 4) {
        const int tj = wv & 1, ti = 2 + (wv >> 1);
        for (int kb = tj; kb < 2; ++kb) mma16(pw, row4(sM, ti, kb), beta4(kb) * tile4(sW, kb, tj));
        pw = tile4(sM, ti, tj) - pw;
        if (ti == 2) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sP0[tj * 256 + (4 * r + q4) * 16 + c16] = pw[r];
        }
      }
      __syncthreads();
      if (wv < 4) {
        const int tj = wv & 1, ti = 2 + (wv >> 1);
        f64x4 w0 = zero4;
        if (ti == 3) {
          f64x4 p0;
#pragma unroll
          for (int r = 0; r < 4; ++r) p0[r] = sP0[tj * 256 + (4 * r + q4) * 16 + c16];
          mma16(w0, row4(sW, 3, 2), beta4(2) * p0);
        }
        mma16(w0, row4(sW, ti, ti), beta4(ti) * pw);
        put4(ti, tj, pw - w0);
      }
      __syncthreads();

      fresh_lane();
      // -------- y, for the state before the chunk: Y = X + (W beta) (V - X)
      f32x4 Y[4];
      // 8 consecutive-pair elements of W beta's row t = 16 i + c16 for K step kk
      // (tokens 32 kk + 4 q4 + e and 16 further), zero for tokens before lo
      auto wrow = [&](int i, int kk, int lo) __attribute__((always_inline)) -> f32x8 {
        f32x8 x;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bool in = 2 * kk + j <= i;  // (else above the diagonal)
          const double* wp = sW + (in ? tile(i, 2 * kk + j) : 0) + c16 * MRS + 4 * q4;
          const float4 b = *reinterpret_cast<const float4*>(sBeta + 32 * kk + 16 * j + 4 * q4);
          x[4 * j] = in ? (float)wp[0] * b.x : 0.f;
          x[4 * j + 1] = in ? (float)wp[1] * b.y : 0.f;
          x[4 * j + 2] = in ? (float)wp[2] * b.z : 0.f;
          x[4 * j + 3] = in ? (float)wp[3] * b.w : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (32 * kk + 16 * (e >> 2) + 4 * q4 + (e & 3) < lo) x[e] = 0.f;
        return x;
      };
      if (own) {
#pragma unroll
        for (int i = 0; i < 4; ++i) Y[i] = X[i];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          f32x8 z;
#pragma unroll
          for (int e = 0; e < 8; ++e) z[e] = Vr[2 * kk + (e >> 2)][e & 3] - X[2 * kk + (e >> 2)][e & 3];
          const XT zb(z);
#pragma unroll
          for (int i = 2 * kk; i < 4; ++i) {
            const XT wa(wrow(i, kk, 0));
            f32x4 y = {0.f, 0.f, 0.f, 0.f};
            if constexpr (P::E == 2)
              mma16_split(y, wa, zb);
            else
              mma16(y, wa, zb);
            Y[i] += y;
          }
        }
        // the wave's shares of y . v and |y|^2, summed over its 16 columns
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float cy = Y[i][r] * Vr[i][r], qy = Y[i][r] * Y[i][r];
            cy += dpp_f<0x111, 0xF>(0.f, cy);
            qy += dpp_f<0x111, 0xF>(0.f, qy);
            cy += dpp_f<0x112, 0xF>(0.f, cy);
            qy += dpp_f<0x112, 0xF>(0.f, qy);
            cy += dpp_f<0x114, 0xF>(0.f, cy);
            qy += dpp_f<0x114, 0xF>(0.f, qy);
            cy += dpp_f<0x118, 0xF>(0.f, cy);
            qy += dpp_f<0x118, 0xF>(0.f, qy);
            if (c16 == 15) {
              sPc[wv * SL + 16 * i + 4 * q4 + r] = cy;
              sPq[wv * SL + 16 * i + 4 * q4 + r] = qy;
            }
          }
      }
      __syncthreads();

      fresh_lane();
      // ------------------------------------------------------- decisions
      RowIn<double> rin;
      rin.nrow = nrow;
      rin.C = C;
      rin.tau = a.tau;
      rin.eps = a.eps;
      const double kk2 = sKK[lane], vv2 = sV2[lane], bet = (double)sBeta[lane];
      rin.sc = ScoreIn<double>::of((double)a.eps_rms, (double)D, kk2 * vv2);
      rin.al2n = (lane + 1 < SL) ? sAl2[lane + 1] : 0.0;
      rin.bo = sBo[lane];
      // growth of |S|^2 with a token of y . v = c and |y|^2 = q: S + k u^T, u =
      // beta (v - y)
      auto grow = [&](double c, double q) __attribute__((always_inline)) -> double {
        const double u2 = vv2 - 2.0 * c + q;
        return 2.0 * bet * (c - q) + kk2 * bet * bet * (u2 < 0.0 ? 0.0 : u2);
      };
      auto row = [&](int p, double& ct, double& inc) __attribute__((always_inline)) {
        ct = (lane > p) ? (double)sR[lane * RRS + p] : 0.0;
        inc = grow(ct, (lane > p) ? (double)sQ[lane * RRS + p] : 0.0);
      };
      if (wv == 0) {
        if (dec.m == 0) {
          // the first token of an empty cache opens a state with score 0
          dec.st.push(0, 0.0, c0);
          dec.m = 1;
          dec.p = 0;
          dec.B = 1;
          if (lane == 0) dec.dc = T;
        }
        const bool more = dec.first_rows(
            rin, 1,
            [&](int p, double& ct, double& inc, double& binit) __attribute__((always_inline)) {
              // (an empty cache's first token starts from S = 0)
              double c = 0.0, q = 0.0;
#pragma unroll
              for (int i = 0; i < NW; ++i) {
                c += (double)sPc[i * SL + lane];
                q += (double)sPq[i * SL + lane];
              }
              ct = c;
              inc = grow(c, q);
              binit = sAl2[0] * b0;
            },
            open_at);
        if (lane == 0) {
          sMisc[0] = (int)(uint32_t)dec.B;
          sMisc[1] = (int)(uint32_t)(dec.B >> 32);
          sMisc[2] = more ? dec.p : -1;
          sMisc[6] = dec.tn;
        }
      }
      __syncthreads();
      if (sMisc[2] >= 0) {  // (workgroup-uniform) a state began in the chunk
        fresh_lane();
        // Tables for every start p in the chunk: y . v = sum_{r=p}^{t-1} (W
        // beta)[t][r] (v_r . v_t), and |y|^2 = sum_{r>=p} x_r (2 sum_{r'>r} x_r'
        // (v_r . v_r') + x_r |v_r|^2) with x_r = (W beta)[t][r].
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int x = wv + SWAVE * u;
          if (x >= 10) break;
          const int tr = x < 1 ? 0 : (x < 3 ? 1 : (x < 6 ? 2 : 3));
          const int tc = x - tr * (tr + 1) / 2;
          f64x4 z = zero4;
          for (int kb = tc; kb <= tr; ++kb) {
            f64x4 b = tile4(sVV, kb, tc);  // rows r' of block kb, column r
            if (kb == tc) {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (4 * r + q4 <= c16) b[r] = 0.0;
            }
            mma16(z, row4(sW, tr, kb) * beta4(kb), b);
          }
          const double br = (double)sBeta[16 * tc + c16], vr2 = sV2[16 * tc + c16];
          const f64x4 wt = tile4(sW, tr, tc);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double xr = wt[r] * br;
            sQ[(16 * tr + 4 * r + q4) * RRS + 16 * tc + c16] = (float)(xr * (2.0 * z[r] + vr2 * xr));
          }
        }
        __syncthreads();
        {
          // suffix sums over s: lane t, wave w terms 8 w .. 8 w + 7, then the
          // totals of the waves behind (in the bytes of sPc and past sR)
          double* sTx = reinterpret_cast<double*>(sPc);
          double* sTy = sM + SL * RRS / 2;
          const int t = lane;
          double x[8], y[8], ax = 0.0, ay = 0.0;
#pragma unroll
          for (int j = 7; j >= 0; --j) {
            const int s = 8 * wv + j;
            const int at = tile(t >> 4, min(s >> 4, t >> 4)) + (t & 15) * MRS + (s & 15);
            if (s < t) {
              ax += sW[at] * (double)sBeta[s] * sVV[at];
              ay += (double)sQ[t * RRS + s];
            }
            x[j] = ax;
            y[j] = ay;
          }
          sTx[wv * SL + t] = ax;
          sTy[wv * SL + t] = ay;
          __syncthreads();
          ax = ay = 0.0;
          for (int w2 = wv + 1; w2 < SWAVE; ++w2) {
            ax += sTx[w2 * SL + t];
            ay += sTy[w2 * SL + t];
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            sR[t * RRS + 8 * wv + j] = (float)(x[j] + ax);
            sQ[t * RRS + 8 * wv + j] = (float)(y[j] + ay);
          }
        }
        __syncthreads();
        if (wv == 0) {
          bool more = true;
          if (!dense)
            more = dec.first_rows(
                rin, NSEQ - 1,
                [&](int p, double& ct, double& inc, double& binit) __attribute__((always_inline)) {
                  row(p, ct, inc);
                  binit = 0.0;
                },
                open_at);
          if (lane == 0) sMisc[3] = more ? dec.p : -1;
        }
        __syncthreads();
        const int prow = sMisc[3];
        if (prow >= 0) {  // (workgroup-uniform)
          fill_rows(rin, prow, rows, row);
          __syncthreads();
          if (wv == 0) dec.finish_rows(rin, rows, open_at);
        }
        if (wv == 0 && lane == 0) {
          sMisc[0] = (int)(uint32_t)dec.B;
          sMisc[1] = (int)(uint32_t)(dec.B >> 32);
          sMisc[6] = dec.tn;
        }
        __syncthreads();
      }

      fresh_lane();
      // -------------------------------- pseudo-values, and the state's advance
      const uint64_t B = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(sMisc[0]) |
                         ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(sMisc[1]) << 32);
      auto start_of = [&](int t) __attribute__((always_inline)) -> int {  // of token t's state
        const uint64_t x = B & (~0ull >> (63 - t));
        return x ? 63 - __clzll((long long)x) : -1;
      };
      const int plast = start_of(SL - 1);
      tn = __builtin_amdgcn_readfirstlane(sMisc[6]);
      hold = tn < nrow ? 2 * hold + 1 : 0;
      wait = hold;
      if (tn > 0 && tn < nrow) {  // (workgroup-uniform) decays to the last of the tokens taken
        if (tid < SL) sDe[tid] = tid < tn ? (float)exp_gate(sG[tn - 1] - sG[tid]) : 0.f;
        __syncthreads();
      }
      if (own && tn > 0) {
        if (B) {
          // tokens whose state began in the chunk: Y = (W beta) V over its tokens
          f32x4 Z[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) Z[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            f32x8 z;
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = Vr[2 * kk + (e >> 2)][e & 3];
            FT vb;
            if constexpr (P::E == 2) {
#pragma unroll
              for (int e = 0; e < 8; ++e) vb[e] = (__bf16)z[e];  // (exact)
            } else {
              vb = z;
            }
#pragma unroll
            for (int i = 2 * kk; i < 4; ++i) {
              const XT wa(wrow(i, kk, start_of(16 * i + c16)));
              if constexpr (P::E == 2)
                mma16_split(Z[i], wa, vb);
              else
                mma16(Z[i], wa, vb);
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (start_of(16 * i + 4 * q4 + r) >= 0) Y[i][r] = Z[i][r];
        }
        fresh_lane();
        const int s0 = plast < 0 ? 0 : plast;
        const float sc = (plast < 0) ? sA[tn - 1] : 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) S[i] *= sc;
        f32x4 ud[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 de = [&]() __attribute__((always_inline)) {
            const float4 x = *reinterpret_cast<const float4*>(sDe + 16 * i + 4 * q4);
            return f32x4{x.x, x.y, x.z, x.w};
          }();
          const float4 bi = *reinterpret_cast<const float4*>(sBeta + 16 * i + 4 * q4);
          const f32x4 u = f32x4{bi.x, bi.y, bi.z, bi.w} * (Vr[i] - Y[i]);
          ud[i] = u * de;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int t = 16 * i + 4 * q4 + r;
            if (t < s0) ud[i][r] = 0.f;
            if (t < tn) {
              Uh[(size_t)(c0 + t) * DV + col] = u[r];
              if (U16h) U16h[(size_t)(c0 + t) * DV + col] = from_f32<bf16_t>(u[r]);
            }
          }
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          if (32 * kk + 31 < s0 || 32 * kk >= tn) continue;  // (uniform)
          f32x8 z;
#pragma unroll
          for (int e = 0; e < 8; ++e) z[e] = ud[2 * kk + (e >> 2)][e & 3];
          const XT ub(z);
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            FT ka;
            if constexpr (P::TRANS) {
              const Tin* kp = sKt + (16 * i + c16) * TRS + 32 * kk + 4 * q4;
              ka = load_4x2<Tin>(kp, kp + 16);
              mma16_split(S[i], ka, ub);
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e)
                ka[e] = sK[(32 * kk + 16 * (e >> 2) + 4 * q4 + (e & 3)) * KRS + 16 * i + c16];
              mma16(S[i], ka, ub);
            }
          }
        }
      }
      if (tn < nrow) {  // the values again, over sQ
        __syncthreads();
#pragma unroll
        for (int u = 0; u < V16; ++u) {
          const int pi = tid + STHR * u;
          const int r = pi % SL, pc = pi / SL;
          *reinterpret_cast<u32x4*>(sV + r * VRS + pc * P::EPP) =
              reinterpret_cast<const u32x4*>(Vin + (size_t)(c0 + min(r, nrow - 1)) * DV)[pc];
        }
        __syncthreads();
      }
    }
    if (tn < nrow) {
      fresh_lane();
      // ---------------------------------------------------- token by token
      // One barrier per token, for LDS only (the pseudo-values' stores stay in
      // flight): every wave that holds state columns adds the waves' shares of
      // |S|^2 and y . v and takes the decision itself, wave 0 keeps the books.
      if (serial) {  // (else the Gram products left them)
        for (int t = wv; t < nrow; t += SWAVE) {
          float kk2 = 0.f, vv2 = 0.f;
          for (int i = lane; i < DK; i += 64) kk2 += to_f32(sK[t * KRS + i]) * to_f32(sK[t * KRS + i]);
          for (int i = lane; i < DV; i += 64) vv2 += to_f32(sV[t * VRS + i]) * to_f32(sV[t * VRS + i]);
          kk2 = wave_total_dpp(kk2);
          vv2 = wave_total_dpp(vv2);
          if (lane == 0) {
            sKK[t] = (double)kk2;
            sV2[t] = (double)vv2;
          }
        }
        lds_barrier();
      }
      for (int t = tn; t < nrow; ++t) {
        // shares of |S|^2, y . v: two sets in turn, so that the next token's need
        // not wait for this one's readers
        float2* sh = reinterpret_cast<float2*>(sPc) + (t & 1) * SWAVE;
        float y = 0.f, kr[NI][4];
        const float vt = own ? to_f32(sV[t * VRS + col]) : 0.f;
        if (own) {
          const float al = sAl[t];
          float b = 0.f;
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            load4f(sK + t * KRS + 16 * i + 4 * q4, kr[i]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              S[i][r] *= al;
              y += kr[i][r] * S[i][r];
              b += S[i][r] * S[i][r];
            }
          }
          b = wave_total_dpp(b);
          const float c = wave_total_dpp(y * vt);
          if (lane == 0) sh[wv] = make_float2(b, c);
          y += __shfl_xor(y, 16, 64);
          y += __shfl_xor(y, 32, 64);
        }
        lds_barrier();
        if (own) {
          double bs = 0.0, cs = 0.0;
#pragma unroll
          for (int i = 0; i < NW; ++i) {
            const float2 x = sh[i];
            bs += (double)x.x;
            cs += (double)x.y;
          }
          int bd = 1;
          float It = 0.f;  // the first token of an empty cache opens a state with score 0
          if (m0 > 0 || c0 + t > 0) {
            It = score_f((float)sKK[t] * (float)sV2[t], (float)bs, (float)cs, (float)D, a.eps,
                         a.eps_rms);
            bd = (It >= a.tau) ? 1 : 0;
            if (sBo[t] != -1) bd = sBo[t] ? 1 : 0;
            if (C == 1) bd = 0;
          }
          bd = __builtin_amdgcn_readfirstlane(bd);
          const float u = sBeta[t] * (vt - (bd ? 0.f : y));
          if (q4 == 0) {
            Uh[(size_t)(c0 + t) * DV + col] = u;
            if (U16h) U16h[(size_t)(c0 + t) * DV + col] = from_f32<bf16_t>(u);
          }
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[i][r] = (bd ? 0.f : S[i][r]) + kr[i][r] * u;
          if (wv == 0) {
            if (bd) {
              open_at(t, It);
            } else {
              dec.st.join(dec.m - 1, 1, (double)It);
              if (lane == t) dec.io = It;
            }
          }
        }
      }
    }
    fresh_lane();
    norm_share();
    if (wv == 0 && lane < nrow) {
      death[c0 + lane] = dec.dc;
      if (a.b_out) a.b_out[tok0 + c0 + lane] = (int8_t)((dec.B >> lane) & 1);
      if (a.merge_out) a.merge_out[tok0 + c0 + lane] = dec.mo;
      if (a.score_out) a.score_out[tok0 + c0 + lane] = dec.io;
    }
    Gprev = Gnext;
  }
  if (te == T) {
    if (wv == 0) dec.st.store(M.ibar, M.n, nullptr, dec.m);
    return;
  }
  // the carry for the next segment
  if (wv == 0) {
    dec.st.store(sv.ibar, sv.n, sv.lead, dec.m);
    if (lane == 0) *sv.m = dec.m;
  }
  if (own) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) sv.S[(((size_t)wv * NI + i) * 4 + r) * 64 + lane] = S[i][r];
  }
}

template <int DK, int DV>
static size_t delta_smem(int C) {
  const size_t f = DeltaP<DK, DV, float>::smem_bytes(C), b = DeltaP<DK, DV, bf16_t>::smem_bytes(C);
  return f > b ? f : b;
}

size_t prefill_delta_scan_smem(const dla_cache_desc& d) {
  if (d.d_k == 128 && d.d_v == 128) return delta_smem<128, 128>(d.C);
  if (d.d_k == 64 && d.d_v == 64) return delta_smem<64, 64>(d.C);
  if (d.d_k == 128 && d.d_v == 64) return delta_smem<128, 64>(d.C);
  return delta_smem<64, 128>(d.C);
}

template <int DK, int DV, typename Tin>
static hipError_t launch_delta_scan_t(const PrefillArgs& a, const PrefillWS& w, int tb, int te,
                                      const float* beta, float* U, bf16_t* U16, hipStream_t s) {
  const size_t shm = DeltaP<DK, DV, Tin>::smem_bytes(a.desc.C);
  if (shm > 160 * 1024) return hipErrorInvalidValue;
  auto launch = [&](auto k) -> hipError_t {
    if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) !=
        hipSuccess)
      return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(a.desc.B * a.desc.H), dim3(STHR), shm, s, a, w, tb, te, beta, U, U16);
    return hipGetLastError();
  };
  // (Four registers per lane and field for C up to 256, as in the gated scan,
  // spill 50 to 120 of this kernel's: 48 float32 heads of 128 x 128, 2048 tokens, C =
  // 128 took 2238 us, with the states in LDS 1374 without the readout.)
  if (a.desc.C > 64) return launch(prefill_delta_scan_kernel<DK, DV, Tin, 0>);
  return launch(prefill_delta_scan_kernel<DK, DV, Tin, 1>);
}

template <int DK, int DV>
static hipError_t launch_delta_scan_dims(const PrefillArgs& a, const PrefillWS& w, int tb, int te,
                                         const float* beta, float* U, bf16_t* U16,
                                         hipStream_t s) {
  if (a.in_dtype == DLA_F32) return launch_delta_scan_t<DK, DV, float>(a, w, tb, te, beta, U, U16, s);
  return launch_delta_scan_t<DK, DV, bf16_t>(a, w, tb, te, beta, U, U16, s);
}

static hipError_t launch_delta_scan(const PrefillArgs& a, const PrefillWS& w, int tb, int te,
                                    const float* beta, float* U, bf16_t* U16, hipStream_t s) {
  const int dk = a.desc.d_k, dv = a.desc.d_v;
  if (dk == 128 && dv == 128) return launch_delta_scan_dims<128, 128>(a, w, tb, te, beta, U, U16, s);
  if (dk == 64 && dv == 64) return launch_delta_scan_dims<64, 64>(a, w, tb, te, beta, U, U16, s);
  if (dk == 128 && dv == 64) return launch_delta_scan_dims<128, 64>(a, w, tb, te, beta, U, U16, s);
  return launch_delta_scan_dims<64, 128>(a, w, tb, te, beta, U, U16, s);
}

// Workspace of a delta-form prefill: the stages' workspace (for the serial or
// the pipelined plan; the float32 stages for float32 inputs), then the write
// vectors u (float32), and for 16-bit inputs a bfloat16 copy of them.
struct DeltaWS {
  size_t u, u16, total;
};

static DeltaWS delta_ws(const dla_cache_desc& d, int T, dla_dtype in, bool readout, bool serial,
                        size_t budget) {
  DeltaWS r;
  const size_t nh = (size_t)d.B * d.H;
  size_t off = round_up(prefill_workspace_bytes(d, T, in, readout, serial, budget), 256);
  r.u = off;
  off = round_up(off + nh * T * d.d_v * 4, 256);
  r.u16 = off;
  off = round_up(off + (in != DLA_F32 && readout ? nh * T * d.d_v * 2 : 0), 256);
  r.total = off;
  return r;
}

size_t prefill_delta_workspace_bytes(const dla_cache_desc& d, int T, dla_dtype in, bool readout,
                                     bool serial, size_t budget) {
  return delta_ws(d, T, in, readout, serial, budget).total;
}

// The stages of the gated prefill's schedule: serial (frames, the whole scan,
// then update and readout segment by segment, on s), or pipelined (the scan
// segment by segment on a second stream forked from s after the frames, and
// segment k's update and readout on s after scan segment k; the last
// segment's wait joins the second stream into s, and so does every error
// path after the fork).
hipError_t launch_prefill_delta(const PrefillArgs& a, const float* beta, hipStream_t s) {
  const bool readout = !a.skip_readout;
  const bool wide = a.in_dtype != DLA_F32;
  const bool serial = a.serial != 0;
  const DeltaWS L = delta_ws(a.desc, a.T, a.in_dtype, readout, serial, a.pool_budget);
  const size_t nh = (size_t)a.desc.B * a.desc.H;
  char* base = a.workspace;
  float* U = reinterpret_cast<float*>(base + L.u);
  bf16_t* U16 = wide && readout ? reinterpret_cast<bf16_t*>(base + L.u16) : nullptr;
  // the update takes u (float32), the readout u in the inputs' type
  PrefillArgs fu = a;
  fu.v = U;
  fu.v_f32 = wide ? 1 : 0;
  PrefillArgs fr = fu;
  fr.v_f32 = 0;
  if (wide) fr.v = U16;
  const bool pipe = pipelined(a.T, a.in_dtype, readout, serial);
  SegPlan p = seg_plan(a.desc, a.T, a.in_dtype, readout, serial, a.pool_budget);
  if (pipe && p.shared) {
    // The scan is the long stage where heads are few, inputs are float32 or chunks
    // go token by token, so the segments stay at the ramp's first size instead of
    // growing: what remains after the scan, the last segment's update and readout,
    // is then short (48 heads of 128 x 128, 2048 tokens: float32 2456 -> 2265 us,
    // bfloat16 1306 -> 1225, token by token 4226 -> 3446 and 3356 -> 3225).  The
    // pool is shared, so the segments change neither the workspace nor the results.
    p.fit = p.first;
    p.nseg = 0;
    p.nch_seg = 0;
    for (int b = 0; b < p.nch; ++p.nseg) {
      const int n = ramp_size(p.first, p.fit, p.nseg, p.nch - b);
      p.nch_seg = n > p.nch_seg ? n : p.nch_seg;
      b += n;
    }
  }
  const PrefillWS w = ws_layout(base, nh, a.T, a.desc.C, a.desc.d_k * a.desc.d_v, p.nch);
  hipError_t e;
  if ((e = launch_prefill_prep(fu, s)) != hipSuccess) return e;
  hipStream_t side = s;
  hipEvent_t* pev = nullptr;
  bool forked = false;
  auto fail = [&](hipError_t err) -> hipError_t {
    if (forked && hipEventRecord(pev[0], side) == hipSuccess) (void)hipStreamWaitEvent(s, pev[0], 0);
    return err;
  };
  if (pipe) {
    if ((e = pipe_resources(s, p.nseg + 1, &side, &pev)) != hipSuccess) return e;
    if ((e = hipEventRecord(pev[0], s)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(side, pev[0], 0)) != hipSuccess) return e;
    forked = true;
    for (int seg = 0; seg < p.nseg; ++seg) {
      int cs, ce;
      seg_range(p, seg, &cs, &ce);
      const int te = (seg + 1 == p.nseg) ? a.T : ce * p.RL;
      if ((e = launch_delta_scan(a, w, cs * p.RL, te, beta, U, U16, side)) != hipSuccess)
        return fail(e);
      if ((e = hipEventRecord(pev[1 + seg], side)) != hipSuccess) return fail(e);
    }
  } else if ((e = launch_delta_scan(a, w, 0, a.T, beta, U, U16, s)) != hipSuccess) {
    return e;
  }
  for (int seg = 0; seg < p.nseg; ++seg) {
    if (pipe && (e = hipStreamWaitEvent(s, pev[1 + seg], 0)) != hipSuccess) return fail(e);
    if ((e = launch_prefill_update(fu, p, seg, s)) != hipSuccess) return fail(e);
    if (readout && (e = launch_prefill_readout(fr, p, seg, s)) != hipSuccess) return fail(e);
  }
  // (the last segment's wait on pev[nseg] has joined the second stream)
  return hipSuccess;
}

}  // namespace dla
