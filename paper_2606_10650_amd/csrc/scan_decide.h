// The decisions of a 64-token scan chunk (Alg. 1 and Alg. 2, Sec. 3.1-3.2),
// shared by the gated scan and the delta-form scan.
//
// The scores of the chunk's tokens against a newest state that began at token
// p of the chunk (p = -1: before it) are one "row": lane t holds token t.  Wave
// 0 evaluates row after row, each boundary starting the next.  A row is a chain
// of about 2.5 k cycles (an affine scan over the lanes and the score's
// divisions), so where boundaries are dense all eight waves evaluate the rows
// of every start still possible at once, and what is left per boundary is a
// lookup and the capacity schedule.  That costs a chunk about as much as three
// rows; it is taken from the NSEQ-th boundary of a chunk on, and from the first
// when the two chunks before had that many.  (With four instead of eight, and one
// chunk before, prompts of two to four independent boundaries per chunk paid for
// both: 48 heads of 64 x 128, 4.4k tokens, a state per 18 / 24 / 32 tokens 1684 /
// 1359 / 1233 us, now 1582 / 1276 / 1178; row by row alone 1580 / 1272 / 1180, but
// a state per token, 1k tokens, 964 us instead of 658.)
#pragma once
#include "mfma.h"
#include "prefill.h"

namespace dla {

constexpr int SL = 64;      // tokens per scan chunk (one per lane of a wavefront)
constexpr int SWAVE = 8;    // waves per scan workgroup
constexpr int STHR = 64 * SWAVE;
constexpr int NSEQ = 8;     // boundaries of a chunk taken row by row

// Transposed copy of a 16-bit piece (columns 8 pc .. 8 pc + 7 of token r, r =
// lane): the lane pair (2i, 2i + 1) swaps halves, so each lane writes 32-bit
// words holding both tokens of the pair, 4 columns each.
template <int TRS>
__device__ __forceinline__ void put_transposed(bf16_t* dst, int pc, int r, const u32x4& val) {
  const bool odd = (r & 1) != 0;
  const uint32_t s0 = odd ? val[0] : val[2], s1 = odd ? val[1] : val[3];
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)s0, 0xB1, 0xF, 0xF, false);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)s1, 0xB1, 0xF, 0xF, false);
  // even lane: columns 0..3, own token first; odd lane: columns 4..7, the
  // partner's token (r - 1) first
  const uint32_t m0 = odd ? val[2] : val[0], m1 = odd ? val[3] : val[1];
  const uint32_t lo0 = odd ? r0 : m0, hi0 = odd ? m0 : r0;
  const uint32_t lo1 = odd ? r1 : m1, hi1 = odd ? m1 : r1;
  uint32_t* row = reinterpret_cast<uint32_t*>(dst + (pc * 8 + (odd ? 4 : 0)) * TRS + (r & ~1));
  row[0] = __builtin_amdgcn_perm(hi0, lo0, 0x05040100u);
  row[TRS / 2] = __builtin_amdgcn_perm(hi0, lo0, 0x07060302u);
  row[TRS] = __builtin_amdgcn_perm(hi1, lo1, 0x05040100u);
  row[3 * (TRS / 2)] = __builtin_amdgcn_perm(hi1, lo1, 0x07060302u);
}

// value of the next lane (lane 63: `last`)
__device__ __forceinline__ int next_lane_i(int x, int last) { return dpp_i<0x130, 0xF>(last, x); }
__device__ __forceinline__ double next_lane_d(double x, double last) {
  return dpp_d<0x130, 0xF>(last, x);
}

// The (aggregated score, token count, leader token) of every state in
// chronological order, held by one wave: lane l has states l + 64 r, r < NR (C
// at most 64 NR).  Leaders of states present before the call are negative.
template <int NR>
struct StatesInRegs {
  double I[NR];
  int n[NR], ld[NR];
  int C;

  __device__ __forceinline__ int lane() const { return threadIdx.x & 63; }
  __device__ __forceinline__ void load(const double* ib, const int32_t* nn, const int32_t* lead,
                                       int m0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int j = lane() + 64 * r;
      I[r] = j < C ? ib[j] : 0.0;
      n[r] = j < C ? nn[j] : 0;
      ld[r] = j < C && lead ? lead[j] : j - m0;
    }
  }
  __device__ __forceinline__ void store(double* ib, int32_t* nn, int32_t* lead, int m) const {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int j = lane() + 64 * r;
      if (j < m) {
        ib[j] = I[r];
        nn[j] = n[r];
        if (lead) lead[j] = ld[r];
      }
    }
  }
  __device__ __forceinline__ int lead(int j) const {  // (j uniform)
    int x = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if ((j >> 6) == r) x = __builtin_amdgcn_readlane(ld[r], j & 63);
    return x;
  }
  __device__ __forceinline__ void next(int r, double& In, int& nn, int& ln) const {
    const bool more = r + 1 < NR;
    const double I0 = more ? readlane_d(I[more ? r + 1 : r], 0) : 0.0;
    const int n0 = more ? __builtin_amdgcn_readlane(n[more ? r + 1 : r], 0) : 0;
    const int l0 = more ? __builtin_amdgcn_readlane(ld[more ? r + 1 : r], 0) : 0;
    In = next_lane_d(I[r], I0);
    nn = next_lane_i(n[r], n0);
    ln = next_lane_i(ld[r], l0);
  }
  // the adjacent pair of lowest density of a full cache, ties to the lowest
  // index; NaN densities (scores from non-finite inputs) compare false, so a
  // sequential argmin that starts at pair 0 never moves to them, and stays at
  // pair 0 when pair 0's density is NaN or none is a number
  __device__ __forceinline__ int argmin() const {
    double d[NR];
    double best = INFINITY;
    bool nan0 = false;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      d[r] = INFINITY;
      if (64 * r + 1 < C) {  // (uniform)
        double In;
        int nn, ln;
        next(r, In, nn, ln);
        const double x = (I[r] + In) / (double)(n[r] + nn);
        if (lane() + 64 * r + 1 < C && x < INFINITY) d[r] = x;
        if (r == 0) nan0 = (__ballot(__builtin_isnan(x)) & 1ull) != 0;
        best = d[r] < best ? d[r] : best;
      }
    }
    min_step<0x111, 0xF>(best);
    min_step<0x112, 0xF>(best);
    min_step<0x114, 0xF>(best);
    min_step<0x118, 0xF>(best);
    min_step<0x142, 0xA>(best);
    min_step<0x143, 0xC>(best);
    best = readlane_d(best, 63);
    if (nan0 || !(best < INFINITY)) return 0;
    int at = 0;
#pragma unroll
    for (int r = NR - 1; r >= 0; --r)
      if (64 * r + 1 < C) {
        const uint64_t eq = __ballot(d[r] == best);
        if (eq) at = 64 * r + __ffsll((unsigned long long)eq) - 1;
      }
    return at;
  }
  template <int CTRL, int RMASK>
  __device__ static __forceinline__ void min_step(double& x) {
    const double o = dpp_d<CTRL, RMASK>(INFINITY, x);
    x = o < x ? o : x;
  }
  // merge states i and i + 1, the later ones move down by one
  __device__ __forceinline__ void merge(int i, int m) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (64 * r < C) {
        double In;
        int nn, ln;
        next(r, In, nn, ln);
        const int j = lane() + 64 * r;
        I[r] = j < i ? I[r] : (j == i ? I[r] + In : In);
        n[r] = j < i ? n[r] : (j == i ? n[r] + nn : nn);
        ld[r] = j <= i ? ld[r] : ln;
      }
  }
  __device__ __forceinline__ void push(int m, double Iv, int lead) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (lane() + 64 * r == m) {
        I[r] = Iv;
        n[r] = 1;
        ld[r] = lead;
      }
  }
  __device__ __forceinline__ void join(int j, int cnt, double sI) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (lane() + 64 * r == j) {
        I[r] += sI;
        n[r] += cnt;
      }
  }
};

// Largest capacity whose bookkeeping stays in registers in a scan of d_k x d_v
// states: 64 (NR = 1) at 128 x 128, where NR = 4 spills 19 registers and the LDS
// form none (48 heads, 4k tokens, 200 / 100 states: NR = 4 1312 / 1017 us, LDS 1290 /
// 986; 4 x 16 heads x 16k tokens, 128 states, 5032 and 4974); else 256 (NR = 4; 48
// heads of 64 x 128, 4.4k tokens, 256 states: NR = 4 1582 us, LDS 1625).
constexpr int max_reg_c(int dk, int dv) { return dk * dv >= 128 * 128 ? 64 : 256; }

// The same in LDS, for larger capacities.
struct StatesInLds {
  double* I;
  int32_t *n, *ld;
  int C;

  __device__ __forceinline__ int lane() const { return threadIdx.x & 63; }
  __device__ __forceinline__ void load(const double* ib, const int32_t* nn, const int32_t* lead,
                                       int m0) {
    for (int j = lane(); j < C; j += 64) {
      I[j] = ib[j];
      n[j] = nn[j];
      ld[j] = lead ? lead[j] : j - m0;
    }
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void store(double* ib, int32_t* nn, int32_t* lead, int m) const {
    for (int j = lane(); j < m; j += 64) {
      ib[j] = I[j];
      nn[j] = n[j];
      if (lead) lead[j] = ld[j];
    }
  }
  __device__ __forceinline__ int lead(int j) const { return ld[j]; }
  __device__ __forceinline__ int argmin() const {
    double best = INFINITY;
    int bi = 0x7fffffff;
    for (int i = lane(); i + 1 < C; i += 64) {
      const double d = (I[i] + I[i + 1]) / (double)(n[i] + n[i + 1]);
      if (d < best) {
        best = d;
        bi = i;
      }
    }
    wave_argmin_d(best, bi);
    if (__builtin_isnan((I[0] + I[1]) / (double)(n[0] + n[1]))) return 0;
    return (bi >= 0 && bi <= C - 2) ? bi : 0;
  }
  // 64 entries at a time in increasing order (a block's writes never touch
  // entries that a later block still has to read)
  __device__ __forceinline__ void merge(int i, int m) {
    for (int j0 = i; j0 + 1 < m; j0 += 64) {
      const int j = j0 + lane();
      const bool act = j + 1 < m;
      double nI = 0.0;
      int nN = 0, nL = 0;
      if (act) {
        nI = (j == i) ? I[j] + I[j + 1] : I[j + 1];
        nN = (j == i) ? n[j] + n[j + 1] : n[j + 1];
        nL = (j == i) ? ld[j] : ld[j + 1];
      }
      __builtin_amdgcn_wave_barrier();
      if (act) {
        I[j] = nI;
        n[j] = nN;
        ld[j] = nL;
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  __device__ __forceinline__ void push(int m, double Iv, int lead) {
    if (lane() == 0) {
      I[m] = Iv;
      n[m] = 1;
      ld[m] = lead;
    }
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void join(int j, int cnt, double sI) {
    if (lane() == 0) {
      I[j] += sI;
      n[j] += cnt;
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// The score's part that does not depend on the row, and the score of the token
// against a state of |S|^2 = b, k^T S v = c.
template <typename N>
struct ScoreIn;
template <>
struct ScoreIn<float> {
  float eps_rms, D;
  float a;  // |k|^2 |v|^2
  __device__ __forceinline__ float at(float b, float c, float eps) const {
    return score_f(a, b, c, D, eps, eps_rms);
  }
};
// The delta form: the three terms of |N(s) - N(S)|^2, which cancel where the token
// fits the state, in float64.
template <>
struct ScoreIn<double> {
  double eps_rms, rD;
  double na, ra;  // a / rs^2, 1 / rs
  __device__ static __forceinline__ double rsq(double x) {  // one Newton step
    const double r = __builtin_amdgcn_rsq(x);
    return r * (1.5 - 0.5 * x * r * r);
  }
  __device__ static __forceinline__ ScoreIn of(double eps_rms, double D, double a) {
    ScoreIn s;
    s.eps_rms = eps_rms;
    s.rD = 1.0 / D;
    s.ra = rsq(a * s.rD + eps_rms);
    s.na = a * s.ra * s.ra;
    return s;
  }
  __device__ __forceinline__ float at(double b, double c, float eps) const {
    const double r = rsq(b * rD + eps_rms);
    const double nb = b * r * r;
    const float num = (float)(na + nb - 2.0 * c * ra * r);
    return sqrtf(num < 0.f ? 0.f : num) / (sqrtf((float)nb) + eps);
  }
};

// Scan-chunk constants of the lane's token, and of the layer.  N: the type of
// |S|^2's recurrence (float64 in the delta form, whose steps can also shrink it).
template <typename N>
struct RowIn {
  ScoreIn<N> sc;
  N al2n;       // alpha^2 of the next token
  int bo;       // boundary override
  int nrow, C;
  float tau, eps;
};

// |S|^2 as a share of the sum of its terms' sizes below which a row stops: the
// terms carry float32 roundings, so that above it |S|^2 is good to 16 x 2^-24.  Every
// token of ordinary prompts (beta in (0, 1), one state per 30 or more tokens) is
// above 1/8, with beta in 1.8 .. 2 above 1/16.
constexpr float kLost = 1.f / 16;

// Row p: the score of the lane's token against the newest state that began at
// p, with c = k^T S v of the decayed state and |S|^2 growing by inc when the
// token joins: b(t + 1) = alpha_{t+1}^2 (b(t) + inc(t)), b(start) = binit.
// Returns whether the token is scored by this row and opens a state.  lost: the
// token is scored by this row, but too little is left of the terms of its b for
// their sum to hold |S|^2 (delta form, whose inc may be negative).
template <typename N>
__device__ __forceinline__ bool score_row(const RowIn<N>& x, int t, int p, N ct, N inc,
                                          N binit, float& It, bool& valid, bool& lost) {
  const int ustart = p < 0 ? 0 : p;
  N Am = 1, Bm = 0;
  if (t >= ustart) {
    Am = x.al2n;
    Bm = x.al2n * inc;
  }
  valid = t < x.nrow && t > p;
  // inclusive scan of the affine maps b -> Am b + Bm over the lanes
  N bt;  // b(t) = b(lane t - 1's t + 1)
  if constexpr (sizeof(N) == 8) {
    float Sm = fabsf((float)Bm);  // the same sum over |inc|
    wave_scan_affine(Am, Bm, Sm);
    bt = dpp_d<0x138, 0xF>(binit, Am * binit + Bm);
    float st = dpp_f<0x138, 0xF>((float)binit, (float)(Am * binit) + Sm);
    if (t == ustart) st = (float)binit;
    if (t == ustart) bt = binit;
    lost = valid && !(bt >= (double)(kLost * st) && bt < 3.4e38);
  } else {
    wave_scan_affine(Am, Bm);
    bt = dpp_f<0x138, 0xF>(binit, Am * binit + Bm);
    if (t == ustart) bt = binit;
    lost = false;
  }
  It = valid ? x.sc.at(bt, ct, x.eps) : 0.f;
  int bd = (It >= x.tau) ? 1 : 0;
  if (x.bo != -1) bd = x.bo ? 1 : 0;
  if (x.C == 1) bd = 0;
  return valid && bd;
}

// LDS tables of the rows evaluated by all waves: scores [p][t], and per row the
// next boundary, its score and the sum of the scores of the tokens before it (or,
// with kStop added, the token before the first lost one if that comes no later).
struct RowTables {
  static constexpr int STRIDE = SL + 1;
  static constexpr int kStop = 256;
  float* It;     // [SL][STRIDE]
  double* sum;   // [SL]
  int32_t* nx;   // [SL]
  float* Inx;    // [SL]
  static constexpr size_t BYTES = (size_t)SL * STRIDE * 4 + SL * 16;
  __device__ __forceinline__ explicit RowTables(char* base) {  // (16-byte aligned)
    sum = reinterpret_cast<double*>(base);
    nx = reinterpret_cast<int32_t*>(sum + SL);
    Inx = reinterpret_cast<float*>(nx + SL);
    It = Inx + SL;
  }
};

// Rows p0 .. nrow - 1, one workgroup; row(p, ct, inc) gives the lane's c and
// growth for a state that began at p.
template <typename N, typename RowFn>
__device__ __forceinline__ void fill_rows(const RowIn<N>& x, int p0, RowTables tb, RowFn row) {
  const int t = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  auto finish = [&](int p, bool open, bool lost, float It) __attribute__((always_inline)) {
    const uint64_t mask = __ballot(open), lmask = __ballot(lost);
    const int ts = mask ? (__ffsll((unsigned long long)mask) - 1) : x.nrow;
    const int tl = lmask ? (__ffsll((unsigned long long)lmask) - 1) : SL + 1;
    const int e = tl <= ts ? max(tl - 1, p + 1) : ts;
    const double s = wave_sum_d((t > p && t < e) ? (double)It : 0.0);
    tb.It[p * RowTables::STRIDE + t] = It;
    if (t == 0) {
      tb.nx[p] = tl <= ts ? e + RowTables::kStop : e;
      tb.sum[p] = s;
    }
    if (t == ts) tb.Inx[p] = It;
  };
  // two rows at a time, so that their chains overlap
  for (int p = p0 + wv; p < x.nrow; p += 2 * SWAVE) {
    const int q = min(p + SWAVE, SL - 1);
    float Ip, Iq;
    N cp, cq, ip, iq;
    bool vp, vq, lp, lq;
    row(p, cp, ip);
    row(q, cq, iq);
    const bool op = score_row(x, t, p, cp, ip, N(0), Ip, vp, lp);
    const bool oq = score_row(x, t, q, cq, iq, N(0), Iq, vq, lq);
    finish(p, op, lp, Ip);
    if (p + SWAVE < x.nrow) finish(p + SWAVE, oq, lq, Iq);
  }
}

// One chunk's decisions, by wave 0: lane t ends with token t's boundary (bit t
// of B), merge index, score and death token (T or later merged: its state's;
// -1: opens no state).
template <typename States>
struct ChunkDecider {
  States st;
  int m;        // states in the cache
  int p;        // where the newest state began (-1: before the chunk)
  // tokens of the chunk that the rows decide (set to nrow before them): up to the
  // one whose step leaves the lost |S|^2
  int tn;
  uint64_t B;
  int runs = 0;  // chunks in a row with NSEQ boundaries or more
  int mo, dc;
  float io;

  // whether the chunk to come is taken by the row tables from its first boundary
  __device__ __forceinline__ bool dense() {  // (B: the chunk before)
    runs = __popcll(B) >= NSEQ ? runs + 1 : 0;
    return runs >= 2;
  }

  // a state opens at token ts of the chunk with score Is: Alg. 2 when the cache
  // is full, then the new state.  kill(lead, token) records the death of a state
  // that began before the chunk.
  template <typename Kill>
  __device__ __forceinline__ void open(int ts, float Is, int mpre, int c0, int C, int T,
                                       uint32_t* flags, Kill kill) {
    const int t = threadIdx.x & 63;
    int istar = -1;
    if (m == C) {
      const int fo = __builtin_amdgcn_readlane(mpre, ts);
      if (fo >= 0 && fo <= C - 2) {
        istar = fo;
      } else {
        if (fo != -1 && t == 0) atomicOr(flags, DLA_FLAG_BAD_MERGE_OVERRIDE);
        istar = st.argmin();
      }
      // the state right of the pair dies at this token
      const int ld = st.lead(istar + 1);
      if (ld >= c0) {
        if (t == ld - c0) dc = c0 + ts;
      } else if (t == 0) {
        kill(ld, c0 + ts);
      }
      st.merge(istar, m);
      m -= 1;
    }
    st.push(m, (double)Is, c0 + ts);
    m += 1;
    if (t == ts) {
      mo = istar;
      dc = T;
      io = Is;
    }
    B |= 1ull << ts;
    p = ts;
  }

  // Rows one at a time until the chunk or, at a lost token, the rows end (returns
  // false) or nseq boundaries were taken with tokens left (returns true; fill_rows
  // and finish_rows go on from p).  row(p, ct, inc, binit) as for fill_rows.
  template <typename N, typename RowFn, typename OpenFn>
  __device__ __forceinline__ bool first_rows(const RowIn<N>& x, int nseq, RowFn row,
                                             OpenFn open_at) {
    const int t = threadIdx.x & 63;
    int taken = 0;
    while (p + 1 < x.nrow) {
      float It;
      N ct, inc, binit;
      bool valid, lost;
      row(p, ct, inc, binit);
      const bool op = score_row(x, t, p, ct, inc, binit, It, valid, lost);
      const uint64_t mask = __ballot(op), lmask = __ballot(lost);
      const int ts = mask ? (__ffsll((unsigned long long)mask) - 1) : x.nrow;
      const int tl = lmask ? (__ffsll((unsigned long long)lmask) - 1) : SL + 1;
      const int e = tl <= ts ? max(tl - 1, p + 1) : ts;
      const bool joins = valid && t < e;
      if (joins) io = It;
      if (e > p + 1) st.join(m - 1, e - (p + 1), wave_sum_d(joins ? (double)It : 0.0));
      if (tl <= ts) {
        tn = e;
        return false;
      }
      if (ts >= x.nrow) return false;
      open_at(ts, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(It), ts)));
      if (++taken == nseq) return p + 1 < x.nrow;
    }
    return false;
  }

  // The rest of the chunk from the tables of fill_rows(p0 = p).
  template <typename N, typename OpenFn>
  __device__ __forceinline__ void finish_rows(const RowIn<N>& x, RowTables tb, OpenFn open_at) {
    const int t = threadIdx.x & 63;
    const int p0 = p;
    const int tt = min(max(t, p0), x.nrow - 1);  // (rows before p0 hold nothing)
    const int nx = tb.nx[tt];
    const float In = nx < x.nrow ? tb.Inx[tt] : 0.f;
    const double sm = tb.sum[tt];
    while (true) {
      const int n = __builtin_amdgcn_readlane(nx, p);
      const int ts = n & (RowTables::kStop - 1);
      if (ts > p + 1) st.join(m - 1, ts - (p + 1), readlane_d(sm, p));
      if (n >= RowTables::kStop) tn = ts;
      if (n >= x.nrow) break;
      open_at(ts, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(In), p)));
      if (p + 1 >= x.nrow) break;
    }
    // every later token was scored by the row of the last boundary before it
    if (t > p0 && t < x.nrow) {
      const uint64_t below = B & ((1ull << t) - 1ull);
      io = tb.It[(63 - __clzll((long long)below)) * RowTables::STRIDE + t];
    }
  }
};

}  // namespace dla
