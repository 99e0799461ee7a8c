// LinSimp forward on gfx950: feature-bank preparation, chunk prefix states,
// the chunk scan with a causal log-space frame, and the anchor-window readout.
//
// Method (per head, 0-based rows; the paper counts from 1):
//   phi(x) = m^{-1/2} exp(Omega x - |x|^2/2)                  [Sec. 3.2, eq:prf]
//   M_i = sum_{j<=i} phi(k_j) v_j^T, a_i = sum_{j<=i} phi(k_j) [eq:Mstate, eq:astate]
//   z_ic = q_i (*) r_c,  C_i = {max(0,i-w+1) .. i}              [Sec. 3.2, 3.3]
//   N_i = sum_c [phi(z_ic)^T M_i] (*) u_c,  Z_i = sum_c phi(z_ic)^T a_i,
//   out_i = N_i / (Z_i + eps)                                   [eq:Ni, eq:Zi, eq:linearized-output]
//
// Everything is evaluated in log2 space.  Query side (App. B.2): one shift
// L_i = max over valid (c, p) of the log features, kept online across anchor
// tiles and feature blocks.  Key side: a causal running maximum R_j of the key
// log features; key features are exp2(lambda_j - R_j)/sqrt(m) and every state
// carries its frame, so neither side can overflow and a row never sees a
// future token's scale.  The 1/sqrt(m) of the query feature is dropped (it
// cancels in the ratio, App. A "Feature scaling").
#include <type_traits>

#include "common.h"
#include "linsimp_internal.h"
#include "prof.h"
#include "keyfeat.h"

namespace linsimp {

struct FwdArgs {
  const void* q; const void* k; const void* v; const void* r; const void* u;
  const float* omega;
  void* out; float* stats;
  void* omq; void* omk; void* omh;
  float* states; float* rho; float* rex;
  void* states16;     // [BH][nch][m][Dv] bf16 inputs: the boundary states' M in bf16; null for float32
  float* part;                                        // [NFB][BH][n][Dv+2] when m > 128
  void* chi;          // [BH][n][m] key features 2^(lambda_j - R_j)/sqrt(m), p permuted in 16-blocks
  float* rj;          // [BH][n]    running key frame R_j (log2)
  int H; int n; int w; int nch; int BH; float eps;
  // bf16 scan in segments (G > 1): chunks per segment; [BH][G-1][m*Dv] states of
  // the segments before the last (matrix-core tiles), [BH][G-1][m], [BH][G-1]
  int G; int cps;
  float* seg_M; float* seg_a; float* seg_R;
};

// ---------------------------------------------------------------------------
// K0: Omega * log2(e) in the operand type; key side keeps a hi/lo bf16 split so
// that key log features are accurate to ~2^-16 relative (bf16 keys are exact).
// bf16 inputs also get an f16 copy for the query-side logits (f16 matrix cores).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_prep_omega(const float* __restrict__ omega, T* __restrict__ omq,
                                                    T* __restrict__ omk, f16* __restrict__ omh, int H, int MD,
                                                    int D) {
  using F = MF<T>;
  int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= H * MD) return;
  float x = omega[idx] * kLog2e;
  omq[idx] = (T)x;
  // the key-side copy in fragment order (the order of bank_frag)
  const int hh = idx / MD, e = idx % MD, p = e / D, k = e % D;
  const size_t f = ((size_t)((p >> 5) * (D / F::KS) + k / F::KS) * 64 + ((k % F::KS) / F::KPL) * 32 + (p & 31))
                   * F::KPL + k % F::KPL;
  if constexpr (sizeof(T) == 2) {
    omh[idx] = (f16)x;
    bf16 hi = (bf16)x;
    omk[(size_t)hh * 2 * MD + f] = hi;
    omk[(size_t)hh * 2 * MD + MD + f] = (bf16)(x - (float)hi);
  } else {
    omk[(size_t)hh * MD + f] = (T)x;
  }
}

// ---------------------------------------------------------------------------
// K2: per 32-token chunk b, its contribution to the prefix state in the frame
// rho_b = max key log2-feature of the chunk:
//   Mt_b = sum_j chi_j v_j^T, at_b = sum_j chi_j, chi_j = exp2(lambda_j - rho_b)/sqrt(m)
// One wave per chunk.  [App. C "Host preparation": per-chunk contributions]
// ---------------------------------------------------------------------------
template <typename T, int D, int DV, int M>
__global__ __launch_bounds__(256) void k_chunk_state(FwdArgs a) {
  using F = MF<T>;
  constexpr int PAD = F::PAD;
  constexpr int S = M * DV + M;
  __shared__ __align__(16) T sVt[4][DV][32 + PAD];
  __shared__ __align__(16) float snk[4][32];
  const int tid = threadIdx.x, l = tid & 63, col = l & 31, h = l >> 5, wv = uniform(tid >> 6);
  const int b = blockIdx.x * 4 + wv;
  const int bh = blockIdx.y, hh = bh % a.H, n = a.n;
  const bool active = b < a.nch;
  const int tok0 = b * 32;
  const T* ks = (const T*)a.k + (size_t)bh * n * D;
  const T* vs = (const T*)a.v + (size_t)bh * n * DV;
  const T* omk_h = (const T*)a.omk + (size_t)hh * (sizeof(T) == 2 ? 2 : 1) * M * D;
  f32x16 acc[M / 32];
  float nk = 0.0f;
  if (active) {
    // V^T of the chunk, token index permuted (it pairs with a register operand):
    // every 16-byte row piece is loaded first (rows clamped), then stored transposed
    constexpr int VE = 16 / (int)sizeof(T);
    constexpr int IT = 32 * (DV / VE) / 64;
    static_assert(32 * (DV / VE) % 64 == 0, "whole pieces per lane");
    typedef T VP __attribute__((ext_vector_type(VE)));
    VP xv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int idx = l + 64 * it, jj = idx % 32, d0 = (idx / 32) * VE;
      xv[it] = *(const VP*)(vs + (size_t)min(tok0 + jj, n - 1) * DV + d0);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int idx = l + 64 * it, jj = idx % 32, d0 = (idx / 32) * VE;
      const bool ok = tok0 + jj < n;
#pragma unroll
      for (int e = 0; e < VE; ++e) sVt[wv][d0 + e][F::sigma(jj)] = ok ? xv[it][e] : (T)0.0f;
    }
    key_logits<T, D, M, false>(acc, nk, ks, tok0, n, omk_h);
    if (h == 0) snk[wv][col] = nk;
  }
  __syncthreads();
  if (!active) return;
  float mx = kNegInf;
  float nkt[16];
  crow_vals(snk[wv], nkt);
#pragma unroll
  for (int pt = 0; pt < M / 32; ++pt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float x = acc[pt][v] - 0.5f * kLog2e * nkt[v];
      acc[pt][v] = (tok0 + crow(v, h) < n) ? x : kNegInf;
      mx = fmaxf(mx, acc[pt][v]);
    }
  const float rb = wave_max(mx);
  const float rs = rsqrtf((float)M);
  float* st = a.states + ((size_t)bh * a.nch + b) * S;
  // bf16 inputs: the two operands of Mt_b = chi^T V are left in the chunk's
  // (otherwise unused) float32 M slot, as the 16-byte fragments the matrix
  // cores take: chi^T [p][sigma(j)] (m x 32) and V^T [d][sigma(j)] (DV x 32);
  // k_state_scan_mma forms the product and scans it
  bf16* cx = (bf16*)st;
  bf16* vx = cx + M * 32;
#pragma unroll
  for (int pt = 0; pt < M / 32; ++pt) {
    float asum = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float c = fast_exp2(acc[pt][v] - rb) * rs;
      acc[pt][v] = c;
      asum += c;
    }
    asum = half_swap_add(asum);
    if (h == 0) st[M * DV + pt * 32 + col] = asum;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int sp = 0; sp < F::CSTEPS; ++sp)
        *(bf16x8*)(cx + (pt * 32 + col) * 32 + 16 * sp + 8 * h) = F::cfrag(acc[pt], sp);
    } else {
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt) {
        f32x16 o = zero16();
#pragma unroll
        for (int sp = 0; sp < F::CSTEPS; ++sp)
          o = F::mma(F::cfrag(acc[pt], sp), F::ldc(&sVt[wv][dt * 32 + col][0], 0, sp, h), o);
#pragma unroll
        for (int v = 0; v < 16; ++v) st[(size_t)(pt * 32 + crow(v, h)) * DV + dt * 32 + col] = o[v];
      }
    }
  }
  if constexpr (sizeof(T) == 2) {
    for (int idx = l; idx < DV * 4; idx += 64)
      *(bf16x8*)(vx + (idx >> 2) * 32 + 8 * (idx & 3)) = *(const bf16x8*)(&sVt[wv][idx >> 2][8 * (idx & 3)]);
  }
  if (l == 0) a.rho[(size_t)bh * a.nch + b] = rb;
}

// ---------------------------------------------------------------------------
// K2b: exclusive scan over chunks with the log-scale monoid
//   (M1, R1) + (M2, r2) = (e^{R1-R} M1 + e^{r2-R} M2, R = max(R1, r2))
// in place: chunk b's contribution is replaced by the state of every token
// before chunk b, in frame rex[b] (-inf for the empty state).  With bf16
// inputs the M part of that state goes to states16 in bf16 instead (the
// operand type of every kernel that reads it, rounded once here; half the
// bytes for the scan and its readers) and only a stays in place.
// Element-parallel, sequential over chunks, loads issued PF chunks ahead.
// [App. C "Host preparation": exclusive cumulative sum -> boundary states]
// ---------------------------------------------------------------------------
template <int M, int DV>
__global__ __launch_bounds__(256) void k_state_scan(FwdArgs a) {
  constexpr int PF = 8;
  constexpr int S = M * DV + M;
  const int bh = blockIdx.y;
  const int i4 = (blockIdx.x * 256 + threadIdx.x) * 4;
  const bool act = i4 < S;
  const int nch = a.nch;
  float* st = a.states + (size_t)bh * nch * S;
  bf16* s16 = a.states16 != nullptr ? (bf16*)a.states16 + (size_t)bh * nch * M * DV : nullptr;
  const float* rh = a.rho + (size_t)bh * nch;
  float* rx = a.rex + (size_t)bh * (nch + 1);
  const bool writer = (blockIdx.x == 0 && threadIdx.x == 0);
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  float R = kNegInf;
  for (int b0 = 0; b0 < nch; b0 += PF) {
    f32x4 x[PF];
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      if (act && b0 + e < nch) x[e] = *(const f32x4*)(st + (size_t)(b0 + e) * S + i4);
      else x[e] = run * 0.0f;
    }
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      int b = b0 + e;
      if (b >= nch) break;
      float rb = rh[b];
      float Rn = fmaxf(R, rb);
      float sa = fast_exp2(R - Rn);      // 0 when R = -inf
      float sb = fast_exp2(rb - Rn);
      if (s16 != nullptr && i4 < M * DV) {
        if (act) {
          bf16x4 y;
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = (bf16)run[e];
          *(bf16x4*)(s16 + (size_t)b * M * DV + i4) = y;
        }
      } else if (act) {
        *(f32x4*)(st + (size_t)b * S + i4) = run;
      }
      if (writer) rx[b] = R;
      run = run * sa + x[e] * sb;
      R = Rn;
    }
  }
  if (writer) rx[nch] = R;
}

// ---------------------------------------------------------------------------
// Key features of every token in the causal running frame (one wave per chunk,
// after the scan has fixed each chunk's entry frame Rex_b):
//   R_j = max(Rex_b, max_{s0 <= j' <= j} max_p lambda_j'p),  chi_j = 2^(lambda_j - R_j)/sqrt(m)
// stored with p permuted inside 16-blocks (the LDS operand layout), for the
// readout's intra-chunk correction and, through the shared workspace, the
// backward sweeps.
// ---------------------------------------------------------------------------
template <typename T, int D, int M>
// (two waves per SIMD also at m = 256, where 267 registers would leave one: 32
// heads x 65536 tokens 2.61 -> 0.75 ms; at d = m = 128, 2 x 16 x 16384, 0.115 -> 0.102)
__global__ __launch_bounds__(256, (D * M >= 128 * 128 ? 2 : 1)) void k_keyfeat(FwdArgs a) {
  using F = MF<T>;
  const int tid = threadIdx.x, l = tid & 63, col = l & 31, h = l >> 5, wv = uniform(tid >> 6);
  const int bh = blockIdx.y, hh = bh % a.H, n = a.n, nch = a.nch;
  const int cb = blockIdx.x * 4 + wv;
  if (cb >= nch) return;
  const int s0 = cb * 32;
  const size_t seq = (size_t)bh * n;
  const T* ks = (const T*)a.k + seq * D;
  const T* omk_h = (const T*)a.omk + (size_t)hh * (sizeof(T) == 2 ? 2 : 1) * M * D;
  f32x16 acc[M / 32];
  float nk;
  key_logits<T, D, M, true>(acc, nk, ks, s0, n, omk_h);
  const bool vt = s0 + col < n;
  float mx = kNegInf;
#pragma unroll
  for (int pt = 0; pt < M / 32; ++pt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float x = vt ? acc[pt][v] - 0.5f * kLog2e * nk : kNegInf;
      acc[pt][v] = x;
      mx = fmaxf(mx, x);
    }
  mx = half_swap_max(mx);
  float R = mx;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    float t = __shfl_up(R, o, 32);
    if (col >= o) R = fmaxf(R, t);
  }
  R = fmaxf(R, a.rex[(size_t)bh * (nch + 1) + cb]);
  if (vt && h == 0) a.rj[seq + s0 + col] = R;
  const float rsm = rsqrtf((float)M);
  // the wave's 32 x M tile goes through LDS, so that the global stores are
  // whole 16-byte pieces of rows (lanes along a row) instead of 8-byte pieces
  // of 32 different rows
  constexpr int CP = M + 16 / (int)sizeof(T);              // row pitch (elements)
  __shared__ __align__(16) T sX[4][32][CP];
  T* xr = &sX[wv][col][0];
#pragma unroll
  for (int pt = 0; pt < M / 32; ++pt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      typedef T V4 __attribute__((ext_vector_type(4)));
      V4 x4;
#pragma unroll
      for (int e = 0; e < 4; ++e) x4[e] = (T)(fast_exp2(acc[pt][4 * g + e] - R) * rsm);
      *(V4*)(xr + F::sigma(pt * 32 + 8 * g + 4 * h)) = x4;   // sigma keeps 4-groups contiguous
    }
  wave_lds_sync();
  constexpr int VE = 16 / (int)sizeof(T), PPR = M / VE;    // 16-byte pieces per row
  typedef T V __attribute__((ext_vector_type(VE)));
  T* dst = (T*)a.chi + (seq + s0) * M;
  const int nrow = min(32, n - s0);
  // every piece read from LDS first, only the stores conditional (a read under
  // the condition would be a branch that waits for it)
  constexpr int IT = 32 * PPR / 64;
  V xs[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = l + 64 * it, r = idx / PPR, c = (idx % PPR) * VE;
    xs[it] = *(const V*)(&sX[wv][r][c]);
  }
  no_hoist();                                   // (and not sunk into the branches)
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = l + 64 * it, r = idx / PPR, c = (idx % PPR) * VE;
    if (r < nrow) *(V*)(dst + (size_t)r * M + c) = xs[it];
  }
}

// ---------------------------------------------------------------------------
// K2b for bf16 inputs: the same exclusive scan, with each chunk's contribution
// Mt_b = chi^T V formed here on the matrix cores from the operand fragments the
// chunk kernel left in the chunk's M slot (0.2 of the bytes of a float32
// contribution).  One wave per (sequence-head, 32 features, 32 columns): the
// running state tile stays in its registers, the fragments of the chunks ahead
// are loaded PF chunks in advance (they do not depend on the recurrence), and
// each chunk's boundary state is written in bf16 to states16.  The wave of the
// first 32 columns also scans a in place.  Workgroups are dealt to the eight
// XCDs in turn; the waves of one sequence-head are numbered to land on one XCD,
// so the fragments they share come through one L2.
// A wave's chain is one chunk after the other (0.55-0.7 us each), so a short
// batch is cut into G segments: k_scan_totals forms each segment's state, and
// every segment's scan starts from the sum of those before it.
// [App. C "Host preparation": exclusive cumulative sum -> boundary states]
// ---------------------------------------------------------------------------
// A wave's place: sequence-head, state tile (features p0.., columns d0..) and segment
template <int M, int DV>
struct ScanPlace {
  static constexpr int NDT = DV / 32, NPD = (M / 32) * NDT;
  int bh, tt, g, p0, d0;
  LS_DEV explicit ScanPlace(int nseg) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    g = slot % nseg;
    tt = (slot / nseg) % NPD;
    bh = xcd + 8 * (slot / (nseg * NPD));
    p0 = (tt / NDT) * 32;
    d0 = (tt % NDT) * 32;
  }
};

// The operands of chunk b's contribution to a wave's tile, PF chunks in flight:
// every load unconditional (clamped chunk index), so that the compiler's
// memory-counter waits see them all
template <int M, int DV, int PF>
struct ScanRing {
  bf16x8 xq[PF][4];
  float aq[PF], rq[PF];
  LS_DEV void fetch(const float* stb, const float* rh, int p0, int d0, int b, int e) {
    constexpr int S = M * DV + M;
    const int l = threadIdx.x, col = l & 31, h = l >> 5;
    const bf16* cx = (const bf16*)(stb + (size_t)b * S);
    const bf16* vx = cx + M * 32;
    xq[e][0] = *(const bf16x8*)(cx + (p0 + col) * 32 + 8 * h);
    xq[e][1] = *(const bf16x8*)(cx + (p0 + col) * 32 + 16 + 8 * h);
    xq[e][2] = *(const bf16x8*)(vx + (d0 + col) * 32 + 8 * h);
    xq[e][3] = *(const bf16x8*)(vx + (d0 + col) * 32 + 16 + 8 * h);
    aq[e] = stb[(size_t)b * S + M * DV + p0 + col];
    rq[e] = rh[b];
  }
  // run, runa, R <- the state with chunk b's contribution (ring slot e)
  LS_DEV void add(int e, f32x16& run, float& runa, float& R) const {
    f32x16 c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xq[e][0], xq[e][2], zero16(), 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xq[e][1], xq[e][3], c, 0, 0, 0);
    const float rb = uniform(rq[e]);
    const float Rn = fmaxf(R, rb);
    const float sa = fast_exp2(R - Rn);                // 0 when R = -inf
    const float sb = fast_exp2(rb - Rn);
#pragma unroll
    for (int v = 0; v < 16; ++v) run[v] = run[v] * sa + c[v] * sb;
    runa = runa * sa + aq[e] * sb;
    R = Rn;
  }
};

// The state of every segment but the last, one wave per (sequence-head, tile,
// segment), tiles as the accumulator holds them
template <int M, int DV>
__global__ __launch_bounds__(64) void k_scan_totals(FwdArgs a) {
  constexpr int S = M * DV + M, PF = 6;
  using P = ScanPlace<M, DV>;
  const P w(a.G - 1);
  if (w.bh >= a.BH) return;                            // wave-uniform
  const int l = threadIdx.x, col = l & 31, h = l >> 5;
  const int b0 = w.g * a.cps, b1 = b0 + a.cps;         // (whole segments: only the last may be short)
  const float* stb = a.states + (size_t)w.bh * a.nch * S;
  const float* rh = a.rho + (size_t)w.bh * a.nch;
  ScanRing<M, DV, PF> ring;
#pragma unroll
  for (int e = 0; e < PF; ++e) ring.fetch(stb, rh, w.p0, w.d0, min(b0 + e, b1 - 1), e);
  f32x16 run = zero16();
  float runa = 0.0f, R = kNegInf;
  int b = b0;
  for (; b + PF <= b1; b += PF) {
#pragma unroll
    for (int e = 0; e < PF; ++e) {
      ring.add(e, run, runa, R);
      ring.fetch(stb, rh, w.p0, w.d0, min(b + e + PF, b1 - 1), e);
    }
  }
#pragma unroll
  for (int e = 0; e < PF; ++e)
    if (b + e < b1) ring.add(e, run, runa, R);
  const size_t sg = (size_t)w.bh * (a.G - 1) + w.g;
  float* o = a.seg_M + (sg * P::NPD + w.tt) * 1024 + l * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) *(f32x4*)(o + 256 * q) = f32x4{run[4 * q], run[4 * q + 1], run[4 * q + 2], run[4 * q + 3]};
  if (w.d0 == 0 && h == 0) a.seg_a[sg * M + w.p0 + col] = runa;
  if (w.tt == 0 && l == 0) a.seg_R[sg] = R;
}

template <int M, int DV>
__global__ __launch_bounds__(64) void k_state_scan_mma(FwdArgs a) {
  constexpr int S = M * DV + M, PF = 6;
  using P = ScanPlace<M, DV>;
  // the state tile passes through LDS so that each lane stores 32 contiguous
  // bytes (16 two-byte stores per lane would take most of the memory counter
  // that the loads in flight need)
  __shared__ __align__(16) bf16 sT[32][40];
  const P w(a.G);
  if (w.bh >= a.BH) return;                            // wave-uniform
  const int l = threadIdx.x, col = l & 31, h = l >> 5;
  const int bh = w.bh, p0 = w.p0, d0 = w.d0, nch = a.nch;
  const int bs = w.g * a.cps, be = min(bs + a.cps, nch);
  float* stb = a.states + (size_t)bh * nch * S;
  bf16* s16 = (bf16*)a.states16 + (size_t)bh * nch * M * DV;
  const float* rh = a.rho + (size_t)bh * nch;
  float* rx = a.rex + (size_t)bh * (nch + 1);
  const bool aw = d0 == 0;                              // also scans a (lanes of half 0)
  const bool writer = w.tt == 0 && l == 0;
  ScanRing<M, DV, PF> ring;
#pragma unroll
  for (int e = 0; e < PF; ++e) ring.fetch(stb, rh, p0, d0, min(bs + e, be - 1), e);
  f32x16 run = zero16();
  float runa = 0.0f, R = kNegInf;
  // the segments before this one
#pragma unroll 2
  for (int g = 0; g < w.g; ++g) {
    const size_t sg = (size_t)bh * (a.G - 1) + g;
    const float* x = a.seg_M + (sg * P::NPD + w.tt) * 1024 + l * 4;
    f32x4 t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) t[q] = *(const f32x4*)(x + 256 * q);
    const float ta = a.seg_a[sg * M + p0 + col], rb = a.seg_R[sg];
    const float Rn = fmaxf(R, rb), sa = fast_exp2(R - Rn), sb = fast_exp2(rb - Rn);
#pragma unroll
    for (int v = 0; v < 16; ++v) run[v] = run[v] * sa + t[v >> 2][v & 3] * sb;
    runa = runa * sa + ta * sb;
    R = Rn;
  }
  // chunk b from ring slot e, then slot e takes chunk b + PF
  auto step = [&](int b, int e) {
    // the state of every token before chunk b (frame R)
#pragma unroll
    for (int v = 0; v < 16; ++v) sT[crow(v, h)][col] = (bf16)run[v];
    wave_lds_sync();
    {
      const int rr = l >> 1, c0 = 16 * (l & 1);
      const bf16x8 y0 = *(const bf16x8*)&sT[rr][c0], y1 = *(const bf16x8*)&sT[rr][c0 + 8];
      bf16* o = s16 + ((size_t)b * M + p0 + rr) * DV + d0 + c0;
      *(bf16x8*)o = y0;
      *(bf16x8*)(o + 8) = y1;
    }
    if (aw) stb[(size_t)b * S + M * DV + p0 + col] = runa;   // both halves: the same value
    if (writer) rx[b] = R;
    ring.add(e, run, runa, R);
    ring.fetch(stb, rh, p0, d0, min(b + PF, be - 1), e);
  };
  int b0 = bs;
  for (; b0 + PF <= be; b0 += PF) {
#pragma unroll
    for (int e = 0; e < PF; ++e) step(b0 + e, e);
  }
#pragma unroll
  for (int e = 0; e < PF; ++e)
    if (b0 + e < be) step(b0 + e, e);
  if (writer && be == nch) rx[nch] = R;
}

// ---------------------------------------------------------------------------
// K3: anchor-window readout for one chunk of 32 rows.
// ---------------------------------------------------------------------------
template <typename T, int D, int DV, int M, int NW, int NA>
struct RCfg {
  static constexpr int PAD = MF<T>::PAD;
  static constexpr int BC = 32;
  static constexpr int FB = M < 128 ? M : 128;          // feature block (<= 128 as in Alg. 1)
  static constexpr int NFB = M / FB;
  static constexpr int WIN = BC + 32 * NA - 1;           // anchor rows the chunk can touch
  static constexpr int UST = ((WIN + 2) / 4) * 4 + 2;   // odd dword stride: conflict-free 2-byte column reads
  static constexpr int RPW = (BC + NW - 1) / NW;
  static constexpr int ES = sizeof(T);
  static constexpr int a16(int x) { return (x + 15) & ~15; }
  static constexpr int oOm = 0;
  static constexpr int oMt = oOm + a16(FB * (D + PAD) * ES);
  static constexpr int oA = oMt + a16(DV * (FB + PAD) * ES);
  static constexpr int oChi = oA + (sizeof(T) == 4 ? a16(M * 4) : 0);   // float32: a of the boundary
  static constexpr int oVt = oChi + a16(BC * (FB + PAD) * ES);
  static constexpr int oR = oVt + a16(DV * (BC + PAD) * ES);
  // u of the window: bf16 inputs as f16 [window row][d] (read transposed, rows
  // in crow order, then multiplied in mixed precision); float32 transposed
  // [d][window row]
  static constexpr int TPU = tr_pad<T, DV>();
  static constexpr int UBYTES = sizeof(T) == 2 ? WIN * (DV + TPU) * ES : DV * UST * ES;
  static constexpr int oUt = oR + a16(WIN * (D + PAD) * ES);
  static constexpr int oQ = oUt + a16(UBYTES);
  static constexpr int oRj = oQ + a16(BC * (D + PAD) * ES);
  // bf16: the block's slice of a as a 3-row B operand (hi, lo, zero), permuted
  static constexpr int oAz = oRj + a16(BC * 4);
  static constexpr int BYTES = oAz + (sizeof(T) == 2 ? a16(3 * (FB + PAD) * ES) : 0);
};

template <typename T, int D, int DV, int M, int NW, int NA>
__global__ __launch_bounds__(64 * NW) void k_readout(FwdArgs a) {
  using F = MF<T>;
  using C = RCfg<T, D, DV, M, NW, NA>;
  constexpr int PAD = C::PAD, FB = C::FB, WIN = C::WIN, UST = C::UST, RPW = C::RPW;
  static_assert(C::BYTES <= 160 * 1024, "readout LDS budget");
  static_assert(64 * NW >= FB, "one thread per feature of the block");
  __shared__ __align__(16) char smem[C::BYTES];
  T* sOm = (T*)(smem + C::oOm);
  T* sMt = (T*)(smem + C::oMt);
  float* sA = (float*)(smem + C::oA);
  T* sChi = (T*)(smem + C::oChi);
  T* sVt = (T*)(smem + C::oVt);
  T* sR = (T*)(smem + C::oR);
  T* sUt = (T*)(smem + C::oUt);
  T* sQ = (T*)(smem + C::oQ);
  float* sRj = (float*)(smem + C::oRj);
  T* sAz = (T*)(smem + C::oAz);

  const int tid = threadIdx.x, l = tid & 63, col = l & 31, h = l >> 5, wv = uniform(tid >> 6);
  constexpr int NT = 64 * NW;
  const int2 gxy = xcd_grid_xy();
  const int cb = gxy.x, bh = gxy.y, hh = bh % a.H, n = a.n, nch = a.nch;
  const int s0 = cb * 32;
  const int wb = s0 - (32 * NA - 1);
  constexpr int S = M * DV + M;
  const size_t seq = (size_t)bh * n;
  const T* qs = (const T*)a.q + seq * D;
  const T* vs = (const T*)a.v + seq * DV;
  const T* rs_ = (const T*)a.r + seq * D;
  const T* us = (const T*)a.u + seq * DV;
  const T* omq_h = (const T*)a.omq + (size_t)hh * M * D;
  const float* bst = a.states + ((size_t)bh * nch + cb) * S;
  const float Rexb = a.rex[(size_t)bh * (nch + 1) + cb];
  const bool has_bnd = cb > 0;

  // ---- prologue ----
  const int fbk = blockIdx.z % C::NFB;
  {
    // every global load of the prologue first, then the LDS stores; the
    // transposed copies take the row index fastest across lanes, so the
    // 2-byte LDS writes of one instruction fall in one row
    using OmT = typename std::conditional<sizeof(T) == 2, f16, T>::type;
    StageRows<OmT, FB, D, NT> so;
    StageState<FB, DV, NT, true> sm;
    StageRowsT<T, FB, DV, NT> sm16;
    StageRowsT<T, 32, DV, NT> sv;
    StageRows<T, WIN, D, NT> sr;
    typename std::conditional<sizeof(T) == 2, StageRows<T, WIN, DV, NT>, StageRowsT<T, WIN, DV, NT>>::type su;
    StageRows<T, 32, D, NT> sq;
    StageRows<T, 32, FB, NT> sc;
    if constexpr (sizeof(T) == 2) so.load((const f16*)a.omh + ((size_t)hh * M + (size_t)fbk * FB) * D, D, 0, 0, FB, tid);
    else so.load(omq_h + (size_t)fbk * FB * D, D, 0, 0, FB, tid);
    if constexpr (sizeof(T) == 2) {
      if (has_bnd) sm16.load((const T*)a.states16 + (((size_t)bh * nch + cb) * M + (size_t)fbk * FB) * DV, DV, 0, 0, FB, tid);
    } else {
      if (has_bnd) sm.load(bst + (size_t)fbk * FB * DV, tid);
    }
    sv.load(vs, DV, s0, 0, n, tid);
    sr.load(rs_, D, wb, 0, n, tid);
    su.load(us, DV, wb, 0, n, tid);
    sq.load(qs, D, s0, 0, n, tid);
    sc.load((const T*)a.chi + seq * M + fbk * FB, M, s0, 0, n, tid);   // this block's features
    const float rjv = (tid < 32) ? a.rj[seq + min(s0 + tid, n - 1)] : 0.0f;
    const float azv = (sizeof(T) == 2 && has_bnd && tid < FB) ? bst[(size_t)M * DV + fbk * FB + tid] : 0.0f;
    float av[(M + NT - 1) / NT];
#pragma unroll
    for (int k = 0; k < (M + NT - 1) / NT; ++k) {
      const int p = tid + NT * k;
      av[k] = (sizeof(T) == 4 && has_bnd && p < M) ? bst[(size_t)M * DV + p] : 0.0f;
    }
    if constexpr (sizeof(T) == 2) so.store((f16*)sOm, D + PAD, 0, 0, FB, tid);
    else so.store(sOm, D + PAD, 0, 0, FB, tid);
    if constexpr (sizeof(T) == 2) {
      sm16.store(0, 0, FB, tid, [&](int p, int d0, const typename StageRowsT<T, FB, DV, NT>::V4& x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sMt[(d0 + e) * (FB + PAD) + F::sigma(p)] = has_bnd ? x[e] : (T)0.0f;
      });
    } else {
      sm.store(tid, [&](int p, int d0, const f32x4& x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sMt[(d0 + e) * (FB + PAD) + F::sigma(p)] = has_bnd ? (T)x[e] : (T)0.0f;
      });
    }
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int k = 0; k < (M + NT - 1) / NT; ++k)
        if (tid + NT * k < M) sA[tid + NT * k] = av[k];
    }
    sv.store(s0, 0, n, tid, [&](int jj, int d0, const typename StageRowsT<T, 32, DV, NT>::V4& x) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sVt[(d0 + e) * (32 + PAD) + F::sigma(jj)] = x[e];
    });
    if constexpr (sizeof(T) == 2) sr.store((f16*)sR, D + PAD, wb, 0, n, tid);
    else sr.store(sR, D + PAD, wb, 0, n, tid);
    if constexpr (sizeof(T) == 2) {
      su.store((f16*)sUt, DV + C::TPU, wb, 0, n, tid);      // f16: exact for bf16 in its range
    } else {
      su.store(wb, 0, n, tid, [&](int wi, int d0, const typename StageRowsT<T, WIN, DV, NT>::V4& x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sUt[(d0 + e) * UST + wi] = x[e];
      });
    }
    if constexpr (sizeof(T) == 2) sq.store((f16*)sQ, D + PAD, s0, 0, n, tid);
    else sq.store(sQ, D + PAD, s0, 0, n, tid);
    sc.store(sChi, FB + PAD, s0, 0, n, tid);
    if (tid < 32) sRj[tid] = (s0 + tid < n) ? rjv : 0.0f;
    if constexpr (sizeof(T) == 2) {
      if (tid < FB) {
        const T hi = (T)azv;
        const int ps = F::sigma(tid);
        sAz[ps] = hi;
        sAz[FB + PAD + ps] = (T)(azv - (float)hi);
        sAz[2 * (FB + PAD) + ps] = (T)0.0f;
      }
    }
  }
  __syncthreads();

  const int fb = fbk;              // feature block handled by this workgroup
  // the chunk's rows, by gridDim.z / NFB workgroups (more than one for small grids)
#pragma unroll 1
  for (int rr = blockIdx.z / C::NFB; rr < RPW; rr += gridDim.z / C::NFB) {
    const int t = wv + NW * rr;
    const int i = s0 + t;
    if (t >= C::BC || i >= n) continue;
    float nacc[DV / 32];
    float zacc = 0.0f, Lrun = kNegInf;
#pragma unroll
    for (int dt = 0; dt < DV / 32; ++dt) nacc[dt] = 0.0f;
    const float Ri = uniform(sRj[t]);
    const float sb = uniform(has_bnd ? fast_exp2(Rexb - Ri) : 0.0f);
    // frame ratios 2^(R_j - R_i) of the registers' rows j = crow(v, h), zero for
    // j > t: all sixteen read and formed, then selected (a load under the
    // condition would be a branch per register, each waiting for its read)
    float sj[16];
    const float* sRjh = sRj + 4 * h;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 r4 = *(const f32x4*)(sRjh + 8 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = fast_exp2(r4[e] - Ri);
        sj[4 * g + e] = (8 * g + 4 * h + e <= t) ? x : 0.0f;
      }
    }
    const T* qrow = sQ + t * (D + PAD);
#pragma unroll 1
    for (int an = 0; an < NA; ++an) {
      // keep the loop-invariant LDS operand reads inside the loop (hoisting
      // them all would exhaust the register file)
      no_hoist();
      const int c = i - 32 * an - col;
      const bool valid = (32 * an + col < a.w) && (c >= 0);
      const int wi = t + 32 * NA - 1 - 32 * an - col;
      const T* rrow = sR + wi * (D + PAD);
      // G1: log2 features of the composite queries, lanes <-> anchor, regs <-> p
      f32x16 accL[FB / 32];
      float nz;
      if constexpr (sizeof(T) == 2) {
        nz = logits_f16<D, FB, D + PAD>(accL, (const f16*)qrow, (const f16*)rrow, (const f16*)sOm);
      } else {
#pragma unroll
        for (int pt = 0; pt < FB / 32; ++pt) accL[pt] = zero16();
        nz = 0.0f;
#pragma unroll 2
        for (int s = 0; s < D / F::KS; ++s) {
          const int k0 = s * F::KS + h * F::KPL;
          const float p = F::ld(qrow, k0) * F::ld(rrow, k0);
          nz += p * p;
#pragma unroll
          for (int pt = 0; pt < FB / 32; ++pt)
            accL[pt] = F::mma(F::ld(sOm + (pt * 32 + col) * (D + PAD), k0), p, accL[pt]);
        }
        nz = half_swap_add(nz);
      }
      // invalid anchors: z is finite (zero-filled rows) and the bias removes them
      const float bias = valid ? -0.5f * kLog2e * nz : kNegInf;
      float tm = kNegInf;
#pragma unroll
      for (int pt = 0; pt < FB / 32; ++pt)
#pragma unroll
        for (int v = 0; v < 16; ++v) tm = fmaxf(tm, accL[pt][v]);
      tm = wave_max(valid ? tm + bias : kNegInf);
      const float Lnew = fmaxf(Lrun, tm);
      if (Lnew > Lrun) {
        const float sc = fast_exp2(Lrun - Lnew);
        zacc *= sc;
#pragma unroll
        for (int dt = 0; dt < DV / 32; ++dt) nacc[dt] *= sc;
        Lrun = Lnew;
      }
      const float off = bias - Lnew;
      float zc = 0.0f;
      // psi in place, boundary part of Z, then the operand-typed copy
      typename F::frag pf[FB / 32][F::CSTEPS];
      if constexpr (sizeof(T) == 2) {
        // bf16: the boundary part of Z (phi(z)^T a over the block's features)
        // is one more matrix product, of psi as rounded for the boundary
        // readout of N against the columns (a_hi, a_lo, 0, ...), a_hi + a_lo
        // being a to 16 significant bits; so N and Z see the same psi
#pragma unroll
        for (int pt = 0; pt < FB / 32; ++pt) {
#pragma unroll
          for (int v = 0; v < 16; ++v) accL[pt][v] = fast_exp2(accL[pt][v] + off);
#pragma unroll
          for (int sp = 0; sp < F::CSTEPS; ++sp) pf[pt][sp] = F::cfrag(accL[pt], sp);
        }
        f32x16 accZ = zero16();
        const T* zrow = sAz + min(col, 2) * (FB + PAD);
#pragma unroll
        for (int pt = 0; pt < FB / 32; ++pt)
#pragma unroll
          for (int sp = 0; sp < F::CSTEPS; ++sp)
            accZ = F::mma(pf[pt][sp], F::ldc(zrow, pt * 32, sp, h), accZ);
#pragma unroll
        for (int v = 0; v < 16; ++v) zc += accZ[v];
      } else {
        const float* sAh = sA + fb * FB + 4 * h;      // + pt*32 + 8*(v>>2) + (v&3)
#pragma unroll
        for (int pt = 0; pt < FB / 32; ++pt) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 av = *(const f32x4*)(sAh + pt * 32 + 8 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float psi = fast_exp2(accL[pt][4 * g + e] + off);
              accL[pt][4 * g + e] = psi;
              zc += psi * av[e];
            }
          }
#pragma unroll
          for (int sp = 0; sp < F::CSTEPS; ++sp) pf[pt][sp] = F::cfrag(accL[pt], sp);
        }
      }
      zc *= sb;
      // intra-chunk causal correction: P^T[j, anchor] = chi_j . psi_anchor, scaled
      // by the frame ratio 2^(R_j - R_i) and masked to j <= i
      f32x16 accP = zero16();
      const T* chirow = sChi + col * (FB + PAD);
#pragma unroll
      for (int pt = 0; pt < FB / 32; ++pt)
#pragma unroll
        for (int sp = 0; sp < F::CSTEPS; ++sp)
          accP = F::mma(F::ldc(chirow, pt * 32, sp, h), pf[pt][sp], accP);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        accP[v] *= sj[v];
        zc += accP[v];
      }
      typename F::frag ppf[F::CSTEPS];
#pragma unroll
      for (int sp = 0; sp < F::CSTEPS; ++sp) ppf[sp] = F::cfrag(accP, sp);
      // per 32-wide slice of d: boundary readout + correction, then the anchor
      // combine N += A_c (*) u_c  (lanes <-> d, regs <-> anchor)
      // (unrolled up to two slices; four would spill 47 of the 168 registers that
      // three waves per SIMD leave; float32 d = m = 64 spills 12 to 14 with two)
      constexpr int kUnroll = DV / 32 <= 2 ? DV / 32 : 1;
#pragma unroll kUnroll
      for (int dt = 0; dt < DV / 32; ++dt) {
        no_hoist();
        f32x16 accA = zero16();
        if (has_bnd) {
          const T* mrow = sMt + (dt * 32 + col) * (FB + PAD);
#pragma unroll
          for (int pt = 0; pt < FB / 32; ++pt)
#pragma unroll
            for (int sp = 0; sp < F::CSTEPS; ++sp)
              accA = F::mma(pf[pt][sp], F::ldc(mrow, pt * 32, sp, h), accA);
          if (sb != 1.0f) accA *= sb;
        }
        const T* vrow = sVt + (dt * 32 + col) * (32 + PAD);
#pragma unroll
        for (int sp = 0; sp < F::CSTEPS; ++sp) accA = F::mma(ppf[sp], F::ldc(vrow, 0, sp, h), accA);
        // anchor row index crow(v,h) = 8*(v>>2) + 4h + (v&3) -> window index falls with it
        float sacc = 0.0f, sacc1 = 0.0f;
        if constexpr (sizeof(T) == 2) {
          // u of the register's anchor at this lane's d: transposed reads of rows
          // t + 32 NA - 1 - 32 an - crow, in crow order
          auto rmap = [&](int ar) { return t + 32 * NA - 1 - 32 * an - ar; };
#pragma unroll
          for (int sp = 0; sp < F::CSTEPS; ++sp) {
            const f16x8 uf = __builtin_bit_cast(f16x8, F::tld_crow_map(sUt, DV + C::TPU, sp, dt * 32, rmap));
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              sacc = __builtin_fmaf(accA[8 * sp + e], (float)uf[e], sacc);
              sacc1 = __builtin_fmaf(accA[8 * sp + e + 1], (float)uf[e + 1], sacc1);
            }
          }
          sacc += sacc1;
        } else {
          const T* urow = sUt + (dt * 32 + col) * UST + (t + 32 * NA - 1 - 32 * an) - 4 * h;
#pragma unroll
          for (int v = 0; v < 16; ++v) sacc += accA[v] * tof(urow[-(8 * (v >> 2) + (v & 3))]);
        }
        // nacc[dt] += sacc with the slices rotated through nacc[0], so that the
        // register is fixed (an index by dt would be a chain of selects)
        const float x0 = nacc[0] + sacc;
#pragma unroll
        for (int i = 1; i < DV / 32; ++i) nacc[i - 1] = nacc[i];
        nacc[DV / 32 - 1] = x0;
      }
        zacc += zc;
    }
    // ---- row epilogue ----
    const float Z = wave_sum(zacc);
    if constexpr (C::NFB == 1) {
      const float inv = 1.0f / (Z + a.eps);
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt) {
        float N = half_swap_add(nacc[dt]);
        if (h == 0) ((T*)a.out)[(seq + i) * DV + dt * 32 + col] = (T)(N * inv);
      }
      if (l == 0 && a.stats != nullptr) {
        a.stats[(seq + i) * 2 + 0] = Lrun;
        a.stats[(seq + i) * 2 + 1] = Z;
      }
    } else {
      // partial (N, Z, L) of this feature block; merged by k_merge_blocks
      float* pr = a.part + (((size_t)fb * a.BH + bh) * n + i) * (DV + 2);
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt) {
        float N = half_swap_add(nacc[dt]);
        if (h == 0) pr[dt * 32 + col] = N;
      }
      if (l == 0) { pr[DV] = Z; pr[DV + 1] = Lrun; }
    }
  }
}

// Merge the per-feature-block partials (online-max combine of Alg. 1 across
// blocks):  L = max_b L_b,  N = sum_b 2^(L_b - L) N_b,  Z likewise.
template <typename T, int DV, int NFB>
__global__ __launch_bounds__(256) void k_merge_blocks(FwdArgs a) {
  const size_t rows = (size_t)a.BH * a.n;
  const size_t row = (size_t)blockIdx.x * (256 / 32) + (threadIdx.x >> 5);
  const int lane = threadIdx.x & 31;
  if (row >= rows) return;
  float L = kNegInf;
#pragma unroll
  for (int b = 0; b < NFB; ++b) L = fmaxf(L, a.part[((size_t)b * rows + row) * (DV + 2) + DV + 1]);
  float Z = 0.0f;
  float sc[NFB];
#pragma unroll
  for (int b = 0; b < NFB; ++b) {
    const float* pr = a.part + ((size_t)b * rows + row) * (DV + 2);
    sc[b] = fast_exp2(pr[DV + 1] - L);
    Z += sc[b] * pr[DV];
  }
  const float inv = 1.0f / (Z + a.eps);
  for (int d = lane; d < DV; d += 32) {
    float N = 0.0f;
#pragma unroll
    for (int b = 0; b < NFB; ++b) N += sc[b] * a.part[((size_t)b * rows + row) * (DV + 2) + d];
    ((T*)a.out)[row * DV + d] = (T)(N * inv);
  }
  if (lane == 0 && a.stats != nullptr) {
    a.stats[row * 2 + 0] = L;
    a.stats[row * 2 + 1] = Z;
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Segments of the bf16 scan: the count that minimises the estimated time of the
// scan (a chunk's step 0.6 us in each wave's chain, or its bytes at 4.5 TB/s)
// and, for more than one segment, of the totals before it (0.35 us a chunk, or
// the operands' bytes, the launch, the earlier segments' states), at most
// room + 1 of them.  4 x 8 heads x 2048 tokens, d = m = 64: 33 -> 20 us with
// both kernels; 2 x 8 x 3001, d = 128, m = 64: 48 -> 25.  Above 64 MB of
// operands and states, which the caches no longer hold, the chains of many
// segments only share the memory: 2 x 16 x 16384, d = m = 128, 0.36 ms whole
// and 0.47 in two; 8 x 6 x 2048, d = 64, m = 128 (88 MB), 35 us and 39.
static int scan_segments(int nch, int64_t room, int BH, int M, int DV) {
  const double frag = 64.0 * BH * nch * (M + DV), out = 2.0 * BH * nch * M * DV;
  if (frag + out > 64e6) return 1;
  int best = 1;
  double best_t = 1e300;
  for (int G = 1; G <= 32 && G <= room + 1 && G <= nch; ++G) {
    const int cps = (nch + G - 1) / G;
    if ((nch + cps - 1) / cps != G) continue;              // the last segment would be empty
    double t = fmax(cps * 0.6, (frag + out) / 4.5e6);
    if (G > 1) t += fmax(cps * 0.35, frag / 4.5e6) + 5.0 + 0.3 * G;
    if (t < best_t) { best_t = t; best = G; }
  }
  return best;
}

template <typename T, int D, int DV, int M, int NA>
static int run_fwd(const Shape& s, FwdArgs a, hipStream_t st) {
  // readout waves per workgroup: the workgroup's LDS fills a CU, so its wave
  // count sets the occupancy; 12 waves (three per SIMD, at most 168 registers
  // each) hide more of each row's dependent matrix-core / VALU chain than 8,
  // although four of them get two of the chunk's 32 rows instead of three
  constexpr int NW = 12;
  const int BH = (int)s.BH();
  const int nch = (int)s.nch();
  // (asked before the first launch: a failing query clears the last error)
  using R = RCfg<T, D, DV, M, NW, NA>;
  static const int64_t slots = kernel_slots(k_readout<T, D, DV, M, NW, NA>, 64 * NW);
  {
    int tot = (int)s.H * M * D;
    ProfScope ps("prep_omega", st);
    k_prep_omega<T><<<(tot + 255) / 256, 256, 0, st>>>(a.omega, (T*)a.omq, (T*)a.omk, (f16*)a.omh, (int)s.H, M * D, D);
  }
  { ProfScope ps("chunk_state", st);
  k_chunk_state<T, D, DV, M><<<dim3((nch + 3) / 4, BH), 256, 0, st>>>(a); }
  if constexpr (sizeof(T) == 2) {
    constexpr int NPD = (M / 32) * (DV / 32);
    const unsigned waves = (unsigned)((BH + 7) / 8 * 8 * NPD);
    // the segments' states use the space of chi, which k_keyfeat fills after the scan
    const int64_t room = (int64_t)s.n * M * (int)sizeof(T) / (4 * (M * DV + M + 1));
    a.G = scan_segments(nch, room, BH, M, DV);
    a.cps = (nch + a.G - 1) / a.G;
    a.seg_M = (float*)a.chi;
    a.seg_a = a.seg_M + (size_t)BH * (a.G - 1) * M * DV;
    a.seg_R = a.seg_a + (size_t)BH * (a.G - 1) * M;
    if (a.G > 1) {
      ProfScope ps("scan_totals", st);
      k_scan_totals<M, DV><<<waves * (a.G - 1), 64, 0, st>>>(a);
    }
    ProfScope ps("state_scan", st);
    k_state_scan_mma<M, DV><<<waves * a.G, 64, 0, st>>>(a);
  } else {
    constexpr int S = M * DV + M;
    ProfScope ps("state_scan", st);
    k_state_scan<M, DV><<<dim3((S / 4 + 255) / 256, BH), 256, 0, st>>>(a);
  }
  { ProfScope ps("keyfeat", st);
  k_keyfeat<T, D, M><<<dim3((nch + 3) / 4, BH), 256, 0, st>>>(a); }
  if (a.out != nullptr) {
    constexpr int NFB = R::NFB;
    // a grid that leaves CUs idle gives each round of a chunk's rows a workgroup
    // of its own (it stages the chunk's window again, beside the others): one
    // float32 head of 256 tokens, 8 chunks, 44 -> 21 us
    const int parts = (int64_t)nch * BH * NFB * R::RPW <= slots ? R::RPW : 1;
    { ProfScope ps("fwd_readout", st);
    k_readout<T, D, DV, M, NW, NA><<<dim3(nch, BH, NFB * parts), 64 * NW, 0, st>>>(a); }
    if constexpr (NFB > 1) {
      ProfScope ps("fwd_merge", st);
      size_t rows = (size_t)BH * s.n;
      k_merge_blocks<T, DV, NFB><<<(unsigned)((rows + 7) / 8), 256, 0, st>>>(a);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("forward launch failed: %s", hipGetErrorString(e));
    return -4;
  }
  return 0;
}

// Supported (dtype, D = Dv, m) combinations; w <= 64, and up to 128 where
// wide_window_ok allows it.
#define LS_FWD_CASES(X)               \
  X(bf16, 32, 32, 32)                 \
  X(bf16, 64, 64, 64)                 \
  X(bf16, 64, 64, 128)                \
  X(bf16, 128, 128, 64)               \
  X(bf16, 128, 128, 128)              \
  X(bf16, 128, 128, 256)              \
  X(float, 32, 32, 32)                \
  X(float, 32, 32, 64)                \
  X(float, 64, 64, 32)                \
  X(float, 64, 64, 64)

bool fwd_combo_supported(int dtype, int D, int Dv, int m) {
#define X(T, D_, DV_, M_) \
  if (dtype == (sizeof(T) == 2 ? 1 : 0) && D == D_ && Dv == DV_ && m == M_) return true;
  LS_FWD_CASES(X)
#undef X
  return false;
}

int launch_forward(const Shape& s, const void* q, const void* k, const void* v, const void* r,
                   const void* u, const float* omega, void* out, float* stats, const Workspace& ws,
                   hipStream_t st) {
  FwdArgs a;
  a.q = q; a.k = k; a.v = v; a.r = r; a.u = u; a.omega = omega;
  a.out = out; a.stats = stats;
  a.omq = ws.omq; a.omk = ws.omk; a.omh = ws.omh; a.states = ws.states; a.states16 = ws.states16; a.rho = ws.rho; a.rex = ws.rex;
  a.H = (int)s.H; a.n = (int)s.n; a.w = s.w; a.nch = (int)s.nch(); a.BH = (int)s.BH(); a.eps = s.eps;
  a.part = ws.part;
  a.chi = ws.chi; a.rj = ws.rj;
  const int NA = (s.w + 31) / 32;
#define X(T, D_, DV_, M_)                                                          \
  if (s.dtype == (sizeof(T) == 2 ? 1 : 0) && s.D == D_ && s.Dv == DV_ && s.m == M_) { \
    if (NA == 1) return run_fwd<T, D_, DV_, M_, 1>(s, a, st);                      \
    if (NA == 2) return run_fwd<T, D_, DV_, M_, 2>(s, a, st);                      \
    if constexpr (wide_window_ok(sizeof(T) == 2 ? 1 : 0, D_, M_, 3)) {              \
      if (NA == 3) return run_fwd<T, D_, DV_, M_, 3>(s, a, st);                    \
    }                                                                              \
    if constexpr (wide_window_ok(sizeof(T) == 2 ? 1 : 0, D_, M_, 4)) {              \
      if (NA == 4) return run_fwd<T, D_, DV_, M_, 4>(s, a, st);                    \
    }                                                                              \
  }
  LS_FWD_CASES(X)
#undef X
  set_error("unsupported shape (dtype=%d D=%d Dv=%d m=%d)", s.dtype, s.D, s.Dv, s.m);
  return -2;
}

}  // namespace linsimp
