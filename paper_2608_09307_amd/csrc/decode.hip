// LinSimp autoregressive decode on gfx950 (Theorem 1: the persistent state of a
// head is M, a and the last w anchor rows (r_c, u_c)).
//
// Per (sequence s, head h), token t = pos[s]:
//   lambda = log2-features of k_t;  R' = max(R, max_p lambda_p)
//   M <- 2^(R-R') M + chi v_t^T,  a <- 2^(R-R') a + chi,  chi = 2^(lambda - R')/sqrt(m)
//   (eq:Mstate / eq:astate in the frame R'; M_true = 2^R' M)
//   ring slot t mod w <- (r_t, u_t)
//   out = N / (Z + eps) over the min(t+1, w) most recent anchors (eq:Ni, eq:Zi)
// The readout uses the contraction order W = Psi^T U (matrix cores, sum over
// anchors), then N_d = sum_p M[p,d] W[p,d] fused with the state update, so
// every float32 state element is read once and written once.
#include <type_traits>

#include "common.h"
#include "linsimp_internal.h"
#include "prof.h"

namespace linsimp {

struct DecArgs {
  const void* q; const void* k; const void* v; const void* r; const void* u;
  const float* omega;
  float* M; float* a; float* rho;
  void* ring_r; void* ring_u;
  int64_t* pos;
  void* out;
  int H; int w; float eps;
};

// ---------------------------------------------------------------------------
// Decode: ntok tokens per sequence in one launch (token j of sequence s is
// position pos[s] + j), in blocks of TB: TB = 1 for the single step, whose
// token loop unrolls away, 8 otherwise; a token's arithmetic is the same in
// both, so T tokens in one call give the bits of T single steps.  One workgroup
// per (sequence, head), one wave per 32 features (with one feature tile, per
// group of its anchors); each wave keeps its rows of M and of the bank (float32)
// in registers, its entries of a, and a row shift L_w of its own (over its
// features only), so the waves walk the tokens of a block without meeting; the
// parts of N and Z are brought together, in order, once per block.
//
// The anchors r, u of the last 32 NA - 1 tokens and of the block's tokens sit in
// LDS, one row per token in a ring of E = 32 NA + TB rows: token i of the call
// (i < 0: before it) has row (i + 32 NA) mod E, and its anchor at offset dl the
// row of token i - dl; offsets past the window read the one row that is free
// in a block, kept zero (a -inf bias alone would let an inf or NaN of a token
// outside the window through).  Per block: lambda by float32 dot products (their
// maxima give every token's frame R) and the table of |z|^2.  Per token and wave:
// the state update, the logits L[c, p] = sum_d r_c[d] (q[d] Omega[p, d]) with
// q (*) Omega rounded once, psi = 2^(L - |z|^2 log2(e)/2 - L_w), W = Psi^T U on
// the matrix cores, N += M (*) W.
//
// Several tokens: bound by the per-token work of two waves per SIMD (about 620
// VALU instructions and 32 matrix products each).  A form that met at five
// barriers per token (key frame, row shift, sums), formed z = q (*) r in every
// wave and read the bank from L2 for each token took 161 us for 16 tokens of
// 32 sequences x 16 heads (d = m = 128, w = 64), this one 86.  A single step
// moves each state element once: 256 x 16 at d = m = 128 0.145 ms, 4.8 TB/s,
// the rate of a copy.
// ---------------------------------------------------------------------------
template <typename T, int D, int DV, int M, int NA, int TB>
struct DCfg {
  static constexpr int FT = M / 32;                              // feature tiles
  // Anchor groups.  N and Z are linear in the anchors, so in a workgroup of one
  // feature tile every group of anchor tiles gets a wave of its own, with its own
  // copy of the state and its own row shift; their parts are added with the other
  // waves'.  One wave alone ran a wide window's tiles in series and, in float32,
  // kept their logits in accumulation registers at one wave per SIMD: one step of
  // 16 heads, w = 128, float32 d = 64 22.0 -> 14.2 us, bf16 d = 32 9.2 -> 7.7;
  // 32 x 16, 16 tokens, float32 d = 64 480 -> 166.  (The copies of the state cost
  // more than the waves give only where a batch fills the chip: 64 x 16, 64
  // tokens, w = 96, bf16 164 -> 175, float32 d = 32 374 -> 410.)
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int AH = FT > 1 ? 1 : F32 ? (D * NA >= 96 ? NA : 1) : NA == 4 ? 2 : NA == 3 ? 3 : 1;
  static constexpr int WPE = AH > 1 && F32 && D == 32 ? 3 : 2;   // waves per SIMD
  static constexpr int NAW = NA / AH;                            // anchor tiles per wave
  static constexpr int NW = FT * AH, NT = 64 * NW;
  static constexpr int AW = 32 * NA, E = AW + TB;
  static constexpr int RST = D + MF<T>::PAD, UST = DV + tr_pad<T, DV>();
  static constexpr int ES = sizeof(T);
  static constexpr int a16(int x) { return (x + 15) & ~15; }
  static constexpr int oR = 0;                                   // r rows of the ring
  static constexpr int oU = oR + a16(E * RST * ES);              // u rows (read transposed)
  static constexpr int oQ = oU + a16(E * UST * ES);              // float32 q, k, v of the block
  static constexpr int oK = oQ + a16(TB * D * 4);
  static constexpr int oV = oK + a16(TB * D * 4);
  static constexpr int oNz = oV + a16(TB * DV * 4);              // [j][dl]: -|z|^2 log2(e)/2, -inf if not a pair
  static constexpr int oLam = oNz + a16(TB * AW * 4);            // [wave][j][32]: key log2-features
  static constexpr int oChi = oLam + a16(NW * TB * 32 * 4);      // per wave: chi of its features
  static constexpr int oN = oChi + a16(NW * 32 * 4);             // [wave][j][d]: N in the wave's row shift
  static constexpr int oZ = oN + a16(NW * TB * DV * 4);          // [wave][j]: Z, L_w, largest lambda
  static constexpr int BYTES = oZ + a16(3 * NW * TB * 4);
};

template <typename T, int D, int DV, int M, int NA, int TB>
__global__ __launch_bounds__((DCfg<T, D, DV, M, NA, TB>::NT), (DCfg<T, D, DV, M, NA, TB>::WPE)) void k_decode(DecArgs A, int ntok) {
  using F = MF<T>;
  using C = DCfg<T, D, DV, M, NA, TB>;
  constexpr int NW = C::NW, NT = C::NT, AW = C::AW, E = C::E, NS = D / F::KS;
  constexpr int FT = C::FT, AH = C::AH, NAW = C::NAW;
  const int NTOK = TB == 1 ? 1 : ntok;
  static_assert(C::BYTES <= 160 * 1024, "decode LDS budget");
  __shared__ __align__(16) char smem[C::BYTES];
  T* sR = (T*)(smem + C::oR);
  T* sU = (T*)(smem + C::oU);
  float* sq = (float*)(smem + C::oQ);
  float* sk = (float*)(smem + C::oK);
  float* sv = (float*)(smem + C::oV);
  float* sNz = (float*)(smem + C::oNz);
  float* sN = (float*)(smem + C::oN);
  float* sZ = (float*)(smem + C::oZ);

  const int tid = threadIdx.x, l = tid & 63, col = l & 31, h = l >> 5, wv = uniform(tid >> 6);
  const int wp = AH == 1 ? wv : wv % FT;                       // this wave's feature tile
  const int a0 = AH == 1 ? 0 : 32 * NAW * (wv / FT);           // first anchor offset of its group
  float* schi = (float*)(smem + C::oChi) + wv * 32;
  float* slam = (float*)(smem + C::oLam) + wv * TB * 32;
  const int sh = blockIdx.x, H = A.H, w = A.w;
  const int s = sh / H, hh = sh % H;
  const int64_t t0 = A.pos[s];
  const int told = (int)(t0 < AW ? t0 : AW);                   // tokens before the call that can be anchors
  const int slot0 = (int)(t0 % w);                             // ring slot of the call's first token
  T* rr = (T*)A.ring_r + (size_t)sh * w * D;
  T* ru = (T*)A.ring_u + (size_t)sh * w * DV;
  const size_t tok0 = (size_t)sh * NTOK;
  const T *rg = (const T*)A.r + tok0 * D, *ug = (const T*)A.u + tok0 * DV;
  float* Ms = A.M + (size_t)sh * M * DV;
  float* as = A.a + (size_t)sh * M;

  // LDS row of token i of the call, i >= -AW (i < 0: before the call)
  auto row_of = [](int i) { return (i + AW) % E; };
  constexpr int VE = 16 / (int)sizeof(T);
  typedef T V __attribute__((ext_vector_type(VE)));
  // a block's token rows: q, k, v as float32, r and u into the ring
  static_assert(D == DV, "rows of one width");
  constexpr int PD = D / VE, PT = 5 * PD, NP = TB * PT, PIT = (NP + NT - 1) / NT;
  // (thread numbers made opaque where a block or a token starts: the addresses
  // are formed there instead of being held in registers across the loops)
  auto opaque = [](int x, auto count) {
    constexpr int N = decltype(count)::value;
    asm volatile("" : "+v"(x));
    if constexpr ((N & (N - 1)) == 0) return x & (N - 1);      // (its range, which the compiler no longer knows)
    __builtin_assume(x >= 0 && x < N);
    return x;
  };
  constexpr std::integral_constant<int, NT> threads{};
  constexpr std::integral_constant<int, 64> lanes{};
  // one piece into an LDS row (float32 rows are padded by one element: not 16-byte aligned)
  auto put = [](T* dst, const V& x) {
    if constexpr (sizeof(T) == 2) *(V*)dst = x;
    else {
#pragma unroll
      for (int e = 0; e < VE; ++e) dst[e] = x[e];
    }
  };
  V xt[PIT];
  auto fetch = [&](int j0) {
    const int tid = opaque(threadIdx.x, threads);
#pragma unroll
    for (int it = 0; it < PIT; ++it) {
      const int idx = min(tid + NT * it, NP - 1), j = min(j0 + idx / PT, NTOK - 1), ti = idx % PT / PD, c = idx % PD;
      uintptr_t p = (uintptr_t)A.q;
      p = ti == 1 ? (uintptr_t)A.k : p;
      p = ti == 2 ? (uintptr_t)A.v : p;
      p = ti == 3 ? (uintptr_t)A.r : p;
      p = ti == 4 ? (uintptr_t)A.u : p;
      xt[it] = *(const V*)((const T*)p + (tok0 + j) * D + c * VE);
    }
  };
  auto place = [&](int j0) {
    const int tid = opaque(threadIdx.x, threads);
#pragma unroll
    for (int it = 0; it < PIT; ++it) {
      const int idx = tid + NT * it, jj = idx / PT, ti = idx % PT / PD, c = idx % PD;
      if (NP % NT != 0 && idx >= NP) continue;
      if (ti < 3) {
        float* dst = sq + (ti * TB + jj) * D + c * VE;         // q, k, v lie one after the other
#pragma unroll
        for (int e = 0; e < VE; ++e) dst[e] = tof(xt[it][e]);
      } else {
        const int row = row_of(j0 + jj);
        put((ti == 3 ? sR + row * C::RST : sU + row * C::UST) + c * VE, xt[it]);
      }
    }
    // the row no token of the block's windows has
    for (int e = tid; e < D; e += NT) sR[row_of(j0 - AW) * C::RST + e] = (T)0.0f;
    for (int e = tid; e < DV; e += NT) sU[row_of(j0 - AW) * C::UST + e] = (T)0.0f;
  };
  // The loads of the prologue in the order they are waited for: the first
  // block's tokens, the ring and the bank, staged, then the state, which arrives
  // under the key features and the logits (the memory counter drains in order).
  fetch(0);
  // ---- this wave's bank rows (Omega log2 e, lanes <-> p, the operand's pieces of D) ----
  float om[NS][F::KPL];
  {
    const float* orow = A.omega + ((size_t)hh * M + wp * 32 + col) * D + h * F::KPL;
#pragma unroll
    for (int ks = 0; ks < NS; ++ks)
#pragma unroll
      for (int e = 0; e < F::KPL; ++e) om[ks][e] = orow[ks * F::KS + e] * kLog2e;
  }
  // ---- anchors before the call: tokens -(AW - 1) .. -1 from the ring slots
  // (t0 + i) mod w, zero rows where the window or the sequence ends ----
  {
    constexpr int PR = D / VE, PW = PR + DV / VE, N = (AW - 1) * PW, IT = (N + NT - 1) / NT;
    V x[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int idx = min(tid + NT * it, N - 1), back = idx / PW + 1, c = idx % PW;
      const int slot = slot0 - min(back, w);                   // (rows past the window or the sequence: dropped below)
      const int sl = slot < 0 ? slot + w : slot;
      x[it] = *(const V*)(c < PR ? rr + (size_t)sl * D + c * VE : ru + (size_t)sl * DV + (c - PR) * VE);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int idx = tid + NT * it, back = idx / PW + 1, c = idx % PW;
      if (N % NT != 0 && idx >= N) continue;
      const bool ok = back < w && back <= told;
      const V zero = {};
      put(c < PR ? sR + row_of(-back) * C::RST + c * VE : sU + row_of(-back) * C::UST + (c - PR) * VE, ok ? x[it] : zero);
    }
    place(0);
  }
  // ---- this wave's rows of M and entries of a ----
  float Mreg[DV / 32][16];
#pragma unroll
  for (int dt = 0; dt < DV / 32; ++dt)
#pragma unroll
    for (int vv = 0; vv < 16; ++vv) Mreg[dt][vv] = Ms[(size_t)(wp * 32 + crow(vv, h)) * DV + dt * 32 + col];
  float areg = as[wp * 32 + col];
  float R = A.rho[sh];

#pragma unroll 1
  for (int j0 = 0; j0 < NTOK; j0 += TB) {
    const int nb = TB == 1 ? 1 : min(TB, NTOK - j0);
    __syncthreads();
    // ---- |z|^2 of the block's (token, anchor) pairs in float32: TPA threads an
    // anchor, each every TPA-th 16-byte piece of the row, their sums added in order ----
    {
      constexpr int TPA = NT >= AW ? (NT / AW >= 4 ? 4 : NT / AW >= 2 ? 2 : 1) : 1, APP = NT / TPA;
      const int tid = opaque(threadIdx.x, threads), part = tid % TPA;
#pragma unroll 1
      for (int idx = tid / TPA; idx < nb * AW; idx += APP) {
        const int j = idx / AW, dl = idx % AW, i = j0 + j;
        const int rrow = row_of(i) - dl;
        const T* rp = sR + (rrow < 0 ? rrow + E : rrow) * C::RST;
        const float* qp = sq + j * D;
        float x = 0.0f;
#pragma unroll
        for (int c = 0; c < D / VE / TPA; ++c) {
          const int e0 = (c * TPA + part) * VE;
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            const float z = qp[e0 + e] * tof(rp[e0 + e]);
            x = __builtin_fmaf(z, z, x);
          }
        }
        if constexpr (TPA >= 2) x += dpp<0xB1>(x);             // quad_perm [1,0,3,2]
        if constexpr (TPA >= 4) x += dpp<0x4E>(x);             // quad_perm [2,3,0,1]
        if (part == 0) sNz[idx] = dl < w && t0 + i - dl >= 0 ? -0.5f * kLog2e * x : kNegInf;
      }
    }
    // ---- key log2-features of the block's tokens (float32) and their maxima ----
#pragma unroll 1
    for (int j = 0; j < nb; ++j) {
      const int l = opaque(lane_id(), lanes), col = l & 31, h = l >> 5;
      const float* kr = sk + j * D;
      float nk = 0.0f, lam = 0.0f;
#pragma unroll
      for (int e = l; e < D; e += 64) nk = __builtin_fmaf(kr[e], kr[e], nk);
      nk = wave_sum(nk);
#pragma unroll
      for (int ks = 0; ks < NS; ++ks) {
        if (ks % (sizeof(T) == 4 ? 16 : 4) == 0) no_hoist();                         // a few reads in flight, not all of the row
#pragma unroll
        for (int e = 0; e < F::KPL; ++e) lam = __builtin_fmaf(om[ks][e], kr[ks * F::KS + h * F::KPL + e], lam);
      }
      lam = __builtin_fmaf(-0.5f * kLog2e, nk, half_swap_add(lam));
      const float mx = wave_max(lam);
      if (h == 0) slam[j * 32 + col] = lam;
      if (l == 0) sZ[3 * (wv * TB + j) + 2] = mx;
    }
    __syncthreads();

#pragma unroll 1
    for (int j = 0; j < nb; ++j) {
      const int l = opaque(lane_id(), lanes), col = l & 31, h = l >> 5;
      // ---- the frame, chi and a ----
      float Rn = R;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) Rn = fmaxf(Rn, sZ[3 * (ww * TB + j) + 2]);
      Rn = uniform(Rn);
      const float sa = uniform(fast_exp2(R - Rn));             // 0 for an empty state (R = -inf)
      const float chi = fast_exp2(slam[j * 32 + col] - Rn) * rsqrtf((float)M);
      areg = __builtin_fmaf(sa, areg, chi);
      R = Rn;
      if (h == 0) schi[col] = chi;
      if (sa != 1.0f) {
#pragma unroll
        for (int dt = 0; dt < DV / 32; ++dt)
#pragma unroll
          for (int vv = 0; vv < 16; ++vv) Mreg[dt][vv] *= sa;
      }
      // ---- logits (registers <-> anchor offset, lanes <-> p) ----
      const int ib = row_of(j0 + j);
      // row of the anchor at offset dl <= AW - 1 < E (one token: the rows past the window are zero already)
      auto ring_row = [&](int dl, bool last) {
        const int e = ib - dl;
        return TB > 1 && last && dl >= w ? row_of(j0 - AW) : e < 0 ? e + E : e;
      };
      const float* qr = sq + j * D;
      const T* arow[NAW];
#pragma unroll
      for (int an = 0; an < NAW; ++an) arow[an] = sR + ring_row(a0 + 32 * an + col, AH > 1 || an == NA - 1) * C::RST;
      f32x16 acc[NAW];
#pragma unroll
      for (int an = 0; an < NAW; ++an) acc[an] = zero16();
#pragma unroll
      for (int ks = 0; ks < NS; ++ks) {
        if (ks % (sizeof(T) == 4 ? 4 : 2) == 0) no_hoist();
        const int k0 = ks * F::KS + h * F::KPL;
        typename F::frag b;
        if constexpr (sizeof(T) == 2) {
          const f32x4 q0 = *(const f32x4*)(qr + k0), q1 = *(const f32x4*)(qr + k0 + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) b[e] = (bf16)(om[ks][e] * (e < 4 ? q0[e] : q1[e - 4]));
        } else {
          b = om[ks][0] * qr[k0];
        }
#pragma unroll
        for (int an = 0; an < NAW; ++an) acc[an] = F::mma(F::ld(arow[an], k0), b, acc[an]);
      }
      float tm = kNegInf;
#pragma unroll
      for (int an = 0; an < NAW; ++an) {
        float bias[16];
        crow_vals(sNz + j * AW + a0 + 32 * an, bias);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[an][v] += bias[v];
          tm = fmaxf(tm, acc[an][v]);
        }
      }
      const float L = wave_max(tm);
      const float Ls = AH > 1 && L == kNegInf ? 0.0f : L;      // (a group without an anchor yet: psi = 0)
      float ps = 0.0f;
      typename F::frag pf[NAW][F::CSTEPS];
#pragma unroll
      for (int an = 0; an < NAW; ++an) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[an][v] = fast_exp2(acc[an][v] - Ls);
          ps += acc[an][v];
        }
#pragma unroll
        for (int sp = 0; sp < F::CSTEPS; ++sp) pf[an][sp] = F::cfrag(acc[an], sp);
      }
      const float zw = wave_sum(ps * areg);
      // ---- W = Psi^T U, the state update and N = sum_p M (*) W (lanes <-> d, registers <-> p) ----
      wave_lds_sync();                                         // chi
      float cr[16];
      crow_vals(schi, cr);
      float* nrow = sN + (wv * TB + j) * DV;
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt) {
        no_hoist();
        f32x16 accW = zero16();
#pragma unroll
        for (int an = 0; an < NAW; ++an) {
          auto rmap = [&](int ar) { return ring_row(a0 + 32 * an + ar, AH > 1 || an == NA - 1); };
#pragma unroll
          for (int sp = 0; sp < F::CSTEPS; ++sp)
            accW = F::mma(pf[an][sp], F::tld_crow_map(sU, C::UST, sp, dt * 32, rmap), accW);
        }
        const float vd = sv[j * DV + dt * 32 + col];
        float np = 0.0f;
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) {
          Mreg[dt][vv] = __builtin_fmaf(cr[vv], vd, Mreg[dt][vv]);
          np = __builtin_fmaf(Mreg[dt][vv], accW[vv], np);
        }
        np = half_swap_add(np);
        if (h == 0) nrow[dt * 32 + col] = np;
      }
      if (l == 0) {
        float* z = sZ + 3 * (wv * TB + j);
        z[0] = zw;
        z[1] = L;
      }
    }
    const bool more = TB > 1 && j0 + TB < NTOK;
    if (more) fetch(j0 + TB);
    __syncthreads();
    if (more) place(j0 + TB);
    // ---- outputs: the waves' parts at the largest row shift ----
    for (int idx = tid; idx < nb * DV; idx += NT) {
      const int j = idx / DV, d = idx % DV;
      float Lm = kNegInf;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) Lm = fmaxf(Lm, sZ[3 * (ww * TB + j) + 1]);
      float Z = 0.0f, N = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float* z = sZ + 3 * (ww * TB + j);
        const float f = fast_exp2(z[1] - Lm);
        Z = __builtin_fmaf(z[0], f, Z);
        N = __builtin_fmaf(sN[(ww * TB + j) * DV + d], f, N);
      }
      ((T*)A.out)[(tok0 + j0 + j) * DV + d] = (T)(N / (Z + A.eps));
    }
  }

  // ---- state back ----
  if (AH == 1 || wv < FT) {
#pragma unroll
    for (int dt = 0; dt < DV / 32; ++dt)
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) Ms[(size_t)(wp * 32 + crow(vv, h)) * DV + dt * 32 + col] = Mreg[dt][vv];
    if (h == 0) as[wp * 32 + col] = areg;
  }
  if (tid == 0) A.rho[sh] = R;
  // the last min(NTOK, w) tokens into their ring slots
  {
    constexpr int PR = D / VE, PW = PR + DV / VE;
    const int jlo = NTOK > w ? NTOK - w : 0, total = (NTOK - jlo) * PW;
    for (int base = 0; base < total; base += 4 * NT) {
      V x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int idx = min(base + tid + NT * i, total - 1), j = jlo + idx / PW, c = idx % PW;
        x[i] = *(const V*)(c < PR ? rg + (size_t)j * D + c * VE : ug + (size_t)j * DV + (c - PR) * VE);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int idx = base + tid + NT * i, j = jlo + idx / PW, c = idx % PW;
        if (idx >= total) continue;
        const int slot = (slot0 + j) % w;
        *(V*)(c < PR ? rr + (size_t)slot * D + c * VE : ru + (size_t)slot * DV + (c - PR) * VE) = x[i];
      }
    }
  }
}

// pos[s] += step after every head of sequence s has read it
__global__ __launch_bounds__(256) void k_decode_advance(int64_t* pos, int64_t S, int step) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < S) pos[i] += step;
}

template <typename T, int D, int DV, int M, int NA>
static int run_decode(int64_t S, DecArgs a, int ntok, hipStream_t st) {
  // the caller bounds S*H by max_decode_groups (one workgroup each)
  static_assert(max_decode_groups(M) * DCfg<T, D, DV, M, NA, 8>::NT < ((int64_t)1 << 32), "decode grid");
  (void)hipGetLastError();                             // an earlier call's error is not this one's
  const unsigned groups = (unsigned)(S * a.H);
  if (ntok == 1) {
    ProfScope ps("decode", st);
    k_decode<T, D, DV, M, NA, 1><<<groups, DCfg<T, D, DV, M, NA, 1>::NT, 0, st>>>(a, ntok);
  } else {
    ProfScope ps("decode_chunk", st);
    k_decode<T, D, DV, M, NA, 8><<<groups, DCfg<T, D, DV, M, NA, 8>::NT, 0, st>>>(a, ntok);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {                               // pos must not advance past a step not taken
    set_error("decode launch failed: %s", hipGetErrorString(e));
    return -4;
  }
  k_decode_advance<<<(unsigned)((S + 255) / 256), 256, 0, st>>>(a.pos, S, ntok);
  e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("decode position update launch failed: %s", hipGetErrorString(e));
    return -4;
  }
  return 0;
}

#define LS_DEC_CASES(X)   \
  X(bf16, 32, 32, 32)     \
  X(bf16, 64, 64, 64)     \
  X(bf16, 64, 64, 128)    \
  X(bf16, 128, 128, 64)   \
  X(bf16, 128, 128, 128)  \
  X(bf16, 128, 128, 256)  \
  X(float, 32, 32, 32)    \
  X(float, 32, 32, 64)    \
  X(float, 64, 64, 32)    \
  X(float, 64, 64, 64)

int launch_decode(int64_t S, int H, int ntok, int D, int Dv, int m, int w, int dtype, float eps,
                  const void* q, const void* k, const void* v, const void* r, const void* u,
                  const float* omega, float* M, float* a, float* rho, void* ring_r, void* ring_u,
                  int64_t* pos, void* out, hipStream_t st) {
  DecArgs A;
  A.q = q; A.k = k; A.v = v; A.r = r; A.u = u; A.omega = omega;
  A.M = M; A.a = a; A.rho = rho; A.ring_r = ring_r; A.ring_u = ring_u; A.pos = pos; A.out = out;
  A.H = H; A.w = w; A.eps = eps;
  const int NA = (w + 31) / 32;
#define X(T, D_, DV_, M_)                                                              \
  if (dtype == (sizeof(T) == 2 ? 1 : 0) && D == D_ && Dv == DV_ && m == M_) {          \
    if (NA == 1) return run_decode<T, D_, DV_, M_, 1>(S, A, ntok, st);                 \
    if (NA == 2) return run_decode<T, D_, DV_, M_, 2>(S, A, ntok, st);                 \
    if constexpr (wide_window_ok(sizeof(T) == 2 ? 1 : 0, D_, M_, 3)) {                  \
      if (NA == 3) return run_decode<T, D_, DV_, M_, 3>(S, A, ntok, st);               \
    }                                                                                  \
    if constexpr (wide_window_ok(sizeof(T) == 2 ? 1 : 0, D_, M_, 4)) {                  \
      if (NA == 4) return run_decode<T, D_, DV_, M_, 4>(S, A, ntok, st);               \
    }                                                                                  \
  }
  LS_DEC_CASES(X)
#undef X
  set_error("decode: unsupported shape (dtype=%d D=%d Dv=%d m=%d)", dtype, D, Dv, m);
  return -2;
}

}  // namespace linsimp
