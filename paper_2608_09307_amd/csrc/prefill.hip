// Prefill of the decode state on gfx950 (Theorem 1): the prefix state after all
// n tokens of each (sequence, head), eq:Mstate / eq:astate summed over the whole
// prefix, and the ring of the last w anchor rows.
//
//   lambda_jp = log2(e) (omega_p . k_j - |k_j|^2 / 2),   R = max_{j, p} lambda_jp
//   M = sum_j 2^(lambda_j - R) v_j^T / sqrt(m),  a likewise,  rho = R
#include <type_traits>

#include "common.h"
#include "linsimp_internal.h"
#include "prof.h"

namespace linsimp {

struct PreArgs {
  const void *k, *v, *r, *u;
  const float* omega;
  float *M, *a, *rho;      // the state, written by the segment kernel (G = 1) or by the combine
  float *part, *prho;      // G > 1: [BH][G][m*DV + m] segment states, [BH][G] their frames
  void *ring_r, *ring_u;
  int64_t* pos;
  int BH, H, n, w, nch, G, cps;   // chunks in all, segments, chunks per segment
  bool rings;                     // rings copied by blocks of their own
};

// The ring of one (sequence, head): slot j mod w holds token j of the last
// min(n, w) tokens; the slots no token reaches (n < w) are zero.  16-byte
// pieces of the rows, every piece of a batch loaded (row index clamped) before
// the first is stored.
template <typename T, int D, int DV, int NT>
LS_DEV void copy_ring(const PreArgs& a, int bh) {
  constexpr int VE = 16 / (int)sizeof(T), NB = 8;
  typedef T V __attribute__((ext_vector_type(VE)));
  constexpr int pr = D / VE, pw = pr + DV / VE;
  const int n = a.n, w = a.w, total = w * pw, tid = threadIdx.x;
  const T *r = (const T*)a.r + (size_t)bh * n * D, *u = (const T*)a.u + (size_t)bh * n * DV;
  T *rr = (T*)a.ring_r + (size_t)bh * w * D, *ru = (T*)a.ring_u + (size_t)bh * w * DV;
  // the newest token j <= n - 1 with j mod w == slot (negative: none)
  auto token = [&](int slot) { return (n - 1) - (((n - 1 - slot) % w + w) % w); };
  for (int base = 0; base < total; base += NT * NB) {
    V x[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int idx = min(base + tid + NT * i, total - 1);
      const int slot = idx / pw, c = idx % pw;
      const size_t j = (size_t)max(token(slot), 0);
      x[i] = *(const V*)(c < pr ? r + j * D + c * VE : u + j * DV + (c - pr) * VE);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int idx = base + tid + NT * i;
      if (idx >= total) continue;
      const int slot = idx / pw, c = idx % pw;
      const bool ok = token(slot) >= 0;
      V y;
#pragma unroll
      for (int e = 0; e < VE; ++e) y[e] = ok ? x[i][e] : (T)0.0f;
      *(V*)(c < pr ? rr + (size_t)slot * D + c * VE : ru + (size_t)slot * DV + (c - pr) * VE) = y;
    }
  }
  if (tid == 0 && bh % a.H == 0) a.pos[bh / a.H] = n;
}

// ---------------------------------------------------------------------------
// State of one segment of the prefix (cps chunks of 32 tokens) of one
// (sequence, head).  Wave wv owns features 32 wv .. 32 wv + 31: its rows of M
// and a stay in registers over the whole segment, in a running frame of its
// own (the largest log2-feature of its tile so far), so the waves meet only at
// the one barrier per chunk that hands over the staged rows; the frames are
// brought together at the end.
//
// Per chunk: the key log2-features on the matrix cores (bf16: Omega log2 e as
// hi + lo, hi in registers and lo in LDS; -|k|^2 log2(e)/2 is one more k-step,
// three bf16 terms against ones, which also carries the -inf of tokens past
// n), the features, then M += chi^T V with V read transposed from LDS.  The
// rows are loaded three chunks ahead of their use and staged one ahead.
// Bound by the chunk's dependent chain at two waves per SIMD: 64 x 16 heads x
// 8192 tokens (d = m = 128) 1.40 -> 1.17 ms, 3.8 TB/s of rows, against the
// form with one frame for all waves (a second barrier per chunk), |k|^2 through
// LDS and V stored transposed.
// ---------------------------------------------------------------------------
template <typename T, int D, int DV, int M>
struct PfCfg {
  static constexpr int NW = M / 32, NT = 64 * NW;
  static constexpr int PAD = MF<T>::PAD;
  static constexpr int KST = D + PAD, VST = DV + tr_pad<T, DV>();
  static constexpr int ES = sizeof(T);
  static constexpr int a16(int x) { return (x + 15) & ~15; }
  static constexpr int oK = 0;                                   // two chunks of key rows
  static constexpr int oV = oK + 2 * a16(32 * KST * ES);         // two chunks of value rows
  static constexpr int oOl = oV + 2 * a16(32 * VST * ES);        // bf16: lo half of the bank [p][D]
  static constexpr int oMx = oOl + (ES == 2 ? a16(M * KST * ES) : 0);
  static constexpr int BYTES = oMx + a16(NW * 4);
};

LS_DEV float sq_add(const bf16x8& f, float acc) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const bf16x2 x = {f[e], f[e + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(x, x, acc, false);
  }
  return acc;
}
LS_DEV float sq_add(const float& f, float acc) { return __builtin_fmaf(f, f, acc); }

template <typename T, int D, int DV, int M>
LS_DEV void prefill_segment(const PreArgs& a, char* smem) {
  using F = MF<T>;
  using C = PfCfg<T, D, DV, M>;
  constexpr int NT = C::NT, NS = D / F::KS;
  constexpr int S = M * DV + M;
  float* smx = (float*)(smem + C::oMx);
  T* sOl = (T*)(smem + C::oOl);
  auto bufK = [&](int i) { return (T*)(smem + C::oK) + i * (C::a16(32 * C::KST * C::ES) / C::ES); };
  auto bufV = [&](int i) { return (T*)(smem + C::oV) + i * (C::a16(32 * C::VST * C::ES) / C::ES); };
  const int tid = threadIdx.x, l = tid & 63, col = l & 31, h = l >> 5, wv = uniform(tid >> 6);
  const int g = blockIdx.x, bh = blockIdx.y, hh = bh % a.H, n = a.n;
  const int cb0 = g * a.cps, ncb = min(a.cps, a.nch - cb0);     // (the host leaves no segment empty)
  const size_t seq = (size_t)bh * n;
  const T* ks = (const T*)a.k + seq * D;
  const T* vs = (const T*)a.v + seq * DV;

  StageRows<T, 32, D, NT> sk[2];
  StageRows<T, 32, DV, NT> sv[2];
  auto load = [&](int b, int i) {
    sk[i].load(ks, D, (cb0 + b) * 32, 0, n, tid);
    sv[i].load(vs, DV, (cb0 + b) * 32, 0, n, tid);
  };
  auto stage = [&](int b, int i) {
    sk[i].store(bufK(i), C::KST, (cb0 + b) * 32, 0, n, tid);
    sv[i].store(bufV(i), C::VST, (cb0 + b) * 32, 0, n, tid);
  };
  load(0, 0);
  load(1, 1);
  // this wave's tile of Omega log2 e as B operands (lanes <-> feature p), straight
  // from the caller's float32 bank
  typename F::frag oh[NS];
  {
    const float* orow = a.omega + ((size_t)hh * M + wv * 32 + col) * D + h * F::KPL;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (sizeof(T) == 2) {
        const f32x4 x0 = *(const f32x4*)(orow + s * F::KS), x1 = *(const f32x4*)(orow + s * F::KS + 4);
        typename F::frag lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = (e < 4 ? x0[e] : x1[e - 4]) * kLog2e;
          oh[s][e] = (bf16)x;
          lo[e] = (bf16)(x - (float)oh[s][e]);
        }
        *(typename F::frag*)(sOl + (wv * 32 + col) * C::KST + s * F::KS + h * F::KPL) = lo;   // read by this wave only
      } else {
        oh[s] = orow[s * F::KS] * kLog2e;
      }
    }
  }
  const T* olrow = sOl + (wv * 32 + col) * C::KST;
  f32x16 Macc[DV / 32];
#pragma unroll
  for (int dt = 0; dt < DV / 32; ++dt) Macc[dt] = zero16();
  float apart = 0.0f;                          // sum over this lane's tokens of chi_p, p = 32 wv + col
  float R = kNegInf;
  stage(0, 0);
  load(2, 0);

  auto chunk = [&](int b, auto cur_c) {
    constexpr int cur = decltype(cur_c)::value;
    __syncthreads();                           // chunk b is staged; the other buffer is free
    if (b + 1 < ncb) stage(b + 1, cur ^ 1);
    load(b + 3, cur ^ 1);
    const T* krow = bufK(cur) + col * C::KST;
    // two accumulation chains; registers <-> token crow(v, h), lanes <-> p
    f32x16 acc = zero16(), acc2 = zero16();
    float nk = 0.0f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const typename F::frag kf = F::ld(krow, s * F::KS + h * F::KPL);
      nk = sq_add(kf, nk);
      if constexpr (sizeof(T) == 2) {
        acc = F::mma(kf, oh[s], acc);
        acc2 = F::mma(kf, F::ld(olrow, s * F::KS + h * F::KPL), acc2);
      } else {
        if (s & 1) acc2 = F::mma(kf, oh[s], acc2);
        else acc = F::mma(kf, oh[s], acc);
      }
    }
    nk = half_swap_add(nk);                    // |k|^2 of token col
    const bool ok = (cb0 + b) * 32 + col < n;
    const float x = fmaxf(-0.5f * kLog2e * nk, -3e38f);   // (finite, so that the split below is)
    typename F::frag xf = F::zero(), one = F::zero();
    if constexpr (sizeof(T) == 2) {
      const bf16 x0 = (bf16)x;
      const float r1 = x - (float)x0;
      const bf16 x1 = (bf16)r1;
      if (h == 0) {
        xf[0] = ok ? x0 : (bf16)kNegInf;
        xf[1] = ok ? x1 : (bf16)0.0f;
        xf[2] = ok ? (bf16)(r1 - (float)x1) : (bf16)0.0f;
        one[0] = one[1] = one[2] = (bf16)1.0f;
      }
    } else {
      if (h == 0) { xf = ok ? x : kNegInf; one = 1.0f; }
    }
    acc2 = F::mma(xf, one, acc2);
    float mx = kNegInf;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[v] += acc2[v];
      mx = fmaxf(mx, acc[v]);
    }
    mx = wave_max(mx);
    if (mx > R) {
      const float sa = fast_exp2(R - mx);      // 0 while the state is empty
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt) Macc[dt] *= sa;
      apart *= sa;
      R = mx;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[v] = fast_exp2(acc[v] - R);
      apart += acc[v];
    }
#pragma unroll
    for (int sp = 0; sp < F::CSTEPS; ++sp)
#pragma unroll
      for (int dt = 0; dt < DV / 32; ++dt)
        Macc[dt] = F::mma(F::cfrag(acc, sp), F::tld_crow(bufV(cur), C::VST, 0, sp, dt * 32), Macc[dt]);
  };
#pragma unroll 1
  for (int b = 0; b < ncb; b += 2) {
    chunk(b, std::integral_constant<int, 0>{});
    if (b + 1 < ncb) chunk(b + 1, std::integral_constant<int, 1>{});
  }

  // one frame for the workgroup's features
  if (l == 0) smx[wv] = R;
  __syncthreads();
  float Rm = smx[0];
#pragma unroll
  for (int i = 1; i < C::NW; ++i) Rm = fmaxf(Rm, smx[i]);
  const float f = fast_exp2(R - Rm) * rsqrtf((float)M);
  const bool whole = a.G == 1;
  float* Mo = whole ? a.M + (size_t)bh * M * DV : a.part + ((size_t)bh * a.G + g) * S;
  float* ao = whole ? a.a + (size_t)bh * M : Mo + (size_t)M * DV;
  // M rows p = 32 wv + crow(v, h) (lanes <-> d), a[p], the frame
#pragma unroll
  for (int dt = 0; dt < DV / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) Mo[(size_t)(wv * 32 + crow(v, h)) * DV + dt * 32 + col] = Macc[dt][v] * f;
  const float at = half_swap_add(apart) * f;
  if (h == 0) ao[wv * 32 + col] = at;
  if (tid == 0) *(whole ? a.rho + bh : a.prho + (size_t)bh * a.G + g) = Rm;
}

template <typename T, int D, int DV, int M>
__global__ __launch_bounds__(64 * (M / 32)) __attribute__((amdgpu_waves_per_eu(2))) void k_prefill(PreArgs a) {
  using C = PfCfg<T, D, DV, M>;
  static_assert(C::BYTES <= 160 * 1024, "prefill LDS budget");
  __shared__ __align__(16) char smem[C::BYTES];
  // blockIdx.y: the states, then (one segment, idle CUs) the rings in blocks of their own
  const int y = blockIdx.y, ring = y - (a.rings ? a.BH : 0);
  if (y < a.BH) prefill_segment<T, D, DV, M>(a, smem);
  if (a.G == 1 && ring >= 0) copy_ring<T, D, DV, C::NT>(a, ring);
}

// The segments' states brought to the largest frame and added, in order; four
// elements per thread.  The last block of each (sequence, head) copies its ring.
template <typename T, int D, int DV, int M>
__global__ __launch_bounds__(256) void k_prefill_combine(PreArgs a) {
  constexpr int S = M * DV + M, NX = (S / 4 + 255) / 256;
  const int bh = blockIdx.y, G = a.G;
  if (blockIdx.x == NX) {
    copy_ring<T, D, DV, 256>(a, bh);
    return;
  }
  const int i4 = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 >= S) return;
  const float* pr = a.prho + (size_t)bh * G;
  const float* p = a.part + (size_t)bh * G * S + i4;
  float R = kNegInf;
  for (int g = 0; g < G; ++g) R = fmaxf(R, pr[g]);
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int g = 0; g < G; ++g) sum += *(const f32x4*)(p + (size_t)g * S) * fast_exp2(pr[g] - R);
  if (i4 < M * DV) *(f32x4*)(a.M + (size_t)bh * M * DV + i4) = sum;
  else *(f32x4*)(a.a + (size_t)bh * M + (i4 - M * DV)) = sum;
  if (i4 == 0) a.rho[bh] = R;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static int launch_status(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return 0;
  set_error("%s launch failed: %s", what, hipGetErrorString(e));
  return -4;
}

// Segments per (sequence, head): the count that minimises the time in units of
// one chunk's work (2.3 us at d = m = 128), `slots` workgroups running at once:
// rounds of workgroups times (chunks per segment + the prologue and the stores
// of a segment, about kEnds chunks), and for more than one segment the combine
// (its launch, and the partial states written and read again against the
// `chunk_kb` of a chunk's rows).  One workgroup per (sequence, head) leaves a
// short batch's chunks in series on a few CUs: 16 heads of one 16384-token
// prompt took 0.85 ms on 16 CUs, 0.054 ms as 32 segments each.
static int prefill_segments(int BH, int nch, int slots, double state_kb, double chunk_kb) {
  constexpr double kEnds = 4.0, kLaunch = 6.0;
  int best = 1;
  double best_t = 1e300;
  for (int G = 1; G <= 128 && G <= nch; ++G) {
    const int cps = (nch + G - 1) / G;
    if ((nch + cps - 1) / cps != G) continue;              // the last segment would be empty
    const double rounds = (double)(((int64_t)BH * G + slots - 1) / slots);
    double t = rounds * (cps + kEnds);
    if (G > 1) t += kLaunch + 2.0 * BH * G * state_kb / (slots * chunk_kb);
    if (t < best_t) { best_t = t; best = G; }
  }
  return best;
}

template <typename T, int D, int DV, int M>
static int run_prefill(const Shape& s, PreArgs a, hipStream_t st) {
  using C = PfCfg<T, D, DV, M>;
  constexpr int S = M * DV + M;
  const int BH = (int)s.BH();
  // workgroups at once: eight waves per CU (two per SIMD) where the LDS allows
  constexpr int kPerCu = 8 / C::NW < 160 * 1024 / C::BYTES ? 8 / C::NW : 160 * 1024 / C::BYTES;
  a.G = prefill_segments(BH, a.nch, 256 * kPerCu, S * 4 / 1024.0, 32 * (D + DV) * sizeof(T) / 1024.0);
  a.cps = (a.nch + a.G - 1) / a.G;
  a.BH = BH;
  // A workgroup of one segment copies its ring after the state, with as little as
  // one wave; beside idle CUs a second one copies it meanwhile (float32 d = 64,
  // m = 32: one head of 100 tokens 24.3 -> 16.7 us)
  a.rings = a.G == 1 && 2 * (int64_t)BH <= 256 * kPerCu;
  (void)hipGetLastError();
  {
    ProfScope ps("prefill_state", st);
    k_prefill<T, D, DV, M><<<dim3(a.G, a.rings ? 2 * BH : BH), C::NT, 0, st>>>(a);
  }
  if (int rc = launch_status("prefill")) return rc;
  if (a.G > 1) {
    ProfScope ps("prefill_combine", st);
    k_prefill_combine<T, D, DV, M><<<dim3((S / 4 + 255) / 256 + 1, BH), 256, 0, st>>>(a);
    return launch_status("prefill combine");
  }
  return 0;
}

int launch_prefill(const Shape& s, const void* k, const void* v, const void* r, const void* u,
                   const float* omega, float* M, float* A, float* rho, void* ring_r, void* ring_u,
                   int64_t* pos, const Workspace& ws, hipStream_t st) {
  PreArgs a;
  a.k = k; a.v = v; a.r = r; a.u = u; a.omega = omega;
  a.M = M; a.a = A; a.rho = rho;
  a.part = ws.states; a.prho = ws.rho;                   // [BH][nch][...]: at most nch segments
  a.ring_r = ring_r; a.ring_u = ring_u; a.pos = pos;
  a.H = (int)s.H; a.n = (int)s.n; a.w = s.w; a.nch = (int)s.nch(); a.G = 1; a.cps = a.nch;
#define X(T, D_, DV_, M_)                                                             \
  if (s.dtype == (sizeof(T) == 2 ? 1 : 0) && s.D == D_ && s.Dv == DV_ && s.m == M_)   \
    return run_prefill<T, D_, DV_, M_>(s, a, st);
  X(bf16, 32, 32, 32)
  X(bf16, 64, 64, 64)
  X(bf16, 64, 64, 128)
  X(bf16, 128, 128, 64)
  X(bf16, 128, 128, 128)
  X(bf16, 128, 128, 256)
  X(float, 32, 32, 32)
  X(float, 32, 32, 64)
  X(float, 64, 64, 32)
  X(float, 64, 64, 64)
#undef X
  set_error("prefill: unsupported shape (dtype=%d D=%d Dv=%d m=%d)", s.dtype, s.D, s.Dv, s.m);
  return -2;
}

}  // namespace linsimp
