// Kernels and launches of tridiag.hpp, included by eigh.hip.
// Eigenvectors of a batch of symmetric matrices through tridiagonal form:
// H = Q T Q^T by Householder reflections (FP32), the eigenvalues of T by
// bisection and its eigenvectors by twisted factorisation (both FP64, one
// thread per eigenpair), V = Q Z.
//
//   * k_tri_reduce: the columns before the last kTail ones, one workgroup per
//     matrix, blocked: a panel of NB columns is reduced with the trailing
//     matrix unchanged (each column takes one product of it with a vector,
//     corrected by the panel's own update held in LDS), then the trailing
//     matrix gets the panel's rank-2 NB update on MFMA.
//   * k_tri_tail: the last kTail columns, with the whole remaining matrix in
//     the registers of one workgroup.
//   * k_tri_vectors: bisection on Sturm counts, then the vector.
//   * k_tri_larft, k_tri_back: V = Q Z on MFMA, 32 columns of V per workgroup
//     held in registers, with compact-WY factors of 32 reflectors.
//
// A matrix is scaled by a power of two to max |h| in [1, 2).  T's diagonal
// gets a perturbation of at most 2^-26, different for every index: it
// separates eigenvalues that coincide (a split T, or eigenvalues that agree
// to FP64 rounding), whose vectors would otherwise come out the same, and is
// below the FP32 rounding of the reduction.
#pragma once
#include <algorithm>

#include "common.hpp"
#include "tridiag.hpp"

namespace {

constexpr int TS = 64;  // setup tile

SVDP_DEV f16v mfma2(float a, float b, f16v acc) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0); }

// orders the wave's own LDS traffic
SVDP_DEV void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// sums over the lanes of a wave by DPP moves (no LDS): rows of 16 lanes, then
// pairs of rows (lanes 31 and 63 hold their halves' sums), then lane 63
template <int CTRL, int ROWS>
SVDP_DEV float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, true));
}
SVDP_DEV float row16_sum(float v) {  // lane 15 of each row of 16
  v = dpp_add<0x111, 0xF>(v);
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  return dpp_add<0x118, 0xF>(v);
}
SVDP_DEV float half_sum(float v) { return dpp_add<0x142, 0xA>(row16_sum(v)); }
SVDP_DEV float wave_sum(float v) {  // in every lane
  v = dpp_add<0x143, 0xC>(half_sum(v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// 1 / x to an ulp: the hardware estimate and one Newton step (a reflector's
// chain; its x is neither tiny nor huge)
SVDP_DEV float rcp32(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, r, 1.f), r, r);
}

// The reflector I - tau v v^T with v = (1, x / (alpha - beta)) that takes
// (alpha, x) to (beta, 0); sig = |x|^2.  Below 1e-30 (entries of 1e-15 in a
// matrix scaled to 1) the squares lose their bits to underflow: x is dropped.
SVDP_DEV void reflector(float alpha, float sig, float& beta, float& tau, float& inv) {
  beta = alpha;
  tau = 0.f;
  inv = 0.f;
  if (sig > 1e-30f) {
    beta = -copysignf(sqrtf(alpha * alpha + sig), alpha);
    tau = (beta - alpha) * rcp32(beta);
    inv = rcp32(alpha - beta);
  }
}

// exact power of two near 1 / max |h| from the setup workgroups' maxima; 1 for
// a zero or non-finite matrix.  The same in every thread of the workgroup.
SVDP_DEV float tri_scale(const TriWs& t, int b) {
  const int cnt = (t.np / TS) * (t.np / TS), lane = threadIdx.x & 63;
  float m = 0.f;
  for (int i = lane; i < cnt; i += 64) m = fmaxf(m, t.mx[(int64_t)b * cnt + i]);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if (!(m > 0.f) || !isfinite(m)) return 1.f;
  return ldexpf(1.f, -min(max(ilogbf(m), -126), 126));
}

// A = sym(H), zero padded to np, both triangles, and max |h| per tile (a NaN
// is dropped).  One 64 x 64 tile per workgroup, its mirror through LDS.
__global__ __launch_bounds__(256) void k_tri_setup(TriWs t, const float* Hin, int64_t ldh, int64_t sH, int* sweeps,
                                                   const int* mask) {
  const int b = blockIdx.y;
  if (mask && !mask[b]) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sweeps[b] = 0;
    t.risk[b] = 0;
    t.bad[b] = 0;
  }
  __shared__ float Tb[TS][TS + 1];
  __shared__ float wmx[4];
  const int nq = t.np / TS;
  const int I = blockIdx.x / nq, J = blockIdx.x - I * nq;
  const float* Hb = Hin + b * sH;
  const int tid = threadIdx.x, c = tid & 63, r0 = tid >> 6;
  for (int r = r0; r < TS; r += 4) {
    const int i = TS * J + r, j = TS * I + c;
    Tb[r][c] = (i < t.n && j < t.n) ? Hb[(int64_t)i * ldh + j] : 0.f;
  }
  __syncthreads();
  float* A = t.A + (int64_t)b * t.np * t.np;
  float mx = 0.f;
  for (int r = r0; r < TS; r += 4) {
    const int i = TS * I + r, j = TS * J + c;
    const float h = (i < t.n && j < t.n) ? Hb[(int64_t)i * ldh + j] : 0.f;
    const float v = 0.5f * h + 0.5f * Tb[c][r];
    A[(int64_t)i * t.np + j] = v;
    mx = fmaxf(mx, fabsf(v));
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if ((tid & 63) == 0) wmx[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) t.mx[(int64_t)b * nq * nq + blockIdx.x] = fmaxf(fmaxf(wmx[0], wmx[1]), fmaxf(wmx[2], wmx[3]));
}

// Householder reduction of the first `cols` columns of one matrix, blocked;
// only A's upper triangle is read and updated.  Per column j (panel index i):
//   x = A[j, :] - sum_k (V_k W_k[j] + W_k V_k[j])     the panel's update of row j
//   v, tau, beta from x[j + 1:]                        reflector, T's entries
//   p = A v - V (W^T v) - W (V^T v)                    A streamed from memory
//   w = tau (p - tau (p^T v) / 2 v)
// and after the panel A -= V W^T + W V^T.  The stream of A bounds the kernel at
// large batches: an element a_rc above the diagonal is read once and used
// twice, p_c += a v_r in the lane's own columns and p_r += a v_c, summed over
// the wave's lanes by DPP, which halves it.  A wave takes whole rows, four at
// a time; a row's 256-column chunks left of the diagonal are skipped and only
// the chunk on it is masked.
template <int NMAX, int NB, int NT>
__global__ __launch_bounds__(NT) void k_tri_reduce(TriWs t, int cols, const int* mask) {
  constexpr int KS = NT / NMAX;  // threads per row in the panel passes
  constexpr int NW = NT / 64;
  constexpr int NC = NMAX / 256;  // 256-column chunks of a row: four columns a lane
  static_assert(KS >= 1 && NT % NMAX == 0, "a thread owns at most one row");
  const int b = blockIdx.x;
  if (mask && !mask[b]) return;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Vp = lds;                 // NB x NMAX
  float* Wp = Vp + NB * NMAX;      // NB x NMAX
  float* vv = Wp + NB * NMAX;      // NMAX
  float* part = vv + NMAX;         // NW x NMAX: each wave's column sums
  float* rp = part + NW * NMAX;    // NMAX: row sums
  float* dg = rp + NMAX;           // NMAX: A's diagonal
  float* red = dg + NMAX;          // 32
  float* gk = red + 32;            // NB: W_k . v
  float* hk = gk + NB;             // NB: V_k . v
  const int n = t.n;
  const int64_t ld = t.np;
  float* A = t.A + (int64_t)b * ld * ld;
  float* HV = t.HV + (int64_t)b * ld * ld;
  double* dd = t.d + (int64_t)b * ld;
  double* ee = t.e + (int64_t)b * ld;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r = tid % NMAX, ks = tid / NMAX;
  const float sc = tri_scale(t, b), isc = 1.f / sc;
  for (int i = tid; i < 2 * NB * NMAX; i += NT) lds[i] = 0.f;
  for (int j0 = 0; j0 < cols; j0 += NB) {
    const int nbk = min(NB, cols - j0);
    __syncthreads();
    if (tid < n) dg[tid] = A[(int64_t)tid * ld + tid];
    for (int i = 0; i < nbk; ++i) {
      const int j = j0 + i;
      // column j of the updated matrix
      float x = 0.f;
      if (r >= j && r < n) {
        if (ks == 0) x = sc * A[(int64_t)j * ld + r];
#pragma unroll 4
        for (int k = ks; k < i; k += KS) x -= Vp[k * NMAX + r] * Wp[k * NMAX + j] + Wp[k * NMAX + r] * Vp[k * NMAX + j];
      }
      if (KS > 1) {
        if (ks > 0) part[(ks - 1) * NMAX + r] = x;
        __syncthreads();
        if (ks == 0)
#pragma unroll
          for (int q = 0; q < KS - 1; ++q) x += part[q * NMAX + r];
      }
      // the reflector: sum of squares below the first entry
      if (ks == 0) {
        if (r == j) dd[j] = (double)x;
        if (r == j + 1) red[31] = x;
        const float sq = wave_sum(r > j + 1 ? x * x : 0.f);
        if (lane == 0) red[w] = sq;
      }
      __syncthreads();
      float sig = 0.f;
#pragma unroll
      for (int q = 0; q < NMAX / 64; ++q) sig += red[q];
      float beta, tau, inv;
      reflector(red[31], sig, beta, tau, inv);
      if (ks == 0) {
        const float v = r == j + 1 ? 1.f : (r > j + 1 ? x * inv : 0.f);
        vv[r] = v;
        Vp[i * NMAX + r] = v;
        if (r < ld) HV[(int64_t)j * ld + r] = v;
        if (r == j) {
          ee[j] = (double)beta;
          t.tau[(int64_t)b * ld + j] = tau;
        }
      }
      __syncthreads();
      // p = A v over rows and columns > j: the diagonal element is in both
      // sums and taken off below
      {
        f4v acc[NC], vc[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          acc[q] = f4v{0.f, 0.f, 0.f, 0.f};
          vc[q] = *(const f4v*)(vv + 256 * q + 4 * lane);
        }
        for (int rr = j + 1 + w; rr < n; rr += 4 * NW) {
          float s[4] = {0.f, 0.f, 0.f, 0.f};
          const int q0 = rr >> 8;  // chunks before it are left of all four rows' diagonals
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            if (q < q0) continue;
            f4v a[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              a[u] = *(const f4v*)(A + (int64_t)min(rr + u * NW, n - 1) * ld + 256 * q + 4 * lane);
            if (256 * q > rr + 3 * NW) {
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const float vr = rr + u * NW < n ? vv[rr + u * NW] : 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  acc[q][c] = fmaf(a[u][c], vr, acc[q][c]);
                  s[u] = fmaf(a[u][c], vc[q][c], s[u]);
                }
              }
            } else {
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const int ru = rr + u * NW;
                const float vr = ru < n ? vv[ru] : 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  const float up = 256 * q + 4 * lane + c >= ru ? a[u][c] : 0.f;
                  acc[q][c] = fmaf(up, vr, acc[q][c]);
                  s[u] = fmaf(up, vc[q][c], s[u]);
                }
              }
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float t4 = wave_sum(s[u]);
            if (lane == 0 && rr + u * NW < n) rp[rr + u * NW] = t4;
          }
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) *(f4v*)(part + w * NMAX + 256 * q + 4 * lane) = acc[q];
      }
      // the panel's dot products with v
      for (int k = w; k < 2 * i; k += NW) {
        const float* src = (k < i ? Wp + k * NMAX : Vp + (k - i) * NMAX);
        float s = 0.f;
        for (int c = (j + 1) / 64 * 64 + lane; c < NMAX; c += 64) s += src[c] * vv[c];
        s = wave_sum(s);
        if (lane == 0) (k < i ? gk[k] : hk[k - i]) = s;
      }
      __syncthreads();
      // p with the panel's correction
      float p = 0.f;
      if (r > j && r < n) {
#pragma unroll
        for (int k = 0; k < NW; k += KS) p += part[(k + ks) * NMAX + r];
        if (ks == 0) p += rp[r] - dg[r] * vv[r];
        p *= sc;
#pragma unroll 4
        for (int k = ks; k < i; k += KS) p -= Vp[k * NMAX + r] * gk[k] + Wp[k * NMAX + r] * hk[k];
      }
      if (KS > 1) {
        __syncthreads();  // part has been read
        if (ks > 0) part[(ks - 1) * NMAX + r] = p;
        __syncthreads();
        if (ks == 0)
#pragma unroll
          for (int q = 0; q < KS - 1; ++q) p += part[q * NMAX + r];
      }
      const float vr = vv[r];
      if (ks == 0) {
        const float pv = wave_sum(p * vr);
        if (lane == 0) red[w] = pv;
      }
      __syncthreads();
      if (ks == 0) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NMAX / 64; ++q) s += red[q];
        Wp[i * NMAX + r] = tau * (p - 0.5f * tau * s * vr);
      }
      __syncthreads();
    }
    // trailing update, the 32 x 32 tiles on and above the diagonal; panel rows
    // beyond nbk are cleared
    for (int i = nbk; i < NB; ++i)
      for (int c = tid; c < NMAX; c += NT) Vp[i * NMAX + c] = Wp[i * NMAX + c] = 0.f;
    __syncthreads();
    const int s0 = (j0 + nbk) & ~31, nt = (n - s0 + 31) / 32;
    const int kh = lane >> 5, ic = lane & 31;
    for (int tile = w; tile < nt * (nt + 1) / 2; tile += NW) {
      int tr = 0, tc = tile;
      while (tc >= nt - tr) { tc -= nt - tr; ++tr; }
      tc += tr;
      const int rb = s0 + 32 * tr, cb = s0 + 32 * tc;
      float* At = A + (int64_t)rb * ld + cb + ic;
      f16v acc;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[4 * g + q] = sc * At[(int64_t)(8 * g + 4 * kh + q) * ld];
#pragma unroll 4
      for (int k = 0; k < NB; k += 2) {
        acc = mfma2(-Vp[(k + kh) * NMAX + rb + ic], Wp[(k + kh) * NMAX + cb + ic], acc);
        acc = mfma2(-Wp[(k + kh) * NMAX + rb + ic], Vp[(k + kh) * NMAX + cb + ic], acc);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) At[(int64_t)(8 * g + 4 * kh + q) * ld] = isc * acc[4 * g + q];
    }
    __syncthreads();
  }
}

// One column of the reduction spread over G workgroups per matrix, a launch per
// column: for few or large matrices, where k_tri_reduce leaves most of the chip
// idle.  Launch j ends column j - 1 and begins column j; every workgroup does
// the vector part for itself (4 columns a thread):
//   w = tau (p - tau (p^T v) / 2 v)              v, tau of column j - 1, p = A v
//   x = A[j, :] - w - w[j] v                     row j with that update
//   v', tau', beta' from x[j + 1:]
// and then its rows r > j: A[r, :] -= v[r] w + w[r] v, p'[r] = A[r, :] v', both
// triangles, so that p' needs no sum over workgroups.  A wave takes U rows of
// NCH chunks of 256 columns at a time; the first rows are loaded before the
// vector part, whose two workgroup sums hide their latency.  Launch js only
// updates.  p (by parity of j) and the scale are kept in T, which is free here.
// Latency and the launch bound it for few matrices (5.5 us a column of one
// 1024^2 matrix, where k_tri_reduce takes 23), the stream of A for more and for
// large ones (11.5 us on average at 4096^2: 50 MB read and written beyond the L2,
// 4.4 TB/s, where a large copy reaches 4.7).
template <int NT, int NCH>
__global__ __launch_bounds__(NT) void k_tri_column(TriWs t, int j, int js, int G, const int* mask) {
  constexpr int NW = NT / 64, U = 16 / NCH;
  const int L = blockIdx.x;
  int b, g;
  if (t.batch >= 8) {  // all of a matrix on one XCD
    const int q = L >> 3;
    b = q / G * 8 + (L & 7);
    g = q % G;
  } else {
    b = L / G;
    g = L - b * G;
  }
  if (b >= t.batch || (mask && !mask[b])) return;
  __shared__ __attribute__((aligned(16))) float sv[4 * NT], sw[4 * NT], sn[4 * NT];
  __shared__ float red[2][NW], alpha_s;
  const int n = t.n, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t ld = t.np;
  float* A = t.A + (int64_t)b * ld * ld;
  float* HV = t.HV + (int64_t)b * ld * ld;
  float* scr = t.T + (int64_t)b * ld * 32;
  const float* p0 = scr + (j & 1) * ld;   // p of column j - 1
  float* p1 = scr + (~j & 1) * ld;        // of column j
  const bool last = j == js;
  // the first rows of this wave
  const int rb = last ? j : j + 1, q0 = rb >> 8;
  int r0 = rb + (g * NW + w) * U;
  f4v a[U][NCH];
  const int q1 = (int)(ld >> 8);
  auto load_rows = [&] {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      if (q < q0 || q >= q1) continue;
#pragma unroll
      for (int u = 0; u < U; ++u)
        a[u][q] = *(const f4v*)(A + (int64_t)min(r0 + u, n - 1) * ld + 256 * q + 4 * lane);
    }
  };
  const int c = 4 * tid, cl = min(c, (int)ld - 4);
  f4v pv4 = *(const f4v*)(p0 + cl), vv4 = *(const f4v*)(HV + (int64_t)max(j - 1, 0) * ld + cl);
  const f4v aj = *(const f4v*)(A + (int64_t)j * ld + cl);
  float pj = p0[j], tau = t.tau[(int64_t)b * ld + max(j - 1, 0)];
  const float sc = j == 0 ? tri_scale(t, b) : scr[2 * ld];
  load_rows();
  if (j == 0) tau = pj = 0.f;
  float dot = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bool in = j > 0 && c + e >= j && c + e < n;
    pv4[e] = in ? pv4[e] : 0.f;
    vv4[e] = in ? vv4[e] : 0.f;
    dot = fmaf(pv4[e], vv4[e], dot);
  }
  dot = wave_sum(dot);
  if (lane == 0) red[0][w] = dot;
  __syncthreads();
  float h = 0.f;
#pragma unroll
  for (int q = 0; q < NW; ++q) h += red[0][q];
  h *= 0.5f * tau;
  const float wj = tau * (pj - h);  // v[j] = 1
  f4v x, ww;
  float sig = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ww[e] = tau * (pv4[e] - h * vv4[e]);
    x[e] = sc * aj[e] - (ww[e] + wj * vv4[e]);
    if (c + e == j + 1) alpha_s = x[e];
    sig += c + e > j + 1 && c + e < n ? x[e] * x[e] : 0.f;
  }
  sig = wave_sum(sig);
  if (lane == 0) red[1][w] = sig;
  __syncthreads();
  sig = 0.f;
#pragma unroll
  for (int q = 0; q < NW; ++q) sig += red[1][q];
  float beta, taun, inv;
  reflector(alpha_s, sig, beta, taun, inv);
  const float isc = 1.f / sc;
  f4v vn;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    vn[e] = c + e == j + 1 ? 1.f : (c + e > j + 1 && c + e < n ? x[e] * inv : 0.f);
    ww[e] *= isc;
  }
  *(f4v*)(sv + c) = vv4;
  *(f4v*)(sw + c) = ww;
  *(f4v*)(sn + c) = vn;
  if (g == 0 && !last) {
    if (c < ld) *(f4v*)(HV + (int64_t)j * ld + c) = vn;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e == j) t.d[(int64_t)b * ld + j] = (double)x[e];
    if (tid == 0) {
      t.e[(int64_t)b * ld + j] = (double)beta;
      t.tau[(int64_t)b * ld + j] = taun;
      scr[2 * ld] = sc;
    }
  }
  __syncthreads();
  for (;;) {
    float s[U], vr[U], wr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(r0 + u, n - 1);
      vr[u] = sv[r];
      wr[u] = sw[r];
      s[u] = 0.f;
    }
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      if (q < q0 || q >= q1) continue;
      const int o = 256 * q + 4 * lane;
      const f4v v = *(const f4v*)(sv + o), wc = *(const f4v*)(sw + o), nx = *(const f4v*)(sn + o);
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[u][q][e] -= fmaf(vr[u], wc[e], wr[u] * v[e]);
          s[u] = fmaf(a[u][q][e], nx[e], s[u]);
        }
        if (r0 + u < n) *(f4v*)(A + (int64_t)(r0 + u) * ld + o) = a[u][q];
      }
    }
    if (!last) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float d = wave_sum(s[u]);
        if (lane == 0 && r0 + u < n) p1[r0 + u] = sc * d;
      }
    }
    r0 += G * NW * U;
    if (r0 >= n) break;
    load_rows();
  }
}

// The last n - js <= 32 TC columns, the remaining matrix in registers: wave w
// holds the 32 columns 32 w .. of it as TC tiles in the MFMA accumulator
// layout (slot 4 g + q of lane (kh, ic): row 8 g + 4 kh + q, column ic).  By
// symmetry row j is column j: it sits in one slot of every wave, at the same
// place.  Per column (three barriers):
//   x = row j to LDS                            every wave its 32 values
//   |x|^2, v                                    the sum by every wave for itself
//   p = A v                                     column sums, in the lane
//   A -= v w^T + w v^T                          one 32x32x2 MFMA per tile
// Tiles of finished rows are skipped at compile time (S: rows below 32 S are
// done), waves of finished columns only keep the barriers.  Latency bounds it:
// 0.8 us per column at n = 256, where thread-per-element VALU code took 3.5.
template <int TC>
struct TailLds {
  float x[32 * TC], v[32 * TC], p[32 * TC], red[TC];
};
// slot `s` (uniform) of tile S of the wave's tiles
template <int TC, int S>
SVDP_DEV float tail_slot(const f16v (&A)[TC], int s) {
  float r = A[S][0];
#pragma unroll
  for (int q = 1; q < 16; ++q)
    if (s == q) r = A[S][q];
  return r;
}
template <int TC, int S>
SVDP_DEV void tail_cols(const TriWs& t, TailLds<TC>& L, f16v (&A)[TC], int b, int js, int nt, int w, int lane) {
  const int kh = lane >> 5, ic = lane & 31, c = 32 * w + ic;
  const int64_t ld = t.np;
  const bool live = w >= S;
  for (int j = 32 * S; j < min(32 * S + 32, nt - 1); ++j) {
    const int jr = j & 31, slot = 4 * (jr >> 3) + (jr & 3), kj = (jr >> 2) & 1;
    if (live) {
      const float x = tail_slot<TC, S>(A, slot);
      if (kh == kj) L.x[c] = x;
    }
    __syncthreads();
    float sq = 0.f;
#pragma unroll
    for (int q = (32 * S) / 64 * 64; q < 32 * TC; q += 64) {
      const int i = q + lane;
      const float xv = i < 32 * TC && i > j + 1 ? L.x[i] : 0.f;
      sq += xv * xv;
    }
    sq = wave_sum(sq);
    float beta, tau, inv;
    reflector(L.x[j + 1], sq, beta, tau, inv);
    const float vc = c > j + 1 ? L.x[c] * inv : (c == j + 1 ? 1.f : 0.f);
    if (kh == 0) L.v[c] = vc;
    if (w == TC - 1 && lane == 0) {
      t.d[(int64_t)b * ld + js + j] = (double)L.x[j];
      t.e[(int64_t)b * ld + js + j] = (double)beta;
      t.tau[(int64_t)b * ld + js + j] = tau;
    }
    float* hv = t.HV + (int64_t)b * ld * ld + (int64_t)(js + j) * ld;
    if (kh == 0 && js + c < ld) hv[js + c] = vc;
    __syncthreads();
    float pc = 0.f;
    if (live) {
      float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = S; x < TC; ++x)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f4v vr = *(const f4v*)&L.v[32 * x + 8 * g + 4 * kh];
#pragma unroll
          for (int q = 0; q < 4; ++q) ps[q] = fmaf(A[x][4 * g + q], vr[q], ps[q]);
        }
      float p = (ps[0] + ps[1]) + (ps[2] + ps[3]);
      p += __shfl_xor(p, 32);
      pc = p;
      if (kh == 0) L.p[c] = p;
    }
    const float pv = half_sum(pc * vc);  // lanes 31 and 63, the same
    if (lane == 31) L.red[w] = pv;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int q = S; q < TC; ++q) s += L.red[q];
    const float h = 0.5f * tau * s;
    if (live) {
      // MFMA operands: contraction index kh = 0: v_r w_c, kh = 1: w_r v_c
      const float wc = c > j ? tau * (pc - h * vc) : 0.f;
      const float bo = kh ? -vc : -wc;
#pragma unroll
      for (int x = S; x < TC; ++x) {
        const int r = 32 * x + ic;
        const float vr = L.v[r];
        const float wr = r > j ? tau * (L.p[r] - h * vr) : 0.f;
        A[x] = mfma2(kh ? wr : vr, bo, A[x]);
      }
    }
  }
  if constexpr (S + 1 < TC) tail_cols<TC, S + 1>(t, L, A, b, js, nt, w, lane);
}
template <int TC>
__global__ __launch_bounds__(64 * TC) void k_tri_tail(TriWs t, int js, const int* mask) {
  const int b = blockIdx.x;
  if (mask && !mask[b]) return;
  __shared__ __attribute__((aligned(16))) TailLds<TC> L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kh = lane >> 5, ic = lane & 31;
  const int nt = t.n - js;
  const int64_t ld = t.np;
  const float sc = tri_scale(t, b);
  const float* Ag = t.A + (int64_t)b * ld * ld + (int64_t)js * ld + js;
  for (int i = tid; i < 32 * TC; i += 64 * TC) L.x[i] = L.v[i] = L.p[i] = 0.f;
  f16v A[TC];
#pragma unroll
  for (int x = 0; x < TC; ++x)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // from the upper triangle (zero from row and column nt to np >= 32 TC)
        const int r = 32 * x + 8 * g + 4 * kh + q, c = 32 * w + ic;
        const int i = min(r, c), j = max(r, c);
        A[x][4 * g + q] = sc * Ag[(int64_t)i * ld + j];
      }
  // columns before js of the reflectors' rows
  float* hv = t.HV + (int64_t)b * ld * ld + (int64_t)js * ld;
  for (int i = w; i < nt; i += TC)
    for (int c = lane; c < js; c += 64) hv[(int64_t)i * ld + c] = 0.f;
  for (int i = w; i < nt; i += TC)
    for (int c = js + 32 * TC + lane; c < ld; c += 64) hv[(int64_t)i * ld + c] = 0.f;
  __syncthreads();
  tail_cols<TC, 0>(t, L, A, b, js, nt, w, lane);
  // the last diagonal entry
  const int jl = nt - 1, jr = jl & 31;
  if (w == jl >> 5 && ic == jr && kh == ((jr >> 2) & 1)) {
    float x = 0.f;
#pragma unroll
    for (int y = 0; y < TC; ++y)
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (y == jl >> 5 && q == 4 * (jr >> 3) + (jr & 3)) x = A[y][q];
    t.d[(int64_t)b * ld + js + jl] = (double)x;
  }
}

// Compact-WY factor of 32 reflectors, I - V T V^T: T_ii = tau_i and
// T[:i, i] = -tau_i T[:i, :i] (V^T v_i).  One panel per workgroup: V^T V on
// MFMA (one load feeds both operands), then the first wave forms T column by column
// in LDS, lane k its row k.
__global__ __launch_bounds__(256) void k_tri_larft(TriWs t, const int* mask) {
  const int b = blockIdx.y;
  if (mask && !mask[b]) return;
  __shared__ __attribute__((aligned(16))) float Gp[4][32][36];
  const int n = t.n, n32 = (n + 31) & ~31;
  const int64_t ld = t.np;
  const int j0 = blockIdx.x * 32, nbk = min(32, n - 1 - j0);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kh = lane >> 5, ic = lane & 31;
  const float* vrow = t.HV + (int64_t)b * ld * ld + (int64_t)(j0 + min(ic, nbk - 1)) * ld + 4 * kh;
  f16v acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  for (int r0 = ((j0 + 1) & ~31) + 8 * w; r0 < n32; r0 += 32) {
    const f4v a = *(const f4v*)(vrow + r0);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = mfma2(a[u], a[u], acc);
  }
  // stored transposed (the matrix is symmetric): row = second index
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *(f4v*)&Gp[w][ic][8 * g + 4 * kh] = f4v{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
  __syncthreads();
  for (int i = tid; i < 1024; i += 256) {
    const int r = i >> 5, c = i & 31;
    Gp[0][r][c] = (Gp[0][r][c] + Gp[1][r][c]) + (Gp[2][r][c] + Gp[3][r][c]);
  }
  __syncthreads();
  if (w != 0) return;
  // row k of T in lane k (and k + 32), in the space of the second partial sum
  float (*Tl)[36] = Gp[1];
  const float* tg = t.tau + (int64_t)b * ld + j0;
  const float tau = ic < nbk ? tg[ic] : 0.f;
  for (int i = 0; i < 32; ++i) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll 4
    for (int m = 0; m + 1 < i; m += 2) {
      s0 += Tl[ic][m] * Gp[0][i][m];
      s1 += Tl[ic][m + 1] * Gp[0][i][m + 1];
    }
    if (i & 1) s0 += Tl[ic][i - 1] * Gp[0][i][i - 1];
    const float ti = __shfl(tau, i);
    const float v = ic < i ? -ti * (s0 + s1) : (ic == i ? ti : 0.f);
    wave_fence();
    Tl[ic][i] = v;
    wave_fence();
  }
  float* Tg = t.T + (int64_t)b * ld * 32 + (int64_t)blockIdx.x * 1024;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *(f4v*)(Tg + ic * 32 + 16 * kh + 4 * g) = *(const f4v*)&Tl[ic][16 * kh + 4 * g];
}

SVDP_DEV double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
constexpr double kPivMin = 1e-30;  // T is scaled to entries of order 1
SVDP_DEV double pivot(double q) { return fabs(q) < kPivMin ? -kPivMin : q; }

// Eigenpair k of T (ascending) in one thread.
//   * Eigenvalue: number of sign changes of p_(i+1) = (d_i - x) p_i -
//     e_(i-1)^2 p_(i-1), a multiply-add recurrence rescaled every eight steps
//     (the quotient form has a division in its chain: 2.6 times the time).
//     |e| is at least 2^-100, so that p does not vanish where T splits.
//     Three shifts a pass, whose chains hide each other's latency: quarters
//     of the bracket until it holds one eigenvalue, then the regula falsi
//     point on p_n and a point on either side at 2^-s of the bracket, s doubled
//     after a hit; after a miss one pass of quarters.  To 2^-52 |lam|, at least
//     2^-60 of the spectrum's width.
//   * Vector: pivots D+ of T - lam = L D+ L^T from the top and D- from the
//     bottom, both chains at once; at the index r of the smallest |D+ + D- -
//     (d - lam)| the twisted factorisation is most nearly singular, and z_r = 1,
//     z_(i-1) = -e z_i / D+_(i-1) upwards, z_(i+1) = -e z_i / D-_(i+1)
//     downwards.  All lanes walk the same rows (each starts at its own r), so
//     that the loads are contiguous.
// Its FP64 chains bound the kernel (about 14 passes for the eigenvalues; one shift a
// pass took 30): at 256 x 512^2 with 1.3 waves a SIMD the VALU is busy 44% of the
// time, and 3.2 GB of pivots and vectors move at 2.0 TB/s.  256 x 512^2: 2.33 ->
// 1.34 ms, 64 x 256^2: 352 -> 290 us, 8 x 1024^2: 1.30 -> 1.07 ms, against one shift
// a pass, one chain of pivots at a time and a walk from each lane's own r.
// T lies in LDS; the pivots go to global scratch (64 threads of a block on
// consecutive addresses).
__global__ __launch_bounds__(64) void k_tri_vectors(TriWs t, const int* mask) {
  const int b = blockIdx.y;
  if (mask && !mask[b]) return;
  extern __shared__ __attribute__((aligned(16))) double de[];  // n8 + 1 pairs: d_i, e_(i-1)
  const int n = t.n, n8 = (n + 7) & ~7;
  const int64_t ld = t.np;
  const int lane = threadIdx.x;
  double lo = 1e300, hi = -1e300;
  for (int i = lane; i <= n8; i += 64) {
    double d = 8192.0, e0 = 0.0;  // padding: no sign change
    if (i < n) {
      const double h = (double)((i * 40503u) & 0xffffu) * (1.0 / 65536.0) - 0.5;
      d = t.d[(int64_t)b * ld + i] + h * 2.98023223876953125e-08;
      const double e1 = i + 1 < n ? t.e[(int64_t)b * ld + i] : 0.0;
      if (i > 0) {
        e0 = t.e[(int64_t)b * ld + i - 1];
        e0 = copysign(fmax(fabs(e0), 7.8886090522101181e-31), e0);
      }
      lo = fmin(lo, d - (fabs(e0) + fabs(e1)));
      hi = fmax(hi, d + (fabs(e0) + fabs(e1)));
    }
    de[2 * i] = d;
    de[2 * i + 1] = e0;
  }
  __syncthreads();
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off));
    hi = fmax(hi, __shfl_xor(hi, off));
  }
  // A spectrum further from zero than it is wide is moved to that distance:
  // eigenvalues, and with them the vectors, are resolved to 2^-52 |lam|, which has
  // to be small against the spectrum's width (the rule of `risk`), not its offset
  // (H near a multiple of I: max |V^T V - I| 1.5e-5 with the offset, 3e-11
  // without).  Nearer to zero, values near it would take passes of their own.
  const double wd = hi - lo, sh = lo > wd ? lo - wd : (hi < -wd ? hi + wd : 0.0);
  for (int i = lane; i < n; i += 64) de[2 * i] -= sh;
  __syncthreads();
  lo -= sh;
  hi -= sh;
  const double w0 = hi - lo;
  lo -= 1e-14 * w0 + 1e-20;
  hi += 1e-14 * w0 + 1e-20;
  const int k = blockIdx.x * 64 + lane;
  const int kk = min(k, n - 1);
  int clo = 0, chi = n, elo = 0, ehi = 0, narrow = 4;
  bool quarters = false;
  double flo = 0.0, fhi = 0.0;  // p_n at the ends (scaled by 2^elo, 2^ehi); 0: not known
  for (int it = 0; it < 96; ++it) {
    const double mid = 0.5 * (lo + hi), w = hi - lo;
    const double tol = fmax(2.220446049250313e-16 * fabs(mid), 8.6736173798840355e-19 * w0);
    const bool open = w > tol;
    if (!__any(open)) break;
    double x[3] = {lo + 0.25 * w, mid, lo + 0.75 * w};
    const bool falsi = chi - clo == 1 && flo != 0.0 && fhi != 0.0 && !quarters;
    if (falsi) {
      const double r = __builtin_amdgcn_ldexp(fabs(fhi) * __builtin_amdgcn_rcp(fabs(flo)), min(max(ehi - elo, -200), 200));
      const double side = fmax(__builtin_amdgcn_ldexp(w, -narrow), 0.5 * tol);
      x[1] = fmin(fmax(lo + w * __builtin_amdgcn_rcp(1.0 + r), lo + 0.5 * tol), hi - 0.5 * tol);
      x[0] = fmax(x[1] - side, lo);
      x[2] = fmin(x[1] + side, hi);
    }
    double p[3] = {1.0, 1.0, 1.0}, pp[3] = {0.0, 0.0, 0.0};
    int cnt[3] = {0, 0, 0};
    int ex[3] = {0, 0, 0};
    for (int i = 0; i < n8; i += 8) {
      // the signs of p before and after each of the eight steps, a bit each
      unsigned sg[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) sg[c] = (unsigned)__double2hiint(p[c]) >> 31;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double di = de[2 * (i + u)], ei = de[2 * (i + u) + 1];
        const double e2 = ei * ei;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double nx = fma(di - x[c], p[c], -(e2 * pp[c]));
          sg[c] = __builtin_amdgcn_alignbit(sg[c], (unsigned)__double2hiint(nx), 31);
          pp[c] = p[c];
          p[c] = nx;
        }
      }
      // scale by the power of two that takes the larger of |p|, |pp| to [1, 2)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        cnt[c] += __popc((sg[c] ^ (sg[c] >> 1)) & 0xffu);
        const int hx = max(__double2hiint(p[c]) & 0x7ff00000, __double2hiint(pp[c]) & 0x7ff00000);
        const double sc = __hiloint2double(0x7fe00000 - min(hx, 0x7fd00000), 0);
        p[c] *= sc;
        pp[c] *= sc;
        ex[c] += hx >> 20;
      }
    }
    if (!open) continue;
    const bool above0 = cnt[0] > kk, above1 = cnt[1] > kk, above2 = cnt[2] > kk;
    const bool hit = !above0 && above2;
    if (above0 || above1 || above2) {
      hi = above0 ? x[0] : (above1 ? x[1] : x[2]);
      chi = above0 ? cnt[0] : (above1 ? cnt[1] : cnt[2]);
      fhi = above0 ? p[0] : (above1 ? p[1] : p[2]);
      ehi = above0 ? ex[0] : (above1 ? ex[1] : ex[2]);
    }
    if (!above0) {
      lo = above1 ? x[0] : (above2 ? x[1] : x[2]);
      clo = above1 ? cnt[0] : (above2 ? cnt[1] : cnt[2]);
      flo = above1 ? p[0] : (above2 ? p[1] : p[2]);
      elo = above1 ? ex[0] : (above2 ? ex[1] : ex[2]);
    }
    if (falsi) narrow = hit ? min(2 * narrow, 48) : max(narrow / 2, 2);
    quarters = falsi && !hit;
  }
  // lanes beyond n repeat the last eigenpair (no store): all walk together
  const bool live = k < n;
  const double lam = 0.5 * (lo + hi);
  if (live) t.lam[(int64_t)b * ld + k] = lam;
  double* Dp = t.Z + (int64_t)b * ld * ld + k;   // k < ld: ld is a multiple of 64
  double* Dm = t.Zb + (int64_t)b * ld * ld + k;
  double qf = 0.0, qb = 0.0, best = INFINITY;
  int r = 0;
  // D+_i forwards and D-_j, j = n - 1 - i, backwards; from the middle on each
  // meets the pivot that the other one left there
  const int half = n / 2;
  auto pivots = [&](int i) {
    const int j = n - 1 - i;
    const double ef = de[2 * i + 1], eb = de[2 * j + 3];
    const double df = de[2 * i] - lam, db = de[2 * j] - lam;
    qf = pivot(i == 0 ? df : df - ef * ef * rcp64(qf));
    qb = pivot(i == 0 ? db : db - eb * eb * rcp64(qb));
    Dp[(int64_t)i * ld] = qf;
    Dm[(int64_t)j * ld] = qb;
  };
  auto take = [&](double g, int i) {
    const bool better = fabs(g) < best;
    best = better ? fabs(g) : best;
    r = better ? i : r;
  };
  for (int i = 0; i < half; ++i) pivots(i);
  if (n & 1) {
    pivots(half);
    take(qf + qb - (de[2 * half] - lam), half);
  }
  for (int i0 = n - half; i0 < n; i0 += 8) {
    double om[8], op[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = min(i0 + u, n - 1);
      om[u] = Dm[(int64_t)i * ld];
      op[u] = Dp[(int64_t)(n - 1 - i) * ld];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u, j = n - 1 - i;
      if (i < n) {
        pivots(i);
        take(qf + om[u] - (de[2 * i] - lam), i);
        take(qb + op[u] - (de[2 * j] - lam), j);
      }
    }
  }
  int rmin = r, rmax = r;
  for (int off = 32; off > 0; off >>= 1) {
    rmin = min(rmin, __shfl_xor(rmin, off));
    rmax = max(rmax, __shfl_xor(rmax, off));
  }
  double nz = 1.0, z = 1.0;
  for (int i0 = rmax - 1; i0 >= 0; i0 -= 8) {
    double dp[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) dp[u] = Dp[(int64_t)max(i0 - u, 0) * ld];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 - u;
      const double zn = z * (-de[2 * max(i, 0) + 3] * rcp64(dp[u]));
      if (i >= 0 && i < r) {
        z = zn;
        nz += z * z;
        Dp[(int64_t)i * ld] = z;
      }
    }
  }
  z = 1.0;
  Dp[(int64_t)r * ld] = 1.0;
  for (int i0 = rmin + 1; i0 < n; i0 += 8) {
    double dm[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) dm[u] = Dm[(int64_t)min(i0 + u, n - 1) * ld];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u;
      const double zn = z * (-de[2 * min(i, n - 1) + 1] * rcp64(dm[u]));
      if (i < n && i > r) {
        z = zn;
        nz += z * z;
        Dp[(int64_t)i * ld] = z;
      }
    }
  }
  if (live) t.zinv[(int64_t)b * ld + k] = 1.0 / sqrt(nz);
}

// V[:, slab] = Q Z[:, slab], 32 columns per workgroup of W waves, wave w
// holding the 32-row tiles w, w + W, ... of the slab in MFMA accumulators for
// the whole product.  Panel by panel from the last: C = V^T Z (each wave its
// rows; the partial sums meet in LDS and are added in order), then
// Z -= V (T C).  An accumulator's slot order is used as the contraction order
// of the products that read it, so Z, C and T C go from result to operand
// without leaving their lanes; a 32 x 32 tile of V is loaded once, row by row,
// and transposed through the wave's own LDS for the first product.
template <int W, int TPW>
__global__ __launch_bounds__(64 * W, TPW <= 2 ? 3 : 2) void k_tri_back(TriWs t, const int* mask) {
  const int n = t.n, slabs = (n + 31) / 32;
  // every slab of matrix b runs on XCD b % 8 and reads its reflectors from one L2
  const int qd = blockIdx.x >> 3, grp = qd / slabs, slab = qd - grp * slabs, b = 8 * grp + (blockIdx.x & 7);
  if (b >= t.batch) return;
  if (mask && !mask[b]) return;
  __shared__ float Cp[2][W][16][64];
  __shared__ __attribute__((aligned(16))) float Tr[W][32][36];
  const int64_t ld = t.np;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kh = lane >> 5, ic = lane & 31;
  const int c = slab * 32 + ic;
  // eigenvalues closer than 1e-8 of the spectrum: their FP64 vectors may be
  // short of orthogonal by more than FP32 rounding.  Up to kTriPolish every matrix
  // counts: its few reflections leave more than the Newton-Schulz step does
  if (slab == 0) {
    const double* lam = t.lam + (int64_t)b * ld;
    const double gap = 1e-8 * (lam[n - 1] - lam[0]);
    for (int i = tid; i < n; i += 64 * W)
      if (n <= kTriPolish || (i > 0 && !(lam[i] - lam[i - 1] > gap))) t.risk[b] = 1;
  }
  const double* Z = t.Z + (int64_t)b * ld * ld;
  const float* HV = t.HV + (int64_t)b * ld * ld;
  const double zs = c < n ? t.zinv[(int64_t)b * ld + c] : 0.0;
  f16v acc[TPW];
  // loads without conditions (a branch around each would serialise them): rows
  // from n on are read from row n - 1 and cleared
  const double* Zc = Z + min(c, n - 1);
#pragma unroll
  for (int x = 0; x < TPW; ++x)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double z[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = 32 * (w + W * x) + 16 * h + 8 * (q >> 2) + 4 * kh + (q & 3);
        z[q] = Zc[(int64_t)min(r, n - 1) * ld];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = 32 * (w + W * x) + 16 * h + 8 * (q >> 2) + 4 * kh + (q & 3);
        acc[x][8 * h + q] = r < n ? (float)(z[q] * zs) : 0.f;
      }
    }
  const int np = (n - 1 + 31) / 32;
  for (int pn = np - 1; pn >= 0; --pn) {
    const int j0 = 32 * pn, nbk = min(32, n - 1 - j0);
    // row tiles below pn are zero in every reflector of the panel
    f16v C;
#pragma unroll
    for (int q = 0; q < 16; ++q) C[q] = 0.f;
    float a[TPW][16];  // row 32 tile + ic of reflectors 8 g + 4 kh + q
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
      const int tile = w + W * x;
      if (tile < pn || 32 * tile >= n) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = 8 * g + 4 * kh + q;
          a[x][4 * g + q] = HV[(int64_t)(j0 + min(k, nbk - 1)) * ld + 32 * tile + ic];
        }
    }
    if (nbk < 32) {  // the first panel applied
#pragma unroll
      for (int x = 0; x < TPW; ++x)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (8 * (q >> 2) + 4 * kh + (q & 3) >= nbk) a[x][q] = 0.f;
    }
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
      const int tile = w + W * x;
      if (tile < pn || 32 * tile >= n) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) Tr[w][8 * g + 4 * kh + q][ic] = a[x][4 * g + q];
      wave_fence();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f4v at = *(const f4v*)&Tr[w][ic][8 * g + 4 * kh];
#pragma unroll
        for (int q = 0; q < 4; ++q) C = mfma2(at[q], acc[x][4 * g + q], C);
      }
      wave_fence();
    }
    float (*cp)[16][64] = Cp[pn & 1];
#pragma unroll
    for (int q = 0; q < 16; ++q) cp[w][q][lane] = C[q];
    const float* Tg = t.T + (int64_t)b * ld * 32 + (int64_t)pn * 1024 + ic * 32 + 4 * kh;
    f4v tf[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) tf[g] = *(const f4v*)(Tg + 8 * g);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      float s = cp[0][q][lane];
#pragma unroll
      for (int u = 1; u < W; ++u) s += cp[u][q][lane];
      C[q] = s;
    }
    f16v TC;
#pragma unroll
    for (int q = 0; q < 16; ++q) TC[q] = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) TC = mfma2(tf[g][q], C[4 * g + q], TC);
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
      const int tile = w + W * x;
      if (tile < pn || 32 * tile >= n) continue;
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[x] = mfma2(-a[x][q], TC[q], acc[x]);
    }
  }
  float* V = t.V + (int64_t)b * ld * ld;
#pragma unroll
  for (int x = 0; x < TPW; ++x)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 32 * (w + W * x) + 8 * g + 4 * kh + q;
        if (r < n && c < n) V[(int64_t)r * ld + c] = acc[x][4 * g + q];
      }
}

// bad[b] = 1 where some |G - I| entry is above 1e-4: one Newton-Schulz step
// alone would leave more than FP32 rounding
__global__ __launch_bounds__(256) void k_tri_dev(TriWs t, const float* G, const int* mask) {
  const int b = blockIdx.y;
  if ((mask && !mask[b]) || !t.risk[b]) return;
  const float* Gb = G + (int64_t)b * t.np * t.np;
  float m = 0.f;
  for (int i = blockIdx.x; i < t.n; i += gridDim.x)
    for (int j = threadIdx.x; j < t.n; j += 256) m = fmaxf(m, fabsf(Gb[(int64_t)i * t.np + j] - (i == j ? 1.f : 0.f)));
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0 && m > 1e-4f && isfinite(m)) t.bad[b] = 1;
}

// The same two in one launch for matrices up to kTriPolish, with the Newton-Schulz
// step V2 = V (3 I - G) / 2 of all of them: one workgroup per matrix, V and G in LDS
// (pitch NP + 4), 16 x 16 x 4 products in the index order of k_cans_small.  The G of
// a matrix of bad goes to Gm, for tri_rescue; again: those alone, after it.  Bound by
// the loads of V and its barriers; as launches of their own, Gram matrix, test and
// step took the EVD of 1 x 64^2 from 193 to 205 us and of 512 x 128^2 from 613 to 683.
template <int NP>
__global__ __launch_bounds__(8 * NP) void k_tri_polish(TriWs t, float* Gm, float* V2, int again, const int* mask) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  static_assert(NP == 64 || NP == 128, "two waves for 16 rows");
  constexpr int LD = NP + 4, NT = 8 * NP, NW = NT / 64, T = NP / 16, TH = T / 2;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float *X = lds, *G = lds + NP * LD;
  __shared__ float red[NW];
  const int n = t.n, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, kq = lane >> 4;
  for (int b = blockIdx.x; b < t.batch; b += gridDim.x) {
    if ((mask && !mask[b]) || (again && !t.bad[b])) continue;
    const int64_t o = (int64_t)b * t.np * t.np;
    __syncthreads();  // the matrix before is done
#pragma unroll
    for (int q = 4 * tid; q < NP * NP; q += 4 * NT) {
      const int i = q / NP, j = q - i * NP;
      f4 v = *(const f4*)(t.V + o + (int64_t)min(i, n - 1) * t.np + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = i < n && j + e < n ? v[e] : 0.f;
      *(f4*)&X[i * LD + j] = v;
    }
    __syncthreads();
    float m = 0.f;
    for (int q = w; q < T * (T + 1) / 2; q += NW) {
      int ti = 0, r = q;
      while (r >= T - ti) { r -= T - ti; ++ti; }
      const int tj = ti + r;
      f4 acc = {0.f, 0.f, 0.f, 0.f};
      const float* p = X + 4 * kq * LD + li;
#pragma unroll
      for (int k0 = 0; k0 < NP; k0 += 16, p += 16 * LD)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(p[u * LD + 16 * ti], p[u * LD + 16 * tj], acc, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * ti + 4 * kq + e, j = 16 * tj + li;
        G[i * LD + j] = acc[e];
        G[j * LD + i] = acc[e];
        if (i < n && j < n) m = fmaxf(m, fabsf(acc[e] - (i == j ? 1.f : 0.f)));
      }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if (lane == 0) red[w] = m;
    __syncthreads();
    for (int q = 0; q < NW; ++q) m = fmaxf(m, red[q]);
    if (!again && m > 1e-4f && isfinite(m)) {
      if (tid == 0) t.bad[b] = 1;
      for (int q = tid; q < NP * NP; q += NT) {
        const int i = q / NP, j = q - i * NP;
        if (i < n && j < n) Gm[o + (int64_t)i * t.np + j] = G[i * LD + j];
      }
      continue;
    }
    // a wave: 16 rows, half of the columns
    const int s = w >> 1, c0 = (w & 1) * TH;
    f4 acc[TH];
#pragma unroll
    for (int c = 0; c < TH; ++c) acc[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int k0 = 0; k0 < NP; k0 += 16) {
      const f4 av = *(const f4*)&X[(16 * s + li) * LD + k0 + 4 * kq];
      f4 bv[TH];
#pragma unroll
      for (int c = 0; c < TH; ++c) bv[c] = *(const f4*)&G[(16 * (c0 + c) + li) * LD + k0 + 4 * kq];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < TH; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[c][u], acc[c], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < TH; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * s + 4 * kq + e, j = 16 * (c0 + c) + li;
        if (i < n && j < n) V2[o + (int64_t)i * t.np + j] = 1.5f * X[i * LD + j] - 0.5f * acc[c][e];
      }
  }
}

// lam_k = v_k^T (H v_k) / v_k^T v_k, Y = H V, summed in FP64 (the norm of an FP32
// vector is off by as much as the quotient otherwise): a wave takes every blockDim /
// 64-th row of 64 columns.  Bound by reading V and Y once (256 x 512^2: 104 us,
// where the full product V^T Y took 500; 4096^2: 42 for 772, and its FP32 sums of
// one sign were the largest error of the eigenvalues there).
__global__ __launch_bounds__(1024) void k_tri_rayleigh(TriWs t, const float* V2, const float* Y, float* lam,
                                                       const int* mask) {
  const int b = blockIdx.y;
  if (mask && !mask[b]) return;
  __shared__ double part[2][16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int c = blockIdx.x * 64 + lane;  // c < np: a multiple of 64
  const int64_t o = (int64_t)b * t.np * t.np + c;
  const float* v = (t.risk[b] ? V2 : t.V) + o;
  double s = 0.0, vv = 0.0;
#pragma unroll 8
  for (int r = w; r < t.n; r += nw) {
    const double x = (double)v[(int64_t)r * t.np];
    s = fma(x, (double)Y[o + (int64_t)r * t.np], s);
    vv = fma(x, x, vv);
  }
  part[0][w][lane] = s;
  part[1][w][lane] = vv;
  __syncthreads();
  if (w == 0 && c < t.n) {
    for (int q = 1; q < nw; ++q) {
      s += part[0][q][lane];
      vv += part[1][q][lane];
    }
    lam[(int64_t)b * t.n + c] = (float)(vv > 0.0 ? s / vv : s);
  }
}

// ---- back-transformation above kTriSlab: 128 reflectors at a time, products of
// gemm_launch (one 4096^2 matrix: 32 pairs of products)

// V = Z / |z| in FP32, zero beyond n, and the risk of close eigenvalues as in
// k_tri_back; the rows of HV that hold no reflector are cleared.
__global__ __launch_bounds__(256) void k_tri_unscaled(TriWs t, const int* mask) {
  const int b = blockIdx.z;
  if (mask && !mask[b]) return;
  const int n = t.n, c = blockIdx.x * 256 + threadIdx.x;
  const int64_t ld = t.np, o = (int64_t)b * ld * ld;
  const double* lam = t.lam + (int64_t)b * ld;
  if (blockIdx.y == 0 && c > 0 && c < n && !(lam[c] - lam[c - 1] > 1e-8 * (lam[n - 1] - lam[0]))) t.risk[b] = 1;
  const double zs = c < n ? t.zinv[(int64_t)b * ld + c] : 0.0;
  for (int r = blockIdx.y; r < ld; r += gridDim.y) {
    const double z = t.Z[o + (int64_t)r * ld + c];
    t.V[o + (int64_t)r * ld + c] = r < n && c < n ? (float)(z * zs) : 0.f;
    if (r >= n - 1) t.HV[o + (int64_t)r * ld + c] = 0.f;
  }
}

// The 128 x 128 factor T of four panels from theirs and S = V^T V: for
// neighbours a, b the block above the diagonal is -T_a S_ab T_b; 32s to 64s, then
// 64s to 128.  One group per workgroup; the lower triangle of S holds S_ab T_b.
__global__ __launch_bounds__(256) void k_tri_merge(TriWs t) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* S = lds;              // 128 x 129
  float* T = lds + 128 * 129;  // 128 x 129
  const int groups = t.np / 128, b = blockIdx.x / groups, g = blockIdx.x - b * groups;
  const int tid = threadIdx.x;
  const float* Sg = t.S + (int64_t)blockIdx.x * 128 * 128;
  const float* Tp = t.T + (int64_t)b * t.np * 32 + (int64_t)g * 4 * 1024;
  const int panels = (t.n - 1 + 31) / 32;  // with reflectors
  for (int q = tid; q < 128 * 128; q += 256) {
    const int i = q >> 7, j = q & 127;
    S[i * 129 + j] = Sg[q];
    const float v = Tp[(i >> 5) * 1024 + (i & 31) * 32 + (j & 31)];
    T[i * 129 + j] = i >> 5 == j >> 5 && 4 * g + (i >> 5) < panels ? v : 0.f;
  }
  __syncthreads();
  for (int h = 32; h <= 64; h *= 2) {
    const int sh = h == 32 ? 5 : 6, cnt = 64 / h;  // pairs
    for (int q = tid; q < cnt << (2 * sh); q += 256) {
      const int p = q >> (2 * sh), i = (q >> sh) & (h - 1), j = q & (h - 1), a0 = 2 * h * p, b0 = a0 + h;
      float x = 0.f;
      for (int k = 0; k <= j; ++k) x += S[(a0 + i) * 129 + b0 + k] * T[(b0 + k) * 129 + b0 + j];
      S[(b0 + i) * 129 + a0 + j] = x;
    }
    __syncthreads();
    for (int q = tid; q < cnt << (2 * sh); q += 256) {
      const int p = q >> (2 * sh), i = (q >> sh) & (h - 1), j = q & (h - 1), a0 = 2 * h * p, b0 = a0 + h;
      float x = 0.f;
      for (int k = i; k < h; ++k) x += T[(a0 + i) * 129 + a0 + k] * S[(b0 + k) * 129 + a0 + j];
      T[(a0 + i) * 129 + b0 + j] = -x;
    }
    __syncthreads();
  }
  float* Tg = t.T4 + (int64_t)blockIdx.x * 128 * 128;
  for (int q = tid; q < 128 * 128; q += 256) Tg[q] = T[(q >> 7) * 129 + (q & 127)];
}

// Orthogonalises the columns of V whose entries of the Gram matrix G are above
// 3e-5 (eigenvalues that agree to 1e-11 or so of their size, where FP64 leaves
// eps |lam| / gap), one workgroup per matrix of bad; what is left is a
// Newton-Schulz step's.  Columns ascend by eigenvalue, so such columns are
// neighbours: a cluster is a run of columns bridged by large entries, and within
// it column j loses its components along the earlier ones, which mixes vectors
// of eigenvalues that differ by less than FP32 resolves.  A column that keeps less
// than 0.3 of itself (FP64 gave the same vector twice) is replaced in the end by a
// random one with the components along every other column taken off: those
// leave it the rest of the same eigenspace.  Latency bounds it: a pair takes a sum
// over the workgroup, a replacement three passes over V.  Above kTriSlab, more than
// 128 n pairs or 2^32 / n^2 replacements (seconds) end it: bad = 2, and the matrix
// is flagged when flags is given.
__global__ __launch_bounds__(1024) void k_tri_rescue(TriWs t, const float* G, int* flags, const int* mask) {
  const int b = blockIdx.x;
  if ((mask && !mask[b]) || !t.bad[b]) return;
  constexpr int PER = kTriMax / 1024;
  __shared__ int start[kTriMax];  // a row's first large entry, then its cluster's first column
  __shared__ unsigned char lost[kTriMax];
  __shared__ double part[2][16];
  extern __shared__ __attribute__((aligned(16))) double xy[];  // n and n
  const int n = t.n, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t ld = t.np;
  double *x = xy, *y = xy + n;
  float* V = t.V + (int64_t)b * ld * ld;
  const float* Gb = G + (int64_t)b * ld * ld;
  for (int j = w; j < n; j += 16) {
    int first = j;
    for (int i = lane; i < j; i += 64)
      if (fabsf(Gb[(int64_t)j * ld + i]) > 3e-5f) first = min(first, i);
    for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
    if (lane == 0) start[j] = first;
  }
  for (int j = tid; j < n; j += 1024) lost[j] = 0;
  __syncthreads();
  if (tid == 0) {
    // columns j - 1 and j are bridged if some row from j on reaches before j
    int reach = n;
    for (int j = n - 1; j >= 0; --j) {
      reach = min(reach, start[j]);
      start[j] = reach < j ? -1 : j;
    }
    for (int j = 1; j < n; ++j)
      if (start[j] < 0) start[j] = start[j - 1];
  }
  __syncthreads();
  int par = 0;
  auto total = [&](double x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    par ^= 1;
    if (lane == 0) part[par][w] = x;
    __syncthreads();
    x = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) x += part[par][q];
    return x;
  };
  double v[PER];
  // v loses its component along column i
  auto take_off = [&](int i) {
    double c[PER], s = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = tid + 1024 * u;
      c[u] = r < n ? (double)V[(int64_t)r * ld + i] : 0.0;
      s = fma(c[u], v[u], s);
    }
    s = total(s);
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = fma(-s, c[u], v[u]);
  };
  auto store = [&](int j, double scale) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = tid + 1024 * u;
      if (r < n) V[(int64_t)r * ld + j] = (float)(v[u] * scale);
    }
  };
  auto norm2 = [&] {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) s = fma(v[u], v[u], s);
    return total(s);
  };
  const bool bounded = n > kTriSlab;
  int64_t budget = bounded ? 128 * n : INT64_MAX;  // pairs
  int dropped = 0;
  for (int j = 1; j < n && budget > 0; ++j) {
    if (start[j] == j) continue;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = tid + 1024 * u;
      v[u] = r < n ? (double)V[(int64_t)r * ld + j] : 0.0;
    }
    for (int i = start[j]; i < j; ++i)
      if (!lost[i]) {
        take_off(i);
        --budget;
      }
    const double s = norm2();
    const bool drop = s < 0.09;
    store(j, drop ? 0.0 : 1.0 / sqrt(s));
    if (tid == 0) lost[j] = drop;
    dropped += drop;
    __syncthreads();
  }
  if (bounded && (int64_t)dropped * n * n > int64_t(1) << 32) budget = 0;
  for (int j = 1; dropped && j < n && budget > 0; ++j) {
    if (!lost[j]) continue;
    for (int r = tid; r < n; r += 1024) {
      unsigned h = (unsigned)(r * 4096 + j) * 2654435761u + 974711u;
      h = (h ^ (h >> 15)) * 2246822519u;
      h = (h ^ (h >> 13)) * 3266489917u;
      x[r] = (double)(int)(h ^ (h >> 16)) * (1.0 / 2147483648.0);
    }
    for (int pass = 0; pass < 3; ++pass) {  // x -= V (V^T x); lost columns are zero
      __syncthreads();
      for (int i = tid; i < n; i += 1024) {
        double s = 0.0;
#pragma unroll 8
        for (int r = 0; r < n; ++r) s = fma((double)V[(int64_t)r * ld + i], x[r], s);
        y[i] = s;
      }
      __syncthreads();
      for (int r = w; r < n; r += 16) {
        double s = 0.0;
        for (int i = lane; i < n; i += 64) s = fma((double)V[(int64_t)r * ld + i], y[i], s);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) x[r] -= s;
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = tid + 1024 * u;
      v[u] = r < n ? x[r] : 0.0;
    }
    const double s = norm2();
    store(j, 1.0 / sqrt(s));
    __syncthreads();
  }
  if (budget <= 0 && tid == 0) {
    t.bad[b] = 2;
    if (flags) atomicOr(flags + b, 32);  // SVDP_FLAG_EIGH_NOT_CONVERGED
  }
}

// columns left to k_tri_tail: as many as one workgroup's registers hold
constexpr int kTail = 256;

template <int NMAX, int NB, int NT>
hipError_t reduce_launch(const TriWs& t, int cols, const int* mask, hipStream_t st) {
  const size_t sh = (size_t)(2 * NB * NMAX + 3 * NMAX + NT / 64 * NMAX + 32 + 2 * NB) * 4;
  hipLaunchKernelGGL((k_tri_reduce<NMAX, NB, NT>), dim3(t.batch), dim3(NT), sh, st, t, cols, mask);
  return hipGetLastError();
}

template <int NT, int NCH>
hipError_t column_launch(const TriWs& t, int js, const int* mask, hipStream_t st) {
  constexpr int rows = NT / 64 * (16 / NCH);
  const int cap = std::max(1, 256 * 1024 / NT / t.batch);  // 16 waves a CU
  for (int j = 0; j <= js; ++j) {
    const int G = std::min(cap, cdiv(t.n - j, rows));
    const int grid = t.batch >= 8 ? cdiv(t.batch, 8) * 8 * G : t.batch * G;
    hipLaunchKernelGGL((k_tri_column<NT, NCH>), dim3(grid), dim3(NT), 0, st, t, j, js, G, mask);
    const hipError_t e = hipGetLastError();
    if (e) return e;
  }
  return hipSuccess;
}

}  // namespace

static int64_t tri_t_floats(int64_t np) { return np * 32; }  // 32 x 32 per 32 columns

// V = Q Z above kTriSlab: Z -= Y_g^T (P_g Z), group by group from the last (P_g
// the 128 reflectors as rows, zero in columns up to 128 g; Y_g = T_g^T P_g).
// The matrices outside a mask are computed with: their V is scratch.
static hipError_t tri_back_products(const TriWs& t, const int* mask, hipStream_t st) {
  const int np = t.np, n = t.n, groups = np / 128;
  const int64_t m2 = (int64_t)np * np, gs = 128 * 128;
  hipLaunchKernelGGL(k_tri_unscaled, dim3(np / 256, std::min(np, 256), t.batch), dim3(256), 0, st, t, mask);
  hipError_t e = hipGetLastError();
  if (e) return e;
  GemmArgs s = {};
  s.alpha = 1.f;
  s.M = s.N = 128; s.K = np; s.batch = t.batch * groups;
  s.A = s.B = t.HV; s.lda = s.ldb = np; s.sA = s.sB = (int64_t)128 * np;
  s.C = t.S; s.ldc = 128; s.sC = gs;
  if ((e = gemm_launch(s, PREC_F32, 0, 1, st))) return e;
  const size_t lds = 2 * 128 * 129 * sizeof(float);
  hipLaunchKernelGGL(k_tri_merge, dim3(t.batch * groups), dim3(256), lds, st, t);
  if ((e = hipGetLastError())) return e;
  GemmArgs y = {};
  y.alpha = 1.f;
  y.M = 128; y.N = np; y.K = 128; y.batch = t.batch * groups;
  y.A = t.T4; y.lda = 128; y.sA = gs;
  y.B = t.HV; y.ldb = np; y.sB = (int64_t)128 * np;
  y.C = t.Y; y.ldc = np; y.sC = (int64_t)128 * np;
  if ((e = gemm_launch(y, PREC_F32, 1, 0, st))) return e;
  for (int g = cdiv(n - 1, 128) - 1; g >= 0; --g) {
    const int64_t o = 128 * (int64_t)g;
    GemmArgs c = {};
    c.alpha = 1.f;
    c.M = 128; c.N = n; c.K = n - (int)o; c.batch = t.batch;
    c.A = t.HV + o * np + o; c.lda = np; c.sA = m2;
    c.B = t.V + o * np; c.ldb = np; c.sB = m2;
    c.C = t.C; c.ldc = np; c.sC = (int64_t)128 * np;
    if ((e = gemm_launch(c, PREC_F32, 0, 0, st))) return e;
    GemmArgs u = {};
    u.alpha = -1.f; u.beta = 1.f;
    u.M = n - (int)o; u.N = n; u.K = 128; u.batch = t.batch;
    u.A = t.Y + o * np + o; u.lda = np; u.sA = m2;
    u.B = t.C; u.ldb = np; u.sB = (int64_t)128 * np;
    u.C = t.V + o * np; u.ldc = np; u.sC = m2;
    u.Cin = t.V + o * np; u.ldcin = np; u.sCin = m2;
    if ((e = gemm_launch(u, PREC_F32, 1, 0, st))) return e;
  }
  return hipSuccess;
}

static hipError_t tri_eig(const TriWs& t, const float* H, int64_t ldh, int64_t sH, const int* mask, int* sweeps,
                   hipStream_t st) {
  hipError_t e;
  const int nq = t.np / TS;
  hipLaunchKernelGGL(k_tri_setup, dim3(nq * nq, t.batch), dim3(256), 0, st, t, H, ldh, sH, sweeps, mask);
  if ((e = hipGetLastError())) return e;
  const int js = std::max(0, t.n - kTail), nt = t.n - js;
  // panels of V and W in LDS: 2 NB n floats
  if (js > 0) {
    // A launch per column streams A's square twice a column, k_tri_reduce its
    // triangle once.  EVD in ms, columns / k_tri_reduce: 1 x 512^2 2.7 / 4.2,
    // 32 x 512^2 3.7 / 4.6, 64 x 512^2 6.3 / 5.5; 8 x 1024^2 8.0 / 20.1,
    // 32 x 1024^2 21.3 / 27.9, 64 x 1024^2 41.5 / 32.6
    const bool columns = t.batch <= 40;
    if (t.np == 512) e = columns ? column_launch<256, 2>(t, js, mask, st) : reduce_launch<512, 28, 1024>(t, js, mask, st);
    else if (t.np == 1024) e = columns ? column_launch<256, 4>(t, js, mask, st) : reduce_launch<1024, 8, 1024>(t, js, mask, st);
    else if (t.np == 2048) e = column_launch<512, 8>(t, js, mask, st);
    else if (t.np == 4096) e = column_launch<1024, 16>(t, js, mask, st);
    else return hipErrorInvalidValue;
    if (e) return e;
  }
  if (nt <= 32) hipLaunchKernelGGL(k_tri_tail<1>, dim3(t.batch), dim3(64), 0, st, t, js, mask);
  else if (nt <= 64) hipLaunchKernelGGL(k_tri_tail<2>, dim3(t.batch), dim3(128), 0, st, t, js, mask);
  else if (nt <= 128) hipLaunchKernelGGL(k_tri_tail<4>, dim3(t.batch), dim3(256), 0, st, t, js, mask);
  else hipLaunchKernelGGL(k_tri_tail<8>, dim3(t.batch), dim3(512), 0, st, t, js, mask);
  if ((e = hipGetLastError())) return e;
  if (t.n > 1) {
    hipLaunchKernelGGL(k_tri_larft, dim3(cdiv(t.n - 1, 32), t.batch), dim3(256), 0, st, t, mask);
    if ((e = hipGetLastError())) return e;
  }
  const size_t shv = (size_t)(((t.n + 7) & ~7) + 1) * 16;
  hipLaunchKernelGGL(k_tri_vectors, dim3(cdiv(t.n, 64), t.batch), dim3(64), shv, st, t, mask);
  if ((e = hipGetLastError())) return e;
  const dim3 grid((unsigned)(cdiv(t.batch, 8) * 8 * cdiv(t.n, 32)));
  switch (t.np) {
    case 64: hipLaunchKernelGGL((k_tri_back<2, 1>), grid, dim3(128), 0, st, t, mask); break;
    case 128: hipLaunchKernelGGL((k_tri_back<4, 1>), grid, dim3(256), 0, st, t, mask); break;
    case 256: hipLaunchKernelGGL((k_tri_back<4, 2>), grid, dim3(256), 0, st, t, mask); break;
    case 512: hipLaunchKernelGGL((k_tri_back<4, 4>), grid, dim3(256), 0, st, t, mask); break;
    case 1024: hipLaunchKernelGGL((k_tri_back<8, 4>), grid, dim3(512), 0, st, t, mask); break;
    default: return tri_back_products(t, mask, st);
  }
  return hipGetLastError();
}

static hipError_t tri_check(const TriWs& t, const float* G, const int* mask, hipStream_t st) {
  hipLaunchKernelGGL(k_tri_dev, dim3(std::min(t.n, 64), t.batch), dim3(256), 0, st, t, G, mask);
  return hipGetLastError();
}

static hipError_t tri_rayleigh(const TriWs& t, const float* V2, const float* Y, float* lam, const int* mask,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_tri_rayleigh, dim3(cdiv(t.n, 64), t.batch), dim3(t.n <= 128 ? 256 : 1024), 0, st, t, V2, Y, lam,
                     mask);
  return hipGetLastError();
}

static hipError_t tri_rescue(const TriWs& t, const float* G, int* flags, const int* mask, hipStream_t st) {
  hipLaunchKernelGGL(k_tri_rescue, dim3(t.batch), dim3(1024), (size_t)t.n * 16, st, t, G, flags, mask);
  return hipGetLastError();
}

static hipError_t tri_polish(const TriWs& t, float* G, float* V2, int again, const int* mask, hipStream_t st) {
  const size_t lds = (size_t)2 * t.np * (t.np + 4) * sizeof(float);
  const dim3 grid(again ? std::min(t.batch, 64) : t.batch);
  if (t.np == 64) hipLaunchKernelGGL(k_tri_polish<64>, grid, dim3(512), lds, st, t, G, V2, again, mask);
  else if (t.np == 128) hipLaunchKernelGGL(k_tri_polish<128>, grid, dim3(1024), lds, st, t, G, V2, again, mask);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
