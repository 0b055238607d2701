// The l x l symmetric eigenproblem of the Rayleigh-Ritz step (l = 32, 64, 96 or 128), one workgroup per problem.
#include <algorithm>

#include "dense_device.h"
#include "kernels.h"
#include "profiler.h"

namespace lq {

constexpr int EIG_THREADS = 256;

// Sums of N values over the 16 lanes of a DPP row with the values dealt out on the way: each of the first log2(N) steps
// hands half of a lane's values to its partner, so a lane ends with the total of value row_sum_index<N>(lane) alone.
template <int N>
__device__ __forceinline__ double row_sum_dealt(double (&v)[N], int tx) {
  static_assert(N == 2 || N == 4 || N == 8, "");
  const bool b3 = tx & 8, b2 = tx & 4, b1 = tx & 2;
#pragma unroll
  for (int e = 0; e < N / 2; ++e) {
    const double keep = b3 ? v[e + N / 2] : v[e], give = b3 ? v[e] : v[e + N / 2];
    v[e] = keep + dpp_move<XOR15>(give);
  }
  if constexpr (N >= 4) {
#pragma unroll
    for (int e = 0; e < N / 4; ++e) {
      const double keep = b2 ? v[e + N / 4] : v[e], give = b2 ? v[e] : v[e + N / 4];
      v[e] = keep + dpp_move<XOR7>(give);
    }
  } else {
    v[0] += dpp_move<XOR7>(v[0]);
  }
  if constexpr (N >= 8) {
    const double keep = b1 ? v[1] : v[0], give = b1 ? v[0] : v[1];
    v[0] = keep + dpp_move<XOR2>(give);
  } else {
    v[0] += dpp_move<XOR2>(v[0]);
  }
  return v[0] + dpp_move<XOR1>(v[0]);
}
template <int N>
__device__ __forceinline__ int row_sum_index(int tx) {
  return N == 8 ? ((tx >> 3) & 1) * 4 + ((tx >> 2) & 1) * 2 + ((tx >> 1) & 1)
       : N == 4 ? ((tx >> 3) & 1) * 2 + ((tx >> 2) & 1) : (tx >> 3) & 1;
}

// ---- one-sided Jacobi, for matrices whose eigenvalues are not separated ------------------------------
__device__ __forceinline__ float row_sum16(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), XOR1, 0xf, 0xf, false));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), XOR2, 0xf, 0xf, false));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), XOR7, 0xf, 0xf, false));
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), XOR15, 0xf, 0xf, false));
  return x;
}

// One-sided (Hestenes) Jacobi in fp32 with X = M and V = I in LDS: rotating the columns of X = M J until they are mutually
// orthogonal makes J^T M^2 J diagonal, so J holds the eigenvectors of the symmetric M and the column norms are the
// eigenvalues.  16 lanes per column pair, l/32 pairs per lane group and round, one barrier per round; every LDS read of a
// round is issued before the first store.  The squared column norms are kept in LDS and updated with the rotation.
// Rows of Ut come out orthonormal to about 1e-6 whatever the spectrum is (repeated and zero eigenvalues included).
template <int NE>
__device__ void jacobi_onesided(const double* __restrict__ G, double mscale, float* fl, float* s_n2, float* s_vscale,
                                int* s_rank, int* s_flags, float* __restrict__ Ut, double* __restrict__ lam) {
  constexpr int l = 16 * NE, P = l + 4, CE = NE, PP = l / 32;
  float* X = fl;
  float* V = fl + l * P;
  const int tid = threadIdx.x, g = tid >> 4, sub = tid & 15, eo = CE * sub;
  for (int idx = tid; idx < l * l; idx += EIG_THREADS) {
    const int c = idx / l, i = idx % l;
    X[c * P + i] = (float)(G[idx] * mscale);            // symmetric: row c of M is column c
    V[c * P + i] = (c == i) ? 1.0f : 0.0f;
  }
  __syncthreads();
  for (int sweep = 0; sweep < 30; ++sweep) {
    if (tid == 0) s_flags[0] = 0;
    for (int c = g; c < l; c += 16) {
      float n2 = 0.f;
#pragma unroll
      for (int e = 0; e < CE; ++e) { const float x = X[c * P + eo + e]; n2 = fmaf(x, x, n2); }
      n2 = row_sum16(n2);
      if (sub == 0) s_n2[c] = n2;
    }
    __syncthreads();
    float worst = 0.0f;
    for (int round = 0; round < l - 1; ++round) {
      int p[PP], q[PP];
      float xp[PP][CE], xq[PP][CE], vp[PP][CE], vq[PP][CE], al[PP], be[PP];
#pragma unroll
      for (int a = 0; a < PP; ++a) {
        circle_pair(g + 16 * a, round, l, p[a], q[a]);
#pragma unroll
        for (int e = 0; e < CE; e += 2) {
          float2 t;
          t = *reinterpret_cast<const float2*>(X + p[a] * P + eo + e); xp[a][e] = t.x; xp[a][e + 1] = t.y;
          t = *reinterpret_cast<const float2*>(X + q[a] * P + eo + e); xq[a][e] = t.x; xq[a][e + 1] = t.y;
          t = *reinterpret_cast<const float2*>(V + p[a] * P + eo + e); vp[a][e] = t.x; vp[a][e + 1] = t.y;
          t = *reinterpret_cast<const float2*>(V + q[a] * P + eo + e); vq[a][e] = t.x; vq[a][e + 1] = t.y;
        }
        al[a] = s_n2[p[a]]; be[a] = s_n2[q[a]];
      }
#pragma unroll
      for (int a = 0; a < PP; ++a) {
        float ga = 0.f;
#pragma unroll
        for (int e = 0; e < CE; ++e) ga = fmaf(xp[a][e], xq[a][e], ga);
        ga = row_sum16(ga);
        // hardware reciprocal / square-root approximations (1 ulp) are enough: a rotation that is orthogonal to 1e-7 and
        // an angle that misses the exact one by 1e-7 change nothing in the convergence
        const float ab = al[a] * be[a];
        if (ga != 0.0f && ga * ga > 4e-12f * ab) {
          worst = fmaxf(worst, fabsf(ga) * __builtin_amdgcn_rsqf(ab));
          const float zeta = (be[a] - al[a]) * 0.5f * __builtin_amdgcn_rcpf(ga);
          const float tt = copysignf(__builtin_amdgcn_rcpf(fabsf(zeta) + __builtin_amdgcn_sqrtf(1.0f + zeta * zeta)), zeta);
          const float cs = __builtin_amdgcn_rsqf(1.0f + tt * tt), sn = cs * tt;
#pragma unroll
          for (int e = 0; e < CE; e += 2) {
            *reinterpret_cast<float2*>(X + p[a] * P + eo + e) =
                make_float2(cs * xp[a][e] - sn * xq[a][e], cs * xp[a][e + 1] - sn * xq[a][e + 1]);
            *reinterpret_cast<float2*>(X + q[a] * P + eo + e) =
                make_float2(sn * xp[a][e] + cs * xq[a][e], sn * xp[a][e + 1] + cs * xq[a][e + 1]);
            *reinterpret_cast<float2*>(V + p[a] * P + eo + e) =
                make_float2(cs * vp[a][e] - sn * vq[a][e], cs * vp[a][e + 1] - sn * vq[a][e + 1]);
            *reinterpret_cast<float2*>(V + q[a] * P + eo + e) =
                make_float2(sn * vp[a][e] + cs * vq[a][e], sn * vp[a][e + 1] + cs * vq[a][e + 1]);
          }
          if (sub == 0) {                               // the pairs of a round are disjoint: nobody else touches these two
            s_n2[p[a]] = fmaxf(al[a] - tt * ga, 0.0f);
            s_n2[q[a]] = be[a] + tt * ga;
          }
        }
      }
      __syncthreads();
    }
    if (worst > 1e-4f) s_flags[0] = 1;                  // every writer stores the same value
    __syncthreads();
    const bool more = s_flags[0] != 0;                  // quadratic convergence: a sweep whose worst pair was below 1e-4
    __syncthreads();                                    // leaves nothing above ~1e-7 behind
    if (!more) break;
  }
  for (int c = tid; c < l; c += EIG_THREADS) {          // eigenvalue estimates = column norms
    float n2 = 0.f;
    double v2 = 0.0;
    for (int i = 0; i < l; ++i) {
      n2 = fmaf(X[c * P + i], X[c * P + i], n2);
      const double vv = V[c * P + i];
      v2 = fma(vv, vv, v2);
    }
    s_n2[c] = sqrtf(n2);
    s_vscale[c] = (float)(1.0 / sqrt(v2));              // accumulated rotations drift from unit norm by ~1e-6
  }
  __syncthreads();
  for (int c = tid; c < l; c += EIG_THREADS) {
    const float li = s_n2[c];
    int r = 0;
    for (int j = 0; j < l; ++j) r += (s_n2[j] > li || (s_n2[j] == li && j < c)) ? 1 : 0;
    s_rank[c] = r;
    lam[r] = (double)li / mscale;
  }
  __syncthreads();
  for (int idx = tid; idx < l * l; idx += EIG_THREADS) {
    const int c = idx / l, i = idx % l;
    Ut[(size_t)s_rank[c] * l + i] = V[c * P + i] * s_vscale[c];
  }
}

// ---- tridiagonal route ---------------------------------------------------------------------------------
// Householder tridiagonalisation, eigenvalues by multisection on Sturm counts, eigenvectors by twisted factorisation,
// back-transformation; all in fp64.  256 threads form a 16 x 16 grid, thread (ty, tx) keeps the elements (i, k) with
// i = ty, k = tx (mod 16) of the matrix in registers.  Every phase is a serial chain of l steps, so what bounds the
// kernel is latency, and the layout is chosen for short steps: four wavefronts (one per SIMD; with 16 the redundant
// per-wavefront work and the LDS reads of the vectors quadruple), two barriers per column, and scalar parts that every
// wavefront computes for itself instead of waiting for one.
// Eigenvectors computed one by one are orthogonal to about 1e-16 lambda_1 / gap.  Where a gap is below 2e-9 lambda_1 (so
// that 1e-6 could be missed; in a sweep the Ritz values of the quantization noise of 8-bit configurations, 1e-8 lambda_1
// themselves, are such a cluster) the rows are orthonormalised together at the end, and where they have come out too
// dependent for that (repeated eigenvalues, a singular matrix) the problem is solved by one-sided Jacobi, in the same launch.
// Measured on a weight matrix's spectrum in a random basis (one problem, us): l = 32 98 -> 45, l = 64 297 -> 100,
// l = 96 687 -> 192, l = 128 1491 -> 273 against one-sided Jacobi with 8 l threads, whose six to nine sweeps of l - 1
// rounds are bound by LDS bandwidth (every round reads and writes X and V); Rayleigh quotients come out 10 to 70 times
// closer, because the tridiagonal route keeps G in fp64.
template <int NE>
__global__ __launch_bounds__(EIG_THREADS) void sym_eig_kernel(const double* __restrict__ Gall, double* __restrict__ work,
                                                              float* __restrict__ Utall, double* __restrict__ lamall) {
  constexpr int l = 16 * NE, NP = NE <= 2 ? 2 : (NE <= 4 ? 4 : 8);
  constexpr int TPE = l > 64 ? 2 : (l > 32 ? 4 : 8);        // threads per eigenvalue in the multisection
  constexpr int ROUNDS = TPE == 2 ? 34 : (TPE == 4 ? 23 : 17);   // (TPE + 1)^ROUNDS > 2^53
  extern __shared__ __attribute__((aligned(16))) double lds[];   // reflectors [l][l]; the Jacobi route's X and V
  double* Vr = lds;
  __shared__ double s_col[l], s_p[l], s_h[l], s_e[l], s_lam[l], s_inv[l];
  __shared__ double2 s_de[l + 1];                            // {d_i, e_{i-1}^2}
  __shared__ double s_best[2][128], s_sum[2][128];
  __shared__ int s_at[2][128], s_k[128];
  __shared__ float s_n2[128], s_vscale[128];
  __shared__ int s_rank[128], s_flags[1];
  __shared__ double s_wmax[4];
  const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63, ty = tid >> 4, tx = tid & 15;
  const double* G = Gall + (size_t)z * l * l;
  double* Sp = work + (size_t)z * 2 * l * l;
  double* Sm = Sp + l * l;
  float* Ut = Utall + (size_t)z * l * l;
  double* lam = lamall + (size_t)z * l;

  // In a sweep the streaming kernels of other streams share the compute unit: this one is a serial chain that the next
  // kernel of its stream waits for, they have thousands of wavefronts in flight.
  __builtin_amdgcn_s_setprio(3);

  // unit scale by a power of two of the largest diagonal entry
  double a[NE][NE];
  double mx = 0.0;
#pragma unroll
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int f = 0; f < NE; ++f) {
      a[e][f] = G[(size_t)(ty + 16 * e) * l + tx + 16 * f];
      if (e == f && ty == tx) mx = fmax(mx, fabs(a[e][f]));
    }
  for (int off = 1; off < 64; off <<= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if (lane == 0) s_wmax[tid >> 6] = mx;
  __syncthreads();
  mx = fmax(fmax(s_wmax[0], s_wmax[1]), fmax(s_wmax[2], s_wmax[3]));
  const double mscale = (mx > 0.0 && mx < 1.0e300) ? ldexp(1.0, -ilogb(mx)) : 1.0;
#pragma unroll
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int f = 0; f < NE; ++f) a[e][f] *= mscale;

  // Reduction of column j: x = A[j+1.., j], v = x - beta e_1, A <- H A H with H = I - h v v^T, as A -= v w^T + w v^T
  for_each_block<NE>([&](auto block) {
    constexpr int jb = decltype(block)::value;
    for (int jt = 0; jt < 16; ++jt) {
      const int j = 16 * jb + jt;
      if (tx == jt) {
#pragma unroll
        for (int e = jb; e < NE; ++e) s_col[ty + 16 * e] = a[e][jb];
      }
      __syncthreads();
      double x0 = lane > j && lane < l ? s_col[lane < l ? lane : 0] : 0.0;
      double x1 = 0.0;
      if constexpr (l > 64) x1 = lane + 64 > j && lane + 64 < l ? s_col[lane + 64 < l ? lane + 64 : 0] : 0.0;
      const double alpha = j + 1 < l ? s_col[j + 1 < l ? j + 1 : j] : 0.0;
      const double s2 = wave_sum((lane == j + 1 ? 0.0 : x0 * x0) + (lane + 64 == j + 1 ? 0.0 : x1 * x1));
      const double n2 = fma(alpha, alpha, s2);
      const bool reflect = s2 > 1e-280;
      const double norm = reflect ? n2 * rsqrt64(n2) : 0.0;
      const double beta = reflect ? -copysign(norm, alpha) : alpha;
      const double h = reflect ? rcp64(fma(fabs(alpha), norm, n2)) : 0.0;     // 2 / v^T v
      const double v1 = reflect ? alpha - beta : 0.0;
      if (lane == j + 1) x0 = v1;
      if (lane + 64 == j + 1) x1 = v1;
      double vi[NE], vk[NE];
#pragma unroll
      for (int e = jb; e < NE; ++e) {
        const int i = ty + 16 * e, k = tx + 16 * e;
        vi[e] = s_col[i]; vk[e] = s_col[k];
        if (e <= jb + 1) {
          vi[e] = i > j + 1 ? vi[e] : (i == j + 1 ? v1 : 0.0);
          vk[e] = k > j + 1 ? vk[e] : (k == j + 1 ? v1 : 0.0);
        }
      }
      if (tid < l) Vr[j * l + tid] = tid > j + 1 ? s_col[tid] : (tid == j + 1 ? v1 : 0.0);
      if (tid == 0) { s_h[j] = h; s_e[j] = beta; s_de[j].x = s_col[j]; }
      double part[NP];
#pragma unroll
      for (int e = 0; e < NP; ++e) {
        part[e] = 0.0;
        if (e >= jb && e < NE) {
#pragma unroll
          for (int f = jb; f < NE; ++f) part[e] = fma(a[e][f], vk[f], part[e]);
        }
      }
      const double total = row_sum_dealt<NP>(part, tx);
      const int re = row_sum_index<NP>(tx);
      if (re < NE) {
        const int i = ty + 16 * re;
        s_p[i] = i > j ? total * h : 0.0;
      }
      __syncthreads();
      double pv = x0 * (lane < l ? s_p[lane < l ? lane : 0] : 0.0);
      if constexpr (l > 64) pv = fma(x1, lane + 64 < l ? s_p[lane + 64 < l ? lane + 64 : 0] : 0.0, pv);
      const double K = 0.5 * h * wave_sum(pv);
      double wi[NE], wk[NE];
#pragma unroll
      for (int e = jb; e < NE; ++e) {
        wi[e] = fma(-K, vi[e], s_p[ty + 16 * e]);
        wk[e] = fma(-K, vk[e], s_p[tx + 16 * e]);
      }
#pragma unroll
      for (int e = jb; e < NE; ++e)
#pragma unroll
        for (int f = jb; f < NE; ++f) a[e][f] = fma(-vi[e], wk[f], fma(-wi[e], vk[f], a[e][f]));
    }
  });
  __syncthreads();

  // Gershgorin interval, squared off-diagonals (kept above zero so that a Sturm sequence that hits zero goes on)
  double lo = 1e300, hi = -1e300;
#pragma unroll
  for (int c = 0; c < (l + 63) / 64; ++c) {
    const int i = lane + 64 * c;
    if (i < l) {
      const double r = (i > 0 ? fabs(s_e[i - 1]) : 0.0) + (i + 1 < l ? fabs(s_e[i]) : 0.0), d = s_de[i].x;
      lo = fmin(lo, d - r); hi = fmax(hi, d + r);
    }
  }
  for (int off = 1; off < 64; off <<= 1) { lo = fmin(lo, __shfl_xor(lo, off)); hi = fmax(hi, __shfl_xor(hi, off)); }
  const double bound = fmax(fabs(lo), fabs(hi));
  lo -= 1e-14 * bound; hi += 1e-14 * bound;
  __syncthreads();
  if (tid < l) {
    const double e = tid > 0 ? s_e[tid - 1] : 0.0;
    s_de[tid].y = tid > 0 ? fmax(e * e, 1e-36 * bound * bound) : 0.0;
  }
  if (tid == 0) { s_de[l].x = 0.0; s_de[l].y = 0.0; }
  __syncthreads();

  // Eigenvalue g (ascending): TPE threads count the eigenvalues below the inner points of its interval.  The count is the
  // number of sign changes of p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}, which needs no division; sign bits are
  // collected 32 at a time and the pair is brought back to unit size every eight steps.
  {
    const int g = tid / TPE, sub = tid % TPE;
    if (g < l) {
      for (int round = 0; round < ROUNDS; ++round) {
        const double x = fma(hi - lo, (sub + 1) * (1.0 / (TPE + 1)), lo);
        double pa = 0.0, pb = 1.0;
        int count = 0;
        unsigned last = 0;
        for (int i0 = 0; i0 < l; i0 += 32) {
          unsigned bits = 0;
#pragma unroll
          for (int i1 = 0; i1 < 32; i1 += 8) {
#pragma unroll
            for (int i2 = 0; i2 < 8; ++i2) {
              const double2 de = s_de[i0 + i1 + i2];
              const double pn = fma(de.x - x, pb, -de.y * pa);
              bits = __builtin_amdgcn_alignbit(bits, (unsigned)__double2hiint(pn), 31);
              pa = pb; pb = pn;
            }
            const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(pa), fabs(pb)));
            pa = ldexp(pa, -ex); pb = ldexp(pb, -ex);
          }
          count += __popc(bits ^ ((bits >> 1) | (last << 31)));
          last = bits & 1u;
        }
        const bool below = count <= g;                   // the eigenvalue is at x or above
        double nlo = below ? x : lo, nhi = below ? hi : x;
        nlo = fmax(nlo, dpp_move<XOR1>(nlo)); nhi = fmin(nhi, dpp_move<XOR1>(nhi));
        if constexpr (TPE >= 4) { nlo = fmax(nlo, dpp_move<XOR2>(nlo)); nhi = fmin(nhi, dpp_move<XOR2>(nhi)); }
        if constexpr (TPE >= 8) { nlo = fmax(nlo, dpp_move<XOR7>(nlo)); nhi = fmin(nhi, dpp_move<XOR7>(nhi)); }
        lo = nlo; hi = nhi;
      }
      if (sub == 0) s_lam[g] = 0.5 * (lo + hi);
    }
  }
  __syncthreads();
  bool close = false;
  if (tid < l - 1) close = !(s_lam[tid + 1] - s_lam[tid] > 2e-9 * bound);
  const bool clustered = __syncthreads_or(close);
  if (tid < l) lam[l - 1 - tid] = fmax(s_lam[tid], 0.0) / mscale;

  // Eigenvectors of the tridiagonal matrix: T - lambda = L D+ L^T from the top (lower half of the threads) and U D- U^T
  // from the bottom (upper half), joined at the index k where |gamma_k| is smallest.  The reciprocal pivots go through
  // the scratch in memory, one eigenvector per lane.
  const int half = tid >> 7, g = tid & 127;
  const bool has = g < l;
  const double lg = has ? s_lam[g] : 0.0;
  const double tiny = 1e-30 * bound;
  if (has) {
    double* S = half == 0 ? Sp : Sm;
    double r = 0.0;
#pragma unroll 4
    for (int s = 0; s < l; ++s) {
      const int i = half == 0 ? s : l - 1 - s;
      double D = (s_de[i].x - lg) - (half == 0 ? s_de[i].y : s_de[i + 1].y) * r;
      if (!(fabs(D) > tiny)) D = copysign(tiny, D);
      r = rcp64(D);
      S[i * l + g] = r;
    }
  }
  __syncthreads();
  if (has) {
    double best = INFINITY;
    int at = half * (l / 2);
#pragma unroll 8
    for (int s = 0; s < l / 2; ++s) {
      const int i = half * (l / 2) + s;
      const double up = i > 0 ? Sp[(i - 1) * l + g] : 0.0, dn = i + 1 < l ? Sm[(i + 1) * l + g] : 0.0;
      const double ga = fabs((s_de[i].x - lg) - s_de[i].y * up - s_de[i + 1].y * dn);
      if (ga < best) { best = ga; at = i; }
    }
    s_best[half][g] = best; s_at[half][g] = at;
  }
  __syncthreads();
  if (has) {
    const int k = s_best[1][g] < s_best[0][g] ? s_at[1][g] : s_at[0][g];
    double zz = 1.0, sum = half == 0 ? 1.0 : 0.0;
    if (half == 0) {
      s_k[g] = k;
#pragma unroll 8
      for (int i = l - 1; i >= 0; --i) {
        const double r = Sp[i * l + g];
        if (i < k) { zz *= -s_e[i] * r; sum = fma(zz, zz, sum); }
        if (i <= k) Sp[i * l + g] = zz;
      }
    } else {
#pragma unroll 8
      for (int i = 1; i < l; ++i) {
        const double r = Sm[i * l + g];
        if (i > k) { zz *= -s_e[i - 1] * r; sum = fma(zz, zz, sum); Sm[i * l + g] = zz; }
      }
    }
    s_sum[half][g] = sum;
  }
  __syncthreads();
  if (tid < l) s_inv[tid] = 1.0 / sqrt(s_sum[0][tid] + s_sum[1][tid]);
  __syncthreads();

  // Back-transformation: 8 lanes per eigenvector, l/32 eigenvectors per lane group, entries 16 m + 2 sub + {0, 1}
  constexpr int NV = l / 32;
  const int grp = tid >> 3, sub = tid & 7;
  double u[NV][NE][2];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = grp + 32 * v, k = s_k[c];
    const double inv = s_inv[c];
#pragma unroll
    for (int m = 0; m < NE; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int i = 16 * m + 2 * sub + q;
        u[v][m][q] = (i <= k ? Sp : Sm)[i * l + c] * inv;
      }
  }
  for_each_block_down<NE>([&](auto block) {
    constexpr int jb = decltype(block)::value;
    for (int jt = 15; jt >= 0; --jt) {
      const int j = 16 * jb + jt;
      const double h = s_h[j];
      double2 w[NE];
#pragma unroll
      for (int m = jb; m < NE; ++m) w[m] = *reinterpret_cast<const double2*>(Vr + j * l + 16 * m + 2 * sub);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        double dot = 0.0;
#pragma unroll
        for (int m = jb; m < NE; ++m) dot = fma(w[m].x, u[v][m][0], fma(w[m].y, u[v][m][1], dot));
        dot += dpp_move<XOR1>(dot);
        dot += dpp_move<XOR2>(dot);
        dot += dpp_move<XOR7>(dot);
        dot *= -h;
#pragma unroll
        for (int m = jb; m < NE; ++m) { u[v][m][0] = fma(dot, w[m].x, u[v][m][0]); u[v][m][1] = fma(dot, w[m].y, u[v][m][1]); }
      }
    }
  });
  if (!clustered) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int c = grp + 32 * v;
#pragma unroll
      for (int m = 0; m < NE; ++m)
        *reinterpret_cast<float2*>(Ut + (size_t)(l - 1 - c) * l + 16 * m + 2 * sub) =
            make_float2((float)u[v][m][0], (float)u[v][m][1]);
    }
    return;
  }

  // Close eigenvalues: the rows are nearly orthonormal still, and steps U <- U + (I - U U^T) U / 2 make them so; the
  // correction mixes only rows that overlap, which are those of close eigenvalues.  U lies in LDS (the reflectors are
  // done with), thread (ty, tx) computes the elements (ty + 16 e, tx + 16 f) of both products.
  constexpr int PU = l + 2;
  double* Us = lds;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int m = 0; m < NE; ++m)
      *reinterpret_cast<double2*>(Us + (grp + 32 * v) * PU + 16 * m + 2 * sub) = make_double2(u[v][m][0], u[v][m][1]);
  for (int step = 0;; ++step) {
    __syncthreads();
    double s[NE][NE];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int f = 0; f < NE; ++f) s[e][f] = 0.0;
    for (int i = 0; i < l; ++i) {
      double p[NE], q[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e) { p[e] = Us[(ty + 16 * e) * PU + i]; q[e] = Us[(tx + 16 * e) * PU + i]; }
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int f = 0; f < NE; ++f) s[e][f] = fma(p[e], q[f], s[e][f]);
    }
    bool off = false, far = false;
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int f = 0; f < NE; ++f) {
        const double d = (e == f && ty == tx ? 1.0 : 0.0) - s[e][f];
        off = off || !(fabs(d) < 1e-8);
        far = far || !(fabs(d) < 0.02);
        s[e][f] = 0.5 * d;
      }
    if (__syncthreads_or(far) || step == 4) {   // the vectors of a cluster came out too much alike (or not finite)
      jacobi_onesided<NE>(G, mscale, reinterpret_cast<float*>(lds), s_n2, s_vscale, s_rank, s_flags, Ut, lam);
      return;
    }
    if (!__syncthreads_or(off)) break;
    double t[NE][NE];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int f = 0; f < NE; ++f) t[e][f] = Us[(ty + 16 * e) * PU + tx + 16 * f];
    for_each_block<16 * NE>([&](auto column) {           // column 16 fb + b of s sits in lane b of the DPP row
      constexpr int fb = decltype(column)::value / 16, b = decltype(column)::value % 16;
      double q[NE];
#pragma unroll
      for (int f = 0; f < NE; ++f) q[f] = Us[(16 * fb + b) * PU + tx + 16 * f];
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const double d = dpp_move<0x150 + b>(s[e][fb]);  // row_newbcast
#pragma unroll
        for (int f = 0; f < NE; ++f) t[e][f] = fma(d, q[f], t[e][f]);
      }
    });
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int f = 0; f < NE; ++f) Us[(ty + 16 * e) * PU + tx + 16 * f] = t[e][f];
  }
  for (int idx = tid; idx < l * l; idx += EIG_THREADS) {
    const int c = idx / l, i = idx % l;
    Ut[(size_t)(l - 1 - c) * l + i] = (float)Us[c * PU + i];
  }
}

bool sym_eig_supported(int l) { return l % 32 == 0 && l >= 32 && l <= 128; }

template <int NE>
static int launch_eig(const double* G, double* work, float* Ut, double* lambda, int batch, hipStream_t st) {
  constexpr int l = 16 * NE;
  const size_t reflectors = (size_t)l * l * sizeof(double), jacobi = (size_t)2 * l * (l + 4) * sizeof(float);
  const size_t rows = (size_t)l * (l + 2) * sizeof(double);
  const size_t need = std::max(reflectors, std::max(jacobi, rows));
  static LdsLimit limit;
  LQ_TRY(limit.raise(reinterpret_cast<const void*>(sym_eig_kernel<NE>), need));
  hipLaunchKernelGGL((sym_eig_kernel<NE>), dim3(batch), dim3(EIG_THREADS), need, st, G, work, Ut, lambda);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

int launch_sym_eig(const double* G, int l, double* work, float* Ut, double* lambda, int batch, hipStream_t st) {
  prof::Scope ps(prof::SYM_EIG, st, (double)l * l * 8.0 * batch);
  switch (l / 16) {
    case 2: return launch_eig<2>(G, work, Ut, lambda, batch, st);
    case 4: return launch_eig<4>(G, work, Ut, lambda, batch, st);
    case 6: return launch_eig<6>(G, work, Ut, lambda, batch, st);
    case 8: return launch_eig<8>(G, work, Ut, lambda, batch, st);
    default: return LQ_ERR_ARG;
  }
}

}  // namespace lq
