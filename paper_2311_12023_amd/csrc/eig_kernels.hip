// The l x l symmetric eigenproblem of the Rayleigh-Ritz step (l = 32, 64, 96 or 128), one workgroup per problem.
#include <algorithm>

#include "dense_device.h"
#include "kernels.h"
#include "profiler.h"

namespace lq {

constexpr int EIG_THREADS = 256;
typedef double doublex2 __attribute__((ext_vector_type(2)));   // native vector: arrays of it stay in registers

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
    for (int j = 0; j < l; ++j) r += sorts_before(s_n2[j], j, li, c) ? 1 : 0;
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
// Householder tridiagonalisation, eigenvalues by Sturm counts (multisection until each is alone, then secant steps inside
// the counts' brackets), eigenvectors by twisted factorisation, back-transformation; all in fp64.  256 threads form a 16 x 16 grid,
// thread (ty, tx) keeps the elements (i, k) with i = ty, k = tx (mod 16) of the matrix in registers.  Every phase is a serial chain of l steps, so what bounds the
// kernel is latency, and the layout is chosen for short steps: four wavefronts (one per SIMD; with 16 the redundant
// per-wavefront work and the LDS reads of the vectors quadruple), two barriers per column, and scalar parts that every
// wavefront computes for itself instead of waiting for one.
// Eigenvectors computed one by one are orthogonal to about 1e-16 lambda_1 / gap.  Where a gap is below 2e-9 lambda_1 (so
// that 1e-6 could be missed; in a sweep the Ritz values of the quantization noise of 8-bit configurations, 1e-8 lambda_1
// themselves, are such a cluster) the rows are orthonormalised together at the end, and where they have come out too
// dependent for that (repeated eigenvalues, a singular matrix) the problem is solved by one-sided Jacobi, in the same launch.
// Measured on a weight matrix's spectrum in a random basis (one problem, us), with one-sided Jacobi (8 l threads, six to nine
// sweeps of l - 1 rounds bound by LDS bandwidth, every one of which reads and writes X and V), with a first form of this route (a
// chain of two wavefront sums and roots per column before anything else, 34 rounds of trisection, reciprocal pivots in memory
// behind branches), with this one and the vectors in the same launch, and as it is: l = 32 98, 45, 35, 35; l = 64 297, 99, 79, 78;
// l = 96 687, 193, 138, 131; l = 128 1491, 275, 210, 184.  Rayleigh quotients come out 10 to 70 times closer than Jacobi's, because G
// stays in fp64.  In the one launch of l = 128 the phases took 275, 61, 47 and 94 thousand cycles (tridiagonal form, eigenvalues,
// vectors, back-transformation); the first launch keeps the first two.  A column of the form is 1400 cycles of latency, by
// what it takes at l = 32, and its share of 3 l^2 fp64 operations.
// The pivots of l = 64 beside the reflectors make 96 KB of LDS, which leaves room for one workgroup of a kernel with 64 KB on
// the compute unit: sweeps that solve l = 64 in batches gain all the same (36 configurations of 4096 x 4096, rank 16, 32 and 40: 25.8 ->
// 24.5, 26.4 -> 25.2, 26.8 -> 25.6 ms; nine of 1024 x 4096, rank 16: 6.0 -> 4.7).
//
// Eigenvalues below x of the tridiagonal matrix with {d_i, e_{i-1}^2} in de: the sign changes of p_i = (d_i - x) p_{i-1} -
// e_{i-1}^2 p_{i-2}, which needs no division; sign bits are collected 32 at a time.  The pair is brought back to unit size every
// 16 steps: with a norm of at most 2 l (a Gram matrix whose diagonal is below 2) and e^2 kept above 1e-36 of its square, a
// step makes it no more than 2^17 larger and two steps no more than 1e-36 smaller.  p_l = f 2^e.
template <int l>
__device__ __forceinline__ int sturm(const double2* de, double x, double& f, int& e) {
  double pa = 0.0, pb = 1.0;
  int count = 0;
  unsigned last = 0;
  e = 0;
  for (int i0 = 0; i0 < l; i0 += 32) {
    unsigned bits = 0;
#pragma unroll
    for (int i1 = 0; i1 < 32; i1 += 16) {
#pragma unroll
      for (int i2 = 0; i2 < 16; ++i2) {
        const double2 v = de[i0 + i1 + i2];
        const double pn = fma(v.x - x, pb, -v.y * pa);
        bits = __builtin_amdgcn_alignbit(bits, (unsigned)__double2hiint(pn), 31);
        pa = pb; pb = pn;
      }
      const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(pa), fabs(pb)));
      pa = ldexp(pa, -ex); pb = ldexp(pb, -ex);
      e += ex;
    }
    count += __popc(bits ^ ((bits >> 1) | (last << 31)));
    last = bits & 1u;
  }
  f = pb;
  return count;
}

// From l = 96 on the vectors of separated eigenvalues take a launch of their own with a workgroup for every 16 of them: one
// workgroup's pivots do not fit LDS beside the reflectors, and its l / 32 vectors per 8 lanes are a third of its time (one problem, as
// traced beside the rest of a call: l = 128 212 -> 149 + 36 us, l = 96 147 -> 110 + 27; at l = 64 and below everything is in LDS
// and the whole solve takes 80 us).  What is handed on lies in the scratch: the reflectors from the diagonal block on (block row jb: 16 rows of l - 16 jb), then this.
template <int NE> constexpr bool EIG_HANDS_ON = NE > 4;
template <int NE> constexpr __host__ __device__ int packed_block(int jb) { return 256 * (jb * NE - jb * (jb - 1) / 2); }
template <int NE>
struct EigHandOn { double2 de[16 * NE + 1]; double e[16 * NE], h[16 * NE], lam[16 * NE], bound; int vectors_wanted; };
// vectors_wanted is written by the first launch for every problem, whatever the scratch held: 0 where that launch has made the
// vectors itself (which it says once it is done with the pivots, whose place this is).

template <int NE>
__global__ __launch_bounds__(EIG_THREADS) void sym_eig_kernel(const double* __restrict__ Gall, double* __restrict__ work,
                                                              float* __restrict__ Utall, double* __restrict__ lamall) {
  constexpr int l = 16 * NE;
  extern __shared__ __attribute__((aligned(16))) double lds[];   // reflectors [l][l]; the Jacobi route's X and V
  double* Vr = lds;
  __shared__ double s_col[l], s_next[l], s_p[l], s_h[l], s_e[l], s_lam[l], s_inv[l];
  __shared__ double2 s_de[l + 1];                            // {d_i, e_{i-1}^2}
  __shared__ double s_best[2][128], s_sum[2][128];
  __shared__ int s_at[2][128], s_k[128];
  __shared__ float s_n2[128], s_vscale[128];
  __shared__ int s_rank[128], s_flags[1];
  __shared__ double s_wmax[4], s_x[EIG_THREADS], s_f[EIG_THREADS];
  __shared__ int s_cnt[EIG_THREADS], s_ex[EIG_THREADS];
  const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63, ty = tid >> 4, tx = tid & 15;
  const double* G = Gall + (size_t)z * l * l;
  double* Sp;                                                // reciprocal pivots: in LDS where all three arrays fit
  if constexpr (NE <= 4) Sp = lds + l * l;
  else Sp = work + (size_t)z * 2 * l * l;
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

  // Reduction of column j: x = A[j+1.., j], v = x - beta e_1, A <- H A H with H = I - h v v^T, as A -= v w^T + w v^T with
  // p = h A v, w = p - (h/2) (p^T v) v.  A step is two exchanges through LDS (x, p) and two short chains of dependent
  // operations, the norm of x with its roots and reciprocals and then p^T v; every 16 lanes hold whole vectors (vk, wk, p), so
  // sums take four cross-lane moves and no wavefront waits for another.  What else there is to do is dealt out between the
  // links of the first chain: the last reflector's update, of which only the tile column that holds column j + 1 was done
  // before that column went to LDS, and A x, which does not need beta (A v = A x - beta A e_1, and column j + 1 goes to LDS
  // with column j).
  double vi[NE], vk[NE], wi[NE], wk[NE];       // the last reflector, not yet applied to the tile columns past the current one
#pragma unroll
  for (int e = 0; e < NE; ++e) vi[e] = vk[e] = wi[e] = wk[e] = 0.0;
  if (tx < 2) {
#pragma unroll
    for (int e = 0; e < NE; ++e) (tx ? s_next : s_col)[ty + 16 * e] = a[e][0];
  }
  for_each_block<NE>([&](auto block) {
    constexpr int jb = decltype(block)::value, LEFT = NE - jb, NP = LEFT <= 2 ? 2 : (LEFT <= 4 ? 4 : 8);
    const int re = row_sum_index<NP>(tx), mine = ty + 16 * (jb + (re < LEFT ? re : 0));      // the row whose sum this lane ends up with
#pragma nounroll
    for (int jt = 0; jt < 16; ++jt) {
      const int j = 16 * jb + jt;
      __syncthreads();
      double xi[NE], xk[NE], part[NP];
#pragma unroll
      for (int e = jb; e < NE; ++e) { xk[e] = s_col[tx + 16 * e]; xi[e] = s_col[ty + 16 * e]; }
      const double alpha = s_col[j + 1 < l ? j + 1 : j], next = s_next[mine];
      if (tid < l && tid != j + 1) Vr[j * l + tid] = tid > j ? s_col[tid] : 0.0;
      if (tid == 0) s_de[j].x = s_col[j];
      xk[jb] = tx > jt ? xk[jb] : 0.0;
      auto piece = [&](auto row) __attribute__((always_inline)) {   // row e of the pending update and of A x
        constexpr int e = jb + decltype(row)::value;
        if constexpr (e - jb < NP) part[e - jb] = 0.0;
        if constexpr (e < NE) {
          part[e - jb] = a[e][jb] * xk[jb];
#pragma unroll
          for (int f = jb + 1; f < NE; ++f) {
            a[e][f] = fma(-vi[e], wk[f], fma(-wi[e], vk[f], a[e][f]));
            part[e - jb] = fma(a[e][f], xk[f], part[e - jb]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
#define LQ_PIECE(E) piece(std::integral_constant<int, E>{})
      __builtin_amdgcn_sched_barrier(0);
      double s2 = 0.0;                         // squares of x past its first element
#pragma unroll
      for (int e = jb; e < NE; ++e) s2 = fma(e <= jb + 1 && tx + 16 * e == j + 1 ? 0.0 : xk[e], xk[e], s2);
      LQ_PIECE(0);
      s2 += dpp_move<XOR1>(s2);
      LQ_PIECE(1);
      s2 += dpp_move<XOR2>(s2);
      LQ_PIECE(2);
      s2 += dpp_move<XOR7>(s2);
      LQ_PIECE(3);
      s2 += dpp_move<XOR15>(s2);
      LQ_PIECE(4);
      const double n2 = fma(alpha, alpha, s2);
      const bool reflect = s2 > 1e-280;
      LQ_PIECE(5);
      const double root = n2 * rsqrt64(n2);
      LQ_PIECE(6);
      const double norm = reflect ? root : 0.0;
      const double beta = reflect ? -copysign(norm, alpha) : alpha;
      const double h = reflect ? rcp64(fma(fabs(alpha), norm, n2)) : 0.0;     // 2 / v^T v
      const double v1 = reflect ? alpha - beta : 0.0;
      LQ_PIECE(7);
#undef LQ_PIECE
      const double total = row_sum_dealt<NP>(part, tx);
      if (re < LEFT) s_p[mine] = mine > j ? fma(-beta, next, total) * h : 0.0;
      if (tid == 0) { s_h[j] = h; s_e[j] = beta; if (j + 1 < l) Vr[j * l + j + 1] = v1; }
#pragma unroll
      for (int e = jb; e < NE; ++e) {
        vi[e] = e <= jb + 1 && ty + 16 * e == j + 1 ? v1 : (e > jb || ty > jt ? xi[e] : 0.0);
        vk[e] = e <= jb + 1 && tx + 16 * e == j + 1 ? v1 : xk[e];
      }
      __syncthreads();
      double pv = 0.0;
#pragma unroll
      for (int e = jb; e < NE; ++e) { wk[e] = s_p[tx + 16 * e]; wi[e] = s_p[ty + 16 * e]; pv = fma(vk[e], wk[e], pv); }
      pv += dpp_move<XOR1>(pv);
      pv += dpp_move<XOR2>(pv);
      pv += dpp_move<XOR7>(pv);
      pv += dpp_move<XOR15>(pv);
      const double K = 0.5 * h * pv;
#pragma unroll
      for (int e = jb; e < NE; ++e) { wi[e] = fma(-K, vi[e], wi[e]); wk[e] = fma(-K, vk[e], wk[e]); }
      // the tile column that holds column j + 1 (and, at its edge, j + 2)
      if (jt < 15) {
#pragma unroll
        for (int e = jb; e < NE; ++e) a[e][jb] = fma(-vi[e], wk[jb], fma(-wi[e], vk[jb], a[e][jb]));
        if (tx == jt + 1 || tx == jt + 2) {
#pragma unroll
          for (int e = jb; e < NE; ++e) (tx == jt + 1 ? s_col : s_next)[ty + 16 * e] = a[e][jb];
        }
        if constexpr (jb + 1 < NE) {
          if (jt == 14 && tx == 0) {           // not yet updated there: the piece of the next step does that
#pragma unroll
            for (int e = jb; e < NE; ++e)
              s_next[ty + 16 * e] = fma(-vi[e], wk[jb + 1], fma(-wi[e], vk[jb + 1], a[e][jb + 1]));
          }
        }
      } else if constexpr (jb + 1 < NE) {
#pragma unroll
        for (int e = jb + 1; e < NE; ++e) {
          a[e][jb + 1] = fma(-vi[e], wk[jb + 1], fma(-wi[e], vk[jb + 1], a[e][jb + 1]));
          if (tx < 2) (tx ? s_next : s_col)[ty + 16 * e] = a[e][jb + 1];
        }
      }
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

  if constexpr (NE <= 2) {
    // Eigenvalue g (ascending): eight threads count the eigenvalues below the inner points of its interval.  (Sequences this
    // short cost less than the bookkeeping of fewer rounds: l = 32 14 against 22 thousand cycles, l = 64 36 against 34.)
    constexpr int TPE = 8;
    const int g = tid / TPE, sub = tid % TPE;
    for (int round = 0; round < 17; ++round) {               // 9^17 > 2^53
      const double x = fma(hi - lo, (sub + 1) * (1.0 / (TPE + 1)), lo);
      double f; int e;
      const bool over = sturm<l>(s_de, x, f, e) <= g;        // the eigenvalue is at x or above
      double nlo = over ? x : lo, nhi = over ? hi : x;
      nlo = fmax(nlo, dpp_move<XOR1>(nlo)); nhi = fmin(nhi, dpp_move<XOR1>(nhi));
      nlo = fmax(nlo, dpp_move<XOR2>(nlo)); nhi = fmin(nhi, dpp_move<XOR2>(nhi));
      lo = fmax(nlo, dpp_move<XOR7>(nlo)); hi = fmin(nhi, dpp_move<XOR7>(nhi));
    }
    if (sub == 0) s_lam[g] = 0.5 * (lo + hi);
  } else {
    // Eigenvalue g (ascending) lies in [lo, hi), with clo <= g eigenvalues below lo and chi > g below hi.
    double xlo = lo, xhi = hi, flo = 0.0, fhi = 0.0;        // the sequence's last value at both ends, f 2^e (0: not known)
    int elo = 0, ehi = 0, clo = 0, chi = l;
    // First every thread takes a point of its own: the eigenvalues that still share an interval share their threads' points,
    // so that a round cuts it 256 / l times as often as it holds eigenvalues.  (A pair of a point and its count is true for any
    // eigenvalue: what a thread reads of another group, should rounding make counts disagree, narrows no interval wrongly.)
    constexpr int TPE = EIG_THREADS / l;
    for (int round = 0; round < 3; ++round) {
      const int g = tid / TPE;
      if (g < l) {
        const int t = tid - clo * TPE + 1, m = (chi - clo) * TPE + 1;
        const double x = fma(xhi - xlo, (double)t / (double)m, xlo);
        double f; int e;
        s_cnt[tid] = sturm<l>(s_de, x, f, e);
        s_x[tid] = x; s_f[tid] = f; s_ex[tid] = e;
      }
      __syncthreads();
      if (g < l) {
        int below = clo * TPE - 1, above = chi * TPE;        // points of the group at or below eigenvalue g, and above it
        while (above - below > 1) {
          const int mid = (below + above) >> 1;
          if (s_cnt[mid] <= g) below = mid; else above = mid;
        }
        const bool up = below >= clo * TPE && s_x[below < 0 ? 0 : below] >= xlo, dn = above < chi * TPE && s_x[above < l * TPE ? above : 0] <= xhi;
        if (up) { xlo = s_x[below]; flo = s_f[below]; elo = s_ex[below]; clo = s_cnt[below]; }
        if (dn) { xhi = s_x[above]; fhi = s_f[above]; ehi = s_ex[above]; chi = s_cnt[above]; }
      }
      __syncthreads();
    }
    if (tid % TPE == 0 && tid / TPE < l) {                   // handed to pairs of threads
      const int g = tid / TPE;
      s_x[2 * g] = xlo; s_f[2 * g] = flo; s_ex[2 * g] = elo; s_cnt[2 * g] = clo;
      s_x[2 * g + 1] = xhi; s_f[2 * g + 1] = fhi; s_ex[2 * g + 1] = ehi; s_cnt[2 * g + 1] = chi;
    }
    __syncthreads();
    // Then two threads per eigenvalue.  Once it is alone in its interval the two points stand q of the width to either side of
    // the secant's zero; the secant's error shrinks with the square of the width, so q -> 2 q^2 where the eigenvalue was
    // between them, and thirds after a miss.
    const int g = tid >> 1, sub = tid & 1;
    if (g < l) {
      xlo = s_x[2 * g]; flo = s_f[2 * g]; elo = s_ex[2 * g]; clo = s_cnt[2 * g];
      xhi = s_x[2 * g + 1]; fhi = s_f[2 * g + 1]; ehi = s_ex[2 * g + 1]; chi = s_cnt[2 * g + 1];
      const double tol = 2.3e-16 * bound;
      double q = 0.125;
      bool missed = false;
      for (int round = 0; round < 64 && __any(xhi - xlo > tol); ++round) {
        const SearchPoints at = search_points(flo, elo, fhi, ehi, !missed && chi - clo == 1, q);
        const double x = fma(xhi - xlo, sub ? at.b : at.a, xlo);
        double f; int e;
        const int c = sturm<l>(s_de, x, f, e);
        const double x2 = dpp_move<XOR1>(x), f2 = dpp_move<XOR1>(f);
        const int e2 = __builtin_amdgcn_mov_dpp(e, XOR1, 0xf, 0xf, false), c2 = __builtin_amdgcn_mov_dpp(c, XOR1, 0xf, 0xf, false);
        const double xa = sub ? x2 : x, fa = sub ? f2 : f, xb = sub ? x : x2, fb = sub ? f : f2;
        const int ea = sub ? e2 : e, ca = sub ? c2 : c, eb = sub ? e : e2, cb = sub ? c : c2;
        const bool over_a = ca <= g, over_b = cb <= g;       // the eigenvalue is at the point or above it
        const bool between = over_a != over_b;
        if (over_b) { xlo = xb; flo = fb; elo = eb; clo = cb; }
        else if (over_a) { xlo = xa; flo = fa; elo = ea; clo = ca; }
        if (!over_a) { xhi = xa; fhi = fa; ehi = ea; chi = ca; }
        else if (!over_b) { xhi = xb; fhi = fb; ehi = eb; chi = cb; }
        if (at.secant) q = between ? fmax(2.0 * q * q, 1e-9) : 0.125;
        missed = at.secant && !between;
      }
      if (sub == 0) s_lam[g] = 0.5 * (xlo + xhi);
    }
  }
  __syncthreads();
  bool close = false;
  if (tid < l - 1) close = !(s_lam[tid + 1] - s_lam[tid] > 2e-9 * bound);
  const bool clustered = __syncthreads_or(close);
  if (tid < l) lam[l - 1 - tid] = fmax(s_lam[tid], 0.0) / mscale;
  if constexpr (EIG_HANDS_ON<NE>) {
    if (!clustered) {                          // the vectors are eig_vectors_kernel's
      double* const out = work + (size_t)z * 2 * l * l;
      for_each_block<NE>([&](auto block) {
        constexpr int jb = decltype(block)::value, W = l - 16 * jb;
        for (int i = tid; i < 16 * W; i += EIG_THREADS) out[packed_block<NE>(jb) + i] = Vr[(16 * jb + i / W) * l + 16 * jb + i % W];
      });
      EigHandOn<NE>& on = *reinterpret_cast<EigHandOn<NE>*>(out + packed_block<NE>(NE));
      if (tid <= l) on.de[tid] = s_de[tid];
      if (tid < l) { on.e[tid] = s_e[tid]; on.h[tid] = s_h[tid]; on.lam[tid] = s_lam[tid]; }
      if (tid == 0) { on.bound = bound; on.vectors_wanted = 1; }
      return;
    }
  }

  // Eigenvectors of the tridiagonal matrix: T - lambda = L D+ L^T from the top (lower half of the threads) and U D- U^T
  // from the bottom (upper half), joined at the index k where |gamma_k| is smallest.  The reciprocal pivots go through
  // the scratch in memory, one eigenvector per lane.
  const int half = __builtin_amdgcn_readfirstlane(tid >> 7), g = tid & 127;
  const bool has = g < l;
  const double lg = has ? s_lam[g] : 0.0;
  const double tiny = 1e-30 * bound;
  if (has) {
    auto pivot = [&](double D) { return rcp64(fabs(D) > tiny ? D : copysign(tiny, D)); };
    double r = 0.0;
    if (half == 0) {
#pragma unroll 16
      for (int i = 0; i < l; ++i) Sp[i * l + g] = r = pivot(fma(-s_de[i].y, r, s_de[i].x - lg));
    } else {
#pragma unroll 16
      for (int i = l - 1; i >= 0; --i) Sm[i * l + g] = r = pivot(fma(-s_de[i + 1].y, r, s_de[i].x - lg));
    }
  }
  __syncthreads();
  if (has) {
    double best = INFINITY;
    int at = half * (l / 2);
#pragma unroll 32
    for (int s = 0; s < l / 2; ++s) {
      const int i = half * (l / 2) + s;
      const double up = i > 0 ? Sp[(i > 0 ? i - 1 : 0) * l + g] : 0.0, dn = i + 1 < l ? Sm[(i + 1 < l ? i + 1 : i) * l + g] : 0.0;
      const double ga = fabs((s_de[i].x - lg) - s_de[i].y * up - s_de[i + 1].y * dn);
      if (ga < best) { best = ga; at = i; }
    }
    s_best[half][g] = best; s_at[half][g] = at;
  }
  __syncthreads();
  if (has) {
    const int k = s_best[1][g] < s_best[0][g] ? s_at[1][g] : s_at[0][g];
    double zz = 1.0, sum = half == 0 ? 1.0 : 0.0;
    if (half == 0) {                           // every element is stored (those of the other half's vector as they were): no
      s_k[g] = k;                              // branch keeps the loads from being issued ahead
#pragma unroll 32
      for (int i = l - 1; i >= 0; --i) {
        const double r = Sp[i * l + g];
        double m = -s_e[i] * r;
        asm("" : "+v"(m));                     // computed whether needed or not
        zz *= i < k ? m : 1.0;
        const double t = i < k ? zz : 0.0;
        sum = fma(t, t, sum);
        Sp[i * l + g] = i <= k ? zz : r;
      }
    } else {
#pragma unroll 32
      for (int i = 1; i < l; ++i) {
        const double r = Sm[i * l + g];
        double m = -s_e[i - 1] * r;
        asm("" : "+v"(m));
        zz *= i > k ? m : 1.0;
        const double t = i > k ? zz : 0.0;
        sum = fma(t, t, sum);
        Sm[i * l + g] = i > k ? zz : r;
      }
    }
    s_sum[half][g] = sum;
  }
  __syncthreads();
  if (tid < l) s_inv[tid] = rsqrt64(s_sum[0][tid] + s_sum[1][tid]);
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
#pragma nounroll
    for (int jt = 15; jt >= 1; jt -= 2) {      // H_j, then H_{j-1}: their sums over a vector are taken together
      const int j = 16 * jb + jt;
      const double h1 = s_h[j], h0 = s_h[j - 1];
      double2 w1[NE], w0[NE];
#pragma unroll
      for (int m = jb; m < NE; ++m) {
        w1[m] = *reinterpret_cast<const double2*>(Vr + j * l + 16 * m + 2 * sub);
        w0[m] = *reinterpret_cast<const double2*>(Vr + (j - 1) * l + 16 * m + 2 * sub);
      }
      double d1[NV], d0[NV], c = 0.0;
#pragma unroll
      for (int m = jb; m < NE; ++m) c = fma(w1[m].x, w0[m].x, fma(w1[m].y, w0[m].y, c));
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        d1[v] = d0[v] = 0.0;
#pragma unroll
        for (int m = jb; m < NE; ++m) {
          d1[v] = fma(w1[m].x, u[v][m][0], fma(w1[m].y, u[v][m][1], d1[v]));
          d0[v] = fma(w0[m].x, u[v][m][0], fma(w0[m].y, u[v][m][1], d0[v]));
        }
      }
      auto sum8 = [](double x) { x += dpp_move<XOR1>(x); x += dpp_move<XOR2>(x); return x + dpp_move<XOR7>(x); };
      c = sum8(c);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        d1[v] = -h1 * sum8(d1[v]);
        d0[v] = -h0 * fma(d1[v], c, sum8(d0[v]));
#pragma unroll
        for (int m = jb; m < NE; ++m) {
          u[v][m][0] = fma(d0[v], w0[m].x, fma(d1[v], w1[m].x, u[v][m][0]));
          u[v][m][1] = fma(d0[v], w0[m].y, fma(d1[v], w1[m].y, u[v][m][1]));
        }
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
  if constexpr (EIG_HANDS_ON<NE>) {
    if (tid == 0) reinterpret_cast<EigHandOn<NE>*>(work + (size_t)z * 2 * l * l + packed_block<NE>(NE))->vectors_wanted = 0;
  }
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

// Eigenvectors 16 b .. 16 b + 15 (ascending) of a problem whose tridiagonal form and eigenvalues sym_eig_kernel has handed on:
// the same twisted factorisation, two lanes of the first wavefront per vector, with the pivots in LDS, while the reflectors are on their way;
// then 16 lanes per vector apply those, entries 32 m + 2 tx + {0, 1}.
template <int NE>
__global__ __launch_bounds__(EIG_THREADS, 2) void eig_vectors_kernel(const double* __restrict__ work, float* __restrict__ Utall) {
  constexpr int l = 16 * NE, PK = packed_block<NE>(NE);
  extern __shared__ __attribute__((aligned(16))) double lds[];
  double* piv = lds;                                         // pivots, [2][l][16]
  double* Vp = lds;                                          // then the packed reflectors
  __shared__ double2 s_de[l + 1];
  __shared__ double s_e[l], s_h[l], s_best[16][16], s_sum[2][16];
  __shared__ int s_at[16][16], s_k[16];
  const int b = blockIdx.x, z = blockIdx.y, tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  float* Ut = Utall + (size_t)z * l * l;
  const double* in = work + (size_t)z * 2 * l * l;
  const EigHandOn<NE>& on = *reinterpret_cast<const EigHandOn<NE>*>(in + PK);
  if (on.vectors_wanted != 1) return;                        // the same for all of the problem's workgroups
  __builtin_amdgcn_s_setprio(3);
  if (tid <= l) s_de[tid] = on.de[tid];
  if (tid < l) { s_e[tid] = on.e[tid]; s_h[tid] = on.h[tid]; }
  const double bound = on.bound, tiny = 1e-30 * bound, lg = on.lam[16 * b + tx];
  constexpr int PIECES = (PK / 2 + EIG_THREADS - 1) / EIG_THREADS;
  doublex2 held[PIECES];                                     // in flight behind the factorisation, whose LDS they take over
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int at = tid + EIG_THREADS * i;
    held[i] = reinterpret_cast<const doublex2*>(in)[at < PK / 2 ? at : 0];
  }
  __syncthreads();
  const int half = ty & 1;                                   // 0: from the top, 1: from the bottom
  if (tid < 32) {
    auto pivot = [&](double D) { return rcp64(fabs(D) > tiny ? D : copysign(tiny, D)); };
    const int step = half ? -1 : 1, first = half ? l - 1 : 0;
    double r = 0.0;
#pragma nounroll
    for (int s0 = 0; s0 < l; s0 += 16) {       // loads by hand in front of stores that they might alias for all the compiler knows
      const int i0 = first + step * s0;
      double x[16], y[16];
#pragma unroll
      for (int s = 0; s < 16; ++s) { x[s] = s_de[i0 + step * s].x - lg; y[s] = -s_de[i0 + step * s + half].y; }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        r = pivot(fma(y[s], r, x[s]));
        piv[(half * l + i0 + step * s) * 16 + tx] = r;
      }
    }
  }
  __syncthreads();
  {
    double best = INFINITY;
    int at = ty;
#pragma unroll
    for (int s = 0; s < NE; ++s) {
      const int i = ty + 16 * s;
      const double up = i > 0 ? piv[(i > 0 ? i - 1 : 0) * 16 + tx] : 0.0, dn = i + 1 < l ? piv[(l + (i + 1 < l ? i + 1 : i)) * 16 + tx] : 0.0;
      const double ga = fabs((s_de[i].x - lg) - s_de[i].y * up - s_de[i + 1].y * dn);
      if (ga < best) { best = ga; at = i; }
    }
    s_best[ty][tx] = best; s_at[ty][tx] = at;
  }
  __syncthreads();
  if (tid < 32) {
    double best = s_best[0][tx];
    int k = s_at[0][tx];
#pragma unroll
    for (int p = 1; p < 16; ++p)
      if (s_best[p][tx] < best) { best = s_best[p][tx]; k = s_at[p][tx]; }
    if (half == 0) s_k[tx] = k;
    double zz = 1.0, sum = half == 0 ? 1.0 : 0.0;
    const int step = half ? 1 : -1, first = half ? 0 : l - 1;
#pragma nounroll
    for (int s0 = 0; s0 < l; s0 += 16) {       // away from k; every element is stored, those of the other half as they were
      const int i0 = first + step * s0;
      double* at = piv + (half * l + i0) * 16 + tx;
      double r[16], m[16];
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const int ie = i0 + step * s - half;
        r[s] = at[16 * step * s];
        m[s] = -s_e[ie > 0 ? ie : 0] * r[s];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const int i = i0 + step * s;
        const bool mine = half ? i > k : i < k;
        zz *= mine ? m[s] : 1.0;
        const double t = mine ? zz : 0.0;
        sum = fma(t, t, sum);
        at[16 * step * s] = mine || i == k ? zz : r[s];
      }
    }
    s_sum[half][tx] = sum;
  }
  __syncthreads();
  const int k = s_k[ty], M = NE / 2;
  const double inv = rsqrt64(s_sum[0][ty] + s_sum[1][ty]);
  double u[NE / 2][2];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = 32 * m + 2 * tx + q;
      u[m][q] = piv[((i <= k ? 0 : l) + i) * 16 + ty] * inv;
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int at = tid + EIG_THREADS * i;
    if (at < PK / 2) reinterpret_cast<doublex2*>(Vp)[at] = held[i];
  }
  __syncthreads();
  for_each_block_down<NE>([&](auto block) {
    constexpr int jb = decltype(block)::value, W = l - 16 * jb, M0 = jb / 2;
    const double* rows = Vp + packed_block<NE>(jb);
    double h1, h0, n1, n0;
    double2 w1[NE / 2], w0[NE / 2], next1[NE / 2], next0[NE / 2];
    auto fetch = [&](int jt) {
      n1 = s_h[16 * jb + jt]; n0 = s_h[16 * jb + jt - 1];
#pragma unroll
      for (int m = M0; m < NE / 2; ++m) {
        const int at = (jb & 1) && m == M0 && tx < 8 ? 0 : 32 * m + 2 * tx - 16 * jb;
        next1[m] = *reinterpret_cast<const double2*>(rows + jt * W + at);
        next0[m] = *reinterpret_cast<const double2*>(rows + (jt - 1) * W + at);
      }
    };
    fetch(15);
#pragma nounroll
    for (int jt = 15; jt >= 1; jt -= 2) {      // H_j, then H_{j-1}: their sums over a vector are taken together
      h1 = n1; h0 = n0;
#pragma unroll
      for (int m = M0; m < NE / 2; ++m) {
        const bool before = (jb & 1) && m == M0 && tx < 8;                 // columns in front of the block row
        w1[m] = before ? make_double2(0.0, 0.0) : next1[m];
        w0[m] = before ? make_double2(0.0, 0.0) : next0[m];
      }
      fetch(jt > 2 ? jt - 2 : 1);
      __builtin_amdgcn_sched_barrier(0);
      double c = 0.0, d1 = 0.0, d0 = 0.0;
#pragma unroll
      for (int m = M0; m < NE / 2; ++m) {
        c = fma(w1[m].x, w0[m].x, fma(w1[m].y, w0[m].y, c));
        d1 = fma(w1[m].x, u[m][0], fma(w1[m].y, u[m][1], d1));
        d0 = fma(w0[m].x, u[m][0], fma(w0[m].y, u[m][1], d0));
      }
      auto sum16 = [](double x) {
        x += dpp_move<XOR1>(x); x += dpp_move<XOR2>(x); x += dpp_move<XOR7>(x);
        return x + dpp_move<XOR15>(x);
      };
      c = sum16(c);
      d1 = -h1 * sum16(d1);
      d0 = -h0 * fma(d1, c, sum16(d0));
#pragma unroll
      for (int m = M0; m < NE / 2; ++m) {
        u[m][0] = fma(d0, w0[m].x, fma(d1, w1[m].x, u[m][0]));
        u[m][1] = fma(d0, w0[m].y, fma(d1, w1[m].y, u[m][1]));
      }
    }
  });
#pragma unroll
  for (int m = 0; m < M; ++m)
    *reinterpret_cast<float2*>(Ut + (size_t)(l - 1 - 16 * b - ty) * l + 32 * m + 2 * tx) = make_float2((float)u[m][0], (float)u[m][1]);
}

bool sym_eig_supported(int l) { return l % 32 == 0 && l >= 32 && l <= 128; }

template <int NE>
static int launch_eig(const double* G, double* work, float* Ut, double* lambda, int batch, hipStream_t st) {
  constexpr int l = 16 * NE;
  const size_t reflectors = (size_t)l * l * (NE <= 4 ? 3 : 1) * sizeof(double), jacobi = (size_t)2 * l * (l + 4) * sizeof(float);
  const size_t rows = (size_t)l * (l + 2) * sizeof(double);
  const size_t need = std::max(reflectors, std::max(jacobi, rows));
  static LdsLimit limit;
  LQ_TRY(limit.raise(reinterpret_cast<const void*>(sym_eig_kernel<NE>), need));
  hipLaunchKernelGGL((sym_eig_kernel<NE>), dim3(batch), dim3(EIG_THREADS), need, st, G, work, Ut, lambda);
  LQ_HIP_TRY(hipGetLastError());
  if constexpr (EIG_HANDS_ON<NE>) {
    constexpr size_t lds = (size_t)std::max(packed_block<NE>(NE), 32 * l) * sizeof(double);
    if constexpr (lds > 57344) {               // beside what the kernel has without asking
      static LdsLimit vectors;
      LQ_TRY(vectors.raise(reinterpret_cast<const void*>(eig_vectors_kernel<NE>), lds));
    }
    hipLaunchKernelGGL((eig_vectors_kernel<NE>), dim3(NE, batch), dim3(EIG_THREADS), lds, st, work, Ut);
    LQ_HIP_TRY(hipGetLastError());
  }
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
