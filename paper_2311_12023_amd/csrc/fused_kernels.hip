// Fused kernels of one LQ iteration (Algorithm 2):  Q <- Quantize(W - L1 L2, c)  and the error
// eps_t = || sqrt(F) .* (W - Q - L1 L2) ||_F, for a lock-step batch of configurations that share W.
//
// The residual T = W - L1 L2 is never written to memory.  Three phases, because the reconstructed block
// scale needs the absmax of a whole scale group (B0*B1 consecutive weights, which in general straddles
// rows) while T is produced in 2-D MFMA tiles:
//   1  per 64x128 tile: L1 L2 by MFMA (K = rank), T, block absmax s, codes against s (the codes depend on
//      the exact block absmax only), and three sums per block from which the error follows for any
//      reconstructed scale s^ = s + delta:  sum w (t - q s^)^2 = e2 - 2 delta eq + delta^2 q2.
//   2  per scale group: v = max s, scale indices, cast of v, and the error of the iteration.
//   3  per weight: R = D_row (W - Q) D_col, the input of the next Factorize (and / or dense Q).
#include "kernels.h"
#include "nf_device.h"
#include "profiler.h"

namespace lq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int TM = 64;     // tile rows
constexpr int TN = 128;    // tile columns
constexpr int PP = TN + 4; // pitch of the product tile in LDS
constexpr int KC = 32;     // rank chunk staged in LDS
constexpr int NTHR1 = 512; // threads of the phase-1 workgroup: 8 wavefronts, one 32x32 MFMA tile each
constexpr int KC2 = 64;    // rank chunk of the split-precision product
constexpr int KP = KC2 + 8;// LDS row pitch of its operand planes in bf16 elements (144 B: conflict-free b128 reads)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------------
// Split-precision operands of L1 L2 = Y_r^T B_r: every factor entry x is stored as bf16 hi + bf16 lo
// (x = hi + lo + O(2^-17 x)), transposed so that the reduction index is contiguous:
//   plane[i][p], i < rows_pad (zero rows past the matrix), p < RK = round_up16(rank) (zeros past the rank);
// per problem: Y hi, Y lo (dpad x RK each), then B hi, B lo (kpad x RK each).
int64_t packed_rows_y(int64_t d) { return (d + TM - 1) / TM * TM; }
int64_t packed_rows_b(int64_t k) { return (k + TN - 1) / TN * TN; }
int packed_rank(int rank) { return (rank + 15) / 16 * 16; }
size_t packed_factor_elems(int64_t d, int64_t k, int rank) {
  return (size_t)2 * (packed_rows_y(d) + packed_rows_b(k)) * packed_rank(rank);
}

// Bound by memory (both factors once in 32 bits, once out as two 16-bit planes).  A workgroup transposes PACK_ROWS rows
// through LDS so that loads run along the factor's rows and stores are contiguous; a thread per row stored 16 bytes every
// 2 RK bytes (12 problems of 4096 + 4096 rows, rank 64,
// beside two other streams: 78 -> 46 us per launch).
constexpr int PACK_ROWS = 32, PACK_MAX_RANK = 128;
static_assert(TM % PACK_ROWS == 0 && TN % PACK_ROWS == 0, "a workgroup's rows belong to one factor");
__global__ __launch_bounds__(256) void pack_factors_kernel(PhaseArgs a, int64_t dpad, int64_t kpad, int rk) {
  __shared__ float s_x[PACK_MAX_RANK][PACK_ROWS + 1];
  const int z = blockIdx.y, tid = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * PACK_ROWS;                 // rows of the packed planes, Y rows first
  const bool isy = i0 < dpad;                                         // dpad and kpad are multiples of PACK_ROWS
  const int64_t r0 = isy ? i0 : i0 - dpad, rows = isy ? dpad : kpad, lim = isy ? a.d : a.k, ld = isy ? a.ldy : a.ldb;
  const float* src = (isy ? a.Y + (size_t)z * a.strideY : a.B + (size_t)z * a.strideB) + r0;
  __bf16* hi = reinterpret_cast<__bf16*>(a.packed) + (size_t)z * a.stridePacked + (isy ? 0 : (size_t)2 * dpad * rk) +
               (size_t)r0 * rk;
  __bf16* lo = hi + (size_t)rows * rk;
  for (int idx = tid; idx < rk * PACK_ROWS; idx += 256) {
    const int p = idx / PACK_ROWS, r = idx % PACK_ROWS;
    s_x[p][r] = (r0 + r < lim && p < a.rank) ? src[(size_t)p * ld + r] : 0.0f;
  }
  __syncthreads();
  const int units = rk >> 3;
  for (int idx = tid; idx < units * PACK_ROWS; idx += 256) {
    const int r = idx / units, p0 = 8 * (idx % units);
    bf16x8 h, l;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = s_x[p0 + e][r];
      const __bf16 xh = (__bf16)x;
      h[e] = xh;
      l[e] = (__bf16)(x - (float)xh);
    }
    *reinterpret_cast<bf16x8*>(hi + (size_t)8 * idx) = h;
    *reinterpret_cast<bf16x8*>(lo + (size_t)8 * idx) = l;
  }
}

int launch_pack_factors(const PhaseArgs& a, hipStream_t st) {
  const int64_t dpad = packed_rows_y(a.d), kpad = packed_rows_b(a.k);
  if (packed_rank(a.rank) > PACK_MAX_RANK) return LQ_ERR_RANK;
  prof::Scope ps(prof::MISC, st, (double)(a.d + a.k) * a.rank * 8.0 * a.batch);
  hipLaunchKernelGGL(pack_factors_kernel, dim3((unsigned)((dpad + kpad) / PACK_ROWS), (unsigned)a.batch), dim3(256), 0, st,
                     a, dpad, kpad, packed_rank(a.rank));
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// Stores the 4 codes of one quad.  `base`: address of the codes of a quad whose index is a multiple of 4 (uniform across
// the wavefront in phase 1), `lq`: this lane's quad index relative to it.  2, 4, 8 bits: 1, 2, 4 bytes per lane,
// contiguous across lanes.  3 bits: the four lanes of a 16-weight run gather their 12-bit pieces into the run's 48-bit
// word and three of them store 16 bits each.  All 64 lanes must call (cross-lane exchange inside).
template <int BITS>
__device__ __forceinline__ void store_quad_codes(uint8_t* __restrict__ base, uint32_t lq, const uint32_t (&c)[4],
                                                 bool live) {
  const uint32_t w = c[0] | (c[1] << BITS) | (c[2] << (2 * BITS)) | (c[3] << (3 * BITS));
  if constexpr (BITS == 8) {
    if (live) *reinterpret_cast<uint32_t*>(base + lq * 4u) = w;
  } else if constexpr (BITS == 4) {
    if (live) *reinterpret_cast<uint16_t*>(base + lq * 2u) = (uint16_t)w;
  } else if constexpr (BITS == 2) {
    if (live) base[lq] = (uint8_t)w;
  } else {
    const int sub = threadIdx.x & 3;
    uint32_t lo = sub < 2 ? (w << (12 * sub)) : (sub == 2 ? (w << 24) : 0u);        // bits 0..31 of the run word
    uint32_t hi = sub == 2 ? (w >> 8) : (sub == 3 ? (w << 4) : 0u);                 // bits 32..47
    lo |= dpp_move_u32<DPP_QUAD_XOR1>(lo); hi |= dpp_move_u32<DPP_QUAD_XOR1>(hi);
    lo |= dpp_move_u32<DPP_QUAD_XOR2>(lo); hi |= dpp_move_u32<DPP_QUAD_XOR2>(hi);
    if (live && sub < 3) {
      const uint16_t piece = sub == 0 ? (uint16_t)lo : (sub == 1 ? (uint16_t)(lo >> 16) : (uint16_t)hi);
      *reinterpret_cast<uint16_t*>(base + (lq >> 2) * 6u + 2u * sub) = piece;
    }
  }
}

// Copies the search table of phase 1 to LDS.
__device__ __forceinline__ void load_search_nosync(const DevTables* __restrict__ tab, int slot, SearchEntry* s_search) {
  const int n = slot == Slot<8>::value ? search_entries(8) : search_entries(4);
  for (int j = threadIdx.x; j < n; j += blockDim.x) s_search[j] = tab->search[slot][j];
}

// max |t| of a quad, as the bit pattern of a non-negative float (unsigned order = numeric order).
__device__ __forceinline__ uint32_t quad_absmax_bits(const float (&t)[4]) {
  float m;
  asm("v_max3_f32 %0, |%1|, |%2|, |%3|\n\tv_max_f32 %0, |%4|, %0" : "=&v"(m) : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]));
  return __float_as_uint(m);
}
// Reductions over the QPB = 4, 8, 16 or 32 lanes that hold a block, for the four quads of a lane at once (lane i of every
// hardware quad, 4 consecutive lanes, ends with the result of quad i): the two steps inside a hardware quad hand half of the
// values to the partner, so four results take the moves of less than two.  Beyond it lanes meet others of the same i: the
// half-row mirror with the quads' order put back is xor 4, a rotation of a row by 8 is xor 8.
constexpr int DPP_QUAD_REVERSE = 0x1B, DPP_ROW_ROR8 = 0x128;
template <int QPB, typename T, typename Op>
__device__ __forceinline__ T block_reduce_dealt(const T (&v)[4], bool odd, bool high, Op op) {
  auto move = [](T x, auto ctrl) __attribute__((always_inline)) {
    return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
#define LQ_MOVE(X, CTRL) move(X, std::integral_constant<int, CTRL>{})
  const T a = op(odd ? v[1] : v[0], LQ_MOVE(odd ? v[0] : v[1], DPP_QUAD_XOR1));
  const T b = op(odd ? v[3] : v[2], LQ_MOVE(odd ? v[2] : v[3], DPP_QUAD_XOR1));
  T x = op(high ? b : a, LQ_MOVE(high ? a : b, DPP_QUAD_XOR2));
  if constexpr (QPB >= 8) x = op(x, LQ_MOVE(LQ_MOVE(x, DPP_ROW_HALF_MIRROR), DPP_QUAD_REVERSE));
  if constexpr (QPB >= 16) x = op(x, LQ_MOVE(x, DPP_ROW_ROR8));
  if constexpr (QPB >= 32) x = op(x, __builtin_bit_cast(T, __shfl_xor(__builtin_bit_cast(int, x), 16)));
#undef LQ_MOVE
  return x;
}
// Value of lane I of each hardware quad.
template <int I>
__device__ __forceinline__ float quad_lane(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x55 * I, 0xf, 0xf, true));
}

// What a lane of phase 1 holds of W and of the Fisher scales beside its product tile: its four quads (rows tid / 32 + 16 u),
// 1/sqrt(row_w) of their rows, 1/sqrt(col_w) and col_w of their columns.
struct PhaseQuads { float4 w[4]; float rs[4]; float4 rc, cw; };

// Epilogue of phase 1 in quad layout: lane `tid` handles quads tid, tid+512, ... of the 64 x 128 tile (32 quads
// per row), so W loads, LDS reads of the product and code stores are all contiguous across lanes.  QPB = B0/4
// lanes hold one block.  The four quads of a lane lie in four different blocks; their block maxima are found first,
// then one division serves all four (lane i of every hardware quad has the maximum of quad i and divides, the quotients go back
// by quad broadcasts: the four lanes of a hardware quad always share their blocks), then the codes.  Blocks lie
// inside the matrix or outside it, so whatever the quads past its edge hold stays there and is never stored.
template <int BITS, int QPB, bool WITH_ERR, bool WEIGHTED>
__device__ __forceinline__ void phase1_epilogue(const PhaseArgs& a, int z, const float* pt, const SearchEntry* s_search,
                                                const float* s_code, int64_t r0, int64_t c0, const PhaseQuads& in) {
  const int tid = threadIdx.x, sub = tid & 3;
  const bool odd = sub & 1, high = sub & 2;
  uint8_t* codes = a.codes + (size_t)z * a.strideCodes;
  BlockRec* blk = a.blk + (size_t)z * a.strideBlk;
  // quad indices: a uniform part per quad u (first quad of the tile, NTHR1 / 32 rows further down for each u) plus a
  // 32-bit lane part; both are multiples of QPB where a block starts, so block indices split the same way
  const int cq = tid & 31;
  const int64_t tq0 = (r0 * a.k + c0) >> 2;
  const uint32_t quad_step = (uint32_t)((NTHR1 / 32) * (a.k >> 2));
  const uint32_t lq = (uint32_t)((tid >> 5) * (a.k >> 2) + cq);
  constexpr int CODE_BYTES_X2 = BITS;            // bytes per quad = BITS / 2
  const bool col_live = c0 + 4 * cq < a.k;
  const int rows_left = (int)(a.d - r0 < TM ? a.d - r0 : TM) - (tid >> 5);
  float t[4][4];
  uint32_t qmax[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int lr = (tid >> 5) + (NTHR1 / 32) * u;
    const float4 p = *reinterpret_cast<const float4*>(pt + lr * PP + 4 * cq);
    float pv[4] = {p.x, p.y, p.z, p.w};
    const float fv[4] = {in.w[u].x, in.w[u].y, in.w[u].z, in.w[u].w};
    if constexpr (WEIGHTED) {
      const float rs = in.rs[u];
      pv[0] *= rs * in.rc.x; pv[1] *= rs * in.rc.y; pv[2] *= rs * in.rc.z; pv[3] *= rs * in.rc.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) t[u][e] = fv[e] - pv[e];
    qmax[u] = quad_absmax_bits(t[u]);
  }
  const float mine = __uint_as_float(block_reduce_dealt<QPB>(qmax, odd, high, [](uint32_t x, uint32_t y) { return x > y ? x : y; }));
  const float rmine = safe_reciprocal(mine);
  const float rcp[4] = {quad_lane<0>(rmine), quad_lane<1>(rmine), quad_lane<2>(rmine), quad_lane<3>(rmine)};
  const float amax[4] = {quad_lane<0>(mine), quad_lane<1>(mine), quad_lane<2>(mine), quad_lane<3>(mine)};
  float e2[4], eq[4], q2[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    uint32_t c[4];
    e2[u] = eq[u] = q2[u] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c[e] = search_code<BITS>(s_search, t[u][e] * rcp[u]);
      if constexpr (WITH_ERR) {
        const float q = s_code[c[e]];
        const float err = t[u][e] - q * amax[u];
        float werr = err, wq = q;
        if constexpr (WEIGHTED) {
          const float w = e == 0 ? in.cw.x : e == 1 ? in.cw.y : e == 2 ? in.cw.z : in.cw.w;
          werr = w * err; wq = w * q;
        }
        e2[u] = fmaf(werr, err, e2[u]);
        eq[u] = fmaf(werr, q, eq[u]);
        q2[u] = fmaf(wq, q, q2[u]);
      }
    }
    const int64_t quad_u = tq0 + (int64_t)u * quad_step;                   // uniform
    store_quad_codes<BITS>(codes + ((quad_u * CODE_BYTES_X2) >> 1), lq, c, col_live && (NTHR1 / 32) * u < rows_left);
  }
  // lane i of a block's first hardware quad stores the record of quad i
  const bool writes = col_live && (cq & (QPB - 1)) < 4 && (NTHR1 / 32) * sub < rows_left;
  const uint32_t at = (uint32_t)sub * (quad_step / QPB) + lq / QPB;
  if constexpr (WITH_ERR) {
    auto add = [](float x, float y) { return x + y; };
    BlockRec rec;
    rec.s = mine;
    rec.e2 = block_reduce_dealt<QPB>(e2, odd, high, add);
    rec.eq = block_reduce_dealt<QPB>(eq, odd, high, add);
    rec.q2 = block_reduce_dealt<QPB>(q2, odd, high, add);
    if (writes) (blk + tq0 / QPB)[at] = rec;
  } else {
    if (writes) (reinterpret_cast<float*>(blk) + tq0 / QPB)[at] = mine;    // without error sums a record is the absmax alone
  }
}

template <int BITS, bool WITH_ERR, bool WEIGHTED>
__device__ __forceinline__ void phase1_dispatch_block(const PhaseArgs& a, int block, int z, const float* pt,
                                                      const SearchEntry* s_search, const float* s_code, int64_t r0,
                                                      int64_t c0, const PhaseQuads& in) {
  switch (block) {
    case 16: phase1_epilogue<BITS, 4, WITH_ERR, WEIGHTED>(a, z, pt, s_search, s_code, r0, c0, in); break;
    case 32: phase1_epilogue<BITS, 8, WITH_ERR, WEIGHTED>(a, z, pt, s_search, s_code, r0, c0, in); break;
    case 64: phase1_epilogue<BITS, 16, WITH_ERR, WEIGHTED>(a, z, pt, s_search, s_code, r0, c0, in); break;
    default: phase1_epilogue<BITS, 32, WITH_ERR, WEIGHTED>(a, z, pt, s_search, s_code, r0, c0, in); break;
  }
}
template <bool WITH_ERR, bool WEIGHTED>
__device__ __forceinline__ void phase1_dispatch(const PhaseArgs& a, const lq_config& cfg, int z, const float* pt, const SearchEntry* s_search,
                                                const float* s_code, int64_t r0, int64_t c0, const PhaseQuads& in) {
  switch (cfg.bits) {
    case 2: phase1_dispatch_block<2, WITH_ERR, WEIGHTED>(a, cfg.block, z, pt, s_search, s_code, r0, c0, in); break;
    case 3: phase1_dispatch_block<3, WITH_ERR, WEIGHTED>(a, cfg.block, z, pt, s_search, s_code, r0, c0, in); break;
    case 4: phase1_dispatch_block<4, WITH_ERR, WEIGHTED>(a, cfg.block, z, pt, s_search, s_code, r0, c0, in); break;
    default: phase1_dispatch_block<8, WITH_ERR, WEIGHTED>(a, cfg.block, z, pt, s_search, s_code, r0, c0, in); break;
  }
}

// The quads of W and the row scales of the band of TM rows at r0, columns from c0; rows and columns past the matrix repeat the
// last row and the first column of the stretch.  Addresses are a uniform base per quad plus a 32-bit lane offset (rows of a band are
// at most 63 apart).
template <bool WEIGHTED>
__device__ __forceinline__ void fetch_phase_quads(const PhaseArgs& a, int64_t r0, int64_t c0, PhaseQuads& q) {
  const int tr = threadIdx.x >> 5;
  const uint32_t col = c0 + 4 * (threadIdx.x & 31) < a.k ? 4 * (threadIdx.x & 31) : 0;
  int row[4] = {tr, tr, tr, tr};
  uint32_t off[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) off[u] = (uint32_t)((tr * a.k + col) * 4);
  if (r0 + TM > a.d) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t left = a.d - 1 - (r0 + (NTHR1 / 32) * u);
      row[u] = left > 0 ? (tr < left ? tr : (int)left) : 0;
      off[u] = (uint32_t)((row[u] * a.k + col) * 4);
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t ru = r0 + (NTHR1 / 32) * u, row_u = ru < a.d ? ru : a.d - 1;              // uniform
    q.w[u] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(a.W + (size_t)row_u * a.k + c0) + off[u]);
    if constexpr (WEIGHTED) q.rs[u] = (a.rsr + row_u)[row[u]];
  }
}
template <bool WITH_ERR>
__device__ __forceinline__ void fetch_phase_columns(const PhaseArgs& a, int64_t c0, PhaseQuads& q) {
  const int64_t col = c0 + (c0 + 4 * (threadIdx.x & 31) < a.k ? 4 * (threadIdx.x & 31) : 0);
  q.rc = *reinterpret_cast<const float4*>(a.rsc + col);
  if constexpr (WITH_ERR) q.cw = *reinterpret_cast<const float4*>(a.col_w + col);
}

// SPLIT: L1 L2 from the packed bf16 hi/lo planes with three v_mfma_f32_32x32x16_bf16 per 16-deep group
// (hi*hi + hi*lo + lo*hi, fp32 accumulation; products good to about 2^-16 relative) instead of fp32 MFMAs.
// Launch: one-dimensional, batch * tiles8 workgroups (tiles8 = number of 64 x 128 tiles rounded up to a multiple
// of 8).  Workgroups go to the 8 XCDs round-robin by index; the index is decoded as (tile mod 8, problem, tile div 8),
// so the problems of a batch that share a tile of W run on one XCD and fetch it into that XCD's L2 once.
template <bool WITH_ERR, bool SPLIT, bool WEIGHTED>
__global__ __launch_bounds__(NTHR1) void lowrank_blockquant_kernel(PhaseArgs a, int tiles, int tiles_n) {
  // The operand chunks and the product tile share one LDS buffer: the product is written after the last MFMA has
  // read its operands.  fp32: Y chunk KC x TM, B chunk KC x TN.  Split: four planes (Y hi, Y lo: TM rows; B hi, B lo:
  // TN rows) of KC2 reduction indices, pitch KP.
  constexpr int SMEM_FLOATS = SPLIT ? ((2 * (TM + TN) * KP * 2 + 3) / 4 > TM * PP ? (2 * (TM + TN) * KP * 2 + 3) / 4 : TM * PP)
                                    : TM * PP;
  __shared__ __attribute__((aligned(16))) float smem[SMEM_FLOATS];
  __shared__ __attribute__((aligned(16))) SearchEntry s_search[SEARCH_ENTRIES];
  __shared__ float s_code[WITH_ERR ? 256 : 1];
  float* pt = smem;
  static_assert(KC * TM + KC * TN <= TM * PP, "operand chunks must fit in the product tile");
  const int tid = threadIdx.x;
  const int slot8 = blockIdx.x >> 3;
  const int z = slot8 % a.batch;
  const int tile = (int)(blockIdx.x & 7) + 8 * (slot8 / a.batch);
  if (tile >= tiles) return;                   // padding of the tile count to a multiple of 8
  const LoopProblem pr = a.prob[z];
  const int64_t r0 = (int64_t)(tile / tiles_n) * TM, c0 = (int64_t)(tile % tiles_n) * TN;
  const int wave = tid >> 6, lane = tid & 63, ln = lane & 31, lh = lane >> 5;
  const int wr = wave >> 2, wc = wave & 3;      // 2 x 4 grid of 32x32 tiles

  // search table (and, for the error sums, the code book) of this problem's bit width, visible after the barriers of
  // the product stage
  const int slot = pr.cfg.bits == 2 ? 0 : pr.cfg.bits == 3 ? 1 : pr.cfg.bits == 4 ? 2 : 3;
  load_search_nosync(a.tables, slot, s_search);
  if constexpr (WITH_ERR)
    for (int i = tid; i < 256; i += NTHR1) s_code[i] = a.tables->code[slot][i];
  // this lane's 4 quads of W, fetched now so that the loads overlap the MFMA stage
  PhaseQuads quads;
  fetch_phase_quads<WEIGHTED>(a, r0, c0, quads);
  if constexpr (WEIGHTED) fetch_phase_columns<WITH_ERR>(a, c0, quads);

  floatx16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;

  if constexpr (SPLIT) {
    __bf16* planes = reinterpret_cast<__bf16*>(smem);          // [Yh | Yl | Bh | Bl], rows x KP
    const int rk = (a.rank + 15) / 16 * 16;
    const int64_t dpad = (a.d + TM - 1) / TM * TM, kpad = (a.k + TN - 1) / TN * TN;
    const __bf16* gy = reinterpret_cast<const __bf16*>(a.packed) + (size_t)z * a.stridePacked;
    const __bf16* gb = gy + (size_t)2 * dpad * rk;
    // piece idx = tid + 512 i, i < 6: 16 bytes (8 reduction indices) of one row of one plane.  Rows tid / 8 + 64 i of the
    // stacked planes [Yh | Yl | Bh | Bl]: piece i always falls into the same plane, at row (tid / 8) (+ 64 for the second
    // half of a B plane), so its address is a uniform base plus the lane offset all pieces share.
    constexpr int PIECES = 2 * (TM + TN) * (KC2 / 8) / NTHR1;
    static_assert(PIECES == 6 && TM == 64 && TN == 128 && NTHR1 == 512, "piece-to-plane map below");
    floatx4 st[PIECES];
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const uint32_t p_lane = (uint32_t)(((tid >> 3) * rk + 8 * (tid & 7)) * 2);
    const char* pbase[PIECES] = {
        reinterpret_cast<const char*>(gy + (size_t)r0 * rk),                   // Y hi
        reinterpret_cast<const char*>(gy + (size_t)(dpad + r0) * rk),          // Y lo
        reinterpret_cast<const char*>(gb + (size_t)c0 * rk),                   // B hi, rows 0..63
        reinterpret_cast<const char*>(gb + (size_t)(c0 + 64) * rk),            // B hi, rows 64..127
        reinterpret_cast<const char*>(gb + (size_t)(kpad + c0) * rk),          // B lo, rows 0..63
        reinterpret_cast<const char*>(gb + (size_t)(kpad + c0 + 64) * rk)};    // B lo, rows 64..127
    auto fetch_planes = [&](int k0) {
      const bool ok = k0 + 8 * (tid & 7) < rk;
#pragma unroll
      for (int i = 0; i < PIECES; ++i)
        st[i] = ok ? *reinterpret_cast<const floatx4*>(pbase[i] + p_lane + 2 * k0) : zero4;
    };
    fetch_planes(0);
    for (int k0 = 0; k0 < rk; k0 += KC2) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PIECES; ++i) {
        const int idx = tid + NTHR1 * i;
        *reinterpret_cast<floatx4*>(planes + (size_t)(idx >> 3) * KP + 8 * (idx & 7)) = st[i];
      }
      __syncthreads();
      if (k0 + KC2 < rk) fetch_planes(k0 + KC2);
      const __bf16* yh = planes + (size_t)(32 * wr + ln) * KP + 8 * lh;
      const __bf16* yl = yh + (size_t)TM * KP;
      const __bf16* bh = planes + (size_t)(2 * TM + 32 * wc + ln) * KP + 8 * lh;
      const __bf16* bl = bh + (size_t)TN * KP;
#pragma unroll
      for (int kg = 0; kg < KC2 / 16; ++kg) {
        if (k0 + 16 * kg < rk) {
          const bf16x8 ah = *reinterpret_cast<const bf16x8*>(yh + 16 * kg), al = *reinterpret_cast<const bf16x8*>(yl + 16 * kg);
          const bf16x8 vh = *reinterpret_cast<const bf16x8*>(bh + 16 * kg), vl = *reinterpret_cast<const bf16x8*>(bl + 16 * kg);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, vh, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, vl, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, vh, acc, 0, 0, 0);
        }
      }
    }
  } else {
    float (*ys)[TM] = reinterpret_cast<float (*)[TM]>(smem);
    float (*bs)[TN] = reinterpret_cast<float (*)[TN]>(smem + KC * TM);
    const float* __restrict__ Y = a.Y + (size_t)z * a.strideY;
    const float* __restrict__ B = a.B + (size_t)z * a.strideB;
    // operand chunk staging through registers, 128-bit pieces: piece idx = tid + 512*i of the chunk.  The wide
    // bases have at least round_up32(rank) rows and zero-padded leading dimensions, so only the column offset
    // needs clamping; rows past `rank` and columns past the matrix are replaced by zeros after the load.
    floatx4 yst[KC * TM / (4 * NTHR1)], bst[KC * TN / (4 * NTHR1)];
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    auto fetch_chunk = [&](int k0) {
#pragma unroll
      for (int i = 0; i < KC * TM / (4 * NTHR1); ++i) {
        const int idx = tid + NTHR1 * i, kk = idx / (TM / 4), rr = 4 * (idx % (TM / 4));
        const int64_t off = r0 + rr;
        const bool ok = k0 + kk < a.rank && off < a.d;
        const floatx4 v = *reinterpret_cast<const floatx4*>(Y + (size_t)(k0 + kk) * a.ldy + (off + 4 <= a.ldy ? off : a.ldy - 4));
        yst[i] = ok ? v : zero4;
      }
#pragma unroll
      for (int i = 0; i < KC * TN / (4 * NTHR1); ++i) {
        const int idx = tid + NTHR1 * i, kk = idx / (TN / 4), cc = 4 * (idx % (TN / 4));
        const int64_t off = c0 + cc;
        const bool ok = k0 + kk < a.rank && off < a.k;
        const floatx4 v = *reinterpret_cast<const floatx4*>(B + (size_t)(k0 + kk) * a.ldb + (off + 4 <= a.ldb ? off : a.ldb - 4));
        bst[i] = ok ? v : zero4;
      }
    };
    fetch_chunk(0);
    for (int k0 = 0; k0 < a.rank; k0 += KC) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < KC * TM / (4 * NTHR1); ++i) {
        const int idx = tid + NTHR1 * i;
        *reinterpret_cast<floatx4*>(&ys[idx / (TM / 4)][4 * (idx % (TM / 4))]) = yst[i];
      }
#pragma unroll
      for (int i = 0; i < KC * TN / (4 * NTHR1); ++i) {
        const int idx = tid + NTHR1 * i;
        *reinterpret_cast<floatx4*>(&bs[idx / (TN / 4)][4 * (idx % (TN / 4))]) = bst[i];
      }
      __syncthreads();
      if (k0 + KC < a.rank) fetch_chunk(k0 + KC);
#pragma unroll
      for (int s = 0; s < KC / 2; ++s) {
        const float av = ys[2 * s + lh][32 * wr + ln];
        const float bv = bs[2 * s + lh][32 * wc + ln];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
      }
    }
  }
  __syncthreads();          // all operand reads done before the product overwrites the buffer
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int row = 32 * wr + 8 * (e >> 2) + 4 * lh + (e & 3);
    pt[row * PP + 32 * wc + ln] = acc[e];
  }
  __syncthreads();
  phase1_dispatch<WITH_ERR, WEIGHTED>(a, pr.cfg, z, pt, s_search, s_code, r0, c0, quads);
}

// ---- the form for split products of up to 64 ranks, used by default --------------------------------------------------
// A workgroup keeps the planes of one 128-column stretch of B in LDS; its eight wavefronts walk over bands of 16 rows of W, each
// for itself, without barriers.  v_mfma_f32_16x16x32_bf16 with the planes of B as its first operand leaves lane 16 q + n, in the accumulator of
// column tile t, with columns 16 t + 4 q + 0..3 of row n: quads of W, subtracted where they are.  A block of B0 weights lies in
// B0 / 16 tiles of the four lanes n, 16 + n, 32 + n, 48 + n, so block maxima and error sums are taken within a lane first;
// for the rest v_permlane32_swap and v_permlane16_swap exchange a value for a value, so that every step halves
// the number of blocks a lane has to do with.  The codes of 32 consecutive weights meet in one lane the same way and are
// stored at once.  The loads of a band are in flight while the band before it is quantized.
// Bound by instruction issue (vector ALU and LDS half busy each, matrix cores a sixth).  12 problems of 4096 x 4096, rank 64,
// with error sums, per weight: tiles of 64 x 128 by the whole workgroup with the product turned into rows through LDS 38 vector
// and 3.9 LDS instructions and four barriers per tile, 285 us; this form 19 and 3.0, 212 us.  One Fisher-weighted 4096 x 11008:
// 102 -> 78 us.
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {      // upper 32 lanes of a <-> lower 32 lanes of b
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap_rows(uint32_t& a, uint32_t& b) {        // lanes 16..31, 48..63 of a <-> 0..15, 32..47 of b
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
// v[b]: what this lane has of block b < NB of its row -> y[i]: block (NB == 8 ? 2 q + i : q * NB / 4) from all four lanes.
template <int NB, typename Op>
__device__ __forceinline__ void quarter_reduce(uint32_t (&v)[8], uint32_t (&y)[2], Op op) {
  constexpr int NX = NB > 1 ? NB / 2 : 1;
  uint32_t x[NX];
#pragma unroll
  for (int b = 0; b < NX; ++b) {
    uint32_t other = NB > 1 ? v[b + NX] : v[b];
    swap_halves(v[b], other);
    x[b] = op(v[b], other);
  }
#pragma unroll
  for (int b = 0; b < (NX > 1 ? NX / 2 : 1); ++b) {
    uint32_t other = NX > 1 ? x[b + NX / 2] : x[b];
    swap_rows(x[b], other);
    y[b] = op(x[b], other);
  }
}
// Codes of 32 consecutive weights from the four lanes' quads: w[t] holds the codes of quad 4 t + q of the lane's row; out: weights
// 32 q .. 32 q + 31 in order.
template <int BITS>
__device__ __forceinline__ void gather_codes(uint32_t (&w)[8], uint32_t (&out)[BITS]) {
  if constexpr (BITS == 8) {
#pragma unroll
    for (int t = 0; t < 4; ++t) swap_halves(w[t], w[t + 4]);
#pragma unroll
    for (int t = 0; t < 8; t += 4) { swap_rows(w[t], w[t + 2]); swap_rows(w[t + 1], w[t + 3]); }
#pragma unroll
    for (int i = 0; i < 4; ++i) { out[i] = w[2 * i]; out[4 + i] = w[2 * i + 1]; }
  } else {
    uint32_t p[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) p[s] = w[2 * s] | (w[2 * s + 1] << 16);
    swap_halves(p[0], p[2]); swap_halves(p[1], p[3]);
    swap_rows(p[0], p[1]); swap_rows(p[2], p[3]);
    if constexpr (BITS == 4) {
      out[0] = __builtin_amdgcn_perm(p[1], p[0], 0x05040100); out[1] = __builtin_amdgcn_perm(p[3], p[2], 0x05040100);
      out[2] = __builtin_amdgcn_perm(p[1], p[0], 0x07060302); out[3] = __builtin_amdgcn_perm(p[3], p[2], 0x07060302);
    } else if constexpr (BITS == 2) {
      const uint32_t a = __builtin_amdgcn_perm(p[1], p[0], 0x06020400), b = __builtin_amdgcn_perm(p[3], p[2], 0x06020400);
      out[0] = __builtin_amdgcn_perm(b, a, 0x05040100); out[1] = __builtin_amdgcn_perm(b, a, 0x07060302);
    } else {
      uint32_t a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = p[i] & 0xfffu; b[i] = p[i] >> 16; }
      out[0] = a[0] | (a[1] << 12) | (a[2] << 24);
      out[1] = (a[2] >> 8) | (a[3] << 4) | (b[0] << 16) | (b[1] << 28);
      out[2] = (b[1] >> 4) | (b[2] << 8) | (b[3] << 20);
    }
  }
}

constexpr int BAND = 16;
struct BandShared {
  __attribute__((aligned(16))) __bf16 b[2 * TN * KP];            // planes of B, hi then lo, zero past the rank
  __attribute__((aligned(16))) SearchEntry search[SEARCH_ENTRIES];
  __attribute__((aligned(16))) float rc[TN], cw[TN];             // 1/sqrt(col_w), col_w of the stretch
  float code[256];
};

template <int BITS, int QPB, bool WITH_ERR, bool WEIGHTED>
__device__ __forceinline__ void walk_bands(const PhaseArgs& a, int z, const BandShared& sh, int64_t c0, int band0, int band1) {
  constexpr int TPB = QPB / 4, NB = 8 / TPB, NX = NB > 1 ? NB / 2 : 1, NY = NB == 8 ? 2 : 1;   // tiles per block, blocks per row
  const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int rk = (a.rank + 15) / 16 * 16;
  const int64_t dpad = (a.d + TM - 1) / TM * TM;
  const char* yhi = reinterpret_cast<const char*>(reinterpret_cast<const __bf16*>(a.packed) + (size_t)z * a.stridePacked);
  const char* ylo = yhi + (size_t)dpad * rk * 2;
  uint8_t* codes = a.codes + (size_t)z * a.strideCodes;
  BlockRec* blk = a.blk + (size_t)z * a.strideBlk;
  const int tiles = a.k - c0 < TN ? (int)((a.k - c0) / 16) : 8;             // of this stretch inside the matrix
  const bool wide = a.k % 32 == 0;                                           // a lane's 32 codes lie inside or outside
  const uint32_t y_lane = (uint32_t)((n * rk + 8 * q) * 2);
  const uint32_t code_lane = (uint32_t)(n * (a.k / 16) + 2 * q) * (2 * BITS);
  const int block0 = NB == 8 ? 2 * q : q * NB / 4;
  const uint32_t blk_lane = (uint32_t)(n * (a.k / (4 * QPB)) + block0);
  const bool blk_live = (NB >= 4 || q % (4 / NB) == 0) && 4 * QPB * block0 < 16 * tiles;

  floatx4 wq[8], yv[2][2];
  float rs = 1.0f;
  auto fetch = [&](int band) {
    const int64_t r0 = (int64_t)band * BAND;
    int row = n;
    if (r0 + BAND > a.d) row = n < (int)(a.d - 1 - r0) ? n : (int)(a.d - 1 - r0);          // rows past the end: the last one
    const char* base = reinterpret_cast<const char*>(a.W + (size_t)r0 * a.k + c0);
    const uint32_t off = (uint32_t)(row * a.k + 4 * q) * 4u;
#pragma unroll
    for (int t = 0; t < 8; ++t) wq[t] = *reinterpret_cast<const floatx4*>(base + (off + (t < tiles ? 64u * t : 0u)));
    if constexpr (WEIGHTED) rs = (a.rsr + r0)[row];
  };
  auto fetch_y = [&](int band) {
    const uint64_t at = (uint64_t)band * (BAND * 2 * rk);
#pragma unroll
    for (int g = 0; g < 2; ++g)
      if (32 * g < rk) {
        const uint32_t lane_at = y_lane + (32 * g + 8 * q < rk ? 64u * g : 0u);           // past the rank: anything
        yv[g][0] = *reinterpret_cast<const floatx4*>(yhi + at + lane_at);
        yv[g][1] = *reinterpret_cast<const floatx4*>(ylo + at + lane_at);
      }
  };
  if (band0 < band1) { fetch(band0); fetch_y(band0); }
  __syncthreads();                             // what the workgroup shares is in LDS
  for (int band = band0; band < band1; band += 8) {
    const int64_t r0 = (int64_t)band * BAND;
    floatx4 t[8];
    const __bf16* bop = sh.b + n * KP + 8 * q;
    auto products = [&](int g) {
      if (32 * g + 32 > rk && 32 * g + 8 * q >= rk) yv[g][0] = yv[g][1] = floatx4{0.f, 0.f, 0.f, 0.f};
      const bf16x8 yh = __builtin_bit_cast(bf16x8, yv[g][0]), yl = __builtin_bit_cast(bf16x8, yv[g][1]);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bf16x8 bh = *reinterpret_cast<const bf16x8*>(bop + 16 * i * KP + 32 * g);
        const bf16x8 bl = *reinterpret_cast<const bf16x8*>(bop + (TN + 16 * i) * KP + 32 * g);
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        t[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, yl, g ? t[i] : zero, 0, 0, 0);
        t[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl, yh, t[i], 0, 0, 0);
        t[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, yh, t[i], 0, 0, 0);
      }
    };
    products(0);
    if (rk > 32) products(1);
    uint32_t m[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (WEIGHTED) t[i] *= rs * *reinterpret_cast<const floatx4*>(sh.rc + 16 * i + 4 * q);
      t[i] = wq[i] - t[i];
      const float e[4] = {t[i][0], t[i][1], t[i][2], t[i][3]};
      const uint32_t mq = quad_absmax_bits(e);
      if (i % TPB == 0) m[i / TPB] = mq;
      else m[i / TPB] = m[i / TPB] > mq ? m[i / TPB] : mq;
    }
    const int following = band + 8 < band1 ? band + 8 : band;                 // past the end: the same band again
    fetch(following);
    fetch_y(following);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t ymax[2];
    quarter_reduce<NB>(m, ymax, [](uint32_t x, uint32_t y) { return x > y ? x : y; });
    float mine[NY], inv[NY];
#pragma unroll
    for (int i = 0; i < NY; ++i) { mine[i] = __uint_as_float(ymax[i]); inv[i] = safe_reciprocal(mine[i]); }
    // The way back for the reciprocals and maxima and, behind the weights, the sums' way in, pair by pair: what a pair needs
    // does not stay in registers.
    uint32_t w[8];
    float y[NY][3];
    auto add = [](uint32_t x, uint32_t other) { return __uint_as_float(x) + __uint_as_float(other); };
    auto block_codes = [&](int b, float rcp, float amax, float (&sum)[3]) __attribute__((always_inline)) {
      sum[0] = sum[1] = sum[2] = 0.f;
#pragma unroll
      for (int i = b * TPB; i < (b + 1) * TPB; ++i) {
        if constexpr (WITH_ERR) asm volatile("" : "+v"(t[i]));            // tile by tile, or registers run out
        floatx4 cw = {1.f, 1.f, 1.f, 1.f};
        if constexpr (WITH_ERR && WEIGHTED) cw = *reinterpret_cast<const floatx4*>(sh.cw + 16 * i + 4 * q);
        uint32_t c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          c[e] = search_code<BITS>(sh.search, t[i][e] * rcp);
          if constexpr (WITH_ERR) {
            const float qv = sh.code[c[e]], err = t[i][e] - qv * amax;
            float werr = err, wqv = qv;
            if constexpr (WEIGHTED) { werr = cw[e] * err; wqv = cw[e] * qv; }
            sum[0] = fmaf(werr, err, sum[0]);
            sum[1] = fmaf(werr, qv, sum[1]);
            sum[2] = fmaf(wqv, qv, sum[2]);
          }
        }
        w[i] = c[0] | (c[1] << BITS) | (c[2] << (2 * BITS)) | (c[3] << (3 * BITS));
      }
    };
#pragma unroll
    for (int i = 0; i < NY; ++i) {
      uint32_t xr[2] = {__float_as_uint(inv[i]), __float_as_uint(inv[i])}, xm[2] = {ymax[i], ymax[i]};
      if constexpr (NX > 1) { swap_rows(xr[0], xr[1]); if constexpr (WITH_ERR) swap_rows(xm[0], xm[1]); }
      float xs[2][3];
#pragma unroll
      for (int j = 0; j < (NX > 1 ? 2 : 1); ++j) {
        const int b = i + j * (NX / 2);
        uint32_t vr[2] = {xr[j], xr[j]}, vm[2] = {xm[j], xm[j]};
        if constexpr (NB > 1) { swap_halves(vr[0], vr[1]); if constexpr (WITH_ERR) swap_halves(vm[0], vm[1]); }
        float vs[2][3];
#pragma unroll
        for (int h = 0; h < (NB > 1 ? 2 : 1); ++h)
          block_codes(b + h * NX, __uint_as_float(vr[h]), __uint_as_float(vm[h]), vs[h]);
        if constexpr (WITH_ERR) {
#pragma unroll
          for (int e = 0; e < 3; ++e) {
            uint32_t l = __float_as_uint(vs[0][e]), u = __float_as_uint(vs[NB > 1 ? 1 : 0][e]);
            swap_halves(l, u);
            xs[j][e] = add(l, u);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (WITH_ERR) {
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          uint32_t l = __float_as_uint(xs[0][e]), u = __float_as_uint(xs[NX > 1 ? 1 : 0][e]);
          swap_rows(l, u);
          y[i][e] = add(l, u);
        }
      }
    }
    uint32_t out[BITS];
    gather_codes<BITS>(w, out);
    const bool row_live = r0 + n < a.d;
    uint8_t* to = codes + (((uint64_t)r0 * a.k + c0) / 16 * (2 * BITS)) + code_lane;
    if (wide) {
      if (row_live && 2 * q < tiles) {
        if constexpr (BITS == 8) {
          reinterpret_cast<uint4*>(to)[0] = make_uint4(out[0], out[1], out[2], out[3]);
          reinterpret_cast<uint4*>(to)[1] = make_uint4(out[4], out[5], out[6], out[7]);
        } else if constexpr (BITS == 4) {
          *reinterpret_cast<uint4*>(to) = make_uint4(out[0], out[1], out[2], out[3]);
        } else if constexpr (BITS == 3) {
          *reinterpret_cast<uint3*>(to) = make_uint3(out[0], out[1], out[2]);
        } else {
          *reinterpret_cast<uint2*>(to) = make_uint2(out[0], out[1]);
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)                     // runs of 16 weights; 3 bits: 48 bits, 2-byte aligned
        if (row_live && 2 * q + h < tiles) {
          if constexpr (BITS == 3) {
            uint16_t* p = reinterpret_cast<uint16_t*>(to + 6 * h);
            p[0] = (uint16_t)(h ? out[1] >> 16 : out[0]);
            p[1] = (uint16_t)(h ? out[2] : out[0] >> 16);
            p[2] = (uint16_t)(h ? out[2] >> 16 : out[1]);
          } else {
#pragma unroll
            for (int i = 0; i < BITS / 2; ++i) reinterpret_cast<uint32_t*>(to + 2 * BITS * h)[i] = out[h * (BITS / 2) + i];
          }
        }
    }
    if constexpr (WITH_ERR) {
      BlockRec* at = blk + ((uint64_t)r0 * a.k + c0) / (4 * QPB) + blk_lane;
      if (row_live && blk_live) {
#pragma unroll
        for (int i = 0; i < NY; ++i) {
          BlockRec rec;
          rec.s = mine[i]; rec.e2 = y[i][0]; rec.eq = y[i][1]; rec.q2 = y[i][2];
          if (i == 0 || 4 * QPB * (block0 + i) < 16 * tiles) at[i] = rec;
        }
      }
    } else {
      float* at = reinterpret_cast<float*>(blk) + ((uint64_t)r0 * a.k + c0) / (4 * QPB) + blk_lane;    // the absmax alone
      if (row_live && blk_live) {
#pragma unroll
        for (int i = 0; i < NY; ++i)
          if (i == 0 || 4 * QPB * (block0 + i) < 16 * tiles) at[i] = mine[i];
      }
    }
  }
}

template <int BITS, bool WITH_ERR, bool WEIGHTED>
__device__ __forceinline__ void walk_bands_block(const PhaseArgs& a, int block, int z, const BandShared& sh, int64_t c0, int band0, int band1) {
  switch (block) {
    case 16: walk_bands<BITS, 4, WITH_ERR, WEIGHTED>(a, z, sh, c0, band0, band1); break;
    case 32: walk_bands<BITS, 8, WITH_ERR, WEIGHTED>(a, z, sh, c0, band0, band1); break;
    case 64: walk_bands<BITS, 16, WITH_ERR, WEIGHTED>(a, z, sh, c0, band0, band1); break;
    default: walk_bands<BITS, 32, WITH_ERR, WEIGHTED>(a, z, sh, c0, band0, band1); break;
  }
}

// Launch: one-dimensional, batch * units8 workgroups, units = column stretches x groups of 8 nb bands, rounded up to a
// multiple of 8; index decoded as (unit mod 8, problem, unit div 8) so that the problems of a batch that share a
// stretch of W run on one XCD at the same time.
template <bool WITH_ERR, bool WEIGHTED>
__global__ __launch_bounds__(NTHR1, 4) void lowrank_blockquant_bands_kernel(PhaseArgs a, int units, int tiles_n, int nb) {
  __shared__ BandShared sh;
  const int tid = threadIdx.x;
  const int slot8 = blockIdx.x >> 3;
  const int z = slot8 % a.batch;
  const int unit = (int)(blockIdx.x & 7) + 8 * (slot8 / a.batch);
  if (unit >= units) return;                   // padding of the unit count to a multiple of 8
  const lq_config cfg = a.prob[z].cfg;
  const int64_t c0 = (int64_t)(unit % tiles_n) * TN;
  const int slot = cfg.bits == 2 ? 0 : cfg.bits == 3 ? 1 : cfg.bits == 4 ? 2 : 3;
  load_search_nosync(a.tables, slot, sh.search);
  if constexpr (WITH_ERR)
    for (int i = tid; i < (1 << cfg.bits); i += NTHR1) sh.code[i] = a.tables->code[slot][i];
  if constexpr (WEIGHTED)
    for (int i = tid; i < TN; i += NTHR1) {
      const bool live = c0 + i < a.k;
      sh.rc[i] = live ? a.rsc[c0 + i] : 1.0f;
      if constexpr (WITH_ERR) sh.cw[i] = live ? a.col_w[c0 + i] : 1.0f;
    }
  {
    // planes of B: 16-byte piece tid & 7 of rows tid / 8 and tid / 8 + 64, of hi and of lo
    const int rk = (a.rank + 15) / 16 * 16;
    const int64_t dpad = (a.d + TM - 1) / TM * TM, kpad = (a.k + TN - 1) / TN * TN;
    const __bf16* gb = reinterpret_cast<const __bf16*>(a.packed) + (size_t)z * a.stridePacked + (size_t)2 * dpad * rk;
    const int piece = 8 * (tid & 7);
    floatx4 bp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const __bf16* from = gb + (size_t)((i >> 1) * kpad + c0 + 64 * (i & 1) + (tid >> 3)) * rk;
      bp[i] = piece < rk ? *reinterpret_cast<const floatx4*>(from + piece) : floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<floatx4*>(sh.b + (size_t)((tid >> 3) + 64 * i) * KP + piece) = bp[i];
  }
  const int nbands = (int)((a.d + BAND - 1) / BAND), first = (unit / tiles_n) * (8 * nb);
  const int band0 = first + __builtin_amdgcn_readfirstlane(tid >> 6), band1 = first + 8 * nb < nbands ? first + 8 * nb : nbands;
  switch (cfg.bits) {
    case 2: walk_bands_block<2, WITH_ERR, WEIGHTED>(a, cfg.block, z, sh, c0, band0, band1); break;
    case 3: walk_bands_block<3, WITH_ERR, WEIGHTED>(a, cfg.block, z, sh, c0, band0, band1); break;
    case 4: walk_bands_block<4, WITH_ERR, WEIGHTED>(a, cfg.block, z, sh, c0, band0, band1); break;
    default: walk_bands_block<8, WITH_ERR, WEIGHTED>(a, cfg.block, z, sh, c0, band0, band1); break;
  }
}

// Steps of eight bands per workgroup: the fewest rounds of 512 resident workgroups times what one of them takes, a step each and
// about as much as one more for the tables, the planes of B and the first loads.  (At most 4 steps instead of 16: the passes of a
// layer's sweep, 36 configurations at a time, 68.3 -> 76.1 ms.)
static int bands_per_wave(int64_t steps, int64_t stretches, int64_t batch) {
  double least = 1e300;
  int best = 1;
  for (int64_t nb = 1; nb <= steps && nb <= 16; ++nb) {
    const int64_t wgs = stretches * ((steps + nb - 1) / nb) * batch;
    const double t = (double)((wgs + 511) / 512) * ((double)nb + 1.0);
    if (t < least) { least = t; best = (int)nb; }
  }
  return best;
}

int launch_lowrank_blockquant(const PhaseArgs& a, bool with_err, hipStream_t st) {
  const int tiles_n = (int)((a.k + TN - 1) / TN);
  const int64_t nbands = (a.d + TM - 1) / TM;
  const int64_t tiles = (int64_t)tiles_n * nbands;
  if ((tiles + 7) / 8 * 8 * a.batch >= (1ll << 31)) return LQ_ERR_SHAPE;
  if (a.k > (1ll << 25)) return LQ_ERR_SHAPE;      // lane offsets within a tile (up to 63 rows apart) are 32-bit byte offsets
  // algorithmic bytes: W and the factors in, the quantized form out, per configuration (the scale part of the latter is
  // finished by the scale kernel that follows)
  prof::Scope ps(prof::LOWRANK_BLOCKQUANT, st,
                 (double)a.d * a.k * (4.0 * a.batch + a.quant_bytes_per_weight) + 4.0 * a.rank * (double)(a.d + a.k) * a.batch);
  const bool split = a.packed != nullptr;
  if (split && a.rank <= KC2) {
    const int64_t steps = ((a.d + BAND - 1) / BAND + 7) / 8;
    const int nb = bands_per_wave(steps, tiles_n, a.batch);
    const int64_t units = (int64_t)tiles_n * ((steps + nb - 1) / nb);
    const dim3 grid((unsigned)((units + 7) / 8 * 8 * a.batch));
    auto go = [&](auto err, auto weighted) {
      hipLaunchKernelGGL((lowrank_blockquant_bands_kernel<decltype(err)::value, decltype(weighted)::value>), grid, dim3(NTHR1), 0, st, a,
                         (int)units, tiles_n, nb);
    };
    if (a.rsc) { if (with_err) go(std::true_type{}, std::true_type{}); else go(std::false_type{}, std::true_type{}); }
    else { if (with_err) go(std::true_type{}, std::false_type{}); else go(std::false_type{}, std::false_type{}); }
    LQ_HIP_TRY(hipGetLastError());
    return LQ_OK;
  }
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8 * a.batch));
  auto go = [&](auto err, auto weighted) {
    constexpr bool E = decltype(err)::value, F = decltype(weighted)::value;
    if (split) hipLaunchKernelGGL((lowrank_blockquant_kernel<E, true, F>), grid, dim3(NTHR1), 0, st, a, (int)tiles, tiles_n);
    else hipLaunchKernelGGL((lowrank_blockquant_kernel<E, false, F>), grid, dim3(NTHR1), 0, st, a, (int)tiles, tiles_n);
  };
  if (a.rsc) { if (with_err) go(std::true_type{}, std::true_type{}); else go(std::false_type{}, std::true_type{}); }
  else { if (with_err) go(std::true_type{}, std::false_type{}); else go(std::false_type{}, std::false_type{}); }
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
// Phase 2: one lane per block.
// WITH_ERR: phase 1 left full block records {s, e2, eq, q2}; otherwise only the block absmax values (4 B per block)
// and the error output is zero.
template <bool WITH_ERR>
__global__ __launch_bounds__(256) void scalequant_error_kernel(PhaseArgs a) {
  __shared__ float s_wave[4];
  __shared__ double s_sum[4];
  const int z = blockIdx.y, tid = threadIdx.x;
  const LoopProblem pr = a.prob[z];
  const int64_t nb = (a.d * a.k) / pr.cfg.block;
  const int64_t b = (int64_t)blockIdx.x * 256 + tid;
  double* part = a.err_part + (size_t)z * a.strideErrPart;
  if ((int64_t)blockIdx.x * 256 >= nb) {           // whole workgroup past this problem's blocks
    if (WITH_ERR && tid == 0) part[blockIdx.x] = 0.0;
    return;
  }
  BlockRec rec; rec.s = 0.f; rec.e2 = 0.f; rec.eq = 0.f; rec.q2 = 0.f;
  if (b < nb) {
    if (WITH_ERR) rec = a.blk[(size_t)z * a.strideBlk + b];
    else rec.s = reinterpret_cast<const float*>(a.blk + (size_t)z * a.strideBlk)[b];
  }
  const float vmax = group_max(rec.s, pr.cfg.scale_block, s_wave);
  const float sigma = vmax / (float)pr.levels;
  const float vhat = cast_group_scale(vmax, pr.cfg.v_dtype);
  double err = 0.0;
  if (b < nb) {
    const uint32_t idx = scale_index(rec.s, sigma, pr.levels);
    a.sidx[(size_t)z * a.strideSidx + b] = (uint8_t)idx;
    if ((b & (pr.cfg.scale_block - 1)) == 0) a.v[(size_t)z * a.strideV + b / pr.cfg.scale_block] = vhat;
    if constexpr (WITH_ERR) {
      const float shat = block_scale(idx, vhat, pr.levels);
      const double delta = (double)shat - (double)rec.s;
      err = (double)rec.e2 - 2.0 * delta * (double)rec.eq + delta * delta * (double)rec.q2;
      if (a.row_w) err *= (double)a.row_w[(b * pr.cfg.block) / a.k];
    }
  }
  if constexpr (WITH_ERR) {
    for (int off = 1; off < 64; off <<= 1) err += __shfl_xor(err, off);
    if ((tid & 63) == 0) s_sum[tid >> 6] = err;
    __syncthreads();
    if (tid == 0) part[blockIdx.x] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
  }
}

// eps = sqrt(sum of the partials), one workgroup per problem, fixed summation order.
__global__ __launch_bounds__(256) void error_finalize_kernel(const double* __restrict__ part, size_t stride,
                                                             int64_t count, double* __restrict__ out,
                                                             size_t out_stride) {
  __shared__ double s_sum[256];
  const int z = blockIdx.x, tid = threadIdx.x;
  const double* p = part + (size_t)z * stride;
  double s = 0.0;
  for (int64_t i = tid; i < count; i += 256) s += p[i];
  s_sum[tid] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (tid < w) s_sum[tid] += s_sum[tid + w];
    __syncthreads();
  }
  if (tid == 0) out[(size_t)z * out_stride] = sqrt(s_sum[0] > 0.0 ? s_sum[0] : 0.0);
}

int64_t err_partials_per_problem(int64_t n, int block) { return (n / block + 255) / 256; }

int launch_scalequant_error(const PhaseArgs& a, int min_block, bool with_err, hipStream_t st) {
  const int64_t nwg = err_partials_per_problem(a.d * a.k, min_block);
  prof::Scope ps(prof::SCALEQUANT_ERROR, st, (double)(a.d * a.k / min_block) * (with_err ? 17.0 : 5.0) * a.batch);
  if (with_err) hipLaunchKernelGGL(scalequant_error_kernel<true>, dim3((unsigned)nwg, (unsigned)a.batch), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(scalequant_error_kernel<false>, dim3((unsigned)nwg, (unsigned)a.batch), dim3(256), 0, st, a);
  LQ_HIP_TRY(hipGetLastError());
  if (with_err) {
    hipLaunchKernelGGL(error_finalize_kernel, dim3((unsigned)a.batch), dim3(256), 0, st, (const double*)a.err_part,
                       a.strideErrPart, nwg, a.err_out, a.strideErrOut);
    LQ_HIP_TRY(hipGetLastError());
  }
  return LQ_OK;
}

// ------------------------------------------------------------------------------------------------
// Phase 3: one quad (4 consecutive weights) per lane and step, so each wavefront instruction reads / writes
// 1 KB of contiguous fp32.
// A workgroup takes a stretch of 512 quads (RES_U = 2 per lane) of W and keeps it in registers for several problems of
// the batch, so W crosses the L2 / L1 fabric a few times per batch instead of once per problem (R is 4 B per weight
// out; W would be another 4 B per weight in).
constexpr int RES_U = 2;

struct ResidualFetch {                 // what one lane needs of one problem besides W
  uint32_t cw[RES_U];                  // packed codes of the quad (4 * bits bits)
  uint32_t si[RES_U];
  float vv[RES_U];
};

__device__ __forceinline__ uint32_t load_quad_word(const uint8_t* __restrict__ codes, int64_t quad, int bits) {
  if (bits == 8) return *reinterpret_cast<const uint32_t*>(codes + quad * 4);
  if (bits == 4) return *reinterpret_cast<const uint16_t*>(codes + quad * 2);
  if (bits == 2) return codes[quad];
  const int64_t byte = (quad * 3) >> 1;     // 3 bits: 12 bits starting at bit 12*quad, nibble-aligned
  return (((uint32_t)codes[byte] | ((uint32_t)codes[byte + 1] << 8)) >> ((quad & 1) * 4)) & 0xfffu;
}

__device__ __forceinline__ void residual_fetch(const PhaseArgs& a, const LoopProblem& pr, int z, const int64_t (&qq)[RES_U],
                                               ResidualFetch& f) {
  const int qpb_shift = __builtin_ctz(pr.cfg.block / 4), sb_shift = __builtin_ctz(pr.cfg.scale_block);
  const uint8_t* codes = a.codes + (size_t)z * a.strideCodes;
  const uint8_t* sidx = a.sidx + (size_t)z * a.strideSidx;
  const float* v = a.v + (size_t)z * a.strideV;
#pragma unroll
  for (int u = 0; u < RES_U; ++u) {
    const int64_t blk = qq[u] >> qpb_shift;
    f.cw[u] = load_quad_word(codes, qq[u], pr.cfg.bits);
    f.si[u] = sidx[blk];
    f.vv[u] = v[blk >> sb_shift];
  }
}

// A workgroup serves RES_G problems for its stretch of W: every load is issued first, then everything is computed
// and stored, and the wavefront ends without ever waiting for a store.  (Loads and stores share one in-order
// counter on this architecture, so a wait for a load also waits for every store issued before it: a loop that
// alternates loads and stores runs at the pace of the store latency.)  Measured on 36 x 4096 x 11008: 3.7 TB/s
// written; a kernel that only stores reaches 5.7 - 6.9 TB/s, one that loads 2 B per quad before storing 3.8 TB/s.  The problem group is the fastest launch
// index, so the groups of a batch that read the same stretch of W run together and share it in L2.
// The lo plane of the fp16 residual: what the rounding of sv to hi dropped, times 2^11, rounded to the upper byte of
// its fp16 form (sign, five exponent bits, two fraction bits; round to nearest even on the bit pattern, which carries
// into the exponent where it has to).  |sv - hi| <= 16 for |sv| <= 65504, so the scaled value stays below 2^15 + 1.
__device__ __forceinline__ uint32_t lo_plane_byte(float sv, _Float16 hi) {
  const _Float16 l = (_Float16)((sv - (float)hi) * 2048.0f);
  const uint32_t b = (uint32_t)__builtin_bit_cast(uint16_t, l);
  return (b + 0x7Fu + ((b >> 8) & 1u)) >> 8;
}

constexpr int RES_G = 6;

__global__ __launch_bounds__(256) void residual_kernel(PhaseArgs a, int groups) {
  __shared__ float s_code[4][256];
  const int tid = threadIdx.x;
  for (int i = tid; i < 1024; i += 256) s_code[i >> 8][i & 255] = a.tables->code[i >> 8][i & 255];
  const int zfirst = (int)(blockIdx.x % groups) * RES_G;
  const int64_t nquads = (a.d * a.k) >> 2;
  const int64_t q0 = (int64_t)(blockIdx.x / groups) * (256 * RES_U) + tid;
  int64_t qq[RES_U];                   // clamped quad indices (loads stay in bounds; stores are guarded)
  float4 w[RES_U];
#pragma unroll
  for (int u = 0; u < RES_U; ++u) {
    const int64_t quad = q0 + 256 * u;
    qq[u] = quad < nquads ? quad : nquads - 1;
    w[u] = *reinterpret_cast<const float4*>(a.W + (qq[u] << 2));
  }
  LoopProblem pr[RES_G];
  ResidualFetch f[RES_G];
#pragma unroll
  for (int gI = 0; gI < RES_G; ++gI) {
    const int z = zfirst + gI < a.batch ? zfirst + gI : a.batch - 1;      // clamped: loaded, never stored
    pr[gI] = a.prob[z];
    residual_fetch(a, pr[gI], z, qq, f[gI]);
  }
  float srow[RES_U];
  float4 cs[RES_U];
  if (a.sr) {
#pragma unroll
    for (int u = 0; u < RES_U; ++u) {
      const int64_t e0 = qq[u] << 2;
      srow[u] = a.sr[e0 / a.k];
      cs[u] = *reinterpret_cast<const float4*>(a.sc + e0 % a.k);
    }
  }
  __syncthreads();                     // code books in LDS
#pragma unroll
  for (int gI = 0; gI < RES_G; ++gI) {
    const int z = zfirst + gI;
    if (z >= a.batch) break;
    const int bits = pr[gI].cfg.bits, levels = pr[gI].levels;
    const float* code = s_code[bits == 2 ? 0 : bits == 3 ? 1 : bits == 4 ? 2 : 3];
    const uint32_t mask = (1u << bits) - 1u;
    float* R = a.R ? a.R + (size_t)z * a.strideR : nullptr;
    _Float16* R16 = a.R16 ? reinterpret_cast<_Float16*>(a.R16) + (size_t)z * a.strideR : nullptr;
    uint8_t* R16lo = a.R16lo ? a.R16lo + (size_t)z * a.strideR : nullptr;
    float* Qd = a.Qd ? a.Qd + (size_t)z * a.strideQd : nullptr;
#pragma unroll
    for (int u = 0; u < RES_U; ++u) {
      const int64_t quad = q0 + 256 * u;
      if (quad >= nquads) break;
      const float sh = block_scale(f[gI].si[u], f[gI].vv[u], levels);
      const uint32_t cw = f[gI].cw[u];
      float4 qv, rv;
      qv.x = code[cw & mask] * sh; qv.y = code[(cw >> bits) & mask] * sh;
      qv.z = code[(cw >> (2 * bits)) & mask] * sh; qv.w = code[(cw >> (3 * bits)) & mask] * sh;
      rv.x = w[u].x - qv.x; rv.y = w[u].y - qv.y; rv.z = w[u].z - qv.z; rv.w = w[u].w - qv.w;
      if (a.sr) {
        rv.x = srow[u] * rv.x * cs[u].x; rv.y = srow[u] * rv.y * cs[u].y;
        rv.z = srow[u] * rv.z * cs[u].z; rv.w = srow[u] * rv.w * cs[u].w;
      }
      if (R) __builtin_nontemporal_store(floatx4{rv.x, rv.y, rv.z, rv.w}, reinterpret_cast<floatx4*>(R + (quad << 2)));
      if (R16) {
        const float lim = 65504.0f;        // largest fp16: out-of-range entries saturate instead of becoming infinite
        const float sv[4] = {__builtin_amdgcn_fmed3f(rv.x * a.r_scale, -lim, lim), __builtin_amdgcn_fmed3f(rv.y * a.r_scale, -lim, lim),
                             __builtin_amdgcn_fmed3f(rv.z * a.r_scale, -lim, lim), __builtin_amdgcn_fmed3f(rv.w * a.r_scale, -lim, lim)};
        halfx4 h;
        uint32_t l = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          h[e] = (_Float16)sv[e];
          l |= lo_plane_byte(sv[e], h[e]) << (8 * e);
        }
        // streamed out: nothing reads these lines before they have left the caches anyway
        __builtin_nontemporal_store(h, reinterpret_cast<halfx4*>(R16 + (quad << 2)));
        if (R16lo) __builtin_nontemporal_store(l, reinterpret_cast<uint32_t*>(R16lo + (quad << 2)));
      }
      if (Qd) __builtin_nontemporal_store(floatx4{qv.x, qv.y, qv.z, qv.w}, reinterpret_cast<floatx4*>(Qd + (quad << 2)));
    }
  }
}

// The form of phase 3 that the warm iterations use: only the scaled fp16 planes of the residual are written.  A
// workgroup owns one stretch of W (RP_U runs of 8 consecutive weights per lane, kept in registers) and walks through the
// problems of the batch with it, so W is read once per batch; the codes and scales of problem z + 1 are fetched before
// problem z is computed and stored, so no load ever waits behind a store; every store of a plane is 16 bytes per lane,
// 1 KB contiguous per wavefront, and is streamed past the caches (measured: the kernel is bound by the bytes it moves;
// per-problem workgroups that re-read W, in either launch order, took 1.29 - 1.36 ms per 36 problems where this takes
// less).
constexpr int RP_U = 2;
typedef _Float16 halfx8r __attribute__((ext_vector_type(8)));
typedef uint32_t uintx2r __attribute__((ext_vector_type(2)));

struct PlaneFetch { uint32_t cw[RP_U][2]; uint32_t si[RP_U]; float vv[RP_U]; };

template <int BITS>
__device__ __forceinline__ void residual_planes_fetch(const PhaseArgs& a, int blk_shift, int sb_shift, int z,
                                                      const int64_t (&oct)[RP_U], PlaneFetch& f) {
  const uint8_t* codes = a.codes + (size_t)z * a.strideCodes;
  const uint8_t* sidx = a.sidx + (size_t)z * a.strideSidx;
  const float* v = a.v + (size_t)z * a.strideV;
#pragma unroll
  for (int u = 0; u < RP_U; ++u) {
    const int64_t o = oct[u];
    f.cw[u][1] = 0;
    if constexpr (BITS == 8) {
      const uint2 c2 = *reinterpret_cast<const uint2*>(codes + o * 8);
      f.cw[u][0] = c2.x; f.cw[u][1] = c2.y;
    } else if constexpr (BITS == 4) {
      f.cw[u][0] = *reinterpret_cast<const uint32_t*>(codes + o * 4);
    } else if constexpr (BITS == 2) {
      f.cw[u][0] = *reinterpret_cast<const uint16_t*>(codes + o * 2);
    } else {       // 24 bits at byte 3 * oct: a 16-bit and an 8-bit piece, the 16-bit one at the even address
      const int64_t b = o * 3;
      const uint32_t h = *reinterpret_cast<const uint16_t*>(codes + b + (o & 1));
      const uint32_t q = codes[b + ((o & 1) ? 0 : 2)];
      f.cw[u][0] = (o & 1) ? (q | (h << 8)) : (h | (q << 16));
    }
    const int64_t blk = o >> blk_shift;
    f.si[u] = sidx[blk];
    f.vv[u] = v[blk >> sb_shift];
  }
}

// zmask: the problems of the batch (bit z) this launch serves; all of them have BITS code bits.
// The loop over them is unrolled twice over two fetch buffers and has no conditional load or store inside (past the
// last problem it fetches the last one again; lanes past the end of the matrix work on the last run of 8 weights again
// and store the same values as its owner), so the compiler's wait for the loads of problem i + 1 never includes the
// stores of problem i that were issued after them.
template <int BITS, bool WEIGHTED>
__global__ __launch_bounds__(256) void residual_planes_kernel(PhaseArgs a, uint64_t zmask) {
  __shared__ float s_code[1 << BITS];
  __shared__ int s_list[64];
  __shared__ int s_par[64][4];         // per problem: log2(B0 / 8), log2(B1), levels
  const int tid = threadIdx.x;
  for (int i = tid; i < (1 << BITS); i += 256) s_code[i] = a.tables->code[Slot<BITS>::value][i];
  if (tid < 64 && ((zmask >> tid) & 1)) {
    const LoopProblem p = a.prob[tid];
    s_list[__builtin_popcountll(zmask & ((1ull << tid) - 1ull))] = tid;
    s_par[tid][0] = __builtin_ctz(p.cfg.block / 8); s_par[tid][1] = __builtin_ctz(p.cfg.scale_block); s_par[tid][2] = p.levels;
  }
  const int count = __builtin_popcountll(zmask);
  const int64_t nocts = (a.d * a.k) >> 3;
  const int64_t oct0 = (int64_t)blockIdx.x * (256 * RP_U) + tid;
  int64_t oct[RP_U];
  float wv[RP_U][8], cv[RP_U][8], srow[RP_U];
#pragma unroll
  for (int u = 0; u < RP_U; ++u) {
    oct[u] = oct0 + 256 * u < nocts ? oct0 + 256 * u : nocts - 1;
    const float4 w0 = *reinterpret_cast<const float4*>(a.W + (oct[u] << 3));
    const float4 w1 = *reinterpret_cast<const float4*>(a.W + (oct[u] << 3) + 4);
    wv[u][0] = w0.x; wv[u][1] = w0.y; wv[u][2] = w0.z; wv[u][3] = w0.w;
    wv[u][4] = w1.x; wv[u][5] = w1.y; wv[u][6] = w1.z; wv[u][7] = w1.w;
    if constexpr (WEIGHTED) {
      const int64_t e0 = oct[u] << 3;
      srow[u] = a.sr[e0 / a.k];
      const float4 c0 = *reinterpret_cast<const float4*>(a.sc + e0 % a.k);
      const float4 c1 = *reinterpret_cast<const float4*>(a.sc + e0 % a.k + 4);
      cv[u][0] = c0.x; cv[u][1] = c0.y; cv[u][2] = c0.z; cv[u][3] = c0.w;
      cv[u][4] = c1.x; cv[u][5] = c1.y; cv[u][6] = c1.z; cv[u][7] = c1.w;
    }
  }
  __syncthreads();                     // code book, problem list and parameters in LDS
  const float lim = 65504.0f;          // largest fp16: out-of-range entries saturate instead of becoming infinite
  constexpr uint32_t mask = (1u << BITS) - 1u;
  auto fetch = [&](int i, PlaneFetch& f) {
    const int z = s_list[i < count ? i : count - 1];
    residual_planes_fetch<BITS>(a, s_par[z][0], s_par[z][1], z, oct, f);
  };
  auto emit = [&](int i, const PlaneFetch& f) {
    const int z = s_list[i];
    const int levels = s_par[z][2];
    _Float16* hi = reinterpret_cast<_Float16*>(a.R16) + (size_t)z * a.strideR;
    uint8_t* lo = a.R16lo + (size_t)z * a.strideR;
#pragma unroll
    for (int u = 0; u < RP_U; ++u) {
      const float sh = block_scale(f.si[u], f.vv[u], levels);
      halfx8r h;
      uint32_t l[2] = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t c = BITS == 8 ? (f.cw[u][e >> 2] >> (8 * (e & 3))) & mask : (f.cw[u][0] >> (BITS * e)) & mask;
        float r = wv[u][e] - s_code[c] * sh;
        if constexpr (WEIGHTED) r = srow[u] * r * cv[u][e];
        const float sv = __builtin_amdgcn_fmed3f(r * a.r_scale, -lim, lim);
        h[e] = (_Float16)sv;
        l[e >> 2] |= lo_plane_byte(sv, h[e]) << (8 * (e & 3));
      }
      __builtin_nontemporal_store(h, reinterpret_cast<halfx8r*>(hi + (oct[u] << 3)));
      __builtin_nontemporal_store(uintx2r{l[0], l[1]}, reinterpret_cast<uintx2r*>(lo + (oct[u] << 3)));
    }
  };
  PlaneFetch fa, fb;
  fetch(0, fa);
  for (int i = 0;;) {
    fetch(i + 1, fb);
    emit(i, fa);
    if (++i >= count) break;
    fetch(i + 1, fa);
    emit(i, fb);
    if (++i >= count) break;
  }
}

template <int BITS>
static void launch_residual_planes(const PhaseArgs& a, uint64_t zmask, dim3 grid, hipStream_t st) {
  if (a.sr) hipLaunchKernelGGL((residual_planes_kernel<BITS, true>), grid, dim3(256), 0, st, a, zmask);
  else hipLaunchKernelGGL((residual_planes_kernel<BITS, false>), grid, dim3(256), 0, st, a, zmask);
}

int launch_residual(const PhaseArgs& a, hipStream_t st) {
  const int64_t nquads = (a.d * a.k) >> 2;
  const int groups = (a.batch + RES_G - 1) / RES_G;
  const int64_t nwg = (nquads + 256 * RES_U - 1) / (256 * RES_U) * groups;
  if (nwg >= (1ll << 31)) return LQ_ERR_SHAPE;
  // R (or dense Q) out per problem, the quantized form in per problem, W in once
  const double out_bytes = (a.R ? 4.0 : 0.0) + (a.R16 ? 2.0 : 0.0) + (a.R16 && a.R16lo ? 1.0 : 0.0) + (a.Qd ? 4.0 : 0.0);
  prof::Scope ps(prof::RESIDUAL, st, (double)a.d * a.k * (out_bytes * a.batch + 4.0 + a.quant_bytes_per_weight));
  if (a.R16 && a.R16lo && !a.R && !a.Qd && ((a.d * a.k) & 7) == 0 && a.batch <= 64 && a.bits_host) {
    const int64_t nwg2 = (((a.d * a.k) >> 3) + 256 * RP_U - 1) / (256 * RP_U);
    if (nwg2 >= (1ll << 31)) return LQ_ERR_SHAPE;
    const dim3 grid((unsigned)nwg2);
    // one launch per code width present in the batch (the kernel's loads depend on it)
    uint64_t m[4] = {0, 0, 0, 0};
    for (int z = 0; z < a.batch; ++z) {
      const int b = a.bits_host[z];
      m[b == 2 ? 0 : b == 3 ? 1 : b == 4 ? 2 : 3] |= 1ull << z;
    }
    if (m[0]) launch_residual_planes<2>(a, m[0], grid, st);
    if (m[1]) launch_residual_planes<3>(a, m[1], grid, st);
    if (m[2]) launch_residual_planes<4>(a, m[2], grid, st);
    if (m[3]) launch_residual_planes<8>(a, m[3], grid, st);
    LQ_HIP_TRY(hipGetLastError());
    return LQ_OK;
  }
  hipLaunchKernelGGL(residual_kernel, dim3((unsigned)nwg), dim3(256), 0, st, a, groups);
  LQ_HIP_TRY(hipGetLastError());
  return LQ_OK;
}

}  // namespace lq
