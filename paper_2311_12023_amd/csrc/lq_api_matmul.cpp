// C ABI of the forward product with a decomposed weight (Section 3.2 "Implementation", Appendix A).
#include <algorithm>
#include <mutex>

#include "kernels.h"

namespace lq {
int check_quant_args(int64_t n, lq_config& c);

static size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }
static int64_t up32(int64_t x) { return (x + 31) & ~(int64_t)31; }

// Few rows of X: the product is bound by reading the weights and runs on the vector ALU (measured faster than the
// MFMA path up to 8 rows).
constexpr int64_t SMALL_M = QMATVEC_MAX_ROWS;
constexpr int SMALL_RANK = 512;
// Above this many rows precision 1 decodes the weights into a bf16 plane first (see planes_kernels.hip for both sides).
// On small weights without a low-rank part of more than 32 the launch more cost what it gained up to 1024 rows when the line was
// drawn.  Since the launch that adds T's partial tiles is gone it gains a little there too (1024 x 1024, 640 rows, with a plane
// against without: rank 0 32.4 and 29.2 us, rank 16 34.8 and 35.1, rank 32 34.7 and 37.3; 1024 rows, rank 16: 34.9 and 38.3).
constexpr int64_t PLANE_M = 512, PLANE_M_SMALL = 1024;

// Between 9 and 128 rows: whether qrows_kernel is ahead of qmatmul_kernel, whose time is that of 256 rows whatever m is.
// qrows_kernel decodes the weights once for every group of up to 48 rows, so it loses on large weights where it has three
// groups (97 rows and more; qrows against qmatmul in us at 112 rows, whole calls, precision 0 / 1, blocks of 64, with 32 within 4 %
// but for the largest):
//   rows of L1 that cannot be read as float4  8192^2, rank 65         135 / 139 against 142 / 98
//   T L2, on the vector ALU, for high ranks   4096 x 11008, rank 512  143 / 120 against 134 / 111  (11008 x 4096: 109 / 85 against 164 / 136)
//   bf16 operands and the largest weights     8192^2, rank 64         - / 83 against - / 80        (blocks of 32: 94 against 81)
// and elsewhere wins (4096 x 11008, 4 bits, rank 64: 79 / 58 against 88 / 67; rank 256: 103 / 81 against 124 / 103).  3-bit codes were
// 112 / 89 against 98 / 75 (4096 x 11008, rank 64) while each of their loads was waited for and are kept from it from 97 rows on; they
// are 87 / 64 against 96 / 71 now (4096^2 42 / 32 against 58 / 46), so that line could be taken out.
static bool rows_kernel_ahead(int64_t m, int64_t d, int64_t k, int rank, int bits, int precision) {
  const int64_t weights = d * k;
  const bool wide = k > d, odd = rank % 4 != 0;
  if (m <= 64 || weights < ((int64_t)1 << 24)) return true;
  if (m <= 96)
    return !(bits == 3 && rank >= 384 && wide && weights >= ((int64_t)1 << 25)) && !(odd && precision == 1 && weights >= ((int64_t)1 << 26));
  if (bits == 3 && rank == 0) return false;
  if (weights < ((int64_t)1 << 25)) return true;
  if (bits == 3 && (rank <= SPLIT_PROJECT_MAX_RANK || d <= k)) return false;
  if (rank >= 384 && wide) return false;
  if (odd && (precision == 1 || (wide && weights >= ((int64_t)1 << 26)))) return false;
  return !(weights >= ((int64_t)1 << 26) && rank <= SPLIT_PROJECT_MAX_RANK && (precision == 1 || rank == 0 || wide));
}

// The kernels a call can take.  Each needs a workspace of its own; where the one given is too small for the route that the
// sizes call for but holds the other that can serve the call, that one is taken.
enum Route { ROUTE_FEW, ROUTE_ROWS, ROUTE_PLANE, ROUTE_GENERAL };
static bool rows_route_serves(int64_t m, int rank) { return m <= QROWS_MAX_ROWS && rank <= QROWS_MAX_RANK; }
static Route preferred_route(int64_t m, int64_t d, int64_t k, int rank, int bits, int precision) {
  if (m <= SMALL_M && rank <= SMALL_RANK) return ROUTE_FEW;
  if (rows_route_serves(m, rank)) return rows_kernel_ahead(m, d, k, rank, bits, precision) ? ROUTE_ROWS : ROUTE_GENERAL;
  const int64_t from = d * k < ((int64_t)1 << 22) && rank <= 32 ? PLANE_M_SMALL : PLANE_M;
  return precision == 1 && m > from && rank <= SPLIT_PROJECT_MAX_RANK ? ROUTE_PLANE : ROUTE_GENERAL;
}
static int64_t padded_rows(int64_t m) { return (m + 255) / 256 * 256; }

struct MatmulPlan {
  bool fused;      // T = X L1 comes out of the pass that splits X (rank up to SPLIT_PROJECT_MAX_RANK)
  int64_t r32, rows_pad;
  // elements of the regions, in the order in which they lie in the workspace
  size_t xh, xl, t_floats, t_plane, part_floats, scale_floats;
  size_t w_plane, l_plane;   // ROUTE_PLANE: the weights and L2 in bf16
};
static MatmulPlan plan_matmul(Route route, int64_t m, int64_t d, int64_t k, int rank) {
  MatmulPlan p{};
  if (route == ROUTE_FEW) {
    p.part_floats = qmatvec_part_floats((int)std::min<int64_t>(m, QMATVEC_MAX_ROWS), d, k, rank);
    return p;
  }
  if (route == ROUTE_ROWS) {
    p.part_floats = qrows_part_floats(m, d, k, rank);
    return p;
  }
  p.r32 = up32(rank);
  p.rows_pad = padded_rows(m);
  p.fused = rank > 0 && rank <= SPLIT_PROJECT_MAX_RANK;
  p.xh = (size_t)p.rows_pad * (size_t)(route == ROUTE_PLANE ? plane_pitch(d) : d);
  p.xl = route == ROUTE_PLANE && p.fused ? 0 : p.xh;   // split_project_kernel leaves it alone for bf16 operands
  p.t_floats = rank > 0 && !p.fused ? (size_t)m * (size_t)p.r32 : 0;
  p.t_plane = rank > 0 ? (size_t)p.rows_pad * (size_t)p.r32 : 0;
  const size_t p1 = p.fused ? split_project_part_floats(p.rows_pad, d)
                            : rank > 0 ? qmatmul_part_floats(m, p.r32, (int)(d / 32)) : 0;
  const size_t p2 = qmatmul_part_floats(m, k, (int)(d / 32 + p.r32 / 32));
  p.part_floats = p1 > p2 ? p1 : p2;
  if (route == ROUTE_PLANE) {
    p.w_plane = weight_plane_elems(plane_pitch(d), k);
    p.l_plane = rank > 0 ? weight_plane_elems(p.r32, k) : 0;
  } else {
    p.scale_floats = (size_t)(d * k / 16);          // one scale per block, block size at least 16
  }
  return p;
}
static size_t plan_bytes(const MatmulPlan& p) {
  return up256(p.xh * 2) + up256(p.xl * 2) + up256(p.t_floats * 4) + 2 * up256(p.t_plane * 2) + up256(p.part_floats * 4) +
         up256(p.scale_floats * 4) + up256(p.w_plane * 2) + up256(p.l_plane * 2) + 256;
}
static size_t route_bytes(Route route, int64_t m, int64_t d, int64_t k, int rank) {
  return plan_bytes(plan_matmul(route, m, d, k, rank));
}

// What m rows need, whatever the code width, and, beyond the few, no less than any number of rows up to QROWS_MAX_ROWS needs: those sizes rise and fall
// with m as reductions are cut less, and a caller sizes once for batches that come and go.  Among the rows of ROUTE_ROWS
// only whole tiles of 16 have to be looked at, between which the cut stays the same.
static size_t workspace_bytes_for(int64_t m, int64_t d, int64_t k, int rank, int precision) {
  if (m <= SMALL_M && rank <= SMALL_RANK) return route_bytes(ROUTE_FEW, m, d, k, rank);
  size_t need = 0;
  for (int bits : {3, 4}) need = std::max(need, route_bytes(preferred_route(m, d, k, rank, bits, precision), m, d, k, rank));
  if (rank <= SMALL_RANK)
    for (int64_t r = 1; r <= SMALL_M; ++r) need = std::max(need, route_bytes(ROUTE_FEW, r, d, k, rank));
  if (rank <= QROWS_MAX_RANK)
    for (int64_t r = 16; r <= QROWS_MAX_ROWS; r += 16) need = std::max(need, route_bytes(ROUTE_ROWS, r, d, k, rank));
  return need;
}

// Scratch of lq_matmul_few_rows_static: a fixed array in device memory (every GPU the library runs on holds its own copy
// until the process ends).  Host code never uses the array's name as an address: the device address is looked up once per
// device and kept.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[64] = {nullptr};

static int static_scratch(void** out) {
  int dev = 0;
  LQ_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return LQ_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    LQ_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return LQ_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LQ_OK;
}
}  // namespace lq

using namespace lq;

extern "C" {

size_t lq_matmul_workspace_bytes_precision(int64_t m, int64_t d, int64_t k, int rank, int precision) {
  if (m <= 0 || d <= 0 || k <= 0 || rank < 0 || (d % 32) != 0 || (precision != 0 && precision != 1)) return 0;
  return workspace_bytes_for(m, d, k, rank, precision);
}

size_t lq_matmul_workspace_bytes(int64_t m, int64_t d, int64_t k, int rank) {
  return std::max(lq_matmul_workspace_bytes_precision(m, d, k, rank, 0),
                  lq_matmul_workspace_bytes_precision(m, d, k, rank, 1));
}

int lq_matmul(const float* X, int64_t m, int64_t d, int64_t k, const uint8_t* codes_packed, const uint8_t* scale_idx,
              const float* v, lq_config c, const float* L1, const float* L2, int rank, int precision, float* Y,
              void* workspace, size_t workspace_bytes, void* stream) {
  if (!X || !codes_packed || !scale_idx || !v || !Y) return LQ_ERR_NULL;
  if (rank < 0 || rank > 1024) return LQ_ERR_RANK;
  if (rank > 0 && (!L1 || !L2)) return LQ_ERR_NULL;
  if (m <= 0 || d <= 0 || k <= 0 || m >= ((int64_t)1 << 31) || d >= ((int64_t)1 << 31) || k >= ((int64_t)1 << 31))
    return LQ_ERR_SHAPE;
  if ((d % 32) != 0) return LQ_ERR_SHAPE;
  LQ_TRY(check_quant_args(d * k, c));
  if ((k % c.block) != 0) return LQ_ERR_SHAPE;
  if (precision != 0 && precision != 1) return LQ_ERR_ARG;
  if (((uintptr_t)X & 15) != 0 || ((uintptr_t)Y & 15) != 0 || (rank > 0 && ((uintptr_t)L2 & 15) != 0)) return LQ_ERR_ARG;
  Route route = preferred_route(m, d, k, rank, c.bits, precision);
  // 32-bit byte offsets into the planes of X and into the codes
  if (route != ROUTE_FEW && (padded_rows(m) * d >= ((int64_t)1 << 31) || d * k >= ((int64_t)1 << 31))) return LQ_ERR_SHAPE;
  MatmulPlan p = plan_matmul(route, m, d, k, rank);
  if (workspace_bytes < plan_bytes(p) && route != ROUTE_FEW) {
    route = route == ROUTE_GENERAL && rows_route_serves(m, rank) ? ROUTE_ROWS : ROUTE_GENERAL;
    p = plan_matmul(route, m, d, k, rank);
  }
  if (!workspace || ((uintptr_t)workspace & 255) != 0 || workspace_bytes < plan_bytes(p)) return LQ_ERR_WORKSPACE;
  char* w = reinterpret_cast<char*>(workspace);
  hipStream_t st = (hipStream_t)stream;
  if (route == ROUTE_FEW) {
    float* part = reinterpret_cast<float*>(w);           // the only region of the plan that is not empty
    const MvWeights q{codes_packed, scale_idx, v, c.bits, c.block, c.scale_block, scale_levels(c)};
    for (int64_t r0 = 0; r0 < m; r0 += QMATVEC_MAX_ROWS) {
      const int mc = (int)std::min<int64_t>(QMATVEC_MAX_ROWS, m - r0);
      LQ_TRY(launch_qmatvec(q, X + r0 * d, d, d, L1, L2, k, rank, mc, k, Y + r0 * k, k, part, p.part_floats, st));
    }
    return LQ_OK;
  }
  if (route == ROUTE_ROWS) {
    const MvWeights q{codes_packed, scale_idx, v, c.bits, c.block, c.scale_block, scale_levels(c)};
    return launch_qrows(q, X, d, d, L1, L2, k, rank, m, k, precision, Y, k, reinterpret_cast<float*>(w), p.part_floats, st);
  }
  uint16_t* xh = reinterpret_cast<uint16_t*>(w); w += up256(p.xh * 2);
  uint16_t* xl = reinterpret_cast<uint16_t*>(w); w += up256(p.xl * 2);
  float* T = reinterpret_cast<float*>(w); w += up256(p.t_floats * 4);
  uint16_t* th = reinterpret_cast<uint16_t*>(w); w += up256(p.t_plane * 2);
  uint16_t* tl = reinterpret_cast<uint16_t*>(w); w += up256(p.t_plane * 2);
  float* part = reinterpret_cast<float*>(w); w += up256(p.part_floats * 4);
  float* bscale = reinterpret_cast<float*>(w); w += up256(p.scale_floats * 4);
  uint16_t* wt = reinterpret_cast<uint16_t*>(w); w += up256(p.w_plane * 2);
  uint16_t* lt = reinterpret_cast<uint16_t*>(w);

  if (route == ROUTE_PLANE) {
    ProjectSum t{};
    if (p.fused)
      LQ_TRY(launch_split_project(X, m, d, d, p.rows_pad, L1, rank, precision, plane_pitch(d), xh, xl, part, p.part_floats, th, tl,
                                  (int)p.r32, BlockScales{}, &t, st));
    else
      LQ_TRY(launch_split_planes(X, m, d, d, p.rows_pad, plane_pitch(d), xh, xl, st));
    const MvWeights q{codes_packed, scale_idx, v, c.bits, c.block, c.scale_block, scale_levels(c)};
    return launch_plane_product(q, xh, d, th, (int)p.r32, L2, rank, m, p.rows_pad, k, wt, lt, Y, k, part, p.part_floats, t, st);
  }
  QmmPart none{};
  if (p.fused) {    // planes of X and of T = X L1 from one pass over X, the block scales of Q in the same launch
    const BlockScales bs{scale_idx, v, d * k / c.block, c.scale_block, scale_levels(c), bscale};
    LQ_TRY(launch_split_project(X, m, d, d, p.rows_pad, L1, rank, precision, d, xh, xl, part, p.part_floats, th, tl,
                                (int)p.r32, bs, nullptr, st));
  } else {
    LQ_TRY(launch_block_scales(scale_idx, v, d * k / c.block, c.scale_block, scale_levels(c), bscale, st));
    LQ_TRY(launch_split_planes(X, m, d, d, p.rows_pad, d, xh, xl, st));
  }
  if (rank > 0 && !p.fused) {   // T = X L1, m x r32 with zero columns beyond r, then its planes
    DensePart xl1{xh, xl, d, L1, rank, d, rank};
    LQ_TRY(launch_qmatmul(none, xl1, m, p.rows_pad, p.r32, T, p.r32, part, p.part_floats, precision, st));
    LQ_TRY(launch_split_planes(T, m, p.r32, p.r32, p.rows_pad, p.r32, th, tl, st));
  }
  QmmPart q{xh, xl, d, codes_packed, bscale, c.bits, c.block};
  DensePart tl2{th, tl, rank > 0 ? p.r32 : 0, L2, k, rank, k};
  return launch_qmatmul(q, tl2, m, p.rows_pad, k, Y, k, part, p.part_floats, precision, st);
}

size_t lq_matmul_few_rows_static_scratch_bytes(void) { return STATIC_SCRATCH_BYTES; }

int lq_matmul_few_rows_static(const float* X, int64_t m, int64_t d, int64_t k, const uint8_t* codes_packed,
                              const uint8_t* scale_idx, const float* v, lq_config c, const float* L1, const float* L2,
                              int rank, float* Y, void* stream) {
  if (!X || !codes_packed || !scale_idx || !v || !Y) return LQ_ERR_NULL;
  if (rank < 0 || rank > SMALL_RANK) return LQ_ERR_RANK;
  if (rank > 0 && (!L1 || !L2)) return LQ_ERR_NULL;
  if (m <= 0 || m > SMALL_M || d <= 0 || k <= 0 || d >= ((int64_t)1 << 31) || k >= ((int64_t)1 << 31)) return LQ_ERR_SHAPE;
  if ((d % 32) != 0) return LQ_ERR_SHAPE;
  LQ_TRY(check_quant_args(d * k, c));
  if ((k % c.block) != 0) return LQ_ERR_SHAPE;
  if (((uintptr_t)X & 15) != 0 || ((uintptr_t)Y & 15) != 0 || (rank > 0 && ((uintptr_t)L2 & 15) != 0)) return LQ_ERR_ARG;
  const size_t part_floats = qmatvec_part_floats((int)m, d, k, rank);
  if (part_floats * sizeof(float) > STATIC_SCRATCH_BYTES) return LQ_ERR_WORKSPACE;   // beyond the fixed scratch: use lq_matmul
  void* sp = nullptr;
  LQ_TRY(static_scratch(&sp));
  const MvWeights q{codes_packed, scale_idx, v, c.bits, c.block, c.scale_block, scale_levels(c)};
  // every partial sum the second kernel reads is written by the first in the same call: nothing has to start at zero
  return launch_qmatvec(q, X, d, d, L1, L2, k, rank, (int)m, k, Y, k, reinterpret_cast<float*>(sp),
                        STATIC_SCRATCH_BYTES / sizeof(float), (hipStream_t)stream);
}

}  // extern "C"
