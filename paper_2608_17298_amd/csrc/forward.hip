// Forward software trace (Sec. 3.2-3.3, Eq. 3-8) writing the (L, T)
// intermediate buffer in primitive-major order (Sec. 4.3, Eq. 16).
//
// One wave per 8x8 pixels, one lane per pixel.  The tile's Gaussian list is
// ordered by a lower bound on the depth at which each Gaussian can be hit by
// a pixel ray of the tile, so a lane can stream it front to back with a small
// sorted pool of pending hits: a pending hit is final -- and is composited
// -- as soon as its depth is below the bound of the next Gaussian in the list.
// The result is exactly the (tau, index) order.
//
// What bounds it: the instructions of a wave's chain (33 steps of four
// candidates and 60 compositing steps per tile at 1M Gaussians, half of them
// fp64) at the two waves per SIMD that the pools' LDS leaves, and about a
// sixth of the time the waits for rows.  A branch costs a lone wave some 45
// cycles, ten times an fp64 operation, and a load issued in the chain its
// whole latency.  So:
//  - The list is taken in chunks of 64 positions, one per lane: rectangles
//    become 64-bit masks of the wave's pixels, and the candidates that no
//    working lane can hit are dropped by a permutation of the lanes.
//  - The rest come in groups of four, whose rows (geometry, SH) are loaded a
//    group ahead and staged in LDS.  The four ray tests, exponentials and pool
//    insertions are straight-line code for all lanes.
//  - Colours are evaluated where a Gaussian is the same for the whole wave, on
//    the matrix cores (4x4x1 fp32: one block per four pixels, the SH block of
//    the four candidates broadcast), instead of 3K scattered loads and 3K
//    FMAs per composited hit.
//  - The pool is a sorted list of 32-bit keys in registers (the depth as a
//    float, its low bits replaced by the hit's payload slot) and the payload
//    (alpha, colour, list position) in LDS; a chain of medians inserts a key.
//    Hits whose keys tie are ordered on their exact depths, recomputed.
// Against one candidate at a time, branches around each part and colours at
// the compositing (ms): 1M Gaussians 1.47 -> 0.93, 4M 2.52 -> 1.56, 100k 0.57
// -> 0.36, 150k large 9.9 -> 5.64, 250k on 16x16 tiles 1.91 -> 0.54, 4k 0.41
// -> 0.12.
// If a pool overflows, its largest hit in (depth, index) order is dropped --
// exact depths, recomputed, decide between equal keys -- and the lane later
// rescans the list from the first Gaussian it dropped, skipping hits already
// composited, so that every pass composites at least a pool of hits, also where
// all depths are equal (copies of one Gaussian, flat Gaussians in one plane);
// compositing stops once the transmittance falls below t_min.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>

#include "ops.h"

namespace gart {
namespace {

constexpr int kGroup = 4;     // candidates per step (sixteen lanes load each one's row)
constexpr int kChunk = 64;    // list positions looked at together, one per lane
constexpr int kWindow = 128;  // list positions whose (L,T) addressing is kept in LDS
constexpr int kPoolSpare = 4;  // free entries below which a lane's final hits are composited

// Each pass composites at least a pool of hits per lane that rescans after it,
// so the pass count is bounded by the hits of a tile; this cap only guards against a
// defect turning into a hang, and is reported in the frame status if reached.
constexpr int kMaxPasses = 1 << 20;

using f32x4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;

// Orders LDS accesses of the (single-wave) block: LDS executes a wave's
// accesses in issue order, so only the compiler has to keep them.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane(int(uint32_t(v)), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(int(uint32_t(v >> 32)), lane);
  return uint64_t(hi) << 32 | lo;
}

__device__ __forceinline__ bool lane_bit(uint64_t wave_mask) { return __builtin_amdgcn_inverse_ballot_w64(wave_mask); }

// d[r] (r = 0..3) += sum_k a_k[r] * Y[k] per lane, a_k[r] = a of lane 4k + r:
// the SH sums of four Gaussians (one channel) at the lane's pixel.
template <int... Ks>
__device__ __forceinline__ void sh_mfma(std::integer_sequence<int, Ks...>, float r, float g, float b, const float* Y,
                                        f32x4& dr, f32x4& dg, f32x4& db) {
  ((dr = __builtin_amdgcn_mfma_f32_4x4x1f32(r, Y[Ks], dr, 4, Ks, 0),
    dg = __builtin_amdgcn_mfma_f32_4x4x1f32(g, Y[Ks], dg, 4, Ks, 0),
    db = __builtin_amdgcn_mfma_f32_4x4x1f32(b, Y[Ks], db, 4, Ks, 0)),
   ...);
}

// Non-negative colour -> the frame's fixed point, rounded to nearest by the
// addition of 2^52 (the integer is the low word of the sum); values from 2^32
// on and NaN saturate.
__device__ __forceinline__ uint32_t color_fixed_fma(double v, double inv_step) {
  const uint64_t u = __double_as_longlong(fma(v, inv_step, 0x1p52));
  return uint32_t(u >> 32) == 0x43300000u ? uint32_t(u) : 0xffffffffu;
}

// 2^(j / 64) for j = 0 .. 63 is kept in LDS: exp(-D2 / 2) = 2^(n / 64) 2^(r / 64)
// with n integer and |r| <= 1/2, the second factor by its Taylor series to the
// fifth order (remainder below 2^-54).
constexpr int kExpSteps = 64;
__constant__ const double kExp2[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};
__device__ __forceinline__ double exp_neg_half(double D2, const double* table) {
  constexpr double kC = -0x1.71547652b82fep+5;  // -64 log2(e) / 2, and what its rounding leaves
  constexpr double kCLow = -0x1.777d0ffda0d24p-51;
  constexpr double k1 = 0x1.62e42fefa39efp-7;  // ln 2 / 64, and its powers over i!
  constexpr double k2 = k1 * k1 / 2, k3 = k2 * k1 / 3, k4 = k3 * k1 / 4, k5 = k4 * k1 / 5;
  const double t = fma(D2, kC, 0x1.8p52);
  const int n = int(uint32_t(__double_as_longlong(t)));
  const double nd = t - 0x1.8p52;
  const double r = fma(D2, kCLow, fma(D2, kC, -nd));
  const double q = r * fma(r, fma(r, fma(r, fma(r, k5, k4), k3), k2), k1);
  const uint64_t u = __double_as_longlong(table[n & (kExpSteps - 1)]);
  const double f = __longlong_as_double(u + (uint64_t(uint32_t((n & ~(kExpSteps - 1)) << 14)) << 32));
  return fma(f, q, f);
}

// max(x, 0); 0 for NaN.
__device__ __forceinline__ float max_zero(float x) {
  float r;
  asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(x));
  return r;
}

// LDS writes by the lanes of the mask (a branch around them would cost more
// than they do).
__device__ __forceinline__ void lds_write_masked(uint64_t mask, uint4* p4, uint4 v4, uint2* p2, uint2 v2) {
  using u32x4 = __attribute__((__vector_size__(16))) uint32_t;
  using u32x2 = __attribute__((__vector_size__(8))) uint32_t;
  const uint32_t a4 = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint4*)p4));
  const uint32_t a2 = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint2*)p2));
  const u32x4 w4 = {v4.x, v4.y, v4.z, v4.w};
  const u32x2 w2 = {v2.x, v2.y};
  uint64_t exec;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %1\n\t"
      "ds_write_b128 %2, %3\n\t"
      "ds_write_b64 %4, %5\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(exec)
      : "s"(mask), "v"(a4), "v"(w4), "v"(a2), "v"(w2)
      : "memory");
}

__device__ __forceinline__ f32x4 rot(f32x4 v) { return f32x4{v[1], v[2], v[3], v[0]}; }

// Pixels of the wave's 8x8 block (bit 8 y + x) inside the rectangle r.
__device__ __forceinline__ uint64_t rect_mask(int4 r, int ox, int oy) {
  // columns and rows as 8-bit masks; a row bit becomes a byte of columns
  const int x0 = min(max(r.x - ox, 0), 8), x1 = max(min(r.z - ox, 7), -1);
  const int y0 = min(max(r.y - oy, 0), 8), y1 = max(min(r.w - oy, 7), -1);
  const uint32_t col = (0xffu >> (7 - x1)) & (0xffu << x0) & 0xffu, row = (0xffu >> (7 - y1)) & (0xffu << y0) & 0xffu;
  const uint32_t lo = ((row & 15u) * 0x204081u & 0x01010101u) * col;
  const uint32_t hi = ((row >> 4) * 0x204081u & 0x01010101u) * col;
  return uint64_t(hi) << 32 | lo;
}

template <int TILE, int K, int FMT, int KB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void forward_kernel(ForwardArgs A) {
  constexpr int NT = TILE * TILE;
  constexpr int G = NT / 64;  // 8x8 blocks (waves) per tile
  constexpr uint32_t SM = 15u;  // payload slot bits of a pool key
  constexpr uint32_t kEmpty = UINT_MAX;
  constexpr double kInf = __builtin_huge_val();
  static_assert(KB >= 2 && KB <= 15, "pool slots fit the key's low bits (15 is an empty entry's)");

  __shared__ __align__(16) double s_row[kGroup * 16];  // W (9), o_g (3), D2c, sigma, -, -
  __shared__ uint4 s_win[kWindow];                     // (L,T) address (64 bits), row length, Gaussian index
  __shared__ double s_exp[kExpSteps];
  __shared__ uint4 s_pa[KB * 64];                      // payload: alpha (fp64), colour r, g
  __shared__ uint2 s_pb[KB * 64];                      //          colour b, list position

  const int n_tiles = A.tiles_x * A.tiles_y;
  const int lane = threadIdx.x;
  int slot_of_tile = blockIdx.x, grp = 0;
  if constexpr (G > 1) {  // the waves of a tile on one XCD (blocks reach the XCDs round-robin)
    slot_of_tile = int(blockIdx.x / (8 * G)) * 8 + int(blockIdx.x % 8);
    grp = int(blockIdx.x / 8) % G;
    if (slot_of_tile >= n_tiles) return;
  }
  const int tile = xcd_tile(slot_of_tile, n_tiles, A.tiles_x);
  const int tx = tile % A.tiles_x, ty = tile / A.tiles_x;
  constexpr int kBlocksX = TILE / 8;
  const int ox = tx * TILE + 8 * (grp % kBlocksX), oy = ty * TILE + 8 * (grp / kBlocksX);
  const int px = ox + lane % 8, py = oy + lane / 8;
  const int q_tile = (py - ty * TILE) * TILE + (px - tx * TILE);  // pixel of the tile, row-major
  const bool valid = px < A.cam.W && py < A.cam.H;

  // The tile's list keys are depths along the tile's axis; key k bounds the
  // depth of a hit on this pixel's ray by k * kscale (0: by nothing).
  double d[3];
  const float kscale = pixel_ray_scale(A.cam, valid ? px : 0, valid ? py : 0, tx, ty, TILE, d);
  float Y[K];  // SH basis of this pixel's ray
  sh_basis<K>(float(d[0]), float(d[1]), float(d[2]), Y);

  const int64_t beg = A.tile_range[tile];
  const int n = int(A.tile_range[tile + 1] - beg);  // below the number of Gaussians, 2^31
  const int64_t hl_beg = A.hl_off[tile];  // this tile's first hit_list row
  // its rows (>= 1 if the tile has pairs); a hit beyond them, which the
  // bound on hits per pixel excludes, would overwrite the last row and is
  // reported in the frame status after the trace
  const uint32_t hl_last = uint32_t(max<int64_t>(A.hl_off[tile + 1] - hl_beg, 1) - 1);
  uint32_t* const hl = A.hit_list + int64_t(NT) * hl_beg;
  s_exp[lane] = kExp2[lane];
  const uint32_t* prim = A.pair_prim + beg;
  const float* pkey = A.pair_key + beg;

  double T = 1.0, L0 = 0.0, L1 = 0.0, L2 = 0.0;
  uint32_t n_hits = 0, n_drops = 0;
  uint32_t n_tests = 0;  // of the wave
  uint32_t visited = 0;  // one past the largest list position composited
  double last_tau = -kInf;
  uint32_t last_id = 0;

  // Pool: keys a[0 .. cnt) ascending, the rest kEmpty; the free payload slots
  // as a stack of 4-bit numbers.
  uint32_t a[KB];
#pragma unroll
  for (int s = 0; s < KB; ++s) a[s] = kEmpty;
  uint32_t cnt = 0;
  uint64_t free_slots = 0xfedcba9876543210ull;
  // The smallest dropped hit in (depth, index) order; every pooled hit is
  // before it.  Its depth and index are found from its list position when
  // first needed (e_tau: NaN until then).
  uint32_t e_key = UINT_MAX;  // its depth key (low bits clear)
  double e_tau = kInf;
  uint32_t e_id = kNoPrim, e_pos = 0;
  uint32_t jr = UINT_MAX;  // first list position holding a dropped hit
  // A rescan starts the wave at the smallest jr of its lanes; a lane skips
  // the positions before its own jr (from): every hit there was composited
  // in an earlier pass.
  uint32_t from = 0;
  uint32_t win_lo = 0;  // list positions from here on are in s_win

  auto exact_tau = [&](uint32_t id) {
    const double* Gm = A.geom + int64_t(kGeomStride) * id;
    double W[9], og[3];
#pragma unroll
    for (int k = 0; k < 9; ++k) W[k] = Gm[kGeoW + k];
#pragma unroll
    for (int k = 0; k < 3; ++k) og[k] = Gm[kGeoOg + k];
    double tau, D2, xg[3];
    ray_hit(W, og, Gm[kGeoD2c], d, &tau, &D2, xg);
    return tau;
  };

  // Among the pooled hits of key top, which are the pool's first (FIRST) or
  // last ones: the payload slot of the smallest (FIRST) or largest one in
  // (depth, index) order, if it is before (after) (t, i), which it replaces;
  // else UINT_MAX.  Four ray tests at a time, for the latency of their rows (60000
  // flat Gaussians in one plane, 116 hits a ray, ms: 59, two 53, four 48).
  auto tied_entry = [&](auto first, uint32_t top, double& t, uint32_t& i) {
    constexpr bool FIRST = decltype(first)::value;
    constexpr int N = 4;
    uint32_t slot = UINT_MAX;
#pragma unroll 1
    for (int s0 = 0; s0 < KB; s0 += N) {
      uint32_t as[N], id[N];
      double ts[N];
      bool ok[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int s = FIRST ? s0 + j : KB - 1 - s0 - j;
        as[j] = kEmpty;
#pragma unroll
        for (int k = 0; k < KB; ++k) as[j] = k == s ? a[k] : as[j];
        ok[j] = as[j] != kEmpty && (as[j] & ~SM) == top;
        const uint32_t pos = s_pb[min(as[j] & SM, uint32_t(KB - 1)) * 64 + lane].y;
        id[j] = prim[ok[j] ? pos : 0u];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) ts[j] = exact_tau(id[j]);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const bool take = ok[j] && (FIRST ? key_less(ts[j], id[j], t, i) : key_less(t, i, ts[j], id[j]));
        slot = take ? as[j] & SM : slot;
        t = take ? ts[j] : t;
        i = take ? id[j] : i;
      }
      if (!ok[N - 1]) break;
    }
    return slot;
  };

  // (L,T) entry of pixel (ox + x, oy + y) = that of (ox, oy) + y w + x inside
  // rect cap tile (Eq. 16).  Returns the address of pixel (ox, oy)'s, which
  // may itself lie outside the rectangle.
  constexpr int kEntryBytes = FMT == GART_LT_FULL ? 16 : FMT == GART_LT_T_ONLY ? 4
                              : FMT == GART_LT_HALF || FMT == GART_LT_FIXED16 ? 8 : 2;
  auto lt_origin = [&](int4 r, int64_t off, int* w) -> uint64_t {
    const int xa = max(r.x, tx * TILE), xb = min(r.z, tx * TILE + TILE - 1);
    const int ya = max(r.y, ty * TILE), yb = min(r.w, ty * TILE + TILE - 1);
    *w = xb - xa + 1;
    const int64_t e = off + int64_t(r.z - r.x + 1) * (ya - r.y) + int64_t(yb - ya + 1) * (xa - r.x) +
                      (oy - ya) * *w + (ox - xa);
    return reinterpret_cast<uint64_t>(A.lt) + uint64_t(e * kEntryBytes);
  };

  // Smallest depth a key can stand for is below its float; the float above
  // the key's low bits exceeds every depth it can stand for.  nb: float bits
  // at or below the depth bound of everything not yet tested.
  auto is_final = [&](uint32_t key, uint32_t nb) { return (key | SM) < nb; };
  auto bound_bits = [&](float key) {
    const float b = key * kscale;  // rounded; one ulp less is below the product
    return b > 0.0f ? __float_as_uint(b) - 1u : 0u;  // 0 * inf (no scale, the list's end) bounds nothing either
  };

  // Payload of the lane's smallest pooled hit (any, if there is none).
  uint4 pa;
  uint2 pb;
  auto load_head = [&]() {
    const uint32_t slot = min(a[0] & SM, uint32_t(KB - 1));
    pa = s_pa[slot * 64 + lane];
    pb = s_pb[slot * 64 + lane];
  };

  // Composites the lane's smallest pooled hit, whose payload is loaded, and
  // loads the payload of the next.
  auto composite = [&]() {
    uint32_t slot = a[0] & SM;
    uint4 wn = s_win[pb.y % kWindow];
    const bool tie = (a[0] ^ a[1]) <= SM;
    const bool staged = pb.y >= win_lo;  // its addressing is in s_win
    if (__builtin_expect(__ballot(tie || !staged) == 0, 1)) {
#pragma unroll
      for (int s = 0; s + 1 < KB; ++s) a[s] = a[s + 1];
    } else {
      bool past = true;  // the entries from this hit's on move down
      if (tie) {
        double bt = kInf;
        uint32_t bid = kNoPrim;
        slot = tied_entry(std::true_type{}, a[0] & ~SM, bt, bid);
        past = false;
        pa = s_pa[slot * 64 + lane];
        pb = s_pb[slot * 64 + lane];
      }
#pragma unroll
      for (int s = 0; s + 1 < KB; ++s) {
        past = past || (a[s] & SM) == slot;
        a[s] = past ? a[s + 1] : a[s];
      }
      if (pb.y >= win_lo) {
        wn = s_win[pb.y % kWindow];
      } else {
        const uint32_t id = prim[pb.y];
        int w;
        const uint64_t at = lt_origin(*reinterpret_cast<const int4*>(A.rect + 4 * int64_t(id)), A.lt_offset[id], &w);
        wn = make_uint4(uint32_t(at), uint32_t(at >> 32), uint32_t(w), id);
      }
    }
    a[KB - 1] = kEmpty;
    --cnt;
    free_slots = free_slots << 4 | slot;
    const uint32_t cpos = pb.y;
    const uint32_t ofs = uint32_t(lane / 8) * wn.z + uint32_t(lane % 8);
    void* const lt = reinterpret_cast<void*>((uint64_t(wn.y) << 32 | wn.x) + ofs * uint32_t(kEntryBytes));
    const double al = __longlong_as_double(int64_t(uint64_t(pa.y) << 32 | pa.x));
    const float c[3] = {max_zero(__uint_as_float(pa.z)), max_zero(__uint_as_float(pa.w)),
                        max_zero(__uint_as_float(pb.x))};
    load_head();
    visited = max(visited, cpos + 1u);
    // k-th composited hit of this pixel -> its list position (read by the
    // gather backward)
    hl[uint64_t(min(n_hits, hl_last)) * NT + q_tile] = cpos;
    if constexpr (FMT == GART_LT_FULL) {
      *static_cast<uint4*>(lt) = make_uint4(color_fixed_fma(L0, A.inv_color_step), color_fixed_fma(L1, A.inv_color_step),
                           color_fixed_fma(L2, A.inv_color_step), __float_as_uint(float(T)));
    } else if constexpr (FMT == GART_LT_T_ONLY) {
      *static_cast<float*>(lt) = float(T);
    } else if constexpr (FMT == GART_LT_HALF) {
      *static_cast<uint2*>(lt) = make_uint2(half_bits(float(L0)) | (half_bits(float(L1)) << 16),
                                                     half_bits(float(L2)) | (half_bits(float(T)) << 16));
    } else if constexpr (FMT == GART_LT_FIXED16) {
      const double inv16 = A.inv_color_step * (1.0 / 65536.0);
      *static_cast<uint2*>(lt) = make_uint2(
          min(color_fixed_fma(L0, inv16), 65535u) | (min(color_fixed_fma(L1, inv16), 65535u) << 16),
          min(color_fixed_fma(L2, inv16), 65535u) | (t_log16(float(T)) << 16));
    } else if constexpr (FMT == GART_LT_T_LOG16) {
      *static_cast<uint16_t*>(lt) = uint16_t(t_log16(float(T)));
    } else {
      *static_cast<uint16_t*>(lt) = uint16_t(half_bits(float(T)));
    }
    const double w = T * al;
    L0 = fma(w, double(c[0]), L0);
    L1 = fma(w, double(c[1]), L1);
    L2 = fma(w, double(c[2]), L2);
    T = T * (1.0 - al);
    ++n_hits;
    last_id = wn.w;
  };

  // A hit into the pool (which has room): payload, then the key by a chain of
  // medians (each entry: the middle of itself, its lower neighbour and x).
  auto payload = [&](double alpha, float c0, float c1, float c2, uint32_t cpos, uint4* pa, uint2* pb) {
    const uint64_t ab = uint64_t(__double_as_longlong(alpha));
    *pa = make_uint4(uint32_t(ab), uint32_t(ab >> 32), __float_as_uint(c0), __float_as_uint(c1));
    *pb = make_uint2(__float_as_uint(c2), cpos);
  };
  auto sort_in = [&](uint32_t x) {
#pragma unroll
    for (int s = KB - 1; s >= 1; --s) a[s] = max(min(a[s], x), min(max(a[s], x), a[s - 1]));
    a[0] = min(a[0], x);
  };
  auto insert = [&](uint32_t key, double alpha, float c0, float c1, float c2, uint32_t cpos) {
    const uint32_t slot = uint32_t(free_slots) & SM;
    payload(alpha, c0, c1, c2, cpos, &s_pa[slot * 64 + lane], &s_pb[slot * 64 + lane]);
    free_slots >>= 4;
    ++cnt;
    sort_in(key | slot);
  };

  // The chunk of the list after the current one, a position per lane.
  int4 nx_rect;
  int64_t nx_off;
  float nx_key, nx_key_end;
  uint32_t nx_id, nx2_id;
  auto load_id = [&](int p0) { return prim[min(p0 + lane, n - 1)]; };
  auto load_chunk = [&](int p0) {  // of the candidates nx_id from list position p0 on
    nx_rect = *reinterpret_cast<const int4*>(A.rect + 4 * int64_t(nx_id));
    nx_off = A.lt_offset[nx_id];
    nx_key = pkey[min(p0 + lane, n - 1)];
    nx_key_end = pkey[min(p0 + kChunk, n - 1)];
  };
  // The rows of the group after the current one: lane 16 c + v loads double v
  // of candidate c, lane 4 k + c the SH coefficient k of candidate c.
  double nx_row;
  float nx_sh[3];
  auto load_rows = [&](uint32_t ids, int g) {  // ids: one per lane, the group starts at lane g
    nx_row = A.geom[int64_t(kGeomStride) * uint32_t(__shfl(int(ids), min(g + lane / 16, 63))) + lane % 16];
    const uint32_t id = __shfl(int(ids), min(g + lane % 4, 63));
    const float* sp = A.sh + (int64_t(id) * K + (K == 16 ? lane / 4 : min(lane / 4, K - 1))) * 3;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) nx_sh[ch] = sp[ch];
  };

  uint32_t restart = 0;
  int passes = 0;  // rescans so far

  // Lane states as wave masks: working lanes (neither terminated, nor at the
  // end of their hits, nor stalled until a rescan), terminated lanes.
  uint64_t work = __ballot(valid), term = ~work;
  for (; n > 0 && work != 0;) {  // (a block of the tile may lie outside the image)
    bool careful = passes > 0;  // hits may have to be skipped or dropped
    nx_id = load_id(int(restart));
    load_chunk(int(restart));
    nx2_id = load_id(int(restart) + kChunk);
    // The current chunk's candidates with a working pixel, moved to the first
    // lanes in list order: index, pixel mask, list key, list position.
    uint32_t c_id = 0, c_lo = 0, c_hi = 0, c_key = 0, c_pos = 0;
    float key_end = 0.0f;  // list key after the chunk
    int n_live = 0;
    auto next_chunk = [&](int base) {
      lds_order();
      const int pos = base + lane;
      int w;
      const uint64_t at = lt_origin(nx_rect, nx_off, &w);
      s_win[uint32_t(pos) % kWindow] = make_uint4(uint32_t(at), uint32_t(at >> 32), uint32_t(w), nx_id);
      const uint64_t mask = pos < n ? rect_mask(nx_rect, ox, oy) : 0;
      const uint64_t live = __ballot((mask & work) != 0);
      n_live = __popcll(live);
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(live >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(live), 0u));
      const int to = 4 * int((mask & work) != 0 ? below : uint32_t(n_live) + uint32_t(lane) - below);
      c_id = __builtin_amdgcn_ds_permute(to, int(nx_id));
      c_lo = __builtin_amdgcn_ds_permute(to, int(uint32_t(mask)));
      c_hi = __builtin_amdgcn_ds_permute(to, int(uint32_t(mask >> 32)));
      c_key = __builtin_amdgcn_ds_permute(to, __float_as_int(nx_key));
      c_pos = __builtin_amdgcn_ds_permute(to, pos);
      key_end = base + kChunk < n ? nx_key_end : __int_as_float(0x7f800000);
      win_lo = uint32_t(max(base + kChunk - kWindow, 0));
      // all of the above is done before the next loads are issued: a loaded
      // value that stayed live past them would be copied, and so waited for,
      // at the end of the step
      uint32_t id2 = nx2_id;
      asm volatile("" : "+v"(c_id), "+v"(c_lo), "+v"(c_hi), "+v"(c_key), "+v"(c_pos), "+v"(key_end), "+v"(id2));
      nx_id = id2;
      load_chunk(base + kChunk);
      nx2_id = load_id(base + 2 * kChunk);
    };
    float sh[3] = {0.0f, 0.0f, 0.0f};  // the current group's SH coefficients
    // Makes the loaded rows the current ones, and loads the group from lane g on.
    auto stage = [&](int g) {
      lds_order();
      s_row[lane] = nx_row;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) sh[ch] = nx_sh[ch];
      asm volatile("" : "+v"(sh[0]), "+v"(sh[1]), "+v"(sh[2]));
      load_rows(c_id, g);
      lds_order();
    };
    // A group of the chunk's candidates per step; the next chunk is taken
    // when the current one ends.
    int base = int(restart) - kChunk, g = 0;
    for (;;) {
      const uint64_t my_mask = uint64_t(c_hi) << 32 | c_lo;
      if ((__ballot((my_mask & work) != 0) >> g & 15u) != 0) {  // a candidate with a working pixel
        uint64_t m[kGroup];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) m[i] = readlane64(my_mask, g + i) & work;
        n_tests += uint32_t(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
        f32x4 cr = {0.5f, 0.5f, 0.5f, 0.5f}, cg = cr, cb = cr;
        sh_mfma(std::make_integer_sequence<int, K>{}, sh[0], sh[1], sh[2], Y, cr, cg, cb);
        if (!careful) {
          // straight-line code for the four candidates (a branch costs
          // about as much as ten of its instructions)
          uint32_t key[kGroup];
          double D2[kGroup];
          uint64_t h[kGroup];
          uint32_t more = cnt;
#pragma unroll
          for (int i = 0; i < kGroup; ++i) {
            const double* row = s_row + 16 * i;
            double W[9], og[3];
#pragma unroll
            for (int k = 0; k < 9; ++k) W[k] = row[k];
#pragma unroll
            for (int k = 0; k < 3; ++k) og[k] = row[9 + k];
            double tau, xg[3];
            const bool hit = ray_hit(W, og, row[12], d, &tau, &D2[i], xg);
            h[i] = __ballot(hit) & m[i];
            key[i] = __float_as_uint(float(tau)) & ~SM;
            more += lane_bit(h[i]) ? 1u : 0u;
          }
          if (__builtin_expect(__ballot(more > uint32_t(KB)) == 0, 1)) {
#pragma unroll
            for (int i = 0; i < kGroup; ++i) {
              const uint32_t slot = uint32_t(free_slots) & SM;
              uint4 pa;
              uint2 pb;
              payload(s_row[16 * i + 13] * exp_neg_half(D2[i], s_exp), cr[i], cg[i], cb[i],
                      __builtin_amdgcn_readlane(int(c_pos), g + i), &pa, &pb);
              lds_write_masked(h[i], &s_pa[slot * 64 + lane], pa, &s_pb[slot * 64 + lane], pb);
              sort_in(lane_bit(h[i]) ? key[i] | slot : kEmpty);
              free_slots = lane_bit(h[i]) ? free_slots >> 4 : free_slots;
            }
            cnt = more;
          } else {
            careful = true;
          }
        }
        if (careful) {
          // one candidate at a time
#pragma unroll 1
          for (int i = 0; i < kGroup; ++i, cr = rot(cr), cg = rot(cg), cb = rot(cb)) {
            const uint64_t mi = readlane64(my_mask, g + i) & work;
            const uint32_t cpos = __builtin_amdgcn_readlane(int(c_pos), g + i);
            const double* row = s_row + 16 * i;
            double W[9], og[3];
#pragma unroll
            for (int k = 0; k < 9; ++k) W[k] = row[k];
#pragma unroll
            for (int k = 0; k < 3; ++k) og[k] = row[9 + k];
            double tau, D2, xg[3];
            bool hit = ray_hit(W, og, row[12], d, &tau, &D2, xg) && lane_bit(mi);
            // in a rescan, hits up to the last composited one were composited before
            const uint32_t id = __builtin_amdgcn_readlane(int(c_id), g + i);
            hit = hit && cpos >= from && key_less(last_tau, last_id, tau, id);
            const uint32_t key = __float_as_uint(float(tau)) & ~SM;
            if (hit && key >= e_key) {
              bool drop = key > e_key;
              if (!drop) {
                if (e_tau != e_tau) {
                  e_id = prim[e_pos];
                  e_tau = exact_tau(e_id);
                }
                drop = !key_less(tau, id, e_tau, e_id);
              }
              if (drop) {
                ++n_drops;
                jr = min(jr, cpos);
                hit = false;
              }
            }
            if (hit && cnt == uint32_t(KB)) {  // a full pool: the largest of its hits and the new one is dropped
              const uint32_t top = max(a[KB - 1] & ~SM, key);
              bool drop_new = key == top;
              e_tau = drop_new ? tau : __builtin_nan("");
              e_id = id;
              if ((a[KB - 1] & ~SM) == top && (key == top || (a[KB - 2] & ~SM) == top)) {
                // among equal keys the exact depths decide, then the indices
                if (key != top) e_tau = -kInf;
                const uint32_t slot = tied_entry(std::false_type{}, top, e_tau, e_id);
                drop_new = slot == UINT_MAX;
                if (!drop_new) {  // to the end of the pool
                  bool past = false;
#pragma unroll
                  for (int s = 0; s + 1 < KB; ++s) {
                    past = past || (a[s] & SM) == slot;
                    a[s] = past ? a[s + 1] : a[s];
                  }
                  a[KB - 1] = top | slot;
                }
              }
              ++n_drops;
              e_key = top;
              e_pos = cpos;
              if (drop_new) {
                hit = false;
              } else {
                const uint32_t slot = a[KB - 1] & SM;
                e_pos = s_pb[slot * 64 + lane].y;
                free_slots = free_slots << 4 | slot;
                a[KB - 1] = kEmpty;
                --cnt;
              }
              jr = min(jr, e_pos);
            }
            if (hit) insert(key, row[13] * exp_neg_half(D2, s_exp), cr[0], cg[0], cb[0], cpos);
          }
        }
      }
      // everything after the group: the next candidate, or the next chunk
      const uint32_t nb = n_live == 0 ? 0u : bound_bits(g + kGroup < n_live ? __uint_as_float(__builtin_amdgcn_readlane(int(c_key), min(g + kGroup, 63))) : key_end);
      // The next group's rows are waited for here, between the tests and the
      // stores of the compositing (loads and stores complete in issue order).
      g += kGroup;
      if (g >= n_live) {
        do {
          base += kChunk;
          next_chunk(base);
        } while (n_live == 0 && base + kChunk < n);
        g = 0;
        load_rows(c_id, 0);
      }
      stage(g + kGroup);
      // Composite final hits only while some lane needs the room, so that
      // each step serves many lanes (at 1M Gaussians 60 steps a tile, each for
      // 41 of 64 lanes on average).
      load_head();
      for (;;) {
        const bool rdy = is_final(a[0], nb) && !lane_bit(term);
        if (__ballot(rdy && cnt > uint32_t(KB - kPoolSpare)) == 0) break;
        if (rdy) composite();
        term |= __ballot(T < A.t_min);
      }
      work &= ~(term | __ballot(e_key != UINT_MAX && nb > (e_key | SM) + 1u));
      if (n_live == 0 || work == 0) break;
    }
    // End of the pass (the list's end, or no working lane): every pooled hit
    // is below the smallest dropped one, and no unscanned Gaussian can
    // precede it.
    for (load_head(); __ballot(cnt != 0 && !lane_bit(term)) != 0; term |= __ballot(T < A.t_min)) {
      if (cnt != 0 && !lane_bit(term)) composite();
    }
    const bool need = e_key != UINT_MAX && !lane_bit(term);
    if (__ballot(need) == 0) break;
    if (passes >= kMaxPasses) {  // never expected: reported, not hidden
      if (lane == 0) atomicOr(A.status, unsigned(GART_FRAME_FORWARD_INCOMPLETE));
      break;
    }
    uint32_t rs = need ? jr : UINT_MAX;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rs = min(rs, uint32_t(__shfl_xor(int(rs), off)));
    restart = __builtin_amdgcn_readfirstlane(int(rs));
    if (need) {
      from = jr;
      last_tau = n_hits ? exact_tau(last_id) : -kInf;  // for the skip test of the rescan
    }
    ++passes;
    e_key = UINT_MAX;
    jr = UINT_MAX;
    term |= __ballot(T < A.t_min);
    work = __ballot(need) & ~term;
  }

  // the wave's visited prefix for the backward: its largest
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) visited = max(visited, uint32_t(__shfl_xor(int(visited), off)));
  if (lane == 0) A.tile_visit[tile * G + grp] = visited;
  double end_tau = kInf;
  uint32_t end_id = kNoPrim;
  if (valid && T < A.t_min) {  // terminated at its last hit
    end_id = last_id;
    end_tau = exact_tau(end_id);
  }
  if (__ballot(n_hits > hl_last + 1u) != 0 && lane == 0) atomicOr(A.status, unsigned(GART_FRAME_HIT_LIST_FULL));
  if (valid) {
    const int64_t p = int64_t(py) * A.cam.W + px;
    A.image[3 * p + 0] = float(L0);
    A.image[3 * p + 1] = float(L1);
    A.image[3 * p + 2] = float(L2);
    gart_pixel_state st;
    st.tau_end = end_tau;
    st.id_end = end_id;
    st.n_hits = n_hits;
    st.color_fixed[0] = color_fixed_fma(L0, A.inv_color_step);
    st.color_fixed[1] = color_fixed_fma(L1, A.inv_color_step);
    st.color_fixed[2] = color_fixed_fma(L2, A.inv_color_step);
    st.t_final = float(T);
    A.pixel_state[p] = st;
  }
  if (A.counters) {
    count_add(A.counters + GART_CNT_FWD_HITS, n_hits);
    count_add(A.counters + GART_CNT_FWD_TESTS, lane == 0 ? n_tests : 0u);
    count_add(A.counters + GART_CNT_FWD_DROPS, n_drops);
    if (lane == 0 && passes)
      atomicAdd(reinterpret_cast<unsigned long long*>(A.counters + GART_CNT_FWD_RESCANS), (unsigned long long)passes);
  }
}

// Pool sizes, by what a pool holds and what its LDS (1.5 KB an entry) costs in
// resident waves.  8x8 tiles: 11 entries (ms at 1M / 100k Gaussians: 8: 1.00 /
// 0.38, 9: 0.95 / 0.36, 10: 0.94 / 0.36, 11: 0.93 / 0.36, 12: 0.98 / 0.39; a
// pool that overflows costs a rescan, 1640 of them at 8 entries and 13 at 11).
// 16x16 tiles, whose list keys bound the depths more loosely: 12 (us with 10,
// 11, 12, 13, 14 entries at 250k Gaussians 979x546: 645, 576, 573, 559, 616; at
// 100k 640x480: 418, 415, 410, 398, 420; at 1M 1237x822: 1185, 1134, 1160, 1136,
// 1266).  Deep frames (long tile lists, many pending hits per ray): 15 (150k
// large Gaussians, 8x8 tiles, ms: 13: 6.93, 14: 6.16, 15: 5.59; one more entry
// leaves five waves per CU instead of six).  Where a frame becomes deep was
// measured on 8x8 tiles; large Gaussians on 16x16 tiles gain from 15 entries
// below it too (1024x680, ms with 12 and 15: 30k 3.93 and 3.84, 60k 8.6 and 5.5).
constexpr int64_t kDeepListPairs = 2048;  // mean pairs per tile from which a frame counts as deep

template <int TILE, int K, int KB>
hipError_t launch_pool(const ForwardArgs& a, hipStream_t s) {
  const int n_tiles = a.tiles_x * a.tiles_y;
  constexpr int G = TILE * TILE / 64;
  const int grid = G == 1 ? n_tiles : (n_tiles + 7) / 8 * 8 * G;
  switch (a.lt_format) {
    case GART_LT_FULL: forward_kernel<TILE, K, GART_LT_FULL, KB><<<grid, 64, 0, s>>>(a); break;
    case GART_LT_T_ONLY: forward_kernel<TILE, K, GART_LT_T_ONLY, KB><<<grid, 64, 0, s>>>(a); break;
    case GART_LT_HALF: forward_kernel<TILE, K, GART_LT_HALF, KB><<<grid, 64, 0, s>>>(a); break;
    case GART_LT_T_HALF: forward_kernel<TILE, K, GART_LT_T_HALF, KB><<<grid, 64, 0, s>>>(a); break;
    case GART_LT_FIXED16: forward_kernel<TILE, K, GART_LT_FIXED16, KB><<<grid, 64, 0, s>>>(a); break;
    case GART_LT_T_LOG16: forward_kernel<TILE, K, GART_LT_T_LOG16, KB><<<grid, 64, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TILE, int K>
hipError_t launch_t(const ForwardArgs& a, hipStream_t s) {
  hipError_t e = record(a.ev_begin, s);
  if (e != hipSuccess) return e;
  const int64_t n_tiles = int64_t(a.tiles_x) * a.tiles_y;
  const bool deep = a.pair_count > kDeepListPairs * n_tiles;
  e = deep ? launch_pool<TILE, K, 15>(a, s) : launch_pool<TILE, K, TILE == 8 ? 11 : 12>(a, s);
  if (e != hipSuccess) return e;
  return record(a.ev_end, s);
}

template <int TILE>
hipError_t launch_k(const ForwardArgs& a, hipStream_t s) {
  switch (a.sh_k) {
    case 1: return launch_t<TILE, 1>(a, s);
    case 4: return launch_t<TILE, 4>(a, s);
    case 9: return launch_t<TILE, 9>(a, s);
    case 16: return launch_t<TILE, 16>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_forward(const ForwardArgs& a, hipStream_t s) {
  if (a.tiles_x * a.tiles_y <= 0) return hipSuccess;
  return a.tile == 16 ? launch_k<16>(a, s) : launch_k<8>(a, s);
}

}  // namespace gart
