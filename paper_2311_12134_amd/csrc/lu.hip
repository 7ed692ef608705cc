// Batched complex LU with partial pivoting (the tau inverse of Eq. (3) is the dominant
// cost of the method, Sec. II.A), blocked with panel width NB: right-looking over groups of
// 2 to 4 panels, left-looking within a group (see lu_factor_any).
//
// All jobs of a wave advance through the same panel steps; every panel is a few
// launches over the whole batch:
//   panel_kernel      one workgroup per job factors rows [k, n) x cols [k, k+NB) with
//                     partial pivoting (pivot = largest |re|+|im|, first on ties, keys
//                     compared in FP64): IB-wide leaves live in registers (rows distributed
//                     cyclically over the workgroup) and are updated in the storage
//                     precision, a leaf's interchanges then move whole panel rows, and the rest
//                     of the panel is updated by the leaf (triangular solve + rank-IB).
//   swap_trsm_kernel  applies the panel's row interchanges to the trailing columns and
//                     forms U12 = L11^-1 A12 (one workgroup per 64-column tile).
//   gemm_*_kernel     (gemm.hip) trailing update A22 -= L21 U12 on the matrix cores:
//                     FP64 MFMA 16x16x4 with the four real products of a complex product,
//                     or (split mode) FP32 MFMA 16x16x4 with three real products
//                     (Ar Br, Ai Bi, (Ar+Ai)(Br+Bi)).
// Interchanges are applied only to the right of each panel (and to the L columns of the
// earlier panels of its group); the solves apply them panel by panel in the same order,
// so the columns of earlier groups never need swapping.
// Matrices are row-major with leading dimension npad (a multiple of 64); the padding
// is an identity block that no pivot ever selects.
#include <algorithm>
#include <type_traits>

#include "lsms_internal.h"
#include "strip_mma.h"

namespace lsms {

typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------
// panel factorization
// ------------------------------------------------------------------------------------
// Pivot keys: a non-negative double orders like its bit pattern, so the magnitude with
// its 13 lowest mantissa bits replaced by (8191 - position) is one 64-bit integer whose
// maximum is the largest magnitude, the lowest position on ties (relative resolution 2^-39).
// NaN magnitudes get key 0 and never win; key 0 overall means "keep the diagonal row".
struct PivotKey {
  unsigned hi, lo;
};
__device__ inline PivotKey pivot_key(double mag, int pos) {
  if (!(mag == mag)) return PivotKey{0u, 0u};
  const unsigned long long b = (unsigned long long)__double_as_longlong(mag);
  return PivotKey{(unsigned)(b >> 32), ((unsigned)b & ~0x1FFFu) | (unsigned)(0x1FFF - pos)};
}
__device__ inline bool key_less(PivotKey a, PivotKey b) { return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo); }
__device__ inline int pivot_pos(unsigned lo) { return 0x1FFF - (int)(lo & 0x1FFFu); }

// One lane's value moved within its 16-lane row by the DPP pattern CTRL.
template <int CTRL>
__device__ inline unsigned dpp_u32(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ inline unsigned lane_u32(unsigned x, int l) { return (unsigned)__builtin_amdgcn_readlane((int)x, l); }
// Largest value of lanes 0 .. N - 1 (N <= 16: the other lanes of the row hold 0; 64: the wavefront), a
// scalar: the maximum within each 16-lane row by DPP (quad exchanges 1 and 2, half-row mirror, row
// mirror; each step combines groups that already agree), then the four rows' maxima.
template <int N>
__device__ inline unsigned lanes_max(unsigned x) {
  x = max(x, dpp_u32<0xB1>(x));              // quad_perm [1, 0, 3, 2]
  if (N > 2) x = max(x, dpp_u32<0x4E>(x));   // quad_perm [2, 3, 0, 1]
  if (N > 4) x = max(x, dpp_u32<0x141>(x));  // row_half_mirror
  if (N > 8) x = max(x, dpp_u32<0x140>(x));  // row_mirror
  if (N <= 16) return lane_u32(x, 0);
  return max(max(lane_u32(x, 0), lane_u32(x, 16)), max(lane_u32(x, 32), lane_u32(x, 48)));
}
// The lane (of lanes 0 .. N - 1) with the largest key, the same in every lane; hi is the largest high
// word, and the low words count only where it ties.
template <int N>
__device__ inline int best_lane(PivotKey key, unsigned hi) {
  unsigned long long m = __ballot(key.hi == hi);
  if (m & (m - 1)) {  // uniform
    const unsigned lo = lanes_max<N>(key.hi == hi ? key.lo : 0u);
    m = __ballot(key.hi == hi && key.lo == lo);
  }
  return __ffsll((long long)m) - 1;
}

__device__ inline float2 lane_value(float2 x, int l) {
  return make_float2(__uint_as_float(lane_u32(__float_as_uint(x.x), l)), __uint_as_float(lane_u32(__float_as_uint(x.y), l)));
}
__device__ inline double2 lane_value(double2 x, int l) {
  return make_double2(__hiloint2double(lane_u32(__double2hiint(x.x), l), lane_u32(__double2loint(x.x), l)),
                      __hiloint2double(lane_u32(__double2hiint(x.y), l), lane_u32(__double2loint(x.y), l)));
}

// Inverse of a pivot in FP64, conj(a) / |a|^2.  Values stored in FP32 have squared magnitudes well
// inside the FP64 range; FP64 values are first scaled by a power of two that brings the larger
// component to [1/2, 1).  1 / |a|^2 by Newton steps on the hardware's reciprocal (24 bits or more), a
// third of the chain of a division: two of them for values stored in FP32, which end at FP64's own
// rounding.
__device__ inline double recip_step(double n, double r) { return __builtin_fma(__builtin_fma(-n, r, 1.0), r, r); }
__device__ inline double2 pivot_inverse(double2 a, float2) {
  const double n = __builtin_fma(a.x, a.x, a.y * a.y);
  const double rn = recip_step(n, recip_step(n, __builtin_amdgcn_rcp(n)));
  return make_double2(a.x * rn, -a.y * rn);
}
// FP64 values: one step on 1 / |a|^2, then one on the complex inverse, z (2 - a z), so that the inverse of a real or an
// imaginary pivot is the rounded quotient: rows that are exact multiples of the pivot row then cancel
// exactly where they do with a division, and a singular matrix of such rows is reported as one.
__device__ inline double2 pivot_inverse(double2 a, double2) {
  const double m = fmax(fabs(a.x), fabs(a.y));
  const int e = -__builtin_amdgcn_frexp_exp(m);
  const double x = __builtin_amdgcn_ldexp(a.x, e), y = __builtin_amdgcn_ldexp(a.y, e);
  const double n = __builtin_fma(x, x, y * y);
  const double rn = recip_step(n, __builtin_amdgcn_rcp(n));
  const double u = x * rn, v = -y * rn;
  const double er = __builtin_fma(y, v, __builtin_fma(-x, u, 1.0)), ei = __builtin_fma(-x, v, -y * u);
  const double zr = __builtin_fma(u, er, __builtin_fma(-v, ei, u)), zi = __builtin_fma(u, ei, __builtin_fma(v, er, v));
  // one infinite component: 0, as a division gives (the Newton steps would make it NaN)
  const double z = 0.0 * fmin(fabs(a.x), fabs(a.y));
  const bool inf = m == INFINITY;
  return make_double2(inf ? z : __builtin_amdgcn_ldexp(zr, e), inf ? -z : __builtin_amdgcn_ldexp(zi, e));
}

// a - b c for the leaf's rank-1 updates: each component as two fused multiply-adds (two
// roundings, where the product-then-difference form takes three operations and three roundings)
__device__ inline float2 leaf_fms(float2 a, float2 b, float2 c) {
  return make_float2(__builtin_fmaf(-b.x, c.x, __builtin_fmaf(b.y, c.y, a.x)),
                     __builtin_fmaf(-b.x, c.y, __builtin_fmaf(-b.y, c.x, a.y)));
}
__device__ inline double2 leaf_fms(double2 a, double2 b, double2 c) {
  return make_double2(__builtin_fma(-b.x, c.x, __builtin_fma(b.y, c.y, a.x)),
                      __builtin_fma(-b.x, c.y, __builtin_fma(-b.y, c.x, a.y)));
}

__device__ inline double2 wide(double2 a) { return a; }
__device__ inline double2 wide(float2 a) { return make_double2((double)a.x, (double)a.y); }
__device__ inline void narrow_to(double2& d, double2 a) { d = a; }
__device__ inline void narrow_to(float2& d, double2 a) { d = make_float2((float)a.x, (float)a.y); }

// c ? a : b by components (a choice between two array elements as a whole would be a choice of their
// addresses, and put the arrays in memory)
__device__ inline float2 sel(bool c, float2 a, float2 b) { return make_float2(c ? a.x : b.x, c ? a.y : b.y); }
__device__ inline double2 sel(bool c, double2 a, double2 b) { return make_double2(c ? a.x : b.x, c ? a.y : b.y); }
// a 16-byte piece of a staged row, to and from LDS (FP32 rows are only 8-byte aligned there)
__device__ inline void chunk_put(float2* d, float4 x) {
  d[0] = make_float2(x.x, x.y);
  d[1] = make_float2(x.z, x.w);
}
__device__ inline void chunk_put(double2* d, float4 x) { *(float4*)d = x; }
__device__ inline float4 chunk_get(const float2* d) {
  const float2 a = d[0], b = d[1];
  return make_float4(a.x, a.y, b.x, b.y);
}
__device__ inline float4 chunk_get(const double2* d) { return *(const float4*)d; }
// Orders LDS traffic between the lanes of one wavefront (its LDS operations run in order).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline double2 shfl2(double2 v, int src) { return make_double2(__shfl(v.x, src), __shfl(v.y, src)); }

// nopiv: keep the diagonal row at every step (the symmetric factorization below); the
// permutation list is then the identity.
//
// One workgroup per job; thread t holds rows t, t + PT, .. of the panel (S of them), one leaf of IB
// columns at a time, in registers.  Rows stay with their threads while a leaf is factored: an
// interchange only exchanges two numbers, the positions pos[] of the rows, and the leaf is stored at
// its rows' positions at the end, from which the list of the rows that moved follows in parallel.
// A pivot column has two barriers: before the first every wavefront posts its best key and that
// pivot's inverse (formed by every lane for its own best row while the keys are reduced, so it is
// off the chain); then the winner alone posts its row (a row posted by every wavefront, one lane's
// 16-byte stores at a time, fills the LDS pipe: 150 000 cycles for the 64 columns of 256 FP32
// rows, 137 000 this way), and every wavefront reads it once, entry q in lane q.
// Bound by that chain, about 2200 cycles a column, by the update's arithmetic from three row
// slots on, and for tall panels by the rank-IB updates' traffic (320 FP64 systems, three and four row slots: 4.2 and
// 4.3 TB/s, nearly five times the panels' own bytes, where a copy reaches 5.0).  Leaves are as wide as the
// registers allow, since every leaf pays once for loading, storing, interchanging the other columns
// and the rank update.  One panel, on 2 and on 320 systems (us; before: rows exchanged in
// registers, the moved rows listed by one thread, leaves of 8 and 16): FP64 256 rows 112 / 180
// (173 / 356), 320 rows 153 / 333 (195 / 402), 768 rows 195 / 499 (283 / 690), 2048 rows 430 / 1437
// (515 / 1633); FP32 256 rows 88 (147), 512 rows 118 / 176 (199 / 282), 1024 rows 160 / 380 (211 / 469),
// 2048 rows 250 / 635 (283 / 689), 2176 rows 320 / 936 (354 / 929).
template <typename T, int PT, int S, int IB>
__global__ __launch_bounds__(PT, 2) void panel_kernel(const JobDesc* jobs, int k, int left, T* work, int32_t* piv,
                                                   int32_t* info, int nopiv) {
  const JobDesc jd = jobs[blockIdx.x];
  if (k >= jd.npad) return;  // uniform over the workgroup
  const int ld = jd.ld > 0 ? jd.ld : jd.npad;
  // row r, column c of the matrix, r from the panel's first row: 32-bit byte offsets (a panel of at most
  // 4096 rows of at most 16384 columns spans 1 GiB).  Each section takes the leading dimension
  // through here(), which keeps its addresses from being formed ahead and held across the leaves.
  char* const A = (char*)(work + jd.a_off + (int64_t)k * ld);
  auto at = [A](int r, int c, int ldx) -> T* { return (T*)(A + (unsigned)(r * ldx + c) * (unsigned)sizeof(T)); };
  auto here = [ld]() {
    int x = ld;
    asm volatile("" : "+s"(x));
    return x;
  };
  const int nrows = jd.npad - k;             // rows, positions and pivots below are relative to k
  int32_t* ip = piv + jd.piv_off;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  constexpr int NW = PT / 64;
  constexpr int SEG = IB * (int)sizeof(T) < 128 ? IB : 128 / (int)sizeof(T);  // columns moved per staged access
  constexpr int CPR = SEG * (int)sizeof(T) / 16, RPI = 64 / CPR;  // 16-byte chunks per row, rows per access
  constexpr int PER = 16 / (int)sizeof(T);                        // elements per chunk
  constexpr int BB = IB >= 32 ? 8 : 4;                            // columns per block of the leaf
  static_assert(IB < NB && IB / BB <= 4 && BB % 2 == 0, "the blocks below; buffers alternate across blocks");
  // the leaf's register that holds column j once it is factored
  auto reg_of = [](int j) { return IB - (j / BB + 1) * BB + j % BB; };

  __shared__ PivotKey s_key[NW];
  __shared__ T s_inv[NW];
  __shared__ __align__(16) T s_prow[IB];
  __shared__ int s_pivall[NB];
  __shared__ T s_L11[IB][IB + 1];
  __shared__ T s_U[IB][NB - IB];
  __shared__ unsigned short s_org[S * PT];  // original row at each position, over all leaves
  __shared__ int s_lpos[2 * IB], s_lorg[2 * IB], s_lcnt;
  __shared__ int s_row[PT];
  // The next leaf stays on chip for 16-wide FP32 leaves of three or four row slots (the other
  // shapes run out of registers or occupancy with it).
  constexpr bool KEEP_NEXT = sizeof(T) == sizeof(float2) && IB == 16 && S * IB * 2 <= 128;
  // A row of the leaf is moved in pieces of 128 bytes through the wave's own rows of s_X: a
  // wavefront's 16-byte access then covers eight whole pieces instead of one chunk of 64 different
  // rows, which costs one L2 request per lane.  The same rows carry the next leaf out of the
  // rank update.
  __shared__ __align__(16) T s_X[PT][SEG + 1];  // one row per thread (wave-private rows)

  T v[S][IB];
  int pos[S];
  int first_zero = 0;
  for (int i = t; i < S * PT; i += PT) s_org[i] = (unsigned short)i;

  const int ch = lane % CPR, rsub = lane / CPR;
  for (int c = 0; c < NB / IB; ++c) {
    const int cl = c * IB;       // the leaf's first row and column
    const int w = NB - cl - IB;  // panel columns right of the leaf
    if (t == 0) s_lcnt = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) pos[s] = t + s * PT < nrows ? t + s * PT : -1;
    int ldx = here();
    if (c == 0 || !KEEP_NEXT) {  // otherwise the leaf came from the previous leaf's rank update
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int rw = s * PT + wave * 64;  // the wave's first row in this slot
        if (rw >= nrows) {                  // uniform per wave
#pragma unroll
          for (int q = 0; q < IB; ++q) v[s][q] = T{0, 0};
          continue;
        }
        float4 x[IB / SEG][CPR];
#pragma unroll
        for (int g = 0; g < IB / SEG; ++g)
#pragma unroll
          for (int u = 0; u < CPR; ++u) {
            const int r = rw + u * RPI + rsub;
            x[g][u] = (r >= cl && r < nrows) ? *(const float4*)at(r, k + cl + g * SEG + PER * ch, ldx)
                                             : make_float4(0.f, 0.f, 0.f, 0.f);
          }
#pragma unroll
        for (int g = 0; g < IB / SEG; ++g) {
#pragma unroll
          for (int u = 0; u < CPR; ++u) chunk_put(s_X[wave * 64 + u * RPI + rsub] + PER * ch, x[g][u]);
          wave_sync();
#pragma unroll
          for (int q = 0; q < SEG; ++q) v[s][g * SEG + q] = s_X[t][q];
          wave_sync();  // every lane has its row before the next piece rewrites them
        }
      }
    }
    // The columns in blocks of BB.  A block's columns run through one rolled loop: registers
    // 0 .. W - 1 hold the W columns from the block on, the current one in register 0; each step
    // shifts them down by one as it updates them and puts the finished column last.  The pivot row
    // takes zeros in the places of the block's finished columns, which keeps those as they are.
    // After the leaf, register reg_of(j) holds column j.
    // A column's search (its keys, the wave's best, the pivot's inverse) starts when the step before
    // has updated that column, and runs beside the rest of that step's update.
    PivotKey key;
    T inv;
    unsigned whi;
    auto search = [&](int d) {
      key = PivotKey{0u, 0u};
      T e = v[0][0];  // the lane's best row's entry
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const double2 x = wide(v[s][0]);
        PivotKey kk = pivot_key(nopiv ? 1.0 : fabs(x.x) + fabs(x.y), pos[s]);
        const bool in = nopiv ? pos[s] == d : pos[s] >= d;
        kk.hi = in ? kk.hi : 0u;
        kk.lo = in ? kk.lo : 0u;
        const bool more = s == 0 || key_less(key, kk);
        key.hi = more ? kk.hi : key.hi;
        key.lo = more ? kk.lo : key.lo;
        if (s > 0) e = sel(more, v[s][0], e);
      }
      const double2 x = wide(e);
      // the pivot's inverse in FP64, rounded once to the storage precision
      narrow_to(inv, sel(x.x == 0.0 && x.y == 0.0, make_double2(0.0, 0.0), pivot_inverse(x, T{})));
      whi = lanes_max<64>(key.hi);
    };
    search(cl);
    auto block = [&](auto jb_tag) {
      constexpr int JB = decltype(jb_tag)::value, W = IB - JB * BB;
#pragma clang loop unroll(disable)
      for (int jj = 0; jj < BB; ++jj) {
        const int d = cl + JB * BB + jj;
        const int post = best_lane<64>(key, whi);
        if (lane == post) {  // (a wave without eligible rows posts key 0)
          s_inv[wave] = inv;
          s_key[wave] = key;
        }
        lds_barrier();
        PivotKey kw{0u, 0u};
        T iw{};
        if (lane < NW) {
          kw = s_key[lane];
          iw = s_inv[lane];
        }
        const int from = best_lane<NW>(kw, lanes_max<NW>(kw.hi));
        const unsigned bhi = lane_u32(kw.hi, from), blo = lane_u32(kw.lo, from);
        T il = lane_value(iw, from);
        int p = pivot_pos(blo);
        if ((bhi | blo) == 0u) {  // no row has a comparable magnitude (all NaN): the diagonal row (uniform)
          p = d;
          il = T{(decltype(il.x))NAN, (decltype(il.x))NAN};
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (pos[s] == p) {
#pragma unroll
            for (int q = 0; q < W; ++q) s_prow[q] = v[s][q];
          }
        if (t == 0) s_pivall[d] = p;
        lds_barrier();
        // the pivot row, entry q in lane q
        const T row = sel(lane + jj < W, s_prow[min(lane, W - 1)], T{0, 0});
        if (nopiv || (bhi == 0u && blo < 0x2000u)) {  // perhaps an exact zero (uniform; without pivoting the key says nothing)
          const T pv = lane_value(row, 0);
          if (pv.x == 0 && pv.y == 0 && first_zero == 0) first_zero = k + d + 1;
        }
        // the interchange, and the leaf's rank-1 update in the storage precision (FP32 in split mode,
        // like the trailing updates; the pivot keys above compare these values in FP64).  Rows on
        // or above the pivot take a zero multiplier, which leaves them as they are.
        T l[S], last[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          pos[s] = pos[s] == p ? d : pos[s] == d ? p : pos[s];
          const bool below = pos[s] > d;
          const T m = cmul(v[s][0], il);
          l[s] = sel(below, m, T{0, 0});
          last[s] = sel(below, m, v[s][0]);
        }
        auto update = [&](int q) {
          const T u = lane_value(row, q);
#pragma unroll
          for (int s = 0; s < S; ++s) v[s][q - 1] = leaf_fms(v[s][q], l[s], u);
        };
        if (W > 1)
          update(1);
        else
#pragma unroll
          for (int s = 0; s < S; ++s) v[s][0] = last[s];
        search(d + 1);
#pragma unroll
        for (int q = 2; q < W; ++q) update(q);
#pragma unroll
        for (int s = 0; s < S; ++s) v[s][W - 1] = last[s];
      }
    };
    block(std::integral_constant<int, 0>{});
    if constexpr (IB / BB > 1) block(std::integral_constant<int, 1>{});
    if constexpr (IB / BB > 2) block(std::integral_constant<int, 2>{});
    if constexpr (IB / BB > 3) block(std::integral_constant<int, 3>{});
    // the rows that moved, the leaf's diagonal block to LDS, and the leaf back to memory (the
    // registers of a row slot are free once it is staged)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int home = t + s * PT;
      if (pos[s] >= 0 && pos[s] != home) {
        const int i = atomicAdd(&s_lcnt, 1);
        s_lpos[i] = pos[s];
        s_lorg[i] = home;
      }
      if (pos[s] >= cl && pos[s] < cl + IB) {
#pragma unroll
        for (int q = 0; q < IB; ++q) s_L11[pos[s] - cl][q] = v[s][reg_of(q)];
      }
    }
    ldx = here();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int rw = s * PT + wave * 64;
      if (rw >= nrows) continue;  // uniform per wave
      s_row[t] = pos[s];
#pragma unroll
      for (int g = 0; g < IB / SEG; ++g) {
#pragma unroll
        for (int q = 0; q < SEG; ++q) s_X[t][q] = v[s][reg_of(g * SEG + q)];
        wave_sync();
#pragma unroll
        for (int u = 0; u < CPR; ++u) {
          const int i = wave * 64 + u * RPI + rsub, r = s_row[i];
          const float4 x = chunk_get(s_X[i] + PER * ch);
          if (r >= cl) *(float4*)at(r, k + cl + g * SEG + PER * ch, ldx) = x;
        }
        wave_sync();  // read before the next piece rewrites the rows
      }
    }
    __syncthreads();
    const int cnt = s_lcnt;
    // the leaf's interchanges on the other columns of the panel (whole panel rows), and on
    // the `left` columns before it (the earlier panels of its group, see lu_factor_any): the at
    // most 2 IB rows that moved, 64 columns at a time, a column per lane
    {
      constexpr int HELD = (2 * IB + NW - 1) / NW;
      ldx = here();
      const int ncols = left + NB - IB;
      unsigned short org = 0;
      if (t < cnt) org = s_org[s_lorg[t]];
      for (int c0 = 0; c0 < ncols; c0 += 64) {
        const int cc = c0 + lane, cr = cc - left;
        const int colx = cc < left ? k - left + cc : k + (cr < cl ? cr : cr + IB);
        T held[HELD];
#pragma unroll
        for (int u = 0; u < HELD; ++u) {
          const int i = wave + NW * u;
          T x{0, 0};
          if (i < cnt && cc < ncols) x = *at(s_lorg[i], colx, ldx);
          held[u] = x;
        }
        __syncthreads();  // every source row is read before any destination row is written
#pragma unroll
        for (int u = 0; u < HELD; ++u) {
          const int i = wave + NW * u;
          if (i < cnt && cc < ncols) *at(s_lpos[i], colx, ldx) = held[u];
        }
      }
      if (t < cnt) s_org[s_lpos[t]] = org;
    }
    __syncthreads();
    if (w > 0) {
      // U rows of the leaf, U = L11^-1 A[leaf rows, right of the leaf], by forward substitution in FP64:
      // eight columns per wavefront, lane = column + 8 g holding rows g, g + 8, ..; every
      // finished row goes to the other lanes of its column by a shuffle
      ldx = here();
      for (int cb = wave * 8; cb < w; cb += NW * 8) {
        constexpr int RPL = (IB + 7) / 8;
        const int cc = cb + (lane & 7), g = lane >> 3;
        const bool in = cc < w && g < IB;  // (always, but for leaves of four columns)
        auto up = [&](int q) { return at(cl + g + 8 * q, k + cl + IB + cc, ldx); };
        double2 u[RPL];
#pragma unroll
        for (int q = 0; q < RPL; ++q) u[q] = in ? wide(*up(q)) : make_double2(0.0, 0.0);
#pragma unroll
        for (int r = 0; r < IB - 1; ++r) {
          const double2 ur = shfl2(u[r / 8], (lane & 7) + 8 * (r & 7));
#pragma unroll
          for (int q = r / 8; q < RPL; ++q) {
            if ((q > r / 8 || g > (r & 7)) && g < IB) u[q] = leaf_fms(u[q], wide(s_L11[g + 8 * q][r]), ur);
          }
        }
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
          T x;
          narrow_to(x, u[q]);
          if (in) {
            *up(q) = x;
            s_U[g + 8 * q][cc] = x;
          }
        }
      }
      __syncthreads();
      // rank-IB update of the panel right of the leaf on the matrix cores: each wave updates
      // its own 64 rows of every PT-row slab, RBP 16-row blocks at a time.  The leaf's L rows
      // are read back from memory (stored before the barrier above), and all old values and
      // L operands of a group are loaded before its first product, so a group waits for
      // memory once instead of once per 16 x 16 tile.  The first IB columns right of the leaf
      // are the next leaf: where it stays on chip their results go through the wave's own rows of
      // s_X straight into the leaf registers (the slab's old leaf values are dead by then), so
      // the next leaf is neither stored here nor loaded again; the other columns are written
      // back.  Rows above the leaf's last row and columns past w are masked at the load and store.
      constexpr int CBM = (NB - IB + 15) / 16;  // 16-column blocks, at most
      constexpr int VRB = CBM * (int)sizeof(T) + IB / 4 * (int)sizeof(T) / 4;  // registers per block
      // with the next leaf kept on chip its registers stay live through the update, so the
      // groups are two blocks (one with four row slots)
      constexpr int RBP = KEEP_NEXT ? (S >= 4 ? 1 : 2) : (VRB * 4 <= 160 ? 4 : (VRB * 2 <= 160 ? 2 : 1));
      // the kept leaves take their L operand from LDS, which shortens their rank updates
      constexpr bool LOP_LDS = KEEP_NEXT;
      typedef StripMma<T, 1, IB> Mma;
      const int ii = lane & 15, kq = lane >> 4;
#pragma unroll 1
      for (int s = 0; s < S; ++s) {
        const int r0 = s * PT;
        ldx = here();
        if constexpr (LOP_LDS) {
          // the slab's leaf rows, the L operand of its products, into the wave's rows of s_X (rows
          // past the matrix hold zeros), and those that moved here from memory, where the leaf is
          // stored; a group's rows take the next leaf only after the group's own products have
          // read them
          wave_sync();
#pragma unroll
          for (int ss = 0; ss < S; ++ss)
            if (ss == s) {
#pragma unroll
              for (int q = 0; q < IB; ++q) s_X[t][q] = v[ss][reg_of(q)];
            }
          wave_sync();
          const int rw = r0 + wave * 64;
          if (lane < cnt && s_lpos[lane] >= rw && s_lpos[lane] < rw + 64) {  // cnt <= 2 IB = 32
            const int r = s_lpos[lane];
#pragma unroll
            for (int u = 0; u < CPR; ++u)
              chunk_put(s_X[wave * 64 + r - rw] + PER * u, *(const float4*)at(r, k + cl + PER * u, ldx));
          }
          wave_sync();
        }
#pragma unroll 1
        for (int g = 0; g < 4; g += RBP) {
          const int gbase = r0 + wave * 64 + g * 16;
          if (gbase >= nrows || gbase + RBP * 16 <= cl + IB) continue;  // uniform per wave
          T lop[RBP][IB / 4];
          T old[RBP][CBM][4];
#pragma unroll
          for (int b = 0; b < RBP; ++b) {
            const int rl = gbase + b * 16 + ii;
            if constexpr (LOP_LDS) {
#pragma unroll
              for (int q = 0; q < IB / 4; ++q) lop[b][q] = s_X[wave * 64 + (g + b) * 16 + ii][4 * q + kq];
            } else {
#pragma unroll
              for (int q = 0; q < IB / 4; ++q) lop[b][q] = rl < nrows ? *at(rl, k + cl + 4 * q + kq, ldx) : T{0, 0};
            }
#pragma unroll
            for (int cb = 0; cb < CBM; ++cb)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int row = gbase + b * 16 + Mma::row(r, lane), cc = cb * 16 + ii;
                old[b][cb][r] =
                    (row >= cl + IB && row < nrows && cc < w) ? *at(row, k + cl + IB + cc, ldx) : T{0, 0};
              }
          }
#pragma unroll
          for (int b = 0; b < RBP; ++b) {
            const int rbase = gbase + b * 16;
            if (rbase + 16 <= cl + IB || rbase >= nrows) continue;  // uniform per wave
#pragma unroll
            for (int cb = 0; cb < CBM; ++cb) {
              if (cb * 16 >= w) continue;  // uniform
              Mma acc;
              acc.zero();
              acc.run_regs(lop[b], [&](int kk, int cc) { return s_U[kk][min(cb * 16 + cc, NB - IB - 1)]; }, lane);
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int row = rbase + Mma::row(r, lane), cc = cb * 16 + ii;
                if (row >= cl + IB && row < nrows && cc < w) {
                  T nv;
                  narrow_to(nv, csub(wide(old[b][cb][r]), acc.value(0, r)));
                  if (KEEP_NEXT && cc < IB)
                    s_X[row - r0][cc] = nv;
                  else
                    *at(row, k + cl + IB + cc, ldx) = nv;
                }
              }
            }
          }
        }
        if constexpr (KEEP_NEXT) {
          wave_sync();
          // the next leaf's rows of this slab (rows above it or past the matrix are zero);
          // register slots are indexed by constants only
          const int r = r0 + t;
          const bool in = r >= cl + IB && r < nrows;
#pragma unroll
          for (int ss = 0; ss < S; ++ss)
            if (ss == s) {
#pragma unroll
              for (int q = 0; q < IB; ++q) v[ss][q] = sel(in, s_X[t][q], T{0, 0});
            }
          wave_sync();  // every lane has its row before the next slab writes s_X
        }
      }
    }
    // the next leaf reads columns written above by other threads, and s_U / s_L11 / s_lcnt
    // are rewritten by it
    __syncthreads();
  }
  // The panel's NB interchanges as one permutation of at most 2 NB rows: entries 0 .. NB - 1 are the
  // positions k .. k + NB - 1, the others the rows below that moved (in no particular order).
  int32_t* lst = ip + perm_off(jd.npad, k);
  __shared__ int s_cnt;
  if (t == 0) s_cnt = NB;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int at = t + s * PT;
    if (at >= nrows) continue;
    const int org = s_org[at];
    int i = at;
    if (at >= NB) {
      if (at == org) continue;
      i = atomicAdd(&s_cnt, 1);
    }
    lst[2 + i] = k + at;
    lst[2 + PERM_MAX + i] = k + org;
  }
  for (int q = t; q < NB; q += PT) ip[k + q] = k + s_pivall[q];
  __syncthreads();
  if (t == 0) {
    lst[0] = s_cnt;
    if (first_zero != 0 && info[blockIdx.x] == 0) info[blockIdx.x] = first_zero;
  }
}

// ------------------------------------------------------------------------------------
// inverses of the panel's diagonal triangles, in place
// ------------------------------------------------------------------------------------
// After panel(k) the diagonal block holds L11 (strictly lower, unit diagonal implied) and
// U11 (upper with diagonal).  One workgroup per job overwrites the block with X = L11^-1 below
// the diagonal and Y = U11^-1 on and above it.  Every later use of the block wants an inverse:
// U12 = L11^-1 A12 in swap_trsm_kernel and the four diagonal steps of the solves, which
// thereby become products on the matrix cores.  No later interchange touches the block (pivots
// of later panels lie below it), and nothing else reads U11.
//
// Blocked in 16 x 16 blocks: one wavefront per diagonal block forms X_ii = L_ii^-1 or
// Y_ii = U_ii^-1 (16-step FP64 substitutions, the sixteen pivots inverted beforehand side by side),
// then the off-diagonal blocks follow from FP64 matrix-core products, for two halves within each
// 32 x 32 triangle and then for the 32 x 32 block between them:
//   X_ij = -X_ii (L_ij X_jj),  (i, j) = (1, 0), (3, 2);
//   W_ij = sum_m L_im X_mj,  X_ij = -sum_m X_im W_mj,  i = 2, 3, j = 0, 1;
// the upper triangle is the same with its blocks counted from the end.  Waves 0 - 3 take the lower
// triangle, 4 - 7 the upper one in opposite order, so that a SIMD's two wavefronts have three
// products together where one has one and the other two.  A first product is the operand of the second
// without leaving its registers (accumulators and right operands have one layout).  Results
// are kept in FP64 and rounded once to the storage precision at the store.
// A chain of about 50 dependent steps bounds it.  FP64 storage on one system: 12 us, against 18 with
// divisions in the substitution and one diagonal of blocks after the other (8 products deep on the
// busiest SIMD's two wavefronts), and 83 for two 64-step substitutions.
template <typename T>
__global__ __launch_bounds__(512) void linv_kernel(const JobDesc* jobs, int k, T* work) {
  constexpr int B = 16;
  const JobDesc jd = jobs[blockIdx.x];
  if (k >= jd.npad) return;  // uniform
  T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  __shared__ T s_T[NB][NB + 1];        // L11 \ U11 as factored
  __shared__ double2 s_V[NB][NB + 1];  // X = L11^-1 below the diagonal, Y = U11^-1 on and above
  __shared__ double2 s_W[2][2][B][B + 1];  // W_2j of either triangle
  for (int idx = t; idx < NB * NB; idx += 512) {
    const int q = idx / NB, pp = idx % NB;
    s_T[q][pp] = A[(k + q) * ld + k + pp];
  }
  __syncthreads();
  const int c = lane & 15, g = lane >> 4;  // a lane's column and row group (rows g + 4 j)
  const bool lower = wave < 4;
  // diagonal blocks
  {
    const int o = (wave & 3) * B;
    double2 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = make_double2(g + 4 * j == c ? 1.0 : 0.0, 0.0);
    if (lower) {
#pragma unroll
      for (int q = 0; q < B; ++q) {  // x_q is final: broadcast it down its column
        const double2 xq = shfl2(x[q / 4], (q & 3) * 16 + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = g + 4 * j;
          if (r > q) x[j] = cfms(x[j], ld2(&s_T[o + r][o + q]), xq);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (g + 4 * j > c) s_V[o + g + 4 * j][o + c] = x[j];
    } else {
      const double2 inv = cinv(ld2(&s_T[o + c][o + c]));
#pragma unroll
      for (int q = B - 1; q >= 0; --q) {  // y_q /= U_qq, then broadcast it up its column
        const double2 iq = shfl2(inv, q);
        if (g == (q & 3)) x[q / 4] = cmul(x[q / 4], iq);
        const double2 yq = shfl2(x[q / 4], (q & 3) * 16 + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = g + 4 * j;
          if (r < q) x[j] = cfms(x[j], ld2(&s_T[o + r][o + q]), yq);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (g + 4 * j <= c) s_V[o + g + 4 * j][o + c] = x[j];
    }
  }
  __syncthreads();
  typedef StripMma<double2, 1, B> Mma;
  const int w4 = lower ? wave : 7 - wave;                        // this wavefront's place in its triangle
  auto org = [&](int b) { return (lower ? b : 3 - b) * B; };     // first row or column of its block b
  // the inverted diagonal block b (unit diagonal of X implied, zeros outside) and others as operands
  auto D = [&](int b) {
    return [&, o = org(b)](int r, int cc) -> double2 {
      const bool in = lower ? r > cc : r <= cc;
      return in ? s_V[o + r][o + cc] : make_double2(lower && r == cc ? 1.0 : 0.0, 0.0);
    };
  };
  auto V = [&](int i, int j) { return [&, a = org(i), b = org(j)](int r, int cc) { return s_V[a + r][b + cc]; }; };
  auto F = [&](int i, int j) { return [&, a = org(i), b = org(j)](int r, int cc) { return ld2(&s_T[a + r][b + cc]); }; };
  auto times = [&](Mma& acc, auto a_at, const Mma& w) {  // acc += a w, w in its accumulators
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double2 a = a_at(c, 4 * q + g), b = w.value(0, q);
      acc.re[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc.re[0], 0, 0, 0);
      acc.im[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acc.im[0], 0, 0, 0);
      acc.re[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, acc.re[0], 0, 0, 0);
      acc.im[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acc.im[0], 0, 0, 0);
    }
  };
  auto put = [&](const Mma& acc, int i, int j) {  // block (i, j) = -acc
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 v = acc.value(0, r);
      s_V[org(i) + Mma::row(r, lane)][org(j) + c] = make_double2(-v.x, -v.y);
    }
  };
  if (w4 < 2) {
    const int i = 2 * w4 + 1, j = 2 * w4;
    Mma w, x;
    w.zero();
    w.run(F(i, j), D(j), lane);
    x.zero();
    times(x, D(i), w);
    put(x, i, j);
  }
  __syncthreads();
  {
    const int i = 2 + (w4 >> 1), j = w4 & 1;
    double2(*const w2)[B + 1] = s_W[lower ? 0 : 1][j];
    Mma w, x;
    w.zero();
    w.run(F(i, j), D(j), lane);
    if (j == 0) w.run(F(i, 1), V(1, 0), lane);
    x.zero();
    if (i == 2) {
#pragma unroll
      for (int r = 0; r < 4; ++r) w2[Mma::row(r, lane)][c] = w.value(0, r);
    }
    __syncthreads();
    times(x, D(i), w);
    if (i == 3) x.run(V(3, 2), [&](int r, int cc) { return w2[r][cc]; }, lane);
    put(x, i, j);
  }
  __syncthreads();
  for (int idx = t; idx < NB * NB; idx += 512) {
    const int q = idx / NB, pp = idx % NB;
    st2(A + (k + q) * ld + k + pp, s_V[q][pp]);
  }
}

template <typename T>
static void launch_linv(const JobDesc* jobs, int njobs, int k, T* work, hipStream_t s) {
  linv_kernel<T><<<njobs, 512, 0, s>>>(jobs, k, work);
}

// ------------------------------------------------------------------------------------
// interchanges + U12 = L11^-1 A12 on one 64-column tile of the trailing matrix
// ------------------------------------------------------------------------------------
// The tile's panel rows are gathered through LDS with the panel's permutation (the other
// permuted rows are written back directly), then U12 = L11^-1 A12 is one 64 x 64 x 64
// product on the matrix cores with the inverse stored by the inverse kernel (FP32 three-product
// MFMA for FP32 storage, FP64 MFMA otherwise).
// SECOND: k is panel nprev >= 1 of a group whose first panel starts at k - nprev NB.  Its
// trailing columns have not yet received the updates of the group's earlier panels, so
// after the gather the panel rows get  A12 -= L[k.., k - nprev NB .. k) U12_earlier  (the
// same 64 x 64 products, one per earlier panel, in panel order) before U12.
template <typename T, bool SECOND>
__global__ __launch_bounds__(256, sizeof(T) == sizeof(float2) ? 4 : 2) void swap_trsm_kernel(const JobDesc* jobs, int k, int nprev, T* work,
                                                        const int32_t* piv) {
  const JobDesc jd = jobs[blockIdx.y];
  const int col0 = k + NB + blockIdx.x * 64;
  if (k >= jd.npad || col0 >= jd.npad) return;  // uniform
  T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  typedef typename LdsOf<T>::type S;
  // Only the gathered tile lives in LDS; the 64 x 64 left operands (the inverse of the
  // panel's unit lower triangle, and for SECOND the first panel's facing L rows) are the
  // same for every tile of a job and are read through the cache by the MFMA operand loads.
  __shared__ S s_X[NB][64 + 4];
  __shared__ int s_dst[PERM_MAX], s_src[PERM_MAX];
  const int32_t* lst = piv + jd.piv_off + perm_off(jd.npad, k);
  const int cnt = lst[0];
  for (int i = t; i < cnt; i += 256) {
    s_dst[i] = lst[2 + i];
    s_src[i] = lst[2 + PERM_MAX + i];
  }
  __syncthreads();
  // the panel's permutation as a gather on this tile: entry i = wave + 4 s, column = lane
  T held[PERM_MAX / 4];
#pragma unroll
  for (int u = 0; u < PERM_MAX / 4; ++u) {
    const int i = wave + 4 * u;
    if (i < cnt) {
      const int dst = s_dst[i];
      const T v = A[s_src[i] * ld + col0 + lane];
      if (dst < k + NB)
        s_X[dst - k][lane] = v;
      else
        held[u] = v;
    }
  }
  __syncthreads();  // every source row is read before any destination row is written
#pragma unroll
  for (int u = 0; u < PERM_MAX / 4; ++u) {
    const int i = wave + 4 * u;
    if (i < cnt) {
      const int dst = s_dst[i];
      if (dst >= k + NB) A[dst * ld + col0 + lane] = held[u];
    }
  }
  const int ii = lane & 15;
  // this wavefront's 16 panel rows: a strip's last product is as long as its place in the triangle, so
  // the strips rotate with the tile, for the wavefronts of one SIMD to take a mix (250 FP32 systems of
  // n = 1472 357 -> 344 us, 160 FP64 ones of 2176 339 -> 320 without delayed updates)
  const int strip = (wave + blockIdx.x) & 3;
  const int row0 = k + strip * 16;
  if (SECOND) {
    // s_X -= L[k.., kl..k) U[kl.., col0..], kl = k - nprev NB: a wave owns its strip's 16 rows.
    StripMma<T, 4, sizeof(T) == sizeof(float2) ? NB / 2 : NB> d;
    d.zero();
    if constexpr (sizeof(T) == sizeof(float2)) {
      // FP32 storage: the wave's gathered rows move to registers (accumulator layout), so that
      // s_X can stage each earlier panel's 64 x 64 block of U rows, loaded once per workgroup
      // 16 bytes of a row per access instead of once per wave through the cache
      S xs[4][4];
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) xs[cb][r] = s_X[strip * 16 + d.row(r, lane)][cb * 16 + ii];
      constexpr int P4 = 64 * (int)sizeof(T) / 16;  // 16-byte pieces per row of the block
#pragma unroll 1
      for (int q = 0; q < nprev; ++q) {
        const int kq = k - (nprev - q) * NB;  // the earlier panel's first column
        __syncthreads();                      // s_X is free (copied out, or the last products done)
        for (int idx = t; idx < NB * P4; idx += 256) {
          const int row = idx / P4, p4 = idx - row * P4;
          ((float4*)&s_X[row][0])[p4] = ((const float4*)(A + (int64_t)(kq + row) * ld + col0))[p4];
        }
        // the left operand in two halves of K (the same products in the same order), so that
        // its registers fit beside the held rows and the accumulators
        T la[NB / 8];
#pragma unroll
        for (int s4 = 0; s4 < NB / 8; ++s4) la[s4] = A[(int64_t)(row0 + ii) * ld + kq + 4 * s4 + (lane >> 4)];
        __syncthreads();
        d.run_regs(la, [&](int kk, int c) { return s_X[kk][c]; }, lane);
#pragma unroll
        for (int s4 = 0; s4 < NB / 8; ++s4)
          la[s4] = A[(int64_t)(row0 + ii) * ld + kq + NB / 2 + 4 * s4 + (lane >> 4)];
        d.run_regs(la, [&](int kk, int c) { return s_X[NB / 2 + kk][c]; }, lane);
      }
      __syncthreads();  // every wave's products read s_X before it takes the updated rows
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          S* xp = &s_X[strip * 16 + d.row(r, lane)][cb * 16 + ii];
          st2(xp, csub(wide(xs[cb][r]), d.value(cb, r)));
        }
    } else {
      // FP64 storage (half the occupancy already): operands through the cache
#pragma unroll 1
      for (int q = 0; q < nprev; ++q) {
        const int kq = k - (nprev - q) * NB;
        T la[NB / 4];
#pragma unroll
        for (int s4 = 0; s4 < NB / 4; ++s4) la[s4] = A[(int64_t)(row0 + ii) * ld + kq + 4 * s4 + (lane >> 4)];
        d.run_regs(la, [&](int kk, int c) { return A[(int64_t)(kq + kk) * ld + col0 + c]; }, lane);
      }
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          S* xp = &s_X[strip * 16 + d.row(r, lane)][cb * 16 + ii];
          st2(xp, csub(ld2(xp), d.value(cb, r)));
        }
    }
  }
  // U12 = L11^-1 A12 straight from the accumulators to the panel rows (the inverse is
  // stored below the diagonal; its unit diagonal and zero upper part are implied).  The
  // lane's sixteen inverse entries are loaded before the barrier, in one batch.
  T li[4][4];  // [16 columns][step]; columns past the strip's own rows are zero and drop out
  {
    const int q = strip * 16 + ii;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const int kk = kb * 16 + 4 * s4 + (lane >> 4);
        li[kb][s4] = kk < q ? A[(int64_t)(k + q) * ld + k + kk] : T{kk == q ? 1.0f : 0.0f, 0.0f};
      }
  }
  __syncthreads();
  StripMma<T, 4, 16> u;
  u.zero();
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
    if (kb <= strip) u.run_regs(li[kb], [&](int kk, int c) { return s_X[kb * 16 + kk][c]; }, lane);
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      st2(A + (int64_t)(row0 + u.row(r, lane)) * ld + col0 + cb * 16 + ii, u.value(cb, r));
}

// ------------------------------------------------------------------------------------
// tall panels: tournament pivoting
// ------------------------------------------------------------------------------------
// A panel of R rows keeps R / PT rows per thread in registers, which bounds the
// one-workgroup panel kernel to 4096 rows.  Taller panels (LIZ of several hundred to
// ~1000 sites) choose their NB pivot rows by a tournament over many workgroups instead
// (communication-avoiding LU, Grigori, Demmel and Xiang 2011):
//   1. the panel is cut into chunks of C rows, copied to scratch, and every chunk is
//      factored with partial pivoting by the panel kernel (one workgroup each); the NB
//      rows its pivots bring to the top are the chunk's candidates;
//   2. the original values of all candidates are gathered into one block and factored
//      with partial pivoting once more; the NB rows chosen there, in that order, are the
//      panel's pivot rows, and that block's top NB x NB factors are the panel's L11, U11;
//   3. the interchanges that bring those rows to the top (same permutation-list format
//      as the panel kernel's) are applied to the panel (and the `left` columns), L11\U11
//      is written over the diagonal block, and after the inverses the rows below are
//      L21 = A21 U11^-1, one 64 x 64 x 64 product per 16-row strip on the matrix cores.
// Every step is an ordinary launch over the batch: no workgroup waits for another.

struct TallLayout {
  int nc_max;
  int64_t w1, w2, p1, p2, g2, sub1, sub2, si1, si2, total;  // byte offsets
};

static TallLayout tall_layout(int njobs, int npad_max, int chunk) {
  TallLayout L{};
  L.nc_max = (npad_max + chunk - 1) / chunk;
  auto al = [](int64_t b) { return (b + 255) / 256 * 256; };
  int64_t off = 0;
  L.w1 = off;  // [job][npad_max][NB] elements of at most 16 bytes
  off += al((int64_t)njobs * npad_max * NB * 16);
  L.w2 = off;  // [job][nc_max * NB][NB]
  off += al((int64_t)njobs * L.nc_max * NB * NB * 16);
  L.p1 = off;  // [job][nc_max][piv_ints(chunk)]
  off += al((int64_t)njobs * L.nc_max * piv_ints(chunk) * 4);
  L.p2 = off;  // [job][piv_ints(nc_max * NB)]
  off += al((int64_t)njobs * piv_ints(L.nc_max * NB) * 4);
  L.g2 = off;  // [job][nc_max * NB] global row of each candidate
  off += al((int64_t)njobs * L.nc_max * NB * 4);
  L.sub1 = off;
  off += al((int64_t)njobs * L.nc_max * sizeof(JobDesc));
  L.sub2 = off;
  off += al((int64_t)njobs * sizeof(JobDesc));
  L.si1 = off;
  off += al((int64_t)njobs * L.nc_max * 4);
  L.si2 = off;
  off += al((int64_t)njobs * 4);
  L.total = off;
  return L;
}

size_t tall_scratch_bytes(int njobs, int npad_max, int chunk, int above) {
  if (chunk <= 0 || npad_max <= above) return 0;
  return (size_t)tall_layout(njobs, npad_max, chunk).total;
}

// Sub-problem descriptors for this panel: chunk c of job j is rows [c C, ...) of the
// job's panel copy (leading dimension NB); chunks past a job's rows are empty (npad 0).
__global__ void tslu_setup_kernel(const JobDesc* jobs, int njobs, int k, int chunk, int nc_max, int npad_max,
                                  JobDesc* sub1, JobDesc* sub2, int32_t* si1, int32_t* si2) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= njobs * nc_max) return;
  const int j = idx / nc_max, c = idx - j * nc_max;
  const int rows = jobs[j].npad - k;
  const int nc = rows > 0 ? (rows + chunk - 1) / chunk : 0;
  JobDesc d{};
  if (c < nc) {
    const int r = min(chunk, rows - c * chunk);  // a multiple of NB, at least NB
    d.a_off = ((int64_t)j * npad_max + (int64_t)c * chunk) * NB;
    d.piv_off = ((int64_t)j * nc_max + c) * piv_ints(chunk);
    d.n = r;
    d.npad = r;
    d.ld = NB;
  }
  sub1[idx] = d;
  si1[idx] = 0;
  if (c == 0) {
    JobDesc e{};
    if (nc > 0) {
      e.a_off = (int64_t)j * nc_max * NB * NB;
      e.piv_off = (int64_t)j * piv_ints(nc_max * NB);
      e.n = nc * NB;
      e.npad = nc * NB;
      e.ld = NB;
    }
    sub2[j] = e;
    si2[j] = 0;
  }
}

// rows [k, npad) x cols [k, k + NB) of each job into its panel copy
template <typename T>
__global__ void tslu_copy_kernel(const JobDesc* jobs, int k, int npad_max, const T* work, T* w1) {
  const JobDesc jd = jobs[blockIdx.y];
  const int rows = jd.npad - k;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (rows <= 0 || idx >= (int64_t)rows * NB) return;
  const int r = (int)(idx / NB), q = (int)(idx - (int64_t)r * NB);
  w1[((int64_t)blockIdx.y * npad_max + r) * NB + q] = work[jd.a_off + (int64_t)(k + r) * jd.npad + k + q];
}

// Candidates of chunk (blockIdx.x) of job (blockIdx.y): the original rows that the chunk's
// interchanges moved to its first NB positions, gathered from the (unmodified) panel.
template <typename T>
__global__ __launch_bounds__(256) void tslu_gather_kernel(const JobDesc* jobs, int k, int chunk, int nc_max,
                                                          const JobDesc* sub1, const int32_t* p1, const T* work,
                                                          T* w2, int32_t* g2) {
  const int j = blockIdx.y, c = blockIdx.x;
  const JobDesc sd = sub1[j * nc_max + c];
  if (sd.npad == 0) return;
  const JobDesc jd = jobs[j];
  const int32_t* lst = p1 + sd.piv_off + perm_off(sd.npad, 0);
  const int64_t base = (int64_t)j * nc_max * NB + (int64_t)c * NB;
  for (int idx = threadIdx.x; idx < NB * NB; idx += 256) {
    const int e = idx / NB, q = idx - e * NB;
    const int gid = k + c * chunk + lst[2 + PERM_MAX + e];
    w2[(base + e) * NB + q] = work[jd.a_off + (int64_t)gid * jd.npad + k + q];
    if (q == 0) g2[base + e] = gid;
  }
}

// The tournament's winners become the panel's pivot rows: interchanges, permutation list,
// L11\U11 from the final factorization, zero-pivot report.  One workgroup per job.
// Bound by latency: the interchanges run through one wavefront's registers (lane i follows the row
// that began at position k + i; the chosen rows' own places are known), and the rows move in rounds
// of 128 (FP64 64) columns.  8 systems of n = 15,440: 66 -> 20 us, against interchanges and list
// kept in LDS, one after the other, and rounds of 32 columns.  At most 64 registers a lane, so that the sixteen
// wavefronts fit where one workgroup of the trailing update has left (on the look-ahead stream).
template <typename T>
__global__ __launch_bounds__(1024, 8) void tslu_apply_kernel(const JobDesc* jobs, int k, int left, int nc_max,
                                                          const JobDesc* sub2, const int32_t* p2, const T* w2,
                                                          const int32_t* g2, const int32_t* si2, T* work,
                                                          int32_t* piv, int32_t* info) {
  const int j = blockIdx.x;
  const JobDesc jd = jobs[j];
  if (k >= jd.npad) return;  // uniform
  const JobDesc rd = sub2[j];
  T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  int32_t* ip = piv + jd.piv_off;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  __shared__ int s_pos[PERM_MAX], s_org[PERM_MAX], s_cnt;
  const int32_t* lst2 = p2 + rd.piv_off + perm_off(rd.npad, 0);
  if (wave == 0) {
    // Interchanges that bring the chosen row of lane q to position k + q for q = 0, 1, ... in turn, as
    // partial pivoting records them.  Rows from below the panel stay where they are until chosen.
    const int sel = g2[(int64_t)j * nc_max * NB + lst2[2 + PERM_MAX + lane]];
    int now = k + lane, pivot = 0;  // where the row that began at k + lane is
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int row = __builtin_amdgcn_readlane(sel, q), d = k + q, top = row - k;
      const int p = top < NB ? __builtin_amdgcn_readlane(now, top & (NB - 1)) : row;
      now = lane == top ? d : now == d ? p : now;
      if (lane == q) pivot = p;
    }
    ip[k + lane] = pivot;
    // position k + i ends with row sel of lane i; the panel's rows that left it follow
    const bool out = now >= k + NB;
    const unsigned long long m = __ballot(out);
    const int cnt = NB + __popcll(m), slot = NB + __popcll(m & ((1ull << lane) - 1));
    s_pos[lane] = k + lane;
    s_org[lane] = sel;
    if (out) {
      s_pos[slot] = now;
      s_org[slot] = k + lane;
    }
    if (lane == 0) s_cnt = cnt;
    int32_t* lst = ip + perm_off(jd.npad, k);
    if (lane == 0) lst[0] = cnt;
    lst[2 + lane] = k + lane;
    lst[2 + PERM_MAX + lane] = sel;
    if (out) {
      lst[2 + slot] = now;
      lst[2 + PERM_MAX + slot] = k + lane;
    }
  }
  __syncthreads();
  // the permutation on the panel's columns and the `left` columns before them, a wavefront per 64
  // entries of a row, every source read before any destination is written
  constexpr int CB = sizeof(T) == sizeof(float2) ? 2 : 1;  // 64-column blocks per round
  constexpr int HELD = PERM_MAX * CB / 16;
  const int cnt = s_cnt, blocks = left / NB + 1;
  for (int b0 = 0; b0 < blocks; b0 += CB) {
    const int nb = min(CB, blocks - b0);  // uniform
    T* P = A + (k - left) + b0 * NB + lane;
    typedef decltype(T::x) V2 __attribute__((ext_vector_type(2)));
    V2 held[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const int id = wave + 16 * u, e = id / nb;
      if (e < cnt) held[u] = *(const V2*)(P + (int64_t)s_org[e] * ld + (id - e * nb) * NB);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const int id = wave + 16 * u, e = id / nb;
      if (e < cnt) *(V2*)(P + (int64_t)s_pos[e] * ld + (id - e * nb) * NB) = held[u];
    }
  }
  __syncthreads();
  // L11\U11 of the chosen rows, as the final factorization left them
  const T* top = w2 + (int64_t)j * nc_max * NB * NB;
  for (int idx = t; idx < NB * NB; idx += 1024) {
    const int q = idx / NB, pp = idx - q * NB;
    A[(int64_t)(k + q) * ld + k + pp] = top[(int64_t)q * NB + pp];
  }
  if (t == 0 && si2[j] != 0 && info[j] == 0) info[j] = k + si2[j];
}

// L21 = A21 U11^-1 below the diagonal block (U11^-1 on and above the block's diagonal,
// written by the inverse kernel): wave w of workgroup (x, job) takes rows k + NB + 64 x + 16 w.
// Bound by latency and memory (64 KB of L21 a workgroup): every load is issued before the first
// product, U11^-1 comes once per workgroup through LDS (four wavefronts read it), and its zero
// blocks are left out (10 of 16).  23 launches on 125 systems of n = 1472: 87 -> 58 us each; 8
// of 15,440: 41 -> 27.
template <typename T>
__global__ __launch_bounds__(256) void tslu_l21_kernel(const JobDesc* jobs, int k, T* work) {
  const JobDesc jd = jobs[blockIdx.y];
  const int t = threadIdx.x, lane = t & 63, ii = lane & 15, h = lane >> 4;
  const int r0 = k + NB + blockIdx.x * 64 + (t >> 6) * 16;
  if (k >= jd.npad || k + NB + (int)blockIdx.x * 64 >= jd.npad) return;  // uniform; npad is a multiple of 64
  T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  typedef typename LdsOf<T>::type S;
  constexpr bool F32 = sizeof(T) == sizeof(float2);
  // the k of step q of a 16-column block in lane quarter h: 64 bytes of a row per load
  auto kof = [](int q, int hh) { return F32 ? 8 * (q >> 1) + 2 * hh + (q & 1) : 4 * q + hh; };
  __shared__ S s_U[NB][NB + (F32 ? 8 : 2)];
  constexpr int P = 16 / (int)sizeof(T), PR = NB / P;  // elements per 16-byte piece, pieces per row
  T a[4][4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int q = 0; q < 4; ++q) a[kb][q] = A[(int64_t)(r0 + ii) * ld + k + kb * 16 + kof(q, h)];
#pragma unroll
  for (int u = 0; u < NB * PR / 256; ++u) {
    const int idx = t + 256 * u, row = idx / PR, c = idx % PR * P;
    T v[P];
    *(float4*)v = *(const float4*)(A + (int64_t)(k + row) * ld + k + c);
#pragma unroll
    for (int e = 0; e < P; ++e) st2(&s_U[row][c + e], row <= c + e ? wide(v[e]) : double2{0, 0});
  }
  __syncthreads();
  StripMma<T, 1, 16> d[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) d[cb].zero();
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int cb = kb; cb < 4; ++cb)  // U11^-1 is zero below its diagonal
      d[cb].run_regs(a[kb], [&](int kk, int c) { return s_U[kb * 16 + kof(kk >> 2, kk & 3)][cb * 16 + c]; }, lane);
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) st2(A + (int64_t)(r0 + d[cb].row(r, lane)) * ld + k + cb * 16 + ii, d[cb].value(0, r));
}

// ------------------------------------------------------------------------------------
// drivers
// ------------------------------------------------------------------------------------
// Leaf width: up to 512 bytes of leaf per thread (FP32: 32 columns up to two row slots, 16 up to five;
// FP64: half of that), so that two wavefronts per SIMD still hold it; past that it is halved to
// stay in registers.
// FP32 panels of at most small_rows (at most PANEL_SMALL_MAX = 768) rows take 256-thread
// workgroups, two per compute unit: 320 panels of 512 rows 176 us against 258 in 512-thread
// workgroups, of 768 rows 236 against 348 (2 panels: 118 and 116, 157 and 150).  FP64 panels do up to 256
// rows, where one row slot holds a 32-wide leaf.
// FP32 panels of 64 rows, more than two per compute unit, take one wavefront each (six per compute unit):
// bitwise the same, and slower by itself, but 256 threads would go round again.  A solve of one-member
// systems, 512 of them 350 us against 372 by one wavefront, 600 450 against 409, 2400 1110 against 943, 5000 2136
// against 1800; of 5000 of n = 144 in the symmetric form, whose every panel has 64 rows, 9.66 ms against 8.75.
constexpr int MANY_SMALL = 2 * 256;  // of an MI355X's 256 compute units
template <typename T>
static void launch_panel(const JobDesc* jobs, int njobs, int k, int left, int rows, T* work, int32_t* piv,
                         int32_t* info, hipStream_t s, int nopiv = 0, int small_rows = PANEL_SMALL_ROWS) {
  auto run = [&](auto pt, auto slots, auto ib) {
    constexpr int PT = decltype(pt)::value;
    panel_kernel<T, PT, decltype(slots)::value, decltype(ib)::value>
        <<<njobs, PT, 0, s>>>(jobs, k, left, work, piv, info, nopiv);
  };
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  typedef std::integral_constant<int, 4> I4;
  typedef std::integral_constant<int, 5> I5;
  typedef std::integral_constant<int, 6> I6;
  typedef std::integral_constant<int, 7> I7;
  typedef std::integral_constant<int, 8> I8;
  typedef std::integral_constant<int, 16> I16;
  typedef std::integral_constant<int, 32> I32;
  typedef std::integral_constant<int, 64> P64;
  typedef std::integral_constant<int, 256> P256;
  typedef std::integral_constant<int, 512> P512;
  if constexpr (sizeof(T) == sizeof(float2)) {
    if (rows <= std::min(small_rows, PANEL_SMALL_MAX)) {
      if (rows <= 64 && njobs > MANY_SMALL) return run(P64{}, I1{}, I32{});
      switch ((rows + 255) / 256) {
        case 1: return run(P256{}, I1{}, I32{});
        case 2: return run(P256{}, I2{}, I32{});
        default: return run(P256{}, I3{}, I16{});
      }
    }
    switch ((rows + 511) / 512) {
      case 1: return run(P512{}, I1{}, I32{});
      case 2: return run(P512{}, I2{}, I32{});
      case 3: return run(P512{}, I3{}, I16{});
      case 4: return run(P512{}, I4{}, I16{});
      case 5: return run(P512{}, I5{}, I16{});
      case 6: return run(P512{}, I6{}, I8{});
      case 7: return run(P512{}, I7{}, I8{});
      default: return run(P512{}, I8{}, I8{});
    }
  } else {
    if (rows <= 256) return run(P256{}, I1{}, I32{});
    switch ((rows + 511) / 512) {
      case 1: return run(P512{}, I1{}, I32{});
      case 2: return run(P512{}, I2{}, I16{});
      case 3: return run(P512{}, I3{}, I8{});
      case 4: return run(P512{}, I4{}, I8{});
      case 5: return run(P512{}, I5{}, I8{});
      case 6: return run(P512{}, I6{}, I4{});
      case 7: return run(P512{}, I7{}, I4{});
      default: return run(P512{}, I8{}, I4{});
    }
  }
}

// The split-mode panel at k = 0 of systems of `rows` rows, for the autotuner: variant 0 the
// 256-thread workgroups (rows <= PANEL_SMALL_MAX), 1 the 512-thread ones.
void launch_panel_f32_variant(int variant, const JobDesc* jobs, int njobs, int rows, float2* work, int32_t* piv,
                              int32_t* info, hipStream_t s) {
  launch_panel<float2>(jobs, njobs, 0, 0, rows, work, piv, info, s, 0, variant == 0 ? PANEL_SMALL_MAX : 0);
}

// One panel (and the inverses of its diagonal triangles): the register-resident panel
// kernel, or the tournament for taller panels.
template <typename T>
static void panel_step(const JobDesc* jobs, int njobs, int npad_max, int k, int left, T* work, int32_t* piv,
                       int32_t* info, const TallScratch& ts, hipStream_t s, int small_rows) {
  const int rows = npad_max - k;
  if (ts.chunk > 0 && rows > ts.above && ts.base) {
    const TallLayout L = tall_layout(ts.njobs, ts.npad_max, ts.chunk);
    char* b = (char*)ts.base;
    T* w1 = (T*)(b + L.w1);
    T* w2 = (T*)(b + L.w2);
    int32_t* p1 = (int32_t*)(b + L.p1);
    int32_t* p2 = (int32_t*)(b + L.p2);
    int32_t* g2 = (int32_t*)(b + L.g2);
    JobDesc* sub1 = (JobDesc*)(b + L.sub1);
    JobDesc* sub2 = (JobDesc*)(b + L.sub2);
    int32_t* si1 = (int32_t*)(b + L.si1);
    int32_t* si2 = (int32_t*)(b + L.si2);
    const int nc_max = L.nc_max;
    tslu_setup_kernel<<<(njobs * nc_max + 255) / 256, 256, 0, s>>>(jobs, njobs, k, ts.chunk, nc_max, ts.npad_max,
                                                                 sub1, sub2, si1, si2);
    tslu_copy_kernel<T><<<dim3((unsigned)(((int64_t)rows * NB + 255) / 256), njobs), 256, 0, s>>>(
        jobs, k, ts.npad_max, work, w1);
    launch_panel<T>(sub1, njobs * nc_max, 0, 0, ts.chunk, w1, p1, si1, s);
    tslu_gather_kernel<T><<<dim3(nc_max, njobs), 256, 0, s>>>(jobs, k, ts.chunk, nc_max, sub1, p1, work, w2, g2);
    launch_panel<T>(sub2, njobs, 0, 0, ((rows + ts.chunk - 1) / ts.chunk) * NB, w2, p2, si2, s);
    tslu_apply_kernel<T><<<njobs, 1024, 0, s>>>(jobs, k, left, nc_max, sub2, p2, w2, g2, si2, work, piv, info);
    launch_linv<T>(jobs, njobs, k, work, s);
    if (rows > NB) tslu_l21_kernel<T><<<dim3((rows - NB + 63) / 64, njobs), 256, 0, s>>>(jobs, k, work);
    return;
  }
  launch_panel<T>(jobs, njobs, k, left, rows, work, piv, info, s, 0, small_rows);
  launch_linv<T>(jobs, njobs, k, work, s);
}

// Algorithmic flops and bytes of one trailing-update launch over the unpadded rows m and
// columns c of each job's updated block: 8 m c kd flops (complex multiply-add count) and
// es (m kd + kd c + 2 m c) bytes (L21 and U12 read once, A22 read and written once).
static void update_cost(const GemmProfiler* prof, int njobs, int kd, int r_begin, int c_begin, int c_end, int es,
                        double* flops, double* bytes) {
  double f = 0.0, b = 0.0;
  for (int j = 0; j < njobs; ++j) {
    const int n = prof->n_true[j];
    const double m = (double)(n - r_begin);
    const double c = (double)((c_end > 0 ? std::min(c_end, n) : n) - c_begin);
    if (m > 0 && c > 0) {
      f += 8.0 * m * c * kd;
      b += (double)es * (m * kd + kd * c + 2.0 * m * c);
    }
  }
  *flops = f;
  *bytes = b;
}

// Blocked LU over groups of G panels (G = group, 2 .. GROUP_MAX): groups start at every
// multiple of G NB, and the big trailing update runs once per group with K = G NB, so the
// trailing matrix is streamed once per G NB columns.  Within a group the panels are
// left-looking: for panel j of the group (first column kj = k + j NB)
//   update of panel j's columns by the group's earlier panels (K = j NB, rows from kj) ->
//   panel(kj), whose interchanges also permute the earlier panels' L columns (j NB of them)
//   -> interchanges + delayed update by the earlier panels + U12 on every column past the
//   panel (swap_trsm_kernel).
// Then one trailing update A22 -= L21 U12 with K = G NB over the rows and columns past the
// group.  Every element thus receives the same updates as in the right-looking order, in
// a different association.  The solves apply each panel's permutation right after the
// earlier panels of its group (see solve.hip).
// With a side stream, the trailing update is split at the next group's first panel: its
// NB columns are updated first, then that panel (and its inverses) is factored on the
// side stream while the rest of the update runs on the main one.  The two touch disjoint
// data (the panel reads and writes only its own columns and the diagonal block; the
// update reads the L and U12 rows of this group and writes columns past the panel), and
// the next group's interchanges wait for both.
template <typename T, typename Gemm>
static void lu_factor_any(const JobDesc* jobs, int njobs, int npad_max, T* work, int32_t* piv, int32_t* info,
                          hipStream_t s, GemmProfiler* prof, const TallScratch& tall, const SideStream* side,
                          int small_rows, int group, Gemm gemm) {
  auto timed_gemm = [&](int k, int kd, int r_begin, int c_begin, int c_end) {
    const int rows = npad_max - r_begin;
    const int cols = (c_end > 0 ? std::min(c_end, npad_max) : npad_max) - c_begin;
    if (rows <= 0 || cols <= 0) return;
    if (prof) prof->before(s);
    gemm(rows, cols, k, kd, r_begin, c_begin, c_end);
    if (prof) {
      double f, b;
      update_cost(prof, njobs, kd, r_begin, c_begin, c_end, (int)sizeof(T), &f, &b);
      prof->after(s, f, b, c_end > 0 ? 0 : 1);
    }
  };
  const int GW = group * NB;
  bool ahead = false;  // this group's first panel was factored on the side stream
  for (int k = 0; k < npad_max; k += GW) {
    for (int j = 0; j < group; ++j) {
      const int kj = k + j * NB;
      if (j > 0) timed_gemm(k, j * NB, kj, kj, kj + NB);  // panel j's columns, K = j NB
      if (j == 0 && ahead)
        (void)hipStreamWaitEvent(s, side->panel_done, 0);
      else
        panel_step<T>(jobs, njobs, npad_max, kj, j * NB, work, piv, info, tall, s, small_rows);
      const int rest = npad_max - kj - NB;
      if (rest <= 0) return;
      if (j == 0)
        swap_trsm_kernel<T, false><<<dim3(rest / 64, njobs), 256, 0, s>>>(jobs, kj, 0, work, piv);
      else
        swap_trsm_kernel<T, true><<<dim3(rest / 64, njobs), 256, 0, s>>>(jobs, kj, j, work, piv);
    }
    ahead = false;
    const int rest = npad_max - k - GW;  // > 0: the group's last panel had columns past it
    if (side && rest > NB) {
      timed_gemm(k, GW, k + GW, k + GW, k + GW + NB);  // the next first panel's columns
      (void)hipEventRecord(side->update_done, s);
      (void)hipStreamWaitEvent(side->stream, side->update_done, 0);
      panel_step<T>(jobs, njobs, npad_max, k + GW, 0, work, piv, info, tall, side->stream, small_rows);
      (void)hipEventRecord(side->panel_done, side->stream);
      ahead = true;
      timed_gemm(k, GW, k + GW, k + GW + NB, 0);
    } else {
      timed_gemm(k, GW, k + GW, k + GW, 0);
    }
  }
}

// ------------------------------------------------------------------------------------
// symmetric factorization (complex-symmetric S, no pivoting)
// ------------------------------------------------------------------------------------
// For S = S^T the unpivoted LU has U = D L^T (D = diag U).  So after each panel the U12 rows
// are the transpose of the panel's L21 scaled by D (no triangular solve, no interchanges),
// the trailing matrix is kept only on and below the diagonal, and every trailing update is
// the lower-triangle half of A22 -= L21 U12: (4/3) n^3 instead of (8/3) n^3.  The factors
// are stored exactly as the LU's (L below, U above the diagonal, identity permutations), so
// the LU solves and the diagonal-block inverses apply unchanged.

// U[k + q][c] = D[q] L[c][k + q] for c in [k + NB, npad): one 64-column tile per workgroup,
// transposed through LDS.  Runs before the inverse kernel (D is read off the diagonal block).
// from_inverse: the diagonal block already holds the inverses (tall panels), D = 1 / diag.
template <typename T>
__global__ __launch_bounds__(256) void sym_u12_kernel(const JobDesc* jobs, int k, T* work, int from_inverse) {
  const JobDesc jd = jobs[blockIdx.y];
  const int c0 = k + NB + blockIdx.x * 64;
  if (k >= jd.npad || c0 >= jd.npad) return;  // uniform
  T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  __shared__ T s_t[64][NB + 1];
  __shared__ T s_d[NB];
  const int t = threadIdx.x;
  if (t < NB) {
    const T dd = A[(int64_t)(k + t) * ld + k + t];
    if (from_inverse)
      narrow_to(s_d[t], cinv(wide(dd)));
    else
      s_d[t] = dd;
  }
  for (int idx = t; idx < 64 * NB; idx += 256) {
    const int i = idx / NB, q = idx - i * NB;
    s_t[i][q] = A[(int64_t)(c0 + i) * ld + k + q];
  }
  __syncthreads();
  for (int idx = t; idx < NB * 64; idx += 256) {
    const int q = idx >> 6, i = idx & 63;
    A[(int64_t)(k + q) * ld + c0 + i] = cmul(s_d[q], s_t[i][q]);
  }
}

// Panels of the symmetric factorization: without pivoting a panel is its diagonal block
// (factored in place by the panel kernel as a 64-row sub-problem with the job's leading
// dimension) and L21 = A21 U11^-1 below it (tslu_l21_kernel), so no pass over the panel's
// whole height is needed; panels of at most tall_rows rows may instead use the panel kernel.  Sub-problem j of a
// step covers job j's block at (k, k); its pivots and list go to scratch, and the job's own
// list for the panel is the identity.
__global__ void sym_tall_setup_kernel(const JobDesc* jobs, int njobs, int k, JobDesc* sub, int32_t* sinfo,
                                      int32_t* piv) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= njobs) return;
  const JobDesc jd = jobs[j];
  JobDesc d{};
  if (k < jd.npad) {
    d.a_off = jd.a_off + (int64_t)k * jd.npad + k;
    d.ld = jd.npad;
    d.n = NB;
    d.npad = NB;
    d.piv_off = (int64_t)j * piv_ints(NB);
    // the job's permutation list for this panel: the identity
    int32_t* ip = piv + jd.piv_off;
    int32_t* lst = ip + perm_off(jd.npad, k);
    lst[0] = NB;
    for (int i = 0; i < NB; ++i) {
      ip[k + i] = k + i;
      lst[2 + i] = k + i;
      lst[2 + PERM_MAX + i] = k + i;
    }
  }
  sub[j] = d;
  sinfo[j] = 0;
}

__global__ void sym_tall_info_kernel(int njobs, int k, const int32_t* sinfo, int32_t* info) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < njobs && sinfo[j] != 0 && info[j] == 0) info[j] = k + sinfo[j];
}

size_t ldlt_scratch_bytes(int njobs) {
  return (size_t)njobs * (sizeof(JobDesc) + 4 * (size_t)piv_ints(NB) + 4) + 3 * 256;
}

void ldlt_factor_f32(const JobDesc* jobs, int njobs, int npad_max, float2* work, int32_t* piv, int32_t* info,
                     hipStream_t s, GemmProfiler* prof, const Half2Scratch& half2, int tall_rows, void* scratch) {
  JobDesc* sub = (JobDesc*)scratch;
  int32_t* spiv = (int32_t*)((char*)scratch + (njobs * sizeof(JobDesc) + 255) / 256 * 256);
  int32_t* sinfo = spiv + (int64_t)njobs * piv_ints(NB);
  // one panel with its U12 rows and inverses; tall panels as above
  auto panel = [&](int k) {
    const int rows = npad_max - k, rest = rows - NB;
    if (rows > tall_rows && scratch) {
      sym_tall_setup_kernel<<<(njobs + 255) / 256, 256, 0, s>>>(jobs, njobs, k, sub, sinfo, piv);
      launch_panel<float2>(sub, njobs, 0, 0, NB, work, spiv, sinfo, s, 1);
      sym_tall_info_kernel<<<(njobs + 255) / 256, 256, 0, s>>>(njobs, k, sinfo, info);
      launch_linv<float2>(jobs, njobs, k, work, s);
      if (rest > 0) {
        tslu_l21_kernel<float2><<<dim3((rest + 63) / 64, njobs), 256, 0, s>>>(jobs, k, work);
        sym_u12_kernel<float2><<<dim3(rest / 64, njobs), 256, 0, s>>>(jobs, k, work, 1);
      }
      return;
    }
    launch_panel<float2>(jobs, njobs, k, 0, rows, work, piv, info, s, 1);
    if (rest > 0) sym_u12_kernel<float2><<<dim3(rest / 64, njobs), 256, 0, s>>>(jobs, k, work, 0);
    launch_linv<float2>(jobs, njobs, k, work, s);
  };
  auto timed = [&](int k, int kd, int rb, bool lower, int c_end) {
    const int rows = npad_max - rb;
    if (rows <= 0) return;
    if (prof) prof->before(s);
    if (lower && half2.p && half2_update(rows, kd))
      launch_gemm_half2(jobs, njobs, rows, rows, k, kd, rb, rb, 0, work, half2, s, true);
    else if (lower)
      launch_gemm_f32_lower(jobs, njobs, rows, k, kd, rb, work, s);
    else
      launch_gemm_f32(7, jobs, njobs, rows, std::min(c_end, npad_max) - rb, k, kd, rb, rb, c_end, work, s);
    if (prof) {
      // algorithmic work: the lower triangle (with diagonal) of each job's unpadded block
      double f = 0.0, b = 0.0;
      for (int j = 0; j < njobs; ++j) {
        const double m = (double)(prof->n_true[j] - rb);
        if (m <= 0) continue;
        const double c = lower ? m : std::min((double)(c_end - rb), m);
        const double e = lower ? m * (m + 1) / 2 : m * c;
        f += 8.0 * e * kd;
        b += 8.0 * (m * kd + kd * c + 2.0 * e);
      }
      prof->after(s, f, b, lower ? 1 : 0);
    }
  };
  constexpr int GW = LDLT_GROUP * NB;
  for (int k = 0; k < npad_max; k += GW) {
    for (int kj = k; kj < std::min(k + GW, npad_max); kj += NB) {
      if (kj > k) timed(k, kj - k, kj, false, kj + NB);  // the panel's columns
      panel(kj);
    }
    if (npad_max > k + GW) timed(k, GW, k + GW, true, 0);
  }
}

// The updates of a panel's columns within its group (64 columns, K < G NB) take the narrow
// tiling; the K = G NB updates (split or not at the look-ahead panel) take the wide one, so
// every element sums in the same order with and without the look-ahead stream.
void lu_factor_f64(const JobDesc* jobs, int njobs, int npad_max, double2* work, int32_t* piv, int32_t* info,
                   hipStream_t s, GemmProfiler* prof, Tiling tiling, const TallScratch& tall, const SideStream* side) {
  lu_factor_any<double2>(jobs, njobs, npad_max, work, piv, info, s, prof, tall, side, tiling.panel_small_rows,
                         tiling.group, [&](int rows, int cols, int k, int kd, int rb, int cb, int ce) {
                           launch_gemm_f64_variant(kd < tiling.group * NB ? tiling.narrow : tiling.wide, jobs, njobs,
                                                   rows, cols, k, kd, rb, cb, ce, work, s);
                         });
}

void lu_factor_f32(const JobDesc* jobs, int njobs, int npad_max, float2* work, int32_t* piv, int32_t* info,
                   hipStream_t s, GemmProfiler* prof, Tiling tiling, const TallScratch& tall,
                   const Half2Scratch& half2, const SideStream* side) {
  lu_factor_any<float2>(jobs, njobs, npad_max, work, piv, info, s, prof, tall, side, tiling.panel_small_rows,
                        tiling.group, [&](int rows, int cols, int k, int kd, int rb, int cb, int ce) {
                          const bool wide = kd == tiling.group * NB;
                          launch_gemm_f32_any(wide ? tiling.wide : tiling.narrow, jobs, njobs, rows, cols, k, kd, rb,
                                              cb, ce, work, wide ? half2 : Half2Scratch{}, s);
                        });
}

}  // namespace lsms
