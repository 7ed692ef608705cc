// Solves with the blocked LU factors (forward substitution, back substitution, and the
// transposed pair used by the adjoint).
//
// The factorization is the product M = P_1^T L_1 P_2^T L_2 ... P_K^T L_K U of panel
// permutations P_p and unit-lower panel factors L_p (stored in the panel's columns,
// never re-permuted by later panels; the factorization leaves the inverses of the unit
// lower and the upper diagonal triangles in each diagonal block).  Hence
//   M X = B   :  X = U^-1 L_K^-1 P_K ... L_1^-1 P_1 B          (trans = 0)
//   M^T X = B :  X = P_1^T L_1^-T ... P_K^T L_K^-T U^-T B      (trans = 1)
// Panels come in groups of G (2 .. 4, as the factorization had them: the L rows of a
// panel are stored after the permutations of the later panels of its group) and every group
// costs two launches over the whole batch:
//   solve_group_diag_kernel    one workgroup per job: the group's permutations in one gather, then
//                              panel by panel the NB x NB diagonal step as a product with the
//                              stored inverse (or its transpose) and the coupling blocks of the
//                              panels still to come with it;
//   solve_group_update_kernel  one workgroup per (64-row strip, job): the strip against the
//                              group's G NB solved rows (K = G NB) on the matrix cores,
//                              operands read straight from the factors (FP32 factors widened in
//                              registers for FP64 solves) and the solution, so the factors
//                              stream from HBM once per solve and the solution rows are read
//                              and written once per group.
// The update is column-oriented (rows below for L and U^T, rows above for U) except for
// L^T, whose group rows need a sum over all rows below: there every strip adds its partial
// product to the group rows with FP64 atomics.  Arithmetic is FP64 for both storage types of
// the factors, except in the split-mode refinement: its forward solves (L and U) with the
// FP32 factors run in FP32 (three-product FP32 MFMA) on an FP32 copy of the right-hand side,
// since a solve with FP32 factors is no more accurate than FP32 however it is summed; the
// residuals and the accumulation of the solution stay FP64.
#include <type_traits>

#include "lsms_internal.h"
#include "strip_mma.h"

namespace lsms {

typedef double d4 __attribute__((ext_vector_type(4)));

enum { MODE_L = 0, MODE_U = 1, MODE_UT = 2, MODE_LT = 3 };

// The solution block of a job: FP64 rows of NRHS_MAX columns, or the FP32 copy the split-mode
// refinement solves on, which lives in columns 16 .. 23 of the same rows (2 NRHS_MAX float2
// per row; the forward solves use columns 0 .. 15 only).
template <typename XT>
struct XView;
template <>
struct XView<double2> {
  static constexpr int LD = NRHS_MAX;
  __device__ static double2* base(double2* xbuf, const JobDesc& jd, int64_t col_off) {
    return xbuf + jd.x_off + col_off;
  }
};
template <>
struct XView<float2> {
  static constexpr int LD = 2 * NRHS_MAX;
  __device__ static float2* base(double2* xbuf, const JobDesc& jd, int64_t) {
    return (float2*)(xbuf + jd.x_off) + 2 * 16;
  }
};
// a factor element in the solve's precision
template <typename XT, typename T>
__device__ inline XT fac(const T* p);
template <>
__device__ inline double2 fac<double2, double2>(const double2* p) { return *p; }
template <>
__device__ inline double2 fac<double2, float2>(const float2* p) { return ld2(p); }
template <>
__device__ inline float2 fac<float2, float2>(const float2* p) { return *p; }
__device__ inline double2 xminus(double2 x, double2 v) { return csub(x, v); }
__device__ inline float2 xminus(float2 x, double2 v) { return make_float2(x.x - (float)v.x, x.y - (float)v.y); }
__device__ inline void xput(double2& d, double2 v) { d = v; }
__device__ inline void xput(float2& d, double2 v) { d = make_float2((float)v.x, (float)v.y); }

// The permutations of a group's panels, as one: every moved row's source is traced back through
// the panels' lists (one hash table of destinations per list), so the solution rows are
// gathered and scattered once instead of once per panel.  lists(o) is the o-th list in the
// order of application, inverse takes (source, destination) pairs for (destination, source).
// NT threads; every source row is read into registers before any destination row is written.
constexpr int HASH_BITS = 8, HASH = 1 << HASH_BITS;  // slots of a table
static_assert(HASH >= 2 * PERM_MAX, "at most half of the slots taken");
struct PermScratch {
  int key[4][HASH], val[4][HASH];
  int dst[4 * PERM_MAX], src[4 * PERM_MAX];
};
template <int NRHS, int NT, typename XT, typename LIST>
__device__ inline void apply_perms(LIST lists, int np, bool inverse, XT* X, PermScratch& ps, int t) {
  static_assert((NT / 256) * PERM_MAX <= NT, "one entry per thread");
  constexpr int G = NT / 256, LD = XView<XT>::LD;
  // multiplicative: a panel's 64 rows would be one run of taken slots under a mask, 20 us to walk
  auto slot = [](int row) { return (int)(((unsigned)row * 2654435761u) >> (32 - HASH_BITS)); };
  const int o = t / PERM_MAX, i = t % PERM_MAX;
  int to = -1, from = -1;
  if (o < np) {
    const int32_t* lst = lists(o);
    const int cnt = lst[0], a = lst[2 + i], b = lst[2 + PERM_MAX + i];  // entries past cnt are not used
    if (i < cnt) {
      to = inverse ? b : a;
      from = inverse ? a : b;
    }
  }
  for (int q = t; q < G * HASH; q += NT) ps.key[q / HASH][q % HASH] = -1;
  __syncthreads();
  if (to >= 0) {
    int h = slot(to);
    while (atomicCAS(&ps.key[o][h], -1, to) != -1) h = (h + 1) & (HASH - 1);  // destinations of a list differ
    ps.val[o][h] = from;
  }
  __syncthreads();
  auto find = [&](int l, int row) {
    int h = slot(row), k;
    while ((k = ps.key[l][h]) != -1 && k != row) h = (h + 1) & (HASH - 1);
    return k == -1 ? -1 : ps.val[l][h];
  };
  if (to >= 0) {
    for (int l = o - 1; l >= 0; --l) {
      const int f = find(l, from);
      if (f >= 0) from = f;
    }
    for (int l = o + 1; l < np; ++l)
      if (find(l, to) >= 0) to = -1;  // a later list writes this row
  }
  if (t < G * PERM_MAX) {
    ps.dst[t] = to;
    ps.src[t] = from;
  }
  __syncthreads();
  constexpr int HELD = G * PERM_MAX * NRHS / NT;
  XT held[HELD];
#pragma unroll
  for (int u = 0; u < HELD; ++u) {
    const int idx = t + NT * u, e = idx / NRHS, c = idx % NRHS;
    held[u] = ps.dst[e] >= 0 ? X[(int64_t)ps.src[e] * LD + c] : XT{};
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < HELD; ++u) {
    const int idx = t + NT * u, e = idx / NRHS, c = idx % NRHS;
    if (ps.dst[e] >= 0) X[(int64_t)ps.dst[e] * LD + c] = held[u];
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------------
// group solves: the panels of the factorization come in groups (k, k + NB, ..), k a
// multiple of G NB (see lu_factor_any).  One launch per group solves its diagonal blocks and
// the coupling blocks between them; one launch per group updates every other 64-row strip
// with K = G NB (less when the job's matrix ends inside the group).  MFMA operands of the
// update are read straight from the factors and the solution rows (through the caches); no
// LDS stage, no barriers in the update.
// ------------------------------------------------------------------------------------

// The group's diagonal step: one wavefront per 16 rows of the group (4 G wavefronts).  Panel j's
// wavefronts form X_j = inv_j (X_j - sum of couplings), the wavefronts of the panels still to come
// then subtract their coupling with X_j, in accumulators that they keep, so a group is 2 G
// dependent 16 x 64 products on each wavefront's own rows, with a barrier after each.
// Sixteen columns a workgroup (blockIdx.y); 32 would not fit the registers of sixteen wavefronts.
// Bound by latency (a group holds 10 products of 64 x 64 x NRHS): the factors do not depend on
// the solution, so a wavefront's operands load a product ahead (FP32 factors in a second register
// set; FP64 factors into the set just used, while the other panels' wavefronts work), 64 consecutive
// bytes of a row per instruction.  A forward and a back step of four panels, n = 2176, against
// four wavefronts that went through the ten products one by one, each loading its own operands:
// FP32 on 6 systems 53 -> 24 and 22 us, FP64 on 2 46 -> 38; on 250 (n = 1984) 83 -> 60 and 77 -> 57,
// where the blocks' scattered rows from memory bound it (neither two workgroups a compute unit, nor
// touching the lines ahead, nor other offsets between the systems changed that).
template <typename T, typename XT, int MODE, int G>
__global__ __launch_bounds__(256 * G) void solve_group_diag_kernel(const JobDesc* jobs, int k, const T* work,
                                                                   const int32_t* piv, double2* xbuf, int64_t col_off,
                                                                   const int32_t* skip) {
  const int job = blockIdx.x;
  if (skip && skip[job]) return;
  const JobDesc jd = jobs[job];
  if (k >= jd.npad) return;  // uniform
  constexpr bool TRANS = MODE == MODE_UT || MODE == MODE_LT, FORWARD = MODE == MODE_L || MODE == MODE_UT;
  constexpr bool LOWER = MODE == MODE_L || MODE == MODE_LT, AHEAD = sizeof(T) == sizeof(float2);
  const T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  constexpr int NRHS = 16;
  XT* X = XView<XT>::base(xbuf, jd, col_off + NRHS * blockIdx.y);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int np = min(G, (jd.npad - k) / NB);  // panels of the group inside this job
  const int b = wave >> 2, row0 = (wave & 3) * 16;  // this wavefront's panel and its rows in it
  const int ii = lane & 15, kq = lane >> 4;
  constexpr int XLD = NRHS + (sizeof(XT) == sizeof(float2) ? 8 : 0);  // FP32: the lane quarters read 2 rows apart, in two bank halves
  __shared__ XT s_a[NB * XLD];
  __shared__ XT s_x[NB * XLD];
  auto list = [&](int o) {
    return piv + jd.piv_off + perm_off(jd.npad, k + (MODE == MODE_LT ? np - 1 - o : o) * NB);
  };
  __shared__ PermScratch ps;  // MODE_L and MODE_LT
  // the k of step q in lane quarter h: four quarters' 16-byte pieces side by side
  auto kof = [](int q, int h) { return sizeof(T) == sizeof(float2) ? 8 * (q >> 1) + 2 * h + (q & 1) : 4 * q + h; };
  // Panel i's block of this wavefront's rows: lane's row ii, its sixteen k's (i == b: the diagonal block)
  auto load = [&](T* a, int i) {
    const int r = k + b * NB + row0, c = k + i * NB;
    const T* p = TRANS ? A + (int64_t)c * ld + r : A + (int64_t)r * ld + c;  // uniform
    const int mine = TRANS ? kof(0, kq) * (int)ld + ii : ii * (int)ld + kof(0, kq);
#pragma unroll
    for (int q = 0; q < 16; ++q) a[q] = (p + kof(q, 0) * (TRANS ? ld : 1))[mine];
  };
  auto order = [&](int o) { return FORWARD ? o : np - 1 - o; };
  const bool active = b < np;
  const int pos = order(b);  // the step at which this wavefront's panel is solved
  typedef StripMma<XT, 1> Mma;
  T buf[2][16];  // the operand of step o is in buf[o & 1] with AHEAD, else in buf[0]
  if (active) load(buf[0], order(0));
  if constexpr (MODE == MODE_L) apply_perms<NRHS, 256 * G>(list, np, false, X, ps, t);
  auto xrow = [&](int r) { return X + (int64_t)(k + b * NB + row0 + r) * XView<XT>::LD; };
  auto slot = [&](int r) { return (row0 + r) * XLD + ii; };
  XT x0[4];
  Mma y;
  y.zero();
  if (active) {
#pragma unroll
    for (int r = 0; r < 4; ++r) x0[r] = xrow(Mma::row(r, lane))[ii];
  }
  auto product = [&](Mma& m, const T* a, const XT* xin) {
    XT w[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) w[q] = fac<XT>(a + q);
    m.run_regs(w, [&](int kk, int c) { return xin[kof(kk >> 2, kk & 3) * XLD + c]; }, lane);
  };
#pragma unroll
  for (int o = 0; o < G; ++o) {
    if (o >= np) break;  // uniform
    T* cur = buf[AHEAD ? o & 1 : 0];
    if (active && o == pos) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s_a[slot(Mma::row(r, lane))] = xminus(x0[r], y.value(0, r));
    }
    lds_barrier();
    if (active && o == pos) {
      // the diagonal block holds the inverses of both triangles: the other one's entries drop out,
      // and the unit lower triangle's diagonal is not stored
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int kk = kof(q, kq), r = row0 + ii;
        const bool mine = MODE == MODE_L ? kk < r : MODE == MODE_LT ? kk > r : MODE == MODE_U ? kk >= r : kk <= r;
        cur[q].x = mine ? cur[q].x : LOWER && kk == r ? 1 : 0;
        cur[q].y = mine ? cur[q].y : 0;
      }
      y.zero();
      product(y, cur, s_a);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        XT v;
        xput(v, y.value(0, r));
        s_x[slot(Mma::row(r, lane))] = v;
        xrow(Mma::row(r, lane))[ii] = v;
      }
    }
    if (o + 1 == np) break;  // uniform
    lds_barrier();
    if (active && o < pos) {
      if (AHEAD) load(buf[(o + 1) & 1], order(o + 1));
      product(y, cur, s_x);
      if (!AHEAD) load(cur, order(o + 1));
    }
  }
  if constexpr (MODE == MODE_LT) {
    __syncthreads();
    apply_perms<NRHS, 256 * G>(list, np, true, X, ps, t);
  }
}

// One 64-row strip s against the group's K = KD rows (KD = G NB, or fewer where the job's
// matrix ends inside the group):
//          MODE_L   X[s] -= L[s, group] X[group]      (s below the group)
//          MODE_U   X[s] -= U[s, group] X[group]      (s above)
//          MODE_UT  X[s] -= U[group, s]^T X[group]    (s below)
//          MODE_LT  X[group] -= L[s, group]^T X[s]    (s below; FP64 atomics into the group rows)
template <typename T, typename XT, int NRHS, int MODE, int KD>
__device__ inline void group_update(const T* A, int64_t ld, XT* X, int k, int s0, int wave, int lane) {
  auto xrow = [&](int r) { return X + (int64_t)r * XView<XT>::LD; };
  const int ii = lane & 15;
  if constexpr (MODE == MODE_LT) {
    // out rows = the group's KD rows (KD / 16 blocks, dealt to the four waves), K = 64 strip rows
    for (int rb = wave; rb < KD / 16; rb += 4) {
      StripMma<double2, NRHS / 16> y;
      y.zero();
      y.run([&](int i, int kk) { return ld2(A + (int64_t)(s0 + kk) * ld + k + rb * 16 + i); },
            [&](int kk, int c) { return xrow(s0 + kk)[c]; }, lane);
#pragma unroll
      for (int cb = 0; cb < NRHS / 16; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double2* xp = xrow(k + rb * 16 + y.row(r, lane)) + cb * 16 + ii;
          const double2 v = y.value(cb, r);
          atomicAdd(&xp->x, -v.x);
          atomicAdd(&xp->y, -v.y);
        }
    }
    return;
  }
  StripMma<XT, NRHS / 16, KD> y;
  y.zero();
  const int r0 = s0 + wave * 16;
  y.run(
      [&](int i, int kk) {
        return MODE == MODE_UT ? fac<XT>(A + (int64_t)(k + kk) * ld + r0 + i)
                               : fac<XT>(A + (int64_t)(r0 + i) * ld + k + kk);
      },
      [&](int kk, int c) { return xrow(k + kk)[c]; }, lane);
#pragma unroll
  for (int cb = 0; cb < NRHS / 16; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      XT* xp = xrow(r0 + y.row(r, lane)) + cb * 16 + ii;
      *xp = xminus(*xp, y.value(cb, r));
    }
}

// MODE_L and MODE_U with the strip's factor rows staged through LDS: the 64 x KD block
// A[s0 .., k ..] streams from HBM in chunks of 256 bytes per row (32 FP32 or 16 FP64
// complex columns), each thread moving 16-byte pieces of whole rows (coalesced), through two
// buffers (35 KB, four workgroups per compute unit) with the next chunk's loads issued before
// the current chunk's products; each wave then takes its 16 rows' operands from LDS.  Same
// products, same order as group_update.
template <typename T, typename XT, int NRHS, int KD>
__device__ inline void group_update_staged(const T* A, int64_t ld, XT* X, int k, int s0, int t, int wave, int lane,
                                           float4 (*sL)[64][17]) {
  constexpr int KCH = 256 / (int)sizeof(T);  // complex columns per chunk
  constexpr int NCH = KD / KCH;
  constexpr int Q = 64 * 16 / 256;            // 16-byte pieces per thread and chunk
  auto xrow = [&](int r) { return X + (int64_t)r * XView<XT>::LD; };
  float4 held[Q];
  auto load = [&](int c) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int idx = t + 256 * q, row = idx >> 4, p4 = idx & 15;
      held[q] = ((const float4*)(A + (int64_t)(s0 + row) * ld + k + c * KCH))[p4];
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int idx = t + 256 * q;
      sL[buf][idx >> 4][idx & 15] = held[q];
    }
  };
  StripMma<XT, NRHS / 16, KCH> y;
  y.zero();
  load(0);
  store(0);
  __syncthreads();
  for (int c = 0; c < NCH; ++c) {
    const int cur = c & 1;
    if (c + 1 < NCH) load(c + 1);
    const T* rows = (const T*)&sL[cur][wave * 16][0];
    y.run([&](int i, int kk) { return fac<XT>(rows + (int64_t)i * (17 * 16 / sizeof(T)) + kk); },
          [&](int kk, int cc) { return xrow(k + c * KCH + kk)[cc]; }, lane);
    if (c + 1 < NCH) store(cur ^ 1);
    __syncthreads();
  }
  const int ii = lane & 15;
  const int r0 = s0 + wave * 16;
#pragma unroll
  for (int cb = 0; cb < NRHS / 16; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      XT* xp = xrow(r0 + y.row(r, lane)) + cb * 16 + ii;
      *xp = xminus(*xp, y.value(cb, r));
    }
}

template <typename T, typename XT, int NRHS, int MODE>
__global__ __launch_bounds__(256) void solve_group_update_kernel(const JobDesc* jobs, int k, int group, const T* work,
                                                                 double2* xbuf, int64_t col_off, const int32_t* skip) {
  const int job = blockIdx.y;
  if (skip && skip[job]) return;
  const JobDesc jd = jobs[job];
  if (k >= jd.npad) return;
  const int s0 = (MODE == MODE_U) ? blockIdx.x * 64 : k + group * NB + blockIdx.x * 64;
  if (MODE == MODE_U ? (s0 >= k) : (s0 >= jd.npad)) return;  // uniform
  const T* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  XT* X = XView<XT>::base(xbuf, jd, col_off);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // strips below the group exist only when the whole group lies inside the job
  const int kd = min(group * NB, jd.npad - k);
  if constexpr (MODE == MODE_L || MODE == MODE_U) {
    __shared__ float4 sL[2][64][17];
    const int t = threadIdx.x;
    switch (kd / NB) {
      case 1: group_update_staged<T, XT, NRHS, NB>(A, ld, X, k, s0, t, wave, lane, sL); break;
      case 2: group_update_staged<T, XT, NRHS, 2 * NB>(A, ld, X, k, s0, t, wave, lane, sL); break;
      case 3: group_update_staged<T, XT, NRHS, 3 * NB>(A, ld, X, k, s0, t, wave, lane, sL); break;
      default: group_update_staged<T, XT, NRHS, 4 * NB>(A, ld, X, k, s0, t, wave, lane, sL); break;
    }
    return;
  }
  switch (kd / NB) {
    case 1: group_update<T, XT, NRHS, MODE, NB>(A, ld, X, k, s0, wave, lane); break;
    case 2: group_update<T, XT, NRHS, MODE, 2 * NB>(A, ld, X, k, s0, wave, lane); break;
    case 3: group_update<T, XT, NRHS, MODE, 3 * NB>(A, ld, X, k, s0, wave, lane); break;
    default: group_update<T, XT, NRHS, MODE, 4 * NB>(A, ld, X, k, s0, wave, lane); break;
  }
}

template <typename T, typename XT, int NRHS>
static void solve_all(const JobDesc* jobs, int njobs, int npad_max, const T* work, const int32_t* piv, double2* x,
                      int64_t col_off, int trans, int group, const int32_t* skip, hipStream_t s) {
  const int GW = group * NB;
  const int last = ((npad_max - 1) / GW) * GW;  // start of the last group
  auto diag = [&](auto mode_tag, int k) {
    constexpr int MODE = decltype(mode_tag)::value;
    auto launch = [&](auto g) {
      constexpr int G = decltype(g)::value;
      solve_group_diag_kernel<T, XT, MODE, G>
          <<<dim3(njobs, NRHS / 16), 256 * G, 0, s>>>(jobs, k, work, piv, x, col_off, skip);
    };
    static_assert(GROUP_MAX == 4, "groups of 2 .. 4 panels");
    group == 2 ? launch(std::integral_constant<int, 2>{}) : group == 3 ? launch(std::integral_constant<int, 3>{})
                                                                       : launch(std::integral_constant<int, 4>{});
  };
  auto update = [&](auto mode_tag, int k, int strips) {
    constexpr int MODE = decltype(mode_tag)::value;
    if (strips <= 0) return;
    solve_group_update_kernel<T, XT, NRHS, MODE>
        <<<dim3(strips, njobs), 256, 0, s>>>(jobs, k, group, work, x, col_off, skip);
  };
  using L = std::integral_constant<int, MODE_L>;
  using U = std::integral_constant<int, MODE_U>;
  using UT = std::integral_constant<int, MODE_UT>;
  using LT = std::integral_constant<int, MODE_LT>;
  if (!trans) {
    for (int k = 0; k < npad_max; k += GW) {
      diag(L{}, k);
      update(L{}, k, (npad_max - k - GW) / 64);
    }
    for (int k = last; k >= 0; k -= GW) {
      diag(U{}, k);
      update(U{}, k, k / 64);
    }
  } else if constexpr (std::is_same<XT, double2>::value) {  // transposed solves: FP64 only
    for (int k = 0; k < npad_max; k += GW) {
      diag(UT{}, k);
      update(UT{}, k, (npad_max - k - GW) / 64);
    }
    for (int k = last; k >= 0; k -= GW) {
      update(LT{}, k, (npad_max - k - GW) / 64);
      diag(LT{}, k);
    }
  }
}

template <typename T>
static void solve_dispatch(const JobDesc* jobs, int njobs, int npad_max, const T* work, const int32_t* piv,
                           double2* x, int64_t col_off, int nrhs, int trans, int group, const int32_t* skip,
                           hipStream_t s) {
  if (nrhs == 16)
    solve_all<T, double2, 16>(jobs, njobs, npad_max, work, piv, x, col_off, trans, group, skip, s);
  else
    solve_all<T, double2, 32>(jobs, njobs, npad_max, work, piv, x, col_off, trans, group, skip, s);
}

void lu_solve_f64(const JobDesc* jobs, int njobs, int npad_max, const double2* work, const int32_t* piv,
                  double2* x, int64_t x_col_off, int nrhs, int trans, int group, hipStream_t s) {
  solve_dispatch<double2>(jobs, njobs, npad_max, work, piv, x, x_col_off, nrhs, trans, group, nullptr, s);
}

void lu_solve_f32(const JobDesc* jobs, int njobs, int npad_max, const float2* work, const int32_t* piv,
                  double2* x, int64_t x_col_off, int nrhs, int trans, int group, hipStream_t s) {
  solve_dispatch<float2>(jobs, njobs, npad_max, work, piv, x, x_col_off, nrhs, trans, group, nullptr, s);
}

void lu_solve_f32_single(const JobDesc* jobs, int njobs, int npad_max, const float2* work, const int32_t* piv,
                         double2* x, const int32_t* skip, int group, hipStream_t s) {
  solve_all<float2, float2, 16>(jobs, njobs, npad_max, work, piv, x, 0, 0, group, skip, s);
}

}  // namespace lsms
