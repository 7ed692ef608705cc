// Split-mode trailing update A22 -= L21 U12 (the FP32 part of the LU of Eq. (3)) on the FP16
// matrix cores, which run sixteen times as many products per clock as the FP32 ones.
//
// Every real FP32 operand x is carried by two FP16 numbers, 2^e x = h1 + h2 with
// h1 = fp16(2^e x) and h2 = fp16(2^e x - h1) (both rounded to nearest): h1 and h2 hold 22 bits
// and the sign of h2, so |2^e x - h1 - h2| <= 2^-23 |2^e x| (a unit in the last place of FP32), or 2^-25 in
// units where the largest entry of x's row (of L21) or column (of U12) lies in [2^14, 2^15), whichever is
// larger: entries 2^-16 times smaller than that largest one are still carried that well.  So that
// systems with rows of unlike size do not spread L21's rows and U12's columns over more than that, row q
// of U12 is first scaled by 2^-s_q and column q of L21 by 2^s_q, 2^s_q being the size of U12's row
// (rows of unlike size then only scale rows of L21, columns only columns of U12).  A product is
//   x y = 2^-(e + f) (h1 g1 + h1 g2 + h2 g1),
// three FP16 products accumulated in FP32 (the dropped h2 g2 is at most 2^-22 |x y|, so a product errs by at
// most 2^-21 |x y|), and a complex product four such real ones (no three-product form, whose
// imaginary part cancels).  The FP16 instruction adds 16 products per rounding of the sum where the
// FP32 one adds at most four, so the sums round less often.  Measured at K = 256 against FP64, in units of 2^-24 of the
// sums of moduli |L21| |U12| (root mean square; the FP32 64 x 64 tiling in brackets): random complex
// entries 0.34 (0.55), positive ones 2.5 (4.1); entries that all lie halfway between two FP16 numbers, so
// that every dropped product is as large as it can be and has one sign, 7.5 (3.5).
//
// Scaling by rows and columns cannot bring every matrix to one size (zero blocks between columns of
// unlike size suffice), and where it fails small entries are lost beside large ones.  So these
// kernels run only where an FP64 residual checks the solution (lsms_tau_solve, which falls back to an
// FP64 LU), not for lsms_batched_lu_solve.
//
// Three launches per update and group of jobs: half2_scale_kernel finds s_q, split_half2_kernel writes the pairs of the
// L21 rows and U12 columns once, in the order the matrix instruction takes its operands, and
// gemm_half2_kernel multiplies them.  The pairs live in scratch of bounded size, so a wave
// goes through it in groups of jobs.
#include <algorithm>
#include <climits>

#include "lsms_internal.h"

namespace lsms {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

// One 32-row (L21) or 32-column (U12) block of pairs: per 16 k a fragment of four planes
// (h1 and h2 of the real part, h1 and h2 of the imaginary part), each the operand of one
// v_mfma_f32_32x32x16_f16: lane l holds row or column l % 32 and k = 8 (l / 32) .. + 7.
constexpr int PLANE = 64 * 8;         // FP16 numbers per plane
constexpr int FRAG = 4 * PLANE;       // per block and 16 k (4096 bytes)

// Scratch of one job: L blocks, U blocks, the exponents e of the rows and of the columns, s_q.
struct Half2Layout {
  int rb, cb;  // 32-row and 32-column blocks of the largest job
  int64_t u, el, eu, sk, bytes;
};
static inline __host__ __device__ Half2Layout half2_layout(int rows, int cols, int kd) {
  Half2Layout h;
  h.rb = rows / 32;
  h.cb = cols / 32;
  const int64_t block = (int64_t)(kd / 16) * FRAG * 2;
  h.u = h.rb * block;
  h.el = h.u + h.cb * block;
  h.eu = h.el + (int64_t)rows * 4;
  h.sk = h.eu + (int64_t)cols * 4;
  h.bytes = (h.sk + (int64_t)kd * 4 + 255) / 256 * 256;
  return h;
}

size_t half2_job_bytes(int rows, int cols, int kd) { return (size_t)half2_layout(rows, cols, kd).bytes; }

// s_q of every K row of U12, one wavefront per row: the exponent of the largest finite entry over all
// columns past the group (whatever columns the update is asked for, so that an update in two parts
// rounds as one does).  All of them: a row whose large entries a sample misses would leave the
// other entries of their columns in FP16's subnormals.  Bound by HBM: 102 us a launch on average over
// 1280 systems of n = 2160 and 500 of 1424, 1.5 % of a step (64 sampled entries took 15; four, eight or
// sixteen loads in flight make no difference, and with launches of fewer systems, so that
// split_half2_kernel would find the rows in the last-level cache, a step takes longer).
__global__ __launch_bounds__(256) void half2_scale_kernel(const JobDesc* jobs, int rows, int cols, int k, int kd,
                                                          const float2* work, char* scratch) {
  const JobDesc jd = jobs[blockIdx.y];
  const int c = jd.npad - k - kd, q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c <= 0 || q >= kd) return;  // c is a multiple of 64
  const float4* row = (const float4*)(work + jd.a_off + (int64_t)(k + q) * jd.npad + k + kd);
  float a = 0.f;
  auto take = [&](float x) { a = fmaxf(a, fabsf(x) < INFINITY ? fabsf(x) : 0.f); };
#pragma unroll 4
  for (int i = lane; i < c / 2; i += 64) {
    const float4 v = row[i];
    take(v.x);
    take(v.y);
    take(v.z);
    take(v.w);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) a = fmaxf(a, __shfl_xor(a, o));
  const Half2Layout lay = half2_layout(rows, cols, kd);
  int s = 0;
  if (a > 0.f) (void)frexpf(a, &s);
  if (lane == 0) ((int*)(scratch + (int64_t)blockIdx.y * lay.bytes + lay.sk))[q] = s;
}

// One workgroup per block: thread t takes row (column) t % 32 and the eight-k groups t / 32,
// t / 32 + 8, ...  A wavefront so covers one whole fragment, reads 128-byte pieces of rows
// (256-byte pieces of U12 rows) and writes 1 KB per plane.  Bound by HBM.
__global__ __launch_bounds__(256) void split_half2_kernel(const JobDesc* jobs, int rows, int cols, int k, int kd,
                                                          int r_begin, int c_begin, int c_end, const float2* work,
                                                          char* scratch) {
  const JobDesc jd = jobs[blockIdx.y];
  const Half2Layout lay = half2_layout(rows, cols, kd);
  const bool left = (int)blockIdx.x < lay.rb;
  const int b = left ? blockIdx.x : blockIdx.x - lay.rb;
  const int o0 = (left ? r_begin : c_begin) + 32 * b;
  const int omax = left || c_end == 0 ? jd.npad : min(c_end, jd.npad);
  if (o0 >= omax) return;  // uniform
  const float2* A = work + jd.a_off;
  const int64_t ld = jd.npad;
  const int t = threadIdx.x, i = t & 31, g0 = t >> 5;
  char* base = scratch + (int64_t)blockIdx.y * lay.bytes;
  const int* sk = (const int*)(base + lay.sk);
  float2 v[4][8];
  int sc[4][8];
  int m = INT_MIN / 2;  // the largest exponent after the scaling by s
  auto top = [&](float x, int s) {
    if (x != 0.f) m = max(m, __builtin_amdgcn_frexp_expf(x) + s);
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int kk = (g0 + 8 * j) * 8;
    if (kk < kd) {  // uniform
      if (left) {
        const float4* src = (const float4*)(A + (int64_t)(o0 + i) * ld + k + kk);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 x = src[u];
          v[j][2 * u] = make_float2(x.x, x.y);
          v[j][2 * u + 1] = make_float2(x.z, x.w);
        }
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[j][u] = A[(int64_t)(k + kk + u) * ld + o0 + i];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sc[j][u] = left ? sk[kk + u] : -sk[kk + u];
        top(v[j][u].x, sc[j][u]);
        top(v[j][u].y, sc[j][u]);
      }
    }
  }
  __shared__ int s_max[8][32];
  s_max[g0][i] = m;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 8; ++g) m = max(m, s_max[g][i]);
  // the largest entry to [2^14, 2^15); a row of zeros as it is (infinities and NaN stay what they
  // are and make the row's sums NaN, as in the FP32 tilings)
  const int e = m > INT_MIN / 2 ? 15 - m : 0;
  if (g0 == 0) ((int*)(base + (left ? lay.el : lay.eu)))[32 * b + i] = e;
  _Float16* dst = (_Float16*)(base + (left ? 0 : lay.u)) + (int64_t)b * (kd / 16) * FRAG;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int g = g0 + 8 * j;
    if (g * 8 < kd) {
      h8 r1, r2, i1, i2;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float x = ldexpf(v[j][u].x, sc[j][u] + e), y = ldexpf(v[j][u].y, sc[j][u] + e);
        r1[u] = (_Float16)x;
        r2[u] = (_Float16)(x - (float)r1[u]);
        i1[u] = (_Float16)y;
        i2[u] = (_Float16)(y - (float)i1[u]);
      }
      _Float16* f = dst + (int64_t)(g >> 1) * FRAG + ((g & 1) * 32 + i) * 8;
      *(h8*)(f) = r1;
      *(h8*)(f + PLANE) = r2;
      *(h8*)(f + 2 * PLANE) = i1;
      *(h8*)(f + 3 * PLANE) = i2;
    }
  }
}

// 128 x 128 complex tile per workgroup of four waves, 64 x 64 per wave as 2 x 2 blocks of
// v_mfma_f32_32x32x16_f16 (D lane l, register r -> row 8 (r / 4) + 4 (l / 32) + r % 4, column
// l % 32).  A stage is 16 k: four row and four column fragments (32 KB), copied from global memory
// straight into one of two LDS buffers while the other is multiplied; fragments lie in LDS as
// the lanes read them (16 bytes per lane, no bank conflicts).  Two workgroups per compute unit.
// Bound by HBM and the matrix cores together: on 256 systems of npad 2176 (K = 256) the two
// launches take 6.6 ms (294 TFLOP/s algorithmic) against 12.0 ms on the FP32 matrix cores, the K
// loop alone 3.7, the traffic of A22 at the copy rate 3.3, the pairs 1.1.  The A22 reads are
// what the tile waits for: a block's loads are issued before the last stage and then one
// block ahead of the stores (7.3 ms with one load and store at a time); staging through
// registers instead of straight to LDS 7.0, 128 x 64 tiles at three workgroups per compute
// unit 8.4, touching the tile's lines early to bring them into L2 7.5.
// LOWER: only the tiles on and below the diagonal (rows and columns begin together), numbered row by
// row; of a tile on the diagonal the 64 x 64 block above it is left as it is.  125 systems of npad
// 1472, K = 256: 655 us a launch and 334 for the pairs on average, where two launches of K = 128 took
// 683 each on the FP32 matrix cores.
template <bool LOWER>
__global__ __launch_bounds__(256, 2) void gemm_half2_kernel(const JobDesc* jobs, int tiles_x, int tiles_y, int rows,
                                                            int cols, int kd, int r_begin, int c_begin, int c_end,
                                                            const char* scratch, float2* work) {
  constexpr int BAND = 8;
  int T = blockIdx.x;
  {
    const int N = gridDim.x, q = N >> 3, r = N & 7, x = T & 7;
    T = x * q + min(x, r) + (T >> 3);
  }
  const int tpj = LOWER ? tiles_y * (tiles_y + 1) / 2 : tiles_x * tiles_y;
  const int job = T / tpj;
  int tx, ty;
  if constexpr (LOWER) {
    const int u = T - job * tpj;
    ty = (int)((sqrtf(8.f * u + 1.f) - 1.f) * 0.5f);
    while (ty * (ty + 1) / 2 > u) --ty;
    while ((ty + 1) * (ty + 2) / 2 <= u) ++ty;
    tx = u - ty * (ty + 1) / 2;
  } else {
    const int u = T - job * tpj;
    const int band = u / (BAND * tiles_x), rem = u - band * BAND * tiles_x;
    const int h = min(BAND, tiles_y - band * BAND);
    tx = rem / h;
    ty = band * BAND + (rem - tx * h);
  }
  const JobDesc jd = jobs[job];
  const int npad = jd.npad;
  const int cmax = c_end > 0 ? min(c_end, npad) : npad;
  const int row0 = r_begin + ty * 128, col0 = c_begin + tx * 128;
  if (row0 >= npad || col0 >= cmax) return;  // uniform
  const Half2Layout lay = half2_layout(rows, cols, kd);
  const char* base = scratch + (int64_t)job * lay.bytes;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int ns = kd / 16;

  __shared__ h8 s_f[2][8][FRAG / 8];
  // the tile's four row and four column blocks; blocks past the job's edge repeat the last one
  const h8* src[8];
  {
    const int nrb = (npad - r_begin) / 32, ncb = (cmax - c_begin) / 32;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      src[c] = (const h8*)base + (int64_t)min(ty * 4 + c, nrb - 1) * ns * (FRAG / 8) + t;
      src[4 + c] = (const h8*)(base + lay.u) + (int64_t)min(tx * 4 + c, ncb - 1) * ns * (FRAG / 8) + t;
    }
  }
  float2* A = work + jd.a_off;
  const int64_t ld = npad;
  const int* el = (const int*)(base + lay.el) - r_begin;
  const int* eu = (const int*)(base + lay.eu) - c_begin;
  auto load = [&](int s) {
#pragma unroll
    for (int c = 0; c < 8; ++c)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[c] + s * (FRAG / 8)),
                                       (__attribute__((address_space(3))) void*)&s_f[s & 1][c][wave * 64], 16, 0, 0);
  };
  // the wave's own copies have landed before the barrier that hands the buffer to the others
  auto landed = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
  };
  f16v re[2][2], im[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      re[i][j] = f16v{};
      im[i][j] = f16v{};
    }
  // the wave's C blocks, 0 .. 3 (row half b / 2, column half b % 2), two sets of registers
  // deep, so that a block's loads overlap the previous block's stores
  float2 c[2][16];
  auto cptr = [&](int b) {
    return A + (int64_t)(row0 + wm * 64 + (b >> 1) * 32 + 4 * (lane >> 5)) * ld + col0 + wn * 64 + (b & 1) * 32 +
           (lane & 31);
  };
  auto inside = [&](int b) {  // uniform
    if (LOWER && row0 == col0 && wm < wn) return false;
    return row0 + wm * 64 + (b >> 1) * 32 < npad && col0 + wn * 64 + (b & 1) * 32 < cmax;
  };
  auto load_c = [&](int b) {
    if (!inside(b)) return;
    const float2* cp = cptr(b);
#pragma unroll
    for (int r = 0; r < 16; ++r) c[b & 1][r] = cp[(int64_t)(8 * (r >> 2) + (r & 3)) * ld];
  };
  auto store_c = [&](int b) {
    if (!inside(b)) return;
    float2* cp = cptr(b);
    const int* er = el + row0 + wm * 64 + (b >> 1) * 32 + 4 * (lane >> 5);
    const int ec = eu[col0 + wn * 64 + (b & 1) * 32 + (lane & 31)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int4 e4 = *(const int4*)(er + 8 * q);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 4 * q + u, e = -(ec + (u == 0 ? e4.x : u == 1 ? e4.y : u == 2 ? e4.z : e4.w));
        float2 cv = c[b & 1][r];
        cv.x -= ldexpf(re[b >> 1][b & 1][r], e);
        cv.y -= ldexpf(im[b >> 1][b & 1][r], e);
        cp[(int64_t)(8 * q + u) * ld] = cv;
      }
    }
  };
  auto multiply = [&](int cur) {
    h8 a[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int p = 0; p < 4; ++p) a[i][p] = s_f[cur][wm * 2 + i][p * 64 + lane];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      h8 b[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) b[p] = s_f[cur][4 + wn * 2 + j][p * 64 + lane];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
#define MF(acc, x, y) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, acc, 0, 0, 0)
        MF(im[i][j], a[i][0], b[3]);
        MF(re[i][j], a[i][0], b[1]);
        MF(im[i][j], a[i][1], b[2]);
        MF(re[i][j], a[i][1], b[0]);
        MF(im[i][j], a[i][2], b[1]);
        MF(im[i][j], a[i][3], b[0]);
        MF(im[i][j], a[i][0], b[2]);
        MF(re[i][j], a[i][0], b[0]);
        MF(im[i][j], a[i][2], b[0]);
        const h8 n2 = -a[i][2], n3 = -a[i][3];
        MF(re[i][j], n2, b[3]);
        MF(re[i][j], n3, b[2]);
        MF(re[i][j], n2, b[2]);
#undef MF
      }
    }
  };
  load(0);
  landed();
  int cur = 0;
  for (int s = 0; s < ns - 1; ++s) {
    load(s + 1);  // its buffer's last readers passed the previous barrier
    multiply(cur);
    landed();
    cur ^= 1;
  }
  load_c(0);
  multiply(cur);
  load_c(1);
  store_c(0);
  load_c(2);
  store_c(1);
  load_c(3);
  store_c(2);
  store_c(3);
}

// From 512 rows on (K = 256, 512 systems: 1.15 ms at 448 rows against 1.43 on the FP32 matrix cores, 1.74
// against 2.26 at 576, 0.82 against 1.06 at 384, 0.72 against 0.73 at 320).  Below, few systems
// lose more than many gain: two launches and their latency cost 0.037 ms where the FP32 tile takes
// 0.024 (2 systems of 384 - 576 rows; the same at 1000 rows, 0.063 against 0.119 at 1920).  The
// number of systems is no part of the rule, so systems of one size round alike however a batch is cut into
// waves.  In a wave of unlike sizes the largest decides for all, as it does for the shapes of their
// panels: a smaller system's rounding may depend on its wave.
bool half2_update(int rows, int kd) { return rows >= 512 && kd <= 256; }

size_t half2_scratch_bytes(int njobs, int npad_max, int group) {
  const int kd = group * NB, rows = npad_max - kd;  // the first group's update is the largest
  if (rows <= 0 || !half2_update(rows, kd)) return 0;
  const size_t job = half2_job_bytes(rows, rows, kd);
  return std::max(job, std::min(HALF2_SCRATCH_MAX, job * (size_t)njobs));
}

// The scratch must hold at least one job (half2_job_bytes); kd a multiple of 64 up to 256.
void launch_gemm_half2(const JobDesc* jobs, int njobs, int rows, int cols, int k, int kd, int r_begin, int c_begin,
                       int c_end, float2* work, const Half2Scratch& scratch, hipStream_t s, bool lower) {
  const Half2Layout lay = half2_layout(rows, cols, kd);
  const int group = (int)std::min<int64_t>(njobs, (int64_t)scratch.bytes / lay.bytes);
  const int tx = (cols + 127) / 128, ty = (rows + 127) / 128;
  for (int j = 0; j < njobs; j += group) {
    const int nj = std::min(group, njobs - j);
    half2_scale_kernel<<<dim3(kd / 4, nj), 256, 0, s>>>(jobs + j, rows, cols, k, kd, work, (char*)scratch.p);
    split_half2_kernel<<<dim3(lay.rb + lay.cb, nj), 256, 0, s>>>(jobs + j, rows, cols, k, kd, r_begin, c_begin, c_end,
                                                                 work, (char*)scratch.p);
    if (lower)
      gemm_half2_kernel<true><<<(unsigned)((int64_t)ty * (ty + 1) / 2 * nj), 256, 0, s>>>(
          jobs + j, tx, ty, rows, cols, kd, r_begin, c_begin, c_end, (const char*)scratch.p, work);
    else
      gemm_half2_kernel<false><<<(unsigned)((int64_t)tx * ty * nj), 256, 0, s>>>(
          jobs + j, tx, ty, rows, cols, kd, r_begin, c_begin, c_end, (const char*)scratch.p, work);
  }
}

}  // namespace lsms
