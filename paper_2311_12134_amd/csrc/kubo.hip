// Kubo-Greenwood sums of Eq. (10) and the four-term combination of Eq. (7).
//
// For atom m (one workgroup) and every LIZ member a, with X_a(z) = tau^{a0}(z) and the
// row tau^{0a}(z) = X_a(z)^T (reciprocity of the complex-symmetric T^-1 - g):
//   s_m[c][mu][nu] += Tr[ J^{m mu}(z2,z1) X_a(z1)^T J^{a nu}(z1,z2) X_a(z2) ]
//                  = sum_{ij} (J0_mu X1^T)_{ij} (Ja_nu X2)_{ji}
//                  = Tr[ J0_mu Z_nu ],   Z_nu = sum_a X1_a^T (Ja_nu X2_a)
// One wavefront per (atom, energy combination, nu) keeps its Z_nu in registers over all members,
// laid out as the FP64 matrix cores leave their results: two 16 x 16 x 16 products per member, no entry products
// until the one trace with J0 at the end.  Nothing passes through LDS: the accumulator layout of
// Ja X2 is the operand layout of the second product, X1^T and X2 are both read as the blocks lie
// (1 KB per load instruction), and Ja stays in registers while the species stays.
// Bound by the FP64 matrix cores, 2 x 16 x 16 instructions a member and wavefront; the next member
// is loaded while the products of this one run.  4000 atoms of 135 members (tensor): 10.7 -> 6.8 ms
// against a workgroup per atom that staged both blocks and all matrices through LDS (one such
// workgroup per compute unit, loads between barriers); 6 atoms, where the wavefronts of one nu
// also spread over three times as many compute units, 633 -> 222 us.  The sum over atoms then runs
// in a fixed order in a single workgroup, so sigma is reproducible.
#include <mutex>

#include "lsms_internal.h"

namespace lsms {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ inline int combo_z1(int c) { return c >> 1; }  // (+,+) (+,-) (-,+) (-,-)
__device__ inline int combo_z2(int c) { return c & 1; }

template <bool TENSOR>
__global__ __launch_bounds__(256) void kubo_trace_kernel(int n_atoms, const int64_t* liz_ptr, const int32_t* liz_atom,
                                                         const double2* tau_plus, const double2* tau_minus,
                                                         const int32_t* species, int n_species,
                                                         const double2* J, double2* per_atom) {
  constexpr int NQ = TENSOR ? 36 : 12;  // sums per atom: [combo][mu] or [combo][mu][nu]
  // an atom's three workgroups (nu = 0 .. 2) read the same blocks: they follow each other on one
  // XCD (workgroups go to the eight XCDs round-robin), whose L2 serves the second and third
  const int seq = blockIdx.x >> 3, atom = (seq / 3) * 8 + (blockIdx.x & 7), nu = seq % 3;
  if (atom >= n_atoms) return;
  const int64_t off = liz_ptr[atom];
  const int nl = (int)(liz_ptr[atom + 1] - off);
  const int lane = threadIdx.x & 63, c = threadIdx.x >> 6;
  const int z1 = combo_z1(c), z2 = combo_z2(c), crev = z2 * 2 + z1;
  double2* out = per_atom + (int64_t)atom * NQ + (TENSOR ? c * 9 + nu : c * 3 + nu);
  const int s0 = species[atom];
  // an out-of-range species index poisons this atom's sums instead of reading past J
  bool bad = s0 < 0 || s0 >= n_species;
  for (int a = lane; a < nl; a += 64) {
    const int sa = species[liz_atom[off + a]];
    bad |= sa < 0 || sa >= n_species;
  }
  if (__any(bad)) {  // the same in every wavefront of the atom
    if (lane == 0)
      for (int mu = 0; mu < (TENSOR ? 3 : 1); ++mu) out[3 * mu] = make_double2(NAN, NAN);
    return;
  }
  const int ii = lane & 15, kq = lane >> 4;
  const double2* T1 = (z1 ? tau_minus : tau_plus) + off * NL * NL + lane;
  const double2* T2 = (z2 ? tau_minus : tau_plus) + off * NL * NL + lane;
  const double2* Jc = J + (c * 3 + nu) * NL * NL + ii * NL + kq;  // Ja (row l % 16, column l / 16)
  int sp = 0;                                                     // species of 64 members, one per lane
  auto member_species = [&](int a) {                              // a = 0, 1, 2, .. in turn
    if ((a & 63) == 0) sp = species[liz_atom[off + min(a + lane, nl - 1)]];
    return __builtin_amdgcn_readlane(sp, a & 63);
  };
  constexpr int S = NL / 4;  // steps of a product
  double2 x1[S], x2[S], ja[S], y1[S], y2[S], jn[S];
  auto load_x = [&](int a, double2* u, double2* v) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      u[s] = T1[(int64_t)a * NL * NL + 64 * s];
      v[s] = T2[(int64_t)a * NL * NL + 64 * s];
    }
  };
  auto load_j = [&](int sa, double2* u) {
#pragma unroll
    for (int s = 0; s < S; ++s) u[s] = Jc[(int64_t)sa * 12 * NL * NL + 4 * s];
  };
  d4 sr = {0, 0, 0, 0}, si = {0, 0, 0, 0};  // Z
  int cur = -1;
  if (nl > 0) {
    cur = member_species(0);
    load_j(cur, ja);
    load_x(0, x1, x2);
  }
  for (int a = 0; a < nl; ++a) {
    bool change = false;
    if (a + 1 < nl) {  // uniform
      const int sa = member_species(a + 1);
      load_x(a + 1, y1, y2);
      change = sa != cur;
      if (change) load_j(sa, jn);
      cur = sa;
    }
    d4 wr = {0, 0, 0, 0}, wi = {0, 0, 0, 0};  // Ja X2: entry (row l / 16 + 4 q, column l % 16)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      wr = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[s].x, x2[s].x, wr, 0, 0, 0);
      wi = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[s].x, x2[s].y, wi, 0, 0, 0);
      wr = __builtin_amdgcn_mfma_f64_16x16x4f64(-ja[s].y, x2[s].y, wr, 0, 0, 0);
      wi = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[s].y, x2[s].x, wi, 0, 0, 0);
    }
    // this member's part by itself, then added: one chain through the matrix instructions of all
    // members would round 32 times as often
    d4 zr = {0, 0, 0, 0}, zi = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < S; ++s) {  // register s of W is row 4 s + l / 16, the k of step s
      zr = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[s].x, wr[s], zr, 0, 0, 0);
      zi = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[s].x, wi[s], zi, 0, 0, 0);
      zr = __builtin_amdgcn_mfma_f64_16x16x4f64(-x1[s].y, wi[s], zr, 0, 0, 0);
      zi = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[s].y, wr[s], zi, 0, 0, 0);
    }
    sr += zr;
    si += zi;
    if (change) {
#pragma unroll
      for (int s = 0; s < S; ++s) ja[s] = jn[s];
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      x1[s] = y1[s];
      x2[s] = y2[s];
    }
  }
  // Tr[J0_mu Z]: register q holds Z (row l / 16 + 4 q, column l % 16); fixed order over the lanes
#pragma unroll
  for (int m = 0; m < (TENSOR ? 3 : 1); ++m) {
    const double2* J0 = J + ((int64_t)s0 * 12 + crev * 3 + (TENSOR ? m : nu)) * NL * NL + ii * NL + kq;
    double2 v = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < 4; ++q) v = cfma(v, J0[4 * q], make_double2(sr[q], si[q]));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      v.x += __shfl_xor(v.x, o);
      v.y += __shfl_xor(v.y, o);
    }
    // no member, no sum: an infinity or NaN of J0 times zero would still be one
    if (lane == 0) out[3 * m] = nl > 0 ? v : make_double2(0.0, 0.0);
  }
}

void launch_kubo_trace(int n_atoms, const int64_t* liz_ptr_dev, const int32_t* liz_atom, const double2* tau_plus,
                       const double2* tau_minus, const int32_t* species, int n_species, const double2* J,
                       double2* per_atom, bool tensor, hipStream_t s) {
  const int grid = (n_atoms + 7) / 8 * 24;
  if (tensor)
    kubo_trace_kernel<true><<<grid, 256, 0, s>>>(n_atoms, liz_ptr_dev, liz_atom, tau_plus, tau_minus, species,
                                                 n_species, J, per_atom);
  else
    kubo_trace_kernel<false><<<grid, 256, 0, s>>>(n_atoms, liz_ptr_dev, liz_atom, tau_plus, tau_minus, species,
                                                  n_species, J, per_atom);
}

// sigma~[c][q] = -(1/(pi V)) sum_m s_m[c][q];  sigma[q] = Re 1/4 (s~++ - s~+- - s~-+ + s~--)
// with q = mu (diagonal, NQ = 12) or q = 3 mu + nu (tensor, NQ = 36).  Thread t sums
// atoms t, t + 256, ...; the wavefronts then reduce in a fixed shuffle order.
template <int NQ>
__global__ __launch_bounds__(256) void kubo_reduce_kernel(int n_atoms, const double2* per_atom, double volume,
                                                          double* sigma, double2* sigma_tilde) {
  __shared__ double2 sred[4][NQ];
  __shared__ double2 stot[NQ];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  double2 acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = make_double2(0.0, 0.0);
  for (int a = t; a < n_atoms; a += 256) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = cadd(acc[q], per_atom[(int64_t)a * NQ + q]);
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double2 v = acc[q];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      v.x += __shfl_xor(v.x, o);
      v.y += __shfl_xor(v.y, o);
    }
    if (lane == 0) sred[wave][q] = v;
  }
  __syncthreads();
  const double f = -1.0 / (M_PI * volume);
  if (t < NQ) {
    double2 v = sred[0][t];
    for (int w = 1; w < 4; ++w) v = cadd(v, sred[w][t]);
    stot[t] = v;
    sigma_tilde[t] = make_double2(f * v.x, f * v.y);
  }
  __syncthreads();
  constexpr int NS = NQ / 4;
  if (t < NS) {
    const double re = stot[0 * NS + t].x - stot[1 * NS + t].x - stot[2 * NS + t].x + stot[3 * NS + t].x;
    sigma[t] = 0.25 * f * re;
  }
}

void launch_kubo_reduce(int n_atoms, const double2* per_atom, double volume, double* sigma, double2* sigma_tilde,
                        bool tensor, hipStream_t s) {
  if (tensor)
    kubo_reduce_kernel<36><<<1, 256, 0, s>>>(n_atoms, per_atom, volume, sigma, sigma_tilde);
  else
    kubo_reduce_kernel<12><<<1, 256, 0, s>>>(n_atoms, per_atom, volume, sigma, sigma_tilde);
}

// ------------------------------------------------------------------------------------
// Fixed scratch of the allocation-free Kubo sum: the per-atom partial sums [atom][4][3]
// (complex) for up to NOALLOC_MAX_ATOMS atoms, one copy per GPU for the life of the
// process.  Host code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): noalloc_scratch_init looks up its device address once per
// device, with that device current, and everything else uses that address.
// ------------------------------------------------------------------------------------
static __device__ __align__(256) double2 scratch[(size_t)NOALLOC_MAX_ATOMS * 12];
static constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mu;

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int prev = 0;
  hipError_t e = hipGetDevice(&prev);
  if (e != hipSuccess) return e;
  e = hipSetDevice(device);
  if (e != hipSuccess) return e;
  void* ptr = nullptr;
  e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
  const hipError_t e2 = hipSetDevice(prev);
  if (e != hipSuccess) return e;
  if (e2 != hipSuccess) return e2;
  if (!ptr) return hipErrorInvalidSymbol;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

double2* noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return (double2*)g_scratch_ptr[device];
}

}  // namespace lsms
