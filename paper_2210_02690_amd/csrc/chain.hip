// Dense inverses of directly solved blocks through their block-tridiagonal structure (Sec. 3: a direct
// solver for J_0 d_0 = b_0 on T_0; the paper names no method).
//
// The dense Gauss-Jordan inversion of a block of n unknowns is a chain of n column steps with a pivot
// search over all rows (about 2 us a step: 1.8 ms for the 888 unknowns of the 176 x 32 channel, 7.1 ms
// for 2 060).  Breadth-first level sets of the block's pattern from two ends of the mesh make it block
// tridiagonal (the order of coarse_bt.hip), and the two chains of small blocks are eliminated towards a
// middle block side by side, for every block of the level at once:
//   left,  i < c:  X_i = S_i^{-1} U_i,  S_{i+1} = D_{i+1} - L_{i+1} X_i,   S_0 = D_0,
//   right, i > c:  Y_i = T_i^{-1} L_i,  T_{i-1} = D_{i-1} - U_{i-1} Y_i,   T_{nb-1} = D_{nb-1},
//   middle:        S_c = D_c - L_c X_{c-1} - U_c Y_{c+1},
// the S_i, T_i inverted by the register-resident matrix-core kernel, those wider than VK_ITEM_MAX rows piece by
// piece (block Gauss-Jordan).  Then the whole inverse G grows outwards from G_cc = S_c^{-1}; with M the
// blocks already there, i the next block on the left and j on the right,
//   G_iM = -X_i G_{i+1,M},  G_Mi = -G_{M,i+1} Z_i,  G_jM = -Y_j G_{j-1,M},  G_Mj = -G_{M,j-1} W_j,
//   G_ii = S_i^{-1} - X_i G_{i+1,i},  G_jj = T_j^{-1} - Y_j G_{j-1,j},  G_ij = -X_i G_{i+1,j},
//   G_ji = -Y_j G_{j-1,i},   Z_i = L_{i+1} S_i^{-1},  W_j = U_{j-1} T_j^{-1},
// two launches of matrix-core products a step.  The solve stays one product with the dense inverse.
// Measured in a setup, beside the patch inversions and with the check below, dense -> chain: 592 unknowns (88
// x 16, k = 1) 1.21 -> 0.33 ms, 888 (176 x 32, k = 2) 2.04 -> 0.56 ms, 2 060 (88 x 16, Q4) 7.7 -> 1.46 ms, 3 213 (48 x
// 8 x 8, k = 2) 20.1 -> 4.2 ms, the three levels of 64 systems 5.1, 29.6 and 18.5 -> 1.3, 8.1 and 3.7 ms.  What
// bounds it now is the chain of pivot steps inside the S_i, 0.5 to 0.7 us each, and for single blocks
// the launches between them.
//
// Pivots are sought inside a piece only, so a regular matrix can meet a singular or badly
// conditioned one.  Each inverse is therefore checked; one that fails is refined by a step of Newton's
// iteration for inverses, or, where that does not do, its level is inverted densely before the solve goes on.
#include <algorithm>
#include <climits>
#include <vector>

#include "vk_internal.h"

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One wavefront per row: a chained row's entries go to D, U or L of its chain block, a row of a dense block to
// the block (column-major), and all values to jval: this kernel is the only one that reads the caller's, so
// they may change once it has run.  cb: the row's chain block, or -1 - b for dense block b; ri: the
// row's index in it.
__global__ __launch_bounds__(256) void chain_gather_kernel(int64_t first, int64_t n_rows, const int64_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ col,
                                                           const double* __restrict__ val,
                                                           const int32_t* __restrict__ cb, const int32_t* __restrict__ ri,
                                                           const vk_chain_block* __restrict__ blk,
                                                           const vk_chain_dense* __restrict__ dense, int64_t e_first,
                                                           double* __restrict__ jval, int32_t* status) {
  const int64_t r = first + (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= n_rows) return;
  const int b = cb[r], i = ri[r];
  const int64_t e1 = row_ptr[r + 1];
  if (b < 0) {
    const vk_chain_dense q = dense[-1 - b];
    for (int64_t e = row_ptr[r] + lane; e < e1; e += 64) {
      const int64_t c = (int64_t)col[e] - q.r0;
      const double x = val[e];
      jval[e - e_first] = x;
      if (c < 0 || c >= q.n) atomicOr(&status[1], 1);
      else q.w[c * q.n + i] = x;
    }
    return;
  }
  const vk_chain_block q = blk[b];
  for (int64_t e = row_ptr[r] + lane; e < e1; e += 64) {
    const int64_t c = col[e];
    const double x = val[e];
    jval[e - e_first] = x;
    if (c < q.r0 || c >= q.r1) {
      atomicOr(&status[1], 1);
      continue;
    }
    const int bc = cb[c], j = ri[c];
    if (bc == b) q.D[(int64_t)i * q.s + j] = x;
    else if (bc == b + 1) q.U[(int64_t)i * q.s_next + j] = x;
    else if (bc == b - 1) q.L[(int64_t)i * q.s_prev + j] = x;
    else atomicOr(&status[1], 2);  // the plan makes this impossible
  }
}

// C = beta base + alpha A B per item (blockIdx.y; x: its tile), each row- or column-major (base null: zero, k = 0
// copies; base may be C).  32 x 32 tiles, a 16 x 16 tile per wavefront on the FP64 matrix cores, 32-step
// chunks through LDS with the next chunk's loads in flight: the matrices are 50 to 500 wide, so the
// tiles are small enough to give a launch tens of workgroups.
__global__ __launch_bounds__(256) void chain_gemm_kernel(const vk_gemm_item* __restrict__ items) {
  const vk_gemm_item p = items[blockIdx.y];
  constexpr int KC = 32, LA = KC + 2, LB = 32 + 1;
  __shared__ double As[32 * LA];
  __shared__ double Bs[KC * LB];
  const int tn = (p.n + 31) / 32, m0 = (int)blockIdx.x / tn * 32, n0 = (int)blockIdx.x % tn * 32;
  if (m0 >= p.m || (p.on && *p.on == 0)) return;  // uniform: the grid covers the largest item
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int wm = (wave >> 1) * 16, wn = (wave & 1) * 16;
  double av[4], bv[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // the fast index along the storage
      const int e = tid + 256 * q, s = e >> 5, f = e & 31;
      const int ra = p.a_cm ? f : s, ca = p.a_cm ? s : f, rb = p.b_cm ? f : s, cb = p.b_cm ? s : f;
      const bool oka = m0 + ra < p.m && k0 + ca < p.k, okb = k0 + rb < p.k && n0 + cb < p.n;
      const double a = p.A[oka ? (p.a_cm ? (int64_t)(k0 + ca) * p.lda + m0 + ra : (int64_t)(m0 + ra) * p.lda + k0 + ca) : 0];
      const double b = p.B[okb ? (p.b_cm ? (int64_t)(n0 + cb) * p.ldb + k0 + rb : (int64_t)(k0 + rb) * p.ldb + n0 + cb) : 0];
      av[q] = oka ? a : 0.0;
      bv[q] = okb ? b : 0.0;
    }
  };
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  if (p.k > 0) load(0);
  for (int k0 = 0; k0 < p.k; k0 += KC) {
    if (k0 > 0) __syncthreads();  // the previous chunk has been read
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = tid + 256 * q;
      As[(p.a_cm ? e & 31 : e >> 5) * LA + (p.a_cm ? e >> 5 : e & 31)] = av[q];
      Bs[(p.b_cm ? e & 31 : e >> 5) * LB + (p.b_cm ? e >> 5 : e & 31)] = bv[q];
    }
    __syncthreads();
    if (k0 + KC < p.k) load(k0 + KC);
#pragma unroll
    for (int s4 = 0; s4 < KC / 4; ++s4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(As[(wm + l16) * LA + 4 * s4 + l4], Bs[(4 * s4 + l4) * LB + wn + l16], acc,
                                                 0, 0, 0);
  }
  const int c = n0 + wn + l16;
  if (c >= p.n) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = m0 + wm + 4 * v + l4;
    if (r >= p.m) continue;
    const int64_t at = p.c_cm ? (int64_t)c * p.ldc + r : (int64_t)r * p.ldc + c;
    const double base = p.base ? p.base[p.base_cm ? (int64_t)c * p.ldbase + r : (int64_t)r * p.ldbase + c] : 0.0;
    p.C[at] = p.beta * base + p.alpha * acc[v];
  }
}

// the row and column maps of a densely inverted block's rows are its pivot rows
__global__ void chain_dense_maps_kernel(const vk_chain_dense* __restrict__ real, const int64_t* __restrict__ rows,
                                        const int32_t* __restrict__ q, int32_t* rmap, int32_t* cmap) {
  const vk_chain_dense d = real[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < d.n) rmap[d.r0 + i] = cmap[d.r0 + i] = q[rows[blockIdx.y] + i];
}

// The check of a chained inverse G: the error |G (J v) - v| of a solve whose solution v is known,
// relative to the largest entry of |G| |J| |v|, per directly solved block.  In units of u = 2^-53 dense
// Gauss-Jordan with pivoting over all rows leaves 0.3 to 13 there (coarse levels of 592 and 888
// unknowns, peak velocities 0.3 to 1 000, time steps 0.01 and 100; up to 7 000 at 1e-5), an ordinary chain
// 0.4 to 10 (10 to 600), with solutions as accurate.  A chain whose pieces are badly conditioned
// leaves 20 to 1e8 and solutions worse by as much: 20, 50 and 87 for three strongly convective matrices, 6,
// 5 and 10 times the dense inverse's error.  So up to CHECK_LIMIT a chain is accepted.  Beyond, one
// step G + G (I - J G) squares the defect, after which solutions have one to two digits more than the
// dense inverse's and the measure is 0.1 to 26 (rounding of J v): hence REFINED_LIMIT.  An error above REFINE_MAX
// is not worth the step.  (|v - J G v| would not do: dense Gauss-Jordan leaves 4 to 600 there without
// any loss in its solutions.)
constexpr double CHECK_LIMIT = 16.0, REFINED_LIMIT = 64.0, REFINE_MAX = 1e-3;

__device__ inline double probe_value(int64_t i) { return 1.0 + 0.125 * (double)(i % 13) - 0.0625 * (double)(i % 7); }

// w = J v and wa = |J| v on the chained rows, a wavefront per row
__global__ __launch_bounds__(256) void chain_probe_kernel(int64_t first, int64_t n_rows, const int64_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ col, const double* __restrict__ jval,
                                                          int64_t e_first, const int32_t* __restrict__ cb,
                                                          const vk_chain_block* __restrict__ blk, double* __restrict__ w,
                                                          double* __restrict__ wa) {
  const int64_t r = first + (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= n_rows || cb[r] < 0) return;
  const int64_t r0 = blk[cb[r]].r0;
  double s = 0.0, a = 0.0;
  for (int64_t e = row_ptr[r] + lane; e < row_ptr[r + 1]; e += 64) {
    const double x = jval[e - e_first], v = probe_value(col[e] - r0);
    s = fma(x, v, s);
    a = fma(fabs(x), v, a);
  }
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    a += __shfl_xor(a, o, 64);
  }
  if (lane == 0) {
    w[r] = s;
    wa[r] = a;
  }
}

// rs[2 k], rs[2 k + 1]: the largest |G w - v| and |G| wa of the k-th chained block, as bits (of
// nonnegative numbers: they order alike, NaN above all).  A wavefront per row, four rows' maxima together.
__global__ __launch_bounds__(256) void chain_error_kernel(int64_t first, int64_t n_rows, const int32_t* __restrict__ cb,
                                                          const vk_chain_block* __restrict__ blk,
                                                          const int32_t* __restrict__ rmap, const int32_t* __restrict__ cmap,
                                                          const double* __restrict__ w, const double* __restrict__ wa,
                                                          unsigned long long* rs) {
  __shared__ unsigned long long m0[4], m1[4];
  __shared__ int at[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r = first + (int64_t)blockIdx.x * 4 + wave;
  const bool ok = r < n_rows && cb[r < n_rows ? r : first] >= 0;  // uniform in the wavefront
  if (lane == 0) at[wave] = -1;
  if (ok) {
    const vk_chain_block q = blk[cb[r]];
    const int64_t n = q.r1 - q.r0;
    const double* g = q.W + (int64_t)rmap[r] * n;
    const int32_t* cm = cmap + q.r0;
    const double *x = w + q.r0, *xa = wa + q.r0;
    double s = 0.0, a = 0.0;
#pragma unroll 4
    for (int64_t j = lane; j < n; j += 64) {
      s = fma(g[j], x[cm[j]], s);
      a = fma(fabs(g[j]), xa[cm[j]], a);
    }
    for (int o = 32; o > 0; o >>= 1) {
      s += __shfl_xor(s, o, 64);
      a += __shfl_xor(a, o, 64);
    }
    if (lane == 0) {
      at[wave] = q.chained;
      m0[wave] = (unsigned long long)__double_as_longlong(fabs(s - probe_value(r - q.r0)));
      m1[wave] = (unsigned long long)__double_as_longlong(fabs(a));
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 0; i < 4; ++i) {
    if (at[i] < 0) continue;
    if (i < 3 && at[i + 1] == at[i]) {
      m0[i + 1] = max(m0[i + 1], m0[i]);
      m1[i + 1] = max(m1[i + 1], m1[i]);
      continue;
    }
    atomicMax(&rs[2 * at[i]], m0[i]);
    atomicMax(&rs[2 * at[i] + 1], m1[i]);
  }
}

__global__ __launch_bounds__(256) void chain_judge_kernel(int n_chained, const unsigned long long* __restrict__ rs, double limit,
                                                          int32_t* bad, int32_t* flag) {
  __shared__ int worst;
  if (threadIdx.x == 0) worst = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < n_chained; k += blockDim.x) {
    const double r = __longlong_as_double((long long)rs[2 * k]), a = __longlong_as_double((long long)rs[2 * k + 1]);
    const bool ok = r <= limit * 0x1p-53 * a && a < __builtin_huge_val();
    bad[k] = ok ? 0 : (r <= REFINE_MAX ? 1 : 2);
    if (!ok) atomicMax(&worst, bad[k]);
  }
  __syncthreads();
  if (threadIdx.x == 0) *flag = worst;
}

// The defect R = I - J G of every chained block that the check did not accept, in the chain's order: a workgroup per row of J, its
// entries through LDS, a thread per column.
__global__ __launch_bounds__(256) void chain_defect_kernel(int64_t first, const int64_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ col, const double* __restrict__ jval,
                                                           int64_t e_first, const int32_t* __restrict__ cb,
                                                           const vk_chain_block* __restrict__ blk,
                                                           const int32_t* __restrict__ rmap, const int32_t* __restrict__ cmap,
                                                           const int32_t* __restrict__ bad) {
  __shared__ double sv[256];
  __shared__ const double* sw[256];
  const int64_t r = first + blockIdx.x;
  if (cb[r] < 0) return;  // uniform
  const vk_chain_block q = blk[cb[r]];
  if (bad[q.chained] == 0) return;
  const int64_t n = q.r1 - q.r0, e1 = row_ptr[r + 1];
  const int tid = threadIdx.x;
  for (int64_t j0 = 0; j0 < n; j0 += 256) {
    const int64_t j = j0 + tid;
    double acc = 0.0;
    for (int64_t eb = row_ptr[r]; eb < e1; eb += 256) {
      const int cnt = (int)(e1 - eb < 256 ? e1 - eb : 256);
      __syncthreads();
      if (tid < cnt) {
        sv[tid] = jval[eb + tid - e_first];
        sw[tid] = q.W + (int64_t)rmap[col[eb + tid]] * n;
      }
      __syncthreads();
      if (j < n)
#pragma unroll 4
        for (int k = 0; k < cnt; ++k) acc = fma(sv[k], sw[k][j], acc);
    }
    if (j < n) q.R[(int64_t)rmap[r] * n + j] = (cmap[q.r0 + j] == (int32_t)(r - q.r0) ? 1.0 : 0.0) - acc;
  }
}

// pieces of the elimination of an s-row chain block: as few as the register-resident kernel takes, of equal
// width rounded up to whole 16-row tiles
int64_t piece_width(int64_t s) {
  const int64_t p = (s + VK_ITEM_MAX - 1) / VK_ITEM_MAX;
  return std::min<int64_t>(((s + p - 1) / p + 15) / 16 * 16, s);
}

// A block is chained where the estimated time of its chain is below 0.8 of the dense inversion's.  The
// estimates (us): a piece in the register-resident kernel (64 rows 27, 128 rows 70, 176 rows 121) and its
// four launches; 35 a step for the products; the dense inversion's 16-column panels with their updates
// (20 + 6 and the outer updates: 888 rows 1.8 ms).
double chain_us(int64_t s) {
  const int64_t w = piece_width(s), p = (s + w - 1) / w;
  return p * (w <= 128 ? 0.5 * w : 0.67 * w) + (p > 1 ? 35.0 * p : 0.0);
}
double dense_us(double n) { return 30.0 * std::ceil(n / 16.0) + 40.0; }

// doubles reserved for a block: a chain of blocks of s rows takes about 6 s n, and pays off up to about n = 5 s;
// a refinement takes 1.5 n^2
int64_t reserve(int64_t n) { return n < VK_CHAIN_MIN_N ? 0 : (n <= 1024 ? 2 * n * n : n * n + n * n / 2); }

int64_t up32(int64_t x) { return (x + 31) / 32 * 32; }

}  // namespace

int64_t vk_chain_buffer(const vk_level& L) {
  if (L.cb_rows.size() < 2 || L.cb_max < VK_CHAIN_MIN_N || L.cb_max > VK_TOURNEY_MIN_N) return 0;
  int64_t need = 2 * up32(L.J.n_rows) + 2 * up32(2 * (int64_t)(L.cb_rows.size() - 1));
  for (size_t b = 0; b + 1 < L.cb_rows.size(); ++b) {
    const int64_t n = L.cb_rows[b + 1] - L.cb_rows[b];
    if (n >= VK_CHAIN_MIN_N) need += reserve(n) + n + 64;
  }
  return need;
}

size_t vk_chain_table_bytes(const vk_level& L) {
  if (vk_chain_buffer(L) == 0) return 0;
  return (size_t)L.cb_rows.back() * 24 + (L.cb_rows.size() - 1) * (size_t)(160 * 1024) + 65536;
}

bool vk_chain_plan(vk_level& L) {
  vk_chain& T = L.chain;
  double* const buf = T.buf;
  double* const jval = T.jval;
  char* const table = T.table;
  const int64_t cap = T.cap;
  const size_t table_cap = T.table_cap;
  T = vk_chain();
  T.buf = buf;
  T.jval = jval;
  T.cap = cap;
  T.table = table;
  T.table_cap = table_cap;
  T.planned = true;
  if (!buf || L.cb_rows.size() < 2) return false;
  const int nblk = (int)L.cb_rows.size() - 1;
  const int64_t rows = L.cb_rows.back();
  std::vector<int64_t> rp(rows + 1);
  if (hipMemcpy(rp.data(), L.J.row_ptr, sizeof(int64_t) * (rows + 1), hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  std::vector<int32_t> cj(rp[rows]);
  if (rp[rows] > 0 && hipMemcpy(cj.data(), L.J.col, sizeof(int32_t) * rp[rows], hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  T.first = L.cb_rows[0];
  std::vector<int32_t> cb(rows, -1), ri(rows), rmap(rows), cmap(rows);
  std::vector<vk_chain_block> blocks;
  std::vector<vk_chain_dense>& dense = T.dense;
  struct piece_lists {
    std::vector<vk_dense_item> inv;
    std::vector<vk_gemm_item> qr, up, put;
  };
  struct step_lists {
    std::vector<piece_lists> pieces;
    std::vector<vk_gemm_item> cp, u1, u2;
  };
  std::vector<step_lists> steps;
  std::vector<vk_gemm_item> zw;
  std::vector<std::vector<vk_gemm_item>> ga, gb;
  int64_t used = 0;
  auto take = [&](int64_t n) {
    double* p = buf + used;
    used += up32(n);
    return p;
  };
  auto item = [](int64_t m, int64_t n, int64_t k, double alpha, const double* A, int64_t lda, const double* B, int64_t ldb,
                 const double* base, int64_t ldbase, double* C, int64_t ldc, bool cm) {
    vk_gemm_item g{};
    g.m = (int32_t)m;
    g.n = (int32_t)n;
    g.k = (int32_t)k;
    g.alpha = alpha;
    g.A = A;
    g.lda = (int32_t)lda;
    g.B = B;
    g.ldb = (int32_t)ldb;
    g.base = base;
    g.ldbase = (int32_t)ldbase;
    g.C = C;
    g.ldc = (int32_t)ldc;
    g.c_cm = g.base_cm = cm;
    g.beta = 1.0;
    return g;
  };
  struct block_plan {
    bool ok = false;
    int c = 0;
    std::vector<int32_t> blk;
    std::vector<int64_t> size;
  };
  std::vector<block_plan> plans(nblk);
  // which blocks have a chain that is worth it, and the zero-filled part of the buffer (D, U, L of all)
  int64_t w0 = 0;
  std::vector<int64_t> woff(nblk);
  for (int b = 0; b < nblk; ++b) {
    const int64_t r0 = L.cb_rows[b], n = L.cb_rows[b + 1] - r0;
    woff[b] = w0;
    w0 += n * n;
    if (n < VK_CHAIN_MIN_N) continue;
    block_plan& p = plans[b];
    if (!vk_level_order(r0, n, &rp[r0], cj.data() + rp[r0], VK_CHAIN_MIN_BLOCK, VK_CHAIN_MIN_BLOCK, p.blk, p.size, &p.c)) continue;
    const int nb = (int)p.size.size();
    if (*std::max_element(p.size.begin(), p.size.end()) > 2048 || *std::min_element(p.size.begin(), p.size.end()) < 16)
      continue;
    double us = chain_us(p.size[p.c]) + 60.0;
    for (int k = 0; k < std::max(p.c, nb - 1 - p.c); ++k) {
      const double a = k < p.c ? chain_us(p.size[k]) : 0.0, z = nb - 1 - k > p.c ? chain_us(p.size[nb - 1 - k]) : 0.0;
      us += std::max(a, z) + 35.0;
    }
    int64_t need = 0;
    for (int i = 0; i < nb; ++i) {
      const int64_t w = piece_width(p.size[i]);  // the inverse, or a piece's inverse and products
      need += up32(p.size[i] * p.size[i]) + (w == p.size[i] ? up32(p.size[i] * p.size[i]) : up32(w * w) + 2 * up32(w * p.size[i]));
      if (i + 1 < nb) need += 4 * up32(p.size[i] * p.size[i + 1]);
    }
    if (us > 0.8 * dense_us((double)n) || need > reserve(n)) continue;
    p.ok = true;
  }
  int64_t n_chained = 0;
  for (int b = 0; b < nblk; ++b) n_chained += plans[b].ok;
  if (n_chained == 0) return false;
  T.n_chained = (int)n_chained;
  T.w = take(L.J.n_rows);
  T.wa = take(L.J.n_rows);
  T.bad = reinterpret_cast<int32_t*>(take(n_chained));
  T.zero = buf + used;
  const int64_t used0 = used;
  T.rs = reinterpret_cast<unsigned long long*>(take(2 * n_chained));
  int64_t r_used = used;  // a refinement's buffers take the chain's place
  std::vector<vk_gemm_item> r_mul[2], r_put[2];
  int chained = 0;
  std::vector<int> first(nblk, 0);
  for (int b = 0; b < nblk; ++b) {
    const int64_t r0 = L.cb_rows[b], n = L.cb_rows[b + 1] - r0;
    if (!plans[b].ok) {
      for (int64_t r = 0; r < n; ++r) {
        cb[r0 + r] = -1 - (int32_t)dense.size();
        ri[r0 + r] = (int32_t)r;
      }
      dense.push_back(vk_chain_dense{L.cb_a + woff[b], r0, n});
      T.flops += 2.0 * (double)n * n * n;
      continue;
    }
    const block_plan& p = plans[b];
    const int nb = (int)p.size.size(), f = (int)blocks.size();
    first[b] = f;
    double *const G = L.cb_a + woff[b], *const R = buf + r_used, *const H = R + up32(n * n);
    const int64_t half = (n + 1) / 2;
    r_used += up32(n * n) + up32(half * n);
    for (int k = 0; k < 2; ++k) {  // rows [g0, g0 + m) of G + G R by way of H
      const int64_t g0 = k * half, m = k == 0 ? half : n - half;
      r_mul[k].push_back(item(m, n, n, 1.0, G + g0 * n, n, R, n, G + g0 * n, n, H, n, false));
      r_put[k].push_back(item(m, n, 0, 0.0, H, n, H, n, H, n, G + g0 * n, n, false));
      r_mul[k].back().on = r_put[k].back().on = T.bad + chained;
    }
    std::vector<int64_t> off(nb + 1, 0);
    for (int i = 0; i < nb; ++i) off[i + 1] = off[i] + p.size[i];
    std::vector<int64_t> pos(off.begin(), off.end() - 1);
    for (int64_t v = 0; v < n; ++v) {
      const int i = p.blk[v];
      const int64_t q = pos[i]++;
      cb[r0 + v] = f + i;
      ri[r0 + v] = (int32_t)(q - off[i]);
      rmap[r0 + v] = (int32_t)q;
      cmap[r0 + q] = (int32_t)v;
    }
    for (int i = 0; i < nb; ++i) {
      vk_chain_block q{};
      q.r0 = r0;
      q.r1 = r0 + n;
      q.W = G;
      q.R = R;
      q.chained = chained;
      q.s = (int32_t)p.size[i];
      q.s_prev = i > 0 ? (int32_t)p.size[i - 1] : 0;
      q.s_next = i + 1 < nb ? (int32_t)p.size[i + 1] : 0;
      q.D = take(p.size[i] * p.size[i]);
      q.U = i + 1 < nb ? take(p.size[i] * p.size[i + 1]) : nullptr;
      q.L = i > 0 ? take(p.size[i] * p.size[i - 1]) : nullptr;
      blocks.push_back(q);
    }
    ++chained;
  }
  T.n_zero = used - used0;
  for (int b = 0; b < nblk; ++b) {
    if (!plans[b].ok) continue;
    const block_plan& p = plans[b];
    const int64_t n = L.cb_rows[b + 1] - L.cb_rows[b];
    const int nb = (int)p.size.size(), f = first[b], c = p.c;
    auto sz = [&](int i) { return p.size[i]; };
    std::vector<int64_t> off(nb + 1, 0);
    for (int i = 0; i < nb; ++i) off[i + 1] = off[i] + p.size[i];
    std::vector<double*> inv(nb), X(nb, nullptr), Z(nb, nullptr);
    std::vector<int32_t> cm(nb);  // the inverse is column-major
    for (int i = 0; i < nb; ++i) {
      // a block of one piece is inverted out of place, a wider one in place, piece by piece
      cm[i] = piece_width(sz(i)) == sz(i);
      inv[i] = cm[i] ? take(sz(i) * sz(i)) : blocks[f + i].D;
      const int j = i < c ? i + 1 : (i > c ? i - 1 : -1);  // the next block inwards
      if (j >= 0) {
        X[i] = take(sz(i) * sz(j));  // X_i or Y_i
        Z[i] = take(sz(j) * sz(i));  // Z_i or W_i
      }
    }
    const int ns = std::max(c, nb - 1 - c) + 1;
    if ((int)steps.size() < ns) steps.resize(ns);
    if ((int)ga.size() < ns - 1) {
      ga.resize(ns - 1);
      gb.resize(ns - 1);
    }
    // Block Gauss-Jordan over the pieces K of S (s x s, row-major, in place), P = S_KK^{-1} (column-major):
    //   Q = S_.K P, R = P S_K.;  S_.. -= Q S_K. off row and column K;  S_K. = R, S_.K = -Q, S_KK = P.
    auto invert = [&](step_lists& S, int i) {
      const int64_t s = sz(i), w = piece_width(s);
      T.flops += 2.0 * (double)s * s * s;
      const int np = (int)((s + w - 1) / w);
      if ((int)S.pieces.size() < np) S.pieces.resize(np);
      double* D = blocks[f + i].D;
      if (np == 1) {
        S.pieces[0].inv.push_back(vk_dense_item{D, inv[i], (int32_t)s, (int32_t)s});
        return;
      }
      double *P = take(w * w), *Q = take(w * s), *R = take(w * s);
      for (int q = 0; q < np; ++q) {
        piece_lists& C = S.pieces[q];
        const int64_t k0 = q * w, k1 = std::min(k0 + w, s), h = k1 - k0;
        C.inv.push_back(vk_dense_item{D + k0 * s + k0, P, (int32_t)h, (int32_t)s});
        const int64_t e0[2] = {0, k1}, e1[2] = {k0, s};  // the rows and columns beside the piece
        for (int a = 0; a < 2; ++a) {
          const int64_t n = e1[a] - e0[a];
          if (n == 0) continue;
          vk_gemm_item g = item(n, h, h, 1.0, D + e0[a] * s + k0, s, P, h, nullptr, 0, Q + e0[a] * h, h, false);
          g.b_cm = 1;
          C.qr.push_back(g);
          g = item(h, n, h, 1.0, P, h, D + k0 * s + e0[a], s, nullptr, 0, R + e0[a], s, false);
          g.a_cm = 1;
          C.qr.push_back(g);
          for (int z = 0; z < 2; ++z)
            if (e1[z] > e0[z])
              C.up.push_back(item(n, e1[z] - e0[z], h, -1.0, Q + e0[a] * h, h, D + k0 * s + e0[z], s, D + e0[a] * s + e0[z], s,
                                  D + e0[a] * s + e0[z], s, false));
          C.put.push_back(item(h, n, 0, 0.0, P, h, P, h, R + e0[a], s, D + k0 * s + e0[a], s, false));
          C.put.push_back(item(n, h, 0, 0.0, P, h, P, h, Q + e0[a] * h, h, D + e0[a] * s + k0, s, false));
          C.put.back().beta = -1.0;
        }
        C.put.push_back(item(h, h, 0, 0.0, P, h, P, h, P, h, D + k0 * s + k0, s, false));
        C.put.back().base_cm = 1;
      }
    };
    for (int k = 0; k < ns; ++k) {
      step_lists& S = steps[k];
      if (k == ns - 1) {
        invert(S, c);
        continue;
      }
      bool first_update = true;
      for (int side = 0; side < 2; ++side) {
        const int i = side == 0 ? k : nb - 1 - k;
        if (side == 0 ? i >= c : i <= c) continue;
        const int j = side == 0 ? i + 1 : i - 1;
        invert(S, i);
        const double* out = side == 0 ? blocks[f + i].U : blocks[f + i].L;  // i -> j
        const double* back = side == 0 ? blocks[f + j].L : blocks[f + j].U;  // j -> i
        S.cp.push_back(item(sz(i), sz(j), sz(i), 1.0, inv[i], sz(i), out, sz(j), nullptr, 0, X[i], sz(j), false));
        S.cp.back().a_cm = cm[i];
        const vk_gemm_item u = item(sz(j), sz(j), sz(i), -1.0, back, sz(i), X[i], sz(j), blocks[f + j].D, sz(j),
                                    blocks[f + j].D, sz(j), false);
        // both chains can reach the middle block in one step: its updates run one after the other
        if (j == c && !first_update) S.u2.push_back(u);
        else S.u1.push_back(u);
        if (j == c) first_update = false;
        T.flops += 2.0 * sz(i) * sz(i) * sz(j) + 2.0 * sz(j) * sz(j) * sz(i);
        zw.push_back(item(sz(j), sz(i), sz(i), 1.0, back, sz(i), inv[i], sz(i), nullptr, 0, Z[i], sz(i), false));
        zw.back().b_cm = cm[i];
      }
    }
    // the whole inverse, outwards from the middle
    double* G = L.cb_a + woff[b];
    auto g = [&](int64_t r, int64_t q) { return G + r * n + q; };
    zw.push_back(item(sz(c), sz(c), 0, 0.0, inv[c], sz(c), inv[c], sz(c), inv[c], sz(c), g(off[c], off[c]), n, false));
    zw.back().base_cm = cm[c];
    for (int t = 1; t < ns; ++t) {
      const int i = c - t, j = c + t;
      const int64_t a0 = off[std::max(i + 1, 0)], a1 = off[std::min(j, nb)], M = a1 - a0;
      std::vector<vk_gemm_item>&A = ga[t - 1], &B = gb[t - 1];
      if (i >= 0) {
        A.push_back(item(sz(i), M, sz(i + 1), -1.0, X[i], sz(i + 1), g(off[i + 1], a0), n, nullptr, 0, g(off[i], a0), n, false));
        A.push_back(item(M, sz(i), sz(i + 1), -1.0, g(a0, off[i + 1]), n, Z[i], sz(i), nullptr, 0, g(a0, off[i]), n, false));
        B.push_back(item(sz(i), sz(i), sz(i + 1), -1.0, X[i], sz(i + 1), g(off[i + 1], off[i]), n, inv[i], sz(i),
                         g(off[i], off[i]), n, false));
        B.back().base_cm = cm[i];
        T.flops += 4.0 * sz(i) * sz(i + 1) * M;
      }
      if (j < nb) {
        A.push_back(item(sz(j), M, sz(j - 1), -1.0, X[j], sz(j - 1), g(off[j - 1], a0), n, nullptr, 0, g(off[j], a0), n, false));
        A.push_back(item(M, sz(j), sz(j - 1), -1.0, g(a0, off[j - 1]), n, Z[j], sz(j), nullptr, 0, g(a0, off[j]), n, false));
        B.push_back(item(sz(j), sz(j), sz(j - 1), -1.0, X[j], sz(j - 1), g(off[j - 1], off[j]), n, inv[j], sz(j),
                         g(off[j], off[j]), n, false));
        B.back().base_cm = cm[j];
        T.flops += 4.0 * sz(j) * sz(j - 1) * M;
      }
      if (i >= 0 && j < nb) {
        B.push_back(item(sz(i), sz(j), sz(i + 1), -1.0, X[i], sz(i + 1), g(off[i + 1], off[j]), n, nullptr, 0,
                         g(off[i], off[j]), n, false));
        B.push_back(item(sz(j), sz(i), sz(j - 1), -1.0, X[j], sz(j - 1), g(off[j - 1], off[i]), n, nullptr, 0,
                         g(off[j], off[i]), n, false));
      }
    }
  }
  if (used > cap || r_used > cap) return false;
  // upload the tables
  size_t tused = 0;
  bool ok = true;
  auto put = [&](const void* src, size_t bytes) -> char* {
    tused = (tused + 63) / 64 * 64;
    char* dst = table + tused;
    if (!ok || tused + bytes > table_cap) {
      ok = false;
      return nullptr;
    }
    if (bytes > 0 && hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipGetLastError();
      ok = false;
    }
    tused += bytes;
    return dst;
  };
  auto put_gemm = [&](const std::vector<vk_gemm_item>& v) {
    vk_gemm_list l;
    l.count = (int)v.size();
    for (const vk_gemm_item& g : v) l.tiles = std::max<int64_t>(l.tiles, (int64_t)((g.m + 31) / 32) * ((g.n + 31) / 32));
    l.items = reinterpret_cast<vk_gemm_item*>(put(v.data(), v.size() * sizeof(vk_gemm_item)));
    return l;
  };
  T.cb = reinterpret_cast<int32_t*>(put(cb.data(), rows * 4));
  T.ri = reinterpret_cast<int32_t*>(put(ri.data(), rows * 4));
  T.rmap = reinterpret_cast<int32_t*>(put(rmap.data(), rows * 4));
  T.cmap = reinterpret_cast<int32_t*>(put(cmap.data(), rows * 4));
  T.blocks = reinterpret_cast<vk_chain_block*>(put(blocks.data(), blocks.size() * sizeof(vk_chain_block)));
  T.d_dense = reinterpret_cast<vk_chain_dense*>(put(dense.data(), dense.size() * sizeof(vk_chain_dense)));
  T.rows = rows;
  for (step_lists& S : steps) {
    vk_chain_step st;
    for (piece_lists& C : S.pieces) {
      vk_chain_piece q;
      // the widest first: the launch's longest chains start first
      std::stable_sort(C.inv.begin(), C.inv.end(), [](const vk_dense_item& a, const vk_dense_item& b) { return a.n > b.n; });
      q.n_items = (int)C.inv.size();
      q.n_max = q.n_items ? C.inv[0].n : 0;
      q.items = reinterpret_cast<vk_dense_item*>(put(C.inv.data(), C.inv.size() * sizeof(vk_dense_item)));
      q.qr = put_gemm(C.qr);
      q.up = put_gemm(C.up);
      q.put = put_gemm(C.put);
      st.pieces.push_back(q);
    }
    st.cp = put_gemm(S.cp);
    st.u1 = put_gemm(S.u1);
    st.u2 = put_gemm(S.u2);
    T.steps.push_back(st);
  }
  T.zw = put_gemm(zw);
  for (int k = 0; k < 2; ++k) {
    T.r_mul[k] = put_gemm(r_mul[k]);
    T.r_put[k] = put_gemm(r_put[k]);
  }
  for (size_t t = 0; t < ga.size(); ++t) {
    T.ga.push_back(put_gemm(ga[t]));
    T.gb.push_back(put_gemm(gb[t]));
  }
  // dense blocks in classes of the panel kernels' widths (a class runs at its widest block's speed)
  const int64_t cls[4] = {512, 1024, 1536, VK_TOURNEY_MIN_N};
  for (int k = 0; k < 4; ++k) {
    vk_chain_rest R;
    std::vector<vk_chain_dense> real;
    std::vector<int64_t> gr{0}, gw;
    for (const vk_chain_dense& q : dense) {
      if (q.n > cls[k] || (k > 0 && q.n <= cls[k - 1])) continue;
      real.push_back(q);
      gw.push_back(q.w - L.cb_a);
      gr.push_back(gr.back() + q.n);
    }
    if (real.empty()) continue;
    R.rows = gr;
    R.d_rows = reinterpret_cast<int64_t*>(put(gr.data(), gr.size() * 8));
    R.d_woff = reinterpret_cast<int64_t*>(put(gw.data(), gw.size() * 8));
    R.d_real = reinterpret_cast<vk_chain_dense*>(put(real.data(), real.size() * sizeof(vk_chain_dense)));
    T.rest.push_back(R);
  }
  if (!ok) return false;
  T.active = true;
  return true;
}

vk_csr vk_chain_J(const vk_level& L) {
  vk_csr A = L.J;
  A.val = L.chain.jval - L.cb_e0;
  return A;
}

static hipError_t gemm_list(hipStream_t s, const vk_gemm_list& l) {
  constexpr int per_launch = 32768;  // a grid's y goes to 65 536; thousands of blocks have more products a step
  for (int i = 0; i < l.count; i += per_launch) {
    chain_gemm_kernel<<<dim3((unsigned)l.tiles, (unsigned)std::min(per_launch, l.count - i)), 256, 0, s>>>(l.items + i);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// *flag = 0 where every chained block's inverse is within `limit` (T.rs is zero)
static hipError_t chain_check(hipStream_t s, const vk_level& L, double limit, int32_t* flag) {
  const vk_chain& T = L.chain;
  const int64_t nr = T.rows - T.first;
  hipError_t e;
  const unsigned g = (unsigned)((nr + 3) / 4);
  chain_probe_kernel<<<g, 256, 0, s>>>(T.first, T.rows, L.J.row_ptr, L.J.col, T.jval, L.cb_e0, T.cb, T.blocks, T.w, T.wa);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  chain_error_kernel<<<g, 256, 0, s>>>(T.first, T.rows, T.cb, T.blocks, T.rmap, T.cmap, T.w, T.wa, T.rs);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  chain_judge_kernel<<<1, 256, 0, s>>>(T.n_chained, T.rs, limit, T.bad, flag);
  return hipGetLastError();
}

hipError_t launch_chain_invert(hipStream_t s, const vk_level& L, int32_t* status, int32_t* scratch, int32_t* flag) {
  const vk_chain& T = L.chain;
  hipError_t e;
  auto virtual_level = [&](double* base, const std::vector<int64_t>& rows, int64_t* d_rows, int64_t* d_woff) {
    vk_level V;
    V.cb_rows = rows;
    for (size_t b = 0; b + 1 < rows.size(); ++b) V.cb_max = std::max(V.cb_max, rows[b + 1] - rows[b]);
    V.d_cb_rows = d_rows;
    V.d_cb_woff = d_woff;
    V.cb_a = V.cb_W = base;
    V.cb_q = L.cb_q;
    V.cb_used = L.cb_used;
    V.cb_gi = L.cb_gi;
    V.cb_go = L.cb_go;
    return V;
  };
  if ((e = launch_fill(s, T.n_zero, 0.0, T.zero)) != hipSuccess) return e;
  for (size_t i = 0; i < T.dense.size();) {  // runs of adjacent dense blocks
    size_t j = i;
    int64_t len = 0;
    for (; j < T.dense.size() && T.dense[j].w == T.dense[i].w + len; ++j) len += T.dense[j].n * T.dense[j].n;
    if ((e = launch_fill(s, len, 0.0, T.dense[i].w)) != hipSuccess) return e;
    i = j;
  }
  if ((e = launch_fill_i32(s, 1, INT_MAX, scratch)) != hipSuccess) return e;
  chain_gather_kernel<<<(unsigned)((T.rows - T.first + 3) / 4), 256, 0, s>>>(T.first, T.rows, L.J.row_ptr, L.J.col, L.J.val, T.cb, T.ri,
                                                                   T.blocks, T.d_dense, L.cb_e0, T.jval, status);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (const vk_chain_step& S : T.steps) {
    for (const vk_chain_piece& C : S.pieces) {
      // a chain block without a pivot only marks `scratch`: the check decides
      if ((e = launch_invert_items(s, C.n_items, C.n_max, C.items, scratch)) != hipSuccess) return e;
      if ((e = gemm_list(s, C.qr)) != hipSuccess) return e;
      if ((e = gemm_list(s, C.up)) != hipSuccess) return e;
      if ((e = gemm_list(s, C.put)) != hipSuccess) return e;
    }
    if ((e = gemm_list(s, S.cp)) != hipSuccess) return e;
    if ((e = gemm_list(s, S.u1)) != hipSuccess) return e;
    if ((e = gemm_list(s, S.u2)) != hipSuccess) return e;
  }
  if ((e = gemm_list(s, T.zw)) != hipSuccess) return e;
  for (size_t t = 0; t < T.ga.size(); ++t) {
    if ((e = gemm_list(s, T.ga[t])) != hipSuccess) return e;
    if ((e = gemm_list(s, T.gb[t])) != hipSuccess) return e;
  }
  for (const vk_chain_rest& R : T.rest) {
    const vk_level V = virtual_level(L.cb_a, R.rows, R.d_rows, R.d_woff);
    if ((e = launch_block_invert_dense_any(s, V, status)) != hipSuccess) return e;
    chain_dense_maps_kernel<<<dim3((unsigned)((V.cb_max + 255) / 256), (unsigned)(R.rows.size() - 1)), 256, 0, s>>>(
        R.d_real, R.d_rows, L.cb_q, T.rmap, T.cmap);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return chain_check(s, L, CHECK_LIMIT, flag);
}

hipError_t launch_chain_refine(hipStream_t s, const vk_level& L, int32_t* flag) {
  const vk_chain& T = L.chain;
  hipError_t e;
  if ((e = launch_fill(s, 2 * (int64_t)T.n_chained, 0.0, reinterpret_cast<double*>(T.rs))) != hipSuccess) return e;
  chain_defect_kernel<<<(unsigned)(T.rows - T.first), 256, 0, s>>>(T.first, L.J.row_ptr, L.J.col, T.jval, L.cb_e0, T.cb, T.blocks,
                                                                T.rmap, T.cmap, T.bad);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int k = 0; k < 2; ++k) {
    if ((e = gemm_list(s, T.r_mul[k])) != hipSuccess) return e;
    if ((e = gemm_list(s, T.r_put[k])) != hipSuccess) return e;
  }
  return chain_check(s, L, REFINED_LIMIT, flag);
}
