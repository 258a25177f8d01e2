// Draft map kernels (descriptor equation; Definition 3.1).
//
//   draft_pool     one workgroup per (block, head, Q or K): mean (float64 sum /
//                  n_a) and channel max over the valid tokens, plus the per-head
//                  max|Q|, max|K| used by the NVFP4 tensor scales.
//   draft_logits   128x160 tiles of Qbar Kbar^T / sqrt d or Qmax Kmax^T / sqrt d
//                  on the float64 matrix cores (16x16x4 MFMA).
//   draft_rows     short rows: logits and softmaxes of 16 rows in one workgroup.
//   draft_softmax  one wave per row: the two row softmaxes (max subtracted)
//                  mixed with weight lambda, rounded once to float32.
#include "common.hpp"
#include "launch.hpp"

namespace da2 {

// One workgroup per (block, head, Q or K). The block's slots are read with
// coalesced 16-byte loads into an LDS tile (padding rows repeat the last valid
// row); thread
// (channel pair p, row group q) then reduces rows [q RPQ, (q + 1) RPQ) of its
// two channels: float64 sums, float32 maxima over the valid rows and max |x|
// (written per block; the logits launch reduces it per head, which avoids
// hundreds of workgroups contending for one atomic address).
// The row groups are combined through LDS in order. Sums of bf16 values in
// float64 are exact, so for bf16 inputs the order of the additions does not
// change the mean.
template <int D, typename T>
__global__ __launch_bounds__(256) void draft_pool_kernel(DraftArgs args) {
  constexpr int EPC = 16 / sizeof(T);    // elements per 16-byte load
  constexpr int CPR = D / EPC;           // loads per slot row
  constexpr int LPT = kCap * CPR / 256;  // loads per thread
  constexpr int CP = D / 2;              // channel pairs
  constexpr int RQ = 256 / CP;           // row groups of the reduction
  constexpr int RPQ = kCap / RQ;         // rows per group
  __shared__ __align__(16) T tile[kCap * D];
  // the per-group partial sums and maxima reuse the tile once it is read
  static_assert(RQ * D * (sizeof(double) + sizeof(float)) <= sizeof(T) * kCap * D, "partials fit in the tile");
  double (*s_sum)[D] = reinterpret_cast<double (*)[D]>(tile);
  float (*s_max)[D] = reinterpret_cast<float (*)[D]>(reinterpret_cast<char*>(tile) + RQ * D * sizeof(double));
  __shared__ float s_amax[4];
  const int a = blockIdx.x, bh = blockIdx.y, which = blockIdx.z;
  const int b = bh / args.H, h = bh % args.H, tid = threadIdx.x;
  const Layout L = layout_view(args.layout, args.R, args.Npad);
  const int n = L.n_a[a];
  const int32_t* slots = L.slot2tok + (int64_t)a * kCap;
  const T* X = static_cast<const T*>(which == 0 ? args.Q : args.K) + (int64_t)b * args.sb + (int64_t)h * args.sh;
  // token indices first, then the data loads, all unconditional so that they
  // overlap: padding slots read the last valid row again (a copy changes no
  // maximum; the sums skip those rows)
  int tok[LPT];
#pragma unroll
  for (int k = 0; k < LPT; ++k) tok[k] = slots[min((tid + 256 * k) / CPR, n - 1)];
  uint4 v[LPT];
#pragma unroll
  for (int k = 0; k < LPT; ++k) {
    const int cc = (tid + 256 * k) % CPR;
    v[k] = *reinterpret_cast<const uint4*>(X + (int64_t)tok[k] * args.sn + cc * EPC);
  }
#pragma unroll
  for (int k = 0; k < LPT; ++k) reinterpret_cast<uint4*>(tile)[tid + 256 * k] = v[k];
  __syncthreads();
  const int p = tid % CP, q = tid / CP;
  double s0 = 0.0, s1 = 0.0;
  float m0 = -INFINITY, m1 = -INFINITY, am = 0.0f;
  // A full block needs no test per row: 64 compares and selects of the 340
  // vector instructions (R = 1,260 x 40 heads, bound by its reads: 333 us
  // with them in every block, 320 without).
  auto reduce = [&]<bool FULL>() {
#pragma unroll
    for (int r = 0; r < RPQ; ++r) {
      const int s = q * RPQ + r;
      const float2 f = tile_pair(tile, D, s, p);
      if (FULL || s < n) {
        s0 += (double)f.x;
        s1 += (double)f.y;
      }
      m0 = fmaxf(m0, f.x);
      m1 = fmaxf(m1, f.y);
      am = fmaxf(am, fmaxf(fabsf(f.x), fabsf(f.y)));
    }
  };
  if (n == kCap)
    reduce.template operator()<true>();
  else
    reduce.template operator()<false>();
  __syncthreads();  // every thread is done with the tile
  s_sum[q][2 * p] = s0;
  s_sum[q][2 * p + 1] = s1;
  s_max[q][2 * p] = m0;
  s_max[q][2 * p + 1] = m1;
  am = wave_max(am);
  if ((tid & 63) == 0) s_amax[tid >> 6] = am;
  __syncthreads();
  if (tid < D) {
    double t = s_sum[0][tid];
    float m = s_max[0][tid];
#pragma unroll
    for (int g = 1; g < RQ; ++g) {
      t += s_sum[g][tid];
      m = fmaxf(m, s_max[g][tid]);
    }
    const int64_t o = ((int64_t)bh * args.R + a) * D + tid;
    (which == 0 ? args.Qbar : args.Kbar)[o] = t / (double)n;
    (which == 0 ? args.Qmax : args.Kmax)[o] = (double)m;
  }
  if (tid == 0) {
    const float m = fmaxf(fmaxf(s_amax[0], s_amax[1]), fmaxf(s_amax[2], s_amax[3]));
    args.blkmax[((int64_t)which * args.B * args.H + bh) * args.R + a] = m;
  }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One 128x160 logit tile of one branch (z = 2*head + branch) on the
// float64 matrix cores: each wave owns a 64x80 quarter as 4x5 MFMA tiles of
// 16x16x4, so every query value loaded feeds five MFMAs and every key value
// four. (On R = 588 this makes 1,920 waves, which two waves per SIMD take in
// one round; 64x64 quarters made 2,400 and a thin second round.) The
// reduction over channels may visit them in any order as long as both
// operands agree: lane group q = lane/16 of k-step 2t+h reads channel
// 8t + 2q + h, so one 16-byte load per operand tile feeds two k-steps. The
// loads run one group of 8 channels ahead of the MFMAs, and consecutive MFMAs
// update different accumulators. Operand rows are addressed as 32-bit byte
// offsets from the branch's base (one VGPR each), which keeps the kernel
// within 256 VGPRs. Rows and columns beyond R read row R-1 and are not stored.
// Each XCD takes whole branches: the descriptors of one (2.6 MB at R = 1,260)
// fit its L2, while tiles dealt round-robin had every XCD read every branch
// (L2 hit rate 48%). With the epilogue's multiplication by 1/sqrt(d) instead
// of a float64 division per logit: 690 -> 660 us at R = 1,260, 40 heads; with
// quarters inside the matrix stored without bounds checks 627 us (MFMA busy
// 0.75; all of it busy would be 470).
constexpr int kLogitTile = 128;  // rows per workgroup
constexpr int kLogitCols = 160;  // columns per workgroup
template <int D>
__global__ __launch_bounds__(256) void draft_logits_kernel(DraftArgs args) {
  constexpr int d = D, NI = 4, NJ = 5;
  const int R = args.R;
  // XCD-aware mapping: workgroup b runs on XCD b mod 8 and takes the next tile
  // of that XCD's contiguous segment of the tiles (z-major, then rows)
  const int ntc = (R + kLogitCols - 1) / kLogitCols, tiles = ntc * ((R + kLogitTile - 1) / kLogitTile);
  const int n_items = 2 * args.B * args.H * tiles, seg = (n_items + 7) >> 3;
  const int item = (int)(blockIdx.x & 7) * seg + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;
  const int z = item / tiles, tile = item - z * tiles, ty = tile / ntc, tx = tile - ty * ntc;
  const int bh = z >> 1, br = z & 1;
  const double* Qs = (br == 0 ? args.Qbar : args.Qmax) + (int64_t)bh * R * d;
  const double* Ks = (br == 0 ? args.Kbar : args.Kmax) + (int64_t)bh * R * d;
  double* out = (br == 0 ? args.S1 : args.S2) + (int64_t)bh * R * R;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
  const int r0 = ty * kLogitTile + (wave >> 1) * 64, c0 = tx * kLogitCols + (wave & 1) * 80;
  // byte offsets of each lane's operand rows from the branch's base (one VGPR each)
  uint32_t oa[NI], ob[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) oa[i] = (uint32_t)(min(r0 + 16 * i + li, R - 1) * d + 2 * q) * 8u;
#pragma unroll
  for (int j = 0; j < NJ; ++j) ob[j] = (uint32_t)(min(c0 + 16 * j + li, R - 1) * d + 2 * q) * 8u;
  auto lda = [&](int i, int t) {
    return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(Qs) + oa[i] + 64 * t);
  };
  auto ldb = [&](int j, int t) {
    return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(Ks) + ob[j] + 64 * t);
  };
  f64x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  double2 a[2][NI], b[2][NJ];  // [buffer][tile]
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    a[0][i] = lda(i, 0);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) b[0][j] = ldb(j, 0);
#pragma unroll
  for (int t = 0; t < d / 8; ++t) {
    const int cur = t & 1;
    if (t + 1 < d / 8) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        a[cur ^ 1][i] = lda(i, t + 1);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[cur ^ 1][j] = ldb(j, t + 1);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[cur][i].x, b[cur][j].x, acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[cur][i].y, b[cur][j].y, acc[i][j], 0, 0, 0);
  }
  // the first tile's workgroup of each branch also reduces the per-block max |Q|
  // (branch 0) or max |K| (branch 1) of its head into the statistics entry
  if (tile == 0) {
    __shared__ float s_red[4];
    const float* bm = args.blkmax + ((int64_t)br * args.B * args.H + bh) * R;
    float m = 0.0f;
    for (int i = threadIdx.x; i < R; i += 256) m = fmaxf(m, bm[i]);
    m = wave_max(m);
    if (lane == 0) s_red[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0)
      args.stats[(int64_t)bh * (4 + d) + br] =
          __float_as_uint(fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3])));
  }
  // accumulator element e of lane l: row l/16 + 4e, column l%16
  const double rsqd = 1.0 / sqrt((double)d);
  auto store = [&]<bool INSIDE>() {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = r0 + 16 * i + q + 4 * e, col = c0 + li;
        double* o = out + (int64_t)row * R + col;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (INSIDE || (row < R && col + 16 * j < R)) o[16 * j] = acc[i][j][e] * rsqd;
      }
  };
  if (r0 + 64 <= R && c0 + 80 <= R)  // the wave's quarter needs no bounds checks
    store.template operator()<true>();
  else
    store.template operator()<false>();
}

__device__ inline double wave_max_f64(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// e^x for x <= 0 in float64: Cody-Waite range reduction x = k ln2 + r with
// |r| <= ln2/2 (two multiply-adds, ln2 split into its nearest double and the
// remainder), then the Taylor series of e^r to degree 13 in Horner form (the
// truncation error is below 5e-18 relative on that interval) and ldexp(., k).
// The coefficients are 1/n! rounded to the nearest double; they live in
// constant memory, so the multiply-adds read them from scalar registers
// instead of copying each into a vector register first. Inputs below -746
// give 0, like e^x itself in float64; a NaN gives NaN.
__constant__ double kExpTaylor[14] = {1.0,
                                      1.0,
                                      0.5,
                                      0.16666666666666666,
                                      0.041666666666666664,
                                      0.008333333333333333,
                                      0.001388888888888889,
                                      0.0001984126984126984,
                                      2.48015873015873e-05,
                                      2.7557319223985893e-06,
                                      2.755731922398589e-07,
                                      2.505210838544172e-08,
                                      2.08767569878681e-09,
                                      1.6059043836821613e-10};
__device__ inline double exp_neg(double x) {
  constexpr double kLog2e = 1.4426950408889634, kLn2Hi = 0.6931471805599453, kLn2Lo = 2.3190468138462996e-17;
  x = x < -746.0 ? -746.0 : x;  // (a NaN stays NaN)
  const double k = rint(x * kLog2e);
  double r = fma(-k, kLn2Hi, x);
  r = fma(-k, kLn2Lo, r);
  double p = kExpTaylor[13];
#pragma unroll
  for (int n = 12; n >= 0; --n) p = fma(p, r, kExpTaylor[n]);
  return ldexp(p, static_cast<int>(k));
}

// One wave per row of A (four rows per workgroup): the two row softmaxes (max
// subtracted) mixed with weight lambda, rounded once to float32. Rows of up to
// 64 KMAX entries keep their logits and exponentials in registers (one exp per
// entry and branch); longer rows take the three-pass form below.
template <int KMAX>
__global__ __launch_bounds__(256) void draft_softmax_reg_kernel(DraftArgs args) {
  const int R = args.R, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= (int64_t)args.B * args.H * R) return;
  const double* s1 = args.S1 + row * R;
  const double* s2 = args.S2 + row * R;
  double e1[KMAX], e2[KMAX];
  double m1 = -INFINITY, m2 = -INFINITY;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const int i = lane + 64 * k;
    e1[k] = i < R ? s1[i] : -INFINITY;
    e2[k] = i < R ? s2[i] : -INFINITY;
    m1 = fmax(m1, e1[k]);
    m2 = fmax(m2, e2[k]);
  }
  m1 = wave_max_f64(m1);
  m2 = wave_max_f64(m2);
  double z1 = 0.0, z2 = 0.0;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const bool in = lane + 64 * k < R;
    e1[k] = in ? exp_neg(e1[k] - m1) : 0.0;
    e2[k] = in ? exp_neg(e2[k] - m2) : 0.0;
    z1 += e1[k];
    z2 += e2[k];
  }
  z1 = wave_sum_f64(z1);
  z2 = wave_sum_f64(z2);
  const double lam = args.lambda;
  // both normalizations and the mixing weights folded into one factor per
  // branch (float64; A is rounded once, to float32, at the end)
  const double r1 = (1.0 - lam) / z1, r2 = lam / z2;
  float* out = args.A + row * R;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const int i = lane + 64 * k;
    if (i < R) out[i] = (float)(e1[k] * r1 + e2[k] * r2);
  }
}

__global__ __launch_bounds__(256) void draft_softmax_kernel(DraftArgs args) {
  const int R = args.R, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= (int64_t)args.B * args.H * R) return;
  const double* s1 = args.S1 + row * R;
  const double* s2 = args.S2 + row * R;
  double m1 = -INFINITY, m2 = -INFINITY;
  for (int i = lane; i < R; i += 64) {
    m1 = fmax(m1, s1[i]);
    m2 = fmax(m2, s2[i]);
  }
  m1 = wave_max_f64(m1);
  m2 = wave_max_f64(m2);
  double z1 = 0.0, z2 = 0.0;
  for (int i = lane; i < R; i += 64) {
    z1 += exp_neg(s1[i] - m1);
    z2 += exp_neg(s2[i] - m2);
  }
  z1 = wave_sum_f64(z1);
  z2 = wave_sum_f64(z2);
  const double lam = args.lambda;
  const double r1 = (1.0 - lam) / z1, r2 = lam / z2;
  float* out = args.A + row * R;
  for (int i = lane; i < R; i += 64) out[i] = (float)(exp_neg(s1[i] - m1) * r1 + exp_neg(s2[i] - m2) * r2);
}

// Short rows (R <= 64 KT): one workgroup owns 16 rows of a head, both branches
// and every column, so the row softmaxes follow in the same launch and read the
// logits from registers (they are stored for the workspace only). Wave w holds
// the column tiles w, w + 4, ... (KT of them); row statistics are reduced over
// the 16 lanes of an accumulator row, then over the waves through LDS. At these
// sizes a 128x160 tile per workgroup leaves the chip idle and its one wave round
// is the time: 12.8 + 4 us for the two launches at R = 8 x 2 heads, 14 + 5 us at
// R = 70 x 12 heads. Beyond 256 columns a wave would need more than 64
// accumulator registers, every key operand still feeds one product only, and
// the tiled kernel wins; use_rows() has the limits on the number of workgroups.
template <int D, int KT>
__global__ __launch_bounds__(256) void draft_rows_kernel(DraftArgs args) {
  constexpr int d = D, NT = d / 8;
  constexpr int PF = KT <= 2 ? 4 : 2;  // channel groups in flight
  const int R = args.R, bh = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
  const int r0 = blockIdx.x * 16;
  __shared__ double s_part[2][4][16];
  const int64_t base = (int64_t)bh * R * d;
  const double* Qs[2] = {args.Qbar + base, args.Qmax + base};
  const double* Ks[2] = {args.Kbar + base, args.Kmax + base};
  // 32-bit element offsets of each lane's operand rows
  const int oa = min(r0 + li, R - 1) * d + 2 * q;
  int ob[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) ob[k] = min(16 * (wave + 4 * k) + li, R - 1) * d + 2 * q;
  f64x4 acc[2][KT];
  double2 a[PF][2], b[PF][2][KT];
#pragma unroll
  for (int br = 0; br < 2; ++br)
#pragma unroll
    for (int k = 0; k < KT; ++k) acc[br][k] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto load = [&](int t) {
#pragma unroll
    for (int br = 0; br < 2; ++br) {
      a[t % PF][br] = *reinterpret_cast<const double2*>(Qs[br] + oa + 8 * t);
#pragma unroll
      for (int k = 0; k < KT; ++k) b[t % PF][br][k] = *reinterpret_cast<const double2*>(Ks[br] + ob[k] + 8 * t);
    }
  };
#pragma unroll
  for (int t = 0; t < PF; ++t) load(t);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
      for (int k = 0; k < KT; ++k)
        acc[br][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t % PF][br].x, b[t % PF][br][k].x, acc[br][k], 0, 0, 0);
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
      for (int k = 0; k < KT; ++k)
        acc[br][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t % PF][br].y, b[t % PF][br][k].y, acc[br][k], 0, 0, 0);
    if (t + PF < NT) load(t + PF);
  }
  // accumulator element e of lane l: row l/16 + 4e, column l%16
  const double rsqd = 1.0 / sqrt((double)d);
  // combines v[br][e] over the row's 16 lanes and the four waves
  auto row_reduce = [&](double (&v)[2][4], auto op) {
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        for (int o = 8; o > 0; o >>= 1) v[br][e] = op(v[br][e], __shfl_xor(v[br][e], o, 64));
        if (li == 0) s_part[br][wave][q + 4 * e] = v[br][e];
      }
    __syncthreads();
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = q + 4 * e;
        v[br][e] = op(op(s_part[br][0][row], s_part[br][1][row]), op(s_part[br][2][row], s_part[br][3][row]));
      }
    __syncthreads();
  };
  double m[2][4], z[2][4];
#pragma unroll
  for (int br = 0; br < 2; ++br) {
    // The workspace holds the logits of every row length. No kernel reads them
    // here, so they need not stay in L2: R = 128 x 60 heads, d = 128, 76.7 us with
    // plain stores, 73.6 so, 72.2 without any; 200 x 19, d = 64, 33.4, 32.3, 31.0.
    double* S = (br == 0 ? args.S1 : args.S2) + (int64_t)bh * R * R;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      m[br][e] = -INFINITY;
      const int row = r0 + q + 4 * e;
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        const int col = 16 * (wave + 4 * k) + li;
        const bool in = col < R;
        acc[br][k][e] = in ? acc[br][k][e] * rsqd : -INFINITY;
        if (in && row < R) __builtin_nontemporal_store((double)acc[br][k][e], S + row * R + col);
        m[br][e] = fmax(m[br][e], acc[br][k][e]);
      }
    }
  }
  row_reduce(m, [](double x, double y) { return fmax(x, y); });
#pragma unroll
  for (int br = 0; br < 2; ++br)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      z[br][e] = 0.0;
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        const bool in = 16 * (wave + 4 * k) + li < R;
        acc[br][k][e] = in ? exp_neg(acc[br][k][e] - m[br][e]) : 0.0;
        z[br][e] += acc[br][k][e];
      }
    }
  row_reduce(z, [](double x, double y) { return x + y; });
  const double lam = args.lambda;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = r0 + q + 4 * e;
    const double f1 = (1.0 - lam) / z[0][e], f2 = lam / z[1][e];
    float* out = args.A + ((int64_t)bh * R + row) * R;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      const int col = 16 * (wave + 4 * k) + li;
      if (row < R && col < R) out[col] = (float)(acc[0][k][e] * f1 + acc[1][k][e] * f2);
    }
  }
  // the first workgroup of a head also reduces its per-block max |Q|, max |K|
  if (blockIdx.x == 0 && wave < 2) {
    const float* bm = args.blkmax + ((int64_t)wave * args.B * args.H + bh) * R;
    float t = 0.0f;
    for (int i = lane; i < R; i += 64) t = fmaxf(t, bm[i]);
    t = wave_max(t);
    if (lane == 0) args.stats[(int64_t)bh * (4 + d) + wave] = __float_as_uint(t);
  }
}

// Whether the short-row kernel is the faster one. Its workgroups each read all
// keys of their head, so beyond about one (KT = 4) or two of them per compute
// unit the tiled kernel's reuse of its operands wins. Whole call, tiled against
// short rows, us (d = 64 / d = 128; workgroups), short rows still with plain stores
// of the logits (up to 4% slower):
//   R = 8 x 2 heads  19.3 / 28.2, 13.6 / 13.4 (2)     R = 40 x 80  29.4 / 45.2, 21.5 / 31.5 (240)
//   R = 75 x 12      23.2 / 34.3, 17.9 / 24.2 (60)    R = 75 x 80  39.3 / 62.1, 36.0 / 56.9 (400)
//   R = 128 x 40     38.8 / 59.0, 37.2 / 58.5 (320)   R = 100 x 80 46.7 / 80.0, 47.5 / 84.9 (560)
//   R = 160 x 24     35.2 / 52.3, 31.5 / 46.7 (240)   R = 192 x 24 38.8 / 57.9, 42.9 / 66.4 (288)
//   R = 256 x 12     34.0 / 49.4, 32.5 / 48.0 (192)   R = 256 x 40 70.9 / 127.5, 73.4 / 134.3 (640)
// (R = 192 x 40, 480 workgroups: 60.4 / 100.8, 51.0 / 88.1; it stays with the
// tiled kernel, whose time the head counts around it share.) Up to 48 blocks a
// tile is mostly padding and the short rows win at every head count.
inline bool use_rows(int R, int BH) {
  const int64_t groups = (int64_t)((R + 15) / 16) * BH;
  return R <= 48 || (R <= 128 ? groups <= 512 : R <= 256 && groups <= 256);
}

template <int D>
void launch_rows(const DraftArgs& args, hipStream_t stream) {
  const dim3 grid((args.R + 15) / 16, args.B * args.H);
  if (args.R <= 64)
    hipLaunchKernelGGL((draft_rows_kernel<D, 1>), grid, dim3(256), 0, stream, args);
  else if (args.R <= 128)
    hipLaunchKernelGGL((draft_rows_kernel<D, 2>), grid, dim3(256), 0, stream, args);
  else
    hipLaunchKernelGGL((draft_rows_kernel<D, 4>), grid, dim3(256), 0, stream, args);
}

hipError_t launch_draft(const DraftArgs& args, hipStream_t stream) {
  const int BH = args.B * args.H;
  const dim3 pool_grid(args.R, BH, 2);
  if (args.d == 128) {
    if (args.dtype == DA2_BF16)
      hipLaunchKernelGGL((draft_pool_kernel<128, uint16_t>), pool_grid, dim3(256), 0, stream, args);
    else
      hipLaunchKernelGGL((draft_pool_kernel<128, float>), pool_grid, dim3(256), 0, stream, args);
  } else {
    if (args.dtype == DA2_BF16)
      hipLaunchKernelGGL((draft_pool_kernel<64, uint16_t>), pool_grid, dim3(256), 0, stream, args);
    else
      hipLaunchKernelGGL((draft_pool_kernel<64, float>), pool_grid, dim3(256), 0, stream, args);
  }
  if (use_rows(args.R, BH)) {
    if (args.d == 128)
      launch_rows<128>(args, stream);
    else
      launch_rows<64>(args, stream);
    return hipGetLastError();
  }
  const int64_t nt = (args.R + kLogitTile - 1) / kLogitTile, ntc = (args.R + kLogitCols - 1) / kLogitCols;
  const dim3 lgrid((unsigned)(8 * ((2 * BH * nt * ntc + 7) / 8)));
  if (args.d == 128)
    hipLaunchKernelGGL(draft_logits_kernel<128>, lgrid, dim3(256), 0, stream, args);
  else
    hipLaunchKernelGGL(draft_logits_kernel<64>, lgrid, dim3(256), 0, stream, args);
  const int64_t rows = (int64_t)BH * args.R;
  const dim3 sgrid((unsigned)((rows + 3) / 4));
  if (args.R <= 64 * 10)
    hipLaunchKernelGGL(draft_softmax_reg_kernel<10>, sgrid, dim3(256), 0, stream, args);
  else if (args.R <= 64 * 32)
    hipLaunchKernelGGL(draft_softmax_reg_kernel<32>, sgrid, dim3(256), 0, stream, args);
  else
    hipLaunchKernelGGL(draft_softmax_kernel, sgrid, dim3(256), 0, stream, args);
  return hipGetLastError();
}

}  // namespace da2
