// Planning and dispatch of the weight-streaming projection (kernel in gemm_mfma_kernel.h).
#include "gemm_mfma_kernel.h"

namespace firp {

// the kernel for more than 128 rows (gemm_tall.hip); takes K % 64 == 0 only
void launch_gemm_tall(const bf16* x, int ldx, int rows, const void* w_packed, int n, int K, float* out, int ld,
                      size_t part_stride, const GemmPlan& plan, hipStream_t s);
void launch_gemm_tall_swiglu(const bf16* x, int ldx, int rows, const void* w_packed, int F, int K, const RowScale& rs,
                             const Act& act, const GemmPlan& p, hipStream_t s);
static bool tall_shape(int rows, int K) { return rows > 128 && K % 64 == 0; }

bool gemm_mfma_supported(int rows, int n, int K) {
  return rows >= 1 && n >= 4 && n % 4 == 0 && K >= 8 && K % 8 == 0;
}

// activation tiles of one pass of the streaming kernel: up to 8 (128 rows)
static int pick_nt(int rows) {
  int nt = (std::min(rows, 128) + 15) / 16;
  const int nts[] = {1, 2, 3, 4, 5, 6, 8};
  for (int c : nts)
    if (c >= nt) return c;
  return 8;
}


GemmPlan gemm_mfma_plan_ex(int rows, int n, int K, int S, int nw) {
  GemmPlan p{};
  p.nt = pick_nt(rows);
  p.nw = nw;
  int tiles = (n + nw * 32 - 1) / (nw * 32);
  int stages = (K + KC - 1) / KC;
  int s_eff = std::max(1, std::min(S, stages));
  int per = (stages + s_eff - 1) / s_eff;
  p.S = S;  // splits past the end of K find no stage and leave zeros
  p.k_per = per * KC;
  p.grid = tiles * p.S;
  p.xt = tall_shape(rows, K) && (nw == 8 || nw == 6) ? (rows <= 192 ? 3 : 4) : 0;
  p.row_block = p.xt ? 256 : 128;
  return p;
}

// The plan of the kernel for more than 128 rows: tile (32 nw rows of W x 64 xt rows of X) and split
// factor by the time of its fullest CU, in microseconds:
//   rounds x stages per workgroup x time of a stage   one workgroup per CU (they fill its registers), so
//                                    the grid runs in whole rounds of 256; a 256 x 256 stage takes 2.6
//                                    (two thirds of the matrix units' nominal rate), the smaller tiles as much
//                                    longer than their share of it as the constants say, and with one row block
//                                    none is faster than its weights arrive from HBM (2.2 for 256 rows)
//   + 6                              launch, first loads, last stores
//   + the partial sums written at 5 and read by the consumer at 4 TB/s
// The constants come from launches measured over (nw, xt, S) at the LLaMA-2 7B, 13B and 34B shapes with
// 160 to 2048 rows.
// More than 320 rows fill the chip without splitting K, but one fp32 accumulator over all of K rounds more
// often than the sums of a split: K is cut at least as often as for 128 rows (`min_split`).  Without
// that the rms logit error of the 13B shape behind a prompt of 1024 tokens went from 2.01e-3 to 2.32e-3 of a
// standard deviation.  It costs that prompt 45.2 -> 55.2 ms, one of 8192 tokens at the 7B shape 212 -> 255.
static GemmPlan tall_plan(int rows, int n, int K, int force_split, int min_split) {
  const int stages = K / KC;
  struct Tile { int nw, xt; double us; };
  const Tile tile[] = {{8, 4, 2.6}, {6, 4, 2.15}, {8, 3, 1.93}, {6, 3, 1.75}, {6, 5, 2.55}};
  GemmPlan best{};
  double best_us = -1.0;
  bool best_busy = false;
  for (const Tile& t : tile) {
    const int tiles = (n + 32 * t.nw - 1) / (32 * t.nw), blocks = (rows + 64 * t.xt - 1) / (64 * t.xt);
    if (rows <= 256 && blocks > 1) continue;   // one pass over W
    const double stage_us = blocks == 1 ? std::max(t.us, 0.275 * t.nw) : t.us;
    const int s_lo = force_split > 0 ? force_split : min_split, s_hi = force_split > 0 ? force_split : 16;
    for (int S = s_lo; S <= s_hi; ++S) {
      if (force_split <= 0 && S > s_lo && stages / S < 4) break;
      const long wgs = (long)tiles * blocks * S, rounds = (wgs + 255) / 256;
      if (force_split <= 0 && S > s_lo && rounds > 1) break;   // more splits than fill the chip only add partial sums
      const int per = (stages + std::min(S, stages) - 1) / std::min(S, stages);
      const bool busy = wgs >= 170;   // two thirds of the CUs: fewer cannot pull the weights at the chip's rate
      if (best_us >= 0.0 && best_busy && !busy) continue;
      const double us = rounds * per * stage_us + 6.0 + (double)S * rows * n * 4.0 * (1 / 5.0e6 + 1 / 4.0e6);
      if (best_us < 0.0 || (busy && !best_busy) || us < best_us - 1e-9) {
        best_us = us;
        best_busy = busy;
        best = gemm_mfma_plan_ex(rows, n, K, S, t.nw);
        best.xt = t.xt;
      }
    }
  }
  return best;
}

// A CU moves data at a capped rate however many workgroups it holds (its vector cache keeps only
// so many lines in flight), so a launch is as fast as its busiest CU: the plan puts at most one
// workgroup on each of the 256 CUs and picks waves per workgroup (nw: 32 rows of W each) and
// split factor S by a model of that CU's time, in units of one 4 KiB stage of one wave's W:
//   stages per workgroup x (nw + 0.6 x activation tiles)   W from HBM, the X tile (4 KiB per 16 rows
//                                                          and stage) from L2 at 0.6 of that cost
//   + rows x nw / 32                                       the partial sums it writes
//   + 6 per stage short of 8                               a pipeline that never fills
//   + S x rows x n / 2^18                                  the consumer kernel reading the partial sums
// The constants come from launch times measured over (S, nw) at the LLaMA-2 7B and 13B shapes
// (e.g. 5120 x 5120 at 67 rows: 8 x 5 waves; 4096 x 11008: 16 x 8).  Few waves with many
// activation tiles are excluded: two waves cannot keep a CU's memory pipeline busy.
static double plan_cost(int rows, int n, int K, int S, int nw, int nt) {
  const int stages = (K + KC - 1) / KC;
  const int per = (stages + S - 1) / S;
  const int r = std::min(rows, 128);
  return per * (nw + 0.6 * nt) + r * nw / 32.0 + 6.0 * std::max(0, 8 - per)
         + (double)S * r * n / 262144.0;   // and the consumer reads every partial sum back (spread over 256 CUs)
}

GemmPlan gemm_mfma_plan(int rows, int n, int K, int force_split) {
  const int stages = (K + KC - 1) / KC;
  const int n_cu = 256;
  if (tall_shape(rows, K)) return tall_plan(rows, n, K, force_split, rows > 320 ? gemm_mfma_plan(128, n, K, 0).S : 1);
  const int nt = pick_nt(rows);
  const int nw_hi = 8, nw_lo = std::min(4, std::max(2, nt));
  int best_nw = nw_hi, best_S = std::max(1, force_split);
  double best = -1.0;
  for (int nw = nw_hi; nw >= nw_lo; --nw) {
    int tiles = (n + nw * 32 - 1) / (nw * 32);
    int s_lo = force_split > 0 ? force_split : 1, s_hi = force_split > 0 ? force_split : 16;
    for (int S = s_lo; S <= s_hi; ++S) {
      if (force_split <= 0 && S > 1 && stages / S < 4) break;
      int grid = tiles * S;
      if (grid > n_cu && !(nw == nw_hi && S == s_lo)) continue;   // (the fallback: several rounds)
      double cost = (double)((grid + n_cu - 1) / n_cu) * plan_cost(rows, n, K, S, nw, nt);
      if (best < 0.0 || cost < best - 1e-9) {
        best = cost;
        best_nw = nw;
        best_S = S;
      }
    }
  }
  return gemm_mfma_plan_ex(rows, n, K, best_S, best_nw);
}

size_t gemm_packed_bytes(int n, int K) {
  return (size_t)((n + 15) / 16) * (size_t)(((K + KC - 1) / KC) * 2) * 1024;
}

// One thread per 16-byte piece of the fragment-major copy.
__global__ void k_pack_weights(WSeg src, int n, int K, int kp32, size_t pieces, uint4* __restrict__ dst) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= pieces) return;
  const int lane = (int)(idx & 63);
  const size_t frag = idx >> 6;
  const int t16 = (int)(frag / kp32), ks = (int)(frag % kp32);
  const int row = t16 * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
  union {
    uint4 v;
    unsigned short e[8];
  } u;
  u.v = make_uint4(0, 0, 0, 0);
  if (row < n && k < K) {
    const bf16* r = row < src.n0 ? src.w0 + (size_t)row * K
                    : row < src.n0 + src.n1 ? src.w1 + (size_t)(row - src.n0) * K
                                            : src.w2 + (size_t)(row - src.n0 - src.n1) * K;
    if (k + 8 <= K && (K & 7) == 0) {
      u.v = *(const uint4*)(r + k);
    } else {
      for (int i = 0; i < 8 && k + i < K; ++i) u.e[i] = r[k + i].v;
    }
  }
  dst[idx] = u.v;
}

void launch_pack_weights(const WSeg& src, int n, int K, void* dst, hipStream_t s) {
  const int kp32 = ((K + KC - 1) / KC) * 2;
  const size_t pieces = gemm_packed_bytes(n, K) / 16;
  const unsigned blocks = (unsigned)((pieces + 255) / 256);
  hipLaunchKernelGGL(k_pack_weights, dim3(blocks), dim3(256), 0, s, src, n, K, kp32, pieces, (uint4*)dst);
}

bool gemm_swiglu_fused(int rows, int F, int K) {
  if (!tall_shape(rows, K) || F % 16) return false;
  return gemm_mfma_plan(rows, 2 * F, K, 0).S == 1;
}

void launch_gemm_swiglu(const Act& x, const void* w_packed, int rows, int F, int K, const RowScale& rs, const Act& act,
                        hipStream_t s) {
  launch_gemm_tall_swiglu(x.pl, x.row, rows, w_packed, F, K, rs, act, gemm_mfma_plan(rows, 2 * F, K, 0), s);
}

void launch_gemm_mfma(const Act& x, const void* w_packed, float* out, int ld, size_t part_stride, int rows, int n,
                      int K, const GemmPlan& plan, hipStream_t s) {
  const char* w = (const char*)w_packed;
  const int ldx = x.row;
  if (plan.xt) {
    launch_gemm_tall(x.pl, ldx, rows, w, n, K, out, ld, part_stride, plan, s);
    return;
  }
  // more rows than one pass takes: row blocks (W is streamed once per block)
  const int block = plan.row_block;
  for (int r0 = 0; r0 < rows; r0 += block) {
    int rb = std::min(block, rows - r0);
    GemmPlan p = plan;
    p.nt = pick_nt(rb);
    const bf16* xr = x.pl + (size_t)r0 * ldx;
    float* o = out + (size_t)r0 * ld;
    switch (p.nw) {
      case 2: launch_gemm_mfma_nw<2>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      case 3: launch_gemm_mfma_nw<3>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      case 4: launch_gemm_mfma_nw<4>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      case 5: launch_gemm_mfma_nw<5>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      case 6: launch_gemm_mfma_nw<6>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      case 7: launch_gemm_mfma_nw<7>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
      default: launch_gemm_mfma_nw<8>(xr, ldx, rb, w, n, K, o, ld, part_stride, p, s); break;
    }
  }
}

}  // namespace firp
