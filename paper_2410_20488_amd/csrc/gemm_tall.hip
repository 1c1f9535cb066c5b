// The projection for more than 128 activation rows, any number of them in one launch.
//
//   out[s][r][c] = sum_{k in split s} X[r][k] * W[c][k],   r < rows,  c < n,  K % 64 == 0
//
// Same operands and the same result layout as the weight-streaming kernel (gemm_mfma_kernel.h):
// W in the fragment-major copy, X as interleaved hi/lo bf16 planes, split-K partial sums.  With this
// many rows a launch is bound by the matrix units (two planes: 4 * rows * n * K operations), and what
// keeps them from their rate is everything that makes a wave wait between two products.  So:
//  * a workgroup of 8 waves owns 32 MW rows of W and 64 XT rows of X: up to 256 x 256, the largest
//    tile whose accumulators (a quarter of a MiB) fit the register file with two waves per SIMD;
//  * the waves form a 2 x 4 grid: wave (wg, xg) multiplies 16 MW rows of W by 16 XT rows of X.  X has two
//    planes, so the wave tile that reads the fewest fragment bytes from LDS per product is twice as
//    tall in W as in X (128 x 64: 16 KiB per 32 columns; 64 x 128 reads 20);
//  * columns go by in half-stages of 32, one MFMA step and one 128-byte line of a row of X.  The
//    products of a half-stage are cut into four quadrants (half of the wave's W fragments x half of
//    its X fragments), taken in a snake order that changes one operand at a time, so every fragment
//    is read from LDS one whole quadrant before it is needed, into registers whose last reader
//    is the quadrant before: 16 fragments of registers hold all of it;
//  * the one barrier of a half-stage stands between its second and third quadrant: by then all of
//    its fragments are in registers, so behind the barrier the next products start at once, and the
//    fragments of the next half-stage are read while they run;
//  * X goes from global memory straight into LDS (global_load_lds, no staging registers).  One
//    instruction moves 8 rows x 128 B, whole cache lines, into 1 KiB of LDS in lane order; the lane
//    that lands at piece s of row r fetches piece s ^ (r % 8) of that row, which keeps the 128-bit
//    fragment reads of 8 consecutive rows on distinct banks without padding.  Requested behind the
//    barrier of a half-stage for the one after the next, into the buffer just read;
//  * W goes through LDS too (each fragment is used by four waves): a thread stages two 16-byte pieces
//    per half-stage in registers, two half-stages ahead of the LDS write, which is one ahead of its use;
//    in LDS a fragment keeps its 1 KiB lane order, so the reads are linear.
//
// Measured per launch at the 13B shapes (q|k|v, o, gate|up, down), sustained: 1024 rows 240, 94, 427, 207 us (the
// fastest split, which the plan takes only where it is no coarser than for 128 rows; 1.34 PFLOP/s with both planes counted), 256 rows 85, 35, 129, 72 us.  The kernel before it (one
// launch per 256 rows, two barriers per 64 columns, fragments read from LDS behind the barrier they
// waited for): 328, 157, 538, 310 us and 92, 41, 140, 79 us.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace firp {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t v) { return __builtin_bit_cast(bf16x8_t, v); }

// One wave-wide direct load: lane L's 16 bytes at base + off[L] land at LDS byte lds + 16 L.
// Written as inline assembly on purpose: the compiler would make every later LDS access wait for
// a direct load it knows of (it cannot tell the LDS buffers apart), which would drain the weight
// loads in flight with it.  The waits for these loads are therefore explicit (wait_vmcnt).
__device__ __forceinline__ void load_to_lds_16(const void* base, unsigned off, unsigned lds) {
  // (one wait state between the scalar write of M0 and the instruction that reads it: the hazard
  // the compiler pads for in its own code and cannot see inside an asm statement)
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}

// Workgroup barrier after this wave's LDS accesses have completed.  (Not __syncthreads(): no fence
// is needed beyond LDS, and the clobber keeps the compiler from moving memory accesses across.)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char*)p;
}

// Wait until at most N vector-memory loads of this wave are outstanding.  Inline assembly with a
// memory clobber so that the compiler keeps the loads written before it before it: the count is
// only right for the program order as written.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// XT: 16-row activation tiles per wave; the workgroup takes 64 * XT rows of X.
// MW: 16-row tiles of W per wave (even); the workgroup takes 32 * MW rows of W.
// `blocks` workgroups side by side take the row blocks of one tile of W, so that they share it in L2.
// GLU: W is gate|up stacked (n = 2 F), one split; every wave takes MW / 2 tiles of gate rows and the up rows of
// the same columns, and writes silu(gate) * up to `act` itself.
template <int XT, int MW, bool GLU>
__device__ __forceinline__ void gemm_tall_tile(const bf16* __restrict__ x, int ldx, int rows, const char* __restrict__ wpk,
                                               int n, int K, float* __restrict__ out, int ld_out, size_t part_stride,
                                               int S, int k_per, int tiles, int blocks, const RowScale& rs,
                                               const Act& act) {
  constexpr int XR = 64 * XT;
  constexpr int NF = 2 * MW;                      // W fragments of a half-stage
  constexpr int WH = MW / 2;                      // a wave's W fragments in two halves ...
  constexpr int XA = (XT + 1) / 2, XB = XT - XA;  // ... and its X tiles
  static_assert(MW % 2 == 0 && XT >= 2, "quadrants");
  __shared__ __attribute__((aligned(1024))) unsigned char xb[2][XR * 128];
  __shared__ __attribute__((aligned(1024))) unsigned char wb[2][NF * 1024];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wg = wave & 1, xg = wave >> 1;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  if (item >= tiles * S * blocks) return;
  const int block = item % blocks, ts = item / blocks;
  const int split = ts / tiles, tile = ts - split * tiles;
  const int row0 = block * XR;
  x += (size_t)row0 * ldx;
  out += (size_t)row0 * ld_out;
  rows = min(rows - row0, XR);
  const int k_begin = min(K, split * k_per);
  const int k_end = min(K, k_begin + k_per);
  const int nh = (k_end - k_begin) / 64 * 2;   // 32-column half-stages, an even number
  const int r16 = lane & 15, kb = lane >> 4;

  // W: this thread stages fragments wave and wave + 8 of a half-stage (with 12 fragments the waves 4..7
  // repeat fragment 11: every wave issues the same two loads, and the repeated LDS writes store the
  // same bytes).  Wave-uniform bases, one per-lane offset.
  const int kp32 = (K / 64) * 2;
  const int n16 = (n + 15) >> 4;
  const char* wsrc[2];
  int wdst[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int f = min(wave_u + 8 * i, NF - 1);
    const int fw = f / MW, fi = f % MW;   // the wave column that multiplies it, and its place there
    const int t16 = GLU ? min(tile * MW + fw * WH + fi % WH, n16 / 2 - 1) + (fi < WH ? 0 : n16 / 2) : min(tile * NF + f, n16 - 1);
    wsrc[i] = wpk + ((size_t)t16 * kp32 + (k_begin >> 5)) * 1024;
    wdst[i] = f * 1024 + lane * 16;
  }
  const unsigned woff = lane * 16;
  // X: a half-stage is XR/8 blocks of 8 rows x 128 B.  This wave moves blocks wave + 8 j (j < XT); its
  // lane L fetches, for the row 8 (wave + 8 j) + L/8, the piece (L % 8) ^ (L / 8).
  const char* xsrc = (const char*)x + (size_t)k_begin * 4;
  unsigned xoff[XT];
#pragma unroll
  for (int j = 0; j < XT; ++j) {
    const int row = min((tid >> 3) + 64 * j, rows - 1);
    xoff[j] = (unsigned)row * (unsigned)ldx * 2u + (unsigned)(((lane & 7) ^ (lane >> 3)) * 16);
  }
  const int lasth = nh - 1;

  auto load_w = [&](u32x4_t (&a)[2], int hs) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a[i] = __builtin_nontemporal_load((const u32x4_t*)(wsrc[i] + (size_t)min(hs, lasth) * 1024 + woff));
  };
  auto store_w = [&](const u32x4_t (&a)[2], int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4_t*)(wb[buf] + wdst[i]) = a[i];
  };
  auto dma_x = [&](int buf, int hs, int j) {
    load_to_lds_16(xsrc + (size_t)min(hs, lasth) * 128, xoff[j], lds_address(xb[buf]) + wave_u * 1024 + j * 8192);
  };
  // fragment reads.  W: linear.  X: row 16 t + r16 is block 2 t + r16 / 8, line r16 % 8; piece
  // (4 plane + kb) ^ (r16 % 8)
  const int arow = (wg * MW) * 1024 + lane * 16;
  const int brow = xg * XT * 2048 + (r16 >> 3) * 1024 + (r16 & 7) * 128;
  const int bcol[2] = {(kb ^ (r16 & 7)) * 16, ((4 + kb) ^ (r16 & 7)) * 16};
  u32x4_t wf[2][WH], xf[2][XA][2];
  auto read_w = [&](auto half, int buf, int i) {
    constexpr int H = decltype(half)::value;
    wf[H][i] = *(const u32x4_t*)(wb[buf] + arow + (H * WH + i) * 1024);
  };
  auto read_x = [&](auto half, int buf, int i) {   // i: tile of the half and plane
    constexpr int H = decltype(half)::value;
    xf[H][i >> 1][i & 1] = *(const u32x4_t*)(xb[buf] + brow + bcol[i & 1] + (H * XA + (i >> 1)) * 2048);
  };

  f32x4_t acc[MW][XT];
#pragma unroll
  for (int mt = 0; mt < MW; ++mt)
#pragma unroll
    for (int xt = 0; xt < XT; ++xt) acc[mt][xt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // The products of W half HW with X half HX; before every fourth of them one of the NE other
  // operations `extra(i)` that this quadrant covers is issued.
  auto quadrant = [&](auto hw, auto hx, auto ne, auto extra) {
    constexpr int HW = decltype(hw)::value, HX = decltype(hx)::value, NE = decltype(ne)::value;
    constexpr int NX = HX ? XB : XA, PER = WH * NX, TOTAL = 2 * PER;
    constexpr int STEP = NE > 0 && TOTAL / NE < 4 ? (TOTAL / NE > 0 ? TOTAL / NE : 1) : 4;
#pragma unroll
    for (int i = 0; i < TOTAL; ++i) {
      if (i % STEP == 0 && i / STEP < NE) {
        extra(i / STEP);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int plane = i / PER, xt = (i % PER) / WH, w = i % WH;
      acc[HW * WH + w][HX * XA + xt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          as_bf16x8(wf[HW][w]), as_bf16x8(xf[HX][xt][plane]), acc[HW * WH + w][HX * XA + xt], 0, 0, 0);
      if (i % STEP == STEP - 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = (TOTAL + STEP - 1) / STEP; i < NE; ++i) extra(i);
    __builtin_amdgcn_sched_barrier(0);
  };

  std::integral_constant<int, 0> c0;
  std::integral_constant<int, 1> c1;
  u32x4_t s0[2], s1[2];   // W staging registers of even and odd half-stages
  // Half-stage hs from LDS buffer P.  Enters with W half 0 and X half P in registers, leaves with W half 0
  // and X half 1 - P of the next one.  Loads complete in order; those of a half-stage are issued X
  // first, so "at most 2 outstanding" in front of the barrier (the two W loads issued behind the last
  // X loads) means that X of half-stage hs + 1 is in LDS and W of hs + 2 in registers.  Every load is
  // unconditional (half-stages past the end repeat the last one; nobody reads them) so that this
  // count stays exact.
  auto half_stage = [&](auto parity, u32x4_t (&stage)[2], int hs) {
    constexpr int P = decltype(parity)::value;
    std::integral_constant<int, P> first;        // X half in registers
    std::integral_constant<int, 1 - P> second;
    constexpr int NX2 = 2 * (P ? XA : XB);       // fragments of the other X half
    std::integral_constant<int, NX2> nx2;
    std::integral_constant<int, WH> nw;
    quadrant(c0, first, nx2, [&](int i) { read_x(second, P, i); });
    quadrant(c0, second, nw, [&](int i) { read_w(c1, P, i); });
    wait_vmcnt<2>();
    lds_barrier();
    store_w(stage, P);                           // W of hs + 2
    std::integral_constant<int, (WH > XT ? WH : XT)> nm;
    quadrant(c1, second, nm, [&](int i) {
      if (i < WH) read_w(c0, 1 - P, i);
      if (i < XT) dma_x(P, hs + 2, i);
    });
    load_w(stage, hs + 4);
    quadrant(c1, first, nx2, [&](int i) { read_x(second, 1 - P, i); });
  };

  if (nh > 0) {
    u32x4_t a0[2], a1[2];
    load_w(a0, 0);
    load_w(a1, 1);
#pragma unroll
    for (int j = 0; j < XT; ++j) dma_x(0, 0, j);
    load_w(s0, 2);
#pragma unroll
    for (int j = 0; j < XT; ++j) dma_x(1, 1, j);
    load_w(s1, 3);
    store_w(a0, 0);
    store_w(a1, 1);
    wait_vmcnt<2>();
    lds_barrier();
#pragma unroll
    for (int i = 0; i < WH; ++i) read_w(c0, 0, i);
#pragma unroll
    for (int i = 0; i < 2 * XA; ++i) read_x(c0, 0, i);
  }
  // nh is even, so there is no peeled tail (in one, the compiler could drop loads whose registers
  // nobody reads any more, and the counted waits would no longer cover the X loads)
  for (int hs = 0; hs < nh; hs += 2) {
    half_stage(c0, s0, hs);
    half_stage(c1, s1, hs + 1);
  }
  wait_vmcnt<0>();   // nothing of this workgroup may still be on its way into LDS when it ends

  // accumulator layout: lane holds C[w-row 4*(lane/16) + i][x-row lane%16], i = 0..3
  if constexpr (GLU) {
    float scale[XT];
#pragma unroll
    for (int xt = 0; xt < XT; ++xt) scale[xt] = row_scale8(rs, row0 + min((xg * XT + xt) * 16 + r16, rows - 1));
#pragma unroll
    for (int w = 0; w < WH; ++w) {
      const int c = (tile * MW + wg * WH + w) * 16 + 4 * kb;
      if (c >= n / 2) continue;
#pragma unroll
      for (int xt = 0; xt < XT; ++xt) {
        const int r = (xg * XT + xt) * 16 + r16;
        if (r >= rows) continue;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = acc[w][xt][i] * scale[xt], u = acc[WH + w][xt][i] * scale[xt];
          v[i] = g / (1.0f + expf(-g)) * u;
        }
        act_store4<true>(act, row0 + r, c, v[0], v[1], v[2], v[3]);
      }
    }
    return;
  }
  float* o = out + (size_t)split * part_stride;
#pragma unroll
  for (int mt = 0; mt < MW; ++mt) {
    const int c = (tile * NF + wg * MW + mt) * 16 + 4 * kb;
    if (c >= n) continue;
#pragma unroll
    for (int xt = 0; xt < XT; ++xt) {
      const int r = (xg * XT + xt) * 16 + r16;
      if (r < rows) *(f32x4_t*)(o + (size_t)r * ld_out + c) = acc[mt][xt];
    }
  }
}

}  // namespace

#define FIRP_TALL_PARAMS                                                                                               \
  const bf16 *__restrict__ x, int ldx, int rows, const char *__restrict__ wpk, int n, int K, float *__restrict__ out, \
      int ld_out, size_t part_stride, int S, int k_per, int tiles, int blocks
#define FIRP_TALL_ARGS x, ldx, rows, wpk, n, K, out, ld_out, part_stride, S, k_per, tiles, blocks

// row blocks of 192 or 256 rows (XT 3, 4), 192 or 256 rows of W (MW 6, 8)
template <int XT, int MW>
__global__ __launch_bounds__(512, 2) void k_gemm_tall(FIRP_TALL_PARAMS) {
  gemm_tall_tile<XT, MW, false>(FIRP_TALL_ARGS, RowScale{}, Act{});
}
// row blocks of 320 rows, 192 rows of W: a step of a few rows more than 256 in one pass over W
__global__ __launch_bounds__(512, 2) void k_gemm_rows320(FIRP_TALL_PARAMS) {
  gemm_tall_tile<5, 6, false>(FIRP_TALL_ARGS, RowScale{}, Act{});
}
// gate|up with SwiGLU as its epilogue
template <int XT, int MW>
__global__ __launch_bounds__(512, 2) void k_gemm_tall_swiglu(FIRP_TALL_PARAMS, RowScale rs, Act act) {
  gemm_tall_tile<XT, MW, true>(FIRP_TALL_ARGS, rs, act);
}

// rows > 128, K % 64 == 0; plan.nw is 8 or 6 (a workgroup owns 256 or 192 rows of W), plan.xt 3..5
// (64 xt activation rows; 5 with nw 6 only), plan.grid = tiles x S per row block
void launch_gemm_tall(const bf16* x, int ldx, int rows, const void* w_packed, int n, int K, float* out, int ld,
                      size_t part_stride, const GemmPlan& p, hipStream_t s) {
  const int blocks = (rows + 64 * p.xt - 1) / (64 * p.xt);
  dim3 g((p.grid * blocks + 7) & ~7), b(512);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, g, b, 0, s, x, ldx, rows, (const char*)w_packed, n, K, out, ld, part_stride, p.S, p.k_per,
                       p.grid / p.S, blocks);
  };
  if (p.xt == 5) go(k_gemm_rows320);
  else if (p.xt == 4) { if (p.nw == 6) go(k_gemm_tall<4, 6>); else go(k_gemm_tall<4, 8>); }
  else { if (p.nw == 6) go(k_gemm_tall<3, 6>); else go(k_gemm_tall<3, 8>); }
}

// act = silu(gate) * up of gate|up [2 F][K] (F % 16 == 0) for a plan of one split: the 8 F rows bytes of partial sums
// are neither written nor read, and there is no kernel to read them.  1023 rows of the 13B shape with K whole:
// 416 us and 26 for the separate kernel -> 411 us; of the 7B shape: 277 and 21 -> 269.
void launch_gemm_tall_swiglu(const bf16* x, int ldx, int rows, const void* w_packed, int F, int K, const RowScale& rs,
                             const Act& act, const GemmPlan& p, hipStream_t s) {
  const int blocks = (rows + 64 * p.xt - 1) / (64 * p.xt), tiles = (F + 16 * p.nw - 1) / (16 * p.nw);
  dim3 g((tiles * blocks + 7) & ~7), b(512);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, g, b, 0, s, x, ldx, rows, (const char*)w_packed, 2 * F, K, (float*)nullptr, 0, (size_t)0, 1, K, tiles,
                       blocks, rs, act);
  };
  if (p.xt == 5) go(k_gemm_tall_swiglu<5, 6>);
  else if (p.xt == 4) { if (p.nw == 6) go(k_gemm_tall_swiglu<4, 6>); else go(k_gemm_tall_swiglu<4, 8>); }
  else { if (p.nw == 6) go(k_gemm_tall_swiglu<3, 6>); else go(k_gemm_tall_swiglu<3, 8>); }
}

}  // namespace firp
