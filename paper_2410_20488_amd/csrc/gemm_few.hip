// Projections for up to 16 activation rows, with the step's next elementwise kernel as their epilogue.
//
//   y[r][c] = sum_k X[r][k] * W[c][k],   r < rows <= 16
//
// With this few rows the activations are next to nothing beside the weights, so the split of K that
// keeps a CU's memory pipeline full can stay inside a workgroup: its 8 waves take every eighth
// 64-column stage of the same MT 16-row tiles of W, read W (the fragment-major copy, 1 KiB per
// instruction) and X straight from global memory into MFMA operand layout, several stages ahead,
// and add their accumulators up through LDS.  MT is chosen so that the tiles make one workgroup per
// CU where they can: X is then loaded once per MT tiles and no CU starts a second pipeline.  A
// workgroup holds finished outputs: no split-K partial sums go through memory and the consumer
// needs no launch:
//   FEW_PLAIN   y * row scale, as one "split"
//   FEW_SWIGLU  silu(gate) * up as the activation planes of the down projection (tiles in pairs: 16 gate
//               rows and the 16 up rows of the same columns)
//   FEW_RESID   x += y; x * gain as the planes of the next projection, and the sum of squares of the
//               tile's 16 columns of every row (see RowScale)
// What bounds it is the weight stream.
#include <algorithm>

#include "kernels.h"

namespace firp {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t v) { return __builtin_bit_cast(bf16x8_t, v); }

constexpr int FEW_WAVES = 8;

}  // namespace

template <int EPI, int MT, bool KTAIL>
__global__ __launch_bounds__(64 * FEW_WAVES, 2) void k_gemm_few(const bf16* __restrict__ xpl, int ldx, int rows,
                                                                const char* __restrict__ wpk, int n, int K, RowScale rs,
                                                                FewOut o) {
  constexpr int AHEAD = MT == 1 ? 6 : MT == 2 ? 4 : MT <= 4 ? 3 : 2;   // stages in flight per wave
  constexpr int OUT = EPI == FEW_SWIGLU ? MT / 2 : MT;                 // 16-column tiles of outputs
  __shared__ float red[FEW_WAVES][MT][4][64];
  __shared__ float scale_lds[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kb = lane >> 4;
  const int kp32 = ((K + 63) / 64) * 2, stages = kp32 / 2;
  const int n16 = (n + 15) >> 4;
  const int out0 = blockIdx.x * OUT, outs = EPI == FEW_SWIGLU ? n16 / 2 : n16;   // first tile, tiles of outputs

  // the row scales: this wave sums the pieces of rows `wave` and `wave + 8`; asked for first, used last
  constexpr int PL = FIRP_FEW_PIECES / 64;   // pieces per lane at most
  float ssq[2][PL];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < PL; ++i) ssq[h][i] = 0.f;
  if (EPI != FEW_RESID && rs.ss) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (wave + 8 * h < rows) {
#pragma unroll
        for (int i = 0; i < PL; ++i)
          if (lane + 64 * i < rs.pieces) ssq[h][i] = rs.ss[(size_t)(wave + 8 * h) * rs.stride + lane + 64 * i];
      }
  }

  const char* wp[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    // (gate|up: the second half of the matrix holds the up rows; tiles past the end repeat the last one)
    const int t16 = EPI == FEW_SWIGLU ? min(out0 + mt / 2, outs - 1) + (mt & 1) * outs : min(out0 + mt, outs - 1);
    wp[mt] = wpk + (size_t)t16 * kp32 * 1024 + lane * 16;
  }
  const char* xp = (const char*)(xpl + (size_t)min(r16, rows - 1) * ldx) + kb * 16;

  u32x4_t a[AHEAD][MT][2], x[AHEAD][2][2];
  auto load = [&](int slot, int st) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        a[slot][mt][j] = __builtin_nontemporal_load((const u32x4_t*)(wp[mt] + (size_t)st * 2048 + j * 1024));
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if constexpr (KTAIL) {
          const bool ok = st * 64 + j * 32 + kb * 8 < K;   // (K % 8 == 0; W's padding is zero, X's is not)
          x[slot][j][p] = ok ? *(const u32x4_t*)(xp + (size_t)st * 256 + j * 128 + p * 64) : u32x4_t{0, 0, 0, 0};
        } else {
          x[slot][j][p] = *(const u32x4_t*)(xp + (size_t)st * 256 + j * 128 + p * 64);
        }
      }
  };
  f32x4_t acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[slot][mt][j]), as_bf16x8(x[slot][j][p]), acc[mt], 0, 0, 0);
  };
  // this wave's stages: wave, wave + 8, ...; loads past its last stage repeat that one (unused), so
  // that every load is unconditional and the compiler's wait counters stay exact
  const int cnt = (stages - wave + FEW_WAVES - 1) / FEW_WAVES;
  if (cnt > 0) {
    auto stage_of = [&](int i) { return wave + FEW_WAVES * min(i, cnt - 1); };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load(i, stage_of(i));
    int i = 0;
    for (; i + AHEAD <= cnt; i += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        multiply(u);
        load(u, stage_of(i + u + AHEAD));
      }
    }
#pragma unroll
    for (int u = 0; u < AHEAD - 1; ++u)
      if (i + u < cnt) multiply(u);
  }

  // accumulator layout: lane holds C[w-row 4*(lane/16) + i][x-row lane%16], i = 0..3
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][mt][i][lane] = acc[mt][i];
  if (EPI != FEW_RESID) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < PL; ++i) t += ssq[h][i];
      t = wave_sum(t);
      if (lane == 0) scale_lds[wave + 8 * h] = rs.ss ? 1.0f / sqrtf(t * rs.inv_d + rs.eps) : 1.0f;
    }
  }
  __syncthreads();
  // 256 threads per output tile: x row r, column cl of the tile
  const int r = (tid & 255) >> 4, cl = tid & 15;
  for (int t = tid >> 8; t < OUT; t += 2) {
    const int tile = out0 + t, c = tile * 16 + cl;
    const bool live = r < rows && tile < outs && c < n;
    auto sum = [&](int mt) {
      float y = 0.f;
#pragma unroll
      for (int w = 0; w < FEW_WAVES; ++w) y += red[w][mt][cl & 3][(cl >> 2) * 16 + r];
      return y;
    };
    if constexpr (EPI == FEW_PLAIN) {
      if (live) o.y[(size_t)r * o.ld + c] = sum(t) * scale_lds[r];
    } else if constexpr (EPI == FEW_SWIGLU) {
      if (live) {
        const float g = sum(2 * t) * scale_lds[r], u = sum(2 * t + 1) * scale_lds[r];
        act_store<true>(o.act, r, c, g / (1.0f + expf(-g)) * u);
      }
    } else {
      float v = 0.f;
      if (live) {
        float* xr = o.x + (size_t)r * n + c;
        v = *xr + sum(t);
        *xr = v;
        act_store<true>(o.act, r, c, v * to_f32(o.gain[c]));
      }
      float s = v * v;
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) s += __shfl_xor(s, d, 16);
      if (live && cl == 0) o.ss[(size_t)r * FIRP_FEW_PIECES + tile] = s;
    }
  }
}

// Tiles per workgroup (of outputs): the fewest that make at most one workgroup per CU, up to what the
// registers hold.
static int few_tiles(int epi, int n) {
  const int outs = epi == FEW_SWIGLU ? n / 32 : (n + 15) / 16;
  const int want = (outs + 255) / 256;
  if (epi == FEW_SWIGLU) return std::min(want, 4);
  return want <= 4 ? want : want <= 6 ? 6 : 8;
}

static bool few_pays(int epi, int rows, int n, int K) {
  if (!gemm_mfma_supported(rows, n, K)) return false;
  if (epi == FEW_SWIGLU && n % 32) return false;              // gate and up rows in whole tiles
  if (epi == FEW_RESID && n > 16 * FIRP_FEW_PIECES) return false;
  if ((double)n * K * 2.0 <= 8e6) return true;
  const int outs = epi == FEW_SWIGLU ? n / 32 : (n + 15) / 16, per = few_tiles(epi, n);
  const int rounds = ((outs + per - 1) / per + 255) / 256;
  return rows <= 4 * per * (epi == FEW_SWIGLU ? 2 : 1) && outs >= 0.88 * 256 * per * rounds;
}

// Whether a decoder layer of this many rows runs on these kernels; all of its projections do or none (a norm
// done by one of them leaves its sums of squares in more pieces than the other consumers read well).
//  * The workgroups have to fill whole rounds of the 256 CUs: a launch takes as long as the CU with most
//    of them (each CU pulls at most its share of the HBM rate), and the streaming kernel, which cuts K
//    among workgroups, always fills the chip.  7B shape (d = 4096: rounds full to 0.9 and more): 1 row 50.9
//    -> 48.6 ms for 16 steps, 4 rows 52.5 -> 50.4; 13B shape (d = 5120: 320 tiles, 0.63 of a round, and gate|up
//    0.84): gate|up 51 us against 44 + 5 + a launch, the rest slower.
//  * Every wave loads its own slice of X, two lines per row and 64 columns beside 16 per tile of W: more
//    than 4 rows per tile and X takes too many of the lines that a CU can have in flight (7B shape, 16 rows:
//    54.9 -> 61.9 ms).
//  * Below 8 MB of weights it is the fixed time of the launches that counts, and there are three fewer
//    per layer (4 layers of width 256, 32 steps: 7.8 -> 6.9 ms).
bool gemm_few_pays(int rows, int d_model, int q_dim, int qkv_dim, int d_ffn) {
  return rows >= 1 && rows <= FIRP_FEW_ROWS && few_pays(FEW_PLAIN, rows, qkv_dim, d_model) &&
         few_pays(FEW_RESID, rows, d_model, q_dim) && few_pays(FEW_SWIGLU, rows, 2 * d_ffn, d_model) &&
         few_pays(FEW_RESID, rows, d_model, d_ffn);
}

void launch_gemm_few(int epi, const Act& x, int rows, const void* w_packed, int n, int K, const RowScale& rs,
                     const FewOut& out, hipStream_t s) {
  const int outs = epi == FEW_SWIGLU ? n / 32 : (n + 15) / 16, per = few_tiles(epi, n);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((outs + per - 1) / per), dim3(64 * FEW_WAVES), 0, s, x.pl, x.row, rows,
                       (const char*)w_packed, n, K, rs, out);
  };
  const bool tail = K % 64 != 0;
#define FEW_GO(E, M) do { if (tail) go(k_gemm_few<E, M, true>); else go(k_gemm_few<E, M, false>); } while (0)
  if (epi == FEW_PLAIN) {
    switch (per) {
      case 1: FEW_GO(FEW_PLAIN, 1); break;
      case 2: FEW_GO(FEW_PLAIN, 2); break;
      case 3: FEW_GO(FEW_PLAIN, 3); break;
      case 4: FEW_GO(FEW_PLAIN, 4); break;
      case 6: FEW_GO(FEW_PLAIN, 6); break;
      default: FEW_GO(FEW_PLAIN, 8); break;
    }
  } else if (epi == FEW_SWIGLU) {
    switch (per) {
      case 1: FEW_GO(FEW_SWIGLU, 2); break;
      case 2: FEW_GO(FEW_SWIGLU, 4); break;
      case 3: FEW_GO(FEW_SWIGLU, 6); break;
      default: FEW_GO(FEW_SWIGLU, 8); break;
    }
  } else {
    // (n <= 16 FIRP_FEW_PIECES: at most two tiles)
    if (per == 1) FEW_GO(FEW_RESID, 1); else FEW_GO(FEW_RESID, 2);
  }
#undef FEW_GO
}

}  // namespace firp
