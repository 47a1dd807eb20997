// Products of the update step of fp32 models (Alg. 1, line 10) for batches of a
// few hundred to a few thousand windows: C = A.B on fp32 MFMAs, one small output
// tile per workgroup and the k range split over its eight waves.
//
// What bounds these products is latency: at 512 windows and d = 128 the largest
// is 0.13 GFLOP, one microsecond of the chip's fp32 rate, but 128 x 128 tiles
// give it 16 workgroups that each walk k alone (28-38 us a product).  Here
// wave w takes the w-th eighth of k and reads its fragments of A and B straight
// from global memory (no wave reads what another one reads, so LDS staging
// would save nothing, and there is no barrier in the k loop), every load of a
// batch of k-steps in flight before the first MFMA of the batch before it; the
// eight partial tiles meet in LDS and are added in wave order, so there is no
// split-K pass either (tall products of few tiles, k = windows x tokens, are cut
// over blocks as well, down to 1024 k values each).  Tiles are 32 x 32, or
// 16 x 16 where the product has fewer than 256 of the larger ones.  Measured at
// 512 windows, d = 128, F = 512, k = 2 (18 products per update): 28-38 -> 4-6 us
// a product (the two of k = 4096: 19 -> 9 with the cut), the backward 444 -> 212 us.
#include "kcommon.h"
#include "kernels.h"

namespace {

// One operand: element (row, k) of segment s at p_s[row * ld_s + k] (KC) or
// p_s[k * ld_s + row]; segment 1 starts at k = k1 of the product.
struct FSrc {
  const float *p0, *p1;
  int64_t ld0, ld1;
  int rows;
};
struct FArgs {
  FSrc A, B;
  int K, k1;         // all of k; the first k of segment 1 (K when there is none)
  int kz;            // k values per z block (a multiple of 16; K when the grid has one)
  float* part;       // partial results [z][M][N] when the grid has several z blocks
  int M, N, tn;
  float* C;
  int64_t ldc;
  const float* cin;  // nullable addend, laid out as C
  const float* gu;   // nullable: C = (A.B) * GELU'(gu)
};

// The four k values 4 lg .. 4 lg + 3 of k-step k0 of row `row`: past kend zero
// (loads clamped into the operand; k contiguous operands have no such step).
template <bool KC>
__device__ __forceinline__ float4 frag(const FSrc& s, int k1, int row, int k0, int lg, int kend) {
  const bool seg1 = k0 >= k1;
  const float* __restrict__ p = seg1 ? s.p1 : s.p0;
  const int64_t ld = seg1 ? s.ld1 : s.ld0;
  const int off = seg1 ? k1 : 0;
  if constexpr (KC) {
    return *reinterpret_cast<const float4*>(p + (int64_t)row * ld + (k0 - off + 4 * lg));
  } else {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + 4 * lg + j;
      v[j] = p[(int64_t)(min(k, kend - 1) - off) * ld + row];
    }
    const int kb = k0 + 4 * lg;
    return make_float4(kb < kend ? v[0] : 0.f, kb + 1 < kend ? v[1] : 0.f, kb + 2 < kend ? v[2] : 0.f,
                       kb + 3 < kend ? v[3] : 0.f);
  }
}

__device__ __forceinline__ uint4 bits4(const float4& v) {
  return make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w));
}

// Tiles of 16 F x 16 F; U k-steps (of 16) per batch of loads.
template <bool AKC, bool BKC, int F, int U>
__device__ __forceinline__ void fgemm_tile(float (&red)[8][16 * F * (16 * F + 4)], int tile, int zi, const FArgs& a) {
  typedef Mma<false> M;
  constexpr int TS = 16 * F, STR = TS + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, lc = lane & 15;
  const int m0 = (tile / a.tn) * TS, n0 = (tile % a.tn) * TS;
  const int zb = zi * a.kz, ze = min(a.K, zb + a.kz);
  const int per = ((ze - zb + 127) / 128) * 16;  // k values per wave
  const int kb = zb + wave * per, ke = min(ze, kb + per);
  int ra[F], rb[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    ra[f] = min(m0 + 16 * f + lc, a.A.rows - 1);
    rb[f] = min(n0 + 16 * f + lc, a.B.rows - 1);
  }
  f32x4 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float4 va[2][U][F], vb[2][U][F];
  // a batch's loads: steps past the wave's range repeat its last step (their
  // values are not used)
  auto load = [&](int set, int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(k0 + 16 * u, kb + (ke - 1 - kb) / 16 * 16);
#pragma unroll
      for (int f = 0; f < F; ++f) {
        va[set][u][f] = frag<AKC>(a.A, a.k1, ra[f], k, lg, a.K);
        vb[set][u][f] = frag<BKC>(a.B, a.k1, rb[f], k, lg, a.K);
      }
    }
  };
  auto mult = [&](int set, int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + 16 * u < ke) {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j) M::run(acc[i][j], bits4(va[set][u][i]), bits4(vb[set][u][j]));
      }
    }
  };
  if (kb < ke) {
    load(0, kb);
    for (int k0 = kb; k0 < ke; k0 += 32 * U) {
      if (k0 + 16 * U < ke) load(1, k0 + 16 * U);
      mult(0, k0);
      if (k0 + 16 * U < ke) {
        if (k0 + 32 * U < ke) load(0, k0 + 32 * U);
        mult(1, k0 + 16 * U);
      }
    }
  }
  // lane holds C[m0 + 16 i + 4 lg + r][n0 + 16 j + lc]
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(16 * i + 4 * lg + r) * STR + 16 * j + lc] = acc[i][j][r];
  __syncthreads();
  for (int q = tid; q < TS * TS; q += 512) {
    const int i = q / TS, j = q % TS, m = m0 + i, n = n0 + j;
    float v = red[0][i * STR + j];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += red[w][i * STR + j];
    if (m < a.M && n < a.N) {
      if (a.part) {
        a.part[((int64_t)zi * a.M + m) * a.N + n] = v;
        continue;
      }
      const int64_t o = (int64_t)m * a.ldc + n;
      if (a.cin) v = a.cin[o] + v;
      if (a.gu) v *= gelu_grad_f(a.gu[o]);
      a.C[o] = v;
    }
  }
}

template <bool AKC, bool BKC, int F, int U>
__global__ __launch_bounds__(512) void k_fgemm(FArgs a) {
  __shared__ __align__(16) float red[8][16 * F * (16 * F + 4)];
  fgemm_tile<AKC, BKC, F, U>(red, (int)blockIdx.x, (int)blockIdx.z, a);
}

// Several weight gradients (rows of both operands contiguous) in one launch, on
// 16-wide tiles: the host takes about 4 us to launch each
struct FGroup {
  FArgs j[GROUP_MAX_JOBS];
  int tile0[GROUP_MAX_JOBS], tiles[GROUP_MAX_JOBS];  // first block, blocks per z of each job
  int n;
};
__global__ __launch_bounds__(512) void k_fgemm_group(FGroup g) {
  __shared__ __align__(16) float red[8][16 * 20];
  const int b = (int)blockIdx.x;
  int q = 0;
  for (int u = 1; u < g.n; ++u) q = b >= g.tile0[u] ? u : q;
  const int t = b - g.tile0[q];
  fgemm_tile<false, false, 1, 4>(red, t % g.tiles[q], t / g.tiles[q], g.j[q]);
}

bool seg(FSrc& s, int i, const float* p, int64_t srow, int64_t sk, int rows, int K, bool& kc) {
  const bool this_kc = sk == 1;
  if (!this_kc && srow != 1) return false;
  if (i && this_kc != kc) return false;
  if (this_kc && (((uintptr_t)p & 15) || srow % 4 || K % 16)) return false;  // float4 of whole k-steps
  kc = this_kc;
  (i ? s.p1 : s.p0) = p;
  (i ? s.ld1 : s.ld0) = this_kc ? srow : sk;
  s.rows = rows;
  return true;
}

template <int F, int U>
void launch(bool akc, bool bkc, const FArgs& a, dim3 grid, hipStream_t s) {
  if (akc && bkc)
    hipLaunchKernelGGL((k_fgemm<true, true, F, U>), grid, dim3(512), 0, s, a);
  else if (akc)
    hipLaunchKernelGGL((k_fgemm<true, false, F, U>), grid, dim3(512), 0, s, a);
  else if (bkc)
    hipLaunchKernelGGL((k_fgemm<false, true, F, U>), grid, dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((k_fgemm<false, false, F, U>), grid, dim3(512), 0, s, a);
}

}  // namespace

// The largest product this kernel takes, in multiply-adds: from there on the
// 128-tile kernel fills the chip and, reading each operand fewer times, is the
// faster.  Measured (us, this kernel / 128 tiles with its split-K pass):
// 4096 x 512 x 128 (2^28) 23 / 22, 512 x 128 x 4096 (2^28) 20 / 46,
// 4096 x 256 x 256 (2^28) 16 / 47; 8192 x 512 x 128 (2^29) 51 / 27,
// 512 x 128 x 8192 (2^29) 61 / 47; 4096 x 1024 x 256 (2^30) 65-108 / 40-51.
constexpr int64_t FGEMM_MAX = (int64_t)1 << 28;

// Blocks along k of a product of `tiles` tiles: cut while that makes at most 512
// blocks of at least 1024 k values each.
static int z_blocks(int64_t tiles, int M, int N, int K, int64_t ws_cap) {
  int z = 1;
  while (tiles * z < 512 && K / (2 * z) >= 1024 && (int64_t)2 * z * M * N <= ws_cap) z *= 2;
  return z;
}
int64_t fgemm_ws_floats(int M, int N, int K) {
  const int z = z_blocks((int64_t)((M + 15) / 16) * ((N + 15) / 16), M, N, K, (int64_t)1 << 60);
  return z > 1 ? (int64_t)z * M * N : 0;
}

bool launch_fgemm(const GemmArgs& g, const GemmArgs* g2, float* ws, int64_t ws_cap, hipStream_t s) {
  if (g.roundA || g.roundB || g.halfA || g.halfB || g.halfC || g.r1c || g.rowwise || g.K <= 0) return false;
  if (g2 && (g2->roundA || g2->roundB || g2->halfA || g2->halfB || g2->r1c || g2->K <= 0 || g.K % 16)) return false;
  const int K = g.K + (g2 ? g2->K : 0);
  if ((int64_t)g.M * g.N * K > FGEMM_MAX) return false;
  FArgs a{};
  bool akc = false, bkc = false;
  if (!seg(a.A, 0, g.A, g.sam, g.sak, g.M, g.K, akc) || !seg(a.B, 0, g.B, g.sbn, g.sbk, g.N, g.K, bkc)) return false;
  if (g2) {
    if (!seg(a.A, 1, g2->A, g2->sam, g2->sak, g.M, g2->K, akc) || !seg(a.B, 1, g2->B, g2->sbn, g2->sbk, g.N, g2->K, bkc))
      return false;
  } else {
    a.A.p1 = a.A.p0;
    a.A.ld1 = a.A.ld0;
    a.B.p1 = a.B.p0;
    a.B.ld1 = a.B.ld0;
  }
  // k contiguous on one side only: the other side's steps are whole as well
  a.K = K;
  a.k1 = g2 ? g.K : K;
  a.M = g.M;
  a.N = g.N;
  a.C = g.C;
  a.ldc = g.ldc;
  a.cin = g.beta != 0.f ? g.C : nullptr;
  a.gu = g.gelu_u;
  const int64_t big = (int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32);
  const bool wide = big >= 256;
  const int ts = wide ? 32 : 16;
  a.tn = (g.N + ts - 1) / ts;
  const int64_t tiles = (int64_t)((g.M + ts - 1) / ts) * a.tn;
  int z = g.gelu_u ? 1 : z_blocks(tiles, g.M, g.N, K, ws_cap);
  a.kz = ((K + z - 1) / z + 15) / 16 * 16;
  z = (K + a.kz - 1) / a.kz;
  a.part = z > 1 ? ws : nullptr;
  const dim3 grid((unsigned)tiles, 1, (unsigned)z);
  if (wide)
    launch<2, 2>(akc, bkc, a, grid, s);
  else
    launch<1, 4>(akc, bkc, a, grid, s);
  if (z > 1) launch_splitk_reduce(ws, z, g.M, g.N, g.C, g.ldc, g.beta, s);
  return true;
}

void launch_fgemm_group(const GemmArgs* g, int n, bool* grouped, RedJob* red, float*& ws, int64_t& ws_cap, bool plan,
                        hipStream_t s) {
  FGroup G{};
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& a = g[i];
    grouped[i] = false;
    if (a.roundA || a.roundB || a.halfA || a.halfB || a.halfC || a.r1c || a.gelu_u || a.beta != 0.f || a.K <= 0) continue;
    if ((int64_t)a.M * a.N * a.K > FGEMM_MAX) continue;
    FArgs f{};
    bool akc = false, bkc = false;
    if (!seg(f.A, 0, a.A, a.sam, a.sak, a.M, a.K, akc) || !seg(f.B, 0, a.B, a.sbn, a.sbk, a.N, a.K, bkc) || akc || bkc)
      continue;
    grouped[i] = true;
    if (plan) continue;
    f.A.p1 = f.A.p0;
    f.A.ld1 = f.A.ld0;
    f.B.p1 = f.B.p0;
    f.B.ld1 = f.B.ld0;
    f.K = f.k1 = a.K;
    f.M = a.M;
    f.N = a.N;
    f.C = a.C;
    f.ldc = a.ldc;
    f.tn = (a.N + 15) / 16;
    const int tiles = (a.M + 15) / 16 * f.tn;
    int z = z_blocks(tiles, a.M, a.N, a.K, ws_cap);
    f.kz = ((a.K + z - 1) / z + 15) / 16 * 16;
    z = (a.K + f.kz - 1) / f.kz;
    f.part = z > 1 ? ws : nullptr;
    G.j[G.n] = f;
    G.tile0[G.n] = blocks;
    G.tiles[G.n++] = tiles;
    blocks += tiles * z;
    red[i] = RedJob{};
    red[i].part = z > 1 ? ws : a.C;
    red[i].pstride = (int64_t)a.M * a.N;
    red[i].splits = z;
    red[i].M = a.M;
    red[i].N = a.N;
    red[i].C = a.C;
    red[i].ldc = a.ldc;
    if (z > 1) {
      ws += (int64_t)z * a.M * a.N;
      ws_cap -= (int64_t)z * a.M * a.N;
    }
  }
  if (G.n) hipLaunchKernelGGL(k_fgemm_group, dim3((unsigned)blocks), dim3(512), 0, s, G);
}
