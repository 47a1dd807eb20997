// The chain of input gradients of the update step through the head, the shared
// FFN and the output projection (Alg. 1, line 10), fused: kept logits -> dz ->
// dY_k -> (dU_r, dY_r) for r = k-1 .. 0 -> dO.  Per window every step needs only
// that window's rows, so one workgroup carries a tile of windows through all of
// it, as the forward FFN kernel does in the other direction:
//   dz = (softmax(z) - onehot(y)) / N                    -> HBM, LDS operand
//   dY_k^T = Wout . dz^T                                  (accumulators)
//   per repeat, chunks of 128 features:
//     dU^T = (W2 . dY^T) * GELU'(U)                       -> HBM, LDS operand
//     dY^T += W1 . dU^T;      dY_r after the last chunk     -> HBM, LDS operand
//   dO^T = Wo . dY_0^T                                    -> HBM
// Every product is formed transposed (weights, from fragment-packed copies of
// their transposes, as the MFMA A operand), so a lane's four results are four
// consecutive features of one window.  The weight fragments of a whole product
// are requested one product ahead; G is double-buffered: one barrier per chunk.
//
// Bound by the weights every workgroup streams from L2 (4 MB per repeat at
// d = 512, at about 53 GB/s per CU whatever the shape) and, in fp32, by its MFMAs.
// It replaces 2 k + 3 dependent products, each reading its operands back from HBM
// and taking 5-13 us (d = 128) at a few hundred to a few thousand windows, with the
// softmax pass, the split-K passes and the fp32 passes for GELU and GELU'.  The
// backward with it, and the chain alone: 512 windows, d = 128, fp32 202 -> 134 us
// (chain 38); 4096, d = 128, bf16 211 -> 163 (18); 4096, d = 256 324 -> 257 (56);
// 8192, d = 512 886 -> 830 (238; the products and their passes took about 350).
#include <type_traits>

#include "kcommon.h"
#include "kernels.h"

namespace {

// four fp32 values -> four operand elements at p (8 or 16 bytes)
__device__ __forceinline__ void put4c(uint16_t* p, const f32x4& v) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}
__device__ __forceinline__ void put4c(float* p, const f32x4& v) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

template <bool BF, int D, int NFC>
struct ChainShape {
  typedef Mma<BF> M;
  typedef typename M::T OT;
  static constexpr int NW = D >= 128 ? 8 : 4, NT = 64 * NW, FC = BF && D <= 256 ? 256 : 128, MB = 16 * NFC;
  static constexpr int RF1 = FC / (16 * NW), RF2 = D / (16 * NW);
  static constexpr int KD = D / M::KS, KC = FC / M::KS, KZ = 256 / M::KS;
  static constexpr int ES = (int)sizeof(OT);
  static constexpr int YSTR = D * ES + 16, GSTR = FC * ES + 16, ZSTR = 256 * ES + 16;
  // k-steps in flight: weights of the products of dY_k and dO, weights of W2's
  // product (W1's: all of a chunk), activations (LDS)
  static constexpr int PZ = RF2 >= 4 ? 4 : 8, PA = KD * RF1 <= 16 ? KD : 8 / RF1, PL = 2;
};

template <bool BF, int D, int NFC>
__global__ __launch_bounds__((D >= 128 ? 512 : 256)) void k_bwd_chain(ChainArgs a) {
  typedef ChainShape<BF, D, NFC> S;
  typedef Mma<BF> M;
  typedef typename M::T OT;
  constexpr int NW = S::NW, NT = S::NT, FC = S::FC, MB = S::MB, RF1 = S::RF1, RF2 = S::RF2, KD = S::KD, KC = S::KC;
  constexpr int KZ = S::KZ, YSTR = S::YSTR, GSTR = S::GSTR, ZSTR = S::ZSTR, PZ = S::PZ, PA = S::PA, PL = S::PL, NB2 = D / 16;
  __shared__ __align__(16) unsigned char Ys[MB * YSTR];
  __shared__ __align__(16) unsigned char Gs[2][MB * GSTR];
  __shared__ __align__(16) unsigned char Zs[MB * ZSTR];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, lc = lane & 15;
  const int64_t tile0 = (int64_t)blockIdx.x * MB, N = a.N;
  const int F = a.F, NB1 = F / 16;
  const int d0 = wave * (D / NW), f0 = wave * (FC / NW);

  // acc^T = W^T-copy . rows over KN k-steps, this wave's RF2 row fragments of D
  auto product = [&](const uint4* W, const unsigned char* rows, int str, auto kn_c, f32x4 (&acc)[RF2][NFC]) {
    constexpr int KN = decltype(kn_c)::value, P = PZ < KN ? PZ : KN;
    uint4 w[P][RF2];
    auto ld = [&](int ks) {
#pragma unroll
      for (int rf = 0; rf < RF2; ++rf) w[ks % P][rf] = W[(ks * NB2 + d0 / 16 + rf) * 64 + lane];
    };
#pragma unroll
    for (int ks = 0; ks < P; ++ks) ld(ks);
    __syncthreads();  // the rows are in LDS
    const unsigned char* r0 = rows + lc * str + lg * 16;
    uint4 bb[PL + 1][NFC];
    auto ldr = [&](int ks) {
#pragma unroll
      for (int nf = 0; nf < NFC; ++nf) bb[ks % (PL + 1)][nf] = *(const uint4*)(r0 + nf * 16 * str + ks * 64);
    };
#pragma unroll
    for (int ks = 0; ks < PL; ++ks) ldr(ks);
#pragma unroll
    for (int ks = 0; ks < KN; ++ks) {
      if (ks + PL < KN) ldr(ks + PL);
#pragma unroll
      for (int rf = 0; rf < RF2; ++rf)
#pragma unroll
        for (int nf = 0; nf < NFC; ++nf) M::run(acc[rf][nf], w[ks % P][rf], bb[ks % (PL + 1)][nf]);
      if (ks + P < KN) ld(ks + P);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto zero = [](f32x4 (&x)[RF2][NFC]) {
#pragma unroll
    for (int rf = 0; rf < RF2; ++rf)
#pragma unroll
      for (int nf = 0; nf < NFC; ++nf) x[rf][nf] = f32x4{0.f, 0.f, 0.f, 0.f};
  };

  // dz, 16 threads per window, 16 consecutive logits each
  for (int q = tid; q < MB * 16; q += NT) {
    const int m = q >> 4, p = q & 15;
    const int64_t n = tile0 + m, nn = min(n, N - 1);
    float x[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 v = *reinterpret_cast<const float4*>(a.z + nn * 256 + p * 16 + 4 * i);
      x[4 * i] = v.x;
      x[4 * i + 1] = v.y;
      x[4 * i + 2] = v.z;
      x[4 * i + 3] = v.w;
    }
    const int y = a.tgt[nn] - p * 16;
    float mx = x[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
    mx = wave_max16(mx);
    float sm = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      x[i] = expf(x[i] - mx);
      sm += x[i];
    }
    sm = wave_sum16(sm);
    const float fn = (float)N;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = n < N ? (x[i] / sm - (i == y ? 1.f : 0.f)) / fn : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 v = f32x4{x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]};
      put4c((OT*)(Zs + m * ZSTR) + p * 16 + 4 * i, v);
      if (n < N) *reinterpret_cast<f32x4*>(a.dz + n * 256 + p * 16 + 4 * i) = v;
    }
  }

  // y^T: lane holds dY[nf*16 + lc][d0 + rf*16 + 4*lg + r]
  f32x4 y[RF2][NFC];
  zero(y);
  product(a.WoutT, Zs, ZSTR, std::integral_constant<int, KZ>{}, y);
  // dY_r -> LDS operand and HBM (bf16 models: r >= 1 as operand values, r = 0 fp32)
  auto put_y = [&](int r) {
#pragma unroll
    for (int nf = 0; nf < NFC; ++nf) {
      const int m = nf * 16 + lc;
      const int64_t n = tile0 + m;
#pragma unroll
      for (int rf = 0; rf < RF2; ++rf) {
        const int dd = d0 + rf * 16 + 4 * lg;
        put4c((OT*)(Ys + m * YSTR) + dd, y[rf][nf]);
        if (n < N) {
          if (r > 0)
            put4c((OT*)a.dYr + ((int64_t)(r - 1) * N + n) * D + dd, y[rf][nf]);
          else
            put4c(a.dY0 + n * D + dd, y[rf][nf]);
        }
      }
    }
  };
  // Loads return in order, so a wait for one is a wait for all before it: the U
  // rows (HBM) of a chunk are requested after the weights that the products before
  // their use need, and have a whole GEMM2 and GEMM1 to arrive.
  uint4 wa[PA][RF1], wb[KC][RF2];
  f32x4 uu[RF1][NFC];
  auto load2 = [&](const uint4* W, int c0, int ks) {  // k-step ks of W2's rows c0 .. of this wave
#pragma unroll
    for (int rf = 0; rf < RF1; ++rf) wa[ks % PA][rf] = W[(ks * NB1 + (c0 + f0) / 16 + rf) * 64 + lane];
  };
  auto loadu = [&](int r, int c0) {  // read once: streamed past the caches
#pragma unroll
    for (int nf = 0; nf < NFC; ++nf) {
      const int64_t n = min(tile0 + nf * 16 + lc, N - 1);
#pragma unroll
      for (int rf = 0; rf < RF1; ++rf)
        uu[rf][nf] = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4*>(a.kU + ((int64_t)r * N + n) * F + c0 + f0 + rf * 16 + 4 * lg));
    }
  };
#pragma unroll
  for (int ks = 0; ks < PA; ++ks) load2(a.W2T + (a.k - 1) * a.wstride, 0, ks);
  loadu(a.k - 1, 0);
  const unsigned char* yrow = Ys + lc * YSTR + lg * 16;
  int par = 0;  // G buffer of the chunk
  for (int r = a.k - 1; r >= 0; --r) {
    const uint4* W2p = a.W2T + r * a.wstride;
    const uint4* W1p = a.W1T + r * a.wstride;
    put_y(r + 1);
    // fp32: the repeat's product is summed from zero and added to dY_{r+1} once (its
    // terms are far smaller than dY: summed onto it, each would be rounded at dY's size)
    f32x4 yf[RF2][NFC];
    if constexpr (!BF) zero(yf);
    f32x4(&ya)[RF2][NFC] = BF ? y : yf;
    __syncthreads();
    for (int c0 = 0; c0 < F; c0 += FC) {
#pragma unroll
      for (int ks = 0; ks < KC; ++ks)
#pragma unroll
        for (int rf = 0; rf < RF2; ++rf) wb[ks][rf] = W1p[((c0 / M::KS + ks) * NB2 + d0 / 16 + rf) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
      f32x4 u[RF1][NFC];
#pragma unroll
      for (int rf = 0; rf < RF1; ++rf)
#pragma unroll
        for (int nf = 0; nf < NFC; ++nf) u[rf][nf] = f32x4{0.f, 0.f, 0.f, 0.f};
      uint4 bb[PL + 1][NFC];
      auto ldy = [&](int ks) {
#pragma unroll
        for (int nf = 0; nf < NFC; ++nf) bb[ks % (PL + 1)][nf] = *(const uint4*)(yrow + nf * 16 * YSTR + ks * 64);
      };
#pragma unroll
      for (int ks = 0; ks < PL; ++ks) ldy(ks);
#pragma unroll
      for (int ks = 0; ks < KD; ++ks) {
        if (ks + PL < KD) ldy(ks + PL);
#pragma unroll
        for (int rf = 0; rf < RF1; ++rf)
#pragma unroll
          for (int nf = 0; nf < NFC; ++nf) M::run(u[rf][nf], wa[ks % PA][rf], bb[ks % (PL + 1)][nf]);
        if (ks + PA < KD) load2(W2p, c0, ks + PA);
        __builtin_amdgcn_sched_barrier(0);
      }
      unsigned char* Gb = Gs[par];
      par ^= 1;
#pragma unroll
      for (int nf = 0; nf < NFC; ++nf) {
        const int m = nf * 16 + lc;
        const int64_t n = tile0 + m;
#pragma unroll
        for (int rf = 0; rf < RF1; ++rf) {
          const int fl = f0 + rf * 16 + 4 * lg;
          const int64_t o = ((int64_t)r * N + n) * F + c0 + fl;
          f32x4 g;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            u[rf][nf][i] *= BF ? gelu_grad_as(uu[rf][nf][i]) : gelu_grad_f(uu[rf][nf][i]);
          put4c((OT*)(Gb + m * GSTR) + fl, u[rf][nf]);
          if (n < N) {
            put4c((OT*)a.dU + o, u[rf][nf]);
            if constexpr (!BF) {  // GELU(U), the operand of W2's gradient (kept by the bf16 forward)
#pragma unroll
              for (int i = 0; i < 4; ++i) g[i] = gelu_f(uu[rf][nf][i]);
              put4c(a.G + o, g);
            }
          }
        }
      }
      {  // the next chunk's, or the next repeat's first
        const bool more = c0 + FC < F, last = !more && r == 0;
#pragma unroll
        for (int ks = 0; ks < PA; ++ks) load2(more || last ? W2p : W2p - a.wstride, more ? c0 + FC : 0, ks);
        loadu(more || last ? r : r - 1, more ? c0 + FC : 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      const unsigned char* grow = Gb + lc * GSTR + lg * 16;
      auto ldg = [&](int ks) {
#pragma unroll
        for (int nf = 0; nf < NFC; ++nf) bb[ks % (PL + 1)][nf] = *(const uint4*)(grow + nf * 16 * GSTR + ks * 64);
      };
#pragma unroll
      for (int ks = 0; ks < PL; ++ks) ldg(ks);
#pragma unroll
      for (int ks = 0; ks < KC; ++ks) {
        if (ks + PL < KC) ldg(ks + PL);
#pragma unroll
        for (int rf = 0; rf < RF2; ++rf)
#pragma unroll
          for (int nf = 0; nf < NFC; ++nf) M::run(ya[rf][nf], wb[ks][rf], bb[ks % (PL + 1)][nf]);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!BF) {
#pragma unroll
      for (int rf = 0; rf < RF2; ++rf)
#pragma unroll
        for (int nf = 0; nf < NFC; ++nf) y[rf][nf] += yf[rf][nf];
    }
  }
  put_y(0);
  f32x4 o[RF2][NFC];
  zero(o);
  product(a.WoT, Ys, YSTR, std::integral_constant<int, KD>{}, o);
#pragma unroll
  for (int nf = 0; nf < NFC; ++nf) {
    const int64_t n = tile0 + nf * 16 + lc;
    if (n < N) {
#pragma unroll
      for (int rf = 0; rf < RF2; ++rf)
        *reinterpret_cast<f32x4*>(a.dO + n * D + d0 + rf * 16 + 4 * lg) = o[rf][nf];
    }
  }
}

template <bool BF, int D>
void launch(const ChainArgs& a, hipStream_t s) {
  // 16 windows per workgroup while that is at most one workgroup per CU, then 32
  // (each weight fragment read from L2 serves twice the windows)
  constexpr int NT = D >= 128 ? 512 : 256;
  if (a.N <= 256 * 16)
    hipLaunchKernelGGL((k_bwd_chain<BF, D, 1>), dim3((unsigned)((a.N + 15) / 16)), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((k_bwd_chain<BF, D, 2>), dim3((unsigned)((a.N + 31) / 32)), dim3(NT), 0, s, a);
}

}  // namespace

bool launch_bwd_chain(bool bf, int D, const ChainArgs& a, hipStream_t s) {
  if (a.N <= 0) return true;
#define TRACE_CHAIN(BF_, D_)     \
  if (bf == BF_ && D == D_) {    \
    launch<BF_, D_>(a, s);       \
    return true;                 \
  }
  TRACE_CHAIN(true, 64) TRACE_CHAIN(true, 128) TRACE_CHAIN(true, 256) TRACE_CHAIN(true, 512)
  TRACE_CHAIN(false, 64) TRACE_CHAIN(false, 128) TRACE_CHAIN(false, 256)
#undef TRACE_CHAIN
  return false;
}
