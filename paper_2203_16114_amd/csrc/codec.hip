// Integer code intervals of the estimate (the coding of Alg. 1, line 9).
// For logits z[256] of a window: m = max z, d_s = (m - z_s) log2(e) in float32
// (two correctly rounded operations, no contraction), u_s = trunc(256 d_s +
// 1/2) capped at 32*256 - 1, w_s = T[u_s mod 256] >> (u_s div 256) with
// T[j] = round(2^31 2^(-j/256)), and freq_s = 1 + 65280 w_s div sum w.  Past
// d_s the arithmetic is exact, so the encoder's and the decoder's launches
// (and any implementation of these steps) give the same frequencies.
#include <cmath>

#include "codec.h"

namespace {
struct QuantTab {
  uint32_t t[256];
};

// frequencies of the bytes 4 lane .. 4 lane + 3 from the window's logits at z
__device__ __forceinline__ void quantize4(const float* __restrict__ z, int lane, const QuantTab& tab, uint32_t (&f)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(z + 4 * lane);
  float m = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  const float zz[4] = {v.x, v.y, v.z, v.w};
  uint32_t wt[4];
  uint64_t S = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float d = __fmul_rn(__fsub_rn(m, zz[r]), 1.4426950408889634f);
    int u = QMAX;
    if (d < 32.0f) u = min((int)__fadd_rn(__fmul_rn(d, 256.0f), 0.5f), QMAX);
    wt[r] = tab.t[u & 255] >> (u >> 8);
    S += wt[r];
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) S += (uint64_t)__shfl_xor((long long)S, o);
#pragma unroll
  for (int r = 0; r < 4; ++r) f[r] = (uint16_t)(1 + ((uint64_t)wt[r] * QSPREAD) / S);
}

// one wave per window
__global__ __launch_bounds__(256) void k_quantize(const float* __restrict__ z, int64_t n, uint16_t* __restrict__ freq,
                                                  QuantTab tab) {
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= n) return;  // whole waves
  uint32_t f[4];
  quantize4(z + w * 256, lane, tab, f);
  *reinterpret_cast<uint2*>(freq + w * 256 + 4 * lane) = make_uint2(f[0] | (f[1] << 16), f[2] | (f[3] << 16));
}

// One position of a coder: the frequencies of a window as above, kept in the
// wave, and the interval of the stream's byte among them: a scan over the lanes'
// sums gives the cumulative frequencies and the total.  Encoding, the byte comes
// from the streams; decoding, it is the one whose interval holds code / (range /
// total), the host coder's own integer steps.  state and out are pinned host
// memory: 8 bytes read and 16 written per stream instead of a 512-byte row of
// frequencies copied to the host, whose threads summed and searched it.  Bound by
// latency (a few us a launch).  Per position of 1024 streams, d = 128, forward and
// updates included, with the coders advanced under the next forward: 144 -> 83 us.
template <bool DEC>
__global__ __launch_bounds__(256) void k_code_step(const float* __restrict__ z, int64_t n,
                                                   const RcState* __restrict__ state, uint8_t* bytes, int64_t stride,
                                                   CodedByte* __restrict__ out, QuantTab tab) {
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= n) return;  // whole waves
  RcState st{0, 0};
  int x = 0;
  if constexpr (DEC)
    st = state[w];
  else
    x = bytes[w * stride];
  uint32_t f[4];
  quantize4(z + w * 256, lane, tab, f);
  const uint32_t sum = f[0] + f[1] + f[2] + f[3];
  uint32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  const uint32_t total = __shfl(inc, 63);
  if (total - 1 > 65535u) {  // not a distribution: no finite logit (the host refuses f = 0)
    if (lane == 0) out[w] = CodedByte{0, 0, 0, 0};
    return;
  }
  uint32_t cum = inc - sum;  // of byte 4 lane
  bool mine;
  uint32_t v = 0;
  if constexpr (DEC) {
    v = min(st.code / (st.range / total), total - 1);
    mine = v >= cum && v < inc;
  } else {
    mine = lane == x >> 2;
  }
  if (!mine) return;
  int r = 0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const bool past = r == j && (DEC ? v >= cum + f[j] : (x & 3) > j);
    if (past) {
      cum += f[j];
      r = j + 1;
    }
  }
  const uint32_t fr = r == 0 ? f[0] : r == 1 ? f[1] : r == 2 ? f[2] : f[3];
  const int sym = 4 * lane + r;
  if constexpr (DEC) bytes[w * stride] = (uint8_t)sym;
  out[w] = CodedByte{cum, fr, total, (uint32_t)sym};
}

const QuantTab& quant_tab() {
  static const QuantTab tab = [] {
    QuantTab t;
    // 2^(-j/256) in extended precision, rounded to the nearest integer at 2^31
    for (int j = 0; j < 256; ++j) t.t[j] = (uint32_t)llroundl(ldexpl(exp2l(-(long double)j / 256.0L), 31));
    return t;
  }();
  return tab;
}
}  // namespace

const uint32_t* quant_table() { return quant_tab().t; }

void launch_quantize(const float* z, int64_t n, uint16_t* freq, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_quantize, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, z, n, freq, quant_tab());
}

void launch_encode_step(const float* z, int64_t n, const uint8_t* bytes, int64_t stride, CodedByte* out,
                        hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_code_step<false>), dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, z, n,
                     (const RcState*)nullptr, const_cast<uint8_t*>(bytes), stride, out, quant_tab());
}

void launch_decode_step(const float* z, int64_t n, const RcState* state, uint8_t* bytes, int64_t stride, CodedByte* out,
                        hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_code_step<true>), dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, z, n, state, bytes, stride,
                     out, quant_tab());
}
