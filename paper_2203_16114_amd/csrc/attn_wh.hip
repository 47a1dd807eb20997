// k_attn_wh: the attention block of attn.hip for launches over runs of
// consecutive positions of each stream, with the byte groups shared between the
// windows that hold them and the work cut by head: a wave forms everything of
// its heads with no barrier until the output projection.
//
// A tile is 64 consecutive windows of one stream (fewer at the end of a stream's
// run: the missing windows are computed from zero bytes and not stored).  Window
// i reads its token t from the group that starts i + g t bytes into the tile's
// bytes, so the tile holds 64 + W - g distinct groups ("group rows" o).  With
// X.W = E.W + P.W their E-parts go to LDS once (16-byte unit u of row o at
// u ^ (o & 15): conflict-free fragment reads).  Then, per head, in parts of 32
// features:
//   K^T = Wk^T . X_E^T over all group rows, q^T = Wq^T . E_last^T + (P.Wq)[T-1]
//     (E_last of window i is group row i + g (T-1));
//   a lane's accumulator quads hold group row 16 rf + lc (K) and window
//     16 nf + lc (q), features 4 lg + r of each 16-feature block.  Key row
//     i + g t of window 16 nf + lc is row (lc + g t) % 16 of fragment
//     nf + (lc + g t) / 16: for g t = 16 b + s with s > 0 each lane picks the
//     fragment its partner needs and a DPP rotation within the row of 16 brings
//     it over, once per fragment and s (for_rows);
//   scores q . (K_E[row] + (P.Wk)[t]) as partial sums over the lane's features,
//     summed over the 4 lane groups by a reduce-scatter (shuffles across 32 and
//     16 lanes) that leaves lane (lg, lc) with the T scores of window
//     16 lg + lc: softmax in the lane; shuffles hand the weights to the lanes
//     that hold each window;
//   V^T = Wv^T . X_E^T and O = sum_t a_t (V_E[row] + (P.Wv)[t]) with the same row
//     selection, kept as operand values until every wave is done with the group
//     rows, over which the O tile is then written;
//   h0^T = Wo^T . O^T + X_last (the waves split the output features), rows staged
//     over the O tile and written whole.
// A window's result is the same bit for bit wherever it sits in a tile.
//
// Workgroups have 4 waves (two workgroups per CU, whose vector and matrix phases
// then interleave; the waves of one workgroup run the same phase together) except
// at 1024-byte rows (d = 512, fp32 d = 256), where the group rows of one tile fill most
// of the LDS: 8 waves, and in models of fewer heads: one wave per head.
//
// Bound by the MFMAs and the vector work of scores and weighted sums (about half
// of the cycles each at d = 256).  Measured against the kernels these launches
// took before: d = 256, 2^20 windows (8 waves of one head each, 157 KB of LDS, one
// workgroup per CU) 1.244 -> 1.166 ms; 1021 streams x 203 positions (per-token
// kernel) 690 -> 314 us; d = 512, 2^17 windows (per-token kernel, as the
// shared-group tile did not fit the LDS) 1.494 -> 0.508 ms; d = 128, 2^18 windows
// (shared-group kernel by alignment class) 186 -> 111 us; fp32, d = 128, 2^16 windows
// (per-token kernel; bound by its fp32 MFMAs, T times as many) 342 -> 105 us.
#include <type_traits>

#include "kcommon.h"
#include "kernels.h"

namespace {

template <bool BF, int T, int G, int D, int DH, int NW_>
struct WhShape {
  typedef Mma<BF> M;
  static constexpr int ES = BF ? 2 : 4, EPU = 16 / ES;  // bytes per operand element, elements per 16-byte unit
  static constexpr int MA = 64, W = T * G, H = D / DH;
  static constexpr int NW = NW_, HPW = H / NW, NP = DH / 32;  // heads per wave, 32-feature parts per head
  static constexpr int NRF = (MA + W - G + 15) / 16;                        // group-row fragments
  static constexpr int NWF = MA / 16;                                       // window fragments
  static constexpr int KSTEPS = D / M::KS, NB = D / 16;
  static constexpr int XSTR = D * ES, NUR = D / EPU, XM = (NUR >= 16 ? 16 : NUR) - 1;  // units per row, swizzle mask
  static constexpr int HSTR = D + 4;  // h0 rows staged for the write (floats, padded)
  static constexpr int XG = NRF * 16 * XSTR > MA * HSTR * 4 ? NRF * 16 * XSTR : MA * HSTR * 4;
  static constexpr int WB = NRF * 16 + G;
  static constexpr int PWS = T * DH;  // floats of one head's rows of P.Wk or P.Wv
  static constexpr int LDS = XG + NW * PWS * 4 + WB;
  static constexpr bool ok = H % NW == 0 && H >= NW && HPW <= 2 && LDS <= 160 * 1024;
};

// four consecutive operand elements as floats
__device__ __forceinline__ f32x4 four(const uint16_t* p) {
  const uint2 b = *reinterpret_cast<const uint2*>(p);
  return f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16),
               __uint_as_float(b.y & 0xffff0000u)};
}
__device__ __forceinline__ f32x4 four(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// x from lane (lc + S) % 16 of the same row of 16 lanes (DPP row_ror: lane i
// receives lane i - n)
template <int S>
__device__ __forceinline__ float from_up(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + (16 - S), 0xF, 0xF, false));
}

// f(t, nf, row, p0, p1) for every token t and window fragment nf: row[fr] the
// accumulator quads of key row g t + (16 nf + lc), p0 and p1 the floats at
// pw + t * STR and 16 further (token t's positional rows).  Token t = b NS + si has
// g t = 16 b + g si: its rows are fragment nf + b shifted up by S = g si lanes (lane
// lc takes lane lc + S of that fragment, or lane lc + S - 16 of the next).  A
// window fragment meets the tokens in the order of (si, b).
template <int T, int G, int STR, int NRF, int NWF, class F>
__device__ __forceinline__ void for_rows(const f32x4 (&acc)[NRF][2], int lc, const float* pw, F&& f) {
  constexpr int NS = 16 / G, NB_ = T / NS;  // shifts; tokens per shift
  auto shift = [&](auto sh_c) {
    constexpr int si = decltype(sh_c)::value, S = G * si;
    float4 p0[NB_], p1[NB_];
#pragma unroll
    for (int b = 0; b < NB_; ++b) {
      p0[b] = *reinterpret_cast<const float4*>(pw + (b * NS + si) * STR);
      p1[b] = *reinterpret_cast<const float4*>(pw + (b * NS + si) * STR + 16);
    }
#pragma unroll
    for (int j = 0; j < NWF + NB_ - 1; ++j) {
      f32x4 row[2];
      if constexpr (S == 0) {
        row[0] = acc[j][0];
        row[1] = acc[j][1];
      } else {
        static_assert(NWF + NB_ - 1 < NRF, "rows");
        const bool own = lc >= S;  // this lane's partner is lc - S (same fragment) or lc - S + 16
#pragma unroll
        for (int fr = 0; fr < 2; ++fr)
#pragma unroll
          for (int r = 0; r < 4; ++r) row[fr][r] = from_up<S>(own ? acc[j][fr][r] : acc[j + 1][fr][r]);
      }
#pragma unroll
      for (int b = 0; b < NB_; ++b)
        if (j - b >= 0 && j - b < NWF) f(b * NS + si, j - b, row, p0[b], p1[b]);
      __builtin_amdgcn_sched_barrier(0);  // one row fragment at a time: registers
    }
  };
  shift(std::integral_constant<int, 0>{});
  shift(std::integral_constant<int, 1>{});
  if constexpr (NS == 4) {
    shift(std::integral_constant<int, 2>{});
    shift(std::integral_constant<int, 3>{});
  }
}

template <bool BF, int T, int G, int D, int DH, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_attn_wh(AttnArgs a, int64_t t0, int tps) {
  typedef Mma<BF> M;
  typedef typename M::T OT;
  typedef WhShape<BF, T, G, D, DH, NW> S;
  constexpr int ES = S::ES, EPU = S::EPU, NUR = S::NUR;
  constexpr int HPW = S::HPW, NP = S::NP, MA = S::MA, W = S::W, NRF = S::NRF, NWF = S::NWF;
  constexpr int KSTEPS = S::KSTEPS, NB = S::NB, XSTR = S::XSTR, XM = S::XM, HSTR = S::HSTR, NT = 64 * NW;
  constexpr int EPB = D / G;         // features per byte embedding
  constexpr int QOFF = (T - 1) * G;  // group row of window 0's last token
  constexpr int QFW = NB / NW;
  static_assert(S::ok && NB % NW == 0, "shape");
  __shared__ __align__(16) unsigned char Xg[S::XG];  // group rows (bf16), then O rows (bf16), then h0 rows (fp32)
  __shared__ __align__(16) float PWh[NW][S::PWS];    // this wave's head rows of P.Wk, then of P.Wv
  __shared__ uint8_t Wb[S::WB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, lc = lane & 15;
  const int64_t st = (t0 + blockIdx.x) / tps;  // stream; tiles are numbered stream by stream
  const int s0 = (int)(t0 + blockIdx.x - st * tps) * MA;
  const int nv = min(MA, a.w.n_steps - s0);                // windows of the tile
  const int64_t l0 = st * a.w.n_steps + s0 - a.w.n0;       // local index of window 0
  if (l0 >= a.w.N || l0 + nv <= 0) return;
  const int i_lo = (int)max((int64_t)0, -l0), i_hi = (int)min((int64_t)nv, a.w.N - l0);  // windows stored
  const OT* __restrict__ E = (const OT*)a.E;
  const OT* __restrict__ P = (const OT*)a.P;

  // the tile's bytes: Wb[k] = stream byte at (target of window 0) - W + k, zero
  // past the last window's
  {
    const uint8_t* src = a.w.streams + st * a.w.stride + a.w.pos0 + s0 - W;
    for (int k = tid; k < S::WB; k += NT) Wb[k] = k < nv + W - 1 ? src[k] : 0;
  }
  __syncthreads();
  // group rows o: unit u holds features EPU u .. + EPU - 1, from byte o + u / (units per byte)
  {
    constexpr int UPB = EPB / EPU;
    constexpr int NUT = NRF * 16 * NUR / NT, NU = NUT > 16 ? NUT / 2 : NUT;  // all or half of the loads in flight
    static_assert(NRF * 16 * NUR % NT == 0 && NUT % NU == 0, "group rows");
#pragma unroll 1
    for (int r0 = 0; r0 < NUT; r0 += NU) {
      uint4 ev[NU];
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        const int q = tid + NT * (r0 + r), o = q / NUR, u = q % NUR;
        const int byte = Wb[o + u / UPB];
        ev[r] = *reinterpret_cast<const uint4*>(E + byte * EPB + (u % UPB) * EPU);
      }
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        const int q = tid + NT * (r0 + r), o = q / NUR, u = q % NUR;
        *(uint4*)(Xg + o * XSTR + 16 * (u ^ (o & XM))) = ev[r];
      }
    }
  }
  __syncthreads();

  // fragment reads of rows m (m & 15 = c) at units 4 ks + lg: byte 64 (ks & ~3) + off[ks & 3]
  auto swz = [&](int c, int (&off)[4]) {
    const int q = (c & XM) >> 2, p = lg ^ (c & 3);
#pragma unroll
    for (int j = 0; j < 4; ++j) off[j] = 16 * (((j ^ q) << 2) | p);
  };
  int xo[4], qo[4];
  swz(lc, xo);
  swz((QOFF + lc) & 15, qo);

  float* pw = PWh[wave];
  constexpr int NPW4 = S::PWS / 4 / 64 > 0 ? S::PWS / 4 / 64 : 1;  // float4 per lane of a head's P rows
  auto load_pw = [&](int which, int h, float4 (&v)[NPW4]) {
    const float* src = a.PW + (int64_t)(which * T) * D + h * DH;
#pragma unroll
    for (int i = 0; i < NPW4; ++i) {
      const int q = min(lane + 64 * i, S::PWS / 4 - 1);
      v[i] = *reinterpret_cast<const float4*>(src + (q / (DH / 4)) * D + 4 * (q % (DH / 4)));
    }
  };
  auto put_pw = [&](const float4 (&v)[NPW4]) {
#pragma unroll
    for (int i = 0; i < NPW4; ++i)
      if (lane + 64 * i < S::PWS / 4) *reinterpret_cast<float4*>(pw + 4 * (lane + 64 * i)) = v[i];
  };

  typedef typename std::conditional<BF, uint2, f32x4>::type OQ;
  OQ opk[HPW][NP][NWF][2];  // O of this wave's heads as operand values
#pragma unroll
  for (int hp = 0; hp < HPW; ++hp) {
    const int h = wave * HPW + hp;
    float4 pv4[NPW4];
    {
      float4 pk4[NPW4];
      load_pw(1, h, pk4);
      load_pw(2, h, pv4);
      put_pw(pk4);
    }
    float sc[NWF][T];
#pragma unroll
    for (int nf = 0; nf < NWF; ++nf)
#pragma unroll
      for (int t = 0; t < T; ++t) sc[nf][t] = 0.f;
#pragma unroll
    for (int part = 0; part < NP; ++part) {
      // K over all group rows and q over the windows' last tokens, 32 features
      f32x4 kacc[NRF][2], qacc[NWF][2];
#pragma unroll
      for (int rf = 0; rf < NRF; ++rf) kacc[rf][0] = kacc[rf][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int nf = 0; nf < NWF; ++nf) qacc[nf][0] = qacc[nf][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      {
        const uint4* Wkh = a.Wk + ((h * NP + part) * 2) * 64 + lane;
        const uint4* Wqh = a.Wq + ((h * NP + part) * 2) * 64 + lane;
        uint4 wk[2][2], wq[2][2];
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) {
          wk[0][fr] = Wkh[fr * 64];
          wq[0][fr] = Wqh[fr * 64];
        }
#pragma unroll 1
        for (int k4 = 0; k4 < KSTEPS; k4 += 4) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int kn = min(k4 + j + 1, KSTEPS - 1);  // (the last step's prefetch is not used)
#pragma unroll
            for (int fr = 0; fr < 2; ++fr) {
              wk[(j + 1) & 1][fr] = Wkh[(kn * NB + fr) * 64];
              wq[(j + 1) & 1][fr] = Wqh[(kn * NB + fr) * 64];
            }
            const int kb = k4 * 64;
            uint4 bg[NRF], bq[NWF];
#pragma unroll
            for (int rf = 0; rf < NRF; ++rf) bg[rf] = *(const uint4*)(Xg + (16 * rf + lc) * XSTR + kb + xo[j]);
#pragma unroll
            for (int nf = 0; nf < NWF; ++nf) bq[nf] = *(const uint4*)(Xg + (QOFF + 16 * nf + lc) * XSTR + kb + qo[j]);
#pragma unroll
            for (int rf = 0; rf < NRF; ++rf)
#pragma unroll
              for (int fr = 0; fr < 2; ++fr) M::run(kacc[rf][fr], wk[j & 1][fr], bg[rf]);
#pragma unroll
            for (int nf = 0; nf < NWF; ++nf)
#pragma unroll
              for (int fr = 0; fr < 2; ++fr) M::run(qacc[nf][fr], wq[j & 1][fr], bq[nf]);
            __builtin_amdgcn_sched_barrier(0);  // keep each step's loads in it
          }
        }
      }
      {
        const float* pq = a.PW + (T - 1) * D + h * DH + part * 32 + 4 * lg;
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) {
          const float4 p4 = *reinterpret_cast<const float4*>(pq + 16 * fr);
#pragma unroll
          for (int nf = 0; nf < NWF; ++nf) {
            qacc[nf][fr][0] += p4.x;
            qacc[nf][fr][1] += p4.y;
            qacc[nf][fr][2] += p4.z;
            qacc[nf][fr][3] += p4.w;
          }
        }
      }
      // scores: partial sums over the lane's 8 features of this part
      const float* pk = pw + part * 32 + 4 * lg;
      for_rows<T, G, DH, NRF, NWF>(kacc, lc, pk, [&](int t, int nf, const f32x4 (&k)[2], const float4& p0, const float4& p1) {
        const f32x4& q0 = qacc[nf][0];
        const f32x4& q1 = qacc[nf][1];
        float s = q0[0] * (k[0][0] + p0.x) + q0[1] * (k[0][1] + p0.y) + q0[2] * (k[0][2] + p0.z) +
                  q0[3] * (k[0][3] + p0.w);
        s += q1[0] * (k[1][0] + p1.x) + q1[1] * (k[1][1] + p1.y) + q1[2] * (k[1][2] + p1.z) + q1[3] * (k[1][3] + p1.w);
        sc[nf][t] += s;
      });
      // the sums formed here (see the asm below)
#pragma unroll
      for (int nf = 0; nf < NWF; ++nf)
#pragma unroll
        for (int t = 0; t < T; ++t) asm volatile("" : "+v"(sc[nf][t]));
    }
    // reduce-scatter over the lane groups: lane (lg, lc) ends with window 16 lg + lc
    float stt[T];
    {
      const bool up = lg >= 2, od = (lg & 1) != 0;
      float r1[2][T];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float keep = up ? sc[2 + j][t] : sc[j][t];
          const float send = up ? sc[j][t] : sc[2 + j][t];
          r1[j][t] = keep + __shfl_xor(send, 32, 64);
        }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float keep = od ? r1[1][t] : r1[0][t];
        const float send = od ? r1[0][t] : r1[1][t];
        stt[t] = keep + __shfl_xor(send, 16, 64);
      }
    }
    {
      const float scale = a.scale;
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        stt[t] *= scale;
        mx = fmaxf(mx, stt[t]);
      }
      float sm = 0.f;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        stt[t] = expf(stt[t] - mx);
        sm += stt[t];
      }
      const float rs = __builtin_amdgcn_rcpf(sm);
#pragma unroll
      for (int t = 0; t < T; ++t) stt[t] *= rs;
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_wave_barrier();  // (the rows of P.Wk are read)
    put_pw(pv4);

#pragma unroll
    for (int part = 0; part < NP; ++part) {
      // V over all group rows, 32 features
      f32x4 vacc[NRF][2];
#pragma unroll
      for (int rf = 0; rf < NRF; ++rf) vacc[rf][0] = vacc[rf][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      {
        const uint4* Wvh = a.Wv + ((h * NP + part) * 2) * 64 + lane;
        uint4 wv[2][2];
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) wv[0][fr] = Wvh[fr * 64];
#pragma unroll 1
        for (int k4 = 0; k4 < KSTEPS; k4 += 4) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int kn = min(k4 + j + 1, KSTEPS - 1);
#pragma unroll
            for (int fr = 0; fr < 2; ++fr) wv[(j + 1) & 1][fr] = Wvh[(kn * NB + fr) * 64];
            const int kb = k4 * 64;
            uint4 bg[NRF];
#pragma unroll
            for (int rf = 0; rf < NRF; ++rf) bg[rf] = *(const uint4*)(Xg + (16 * rf + lc) * XSTR + kb + xo[j]);
#pragma unroll
            for (int rf = 0; rf < NRF; ++rf)
#pragma unroll
              for (int fr = 0; fr < 2; ++fr) M::run(vacc[rf][fr], wv[j & 1][fr], bg[rf]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      // O[window 16 nf + lc][features 16 fr + 4 lg + r] of this part; the weights
      // of window 16 nf + lc are in lane (nf, lc)
      f32x4 o[NWF][2];
#pragma unroll
      for (int nf = 0; nf < NWF; ++nf) o[nf][0] = o[nf][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* pv = pw + part * 32 + 4 * lg;
      for_rows<T, G, DH, NRF, NWF>(vacc, lc, pv, [&](int t, int nf, const f32x4 (&v)[2], const float4& p0, const float4& p1) {
        const float at = __shfl(stt[t], 16 * nf + lc, 64);
        o[nf][0][0] += at * (v[0][0] + p0.x);
        o[nf][0][1] += at * (v[0][1] + p0.y);
        o[nf][0][2] += at * (v[0][2] + p0.z);
        o[nf][0][3] += at * (v[0][3] + p0.w);
        o[nf][1][0] += at * (v[1][0] + p1.x);
        o[nf][1][1] += at * (v[1][1] + p1.y);
        o[nf][1][2] += at * (v[1][2] + p1.z);
        o[nf][1][3] += at * (v[1][3] + p1.w);
      });
#pragma unroll
      for (int nf = 0; nf < NWF; ++nf)
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) {
          // formed here: left to the compiler, the sums sink to their use behind
          // the next head's products and spill the value rows
          if constexpr (BF) {
            uint32_t lo = pack_bf16x2(o[nf][fr][0], o[nf][fr][1]), hi = pack_bf16x2(o[nf][fr][2], o[nf][fr][3]);
            asm volatile("" : "+v"(lo), "+v"(hi));
            opk[hp][part][nf][fr] = make_uint2(lo, hi);
          } else {
            asm volatile("" : "+v"(o[nf][fr]));
            opk[hp][part][nf][fr] = o[nf][fr];
          }
        }
    }
    __builtin_amdgcn_wave_barrier();  // (the rows of P.Wv are read)
  }
  __syncthreads();  // the group rows are no longer needed: the O rows go over them
#pragma unroll
  for (int hp = 0; hp < HPW; ++hp)
#pragma unroll
    for (int part = 0; part < NP; ++part)
#pragma unroll
      for (int nf = 0; nf < NWF; ++nf)
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) {
          const int m = 16 * nf + lc;
          const int oe = (wave * HPW + hp) * DH + part * 32 + 16 * fr + 4 * lg;
          *reinterpret_cast<OQ*>(Xg + m * XSTR + 16 * ((oe / EPU) ^ (m & XM)) + (oe % EPU) * ES) = opk[hp][part][nf][fr];
        }
  __syncthreads();

  // h0^T = Wo^T . O^T + X_last (fp32: E + P of the last token)
  f32x4 acc[QFW][NWF];
#pragma unroll
  for (int qi = 0; qi < QFW; ++qi)
#pragma unroll
    for (int nf = 0; nf < NWF; ++nf) acc[qi][nf] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    const uint4* Wop = a.Wo + (wave * QFW) * 64 + lane;
    uint4 wo[2][QFW];
#pragma unroll
    for (int qi = 0; qi < QFW; ++qi) wo[0][qi] = Wop[qi * 64];
#pragma unroll 1
    for (int k4 = 0; k4 < KSTEPS; k4 += 4) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kn = min(k4 + j + 1, KSTEPS - 1);
#pragma unroll
        for (int qi = 0; qi < QFW; ++qi) wo[(j + 1) & 1][qi] = Wop[(kn * NB + qi) * 64];
        uint4 bo[NWF];
#pragma unroll
        for (int nf = 0; nf < NWF; ++nf) bo[nf] = *(const uint4*)(Xg + (16 * nf + lc) * XSTR + k4 * 64 + xo[j]);
#pragma unroll
        for (int qi = 0; qi < QFW; ++qi)
#pragma unroll
          for (int nf = 0; nf < NWF; ++nf) M::run(acc[qi][nf], wo[j & 1][qi], bo[nf]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __syncthreads();  // the O rows are no longer needed: the h0 rows go over them
  float* Hs = reinterpret_cast<float*>(Xg);
#pragma unroll
  for (int qi = 0; qi < QFW; ++qi) {
    const int d = (wave * QFW + qi) * 16 + 4 * lg;
    const int j = d / EPB, cc = d - j * EPB;
    const f32x4 pb = four(P + (T - 1) * D + d);
#pragma unroll
    for (int nf = 0; nf < NWF; ++nf) {
      const int m = 16 * nf + lc;
      const f32x4 eb = four(E + Wb[m + QOFF + j] * EPB + cc);
      float4 r;
      r.x = acc[qi][nf][0] + (eb[0] + pb[0]);
      r.y = acc[qi][nf][1] + (eb[1] + pb[1]);
      r.z = acc[qi][nf][2] + (eb[2] + pb[2]);
      r.w = acc[qi][nf][3] + (eb[3] + pb[3]);
      *reinterpret_cast<float4*>(Hs + m * HSTR + d) = r;
    }
  }
  __syncthreads();
  for (int m = i_lo + wave; m < i_hi; m += NW) {
    float* dst = a.h0 + (l0 + m) * D;
#pragma unroll
    for (int c = 4 * lane; c < D; c += 256)
      *reinterpret_cast<float4*>(dst + c) = *reinterpret_cast<const float4*>(Hs + m * HSTR + c);
  }
}

template <bool BF, int T, int G, int D, int DH, int NW>
void launch_nw(const AttnArgs& a, int64_t t0, int tps, int64_t tiles, hipStream_t s) {
  hipLaunchKernelGGL((k_attn_wh<BF, T, G, D, DH, NW>), dim3((unsigned)tiles), dim3(64 * NW), 0, s, a, t0, tps);
}

template <bool BF, int T, int G, int D, int DH>
void launch(const AttnArgs& a, hipStream_t s) {
  // one block per 64 positions of a stream, from the launch's first window's tile
  // to its last window's
  constexpr int H = D / DH;
  const int tps = (a.w.n_steps + 63) / 64;
  auto tile = [&](int64_t n) { return n / a.w.n_steps * tps + n % a.w.n_steps / 64; };
  const int64_t t0 = tile(a.w.n0), tiles = tile(a.w.n0 + a.w.N - 1) - t0 + 1;
  if constexpr (H <= 4) {
    launch_nw<BF, T, G, D, DH, H>(a, t0, tps, tiles, s);
  } else if constexpr (D * WhShape<BF, T, G, D, DH, 8>::ES == 1024) {
    launch_nw<BF, T, G, D, DH, 8>(a, t0, tps, tiles, s);
  } else {
    // at most one tile per CU: the tile's own latency counts, and eight waves of
    // one head each take less than four of two (64 tiles at d = 256: 21 / 28 us)
    if (tiles <= 256) return launch_nw<BF, T, G, D, DH, 8>(a, t0, tps, tiles, s);
    launch_nw<BF, T, G, D, DH, 4>(a, t0, tps, tiles, s);
  }
}

}  // namespace

bool launch_attn_wh(bool bf, int T, int D, int DH, const AttnArgs& a, hipStream_t s) {
  // Where a stream's run of positions fills its tiles badly, the per-token
  // kernel: it projects T + 1 rows a window (the last one twice: q and Wo) and a
  // tile here NR + 64, filled or not.  Measured (us, this / per token) on 1021
  // streams: T = 8, g = 8, d = 256 (line at 22 positions): 16 positions 71 / 64,
  // 24 74 / 103; d = 512: 205 / 183, 217 / 268; T = 8, g = 4, d = 128 (line at 18):
  // 30 / 26, 32 / 46; fp32 at 24 positions, d = 128: 102 / 173.
  // Small calls of narrow models are the per-token kernel's too: its 16- and
  // 32-window tiles spread them over more CUs, and a tile here has only as many
  // waves as heads.  d = 128: 4096 windows 14 / 13 (fp32 33 / 30), 12992 17 / 26
  // (36 / 90); d = 64 (one head): 16384 33 / 20, 32768 35 / 38.
  // The rules look at the whole call, so its chunks agree.
  const int tps = (a.w.n_steps + 63) / 64, nr = (64 + (T - 1) * a.g + 15) / 16 * 16;
  if ((int64_t)a.w.n_steps * (T + 1) < (int64_t)tps * (nr + 64)) return false;
  if (D <= 128 && a.total <= (D == 64 ? 24576 : 6144)) return false;
#define TRACE_WH(BF_, T_, G_, D_, DH_)                             \
  if (bf == BF_ && T == T_ && a.g == G_ && D == D_ && DH == DH_) { \
    launch<BF_, T_, G_, D_, DH_>(a, s);                            \
    return true;                                                   \
  }
#define TRACE_WH4(BF_, D_, DH_) \
  TRACE_WH(BF_, 8, 8, D_, DH_) TRACE_WH(BF_, 8, 4, D_, DH_) TRACE_WH(BF_, 4, 8, D_, DH_) TRACE_WH(BF_, 4, 4, D_, DH_)
  TRACE_WH4(true, 128, 32) TRACE_WH4(true, 128, 64) TRACE_WH4(true, 256, 32) TRACE_WH4(true, 256, 64) TRACE_WH4(true, 512, 64)
  TRACE_WH4(false, 64, 32) TRACE_WH4(false, 64, 64) TRACE_WH4(false, 128, 32) TRACE_WH4(false, 128, 64)
  TRACE_WH4(false, 256, 32) TRACE_WH4(false, 256, 64)
#undef TRACE_WH4
#undef TRACE_WH
  return false;
}
