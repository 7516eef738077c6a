// float32 path: used by fp32 models (small shapes, where launch latency, not
// arithmetic, bounds the step).  float32 storage, products and softmax sums in
// float64 on the matrix cores (v_mfma_f64_16x16x4: a float32 x float32 product
// is exact in float64), so each stored value is the float32 rounding of a
// nearly exact result; fixed reduction order everywhere, so results are
// run-to-run identical.
//
// v_mfma_f64_16x16x4 layout (lane l): A operand row l % 16, B operand column
// l % 16, both k slot l / 16; D register r: row 4 r + l / 16, column l % 16.
// The four k slots are summed, so which k a slot stands for is free as long as
// A and B agree: here slot g of the four MFMAs of a 16-k step stands for k =
// 4 g + e, e = 0 .. 3, and a lane's operands of the step are one float4.
#include <algorithm>

#include "kernels.h"

namespace dllm {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// ---- GEMM -------------------------------------------------------------------
// C = A W^T with fused epilogues.  A workgroup of NWV waves owns 16 MT rows x
// two 16-column blocks, the pair an epilogue needs together: dimensions j and
// j + hd/2 of one head (QKV), gate and up of the same 16 columns (SWIGLU), or
// two neighbouring blocks (RESID, STORE).  Wave w takes the 16-k steps w, w +
// NWV, ..: operands go straight from memory into registers (FU steps in flight,
// no LDS in the loop), and the waves' float64 accumulators are summed in wave
// order through LDS, where wave r < 4 finishes accumulator register r.
//
// What bounds it: at these sizes the latency of one round of loads, so few
// launches and short k chains per wave.  The kernel this replaces (one float64
// dot product per thread out of LDS, one launch per weight tensor, RoPE, SwiGLU
// and the norms in launches of their own) took 9.8 us a launch at 96 rows and
// 23 us at 948 (tiny model, 256 x 256); now 6.3 / 8.4 us for all of q/k/v / gate/up
// with norm and epilogue at 96 rows, 19 / 30 us at 948 (22 TFLOP/s; 31 at 5840
// rows, of the 54 a float64 library product reaches).
//
// With NORM the rows of A are RMS-normalised first, from the same registers
// (every wave holds its share of the row, its NORM steps, K <= 16 NORM NWV), so
// the norm costs no launch; column block 0 also stores the normed rows.
constexpr int FU = 4;             // 16-k steps in flight per wave
constexpr int NORM_MAX_K = 512;   // widest row a NORM launch holds (8 steps on four waves)

template <int EPI, int MT, int NWV, bool VEC, int NORM>
__global__ void __launch_bounds__(64 * NWV) gemm_f32_kernel(GemmF32 g) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ double red[NWV][MT * 8][64];
  __shared__ double ssq[NORM > 0 ? NWV : 1][16 * MT];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15, kg = lane >> 4;
  const int m0 = blockIdx.y * 16 * MT, t = blockIdx.x;
  const int KS = (g.K + 15) / 16;

  // weight rows of the two column blocks (clamped past the end: never stored)
  const float* w[2];
  if (EPI == F32_QKV) {
    const int half = g.hd / 2, per = half / 16, head = t / per, j0 = 16 * (t % per) + row;
    const int H1 = head - g.Hq, H2 = H1 - g.Hkv;
    const float* base = H1 < 0 ? g.W0 + (size_t)head * g.hd * g.K
                        : H2 < 0 ? g.W1 + (size_t)H1 * g.hd * g.K : g.W2 + (size_t)H2 * g.hd * g.K;
    w[0] = base + (size_t)j0 * g.K;
    w[1] = base + (size_t)(j0 + half) * g.K;
  } else if (EPI == F32_SWIGLU) {
    const int f = min(16 * t + row, g.N - 1);
    w[0] = g.W0 + (size_t)f * g.K;
    w[1] = g.W1 + (size_t)f * g.K;
  } else {
    w[0] = g.W0 + (size_t)min(32 * t + row, g.N - 1) * g.K;
    w[1] = g.W0 + (size_t)min(32 * t + 16 + row, g.N - 1) * g.K;
  }
  // row m of the product reads row (m / rows) Ls + r0 + m % rows of A (the
  // head's rows of every sequence; otherwise rows = M, Ls = r0 = 0)
  const float* a[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = min(m0 + 16 * mt + row, g.M - 1);
    a[mt] = g.A + ((size_t)(m / g.rows) * g.Ls + g.r0 + m % g.rows) * g.K;
  }
  auto ld = [&](const float* p, int s) {
    const int k = 16 * s + 4 * kg;
    if (VEC) return *reinterpret_cast<const float4*>(p + k);
    return make_float4(k < g.K ? p[k] : 0.f, k + 1 < g.K ? p[k + 1] : 0.f, k + 2 < g.K ? p[k + 2] : 0.f,
                       k + 3 < g.K ? p[k + 3] : 0.f);
  };
  f64x4_t acc[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) acc[mt][nb] = f64x4_t{0., 0., 0., 0.};
  auto mma = [&](const float4 (&av)[MT], const float4 (&bv)[2]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[mt][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(&av[mt].x)[e], (double)(&bv[nb].x)[e],
                                                             acc[mt][nb], 0, 0, 0);
  };

  // what the epilogue reads besides the sums, loaded now: the RoPE values of the
  // rows this wave finishes, or the residual it adds to
  float pre[MT][2] = {};
  if (wave < 4) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = min(m0 + 16 * mt + 4 * wave + kg, g.M - 1);
      if (EPI == F32_QKV) {
        const int half = g.hd / 2, per = half / 16, head = t / per, j = 16 * (t % per) + row;
        if (head < g.Hq + g.Hkv) {
          const size_t at = (size_t)(g.pos0 + m % g.Lq) * half + j;
          pre[mt][0] = g.cosb[at];
          pre[mt][1] = g.sinb[at];
        }
      } else if (EPI == F32_RESID) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) pre[mt][nb] = g.C[(size_t)m * g.N + min(32 * t + 16 * nb + row, g.N - 1)];
      }
    }
  }

  if constexpr (NORM > 0) {
    constexpr int NS = NORM;
    float4 av[NS][MT], bv[NS][2], gn[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int s = wave + NWV * i;
      if (s < KS) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[i][mt] = ld(a[mt], s);
        bv[i][0] = ld(w[0], s);
        bv[i][1] = ld(w[1], s);
        gn[i] = ld(g.gain, s);
      } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[i][mt] = make_float4(0.f, 0.f, 0.f, 0.f);
        bv[i][0] = bv[i][1] = gn[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      double ss = 0.0;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const float4 v = av[i][mt];
        ss += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
      }
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      if (kg == 0) ssq[wave][16 * mt + row] = ss;
    }
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      double tot = 0.0;
#pragma unroll
      for (int v = 0; v < NWV; ++v) tot += ssq[v][16 * mt + row];
      const float rstd = (float)(1.0 / sqrt(tot / (double)g.K + (double)g.eps));
      const int m = m0 + 16 * mt + row;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int s = wave + NWV * i;
        if (s >= KS) continue;
        const float4 gv = gn[i];
        float4& v = av[i][mt];
        v = make_float4(v.x * rstd * gv.x, v.y * rstd * gv.y, v.z * rstd * gv.z, v.w * rstd * gv.w);
        if (t == 0 && m < g.M) *reinterpret_cast<float4*>(g.normed + (size_t)m * g.K + 16 * s + 4 * kg) = v;
      }
    }
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if (wave + NWV * i < KS) mma(av[i], bv[i]);
  } else {
    // FU steps per round; the next round's loads are issued before this one's MFMAs
    float4 av[2][FU][MT], bv[2][FU][2];
    auto load = [&](int i0, auto set_c) {
      constexpr int set = decltype(set_c)::value;
#pragma unroll
      for (int i = 0; i < FU; ++i) {
        const int s = wave + NWV * (i0 + i);
        if (s >= KS) break;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[set][i][mt] = ld(a[mt], s);
        bv[set][i][0] = ld(w[0], s);
        bv[set][i][1] = ld(w[1], s);
      }
    };
    auto run = [&](int i0, auto set_c) {
      constexpr int set = decltype(set_c)::value;
#pragma unroll
      for (int i = 0; i < FU; ++i)
        if (wave + NWV * (i0 + i) < KS) mma(av[set][i], bv[set][i]);
    };
    const int n = wave < KS ? (KS - wave + NWV - 1) / NWV : 0;
    using c0 = std::integral_constant<int, 0>;
    using c1 = std::integral_constant<int, 1>;
    load(0, c0{});
    for (int i0 = 0; i0 < n; i0 += 2 * FU) {
      load(i0 + FU, c1{});
      run(i0, c0{});
      load(i0 + 2 * FU, c0{});
      run(i0 + FU, c1{});
    }
  }

#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(mt * 2 + nb) * 4 + r][lane] = acc[mt][nb][r];
  __syncthreads();
  if (wave >= 4) return;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m0 + 16 * mt + 4 * wave + kg;  // accumulator register `wave`
    double c[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      c[nb] = red[0][(mt * 2 + nb) * 4 + wave][lane];
#pragma unroll
      for (int v = 1; v < NWV; ++v) c[nb] += red[v][(mt * 2 + nb) * 4 + wave][lane];
    }
    if (m >= g.M) continue;
    if (EPI == F32_QKV) {
      const int half = g.hd / 2, per = half / 16, head = t / per, j = 16 * (t % per) + row;
      const int b = m / g.Lq, i = m - b * g.Lq, pos = g.pos0 + i;
      const float x1 = (float)c[0], x2 = (float)c[1];
      if (head < g.Hq + g.Hkv) {
        const float cs = pre[mt][0], sn = pre[mt][1];
        float* dst = head < g.Hq ? g.q + (((size_t)b * g.Hq + head) * g.Lq + i) * g.hd
                                 : g.k + (((size_t)b * g.Hkv + (head - g.Hq)) * g.L + pos) * g.hd;
        dst[j] = x1 * cs - x2 * sn;
        dst[j + half] = x2 * cs + x1 * sn;
      } else {
        float* dst = g.vt + ((size_t)b * g.Hkv + (head - g.Hq - g.Hkv)) * g.hd * g.L + pos;
        dst[(size_t)j * g.L] = x1;
        dst[(size_t)(j + half) * g.L] = x2;
      }
    } else if (EPI == F32_SWIGLU) {
      const int f = 16 * t + row;
      if (f >= g.N) continue;
      const float gt = (float)c[0], up = (float)c[1];
      g.C[(size_t)m * g.N + f] = gt / (1.0f + expf(-gt)) * up;
    } else {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const int n = 32 * t + 16 * nb + row;
        if (n >= g.N) continue;
        float* o = g.C + (size_t)m * g.N + n;
        *o = EPI == F32_RESID ? (float)((double)pre[mt][nb] + c[nb]) : (float)c[nb];
      }
    }
  }
#endif
}

namespace {

template <int EPI, bool VEC, bool NORM>
void launch_f32(const GemmF32& g, int tiles, hipStream_t s) {
  auto go = [&](auto mt, auto nwv) {
    constexpr int MT = decltype(mt)::value, NWV = decltype(nwv)::value;
    const dim3 grid(tiles, ceil_div(g.M, 16 * MT)), blk(64 * NWV);
    // a NORM launch keeps every step of the row in registers: as few as hold it
    constexpr int NW = NORM ? NORM_MAX_K / 16 / NWV : 0;
    if (NORM && g.K <= NORM_MAX_K / 2)
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, MT, NWV, VEC, NW / 2>), grid, blk, 0, s, g);
    else
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, MT, NWV, VEC, NW>), grid, blk, 0, s, g);
  };
  using i1 = std::integral_constant<int, 1>;
  using i2 = std::integral_constant<int, 2>;
  using i4 = std::integral_constant<int, 4>;
  using i8 = std::integral_constant<int, 8>;
  // 32-row tiles (half the operand loads per product) once they still give
  // every CU two workgroups (948 rows: q/k/v 19.6 against 20.5 us with 16-row
  // tiles, gate/up 30.4 against 28.7; 5840 rows: down 41.8 against 42.4); eight
  // waves (half the k chain each) while 16-row tiles leave CUs short of two
  const long cus = device_cu_count();
  const long t16 = (long)ceil_div(g.M, 16) * tiles, t32 = (long)ceil_div(g.M, 32) * tiles;
  if (t32 >= 2 * cus)
    go(i2{}, i4{});
  else if (t16 >= 2 * cus)
    go(i1{}, i4{});
  else
    go(i1{}, i8{});
}

template <int EPI>
void launch_f32_epi(const GemmF32& g, int tiles, bool vec, hipStream_t s) {
  if constexpr (EPI != F32_RESID) {
    if (g.gain) {
      launch_f32<EPI, true, true>(g, tiles, s);
      return;
    }
  }
  vec ? launch_f32<EPI, true, false>(g, tiles, s) : launch_f32<EPI, false, false>(g, tiles, s);
}

// float4 operand loads: whole 16-k steps and 16-byte aligned rows
bool f32_vec(const GemmF32& g) {
  const uintptr_t p = (uintptr_t)g.A | (uintptr_t)g.W0 | (uintptr_t)g.W1 | (uintptr_t)g.W2 | (uintptr_t)g.gain |
                      (uintptr_t)g.normed;
  return g.K % 16 == 0 && p % 16 == 0;
}

}  // namespace

bool gemm_f32_fuses_norm(const GemmF32& g) { return f32_vec(g) && g.K <= NORM_MAX_K; }

void launch_gemm_f32(GemmF32 g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return;
  if (g.rows == 0) {
    g.rows = g.M;
    g.Ls = g.r0 = 0;
  }
  if (g.gain && !gemm_f32_fuses_norm(g)) throw HipError("gemm_f32: this shape does not fuse its norm");
  if (ceil_div(g.M, 16) > 65535) throw HipError("gemm_f32: more than 65535 row tiles");
  const bool vec = f32_vec(g);
  switch (g.epi) {
    case F32_QKV:
      if (g.hd % 32 != 0 || g.pos0 < 0 || g.pos0 + g.Lq > g.L) throw HipError("gemm_f32: bad q/k/v rows");
      launch_f32_epi<F32_QKV>(g, (g.Hq + 2 * g.Hkv) * (g.hd / 32), vec, s);
      break;
    case F32_SWIGLU: launch_f32_epi<F32_SWIGLU>(g, ceil_div(g.N, 16), vec, s); break;
    case F32_RESID: launch_f32_epi<F32_RESID>(g, ceil_div(g.N, 32), vec, s); break;
    default: launch_f32_epi<F32_STORE>(g, ceil_div(g.N, 32), vec, s); break;
  }
  DLLM_LAUNCH_CHECK("gemm_f32");
}

// ---- attention ----------------------------------------------------------------
// One workgroup of NW waves per (16 queries, query head, sequence); wave w takes
// the 16-key tiles w, w + NW, .. with a float64 online softmax.  S^T = K Q^T, so
// a lane holds scores of one query; the K rows enter in the order key(i) = 4 (i
// % 4) + i / 4, which leaves a lane with the four consecutive keys 4 g .. 4 g +
// 3 (g = lane / 16) in its four registers, and those registers are as they
// stand the B operands of O^T += V^T P^T (slot g of MFMA r = key 4 g + r).  The
// waves' (max, sum, output) states are merged in wave order through LDS.
// One thread per key and per output dimension, scores in LDS, took 8.3 us at 96
// tokens and 78 us at 4 x 237 (tiny model: 4 heads of 64); this kernel 8.4 and
// 12.6 us (at 96 tokens its chain of loads, MFMAs and merge is all there is).
__device__ __forceinline__ float4 ld4u(const float* p) {  // 4-byte aligned
  float4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

template <int HD>
__global__ void __launch_bounds__(HD == 64 ? 512 : 256) attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                       const float* __restrict__ vt, float* __restrict__ out, int Lq,
                                                       int L, int Hq, int Hkv, double scale) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NS = HD / 16, NW = HD == 64 ? 8 : 4;  // the states to merge take 64 KiB of LDS
  __shared__ double ox[NW][NS * 4][64];
  __shared__ double mx[NW][16], lx[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g = lane >> 4;
  const int q0 = blockIdx.x * 16, h = blockIdx.y, b = blockIdx.z, kvh = h / (Hq / Hkv);
  const float* kh = k + ((size_t)b * Hkv + kvh) * L * HD;
  const float* vh = vt + ((size_t)b * Hkv + kvh) * HD * L;
  const float* qrow = q + (((size_t)b * Hq + h) * Lq + min(q0 + col, Lq - 1)) * HD;
  float4 qf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) qf[s] = *reinterpret_cast<const float4*>(qrow + 16 * s + 4 * g);
  f64x4_t o[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) o[s] = f64x4_t{0., 0., 0., 0.};
  double m = -INFINITY, l = 0.0;
  const int nt = (L + 15) / 16;
  for (int t = wave; t < nt; t += NW) {
    const int t0 = 16 * t, key = min(t0 + 4 * (col & 3) + (col >> 2), L - 1);
    const float* kr = kh + (size_t)key * HD + 4 * g;
    float4 kf[NS], vf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) kf[s] = *reinterpret_cast<const float4*>(kr + 16 * s);
    if (t0 + 16 <= L) {
#pragma unroll
      for (int s = 0; s < NS; ++s) vf[s] = ld4u(vh + (size_t)(16 * s + col) * L + t0 + 4 * g);
    } else {  // the last tile: keys past L take no part
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          (&vf[s].x)[r] = t0 + 4 * g + r < L ? vh[(size_t)(16 * s + col) * L + t0 + 4 * g + r] : 0.f;
    }
    f64x4_t sa = {0., 0., 0., 0.}, sb = {0., 0., 0., 0.};  // two chains
#pragma unroll
    for (int s = 0; s < NS; s += 2)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sa = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(&kf[s].x)[e], (double)(&qf[s].x)[e], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(&kf[s + 1].x)[e], (double)(&qf[s + 1].x)[e], sb, 0, 0, 0);
      }
    double sc[4], mt = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = t0 + 4 * g + r < L ? (sa[r] + sb[r]) * scale : -INFINITY;
      mt = fmax(mt, sc[r]);
    }
    mt = fmax(mt, __shfl_xor(mt, 16, 64));
    mt = fmax(mt, __shfl_xor(mt, 32, 64));
    // While every score of a query is -inf or NaN (which fmax drops) its maximum
    // is -inf: then scores are taken against 0, so that -inf adds nothing and NaN
    // stays NaN.  No branch: queries would differ in it, and the MFMAs below read
    // V of every lane.
    const double mn = fmax(m, mt), ref = mn == -INFINITY ? 0.0 : mn;
    const double alpha = exp(m - ref);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = exp(sc[r] - ref);
      l += sc[r];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      o[s] *= alpha;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        o[s] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(&vf[s].x)[r], sc[r], o[s], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) ox[wave][s * 4 + r][lane] = o[s][r];
  if (g == 0) {
    mx[wave][col] = m;
    lx[wave][col] = l;
  }
  __syncthreads();
  double mm = -INFINITY, ll = 0.0, a[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) mm = fmax(mm, mx[w][col]);
#pragma unroll
  for (int w = 0; w < NW; ++w) {  // a wave that saw no key (m = -inf, sums zero) adds nothing; a NaN sum stays
    a[w] = mx[w][col] == -INFINITY ? 0.0 : exp(mx[w][col] - mm);
    ll += lx[w][col] * a[w];
  }
  if (q0 + col >= Lq) return;
  float* orow = out + ((size_t)b * Lq + q0 + col) * Hq * HD + (size_t)h * HD;
#pragma unroll
  for (int s = wave; s < NS; s += NW)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += ox[w][s * 4 + r][lane] * a[w];
      orow[16 * s + 4 * r + g] = (float)(v / ll);
    }
#endif
}

void launch_attn_f32(const float* q, const float* k, const float* vt, float* out, int B, int Lq, int L, int Hq,
                     int Hkv, int hd, hipStream_t s) {
  if (B * Lq == 0) return;
  const dim3 grid(ceil_div(Lq, 16), Hq, B);
  const double scale = 1.0 / sqrt((double)hd);
  if (hd == 64)
    hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(512), 0, s, q, k, vt, out, Lq, L, Hq, Hkv, scale);
  else if (hd == 128)
    hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(256), 0, s, q, k, vt, out, Lq, L, Hq, Hkv, scale);
  else
    throw HipError("attn_f32: head_dim must be 64 or 128");
  DLLM_LAUNCH_CHECK("attn_f32");
}

// ---- vocabulary reduction -------------------------------------------------------
// One 256-thread block per row.  Thread t scans v = t, t+256, ... so its first
// maximum is its lowest index; the merges prefer the larger value, then the
// lower index.  Both merges run over lanes by shuffles, then over the four waves
// through LDS (16 barriers of an LDS tree: 7.1 us a launch at V = 2048).
__global__ void __launch_bounds__(256) vocab_reduce_f32_kernel(const float* __restrict__ logits, int V, int mask_id,
                                                               float* __restrict__ conf, int32_t* __restrict__ arg) {
  const int r = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* row = logits + (size_t)r * V;
  __shared__ float sm[4];
  __shared__ int si[4];
  __shared__ double sd[4];
  float m = -INFINITY;
  int idx = 0x7fffffff;
#pragma unroll 8
  for (int v = threadIdx.x; v < V; v += 256) {
    const float x = v == mask_id ? -INFINITY : row[v];
    if (x > m) {
      m = x;
      idx = v;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float m2 = __shfl_xor(m, o, 64);
    const int i2 = __shfl_xor(idx, o, 64);
    if (m2 > m || (m2 == m && i2 < idx)) {
      m = m2;
      idx = i2;
    }
  }
  if (lane == 0) {
    sm[wave] = m;
    si[wave] = idx;
  }
  __syncthreads();
  float M = sm[0];
  int I = si[0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (sm[w] > M || (sm[w] == M && si[w] < I)) {
      M = sm[w];
      I = si[w];
    }
  double s = 0.0;
#pragma unroll 4
  for (int v = threadIdx.x; v < V; v += 256)
    if (v != mask_id) s += exp((double)row[v] - (double)M);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) sd[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    conf[r] = (float)(1.0 / ((sd[0] + sd[1]) + (sd[2] + sd[3])));
    arg[r] = I;
  }
}

void launch_vocab_reduce_f32(const float* logits, int R, int V, int mask_id, float* conf, int32_t* argmax,
                             hipStream_t s) {
  if (R == 0) return;
  hipLaunchKernelGGL(vocab_reduce_f32_kernel, dim3(R), dim3(256), 0, s, logits, V, mask_id, conf, argmax);
  DLLM_LAUNCH_CHECK("vocab_reduce_f32");
}

}  // namespace dllm
