// fp32 stages on the matrix cores: products and attention forward on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 multiply-add).
//
// These stages are small (a handful of tokens against widths of a few hundred), so what bounds a launch is not its rate
// but its chain: loads, then dependent multiply-adds, then a store, each a trip through the memory or the pipe.  Both
// kernels therefore cut the work into many short pieces: 16 rows per workgroup, the contraction (keys, for attention)
// dealt to its four waves and their partial results added in a fixed order through LDS.  Operands go straight from global
// memory to the fragments: with 16-deep slices a lane reads 16 consecutive bytes of its row, and the four k it holds are
// the slice's k in an order both operands share, so no LDS staging is needed.
//
// Measured (one block of width 128, 2 x 64 tokens): 128 x 128 outputs, K = 128: 18 us on 4 workgroups of the vector kernel, 3.4 on
// 64 workgroups here; K = 512: 38 -> 8; attention 21 -> 4.6; the whole check 191 -> 44.  Its error against 64 bits: 4.4e-8 ->
// 3.9e-8 (the four partial sums are shorter than the one they replace).  Large stages gain less but gain: from 16 tokens of 256
// columns to 8192 of 1024 and 2048 of 4096 no product and no forward attention was slower than on the vector kernels; 8192 x 1024 and
// 2048 x 4096 run at 63 .. 77 TFLOP/s where those had 43 .. 58 (operands come from L2 without LDS, which is what bounds them there).
#include "common.h"

namespace sv {
namespace {

// One fp32 product.  A workgroup makes (16 MI) x (16 NI) outputs; wave w takes every fourth 16-deep slice of k.
// 16 x 16 outputs per workgroup until that fills the CUs four times over, then 32 x 32 (a quarter of the operand traffic).
template <int MI, int NI, bool KN, bool DUAL>
__global__ __launch_bounds__(256) void f32_gemm_kernel(GemmArgs a) {
  constexpr int NP = DUAL ? 2 : 1;
  __shared__ float red[4][NP * MI * NI][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * 16 * MI, n0 = blockIdx.x * 16 * NI;
  const int M = a.m_dev ? *a.m_dev : a.M;             // grouped form: row count from device memory (the launch covers its bound)
  if (m0 >= M) return;
  const int64_t goff = a.tile_group ? (int64_t)a.tile_group[m0 >> 8] * a.group_stride : 0;

  // this thread's outputs: row 4 (lane / 16) + wave and column lane % 16 of each 16 x 16 block; their epilogue inputs are
  // asked for first, so that they do not add a memory round trip at the end
  float r1[MI][NI], r2[MI][NI];
  const bool with_r = a.epi == EPI_RESID || a.epi == EPI_SWIGLU_BWD || a.epi == EPI_GELU_BWD;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int m = m0 + mi * 16 + 4 * lq + wave, n = n0 + ni * 16 + l15;
      r1[mi][ni] = r2[mi][ni] = 0.0f;
      if (m < M && n < a.N) {
        if (with_r) r1[mi][ni] = ((const float*)a.R)[(int64_t)m * a.ldr + n];
        if (a.epi == EPI_SWIGLU_BWD) r2[mi][ni] = ((const float*)a.R2)[(int64_t)m * a.ldr + n];
        if (a.epi == EPI_ROPE && n < a.rope_cols) {
          const float* cs = a.rope_cs + ((int64_t)(m % a.rope_S) * (a.rope_hd >> 1) + ((n % a.rope_hd) >> 1)) * 2;
          r1[mi][ni] = cs[0]; r2[mi][ni] = cs[1];
        }
      }
    }

  f32x4 acc[NP][MI][NI];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) acc[p][mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  for (int s = 0; s < a.nseg; ++s) {
    const int K = a.seg[s].K;
    const int64_t lda = a.seg[s].lda, ldb = a.seg[s].ldb;
    const float* B = (const float*)a.seg[s].B + goff;
    int nb = n0;                                      // first column inside its weight matrix
    if (a.nbcol > 0) {
      int j = 0;
      while (j + 1 < a.nbcol && nb >= a.ncol[j]) { nb -= a.ncol[j]; ++j; }
      B = (const float*)a.Bcol[j];
    }
    const int nleft = a.N - n0;
    const float* ap[MI];
    const float* bp[NP][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) ap[mi] = (const float*)a.seg[s].A + (int64_t)min(m0 + mi * 16 + l15, M - 1) * lda;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int n = nb + min(ni * 16 + l15, nleft - 1);
      bp[0][ni] = KN ? B + n : B + (int64_t)n * ldb;
      if (DUAL) bp[NP - 1][ni] = KN ? (const float*)a.B2 + goff + n : (const float*)a.B2 + goff + (int64_t)n * a.ldb2;
    }
    auto load = [&](int kb, f32x4 (&x)[MI], f32x4 (&w)[NP][NI]) {
      const int k = kb * 16 + lq * 4;
      const bool ok = k < K;                          // K is a multiple of 4: a lane's four k are all in or all out
      const int kc = ok ? k : 0;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) x[mi] = *reinterpret_cast<const f32x4*>(ap[mi] + kc);
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          if (KN) {
            const int64_t ld = p ? a.ldb2 : ldb;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[p][ni][i] = bp[p][ni][(int64_t)(kc + i) * ld];
          } else {
            w[p][ni] = *reinterpret_cast<const f32x4*>(bp[p][ni] + kc);
          }
        }
      if (!ok) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) x[mi] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) w[p][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    };
    auto mul = [&](f32x4 (&x)[MI], f32x4 (&w)[NP][NI]) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
              acc[p][mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[mi][i], w[p][ni][i], acc[p][mi][ni], 0, 0, 0);
    };
    const int nblk = (K + 15) >> 4;
    f32x4 x0[MI], w0[NP][NI], x1[MI], w1[NP][NI];
    int kb = wave;
    if (kb < nblk) load(kb, x0, w0);
    for (; kb < nblk; kb += 8) {                      // two slices per step, the next one's loads ahead of each multiply
      if (kb + 4 < nblk) load(kb + 4, x1, w1);
      mul(x0, w0);
      if (kb + 8 < nblk) load(kb + 8, x0, w0);
      if (kb + 4 < nblk) mul(x1, w1);
    }
  }

#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][(p * MI + mi) * NI + ni][r * 64 + lane] = acc[p][mi][ni][r];
  __syncthreads();

  float* C = (float*)a.C; float* C2 = (float*)a.C2; float* C3 = (float*)a.C3;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      auto sum = [&](int p) {
        const int b = (p * MI + mi) * NI + ni;
        return (red[0][b][tid] + red[1][b][tid]) + (red[2][b][tid] + red[3][b][tid]);
      };
      const float v = sum(0);
      const float u = DUAL ? sum(NP - 1) : 0.0f;
      const float pair = __shfl_xor(v, 1, 64);         // the other feature of the column's RoPE pair
      const int m = m0 + mi * 16 + 4 * lq + wave, n = n0 + ni * 16 + l15;
      if (m >= M || n >= a.N) continue;
      const int64_t ic = (int64_t)m * a.ldc + n;
      const float e1 = r1[mi][ni], e2 = r2[mi][ni];
      switch (a.epi) {
        case EPI_STORE: C[ic] = v; break;
        case EPI_RESID: C[ic] = v + e1; break;
        case EPI_GELU: C[ic] = gelu_f(v); if (C2) C2[ic] = v; break;
        case EPI_SWIGLU: C[ic] = silu_f(v) * u; if (C2) C2[ic] = v; if (C3) C3[ic] = u; break;
        case EPI_SWIGLU_BWD: C[ic] = v * e2 * silu_grad_f(e1); C2[ic] = v * silu_f(e1); break;
        case EPI_GELU_BWD: C[ic] = v * gelu_grad_f(e1); break;
        case EPI_ROPE: C[ic] = n < a.rope_cols ? (n & 1 ? pair * e2 + v * e1 : v * e1 - pair * e2) : v; break;
      }
    }
}

// Attention forward, fp32: 16 queries of one head per workgroup, wave w takes every fourth block of 16 keys and keeps its own
// running maximum, sum and output; the four are merged through LDS at the end.  S^T = K Q^T leaves a lane four keys of one
// query, which is what the second product takes as its B operand (its k order is the lane's key order), so the
// probabilities never move between lanes.
template <int HD>
__global__ __launch_bounds__(256) void f32_attn_fwd_kernel(const float* __restrict__ qkv, int64_t ld, float* __restrict__ o, float* __restrict__ lse,
                                                           int S, int H, int Hkv, int causal) {
  constexpr int NJ = HD / 16, PITCH = HD + 4;
  __shared__ float ol[4][16][PITCH];
  __shared__ float ml[4][16], ll[4][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, lq = lane >> 4;
  const int q0 = blockIdx.x * 16, h = blockIdx.y, b = blockIdx.z, kvh = h / (H / Hkv);
  const int Dq = H * HD, Dkv = Hkv * HD, q = q0 + l15;
  const float scale = rsqrtf((float)HD);
  const float* qrow = qkv + ((int64_t)b * S + min(q, S - 1)) * ld + h * HD + lq * 4;
  const float* kbase = qkv + (int64_t)b * S * ld + Dq + kvh * HD;
  f32x4 qf[NJ], acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    qf[j] = *reinterpret_cast<const f32x4*>(qrow + j * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) { qf[j][i] *= scale; acc[j][i] = 0.0f; }
  }
  float m = -INFINITY, l = 0.0f;
  const int kend = causal ? min(S, q0 + 16) : S;
  for (int k0 = wave * 16; k0 < kend; k0 += 64) {
    const float* krow = kbase + (int64_t)min(k0 + l15, S - 1) * ld + lq * 4;
    f32x4 kf[NJ];
    float vf[4][NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) kf[j] = *reinterpret_cast<const f32x4*>(krow + j * 16);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* vrow = kbase + (int64_t)min(k0 + 4 * lq + r, S - 1) * ld + Dkv + l15;
#pragma unroll
      for (int j = 0; j < NJ; ++j) vf[r][j] = vrow[j * 16];
    }
    f32x4 s = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][i], qf[j][i], s, 0, 0, 0);
    float mx = -INFINITY;
    const bool masks = k0 + 16 > S || (causal && k0 + 16 > q0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = k0 + 4 * lq + r;
      if (key >= S || (causal && key > q)) s[r] = -INFINITY;      // every block holds at least one key each query sees
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), c = expf(m - mn);
    m = mn;
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = expf(s[r] - mn);
    l = l * c + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j][r] *= c;
    // A masked key enters the product with probability 0, and 0 times an infinite or NaN value is NaN: a block that masks
    // and holds such a value is added key by key, by the queries that see the key.
    bool odd = false;
    if (masks) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < NJ; ++j) odd = odd || !(fabsf(vf[r][j]) < INFINITY);
      odd = __any(odd);
    }
    if (odd) {
      for (int t = 0; t < 16; ++t) {
        const float pt = __shfl(t & 2 ? (t & 1 ? p[3] : p[2]) : (t & 1 ? p[1] : p[0]), (t >> 2) * 16 + l15, 64);
        const int key = k0 + t;
        if (key >= S || (causal && key > q)) continue;
        const float* vrow = kbase + (int64_t)key * ld + Dkv + lq * 4;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[j][r] = fmaf(pt, vrow[j * 16 + r], acc[j][r]);
      }
      continue;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][j], p[r], acc[j], 0, 0, 0);
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (lq == 0) { ml[wave][l15] = m; ll[wave][l15] = l; }
#pragma unroll
  for (int j = 0; j < NJ; ++j) *reinterpret_cast<f32x4*>(&ol[wave][l15][j * 16 + lq * 4]) = acc[j];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < NJ; ++e) {
    const int idx = e * 256 + tid, qi = idx / HD, d = idx % HD;
    if (q0 + qi >= S) continue;
    const float mm = fmaxf(fmaxf(ml[0][qi], ml[1][qi]), fmaxf(ml[2][qi], ml[3][qi]));
    float sum = 0.0f, out = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = ll[w][qi] == 0.0f ? 0.0f : expf(ml[w][qi] - mm);    // a wave that had no keys
      sum = fmaf(f, ll[w][qi], sum);
      out = fmaf(f, ol[w][qi][d], out);
    }
    o[((int64_t)b * S + q0 + qi) * Dq + h * HD + d] = out / sum;
    if (d == 0) lse[((int64_t)b * H + h) * S + q0 + qi] = mm + logf(sum);
  }
}

inline bool a16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <bool KN, bool DUAL>
hipError_t launch(const GemmArgs& a, bool wide, hipStream_t st) {
  if (wide) hipLaunchKernelGGL((f32_gemm_kernel<2, 2, KN, DUAL>), dim3((a.N + 31) / 32, (a.M + 31) / 32), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((f32_gemm_kernel<1, 1, KN, DUAL>), dim3((a.N + 15) / 16, (a.M + 15) / 16), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// Operand rows are read 16 bytes at a time (a [K,N] operand element by element); the column map's matrices start on a tile.
bool f32_gemm_supported(const GemmArgs& a) {
  if (a.M < 1 || a.N < 1 || a.nseg < 1 || a.rscale || a.rowsq) return false;
  for (int s = 0; s < a.nseg; ++s) {
    const GemmSeg& g = a.seg[s];
    if (g.K < 4 || g.K % 4 || g.lda % 4 || !a16(g.A)) return false;
    if (!a.b_is_kn && (g.ldb % 4 || !a16(g.B))) return false;
  }
  if (a.epi == EPI_SWIGLU && (!a.B2 || a.nseg != 1 || (!a.b_is_kn && (a.ldb2 % 4 || !a16(a.B2))))) return false;
  if (a.tile_group && !a.b_is_kn && a.group_stride % 4) return false;
  if (a.nbcol > 0) {
    if (a.b_is_kn || a.nseg != 1 || a.epi == EPI_SWIGLU) return false;
    for (int j = 0; j < a.nbcol; ++j)
      if (a.ncol[j] % 16 || !a16(a.Bcol[j])) return false;
  }
  if (a.epi == EPI_ROPE && (!a.rope_cs || a.rope_hd % 2 || a.rope_cols % 2 || a.rope_S < 1)) return false;
  return (a.M + 15) / 16 <= 65535;
}

hipError_t f32_gemm(const GemmArgs& a, hipStream_t st) {
  if (!f32_gemm_supported(a)) return hipErrorInvalidValue;
  bool wide = (int64_t)((a.M + 31) / 32) * ((a.N + 31) / 32) >= 256;
  for (int j = 0; j < a.nbcol; ++j) wide = wide && a.ncol[j] % 32 == 0;
  const bool dual = a.epi == EPI_SWIGLU;
  if (a.b_is_kn) return dual ? launch<true, true>(a, wide, st) : launch<true, false>(a, wide, st);
  return dual ? launch<false, true>(a, wide, st) : launch<false, false>(a, wide, st);
}

bool f32_attn_supported(const void* qkv, int64_t ld, int B, int H, int hd) {
  return (hd == 16 || hd == 32 || hd == 64 || hd == 128) && ld % 4 == 0 && a16(qkv) && H <= 65535 && B <= 65535;
}

hipError_t f32_attn_fwd(const float* qkv, int64_t ld, float* o, float* lse, int B, int S, int H, int Hkv, int hd, int causal, hipStream_t st) {
  if (B <= 0 || S <= 0) return hipSuccess;
  if (!f32_attn_supported(qkv, ld, B, H, hd)) return hipErrorInvalidValue;
  const dim3 grid((S + 15) / 16, H, B), block(256);
  switch (hd) {
    case 16: hipLaunchKernelGGL(f32_attn_fwd_kernel<16>, grid, block, 0, st, qkv, ld, o, lse, S, H, Hkv, causal); break;
    case 32: hipLaunchKernelGGL(f32_attn_fwd_kernel<32>, grid, block, 0, st, qkv, ld, o, lse, S, H, Hkv, causal); break;
    case 64: hipLaunchKernelGGL(f32_attn_fwd_kernel<64>, grid, block, 0, st, qkv, ld, o, lse, S, H, Hkv, causal); break;
    default: hipLaunchKernelGGL(f32_attn_fwd_kernel<128>, grid, block, 0, st, qkv, ld, o, lse, S, H, Hkv, causal); break;
  }
  return hipGetLastError();
}

}  // namespace sv
