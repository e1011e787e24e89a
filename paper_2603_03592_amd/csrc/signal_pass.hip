// One pass of the verifier loop over a stage's submissions (bf16) and their EMA (fp32): the sums of every statistic, the sum of
// the submissions that are not excluded (for the EMA update) and the projections on the sliced-Wasserstein directions.
//
// As separate passes (score_parts_kernel, sw_project_kernel) the submissions come from memory twice, which is most of what
// a stage call costs: 16 x [8192, 4096] are 1.07 GB, 297 us with the EMA and the sum, and again 202 us for the projections.
// Here it is one read, 371 us in all (3.6 TB/s with the EMA and the sum): about half memory, half the vector ALUs' share.
//
// A workgroup owns 16 tokens and all submissions, a wave up to four of them; the row is walked in chunks of 64 features.  A lane
// holds 8 consecutive features of one token (lane & 15; features 8 (lane >> 4) of each half chunk): that is a B fragment of
// v_mfma_f32_16x16x32_bf16 as it comes from memory, so the submissions go straight to registers, are used there by the
// statistics and by the matrix cores (directions in the A slot, staged through LDS for the workgroup), and are never stored.
// The submissions of a wave share the EMA's values, the reference's own sums and one class mask per element for the
// sign test (as in score_parts_kernel).  A register is asked for again, for the next chunk, right behind its last use: one
// chunk of every wave is always in flight.  The waves' partial sums over submissions meet in LDS, one barrier per chunk.
// Sums are taken over a chunk's 16 elements per lane first and then over the chunks, so that no fp32 sum is longer than
// those of the separate pass.
#include "common.h"

namespace sv {
namespace {

__device__ __forceinline__ double xor_sum(double v, int from, int to) {
  for (int o = from; o <= to; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <int LB, int kCPW, int NW>          // blocks of 16 directions; submissions per wave; waves
__global__ __launch_bounds__(64 * NW, 2) void signal_pass_kernel(const bf16* __restrict__ X, int64_t x_stride, int n, const float* __restrict__ m,
                                                             const bf16* __restrict__ U, int64_t T, int D, int64_t Tpad, uint32_t skip,
                                                             float* __restrict__ sum_out, float* __restrict__ P, int tiles,
                                                             ScorePartial* __restrict__ partials) {
  constexpr int UB = LB * 16 * 128;          // bytes of the directions' chunk: rows of 64 bf16, 16-byte pieces XOR-swizzled by the row
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int nthreads = 64 * NW, nw = NW;
  char* ubuf = smem;                         // two chunks of the directions
  char* sbuf = smem + 2 * UB;                // two chunks of the waves' sums: [wave][16 tokens][64 floats], pieces swizzled too
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, lq = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * 16, t = t0 + l15;
  const bool live = t < T;
  const uint64_t live_lanes = __ballot(live);
  const int nchunk = D >> 6;
  // buffer loads: a descriptor per tensor based at the tile's first token, the lane's place in it, the chunk as scalar offset
  const int rel_row = (int)(min(t, T - 1) - t0);
  const int vx = (rel_row * D + lq * 8) * 2, vm = (rel_row * D + lq * 8) * 4;
  auto desc = [&](const void* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, -1, 0x00020000); };
  const bf16* xp[kCPW];
  uint32_t take[kCPW];                                              // all ones for a submission that enters the sum, else zero
#pragma unroll
  for (int c = 0; c < kCPW; ++c) {
    const int i = wave * kCPW + c;
    xp[c] = X + (int64_t)min(i, n - 1) * x_stride + t0 * D;         // a wave's missing submissions repeat the last one, unused
    take[c] = i < n && !((skip >> i) & 1u) ? ~0u : 0u;
  }
  const float* mp = m + t0 * D;

  // directions: piece p (16 bytes) of the chunk is row p / 8, piece p % 8 of it
  constexpr int UPT = (LB * 16 * 8 + nthreads - 1) / nthreads;
  bf16x8 ureg[UPT];
  auto load_u = [&](int chunk) {
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
      const int p = tid + j * nthreads;
      if (LB * 128 % nthreads == 0 || p < LB * 128) ureg[j] = *reinterpret_cast<const bf16x8*>(U + (int64_t)(p >> 3) * D + chunk * 64 + (p & 7) * 8);
    }
  };
  auto store_u = [&](int buf) {
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
      const int p = tid + j * nthreads, r = p >> 3;
      if (LB * 128 % nthreads == 0 || p < LB * 128) *reinterpret_cast<bf16x8*>(ubuf + buf * UB + r * 128 + (((p & 7) ^ (r & 7)) << 4)) = ureg[j];
    }
  };

  bf16x8 x[kCPW][2];
  f32x4 r[2][2];
  auto load_x = [&](int c, int h, int chunk) {
    x[c][h] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(desc(xp[c]), vx, chunk * 128 + h * 64, 0));
  };
  auto load_r = [&](int h, int chunk) {
    r[h][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(desc(mp), vm, chunk * 256 + h * 128, 0));
    r[h][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(desc(mp), vm + 16, chunk * 256 + h * 128, 0));
  };

  f32x4 acc[kCPW][LB];
  float sc[kCPW], scc[kCPW], sad[kCPW], sdd[kCPW], sr = 0.0f, srr = 0.0f;
  int match[kCPW];
#pragma unroll
  for (int c = 0; c < kCPW; ++c) {
    sc[c] = scc[c] = sad[c] = sdd[c] = 0.0f;
    match[c] = 0;
#pragma unroll
    for (int b = 0; b < LB; ++b) acc[c][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  load_u(0);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    load_r(h, 0);
#pragma unroll
    for (int c = 0; c < kCPW; ++c) load_x(c, h, 0);
  }
  store_u(0);
  __syncthreads();
  for (int k = 0; k < nchunk; ++k) {
    const int next = min(k + 1, nchunk - 1);           // past the end: the last chunk again, unused
    load_u(next);
    const char* ub = ubuf + (k & 1) * UB;
    char* sb = sbuf + (k & 1) * (nw * 4096) + wave * 4096;
    float psr = 0.0f, psrr = 0.0f, psc[kCPW], pscc[kCPW], psad[kCPW], psdd[kCPW];
#pragma unroll
    for (int c = 0; c < kCPW; ++c) psc[c] = pscc[c] = psad[c] = psdd[c] = 0.0f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 u[LB];
#pragma unroll
      for (int b = 0; b < LB; ++b) u[b] = *reinterpret_cast<const bf16x8*>(ub + (b * 16 + l15) * 128 + (((h * 4 + lq) ^ (l15 & 7)) << 4));
      float rv[8], sum[8];
      int cls[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        rv[j] = r[h][j >> 2][j & 3];
        // the classes of a value whose sign (of zero and NaN: 0) is the reference's: -inf, -normal, -subnormal; +subnormal,
        // +normal, +inf; or the zeros and NaNs
        cls[j] = rv[j] > 0.0f ? 0x380 : (rv[j] < 0.0f ? 0x01c : 0x063);
        psr += rv[j];
        psrr = fmaf(rv[j], rv[j], psrr);
        sum[j] = 0.0f;
      }
      asm volatile("" : "+v"(psr), "+v"(psrr));
      load_r(h, next);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < kCPW; ++c) {
        float a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = (float)x[c][h][j];
#pragma unroll
        for (int b = 0; b < LB; ++b) acc[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[b], x[c][h], acc[c][b], 0, 0, 0);
        load_x(c, h, next);
        int pm = 0;                                    // wave-uniform
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float d = a[j] - rv[j];
          psdd[c] = fmaf(d, d, psdd[c]);
          psad[c] += fabsf(d);
          psc[c] += a[j];
          pscc[c] = fmaf(a[j], a[j], pscc[c]);
          uint64_t lanes;                              // counted on the scalar unit
          asm("v_cmp_class_f32_e64 %0, %1, %2" : "=s"(lanes) : "v"(a[j]), "v"(cls[j]));
          pm += __popcll(lanes & live_lanes);
          sum[j] += __uint_as_float(__float_as_uint(a[j]) & take[c]);
        }
        // one submission at a time: left to itself the compiler takes the same sum of all four at the end, with everything they
        // need in registers until then
        asm volatile("" : "+v"(psdd[c]), "+v"(psad[c]), "+v"(psc[c]), "+v"(pscc[c]), "+s"(pm));
        match[c] += pm;
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *reinterpret_cast<f32x4*>(sb + l15 * 256 + (((h * 8 + lq * 2 + q) ^ l15) << 4)) = f32x4{sum[q * 4], sum[q * 4 + 1], sum[q * 4 + 2], sum[q * 4 + 3]};
    }
    sr += psr; srr += psrr;
#pragma unroll
    for (int c = 0; c < kCPW; ++c) { sc[c] += psc[c]; scc[c] += pscc[c]; sad[c] += psad[c]; sdd[c] += psdd[c]; }
    store_u((k + 1) & 1);
    lds_barrier();                                     // orders LDS only: the next chunk's loads stay in flight
    for (int e = tid; e < 256; e += nthreads) {        // 16 tokens x 16 pieces of 4 features
      const int tok = e >> 4, pc = e & 15;
      const char* s0 = sbuf + (k & 1) * (nw * 4096) + tok * 256 + ((pc ^ tok) << 4);
      f32x4 v = *reinterpret_cast<const f32x4*>(s0);
      for (int w = 1; w < nw; ++w) {
        const f32x4 o = *reinterpret_cast<const f32x4*>(s0 + w * 4096);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += o[i];
      }
      if (t0 + tok < T) *reinterpret_cast<f32x4*>(sum_out + (t0 + tok) * (int64_t)D + k * 64 + pc * 4) = v;
    }
  }

  // ---- projections: element i of block b is direction 16 b + 4 lq + i of token l15
#pragma unroll
  for (int c = 0; c < kCPW; ++c) {
    const int i = wave * kCPW + c;
    if (i >= n) break;
    float* out = P + (int64_t)i * (LB * 16) * Tpad + t;
#pragma unroll
    for (int b = 0; b < LB; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (live) out[(int64_t)(b * 16 + lq * 4 + j) * Tpad] = acc[c][b][j];
  }

  // ---- one record per submission: token sums over the four lanes of a token, then over the 16 tokens
  const double dsr = xor_sum(live ? (double)sr : 0.0, 1, 32), dsrr = xor_sum(live ? (double)srr : 0.0, 1, 32);
  float tsrr = srr + __shfl_xor(srr, 16, 64);
  tsrr += __shfl_xor(tsrr, 32, 64);
  const double elements = (double)__popcll(live_lanes) * 0.25 * (double)D;
#pragma unroll
  for (int c = 0; c < kCPW; ++c) {
    const int i = wave * kCPW + c;
    if (i >= n) break;
    float tsdd = sdd[c] + __shfl_xor(sdd[c], 16, 64);
    tsdd += __shfl_xor(tsdd, 32, 64);
    const float rel = sqrtf(tsdd) / fmaxf(sqrtf(tsrr), 1e-30f);
    const bool ok = live && rel <= 3.0e38f;
    const int bad = __ballot(live && !ok) != 0;
    float best = ok ? rel : -1.0f;
    int at = ok ? (int)t : 0;
#pragma unroll
    for (int o = 1; o <= 8; o <<= 1) {
      const float ob = __shfl_xor(best, o, 64);
      const int oa = __shfl_xor(at, o, 64);
      if (ob > best || (ob == best && ob >= 0.0f && oa < at)) { best = ob; at = oa; }
    }
    ScorePartial p;
    p.s[0] = xor_sum(live ? (double)sc[c] : 0.0, 1, 32);
    p.s[1] = dsr;
    p.s[2] = xor_sum(live ? (double)scc[c] : 0.0, 1, 32);
    p.s[3] = dsrr;
    p.s[4] = p.s[0] - dsr;
    p.s[5] = xor_sum(live ? (double)sad[c] : 0.0, 1, 32);
    p.s[6] = xor_sum(live ? (double)sdd[c] : 0.0, 1, 32);
    p.s[7] = elements - (double)match[c];
    p.max_rel = best; p.argmax = at; p.bad = bad; p.pad = 0;
    if (lane == 0) partials[(int64_t)i * tiles + blockIdx.x] = p;
  }
}

template <int LB, int CPW, int NW>
hipError_t launch(const bf16* X, int64_t stride, int n, const float* m, const bf16* U, int64_t T, int D, int64_t Tpad, uint32_t skip, float* sum_out,
                  float* P, ScorePartial* partials, hipStream_t st) {
  auto kern = signal_pass_kernel<LB, CPW, NW>;
  constexpr int lds = 2 * LB * 16 * 128 + 2 * NW * 4096;
  static bool configured = false;   // per process; the attribute is per function
  if (!configured && lds > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  configured = true;
  const int tiles = (int)((T + 15) / 16);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(64 * NW), lds, st, X, stride, n, m, U, T, D, Tpad, skip, sum_out, P, tiles, partials);
  return hipGetLastError();
}

inline bool a16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

bool signal_pass_supported(const void* X, int64_t stride, int n, int dtype, const float* m, const void* U, int L, int64_t T, int D) {
  return dtype == SV_BF16 && n >= 1 && n <= 16 && (L == 32 || L == 64) && D >= 64 && D % 64 == 0 && stride % 8 == 0 && T >= 1 && T <= 0x7fffffffLL &&
         a16(X) && a16(m) && a16(U);
}

// The pass reads every submission once where the separate ones read it twice (three times where the score pass leaves no sum), but a
// workgroup walks its 16 tokens' whole row with all submissions, chunk behind chunk, where those spread submissions and rows over
// the chip.  So it is the longer way where there are too few tokens to be short of memory.  Times of a forward and a
// backward call of one stage, separate -> one pass, us, 32 directions (submissions x tokens x columns):
//   16 x 128 x 4032   226 -> 377     12 x 2000 x 3136  396 -> 384     16 x 8192 x 4032  1636 -> 987     2 x 8192 x 4032  528 -> 548
//   4 x 4000 x 4032   426 -> 400     8 x 128 x 384     160 -> 152     16 x 47 x 384      164 -> 172     4 x 500 x 1024   194 -> 187
// With a sum from the score pass (summed: one read less on that side, but a longer chain of its own) the pass is even or better
// where its waves have work for three of four places: 16 x 128 x 4096 456 -> 381, 9 x 128 x 4096 339 -> 367, 2 x 500 x 4096 263 -> 298.
bool signal_pass_pays(int n, int64_t T, int D, bool summed) {
  if (T * n >= 24576 || D <= 320 || (D <= 1024 && n <= 4)) return true;
  const int places = n <= 4 ? 4 : n <= 8 ? 8 : 16;
  return summed && T >= 16 && 4 * n >= 3 * places;
}

hipError_t launch_signal_pass(const void* X, int64_t stride, int n, const float* m, const void* U, int L, int64_t T, int D, int64_t Tpad,
                              uint32_t skip, float* sum_out, float* P, ScorePartial* partials, hipStream_t st) {
  // Four waves, two workgroups on a CU, or where that many workgroups are not there eight waves with half the submissions each: a
  // workgroup's time is then its chain of chunks, and a chunk takes as long as a wave's work on it.
  const bool few = T <= 16 * cu_count();
#define SV_PASS(CPW, NW)                                                                                                       \
  (L == 32 ? launch<2, CPW, NW>((const bf16*)X, stride, n, m, (const bf16*)U, T, D, Tpad, skip, sum_out, P, partials, st)       \
           : launch<4, CPW, NW>((const bf16*)X, stride, n, m, (const bf16*)U, T, D, Tpad, skip, sum_out, P, partials, st))
  if (n <= 4) return SV_PASS(1, 4);
  if (few) return n <= 8 ? SV_PASS(1, 8) : SV_PASS(2, 8);
  return n <= 8 ? SV_PASS(2, 4) : n <= 12 ? SV_PASS(3, 4) : SV_PASS(4, 4);
#undef SV_PASS
}

}  // namespace sv
