// One pass of the verifier loop over a stage's submissions (bf16) and their EMA (fp32): the sums of every statistic, the EMA's
// next value over the submissions that are not excluded, and the projections on the sliced-Wasserstein directions.
//
// As separate passes (score_parts_kernel, sw_project_kernel) the submissions come from memory twice, which is most of what
// a stage call costs: 16 x [8192, 4096] are 1.07 GB, 297 us with the EMA and the sum, again 202 us for the projections, and 60 us
// for an EMA update from the sum.  In one pass 374 us with the submissions in registers, and those 60; in this form 320 us with the
// update, 4.6 TB/s of reads and writes together (a large copy reaches 4.7).
//
// What bounds it is memory: without its statistics it takes 340 us of 347 (before the non-temporal loads), without the two stores 243.  How
// much is on its way decides: with the submissions in registers, one chunk ahead, 324 us with the statistics and 319 without, while
// loads in this pattern and nothing else read the submissions in 175 us with 8 to 16 KB of every wave in flight.  Two chunks ahead
// do not fit the registers beside the projections' accumulators.  So the submissions go straight to LDS, three to five chunks ahead
// (non-temporal, since nobody reads them twice: 347 -> 320 us), and every wave can read every submission:
//   - A workgroup of eight waves owns 16 tokens and all submissions and walks the rows in chunks of 64 features: per chunk 16 x 128
//     bytes of each submission and the directions' 64 columns.
//   - Statistics: a wave takes two tokens, a lane two neighbouring features of one of them, of all submissions one after the other.
//     They share the EMA's values and one class mask per element for the sign test (as in score_parts_kernel), their sum stays
//     in the lane, and so does the EMA's update: m is written in place and its former value beside it (a verdict that
//     excludes somebody else goes back to it).
//   - Projections on v_mfma_f32_16x16x32_bf16, directions in the A slot: a wave takes half the blocks of 16 directions for every
//     fourth submission; fragments are 16-byte reads of the swizzled rows.  The same fragments against ones and against themselves
//     give a token's sum and, on the diagonal, its sum of squares: exact products, added in fp32 within a chunk.
// No fp32 sum is long.  The matrix cores' sums of a chunk (64 terms; they do not round to nearest) go on in 64 bits, the reference's too, and
// the statistics' many are closed after every turn of the places (4 to 6 chunks: 8 to 12 additions one after the other) into a second
// fp32 sum (16 additions at 4096 columns); the lanes meet in 64 bits.  With one fp32 sum over the row the z-scored statistic of signals whose
// mean is 30 deviations was off by 5.8e-4 (2000 tokens of 4096), with these by 5e-5, and of those around zero by 2.0e-6 and 6e-8 (8192
// tokens).  It costs 0.7 % of a loop call on average and 3 % at most (4 x 47 x 4032 185 -> 191 us, 16 x 2000 x 4032 379 -> 389).
// Workgroups start at different chunks, so that they do not all ask for the same 128 bytes of every 8 KB row at once (374 -> 324 us
// for the register form).
#include <type_traits>

#include "common.h"

namespace sv {
namespace {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kStream = 2;   // of a buffer load: its bytes come by once (non-temporal)

template <int LB, int NS> struct PassCfg {       // blocks of 16 directions; places for submissions (a multiple of 4)
  static constexpr int XB = NS * 2048;           // a chunk's bytes: the submissions' [NS][16 tokens][64 bf16]
  static constexpr int UB = LB * 2048;           // ... the directions' [16 LB][64 bf16]
  static constexpr int NST = NS == 16 ? 4 : NS == 12 ? 5 : 6, NU = 3;      // chunks of either in LDS: NST - 1 and two on their way
  static constexpr int LDS = NST * XB + NU * UB;
  static constexpr int XW = NS / 4, UW = (2 * LB + 7) / 8;                 // direct-to-LDS loads of 1 KB per wave and chunk
  // What a wave has issued behind the directions it needs next: the submissions and the EMA's values of two chunks, the stores of two
  // and the directions of one.  (What it needs of the submissions next is older.)
  static constexpr int YOUNGER = 2 * (XW + 1 + 2) + UW;
  static_assert(YOUNGER < 64 && LDS <= 160 * 1024, "the wait count has 6 bits, a CU 160 KB");
  // the statistics' reduction: the lanes' sums, every token's sums, the matches
  static constexpr int NV = 2 * NS + 2, RED = 8 * NV * 64 * 4, TOK = 16 * (4 * NS + 2) * 8, CNT = 8 * NS * 4;
  static_assert(RED + TOK + CNT <= LDS, "the reduction fits the chunks' place");
};

template <int LB, int NS, bool ALL>              // ALL: every place holds a submission that enters the EMA
__global__ __launch_bounds__(512, 2) void signal_pass_kernel(const bf16* __restrict__ X, int64_t x_stride, int n, float* m, float* m_prev, float beta,
                                                             float w_new, const bf16* __restrict__ U, int64_t T, int D, int64_t Tpad, uint32_t skip,
                                                             float* __restrict__ P, int tiles, ScorePartial* __restrict__ partials) {
  using C = PassCfg<LB, NS>;
  constexpr int NST = C::NST, SPW = NS / 4, BPW = LB / 2;        // submissions and blocks of directions of a wave's projections
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, lq = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * 16;
  const int last_row = (int)(min(t0 + 15, T - 1) - t0);
  const int nchunk = D >> 6;
  auto swz = [](int r) { return (r ^ (r >> 3)) & 7; };           // which 16-byte piece of a 128-byte row goes where

  auto desc = [&](const void* p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000); };
  // ---- the streams.  A load fills 1 KB of LDS: 8 rows of a submission's chunk (load 2 c and 2 c + 1 of submission c) or of the
  // directions'.  Rows past the last token repeat it, places past the last submission repeat that one (neither is used).
  const bf16* xp = X + t0 * D;
  float* mp = m + t0 * D;
  const int r8 = lane >> 3, p8 = lane & 7;
  const int hi_row = (wave & 1) * 8 + r8;                        // a wave's loads are all of one half of the rows
  const unsigned vx = (unsigned)(min(hi_row, last_row) * D * 2 + ((p8 ^ swz(hi_row)) << 4));
  auto load_x = [&](int chunk, int st) {
    const int so = chunk * 128;
#pragma unroll
    for (int j = 0; j < C::XW; ++j) {
      const int i = wave + 8 * j;
      char* dst = smem + st * C::XB + i * 1024;
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(xp + (int64_t)min(i >> 1, n - 1) * x_stride), (short)0, -1, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, (int)vx, so, 0, kStream);
    }
  };
  unsigned vu[C::UW];
#pragma unroll
  for (int j = 0; j < C::UW; ++j) {
    const int r = min(wave + 8 * j, 2 * LB - 1) * 8 + r8;        // a repeated load writes the same bytes
    vu[j] = (unsigned)(r * D * 2 + ((p8 ^ swz(r)) << 4));
  }
  char* ubuf = smem + NST * C::XB;
  auto load_u = [&](int chunk, int st) {
    const int so = chunk * 128;
#pragma unroll
    for (int j = 0; j < C::UW; ++j) {
      char* dst = ubuf + st * C::UB + min(wave + 8 * j, 2 * LB - 1) * 1024;
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(U), (short)0, -1, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, (int)vu[j], so, 0, 0);
    }
  };

  // ---- a wave's places: statistics of token `tok`, features 2 f and 2 f + 1 of the chunk; projections of blocks BPW (wave & 1) ..
  // and submissions (wave >> 1) + 4 j
  const int tok = wave * 2 + (lane >> 5), f = lane & 31;
  const bool live = t0 + tok < T;
  const int live_mask = live ? -1 : 0;
  const int sx = tok * 128 + (((f >> 2) ^ swz(tok)) << 4) + (f & 3) * 4;
  const int fx = (wave >> 1) * 2048 + l15 * 128, fu = (wave & 1) * BPW * 2048 + l15 * 128;
  const int vm = (tok * D + f * 2) * 4, vr = (min(tok, last_row) * D + f * 2) * 4;
  const __amdgpu_buffer_rsrc_t bm = desc(mp, (last_row + 1) * D * 4), bp = desc(m_prev + t0 * D, (last_row + 1) * D * 4);   // rows past the last token are dropped

  f32x4 acc[SPW][BPW];
#pragma unroll
  for (int j = 0; j < SPW; ++j)
#pragma unroll
    for (int b = 0; b < BPW; ++b) acc[j][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  double self[SPW];                                              // of a wave's submissions: sums of c (even waves), of c c' (odd ones)
#pragma unroll
  for (int j = 0; j < SPW; ++j) self[j] = 0.0;
  const bf16x8 ones = {(bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f};
  float sad[NS], sdd[NS], sad_all[NS], sdd_all[NS];              // sums of |d|, d^2: of this turn of the places, of those before
  double sr = 0.0, srr = 0.0;
  int match[NS];
#pragma unroll
  for (int c = 0; c < NS; ++c) { sad[c] = sdd[c] = sad_all[c] = sdd_all[c] = 0.0f; match[c] = 0; }

  auto after = [&](int chunk) { return chunk + 1 == nchunk ? 0 : chunk + 1; };      // behind the last round: chunks again, unused
  f32x2 r[NST];                                                  // the EMA's values, as far ahead as the submissions
  auto load_r = [&](f32x2& v, int chunk) { v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(bm, vr, chunk * 256, 0)); };
  int chunk = (int)((blockIdx.x >> 3) * 5u % (unsigned)nchunk), ahead = chunk, ahead_u = chunk, su = 0;
  for (int s = 0; s < 2; ++s) { load_u(ahead_u, s); ahead_u = after(ahead_u); }
#pragma unroll
  for (int s = 0; s + 1 < NST; ++s) { load_r(r[s], ahead); load_x(ahead, s); ahead = after(ahead); }
  __builtin_amdgcn_s_waitcnt(0);                                 // all of them: the waits below count on it
  __syncthreads();
  auto body = [&](auto st_tag) {
    constexpr int st = decltype(st_tag)::value, fill = (st + NST - 1) % NST;        // fill: the place the last chunk has left
    load_u(ahead_u, su == 0 ? C::NU - 1 : su - 1);
    __builtin_amdgcn_sched_barrier(0);                           // the oldest of the chunk's: the wait below counts what is behind it
    ahead_u = after(ahead_u);
    const f32x2 rv = r[st];
    load_r(r[fill], ahead);
    load_x(ahead, fill);
    ahead = after(ahead);
    const char* base = smem + st * C::XB;
    const char* ub = ubuf + su * C::UB;
    // the statistics' values are asked for first: they arrive behind the projections' products
    uint32_t xx[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) xx[c] = *reinterpret_cast<const uint32_t*>(base + sx + c * 2048);
    __builtin_amdgcn_sched_barrier(0);
    // projections
    bf16x8 u[2][BPW], x[2][SPW];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int b = 0; b < BPW; ++b) {
        const int r = ((wave & 1) * BPW + b) * 16 + l15;
        u[h][b] = *reinterpret_cast<const bf16x8*>(ub + fu + b * 2048 + (((h * 4 + lq) ^ swz(r)) << 4));
      }
#pragma unroll
      for (int j = 0; j < SPW; ++j) x[h][j] = *reinterpret_cast<const bf16x8*>(base + fx + j * 8192 + (((h * 4 + lq) ^ swz(l15)) << 4));
    }
    __builtin_amdgcn_sched_barrier(0);
    // statistics
    f32x4 piece[SPW];                                            // the chunk's part of self: 64 terms
    float sum[2] = {0.0f, 0.0f};
    int cls[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // the classes of a value whose sign (of zero and NaN: 0) is the reference's: -inf, -normal, -subnormal; +subnormal,
      // +normal, +inf; or the zeros and NaNs.  None in the places past the last token.
      cls[e] = (rv[e] > 0.0f ? 0x380 : (rv[e] < 0.0f ? 0x01c : 0x063)) & live_mask;
      sr += (double)rv[e];
      srr = fma((double)rv[e], (double)rv[e], srr);
    }
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      if (c == NS / 2) {
        // the products stand between the statistics' halves: their fragments are there by now, and the matrix cores work beside
        // what follows
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < SPW; ++j) {
#pragma unroll
            for (int b = 0; b < BPW; ++b) acc[j][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[h][b], x[h][j], acc[j][b], 0, 0, 0);
            piece[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16((wave & 1) ? x[h][j] : ones, x[h][j], h ? piece[j] : f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      const uint32_t take = ALL || !((skip >> c) & 1u) ? ~0u : 0u;           // wave-uniform; places past the last submission are skipped
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t bits = e == 0 ? xx[c] << 16 : xx[c] & 0xffff0000u;
        const float a = __uint_as_float(bits), d = a - rv[e];
        sad[c] += fabsf(d);
        sdd[c] = fmaf(d, d, sdd[c]);
        uint64_t lanes;                                          // counted on the scalar unit
        asm("v_cmp_class_f32_e64 %0, %1, %2" : "=s"(lanes) : "v"(a), "v"(cls[e]));
        match[c] += __popcll(lanes);
        sum[e] += __uint_as_float(ALL ? bits : bits & take);
      }
      if constexpr (st == NST - 1) {
        sad_all[c] += sad[c]; sdd_all[c] += sdd[c];
        sad[c] = sdd[c] = 0.0f;
      }
    }
#pragma unroll
    for (int j = 0; j < SPW; ++j)
      self[j] += (double)((l15 & 3) == 0 ? piece[j][0] : (l15 & 3) == 1 ? piece[j][1] : (l15 & 3) == 2 ? piece[j][2] : piece[j][3]);
    f32x2 next;
#pragma unroll
    for (int e = 0; e < 2; ++e) next[e] = beta * rv[e] + w_new * sum[e];
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, rv), bp, vm, chunk * 256, 0);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, next), bm, vm, chunk * 256, 0);
    // this wave's part of the next chunk has landed, its reads of this one are done; behind the barrier everybody's
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070 | (C::YOUNGER & 15) | ((C::YOUNGER >> 4) << 14));       // vmcnt(YOUNGER) lgkmcnt(0)
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    chunk = after(chunk);
    su = su + 1 == C::NU ? 0 : su + 1;
  };
  for (int k = 0;;) {                                            // left by breaks: a turn's end is reached from its last part only
    body(std::integral_constant<int, 0>{});
    if (++k >= nchunk) break;
    body(std::integral_constant<int, 1>{});
    if (++k >= nchunk) break;
    body(std::integral_constant<int, 2>{});
    if (++k >= nchunk) break;
    body(std::integral_constant<int, 3>{});
    if (++k >= nchunk) break;
    if constexpr (NST > 4) { body(std::integral_constant<int, 4>{}); if (++k >= nchunk) break; }
    if constexpr (NST > 5) { body(std::integral_constant<int, 5>{}); if (++k >= nchunk) break; }
  }
  __builtin_amdgcn_s_waitcnt(0);                                 // the last direct-to-LDS loads have landed before their place is used again
  __syncthreads();

  // ---- projections: element i of block b is direction 16 b + 4 lq + i of token l15
  const int64_t t = t0 + l15;
#pragma unroll
  for (int j = 0; j < SPW; ++j) {
    const int i = (wave >> 1) + 4 * j;
    if (i >= n) break;
    float* out = P + (int64_t)i * (LB * 16) * Tpad + t;
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t < T) out[(int64_t)(((wave & 1) * BPW + b) * 16 + lq * 4 + e) * Tpad] = acc[j][b][e];
  }

  // ---- every token's sums: of c in all rows of its column, of c^2 on the diagonal (lane (l15, l15 / 4)); the 32 lanes of a
  // token leave their others in LDS and a thread adds up those of one sum in 64 bits (in an order of its own, so that the lanes of
  // a read meet different banks)
  float* red = reinterpret_cast<float*>(smem);                   // [wave][NV][64 lanes]
  double* tk = reinterpret_cast<double*>(smem + C::RED);         // [token][4 NS + 2]: sums of c, c^2, |d|, d^2; of the reference and its squares
  constexpr int TS = 4 * NS + 2;
#pragma unroll
  for (int j = 0; j < SPW; ++j) {
    const int c = (wave >> 1) + 4 * j;
    if (lq == l15 >> 2) tk[l15 * TS + ((wave & 1) ? NS : 0) + c] = self[j];
  }
#pragma unroll
  for (int c = 0; c < NS; ++c) {
    red[(wave * C::NV + c) * 64 + lane] = sad_all[c] + sad[c];
    red[(wave * C::NV + NS + c) * 64 + lane] = sdd_all[c] + sdd[c];
  }
  red[(wave * C::NV + 2 * NS) * 64 + lane] = (float)sr;
  red[(wave * C::NV + 2 * NS + 1) * 64 + lane] = (float)srr;
  int* cnt = reinterpret_cast<int*>(smem + C::RED + C::TOK);     // [wave][NS]
#pragma unroll
  for (int c = 0; c < NS; ++c)
    if (lane == 0) cnt[wave * NS + c] = match[c];
  __syncthreads();
  for (int e = tid; e < 16 * C::NV; e += 512) {
    const int to = e / C::NV, v = e % C::NV;
    const float* src = red + ((to >> 1) * C::NV + v) * 64 + (to & 1) * 32;
    double a = 0.0;
    for (int l = 0; l < 32; ++l) a += (double)src[(l + tid) & 31];
    tk[to * TS + 2 * NS + v] = a;
  }
  __syncthreads();
  // ---- one record per submission
  if (tid < n) {
    const int c = tid, rows = last_row + 1;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s5 = 0.0, s6 = 0.0;
    float best = -1.0f;
    int at = 0, bad = 0, same = 0;
    for (int r = 0; r < rows; ++r) {
      const double* a = tk + r * TS;
      s0 += a[c]; s2 += a[NS + c]; s5 += a[2 * NS + c]; s6 += a[3 * NS + c];
      s1 += a[4 * NS]; s3 += a[4 * NS + 1];
      const float rel = sqrtf((float)a[3 * NS + c]) / fmaxf(sqrtf((float)a[4 * NS + 1]), 1e-30f);
      if (!(rel <= 3.0e38f)) bad = 1;
      else if (rel > best) { best = rel; at = (int)(t0 + r); }   // the first of equals
    }
    for (int w = 0; w < 8; ++w) same += cnt[w * NS + c];
    ScorePartial p;
    p.s[0] = s0; p.s[1] = s1; p.s[2] = s2; p.s[3] = s3; p.s[4] = s0 - s1; p.s[5] = s5; p.s[6] = s6;
    p.s[7] = (double)rows * (double)D - (double)same;
    p.max_rel = best; p.argmax = at; p.bad = bad; p.launch = 0;
    partials[(int64_t)c * tiles + blockIdx.x] = p;
  }
}

template <int LB, int NS, bool ALL>
hipError_t launch(const bf16* X, int64_t stride, int n, float* m, float* m_prev, float beta, const bf16* U, int64_t T, int D, int64_t Tpad, uint32_t skip,
                  float* P, ScorePartial* partials, hipStream_t st) {
  auto kern = signal_pass_kernel<LB, NS, ALL>;
  constexpr int lds = PassCfg<LB, NS>::LDS;
  static bool configured = false;   // per process; the attribute is per function
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles = (int)((T + 15) / 16);
  int taken = 0;
  for (int i = 0; i < n; ++i) taken += !((skip >> i) & 1u);
  const float keep = taken ? beta : 1.0f, w = taken ? (1.0f - beta) / (float)taken : 0.0f;      // nobody to take: m as it is
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(512), lds, st, X, stride, n, m, m_prev, keep, w, U, T, D, Tpad,
                     skip | (n < 32 ? ~0u << n : 0u), P, tiles, partials);
  return hipGetLastError();
}

inline bool a16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

bool signal_pass_supported(const void* X, int64_t stride, int n, int dtype, const float* m, const void* U, int L, int64_t T, int D) {
  return dtype == SV_BF16 && n >= 1 && n <= 16 && (L == 32 || L == 64) && D >= 64 && D % 64 == 0 && stride % 8 == 0 && T >= 1 && T <= 0x7fffffffLL &&
         a16(X) && a16(m) && a16(U);
}

// The pass reads every submission once where the separate ones read it twice (three times where the score pass leaves no sum), but a
// workgroup walks its 16 tokens' whole row with all submissions, chunk behind chunk (about 1.4 us a chunk of 16), where those spread
// submissions and rows over the chip.  So it is the longer way where there are few tokens of many long submissions.  Times of the pass
// over those of the separate passes, a forward and a backward call of one stage together, 64 directions:
//   columns            16 submissions x 33 / 500 / 1000 / 1500 tokens     5 x 33 / 500 / 2500     2 x 33 / 500 / 2500
//   448                0.98 / 0.94 / 0.95 / 0.88                           0.90 / 0.91 / 0.89      (taken)
//   1088               1.12 / 1.05 / 0.99 / 0.90                           0.96 / 0.96 / 0.89      0.87 / 0.88 / 0.87
//   1984               1.25 / 1.17 / 1.05 / 0.93                           1.01 / 1.00 / 0.88      0.87 / 0.88 / 0.86
//   4032               1.57 / 1.32 / (taken)                               1.15 / 1.13 / (taken)   (taken)
// The lines are on the safe side of these: between them and where the pass begins to win lie calls that it would make up to 16 % shorter,
// up to four submissions of 1025 to 2047 columns among them, which take the separate passes as they always have.  With a sum from the
// score pass (summed: one read less on that side, but a longer chain of its own) the pass is always the shorter way: 16 x 47 x 4096
// 485 -> 346 us, 2 x 47 x 4096 266 -> 200.
bool signal_pass_pays(int n, int64_t T, int D, bool summed) {
  return summed || D <= 320 || T * n >= (D >= 2048 ? 12000 : 24576) || (n <= 4 && (D <= 1024 || D >= 2048));
}

hipError_t launch_signal_pass(const void* X, int64_t stride, int n, float* m, float* m_prev, float beta, const void* U, int L, int64_t T, int D,
                              int64_t Tpad, uint32_t skip, float* P, ScorePartial* partials, hipStream_t st) {
  const bool all = skip == 0 && n % 4 == 0;
#define SV_PASS_(LB, NS, ALL) launch<LB, NS, ALL>((const bf16*)X, stride, n, m, m_prev, beta, (const bf16*)U, T, D, Tpad, skip, P, partials, st)
#define SV_PASS(NS) (L == 32 ? (all ? SV_PASS_(2, NS, true) : SV_PASS_(2, NS, false)) : (all ? SV_PASS_(4, NS, true) : SV_PASS_(4, NS, false)))
  return n <= 4 ? SV_PASS(4) : n <= 8 ? SV_PASS(8) : n <= 12 ? SV_PASS(12) : SV_PASS(16);
#undef SV_PASS_
#undef SV_PASS
}

}  // namespace sv
