// Check statistics between submissions and a reference point, the flag rule, and the EMA
// reference update.  All three kernels are streaming (HBM-bound) passes.
//
//   score_tokens_kernel : one pass over claim and reference.  Per token it forms the sums the
//                         whole distance family needs (Omega_L1, Omega_L2, Omega_SFR of the
//                         paragraph "Choice of Distance Measure", and the per-token relative
//                         L2), then folds 16 tokens into one partial record.
//   score_finalize_kernel: deterministic reduction of the records of one submission (few records: in the
//                         pass itself), the scores, and the flag Gamma > tau (Eq. test_statistic; a submission
//                         is flagged when any enabled metric exceeds its threshold).
//   ema_update_kernel   : Eq. momentum_def over the un-flagged submissions.
#include <mutex>
#include <type_traits>

#include "common.h"

namespace sv {

namespace {

constexpr int kTPW = kScoreTokensPerWG / 4;  // tokens per wave

__device__ __forceinline__ float dpp_add(float v, int ctrl_sel) {
  const int x = __float_as_int(v);
  int y;
  switch (ctrl_sel) {                                            // immediate operands
    case 0: y = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false); break;     // quad_perm [1,0,3,2]
    case 1: y = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false); break;     // quad_perm [2,3,0,1]
    case 2: y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false); break;    // row_half_mirror
    default: y = __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false); break;   // row_mirror
  }
  return v + __int_as_float(y);
}
// Sum over the 64 lanes without the LDS crossbar: four exchange steps inside each row of 16 lanes, then the four row
// sums are read as scalars.  Every lane gets the same value (a fixed order: run-to-run identical).
__device__ __forceinline__ float wave_sum_rows(float v) {
  v = dpp_add(v, 0); v = dpp_add(v, 1); v = dpp_add(v, 2); v = dpp_add(v, 3);
  const int x = __float_as_int(v);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(x, 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(x, 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(x, 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(x, 48));
  return (r0 + r1) + (r2 + r3);
}

struct Tau4 { float v[4]; };

// What turns a submission's records into its scores and flag.
struct Verdict { uint32_t mask; Tau4 tau; int reduce; sv_result* results; };

// What a pass that forms the scores itself is given beside; nothing for the others.
template <bool ALONE> struct Alone { uint32_t launch; Verdict verdict; };
template <> struct Alone<false> {};

inline __host__ __device__ int finalize_threads(int tiles_per_claim) { return tiles_per_claim <= 128 ? 64 : 256; }

// Records that another workgroup of the same launch reads.  The XCDs' L2 caches do not see each other's plain stores within a launch,
// and a release fence would write a whole L2 back for 80 bytes (and leave what follows in the check to find it so): the words go
// past it one by one, and are read past it.
__device__ __forceinline__ void publish(ScorePartial* p, int word, uint64_t v) {      // one of a record's ten 8-byte words
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p) + word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t published(const ScorePartial* p, int word) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p) + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// what this wave has published is there for every XCD
__device__ __forceinline__ void published_so_far() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
  asm volatile("" ::: "memory");
}

// The scores and the flag of one submission, by the first nt threads of a workgroup (all of which call).
template <bool PUBLISHED>
__device__ void finalize_claim(const ScorePartial* p, int tiles_per_claim, int claim, int64_t T, int D, const Verdict& verdict, int nt) {
  const int tid = threadIdx.x;
  const uint32_t mask = verdict.mask;
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float best = -1.0f; int bt = 0, bad = 0;
  for (int i = tid; i < tiles_per_claim && tid < nt; i += nt) {      // tiles visited in increasing order
    ScorePartial q;
    if constexpr (PUBLISHED) {
      struct Words { uint64_t w[10]; } words;
      static_assert(sizeof(Words) == sizeof(ScorePartial), "a record is ten words");
#pragma unroll
      for (int j = 0; j < 10; ++j) words.w[j] = published(p + i, j);
      q = __builtin_bit_cast(ScorePartial, words);
    } else q = p[i];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += q.s[j];
    bad |= q.bad;
    if (q.max_rel > best) { best = q.max_rel; bt = q.argmax; }
  }
  __shared__ double s_acc[256][8];
  __shared__ float s_best[256];
  __shared__ int s_bt[256], s_bad[256];
#pragma unroll
  for (int j = 0; j < 8; ++j) s_acc[tid][j] = acc[j];
  s_best[tid] = best; s_bt[tid] = bt; s_bad[tid] = bad;
  __syncthreads();
  for (int stride = nt >> 1; stride > 0; stride >>= 1) { // fixed tree: run-to-run identical
    if (tid < stride) {
#pragma unroll
      for (int j = 0; j < 8; ++j) s_acc[tid][j] += s_acc[tid + stride][j];
      s_bad[tid] |= s_bad[tid + stride];
      const float o = s_best[tid + stride];
      if (o > s_best[tid] || (o == s_best[tid] && s_bt[tid + stride] < s_bt[tid])) { s_best[tid] = o; s_bt[tid] = s_bt[tid + stride]; }
    }
    __syncthreads();
  }
  if (tid == 0) {
    const double n = (double)T * (double)D;
    const double Sc = s_acc[0][0], Sr = s_acc[0][1], Scc = s_acc[0][2], Srr = s_acc[0][3];
    const double Sd = s_acc[0][4], Sad = s_acc[0][5], Sdd = s_acc[0][6], Ns = s_acc[0][7];
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    double sc[4];
    const double grel = sqrt(Sdd) / fmax(sqrt(Srr), 1e-30);
    const double mrel = s_bad[0] ? nan : (double)fmaxf(s_best[0], 0.0f);
    sc[SV_IDX_RELL2] = (verdict.reduce == SV_REDUCE_MAX_TOKEN) ? mrel : grel;
    sc[SV_IDX_L1] = Sad / n;
    // z-scored L2 = 2 (1 - rho) = (var_d - (sd_c - sd_r)^2) / (sd_c sd_r): no cancellation for rho ~ 1
    const double mc = Sc / n, mr = Sr / n, md = Sd / n;
    const double vc = Scc / n - mc * mc, vr = Srr / n - mr * mr, vd = fmax(Sdd / n - md * md, 0.0);
    const bool const_c = !(vc > 1e-10 * (Scc / n)), const_r = !(vr > 1e-10 * (Srr / n));
    if (Scc != Scc || Srr != Srr) sc[SV_IDX_ZL2] = nan;
    else if (const_c && const_r) sc[SV_IDX_ZL2] = 0.0;
    else if (const_c || const_r) sc[SV_IDX_ZL2] = 2.0;
    else {
      const double a = sqrt(vc), b = sqrt(vr);
      sc[SV_IDX_ZL2] = fmax(vd - (a - b) * (a - b), 0.0) / (a * b);
    }
    sc[SV_IDX_SFR] = Ns / n;
    sv_result r;
    uint32_t flag = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool on = ((mask >> i) & 1u) || i == SV_IDX_RELL2;         // the relative L2 is always formed
      r.score[i] = on ? (float)sc[i] : 0.0f;
      if (((mask >> i) & 1u) && !(r.score[i] <= verdict.tau.v[i])) flag = 1;   // strict '>'; non-finite scores are flagged
    }
    r.flag = flag; r.metric_mask = mask;
    r.max_token_rell2 = (float)mrel; r.argmax_token = s_bt[0];
    verdict.results[claim] = r;
  }
}

__global__ __launch_bounds__(256) void score_finalize_kernel(const ScorePartial* __restrict__ partials, int tiles_per_claim, int64_t T, int D,
                                                             Verdict verdict) {
  finalize_claim<false>(partials + (int64_t)blockIdx.x * tiles_per_claim, tiles_per_claim, blockIdx.x, T, D, verdict, blockDim.x);
}

// NEED_L1 / NEED_Z / NEED_SFR prune the sums a launch does not need (the statistic family is
// requested by mask): with only the relative L2 enabled a token costs two FMAs per element and the
// pass is bound by HBM; with all eight sums it is bound by the vector ALUs (about 18 ops/element).
// TW: tokens per workgroup, and per record.  With few records of 16 (one submission of up to 4096 tokens) the pass is a chain of
// memory round trips, one per token of a wave, on a part of the CUs: 4 tokens then, one per wave on four times the workgroups
// (512 tokens of 4096, both sides bf16: 13 -> 6 us; 2331 of 960: 10 -> 5.5).
// ALONE: the pass forms the scores too, without a second launch (an instantiation of its own: with the code for it behind a branch the
// pass over 4096 tokens of 1024 took 5 us more).  A record carries the launch's number, written behind the rest of it, and a workgroup
// that then finds that number in every record of its submission forms the scores from them, in the order of score_finalize_kernel.  One
// of them does (the one whose number was there last); if several do, they write the same bytes.  Nobody waits, and nothing has to be as an
// earlier launch should have left it: launches that overlapped on one context, which share the records and are not supported, can
// spoil their own scores but not a later launch's.
template <typename EC, typename ER, bool NEED_L1, bool NEED_Z, bool NEED_SFR, int TW, bool ALONE>
__global__ __launch_bounds__(256) void score_tokens_kernel(const EC* __restrict__ claims, int64_t claim_stride,
                                                           const ER* __restrict__ ref, int64_t ref_stride, int64_t T, int D,
                                                           int n_claims, int tiles_per_claim, float* __restrict__ token_scores,
                                                           ScorePartial* __restrict__ partials, Alone<ALONE> alone) {
  // Workgroup ids go round-robin over the 8 XCDs (each with its own L2): ids congruent mod 8 get a contiguous run of
  // token tiles, and within a run the claim index varies fastest, so the submissions that share a tile of the
  // reference run together on one XCD and fetch it from memory once instead of once per XCD.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int claim = slot % n_claims;
  const int tile = xcd * ((tiles_per_claim + 7) >> 3) + slot / n_claims;
  if (tile >= tiles_per_claim) return;               // the last XCD's run may be short (whole workgroup leaves)
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const EC* cbase = claims + (int64_t)claim * claim_stride;
  const ER* rbase = ref + (int64_t)claim * ref_stride;

  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float best = -1.0f;
  int best_t = 0, bad = 0;

  for (int i = 0; i < TW / 4; ++i) {
    const int64_t t = (int64_t)tile * TW + i * 4 + wave;
    if (t >= T) break;  // uniform per wave
    const EC* c = cbase + t * D;
    const ER* r = rbase + t * D;
    float sc = 0, sr = 0, scc = 0, srr = 0, sad = 0, sdd = 0;
    int nsi = 0;
    auto accumulate = [&](const float (&cv)[8], const float (&rv)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = cv[j], b = rv[j], d = a - b;
        srr = fmaf(b, b, srr); sdd = fmaf(d, d, sdd);
        if (NEED_Z) { sc += a; sr += b; scc = fmaf(a, a, scc); }
        if (NEED_L1) sad += fabsf(d);
        // sign(a) != sign(b) with sign(0) = 0: the two signs agree iff both "positive" and both "negative" tests agree
        if (NEED_SFR) nsi += (int)(((a > 0.0f) != (b > 0.0f)) | ((a < 0.0f) != (b < 0.0f)));
      }
    };
    // N units of 512 elements from k0 on, all their loads in flight before the first is used; of the row's last unit the lanes
    // past its end take two equal zeros, which add nothing to any sum
    // (55 submissions of 5338 x 1856, each with its own fp32 reference: 750 -> 560 us, 5.8 TB/s, against one unit at a time)
    auto part = [&](auto n_tag, auto last_tag, int k0) {
      constexpr int N = decltype(n_tag)::value;
      float cv[N][8], rv[N][8];
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const int k = k0 + m * 512 + lane * 8;
        if (decltype(last_tag)::value && m == N - 1) {
#pragma unroll
          for (int j = 0; j < 8; ++j) cv[m][j] = rv[m][j] = 0.0f;
          if (k < D) { load8(c + k, cv[m]); load8(r + k, rv[m]); }
        } else {
          load8(c + k, cv[m]);
          load8(r + k, rv[m]);
        }
      }
#pragma unroll
      for (int m = 0; m < N; ++m) accumulate(cv[m], rv[m]);
    };
    int k0 = 0;
    for (; k0 + 2048 <= D; k0 += 2048) part(std::integral_constant<int, 4>{}, std::false_type{}, k0);
    const int rest = D - k0;
    if (rest > 1536) part(std::integral_constant<int, 4>{}, std::true_type{}, k0);
    else if (rest > 1024) part(std::integral_constant<int, 3>{}, std::true_type{}, k0);
    else if (rest > 512) part(std::integral_constant<int, 2>{}, std::true_type{}, k0);
    else if (rest > 0) part(std::integral_constant<int, 1>{}, std::true_type{}, k0);
    srr = wave_sum_rows(srr); sdd = wave_sum_rows(sdd);
    if (NEED_Z) { sc = wave_sum_rows(sc); sr = wave_sum_rows(sr); scc = wave_sum_rows(scc); }
    if (NEED_L1) sad = wave_sum_rows(sad);
    float ns = 0.0f;
    if (NEED_SFR) ns = wave_sum_rows((float)nsi);      // at most D / 64 per lane: exact in fp32
    const float rel = sqrtf(sdd) / fmaxf(sqrtf(srr), 1e-30f);
    if (lane == 0 && token_scores) token_scores[(int64_t)claim * T + t] = rel;
    acc[0] += sc; acc[1] += sr; acc[2] += scc; acc[3] += srr;
    acc[4] += (double)sc - (double)sr;            // sum of differences, only used for the mean of d in the z-scored L2
    acc[5] += sad; acc[6] += sdd; acc[7] += ns;
    if (!(rel <= 3.0e38f)) bad = 1;           // NaN or inf
    else if (rel > best) { best = rel; best_t = (int)t; }
  }

  __shared__ double s_acc[4][8];
  __shared__ float s_best[4];
  __shared__ int s_bt[4], s_bad[4];
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) s_acc[wave][j] = acc[j];
    s_best[wave] = best; s_bt[wave] = best_t; s_bad[wave] = bad;
  }
  __syncthreads();
  ScorePartial* p = partials + (int64_t)claim * tiles_per_claim + tile;
  // one sum each, the waves in order; the worst token beside them
  auto sum_of = [&](int j) { return s_acc[0][j] + s_acc[1][j] + s_acc[2][j] + s_acc[3][j]; };
  auto worst = [&](float& b, int& bt, int& bd) {
    b = -1.0f; bt = 0; bd = 0;
    for (int w = 0; w < 4; ++w) {
      bd |= s_bad[w];
      if (s_best[w] > b || (s_best[w] == b && s_best[w] >= 0.0f && s_bt[w] < bt)) { b = s_best[w]; bt = s_bt[w]; }
    }
  };
  float b; int bt, bd;
  if constexpr (!ALONE) {                              // the records go to score_finalize_kernel
    if (threadIdx.x < 8) {
      p->s[threadIdx.x] = sum_of(threadIdx.x);
    } else if (threadIdx.x == 64) {
      worst(b, bt, bd);
      p->max_rel = b; p->argmax = bt; p->bad = bd; p->launch = 0;
    }
  } else {
    // 1 x 256 tokens of 512: a call 14.8 -> 11.8 us, the host's time for a launch.  (With a counter between fences the call is as short, but
    // the checks around it were longer, by an L2 written back and emptied: 256 tokens of 512 columns, forward, 45.8 us instead of 44.4.)
    __shared__ int s_all;
    if (wave == 0) {
      worst(b, bt, bd);
      if (lane < 8) publish(p, lane, (uint64_t)__double_as_longlong(sum_of(lane)));
      else if (lane == 8) publish(p, 8, (uint64_t)__float_as_uint(b) | (uint64_t)(uint32_t)bt << 32);
      published_so_far();
      if (lane == 8) publish(p, 9, (uint64_t)(uint32_t)bd | (uint64_t)alone.launch << 32);
      published_so_far();
      int missing = 0;
      for (int i = lane; i < tiles_per_claim; i += 64)
        missing |= (uint32_t)(published(partials + (int64_t)claim * tiles_per_claim + i, 9) >> 32) != alone.launch;
      const bool all = __ballot(missing) == 0;
      if (lane == 0) s_all = all;
    }
    __syncthreads();
    if (!s_all) return;
    finalize_claim<true>(partials + (int64_t)claim * tiles_per_claim, tiles_per_claim, claim, T, D, alone.verdict, finalize_threads(tiles_per_claim));
  }
}

// ---------------------------------------------------------------------------------------------
// The same statistics for several submissions against ONE shared reference.  A wave
// owns a token and takes its row in parts of NU KB (NU = 2 .. 4): it loads the reference part into registers once,
// forms the reference's own sums and -- for the sign-flip ratio -- one class mask per element, and then streams the
// same part of every submission of its group past them, the next submission's loads in flight while the current one
// is reduced.  Compared with score_tokens_kernel the reference is read once per group instead of once per submission,
// and its share of the arithmetic is paid once: 7-8 vector instructions per element instead of 16, which moves the
// all-statistics pass from the vector ALUs' bound to the memory's.
//   sign test: sign(a) == sign(b), with sign(0) = sign(NaN) = 0, is one v_cmp_class of a against the set of classes
//   that b's sign allows; the matches are counted on the scalar unit from the lane mask.
// TAIL: rows of any multiple of 8 elements; the last part's lanes past the row's end see zeros on both sides and no sign class.
// ONCE: the submissions' loads are non-temporal (128 of 8192 x 4096 in bf16 read at 5.4 -> 6.2 TB/s).
// Lane c of a wave adds up submission c's sums over the parts of a token (a predicated add after each wave
// reduction) and closes the token -- per-token relative L2, running sums -- for all submissions at once; the four
// waves' sums are folded per submission at the end, into the same per-(submission, tile) records as above.
// With SUM the kernel also writes, per element, the sum over the group's submissions whose bit in `skip` is clear
// (added in index order, fp32): the mean the EMA update needs, without another pass over the submissions.  SUM needs
// the whole set in one group.
constexpr int kGroupMax = 32;                 // submissions per group (<= 64: one lane each)

template <typename E, int N> struct RawUnit;                     // N consecutive elements as they come from memory
template <> struct RawUnit<bf16, 8> { bf16x8 v; __device__ __forceinline__ void load(const bf16* p) { v = *reinterpret_cast<const bf16x8*>(p); }
                                      __device__ __forceinline__ void load_once(const bf16* p) { v = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p)); }
                                      __device__ __forceinline__ float get(int i) const { return static_cast<float>(v[i]); } };
template <> struct RawUnit<bf16, 4> { bf16x4 v; __device__ __forceinline__ void load(const bf16* p) { v = *reinterpret_cast<const bf16x4*>(p); }
                                      __device__ __forceinline__ void load_once(const bf16* p) { v = __builtin_nontemporal_load(reinterpret_cast<const bf16x4*>(p)); }
                                      __device__ __forceinline__ float get(int i) const { return static_cast<float>(v[i]); } };
template <> struct RawUnit<float, 4> { f32x4 v; __device__ __forceinline__ void load(const float* p) { v = *reinterpret_cast<const f32x4*>(p); }
                                      __device__ __forceinline__ void load_once(const float* p) { v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p)); }
                                       __device__ __forceinline__ float get(int i) const { return v[i]; } };
template <> struct RawUnit<float, 8> { f32x4 a, b; __device__ __forceinline__ void load(const float* p) { a = *reinterpret_cast<const f32x4*>(p); b = *reinterpret_cast<const f32x4*>(p + 4); }
                                      __device__ __forceinline__ void load_once(const float* p) { a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p)); b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p + 4)); }
                                       __device__ __forceinline__ float get(int i) const { return i < 4 ? a[i] : b[i - 4]; } };

template <typename EC, typename ER, int NU, bool FULL, bool SUM, bool TAIL, bool ONCE>
__global__ __launch_bounds__(256) void score_parts_kernel(const EC* __restrict__ claims, int64_t claim_stride, const ER* __restrict__ ref,
                                                          int64_t T, int D, int n_claims, int G, int n_groups, int tiles_per_claim,
                                                          float* __restrict__ token_scores, ScorePartial* __restrict__ partials,
                                                          uint32_t skip, float* __restrict__ sum_out) {
  constexpr int EPU = 16 / (int)sizeof(EC);            // elements per 16-byte unit of a submission's row
  constexpr int PE = NU * 64 * EPU;                    // elements per part
  const int parts = TAIL ? (D + PE - 1) / PE : D / PE;
  static_assert(!(SUM && TAIL), "the sum is written for whole parts");
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int group = slot % n_groups;
  const int tile = xcd * ((tiles_per_claim + 7) >> 3) + slot / n_groups;
  if (tile >= tiles_per_claim) return;
  const int c0 = group * G, nc = min(G, n_claims - c0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};            // lane c: submission c0 + c
  float best = -1.0f;
  int best_t = 0, bad = 0;

  for (int i = 0; i < kTPW; ++i) {
    const int64_t t = (int64_t)tile * kScoreTokensPerWG + i * 4 + wave;
    if (t >= T) break;                                 // uniform per wave
    const EC* cb = claims + (int64_t)c0 * claim_stride + t * D + lane * EPU;
    RawUnit<EC, EPU> bufA[NU], bufB[NU];
    auto fetch = [&](RawUnit<EC, EPU> (&buf)[NU], int q) {       // q = part * nc + submission
      const int part = q / nc, c = q - part * nc;
      const EC* p = cb + (int64_t)c * claim_stride + part * PE;
      // TAIL: lanes past the row's end load its last unit; what they hold counts as zero against a zero of the reference
#pragma unroll
      for (int m = 0; m < NU; ++m) {
        const EC* q_m = TAIL ? p + min(m * 64 * EPU, D - EPU - lane * EPU - part * PE) : p + m * 64 * EPU;
        if (ONCE) buf[m].load_once(q_m); else buf[m].load(q_m);
      }
    };
    float sr = 0, srr = 0;                             // the reference's sums: per lane until the token is closed
    float tsdd = 0, tsc = 0, tscc = 0, tsad = 0;       // lane c: submission c's sums over the parts done so far
    int tmatch = 0;
    fetch(bufA, 0);
    const int nq = parts * nc;
    for (int part = 0; part < parts; ++part) {
      const ER* r = ref + t * D + part * PE + lane * EPU;
      float rv[NU][EPU], ssum[NU][EPU];
      int cls[NU][EPU];
#pragma unroll
      for (int m = 0; m < NU; ++m) {
        RawUnit<ER, EPU> u;
        const bool in = !TAIL || part * PE + (m * 64 + lane) * EPU < D;
        u.load(TAIL ? r + min(m * 64 * EPU, D - EPU - lane * EPU - part * PE) : r + m * 64 * EPU);
#pragma unroll
        for (int j = 0; j < EPU; ++j) {
          const float b = in ? u.get(j) : 0.0f;
          rv[m][j] = b;
          srr = fmaf(b, b, srr);
          if (SUM) ssum[m][j] = 0.0f;
          if (FULL) {
            sr += b;
            // classes a may have for sign(a) == sign(b): {+denormal, +normal, +inf}, {-inf, -normal, -denormal}, {NaNs, -0, +0}
            cls[m][j] = b > 0.0f ? 0x380 : (b < 0.0f ? 0x01C : 0x063);
            if (TAIL) cls[m][j] = in ? cls[m][j] : 0;
          }
        }
      }
      auto reduce = [&](const RawUnit<EC, EPU> (&buf)[NU], int c) {
        float sc = 0, scc = 0, sad = 0, sdd = 0;
        int match = 0;                                  // wave-uniform
        const bool add = SUM && ((skip >> (c0 + c)) & 1u) == 0;
#pragma unroll
        for (int m = 0; m < NU; ++m)
#pragma unroll
          for (int j = 0; j < EPU; ++j) {
            const float a = !TAIL || part * PE + (m * 64 + lane) * EPU < D ? buf[m].get(j) : 0.0f, d = a - rv[m][j];
            sdd = fmaf(d, d, sdd);
            if (SUM && add) ssum[m][j] += a;
            if (FULL) {
              sc += a; scc = fmaf(a, a, scc); sad += fabsf(d);
              // the compare's lane mask goes straight to the scalar unit (through the generic ballot the compiler
              // turns the predicate into a register value and compares again)
              uint64_t lanes;
              asm("v_cmp_class_f32_e64 %0, %1, %2" : "=s"(lanes) : "v"(a), "v"(cls[m][j]));
              match += __builtin_popcountll(lanes);
              asm volatile("" : "+s"(match));        // count now: otherwise all the masks stay live until the predicated adds
            }
          }
        sdd = wave_sum_rows(sdd);
        if (FULL) { sc = wave_sum_rows(sc); scc = wave_sum_rows(scc); sad = wave_sum_rows(sad); }
        if (lane == c) { tsdd += sdd; tsc += sc; tscc += scc; tsad += sad; tmatch += match; }
      };
      // The next (part, submission) is fetched before the current one is reduced -- unconditionally (past the end:
      // the last one again, never used), because a fetch behind a branch makes the compiler's wait for the current
      // buffer cover the younger loads too, and nothing would be in flight during the reduction.
      const int q0 = part * nc;
      for (int c = 0; c < nc; c += 2) {
        fetch(bufB, min(q0 + c + 1, nq - 1));
        reduce(bufA, c);
        if (c + 1 < nc) {
          fetch(bufA, min(q0 + c + 2, nq - 1));
          reduce(bufB, c + 1);
        } else {                                       // odd group: the next part's first submission sits in B
#pragma unroll
          for (int m = 0; m < NU; ++m) bufA[m] = bufB[m];
        }
      }
      if (SUM) {
        float* so = sum_out + t * D + part * PE + lane * EPU;
#pragma unroll
        for (int m = 0; m < NU; ++m) {
          if (EPU == 8) {
            f32x4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) { lo[j] = ssum[m][j]; hi[j] = ssum[m][(EPU == 8) ? 4 + j : j]; }
            *reinterpret_cast<f32x4*>(so + m * 64 * EPU) = lo;
            *reinterpret_cast<f32x4*>(so + m * 64 * EPU + 4) = hi;
          } else {
            f32x4 lo;
#pragma unroll
            for (int j = 0; j < 4; ++j) lo[j] = ssum[m][j];
            *reinterpret_cast<f32x4*>(so + m * 64 * EPU) = lo;
          }
        }
      }
    }
    // close the token: every lane for its own submission
    srr = wave_sum_rows(srr);
    if (FULL) sr = wave_sum_rows(sr);
    const float rel = sqrtf(tsdd) / fmaxf(sqrtf(srr), 1e-30f);
    if (lane < nc) {
      if (token_scores) token_scores[(int64_t)(c0 + lane) * T + t] = rel;
      acc[0] += tsc; acc[1] += sr; acc[2] += tscc; acc[3] += srr;
      acc[4] += (double)tsc - (double)sr;
      acc[5] += tsad; acc[6] += tsdd;
      if (FULL) acc[7] += (double)(D - tmatch);
      if (!(rel <= 3.0e38f)) bad = 1;
      else if (rel > best) { best = rel; best_t = (int)t; }
    }
  }

  __shared__ double s_acc[4][kGroupMax][8];
  __shared__ float s_best[4][kGroupMax];
  __shared__ int s_bt[4][kGroupMax], s_bad[4][kGroupMax];
  if (lane < nc) {
#pragma unroll
    for (int j = 0; j < 8; ++j) s_acc[wave][lane][j] = acc[j];
    s_best[wave][lane] = best; s_bt[wave][lane] = best_t; s_bad[wave][lane] = bad;
  }
  __syncthreads();
  if ((int)threadIdx.x < nc) {
    const int c = threadIdx.x;
    ScorePartial p;
#pragma unroll
    for (int j = 0; j < 8; ++j) p.s[j] = s_acc[0][c][j] + s_acc[1][c][j] + s_acc[2][c][j] + s_acc[3][c][j];
    float b = -1.0f; int bt = 0, bd = 0;
    for (int w = 0; w < 4; ++w) {
      bd |= s_bad[w][c];
      if (s_best[w][c] > b || (s_best[w][c] == b && s_best[w][c] >= 0.0f && s_bt[w][c] < bt)) { b = s_best[w][c]; bt = s_bt[w][c]; }
    }
    p.max_rel = b; p.argmax = bt; p.bad = bd; p.launch = 0;
    partials[(int64_t)(c0 + c) * tiles_per_claim + tile] = p;
  }
}

// m <- beta m + (1 - beta) / n * sum: the EMA update from the sum a score_parts_kernel launch has written
__global__ __launch_bounds__(256) void ema_from_sum_kernel(float* __restrict__ m, const float* __restrict__ sum, int64_t n_vec, float beta, float w) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= n_vec) return;
  float mv[8], sv8[8];
  load8(m + v * 8, mv);
  load8(sum + v * 8, sv8);
#pragma unroll
  for (int j = 0; j < 8; ++j) mv[j] = beta * mv[j] + w * sv8[j];
  store8(m + v * 8, mv);
}

template <typename E>
__global__ __launch_bounds__(256) void ema_update_kernel(float* m, const E* __restrict__ claims, int64_t claim_stride,
                                                         int n_claims, const uint8_t* __restrict__ flags, int64_t n_vec, float beta, const float* m_from) {
  // the un-flagged submissions of this step, compacted once per workgroup
  __shared__ int clean[1024];
  __shared__ int s_n;
  if (threadIdx.x == 0) {
    int n = 0;
    for (int i = 0; i < n_claims && n < 1024; ++i)
      if (flags == nullptr || flags[i] == 0) clean[n++] = i;
    s_n = n;
  }
  __syncthreads();
  const int n_clean = s_n;
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= n_vec) return;
  float mv[8];
  load8(m_from + v * 8, mv);
  if (n_clean == 0) {                       // every submission flagged: the EMA is left as it is
    if (m_from != m) store8(m + v * 8, mv);
    return;
  }
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const E* base = claims + v * 8;
  int i = 0;
  for (; i + 3 < n_clean; i += 4) {
    float x0[8], x1[8], x2[8], x3[8];
    load8(base + (int64_t)clean[i] * claim_stride, x0);
    load8(base + (int64_t)clean[i + 1] * claim_stride, x1);
    load8(base + (int64_t)clean[i + 2] * claim_stride, x2);
    load8(base + (int64_t)clean[i + 3] * claim_stride, x3);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += (x0[j] + x1[j]) + (x2[j] + x3[j]);
  }
  for (; i < n_clean; ++i) {
    float x[8];
    load8(base + (int64_t)clean[i] * claim_stride, x);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += x[j];
  }
  const float w = (1.0f - beta) / (float)n_clean;
#pragma unroll
  for (int j = 0; j < 8; ++j) mv[j] = beta * mv[j] + w * acc[j];
  store8(m + v * 8, mv);
}

}  // namespace

namespace {
Verdict make_verdict(uint32_t mask, const float* tau4, int reduce, sv_result* results) {
  Verdict v{mask, {}, reduce, results};
  for (int i = 0; i < 4; ++i) v.tau.v[i] = tau4 ? tau4[i] : 0.0f;
  return v;
}

// Rows of no multiple of 2 KB against a shared reference: does the kernel that keeps the reference in registers beat the one that reads it
// with every submission?  It saves the more, the more submissions share a part of it (n in groups of G) and the more sums there are to
// form (full), and its workgroups are longer: just above two of them on a CU, the few CUs with a third set the time, and where memory
// takes most of it anyway (the relative L2 alone, rows of 3 KB and more) a fifth does so again, until there are many.  An fp32 reference
// of bf16 submissions (mixed) is the other kernel's cheapest form.  Without -> with it, us, submissions x tokens x columns, bf16 unless
// said, all sums: 8 x 8200 x 960 (4.0 workgroups on a CU) 55 -> 41, 16 x 2060 x 2304 (2.0) 52 -> 57, 16 x 3000 x 2304 (2.9) 65 -> 58; 2 x 8200 x
// 64 (2.0) 19.3 -> 20.5, mixed 17.6 -> 20.3, in fp32 19.4 -> 17.4; 3 x 8200 x 3520 (2.0) 52 -> 59.  The relative L2 alone: 64 x 8200 x 504 (8.0)
// 237 -> 103, 16 x 4100 x 1600 (4.0) 40 -> 48, 16 x 7000 x 1600 (6.8) 78 -> 70, 2 x 20000 x 1600 (4.9) 35 -> 40, 6 x 8200 x 3520 (4.0) 79 -> 88, 10 x
// 7000 x 960 in fp32 (5.1) 53 -> 61, 16 x 2560 x 2304 in fp32 (2.5) 90 -> 69.
bool ragged_parts_pay(int n, int G, int64_t workgroups, int units, bool full, int claim_dtype, int ref_dtype) {
  const double per_cu = (double)workgroups / cu_count();
  const bool past_three = per_cu > 2.6, many = per_cu >= 6.5;
  const bool mixed = claim_dtype == SV_BF16 && ref_dtype == SV_F32, all16 = claim_dtype == SV_BF16 && ref_dtype == SV_BF16;
  const int share = n < G ? n : G;
  if (per_cu < 2.0) return false;
  if (units > 8 && share > 2) return true;               // three parts and more: the start of a chain is a small share of it
  if (units > 4) {
    const bool fifth = per_cu >= 4.0 && per_cu < 4.5;
    return share == 2 ? many : past_three && (!fifth || (share > 3 ? full || !all16 : mixed));
  }
  if (full) return units == 2 || (mixed ? past_three && (units > 2 || share > 2) : past_three || units > 2 || share > 3);
  if (units > 2) return share > 2 && per_cu >= (share == 3 && !mixed ? 6.5 : 5.7);
  return past_three || share > 3;
}

bool being_captured(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(st, &s) != hipSuccess || s != hipStreamCaptureStatusNone;
}
}  // namespace

hipError_t launch_score_finalize(const ScorePartial* partials, int n_claims, int tiles, int64_t T, int D, uint32_t mask, const float* tau4,
                                 int reduce, sv_result* results, hipStream_t st) {
  hipLaunchKernelGGL(score_finalize_kernel, dim3(n_claims), dim3(finalize_threads(tiles)), 0, st, partials, tiles, T, D,
                     make_verdict(mask, tau4, reduce, results));
  return hipGetLastError();
}

bool score_sum_supported(int n_claims, int64_t ref_stride, int claim_dtype, int D) {
  const int64_t row_bytes = (int64_t)D * (claim_dtype == SV_BF16 ? 2 : 4);
  return n_claims >= 1 && n_claims <= kGroupMax && ref_stride == 0 && row_bytes % 2048 == 0;
}

hipError_t launch_ema_from_sum(float* m, const float* sum, int n_summed, int64_t T, int D, float beta, hipStream_t st) {
  if (n_summed <= 0 || T <= 0) return hipSuccess;    // nobody entered the sum: the EMA is left as it is
  const int64_t n_vec = T * D / 8;
  hipLaunchKernelGGL(ema_from_sum_kernel, dim3((unsigned)((n_vec + 255) / 256)), dim3(256), 0, st, m, sum, n_vec, beta,
                     (1.0f - beta) / (float)n_summed);
  return hipGetLastError();
}

hipError_t launch_score(const void* claims, int64_t claim_stride, int n_claims, const void* ref, int64_t ref_stride,
                        int claim_dtype, int ref_dtype, int64_t T, int D, uint32_t mask, const float* tau4, int reduce,
                        float* token_scores, sv_result* results, ScorePartial* scratch, int64_t scratch_elems,
                        hipStream_t st, uint32_t* launches, uint32_t skip, float* sum_out) {
  if (n_claims <= 0 || T <= 0) return hipSuccess;
  if (sum_out && !score_sum_supported(n_claims, ref_stride, claim_dtype, D)) return hipErrorInvalidValue;
  const int64_t tiles = (T + kScoreTokensPerWG - 1) / kScoreTokensPerWG;
  int64_t per_launch = scratch_elems / tiles;
  if (per_launch < 1) return hipErrorInvalidValue;
  if (per_launch * (tiles + 7) > 0x7fffffffLL) per_launch = 0x7fffffffLL / (tiles + 7);
  const int64_t csz = claim_dtype == SV_BF16 ? 2 : 4, rsz = ref_dtype == SV_BF16 ? 2 : 4;
  for (int64_t c0 = 0; c0 < n_claims; c0 += per_launch) {
    const int nc = (int)((n_claims - c0 < per_launch) ? (n_claims - c0) : per_launch);
    const char* cp = (const char*)claims + c0 * claim_stride * csz;
    const char* rp = (const char*)ref + c0 * ref_stride * rsz;
    float* ts = token_scores ? token_scores + c0 * T : nullptr;
    const dim3 grid((unsigned)(8 * ((tiles + 7) / 8) * nc)), block(256);
    const int64_t row_bytes = (int64_t)D * csz;
    const bool full = (mask & (SV_M_L1 | SV_M_ZL2 | SV_M_SFR)) != 0;
    // Shared reference and several submissions (or their sum wanted): the kernel that keeps the reference in registers; where the rows
    // are no multiple of 2 KB, if it pays.
    int G = sum_out ? nc : 16;
    while (!sum_out && G > 4 && tiles * ((nc + G - 1) / G) < 1024) G >>= 1;
    const int n_groups = (nc + G - 1) / G;
    G = (nc + n_groups - 1) / n_groups;                  // groups alike: every group reads the reference once
    const bool whole = row_bytes % 2048 == 0;
    const int units = (int)((row_bytes + 1023) / 1024);  // KB of a row
    if (ref_stride == 0 && (sum_out || nc >= 2) &&
        (whole || ragged_parts_pay(nc, G, tiles * n_groups, units, full, claim_dtype, ref_dtype))) {
      if (sum_out && (nc != n_claims || nc * tiles > scratch_elems)) return hipErrorInvalidValue;   // one launch, one group
      const dim3 ggrid((unsigned)(8 * ((tiles + 7) / 8) * n_groups));
#define SV_LAUNCH_PARTS5(EC, ER, NU, FULL, SUM, TAIL, ONCE)                                                           \
  hipLaunchKernelGGL((score_parts_kernel<EC, ER, NU, FULL, SUM, TAIL, ONCE>), ggrid, block, 0, st, (const EC*)cp, claim_stride, (const ER*)rp, T, D, \
                     nc, G, n_groups, (int)tiles, ts, scratch, skip, sum_out)
#define SV_LAUNCH_PARTS4(EC, ER, NU, SUM, TAIL, ONCE)                                                                 \
  do { if (full) SV_LAUNCH_PARTS5(EC, ER, NU, true, SUM, TAIL, ONCE); else SV_LAUNCH_PARTS5(EC, ER, NU, false, SUM, TAIL, ONCE); } while (0)
#define SV_LAUNCH_PARTS3(EC, ER, NU, TAIL)                                                                            \
  do { if (once) SV_LAUNCH_PARTS4(EC, ER, NU, false, TAIL, true); else SV_LAUNCH_PARTS4(EC, ER, NU, false, TAIL, false); } while (0)
#define SV_LAUNCH_WHOLE(EC, ER, NU)                                                                                   \
  do { if (sum_out) SV_LAUNCH_PARTS4(EC, ER, NU, true, false, false); else SV_LAUNCH_PARTS3(EC, ER, NU, false); } while (0)
#define SV_LAUNCH_PARTS(EC, ER)                                                                                       \
  do { if (!whole) { if (nu == 4) SV_LAUNCH_PARTS3(EC, ER, 4, true); else if (nu == 3) SV_LAUNCH_PARTS3(EC, ER, 3, true); else SV_LAUNCH_PARTS3(EC, ER, 2, true); } \
       else if (row_bytes % 4096 == 0) SV_LAUNCH_WHOLE(EC, ER, 4); else SV_LAUNCH_WHOLE(EC, ER, 2); } while (0)
      // more than the memory-side cache holds (256 MB): loads that leave nothing behind.  128 x 8192 x 4096 1587 -> 1394 us, 16 x 4096 x
      // 4096 (0.5 GB) 121 -> 114.5; but 4 x 2048 x 2048 (33 MB) 27.7 -> 28.6
      const bool once = row_bytes * T * nc > ((int64_t)256 << 20);
      int nu = 4;                                        // units per part: as few as possible for nothing
      for (int u = 3; u >= 2; --u)
        if ((units + u - 1) / u * u < (units + nu - 1) / nu * nu) nu = u;
      if (claim_dtype == SV_BF16 && ref_dtype == SV_BF16) SV_LAUNCH_PARTS(bf16, bf16);
      else if (claim_dtype == SV_BF16) SV_LAUNCH_PARTS(bf16, float);
      else if (ref_dtype == SV_BF16) SV_LAUNCH_PARTS(float, bf16);
      else SV_LAUNCH_PARTS(float, float);
#undef SV_LAUNCH_PARTS
#undef SV_LAUNCH_WHOLE
#undef SV_LAUNCH_PARTS4
#undef SV_LAUNCH_PARTS3
#undef SV_LAUNCH_PARTS5
      hipError_t e = launch_score_finalize(scratch, nc, (int)tiles, T, D, mask, tau4, reduce, results + c0, st);
      if (e != hipSuccess) return e;
      continue;
    }
    const int64_t tiles4 = (T + 3) / 4;                // up to one record of 16 tokens per CU: smaller ones (see the kernel)
    const bool few = tiles * nc <= cu_count() && tiles4 * nc <= scratch_elems;
    const int tpc = (int)(few ? tiles4 : tiles);
    const dim3 gridt((unsigned)(8 * ((tpc + 7) / 8) * nc));
    // Few records, where the host's launches are what a caller waits for: one launch.  32 records 14.7 -> 11.8 us, 64 14.8 -> 11.8; every
    // workgroup pays for publishing its record and reading the others' numbers, about a microsecond of the GPU's time.  Under capture
    // a launch's number would be that of its every replay: two launches.
    uint32_t launch = 0;
    if (launches && few && (int64_t)tpc * nc <= kScoreAloneRecords && !being_captured(st)) {
      if (++*launches == 0) ++*launches;                 // 0 is in the records of other launches
      launch = *launches;
    }
    const Verdict verdict = make_verdict(mask, tau4, reduce, results + c0);
#define SV_LAUNCH_SCORE3(EC, ER, L1, Z, SFR)                                                                           \
  do {                                                                                                                 \
    if (launch) hipLaunchKernelGGL((score_tokens_kernel<EC, ER, L1, Z, SFR, 4, true>), gridt, block, 0, st, (const EC*)cp, claim_stride,  \
                                (const ER*)rp, ref_stride, T, D, nc, tpc, ts, scratch, Alone<true>{launch, verdict});         \
    else if (few) hipLaunchKernelGGL((score_tokens_kernel<EC, ER, L1, Z, SFR, 4, false>), gridt, block, 0, st, (const EC*)cp, claim_stride,  \
                                (const ER*)rp, ref_stride, T, D, nc, tpc, ts, scratch, Alone<false>{});         \
    else hipLaunchKernelGGL((score_tokens_kernel<EC, ER, L1, Z, SFR, kScoreTokensPerWG, false>), gridt, block, 0, st, (const EC*)cp, claim_stride, \
                            (const ER*)rp, ref_stride, T, D, nc, tpc, ts, scratch, Alone<false>{});             \
  } while (0)
#define SV_LAUNCH_SCORE(EC, ER)                                                                                          \
  do {                                                                                                                   \
    const bool l1 = mask & SV_M_L1, z = mask & SV_M_ZL2, sfr = mask & SV_M_SFR;                                          \
    if (!l1 && !z && !sfr) SV_LAUNCH_SCORE3(EC, ER, false, false, false);                                                \
    else if (l1 && !z && !sfr) SV_LAUNCH_SCORE3(EC, ER, true, false, false);                                             \
    else if (!l1 && !z && sfr) SV_LAUNCH_SCORE3(EC, ER, false, false, true);                                             \
    else if (!l1 && z && !sfr) SV_LAUNCH_SCORE3(EC, ER, false, true, false);                                             \
    else SV_LAUNCH_SCORE3(EC, ER, true, true, true);                                                                     \
  } while (0)
    if (claim_dtype == SV_BF16 && ref_dtype == SV_BF16) SV_LAUNCH_SCORE(bf16, bf16);
    else if (claim_dtype == SV_BF16) SV_LAUNCH_SCORE(bf16, float);
    else if (ref_dtype == SV_BF16) SV_LAUNCH_SCORE(float, bf16);
    else SV_LAUNCH_SCORE(float, float);
#undef SV_LAUNCH_SCORE
#undef SV_LAUNCH_SCORE3
    hipError_t e = launch ? hipGetLastError() : launch_score_finalize(scratch, nc, tpc, T, D, mask, tau4, reduce, results + c0, st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

// Alg. gradient_replacement: every signal whose mask byte is set is overwritten with the reference point m
// (rounded to the signal's dtype); the others are left alone.  The workgroups of a signal stride over its 8-element vectors.
template <typename E>
__global__ __launch_bounds__(256) void replace_kernel(E* __restrict__ signals, int64_t stride, const uint8_t* __restrict__ mask,
                                                      const float* __restrict__ m, int64_t n_vec) {
  if (mask[blockIdx.y] == 0) return;
  for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n_vec; v += (int64_t)gridDim.x * 256) {
    float x[8];
    load8(m + v * 8, x);
    store8(signals + (int64_t)blockIdx.y * stride + v * 8, x);
  }
}

hipError_t launch_replace(void* signals, int64_t stride, int n, int dtype, const uint8_t* mask, const float* m, int64_t T, int D,
                          hipStream_t st) {
  if (n <= 0 || T <= 0) return hipSuccess;
  const int64_t n_vec = T * D / 8;
  // few workgroups per signal: most signals are left alone, and a workgroup that only reads its mask byte should be cheap
  const dim3 grid((unsigned)min((n_vec + 255) / 256, (int64_t)1024), (unsigned)n), block(256);
  if (dtype == SV_BF16) hipLaunchKernelGGL(replace_kernel<bf16>, grid, block, 0, st, (bf16*)signals, stride, mask, m, n_vec);
  else hipLaunchKernelGGL(replace_kernel<float>, grid, block, 0, st, (float*)signals, stride, mask, m, n_vec);
  return hipGetLastError();
}

hipError_t launch_ema(float* m, const void* claims, int64_t claim_stride, int n_claims, int claim_dtype,
                      const uint8_t* flags, int64_t T, int D, float beta, hipStream_t st, const float* m_from) {
  if (n_claims <= 0 || T <= 0) return hipSuccess;
  if (!m_from) m_from = m;
  const int64_t n_vec = T * D / 8;
  const dim3 grid((unsigned)((n_vec + 255) / 256)), block(256);
  if (claim_dtype == SV_BF16)
    hipLaunchKernelGGL(ema_update_kernel<bf16>, grid, block, 0, st, m, (const bf16*)claims, claim_stride, n_claims, flags, n_vec, beta, m_from);
  else
    hipLaunchKernelGGL(ema_update_kernel<float>, grid, block, 0, st, m, (const float*)claims, claim_stride, n_claims, flags, n_vec, beta, m_from);
  return hipGetLastError();
}

}  // namespace sv

// ---------------------------------------------------------------------------------------------------------------
// The statistic for callers that cannot allocate.  sv_score_and_flag keeps its per-(submission, token tile) partial
// records in the context's workspace, which sv_create allocates; here the same records live in a file-scope device
// array that exists once per GPU from the moment the library's code object is loaded on it until the process ends.
namespace {

constexpr int64_t kStaticScoreRecords = 1 << 16;          // 5 MiB: e.g. 128 submissions of 8192 tokens
static __device__ __align__(256) unsigned char scratch[kStaticScoreRecords * sizeof(sv::ScorePartial)];

constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
sv::ScorePartial* g_static_ptr[kMaxDevices] = {};          // device address of `scratch` on each GPU, asked for once

// The array's name is a host-side handle, not a device address: the address on the CURRENT device comes from the
// runtime, once per device, and only that pointer is ever handed to a kernel.
hipError_t static_score_scratch(sv::ScorePartial** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (!g_static_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_static_ptr[dev] = (sv::ScorePartial*)p;
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}

}  // namespace

extern "C" sv_status sv_score_and_flag_noalloc(const void* claims, int64_t claim_stride, int32_t n_claims, const void* ref,
                                               int64_t ref_stride, int32_t claim_dtype, int32_t ref_dtype, int64_t T, int32_t D,
                                               uint32_t metric_mask, const float* tau, int32_t reduce, float* token_scores_out,
                                               sv_result* results_dev, void* stream) {
  using sv::set_global_error;
  if (n_claims < 0 || T < 0 || D < 1) { set_global_error("negative size"); return SV_EINVAL; }
  if (n_claims == 0 || T == 0) return SV_OK;
  if (!claims || !ref || !results_dev || !tau) { set_global_error("claims, ref, tau and results_dev must be non-NULL"); return SV_EINVAL; }
  if ((claim_dtype != SV_F32 && claim_dtype != SV_BF16) || (ref_dtype != SV_F32 && ref_dtype != SV_BF16)) {
    set_global_error("unknown dtype");
    return SV_EINVAL;
  }
  if (reduce != SV_REDUCE_GLOBAL && reduce != SV_REDUCE_MAX_TOKEN) { set_global_error("unknown reduce"); return SV_EINVAL; }
  if (D % 8) { set_global_error("D must be a multiple of 8"); return SV_EUNSUPPORTED; }
  if (T > 0x7fffffffLL || claim_stride < 0 || ref_stride < 0) { set_global_error("T or a stride is out of range"); return SV_EINVAL; }
  const int64_t tiles = (T + sv::kScoreTokensPerWG - 1) / sv::kScoreTokensPerWG;
  if (tiles * (int64_t)n_claims > kStaticScoreRecords) {
    set_global_error("n_claims * ceil(T / %d) = %lld exceeds the %lld partial records of the static scratch: split the call or use "
                     "sv_score_and_flag with a context", sv::kScoreTokensPerWG, (long long)(tiles * n_claims), (long long)kStaticScoreRecords);
    return SV_EUNSUPPORTED;
  }
  sv::ScorePartial* records = nullptr;
  hipError_t e = static_score_scratch(&records);
  if (e != hipSuccess) { set_global_error("hipGetSymbolAddress of the static scratch failed: %s", hipGetErrorString(e)); return SV_EHIP; }
  // every record the finalize step reads is written by the pass before it in this same call, so nothing has to be
  // cleared between calls; the records of an earlier, larger call beyond this call's range are simply not read
  e = sv::launch_score(claims, claim_stride, n_claims, ref, ref_stride, claim_dtype, ref_dtype, T, D, metric_mask, tau, reduce,
                       token_scores_out, results_dev, records, kStaticScoreRecords, (hipStream_t)stream, nullptr);
  if (e != hipSuccess) { set_global_error("launching the score pass failed: %s", hipGetErrorString(e)); return SV_EHIP; }
  return SV_OK;
}
