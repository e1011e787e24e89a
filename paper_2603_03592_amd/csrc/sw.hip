// Sliced Wasserstein statistic Omega_SW (paragraph "Choice of Distance Measure"): the mean over L
// directions u of the 1-Wasserstein distance between the two signals projected on u.  The samples
// of a signal are its T token vectors; with equal sample counts W1 on the line is the mean absolute
// difference of the sorted projections.
//
// Three steps, all on the caller's stream:
//   project : P[l][t] = <x_t, u_l>          MFMA, HBM-bound (one read of the signal)
//   sort    : every row P[l][.] ascending   bitonic network in LDS (+ global steps for long rows)
//   W1      : sum_t |P_claim[l][t] - P_ref[l][t]| fused into the claim's last sort stage, fixed
//             summation order; a finalize kernel averages over l and applies the threshold.
#include "common.h"

namespace sv {
namespace {

constexpr int kSortChunkMax = (int)kSwSortChunkMax;   // floats sorted in LDS by one workgroup (64 KB)

// ---------------------------------------------------------------------------------------------
// Projection.  A workgroup of 4 waves owns 128 or 256 tokens (kSwTB blocks of 32 per wave) and all
// L = 32 * LB directions; the contraction runs over the feature axis in steps of 16 on
// v_mfma_f32_32x32x16_bf16 with the directions in the A slot, so a lane ends up with one token
// (lane & 31) and the directions 8q + 4 (lane >> 5) + r of each block of 32.
// The signal is streamed in chunks of 128 bytes per row (64 bf16 or 32 fp32 features): the
// [rows x 128 B] tile goes global -> LDS with global_load_lds (8 lanes fetch one row's 128
// contiguous bytes; the 16-byte pieces are XOR-swizzled by choosing which piece a lane fetches),
// three tiles deep, so that two chunks are always in flight and the wait at the end of a chunk
// leaves the youngest one outstanding.  The matching [L x chunk] piece of the directions takes the same
// road.  Fragments are 16-byte LDS reads, conflict-free with the swizzle.
// fp32 signals are split into three bf16 terms (x = hi + mid + lo exactly), three MFMAs per step:
// every product is exact in fp32, so the result has fp32-accumulation accuracy.
__device__ __forceinline__ int sw_swz(int row) { return (row ^ (row >> 3)) & 7; }

template <int LB>
__device__ __forceinline__ void mac_bf16(const bf16x8 (&u)[LB], const bf16x8& x, f32x16 (&acc)[LB]) {
#pragma unroll
  for (int b = 0; b < LB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[b], x, acc[b], 0, 0, 0);
}

template <int LB>
__device__ __forceinline__ void mac_f32(const bf16x8 (&u)[LB], const f32x4& x0, const f32x4& x1, f32x16 (&acc)[LB]) {
  bf16x8 hi, mid, lo;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float x = i < 4 ? x0[i] : x1[i - 4];
    const bf16 a = (bf16)x;
    const float r1 = x - (float)a;
    const bf16 b = (bf16)r1;
    const float r2 = r1 - (float)b;
    hi[i] = a; mid[i] = b; lo[i] = (bf16)r2;
  }
  mac_bf16<LB>(u, lo, acc);
  mac_bf16<LB>(u, mid, acc);
  mac_bf16<LB>(u, hi, acc);
}

// Blocks of 32 tokens per wave: with up to 64 directions one, so that a tile's three chunks take 72 KB and two workgroups share a
// CU, one streaming while the other starts or ends; with more the directions' chunk is as large as the signal's and two blocks share it.
template <int LB> constexpr int kSwTB = LB <= 2 ? 1 : 2;
template <int LB> constexpr int kSwTile = kSwTB<LB> * 128 * 128;     // bytes of one signal tile in LDS
constexpr int kSwDepth = 3;            // signal tiles (and direction chunks) in LDS: two chunks in flight

template <int N> __device__ __forceinline__ void wait_vm_lds_barrier() {      // wait until at most N vector-memory loads are in flight
  static_assert(N >= 5 && N <= 12, "4 or 8 signal loads + 1..4 direction loads per chunk");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0070 | N);                          // vmcnt(N) lgkmcnt(0)
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <typename E, int LB>
__device__ __forceinline__ void sw_project_body(const char* __restrict__ xbase, const bf16* __restrict__ U, int D, int64_t T, int64_t Tpad,
                                                float* __restrict__ out, char* smem, unsigned sig, bool pad) {
  constexpr bool kBf16 = sizeof(E) == 2;
  constexpr int KC = 128 / (int)sizeof(E);            // features per chunk
  constexpr int NSTEP = KC / 16;                      // MFMA k steps per chunk
  constexpr int UPITCH = KC * 2;                      // bytes of a direction row per chunk: 128 (bf16 signal) or 64 (fp32 signal)
  constexpr int UTILE = LB * 32 * UPITCH;
  constexpr int UINSTR = UTILE / 1024;                // direct-to-LDS instructions per directions' chunk
  constexpr int UW = (UINSTR + 3) / 4;                // ... per wave (every wave issues the same number: the waits count them)
  constexpr int RPI = 1024 / UPITCH;                  // direction rows per instruction: 8 or 16
  constexpr int TB = kSwTB<LB>, XI = 4 * TB, XTILE = kSwTile<LB>;      // direct-to-LDS instructions of a wave per signal chunk
  char* xs = smem;                                    // kSwDepth signal tiles
  char* us = smem + kSwDepth * XTILE;               // kSwDepth direction chunks
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l31 = lane & 31, lhi = lane >> 5;
  const int64_t tile0 = (int64_t)blockIdx.x * (128 * TB);
  // direct-to-LDS plan: instruction i of this wave covers the tile rows (wave + 4 i) * 8 .. + 7
  int64_t xoff[XI];
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int r = (wave + 4 * i) * 8 + (lane >> 3), c = (lane & 7) ^ sw_swz(r);
    xoff[i] = min(tile0 + r, T - 1) * (int64_t)D * (int64_t)sizeof(E) + c * 16;     // rows past the end re-read the last one
  }
  // The directions' chunk [L rows x UPITCH bytes] goes the same way (no registers, so the only vector-memory
  // operations in flight are direct-to-LDS loads and the waits can count them exactly; staged through registers, the
  // compiler's wait before the LDS write also waited for the youngest signal chunk).  Instruction j of this wave covers
  // the rows RPI * i .. + RPI - 1, i = min(wave + 4 j, UINSTR - 1) (a repeated instruction rewrites the same bytes).
  // 16-byte pieces are XOR-swizzled by the row so that the 32 rows a fragment read touches spread over the banks.
  auto u_swz = [](int r) { return kBf16 ? sw_swz(r) : ((r >> 2) & 3); };
  int64_t uoff[UW];
  int ulds[UW];
#pragma unroll
  for (int j = 0; j < UW; ++j) {
    const int i = min(wave + 4 * j, UINSTR - 1);
    const int r = i * RPI + lane / (UPITCH / 16), c = (lane % (UPITCH / 16)) ^ u_swz(r);
    uoff[j] = (int64_t)r * D * 2 + c * 16;
    ulds[j] = i * 1024;
  }
  // Workgroups that run together start at different chunks: with a row pitch that is a multiple of the memory
  // channels' interleave, everybody reading column chunk kc of its rows at the same time would camp on few channels.
  const int nchunk = D / KC;
  const int rot = (int)((blockIdx.x * 5u + sig * 3u) % (unsigned)nchunk);      // sig: index of the signal in its tensor
  auto chunk_of = [&](int kc) { const int c = kc + rot; return c >= nchunk ? c - nchunk : c; };
  auto dma = [&](int kc, int stage) {
    const int ck = chunk_of(kc);
#pragma unroll
    for (int j = 0; j < UW; ++j)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)U + uoff[j] + (int64_t)ck * UPITCH),
                                       (__attribute__((address_space(3))) void*)(us + stage * UTILE + ulds[j]), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < XI; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xbase + xoff[i] + (int64_t)ck * 128),
                                       (__attribute__((address_space(3))) void*)(xs + stage * XTILE + (wave + 4 * i) * 1024), 16, 0, 0);
  };
  f32x16 acc[TB][LB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int b = 0; b < LB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[tb][b][i] = 0.0f;

  dma(0, 0);
  dma(nchunk > 1 ? 1 : 0, 1);                          // a second chunk is always issued: the waits below count on it
  wait_vm_lds_barrier<XI + UW>();
  int st = 0;                                          // LDS tile of chunk kc
  for (int kc = 0; kc < nchunk; ++kc) {
    const int st2 = st == 0 ? kSwDepth - 1 : st - 1;   // tile of chunk kc + 2: the one chunk kc - 1 was read from
    dma(kc + 2 < nchunk ? kc + 2 : nchunk - 1, st2);   // past the end: re-read the last chunk (never used)
    const char* xt = xs + st * XTILE;
    const char* ub = us + st * UTILE;
#pragma unroll
    for (int s = 0; s < NSTEP; ++s) {
      bf16x8 u[LB];
#pragma unroll
      for (int b = 0; b < LB; ++b) {
        const int r = b * 32 + l31;
        u[b] = *reinterpret_cast<const bf16x8*>(ub + r * UPITCH + (((2 * s + lhi) ^ u_swz(r)) << 4));
      }
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        const int r = (wave * TB + tb) * 32 + l31;
        if (kBf16) {
          const bf16x8 x = *reinterpret_cast<const bf16x8*>(xt + r * 128 + (((2 * s + lhi) ^ sw_swz(r)) << 4));
          mac_bf16<LB>(u, x, acc[tb]);
        } else {
          const int c = 2 * (2 * s + lhi);
          const f32x4 x0 = *reinterpret_cast<const f32x4*>(xt + r * 128 + ((c ^ sw_swz(r)) << 4));
          const f32x4 x1 = *reinterpret_cast<const f32x4*>(xt + r * 128 + (((c + 1) ^ sw_swz(r)) << 4));
          mac_f32<LB>(u, x0, x1, acc[tb]);
        }
      }
    }
    // chunk kc + 1 has landed (only the loads of chunk kc + 2 may still be in flight) and this wave is done with
    // tile st; after the barrier that holds for the whole workgroup
    wait_vm_lds_barrier<XI + UW>();
    st = st + 1 >= kSwDepth ? 0 : st + 1;
  }
  __builtin_amdgcn_s_waitcnt(0);                       // every direct-to-LDS load has landed before the LDS is given back
  const int64_t t0 = tile0 + wave * (32 * TB);
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int64_t t = t0 + tb * 32 + l31;
    if (t >= T) continue;
#pragma unroll
    for (int b = 0; b < LB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        out[(int64_t)(b * 32 + (i >> 2) * 8 + lhi * 4 + (i & 3)) * Tpad + t] = acc[tb][b][i];
  }
  // The sort does not look at a row's padding.  Where the rows are the caller's it is filled with infinities all the same, a share by
  // every workgroup of the signal (tiles past the last token, which did it before, read and multiplied for nothing: 191 -> 172 us
  // for 33 signals of 6000 x 2048).
  if (pad) {
    const int64_t w = (Tpad - T + gridDim.x - 1) / gridDim.x, p0 = T + (int64_t)blockIdx.x * w;
    const int n = (int)max((int64_t)0, min(w, Tpad - p0));
    for (int e = tid; e < n * LB * 32; e += 256) out[(int64_t)(e / n) * Tpad + p0 + e % n] = __builtin_huge_valf();
  }
}

// The launch covers n2 (0 or 1) signals of type E2 at X2 -- projected into P2 -- in the grid rows 0 .. n2 - 1, and behind
// them the signals X + i * x_stride of type E, projected into the slots P + i * L * Tpad.  A single reference tensor has
// too few token tiles to fill the chip; in one launch with the submissions it runs beside them.
template <typename E, typename E2, int LB>
__global__ __launch_bounds__(256) void sw_project_kernel(const E* __restrict__ X, int64_t x_stride, const E2* __restrict__ X2, int n2,
                                                         const bf16* __restrict__ U, int D, int64_t T, int64_t Tpad,
                                                         float* __restrict__ P, float* __restrict__ P2, bool pad) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int y = blockIdx.y;                           // uniform
  if constexpr (sizeof(E) == sizeof(E2)) {
    const char* xb = y < n2 ? (const char*)X2 : (const char*)(X + (int64_t)(y - n2) * x_stride);
    float* out = y < n2 ? P2 : P + (int64_t)(y - n2) * (LB * 32) * Tpad;
    sw_project_body<E, LB>(xb, U, D, T, Tpad, out, smem, y < n2 ? y : y - n2, pad);
  } else {
    if (y < n2) sw_project_body<E2, LB>((const char*)X2, U, D, T, Tpad, P2, smem, y, pad);
    else sw_project_body<E, LB>((const char*)(X + (int64_t)(y - n2) * x_stride), U, D, T, Tpad, P + (int64_t)(y - n2) * (LB * 32) * Tpad, smem, y - n2, pad);
  }
}

// ---------------------------------------------------------------------------------------------
// Bitonic sorting network on rows of length Tpad (a power of two), ascending everywhere: in the first stage of level k
// element i of a block of k meets its mirror image k - 1 - i, in the others i meets i + j.  So a comparator is a minimum and a
// maximum and needs no direction.  It works on keys, the float's bits made to order as unsigned numbers: a total order, with
// NaNs at the ends.  Padding is the largest key of all and never leaves the positions from T on, so whatever touches
// padding only is skipped (27 % of the network at T = 6000).  The result is the same for every input.
//
// sw_sort_chunk_kernel keeps a chunk of `ch` consecutive elements in LDS and runs the levels
// k = k_first, 2 k_first, ..., k_last on it.  With k_first = 2 and k_last = ch it sorts the chunk from scratch; with
// k_first = k_last = k > ch it finishes level k after sw_sort_global_kernel has done the strides j >= ch.
// If `ref` is non-null (only for ch == Tpad) the sorted row is not written back; instead the
// workgroup adds up |row[i] - ref_row[i]| over the T real samples in a fixed order and stores the
// sum in w1[first_seg + segment]; the reference row is row (segment % L) of `ref` when ref_shared,
// else row `segment`.
//
// A stage per round trip through LDS would be LDS-bound, so a thread takes eight vectors of four elements
// v0 + m s (m = 0..7; of a mirrored stage's upper half the mirrored ones) into registers and runs up to three stages
// (vector strides 4s, 2s, s) on them per round trip; the last pass of a level (s = 1: 32 consecutive elements) also runs
// the strides 2 and 1 inside the vectors, and the first pass of a sort from scratch all of the levels
// k = 2 .. 32 (15 stages).  13 levels of an 8192-element row take 24 round trips instead of 91.  What is left is about half
// arithmetic (two instructions per comparator; with directions and float comparisons it was three and a scalar one) and half LDS.
// 1024 rows of 8192 against a reference: 71 -> 56 us, 64 rows alone 39 -> 28, 2048 rows at T = 6000 139 -> 100.
// Vectors are XOR-swizzled in LDS (bits 4, 5, 6 of the vector index folded into bits
// 1, 2 and 0 + 3) so that 16 neighbouring lanes hit 16 different 16-byte slots at every stride.
typedef __attribute__((ext_vector_type(4))) uint32_t key4;
constexpr uint32_t kPadKey = 0xffffffffu;

__device__ __forceinline__ uint32_t key_of(float x) {
  const uint32_t b = __float_as_uint(x);
  return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float value_of(uint32_t k) { return __uint_as_float(k ^ (~(uint32_t)((int32_t)k >> 31) | 0x80000000u)); }
__device__ __forceinline__ key4 keys_of(const f32x4& v) { return key4{key_of(v[0]), key_of(v[1]), key_of(v[2]), key_of(v[3])}; }

__device__ __forceinline__ void cx(uint32_t& a, uint32_t& b) {
  const uint32_t lo = min(a, b), hi = max(a, b);
  a = lo; b = hi;
}
template <int A, int B>
__device__ __forceinline__ void cx_in(key4& v) {                     // components A and B of one vector
  uint32_t a = v[A], b = v[B];
  cx(a, b);
  v[A] = a; v[B] = b;
}
template <int FLIP>
__device__ __forceinline__ void cxv(key4& a, key4& b) {              // component i meets component i, or (FLIP) 3 - i
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = FLIP ? 3 - i : i;
    uint32_t x = a[i], y = b[j];
    cx(x, y);
    a[i] = x; b[j] = y;
  }
}
// vectors m and m + SM of the eight
template <int SM>
__device__ __forceinline__ void vec_stage(key4 (&e)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m)
    if ((m & SM) == 0) cxv<0>(e[m], e[m + SM]);
}
// first stage of a level on blocks of N of the eight vectors: vector m meets vector N - 1 - m, last component first
template <int N>
__device__ __forceinline__ void mirror_stage(key4 (&e)[8]) {
#pragma unroll
  for (int b = 0; b < 8; b += N)
#pragma unroll
    for (int m = 0; m < N / 2; ++m) cxv<1>(e[b + m], e[b + N - 1 - m]);
}
// strides 2 and 1 inside every vector
__device__ __forceinline__ void in_stages(key4 (&e)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    cx_in<0, 2>(e[m]); cx_in<1, 3>(e[m]);
    cx_in<0, 1>(e[m]); cx_in<2, 3>(e[m]);
  }
}

__global__ __launch_bounds__(512) void sw_sort_chunk_kernel(const float* src, float* P, int64_t Tpad, int ch, int64_t k_first, int64_t k_last,
                                                            const float* __restrict__ ref, int ref_shared, int L, int64_t T,
                                                            float* __restrict__ w1, int first_seg) {
  extern __shared__ __attribute__((aligned(16))) float s[];
  key4* s4 = reinterpret_cast<key4*>(s);
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t gbase = (int64_t)blockIdx.x * ch;
  const float* from = src + (int64_t)blockIdx.y * Tpad + gbase;   // rows to read; P itself if they are sorted in place
  float* row = P + (int64_t)blockIdx.y * Tpad + gbase;
  const int nvec = ch >> 2, ngroups = ch >> 5;
  const int real = (int)min((int64_t)ch, max((int64_t)0, T - gbase));      // the chunk's elements from here on are padding, always
  const bool swz = nvec >= 128;                       // the swizzle permutes inside blocks of 128 vectors
  auto phys = [&](int v) { return swz ? v ^ ((((v >> 4) & 3) << 1) | (((v >> 6) & 1) * 9)) : v; };
  for (int v = tid; v < nvec; v += nt) {
    key4 e = key4{kPadKey, kPadKey, kPadKey, kPadKey};
    if (4 * v < real) e = keys_of(*reinterpret_cast<const f32x4*>(from + 4 * v));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * v + i >= real) e[i] = kPadKey;
    s4[phys(v)] = e;
  }
  __syncthreads();

  // one round trip: the stages `mask` (4: stride 4s, or with `mirror` the mirrored stage; 2: stride 2s, 1: stride s, in
  // vectors), and with in_vec (s = 1 only) the strides 2 and 1 inside the vectors
  auto pass = [&](bool mirror, int s_log, int mask, bool in_vec) {
    for (int g = tid; g < ngroups; g += nt) {
      const int off = g & ((1 << s_log) - 1), v0 = ((g >> s_log) << (3 + s_log)) + off;
      if (4 * v0 >= real) continue;
      const int up = mirror ? (1 << s_log) - 1 - 2 * off : 0;                // from an offset to its mirror image
      key4 e[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) e[m] = s4[phys(v0 + (m << s_log) + (m >= 4 ? up : 0))];
      if (mask & 4) { if (mirror) mirror_stage<8>(e); else vec_stage<4>(e); }
      if (mask & 2) vec_stage<2>(e);
      if (mask & 1) vec_stage<1>(e);
      if (in_vec) in_stages(e);
#pragma unroll
      for (int m = 0; m < 8; ++m) s4[phys(v0 + (m << s_log) + (m >= 4 ? up : 0))] = e[m];
    }
    __syncthreads();
  };

  int64_t k = k_first;
  if (k_first <= 2) {                                  // levels 2 .. 32 on 32 consecutive elements, one round trip
    for (int g = tid; g < ngroups; g += nt) {
      if (32 * g >= real) continue;
      key4 e[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) e[m] = s4[phys(8 * g + m)];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        cx_in<0, 1>(e[m]); cx_in<2, 3>(e[m]);                                                               // level 2
        cx_in<0, 3>(e[m]); cx_in<1, 2>(e[m]); cx_in<0, 1>(e[m]); cx_in<2, 3>(e[m]);                        // level 4
      }
      mirror_stage<2>(e); in_stages(e);                                                                     // level 8
      mirror_stage<4>(e); vec_stage<1>(e); in_stages(e);                                                    // level 16
      mirror_stage<8>(e); vec_stage<2>(e); vec_stage<1>(e); in_stages(e);                                   // level 32
#pragma unroll
      for (int m = 0; m < 8; ++m) s4[phys(8 * g + m)] = e[m];
    }
    __syncthreads();
    k = 64;
  }
  for (; k <= k_last; k <<= 1) {
    // vector-stride stages of this level inside the chunk: strides min(k, ch) / 8 ... 1; the first one is mirrored if the
    // level's own first stage is inside the chunk
    int cur = 0;
    for (int64_t j = (k < ch ? k : (int64_t)ch) >> 3; j >= 1; j >>= 1) ++cur;
    bool mirror = k <= ch;
    while (cur > 3) {                                  // leading stages: first the remainder, then threes
      const int g = (cur - 3) % 3 == 0 ? 3 : (cur - 3) % 3;
      // the eight vectors always span twice the top stride (s = top / 4); a remainder runs the upper stages only
      pass(mirror, cur - 3, g == 3 ? 7 : (g == 2 ? 6 : 4), false);
      cur -= g;
      mirror = false;
    }
    pass(false, 0, cur == 3 ? 7 : (cur == 2 ? 3 : 1), true);
  }
  if (ref == nullptr) {
    for (int v = tid; v < nvec; v += nt) {
      const key4 e = s4[phys(v)];
      *reinterpret_cast<f32x4*>(row + 4 * v) = f32x4{value_of(e[0]), value_of(e[1]), value_of(e[2]), value_of(e[3])};
    }
    return;
  }
  const int seg = blockIdx.y;
  const float* rrow = ref + (int64_t)(ref_shared ? seg % L : seg) * Tpad;
  float sum = 0.0f;
  for (int v = tid; 4 * (int64_t)v < T; v += nt) {   // the padding is left out
    const key4 a = s4[phys(v)];
    const f32x4 b = *reinterpret_cast<const f32x4*>(rrow + 4 * v);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * (int64_t)v + i < T) sum += fabsf(value_of(a[i]) - b[i]);
  }
  sum = wave_sum(sum);
  __syncthreads();                                  // the row is no longer needed: reuse its first words
  if ((tid & 63) == 0) s[tid >> 6] = sum;
  __syncthreads();
  if (tid == 0) {
    float tot = 0.0f;
    for (int w = 0; w < nt / 64; ++w) tot += s[w];
    w1[first_seg + seg] = tot;
  }
}

// One stage (k, j) with j >= chunk size, straight on global memory (mirrored if it is the level's first).
__global__ __launch_bounds__(256) void sw_sort_global_kernel(float* __restrict__ P, int64_t Tpad, int64_t k, int64_t j) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= (Tpad >> 1)) return;
  float* row = P + (int64_t)blockIdx.y * Tpad;
  const int64_t i = 2 * p - (p & (j - 1)), o = 2 * j == k ? i ^ (k - 1) : i + j;
  const float a = row[i], b = row[o];
  if (key_of(a) > key_of(b)) { row[i] = b; row[o] = a; }
}

// Unfused W1 for rows longer than one chunk: one workgroup per segment, fixed order.
__global__ __launch_bounds__(256) void sw_w1_kernel(const float* __restrict__ P, const float* __restrict__ ref, int ref_shared, int L,
                                                    int64_t T, int64_t Tpad, float* __restrict__ w1, int first_seg) {
  __shared__ float red[4];
  const int seg = blockIdx.x;
  const float* a = P + (int64_t)seg * Tpad;
  const float* b = ref + (int64_t)(ref_shared ? seg % L : seg) * Tpad;
  float sum = 0.0f;
  for (int64_t i = threadIdx.x; i < T; i += 256) sum += fabsf(a[i] - b[i]);
  sum = block_sum_256(sum, red);
  if (threadIdx.x == 0) w1[first_seg + seg] = sum;
}

// Omega_SW = (1 / L) sum_l (1 / T) sum_t |...|; flagged iff not (Omega_SW <= tau).
__global__ void sw_finalize_kernel(const float* __restrict__ w1, int n_claims, int L, int64_t T, float tau, float* __restrict__ sw_out,
                                   sv_result* __restrict__ results) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_claims) return;
  double tot = 0.0;
  for (int l = 0; l < L; ++l) tot += (double)w1[(int64_t)c * L + l];
  const float v = T > 0 ? (float)(tot / ((double)L * (double)T)) : 0.0f;
  if (sw_out) sw_out[c] = v;
  if (results) {
    results[c].metric_mask |= SV_M_SW;
    if (!(v <= tau)) results[c].flag = 1u;
  }
}

// The projection is linear, so the projections of m <- beta m + (1 - beta) mean_clean(x) are the same combination of
// the projections: out = beta pm + w sum_{c not skipped} P_c (index order, fp32), per direction and token; out may be pm.
__global__ __launch_bounds__(256) void sw_proj_ema_kernel(float* out, const float* pm, const float* __restrict__ P, int n, uint32_t skip,
                                                          int64_t slot, int64_t T, int64_t Tpad, float beta, float w) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= T) return;
  const int64_t i = (int64_t)blockIdx.y * Tpad + t;
  float acc = 0.0f;
  for (int c = 0; c < n; ++c)
    if (((skip >> c) & 1u) == 0) acc += P[(int64_t)c * slot + i];
  out[i] = beta * pm[i] + w * acc;
}

template <typename E, typename E2, int LB>
hipError_t project_launch(const void* X, int64_t stride, int count, const void* X2, int n2, const void* U, int D, int64_t T, int64_t Tpad,
                          float* P, float* P2, bool pad, hipStream_t st) {
  auto kern = sw_project_kernel<E, E2, LB>;
  constexpr int lds = kSwDepth * (kSwTile<LB> + LB * 32 * 128);   // direction chunks of 128 (bf16 signal) or 64 bytes per row
  static bool configured = false;   // per process; the attribute is per function
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  constexpr int rows = 128 * kSwTB<LB>;
  dim3 grid((unsigned)((T + rows - 1) / rows), (unsigned)(count + n2));
  hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, (const E*)X, stride, (const E2*)X2, n2, (const bf16*)U, D, T, Tpad, P, P2, pad);
  return hipGetLastError();
}

template <typename E, typename E2>
hipError_t project_dispatch(const void* X, int64_t stride, int count, const void* X2, int n2, const void* U, int L, int D, int64_t T,
                            int64_t Tpad, float* P, float* P2, bool pad, hipStream_t st) {
  switch (L / 32) {
    case 1: return project_launch<E, E2, 1>(X, stride, count, X2, n2, U, D, T, Tpad, P, P2, pad, st);
    case 2: return project_launch<E, E2, 2>(X, stride, count, X2, n2, U, D, T, Tpad, P, P2, pad, st);
    case 3: return project_launch<E, E2, 3>(X, stride, count, X2, n2, U, D, T, Tpad, P, P2, pad, st);
    default: return project_launch<E, E2, 4>(X, stride, count, X2, n2, U, D, T, Tpad, P, P2, pad, st);
  }
}

}  // namespace

int64_t sw_padded_len(int64_t T) {
  int64_t p = 128;
  while (p < T) p <<= 1;
  return p;
}

hipError_t launch_sw_project(const void* X, int64_t stride, int count, int dtype, const void* U, int L, int D, int64_t T, int64_t Tpad,
                             float* P, hipStream_t st, bool pad) {
  if (count <= 0) return hipSuccess;
  return dtype == SV_BF16 ? project_dispatch<bf16, bf16>(X, stride, count, nullptr, 0, U, L, D, T, Tpad, P, nullptr, pad, st)
                          : project_dispatch<float, float>(X, stride, count, nullptr, 0, U, L, D, T, Tpad, P, nullptr, pad, st);
}

bool sw_project_with_ref_supported(int dtype, int ref_dtype) { return dtype == ref_dtype || (dtype == SV_BF16 && ref_dtype == SV_F32); }

hipError_t launch_sw_project_with_ref(const void* X, int64_t stride, int count, int dtype, const void* ref, int ref_dtype, const void* U,
                                      int L, int D, int64_t T, int64_t Tpad, float* P, float* Pref, hipStream_t st) {
  if (count <= 0 || !sw_project_with_ref_supported(dtype, ref_dtype)) return hipErrorInvalidValue;
  if (dtype == SV_BF16 && ref_dtype == SV_F32) return project_dispatch<bf16, float>(X, stride, count, ref, 1, U, L, D, T, Tpad, P, Pref, false, st);
  return dtype == SV_BF16 ? project_dispatch<bf16, bf16>(X, stride, count, ref, 1, U, L, D, T, Tpad, P, Pref, false, st)
                          : project_dispatch<float, float>(X, stride, count, ref, 1, U, L, D, T, Tpad, P, Pref, false, st);
}

hipError_t launch_sw_sort(float* P, int n_seg, int64_t T, int64_t Tpad, const float* ref, int ref_shared, int L, float* w1,
                          int first_seg, hipStream_t st, const float* src) {
  if (n_seg <= 0) return hipSuccess;
  if (!src) src = P;
  const int ch = (int)min(Tpad, (int64_t)kSortChunkMax);
  const int nt = max(64, min(512, ch / 32));      // a thread holds 32 elements in the register passes
  const size_t lds = (size_t)ch * sizeof(float);
  const dim3 grid((unsigned)(Tpad / ch), (unsigned)n_seg);
  if (Tpad == ch) {
    sw_sort_chunk_kernel<<<grid, nt, lds, st>>>(src, P, Tpad, ch, 2, Tpad, ref, ref_shared, L, T, w1, first_seg);
    return hipGetLastError();
  }
  sw_sort_chunk_kernel<<<grid, nt, lds, st>>>(src, P, Tpad, ch, 2, ch, nullptr, 0, L, T, nullptr, 0);
  for (int64_t k = 2 * (int64_t)ch; k <= Tpad; k <<= 1) {
    for (int64_t j = k >> 1; j >= ch; j >>= 1)
      sw_sort_global_kernel<<<dim3((unsigned)((Tpad / 2 + 255) / 256), (unsigned)n_seg), 256, 0, st>>>(P, Tpad, k, j);
    sw_sort_chunk_kernel<<<grid, nt, lds, st>>>(P, P, Tpad, ch, k, k, nullptr, 0, L, T, nullptr, 0);
  }
  if (ref) sw_w1_kernel<<<n_seg, 256, 0, st>>>(P, ref, ref_shared, L, T, Tpad, w1, first_seg);
  return hipGetLastError();
}

hipError_t launch_sw_proj_ema(float* out, const float* pm, const float* P, int n, uint32_t skip, int L, int64_t T, int64_t Tpad, float beta, float w,
                              hipStream_t st) {
  sw_proj_ema_kernel<<<dim3((unsigned)((T + 255) / 256), (unsigned)L), 256, 0, st>>>(out, pm, P, n, skip, (int64_t)L * Tpad, T, Tpad, beta, w);
  return hipGetLastError();
}

hipError_t launch_sw_finalize(const float* w1, int n_claims, int L, int64_t T, float tau, float* sw_out, sv_result* results,
                              hipStream_t st) {
  if (n_claims <= 0) return hipSuccess;
  sw_finalize_kernel<<<(n_claims + 127) / 128, 128, 0, st>>>(w1, n_claims, L, T, tau, sw_out, results);
  return hipGetLastError();
}

}  // namespace sv
