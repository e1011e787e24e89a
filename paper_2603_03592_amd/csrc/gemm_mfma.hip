// bf16 GEMMs of the block recompute on the gfx950 matrix cores.
//
//   C[M,N] = sum_seg A_seg[M,K_seg] * op(B_seg)   fp32 accumulation, fused epilogue
//
// op(B) = B^T with B stored [N,K] (forward: activations times [out,in] weights) or B stored
// [K,N] (backward: gradients times the same [out,in] weights, contraction over "out").
//
// Three kernels.  [N,K] operands take the persistent 256x256 direct-to-LDS kernel or, where its tiles would not fill the
// chip or the columns are no multiple of 256, the direct-to-LDS kernel on smaller tiles, whole or over runs of k slices
// (plan_gemm prices them).  [K,N] operands go through registers, transposed on the way (8x8 blocks, v_perm).
//
// Common shape: a BM x BN output tile per workgroup, K walked in slices of 64.  Both operand
// slices are staged in LDS as rows of 64 bf16 (128 bytes) whose eight 16-byte chunks are
// XOR-swizzled by the row index, so that the 16-byte fragment reads (a lane reads 8 consecutive
// k of one row) and the 16-byte staging writes are bank-conflict free.
//
// The weight tile takes the MFMA "A" slot and the activation tile the "B" slot: each lane then
// owns one token row and groups of 4 consecutive output features, which makes every epilogue
// access an 8-byte vector (4 bf16) and keeps SwiGLU's gate/up pair in the same lane.
//
// Workgroup ids are remapped so that each XCD (ids congruent mod 8) works on a contiguous run
// of tiles, ordered in groups of GROUP_M row tiles, to keep operand panels hot in its L2.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace sv {

int cu_count() {
  static const int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 8) return 256;
    return v;
  }();
  return n;
}

namespace {

constexpr int BK = 64;
constexpr int kGroupM = 4;

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }
__device__ __forceinline__ int lds_off(int row, int chunk) { return row * 128 + ((chunk ^ swz(row)) << 4); }

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

template <int BM, int BN, int WAVES_M, int WAVES_N>
struct Cfg {
  static constexpr int NT = 64 * WAVES_M * WAVES_N;
  static constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  static constexpr int MI = WTM / 32, NI = WTN / 32;
  static constexpr int XCH = BM * 8 / NT;      // 16-byte chunks per thread, activation tile
  static constexpr int WCH = BN * 8 / NT;      // weight tile
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr int LDS = 2 * STAGE;
  static_assert(WCH % 8 == 0, "a [K,N] operand is staged in whole 8x8 blocks per thread");
};

// ---- The last round of the persistent kernel's tiles.  Every XCD has `slots` workgroups and walks per_xcd tiles; what its last round
// would leave idle for a whole tile's time goes to a second launch on smaller tiles: those of the last round only, if they are at most a
// quarter of the workgroups (one round of 128x128), or half of them where the k loop is long enough for two (in groups) or for one of
// 256x128.  50 176 x 1024 in groups, 784 tiles (3.06 rounds, paid as 4), K = 4096 and 8192: 643 -> 516 + 62 us on average; 8568 x 2048,
// K = 6528 in a check 2170 -> 1980 us; 8192 x 5632 gate/up, 5.5 rounds: 340 -> 291 + 36 us (a half-empty round runs at a higher
// clock, so less than the half is saved).  Returns the tiles per XCD that are left to it.
__host__ __device__ inline int tail_tiles(int per_xcd, int slots, int slices) {
  const int rem = per_xcd % slots;
  return per_xcd > slots && rem > 0 && (4 * rem <= slots || (2 * rem <= slots && slices >= 32)) ? rem : 0;
}

// x of the lane N places further on in its row of 16 lanes (cyclic)
template <int N> __device__ __forceinline__ float dpp_row_ror(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + N, 0xf, 0xf, false));
}

// Epilogue on 4 consecutive output features of one token row, in two phases so that a caller can
// issue all loads of a row block before the first store (the output and the residual / gate / up
// buffers may alias as far as the compiler knows, so loads are never hoisted over stores for us).
struct EpiIn { bf16x4 r, r2; f32x4 cs; };

template <int EPI>
__device__ __forceinline__ void epilogue_load4(const GemmArgs& a, int m, int n, EpiIn& in) {
  const int64_t ir = (int64_t)m * a.ldr + n;
  if (EPI == EPI_RESID || EPI == EPI_SWIGLU_BWD || EPI == EPI_GELU_BWD) in.r = *reinterpret_cast<const bf16x4*>((const bf16*)a.R + ir);
  if (EPI == EPI_SWIGLU_BWD) in.r2 = *reinterpret_cast<const bf16x4*>((const bf16*)a.R2 + ir);
  if (EPI == EPI_ROPE && n < a.rope_cols) {      // cos_i, sin_i, cos_i+1, sin_i+1 of the two feature pairs
    const int half = a.rope_hd >> 1, p = m % a.rope_S, i0 = (n % a.rope_hd) >> 1;
    in.cs = *reinterpret_cast<const f32x4*>(a.rope_cs + ((int64_t)p * half + i0) * 2);
  }
}

// rs multiplies the accumulators first (GemmArgs::rscale; the kinds that can follow a norm).  put(w, p) stores the four bf16
// values p into output w (0: C, 1: C2, 2: C3) at the place this call stands for; roped: the features are rotated (EPI_ROPE).
// Returns the sum of squares of the four values as stored in C.
template <int EPI, class Put>
__device__ __forceinline__ float epilogue_math4(const GemmArgs& a, bool roped, const float (&v_in)[4], const float (&u_in)[4], const EpiIn& in,
                                                float rs, Put&& put) {
  const bf16x4& r = in.r;
  const bf16x4& r2 = in.r2;
  constexpr bool kScaled = EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_SWIGLU || EPI == EPI_ROPE;
  float v[4], u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[i] = kScaled ? v_in[i] * rs : v_in[i]; u[i] = kScaled ? u_in[i] * rs : u_in[i]; }
  float o[4];
  switch (EPI) {
    case EPI_STORE:
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[i];
      break;
    case EPI_RESID:
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[i] + (float)r[i];
      break;
    case EPI_GELU: {
      if (a.C2) { bf16x4 p; for (int i = 0; i < 4; ++i) p[i] = (bf16)v[i]; put(1, p); }
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = gelu_epi_f(v[i]);
    } break;
    case EPI_SWIGLU: {
      if (a.C2) { bf16x4 p; for (int i = 0; i < 4; ++i) p[i] = (bf16)v[i]; put(1, p); }
      if (a.C3) { bf16x4 p; for (int i = 0; i < 4; ++i) p[i] = (bf16)u[i]; put(2, p); }
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = silu_f(v[i]) * u[i];
    } break;
    case EPI_SWIGLU_BWD: {
      bf16x4 p;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gf = (float)r[i];
        o[i] = v[i] * (float)r2[i] * silu_grad_f(gf);
        p[i] = (bf16)(v[i] * silu_f(gf));
      }
      put(1, p);
    } break;
    case EPI_ROPE: {
      if (roped) {
        const f32x4 cs = in.cs;
        if (a.rope_bf16) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = (float)(bf16)v[i];
        }
        o[0] = v[0] * cs[0] - v[1] * cs[1];
        o[1] = v[0] * cs[1] + v[1] * cs[0];
        o[2] = v[2] * cs[2] - v[3] * cs[3];
        o[3] = v[2] * cs[3] + v[3] * cs[2];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = v[i];
      }
    } break;
    default:  // EPI_GELU_BWD
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[i] * gelu_grad_epi_f((float)r[i]);
      break;
  }
  bf16x4 p;
  float sq = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) { p[i] = (bf16)o[i]; sq = fmaf((float)p[i], (float)p[i], sq); }
  put(0, p);
  return sq;
}

// the same on the output element (m, n), through plain pointers
template <int EPI>
__device__ __forceinline__ float epilogue_apply4(const GemmArgs& a, int m, int n, const float (&v_in)[4], const float (&u_in)[4], const EpiIn& in,
                                                 float rs = 1.0f) {
  const int64_t ic = (int64_t)m * a.ldc + n;
  return epilogue_math4<EPI>(a, EPI == EPI_ROPE && n < a.rope_cols, v_in, u_in, in, rs, [&](int w, bf16x4 p) {
    *reinterpret_cast<bf16x4*>((bf16*)(w == 0 ? a.C : w == 1 ? a.C2 : a.C3) + ic) = p;
  });
}

// How many trips ahead of its stores the direct-to-LDS kernel's epilogue reads its inputs (a trip: two rows per lane).  One trip
// of work is shorter than a memory round trip, so one trip ahead leaves the epilogue waiting once per trip.  (2, 2 and 3 measure the
// same within 1 %, 8 for the residual spills.)
template <int EPI> constexpr int kEpiAhead = EPI == EPI_ROPE ? 4 : EPI == EPI_SWIGLU_BWD ? 4 : 6;   // as far as the registers go

// does this kind of epilogue take GemmArgs::rscale?
template <int EPI> constexpr bool kEpiScaled = EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_SWIGLU || EPI == EPI_ROPE;

// The accumulators of one 32-row block of a wave tile.  Per feature block: its four loads first, then compute and store.
template <int EPI, int NI, int MI>
__device__ __forceinline__ void epilogue_rows(const GemmArgs& a, int M, const f32x16 (&acc)[NI][MI], int mi, int m, int nbase) {
  if (m >= M) return;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    EpiIn in[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) epilogue_load4<EPI>(a, m, nbase + ni * 32 + q * 8, in[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[4], u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[i] = acc[ni][mi][q * 4 + i]; u[i] = 0.0f; }
      epilogue_apply4<EPI>(a, m, nbase + ni * 32 + q * 8, v, u, in[q]);
    }
  }
}

// B stored [K,N]: both operands staged through registers, the weights transposed on the way.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_mfma_kernel(GemmArgs a, int tiles_m, int tiles_n) {
  using C = Cfg<BM, BN, WAVES_M, WAVES_N>;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int M = a.M;
  // ---- tile assignment (XCD-contiguous, grouped raster)
  const int nblk = tiles_m * tiles_n;
  const int per_xcd = (nblk + 7) >> 3;
  const int pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (pid >= nblk) return;
  const int in_group = kGroupM * tiles_n;
  const int first_m = (pid / in_group) * kGroupM;
  const int gsz = min(tiles_m - first_m, kGroupM);
  const int tile_m = first_m + (pid % in_group) % gsz;
  const int tile_n = (pid % in_group) / gsz;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  // ---- global -> register staging
  // Small tiles keep TWO slices in flight in registers (PF2): with at most two workgroups of four waves on a CU, one
  // slice of multiplies (~500 cycles) does not cover a global load's latency.  Large tiles have no registers for that.
  constexpr bool PF2 = BM * BN <= 128 * 128;
  constexpr int NSET = PF2 ? 2 : 1;
  bf16x8 xregs[NSET][C::XCH], wregs[NSET][C::WCH];
  int seg = 0, kin = 0;       // position of the slice being loaded
  auto load_slice = [&](auto set_tag) {
    bf16x8 (&xreg)[C::XCH] = xregs[decltype(set_tag)::value];
    bf16x8 (&wreg)[C::WCH] = wregs[decltype(set_tag)::value];
    const bf16* A = (const bf16*)a.seg[seg].A;
    const int64_t lda = a.seg[seg].lda, ldb = a.seg[seg].ldb;
#pragma unroll
    for (int i = 0; i < C::XCH; ++i) {
      const int e = tid + i * C::NT, r = e >> 3, c = e & 7;
      const int m = min(m0 + r, M - 1);
      xreg[i] = *reinterpret_cast<const bf16x8*>(A + (int64_t)m * lda + kin + c * 8);
    }
    {
      // thread owns 8x8 blocks: 8 consecutive k rows x 8 consecutive n columns
      const bf16* B = (const bf16*)a.seg[seg].B;
#pragma unroll
      for (int b = 0; b < C::WCH / 8; ++b) {
        const int blk = tid + b * C::NT, ng = blk % (BN / 8), kg = blk / (BN / 8);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          wreg[b * 8 + j] = *reinterpret_cast<const bf16x8*>(B + (int64_t)(kin + kg * 8 + j) * ldb + n0 + ng * 8);
      }
    }
    if (PF2) {                 // branch-free callers load past the end: stay on the last slice then
      if (kin + BK < a.seg[seg].K) kin += BK;
      else if (seg + 1 < a.nseg) { kin = 0; ++seg; }
    } else {
      kin += BK;
      if (kin >= a.seg[seg].K) { kin = 0; ++seg; }
    }
  };
  auto store_slice = [&](int stage, auto set_tag) {
    bf16x8 (&xreg)[C::XCH] = xregs[decltype(set_tag)::value];
    bf16x8 (&wreg)[C::WCH] = wregs[decltype(set_tag)::value];
    char* xs = smem + stage * C::STAGE;
    char* ws = xs + BM * 128;
#pragma unroll
    for (int i = 0; i < C::XCH; ++i) {
      const int e = tid + i * C::NT, r = e >> 3, c = e & 7;
      *reinterpret_cast<bf16x8*>(xs + lds_off(r, c)) = xreg[i];
    }
    {
#pragma unroll
      for (int b = 0; b < C::WCH / 8; ++b) {
        const int blk = tid + b * C::NT, ng = blk % (BN / 8), kg = blk / (BN / 8);
        u32x4 in[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] = __builtin_bit_cast(u32x4, wreg[b * 8 + j]);
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          // column n of the block: element n of rows 0..7 -> one 16-byte chunk (8 consecutive k)
          u32x4 o;
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const uint32_t lo = in[2 * p][n >> 1], hi = in[2 * p + 1][n >> 1];
            o[p] = (n & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
          }
          *reinterpret_cast<u32x4*>(ws + lds_off(ng * 8 + n, kg)) = o;
        }
      }
    }
  };

  int nslices = 0;
  for (int s = 0; s < a.nseg; ++s) nslices += a.seg[s].K / BK;

  f32x16 acc[C::NI][C::MI];
#pragma unroll
  for (int i = 0; i < C::NI; ++i)
#pragma unroll
    for (int j = 0; j < C::MI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // per-lane fragment rows
  const int l31 = lane & 31, lhi = lane >> 5;
  int wrow[C::NI];
#pragma unroll
  for (int ni = 0; ni < C::NI; ++ni) wrow[ni] = wn * C::WTN + ni * 32 + l31;

  auto multiply = [&](int stage) {
    const char* xs = smem + stage * C::STAGE;
    const char* ws = xs + BM * 128;
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      bf16x8 xf[C::MI], wf[C::NI];
#pragma unroll
      for (int mi = 0; mi < C::MI; ++mi)
        xf[mi] = *reinterpret_cast<const bf16x8*>(xs + lds_off(wm * C::WTM + mi * 32 + l31, kk * 2 + lhi));
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni)
        wf[ni] = *reinterpret_cast<const bf16x8*>(ws + lds_off(wrow[ni], kk * 2 + lhi));
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < C::MI; ++mi)
          acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ni], xf[mi], acc[ni][mi], 0, 0, 0);
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, NSET - 1>;
  if constexpr (PF2) {
    // Slice kt is multiplied from LDS stage kt & 1 while slice kt + 1 sits in register set (kt + 1) & 1 (stored to the
    // other stage at the end of the step) and slice kt + 2 is being loaded into set kt & 1.  No branch in a step: loads
    // past the end re-read the last slice, the store after the last multiply fills a stage nobody reads -- so the
    // compiler's wait before a store counts exactly the newer loads still in flight.
    load_slice(Set0{});
    load_slice(Set1{});
    store_slice(0, Set0{});
    __syncthreads();
    int kt = 0;
    for (; kt + 1 < nslices; kt += 2) {
      load_slice(Set0{});
      __builtin_amdgcn_sched_barrier(0);     // the loads stay at the top of the step: sunk below the multiply they
      multiply(0);                           // would be issued one step late
      __builtin_amdgcn_sched_barrier(0);
      store_slice(1, Set1{});
      __syncthreads();
      load_slice(Set1{});
      __builtin_amdgcn_sched_barrier(0);
      multiply(1);
      __builtin_amdgcn_sched_barrier(0);
      store_slice(0, Set0{});
      __syncthreads();
    }
    if (kt < nslices) multiply(0);
  } else {
    load_slice(Set0{});
    store_slice(0, Set0{});
    __syncthreads();
    for (int kt = 0; kt < nslices; ++kt) {
      const bool more = kt + 1 < nslices;
      if (more) load_slice(Set0{});
      multiply(kt & 1);
      if (more) store_slice((kt + 1) & 1, Set0{});
      __syncthreads();
    }
  }

  // ---- epilogue: lane owns token row (lane & 31) of each 32-row block and, per register
  // quad q, output features 8q + 4*(lane>>5) .. +3 of each 32-feature block.
#pragma unroll
  for (int mi = 0; mi < C::MI; ++mi)
    epilogue_rows<EPI, C::NI, C::MI>(a, M, acc, mi, m0 + wm * C::WTM + mi * 32 + l31, n0 + wn * C::WTN + lhi * 4);
}

// Sum of the split-k partial products, in the order of the splits, then the epilogue: one thread per 4 consecutive
// output features of a row.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a, int nsplit) {
  const int n4 = a.N >> 2;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)a.M * n4) return;
  const int m = (int)(idx / n4), n = (int)(idx % n4) * 4;
  const float* p = a.split_ws + (int64_t)m * a.N + n;
  f32x4 sum = *reinterpret_cast<const f32x4*>(p);
  for (int s = 1; s < nsplit; ++s) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + (int64_t)s * a.M * a.N);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[i] += v[i];
  }
  float v[4], u[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = sum[i];
  EpiIn in;
  epilogue_load4<EPI>(a, m, n, in);
  epilogue_apply4<EPI>(a, m, n, v, u, in, kEpiScaled<EPI> && a.rscale ? a.rscale[m] : 1.0f);
}

// ------------------------------------------------------------------------------------------
// 256x256x64 NT kernel with direct global->LDS loads (buffer_load_dwordx4 ... lds, 16 bytes per lane), four waves of 128x128.
//
// Each wave instruction copies 64 x 16 bytes to one contiguous 1 KB block of LDS = 8 tile rows; the XOR swizzle is applied by
// choosing WHICH global chunk each lane fetches, so no VGPR staging or ds_write is needed.  The loads are buffer loads: a
// descriptor per operand panel in scalar registers, the lane's byte offset in one vector register, the slice's k offset as the
// scalar offset.
//
// v_mfma_f32_16x16x32_bf16: a product's accumulators pass the register file once per 32 k instead of once per 16, and at sizes where
// the chip's power sets the clock that shows: 8192 x 28672, K = 4096 1405 -> 1322 us, with the same bits, the same loads and as many
// LDS reads as on v_mfma_f32_32x32x16_bf16.  Its fragment reads (16 rows x 64 bytes) need a swizzle of their own (swz16): with the
// other kernels' it was slower, 1490.
//
// Where the loads go: slice k + 1 of the weights and slice k + 2 of the activations are on their way while slice k is multiplied,
// into two and three buffers of 32 KB, all of the CU's 160 KB.  A slice is two steps of 32 k; a step is 64 MFMAs, and behind
// every second one stands one of the 16 fragment reads of the next step or of 8 loads, activations in the one step and weights in
// the other: loads in one step only left them too little time (K = 14336: 693 against 645 us).  One wait and barrier per slice,
// which leaves the youngest eight loads in flight.
//
// The stream of slices runs on across tiles: behind a tile's last MFMAs the next tile's first slice has landed, its first fragments
// are in registers and the loads of the slices behind it are on their way, so a tile begins without a wait.  A tile's first MFMAs
// take zero for their accumulators, no instruction clears them.
//
// A wave has its SIMD to itself and issues an instruction in about 4 cycles, so three fit behind two 16-cycle MFMAs and every further one
// delays the next.  Most slices are therefore run by a loop that only counts and adds to offsets; what a stream has to do at a segment's
// or a tile's end stands in the slices at which that happens.  With the walk through those conditions in every step a slice took 2456
// cycles, so 2282, of which 2048 are MFMAs.  Where every CU has a tile the clock follows the power and gives a part of that back: 8192 x 4096,
// K = 14336 659 -> 618 us, 8192 x 2048, K = 2048 51.4 -> 50.3; with fewer tiles 6144 x 1536, K = 2048 44.2 -> 41.4 (42.5 on
// v_mfma_f32_32x32x16_bf16), 6144 x 1024, K = 4096 80.5 -> 75.0 (74.6).

// the stores a full tile's epilogue makes last of all (at least: 6 bits of a wait count hold no more than 63 with the eight loads)
template <int EPI> constexpr int kEpiStores = EPI == EPI_SWIGLU ? 16 : EPI == EPI_SWIGLU_BWD ? 55 : 32;
constexpr int meet_wait(int vm) { return 0x0070 | (vm & 15) | ((vm >> 4) << 14); }       // vmcnt(vm) lgkmcnt(0)

// A buffer descriptor, without a bound or of no bytes, from a base that is the same in every lane, said explicitly: kept across the loops, the
// compiler moves one to vector registers otherwise and walks over the lanes at every load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t open_rsrc(const void* base, int bytes = -1) {
  const uint64_t v = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// called where a branch is not expected, lambdas stay calls, and the registers they set go to memory
#define SV_INLINE __attribute__((always_inline))

struct Stream { int vb, m0, n0, seg, k, left; };
__device__ __forceinline__ int swz16(int row) { return (row >> 1) & 7; }

// GROUPED: the grouped form (per-row-block weight group, row count from device memory) as its own instantiation, so
// that the dense form's code -- in particular its waits, which scalar loads in the tile-change path would disturb
// (they share a counter with the LDS reads) -- is unaffected by it.
//
// NF: the forms that stand at the two ends of an RMSNorm run inside the products (their own instantiations, for the same
// reason): the kinds that can follow a norm multiply every row by GemmArgs::rscale, EPI_RESID also writes GemmArgs::rowsq.
template <int EPI, bool GROUPED, bool NF = false>
__global__ __launch_bounds__(256) void gemm_mfma_dma_kernel(GemmArgs a, int tiles_m, int tiles_n) {
  constexpr bool DUAL = EPI == EPI_SWIGLU;
  constexpr bool RS = NF && kEpiScaled<EPI>, SQ = NF && EPI == EPI_RESID;
  constexpr bool kHasInputs = EPI == EPI_RESID || EPI == EPI_SWIGLU_BWD || EPI == EPI_GELU_BWD || EPI == EPI_ROPE;
  constexpr int BM = 256, MI = 8, NI = 8;
  constexpr int NOUT = DUAL ? 128 : 256;
  constexpr int BUF = 256 * 128, WBUF = 3 * BUF;          // activations: three buffers from 0; weights: two from WBUF
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // grouped form: the row count lives in device memory and the launch covers its bound
  const int M = GROUPED ? *a.m_dev : a.M;
  if (GROUPED) tiles_m = (M + BM - 1) / BM;
  // Persistent workgroups: workgroup b works on the virtual block ids b, b + gridDim.x, ...; a virtual id
  // maps to a tile so that ids congruent mod 8 (one XCD) walk a contiguous run of tiles in groups of
  // kGroupM row tiles.  gridDim.x is a multiple of 8, so a workgroup stays on its XCD's run.
  const int nblk = tiles_m * tiles_n;
  const int per_xcd = (nblk + 7) >> 3;
  const int nslices = a.slices;
  const int own = a.tail ? per_xcd - tail_tiles(per_xcd, a.tail, nslices) : per_xcd;     // tiles per XCD of this launch
  auto tile_of = [&](int vb, int& m0, int& n0) SV_INLINE -> bool {
    if (vb >= own * 8) return false;
    const int pid = (vb & 7) * per_xcd + (vb >> 3);
    if (pid >= nblk) return false;
    const int in_group = kGroupM * tiles_n;
    const int first_m = (pid / in_group) * kGroupM;
    const int gsz = min(tiles_m - first_m, kGroupM);
    m0 = (first_m + (pid % in_group) % gsz) * BM;
    n0 = ((pid % in_group) / gsz) * NOUT;
    return true;
  };

  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lhi = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;

  // ---- the two streams of slices across this workgroup's tiles.  State: virtual block vb (tile m0, n0), segment seg, offset k in
  // it, `left` slices to its end, in registers (a per-slice kernel-argument load would share its wait counter with the
  // LDS reads).  A finished stream's loads go on (the loop has no branch for it) through a descriptor of no bytes, which costs no memory.
  Stream sa{(int)blockIdx.x, 0, 0, 0, 0, 0};
  if (!tile_of(sa.vb, sa.m0, sa.n0)) return;
  Stream sb = sa;
  const bf16 *pA, *pB, *pB2;              // first rows of the panels the streams read; their descriptors, without a bound, are made at each step
  int a_bytes = -1, b_bytes = -1;
  unsigned voffA[8], voffB[8];
  // (the lane's number is opaque here: the offsets of a product of one segment would otherwise be kept twice)
  auto set_a = [&](const GemmSeg& sg) SV_INLINE {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    sa.left = __builtin_amdgcn_readfirstlane(sg.K) / BK;
    const unsigned lda2 = (unsigned)sg.lda * 2u;             // panels_fit: a panel's offsets have 32 bits
    pA = (const bf16*)sg.A + (int64_t)sa.m0 * sg.lda;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (wave + 4 * i) * 8 + (ln >> 3), c = (ln & 7) ^ swz16(r);
      voffA[i] = (unsigned)min(r, M - 1 - sa.m0) * lda2 + c * 16u;      // ragged row tail: re-read the last row
    }
  };
  auto set_b = [&](const GemmSeg& sg) SV_INLINE {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    sb.left = __builtin_amdgcn_readfirstlane(sg.K) / BK;
    const unsigned ldb2 = (unsigned)sg.ldb * 2u, ldu2 = DUAL ? (unsigned)a.ldb2 * 2u : 0u;
    const int64_t goff = GROUPED ? (int64_t)a.tile_group[sb.m0 >> 8] * a.group_stride : 0;
    const bf16* B;
    if (!DUAL && a.nbcol > 0) {
      int start = 0, j = 0;
      while (j + 1 < a.nbcol && sb.n0 >= start + a.ncol[j]) { start += a.ncol[j]; ++j; }
      B = (const bf16*)a.Bcol[j] + (int64_t)(sb.n0 - start) * sg.ldb;
    } else {
      B = (const bf16*)sg.B + goff + (int64_t)sb.n0 * sg.ldb;
    }
    pB = B;
    pB2 = DUAL ? (const bf16*)a.B2 + goff + (int64_t)sb.n0 * a.ldb2 : B;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (wave + 4 * i) * 8 + (ln >> 3), c = (ln & 7) ^ swz16(r);
      voffB[i] = (unsigned)(DUAL ? r & 127 : r) * (DUAL && i >= 4 ? ldu2 : ldb2) + c * 16u;
    }
  };
  // to the next slice, at a segment's or a tile's end with all that brings; a finished stream ends at every slice
  auto advance = [&](Stream& s, auto&& set, auto&& close) SV_INLINE {
    s.k += BK;
    s.left = __builtin_amdgcn_readfirstlane(s.left - 1);
    if (__builtin_expect(s.left == 0, 0)) {
      s.k = 0;
      if (s.seg + 1 < a.nseg) { ++s.seg; set(a.seg[s.seg]); return; }
      s.seg = 0;
      s.vb += gridDim.x;
      if (tile_of(s.vb, s.m0, s.n0)) { set(a.seg[0]); return; }
      s.seg = a.nseg - 1; s.vb = own * 8; s.left = 1;
      close();
    }
  };
  auto close_a = [&]() SV_INLINE { a_bytes = 0; };
  auto close_b = [&]() SV_INLINE { b_bytes = 0; };
  // 1 KB: the wave's i-th group of 8 rows
  auto dma_a = [&](__amdgpu_buffer_rsrc_t r, int k, int buf, int i) SV_INLINE {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(smem + buf + (wave + 4 * i) * 1024), 16, (int)voffA[i], k, 0, 0);
  };
  auto dma_b = [&](__amdgpu_buffer_rsrc_t r, __amdgpu_buffer_rsrc_t r2, int k, int buf, int i) SV_INLINE {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(DUAL && i >= 4 ? r2 : r, (__attribute__((address_space(3))) void*)(smem + buf + (wave + 4 * i) * 1024), 16,
                                             (int)voffB[i], k, 0, 0);
  };
  // what the steps' loads go through: the streams' panels (SwiGLU's weights lie in two) and their slices' byte offsets
#define SV_PANELS                                                                                                  \
  const __amdgpu_buffer_rsrc_t rA = open_rsrc(pA, a_bytes), rB = open_rsrc(pB, b_bytes), rB2 = open_rsrc(pB2, b_bytes); \
  int ka = __builtin_amdgcn_readfirstlane(sa.k * 2), kb = __builtin_amdgcn_readfirstlane(sb.k * 2)
  auto behind = [](int buf) { return buf == 2 * BUF ? 0 : buf + BUF; };      // the next of the activations' buffers

  // ---- fragment addresses: rows 16 b + (lane & 15) of an operand, chunk 4 s + (lane >> 4); swz16 does not see b
  unsigned offX[2], offW[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int chunk = ((s * 4 + lhi) ^ swz16(l15)) << 4;
    offX[s] = (unsigned)((wm * 128 + l15) * 128 + chunk);
    offW[s] = (unsigned)((wn * (DUAL ? 64 : 128) + l15) * 128 + chunk);
  }
  auto read_x = [&](int buf, int s, int b) { return *reinterpret_cast<const bf16x8*>(smem + buf + offX[s] + b * 2048); };
  auto read_w = [&](int buf, int s, int b) {                  // SwiGLU: blocks 0..3 gate, 4..7 up, which begin at row 128
    return *reinterpret_cast<const bf16x8*>(smem + buf + offW[s] + (DUAL && b >= 4 ? b + 4 : b) * 2048);
  };

  f32x4 acc[NI][MI];
#define SV_SB __builtin_amdgcn_sched_barrier(0)
  // One step of 32 k: MFMAs on (xc, wc), on zero accumulators if `first`; the fragments of step s of the slice in buffers ra, rw
  // are read into (xn, wn_), and the eight loads of a stream's next slice are issued (into_w: weights) through d and d2, at offset k, into
  // buffer db; `ends`: the stream goes on by itself (advance).
  auto step = [&](auto first, auto into_w, auto reads, auto ends, __amdgpu_buffer_rsrc_t d, __amdgpu_buffer_rsrc_t d2, int k, bf16x8 (&xc)[MI],
                  bf16x8 (&wc)[NI], bf16x8 (&xn)[MI], bf16x8 (&wn_)[NI], int ra, int rw, int s, int db) {
    const f32x4 zero{0.0f, 0.0f, 0.0f, 0.0f};
    auto two = [&](int q) {
      const int g = q >> 2;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = (q & 3) * 2 + h, m = g & 1 ? 7 - j : j; // back and forth, so that neighbours share an operand
        acc[g][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wc[g], xc[m], decltype(first)::value ? zero : acc[g][m], 0, 0, 0);
      }
      SV_SB;
    };
#pragma unroll
    for (int q = 0; q < 24; ++q) {                            // two MFMAs, then one memory instruction
      two(q);
      const int r = q - q / 3;
      if (q % 3 == 2) { if (decltype(into_w)::value) dma_b(d, d2, k, db, q / 3); else dma_a(d, k, db, q / 3); }
      else if (decltype(reads)::value) { if (r < 8) xn[r] = read_x(ra, s, r); else wn_[r - 8] = read_w(rw, s, r - 8); }
      SV_SB;
    }
    // between MFMAs: behind the last of them its scalar chain would idle the matrix pipe
    if (decltype(ends)::value) { if (decltype(into_w)::value) advance(sb, set_b, close_b); else advance(sa, set_a, close_a); }
    SV_SB;
#pragma unroll
    for (int q = 24; q < 32; ++q) two(q);
  };
  // this wave's wait, then the workgroup's barrier: slice k + 1 is complete (its youngest load is older than the last eight), and
  // everybody has read what they need of slice k
#define SV_MEET(imm) do { SV_SB; __builtin_amdgcn_s_waitcnt(imm); asm volatile("s_barrier" ::: "memory"); SV_SB; } while (0)
  constexpr int kLgkm0 = 0xc07f;                              // lgkmcnt(0), nothing else
  using Yes = std::true_type;
  using No = std::false_type;

  bf16x8 x0[MI], w0[NI], x1[MI], w1[NI];
  int ca = 0, cw = WBUF;                                      // the buffers of the slice being multiplied
  constexpr int kOther = WBUF ^ (WBUF + BUF);
  set_a(a.seg[0]);
  set_b(a.seg[0]);
  auto load_a = [&](int buf) SV_INLINE {
    SV_PANELS;
#pragma unroll
    for (int j = 0; j < 8; ++j) dma_a(rA, ka, buf, j);
  };
  auto load_b = [&](int buf) SV_INLINE {
    SV_PANELS;
#pragma unroll
    for (int j = 0; j < 8; ++j) dma_b(rB, rB2, kb, buf, j);
  };
  load_a(0);
  load_b(WBUF);
  advance(sa, set_a, close_a);
  advance(sb, set_b, close_b);
  load_a(BUF);
  advance(sa, set_a, close_a);
  SV_MEET(meet_wait(8));
  load_b(cw ^ kOther);
  advance(sb, set_b, close_b);
  if (!kHasInputs) {
#pragma unroll
    for (int b = 0; b < 8; ++b) { x0[b] = read_x(ca, 0, b); w0[b] = read_w(cw, 0, b); }
  }

  int m0, n0;
  bool stored = false;                                        // this workgroup's stores may be on their way
  for (int vb = blockIdx.x; tile_of(vb, m0, n0); vb += gridDim.x) {
    // ---- what the epilogue's global accesses need, set up here because the first inputs are asked for early.
    // In the read-back of the epilogue a lane serves row er of each group of 4 rows, 8 columns from 8 ec.
    // One buffer descriptor per tensor, based at the tile's first row and the wave's first column, up to the last of the M rows: what
    // lies past them is dropped or read as zero, and a ragged tile runs the same code as a full one.  Inside it a lane's
    // byte offset is (row * ld + column) * 2: no 64-bit address arithmetic per access.  All of it is in the vector register: the
    // bounds test subtracts a scalar offset from the descriptor's size, and a ragged tile's row blocks begin past its end.
    constexpr int PD = kEpiAhead<EPI>;                   // trips the epilogue's global reads run ahead of its stores
    const int er = lhi, ec8 = l15;
    const int ncol0 = n0 + wn * (DUAL ? 64 : 128);
    const int rows = min(M - m0, BM);
    auto desc = [&](const void* base, int ld) {
      return __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16*)base + (int64_t)m0 * ld + ncol0), (short)0, (rows * ld - ncol0) * 2, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t bC = desc(a.C, a.ldc), bC2 = desc(a.C2, a.ldc), bC3 = desc(a.C3, a.ldc);
    const __amdgpu_buffer_rsrc_t bR = desc(a.R, a.ldr), bR2 = desc(a.R2, a.ldr);
    // byte offset of row `row` of the wave's 128 rows, `bytes` into it; a group's first row is added behind it
    auto place = [&](int row, int ld, int bytes) { return (wm * 128 + row) * ld * 2 + bytes; };
    int rope_p0 = 0, rope_v = 0;                         // first row's position; byte offset of the lane's feature pairs in a table row
    if (EPI == EPI_ROPE) {
      rope_p0 = (m0 + wm * 128) % a.rope_S;
      rope_v = (((ncol0 + ec8 * 8) % a.rope_hd) >> 1) * 8;
    }
    const __amdgpu_buffer_rsrc_t bT = __builtin_amdgcn_make_buffer_rsrc((void*)a.rope_cs, (short)0, -1, 0x00020000);
    auto ld16 = [&](__amdgpu_buffer_rsrc_t b, int vo, bf16x4& lo, bf16x4& hi) {
      const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b, vo, 0, 0));
      lo = __builtin_shufflevector(v, v, 0, 1, 2, 3);
      hi = __builtin_shufflevector(v, v, 4, 5, 6, 7);
    };
    // the inputs of trip `trip` (rows 8 trip .. 8 trip + 7 of the wave's 128, two per lane): residual, gate / up, RoPE table
    auto load_inputs = [&](int trip, int er, EpiIn (&lo)[2], EpiIn (&hi)[2]) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int rb = trip * 8 + k * 4;
        if (EPI == EPI_ROPE) {
          // position of the row in its sequence without a division per row: the wave's first row is reduced once
          // per tile, the rows of the tile follow it consecutively
          int p = rope_p0 + rb + er;
          if (a.rope_S >= 256) p -= p >= a.rope_S ? a.rope_S : 0; else p %= a.rope_S;
          const int vo = p * (a.rope_hd >> 1) * 8 + rope_v;         // the table entry (position p, feature pair) is 8 bytes
          lo[k].cs = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bT, vo, 0, 0));
          hi[k].cs = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bT, vo + 16, 0, 0));
        } else if (kHasInputs) {
          const int vo = place(er, a.ldr, ec8 * 16) + rb * a.ldr * 2;
          ld16(bR, vo, lo[k].r, hi[k].r);
          if (EPI == EPI_SWIGLU_BWD) ld16(bR2, vo, lo[k].r2, hi[k].r2);
        }
      }
    };
    EpiIn in_lo[PD][2], in_hi[PD][2];                    // [trip mod PD][row of the pair]
    // the row factors of the wave's 128 rows, lane l those of rows l and 64 + l, are asked for here, a k loop before the epilogue wants them
    float rs_pre0 = 1.0f, rs_pre1 = 1.0f;
    if (RS) {
      rs_pre0 = a.rscale[min(m0 + wm * 128 + lane, M - 1)];
      rs_pre1 = a.rscale[min(m0 + wm * 128 + 64 + lane, M - 1)];
    }
    // ---- the k loop.  The tile's first slice has landed; its first fragments have been asked for, unless the epilogue has inputs,
    // which need the registers.
    if (kHasInputs) {
#pragma unroll
      for (int b = 0; b < 8; ++b) { x0[b] = read_x(ca, 0, b); w0[b] = read_w(cw, 0, b); }
    }
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    SV_SB;
    {
      SV_PANELS;
      step(Yes{}, No{}, Yes{}, Yes{}, rA, rA, ka, x0, w0, x1, w1, ca, cw, 1, behind(behind(ca)));
    }
    ca = behind(ca); cw ^= kOther;
    if (nslices > 1) {
      // the tile's second slice was asked for before the last tile's results were stored: those may still be on their way
      SV_SB;
      __builtin_amdgcn_s_waitcnt(meet_wait(8 + kEpiStores<EPI>));
      if (!stored) __builtin_amdgcn_s_waitcnt(meet_wait(8));
      SV_MEET(meet_wait(63));
      for (int kt = 1;;) {
        // the slices before one at which a stream's segment or the tile ends
        SV_PANELS;
        const int n = __builtin_amdgcn_readfirstlane(min(min(sa.left, sb.left), nslices - kt) - 1);
        for (int i = 0; i < n; ++i) {
          step(No{}, Yes{}, Yes{}, No{}, rB, rB2, kb, x1, w1, x0, w0, ca, cw, 0, cw ^ kOther);
          __builtin_amdgcn_s_waitcnt(kLgkm0);
          SV_SB;
          step(No{}, No{}, Yes{}, No{}, rA, rA, ka, x0, w0, x1, w1, ca, cw, 1, behind(behind(ca)));
          ca = behind(ca); cw ^= kOther;
          ka += BK * 2; kb += BK * 2;
          SV_MEET(meet_wait(8));
        }
        kt += n;
        sa.left -= n; sb.left -= n; sa.k += n * BK; sb.k += n * BK;
        step(No{}, Yes{}, Yes{}, Yes{}, rB, rB2, kb, x1, w1, x0, w0, ca, cw, 0, cw ^ kOther);
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        SV_SB;
        step(No{}, No{}, Yes{}, Yes{}, rA, rA, ka, x0, w0, x1, w1, ca, cw, 1, behind(behind(ca)));
        ca = behind(ca); cw ^= kOther;
        if (++kt == nslices) break;
        SV_MEET(meet_wait(8));
      }
    }
    SV_SB;
    if (kHasInputs) {                                    // the epilogue's first inputs: their round trip hides behind the last step's products
#pragma unroll
      for (int t = 0; t < PD; ++t) load_inputs(t, er, in_lo[t], in_hi[t]);
    }
    SV_MEET(meet_wait(8 + (kHasInputs ? PD * (EPI == EPI_SWIGLU_BWD || EPI == EPI_ROPE ? 4 : 2) : 0)));
    {
      SV_PANELS;
      step(No{}, Yes{}, std::integral_constant<bool, !kHasInputs>{}, Yes{}, rB, rB2, kb, x1, w1, x0, w0, ca, cw, 0, cw ^ kOther);
    }
    SV_SB;
    stored = true;

    // ---- epilogue through LDS (the next tile's first slices are landing meanwhile).
    // In the accumulator layout a lane owns one token row and groups of 4 features, so a store instruction would touch 16 rows
    // with 32 bytes each (with the weights' rows dealt so that a lane holds 8 neighbouring features, 64 or, after an exchange
    // between lanes, 128 bytes, the stores were still 2 - 4 % of a K = 2048 product slower than this way).  Each wave instead turns
    // 16 rows at a time over in a patch of its own of the activations' free buffer and reads them back so that consecutive lanes
    // hold 16 bytes each of an output row: every global access of the epilogue (result, residual, gate / up) is a run of full lines.
    // The patch is what this wave's own loads will fill next, 1 KB pieces 4 KB apart, so that no barrier
    // stands between the waves' epilogues and the loads behind them.
    char* patch = smem + behind(behind(ca)) + wave * 1024;
    {
      // The lane's row and chunk numbers are made opaque once per tile: otherwise every address below is loop invariant, gets
      // hoisted out of the tile loop and crowds the fragments and the epilogue's inputs out of the registers.
      int e15 = l15, eer = er;
      asm volatile("" : "+v"(e15), "+v"(eer));
      // The accumulators stay in the accumulation registers until their row block's turn: seen through, the compiler copies whole
      // blocks of them ahead and spills.
      auto take = [&](int ni, int mi) {
        f32x4 v = acc[ni][mi];
        asm volatile("" : "+a"(v));
        return v;
      };
      auto put16 = [&](__amdgpu_buffer_rsrc_t b, bf16x8 v, int rb, int row, int bytes) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, place(row, a.ldc, bytes) + rb * a.ldc * 2, 0, 0);
      };
      if constexpr (DUAL) {
        // Gate and up of one feature sit in the same lane and register index, so SiLU(g) * u is taken in the accumulator layout
        // and the patch holds bf16 results: 16 rows x 64 features x 2 bytes each of the result and, where backward wants them, gate
        // and up (16-byte chunks XOR-swizzled by bits 1..3 of the row), three quarters of the fp32 way's LDS traffic and half
        // its stores.  A row block's arithmetic stands behind the read-back of the one before.
        const bool stash = a.C2 || a.C3;
        const int lr = eer * 2 + (e15 >> 3), cc = e15 & 7;       // read-back: rows lr and 8 + lr, chunk cc
        char* const wr = patch + (e15 >> 3) * 4096 + (e15 & 7) * 128 + (eer & 1) * 8;
        const int wx = (e15 >> 1) & 7, wc = eer >> 1;
        bf16x4 act[4], gt[4], ut[4];
        auto math = [&](int mi) {
          const float rs = RS ? __shfl(mi < 4 ? rs_pre0 : rs_pre1, (mi & 3) * 16 + e15) : 1.0f;
#pragma unroll
          for (int ni = 0; ni < 4; ++ni) {
            const f32x4 gate = take(ni, mi), up = take(ni + 4, mi);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float g = RS ? gate[i] * rs : gate[i], u = RS ? up[i] * rs : up[i];
              act[ni][i] = (bf16)(silu_f(g) * u); gt[ni][i] = (bf16)g; ut[ni][i] = (bf16)u;
            }
          }
        };
        math(0);
        SV_SB;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
          for (int ni = 0; ni < 4; ++ni) *reinterpret_cast<bf16x4*>(wr + (((ni * 2 + wc) ^ wx) << 4)) = act[ni];
          if (stash) {
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) {
              *reinterpret_cast<bf16x4*>(wr + 8192 + (((ni * 2 + wc) ^ wx) << 4)) = gt[ni];
              *reinterpret_cast<bf16x4*>(wr + 16384 + (((ni * 2 + wc) ^ wx) << 4)) = ut[ni];
            }
          }
          __builtin_amdgcn_s_waitcnt(kLgkm0);            // the patch is complete before it is read back
          __builtin_amdgcn_wave_barrier();
          bf16x8 oc[2], og[2], ou[2];
#pragma unroll
          for (int it = 0; it < 2; ++it) {
            const char* rd = patch + it * 4096 + lr * 128 + ((cc ^ ((it * 4 + (lr >> 1)) & 7)) << 4);
            oc[it] = *reinterpret_cast<const bf16x8*>(rd);
            if (stash) { og[it] = *reinterpret_cast<const bf16x8*>(rd + 8192); ou[it] = *reinterpret_cast<const bf16x8*>(rd + 16384); }
          }
          SV_SB;
          if (mi + 1 < MI) math(mi + 1);
          SV_SB;
#pragma unroll
          for (int it = 0; it < 2; ++it) put16(bC, oc[it], mi * 16 + it * 8, lr, cc * 16);
          if (stash) {
#pragma unroll
            for (int it = 0; it < 2; ++it) {
              if (a.C2) put16(bC2, og[it], mi * 16 + it * 8, lr, cc * 16);
              if (a.C3) put16(bC3, ou[it], mi * 16 + it * 8, lr, cc * 16);
            }
          }
          __builtin_amdgcn_wave_barrier();
        }
      } else {
        // 16 rows of 128 fp32 accumulators in the patch; a lane's 8 columns lie in chunks c and 16 + c of 16 bytes, XOR-swizzled by
        // the row: conflict-free both ways.  Sixteen trips per tile, two rows per lane and trip.  The epilogue's global
        // reads (residual, gate / up, RoPE table) run kEpiAhead trips ahead of its stores; the first of them were asked for before
        // the last step.  (The memory counter retires in order: a read is waited for together with every store issued
        // before it, so the reads of a trip are issued before the stores they must not wait for have piled up.)
        auto prow = [](int row) { return (row >> 1) * 4096 + (row & 1) * 512; };
        float sq0 = 0.0f, sq1 = 0.0f;                    // SQ: the sums of rows 4 l15 + lhi and 64 + 4 l15 + lhi
#pragma unroll
        for (int trip = 0; trip < 16; ++trip) {
          const int mi = trip >> 1, it = (trip & 1) * 2;
          if ((trip & 1) == 0) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
              *reinterpret_cast<f32x4*>(patch + prow(e15) + (((ni * 2 + (eer >> 1) + (eer & 1) * 16) ^ e15) << 4)) = take(ni, mi);
            __builtin_amdgcn_s_waitcnt(kLgkm0);          // the patch is complete before it is read back
            __builtin_amdgcn_wave_barrier();
          }
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int row = (it + k) * 4 + eer, rb = trip * 8 + k * 4;
            const f32x4 a_lo = *reinterpret_cast<const f32x4*>(patch + prow(row) + ((e15 ^ row) << 4));
            const f32x4 a_hi = *reinterpret_cast<const f32x4*>(patch + prow(row) + (((16 + e15) ^ row) << 4));
            float lo[4], hi[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { lo[i] = a_lo[i]; hi[i] = a_hi[i]; }
            bf16x4 olo[2], ohi[2];
            auto put_lo = [&](int w, bf16x4 pk) { olo[w] = pk; };
            auto put_hi = [&](int w, bf16x4 pk) { ohi[w] = pk; };
            const float rs = RS ? __shfl(trip < 8 ? rs_pre0 : rs_pre1, (rb & 63) + eer) : 1.0f;
            const bool roped = EPI == EPI_ROPE && ncol0 + ec8 * 8 < a.rope_cols;
            float sq = epilogue_math4<EPI>(a, roped, lo, hi, in_lo[trip % PD][k], rs, put_lo);
            float sq_hi = epilogue_math4<EPI>(a, roped, hi, lo, in_hi[trip % PD][k], rs, put_hi);
            put16(bC, __builtin_shufflevector(olo[0], ohi[0], 0, 1, 2, 3, 4, 5, 6, 7), rb, eer, e15 * 16);
            if (EPI == EPI_SWIGLU_BWD || (EPI == EPI_GELU && a.C2))
              put16(bC2, __builtin_shufflevector(olo[1], ohi[1], 0, 1, 2, 3, 4, 5, 6, 7), rb, eer, e15 * 16);
            if (SQ) {
              // the 16 lanes of a row hold its 128 stored values, two chunks of 4 each: rotate-and-add within the row of 16 lanes leaves
              // the sum in all of them, and the one whose turn it is keeps it.  Chunk c's sum meets that of chunk c ^ 16 first, then c ^ 8,
              // 4, 2 and, in the lane, 1: a verifier's row factors, and all that follows them, stay the same bits whatever
              // columns a lane holds.
              sq += dpp_row_ror<8>(sq); sq += dpp_row_ror<4>(sq); sq += dpp_row_ror<2>(sq); sq += dpp_row_ror<1>(sq);
              sq_hi += dpp_row_ror<8>(sq_hi); sq_hi += dpp_row_ror<4>(sq_hi); sq_hi += dpp_row_ror<2>(sq_hi); sq_hi += dpp_row_ror<1>(sq_hi);
              sq += sq_hi;
              if (trip < 8) sq0 = e15 == trip * 2 + k ? sq : sq0;
              else sq1 = e15 == trip * 2 + k - 16 ? sq : sq1;
            }
          }
          if (kHasInputs && trip + PD < 16) load_inputs(trip + PD, eer, in_lo[trip % PD], in_hi[trip % PD]);
          SV_SB;                                         // one trip at a time
          if (trip & 1) __builtin_amdgcn_wave_barrier(); // the reads of this block are issued before the next block's writes
        }
        if (SQ) {                                        // 128 consecutive floats of plane (n0 / 128 + wn): two full-line stores
          const int r = wm * 128 + e15 * 4 + eer;
          const __amdgpu_buffer_rsrc_t bQ = __builtin_amdgcn_make_buffer_rsrc((void*)(a.rowsq + (int64_t)((n0 >> 7) + wn) * a.rowsq_ld + m0), (short)0, rows * 4, 0x00020000);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sq0), bQ, r * 4, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sq1), bQ, (r + 64) * 4, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(kLgkm0);                  // the patch has been read: this wave's loads may fill it
    SV_SB;
  }
  // The finished streams' loads write zeros into the free buffers: every one must have done so before the workgroup gives its LDS back.
  __builtin_amdgcn_s_waitcnt(0);
#undef SV_MEET
#undef SV_SB
#undef SV_PANELS
}

// ------------------------------------------------------------------------------------------
// Direct-to-LDS kernel on smaller tiles: (32 MI) x (32 NI) outputs per workgroup of 2 x 2 waves.  It serves what the 256x256 kernel
// cannot fill the chip with (fewer than about one tile per CU) and widths that are no multiple of 256: any multiple of 8
// columns -- weight rows past the end re-read the last group of 8, outputs past the end (rows and columns) are dropped by the bounds
// check of the buffer stores.
//
// What bounds it: on 128x128 and 256x128 tiles the operands' way into LDS, about 40 bytes a clock and CU where all CUs load (750 and 1290
// cycles a slice of 512 and 1024 matrix cycles; the 256x256 tile, with half the loads of the one per multiply-add, stays better wherever it fills
// the chip); on smaller ones instructions: a wave has a SIMD to itself, or half of one, and behind each of its few MFMAs stand a load with
// its LDS address or a fragment read.  RA and RB: buffers of activations and of weights, within one workgroup's 160 KB or two
// workgroups' 80 KB.  The k loop is the 256x256 kernel's: two steps of 32 k a slice on 16x16x32 MFMAs, the fragment reads of the
// next step and the loads of a later slice spread over the first three quarters of a step's MFMAs, activations in the one step and
// weights in the other, one wait and barrier a slice that leaves the youngest loads in flight; the slices at which a segment ends
// stand apart from the others, and so do the last RA - 1, which load nothing.  Before they did, us (and on eight waves with loads and reads
// in groups around the MFMAs of a 16-wide step): 1024^3 on 64x64 6.7 -> 6.3 (7.0); 512 x 4096, K = 4096 on 64x128 24.4 -> 22.0 (26.4);
// 1536 x 1536, K = 2048 on 128x128 16.4 -> 15.7 (16.4); 2048 x 4096, K = 4096 on 256x128 58 -> 58 (62).
template <int MI, int NI, int RA, int RB, bool DUAL>
struct MidCfg {
  static constexpr int BM = 32 * MI, BN = 32 * NI, NOUT = DUAL ? BN / 2 : BN;
  static constexpr int ABUF = BM * 128, WBUF = BN * 128, LDS = RA * ABUF + RB * WBUF;
  static constexpr int OCC = 2 * LDS <= 160 * 1024 ? 2 : 1;                     // workgroups on a CU
  // The loads that may be in flight when a slice with `j` more behind it is to be complete: those of the slices behind it, of which the
  // activations are RA - 2 ahead and the weights RB - 2.  (All of them are younger than that slice's, as long as the activations'
  // ring is at most one longer.)
  static constexpr int left(int j) { return (j < RA - 2 ? j : RA - 2) * MI + (j < RB - 2 ? j : RB - 2) * NI; }
  static constexpr int LEFT = left(RA);
  static_assert(LDS <= 160 * 1024 && RA >= RB && RA <= RB + 1 && RB >= 2 && LEFT < 64 && (!DUAL || NI % 4 == 0), "tile shape");
};

//
// SPLIT: a tile's k slices are dealt to nsplit workgroups in contiguous runs, each leaves its fp32 partial product in
// a.split_ws[run][M][N] and splitk_reduce_kernel adds the runs in order.  SUMMED: the same sum of runs (GemmArgs::runs) in one
// workgroup, the running total beside the accumulators: bit for bit what the partial products and their reduction give.
// TAIL: the last round of a product on 256x256 tiles (GemmArgs::tail).
template <int MI, int NI, int RA, int RB, int EPI, bool GROUPED, bool SPLIT, bool SUMMED, bool TAIL>
__global__ __launch_bounds__(256, (MidCfg<MI, NI, RA, RB, EPI == EPI_SWIGLU>::OCC)) void gemm_mid_kernel(GemmArgs a, int tiles_m, int tiles_n, int nsplit) {
  constexpr bool DUAL = EPI == EPI_SWIGLU;
  static_assert(!SPLIT || (EPI == EPI_STORE && !GROUPED), "a split run stores bare partial products");
  static_assert(!SUMMED || (!DUAL && !GROUPED && !SPLIT), "one sum of runs per output");
  static_assert(NI <= 4 || (EPI != EPI_STORE && EPI != EPI_ROPE), "a panel for each group of weight rows");
  using C = MidCfg<MI, NI, RA, RB, DUAL>;
  constexpr int BM = C::BM, BN = C::BN, ABUF = C::ABUF, WBUF = C::WBUF, W0 = RA * ABUF;     // weights' buffers from W0
  constexpr int kGroup = BM >= 256 ? 4 : BM >= 128 ? 8 : 16;          // row tiles per raster group: about 1024 rows
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int M = GROUPED ? *a.m_dev : a.M;
  if (GROUPED) tiles_m = (M + BM - 1) / BM;
  // tile assignment as in the 256x256 kernel: ids congruent mod 8 (one XCD) walk a contiguous run of tiles.  As that kernel's last
  // round: its map and its tiles, each in SUB pieces next to each other.
  constexpr int SUBN = 256 / BN, SUB = 256 / BM * SUBN;
  static_assert(!TAIL || (!SPLIT && !SUMMED && 256 % BM == 0), "a tail's tiles are whole");
  int group = kGroup, skip = 0, sub = 0, slot = blockIdx.x >> 3;
  if (TAIL) {
    tiles_m = (M + 255) / 256; tiles_n = a.N / (DUAL ? 128 : 256);
    const int all = (tiles_m * tiles_n + 7) >> 3, rem = tail_tiles(all, a.tail, a.slices);
    sub = slot % SUB; slot /= SUB;
    if (slot >= rem) return;
    skip = all - rem;
    group = kGroupM;
  }
  const int nblk = tiles_m * tiles_n, nvb = SPLIT ? nblk * nsplit : nblk;
  const int per_xcd = (nvb + 7) >> 3;
  int pid = (blockIdx.x & 7) * per_xcd + skip + slot;
  if (skip + slot >= per_xcd || pid >= nvb) return;
  int run = 0;
  if (SPLIT) { run = pid / nblk; pid -= run * nblk; }
  const int in_group = group * tiles_n;
  const int first_m = (pid / in_group) * group;
  const int gsz = min(tiles_m - first_m, group);
  const int m0 = (first_m + (pid % in_group) % gsz) * (TAIL ? 256 : BM) + sub / SUBN * BM;
  const int n0 = ((pid % in_group) / gsz) * (TAIL ? SUBN * C::NOUT : C::NOUT) + sub % SUBN * C::NOUT;
  if (TAIL && m0 >= M) return;

  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lhi = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;

  // ---- the two streams of slices: segment seg, offset k in it, `turn` slices to its end
  int nsl = a.slices, seg0 = 0, k0 = 0;
  if (SPLIT) {                                            // run r takes the slices [r * nsl / nsplit, (r + 1) * nsl / nsplit)
    const int ks = (int)((int64_t)run * nsl / nsplit);
    nsl = (int)((int64_t)(run + 1) * nsl / nsplit) - ks;
    k0 = ks * BK;
    while (k0 >= a.seg[seg0].K) { k0 -= a.seg[seg0].K; ++seg0; }
  }
  int a_seg = seg0, a_k = k0, a_turn = 0, w_seg = seg0, w_k = k0, w_turn = 0;
  // The weights' panels: the tile's columns lie in one matrix, or in gate and up, but for products over column blocks of several matrices,
  // where every group of 8 rows has a panel of its own.
  constexpr bool OWN = EPI == EPI_STORE || EPI == EPI_ROPE;
  constexpr int NP = OWN ? NI : DUAL ? 2 : 1;
  auto panel = [](int i) SV_INLINE { return OWN ? i : DUAL ? i / (NI / 2) : 0; };
  const bf16 *pA, *pB[NP];                                // first rows of the panels
  unsigned voffA[MI], voffB[NI];
  auto set_a = [&](const GemmSeg& sg) SV_INLINE {
    a_turn = (__builtin_amdgcn_readfirstlane(sg.K) - a_k) / BK;
    pA = (const bf16*)sg.A + (int64_t)m0 * sg.lda;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int r = (wave + 4 * i) * 8 + (lane >> 3), c = (lane & 7) ^ swz16(r);
      voffA[i] = (unsigned)((int64_t)min(r, M - 1 - m0) * sg.lda + c * 8) * 2u;
    }
  };
  auto set_b = [&](const GemmSeg& sg) SV_INLINE {
    w_turn = (__builtin_amdgcn_readfirstlane(sg.K) - w_k) / BK;
    const int64_t goff = GROUPED ? (int64_t)__builtin_amdgcn_readfirstlane(a.tile_group[m0 >> 8]) * a.group_stride : 0;
    const bf16* B0 = (const bf16*)sg.B + goff;
    if (!OWN) pB[0] = B0 + (int64_t)n0 * sg.ldb;
    if (DUAL) pB[NP - 1] = (const bf16*)a.B2 + goff + (int64_t)n0 * a.ldb2;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int g = (wave + 4 * i) * 8, r = g + (lane >> 3), c = (lane & 7) ^ swz16(r);
      const int64_t ldb = DUAL && panel(i) ? a.ldb2 : sg.ldb;
      int row = min(n0 + g - (DUAL ? panel(i) * (BN / 2) : 0), a.N - 8);      // the group's first weight row
      if (OWN) {
        const bf16* B = B0;
        if (a.nbcol > 0) {
          const int o1 = a.ncol[0], o2 = o1 + a.ncol[1];
          if (a.nbcol > 2 && row >= o2) { B = (const bf16*)a.Bcol[2]; row -= o2; }
          else if (a.nbcol > 1 && row >= o1) { B = (const bf16*)a.Bcol[1]; row -= o1; }
          else B = (const bf16*)a.Bcol[0];
        }
        pB[panel(i)] = B + (int64_t)row * ldb;
        row = 0;
      } else {
        row -= n0;
      }
      voffB[i] = (unsigned)((int64_t)(row + (lane >> 3)) * ldb + c * 8) * 2u;
    }
  };
  // to the next slice, at a segment's end with all that brings (behind the last one there is none)
  auto advance_a = [&]() SV_INLINE {
    a_k += BK;
    if (__builtin_expect(--a_turn == 0 && a_seg + 1 < a.nseg, 0)) { a_k = 0; ++a_seg; set_a(a.seg[a_seg]); }
  };
  auto advance_b = [&]() SV_INLINE {
    w_k += BK;
    if (__builtin_expect(--w_turn == 0 && w_seg + 1 < a.nseg, 0)) { w_k = 0; ++w_seg; set_b(a.seg[w_seg]); }
  };
  // what the steps' loads go through: the activations' panel, the groups of 8 weight rows, the slices' byte offsets
#define SV_PANELS                                                                                                                         \
  const __amdgpu_buffer_rsrc_t rA = open_rsrc(pA), rB0 = open_rsrc(pB[0]), rB1 = open_rsrc(pB[NP > 1 ? 1 : 0]), \
                               rB2 = open_rsrc(pB[NP > 2 ? 2 : 0]), rB3 = open_rsrc(pB[NP > 2 ? 3 : 0]);                \
  int ka = __builtin_amdgcn_readfirstlane(a_k * 2), kb = __builtin_amdgcn_readfirstlane(w_k * 2)
#define SV_PANEL_ARGS rA, rB0, rB1, rB2, rB3
#define SV_PANEL_PARAMS                                                                                                                   \
  __amdgpu_buffer_rsrc_t rA, __amdgpu_buffer_rsrc_t rB0, __amdgpu_buffer_rsrc_t rB1, __amdgpu_buffer_rsrc_t rB2, __amdgpu_buffer_rsrc_t rB3
  // 1 KB: the wave's i-th group of 8 rows
  auto dma_a = [&](SV_PANEL_PARAMS, int k, int buf, int i) SV_INLINE {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (__attribute__((address_space(3))) void*)(smem + buf + (wave + 4 * i) * 1024), 16, (int)voffA[i], k, 0, 0);
  };
  auto dma_b = [&](SV_PANEL_PARAMS, int k, int buf, int i) SV_INLINE {
    const int j = panel(i);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(j == 0 ? rB0 : j == 1 ? rB1 : j == 2 ? rB2 : rB3,
                                             (__attribute__((address_space(3))) void*)(smem + buf + (wave + 4 * i) * 1024), 16, (int)voffB[i], k, 0, 0);
  };
  auto next_a = [](int b) { return b == (RA - 1) * ABUF ? 0 : b + ABUF; };
  auto next_w = [](int b) { return b == W0 + (RB - 1) * WBUF ? W0 : b + WBUF; };
  auto last_a = [](int b) { return b == 0 ? (RA - 1) * ABUF : b - ABUF; };
  auto last_w = [](int b) { return b == W0 ? W0 + (RB - 1) * WBUF : b - WBUF; };

  // ---- the epilogue's places.  Each wave turns its accumulators over 16 rows at a time through an LDS patch of its own and
  // reads them back so that LPR consecutive lanes hold one row's outputs (8 per lane), RPI rows per instruction.
  constexpr bool kHasInputs = EPI == EPI_RESID || EPI == EPI_SWIGLU_BWD || EPI == EPI_GELU_BWD || EPI == EPI_ROPE;
  constexpr int LPR = DUAL ? NI : 2 * NI, RPI = 64 / LPR, TR = 16 / RPI;
  static_assert(RPI <= 16, "a pass is no more than a row block");
  const int er = lane / LPR, ec = lane % LPR;
  const int mw = wm * 16 * MI, n = n0 + wn * (DUAL ? NI * 8 : NI * 16) + ec * 8;     // the lane's first row (+ er) and columns n .. n + 7
  const int rows = min(M - m0, BM);
  // rows past M lie past the descriptor's end, columns past N are sent there
  auto desc = [&](const void* base, int64_t ld, int es) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (int64_t)m0 * ld * es), (short)0, (int)(rows * ld * es), 0x00020000);
  };
  const unsigned vcol = n < a.N ? (unsigned)n : SPLIT ? 0x20000000u : 0x40000000u;     // byte offset 2^31: past every descriptor's end
  const bool rscaled = kEpiScaled<EPI> && !GROUPED && !SPLIT && a.rscale;
  // Plain and SwiGLU results are formed in the accumulators' layout, where a lane's values of a row block are of one row, and turned over in bf16.
  // (GELU, with so much arithmetic in front of the LDS writes: 30.9 -> 32.7 us for 2331 x 3840, K = 960 on 192x256.)
  constexpr bool kPacked = (EPI == EPI_STORE && !SPLIT) || EPI == EPI_SWIGLU;
  EpiIn in_lo[2][TR], in_hi[2][TR];
  float rs[2][TR], rs_row[kPacked ? MI : 1];
  int rope_p0 = 0, rope_i0 = 0;
  if (EPI == EPI_ROPE) { rope_p0 = (m0 + mw) % a.rope_S; rope_i0 = (n % a.rope_hd) >> 1; }
  auto ld16 = [&](__amdgpu_buffer_rsrc_t b, unsigned vo, bf16x4& lo, bf16x4& hi) {
    const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b, (int)vo, 0, 0));
    lo = __builtin_shufflevector(v, v, 0, 1, 2, 3);
    hi = __builtin_shufflevector(v, v, 4, 5, 6, 7);
  };
  auto load_inputs = [&](int mi, EpiIn (&lo)[TR], EpiIn (&hi)[TR], float (&f)[TR]) {
    if (kHasInputs) {
      const __amdgpu_buffer_rsrc_t bR = desc(a.R, a.ldr, 2), bR2 = desc(a.R2, a.ldr, 2);
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const int r = mw + mi * 16 + t * RPI + er;
        if (EPI == EPI_ROPE) {
          int p = rope_p0 + mi * 16 + t * RPI + er;
          if (a.rope_S >= BM) p -= p >= a.rope_S ? a.rope_S : 0; else p %= a.rope_S;
          const float* cs = a.rope_cs + ((int64_t)p * (a.rope_hd >> 1) + rope_i0) * 2;
          lo[t].cs = *reinterpret_cast<const f32x4*>(cs);
          hi[t].cs = *reinterpret_cast<const f32x4*>(cs + 4);
        } else {
          const unsigned vo = ((unsigned)(r * (int)a.ldr) + vcol) * 2u;
          ld16(bR, vo, lo[t].r, hi[t].r);
          if (EPI == EPI_SWIGLU_BWD) ld16(bR2, vo, lo[t].r2, hi[t].r2);
        }
      }
    }
    if (kEpiScaled<EPI> && !kPacked) {
#pragma unroll
      for (int t = 0; t < TR; ++t) f[t] = 1.0f;
      if (rscaled) {
#pragma unroll
        for (int t = 0; t < TR; ++t) f[t] = a.rscale[min(m0 + mw + mi * 16 + t * RPI + er, M - 1)];
      }
    }
  };

  f32x4 acc[NI][MI];

  // ---- fragment addresses: rows 16 b + (lane & 15) of an operand, chunk 4 s + (lane >> 4); swz16 does not see b
  unsigned offX[2], offW[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int chunk = ((s * 4 + lhi) ^ swz16(l15)) << 4;
    offX[s] = (unsigned)((wm * 16 * MI + l15) * 128 + chunk);
    offW[s] = (unsigned)((wn * (DUAL ? 8 : 16) * NI + l15) * 128 + chunk);
  }
  constexpr int kUp = DUAL ? BN / 32 - NI / 2 : 0;         // from the block after the last gate block to the first up block
  auto read_x = [&](int buf, int s, int b) { return *reinterpret_cast<const bf16x8*>(smem + buf + offX[s] + b * 2048); };
  auto read_w = [&](int buf, int s, int b) { return *reinterpret_cast<const bf16x8*>(smem + buf + offW[s] + (DUAL && b >= NI / 2 ? b + kUp : b) * 2048); };
#define SV_SB __builtin_amdgcn_sched_barrier(0)
#define SV_MEET(imm) do { SV_SB; __builtin_amdgcn_s_waitcnt(imm); asm volatile("s_barrier" ::: "memory"); SV_SB; } while (0)
  constexpr int kLgkm0 = 0xc07f;                           // lgkmcnt(0), nothing else
  auto step = [&](auto first, auto into_w, auto reads, auto loads, auto ends, SV_PANEL_PARAMS, int k, bf16x8 (&xc)[MI], bf16x8 (&wc)[NI], bf16x8 (&xn)[MI],
                  bf16x8 (&wn_)[NI], int ra, int rw, int s, int db) {
    constexpr bool W = decltype(into_w)::value;
    constexpr int ND = W ? NI : MI, NMEM = MI + NI + ND, NM = MI * NI, SPAN = NM * 3 / 4;
    const f32x4 zero{0.0f, 0.0f, 0.0f, 0.0f};
    auto mul = [&](int f) {
      const int g = f / MI, j = f % MI, m = g & 1 ? MI - 1 - j : j;       // back and forth, so that neighbours share an operand
      acc[g][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wc[g], xc[m], decltype(first)::value ? zero : acc[g][m], 0, 0, 0);
    };
#pragma unroll
    for (int f = 0; f < SPAN; ++f) {
      mul(f);
      // the memory instructions [lo, hi) stand behind this MFMA
      const int lo = (f * NMEM + SPAN - 1) / SPAN, hi = f + 1 == SPAN ? NMEM : ((f + 1) * NMEM + SPAN - 1) / SPAN;
      if (hi > lo) SV_SB;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = lo + i, d = q * ND / NMEM, r = q - d;
        const bool load = (q + 1) * ND / NMEM > d;
        if (q >= hi || !(load ? decltype(loads)::value : decltype(reads)::value)) continue;
        if (load) { if (W) dma_b(SV_PANEL_ARGS, k, db, d); else dma_a(SV_PANEL_ARGS, k, db, d); }
        else if (r < MI) xn[r] = read_x(ra, s, r);
        else wn_[r - MI] = read_w(rw, s, r - MI);
        SV_SB;
      }
    }
    if (decltype(ends)::value) { if (W) advance_b(); else advance_a(); }   // between MFMAs, as there
    SV_SB;
#pragma unroll
    for (int f = SPAN; f < NM; ++f) mul(f);
  };

  if (kPacked) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) rs_row[mi] = 1.0f;
    if (rscaled) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) rs_row[mi] = a.rscale[min(m0 + mw + mi * 16 + l15, M - 1)];
    }
  } else if (!SPLIT) load_inputs(0, in_lo[0], in_hi[0], rs[0]);      // older than every slice: in order, so landed when the first has
  SV_SB;
  set_a(a.seg[SPLIT ? seg0 : 0]);
  set_b(a.seg[SPLIT ? seg0 : 0]);
  // Slices past the last are not loaded (from memory or as zeros, they were up to half of a short product's way into LDS).
#pragma unroll
  for (int s = 0; s + 1 < RA; ++s) {
    if (s > 0 && s >= nsl) continue;
    SV_PANELS;
#pragma unroll
    for (int j = 0; j < MI; ++j) dma_a(SV_PANEL_ARGS, ka, s * ABUF, j);
    advance_a();
    if (s + 1 < RB) {
#pragma unroll
      for (int j = 0; j < NI; ++j) dma_b(SV_PANEL_ARGS, kb, W0 + s * WBUF, j);
      advance_b();
    }
  }
  bf16x8 x0[MI], w0[NI], x1[MI], w1[NI];
  f32x4 tot[SUMMED ? NI : 1][SUMMED ? MI : 1];
  int run_end = nsl, runs = 1, run_i = 0;                  // SUMMED: the run being summed ends before slice run_end
  if (SUMMED) {
    int j = 0, c = n0;
    while (j + 1 < a.nbcol && c >= a.ncol[j]) { c -= a.ncol[j]; ++j; }
    runs = a.runs[j];
    run_end = nsl / runs;
  }
  int ca = 0, cw = W0;                                     // the buffers of the slice being multiplied
  // this wave's wait for a slice with j more behind it, then the workgroup's barrier: everybody's loads of that slice have landed, their
  // reads of the one before are done
  auto meet = [&](int j) SV_INLINE {
    SV_SB;
    if (j >= RA - 2) __builtin_amdgcn_s_waitcnt(meet_wait(C::LEFT));
    if (j == 0) __builtin_amdgcn_s_waitcnt(meet_wait(C::left(0)));
    if (RA > 3 && j == 1) __builtin_amdgcn_s_waitcnt(meet_wait(C::left(1)));
    if (RA > 4 && j == 2) __builtin_amdgcn_s_waitcnt(meet_wait(C::left(2)));
    SV_MEET(meet_wait(63));
  };
  meet(nsl - 1);
  if (nsl >= RB) {
    SV_PANELS;
#pragma unroll
    for (int j = 0; j < NI; ++j) dma_b(SV_PANEL_ARGS, kb, last_w(cw), j);
    advance_b();
  }
#pragma unroll
  for (int b = 0; b < MI; ++b) x0[b] = read_x(ca, 0, b);
#pragma unroll
  for (int b = 0; b < NI; ++b) w0[b] = read_w(cw, 0, b);
  // SUMMED: the accumulators go to the total (which begins as -0, what every sum leaves as it is) and begin again: from zero operands of the
  // step behind where the registers have room for that step twice, else from zeros.  1077 x 1024, K = 1024 in runs of 2 slices, us: 13.6 with a select
  // for the first run and zeros, 12.8.
  constexpr bool kFresh = SUMMED && C::OCC == 1;
  if constexpr (SUMMED) {
#pragma unroll
    for (int i = 0; i < NI * MI * 4; ++i) tot[i / (MI * 4)][i / 4 % MI][i % 4] = -0.0f;
  }
  auto end_run = [&](auto summed) SV_INLINE {
    if constexpr (decltype(summed)::value) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            tot[ni][mi][r] += acc[ni][mi][r];
            if (!kFresh) acc[ni][mi][r] = 0.0f;
          }
      ++run_i;
      run_end = (int)((int64_t)(run_i + 1) * nsl / runs);
    }
  };
  using Yes = std::true_type;
  using No = std::false_type;
  __builtin_amdgcn_s_waitcnt(kLgkm0);
  SV_SB;
  if (nsl >= RA) {
    SV_PANELS;
    step(Yes{}, No{}, Yes{}, Yes{}, Yes{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
  } else {
    SV_PANELS;
    step(Yes{}, No{}, Yes{}, No{}, No{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
  }
  ca = next_a(ca); cw = next_w(cw);
  meet(nsl - 2);
  int kt = 1;
  while (kt <= nsl - RA) {
    // the slices before one at which a stream's segment ends: as in the 256x256 kernel
    SV_PANELS;
    int n = min(min(a_turn, w_turn) - 1, nsl - RA - kt + 1);
    n = __builtin_amdgcn_readfirstlane(n);
    for (int i = 0; i < n; ++i) {
      step(No{}, Yes{}, Yes{}, Yes{}, No{}, SV_PANEL_ARGS, kb, x1, w1, x0, w0, ca, cw, 0, last_w(cw));
      const bool ended = SUMMED && kt + i == run_end;
      if (__builtin_expect(ended, 0)) end_run(std::integral_constant<bool, SUMMED>{});
      __builtin_amdgcn_s_waitcnt(kLgkm0);
      SV_SB;
      if (kFresh && ended) step(std::integral_constant<bool, kFresh>{}, No{}, Yes{}, Yes{}, No{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
      else step(No{}, No{}, Yes{}, Yes{}, No{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
      ca = next_a(ca); cw = next_w(cw);
      ka += BK * 2; kb += BK * 2;
      SV_MEET(meet_wait(C::LEFT));
    }
    kt += n;
    a_turn -= n; a_k += n * BK;
    w_turn -= n; w_k += n * BK;
    if (kt > nsl - RA) break;
    step(No{}, Yes{}, Yes{}, Yes{}, Yes{}, SV_PANEL_ARGS, kb, x1, w1, x0, w0, ca, cw, 0, last_w(cw));
    const bool ended = SUMMED && kt == run_end;
    if (__builtin_expect(ended, 0)) end_run(std::integral_constant<bool, SUMMED>{});
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    SV_SB;
    if (kFresh && ended) step(std::integral_constant<bool, kFresh>{}, No{}, Yes{}, Yes{}, Yes{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
    else step(No{}, No{}, Yes{}, Yes{}, Yes{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
    ca = next_a(ca); cw = next_w(cw);
    ++kt;
    SV_MEET(meet_wait(C::LEFT));
  }
  // the last slices, with j more behind each: their activations are on their way, and so are their weights but for one slice's where the
  // activations' ring is the longer
  auto ending = [&](auto jc) SV_INLINE {
    constexpr int j = decltype(jc)::value;
    if (nsl < j + 2) return;
    SV_PANELS;
    step(No{}, Yes{}, Yes{}, std::integral_constant<bool, (j >= RB - 1)>{}, No{}, SV_PANEL_ARGS, kb, x1, w1, x0, w0, ca, cw, 0, last_w(cw));
    const bool ended = SUMMED && nsl - 1 - j == run_end;
    if (__builtin_expect(ended, 0)) end_run(std::integral_constant<bool, SUMMED>{});
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    SV_SB;
    if (kFresh && ended) step(std::integral_constant<bool, kFresh>{}, No{}, Yes{}, No{}, No{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
    else step(No{}, No{}, Yes{}, No{}, No{}, SV_PANEL_ARGS, ka, x0, w0, x1, w1, ca, cw, 1, last_a(ca));
    ca = next_a(ca); cw = next_w(cw);
    SV_MEET(meet_wait(C::left(j > 0 ? j - 1 : 0)));
  };
  if constexpr (RA > 4) ending(std::integral_constant<int, 3>{});
  if constexpr (RA > 3) ending(std::integral_constant<int, 2>{});
  ending(std::integral_constant<int, 1>{});
  ending(std::integral_constant<int, 0>{});
  static_assert(RA >= 3 && RA <= 5, "the last slices");
  {
    SV_PANELS;
    step(No{}, Yes{}, No{}, No{}, No{}, SV_PANEL_ARGS, kb, x1, w1, x0, w0, ca, cw, 0, last_w(cw));
  }
  end_run(std::integral_constant<bool, SUMMED>{});

  // ---- epilogue.  The patches lie in the weights' buffer that everybody has read and no load is on its way to.  A wave's LDS accesses are
  // served in their order: block mi + 1 is on its way into the patch and out of it while block mi's results are formed or stored, with no
  // wait between its writes and reads.
  char* patch = smem + last_w(cw) + wave * (NI * 1024);
  const __amdgpu_buffer_rsrc_t bC = SPLIT ? desc(a.split_ws + (int64_t)run * M * a.N, a.N, 4) : desc(a.C, a.ldc, 2);
  const __amdgpu_buffer_rsrc_t bC2 = desc(a.C2, a.ldc, 2), bC3 = desc(a.C3, a.ldc, 2);
  const bool keeps2 = EPI == EPI_SWIGLU_BWD || ((EPI == EPI_GELU || EPI == EPI_SWIGLU) && a.C2), keeps3 = EPI == EPI_SWIGLU && a.C3;
  if constexpr (kPacked) {
    // A row of a patch: LPR chunks of 16 bytes (8 features), XOR-swizzled by the row; a patch for each output.  Half of the LDS traffic of fp32
    // patches: 3000 x 1536 on 256x128, K = 512 10.8 -> 10.3 us.
    constexpr int PB = 16 * LPR * 16;
    static_assert((DUAL ? 3 : 1) * PB <= NI * 1024, "the patches lie in the wave's part of the buffer");
    auto mix = [](int row) { return LPR == 16 ? row : LPR == 8 ? row >> 1 : row >> 2; };
    bf16x8 out[2][TR][3];
    auto turn_over = [&](int mi) SV_INLINE {
#pragma unroll
      for (int ni = 0; ni < (DUAL ? NI / 2 : NI); ++ni) {
        float v[4], u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i] = SUMMED ? tot[SUMMED ? ni : 0][SUMMED ? mi : 0][i] : acc[ni][mi][i];
          u[i] = DUAL ? acc[DUAL ? ni + NI / 2 : ni][mi][i] : 0.0f;
        }
        char* const at = patch + l15 * (LPR * 16) + (((ni * 2 + (lhi >> 1)) ^ mix(l15)) << 4) + (lhi & 1) * 8;
        epilogue_math4<EPI>(a, false, v, u, EpiIn{}, rs_row[mi], [&](int w, bf16x4 x) { *reinterpret_cast<bf16x4*>(at + w * PB) = x; });
      }
      SV_SB;
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const char* const at = patch + (t * RPI + er) * (LPR * 16) + ((ec ^ mix(t * RPI + er)) << 4);
        out[mi & 1][t][0] = *reinterpret_cast<const bf16x8*>(at);
        if (keeps2) out[mi & 1][t][1] = *reinterpret_cast<const bf16x8*>(at + PB);
        if (keeps3) out[mi & 1][t][2] = *reinterpret_cast<const bf16x8*>(at + 2 * PB);
      }
      SV_SB;
    };
    turn_over(0);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      if (mi + 1 < MI) turn_over(mi + 1);
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const int vo = (int)(((unsigned)((mw + mi * 16 + t * RPI + er) * (int)a.ldc) + vcol) * 2u);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[mi & 1][t][0]), bC, vo, 0, 0);
        if (keeps2) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[mi & 1][t][1]), bC2, vo, 0, 0);
        if (keeps3) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[mi & 1][t][2]), bC3, vo, 0, 0);
      }
      SV_SB;
    }
    return;
  }
  // With inputs, and for partial products, in fp32.  A row of a patch: 4 NI chunks of 16 bytes (4 features), those of a lane's 8 columns LPR
  // apart, XOR-swizzled by the row.
  auto mix = [](int row) { return (row >> (NI == 2 ? 1 : 0)) & (2 * NI - 1); };
  f32x4 lo[2][TR], hi[2][TR];
  auto turn_over = [&](int mi) SV_INLINE {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int slot = ni * 2 + (lhi >> 1) + (lhi & 1) * LPR;
      *reinterpret_cast<f32x4*>(patch + l15 * (NI * 64) + ((slot ^ mix(l15)) << 4)) = SUMMED ? tot[SUMMED ? ni : 0][SUMMED ? mi : 0] : acc[ni][mi];
    }
    SV_SB;
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const int row = t * RPI + er;
      auto at = [&](int slot) { return *reinterpret_cast<const f32x4*>(patch + row * (NI * 64) + ((slot ^ mix(row)) << 4)); };
      lo[mi & 1][t] = at(ec); hi[mi & 1][t] = at(LPR + ec);
    }
    SV_SB;
  };
  turn_over(0);
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    if (!SPLIT && mi + 1 < MI) load_inputs(mi + 1, in_lo[(mi + 1) & 1], in_hi[(mi + 1) & 1], rs[(mi + 1) & 1]);
    if (mi + 1 < MI) turn_over(mi + 1);
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const int r = mw + mi * 16 + t * RPI + er;
      if (SPLIT) {
        const int vo = (int)(((unsigned)(r * a.N) + vcol) * 4u);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lo[mi & 1][t]), bC, vo, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hi[mi & 1][t]), bC, vo + 16, 0, 0);
        continue;
      }
      const int vo = (int)(((unsigned)(r * (int)a.ldc) + vcol) * 2u);
      const bool roped = EPI == EPI_ROPE && n < a.rope_cols;
      const float f = kEpiScaled<EPI> ? rs[mi & 1][t] : 1.0f;
      bf16x4 o[2][3];
      auto half = [&](int h, const f32x4& x, const EpiIn& e) {
        float v[4], u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { v[i] = x[i]; u[i] = 0.0f; }
        epilogue_math4<EPI>(a, roped, v, u, e, f, [&](int w, bf16x4 p) { o[h][w] = p; });
      };
      half(0, lo[mi & 1][t], in_lo[mi & 1][t]);
      half(1, hi[mi & 1][t], in_hi[mi & 1][t]);
      auto put = [&](const __amdgpu_buffer_rsrc_t& b, int w) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, __builtin_shufflevector(o[0][w], o[1][w], 0, 1, 2, 3, 4, 5, 6, 7)), b, vo, 0, 0);
      };
      put(bC, 0);
      if (keeps2) put(bC2, 1);
    }
    SV_SB;
  }
#undef SV_MEET
#undef SV_SB
#undef SV_PANELS
#undef SV_PANEL_ARGS
#undef SV_PANEL_PARAMS
}

inline int k_slices(const GemmArgs& a) {
  int n = 0;
  for (int s = 0; s < a.nseg; ++s) n += a.seg[s].K / BK;
  return n;
}

template <int MI, int NI, int RA, int RB, int EPI, bool GROUPED, bool SPLIT = false, bool SUMMED = false, bool TAIL = false>
hipError_t launch_mid(const GemmArgs& a, int nsplit, hipStream_t st, int tail_max = 0) {      // tail_max: tiles per XCD a tail has at most
  using C = MidCfg<MI, NI, RA, RB, EPI == EPI_SWIGLU>;
  auto kern = gemm_mid_kernel<MI, NI, RA, RB, EPI, GROUPED, SPLIT, SUMMED, TAIL>;
  static bool configured = false;   // per process; the attribute is per function
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (a.M + C::BM - 1) / C::BM, tiles_n = (a.N + C::NOUT - 1) / C::NOUT;
  const int64_t per_xcd = TAIL ? (int64_t)tail_max * (256 / C::BM) * (256 / C::BN) : ((int64_t)tiles_m * tiles_n * nsplit + 7) / 8;
  GemmArgs g = a;
  g.slices = k_slices(a);
  hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(256), C::LDS, st, g, tiles_m, tiles_n, nsplit);
  return hipGetLastError();
}

template <int EPI, bool GROUPED, bool NF = false>
hipError_t launch_dma(const GemmArgs& a, hipStream_t st) {
  auto kern = gemm_mfma_dma_kernel<EPI, GROUPED, NF>;
  constexpr int lds = 5 * 256 * 128;                      // three buffers of activations, two of weights
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (a.M + 255) / 256, tiles_n = a.N / (EPI == EPI_SWIGLU ? 128 : 256);
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  const int n_cu = std::max(8, cu_count() / 8 * 8);       // one persistent workgroup per CU (all of its LDS)
  const int grid = per_xcd * 8 < n_cu ? per_xcd * 8 : n_cu;
  GemmArgs g = a;
  g.slices = k_slices(a);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, g, tiles_m, tiles_n);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI>
hipError_t launch_kn(const GemmArgs& a, hipStream_t st) {
  using C = Cfg<BM, BN, WAVES_M, WAVES_N>;
  auto kern = gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, EPI>;
  static bool configured = false;   // per process; the attribute is per function
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = a.N / BN;
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(C::NT), C::LDS, st, a, tiles_m, tiles_n);
  return hipGetLastError();
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// ---- which kernel and tile serves a product.  Every choice is priced as rounds of workgroups over the CUs times (a fixed part
// + slices x time per slice), plus for runs of k slices the reduction launch and the traffic of the partial products; the
// cheapest is taken.  The figures are microseconds fitted to a sweep over 64 .. 8192 rows, 320 .. 14336 columns and K =
// 512 .. 14336 with every tile forced, within 15 % of what the kernels took before their present k loops, one workgroup of 128x128
// a CU.  They stand for the lines between the tiles, which the tests name, and no longer for times: prices fitted later to kernels on
// these loops took tiles that were 0.8 % faster on average over 156 sizes.  They are those of a plain store: the dearer
// epilogues (SwiGLU with its stashes, SwiGLU-backward) cost the same here, and a tile more than the last full round counts as a
// round (on 256x256 tiles: as a second launch on smaller ones, where tail_tiles says so).  Against 256x256 tiles over runs of k, which these replaced, k of 9000 and more for 500 .. 1500 rows of 3072 .. 4096 columns
// was left 5 .. 15 % slower (1453 x 3072, K = 9728: 97 -> 112 us), everything else even or faster.  Where the lines come out, with both
// sides as they were measured on that sweep: 4096 x 1024, K = 1024 (256 tiles of 128 x 128) 13.4 us against 19 on 256 x 128 and 33 on
// 256 x 256 over runs; 8192 x 1024, K = 8192 (256 tiles of 256 x 128) 113 us against 121 and 124; 8192 x 2048, K = 2048
// (256 tiles of 256 x 256) 59 us against 64 on 256 x 128; 512 x 4096, K = 14336 (256 x 128 over 4 runs) 63 us against 85 whole;
// 1024^3 (256 tiles of 64 x 64) 7.0 us against 8.1 on 64 x 128 and 9.6 on 128 x 128.
enum TileKind { kTile256 = 0, kTile256x128, kTile128, kTile64x128, kTile64, kTileKinds, kTile192x256 = kTileKinds };
struct TileCost { int bm, bn; double fixed, slice; };
constexpr TileCost kTileCost[kTileKinds] = {{256, 256, 4.0, 1.55}, {256, 128, 6.5, 0.86}, {128, 128, 5.0, 0.52}, {64, 128, 4.0, 0.36}, {64, 64, 3.5, 0.21}};
struct Plan { int kind, runs; };

// workgroups of the persistent kernel per XCD
int tile_slots() { return std::max(8, cu_count() / 8 * 8) / 8; }

bool panels_fit(const GemmArgs& a) {      // 32-bit byte offsets inside a panel of 256 rows, and inside a tile's outputs
  for (int s = 0; s < a.nseg; ++s)
    if (!(256 * a.seg[s].lda * 2 < (int64_t)1 << 32 && 256 * a.seg[s].ldb * 2 < (int64_t)1 << 32)) return false;
  return !(a.epi == EPI_SWIGLU && 256 * a.ldb2 * 2 >= (int64_t)1 << 32);
}

bool fits_256(const GemmArgs& a) {        // the persistent 256x256 kernel has whole tiles of columns
  if (a.N % (a.epi == EPI_SWIGLU ? 128 : 256)) return false;
  for (int j = 0; j < a.nbcol; ++j)
    if (a.ncol[j] % 256) return false;
  return 256 * a.ldc * 2 < (int64_t)1 << 31 && 256 * a.ldr * 2 < (int64_t)1 << 31;      // a tile's outputs by 32-bit byte offsets
}

bool fits_mid(const GemmArgs& a) {        // buffer descriptors over a tile's rows keep below 2^31 bytes
  return 256 * a.ldc * 2 < (int64_t)1 << 31 && 256 * a.ldr * 2 < (int64_t)1 << 31 && (int64_t)256 * a.N * 4 < (int64_t)1 << 31;
}

bool summed_runs(const GemmArgs& a) { return a.runs[0] > 1 || a.runs[1] > 1 || a.runs[2] > 1; }

// The epilogues that form an activation or its derivative are a fifth to a third of a product's time at K = 1024, and a launch of fewer
// 256x256 tiles than CUs does them on part of the chip.  192x256 tiles, while they too are one round, give every
// CU three quarters of a tile.  256x256 -> 192x256, us: GELU 2331 x 3840, K = 960 (150 tiles, 195 of these) 38.1 -> 31.0, its backward
// 37.4 -> 31.2; 4096 x 2560, K = 1024 39.1 -> 33.1; SwiGLU with its stashes 2331 x 1920, K = 960 30.7 -> 25.6, its backward at 3840
// columns 34.9 -> 32.1; 900 x 5120, K = 2048 48.3 -> 43.3; 800 x 6144, K = 3072 68.2 -> 62.6.  With a longer k loop the bare product
// decides: GELU 768 x 16384, K = 4096 104 -> 112.  (Plain stores and residual sums gain 1 - 9 % and stay where they are: what they run
// on is what sv_gemm_plan tells.)  Where 256x128 tiles were chosen, whole rounds decide, at what a round of either took on kernels with four waves'
// k loop (6.1 us and 0.65 a slice, 6.0 and 0.92; the plan's own price of 256x128 is of the form before).
bool narrower_pays(const GemmArgs& a, int kind, int slices) {
  if (a.epi != EPI_GELU && a.epi != EPI_GELU_BWD && a.epi != EPI_SWIGLU && a.epi != EPI_SWIGLU_BWD) return false;
  const int64_t nout = a.epi == EPI_SWIGLU ? 128 : 256, cus = cu_count(), tiles = (a.M + 191) / 192 * (a.N / nout);
  if (a.tile_group || slices > 48 || !fits_mid(a)) return false;
  if (kind == kTile256) return tiles <= cus;
  const int64_t tiles128 = (int64_t)((a.M + 255) / 256) * (2 * a.N / nout);
  return kind == kTile256x128 && a.N % nout == 0 &&
         (double)((tiles + cus - 1) / cus) * (6.0 + 0.92 * slices) < 0.95 * (double)((tiles128 + cus - 1) / cus) * (6.1 + 0.65 * slices);
}

// Asked twice for a product that may leave row sums, once to know whether it will (mfma_gemm_emits_rowsq) and once to launch it:
// with a.rowsq set the answer does not depend on the scratch, which only runs of k use.
Plan plan_gemm(const GemmArgs& a) {
  if (summed_runs(a)) return Plan{kTile128, 1};
  const bool dual = a.epi == EPI_SWIGLU;
  const int slices = k_slices(a);
  const double cus = cu_count();
  Plan best{-1, 1};
  double best_cost = 0.0;
  for (int k = 0; k < kTileKinds; ++k) {
    if (k == kTile256 ? !fits_256(a) : !fits_mid(a)) continue;
    if (k == kTile64 && dual) continue;                  // a wave of it holds one block of 32 columns: no gate / up pair
    const TileCost& t = kTileCost[k];
    const int nout = dual ? t.bn / 2 : t.bn;
    const int64_t tiles = (int64_t)((a.M + t.bm - 1) / t.bm) * ((a.N + nout - 1) / nout);
    const bool splits = a.split_ws && !a.runs[0] && !a.rowsq && k != kTile256 && !dual && !a.tile_group;
    for (int runs = 1; runs <= (splits ? 8 : 1); ++runs) {
      if (runs > 1 && (slices < 4 * runs || (int64_t)runs * a.M * a.N > a.split_ws_floats)) break;
      const double rounds = (double)((tiles * runs + (int64_t)cus - 1) / (int64_t)cus);
      double cost = rounds * (t.fixed + t.slice * ((slices + runs - 1) / runs));
      if (k == kTile256) {
        cost += 4.0;
        const int per_xcd = (int)((tiles + 7) / 8), slots = tile_slots(), left = a.rowsq || a.tile_group ? 0 : tail_tiles(per_xcd, slots, slices);
        if (left > 0) {                                  // its last round on smaller tiles, in a launch of their own
          const TileCost& s = kTileCost[4 * left <= slots ? kTile128 : kTile256x128];
          cost = 7.0 + per_xcd / slots * (t.fixed + t.slice * slices) + s.fixed + s.slice * slices;
        }
      }
      if (runs > 1) cost += 4.0 + (4.0 * runs + 4.0) * a.M * (double)a.N / 4.5e6;
      if (best.kind < 0 || cost < best_cost) { best = Plan{k, runs}; best_cost = cost; }
    }
  }
  if (best.runs == 1 && narrower_pays(a, best.kind, slices)) best.kind = kTile192x256;      // 192x256 tiles have no form over runs of k
  return best;
}

// Tiles per XCD (at most) that a product on 256x256 tiles leaves to a second launch, or 0.  In groups the rows are known on the device
// only: somewhere between none and 255 of padding per group more than the tokens' rows; the second launch (4.5 us where it
// finds nothing to do) is made if half of the likely counts have a tail.
template <int EPI, bool GROUPED>
int tail_pays(const GemmArgs& a) {
  if (a.rowsq || !fits_mid(a)) return 0;                 // row sums come from whole 256 x 256 tiles only
  const int tiles_n = a.N / (EPI == EPI_SWIGLU ? 128 : 256), slots = tile_slots();
  const int slices = k_slices(a);
  if (!GROUPED) return tail_tiles(((a.M + 255) / 256 * tiles_n + 7) / 8, slots, slices);
  const int most = a.M / 256, pad = std::min(most - 1, a.groups);
  int with = 0, all = 0, left = 0;
  for (int b = most - pad + pad / 4; b <= most - pad / 4; ++b, ++all) {
    const int t = tail_tiles((b * tiles_n + 7) / 8, slots, slices);
    with += t > 0;
  }
  for (int b = std::max(1, most - pad); b <= most; ++b) left = std::max(left, tail_tiles((b * tiles_n + 7) / 8, slots, slices));
  return 2 * with >= all ? left : 0;
}

// 128x128 tiles: two workgroups of 80 KB on a CU where there are tiles for them (4096 x 3072, K = 1024 28.0 -> 25.8 us, 8192 x 1024 19.6 ->
// 17.9; 8192 x 768 with rotation and settled sums, K = 512 23.0 -> 16.6), one with four buffers of each operand where every tile has a CU
// of its own (2304 x 960, K = 960 from memory 13.3 us against 15.2; with five and four of them, 16 KB more to fill before the first MFMA, 13.6).
bool two_per_cu(const GemmArgs& a, int runs) {
  const int nout = a.epi == EPI_SWIGLU ? 64 : 128;
  return (int64_t)((a.M + 127) / 128) * ((a.N + nout - 1) / nout) * runs > cu_count();
}

// the form that scales rows, where there is one
template <int EPI, bool GROUPED>
hipError_t launch_dma_nf(const GemmArgs& a, hipStream_t st) {
  if constexpr (!GROUPED && EPI != EPI_SWIGLU_BWD && EPI != EPI_GELU_BWD) return launch_dma<EPI, false, true>(a, st);
  else return hipErrorInvalidValue;
}

template <int EPI, bool GROUPED>
hipError_t launch_tile(const GemmArgs& a, int kind, hipStream_t st) {
  switch (kind) {
    case kTile256: {
      const int left = tail_pays<EPI, GROUPED>(a);
      if (left > 0) {
        GemmArgs g = a;
        g.tail = tile_slots();
        hipError_t e = g.rscale ? launch_dma_nf<EPI, GROUPED>(g, st) : launch_dma<EPI, GROUPED>(g, st);
        if (e != hipSuccess) return e;
        if (GROUPED || 4 * left <= g.tail) return launch_mid<4, 4, 4, 4, EPI, GROUPED, false, false, true>(g, 1, st, left);
        if constexpr (!GROUPED) return launch_mid<8, 4, 3, 3, EPI, false, false, false, true>(g, 1, st, left);
      }
      if constexpr (!GROUPED && EPI != EPI_SWIGLU_BWD && EPI != EPI_GELU_BWD)
        if (a.rscale || a.rowsq) return launch_dma<EPI, false, true>(a, st);   // the ends of a norm that runs inside the products
      return launch_dma<EPI, GROUPED>(a, st);
    }
    case kTile256x128: return launch_mid<8, 4, 3, 3, EPI, GROUPED>(a, 1, st);
    case kTile128: return two_per_cu(a, 1) ? launch_mid<4, 4, 3, 2, EPI, GROUPED>(a, 1, st) : launch_mid<4, 4, 4, 4, EPI, GROUPED>(a, 1, st);
    case kTile64x128: return launch_mid<2, 4, 4, 3, EPI, GROUPED>(a, 1, st);
    case kTile192x256:
      if constexpr (!GROUPED && (EPI == EPI_GELU || EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_BWD))
        return launch_mid<6, 8, 3, 2, EPI, false>(a, 1, st);
      return hipErrorInvalidValue;
    default:
      if constexpr (EPI != EPI_SWIGLU) return launch_mid<2, 2, 5, 5, EPI, GROUPED>(a, 1, st);
      return hipErrorInvalidValue;
  }
}

// runs of k slices into a.split_ws, then the reduction with the epilogue
template <int EPI>
hipError_t launch_runs(const GemmArgs& a, const Plan& p, hipStream_t st) {
  hipError_t e;
  switch (p.kind) {
    case kTile256x128: e = launch_mid<8, 4, 3, 3, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile128: e = two_per_cu(a, p.runs) ? launch_mid<4, 4, 3, 2, EPI_STORE, false, true>(a, p.runs, st) : launch_mid<4, 4, 4, 4, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile64x128: e = launch_mid<2, 4, 4, 3, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile64: e = launch_mid<2, 2, 5, 5, EPI_STORE, false, true>(a, p.runs, st); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const int64_t threads = (int64_t)a.M * (a.N / 4);
  hipLaunchKernelGGL(splitk_reduce_kernel<EPI>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a, p.runs);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_plan(const GemmArgs& a, const Plan& p, hipStream_t st) {
  if (a.rowsq && (p.kind != kTile256 || p.runs > 1)) return hipErrorInvalidValue;    // somebody will read them: mfma_gemm_emits_rowsq first
  if (summed_runs(a)) {
    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID || EPI == EPI_ROPE)
      return two_per_cu(a, 1) ? launch_mid<4, 4, 3, 2, EPI, false, false, true>(a, 1, st) : launch_mid<4, 4, 4, 4, EPI, false, false, true>(a, 1, st);
    return hipErrorInvalidValue;
  }
  if constexpr (EPI != EPI_SWIGLU)
    if (p.runs > 1) return launch_runs<EPI>(a, p, st);
  return launch_tile<EPI, false>(a, p.kind, st);
}

}  // namespace

// Which expert a token takes is decided by sums that start here, and a near-tie follows their last bits: the products that lead to
// a router keep their sums cut the way verifiers of this library have cut them, while tile and launch are free.  The cut: runs that
// once brought 256x256 tiles to one workgroup per CU, or 128x64 tiles to three.  What it makes alike: the routing of two verifiers of
// one stage and token count whose scratch is the same or holds the runs either way (`fit`; the scratch grows with max_tokens up to
// a cap, and only q | k | v of narrow experts can be short of it), forward only or with backward.  Not covered: widths that were
// no multiple of 128 (of 64 along k, and in the experts' own products), which the vector kernels summed before these tiles took them.
int mfma_settled_runs(int64_t M, int N, int K, int64_t ws_floats) {
  const int slices = K / BK;
  const int64_t fit = ws_floats / std::max<int64_t>(1, M * N);
  if (N % 256 == 0) {
    const int64_t tiles = ((M + 255) / 256) * (N / 256);
    if (tiles >= 192) return 1;
    const int64_t n = std::min<int64_t>(std::min<int64_t>(std::min<int64_t>(8, 256 / tiles), slices / 4), fit);
    if (n >= 2) return (int)n;
  }
  const int64_t rows = (M + 127) / 128;
  if (N % 128 == 0 && rows * (N / 128) < 160) {
    const int64_t wgs = rows * (N / 64);
    const int64_t n = std::min<int64_t>(std::min<int64_t>(std::min<int64_t>(8, slices / 8), (768 + wgs - 1) / wgs), fit);
    if (n >= 2) return (int)n;
  }
  return 1;
}

bool mfma_gemm_emits_rowsq(const GemmArgs& a) {
  return a.rowsq && a.epi == EPI_RESID && !a.tile_group && mfma_gemm_supported(a) && plan_gemm(a).kind == kTile256;
}

void mfma_gemm_plan(const GemmArgs& a, int* tile, int* runs) {
  constexpr int number[kTileKinds + 1] = {1, 3, 2, 4, 5, 6};
  *tile = 0; *runs = 1;
  if (a.b_is_kn || !mfma_gemm_supported(a)) return;
  const Plan p = plan_gemm(a);
  *tile = number[p.kind]; *runs = p.runs;
}

int mfma_gemm_tail(const GemmArgs& a) {
  if (a.b_is_kn || !mfma_gemm_supported(a) || !fits_256(a)) return 0;
  if (a.tile_group) return a.epi == EPI_SWIGLU ? tail_pays<EPI_SWIGLU, true>(a) : tail_pays<EPI_STORE, true>(a);
  return a.epi == EPI_SWIGLU ? tail_pays<EPI_SWIGLU, false>(a) : tail_pays<EPI_STORE, false>(a);
}

bool mfma_gemm_shape(const GemmArgs& a) {
  if (a.M < 1 || a.nseg < 1 || a.nseg > 3) return false;
  if (a.rscale && (a.tile_group || (a.epi != EPI_STORE && a.epi != EPI_GELU && a.epi != EPI_SWIGLU && a.epi != EPI_ROPE))) return false;
  if (a.rowsq && (a.epi != EPI_RESID || a.rowsq_ld < a.M)) return false;
  const bool dual = a.epi == EPI_SWIGLU;
  if (dual && (a.b_is_kn || a.nseg != 1 || !a.B2 || a.ldb2 % 8 || !aligned16(a.B2))) return false;
  if (a.epi < EPI_STORE || a.epi > EPI_ROPE) return false;
  if (a.nbcol > 0 || a.epi == EPI_ROPE) {                // the fused q | k | v form; a group of 8 weight rows belongs to one matrix
    if (a.b_is_kn || a.nseg != 1 || a.nbcol > 3) return false;
    int tot = 0;
    for (int j = 0; j < a.nbcol; ++j) { if (a.ncol[j] % 8 || !aligned16(a.Bcol[j])) return false; tot += a.ncol[j]; }
    if (a.nbcol > 0 && (tot != a.N || a.epi == EPI_SWIGLU)) return false;
    if (a.epi == EPI_ROPE && (!a.rope_cs || a.rope_hd % 8 || a.rope_cols % 8 || a.rope_S < 1)) return false;
  }
  if ((a.tile_group != nullptr) != (a.m_dev != nullptr)) return false;      // the grouped form needs both
  if (a.tile_group && (a.b_is_kn || a.nbcol > 0 || a.group_stride % 8 || a.M % 256)) return false;
  if (a.tile_group && a.epi != EPI_STORE && a.epi != EPI_SWIGLU && a.epi != EPI_SWIGLU_BWD) return false;
  if (summed_runs(a)) {                                  // served by the 128x128 tile, whose columns lie in one matrix
    if (a.b_is_kn || a.tile_group || a.nseg != 1 || a.rowsq || !fits_mid(a) || (a.epi != EPI_STORE && a.epi != EPI_RESID && a.epi != EPI_ROPE)) return false;
    for (int j = 0; j < std::max(1, a.nbcol); ++j)
      if (a.runs[j] < 1 || a.runs[j] > a.seg[0].K / BK || (a.nbcol > 0 && a.ncol[j] % 128)) return false;
  }
  if (a.b_is_kn && (a.epi == EPI_RESID || a.epi == EPI_GELU || a.epi == EPI_SWIGLU)) return false;
  if ((a.epi == EPI_RESID || a.epi == EPI_SWIGLU_BWD || a.epi == EPI_GELU_BWD) && !a.R) return false;
  if (a.epi == EPI_SWIGLU_BWD && (!a.R2 || !a.C2)) return false;
  if (a.N < 8 || a.N % (a.b_is_kn ? 128 : 8)) return false;
  // Row strides are multiples of 4 values: the epilogues' accesses of 16 bytes then stand on 8-byte boundaries, and buffer accesses of any
  // width need whole dwords only.
  if (a.ldc % 4 || !aligned16(a.C)) return false;
  if ((a.C2 && !aligned16(a.C2)) || (a.C3 && !aligned16(a.C3))) return false;
  if ((a.R || a.R2) && (a.ldr % 4 || !aligned16(a.R) || (a.R2 && !aligned16(a.R2)))) return false;
  for (int s = 0; s < a.nseg; ++s) {
    const GemmSeg& g = a.seg[s];
    if (g.K < BK || g.K % BK || g.lda % 8 || g.ldb % 8 || !aligned16(g.A) || !aligned16(g.B)) return false;
  }
  return true;
}

bool mfma_gemm_reaches(const GemmArgs& a, int tile) {
  if (a.b_is_kn) return true;                            // 64-bit addresses
  return panels_fit(a) && ((tile <= 1 && fits_256(a)) || (tile != 1 && fits_mid(a)));
}

bool mfma_gemm_supported(const GemmArgs& a) { return mfma_gemm_shape(a) && mfma_gemm_reaches(a, 0); }

hipError_t mfma_gemm(const GemmArgs& a, hipStream_t st, int tile) {
  if (!mfma_gemm_supported(a)) return hipErrorInvalidValue;
  if ((tile == 1 || tile == 3) && a.N % (a.epi == EPI_SWIGLU ? 128 : 256)) return hipErrorInvalidValue;
  if (a.b_is_kn) {
    const bool big = tile == 1 || tile == 3 || (tile == 0 && a.N % 256 == 0 && (int64_t)((a.M + 255) / 256) * (a.N / 256) >= 192);
    switch (a.epi) {
      case EPI_STORE: return big ? launch_kn<256, 256, 2, 2, EPI_STORE>(a, st) : launch_kn<128, 128, 2, 1, EPI_STORE>(a, st);
      case EPI_SWIGLU_BWD: return big ? launch_kn<256, 256, 2, 2, EPI_SWIGLU_BWD>(a, st) : launch_kn<128, 128, 2, 1, EPI_SWIGLU_BWD>(a, st);
      case EPI_GELU_BWD: return big ? launch_kn<256, 256, 2, 2, EPI_GELU_BWD>(a, st) : launch_kn<128, 128, 2, 1, EPI_GELU_BWD>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  Plan p{tile == 1 ? kTile256 : tile == 2 ? kTile128 : tile == 3 ? kTile256x128 : kTile64x128, 1};
  if (tile == 0) p = plan_gemm(a);
  else if (p.kind == kTile256 ? !fits_256(a) : !fits_mid(a)) return hipErrorInvalidValue;
  if (a.tile_group) {
    switch (a.epi) {                                       // the epilogues the mixture-of-experts products use
      case EPI_STORE: return launch_tile<EPI_STORE, true>(a, p.kind, st);
      case EPI_SWIGLU: return launch_tile<EPI_SWIGLU, true>(a, p.kind, st);
      case EPI_SWIGLU_BWD: return launch_tile<EPI_SWIGLU_BWD, true>(a, p.kind, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (a.epi) {
    case EPI_STORE: return launch_plan<EPI_STORE>(a, p, st);
    case EPI_RESID: return launch_plan<EPI_RESID>(a, p, st);
    case EPI_GELU: return launch_plan<EPI_GELU>(a, p, st);
    case EPI_SWIGLU: return launch_plan<EPI_SWIGLU>(a, p, st);
    case EPI_SWIGLU_BWD: return launch_plan<EPI_SWIGLU_BWD>(a, p, st);
    case EPI_GELU_BWD: return launch_plan<EPI_GELU_BWD>(a, p, st);
    case EPI_ROPE: return launch_plan<EPI_ROPE>(a, p, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t mfma_gemm_runs(const GemmArgs& a, int tile, int runs, hipStream_t st) {
  constexpr int kind[6] = {-1, -1, kTile128, kTile256x128, kTile64x128, kTile64};
  if (a.epi != EPI_STORE || a.b_is_kn || a.nseg != 1 || a.tile_group || a.rowsq || tile < 2 || tile > 5 || runs < 1 || runs > a.seg[0].K / BK ||
      !mfma_gemm_supported(a) || !fits_mid(a))
    return hipErrorInvalidValue;
  if (a.split_ws) return (int64_t)runs * a.M * a.N <= a.split_ws_floats ? launch_runs<EPI_STORE>(a, Plan{kind[tile], runs}, st) : hipErrorInvalidValue;
  if (runs == 1) return launch_tile<EPI_STORE, false>(a, kind[tile], st);
  if (tile != 2) return hipErrorInvalidValue;
  GemmArgs g = a;
  g.runs[0] = runs;
  return mfma_gemm(g, st);
}

}  // namespace sv
