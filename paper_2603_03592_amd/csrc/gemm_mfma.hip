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
// XOR-swizzled by the row index, so that the 16-byte fragment reads of v_mfma_f32_32x32x16_bf16
// (a lane reads 8 consecutive k of one row) and the 16-byte staging writes are bank-conflict
// free.
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
// of work is shorter than a memory round trip, so one trip ahead leaves the epilogue waiting once per trip.
template <int EPI> constexpr int kEpiAhead = EPI == EPI_ROPE ? 2 : EPI == EPI_SWIGLU_BWD ? 3 : 4;   // as far as the registers go

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
// 256x256x64 NT kernel with direct global->LDS loads (buffer_load_dwordx4 ... lds, 16 bytes per lane).
//
// Each wave instruction copies 64 x 16 bytes to one contiguous 1 KB block of LDS = 8 tile rows;
// the XOR swizzle is applied by choosing WHICH global chunk each lane fetches, so the LDS image
// is the same swizzled layout the fragment reads expect and no VGPR staging or ds_write is
// needed.  The loads are buffer loads: a descriptor per operand panel in scalar registers, the
// lane's byte offset in one vector register, the slice's k offset as the scalar offset -- no
// 64-bit address arithmetic per slice.  Two LDS stages; the 16 loads a wave owes for slice k+1 and
// the 8 fragment reads of the next 16-wide k step are issued ONE AT A TIME BEHIND AN MFMA, in the
// 32 cycles the matrix pipe is busy with it (one wave per SIMD: whatever is issued between two
// MFMAs after the pipe has drained idles it; grouping them between blocks of four MFMAs measured
// 1-3 % slower), fragments double buffered in registers.  The loop is rotated so that the one
// full wait + barrier per slice sits at the loop top: after it the compiler's counter tracking
// is exact and no other wait stalls the MFMA stream.
//
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
  constexpr int BM = 256, BN = 256, STAGE = (BM + BN) * 128, MI = 4, NI = 4;
  constexpr int NOUT = DUAL ? 128 : 256;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // grouped form: the row count lives in device memory and the launch covers its bound
  const int M = GROUPED ? *a.m_dev : a.M;
  if (GROUPED) tiles_m = (M + BM - 1) / BM;
  // Persistent workgroups: workgroup b works on the virtual block ids b, b + gridDim.x, ...; a virtual id
  // maps to a tile so that ids congruent mod 8 (one XCD) walk a contiguous run of tiles in groups of
  // kGroupM row tiles.  gridDim.x is a multiple of 8, so a workgroup stays on its XCD's run.
  const int nblk = tiles_m * tiles_n;
  const int per_xcd = (nblk + 7) >> 3;
  int nslices = 0;
  for (int s = 0; s < a.nseg; ++s) nslices += a.seg[s].K / BK;
  const int own = a.tail ? per_xcd - tail_tiles(per_xcd, a.tail, nslices) : per_xcd;     // tiles per XCD of this launch
  auto tile_of = [&](int vb, int& m0, int& n0) -> bool {
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

  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;

  // ---- DMA side: one continuous stream of slices across this workgroup's tiles, always one slice
  // ahead of the multiply.  State: virtual block d_vb (tile d_m0, d_n0), segment dseg, offset dk.
  int d_vb = blockIdx.x, d_m0 = 0, d_n0 = 0, dseg = 0, dk = 0, d_K = 0;   // d_K: length of segment dseg, kept in a register
                                                                           // (a per-slice kernel-argument load would share
                                                                           // its wait counter with the LDS reads)
  bool d_valid = tile_of(d_vb, d_m0, d_n0);
  const char *gA, *gB, *gB2;
  __amdgpu_buffer_rsrc_t rA, rB, rB2;     // buffer descriptors of the panels the stream reads: base = first row, no bound
  unsigned voffA[8], voffB[8];
  auto set_segment = [&]() {
    const GemmSeg& sg = a.seg[dseg];
    d_K = sg.K;
    gA = (const char*)((const bf16*)sg.A + (int64_t)d_m0 * sg.lda);
    const int64_t goff = GROUPED ? (int64_t)a.tile_group[d_m0 >> 8] * a.group_stride : 0;
    if (!DUAL && a.nbcol > 0) {
      int start = 0, j = 0;
      while (j + 1 < a.nbcol && d_n0 >= start + a.ncol[j]) { start += a.ncol[j]; ++j; }
      gB = (const char*)((const bf16*)a.Bcol[j] + (int64_t)(d_n0 - start) * sg.ldb);
    } else {
      gB = (const char*)((const bf16*)sg.B + goff + (int64_t)d_n0 * sg.ldb);
    }
    gB2 = DUAL ? (const char*)((const bf16*)a.B2 + goff + (int64_t)d_n0 * a.ldb2) : gB;
    rA = __builtin_amdgcn_make_buffer_rsrc((void*)gA, (short)0, -1, 0x00020000);
    rB = __builtin_amdgcn_make_buffer_rsrc((void*)gB, (short)0, -1, 0x00020000);
    rB2 = __builtin_amdgcn_make_buffer_rsrc((void*)gB2, (short)0, -1, 0x00020000);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (wave + 4 * i) * 8 + (lane >> 3), c = (lane & 7) ^ swz(r);
      const int ra = min(r, M - 1 - d_m0);                  // ragged row tail: re-read the last row
      voffA[i] = (unsigned)((int64_t)ra * sg.lda + c * 8) * 2u;
      if (DUAL) voffB[i] = (unsigned)((int64_t)(r & 127) * (i >= 4 ? a.ldb2 : sg.ldb) + c * 8) * 2u;
      else voffB[i] = (unsigned)((int64_t)r * sg.ldb + c * 8) * 2u;
    }
  };
  auto dma = [&](int stage, int j) {                          // j: 0..7 activation rows, 8..15 weight rows
    const int i = j & 7;
    const unsigned off = j < 8 ? voffA[i] : voffB[i];
    char* dst = smem + stage * STAGE + (j < 8 ? 0 : BM * 128) + (wave + 4 * i) * 1024;
    // buffer form of the direct-to-LDS load: per-lane byte offset in a register, the slice's offset k * 2 as the scalar offset
    __builtin_amdgcn_raw_ptr_buffer_load_lds(j < 8 ? rA : ((DUAL && i >= 4) ? rB2 : rB), (__attribute__((address_space(3))) void*)dst, 16,
                                             (int)off, dk * 2, 0, 0);
  };
  auto advance = [&]() {                                      // to the next slice of the stream
    dk += BK;
    if (dk < d_K) return;
    dk = 0;
    if (dseg + 1 < a.nseg) { ++dseg; set_segment(); return; }
    dseg = 0;
    d_vb += gridDim.x;
    d_valid = tile_of(d_vb, d_m0, d_n0);
    if (d_valid) set_segment();
  };

  int xrow[MI], wrow[NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) xrow[mi] = wm * 128 + mi * 32 + l31;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) wrow[ni] = (DUAL ? (ni < 2 ? wn * 64 + ni * 32 : 128 + wn * 64 + (ni - 2) * 32) : wn * 128 + ni * 32) + l31;

  f32x16 acc[NI][MI];

#define SV_SB __builtin_amdgcn_sched_barrier(0)
  // One 16-wide k step: MFMAs on (xc, wc); fragments (rstage, rkk) are read into (xn, wn_) and the
  // DMAs [d0, d0 + 8) of the stream's next slice are issued into dstage, both spread over the four MFMA groups.
  auto step = [&](bf16x8 (&xc)[MI], bf16x8 (&wc)[NI], bf16x8 (&xn)[MI], bf16x8 (&wn_)[NI], bool do_read, int rstage, int rkk,
                  bool do_dma, int dstage, int d0) {
    const char* xs = smem + rstage * STAGE;
    const char* ws = xs + BM * 128;
    // The fragments this step multiplies were requested during the previous step, the youngest of them four MFMAs
    // ago: wait for them here, before this step's own requests are queued behind them.
    __builtin_amdgcn_s_waitcnt(0xc07f);
    SV_SB;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // every other instruction of the group is issued behind an MFMA, in the 32 cycles the matrix pipe is busy with it
      acc[g][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc[g], xc[0], acc[g][0], 0, 0, 0);
      SV_SB;
      if (do_read) xn[g] = *reinterpret_cast<const bf16x8*>(xs + lds_off(xrow[g], rkk * 2 + lhi));
      SV_SB;
      acc[g][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc[g], xc[1], acc[g][1], 0, 0, 0);
      SV_SB;
      if (do_read) wn_[g] = *reinterpret_cast<const bf16x8*>(ws + lds_off(wrow[g], rkk * 2 + lhi));
      SV_SB;
      acc[g][2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc[g], xc[2], acc[g][2], 0, 0, 0);
      SV_SB;
      if (do_dma) dma(dstage, d0 + 2 * g);
      SV_SB;
      acc[g][3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc[g], xc[3], acc[g][3], 0, 0, 0);
      SV_SB;
      if (do_dma) dma(dstage, d0 + 2 * g + 1);
      SV_SB;
    }
  };

  if (!d_valid) return;
  bf16x8 xf0[MI], wf0[NI], xf1[MI], wf1[NI];
  set_segment();
#pragma unroll
  for (int j = 0; j < 16; ++j) dma(0, j);                     // slice 0 of the first tile
  advance();
  int par = 0;                                                // LDS stage of the current tile's slice 0

  int m0, n0;
  for (int vb = blockIdx.x; tile_of(vb, m0, n0); vb += gridDim.x) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < MI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // ---- what the epilogue's global accesses need, set up here because a full tile asks for its first inputs a slice early.
    // In the read-back of the epilogue a lane serves row er of each group of 4 rows, 16-byte chunk ec4 (and 16 + ec4).
    // One buffer descriptor per tensor, based at the tile's first row and the wave's first column; inside it a lane's
    // byte offset is (row * ld + column) * 2, of which the lane's part never changes and the row block's part is a scalar:
    // no 64-bit address arithmetic per access.
    constexpr bool kHasInputs = EPI == EPI_RESID || EPI == EPI_SWIGLU_BWD || EPI == EPI_GELU_BWD || EPI == EPI_ROPE;
    constexpr int PD = kEpiAhead<EPI>;                   // trips the epilogue's global reads run ahead of its stores
    const int er = lane >> 4, ec4 = lane & 15;
    const int ncol0 = n0 + wn * (DUAL ? 64 : 128);
    auto desc = [&](const void* base, int ld) {
      return __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16*)base + (int64_t)m0 * ld + ncol0), (short)0, -1, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t bC = desc(a.C, a.ldc), bC2 = desc(a.C2, a.ldc), bC3 = desc(a.C3, a.ldc);
    const __amdgpu_buffer_rsrc_t bR = desc(a.R, a.ldr), bR2 = desc(a.R2, a.ldr);
    const int vC = ((wm * 128 + er) * a.ldc + ec4 * 4) * 2, vR = ((wm * 128 + er) * a.ldr + ec4 * 4) * 2;
    // offsets of row block rb (rows rb .. rb + 3 of the wave's 128): per lane (vo) and scalar (so).  A ragged tile
    // re-reads its last row for the rows past the end, which takes the row into the lane's part.
    auto place = [&](auto check_tag, int rb, int ld, int vlane, int& vo, int& so) {
      if (decltype(check_tag)::value) { vo = (min(wm * 128 + rb + er, M - 1 - m0) * ld + ec4 * 4) * 2; so = 0; }
      else { vo = vlane; so = rb * ld * 2; }
    };
    int rope_p0 = 0, rope_v_lo = 0, rope_v_hi = 0;      // first row's position; byte offsets of the lane's feature pairs in a table row
    if (EPI == EPI_ROPE) {
      rope_p0 = (m0 + wm * 128) % a.rope_S;
      rope_v_lo = (((ncol0 + ec4 * 4) % a.rope_hd) >> 1) * 8;
      rope_v_hi = (((ncol0 + 64 + ec4 * 4) % a.rope_hd) >> 1) * 8 - rope_v_lo;
    }
    const __amdgpu_buffer_rsrc_t bT = __builtin_amdgcn_make_buffer_rsrc((void*)a.rope_cs, (short)0, -1, 0x00020000);
    auto ld8 = [&](__amdgpu_buffer_rsrc_t b, int vo, int so) { return __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(b, vo, so, 0)); };
    // the inputs of trip `trip` (two rows of row block mi = trip / 4 per lane): residual, gate / up, RoPE table
    auto load_inputs = [&](auto check_tag, int trip, EpiIn (&lo)[2], EpiIn (&hi)[2]) {
      const int mi = trip >> 2, it = (trip & 3) * 2;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int rb = mi * 32 + (it + k) * 4;
        if (EPI == EPI_ROPE) {
          // position of the row in its sequence without a division per row: the wave's first row is reduced once
          // per tile, the rows of the tile follow it consecutively
          int p = rope_p0 + rb + er;
          if (a.rope_S >= 256) p -= p >= a.rope_S ? a.rope_S : 0; else p %= a.rope_S;
          const int vo = p * (a.rope_hd >> 1) * 8 + rope_v_lo;      // the table entry (position p, feature pair) is 8 bytes
          lo[k].cs = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bT, vo, 0, 0));
          hi[k].cs = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bT, vo + rope_v_hi, 0, 0));
        } else if (kHasInputs) {
          int vo, so;
          place(check_tag, rb, a.ldr, vR, vo, so);
          lo[k].r = ld8(bR, vo, so);
          hi[k].r = ld8(bR, vo + 128, so);
          if (EPI == EPI_SWIGLU_BWD) { lo[k].r2 = ld8(bR2, vo, so); hi[k].r2 = ld8(bR2, vo + 128, so); }
        }
      }
    };
    EpiIn in_lo[PD][2], in_hi[PD][2];                    // [trip mod PD][row of the pair]
    const bool full_tile = m0 + 256 <= M;
    auto first_inputs = [&]() {                          // of a full tile, a slice before the epilogue
      if (kHasInputs && full_tile) {
#pragma unroll
        for (int t = 0; t < PD; ++t) load_inputs(std::false_type{}, t, in_lo[t], in_hi[t]);
      }
    };
    // ---- slice 0 (its loads were issued during the previous tile's last slice, or above)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    SV_SB;
    // the row factors of the wave's 128 rows are asked for here, a whole k loop before the epilogue wants them (its
    // first loads would otherwise start with a memory round trip per tile); the next wait for memory is a slice away
    float rs_pre0 = 1.0f, rs_pre1 = 1.0f;
    if (RS) {
      rs_pre0 = a.rscale[min(m0 + wm * 128 + lane, M - 1)];
      rs_pre1 = a.rscale[min(m0 + wm * 128 + 64 + lane, M - 1)];
    }
    if (nslices == 1) first_inputs();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      xf0[g] = *reinterpret_cast<const bf16x8*>(smem + par * STAGE + lds_off(xrow[g], lhi));
      wf0[g] = *reinterpret_cast<const bf16x8*>(smem + par * STAGE + BM * 128 + lds_off(wrow[g], lhi));
    }
    step(xf0, wf0, xf1, wf1, true, par, 1, true, par ^ 1, 0);
    step(xf1, wf1, xf0, wf0, true, par, 2, true, par ^ 1, 8);
    if (d_valid) advance();
    step(xf0, wf0, xf1, wf1, true, par, 3, false, 0, 0);
    for (int kt = 1; kt < nslices; ++kt) {
      const int st = (par + kt) & 1;
      __builtin_amdgcn_s_waitcnt(0);   // my DMAs of slice kt have landed, my fragment reads of slice kt-1 are done
      __syncthreads();                 // ... and so have everybody's: stage st is complete, stage st^1 is free
      SV_SB;
      if (kt == nslices - 1) first_inputs();     // their round trip hides behind the last slice's products
      SV_SB;
      step(xf1, wf1, xf0, wf0, true, st, 0, true, st ^ 1, 0);     // MFMAs of (kt-1, k step 3)
      step(xf0, wf0, xf1, wf1, true, st, 1, true, st ^ 1, 8);
      if (d_valid) advance();
      step(xf1, wf1, xf0, wf0, true, st, 2, false, 0, 0);
      step(xf0, wf0, xf1, wf1, true, st, 3, false, 0, 0);
    }
    step(xf1, wf1, xf0, wf0, false, 0, 0, false, 0, 0);

    // ---- epilogue through LDS (the next tile's slice 0 is landing in the other stage meanwhile).
    // In the accumulator layout a lane owns one token row and scattered groups of 4 features, so a
    // store instruction would touch 32 rows with 16 bytes each; the memory pipeline then takes ~11 us
    // per tile.  Each wave instead writes its 32 x 128 fp32 block into its own 16 KB patch of the
    // stage that was just consumed (16-byte chunks XOR-swizzled by the row: conflict-free both ways)
    // and reads it back so that 16 consecutive lanes cover 128 contiguous bytes of an output row;
    // every global access of the epilogue (result, residual, gate / up) becomes a full-line run.
    const int sl = (par + nslices - 1) & 1;
    par = (par + nslices) & 1;
    __syncthreads();                                   // everybody is done reading stage sl
    char* patch = smem + sl * STAGE + wave * 16384;
    // per wave, behind the two stages: the row factors of its 128 rows (each lane of the read-back needs those of the
    // rows it serves) and the rows' sums of squares (stored in one piece when the tile is done)
    float* rsbuf = reinterpret_cast<float*>(smem + 2 * STAGE) + wave * 256;
    float* sqbuf = rsbuf + 128;
    if (RS) { rsbuf[lane] = rs_pre0; rsbuf[64 + lane] = rs_pre1; }
    // Sixteen trips per tile: row block mi = trip / 4, two rows per lane and trip.  The epilogue's global reads (residual,
    // gate / up, RoPE table) run kEpiAhead trips ahead of its stores; the first of them were asked for when the last slice
    // began.  (The memory counter retires in order: a read is waited for together with every store issued before it, so
    // the reads of a trip are issued before the stores they must not wait for have piled up.)  Tiles that lie
    // inside the M rows run without any per-lane condition (CHECK = false): around divergent branches the compiler's
    // wait insertion falls back to waiting for (nearly) everything in flight, one memory round trip per store.
    auto run_epilogue = [&](auto check_tag) {
      constexpr bool CHECK = decltype(check_tag)::value;
      if constexpr (DUAL) {
        if (!a.C2 && !a.C3) {
          // Forward-only check (no stash of g and u).  Gate and up of one feature sit in the same lane and register
          // index, so SiLU(g) * u is taken in the accumulator layout and only its bf16 result goes through the patch:
          // 128 token rows x 64 features x 2 bytes = the 16 KB patch in one piece (16-byte chunks XOR-swizzled by bits
          // 1..3 of the row), a quarter of the fp32 way's LDS traffic, and the read-back gives every lane 16 bytes of a
          // row, so 8 lanes store one full 128-byte line.  (With the stashes, three such passes measured slower than
          // the fp32 way below, which serves them.)
          // The lane's row and chunk numbers are made opaque once per tile: otherwise every address below is loop
          // invariant, gets hoisted out of the tile loop and spilled, and its reloads cost a memory round trip each.
          int r31 = l31, rhi = lhi, ln = lane;
          asm volatile("" : "+v"(r31), "+v"(rhi), "+v"(ln));
          // The accumulators are read where they are, in the accumulation registers, by an instruction the compiler
          // cannot merge with the reads of the other way: left to it, it keeps copies of whole accumulator blocks in
          // ordinary registers from one use to the next and spills them.  The matrix pipe's last write is long
          // finished (a workgroup barrier lies in between); the wait states make that formal, since the compiler's
          // own hazard handling does not look into assembly.
          float rsv[MI];
          if (RS) { __builtin_amdgcn_s_waitcnt(0xc07f); __builtin_amdgcn_wave_barrier(); }   // the factors are in LDS
#pragma unroll
          for (int mi = 0; mi < MI; ++mi) rsv[mi] = RS ? rsbuf[mi * 32 + r31] : 1.0f;
          asm volatile("s_nop 15\n\ts_nop 15");
          auto rd = [&](int ni, int mi, int r) {
            float x;
            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[ni][mi][r]));
            return x;
          };
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                bf16x4 pk;
#pragma unroll
                for (int i = 0; i < 4; ++i) pk[i] = (bf16)(silu_f(rd(ni, mi, q * 4 + i) * rsv[mi]) * (rd(ni + 2, mi, q * 4 + i) * rsv[mi]));
                const int row = mi * 32 + r31;
                *reinterpret_cast<bf16x4*>(patch + row * 128 + (((ni * 4 + q) ^ ((r31 >> 1) & 7)) << 4) + rhi * 8) = pk;
                if (q == 3) SV_SB;                       // one feature block at a time
              }
          __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0): the patch is complete before it is read back
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int it = 0; it < 16; ++it) {
            const int row = it * 8 + (ln >> 3), cc = ln & 7;
            const bf16x8 v = *reinterpret_cast<const bf16x8*>(patch + row * 128 + ((cc ^ ((row >> 1) & 7)) << 4));
            const int m = m0 + wm * 128 + row;
            if (CHECK && m >= M) continue;
            *reinterpret_cast<bf16x8*>((bf16*)a.C + (int64_t)m * a.ldc + n0 + wn * 64 + cc * 8) = v;
            if ((it & 3) == 3) SV_SB;
          }
          return;
        }
      }
      // The lane's row and chunk numbers in the patch are made opaque once per tile, as above: the patch addresses below
      // are the same for every tile, and kept in registers across the k loop they crowd the epilogue's inputs out.
      int e31 = l31, eer = er, ec = ec4;
      asm volatile("" : "+v"(e31), "+v"(eer), "+v"(ec));
      if (kHasInputs && CHECK) {                         // a ragged tile asks for its first inputs here, a full one did so a slice ago
#pragma unroll
        for (int t = 0; t < PD; ++t) load_inputs(check_tag, t, in_lo[t], in_hi[t]);
      }
#pragma unroll
      for (int trip = 0; trip < 16; ++trip) {
        const int mi = trip >> 2, it = (trip & 3) * 2;
        if ((trip & 3) == 0) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              f32x4 v;
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = acc[ni][mi][q * 4 + i];
              const int chunk = ni * 8 + q * 2 + lhi;    // features 4*chunk .. +3 of the wave's 128
              *reinterpret_cast<f32x4*>(patch + e31 * 512 + ((chunk ^ e31) << 4)) = v;
            }
          __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0): the patch is complete before it is read back
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int row = (it + k) * 4 + eer, rb = mi * 32 + (it + k) * 4;
          const f32x4 a_lo = *reinterpret_cast<const f32x4*>(patch + row * 512 + ((ec ^ row) << 4));
          const f32x4 a_hi = *reinterpret_cast<const f32x4*>(patch + row * 512 + (((16 + ec) ^ row) << 4));
          float lo[4], hi[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) { lo[i] = a_lo[i]; hi[i] = a_hi[i]; }
          const bool ok = !CHECK || wm * 128 + rb + er < M - m0;
          int vo, so;
          place(check_tag, rb, a.ldc, vC, vo, so);
          auto put_lo = [&](int w, bf16x4 pk) {
            if (ok) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, pk), w == 0 ? bC : w == 1 ? bC2 : bC3, vo, so, 0);
          };
          auto put_hi = [&](int w, bf16x4 pk) {
            if (ok) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, pk), w == 0 ? bC : w == 1 ? bC2 : bC3, vo + 128, so, 0);
          };
          const float rs = RS ? rsbuf[mi * 32 + row] : 1.0f;
          const EpiIn& i_lo = in_lo[trip % PD][k];
          const EpiIn& i_hi = in_hi[trip % PD][k];
          if (DUAL) epilogue_math4<EPI>(a, false, lo, hi, i_lo, rs, put_lo);   // patch columns 0..63: gate, 64..127: up
          else {
            float sq = epilogue_math4<EPI>(a, EPI == EPI_ROPE && ncol0 + ec4 * 4 < a.rope_cols, lo, hi, i_lo, rs, put_lo);
            sq += epilogue_math4<EPI>(a, EPI == EPI_ROPE && ncol0 + 64 + ec4 * 4 < a.rope_cols, hi, lo, i_hi, rs, put_hi);
            if (SQ) {
              // the 16 lanes of a row hold its 128 stored values: rotate-and-add within the row of 16 lanes leaves the
              // sum in all of them, and all of them write it (one LDS address per row, no per-lane condition)
              sq += dpp_row_ror<8>(sq); sq += dpp_row_ror<4>(sq); sq += dpp_row_ror<2>(sq); sq += dpp_row_ror<1>(sq);
              if (ok) sqbuf[mi * 32 + row] = sq;
            }
          }
        }
        if (kHasInputs && trip + PD < 16) load_inputs(check_tag, trip + PD, in_lo[trip % PD], in_hi[trip % PD]);
      }
      if (SQ) {                                          // 128 consecutive floats of plane (n0 / 128 + wn): two full-line stores
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_wave_barrier();
        float* plane = a.rowsq + (int64_t)((n0 >> 7) + wn) * a.rowsq_ld + m0 + wm * 128;
        if (!CHECK || m0 + wm * 128 + lane < M) plane[lane] = sqbuf[lane];
        if (!CHECK || m0 + wm * 128 + 64 + lane < M) plane[64 + lane] = sqbuf[64 + lane];
      }
    };
    if (m0 + 256 <= M) run_epilogue(std::false_type{});
    else run_epilogue(std::true_type{});
  }
  // A finished stream keeps re-reading its last slice into the free stage (the loop has no branch for it): every
  // such load must have landed before the workgroup gives its LDS back.
  __builtin_amdgcn_s_waitcnt(0);
#undef SV_SB
}

// ------------------------------------------------------------------------------------------
// Direct-to-LDS kernel on smaller tiles: (WM * 32 * MI) x (WN * 32 * NI) outputs per workgroup of WM x WN waves, NST LDS
// stages of one 64-deep slice each.  It serves what the 256x256 kernel cannot fill the chip with (fewer than about one
// tile per CU) and widths that are no multiple of 256: any multiple of 8 columns -- weight rows past the end re-read the
// last group of 8, outputs past the end (rows and columns) are dropped by the bounds check of the buffer stores.
//
// What bounds it: LDS.  A 128x128 tile moves 32 KB into LDS (64 B/clk) and 64 KB out of it (about 200 B/clk) per slice
// of 512 matrix cycles, so a CU is busy with LDS about 1.5 x as long as with MFMAs; the 256x256 tile (0.75 x) stays the
// better one wherever it fills the chip.  NST: the loads of slice k + NST - 1 are issued when slice k is multiplied.  As many
// stages as a CU's 160 KB hold for one workgroup (256x128: 3, 128x128: 4, 64x64: 8), since a CU has about one tile where these
// serve; 64x128 takes 3, and its 72 KB let two workgroups share a CU.  (128x128 with two stages and two workgroups on a CU,
// each under the other's wait for memory, measured slower than one with four.)
//
// The one wait + barrier per slice stands before the last of its four 16-wide k steps, whose fragments are in registers
// by then: behind it the first fragments of the next slice are asked for, and the step's MFMAs hide their latency.
template <int WM, int WN, int MI, int NI, int NST, bool DUAL>
struct MidCfg {
  static constexpr int NW = WM * WN, NT = 64 * NW, BM = WM * 32 * MI, BN = WN * 32 * NI, NOUT = DUAL ? BN / 2 : BN;
  static constexpr int STAGE = (BM + BN) * 128, LDS = NST * STAGE;
  static constexpr int NA = BM / 8 / NW, NB = BN / 8 / NW, ND = NA + NB;      // 1 KB loads per wave and slice
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && (!DUAL || NI % 2 == 0), "tile shape");
  static_assert(NW * 32 * NI * 32 * 4 <= LDS, "the epilogue's patches fit the stages");
  static_assert(ND * (NST - 2) < 64, "the wait count has 6 bits");
};

//
// SPLIT: a tile's k slices are dealt to nsplit workgroups in contiguous runs, each leaves its fp32 partial product in
// a.split_ws[run][M][N] and splitk_reduce_kernel adds the runs in order.  SUMMED: the same sum of runs (GemmArgs::runs) in one
// workgroup, the running total beside the accumulators: bit for bit what the partial products and their reduction give.
// TAIL: the last round of a product on 256x256 tiles (GemmArgs::tail).
template <int WM, int WN, int MI, int NI, int NST, int EPI, bool GROUPED, bool SPLIT, bool SUMMED, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_mid_kernel(GemmArgs a, int tiles_m, int tiles_n, int nsplit) {
  constexpr bool DUAL = EPI == EPI_SWIGLU;
  static_assert(!SPLIT || (EPI == EPI_STORE && !GROUPED), "a split run stores bare partial products");
  static_assert(!SUMMED || (!DUAL && !GROUPED && !SPLIT), "one sum of runs per output");
  using C = MidCfg<WM, WN, MI, NI, NST, DUAL>;
  constexpr int BM = C::BM, BN = C::BN, STAGE = C::STAGE, NW = C::NW, NA = C::NA, NB = C::NB;
  constexpr int kGroup = 1024 / BM;                       // row tiles per raster group: 1024 rows, as on the large tile
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int M = GROUPED ? *a.m_dev : a.M;
  if (GROUPED) tiles_m = (M + BM - 1) / BM;
  // tile assignment as in the 256x256 kernel: ids congruent mod 8 (one XCD) walk a contiguous run of tiles.  As that kernel's last
  // round: its map and its tiles, each in SUB pieces next to each other.
  constexpr int SUBN = 256 / BN, SUB = 256 / BM * SUBN;
  static_assert(!TAIL || (!SPLIT && !SUMMED), "a tail's tiles are whole");
  int group = kGroup, skip = 0, sub = 0, slot = blockIdx.x >> 3;
  if (TAIL) {
    int slices = 0;
    for (int s = 0; s < a.nseg; ++s) slices += a.seg[s].K / BK;
    tiles_m = (M + 255) / 256; tiles_n = a.N / (DUAL ? 128 : 256);
    const int all = (tiles_m * tiles_n + 7) >> 3, rem = tail_tiles(all, a.tail, slices);
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

  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave % WM, wn = wave / WM;

  // ---- the stream of slices: segment dseg, offset dk
  int dseg = 0, dk = 0, d_K = 0, left;
  int nsl = 0;
  for (int s = 0; s < a.nseg; ++s) nsl += a.seg[s].K / BK;
  left = nsl;
  if (SPLIT) {                                            // run r takes the slices [r * nsl / nsplit, (r + 1) * nsl / nsplit)
    const int ks = (int)((int64_t)run * nsl / nsplit);
    nsl = (int)((int64_t)(run + 1) * nsl / nsplit) - ks;
    left = nsl;
    int k = ks * BK;
    while (k >= a.seg[dseg].K) { k -= a.seg[dseg].K; ++dseg; }
    dk = k;
  }
  const bf16* pA;
  const bf16* pB[NB];                                     // first row of the panel; of each group of 8 weight rows
  unsigned voffA[NA], voffB[NB];
  auto set_segment = [&]() {
    const GemmSeg& sg = a.seg[dseg];
    d_K = sg.K;
    pA = (const bf16*)sg.A + (int64_t)m0 * sg.lda;
    const int64_t goff = GROUPED ? (int64_t)a.tile_group[m0 >> 8] * a.group_stride : 0;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int r = (wave + NW * i) * 8 + (lane >> 3), c = (lane & 7) ^ swz(r);
      voffA[i] = (unsigned)((int64_t)min(r, M - 1 - m0) * sg.lda + c * 8) * 2u;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int g = (wave + NW * i) * 8, r = g + (lane >> 3), c = (lane & 7) ^ swz(r);
      const bf16* B = (const bf16*)sg.B + goff;
      int64_t ldb = sg.ldb;
      int row;                                            // the group's first weight row
      if (DUAL) {
        const bool up = g >= BN / 2;
        if (up) { B = (const bf16*)a.B2 + goff; ldb = a.ldb2; }
        row = min(n0 + (up ? g - BN / 2 : g), a.N - 8);
      } else {
        row = min(n0 + g, a.N - 8);
        if ((EPI == EPI_STORE || EPI == EPI_ROPE) && a.nbcol > 0) {
          const int o1 = a.ncol[0], o2 = o1 + a.ncol[1];
          if (a.nbcol > 2 && row >= o2) { B = (const bf16*)a.Bcol[2]; row -= o2; }
          else if (a.nbcol > 1 && row >= o1) { B = (const bf16*)a.Bcol[1]; row -= o1; }
          else B = (const bf16*)a.Bcol[0];
        }
      }
      pB[i] = B + (int64_t)row * ldb;
      voffB[i] = (unsigned)((int64_t)(lane >> 3) * ldb + c * 8) * 2u;
    }
  };
  auto dma = [&](int stage, int j) {                      // j: the wave's NA activation groups, then its NB weight groups
    const int i = j < NA ? j : j - NA;
    char* dst = smem + stage * STAGE + (j < NA ? 0 : BM * 128) + (wave + NW * i) * 1024;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(j < NA ? pA : pB[j < NA ? 0 : i]), (short)0, -1, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16,
                                             (int)(j < NA ? voffA[j < NA ? i : 0] : voffB[j < NA ? 0 : i]), dk * 2, 0, 0);
  };
  auto advance = [&]() {                                  // to the next slice; past the last one the stream re-reads it
    if (--left <= 0) return;
    dk += BK;
    if (dk < d_K) return;
    dk = 0; ++dseg; set_segment();
  };

  // ---- the epilogue's places.  Each wave turns its accumulators over 32 rows at a time through an LDS patch of its own and
  // reads them back so that LPR consecutive lanes hold one row's outputs (4 per lane), RPI rows per instruction.
  constexpr bool kHasInputs = EPI == EPI_RESID || EPI == EPI_SWIGLU_BWD || EPI == EPI_GELU_BWD || EPI == EPI_ROPE;
  constexpr int LPR = DUAL ? NI * 4 : NI * 8, RPI = 64 / LPR, TR = 32 / RPI;
  const int er = lane / LPR, ec = lane % LPR;
  const int mw = wm * 32 * MI, n = n0 + wn * (DUAL ? NI * 16 : NI * 32) + ec * 4;    // the lane's first row (+ er) and columns n .. n + 3
  const int rows = min(M - m0, BM);
  // rows past M lie past the descriptor's end, columns past N are sent there
  auto desc = [&](const void* base, int64_t ld, int es) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (int64_t)m0 * ld * es), (short)0, (int)(rows * ld * es), 0x00020000);
  };
  const unsigned vcol = n < a.N ? (unsigned)n : SPLIT ? 0x20000000u : 0x40000000u;     // byte offset 2^31: past every descriptor's end
  const bool rscaled = kEpiScaled<EPI> && !GROUPED && !SPLIT && a.rscale;
  EpiIn in[2][TR];
  float rs[2][TR];
  int rope_p0 = 0, rope_i0 = 0;
  if (EPI == EPI_ROPE) { rope_p0 = (m0 + mw) % a.rope_S; rope_i0 = (n % a.rope_hd) >> 1; }
  auto load_inputs = [&](int mi, EpiIn (&e)[TR], float (&f)[TR]) {
    if (kHasInputs) {
      const __amdgpu_buffer_rsrc_t bR = desc(a.R, a.ldr, 2), bR2 = desc(a.R2, a.ldr, 2);
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        const int r = mw + mi * 32 + t * RPI + er;
        if (EPI == EPI_ROPE) {
          int p = rope_p0 + mi * 32 + t * RPI + er;
          if (a.rope_S >= BM) p -= p >= a.rope_S ? a.rope_S : 0; else p %= a.rope_S;
          e[t].cs = *reinterpret_cast<const f32x4*>(a.rope_cs + ((int64_t)p * (a.rope_hd >> 1) + rope_i0) * 2);
        } else {
          const unsigned vo = ((unsigned)(r * (int)a.ldr) + vcol) * 2u;
          e[t].r = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(bR, (int)vo, 0, 0));
          if (EPI == EPI_SWIGLU_BWD) e[t].r2 = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(bR2, (int)vo, 0, 0));
        }
      }
    }
    if (kEpiScaled<EPI>) {
#pragma unroll
      for (int t = 0; t < TR; ++t) f[t] = 1.0f;
      if (rscaled) {
#pragma unroll
        for (int t = 0; t < TR; ++t) f[t] = a.rscale[min(m0 + mw + mi * 32 + t * RPI + er, M - 1)];
      }
    }
  };

  f32x16 acc[NI][MI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // ---- fragment addresses: row 32 b + (lane & 31) of a tile, chunk 2 kk + lhi.  The swizzle sees a 32-row block only by
  // its parity, which turns chunk 2 kk into 2 (kk ^ 2): one base per k step and operand, block offsets are immediates.
  const int bx = wm * MI, bw = wn * (DUAL ? NI / 2 : NI);
  unsigned offX[4], offW[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    offX[kk] = (unsigned)(bx * 4096 + lds_off(l31, (kk * 2 + lhi) ^ ((bx & 1) << 2)));
    offW[kk] = (unsigned)(BM * 128 + bw * 4096 + lds_off(l31, (kk * 2 + lhi) ^ ((bw & 1) << 2)));
  }
  constexpr int kUp = DUAL ? BN / 64 - NI / 2 : 0;         // from the block after the last gate block to the first up block
  auto read = [&](const char* base, int kk, bf16x8 (&x)[MI], bf16x8 (&w)[NI]) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int b = DUAL && ni >= NI / 2 ? ni + kUp : ni;
      w[ni] = *reinterpret_cast<const bf16x8*>(base + offW[kk ^ ((b & 1) << 1)] + b * 4096);
    }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) x[mi] = *reinterpret_cast<const bf16x8*>(base + offX[kk ^ ((mi & 1) << 1)] + mi * 4096);
  };
#define SV_SB __builtin_amdgcn_sched_barrier(0)
  constexpr int kLgkm0 = 0xc07f;                           // lgkmcnt(0), nothing else
  constexpr int kLandedCnt = C::ND * (NST - 2);            // loads that may still be in flight when the next slice has landed
  constexpr int kLanded = 0x0070 | (kLandedCnt & 15) | ((kLandedCnt >> 4) << 14);      // vmcnt(kLandedCnt) lgkmcnt(0)
  // this wave's wait, then the workgroup's barrier
#define SV_MEET(imm) do { SV_SB; __builtin_amdgcn_s_waitcnt(imm); asm volatile("s_barrier" ::: "memory"); SV_SB; } while (0)
  auto mul = [&](bf16x8 (&x)[MI], bf16x8 (&w)[NI]) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[ni], x[mi], acc[ni][mi], 0, 0, 0);
  };

  if (!SPLIT) load_inputs(0, in[0], rs[0]);                // older than every slice: in order, so landed when the first has
  SV_SB;
  set_segment();
#pragma unroll
  for (int s = 0; s + 1 < NST; ++s) {
#pragma unroll
    for (int j = 0; j < C::ND; ++j) dma(s, j);
    advance();
  }
  bf16x8 x0[MI], w0[NI], x1[MI], w1[NI];
  f32x16 tot[SUMMED ? NI : 1][SUMMED ? MI : 1];
  int run_end = nsl, runs = 1, run_i = 0;                  // SUMMED: the run being summed ends before slice run_end
  if (SUMMED) {
    int j = 0, c = n0;
    while (j + 1 < a.nbcol && c >= a.ncol[j]) { c -= a.ncol[j]; ++j; }
    runs = a.runs[j];
    run_end = nsl / runs;
  }
  SV_MEET(kLanded);
  read(smem, 0, x0, w0);
  int st = 0;
  for (int kt = 0; kt < nsl; ++kt) {
    const char* base = smem + st * STAGE;
    const int fill = st == 0 ? NST - 1 : st - 1;           // the stage slice kt - 1 has left
    st = st + 1 == NST ? 0 : st + 1;
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    SV_SB;
    read(base, 1, x1, w1);
    SV_SB;
#pragma unroll
    for (int j = 0; j < C::ND; ++j) {                      // the next loads, one behind each MFMA
      if (j < MI * NI) acc[j / MI][j % MI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[j / MI], x0[j % MI], acc[j / MI][j % MI], 0, 0, 0);
      SV_SB;
      dma(fill, j);
      SV_SB;
      if (j + 1 == MI * NI) {
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        SV_SB;
        read(base, 2, x0, w0);
        SV_SB;
      }
      if (j >= MI * NI && j < 2 * MI * NI) {
        const int i = j - MI * NI;
        acc[i / MI][i % MI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[i / MI], x1[i % MI], acc[i / MI][i % MI], 0, 0, 0);
        SV_SB;
      }
    }
#pragma unroll
    for (int i = C::ND; i < MI * NI; ++i) acc[i / MI][i % MI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[i / MI], x0[i % MI], acc[i / MI][i % MI], 0, 0, 0);
    if (C::ND < MI * NI) {
      __builtin_amdgcn_s_waitcnt(kLgkm0);
      SV_SB;
      read(base, 2, x0, w0);
      SV_SB;
    }
#pragma unroll
    for (int i = C::ND > MI * NI ? C::ND - MI * NI : 0; i < MI * NI; ++i)
      acc[i / MI][i % MI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[i / MI], x1[i % MI], acc[i / MI][i % MI], 0, 0, 0);
    advance();
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    SV_SB;
    read(base, 3, x1, w1);
    SV_SB;
    mul(x0, w0);
    SV_SB;
    SV_MEET(kLanded);                                         // everybody's loads of slice kt + 1 have landed, their reads of slice kt are done
    read(smem + st * STAGE, 0, x0, w0);                    // past the last slice: a stage nobody needs
    SV_SB;
    mul(x1, w1);
    SV_SB;
    if constexpr (SUMMED) {
      if (kt + 1 == run_end) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              tot[ni][mi][r] = run_i == 0 ? acc[ni][mi][r] : tot[ni][mi][r] + acc[ni][mi][r];
              acc[ni][mi][r] = 0.0f;
            }
        ++run_i;
        run_end = (int)((int64_t)(run_i + 1) * nsl / runs);
      }
    }
  }
  SV_MEET(0);                                                 // the re-read slices too: the stages become the patches

  // ---- epilogue
  char* patch = smem + wave * (32 * NI * 128);
  const __amdgpu_buffer_rsrc_t bC = SPLIT ? desc(a.split_ws + (int64_t)run * M * a.N, a.N, 4) : desc(a.C, a.ldc, 2);
  const __amdgpu_buffer_rsrc_t bC2 = desc(a.C2, a.ldc, 2), bC3 = desc(a.C3, a.ldc, 2);
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    constexpr int kMask = NI * 8 - 1;
    if (!SPLIT && mi + 1 < MI) load_inputs(mi + 1, in[(mi + 1) & 1], rs[(mi + 1) & 1]);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = SUMMED ? tot[SUMMED ? ni : 0][SUMMED ? mi : 0][q * 4 + i] : acc[ni][mi][q * 4 + i];
        *reinterpret_cast<f32x4*>(patch + l31 * (NI * 128) + (((ni * 8 + q * 2 + lhi) ^ (l31 & kMask)) << 4)) = v;
      }
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    __builtin_amdgcn_wave_barrier();
    f32x4 va[TR], vu[TR];
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const int row = t * RPI + er;
      va[t] = *reinterpret_cast<const f32x4*>(patch + row * (NI * 128) + ((ec ^ (row & kMask)) << 4));
      if (DUAL) vu[t] = *reinterpret_cast<const f32x4*>(patch + row * (NI * 128) + (((ec + NI * 4) ^ (row & kMask)) << 4));
    }
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const int r = mw + mi * 32 + t * RPI + er;
      if (SPLIT) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, va[t]), bC, (int)(((unsigned)(r * a.N) + vcol) * 4u), 0, 0);
        continue;
      }
      float v[4], u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[i] = va[t][i]; u[i] = DUAL ? vu[t][i] : 0.0f; }
      const unsigned vo = ((unsigned)(r * (int)a.ldc) + vcol) * 2u;
      epilogue_math4<EPI>(a, EPI == EPI_ROPE && n < a.rope_cols, v, u, in[mi & 1][t], kEpiScaled<EPI> ? rs[mi & 1][t] : 1.0f, [&](int w, bf16x4 p) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, p), w == 0 ? bC : w == 1 ? bC2 : bC3, (int)vo, 0, 0);
      });
    }
    __builtin_amdgcn_wave_barrier();                       // the reads of this block are issued before the next block's writes
  }
#undef SV_MEET
#undef SV_SB
}

template <int WM, int WN, int MI, int NI, int NST, int EPI, bool GROUPED, bool SPLIT = false, bool SUMMED = false, bool TAIL = false>
hipError_t launch_mid(const GemmArgs& a, int nsplit, hipStream_t st, int tail_max = 0) {      // tail_max: tiles per XCD a tail has at most
  using C = MidCfg<WM, WN, MI, NI, NST, EPI == EPI_SWIGLU>;
  auto kern = gemm_mid_kernel<WM, WN, MI, NI, NST, EPI, GROUPED, SPLIT, SUMMED, TAIL>;
  static bool configured = false;   // per process; the attribute is per function
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (a.M + C::BM - 1) / C::BM, tiles_n = (a.N + C::NOUT - 1) / C::NOUT;
  const int64_t per_xcd = TAIL ? (int64_t)tail_max * (256 / C::BM) * (256 / C::BN) : ((int64_t)tiles_m * tiles_n * nsplit + 7) / 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(C::NT), C::LDS, st, a, tiles_m, tiles_n, nsplit);
  return hipGetLastError();
}

template <int EPI, bool GROUPED, bool NF = false>
hipError_t launch_dma(const GemmArgs& a, hipStream_t st) {
  auto kern = gemm_mfma_dma_kernel<EPI, GROUPED, NF>;
  constexpr int lds = 2 * 512 * 128 + 4 * 1024;           // two stages, and per wave 128 row factors + 128 row sums
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (a.M + 255) / 256, tiles_n = a.N / (EPI == EPI_SWIGLU ? 128 : 256);
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  const int n_cu = std::max(8, cu_count() / 8 * 8);       // one persistent workgroup per CU (128 KB of LDS each)
  const int grid = per_xcd * 8 < n_cu ? per_xcd * 8 : n_cu;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, a, tiles_m, tiles_n);
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
// 512 .. 14336 with every tile forced (within 15 % of the measured times there).  They are those of a plain store: the dearer
// epilogues (SwiGLU with its stashes, SwiGLU-backward) cost the same here, and a tile more than the last full round counts as a
// round (on 256x256 tiles: as a second launch on smaller ones, where tail_tiles says so).  Against 256x256 tiles over runs of k, which these replaced, k of 9000 and more for 500 .. 1500 rows of 3072 .. 4096 columns
// is left 5 .. 15 % slower (1453 x 3072, K = 9728: 97 -> 112 us), everything else even or faster.  Where the lines come out, with both
// sides as measured on that sweep: 4096 x 1024, K = 1024 (256 tiles of 128 x 128) 13.4 us against 19 on 256 x 128 and 33 on
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
  if (256 * a.ldc * 2 >= (int64_t)1 << 31 || 256 * a.ldr * 2 >= (int64_t)1 << 31) return false;   // a tile's outputs by 32-bit byte offsets
  return !(a.epi == EPI_SWIGLU && a.ldc % 8);            // its epilogue stores 16 bytes per lane
}

bool fits_mid(const GemmArgs& a) {        // buffer descriptors over a tile's rows keep below 2^31 bytes
  return 256 * a.ldc * 2 < (int64_t)1 << 31 && 256 * a.ldr * 2 < (int64_t)1 << 31 && (int64_t)256 * a.N * 4 < (int64_t)1 << 31;
}

bool summed_runs(const GemmArgs& a) { return a.runs[0] > 1 || a.runs[1] > 1 || a.runs[2] > 1; }

// The epilogues that form an activation or its derivative are a fifth to a third of a product's time at K = 1024, and a launch of fewer
// 256x256 tiles than CUs does them on part of the chip.  192x256 tiles (eight waves, two stages), while they too are one round, give every
// CU three quarters of a tile.  256x256 -> 192x256, us: GELU 2331 x 3840, K = 960 (150 tiles, 195 of these) 38.1 -> 31.4, its backward
// 37.4 -> 30.9; 4096 x 2560, K = 1024 39.1 -> 33.1; SwiGLU with its stashes 2331 x 1920, K = 960 30.7 -> 25.6, its backward at 3840
// columns 34.9 -> 32.1; 900 x 5120, K = 2048 48.3 -> 43.3; 800 x 6144, K = 3072 68.2 -> 62.6.  With a longer k loop the bare product
// decides: GELU 768 x 16384, K = 4096 104 -> 112.  (Plain stores and residual sums gain 1 - 9 % and stay where they are: what they run
// on is what sv_gemm_plan tells.)
bool narrower_pays(const GemmArgs& a, int slices) {
  if (a.epi != EPI_GELU && a.epi != EPI_GELU_BWD && a.epi != EPI_SWIGLU && a.epi != EPI_SWIGLU_BWD) return false;
  return !a.tile_group && slices <= 48 && fits_mid(a) && (int64_t)((a.M + 191) / 192) * (a.N / (a.epi == EPI_SWIGLU ? 128 : 256)) <= cu_count();
}

// Asked twice for a product that may leave row sums, once to know whether it will (mfma_gemm_emits_rowsq) and once to launch it:
// with a.rowsq set the answer does not depend on the scratch, which only runs of k use.
Plan plan_gemm(const GemmArgs& a) {
  if (summed_runs(a)) return Plan{kTile128, 1};
  const bool dual = a.epi == EPI_SWIGLU;
  int slices = 0;
  for (int s = 0; s < a.nseg; ++s) slices += a.seg[s].K / BK;
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
  if (best.kind == kTile256 && narrower_pays(a, slices)) best.kind = kTile192x256;
  return best;
}

// Tiles per XCD (at most) that a product on 256x256 tiles leaves to a second launch, or 0.  In groups the rows are known on the device
// only: somewhere between none and 255 of padding per group more than the tokens' rows; the second launch (4.5 us where it
// finds nothing to do) is made if half of the likely counts have a tail.
template <int EPI, bool GROUPED>
int tail_pays(const GemmArgs& a) {
  if (a.rowsq || !fits_mid(a)) return 0;                 // row sums come from whole 256 x 256 tiles only
  const int tiles_n = a.N / (EPI == EPI_SWIGLU ? 128 : 256), slots = tile_slots();
  int slices = 0;
  for (int s = 0; s < a.nseg; ++s) slices += a.seg[s].K / BK;
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
        if (GROUPED || 4 * left <= g.tail) return launch_mid<4, 2, 1, 2, 4, EPI, GROUPED, false, false, true>(g, 1, st, left);
        if constexpr (!GROUPED) return launch_mid<4, 2, 2, 2, 3, EPI, false, false, false, true>(g, 1, st, left);
      }
      if constexpr (!GROUPED && EPI != EPI_SWIGLU_BWD && EPI != EPI_GELU_BWD)
        if (a.rscale || a.rowsq) return launch_dma<EPI, false, true>(a, st);   // the ends of a norm that runs inside the products
      return launch_dma<EPI, GROUPED>(a, st);
    }
    case kTile256x128: return launch_mid<4, 2, 2, 2, 3, EPI, GROUPED>(a, 1, st);
    case kTile128: return launch_mid<4, 2, 1, 2, 4, EPI, GROUPED>(a, 1, st);
    case kTile64x128: return launch_mid<2, 2, 1, 2, 3, EPI, GROUPED>(a, 1, st);
    case kTile192x256:
      if constexpr (!GROUPED && (EPI == EPI_GELU || EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_BWD))
        return launch_mid<2, 4, 3, 2, 2, EPI, false>(a, 1, st);
      return hipErrorInvalidValue;
    default:
      if constexpr (EPI != EPI_SWIGLU) return launch_mid<2, 2, 1, 1, 8, EPI, GROUPED>(a, 1, st);
      return hipErrorInvalidValue;
  }
}

// runs of k slices into a.split_ws, then the reduction with the epilogue
template <int EPI>
hipError_t launch_runs(const GemmArgs& a, const Plan& p, hipStream_t st) {
  hipError_t e;
  switch (p.kind) {
    case kTile256x128: e = launch_mid<4, 2, 2, 2, 3, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile128: e = launch_mid<4, 2, 1, 2, 4, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile64x128: e = launch_mid<2, 2, 1, 2, 3, EPI_STORE, false, true>(a, p.runs, st); break;
    case kTile64: e = launch_mid<2, 2, 1, 1, 8, EPI_STORE, false, true>(a, p.runs, st); break;
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
    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID || EPI == EPI_ROPE) return launch_mid<4, 2, 1, 2, 4, EPI, false, false, true>(a, 1, st);
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
    if (a.epi == EPI_ROPE && (!a.rope_cs || a.rope_hd % 4 || a.rope_cols % 4 || a.rope_S < 1)) return false;
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
