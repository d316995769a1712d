// Projection GEMM C[M,N] = A[M,K] * B[N,K]^T on the gfx950 matrix cores:
// bf16 operands, fp32 accumulation (v_mfma_f32_32x32x16_bf16), LDS-staged tiles.
//
// Both operands are K-contiguous, so a lane's MFMA fragment (8 consecutive k of
// one row) is one 16-byte LDS read.  A workgroup of 4 waves owns a 128x128 tile
// of C; each wave owns 64x64 of it as 2x2 MFMA tiles.  K is walked in steps of
// 64 through a double-buffered LDS stage filled by direct-to-LDS global loads
// (global_load_lds_dwordx4), one step ahead of the MFMAs.  16-byte LDS chunks are XOR-swizzled by row/2: a 16-byte
// LDS read is served 16 lanes (256 bytes, all 64 banks) at a time, rows are 128
// bytes, so 16 consecutive rows must spread over (row parity, 8 chunk slots).
//
// Epilogues: store bf16; accumulate into an fp32 residual stream; SwiGLU, where
// the B tile is 64 gate rows and the 64 matching up rows arranged so that one
// lane ends up holding gate and up of the same (row, feature).
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int BM = 128, BN = 128, BK = 64;
constexpr int LDS_TILE = BM * BK;   // elements per operand tile

#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ int lds_off(int row, int chunk) {   // element offset of a 16-byte chunk
  return row * BK + ((chunk ^ ((row >> 1) & 7)) << 3);
}

// fp32 store; in a split-K launch split s stores its partial product to C + s * part_stride.
constexpr int EPI_PARTIAL_F32 = ARB_EPI_STORE_F32;

template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                   void *__restrict__ Cv, int M, int N, int K, int tiles_m,
                                                   int tiles_n, int tile_n0, size_t part_stride) {
  // One array per operand and stage: the compiler orders LDS reads against in-flight direct-to-LDS
  // loads by object, so separate objects let the reads of one stage overlap the loads into the other.
  __shared__ __attribute__((aligned(16))) bf16 As0[LDS_TILE], As1[LDS_TILE], Bs0[LDS_TILE], Bs1[LDS_TILE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  constexpr int TILE_GROUP = 4;
  tile_of<TILE_GROUP>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
  tile_n += tile_n0;                 // this launch covers n-tiles [tile_n0, tile_n0 + tiles_n)
  const int m0 = tile_m * BM;

  // Global source of this thread's four 16-byte chunks per operand.  Tiles are brought in by
  // direct-to-LDS loads: one wave-wide load fills 1 KB of LDS in lane order (8 tile rows of 8
  // chunk slots), so the XOR swizzle is applied on the global side: the lane that owns slot
  // (row, p) fetches logical chunk p ^ swz(row).
  const bf16 *a_src[4], *b_src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + 256 * i, row = c >> 3, chunk = (c & 7) ^ ((row >> 1) & 7);
    int am = m0 + row;
    am = am < M ? am : M - 1;                       // tail rows re-read the last row; never stored
    a_src[i] = A + (size_t)am * K + chunk * 8;
    int bn;
    if (EPI == ARB_EPI_SWIGLU_BF16) {
      // tile-local row r: wave column r/64, MFMA tile (r%64)/32 (0 = gate, 1 = up), feature offset r%32
      const int f = tile_n * 64 + (row >> 6) * 32 + (row & 31);
      bn = ((row >> 5) & 1) ? N + f : f;            // N = F here
    } else {
      bn = tile_n * BN + row;
    }
    b_src[i] = B + (size_t)bn * K + chunk * 8;
  }

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // K range of this workgroup (the whole of K unless the launch is split along K)
  const int nk_all = K / BK;
  const int kt_begin = split_point(nk_all, blockIdx.y, gridDim.y);
  const int nk = split_point(nk_all, blockIdx.y + 1, gridDim.y) - kt_begin;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a_src[i] += (size_t)kt_begin * BK;
    b_src[i] += (size_t)kt_begin * BK;
  }

  // While step kt is multiplied out of LDS buffer kt%2, the loads of step kt+1 stream from global
  // memory straight into the other buffer (no register staging, no LDS-write phase); the barrier
  // that ends the step also waits for them.
  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto dma = [&](int buf, int kt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int slot = (i * 4 + wave_u) * 512;      // 1 KB (8 rows) per wave-wide load
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(a_src[i] + (size_t)kt * BK), LDS_PTR((buf ? As1 : As0) + slot), 16, 0, 0);
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(b_src[i] + (size_t)kt * BK), LDS_PTR((buf ? Bs1 : Bs0) + slot), 16, 0, 0);
    }
  };
  // MFMAs of one K-step; the LDS reads of sub-step kk+1 are issued before the MFMAs of kk.
  auto compute = [&](int buf) {
    bf16x8 fa[2][2], fb[2][2];
    auto frags = [&](int slot, int kk) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[slot][i] = *(const bf16x8 *)&(buf ? As1 : As0)[lds_off(wm * 64 + i * 32 + frag_row, kk * 2 + frag_half)];
        fb[slot][i] = *(const bf16x8 *)&(buf ? Bs1 : Bs0)[lds_off(wn * 64 + i * 32 + frag_row, kk * 2 + frag_half)];
      }
    };
    frags(0, 0);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      if (kk + 1 < BK / 16) frags((kk + 1) & 1, kk + 1);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][i], fb[kk & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // The loop body is branch-free (loads past the end are clamped to the last step; their copy is
  // never read).
  const int last = nk - 1;
  dma(0, 0);
  __syncthreads();
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    dma(1, kt + 1);
    __builtin_amdgcn_sched_barrier(0);      // keep the loads ahead of the MFMAs they overlap with
    compute(0);
    __syncthreads();
    dma(0, min(kt + 2, last));
    __builtin_amdgcn_sched_barrier(0);
    compute(1);
    __syncthreads();
  }
  if (kt < nk) compute(0);     // odd number of steps: the last one sits in buffer 0

  // D layout of the 32x32 MFMA: lane holds column lane%32 and rows 8*(r/4) + 4*(lane/32) + r%4.
  if (EPI == ARB_EPI_SWIGLU_BF16) {
    bf16 *C = (bf16 *)Cv;
    const int col = tile_n * 64 + wn * 32 + frag_row;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * 64 + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
        if (m < M) {
          const float gte = acc[i][0][r], up = acc[i][1][r];
          C[(size_t)m * N + col] = (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = tile_n * BN + wn * 64 + j * 32 + frag_row;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + wm * 64 + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
          if (m < M) {
            if (EPI == ARB_EPI_STORE_BF16) {
              ((bf16 *)Cv)[(size_t)m * N + col] = (bf16)acc[i][j][r];
            } else if (EPI == EPI_PARTIAL_F32) {
              ((float *)Cv)[blockIdx.y * part_stride + (size_t)m * N + col] = acc[i][j][r];
            } else {
              float *dst = (float *)Cv + (size_t)m * N + col;
              *dst += acc[i][j][r];
            }
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Deep-ring kernel for launches of at most one workgroup per CU (narrow projections, remainders,
// split-K launches sized to one round).  Such a launch is bound by what a CU can pull in: it only has
// the loads of its one workgroup in flight, and its one address unit handles a half-used cache line
// like a whole one.  So K is walked in steps of 64 (every row piece is a whole 128-byte line) through
// a ring of LDS stages that fills the CU's LDS: all stages but one are loading or loaded ahead of the
// one being multiplied out.  (Steps of 32 with twice the stages keep the same bytes in flight but
// move half lines: QKV 17.5 -> 14.5 us on the 1.5B shape with steps of 64.)
// MI = 32-row MFMA tiles per wave along M: 2 gives the 128x128 tile (4 stages), 1 a 64x128 tile
// (6 stages) for launches that would otherwise leave more than half of the CUs without a workgroup,
// 4 a 256x128 tile (3 stages) for launches that are one well-filled round of such tiles.
// NT_B: the weights are loaded non-temporal, for launches of a single m-tile, where every weight is used once (8B
// gate/up at 33 rows 50.3 -> 46.6 us); with several m-tiles they meet in L2 and have to stay there.
#ifndef ARB_RING_K
#define ARB_RING_K 64
#endif
constexpr int RK = ARB_RING_K;                      // K per stage: 64 makes every row piece a whole 128-byte line
constexpr int ring_stages(int mi) { return RK == 32 ? 8 : (mi == 1 ? 6 : mi == 2 ? 4 : 3); }   // 144, 128, 144 KB for K 64

__device__ __forceinline__ int lds_off32(int row, int chunk) {   // element offset of a 16-byte chunk, 64-byte rows
  return row * 32 + ((chunk ^ ((row >> 2) & 3)) << 3);
}

__device__ __forceinline__ int lds_off_ring(int row, int chunk) {   // element offset of a 16-byte chunk in a stage row
  // 16 lanes read 16 consecutive rows of one chunk: 64-byte rows put 4 rows into 256 bytes (swizzle by row/4),
  // 128-byte rows 2 (swizzle by row/2)
  return RK == 32 ? row * 32 + ((chunk ^ ((row >> 2) & 3)) << 3) : row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3);
}

// s_waitcnt immediates (vmcnt in bits 3:0 and 15:14, lgkmcnt in 11:8, expcnt 6:4 left at "no wait")
constexpr int waitcnt_vm_lgkm0(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70; }
constexpr int waitcnt_vm(int vm) { return waitcnt_vm_lgkm0(vm) | 0xF00; }       // lgkmcnt at "no wait" too

template <int EPI, int MI, bool NT_B = false>
__global__ __launch_bounds__(256, 1) void gemm_ring_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                   void *__restrict__ Cv, int M, int N, int K, int tiles_m,
                                                   int tiles_n, int tile_n0, size_t part_stride) {
  constexpr int RBM = 64 * MI;                              // rows of the tile
  constexpr int RING_STAGES = ring_stages(MI);
  constexpr int RING_STAGE_ELEMS = (RBM + BN) * RK;         // A rows then B rows
  constexpr int CPR = RK / 8, RPL = 64 / CPR;               // 16-byte chunks per stage row; rows per wave-wide load
  constexpr int A_LOADS = RBM / (4 * RPL), B_LOADS = BN / (4 * RPL);   // wave-wide loads per wave and step
  constexpr int LOADS = A_LOADS + B_LOADS;
  constexpr int NS = RK / 16;                               // MFMA sub-steps per stage
  constexpr int UNUSED = 8;
  // one array per stage (the compiler orders LDS reads against in-flight loads by object)
  __shared__ __attribute__((aligned(16))) bf16 St0[RING_STAGE_ELEMS], St1[RING_STAGE_ELEMS], St2[RING_STAGE_ELEMS],
      St3[RING_STAGES > 3 ? RING_STAGE_ELEMS : UNUSED], St4[RING_STAGES > 4 ? RING_STAGE_ELEMS : UNUSED], St5[RING_STAGES > 5 ? RING_STAGE_ELEMS : UNUSED],
      St6[RING_STAGES > 6 ? RING_STAGE_ELEMS : UNUSED], St7[RING_STAGES > 7 ? RING_STAGE_ELEMS : UNUSED];
  static_assert(RING_STAGES >= 3 && RING_STAGES <= 8, "stage arrays");
#define ARB_ST(s) ((s) == 0 ? St0 : (s) == 1 ? St1 : (s) == 2 ? St2 : (s) == 3 ? St3 : (s) == 4 ? St4 : (s) == 5 ? St5 : (s) == 6 ? St6 : St7)

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  constexpr int TILE_GROUP = 512 / RBM;            // 512 rows
  tile_of<TILE_GROUP>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
  tile_n += tile_n0;                 // this launch covers n-tiles [tile_n0, tile_n0 + tiles_n)
  const int m0 = tile_m * RBM;

  // This thread's 16-byte chunks per step: tile rows row0 + 4 RPL i of A (i < A_LOADS) and of B (i < B_LOADS),
  // the same chunk for all (the swizzle term of a row does not change when 4 RPL is added to it).
  const int row0 = tid / CPR;
  const int chunk = (tid % CPR) ^ (RK == 32 ? ((row0 >> 2) & 3) : ((row0 >> 1) & 7));
  const bf16 *a_src[A_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) {
    int am = m0 + row0 + 4 * RPL * i;
    am = am < M ? am : M - 1;                       // tail rows re-read the last row; never stored
    a_src[i] = A + (size_t)am * K + chunk * 8;
  }
  // B rows.  For SwiGLU the tile-local row r maps to wave column r/64, MFMA tile (r%64)/32 (0 = gate, 1 = up) and
  // feature offset r%32, i.e. feature tile_n*64 + (r/64)*32 + r%32 of the gate or up half; N = F there.
  const bf16 *b_src[B_LOADS];
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) {
    const int r = row0 + 4 * RPL * i;
    const int brow = EPI == ARB_EPI_SWIGLU_BF16 ? tile_n * 64 + (r >> 6) * 32 + (r & 31) + ((r >> 5) & 1) * N : tile_n * BN + r;
    b_src[i] = B + (size_t)brow * K + chunk * 8;
  }

  f32x16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // K range of this workgroup (the whole of K unless the launch is split along K)
  const int nk_all = K / RK;
  const int kt_begin = split_point(nk_all, blockIdx.y, gridDim.y);
  const int nk = split_point(nk_all, blockIdx.y + 1, gridDim.y) - kt_begin, last = nk - 1;
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) a_src[i] += (size_t)kt_begin * RK;
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) b_src[i] += (size_t)kt_begin * RK;

  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto dma_a = [&](int s, int kt) {
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(a_src[i] + (size_t)kt * RK), LDS_PTR(ARB_ST(s) + (i * 4 + wave_u) * 512), 16, 0, 0);
  };
  auto dma_b = [&](int s, int kt) {
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(b_src[i] + (size_t)kt * RK), LDS_PTR(ARB_ST(s) + RBM * RK + (i * 4 + wave_u) * 512), 16, 0, NT_B ? 2 : 0);
  };
  // The swizzle term of a fragment row depends on frag_row only, so each operand needs one LDS offset
  // per sub-step; MFMA tile and stage are constant displacements from it.
  int a_off[NS], b_off[NS];
#pragma unroll
  for (int kk = 0; kk < NS; ++kk) {
    a_off[kk] = lds_off_ring(wm * 32 * MI + frag_row, 2 * kk + frag_half);
    b_off[kk] = RBM * RK + lds_off_ring(wn * 64 + frag_row, 2 * kk + frag_half);
  }
  bf16x8 fa[2][MI], fb[2][2];
  auto frags = [&](int slot, int s, int kk) {
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[slot][i] = *(const bf16x8 *)&ARB_ST(s)[a_off[kk] + i * 32 * RK];
#pragma unroll
    for (int j = 0; j < 2; ++j) fb[slot][j] = *(const bf16x8 *)&ARB_ST(s)[b_off[kk] + j * 32 * RK];
  };
  auto mfmas = [&](int slot) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][i], fb[slot][j], acc[i][j], 0, 0, 0);
  };
  // Step out of stage s (NS sub-steps of 2 MI MFMAs); on entry fragment slot 0 holds its first sub-step.
  // `refill` is the step loaded into the stage before s, which every wave left at the previous barrier
  // (clamped to the last step past the end; those copies are never read).  Before the barrier this
  // wave's reads of stage s have returned and its loads of the next step have landed: they are the
  // oldest of its loads in flight, the LOADS * (RING_STAGES - 3) + A_LOADS issued since may stay in flight.  (A full
  // workgroup fence would wait for all of them.)
  auto step = [&](int s, int refill) {
    const int prev = (s + RING_STAGES - 1) % RING_STAGES, next = (s + 1) % RING_STAGES;
#pragma unroll
    for (int kk = 0; kk + 1 < NS; ++kk) {
      frags((kk + 1) & 1, s, kk + 1);
      if (kk == 0) dma_a(prev, refill);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(kk & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(LOADS * (RING_STAGES - 3) + A_LOADS));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frags(0, next, 0);
    dma_b(prev, refill);
    __builtin_amdgcn_sched_barrier(0);
    mfmas(1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // The same without a refill, for the steps after the last whole turn of the ring: nothing is loaded
  // any more, so the wait is for everything still in flight.
  auto drain_step = [&](int s) {
#pragma unroll
    for (int kk = 0; kk + 1 < NS; ++kk) {
      frags((kk + 1) & 1, s, kk + 1);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(kk & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frags(0, (s + 1) % RING_STAGES, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfmas(1);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int s = 0; s < RING_STAGES - 1; ++s) {
    dma_a(s, min(s, last));
    dma_b(s, min(s, last));
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(LOADS * (RING_STAGES - 2)));   // step 0 has landed
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  frags(0, 0, 0);
  // Whole turns of the ring in a branch-free body, then the 0..RING_STAGES-1 steps that are left.
  int kt = 0;
  for (; kt + RING_STAGES <= nk; kt += RING_STAGES) {
#pragma unroll
    for (int s = 0; s < RING_STAGES; ++s) step(s, min(kt + s + RING_STAGES - 1, last));
  }
  const int rem = nk - kt;
#pragma unroll
  for (int s = 0; s < RING_STAGES - 1; ++s)
    if (s < rem) drain_step(s);
#undef ARB_ST

  // D layout of the 32x32 MFMA: lane holds column lane%32 and rows 8*(r/4) + 4*(lane/32) + r%4.
  if (EPI == ARB_EPI_SWIGLU_BF16) {
    bf16 *C = (bf16 *)Cv;
    const int col = tile_n * 64 + wn * 32 + frag_row;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * 32 * MI + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
        if (m < M) {
          const float gte = acc[i][0][r], up = acc[i][1][r];
          C[(size_t)m * N + col] = (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = tile_n * BN + wn * 64 + j * 32 + frag_row;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + wm * 32 * MI + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
          if (m < M) {
            if (EPI == ARB_EPI_STORE_BF16) {
              ((bf16 *)Cv)[(size_t)m * N + col] = (bf16)acc[i][j][r];
            } else if (EPI == EPI_PARTIAL_F32) {
              ((float *)Cv)[blockIdx.y * part_stride + (size_t)m * N + col] = acc[i][j][r];
            } else {
              float *dst = (float *)Cv + (size_t)m * N + col;
              *dst += acc[i][j][r];
            }
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Large-tile variant for launches that fill the chip with 256x256 tiles.  Global->LDS traffic
// per flop halves against the 128x128 tile (a CU's vector-memory path moves ~50-60 bytes/clock,
// which caps the small tile at about half the MFMA rate), and a fragment read (1 KB per wave)
// serves more MFMAs: 4 waves, one per SIMD, each own 128x128 of the tile as 4x4 MFMA tiles (8
// fragment reads per 16 MFMAs), the 256 accumulator registers in the AGPR half of the wave's 512.
//
// With one wave per SIMD nothing else covers a stall, so every kind of instruction is spread
// evenly through the MFMA stream.  K is walked in steps of 32 through four LDS stages (128 KB):
// while step k is multiplied out of stage k%4, the loads of step k+3 stream into the stage that
// step k-1 has just left, one load per four MFMAs, so the vector-memory path never sees a burst
// and a load has three steps to land.  Per step there are two sub-steps of 16 MFMAs; the fragments
// of the next sub-step are read between the MFMAs of the current one.  The barrier of a step sits
// before its second sub-step: past it every wave is done reading the previous stage and the next
// stage has landed.  LDS rows are 64 bytes here, so the 16-byte chunks are swizzled by row/4.
constexpr int LM = 256, LN = 256, LK = 32;
constexpr int L_TILE = LM * LK;          // elements per operand and stage


// B is the K-blocked copy of the weights, [K/32][rows][32] (arb_pack_k_blocked): the 16 rows of a wave-wide load of one
// K step are then 1 KB of consecutive memory, whole cache lines, instead of 16 half lines.  Launches without such a
// copy go to the eight-wave kernel below; where there is one, this kernel is still the better one on few token rows
// (gate/up 1024x2x8192x1536 in 256 tiles 47.4 us against 50.6, 512x2x16384x4096 112 against 119) and within 3 % on many.
template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm256_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                         void *__restrict__ Cv, int M, int N, int K, int tiles_m,
                                                         int tiles_n) {
  // one array per operand and stage (the compiler orders LDS reads against in-flight loads by object)
  __shared__ __attribute__((aligned(16))) bf16 As0[L_TILE], As1[L_TILE], As2[L_TILE], As3[L_TILE];
  __shared__ __attribute__((aligned(16))) bf16 Bs0[L_TILE], Bs1[L_TILE], Bs2[L_TILE], Bs3[L_TILE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  constexpr int TILE_GROUP = 4;
  tile_of<TILE_GROUP>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * LM;

  // This thread's four 16-byte chunks per operand and step: tile rows tid/4 + 64 i, and the same
  // chunk for every i (the swizzle term (row/4)%4 does not depend on i).  One wave-wide load fills
  // 1 KB of LDS in lane order, i.e. 16 rows of 4 chunk slots.
  const int row0 = tid >> 2, chunk = (tid & 3) ^ ((row0 >> 2) & 3);
  const bf16 *a_src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int am = m0 + row0 + 64 * i;
    am = am < M ? am : M - 1;                       // tail rows re-read the last row; never stored
    a_src[i] = A + (size_t)am * K + chunk * 8;
  }
  // B rows of chunk i are b_row0 + i * b_rows_per_i.  For SwiGLU the tile-local row r maps to wave column
  // r/128, MFMA tile (r%128)/32 (even = gate, odd = up) and feature offset r%32, i.e. feature
  // tile_n*128 + (r/64)*32 + r%32 of the gate (r/32 even) or up (odd) half; N = F there.
  const int b_row0 = EPI == ARB_EPI_SWIGLU_BF16 ? tile_n * 128 + (row0 & 31) + ((row0 >> 5) & 1) * N : tile_n * LN + row0;
  const size_t b_rows = EPI == ARB_EPI_SWIGLU_BF16 ? 2 * (size_t)N : (size_t)N;      // rows of the weight matrix
  const size_t b_row_pitch = 32, b_k_pitch = b_rows * 32;                               // elements between rows, K steps
  const size_t b_step = (size_t)(EPI == ARB_EPI_SWIGLU_BF16 ? 32 : 64) * b_row_pitch;
  const bf16 *b_src = B + (size_t)b_row0 * b_row_pitch + chunk * 8;

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = K / LK, last = nk - 1;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
#define ARB_STAGE(base, s) ((s) == 0 ? base##0 : (s) == 1 ? base##1 : (s) == 2 ? base##2 : base##3)
  auto dma_a = [&](int s, int kt) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(a_src[i] + (size_t)kt * LK), LDS_PTR(ARB_STAGE(As, s) + (i * 4 + wave_u) * 512), 16, 0, 0);
  };
  auto dma_b = [&](int s, int kt) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(b_src + i * b_step + (size_t)kt * b_k_pitch), LDS_PTR(ARB_STAGE(Bs, s) + (i * 4 + wave_u) * 512), 16, 0, 0);
  };
  bf16x8 fa[2][4], fb[2][4];
  // Fragment reads in the order the MFMAs (row-major over the 4x4 tiles) first need them.
  // The swizzle term of a fragment row depends on frag_row only, so each operand needs one LDS
  // offset per sub-step; MFMA tile and stage are constant displacements from it.
  const int a_off[2] = {lds_off32(wm * 128 + frag_row, frag_half), lds_off32(wm * 128 + frag_row, 2 + frag_half)};
  const int b_off[2] = {lds_off32(wn * 128 + frag_row, frag_half), lds_off32(wn * 128 + frag_row, 2 + frag_half)};
  auto frags = [&](int slot, int s, int kk) {
    auto rd_a = [&](int i) { fa[slot][i] = *(const bf16x8 *)&ARB_STAGE(As, s)[a_off[kk] + i * 32 * LK]; };
    auto rd_b = [&](int j) { fb[slot][j] = *(const bf16x8 *)&ARB_STAGE(Bs, s)[b_off[kk] + j * 32 * LK]; };
    rd_a(0); rd_b(0); rd_b(1); rd_b(2); rd_b(3); rd_a(1); rd_a(2); rd_a(3);
  };
  auto mfmas = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][i], fb[slot][j], acc[i][j], 0, 0, 0);
  };
  // 16 MFMAs with at most one other memory instruction between two of them: 8 fragment reads and 4
  // global->LDS loads behind the first twelve, so the reads have returned by the end of the sub-step
  auto spread = [&]() {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // 1 LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // 1 global->LDS load
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Step out of stage s; on entry fragment slot 0 holds its first sub-step.  `refill` is the step
  // loaded into the stage before s (clamped to the last step past the end; those copies are never read).
  auto step = [&](int s, int refill) {
    const int prev = (s + 3) & 3, next = (s + 1) & 3;
    frags(1, s, 1);
    dma_a(prev, refill);
    mfmas(0);
    spread();
    // Hand-over of the stages.  Before the barrier this wave's reads of stage s have returned
    // (lgkmcnt 0) and its loads of the next step have landed: those are the oldest 8 of its loads in
    // flight, the 12 issued since may stay in flight (vmcnt 12).  A full workgroup fence would wait
    // for all of them.
    __builtin_amdgcn_s_waitcnt(0x007C);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frags(0, next, 0);
    dma_b(prev, refill);
    mfmas(1);
    spread();
  };

  dma_a(0, 0); dma_b(0, 0);
  dma_a(1, min(1, last)); dma_b(1, min(1, last));
  dma_a(2, min(2, last)); dma_b(2, min(2, last));
  __builtin_amdgcn_s_waitcnt(0x4070);       // vmcnt(16) lgkmcnt(0): step 0 has landed, steps 1 and 2 may be in flight
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  frags(0, 0, 0);
  int kt = 0;
  for (; kt + 4 <= nk; kt += 4) {
    step(0, min(kt + 3, last));
    step(1, min(kt + 4, last));
    step(2, min(kt + 5, last));
    step(3, min(kt + 6, last));
  }
  if (kt < nk) {                              // K is a multiple of 64, so two steps are left
    step(0, last);
    step(1, last);
  }
#undef ARB_STAGE

  if (EPI == ARB_EPI_SWIGLU_BF16) {
    // A lane holds single elements of 128 rows: stored from registers they would leave in 2-byte
    // pieces (128 stores per lane through the address unit).  The wave's 128 x 64 block goes through
    // the LDS instead (the stages are free now, 16 KB per wave) and leaves in 16-byte pieces of whole
    // 128-byte rows.  The 16-byte chunks of a row are swizzled by bit 2 of the row so that the two
    // lane halves, four rows apart, write different banks.
    bf16 *C = (bf16 *)Cv;
    __syncthreads();                      // every wave is done reading the last stage
    bf16 *stage = wave_u == 0 ? As0 : wave_u == 1 ? As1 : wave_u == 2 ? As2 : As3;
#pragma unroll
    for (int jp = 0; jp < 2; ++jp)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3), f = jp * 32 + frag_row;
          const float gte = acc[i][2 * jp][r], up = acc[i][2 * jp + 1][r];
          stage[row * 64 + ((((f >> 3) ^ (((row >> 2) & 1) << 2))) << 3) + (f & 7)] =
              (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
        }
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const int row = it * 8 + (lane >> 3), chunk = lane & 7;
      const bf16x8 v = *(const bf16x8 *)&stage[row * 64 + ((chunk ^ (((row >> 2) & 1) << 2)) << 3)];
      const int m = m0 + wm * 128 + row;
      if (m < M) *(bf16x8 *)(C + (size_t)m * N + tile_n * 128 + wn * 64 + chunk * 8) = v;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = tile_n * LN + wn * 128 + j * 32 + frag_row;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + wm * 128 + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
          if (m < M) {
            if (EPI == ARB_EPI_STORE_BF16) {
              ((bf16 *)Cv)[(size_t)m * N + col] = (bf16)acc[i][j][r];
            } else if (EPI == ARB_EPI_STORE_F32) {
              ((float *)Cv)[(size_t)m * N + col] = acc[i][j][r];
            } else {
              float *dst = (float *)Cv + (size_t)m * N + col;
              *dst += acc[i][j][r];
            }
          }
        }
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Eight-wave large-tile kernel: the 256x256 tile of row-major operands with two waves per SIMD, so that one wave's
// MFMAs cover the other's LDS reads, barriers and epilogue.  A wave owns 128x64 of the tile as 4x2 MFMA tiles.  K is
// walked in steps of 64 (every row piece is a whole 128-byte line, which the 32-wide steps of the kernel above only
// get from a K-blocked copy) through two LDS stages of four regions: the upper and lower half of every wave's rows
// (A0, A1) and the two 32-column groups of every wave's columns (B0, B1), 16 KB each.
//
// A step is four phases of 8 MFMAs per wave: A0 B0, A0 B1, A1 B1, A1 B0.  A fragment register is read again
// as soon as its last MFMA has been issued (A1 over A0 in the second phase, the next step's A0 and B0 over A1 and
// B0 in the fourth), so the fragments need 64 registers beside the 128 accumulators and two waves fit a SIMD.  A
// region is free once every wave has consumed its fragments, one phase after the phase that reads it; the loads of
// step t+2 go there at once, six phases (1.5 steps, 96 KB in flight) before they are read.  One barrier per phase hands
// regions over in both directions: behind it every wave's share of the region read next has landed (counted vmcnt) and every
// wave is done with the region refilled next.  Fragment reads and their waits are inline assembly: left to the
// compiler, every read would wait for all direct-to-LDS loads in flight.
//
// The rate of a full chip is set by its clock under this load, not by the schedule: with K = 14336, 256 tiles run at
// 1.25 to 1.34 PFLOP/s (1.6 us per step of 64), 192 at 1.1 to 1.14 (1.4 us), 128 at 0.9 (1.17 us), so three quarters of a
// round are 85 % as fast as a whole one, and a launch of 144 tiles already beats smaller tiles that fill the chip.  Measured (before: 128x128
// tiles): down 8208x1536x8960 193 us (262), O 8208x1536x1536 44 (55), down 3001x4096x14336 293 (407), QKV
// 2048x6144x4096 89 (125).
constexpr int W_TM = 256, W_TN = 256;                    // tile
constexpr int W_REGION = 128 * 64;                        // elements of a region

template <int OFF>
__device__ __forceinline__ void wide_request_a(unsigned addr, bf16x8 &f0, bf16x8 &f1) {       // two MFMA tiles, 32 rows apart
  asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4"
               : "=&v"(f0), "=&v"(f1)
               : "v"(addr), "n"(OFF), "n"(OFF + 32 * 64 * 2)
               : "memory");
}
template <int OFF>
__device__ __forceinline__ void wide_request_b(unsigned addr, bf16x8 &f) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(f) : "v"(addr), "n"(OFF) : "memory");
}
// at most N of this wave's LDS reads are outstanding; naming the fragments keeps their MFMAs behind the wait
template <int N>
__device__ __forceinline__ void wide_await(bf16x8 &f0, bf16x8 &f1, bf16x8 &f2) {
  asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(f0), "+v"(f1), "+v"(f2) : "n"(N) : "memory");
}

template <int EPI>
__global__ __launch_bounds__(512, 2) void gemm_wide_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                           void *__restrict__ Cv, int M, int N, int K, int tiles_m,
                                                           int tiles_n, size_t part_stride) {
  __shared__ __attribute__((aligned(1024))) bf16 Regions[8 * W_REGION];    // A [stage][half], then B [stage][group]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  int tile_m, tile_n;
  tile_of<4>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * W_TM;

  // K range of this workgroup (the whole of K unless the launch is split along K)
  const int nk_all = K / 64;
  const int kt_begin = split_point(nk_all, blockIdx.y, gridDim.y);
  const int nk = split_point(nk_all, blockIdx.y + 1, gridDim.y) - kt_begin, last = nk - 1;

  // This wave brings rows [16 wave, 16 wave + 16) of every region, 8 rows of 128 bytes per wave-wide load; the
  // 16-byte chunks of a row are swizzled by row/2 on the global side.  Region row r of A half h is tile row
  // (r/64) 128 + 64 h + r%64; region row r of B group j is column (r/32) 64 + 32 j + r%32 of the tile, or for SwiGLU
  // feature 32 (r/32) + r%32 of the tile's 128, its gate (j = 0) or up (j = 1) row.
  constexpr bool SWIGLU = EPI == ARB_EPI_SWIGLU_BF16;
  const size_t k_bytes = (size_t)K * 2;
  const char *a_base = (const char *)A + (size_t)m0 * k_bytes + (size_t)kt_begin * 128;
  const char *b_base = (const char *)B + (size_t)tile_n * (SWIGLU ? 128 : W_TN) * k_bytes + (size_t)kt_begin * 128;
  unsigned a_off[2][2], b_off[2];                         // byte offsets from the tile's first row, < 256 rows
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = wave * 16 + i * 8 + (lane >> 3);
    const unsigned chunk = (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int row = (r >> 6) * 128 + h * 64 + (r & 63);
      row = row < M - m0 ? row : M - 1 - m0;              // tail rows re-read the last row; never stored
      a_off[h][i] = (unsigned)(row * k_bytes) + chunk;
    }
    b_off[i] = (unsigned)((SWIGLU ? r : (r >> 5) * 64 + (r & 31)) * k_bytes) + chunk;
  }
  const size_t b_group = (size_t)(SWIGLU ? N : 32) * k_bytes;         // from group 0 to group 1
  auto load_a = [&](int s, int h, int kt) {               // steps past the end: the last one again, never multiplied
    const char *src = a_base + (size_t)(kt < last ? kt : last) * 128;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src + a_off[h][i]), LDS_PTR(Regions + (2 * s + h) * W_REGION + (wave * 2 + i) * 512), 16, 0, 0);
  };
  auto load_b = [&](int s, int j, int kt) {
    const char *src = b_base + (size_t)(kt < last ? kt : last) * 128 + (j ? b_group : 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src + b_off[i]), LDS_PTR(Regions + (4 + 2 * s + j) * W_REGION + (wave * 2 + i) * 512), 16, 0, 0);
  };

  f32x16 acc[2][2][2];                                    // [A half][32-row tile][B group]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[h][i][j][r] = 0.f;

  // LDS byte addresses of this lane's fragments of MFMA step kk in stage 0, half / group 0
  const int frag_row = lane & 31, frag_half = lane >> 5;
  unsigned a_addr[4], b_addr[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const unsigned o = (unsigned)(uintptr_t)LDS_PTR(Regions) + 2u * (frag_row * 64 + (((2 * kk + frag_half) ^ ((frag_row >> 1) & 7)) << 3));
    a_addr[kk] = o + 2u * (wm * 64 * 64);
    b_addr[kk] = o + 2u * (4 * W_REGION + wn * 32 * 64);
  }
  bf16x8 fa[2][4], fb[2][4];
  auto products = [&](auto h_, auto j_, int kk) {
    constexpr int h = decltype(h_)::value, j = decltype(j_)::value;
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[h][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][kk], fb[j][kk], acc[h][i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  using std::integral_constant;
  constexpr integral_constant<int, 0> zero{};
  constexpr integral_constant<int, 1> one{};
  constexpr int RB = W_REGION * 2;                        // bytes of a region
  // The counted waits: 12 reads (A0, B0) are outstanding on entry of phase 0, 4 (B1) of phase 1, 8 (A1) of phase 2.
  auto phase0 = [&](auto s_) {                            // A0 B0; reads B1
    constexpr int S = decltype(s_)::value, OFF = (2 * S + 1) * RB;
    __builtin_amdgcn_sched_barrier(0);
    wide_await<9>(fa[0][0], fa[1][0], fb[0][0]); products(zero, zero, 0); wide_request_b<OFF>(b_addr[0], fb[1][0]);
    wide_await<7>(fa[0][1], fa[1][1], fb[0][1]); products(zero, zero, 1); wide_request_b<OFF>(b_addr[1], fb[1][1]);
    wide_await<5>(fa[0][2], fa[1][2], fb[0][2]); products(zero, zero, 2); wide_request_b<OFF>(b_addr[2], fb[1][2]);
    wide_await<3>(fa[0][3], fa[1][3], fb[0][3]); products(zero, zero, 3); wide_request_b<OFF>(b_addr[3], fb[1][3]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto phase1 = [&](auto s_) {                            // A0 B1; reads A1 over A0
    constexpr int S = decltype(s_)::value, OFF = (2 * S + 1) * RB;
    __builtin_amdgcn_sched_barrier(0);
    wide_await<3>(fa[0][0], fa[1][0], fb[1][0]); products(zero, one, 0); wide_request_a<OFF>(a_addr[0], fa[0][0], fa[1][0]);
    wide_await<4>(fa[0][1], fa[1][1], fb[1][1]); products(zero, one, 1); wide_request_a<OFF>(a_addr[1], fa[0][1], fa[1][1]);
    wide_await<5>(fa[0][2], fa[1][2], fb[1][2]); products(zero, one, 2); wide_request_a<OFF>(a_addr[2], fa[0][2], fa[1][2]);
    wide_await<6>(fa[0][3], fa[1][3], fb[1][3]); products(zero, one, 3); wide_request_a<OFF>(a_addr[3], fa[0][3], fa[1][3]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto phase2 = [&]() {                                   // A1 B1
    __builtin_amdgcn_sched_barrier(0);
    wide_await<6>(fa[0][0], fa[1][0], fb[1][0]); products(one, one, 0);
    wide_await<4>(fa[0][1], fa[1][1], fb[1][1]); products(one, one, 1);
    wide_await<2>(fa[0][2], fa[1][2], fb[1][2]); products(one, one, 2);
    wide_await<0>(fa[0][3], fa[1][3], fb[1][3]); products(one, one, 3);
  };
  auto phase3 = [&](auto s_) {                            // A1 B0; reads the next step's A0 and B0 (stage s_) over them
    constexpr int S = decltype(s_)::value, OFF = 2 * S * RB;
    __builtin_amdgcn_sched_barrier(0);
    products(one, zero, 0); wide_request_a<OFF>(a_addr[0], fa[0][0], fa[1][0]); wide_request_b<OFF>(b_addr[0], fb[0][0]);
    products(one, zero, 1); wide_request_a<OFF>(a_addr[1], fa[0][1], fa[1][1]); wide_request_b<OFF>(b_addr[1], fb[0][1]);
    products(one, zero, 2); wide_request_a<OFF>(a_addr[2], fa[0][2], fa[1][2]); wide_request_b<OFF>(b_addr[2], fb[0][2]);
    products(one, zero, 3); wide_request_a<OFF>(a_addr[3], fa[0][3], fa[1][3]); wide_request_b<OFF>(b_addr[3], fb[0][3]);
    __builtin_amdgcn_sched_barrier(0);
  };
#define ARB_HANDOVER(vm)                               \
  do {                                                 \
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(vm));        \
    __builtin_amdgcn_s_barrier();                      \
    __builtin_amdgcn_sched_barrier(0);                 \
  } while (0)
  // Step t out of stage s.  A region is two loads of this wave.  At the end of phase 0 A1(t) has landed (behind it the four
  // regions of t+1), of phase 2 A0 and B0 of t+1 (behind: B1 A1 of t+1 and A0 B0 B1 of t+2), of phase 3 B1 of t+1
  // (behind: A1 of t+1 and the four regions of t+2).
  auto step = [&](auto s_, int t) {
    constexpr int S = decltype(s_)::value;
    phase0(s_);
    ARB_HANDOVER(8);
    load_a(S, 0, t + 2);
    load_b(S, 0, t + 2);
    phase1(s_);
    ARB_HANDOVER(63);                                     // nothing new is read in phase 2
    load_b(S, 1, t + 2);
    phase2();
    ARB_HANDOVER(10);
    load_a(S, 1, t + 2);
    phase3(integral_constant<int, S ^ 1>{});
    ARB_HANDOVER(10);
  };
#pragma unroll
  for (int s = 0; s < 2; ++s) {                           // in the order the waits count
    load_a(s, 0, s); load_b(s, 0, s);
    __builtin_amdgcn_sched_barrier(0);
    load_b(s, 1, s);
    __builtin_amdgcn_sched_barrier(0);
    load_a(s, 1, s);
    __builtin_amdgcn_sched_barrier(0);
  }
  ARB_HANDOVER(12);                                       // A0 and B0 of step 0
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    wide_request_a<0>(a_addr[kk], fa[0][kk], fa[1][kk]);
    wide_request_b<0>(b_addr[kk], fb[0][kk]);
  }
  ARB_HANDOVER(10);                                       // B1 of step 0
  int t = 0;
  for (; t + 2 < nk; t += 2) {
    step(zero, t);
    step(one, t + 1);
  }
  // One or two steps are left, and both stages hold what they need: nothing more is requested, so less may be in flight.
  // (With an odd number of steps the loop's last loads were clamped repeats.)
  phase0(zero);
  ARB_HANDOVER(8);
  phase1(zero);
  phase2();
  if (t + 1 < nk) {
    ARB_HANDOVER(4);
    phase3(one);
    ARB_HANDOVER(2);
    phase0(one);
    ARB_HANDOVER(0);
    phase1(one);
    phase2();
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) products(one, zero, kk);
#undef ARB_HANDOVER
  // every fragment read has returned and every load has landed, in all waves, before the LDS is written again
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  __syncthreads();

  // D layout of the 32x32 MFMA: lane holds column lane%32 and rows 8*(r/4) + 4*(lane/32) + r%4.
  if (SWIGLU) {
    // through the LDS, 8 KB per wave, to leave in 16-byte pieces of 64-byte rows (a lane's own elements are 2-byte
    // pieces of 64 rows); chunks are swizzled by row/4 so that the lane halves write different banks
    bf16 *C = (bf16 *)Cv, *stage = Regions + wave * 4096;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = h * 64 + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
          const float gte = acc[h][i][0][r], up = acc[h][i][1][r];
          stage[row * 32 + (((frag_row >> 3) ^ ((row >> 2) & 3)) << 3) + (frag_row & 7)] =
              (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
        }
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int row = it * 16 + (lane >> 2), chunk = lane & 3;
      const bf16x8 v = *(const bf16x8 *)&stage[row * 32 + ((chunk ^ ((row >> 2) & 3)) << 3)];
      const int m = m0 + wm * 128 + row;
      if (m < M) *(bf16x8 *)(C + (size_t)m * N + tile_n * 128 + wn * 32 + chunk * 8) = v;
    }
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int col = tile_n * W_TN + wn * 64 + j * 32 + frag_row;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm * 128 + h * 64 + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
            if (m < M) {
              if (EPI == ARB_EPI_STORE_BF16) {
                ((bf16 *)Cv)[(size_t)m * N + col] = (bf16)acc[h][i][j][r];
              } else if (EPI == EPI_PARTIAL_F32) {
                ((float *)Cv)[blockIdx.y * part_stride + (size_t)m * N + col] = acc[h][i][j][r];
              } else {
                float *dst = (float *)Cv + (size_t)m * N + col;
                *dst += acc[h][i][j][r];
              }
            }
          }
        }
  }
}

// ---------------------------------------------------------------------------------------------
// Up to 64 token rows beyond the few that the weight-streaming kernel takes (a short step of one sequence): 64 rows by 64
// weight rows per workgroup.  Such a launch streams the weights once and is bound by how evenly and how deeply the CUs
// pull them in; with 128 weight rows per workgroup the projections of the 1.5B shape left half of the CUs idle
// (QKV, O and down 72 to 96 workgroups, gate/up 140).  K is walked in steps of 64 through a ring of D stages of 16 KB,
// direct-to-LDS, weights non-temporal; five stages let two workgroups share a CU, nine fill it with one.  A wave multiplies
// 32 rows by all 64 columns (for SwiGLU 32 features' gate and up rows) over half of a step's k; the two halves are added in
// LDS at the end.  Reads, waits and loads are ordered by hand as in the eight-wave kernel above: with the loads of D - 2
// later steps in flight the stage read next has landed, behind the barrier for all waves, and the one refilled next has been read.
template <int EPI, int D>
__global__ __launch_bounds__(256) void gemm_narrow_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                          void *__restrict__ Cv, int M, int N, int K, size_t part_stride) {
  constexpr int STAGE = 16384, LOADS = 4;                 // bytes: 64 A rows, 64 B rows of 128; loads per wave and step
  constexpr bool SWIGLU = EPI == ARB_EPI_SWIGLU_BF16;
  __shared__ __attribute__((aligned(1024))) char Ring[D * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, kh = wave >> 1, frag_row = lane & 31, frag_half = lane >> 5;

  const int nk_all = K / 64;
  const int kt_begin = split_point(nk_all, blockIdx.y, gridDim.y);
  const int n = split_point(nk_all, blockIdx.y + 1, gridDim.y) - kt_begin, last = n - 1;

  // A load fills 8 rows of 8 pieces (16 bytes); this wave's rows are 8 wave + lane/8 and 32 more.  Pieces are swizzled by
  // row/2 on the global side.  Addresses: a uniform base and a 32-bit lane offset.
  const int row = wave * 8 + (lane >> 3);
  const unsigned k_bytes = (unsigned)K * 2, piece = ((lane & 7) ^ ((row >> 1) & 7)) * 16;
  unsigned a_off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) a_off[i] = (unsigned)min(row + 32 * i, M - 1) * k_bytes + piece;      // rows past M: never stored
  const unsigned b_off = (unsigned)row * k_bytes + piece;
  const char *a_base = (const char *)A + (size_t)kt_begin * 128;
  const char *b_base = (const char *)B + (size_t)blockIdx.x * (SWIGLU ? 32 : 64) * k_bytes + (size_t)kt_begin * 128;
  const size_t b_upper = (size_t)(SWIGLU ? N : 32) * k_bytes;          // from the tile's first 32 weight rows to the others
  auto load = [&](int s, int it) {                        // past the end: the last step again, never multiplied
    const size_t k = (size_t)(it < last ? it : last) * 128;
    char *dst = Ring + s * STAGE + wave * 1024;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(b_base + k + (i ? b_upper : 0) + b_off), LDS_PTR(dst + 8192 + i * 4096), 16, 0, 2 /* nt */);
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(a_base + k + a_off[i]), LDS_PTR(dst + i * 4096), 16, 0, 0);
    }
  };

  f32x16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

  // LDS offsets of this lane's fragments of its two MFMA steps
  unsigned a_addr[2], b_addr[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const unsigned o = (unsigned)(uintptr_t)LDS_PTR(Ring) + frag_row * 128 + (((2 * (2 * kh + u) + frag_half) ^ ((frag_row >> 1) & 7)) << 4);
    a_addr[u] = o + wm * 4096;
    b_addr[u] = o + 8192;
  }
#pragma unroll
  for (int s = 0; s < D - 1; ++s) load(s, s);
  int s = 0;
  for (int it = 0; it < n; ++it) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((D - 2) * LOADS));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    load(s == 0 ? D - 1 : s - 1, it + D - 1);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned stage = s * STAGE;
    bf16x8 fa[2], fb[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      wide_request_b<0>(a_addr[u] + stage, fa[u]);
      wide_request_a<0>(b_addr[u] + stage, fb[u][0], fb[u][1]);       // 32 rows of 128 bytes apart
    }
    wide_await<3>(fa[0], fb[0][0], fb[0][1]);
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[0][j], acc[j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    wide_await<0>(fa[1], fb[1][0], fb[1][1]);
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[1][j], acc[j], 0, 0, 0);
    s = s + 1 == D ? 0 : s + 1;
  }
  // every load has landed and, past the barrier, every stage has been read
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  __syncthreads();
  f32x4 *red = (f32x4 *)Ring;
  if (kh == 1) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        red[((wm * 2 + j) * 4 + q) * 64 + lane] = f32x4{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
  }
  __syncthreads();
  if (kh == 1) return;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = red[((wm * 2 + j) * 4 + q) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][4 * q + e] += v[e];
    }
  // D layout of the 32x32 MFMA: lane holds column lane%32 and rows 8*(r/4) + 4*(lane/32) + r%4.
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = wm * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
    if (m >= M) continue;
    if (SWIGLU) {
      const float gte = acc[0][r], up = acc[1][r];
      ((bf16 *)Cv)[(size_t)m * N + blockIdx.x * 32 + frag_row] = (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const size_t at = (size_t)m * N + blockIdx.x * 64 + j * 32 + frag_row;
        if (EPI == ARB_EPI_STORE_BF16) ((bf16 *)Cv)[at] = (bf16)acc[j][r];
        else if (EPI == EPI_PARTIAL_F32) ((float *)Cv)[blockIdx.y * part_stride + at] = acc[j][r];
        else ((float *)Cv)[at] += acc[j][r];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Weight-streaming kernel for few token rows (M <= 32: drafting token by token, a single short step).
// Such a launch reads every weight once and multiplies it with next to nothing, so it is bound by how many
// bytes of weights are in flight (a plain read of this memory reaches 6.2 TB/s, 7.0 with non-temporal loads).
// A workgroup owns 16 RT weight rows and a K range; its four waves deal the range's chunks of 64 k among
// themselves and each streams its own chunks, weights and activations, through a private ring of D LDS stages: no
// barrier until the end, when the four sums are added in LDS (fixed order) and stored.  Loads are direct-to-LDS and
// cover 8 rows x 128 bytes, i.e. whole cache lines: the same loop with fragments loaded straight into registers (four
// neighbouring lanes on four different rows) stays at 4.1 TB/s.  Weights are loaded non-temporal: each is used once.
// 16x16x32 MFMAs with the weights as rows and 16 MT tokens as columns; a lane ends with 4 consecutive features of one
// token.  Ring depth and rows keep a workgroup at 72 to 80 KB (two per CU) where MT allows.
// Large matrices with a K that fits are the resident-activation kernel's (gemm_few.hip); what is left here are small ones, where the
// start of a launch is all there is (QKV and O of the 1.5B shape at 16 tokens in four K splits 4.3 and 4.2 us by the kernel trace of
// a decode step, 4.8 and 4.6 there, unsplit; a pass takes them there all the same, fused with what follows), and unsplit products of a very long K.
__device__ __forceinline__ int lds_off_stream(int row, int chunk) {   // 128-byte rows; 16 lanes read one chunk of 16 rows
  return row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3);
}

template <int EPI, int MT, int RT, int D>
__global__ __launch_bounds__(256) void gemm_stream_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                          void *__restrict__ Cv, int M, int N, int K, size_t part_stride) {
  constexpr int W = 4;                                  // waves, each with its own chunks of K and its own ring
  constexpr int STAGE = (RT + MT) * 1024;               // elements of a wave's stage: 16 RT weight rows, 16 MT token rows
  constexpr int UNUSED = 8;
  constexpr int LOADS = 2 * (RT + MT);                  // wave-wide 1 KB loads per stage
  constexpr bool SWIGLU = EPI == ARB_EPI_SWIGLU_BF16;
  static_assert(D >= 2 && D <= 4 && (!SWIGLU || RT % 2 == 0), "ring depth, gate/up pairs");
  // one array per stage (the compiler orders LDS reads against in-flight loads by object)
  __shared__ __attribute__((aligned(16))) bf16 St0[W * STAGE], St1[W * STAGE], St2[D > 2 ? W * STAGE : UNUSED],
      St3[D > 3 ? W * STAGE : UNUSED];
#define ARB_ST(s) ((s) == 0 ? St0 : (s) == 1 ? St1 : (s) == 2 ? St2 : St3)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, quarter = lane >> 4, load_row = lane >> 3;

  // K range of this workgroup in chunks of 64, and this wave's share of it: chunks begin + wave, + W, ...
  const int nk_all = K / 64;
  const int kt_begin = split_point(nk_all, blockIdx.y, gridDim.y);
  const int kt_end = split_point(nk_all, blockIdx.y + 1, gridDim.y);
  const int n = (kt_end - kt_begin - wave + W - 1) / W, last = n - 1;

  const bf16 *w_src[2 * RT], *x_src[2 * MT];
#pragma unroll
  for (int i = 0; i < 2 * RT; ++i) {
    const int r = i * 8 + load_row, t = r >> 4;          // tile-local row, its 16-row MFMA tile
    // SwiGLU: the first half of the tiles are gate rows, the second half the matching up rows; N = F there
    const int row = SWIGLU ? blockIdx.x * (RT * 8) + (t % (RT / 2)) * 16 + (r & 15) + (t >= RT / 2 ? N : 0)
                           : blockIdx.x * (RT * 16) + r;
    w_src[i] = B + (size_t)row * K + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
  }
#pragma unroll
  for (int j = 0; j < 2 * MT; ++j) {
    const int r = j * 8 + load_row;
    const int m = r < M ? r : M - 1;                      // rows past M re-read the last one; never stored
    x_src[j] = A + (size_t)m * K + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
  }

  f32x4 acc[RT][MT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto load = [&](int s, int it) {                        // `it` past the end: the last chunk again, never used
    const size_t k = (size_t)(kt_begin + wave + min(it, last) * W) * 64;
    bf16 *dst = ARB_ST(s) + wave * STAGE;
#pragma unroll
    for (int i = 0; i < 2 * RT; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(w_src[i] + k), LDS_PTR(dst + i * 512), 16, 0, 2 /* nt */);
#pragma unroll
    for (int j = 0; j < 2 * MT; ++j)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(x_src[j] + k), LDS_PTR(dst + (2 * RT + j) * 512), 16, 0, 0);
  };
  auto multiply = [&](int s) {
    const bf16 *src = ARB_ST(s) + wave * STAGE;
    bf16x8 wf[2][RT], xf[2][MT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int off = lds_off_stream(r16, h * 4 + quarter);     // the swizzle does not change when 16 is added to the row
#pragma unroll
      for (int i = 0; i < RT; ++i) wf[h][i] = *(const bf16x8 *)&src[i * 1024 + off];
#pragma unroll
      for (int j = 0; j < MT; ++j) xf[h][j] = *(const bf16x8 *)&src[(RT + j) * 1024 + off];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][i], xf[h][j], acc[i][j], 0, 0, 0);
  };
  if (n > 0) {
#pragma unroll
    for (int s = 0; s < D - 1; ++s) load(s, s);
    int it = 0;
    for (; it + D <= n; it += D) {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        load((s + D - 1) % D, it + s + D - 1);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS * (D - 1)));       // this stage has landed; the D - 1 behind it may be in flight
        __builtin_amdgcn_sched_barrier(0);
        multiply(s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __builtin_amdgcn_sched_barrier(0);
    const int rem = n - it;
#pragma unroll
    for (int s = 0; s < D - 1; ++s)
      if (s < rem) multiply(s);
  }
  // Sum of the four waves.  The sums go over stage 0: every load has landed (waited for above) and, past the barrier,
  // every wave is done reading.
  __syncthreads();
  float *red = (float *)St0;
  static_assert(STAGE * sizeof(bf16) >= RT * MT * 256 * sizeof(float), "the sums fit stage 0");
#undef ARB_ST
  constexpr int TILE = 64 * 4;                            // floats of one 16x16 tile, in lane order
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) *(f32x4 *)&red[((wave * RT + i) * MT + j) * TILE + lane * 4] = acc[i][j];
  __syncthreads();
  auto total = [&](int i, int j, int l) {
    f32x4 s = *(const f32x4 *)&red[(i * MT + j) * TILE + l * 4];
#pragma unroll
    for (int w = 1; w < W; ++w) s += *(const f32x4 *)&red[((w * RT + i) * MT + j) * TILE + l * 4];
    return s;
  };
  // D layout of the 16x16 MFMA: lane holds column lane%16 (token) and rows 4*(lane/16) + {0..3} (features)
  for (int t = tid; t < (SWIGLU ? RT / 2 : RT) * MT * 64; t += 256) {
    const int l = t & 63, j = (t >> 6) % MT, i = (t >> 6) / MT;
    const int m = j * 16 + (l & 15);
    if (m >= M) continue;
    const f32x4 s = total(i, j, l);
    if (SWIGLU) {
      const f32x4 up = total(i + RT / 2, j, l);
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)(s[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-s[e])) * up[e]);
      *(bf16x4 *)((bf16 *)Cv + (size_t)m * N + blockIdx.x * (RT * 8) + i * 16 + (l >> 4) * 4) = o;
    } else {
      const size_t at = (size_t)m * N + blockIdx.x * (RT * 16) + i * 16 + (l >> 4) * 4;
      if (EPI == ARB_EPI_STORE_BF16) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)s[e];
        *(bf16x4 *)((bf16 *)Cv + at) = o;
      } else if (EPI == EPI_PARTIAL_F32) {
        *(f32x4 *)((float *)Cv + blockIdx.y * part_stride + at) = s;
      } else {
        *(f32x4 *)((float *)Cv + at) += s;
      }
    }
  }
}

}  // namespace

// Whether a launch runs on the weight-streaming kernel, and in which shape: mt = 16-token tiles, rt = 16-row
// tiles of weights per workgroup.  rows = weight rows (2 F for SwiGLU).  (What gemm_few_takes is asked about first.)
//  - Up to 16 tokens it beats the tiled kernels at every size measured.  Four row tiles instead of two pay where there are still
//    two workgroups per CU.
//  - From 17 to 32 tokens the activations, which every workgroup reads for itself, weigh as much as half of its weights: it
//    still wins where the tiled kernels are short of workgroups, i.e. on small matrices (up to 16 M weights: the narrow
//    projections of the 1.5B shape, whose forward of 20 tokens takes 453 us instead of 523), and on a very large matrix with a K that
//    no other few-token kernel holds: 65536 rows, us at 17 / 24 / 32 tokens, tiled against streaming, K 5120 114 / 119 / 127,
//    115 / 118 / 122; 8192 2 % ahead; 151936 rows equal within 5 %.
//  - Beyond, the 64-row tile, which shares the activations through LDS, is as fast or faster.
static bool stream_shape(int M, int rows, int K, int *mt, int *rt) {
  if (M <= 0 || M > 32) return false;
  const bool wide = rows / 64 >= 512 && rows % 64 == 0;
  *mt = M <= 16 ? 1 : 2;
  *rt = wide ? 4 : 2;
  return M <= 16 || (long long)rows * K <= (16 << 20) || (rows >= 65536 && wide && K >= 4096);
}

// K splits of a projection with fp32 partial products on the tiled kernels
int gemm_residual_splits(int M, int N, int K) {
  // as many workgroups as are resident at once (two per CU on 256 CUs) without starting a second
  // round, each keeping at least 4 K-steps; the partials cost 8 bytes of traffic per element and
  // split, so no more splits than that (measured on the 1.5B shape: 5 beats 4 and 6 for K = 8960).
  // With a short K (at most 32 steps) the launch is kept to one workgroup per CU instead, which the
  // deep-ring kernel serves better and which halves the partial traffic (measured: 2 beats 5 for K = 1536).
  const int tiles = ceil_div(M, BM) * (N / BN), nk = K / BK;
  int s = (nk <= 32 ? 256 : 512) / tiles;
  if (s > nk / 4) s = nk / 4;
  if (s > 8) s = 8;
  return s < 1 ? 1 : s;
}

int gemm_stream_splits(int M, int N, int K) {
  int mt, rt;
  if (!stream_shape(M, N, K, &mt, &rt)) return 0;
  // About one workgroup per CU, two where one split would leave CUs without work; at least six chunks of K per split
  // (the four waves share them) and at most the eight partial products that the workspace holds.  (1.5B shape, 16
  // tokens: O 4.8 / 3.9 / 3.4 us with 1 / 2 / 4 splits, down 7.7 / 8.4 with 5 / 8; 8B: QKV 15.7 / 12.6 with 1 / 2,
  // down 32.9 / 22.2 / 21.7 with 1 / 2 / 4.)
  const int tiles = N / (16 * rt), nk = K / BK;
  int s = tiles >= 256 ? 1 : tiles > 128 ? 2 : 256 / tiles;
  if (s > nk / 6) s = nk / 6;
  if (s > 8) s = 8;
  return s < 1 ? 1 : s;
}

int gemm_large_cols(int M, int N, int K, int epilogue, int splits) {
  int mt, rt;
  if (stream_shape(M, epilogue == ARB_EPI_SWIGLU_BF16 ? 2 * N : N, K, &mt, &rt)) return 0;
  // Large tiles run one per CU, so they go in whole rounds of 256: as many n-tile columns as fill whole
  // rounds (all of them when the last round would be at least 80 % full), the remaining columns in
  // 128x128 tiles.  With less than one round of large tiles everything runs in small ones.
  const int big_n = epilogue == ARB_EPI_SWIGLU_BF16 ? 128 : LN;       // a large n-tile is two small ones
  if (splits != 1 || M <= 64 || N <= 0 || N % big_n != 0) return 0;
  const int tm = ceil_div(M, LM), tn = N / big_n, total = tm * tn, tail = total % 256;
  if (total < 205) return 0;
  return 5 * tail >= 4 * 256 || tail == 0 ? tn : (total - tail) / tm;
}

// Time estimates in us for a launch of m rows with fp32 (or bf16) output, from which the planner below chooses.  Both have
// the form steps x time per step + fixed + what each split's product costs to write here and read in the consumer.  The constants
// are a fit to 8 matrices (QKV, O and down of the 1.5B and 8B shapes, two in between) x 29 row counts from 70 to 8208 x every
// kernel and split, weights from memory, plus each split's products read once at 12 TB/s (they come from the memory-side cache: a norm
// behind 3 and behind 7 of them, 768 rows of 1536: 5.9 and 7.3 us, a rotary kernel behind 1 and 2: 5.1 and 5.2).  Per step of 64 k:
// 64x128 tiles 0.355, 128x128 one per CU 0.53, two per CU 0.83, 256x128 0.9; 256x256 tiles 1.1 up to half of the CUs, 1.33 with
// all (the clock).  What the estimates choose is 0.9 % slower than the best of each (the worst 14 %); with times per step taken at full
// launches of long K, and one split per kernel to choose from, it was 5 % (30 %): 8B O at 160 rows 22 -> 17 us with its share of the
// consumer; passes of 200 / 384 / 512 rows of the 1.5B shape 765 -> 715, 897 -> 821, 1104 -> 1060 us.
static double split_us(int m, int N, int splits, int bytes) { return (double)m * N * bytes * splits / 2.9e6; }
static double tiled_us(int m, int N, int K, int splits, int bytes) {
  const int t128 = ceil_div(m, BM) * (N / BN) * splits, t64 = ceil_div(m, 64) * (N / BN) * splits,
            t256 = ceil_div(m, 256) * (N / BN) * splits;
  double step;
  if (t128 <= 128 || m <= 64) step = 0.355 * ceil_div(t64, 256);
  else if (t128 <= 256) step = 0.53;
  else if (t256 >= 192 && t256 <= 256) step = 0.9;
  else step = (t128 / 512) * 0.83 + (t128 % 512 == 0 ? 0.0 : t128 % 512 <= 256 ? 0.53 : 0.98);
  return step * (K / BK) / splits + 3.9 + split_us(m, N, splits, bytes);
}
static double wide_us(int m, int N, int K, int splits, int bytes) {
  const double f = ceil_div(m, W_TM) * (N / W_TN) * splits / 256.0;          // at most one round
  return (f <= 0.5 ? 1.1 : 1.1 + 0.46 * (f - 0.5)) * (K / BK) / splits + 3.9 + split_us(m, N, splits, bytes);
}

// How a projection without the SwiGLU epilogue is launched.  Rows that make up whole rounds of 256 large tiles go to the
// eight-wave kernel unsplit.  The rows left over (all of them, where there is no whole round) are a launch of their own,
// because what suits them is another kernel or another split of K: it goes to the eight-wave kernel with the number of
// splits that fills its round best, or to the tiled kernels, or (a few rows) to the weight-streaming kernel, whichever is
// estimated to be the fastest, or at most 64 rows to the kernel with resident activations.  max_splits > 0: fp32 output that may come
// as that many partial products; 0: unsplit.  (Down 6144x4096x14336:
// one launch of 384 tiles 635 us; 256 + 128 tiles in two K splits 550.  4943x4096x14336: 619 us in 320 tiles, 568 in
// 128x128 tiles; 256 + 64 in four splits 465.)
GemmPlan gemm_plan(int M, int N, int K, int max_splits) {
  GemmPlan p{};
  int row = 0;
  const bool partials = max_splits > 0;
  const int bytes = partials ? 4 : 2;
  int mt, rt;
  if (M > 64 && N % W_TN == 0 && N / W_TN <= 256 && !stream_shape(M, N, K, &mt, &rt)) {
    const int tn = N / W_TN, per_round = 256 / tn, whole = ceil_div(M, W_TM) / per_round * per_round;
    if (whole > 0) {
      row = whole * W_TM < M ? whole * W_TM : M;
      p.seg[p.n++] = GemmSeg{0, row, 1, true};
    }
  }
  const int m = M - row;
  if (m <= 0) return p;
  GemmSeg rest{row, m, 1, false};
  if (gemm_few_takes(m, N, K, 1) || (partials && gemm_few_splits(m, N, K, max_splits))) {
    if (partials) rest.splits = gemm_few_splits(m, N, K, max_splits);
  } else if (stream_shape(m, N, K, &mt, &rt)) {
    if (partials) rest.splits = std::min(gemm_stream_splits(m, N, K), max_splits);
  } else {
    double best = tiled_us(m, N, K, 1, bytes);
    for (int s = 2; partials && s <= max_splits && K / BK / s >= 4; ++s) {
      const double t = tiled_us(m, N, K, s, bytes);
      if (t < best) {
        best = t;
        rest.splits = s;
      }
    }
    const int tiles = N % W_TN == 0 ? ceil_div(m, W_TM) * (N / W_TN) : 0;
    for (int s = 1; tiles > 0 && tiles * s <= 256 && s <= (partials ? max_splits : 1) && K / BK / s >= 8; ++s) {
      const double t = wide_us(m, N, K, s, bytes);
      if (t < best) {
        best = t;
        rest.splits = s;
        rest.wide = true;
      }
    }
  }
  p.seg[p.n++] = rest;
  return p;
}

static arb_status launch_wide(const bf16 *A, const bf16 *B, void *C, int M, int N, int K, int epilogue, hipStream_t st,
                              int splits, int tiles_n, size_t part_stride) {
  const int tm = ceil_div(M, W_TM);
  const dim3 grid(tm * tiles_n, splits), block(512);
#define ARB_WIDE(E) hipLaunchKernelGGL((gemm_wide_kernel<E>), grid, block, 0, st, A, B, C, M, N, K, tm, tiles_n, part_stride)
  switch (epilogue) {
    case ARB_EPI_STORE_BF16: ARB_WIDE(ARB_EPI_STORE_BF16); break;
    case ARB_EPI_RESIDUAL_F32:
      if (splits > 1) ARB_WIDE(EPI_PARTIAL_F32); else ARB_WIDE(ARB_EPI_RESIDUAL_F32);
      break;
    case ARB_EPI_STORE_F32: ARB_WIDE(ARB_EPI_STORE_F32); break;
    case ARB_EPI_SWIGLU_BF16: ARB_WIDE(ARB_EPI_SWIGLU_BF16); break;
    default: return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
  }
#undef ARB_WIDE
  ARB_CHECK_LAUNCH("gemm_wide");
  return ARB_OK;
}

// One launch that covers all rows: the weight-streaming kernel, or up to two tiled kernels side by side.
static arb_status launch_tiles(const bf16 *A, const bf16 *B, void *C, int M, int N, int K, int epilogue, hipStream_t st,
                               int splits, int part, const bf16 *B_blocked, size_t part_stride) {
  const int tiles_m = ceil_div(M, BM);
  int tiles_n = epilogue == ARB_EPI_SWIGLU_BF16 ? N / 64 : N / BN;
  const int rows = epilogue == ARB_EPI_SWIGLU_BF16 ? 2 * N : N;
  if (gemm_few_takes(M, rows, K, splits))
    return part == GEMM_PART_LARGE ? ARB_OK : launch_gemm_few(A, B, C, M, N, K, epilogue, splits, part_stride, st);
  int mt, rt;
  if (stream_shape(M, rows, K, &mt, &rt)) {
    if (part == GEMM_PART_LARGE) return ARB_OK;
    const dim3 sgrid(rows / (16 * rt), splits), sblock(256);
#define ARB_STREAM(E)                                                                                                 \
  do {                                                                                                                \
    if (mt == 1 && rt == 2)                                                                                           \
      hipLaunchKernelGGL((gemm_stream_kernel<E, 1, 2, 3>), sgrid, sblock, 0, st, A, B, C, M, N, K, part_stride);      \
    else if (mt == 1)                                                                                                 \
      hipLaunchKernelGGL((gemm_stream_kernel<E, 1, 4, 2>), sgrid, sblock, 0, st, A, B, C, M, N, K, part_stride);      \
    else if (rt == 2)                                                                                                 \
      hipLaunchKernelGGL((gemm_stream_kernel<E, 2, 2, 4>), sgrid, sblock, 0, st, A, B, C, M, N, K, part_stride);      \
    else                                                                                                              \
      hipLaunchKernelGGL((gemm_stream_kernel<E, 2, 4, 3>), sgrid, sblock, 0, st, A, B, C, M, N, K, part_stride);      \
  } while (0)
    switch (epilogue) {
      case ARB_EPI_STORE_BF16: ARB_STREAM(ARB_EPI_STORE_BF16); break;
      case ARB_EPI_RESIDUAL_F32:
        if (splits > 1) ARB_STREAM(EPI_PARTIAL_F32); else ARB_STREAM(ARB_EPI_RESIDUAL_F32);
        break;
      case ARB_EPI_SWIGLU_BF16: ARB_STREAM(ARB_EPI_SWIGLU_BF16); break;
      case ARB_EPI_STORE_F32: ARB_STREAM(ARB_EPI_STORE_F32); break;
      default: return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
    }
#undef ARB_STREAM
    ARB_CHECK_LAUNCH("gemm_stream");
    return ARB_OK;
  }
  // At most 64 token rows: 64 weight rows per workgroup where 128 of them would leave half of the CUs idle, or would make
  // more than one round of one workgroup per CU (two of these share a CU).  Measured at 37 tokens against 64x128 tiles: down
  // of the 1.5B shape (96 workgroups of 128 weight rows) 12.7 -> 9.8 us, QKV and O (96, 72) 6.3 -> 6.2 and 6.1 -> 6.0, LM head
  // of the 8B shape (1002, in large tiles before) 248 -> 213.  In between 128 weight rows stay the better ones: gate/up (140) 16.3
  // against 18.5.
  const int wgs128 = rows / BN * splits;
  if (M <= 64 && (wgs128 <= 128 || wgs128 > 256)) {
    if (part == GEMM_PART_LARGE) return ARB_OK;
    const dim3 ngrid(rows / 64, splits), nblock(256);
    const bool one = rows / 64 * splits <= 256;           // one workgroup per CU: the deep ring
#define ARB_NARROW(E)                                                                                                    \
  do {                                                                                                                   \
    if (one) hipLaunchKernelGGL((gemm_narrow_kernel<E, 9>), ngrid, nblock, 0, st, A, B, C, M, N, K, part_stride);         \
    else hipLaunchKernelGGL((gemm_narrow_kernel<E, 5>), ngrid, nblock, 0, st, A, B, C, M, N, K, part_stride);             \
  } while (0)
    switch (epilogue) {
      case ARB_EPI_STORE_BF16: ARB_NARROW(ARB_EPI_STORE_BF16); break;
      case ARB_EPI_RESIDUAL_F32:
        if (splits > 1) ARB_NARROW(EPI_PARTIAL_F32); else ARB_NARROW(ARB_EPI_RESIDUAL_F32);
        break;
      case ARB_EPI_SWIGLU_BF16: ARB_NARROW(ARB_EPI_SWIGLU_BF16); break;
      case ARB_EPI_STORE_F32: ARB_NARROW(ARB_EPI_STORE_F32); break;
      default: return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
    }
#undef ARB_NARROW
    ARB_CHECK_LAUNCH("gemm_narrow");
    return ARB_OK;
  }
  const int big_cols = gemm_large_cols(M, N, K, epilogue, splits);   // n-tile columns given to the large-tile kernel
  if (big_cols > 0 && part != GEMM_PART_SMALL) {
    if (!B_blocked) {
      if (arb_status s = launch_wide(A, B, C, M, N, K, epilogue, st, splits, big_cols, part_stride)) return s;
    } else {
      const int tm = ceil_div(M, LM);
      const dim3 bgrid(tm * big_cols), bblock(256);
#define ARB_BIG(E) hipLaunchKernelGGL((gemm256_kernel<E>), bgrid, bblock, 0, st, A, B_blocked, C, M, N, K, tm, big_cols)
      switch (epilogue) {
        case ARB_EPI_STORE_BF16: ARB_BIG(ARB_EPI_STORE_BF16); break;
        case ARB_EPI_RESIDUAL_F32: ARB_BIG(ARB_EPI_RESIDUAL_F32); break;
        case ARB_EPI_STORE_F32: ARB_BIG(ARB_EPI_STORE_F32); break;
        case ARB_EPI_SWIGLU_BF16: ARB_BIG(ARB_EPI_SWIGLU_BF16); break;
        default: return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
      }
#undef ARB_BIG
      ARB_CHECK_LAUNCH("gemm256");
    }
  }
  const int tile_n0 = big_cols * 2;                   // small n-tiles covered by the large-tile launch
  tiles_n -= tile_n0;
  if (tiles_n == 0 || part == GEMM_PART_LARGE) return ARB_OK;
  const dim3 block(256);
  const bool ring = tiles_m * tiles_n * splits <= 256;      // at most one workgroup per CU: latency-bound
  // not even half of the CUs: 64-row tiles; also for at most 64 token rows, of which a 128-row tile would waste half
  // its loads in flight (gate/up of the 1.5B shape at 33 rows 17.6 -> 16.6 us, of the 8B shape 50 -> 46.6)
  const bool half = tiles_m * tiles_n * splits <= 128 || M <= 64;      // not even half of the CUs: 64-row tiles
  // More than one round of 128-row tiles that is one well-filled round of 256-row tiles (the split-K down
  // projection): the taller tile reads 0.75 KB of LDS per MFMA instead of 1 KB, needs a third less ingest
  // per flop and runs on the deep-ring kernel.
  const int tm256 = ceil_div(M, 256);
  const bool tall = !ring && tm256 * tiles_n * splits <= 256 && tm256 * tiles_n * splits >= 192;
  const int tm64 = ceil_div(M, 64);
  const dim3 grid(tiles_m * tiles_n, splits), grid64(tm64 * tiles_n, splits), grid256(tm256 * tiles_n, splits);
#define ARB_SMALL(E)                                                                                                  \
  do {                                                                                                                \
    if (tall)                                                                                                         \
      hipLaunchKernelGGL((gemm_ring_kernel<E, 4>), grid256, block, 0, st, A, B, C, M, N, K, tm256, tiles_n, tile_n0, part_stride); \
    else if (half && M <= 64)                                                                                         \
      hipLaunchKernelGGL((gemm_ring_kernel<E, 1, true>), grid64, block, 0, st, A, B, C, M, N, K, tm64, tiles_n, tile_n0, part_stride); \
    else if (half)                                                                                                    \
      hipLaunchKernelGGL((gemm_ring_kernel<E, 1>), grid64, block, 0, st, A, B, C, M, N, K, tm64, tiles_n, tile_n0, part_stride);   \
    else if (ring)                                                                                                    \
      hipLaunchKernelGGL((gemm_ring_kernel<E, 2>), grid, block, 0, st, A, B, C, M, N, K, tiles_m, tiles_n, tile_n0, part_stride);  \
    else                                                                                                              \
      hipLaunchKernelGGL((gemm_kernel<E>), grid, block, 0, st, A, B, C, M, N, K, tiles_m, tiles_n, tile_n0, part_stride);          \
  } while (0)
  switch (epilogue) {
    case ARB_EPI_STORE_BF16: ARB_SMALL(ARB_EPI_STORE_BF16); break;
    case ARB_EPI_RESIDUAL_F32:
      if (splits > 1) ARB_SMALL(EPI_PARTIAL_F32); else ARB_SMALL(ARB_EPI_RESIDUAL_F32);
      break;
    case ARB_EPI_SWIGLU_BF16: ARB_SMALL(ARB_EPI_SWIGLU_BF16); break;
    case ARB_EPI_STORE_F32: ARB_SMALL(ARB_EPI_STORE_F32); break;
    default: return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
  }
#undef ARB_SMALL
  ARB_CHECK_LAUNCH("gemm");
  return ARB_OK;
}

arb_status launch_gemm_plan(const GemmPlan &plan, const bf16 *A, const bf16 *B, void *C, int M, int N, int K, int epilogue,
                            hipStream_t st) {
  const size_t elem = epilogue == ARB_EPI_STORE_BF16 ? sizeof(bf16) : sizeof(float), part_stride = (size_t)M * N;
  for (int i = 0; i < plan.n; ++i) {
    const GemmSeg &g = plan.seg[i];
    const bf16 *a = A + (size_t)g.row0 * K;
    void *c = (char *)C + (size_t)g.row0 * N * elem;
    const arb_status s = g.wide ? launch_wide(a, B, c, g.rows, N, K, epilogue, st, g.splits, N / W_TN, part_stride)
                                : launch_tiles(a, B, c, g.rows, N, K, epilogue, st, g.splits, GEMM_PART_ALL, nullptr, part_stride);
    if (s) return s;
  }
  return ARB_OK;
}

arb_status launch_gemm(const bf16 *A, const bf16 *B, void *C, int M, int N, int K, int epilogue, hipStream_t st, int part,
                       const bf16 *B_blocked) {
  if (M == 0) return ARB_OK;
  if (M < 0 || N <= 0 || K <= 0) return arb_fail(ARB_EINVAL, "gemm: M=%d N=%d K=%d", M, N, K);
  if (K % BK != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm: K=%d is not a multiple of %d", K, BK);
  if (epilogue == ARB_EPI_SWIGLU_BF16) {
    if (N % 64 != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm: SwiGLU width %d is not a multiple of 64", N);
  } else {
    if (N % BN != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm: N=%d is not a multiple of %d", N, BN);
    if (epilogue < 0 || epilogue > ARB_EPI_STORE_F32) return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
    if (!B_blocked) return launch_gemm_plan(gemm_plan(M, N, K, 0), A, B, C, M, N, K, epilogue, st);
  }
  return launch_tiles(A, B, C, M, N, K, epilogue, st, 1, part, B_blocked, 0);
}

// packed[(kb * rows + r) * 32 + j] = W[r][kb * 32 + j]: one thread per 16-byte chunk
__global__ __launch_bounds__(256) void pack_k_blocked_kernel(const bf16 *__restrict__ W, size_t rows, int K,
                                                             bf16 *__restrict__ packed) {
  const size_t chunks_per_row = K / 8, total = rows * chunks_per_row;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t r = i / chunks_per_row, c = i - r * chunks_per_row;      // source row and 16-byte chunk
    const size_t kb = c / 4;
    *(bf16x8 *)(packed + (kb * rows + r) * 32 + (c % 4) * 8) = *(const bf16x8 *)(W + r * (size_t)K + c * 8);
  }
}

arb_status launch_pack_k_blocked(const bf16 *W, size_t rows, int K, bf16 *packed, hipStream_t st) {
  if (rows == 0) return ARB_OK;
  if (K <= 0 || K % 32 != 0) return arb_fail(ARB_EUNSUPPORTED, "pack_k_blocked: K=%d is not a multiple of 32", K);
  const size_t chunks = rows * (size_t)(K / 8);
  const int blocks = (int)((chunks + 255) / 256 < 8192 ? (chunks + 255) / 256 : 8192);
  hipLaunchKernelGGL(pack_k_blocked_kernel, dim3(blocks), dim3(256), 0, st, W, rows, K, packed);
  ARB_CHECK_LAUNCH("pack_k_blocked");
  return ARB_OK;
}
