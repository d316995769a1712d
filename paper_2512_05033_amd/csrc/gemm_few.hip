// Projections of few token rows (drafting token by token, one short step): C[M,N] = A[M,K] * B[N,K]^T with M <= 64, and
// the two fusions that such a pass wants, because its launches of a few microseconds each cost more than their bytes:
// the QKV projection that rotates and appends, and the O projection that completes the residual stream and hands the norm
// on as unscaled rows with their sums of squares.
//
// Such a launch reads every weight once, so what bounds it is the memory: how many bytes of weights are in flight, and that
// nothing else is.  One workgroup of eight waves per CU at a time (the O launch of a model wider than 4096 is two
// rounds of them); a wave owns one eighth of the workgroup's K and keeps the
// activations of that slice in registers, as MFMA operands, for the whole launch, so that the LDS holds little but weights: a
// private ring of D stages of 16 rows by 64 k (2 KB) per wave, 48 to 80 KB per CU in flight, filled by non-temporal direct-to-LDS
// loads of whole 128-byte lines.  The activations come first through the same ring, and the ring runs on across the 16-row tiles that the workgroup
// walks through; at the end of a tile the eight partial sums meet in one of two LDS buffers (one barrier per tile, behind which the others
// go on), and the waves take turns in adding them up and storing (the compiler has that wave wait for its own ring first).  (The kernel before it, gemm_stream_kernel, fetches the activations
// again for every 32 weight rows, drains at the end of each of its short workgroups, and its launches were 1.09 or 1.75 rounds of them.)
// By the kernel trace of a pass, us, with that kernel and now: 1.5B shape, 16 tokens: gate/up 15.5 -> 13.7, down (5 splits) 7.6 -> 7.1, LM head
// 87.8 -> 82.2, QKV and the rotary kernel 4.3 + 3.3 -> 5.4, O and the norm 4.2 + 3.5 -> 5.0; 37 tokens: gate/up 16.8 -> 15.2, down
// 10.0 -> 9.1, QKV 6.2 + 3.5 -> 6.3, O 6.0 + 4.8 -> 6.1; 8B shape, 5 tokens: QKV 12.4 + 4.6 -> 11.7, O 12 + 4.6 -> 8.7, down
// 30 -> 20.3, gate/up 39.9 -> 38.7, LM head 193 -> 165 (6.4 TB/s).
#include "common.h"

#include <algorithm>

namespace {

#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// s_waitcnt immediates (vmcnt in bits 3:0 and 15:14, lgkmcnt in 11:8, expcnt 6:4 left at "no wait")
constexpr int waitcnt_vm(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0xF70; }
constexpr int kWaitLgkm0 = 0xC07F;

constexpr int FW = 8;                                    // waves
constexpr int kFewGrid = 256;                            // one workgroup per CU
constexpr long long kFewWeights = 8 << 20;               // fewest weights of an unfused launch
constexpr int kSquarePieces = 16;                        // most partial sums of squares a thread adds up
constexpr double kStageUs = 0.55;                        // of a CU, for one 16 KB stage (all waves together)

// How a launch divides its units and its chunks of 64 k among the workgroups: so many each, one more for the first few.
struct FewSplit {
  int units, units_left, chunks, chunks_left;
};
// chunks per wave
inline int few_chunks(int K, int splits) { return ceil_div(ceil_div(K / 64, splits), FW); }

enum { FEW_BF16, FEW_RESIDUAL, FEW_F32, FEW_SWIGLU, FEW_SCALED_SWIGLU, FEW_ROPE, FEW_NORM };

// LDS reads that the compiler must not order behind the direct-to-LDS loads in flight (it would wait for all of them); each block
// waits for its own reads, so that no register is named before it holds its value.
template <typename T>
__device__ __forceinline__ void few_read(unsigned a0, unsigned a1, T &v0, T &v1) {
  static_assert(sizeof(T) == 16, "16 bytes");
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v0), "=&v"(v1) : "v"(a0), "v"(a1) : "memory");
}
template <typename T>
__device__ __forceinline__ void few_read(unsigned a0, unsigned a1, unsigned a2, T &v0, T &v1, uint32_t &v2) {
  static_assert(sizeof(T) == 16, "16 bytes");
  asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %4\n\tds_read_b32 %2, %5\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v0), "=&v"(v1), "=&v"(v2) : "v"(a0), "v"(a1), "v"(a2) : "memory");
}
__device__ __forceinline__ void few_read4(unsigned a, uint32_t (&v)[4]) {     // 256 bytes apart
  asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\t"
               "ds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(a) : "memory");
}

// Weight rows come in units of eight: eight consecutive rows, or (SwiGLU) four gate rows and their four up rows, or (QKV) four
// rows of the first half of a head and the four that the rotation pairs them with.  A tile is two units.  In the result of
// the 16x16 MFMA lane quarter q holds rows 4 q .. 4 q + 3 of the tile for the token lane % 16, so that the two
// partners of a pair come to lie in neighbouring quarters of the same token.
template <int EPI, int MT, int NC, int D>
__global__ __launch_bounds__(64 * FW, 2) void gemm_few_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ B,
                                                           void *__restrict__ Cv, int M, int N, int K, FewSplit split,
                                                           size_t part_stride, FewFusion fu) {
  constexpr bool SCALED = EPI == FEW_SCALED_SWIGLU, SWIGLU = EPI == FEW_SWIGLU || SCALED, ROPE = EPI == FEW_ROPE, NORM = EPI == FEW_NORM, PAIRED = SWIGLU || ROPE;
  constexpr int P = 16 * MT, NP = 64 * FW / P;             // padded tokens; threads per token that add up sums of squares
  __shared__ __attribute__((aligned(1024))) char Ring[FW * D * 2048];
  __shared__ __attribute__((aligned(16))) f32x4 Red[2][FW][MT][64];
  constexpr int SIDE = SCALED ? kSquarePieces * 256 : ROPE ? 2 * 1024 + 256 : NORM ? 2 * 1024 : 0;      // bytes per wave
  __shared__ __attribute__((aligned(1024))) char Side[SIDE ? FW * SIDE : 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, quarter = lane >> 4, bx = blockIdx.x, by = blockIdx.y;

  // units of this workgroup, K range of this wave (in chunks of 64; a short launch is a chain of few instructions, so no divisions)
  const int u0 = bx * split.units + min(bx, split.units_left), nu = split.units + (bx < split.units_left);
  const int tiles = (nu + 1) / 2;
  const int kt0 = by * split.chunks + min(by, split.chunks_left), kn = split.chunks + (by < split.chunks_left);
  const int c0 = kn * wave / FW, nc = kn * (wave + 1) / FW - c0;
  const unsigned k_bytes = (unsigned)K * 2;
  const char *a_base = (const char *)A + (size_t)(kt0 + c0) * 128, *b_base = (const char *)B + (size_t)(kt0 + c0) * 128;

  // Everything that is not a weight is asked for first, to a place of this wave's in LDS: loads return in order, so it has landed when the
  // first stage has.
  char *side = Side + wave * SIDE;
  const unsigned side_addr = (unsigned)(uintptr_t)LDS_PTR(side);
  if (SCALED) {
#pragma unroll 1
    for (int i = 0; i * NP < fu.n_squares; ++i)             // at most kSquarePieces (gemm_few_norms)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(fu.squares + min(tid / P + i * NP, fu.n_squares - 1) * P + tid % P), LDS_PTR(side + i * 256), 4, 0, 0);
  }
  // the one item (tile, 16 tokens) that this wave finishes: residual stream and gain, or cosines, sines and pool slot
  f32x4 item[2];
  uint32_t slot;
  if (NORM) {
    const unsigned f = u0 * 8 + quarter * 4;
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(fu.h + min(wave * 16 + r16, M - 1) * N + f), LDS_PTR(side), 16, 0, 0);
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(fu.gain + f), LDS_PTR(side + 1024), 16, 0, 0);
  }
  if (ROPE) {
    const int t = min(wave / MT, tiles - 1), m = min(wave % MT * 16 + r16, M - 1), half = fu.head_dim / 2;
    const int u = u0 + min(2 * t + (lane >> 4 & 1), nu - 1);
    const f32x2 *cs = fu.cs + m * half + (u * 4 & (half - 1));
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(cs), LDS_PTR(side), 16, 0, 0);
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(cs + 2), LDS_PTR(side + 1024), 16, 0, 0);
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(fu.tok_slot + m), LDS_PTR(side + 2048), 4, 0, 0);
  }
  // A stage is 16 rows by 64 k: load i of it rows 8 i + lane / 8, lane l piece l % 8 (16 bytes), swizzled by the row / 2
  // on the global side.  The first stages of a wave are its activations, 16 tokens each (rows past M repeat the last one and are never
  // stored), the others weights, a unit per load.  A workgroup's last tile may hold one unit, which it then holds twice.  (Activations
  // loaded straight into registers, in half lines: QKV alone at 16 / 37 tokens 5.7 / 8.0 us instead of 4.8 / 5.8.)
  const int lr = lane >> 3;
  const unsigned piece0 = ((lane & 7) ^ ((lr >> 1) & 7)) * 16, piece1 = ((lane & 7) ^ (((lr + 8) >> 1) & 7)) * 16;
  const unsigned unit_rows = (PAIRED ? (lr & 3) + (lr >> 2) * (SWIGLU ? N : fu.head_dim / 2) : lr) * k_bytes;
  const int head_shift = ROPE ? fu.head_shift : 0;
  // first row of a unit: 8 u, 4 u, or 4 u and the second halves of the heads before it
  auto unit_row = [&](int u) { return (unsigned)(PAIRED ? 4 * u + (ROPE ? u >> head_shift << (head_shift + 2) : 0) : 8 * u); };
  char *ring = Ring + wave * D * 2048;
  const int total = (MT + tiles) * nc;                      // stages of this wave
  int issued = 0, ls = 0, lc = nc, lt = -MT;                // stages asked for; ring offset, chunks left and tile (of tokens: negative) of the next
  const char *base;                                         // addresses: a uniform base and a 32-bit lane offset
  unsigned off0, off1;
  auto aim = [&]() {
    if (lt < 0) {
      base = a_base;
      off0 = min((lt + MT) * 16 + lr, M - 1) * k_bytes + piece0;
      off1 = min((lt + MT) * 16 + 8 + lr, M - 1) * k_bytes + piece1;
    } else {
      const unsigned row = unit_row(u0 + 2 * lt);
      base = b_base + (size_t)row * k_bytes;
      off0 = unit_rows + piece0;
      off1 = unit_rows + piece1 + (unit_row(u0 + min(2 * lt + 1, nu - 1)) - row) * k_bytes;
    }
  };
  aim();
  auto request = [&]() {
    if (lt < 0) {                                           // every workgroup reads them: they have to stay in L2 (non-temporal: QKV 5.8 -> 6.9 us)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(base + off0), LDS_PTR(ring + ls), 16, 0, 0);
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(base + off1), LDS_PTR(ring + ls + 1024), 16, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(base + off0), LDS_PTR(ring + ls), 16, 0, 2 /* nt */);
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(base + off1), LDS_PTR(ring + ls + 1024), 16, 0, 2 /* nt */);
    }
    base += 128;
    ls = ls == (D - 1) * 2048 ? 0 : ls + 2048;
    ++issued;
    if (__builtin_expect(--lc == 0, 0)) {
      lc = nc;
      ++lt;
      aim();
    }
  };
#pragma unroll 1
  for (int i = min(D - 1, total); i > 0; --i) request();

  unsigned addr[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    addr[h] = (unsigned)(uintptr_t)LDS_PTR(ring) + r16 * 128 + (((h * 4 + quarter) ^ ((r16 >> 1) & 7)) << 4);
  int s = 0, done = 0;                                      // ring slot and number of the stage to be read
  // The next stage, as MFMA operands.  It has landed when no more than the stages behind it are in flight (a store in between
  // only makes the wait longer); near the end, where nothing is asked for any more, fewer may be.
  auto take = [&](bf16x8 &f0, bf16x8 &f1) {
    if (issued < total) request();                          // into the slot that was read last
    __builtin_amdgcn_sched_barrier(0);
    const int behind = issued - 1 - done;
    if (behind >= D - 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * (D - 1)));
    else if (behind >= 3) __builtin_amdgcn_s_waitcnt(waitcnt_vm(6));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __builtin_amdgcn_sched_barrier(0);
    few_read(addr[0] + s, addr[1] + s, f0, f1);
    ++done;
    s = s == (D - 1) * 2048 ? 0 : s + 2048;
    __builtin_amdgcn_sched_barrier(0);
  };
  bf16x8 act[NC][2][MT];
#pragma unroll
  for (int j = 0; j < MT; ++j)
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) take(act[c][0][j], act[c][1][j]);
  if (NORM) few_read(side_addr + lane * 16, side_addr + 1024 + lane * 16, item[0], item[1]);
  if (ROPE) few_read(side_addr + lane * 16, side_addr + 1024 + lane * 16, side_addr + 2048 + lane * 4, item[0], item[1], slot);

  // 1 / rms of each token's row, from the partial sums of squares that the O projection left (fixed order)
  float inv_rms[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) inv_rms[j] = 1.0f;
  if (SCALED) {
    float *sums = (float *)Red;                             // [P][NP]
    float sq = 0.f;
#pragma unroll 1
    for (int i = 0; i * NP < fu.n_squares; i += 4) {        // (of four, the ones past the last hold nothing and are not added)
      uint32_t square[4];
      few_read4(side_addr + i * 256 + lane * 4, square);
#pragma unroll
      for (int k = 0; k < 4; ++k) sq += tid / P + (i + k) * NP < fu.n_squares ? __uint_as_float(square[k]) : 0.f;
    }
    if (tid / P < NP) sums[tid % P * NP + tid / P] = sq;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      float all = 0.f;
#pragma unroll
      for (int i = 0; i < NP; ++i) all += sums[(j * 16 + r16) * NP + i];
      inv_rms[j] = 1.0f / sqrtf(all / (float)K + fu.eps);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();                           // read by all before a tile's sums go there
    __builtin_amdgcn_sched_barrier(0);
  }

  for (int t = 0; t < tiles; ++t) {
    f32x4 acc[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) {
        bf16x8 wf[2];
        take(wf[0], wf[1]);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < MT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h], act[c][h][j], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    // Two buffers: one is written again two tiles on, behind the next tile's barrier, which its readers reach after reading.
    f32x4(*red)[MT][64] = Red[t & 1];
#pragma unroll
    for (int j = 0; j < MT; ++j) red[wave][j][lane] = acc[j];
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int units = min(2, nu - 2 * t);                    // units of this tile
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      if (((t * MT + j) & (FW - 1)) != wave) continue;
      const int m = j * 16 + r16;
      auto sum = [&](int l) {
        f32x4 v = red[0][j][l];
#pragma unroll
        for (int w = 1; w < FW; ++w) v += red[w][j][l];
        return v;
      };
      if (PAIRED) {
        const int i = lane >> 4, u = u0 + 2 * t + i;
        if (i >= units || m >= M) continue;                  // half of the lanes: an item is a token and a unit
        f32x4 a = sum(i * 32 + r16), b = sum(i * 32 + 16 + r16);
        if (SWIGLU) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gte = SCALED ? a[e] * inv_rms[j] : a[e], up = SCALED ? b[e] * inv_rms[j] : b[e];
            o[e] = (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
          }
          *(bf16x4 *)((bf16 *)Cv + (size_t)m * N + (size_t)u * 4) = o;
        } else {
          const int head = u >> head_shift, f = u * 4 & (fu.head_dim / 2 - 1);
          bf16x4 oa, ob;
          if (head < fu.n_q_heads + fu.n_kv_heads) {
            const float q = head < fu.n_q_heads ? fu.q_scale : 1.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float cosv = item[e / 2][e % 2 * 2], sinv = item[e / 2][e % 2 * 2 + 1];
              oa[e] = (bf16)((a[e] * cosv - b[e] * sinv) * q);
              ob[e] = (bf16)((b[e] * cosv + a[e] * sinv) * q);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              oa[e] = (bf16)a[e];
              ob[e] = (bf16)b[e];
            }
          }
          bf16 *dst;
          if (head < fu.n_q_heads) {
            dst = (bf16 *)Cv + ((size_t)m * fu.n_q_heads + head) * fu.head_dim;
          } else {
            const int kv = head - fu.n_q_heads, hk = kv < fu.n_kv_heads ? kv : kv - fu.n_kv_heads;
            dst = (kv < fu.n_kv_heads ? fu.k_pool : fu.v_pool) +
                  (((size_t)(slot / ARB_KV_BLOCK) * fu.n_kv_heads + hk) * ARB_KV_BLOCK + slot % ARB_KV_BLOCK) * fu.head_dim;
          }
          *(bf16x4 *)(dst + f) = oa;
          *(bf16x4 *)(dst + f + fu.head_dim / 2) = ob;
        }
      } else {
        f32x4 v = sum(lane);
        const bool mine = m < M && quarter / 2 < units;
        const size_t at = (size_t)m * N + (size_t)(u0 + 2 * t) * 8 + quarter * 4;
        if (NORM) {
          // The residual stream is complete here; its norm needs the whole row.  The row goes on times the gain, unscaled
          // (rounded to bf16 as the scaled one would be), with this tile's share of its sum of squares.
          v += item[0];
          float sq = mine ? v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3] : 0.f;
          sq += __shfl_xor(sq, 16, 64);
          sq += __shfl_xor(sq, 32, 64);
          if (lane < 16) fu.squares_out[(size_t)blockIdx.x * P + m] = sq;
          if (mine) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(v[e] * item[1][e]);
            *(f32x4 *)(fu.h + at) = v;
            *(bf16x4 *)((bf16 *)Cv + at) = o;
          }
        } else if (mine) {
          if (EPI == FEW_BF16) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
            *(bf16x4 *)((bf16 *)Cv + at) = o;
          } else if (EPI == FEW_F32) {
            *(f32x4 *)((float *)Cv + blockIdx.y * part_stride + at) = v;
          } else {
            *(f32x4 *)((float *)Cv + at) += v;
          }
        }
      }
    }
  }
}

template <int EPI>
arb_status launch_few(const bf16 *A, const bf16 *B, void *C, int M, int N, int K, const dim3 &grid, size_t part_stride,
                      const FewFusion &fu, hipStream_t st) {
  const int mt = ceil_div(M, 16), nc = few_chunks(K, grid.y), units = (EPI == FEW_SWIGLU || EPI == FEW_SCALED_SWIGLU ? 2 * N : N) / 8, gx = grid.x, gy = grid.y;
  const FewSplit split{units / gx, units % gx, K / 64 / gy, K / 64 % gy};
#define ARB_FEW(MT, NC, D)                                                                                              \
  hipLaunchKernelGGL((gemm_few_kernel<EPI, MT, NC, D>), grid, dim3(64 * FW), 0, st, A, B, C, M, N, K, split, part_stride, fu)
  // Depth of the ring: what covers the memory's latency (a long K: six stages), and no more: the requests in front of the first wait
  // hold up a short launch.  Passes with nine stages (160 KB with the sums) / eight / six / five, us: 1.5B shape, one token 353 / 350 / 344 / 339,
  // 16 sequences 520 / 517 / 510 / 507; 8B shape, one token 391 / 387 / 382 / 383, 32 tokens 431 / 432 / 429 / 432.
  if (mt == 1) { if (nc <= 4) ARB_FEW(1, 4, 5); else if (nc <= 8) ARB_FEW(1, 8, 6); else ARB_FEW(1, 16, 6); }
  else if (mt == 2) { if (nc <= 4) ARB_FEW(2, 4, 5); else ARB_FEW(2, 8, 6); }
  else if (mt == 3) ARB_FEW(3, 4, 4);
  else ARB_FEW(4, 4, 4);
#undef ARB_FEW
  ARB_CHECK_LAUNCH("gemm_few");
  return ARB_OK;
}

}  // namespace

// Whether a launch of M rows against `rows` weight rows (2 F for SwiGLU), K in so many splits, can run on this kernel.
//  - A wave's slice of the activations has to fit its registers (8 per chunk and 16 tokens): at most 128 of them.
//  - Every wave needs work: at least two of the chunks of K.
//  - A lane's offset from its unit's first row is kept in 32 bits.
static bool few_fits(int M, int rows, int K, int splits) {
  if (M <= 0 || M > 64 || K / 64 / splits < 2 * FW || (long long)(rows + 8) * K * 2 >= (1LL << 32)) return false;
  const int nc = few_chunks(K, splits);
  return nc <= 16 && ceil_div(M, 16) * (nc <= 4 ? 4 : nc <= 8 ? 8 : 16) <= 16;
}

// ... and should.  On small matrices the start of a launch is all there is, and a split K is the faster start.
bool gemm_few_takes(int M, int rows, int K, int splits) {
  return few_fits(M, rows, K, splits) && (long long)rows * K >= kFewWeights;
}

// K splits of a projection with fp32 partial products, 0 if this kernel does not take it.  The time of a launch goes with the
// number of 16 KB stages (all waves together) per workgroup, activations included, of which a CU takes one in about kStageUs; every
// split costs its consumer another row to read.
int gemm_few_splits(int M, int N, int K, int max_splits) {
  int best = 0;
  double best_us = 0;
  for (int s = 1; s <= max_splits; ++s) {
    if (!gemm_few_takes(M, N, K, s)) continue;
    const int per = std::max(2, ceil_div(N / 8, kFewGrid / s));          // units of a workgroup
    const double us = kStageUs * (ceil_div(M, 16) + ceil_div(per, 2)) * K / 64 / s / FW + s * (0.4 + (double)M * N * 8 / 5.0e6);
    if (best == 0 || us < best_us) {
      best = s;
      best_us = us;
    }
  }
  return best;
}

arb_status launch_gemm_few(const bf16 *A, const bf16 *B, void *C, int M, int N, int K, int epilogue, int splits,
                           size_t part_stride, hipStream_t st) {
  const int units = (epilogue == ARB_EPI_SWIGLU_BF16 ? 2 * N : N) / 8;
  const dim3 grid(std::min(kFewGrid / splits, ceil_div(units, 2)), splits);       // whole tiles, one workgroup per CU
  const FewFusion none{};
  switch (epilogue) {
    case ARB_EPI_STORE_BF16: return launch_few<FEW_BF16>(A, B, C, M, N, K, grid, part_stride, none, st);
    case ARB_EPI_RESIDUAL_F32:
      if (splits > 1) return launch_few<FEW_F32>(A, B, C, M, N, K, grid, part_stride, none, st);
      return launch_few<FEW_RESIDUAL>(A, B, C, M, N, K, grid, part_stride, none, st);
    case ARB_EPI_STORE_F32: return launch_few<FEW_F32>(A, B, C, M, N, K, grid, part_stride, none, st);
    case ARB_EPI_SWIGLU_BF16: return launch_few<FEW_SWIGLU>(A, B, C, M, N, K, grid, part_stride, none, st);
  }
  return arb_fail(ARB_EINVAL, "gemm: unknown epilogue %d", epilogue);
}

// ---- the fused launches of a pass ----

// QKV: the epilogue holds both partners of a rotary pair, rotates them and writes q, and k and v to their pool slots, so that neither
// the fp32 products nor the launch that would read them back exist.  Sums are fp32 and q, k are rounded once, after the rotation.  A wave
// fetches what its one item needs (cosines, sines, slot) at the start; that is the limit on tiles.
// K is not split here, so a workgroup with a whole tile more than its even share costs that tile's stages.  The alternative, K splits
// that divide evenly and a rotary kernel, costs a launch: where the uneven share takes more than 4 us of stages, it is the faster one.
// Passes of 1 / 8 / 16 tokens, us per layer, fused against split: 2.2 us (4096 wide, 6144 QKV rows) 98.1 / 102.3 / 104.1, 99.5 / 104.0 /
// 104.6; 3.3 us (8192, 2560) 59.7 / 62.6 / 63.5, 59.8 / 63.7 / 64.7; 4.4 us (8192, 10240) 304.4 / 308.3 / 313.2, 303.0 / 307.2 /
// 312.1; 5.0 us (6144, 5120) 63.3 / 66.0 / 67.1, 61.2 / 65.0 / 66.4; 7.2 us (7680, 8704) 90.9 / 94.8 / 97.1, 89.4 / 93.5 / 94.5.
bool gemm_few_rotates(int M, int rows, int K) {
  if (!few_fits(M, rows, K, 1)) return false;
  const int units = rows / 8, tiles = ceil_div(ceil_div(units, std::min(kFewGrid, ceil_div(units, 2))), 2);
  return tiles * ceil_div(M, 16) <= FW && kStageUs * (tiles - units / (2.0 * kFewGrid)) * K / 64 / FW <= 4.0;
}
arb_status launch_gemm_few_qkv(const bf16 *A, const bf16 *B, bf16 *q, int M, int rows, int K, const FewFusion &fu, hipStream_t st) {
  return launch_few<FEW_ROPE>(A, B, q, M, rows, K, dim3(std::min(kFewGrid, ceil_div(rows / 8, 2)), 1), 0, fu, st);
}

// O, the norm and gate/up: the O epilogue adds its sums to the residual stream and stores the new row times the gain, unscaled, with each
// 16-feature tile's share of the row's sum of squares; every gate/up workgroup adds those up and scales its sums by 1 / rms before the
// activation.  W (r x) = r (W x) row by row, and x is rounded to bf16 once with or without r, so nothing is rounded more than it was.
// A workgroup of the O launch has one tile, so that each wave can fetch the stream and the gain of its one item at the start.  So the launch
// is d / 16 workgroups, each over the whole K, one per CU.  Where they leave CUs idle, in the only round or in the second, K splits
// and a norm kernel can be faster; by the stages that an even division would save, the line lies at 3.1 us in one round (from 96 workgroups
// on the launch has the memory's rate all the same) and at 2.1 us with a second.  Passes of 1 / 8 / 16 tokens, us per layer, fused against split:
// one round, 3.0 us (1280 wide, 4096 of attention) 31.0 / 32.9 / 34.7, 30.5 / 33.6 / 35.4; 3.3 us (1024, 4096) 30.0 / 31.8 / 33.4,
// 29.0 / 30.9 / 32.8; 6.6 us (1024, 8192) 35.3 / 37.1 / 39.3, 32.4 / 34.5 / 37.0; 96 workgroups, 2.8 us (1536, 4096) 31.0 / 33.2 / 35.2,
// 32.8 / 35.4 / 37.5; two rounds, 1.4 us (6144, 2560) 54.1 / 56.2 / 57.7, 54.5 / 56.8 / 58.0; 2.5 us (5120, 3072) 51.1 / 52.7 /
// 55.0, 50.3 / 52.4 / 54.7; 4.1 us (5120, 5120) 62.2 / 65.3 / 66.8, 59.9 / 63.8 / 64.5; 0 us (8192, 8192) 304.4 / 308.3 / 313.2,
// 305.9 / 309.6 / 313.4.
bool gemm_few_norms(int M, int d, int hq, int F) {
  const int pieces = 64 * FW / (16 * ceil_div(M, 16)) * kSquarePieces;     // partial sums that a gate/up workgroup can add up per token
  if (!few_fits(M, d, hq, 1) || !few_fits(M, 2 * F, d, 1) || d / 16 > pieces) return false;
  const int workgroups = d / 16, rounds = ceil_div(workgroups, kFewGrid);
  const double idle_us = kStageUs * (rounds - workgroups / (double)kFewGrid) * hq / 64 / FW;
  return rounds == 1 ? workgroups >= 96 || idle_us <= 3.1 : idle_us <= 2.1;
}
arb_status launch_gemm_few_o(const bf16 *A, const bf16 *B, bf16 *x, int M, int d, int hq, const FewFusion &fu, hipStream_t st) {
  return launch_few<FEW_NORM>(A, B, x, M, d, hq, dim3(d / 16, 1), 0, fu, st);
}
arb_status launch_gemm_few_gate_up(const bf16 *x, const bf16 *B, bf16 *act, int M, int F, int d, const FewFusion &fu, hipStream_t st) {
  return launch_few<FEW_SCALED_SWIGLU>(x, B, act, M, F, d, dim3(std::min(kFewGrid, ceil_div(F / 4, 2)), 1), 0, fu, st);
}
