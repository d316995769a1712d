// Projection GEMM with 4-bit weights and bf16 activations (the weight-quantized draft of the
// self-draft regime, Section 5.1): C[M,N] = A[M,K] * W'[N,K]^T with
// W'[n,k] = q[n,k] * scale[n, k/128], q in [-8, 7] stored as offset-binary nibbles, eight
// consecutive k per uint32, scale bf16.
//
// The tile kernel (more than 32 activation rows) has the geometry of the 128x128x64 bf16 kernel (4 waves of 64x64,
// A by direct-to-LDS loads), except for the weight operand: each thread fetches 16 bytes of packed weights (32 nibbles
// of one row) into registers, expands them to the bf16 integers -8..7 (exact) and stores them into an LDS stage.  The
// MFMAs therefore accumulate sum_k a[m,k] q[n,k] per group of 128 k (two steps) into a temporary accumulator; at the
// end of a group it is folded into the result with one fp32 multiply by the group's scale.  No product q*scale is ever
// rounded to bf16, so the result differs from the definition only by fp32 accumulation.  Weight traffic is a quarter
// of the bf16 kernel's.  Up to 32 rows a weight-streaming kernel runs instead (below).
#include "common.h"

#include <math.h>

#include <type_traits>

namespace {

constexpr int BM = 128, BN = 128, BK = 64, GROUP = 128;
constexpr int LDS_TILE = BM * BK;
constexpr double kTallStepUs = 1.22, kPairStepUs = 1.34, kSingleStepUs = 0.8;     // measured, see w4_tile_us
constexpr int kSkinnyRows = 32;     // up to this many activation rows the weight-streaming kernel runs

#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ int lds_off(int row, int chunk) {   // element offset of a 16-byte chunk, 128-byte rows
  return row * BK + ((chunk ^ ((row >> 1) & 7)) << 3);
}

// nibble of a word that holds input e of its eight: the even inputs in nibbles 0..3, the odd ones in nibbles 4..7
__host__ __device__ constexpr int nibble_of(int e) { return e / 2 + 4 * (e % 2); }

// a packed word -> its eight inputs as the bf16 integers nibble - 8, k ascending
__device__ __forceinline__ bf16x8 expand_nibbles(uint32_t w) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // 2^23 + nibble as a float, minus (2^23 + 8): exact
    const float f = __uint_as_float(0x4B000000u | ((w >> (4 * nibble_of(e))) & 15u)) - 8388616.0f;
    o[e] = (bf16)f;
  }
  return o;
}

// A packed word as the bf16 values 16 + nibble = 24 + q, k ascending, without a conversion instruction (those run at
// a quarter of the rate of plain integer instructions here, and sixteen of them per word bound the kernel): in the
// binade [16, 32) a bf16 is 16 (1 + m / 128), so a nibble placed in the four top bits of the mantissa adds exactly
// its value.  The storage format puts two neighbours 16 bits apart, so one shift and one and-or place a pair.  The
// constant 24 is taken out again in fp32: sum_k a_k (24 + q_k) - 24 sum_k a_k, with the second sum from an MFMA
// against ones; the terms are about five times the size of the result, so fp32 loses two or three more bits than
// without the detour, far below what the rounding of the output, or an fp32 test bar of 1e-5, sees.
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t bits) {      // (x & mask) | bits, one instruction
  uint32_t d;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "s"(mask), "v"(bits));
  return d;
}
__device__ __forceinline__ bf16x8 expand_nibbles_plus24(uint32_t w) {
  const uint32_t mask = 0x00780078u, bits = 0x41804180u;
  u32x4 d;
  d[0] = and_or(w << 3, mask, bits);
  d[1] = and_or(w >> 1, mask, bits);
  d[2] = and_or(w >> 5, mask, bits);
  d[3] = and_or(w >> 9, mask, bits);
  return __builtin_bit_cast(bf16x8, d);
}

// QMAX = 7: 4-bit integers -8..7; QMAX = 3: 3-bit integers -4..3 (same nibble storage)
template <int QMAX>
__global__ __launch_bounds__(256) void w4_quantize_kernel(const bf16 *__restrict__ W, int N, int K,
                                                          uint32_t *__restrict__ packed, bf16 *__restrict__ scales) {
  // 16 threads per group of 128 weights, 8 weights (one word) each
  const int groups_per_row = K / GROUP;
  const long long gid = (long long)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int l16 = threadIdx.x & 15;
  if (gid >= (long long)N * groups_per_row) return;
  const int n = (int)(gid / groups_per_row), g = (int)(gid - (long long)n * groups_per_row);
  const bf16x8 w = *(const bf16x8 *)(W + (size_t)n * K + g * GROUP + l16 * 8);
  float m = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf((float)w[e]));
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 16));
  const bf16 scale = (bf16)(m / (float)QMAX);
  const float sf = (float)scale;
  uint32_t word = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float q = sf == 0.f ? 0.f : rintf((float)w[e] / sf);
    q = fminf(fmaxf(q, -(float)(QMAX + 1)), (float)QMAX);
    word |= (uint32_t)((int)q + 8) << (4 * nibble_of(e));
  }
  packed[(size_t)n * (K / 8) + g * 16 + l16] = word;
  if (l16 == 0) scales[gid] = scale;
}

constexpr int EPI_PARTIAL_F32 = ARB_EPI_STORE_F32;   // in a split-K launch split s stores to C + s*M*N

// Epilogue of a 128x128 tile held as 4 waves x (2 x 2) MFMA results (wave (wm, wn) owns rows 64 wm.., columns 64 wn..).
template <int EPI>
__device__ __forceinline__ void w4_tile_epilogue(const f32x16 (&acc)[2][2], void *__restrict__ Cv, int M, int N, int m0,
                                                 int tile_n, int wm, int wn, int frag_row, int frag_half) {
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
              ((float *)Cv)[((size_t)blockIdx.y * M + m) * N + col] = acc[i][j][r];
            } else {
              float *dst = (float *)Cv + (size_t)m * N + col;
              *dst += acc[i][j][r];
            }
          }
        }
      }
  }
}

// The tile kernel.  Every wait is counted by hand: left to the compiler, a turn of this loop held three round trips to
// memory (it waits for all loads in flight before an LDS read that it cannot tell apart from a direct-to-LDS load in
// flight, and a workgroup fence does so in front of each barrier), and a launch of one tile row (up to 128 tokens, one
// workgroup per CU) has nothing else to run meanwhile: 75 us on the 8B gate/up shape whatever the row count.  Here the
// packed weights go to registers six steps ahead and the scales two groups ahead, by inline assembly (the compiler
// keeps no account of them); the activation tile streams two steps ahead into a ring of three LDS stages; the
// fragments are read by inline assembly one MFMA step ahead (the compiler sees neither an LDS read that could meet a
// load in flight nor a load it would have to wait for), and the one wait of a step, in front of its barrier, lets the
// eight requests made since the tile of the next step stay in flight: loads complete in order, so everything older
// has landed.  A register that a load in flight will write is named by the wait that covers it (and by a last wait
// behind the loop): the compiler then neither reads it earlier nor gives it to another value.
// Two heights: 128 rows (WM = 2, four waves, two workgroups per CU) and 256 (WM = 4, eight waves, one per CU).  The taller tile
// expands every weight for twice the rows; what bounds it is the LDS (64x64 per wave: 16 KB of fragment reads per wave and
// step, as many clocks as the MFMAs, plus the stages' writes).  8B gate/up at 484 rows: 174 us in 128-row tiles, 160 in 256-row ones.
// What bounds the 128-row tile is the expansion (exact: two integer instructions, a subtraction and half a conversion per
// weight; without it the 8B gate/up shape at 128 rows takes 41 instead of 59 us, without the MFMAs 56).  The
// conversion-free expansion of the few-token kernel was tried here too (with the row sums from a third MFMA per
// row block and, in a second version, two accumulator sets so that the fold of a group runs between the MFMAs of
// the next): its longer fold (two fused multiply-adds per element and the reads of accumulator registers) costs what
// the expansion saves, 63-67 us.
template <int AOFF, int BOFF>
__device__ __forceinline__ void w4_request_frags(unsigned a_addr, unsigned b_addr, bf16x8 &fa0, bf16x8 &fa1, bf16x8 &fb0,
                                                 bf16x8 &fb1) {
  asm volatile("ds_read_b128 %0, %4 offset:%6\n\tds_read_b128 %1, %4 offset:%7\n\t"
               "ds_read_b128 %2, %5 offset:%8\n\tds_read_b128 %3, %5 offset:%9"
               : "=&v"(fa0), "=&v"(fa1), "=&v"(fb0), "=&v"(fb1)
               : "v"(a_addr + (AOFF & ~0xFFFF)), "v"(b_addr), "n"(AOFF & 0xFFFF), "n"((AOFF & 0xFFFF) + 32 * BK * 2), "n"(BOFF), "n"(BOFF + 32 * BK * 2)
               : "memory");
}
// the requested fragments have landed (and every LDS write of this wave is done); naming them keeps their readers behind
__device__ __forceinline__ void w4_await_frags(bf16x8 &fa0, bf16x8 &fa1, bf16x8 &fb0, bf16x8 &fb1) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fa0), "+v"(fa1), "+v"(fb0), "+v"(fb1) : : "memory");
}

template <int EPI, int WM>
__global__ __launch_bounds__(128 * WM, 2) void gemm_w4_kernel(const bf16 *__restrict__ A, const uint32_t *__restrict__ Bq,
                                                      const bf16 *__restrict__ Bscale, void *__restrict__ Cv, int M,
                                                      int N, int K, int tiles_m, int tiles_n) {
  constexpr int NA = 3, AHEAD_W = 6;                    // activation stages; steps the packed weights are ahead
  constexpr int WAVES = 2 * WM, ROWS = 64 * WM;          // waves (wm, wn) of 64 x 64; tile rows
  constexpr int A_TILE = ROWS * BK;                      // elements of an activation stage
  constexpr int WORDS = 8 / WM;                          // packed words a thread expands per step: 128 rows of 8 over 128 WM threads
  // Two objects: the activation ring only ever sees direct-to-LDS loads and the assembly's reads, so the stores of
  // expanded weights into the other one are not ordered behind loads in flight.
  __shared__ __attribute__((aligned(16))) bf16 Ring[NA * A_TILE], Bs[2 * LDS_TILE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int tile_m, tile_n;
  constexpr int TILE_GROUP = 8 / WM;
  tile_of<TILE_GROUP>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * ROWS;
  const int frag_row = lane & 31, frag_half = lane >> 5;

  // weight row of tile-local B row r.  SwiGLU: wave column r/64, MFMA tile (r%64)/32 (0 = gate, 1 = up),
  // feature offset r%32; N = F there and the up rows follow the F gate rows.
  auto weight_row = [&](int r) {
    if (EPI == ARB_EPI_SWIGLU_BF16) {
      const int f = tile_n * 64 + (r >> 6) * 32 + (r & 31);
      return ((r >> 5) & 1) ? N + f : f;
    }
    return tile_n * BN + r;
  };

  const int ng_all = K / GROUP;
  const int g_begin = split_point(ng_all, blockIdx.y, gridDim.y);
  const int ng = split_point(ng_all, blockIdx.y + 1, gridDim.y) - g_begin;
  const int nk = 2 * ng, last = nk - 1;

  const bf16 *a_src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + 64 * WAVES * i, row = c >> 3, chunk = (c & 7) ^ ((row >> 1) & 7);
    int am = m0 + row;
    am = am < M ? am : M - 1;                            // tail rows re-read the last row; never stored
    a_src[i] = A + (size_t)am * K + (size_t)g_begin * GROUP + chunk * 8;
  }
  const int b_row = tid / WM, b_word = tid % WM * WORDS;  // a thread's weights: WORDS words of one row
  const uint32_t *bq_src = Bq + (size_t)weight_row(b_row) * (K / 8) + (size_t)g_begin * (GROUP / 8) + b_word;
  const bf16 *sc_src[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) sc_src[j] = Bscale + (size_t)weight_row(wn * 64 + j * 32 + frag_row) * (K / GROUP) + g_begin;

  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto dma_a = [&](int stage, int kt) {                  // four wave-wide direct-to-LDS loads
    kt = kt < last ? kt : last;                          // past the range: a valid step, never read
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(a_src[i] + (size_t)kt * BK), LDS_PTR(Ring + stage * A_TILE + (i * WAVES + wave_u) * 512), 16, 0, 0);
  };
  typedef uint32_t words_t __attribute__((ext_vector_type(WORDS)));
  words_t wq[AHEAD_W];                                     // packed weights of steps kt+1 .. kt+6, slot = step % 6
  unsigned sc[3][2];                                     // scales (bf16 bits) of three groups, slot = group % 3
  auto load_w = [&](int slot, int kt) {
    kt = kt < last ? kt : last;
    if constexpr (WM == 2) asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(wq[slot]) : "v"(bq_src + (size_t)kt * (BK / 8)) : "memory");
    else asm volatile("global_load_dwordx2 %0, %1, off" : "=&v"(wq[slot]) : "v"(bq_src + (size_t)kt * (BK / 8)) : "memory");
  };
  auto load_sc = [&](int slot, int g) {
    g = g < ng ? g : ng - 1;
    asm volatile("global_load_ushort %0, %1, off" : "=&v"(sc[slot][0]) : "v"(sc_src[0] + g) : "memory");
    asm volatile("global_load_ushort %0, %1, off" : "=&v"(sc[slot][1]) : "v"(sc_src[1] + g) : "memory");
  };
  auto store_b = [&](int buf, const words_t &w) {
#pragma unroll
    for (int c = 0; c < WORDS; ++c) *(bf16x8 *)&Bs[buf * LDS_TILE + lds_off(b_row, b_word + c)] = expand_nibbles(w[c]);
  };

  // byte addresses of this lane's fragments of MFMA step kk in stage 0: the row block's first row; the second row
  // block, the stage and the operand's array are constant displacements
  unsigned a_addr[4], b_addr[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    a_addr[kk] = (unsigned)(uintptr_t)LDS_PTR(Ring) + 2u * lds_off(wm * 64 + frag_row, kk * 2 + frag_half);
    b_addr[kk] = (unsigned)(uintptr_t)LDS_PTR(Bs) + 2u * lds_off(wn * 64 + frag_row, kk * 2 + frag_half);
  }

  f32x16 acc[2][2], tmp[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = tmp[i][j][r] = 0.f;
  f32x16 zero;                                           // a group's sums start from the MFMA's own zero operand
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;

  // Request order of the prologue = that of the loop: (tile, weights[, scales]) per step, the scales on even steps.
#pragma unroll
  for (int d = 0; d < AHEAD_W - 1; ++d) load_w(d, d);
  load_sc(0, 0);
  load_sc(1, 1);
  asm volatile("" ::: "memory");
  dma_a(0, 0);
  asm volatile("" ::: "memory");
  dma_a(1, 1);
  asm volatile("" ::: "memory");
  load_w(AHEAD_W - 1, AHEAD_W - 1);
  // all but the second tile and the last weights have landed; a wait names the registers whose loads it covers and
  // that are read before the next wait does so, or the compiler could move their readers above it
  asm volatile("s_waitcnt vmcnt(5)" : "+v"(wq[0]), "+v"(wq[1]), "+v"(sc[0][0]), "+v"(sc[0][1]) : : "memory");
  store_b(0, wq[0]);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  bf16x8 fa[2][2], fb[2][2];
  // One step (64 k): u = its position in a turn of six (three groups), so that stage (u % 3), weight stage (u % 2),
  // register set (u % 6) and scale set are fixed per position.
  auto step = [&](auto u_, int kt) {
    constexpr int U = decltype(u_)::value;
    constexpr int SA = (U % NA) * A_TILE * 2, SB = (U % 2) * LDS_TILE * 2;
    dma_a((U + 2) % NA, kt + 2);                         // into the stage step kt-1 was read from
    asm volatile("" ::: "memory");
    load_w(U % AHEAD_W, kt + AHEAD_W);                   // that set went into LDS during step kt-1
    if (U % 2 == 0) load_sc((U / 2 + 2) % 3, (kt >> 1) + 2);
    asm volatile("" ::: "memory");
    w4_request_frags<SA, SB>(a_addr[0], b_addr[0], fa[0][0], fa[0][1], fb[0][0], fb[0][1]);
    const words_t &next_w = wq[(U + 1) % AHEAD_W];
    bf16 *next_b = Bs + ((U + 1) % 2) * LDS_TILE;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      w4_await_frags(fa[kk & 1][0], fa[kk & 1][1], fb[kk & 1][0], fb[kk & 1][1]);
      if (kk == 0) w4_request_frags<SA, SB>(a_addr[1], b_addr[1], fa[1][0], fa[1][1], fb[1][0], fb[1][1]);
      if (kk == 1) w4_request_frags<SA, SB>(a_addr[2], b_addr[2], fa[0][0], fa[0][1], fb[0][0], fb[0][1]);
      if (kk == 2) w4_request_frags<SA, SB>(a_addr[3], b_addr[3], fa[1][0], fa[1][1], fb[1][0], fb[1][1]);
      // the MFMAs stay behind the request (left alone, the scheduler moves them up and the wave then waits out the
      // LDS latency of every request with nothing to do)
      __builtin_amdgcn_sched_barrier(0);
      // a share of the next step's weights per MFMA step: expanded and stored while the matrix pipe runs
      if (kk * WORDS % 4 == 0) {
        constexpr int PER = 4 / WORDS;
        *(bf16x8 *)&next_b[lds_off(b_row, b_word + kk / PER)] = expand_nibbles(next_w[kk / PER]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          tmp[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][i], fb[kk & 1][j], U % 2 == 0 && kk == 0 ? zero : tmp[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (U % 2 == 1) {                                    // end of a group
      const float s0 = __uint_as_float(sc[U / 2][0] << 16), s1 = __uint_as_float(sc[U / 2][1] << 16);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[i][0][r] = fmaf(tmp[i][0][r], s0, acc[i][0][r]);
          acc[i][1][r] = fmaf(tmp[i][1][r], s1, acc[i][1][r]);
        }
    }
    // The tile of step kt+1 was requested at the top of step kt-1; since then: that step's weights, this step's
    // tile and weights, and the scales of whichever of the two steps is even: 1 + 4 + 1 + 2 = 8 requests.
    // Everything older has landed, among it the weights the next step expands and the scales the next step folds in.
    if (U % 2 == 0)
      asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" : "+v"(wq[(U + 2) % AHEAD_W]), "+v"(sc[U / 2][0]), "+v"(sc[U / 2][1]) : : "memory");
    else
      asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" : "+v"(wq[(U + 2) % AHEAD_W]) : : "memory");
    __builtin_amdgcn_s_barrier();
  };
  for (int kt = 0; kt < nk; kt += 6) {
    step(std::integral_constant<int, 0>{}, kt);
    step(std::integral_constant<int, 1>{}, kt + 1);
    if (kt + 2 >= nk) break;
    step(std::integral_constant<int, 2>{}, kt + 2);
    step(std::integral_constant<int, 3>{}, kt + 3);
    if (kt + 4 >= nk) break;
    step(std::integral_constant<int, 4>{}, kt + 4);
    step(std::integral_constant<int, 5>{}, kt + 5);
  }
  // The clamped requests past the end: their registers stay named until they have landed (a register the compiler
  // takes for dead it hands to something else, and a load that lands in it afterwards overwrites that).
  asm volatile("s_waitcnt vmcnt(0)"
               : "+v"(wq[0]), "+v"(wq[1]), "+v"(wq[2]), "+v"(wq[3]), "+v"(wq[4]), "+v"(wq[5]), "+v"(sc[0][0]), "+v"(sc[0][1]),
                 "+v"(sc[1][0]), "+v"(sc[1][1]), "+v"(sc[2][0]), "+v"(sc[2][1])
               : : "memory");
  w4_tile_epilogue<EPI>(acc, Cv, M, N, m0, tile_n, wm, wn, frag_row, frag_half);
}


// Few tokens (M <= 32: drafting token by token): the product only has to stream the packed weights once.  A workgroup
// owns 128 weight rows (SwiGLU: 64 gate rows and the 64 up rows of the same features) and a K range, walked in chunks
// of 256 k, i.e. whole 128-byte lines of packed weights, through a ring of D LDS stages filled by direct-to-LDS loads
// (non-temporal: each weight is used once).  The activations of a chunk are shared by the workgroup; they are four times
// as wide as the weights, so a wave that fetched its own would read as many bytes of them as of weights.  Eight waves,
// two per SIMD: wave (b, g) multiplies rows 32 b.. with group g of the chunk's two, so that expansion and MFMAs of
// different waves overlap; the two group sums meet in LDS at the end.
// 16x16x32 MFMAs, tokens as rows and weights as columns: a lane ends with 4 tokens of one weight row and needs one
// scale per row tile and group.  Within a group lane quarter q owns k = 32 q ..
// 32 q + 31: one 16-byte LDS read of packed weights feeds four MFMAs (the contraction order is free as long as both
// operands agree).  Weights enter the MFMAs as 24 + q (expand_nibbles_plus24); the sums start from -24 sum_k a_k,
// computed once per group for both row tiles by MFMAs against the constant.  One fp32 multiply by the group's scale per
// group, as in the tile kernel.
// An unsplit launch on a narrow matrix would leave most CUs idle that way, so its workgroups are narrower and deal the
// chunks of K to TEAMS teams of waves instead: 4 / TEAMS row blocks and two groups per team, a step of the ring holds a
// chunk of every team, and all sums of a row block meet in LDS at the end.  Above 16 tokens two workgroups of 16 each share the
// rows where that still is at most one workgroup per CU.  The rule (w4_stream_shape) takes the most teams that are at most one workgroup
// per CU.  Measured at 16 / 32 tokens, fp32 output, us, with 1, 2 and 4 teams: 4096x14336 43.2 / 51.3, 24.2 / 24.1, 17.4 / 17.4;
// 1536x8960 28.4 / 33.1, 16.4 / 16.5, 12.3 / 12.2; 6144x4096 15.1 / 17.5, 9.5 / 9.9, 7.7 / 13.2 (384 workgroups);
// 10240x4096 15.1 / 17.7, 9.9 / 12.7 (32 tokens per workgroup), 13.4 / 19.5; 2x8960x1536 with SwiGLU 8.8 / 9.7, 10.7 / 13.4, 13.3 / 21.
// Split launches fill the chip by their splits and keep one team.
// Measured at 16 tokens, 8B shape, weights from memory (before: 32x32 MFMAs, half empty; weights straight to registers in half
// lines; activations and scales per wave): gate/up 26.1 -> 18.5 us (3.3 TB/s), O and down in 8 splits 16.8 -> 10.9 on
// average, QKV in 4 splits 12.2 -> 8.2.  What is left is the start of so short a launch and, per chunk, the expansion.
// Every wait is counted by hand: loads complete in order, so with the loads of D - 2 later chunks in flight the stage
// read next has landed, and its scales, requested before it (those of a later chunk only make the wait longer); the barrier makes that true of every wave's share, and tells that the stage refilled next has been
// read.  The loop is not unrolled over the ring: a workgroup runs 2 to 16 turns, and code that runs once is fetched from memory.
// s_waitcnt immediate that waits for vector memory only (vmcnt in bits 3:0 and 15:14, the other counts at "no wait")
constexpr int vmcnt_imm(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0xF70; }

template <int OFF>
__device__ __forceinline__ void w4s_read(unsigned addr, u32x4 &f) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(f) : "v"(addr), "n"(OFF) : "memory");
}
// two 16-row tiles: their scales, then their packed weights
__device__ __forceinline__ void w4s_read_scales(unsigned addr0, unsigned addr1, unsigned &s0, unsigned &s1) {
  asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %3" : "=&v"(s0), "=&v"(s1) : "v"(addr0), "v"(addr1) : "memory");
}
template <int N>
__device__ __forceinline__ void w4s_await(u32x4 &f0, u32x4 &f1) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f0), "+v"(f1) : "n"(N) : "memory");
}
__device__ __forceinline__ void w4s_await_tiles(unsigned &s0, unsigned &s1, u32x4 &f0, u32x4 &f1) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(s0), "+v"(s1), "+v"(f0), "+v"(f1) : : "memory");
}

template <int EPI, int MT, int D, int TEAMS>
__global__ __launch_bounds__(512, 2) void gemm_w4_stream_kernel(const bf16 *__restrict__ A, const uint32_t *__restrict__ Bq,
                                                                const bf16 *__restrict__ Bscale, void *__restrict__ Cv,
                                                                int M, int N, int K) {
  const size_t part_stride = (size_t)M * N;
  if (gridDim.z > 1) {                                   // this workgroup's tokens
    const int m0 = blockIdx.z * 16 * MT;
    A += (size_t)m0 * K;
    Cv = (char *)Cv + (size_t)m0 * N * (EPI == ARB_EPI_STORE_BF16 || EPI == ARB_EPI_SWIGLU_BF16 ? sizeof(bf16) : sizeof(float));
    M = min(M - m0, 16 * MT);
  }
  constexpr int RT = 2;                                  // 16-row tiles of weights per wave
  constexpr int BLOCKS = 4 / TEAMS, ROWS = 32 * BLOCKS;  // row blocks of 32 per team; weight rows of the workgroup
  constexpr int W_TEAM = ROWS * 128, X_TEAM = MT * 16 * 512;          // bytes of a chunk
  constexpr int W_BYTES = TEAMS * W_TEAM, X_BYTES = TEAMS * X_TEAM, STAGE = W_BYTES + X_BYTES;
  constexpr int S_CHUNKS = 4, S_BLOCK = ROWS * 32;       // chunks whose scales are fetched together; 32 bytes per row
  constexpr int S_BLOCKS = ((D - 1) * TEAMS + 3) / 4 + 1;             // a block is loaded again D - 1 steps before it is read, behind its last reader
  constexpr int LOADS = 2 + MT * TEAMS;                  // per wave and step: weights, activations
  constexpr bool SWIGLU = EPI == ARB_EPI_SWIGLU_BF16;
  static_assert(D >= 3 && D <= 6 && D * STAGE + S_BLOCKS * S_BLOCK <= 160 * 1024 && (D - 2) * LOADS <= 63 &&
                D * STAGE >= 8 * RT * MT * 1024, "ring");
  __shared__ __attribute__((aligned(1024))) char Ring[D * STAGE + S_BLOCKS * S_BLOCK];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, quarter = lane >> 4, block = wave % BLOCKS, grp = wave / BLOCKS % 2, team = wave / (2 * BLOCKS);
  const int member = wave % (2 * BLOCKS);                // of its team

  // this workgroup's chunks, dealt to the teams: step `it` is chunk it TEAMS + team of each; a last chunk of one group (K
  // an odd multiple of 128) reads that group twice and uses it once
  const int ng_all = K / GROUP, nc_all = (ng_all + 1) / 2;
  const int c_begin = split_point(nc_all, blockIdx.y, gridDim.y);
  const int nc = split_point(nc_all, blockIdx.y + 1, gridDim.y) - c_begin, n = (nc + TEAMS - 1) / TEAMS, last = nc - 1;

  auto weight_row = [&](int r) {                         // r < ROWS: 32-row block of a wave, 16-row tile, row
    if (SWIGLU) return (int)blockIdx.x * (ROWS / 2) + (r >> 5) * 16 + (r & 15) + ((r & 16) ? N : 0);
    return (int)blockIdx.x * ROWS + r;
  };
  // Loads of 1 KB: 8 weight rows of 8 pieces (16 bytes), or 2 activation rows of 32.  The pieces of a row are swizzled
  // on the global side so that the fragment reads (16 rows, one piece) cover all banks.  Addresses are a uniform base
  // (every load stays inside one 16-row tile) and a 32-bit lane offset.
  const char *w_base[2];
  unsigned w_off[2], w_off_half[2], x_off[MT * TEAMS], x_off_half[MT * TEAMS];       // _half: the second group's pieces read the first's
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r0 = (member * 2 + i) * 8, piece = (lane & 7) ^ (4 * i + (lane >> 4));
    w_base[i] = (const char *)(Bq + (size_t)weight_row(r0) * (K / 8));
    w_off[i] = (lane >> 3) * (unsigned)(K / 2) + piece * 16;
    w_off_half[i] = (lane >> 3) * (unsigned)(K / 2) + (piece & 3) * 16;
  }
#pragma unroll
  for (int j = 0; j < MT * TEAMS; ++j) {
    const int r = (member + 2 * BLOCKS * j) * 2 + (lane >> 5), piece = (lane & 31) ^ (r & 15);
    const unsigned row = (unsigned)(r < M ? r : M - 1) * (unsigned)(K * 2);         // rows past M re-read the last one; never stored
    x_off[j] = row + piece * 16;
    x_off_half[j] = row + (piece & 15) * 16;
  }
  // Scales are fetched for four chunks at a time, eight dwords of a row (the eight scales may start in the middle of the
  // first): two bytes per row and chunk would cost the address unit as many cache lines as the weights.  Dwords are aligned; an
  // array that starts in the middle of one counts from that dword's start.  Past the row they hold others, not used; past
  // the array's last dword that one is read again.
  const size_t sc_shift = ((uintptr_t)Bscale & 2) / 2;
  const char *sc_base = (const char *)((uintptr_t)Bscale & ~(uintptr_t)3);
  const size_t sc_last = ((size_t)(SWIGLU ? 2 * (size_t)N : (size_t)N) * ng_all + sc_shift - 1) >> 1;
  auto first_scale = [&](int r) { return (size_t)weight_row(r) * ng_all + sc_shift + 2 * c_begin; };
  size_t sc_dword[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) sc_dword[i] = (first_scale((member * 2 + i) * 8 + (lane >> 3)) >> 1) + (lane & 7);
  auto load_scales = [&](int block_of_chunks) {          // the first team's members, for all teams
    char *dst = Ring + D * STAGE + block_of_chunks % S_BLOCKS * S_BLOCK;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      size_t at = sc_dword[i] + block_of_chunks * S_CHUNKS;
      at = at < sc_last ? at : sc_last;
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(sc_base + at * 4), LDS_PTR(dst + (member * 2 + i) * 256), 4, 0, 0);
    }
  };
  auto load = [&](int s, int it) {                       // past the end: the last chunk again, never used
    if (it * TEAMS % S_CHUNKS == 0 && it < n && team == 0) load_scales(it * TEAMS / S_CHUNKS);
    const int at = it * TEAMS + team, c = c_begin + (at < last ? at : last);
    const bool half = 2 * c + 1 >= ng_all;               // a chunk of one group
    char *dst = Ring + s * STAGE + team * W_TEAM, *dst_x = Ring + s * STAGE + W_BYTES + team * X_TEAM;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(w_base[i] + (size_t)c * 128 + (half ? w_off_half[i] : w_off[i])),
                                       LDS_PTR(dst + (member * 2 + i) * 1024), 16, 0, 2 /* nt */);
#pragma unroll
    for (int j = 0; j < MT * TEAMS; ++j)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR((const char *)A + (size_t)c * 512 + (half ? x_off_half[j] : x_off[j])),
                                       LDS_PTR(dst_x + (member + 2 * BLOCKS * j) * 1024), 16, 0, 0);
  };

  // LDS addresses of this lane's fragments in stage 0: row tile 0 of the weights; word w of the activations' token tile 0
  const unsigned ring = (unsigned)(uintptr_t)LDS_PTR(Ring);
  const unsigned w_addr = ring + team * W_TEAM + (block * 32 + c16) * 128 + (((4 * grp + quarter) ^ (c16 >> 1)) << 4);
  unsigned x_addr[4];
  unsigned s_addr[RT], high[RT];                         // address of a scale's dword in block 0, chunk 0; is it the upper half
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int r = block * 32 + i * 16 + c16;
    const unsigned h = (unsigned)(first_scale(r) & 1) + grp;
    s_addr[i] = ring + D * STAGE + r * 32 + (h >> 1) * 4;
    high[i] = h & 1;
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) x_addr[w] = ring + W_BYTES + team * X_TEAM + c16 * 512 + (((16 * grp + 4 * quarter + w) ^ c16) << 4);

  f32x4 acc[RT][MT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 minus24;
#pragma unroll
  for (int e = 0; e < 8; ++e) minus24[e] = (bf16)-24.0f;

#pragma unroll
  for (int s = 0; s < D - 1; ++s)
    if (n > 0) load(s, s);
  int s = 0;
  for (int it = 0; it < n; ++it) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((D - 2) * LOADS));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    load(s == 0 ? D - 1 : s - 1, it + D - 1);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned stage = s * STAGE;
    s = s + 1 == D ? 0 : s + 1;
    const int chunk = it * TEAMS + team;
    // the chunks past the end of the last step, the missing second group of the last chunk
    if ((TEAMS > 1 && chunk > last) || 2 * (c_begin + chunk) + grp >= ng_all) continue;
    u32x4 wf[RT], xf[MT][4];
    unsigned sc[RT];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      w4s_read<0>(x_addr[w] + stage, xf[0][w]);
      if (MT == 2) w4s_read<16 * 512>(x_addr[w] + stage, xf[MT - 1][w]);
    }
    const unsigned sc_at = chunk / S_CHUNKS % S_BLOCKS * S_BLOCK + chunk % S_CHUNKS * 4;
    w4s_read_scales(s_addr[0] + sc_at, s_addr[1] + sc_at, sc[0], sc[1]);
    w4s_read<0>(w_addr + stage, wf[0]);
    w4s_read<16 * 128>(w_addr + stage, wf[1]);
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      w4s_await<4>(xf[j][0], xf[j][1]);
      w4s_await<4>(xf[j][2], xf[j][3]);
    }
    f32x4 base[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      base[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w)
        base[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xf[j][w]), minus24, base[j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    w4s_await_tiles(sc[0], sc[1], wf[0], wf[1]);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      f32x4 sum[MT];
#pragma unroll
      for (int j = 0; j < MT; ++j) sum[j] = base[j];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const bf16x8 q = expand_nibbles_plus24(wf[i][w]);
#pragma unroll
        for (int j = 0; j < MT; ++j)
          sum[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xf[j][w]), q, sum[j], 0, 0, 0);
      }
      const float scale = __uint_as_float(high[i] ? sc[i] & 0xFFFF0000u : sc[i] << 16);
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(sum[j][e], scale, acc[i][j][e]);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  // the 2 TEAMS sums of a row block meet in LDS: every load has landed and, past the barrier, every stage has been read
  __syncthreads();
  f32x4 *red = (f32x4 *)Ring;
  const int share = wave / BLOCKS;                       // 2 team + grp
  if (share > 0) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) red[((wave * RT + i) * MT + j) * 64 + lane] = acc[i][j];
  }
  __syncthreads();
  if (share > 0) return;
#pragma unroll
  for (int o = 1; o < 2 * TEAMS; ++o)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) acc[i][j] += red[(((o * BLOCKS + block) * RT + i) * MT + j) * 64 + lane];
  // D layout of the 16x16 MFMA: lane holds column lane%16 (a weight row) and rows (tokens) 4*(lane/16) + {0..3}
#pragma unroll
  for (int j = 0; j < MT; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = j * 16 + 4 * quarter + e;
      if (m >= M) continue;
      if (SWIGLU) {
        const float gte = acc[0][j][e], up = acc[1][j][e];
        ((bf16 *)Cv)[(size_t)m * N + blockIdx.x * (ROWS / 2) + block * 16 + c16] = (bf16)(gte * __builtin_amdgcn_rcpf(1.0f + __expf(-gte)) * up);
      } else {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const size_t at = (size_t)m * N + blockIdx.x * ROWS + block * 32 + i * 16 + c16;
          if (EPI == ARB_EPI_STORE_BF16) ((bf16 *)Cv)[at] = (bf16)acc[i][j][e];
          else if (EPI == EPI_PARTIAL_F32) ((float *)Cv)[blockIdx.y * part_stride + at] = acc[i][j][e];
          else ((float *)Cv)[at] += acc[i][j][e];
        }
      }
    }
}

// Teams of the streaming kernel and, for more than 16 tokens, whether its workgroups take 16 tokens each (see the kernel).
struct W4Stream { int teams, token_tiles; };
static W4Stream w4_stream_shape(int M, int tiles_n, int splits) {
  const int tokens16 = M <= 16 ? 1 : 2;
  if (splits > 1) return {1, 1};
  if (tiles_n * 4 * tokens16 <= 256) return {4, tokens16};
  if (tiles_n * 2 * tokens16 <= 256) return {2, tokens16};
  return {tiles_n * 2 <= 256 ? 2 : 1, 1};
}

}  // namespace

arb_status launch_w4_quantize(const bf16 *W, int N, int K, uint32_t *packed, bf16 *scales, int bits, hipStream_t st) {
  if (N == 0) return ARB_OK;
  if (bits != 3 && bits != 4) return arb_fail(ARB_EUNSUPPORTED, "weight quantization to %d bits (3 or 4)", bits);
  if (N < 0 || K <= 0 || K % GROUP != 0) return arb_fail(ARB_EUNSUPPORTED, "w4_quantize: N=%d, K=%d (K must be a multiple of %d)", N, K, GROUP);
  const long long groups = (long long)N * (K / GROUP);
  const dim3 grid((unsigned)((groups + 15) / 16)), block(256);
  if (bits == 4) hipLaunchKernelGGL(w4_quantize_kernel<7>, grid, block, 0, st, W, N, K, packed, scales);
  else hipLaunchKernelGGL(w4_quantize_kernel<3>, grid, block, 0, st, W, N, K, packed, scales);
  ARB_CHECK_LAUNCH("w4_quantize");
  return ARB_OK;
}

// Time estimates in us of the two tile kernels, from which the number of K splits and the kernel are chosen: steps of 64 k
// times the time per step measured with one workgroup per CU, or with two (128-row tiles; 256-row tiles only fit once),
// and what fp32 partial products cost to write here and read in the consumer.
static double w4_tile_us(int M, int tiles_n, int K, int splits, bool tall) {
  const int wgs = ceil_div(M, tall ? 2 * BM : BM) * tiles_n * splits, steps = 2 * ceil_div(K / GROUP, splits);
  double step;
  if (tall) step = ceil_div(wgs, 256) * kTallStepUs;
  else step = wgs / 512 * kPairStepUs + (wgs % 512 == 0 ? 0.0 : wgs % 512 <= 256 ? kSingleStepUs : kPairStepUs);
  return step * steps + 5.0 + (double)M * tiles_n * BN * 4 * (2 * splits - 2) / 5.0e6;
}
static bool w4_tall(int M, int tiles_n, int K, int splits) {
  return M > BM && w4_tile_us(M, tiles_n, K, splits, true) < w4_tile_us(M, tiles_n, K, splits, false);
}

int gemm_w4_splits(int M, int N, int K, int max_splits) {
  int best = 1;
  double best_us = 0.0;
  for (int s = 1; s <= max_splits && (s == 1 || K / GROUP / s >= 4); ++s) {
    double us = w4_tile_us(M, N / BN, K, s, false);
    if (M > BM) us = fmin(us, w4_tile_us(M, N / BN, K, s, true));
    if (s == 1 || us < best_us) { best = s; best_us = us; }
  }
  return best;
}

arb_status launch_gemm_w4(const bf16 *A, const uint32_t *Bq, const bf16 *Bscale, void *C, int M, int N, int K,
                          int epilogue, hipStream_t st, int splits) {
  if (M == 0) return ARB_OK;
  if (M < 0 || N <= 0 || K <= 0) return arb_fail(ARB_EINVAL, "gemm_w4: M=%d N=%d K=%d", M, N, K);
  if (K % GROUP != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm_w4: K=%d is not a multiple of %d", K, GROUP);
  const int tiles_m = ceil_div(M, BM);
  int tiles_n;
  if (epilogue == ARB_EPI_SWIGLU_BF16) {
    if (N % 64 != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm_w4: SwiGLU width %d is not a multiple of 64", N);
    tiles_n = N / 64;
  } else {
    if (N % BN != 0) return arb_fail(ARB_EUNSUPPORTED, "gemm_w4: N=%d is not a multiple of %d", N, BN);
    tiles_n = N / BN;
  }
  if (splits > 1 && epilogue != ARB_EPI_RESIDUAL_F32 && epilogue != ARB_EPI_STORE_F32)
    return arb_fail(ARB_EINVAL, "gemm_w4: split-K needs an fp32 epilogue (partial products)");
  if (splits < 1 || splits > K / GROUP) return arb_fail(ARB_EINVAL, "gemm_w4: %d splits of %d groups", splits, K / GROUP);
  const bool skinny = M <= kSkinnyRows;                // few tokens: the weight-streaming kernel
  const bool tall = !skinny && w4_tall(M, tiles_n, K, splits);
  const int tall_m = ceil_div(M, 2 * BM);
  const W4Stream stream = skinny ? w4_stream_shape(M, tiles_n, splits) : W4Stream{1, 1};
  const int mt = M <= 16 || stream.token_tiles == 2 ? 1 : 2;       // 16-token tiles of a streaming workgroup
  const dim3 grid((tall ? tall_m : tiles_m) * tiles_n * stream.teams, splits, stream.token_tiles), block(skinny || tall ? 512 : 256);
#define ARB_W4(E)                                                                                                    \
  do {                                                                                                               \
    if (skinny && mt == 1 && stream.teams == 4)                                                                      \
      hipLaunchKernelGGL((gemm_w4_stream_kernel<E, 1, 3, 4>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K);       \
    else if (skinny && mt == 1 && stream.teams == 2)                                                                 \
      hipLaunchKernelGGL((gemm_w4_stream_kernel<E, 1, 4, 2>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K);       \
    else if (skinny && mt == 1)                                                                                      \
      hipLaunchKernelGGL((gemm_w4_stream_kernel<E, 1, 6, 1>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K);       \
    else if (skinny && stream.teams == 2)                                                                            \
      hipLaunchKernelGGL((gemm_w4_stream_kernel<E, 2, 3, 2>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K);       \
    else if (skinny)                                                                                                 \
      hipLaunchKernelGGL((gemm_w4_stream_kernel<E, 2, 4, 1>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K);       \
    else if (tall)                                                                                                   \
      hipLaunchKernelGGL((gemm_w4_kernel<E, 4>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K, tall_m, tiles_n);    \
    else hipLaunchKernelGGL((gemm_w4_kernel<E, 2>), grid, block, 0, st, A, Bq, Bscale, C, M, N, K, tiles_m, tiles_n); \
  } while (0)
  switch (epilogue) {
    case ARB_EPI_STORE_BF16: ARB_W4(ARB_EPI_STORE_BF16); break;
    case ARB_EPI_RESIDUAL_F32:
      if (splits > 1) ARB_W4(EPI_PARTIAL_F32); else ARB_W4(ARB_EPI_RESIDUAL_F32);
      break;
    case ARB_EPI_SWIGLU_BF16: ARB_W4(ARB_EPI_SWIGLU_BF16); break;
    case ARB_EPI_STORE_F32: ARB_W4(ARB_EPI_STORE_F32); break;
    default: return arb_fail(ARB_EINVAL, "gemm_w4: unknown epilogue %d", epilogue);
  }
#undef ARB_W4
  ARB_CHECK_LAUNCH("gemm_w4");
  return ARB_OK;
}
