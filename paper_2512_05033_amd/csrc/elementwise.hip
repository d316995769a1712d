// Row-wise and per-token kernels of the step-scoring forward: token metadata
// (position, pool slot), rotary table, embedding gather + RMSNorm, RMSNorm,
// rotary embedding + KV append, final RMSNorm + head dot, segmented pooling +
// threshold.  All are HBM-bound and touch T*d elements a handful of times.
#include "common.h"

// ------------------------------------------------------------------ reductions

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum over a block of 256 threads; every thread gets the result.
__device__ __forceinline__ float block_sum_256(float v, float *lds4) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds4[w] = v;
  __syncthreads();
  return lds4[0] + lds4[1] + lds4[2] + lds4[3];
}

// ---------------------------------------------------------------- token metadata

// The attention work list: for every sequence, split, kv head and query tile that has a visible key one AttnItem, and
// nothing else, so that every workgroup of an attention launch has work.  (The launch used to be the full product
// of batch, most splits and most query tiles; on ragged batches half of its workgroups returned at once, but they took
// their turn in the order in which workgroups are handed to the CUs, which left the working ones unevenly
// spread: 64 contexts of 1 K to 16 K on the 1.5B shape 496 -> 306 us per layer, 32 of 4 K to 32 K on the 8B shape with
// steps of 1 and 64 tokens 613 -> 522.)  Sequences with the longest splits come first, so that a launch ends on
// short ones; the query tiles of a (sequence, split, kv head) are neighbours, the ones that see most keys first.
// Blocks [0, n_parts) each know the whole order and write every n_parts-th run of 256 items.
// The launch is sized by the host's copy of the lengths and the list is written from the device's.  Where the two disagree
// nothing is written or read out of range: the list ends at n_items, places that no item claims hold an empty one (its
// workgroup returns), and splits beyond the max_splits that the partial results have room for are empty too.
constexpr int kListSeqs = 512;             // sequences ordered at a time, two per thread

// Items of a sequence with context p + s cut into parts of c keys: every split that starts inside the prefix has all nq
// query tiles, the few that start inside the step have those whose last row sees their first key.
__device__ __forceinline__ int attention_item_count(int p, int s, int c, int G, int Hkv) {
  const int nq = (s * G + ATTN_QROWS - 1) / ATTN_QROWS, in_prefix = p / c + 1;
  int tiles = in_prefix * nq;
  for (int begin = in_prefix * c; begin < p + s; begin += c) tiles += nq - attn_first_qtile(p, G, begin);
  return tiles * Hkv;
}

__device__ void write_attention_items(const int32_t *__restrict__ prefix_lens, const int32_t *__restrict__ cu, int batch,
                                      int G, int Hkv, int kv_chunk, int max_splits, AttnItem *__restrict__ items,
                                      int n_items, int part, int n_parts) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  __shared__ i32x4 key4[kListSeqs / 4];
  __shared__ int first[kListSeqs], prefix[kListSeqs], step[kListSeqs], order[kListSeqs];
  __shared__ int ends[kListSeqs], wave_total[4];           // ends: inclusive sums of the ordered item counts
  int *key = (int *)key4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int written = 0;
  for (int base = 0; base < batch; base += kListSeqs) {
    const int n = min(kListSeqs, batch - base);
    for (int i = tid; i < n; i += 256) {
      const int p = max(prefix_lens[base + i], 0), t0 = cu[base + i], s = max(cu[base + i + 1] - t0, 0);
      prefix[i] = p;
      first[i] = t0;
      step[i] = s;
      key[i] = s > 0 ? attn_seq_chunk(p + s, kv_chunk) : ATTN_KT;        // without a step: no items
    }
    if (tid < 16 && n + tid < kListSeqs) key[n + tid] = 0;               // below every key: the ranks are counted sixteen at a time
    __syncthreads();
    for (int i = tid; i < n; i += 256) {
      const int k = key[i];
      int rank = 0;
      // (one key per LDS read, each waited for, made this loop the longest part of the opening launch: 200 sequences 13 us)
      for (int j = 0; j < n; j += 16) {
        i32x4 other[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) other[q] = key4[j / 4 + q];
#pragma unroll
        for (int e = 0; e < 16; ++e) rank += other[e / 4][e % 4] > k || (other[e / 4][e % 4] == k && j + e < i);
      }
      order[rank] = i;
    }
    __syncthreads();
    int count[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (2 * tid + e < n) {
        const int i = order[2 * tid + e];
        count[e] = attention_item_count(prefix[i], step[i], key[i], G, Hkv);
      }
    int sum = count[0] + count[1];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(sum, o, 64);
      if (lane >= o) sum += up;
    }
    if (lane == 63) wave_total[wave] = sum;
    __syncthreads();
    for (int w = 0; w < wave; ++w) sum += wave_total[w];
    ends[2 * tid] = sum - count[1];
    ends[2 * tid + 1] = sum;
    __syncthreads();
    const int total = min(ends[n - 1], n_items - written);
    for (int l = part * 256 + tid; l < total; l += n_parts * 256) {
      int lo = 0, hi = n - 1;                              // first r with ends[r] > l
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ends[mid] > l) hi = mid; else lo = mid + 1;
      }
      const int i = order[lo], p = prefix[i], s = step[i], c = key[i], rows = s * G;
      const int nq = (rows + ATTN_QROWS - 1) / ATTN_QROWS;
      const int j0 = lo ? l - ends[lo - 1] : l;
      int split = min(j0 / (nq * Hkv), p / c), j = j0 - split * nq * Hkv, per;
      for (;; ++split) {
        per = nq - attn_first_qtile(p, G, split * c);      // query tiles of this split, the last ones of the sequence
        if (j < per * Hkv) break;
        j -= per * Hkv;
      }
      const int hk = j / per, row0 = (nq - 1 - (j - hk * per)) * ATTN_QROWS;
      const int visible = p + (min(rows, row0 + ATTN_QROWS) - 1) / G + 1;          // keys any row of the tile may see
      items[written + l] = split < max_splits
                               ? AttnItem{base + i, first[i], p, s, row0, split * c, min(visible, split * c + c), split << 16 | hk}
                               : AttnItem{};
    }
    written += total;
    __syncthreads();
  }
  for (int l = written + part * 256 + tid; l < n_items; l += n_parts * 256) items[l] = AttnItem{};
}

// For step token j of sequence b at position pos = p_b + i:
//   slot = block_tables[b][pos / blk] * blk + pos % blk.
struct TokenMeta {
  const int32_t *prefix_lens, *cu, *tables;
  int batch, max_blocks, blk;
  int32_t *tok_pos, *tok_slot;
  int list_blocks, kv_chunk, max_splits, n_items, G, Hkv;       // blocks of the launch that write the attention work list (0: there is none)
  AttnLists lists;
};

// -> the token's position; with `write` also stores what the later kernels read about it
__device__ __forceinline__ int token_meta(const TokenMeta &t, int j, bool write) {
  int lo = 0, hi = t.batch;               // largest b with cu[b] <= j
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (t.cu[mid] <= j) lo = mid; else hi = mid;
  }
  const int b = lo, prefix = t.prefix_lens[b], t0 = t.cu[b], pos = prefix + (j - t0);
  if (write) {
    if (t.tok_pos) t.tok_pos[j] = pos;
    if (t.tok_slot) t.tok_slot[j] = t.tables[(size_t)b * t.max_blocks + pos / t.blk] * t.blk + pos % t.blk;
    if (t.lists.tok_splits) t.lists.tok_splits[j] = min(pos / attn_seq_chunk(prefix + t.cu[b + 1] - t0, t.kv_chunk) + 1, t.max_splits);
  }
  return pos;
}

// The first list_blocks blocks write the attention work list.
__global__ __launch_bounds__(256) void token_meta_kernel(TokenMeta t, int T) {
  if ((int)blockIdx.x < t.list_blocks) {
    write_attention_items(t.prefix_lens, t.cu, t.batch, t.G, t.Hkv, t.kv_chunk, t.max_splits, t.lists.items, t.n_items, blockIdx.x,
                          t.list_blocks);
    return;
  }
  const int j = (blockIdx.x - t.list_blocks) * 256 + threadIdx.x;
  if (j < T) token_meta(t, j, true);
}

static TokenMeta token_meta_args(const int32_t *prefix_lens, const int32_t *cu_step_lens, const int32_t *block_tables,
                                 int batch, int max_blocks_per_seq, int kv_block, int32_t *tok_pos, int32_t *tok_slot,
                                 const AttnPlan *plan, AttnLists lists, int G, int n_kv_heads) {
  const int list_blocks = !plan || plan->n_items == 0 ? 0 : plan->n_items <= 1024 ? 1 : plan->n_items <= 16384 ? ceil_div(plan->n_items, 1024) : 16;
  return TokenMeta{prefix_lens, cu_step_lens, block_tables, batch, max_blocks_per_seq, kv_block, tok_pos, tok_slot,
                   list_blocks, plan ? plan->kv_chunk : ATTN_KT, plan ? plan->max_splits : 1, plan ? plan->n_items : 0, G,
                   n_kv_heads, lists};
}

arb_status launch_token_meta(const int32_t *prefix_lens, const int32_t *cu_step_lens, const int32_t *block_tables,
                             int batch, int total_tokens, int max_blocks_per_seq, int kv_block, int32_t *tok_pos,
                             int32_t *tok_slot, hipStream_t st, const AttnPlan *plan, AttnLists lists, int G, int n_kv_heads) {
  if (total_tokens == 0) return ARB_OK;
  const TokenMeta t = token_meta_args(prefix_lens, cu_step_lens, block_tables, batch, max_blocks_per_seq, kv_block, tok_pos,
                                      tok_slot, plan, lists, G, n_kv_heads);
  hipLaunchKernelGGL(token_meta_kernel, dim3(ceil_div(total_tokens, 256) + t.list_blocks), dim3(256), 0, st, t, total_tokens);
  ARB_CHECK_LAUNCH("token_meta");
  return ARB_OK;
}

// ------------------------------------------------------------- debug: id range check

// err[0]: bit 0 = a token id outside [0, vocab), bit 1 = a referenced block id outside [0, n_blocks);
// err[1] / err[2]: smallest offending index into token_ids / block_tables (INT32_MAX: none).
__global__ void check_ids_init_kernel(int32_t *err) {
  err[0] = 0;
  err[1] = err[2] = INT32_MAX;
  err[3] = 0;
}

// One thread per token id, then one per block-table entry.  Entry j of row b is referenced iff
// j < ceil((p_b + s_b) / blk); the rest of a row may hold anything.
__global__ void check_ids_kernel(const int32_t *__restrict__ token_ids, int T, int vocab,
                                 const int32_t *__restrict__ tables, int batch, int max_blocks,
                                 const int32_t *__restrict__ prefix_lens, const int32_t *__restrict__ cu, int blk,
                                 int n_blocks, int32_t *err) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < T) {
    if (token_ids) {
      const int id = token_ids[i];
      if (id < 0 || id >= vocab) {
        atomicOr(&err[0], 1);
        atomicMin(&err[1], (int)i);
      }
    }
    return;
  }
  const long long e = i - T;
  if (e >= (long long)batch * max_blocks) return;
  const int b = (int)(e / max_blocks), j = (int)(e - (long long)b * max_blocks);
  const int ctx = prefix_lens[b] + cu[b + 1] - cu[b];
  if (j >= (ctx + blk - 1) / blk) return;
  const int id = tables[e];
  if (id < 0 || id >= n_blocks) {
    atomicOr(&err[0], 2);
    atomicMin(&err[2], (int)e);
  }
}

arb_status launch_check_ids(const int32_t *token_ids, int T, int vocab, const int32_t *block_tables, int batch,
                            int max_blocks_per_seq, const int32_t *prefix_lens, const int32_t *cu_step_lens,
                            int kv_block, int n_blocks, int32_t *err, hipStream_t st) {
  hipLaunchKernelGGL(check_ids_init_kernel, dim3(1), dim3(1), 0, st, err);
  ARB_CHECK_LAUNCH("check_ids_init");
  const long long n = (long long)T + (long long)batch * max_blocks_per_seq;
  hipLaunchKernelGGL(check_ids_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, token_ids, T, vocab,
                     block_tables, batch, max_blocks_per_seq, prefix_lens, cu_step_lens, kv_block, n_blocks, err);
  ARB_CHECK_LAUNCH("check_ids");
  return ARB_OK;
}

// -------------------------------------------------------------------- rotary table

// cs[j][t] = (cos, sin) of pos_j * base^(-2t/hd), evaluated in fp64 so that the
// fp32 table is correctly rounded even at positions of tens of thousands.
__device__ __forceinline__ f32x2 rope_cos_sin(int pos, int t, int half, double log2_base) {
  const double inv_freq = exp2(-(double)t / (double)half * log2_base);
  double s, c;
  sincos((double)pos * inv_freq, &s, &c);
  return f32x2{(float)c, (float)s};
}

__global__ void rope_table_kernel(const int32_t *__restrict__ tok_pos, int T, int half, double log2_base,
                                  f32x2 *__restrict__ cs) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= T * half) return;
  const int j = idx / half, t = idx - j * half;
  cs[idx] = rope_cos_sin(tok_pos[j], t, half, log2_base);
}

arb_status launch_rope_table(const int32_t *tok_pos, int total_tokens, int head_dim, float rope_base, f32x2 *cs,
                             hipStream_t st) {
  const int half = head_dim / 2, n = total_tokens * half;
  if (n == 0) return ARB_OK;
  hipLaunchKernelGGL(rope_table_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, tok_pos, total_tokens, half,
                     log2((double)rope_base), cs);
  ARB_CHECK_LAUNCH("rope_table");
  return ARB_OK;
}

// ------------------------------------------------------------------------ RMSNorm

// One block of 256 threads per row; a row is held in registers between the sum-of-squares pass and the scaling
// pass: VECS groups of eight elements per thread (1, 2 or 4, the fewest that hold the row, so that the registers of
// a narrow row do not cost resident waves).  With few rows the kernel is one chain of memory round trips; the gains are
// asked for together with the row, not behind the reduction (16 rows of 1536: 4.2 -> 3.5 us).
#define ROW_VECS 4         // the most

// With partial products the row is first completed by those of the preceding residual projection (their number may
// differ between its head and its tail rows): h = h_in + sum_s parts[s] (fixed order), and written back through
// h_out when that is not null.
// The EMBED launch opens a pass: the row is a token's embedding, and the block also finds the token's position and pool
// slot and its row of the rotary table; its first blocks write the attention work list.  (Three launches before, all of
// them short chains of dependent loads: together 9 to 20 us of a pass, and the gaps between them.)
struct PassOpening {
  TokenMeta meta;
  double log2_base;
  int half;                  // head_dim / 2
  f32x2 *cs;
};

template <bool EMBED, bool HEAD, int VECS>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float *h_in, const float *__restrict__ parts,
                                                      RowParts row_parts, size_t part_stride,
                                                      const bf16 *__restrict__ embed,
                                                      const int32_t *__restrict__ token_ids,
                                                      const float *__restrict__ g, float eps, int d,
                                                      float *h_out, bf16 *__restrict__ x_out,
                                                      const float *__restrict__ w_head,
                                                      const float *__restrict__ w_head1, float *__restrict__ tok_dot,
                                                      PassOpening opening) {
  __shared__ float red[4];
  const int tid = threadIdx.x;
  int row = blockIdx.x;
  if (EMBED) {
    const TokenMeta &m = opening.meta;
    if (row < m.list_blocks) {
      write_attention_items(m.prefix_lens, m.cu, m.batch, m.G, m.Hkv, m.kv_chunk, m.max_splits, m.lists.items, m.n_items, row,
                            m.list_blocks);
      return;
    }
    row -= m.list_blocks;
  }
  const int n_parts = row < row_parts.row ? row_parts.head : row_parts.tail;
  float v[VECS][8];
  f32x4 gain[VECS][2];
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < VECS; ++it) {
    const int c = (it * 256 + tid) * 8;
    if (c < d) {
      gain[it][0] = *(const f32x4 *)(g + c);
      gain[it][1] = *(const f32x4 *)(g + c + 4);
      if (EMBED) {
        const bf16x8 e = *(const bf16x8 *)(embed + (size_t)token_ids[row] * d + c);
#pragma unroll
        for (int k = 0; k < 8; ++k) v[it][k] = (float)e[k];
        float *dst = h_out + (size_t)row * d + c;
        *(f32x4 *)dst = f32x4{v[it][0], v[it][1], v[it][2], v[it][3]};
        *(f32x4 *)(dst + 4) = f32x4{v[it][4], v[it][5], v[it][6], v[it][7]};
      } else {
        const float *src = h_in + (size_t)row * d + c;
        f32x4 a = *(const f32x4 *)src, b = *(const f32x4 *)(src + 4);
        if (n_parts > 0) {
          // The loads of all partial products go out together (a loop over a run-time count waits for each before it asks for
          // the next); the sums keep the fixed order.
          const float *p0 = parts + (size_t)row * d + c;
#define ARB_ADD_PARTS(NP)                                                      \
  {                                                                            \
    f32x4 pa[NP], pb[NP];                                                      \
    _Pragma("unroll") for (int sp = 0; sp < NP; ++sp) {                        \
      pa[sp] = *(const f32x4 *)(p0 + sp * part_stride);                        \
      pb[sp] = *(const f32x4 *)(p0 + sp * part_stride + 4);                    \
    }                                                                          \
    _Pragma("unroll") for (int sp = 0; sp < NP; ++sp) { a += pa[sp]; b += pb[sp]; } \
  }
          switch (n_parts) {
            case 1: ARB_ADD_PARTS(1) break;
            case 2: ARB_ADD_PARTS(2) break;
            case 3: ARB_ADD_PARTS(3) break;
            case 4: ARB_ADD_PARTS(4) break;
            case 5: ARB_ADD_PARTS(5) break;
            case 6: ARB_ADD_PARTS(6) break;
            case 7: ARB_ADD_PARTS(7) break;
            case 8: ARB_ADD_PARTS(8) break;
            default:
              for (int sp = 0; sp < n_parts; ++sp) {
                a += *(const f32x4 *)(p0 + sp * part_stride);
                b += *(const f32x4 *)(p0 + sp * part_stride + 4);
              }
          }
#undef ARB_ADD_PARTS
          if (h_out) {                          // the last norm of a pass has no later reader of h
            float *dst = h_out + (size_t)row * d + c;
            *(f32x4 *)dst = a;
            *(f32x4 *)(dst + 4) = b;
          }
        }
        v[it][0] = a[0]; v[it][1] = a[1]; v[it][2] = a[2]; v[it][3] = a[3];
        v[it][4] = b[0]; v[it][5] = b[1]; v[it][6] = b[2]; v[it][7] = b[3];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) ss += v[it][k] * v[it][k];
    }
  }
  if (EMBED) {
    const int pos = token_meta(opening.meta, row, tid == 0);
    for (int t = tid; t < opening.half; t += 256) opening.cs[(size_t)row * opening.half + t] = rope_cos_sin(pos, t, opening.half, opening.log2_base);
  }
  ss = block_sum_256(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)d + eps);
  float dot = 0.f;
#pragma unroll
  for (int it = 0; it < VECS; ++it) {
    const int c = (it * 256 + tid) * 8;
    if (c < d) {
      const f32x4 g0 = gain[it][0], g1 = gain[it][1];
      float y[8];
#pragma unroll
      for (int k = 0; k < 4; ++k) { y[k] = v[it][k] * r * g0[k]; y[4 + k] = v[it][4 + k] * r * g1[k]; }
      if (HEAD && w_head) {
        f32x4 w0 = *(const f32x4 *)(w_head + c), w1 = *(const f32x4 *)(w_head + c + 4);
        if (w_head1) {           // two-class head: only the difference of the class logits matters (class 1 minus class 0)
          w0 = *(const f32x4 *)(w_head1 + c) - w0;
          w1 = *(const f32x4 *)(w_head1 + c + 4) - w1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) dot += y[k] * w0[k] + y[4 + k] * w1[k];
      }
      if (x_out) {
        bf16x8 o;
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = (bf16)y[k];
        *(bf16x8 *)(x_out + (size_t)row * d + c) = o;
      }
    }
  }
  if (HEAD && tok_dot) {
    dot = block_sum_256(dot, red);
    if (tid == 0) tok_dot[row] = dot;
  }
}

// launches rmsnorm_kernel<EMBED, HEAD, VECS> for rows of d elements
#define ARB_LAUNCH_NORM(EMBED, HEAD, GRID, ...)                                                                            \
  do {                                                                                                                    \
    if (d <= 2048) hipLaunchKernelGGL((rmsnorm_kernel<EMBED, HEAD, 1>), dim3(GRID), dim3(256), 0, st, __VA_ARGS__);        \
    else if (d <= 4096) hipLaunchKernelGGL((rmsnorm_kernel<EMBED, HEAD, 2>), dim3(GRID), dim3(256), 0, st, __VA_ARGS__);   \
    else hipLaunchKernelGGL((rmsnorm_kernel<EMBED, HEAD, ROW_VECS>), dim3(GRID), dim3(256), 0, st, __VA_ARGS__);           \
  } while (0)

static arb_status check_row_width(int d) {
  if (d <= 0 || d % 8 != 0 || d > 256 * 8 * ROW_VECS)
    return arb_fail(ARB_EUNSUPPORTED, "row width %d: need a multiple of 8 up to %d", d, 256 * 8 * ROW_VECS);
  return ARB_OK;
}

arb_status launch_open_pass(const bf16 *embed, const int32_t *token_ids, const float *g, float eps, int T, int d, float *h,
                            bf16 *x, const int32_t *prefix_lens, const int32_t *cu_step_lens, const int32_t *block_tables,
                            int batch, int max_blocks_per_seq, int kv_block, int32_t *tok_slot, float rope_base, int head_dim,
                            f32x2 *cs, const AttnPlan &plan, AttnLists lists, int G, int n_kv_heads, hipStream_t st) {
  if (T == 0) return ARB_OK;
  if (arb_status s = check_row_width(d)) return s;
  const PassOpening o{token_meta_args(prefix_lens, cu_step_lens, block_tables, batch, max_blocks_per_seq, kv_block, nullptr,
                                      tok_slot, &plan, lists, G, n_kv_heads),
                      log2((double)rope_base), head_dim / 2, cs};
  ARB_LAUNCH_NORM(true, false, T + o.meta.list_blocks, (const float *)nullptr,
                     (const float *)nullptr, RowParts{}, (size_t)0, embed, token_ids, g, eps, d, h, x, (const float *)nullptr,
                     (const float *)nullptr, (float *)nullptr, o);
  ARB_CHECK_LAUNCH("open_pass");
  return ARB_OK;
}

arb_status launch_rmsnorm(float *h, const float *parts, RowParts n_parts, const float *g, float eps, int T, int d, bf16 *x,
                          hipStream_t st) {
  if (T == 0) return ARB_OK;
  if (arb_status s = check_row_width(d)) return s;
  ARB_LAUNCH_NORM(false, false, T, (const float *)h, parts, n_parts,
                     (size_t)T * d, (const bf16 *)nullptr, (const int32_t *)nullptr, g, eps, d, h, x,
                     (const float *)nullptr, (const float *)nullptr, (float *)nullptr, PassOpening{});
  ARB_CHECK_LAUNCH("rmsnorm");
  return ARB_OK;
}

arb_status launch_final_norm_head(const float *h, const float *parts, RowParts n_parts, const float *g, float eps, int T,
                                  int d, const float *w_head, const float *w_head1, bf16 *hidden_out, float *tok_dot,
                                  hipStream_t st) {
  if (T == 0) return ARB_OK;
  if (arb_status s = check_row_width(d)) return s;
  // the residual stream is not needed after the last norm, so the completed row is not written back
  ARB_LAUNCH_NORM(false, true, T, h, parts, n_parts, (size_t)T * d,
                     (const bf16 *)nullptr, (const int32_t *)nullptr, g, eps, d, (float *)nullptr, hidden_out, w_head,
                     w_head1, tok_dot, PassOpening{});
  ARB_CHECK_LAUNCH("final_norm_head");
  return ARB_OK;
}

// ------------------------------------------------------- rotary embedding + KV append

// One block per token and 256 work units.  A unit is (head, UNIT adjacent pair indices t..):
// it reads u[t..] and u[t+half..] of that head, rotates q and k heads
// by the token's table row ((a, b) -> (a cos - b sin, b cos + a sin)), writes q
// (bf16) to the qkv row and k, v (bf16) to the token's slot of the pool
// [n_blocks, Hkv, 16, hd].  With PARTS the projection comes as fp32 split-K partial
// products that are added up here (fixed order), so q and k are rounded once; a row of qkv then only holds
// the query heads.  row_heads: heads per row of qkv.
// Many tokens are bound by memory: four pairs, 16-byte loads of the fp32 products (against two pairs and 8-byte loads, us
// per layer: 8B shape 512 tokens 11.0 -> 10.1, 1040 tokens in several splits 13.8 -> 12.4, 4096 tokens 35.0 -> 30.2; 1.5B shape
// 4096 tokens 15.8 -> 15.3).  Few tokens are a chain of dependent loads whose length the width of a unit does not change.
// (With bf16 products to read, 4096 tokens of the 8B shape took 25.3.)
template <bool PARTS, int UNIT>
__global__ __launch_bounds__(256) void rope_append_kernel(bf16 *__restrict__ qkv, const float *__restrict__ parts,
                                                          RowParts row_parts, size_t part_stride,
                                                          const f32x2 *__restrict__ cs,
                                                          const int32_t *__restrict__ tok_slot,
                                                          bf16 *__restrict__ k_pool, bf16 *__restrict__ v_pool,
                                                          int Hq, int Hkv, int hd, float q_scale, int row_heads) {
  typedef float vec_f __attribute__((ext_vector_type(UNIT)));
  typedef bf16 vec_b __attribute__((ext_vector_type(UNIT)));
  const int j = blockIdx.x;
  const int n_parts = j < row_parts.row ? row_parts.head : row_parts.tail;
  const int half = hd / 2, units_per_head = half / UNIT, n_heads = Hq + 2 * Hkv;
  bf16 *row = qkv + (size_t)j * row_heads * hd;
  const float *prow = PARTS ? parts + (size_t)j * n_heads * hd : nullptr;
  const int slot = tok_slot[j];
  const size_t blk = slot / ARB_KV_BLOCK, off = slot % ARB_KV_BLOCK;
  // one unit per thread: blockIdx.y walks the units of the token in groups of 256, so that a token's row is
  // one round of memory latency whatever its width (a loop over the units took one round per 256 of them,
  // 6 rounds per token on the 8B shape: most of the kernel's time in small batches)
  const int u = blockIdx.y * blockDim.x + threadIdx.x;
  if (u < n_heads * units_per_head) {
    const int head = u / units_per_head, t = (u - head * units_per_head) * UNIT;
    bf16 *src = row + head * hd;
    vec_f a, b;
    if (PARTS) {
      // up to eight partial products are asked for together (a loop over a run-time count waits for each before it asks
      // for the next: 16 tokens of the 1.5B shape, 4 partial products, 3.9 -> 3.4 us); the sums keep the fixed order
      const float *p0 = prow + head * hd + t;
      a = b = vec_f(0.f);
      for (int p = 0; p < n_parts; p += 8) {
        vec_f pa[8], pb[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (p + i < n_parts) {
            pa[i] = *(const vec_f *)(p0 + (p + i) * part_stride);
            pb[i] = *(const vec_f *)(p0 + (p + i) * part_stride + half);
          }
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (p + i < n_parts) {
            a += pa[i];
            b += pb[i];
          }
      }
    } else {
      const vec_b va = *(const vec_b *)(src + t), vb = *(const vec_b *)(src + t + half);
#pragma unroll
      for (int e = 0; e < UNIT; ++e) { a[e] = (float)va[e]; b[e] = (float)vb[e]; }
    }
    vec_b oa, ob;
    if (head < Hq + Hkv) {
      f32x4 two[UNIT / 2];                                  // (cos, sin) of two pairs each
#pragma unroll
      for (int e = 0; e < UNIT / 2; ++e) two[e] = *(const f32x4 *)(cs + (size_t)j * half + t + 2 * e);
      const float f = head < Hq ? q_scale : 1.0f;          // queries may carry a constant factor for the attention kernel
#pragma unroll
      for (int e = 0; e < UNIT; ++e) {
        const float c = two[e / 2][e % 2 * 2], s = two[e / 2][e % 2 * 2 + 1];
        oa[e] = (bf16)((a[e] * c - b[e] * s) * f);
        ob[e] = (bf16)((b[e] * c + a[e] * s) * f);
      }
    } else {
#pragma unroll
      for (int e = 0; e < UNIT; ++e) { oa[e] = (bf16)a[e]; ob[e] = (bf16)b[e]; }
    }
    bf16 *dst;
    if (head < Hq) {
      dst = src;
    } else if (head < Hq + Hkv) {
      dst = k_pool + ((blk * Hkv + (head - Hq)) * ARB_KV_BLOCK + off) * hd;
    } else {
      dst = v_pool + ((blk * Hkv + (head - Hq - Hkv)) * ARB_KV_BLOCK + off) * hd;
    }
    *(vec_b *)(dst + t) = oa;
    *(vec_b *)(dst + t + half) = ob;
  }
}

constexpr int kRopeManyTokens = 512;        // below, the two forms are within 0.2 us of each other, two pairs ahead more often

arb_status launch_rope_append(bf16 *qkv, const float *parts, RowParts n_parts, const f32x2 *cs, const int32_t *tok_slot,
                              bf16 *k_pool, bf16 *v_pool, int T, int n_q_heads, int n_kv_heads, int head_dim,
                              float q_scale, hipStream_t st) {
  if (T == 0) return ARB_OK;
  const size_t stride = (size_t)T * (n_q_heads + 2 * n_kv_heads) * head_dim;
  const int unit = T >= kRopeManyTokens ? 4 : 2;                      // half a head is 32 or 64 pairs
  const dim3 grid(T, ceil_div((n_q_heads + 2 * n_kv_heads) * (head_dim / 2 / unit), 256));
  const int row_heads = n_parts.head > 0 ? n_q_heads : n_q_heads + 2 * n_kv_heads;
#define ARB_ROPE(PARTS, UNIT)                                                                                            \
  hipLaunchKernelGGL((rope_append_kernel<PARTS, UNIT>), grid, dim3(256), 0, st, qkv, parts, n_parts, stride, cs, tok_slot, \
                     k_pool, v_pool, n_q_heads, n_kv_heads, head_dim, q_scale, row_heads)
  if (n_parts.head > 0) { if (unit == 4) ARB_ROPE(true, 4); else ARB_ROPE(true, 2); }
  else { if (unit == 4) ARB_ROPE(false, 4); else ARB_ROPE(false, 2); }
#undef ARB_ROPE
  ARB_CHECK_LAUNCH("rope_append");
  return ARB_OK;
}

// ------------------------------------------------------- pooling + head + threshold

// One wave per sequence.  tok_dot[j] = w . y_j, so by linearity of the head
// score_b = mean_j tok_dot[j] + c (mean pooling) or tok_dot[last] + c.
// The sum runs in a fixed order, so repeated calls give identical bits.
// With `probability` the pooled value is the difference of two class logits and the score is the
// softmax probability of class 1, 1 / (1 + exp(-z)) (Sec. 4.2: the router's y_hat).
// Decision (Alg. 1): accept iff score <= tau, i.e. escalate = !(score <= tau).
__global__ __launch_bounds__(64) void pool_route_kernel(const float *__restrict__ tok_dot,
                                                        const int32_t *__restrict__ cu, float b_head, int pool,
                                                        int probability, float tau, float *__restrict__ scores,
                                                        uint8_t *__restrict__ escalate) {
  const int b = blockIdx.x, lo = cu[b], hi = cu[b + 1];
  float acc = 0.f;
  if (pool == ARB_POOL_LAST) {
    acc = tok_dot[hi - 1];
  } else {
    for (int j = lo + (int)threadIdx.x; j < hi; j += 64) acc += tok_dot[j];
    acc = wave_sum(acc) / (float)(hi - lo);
  }
  float score = acc + b_head;
  if (probability) score = 1.0f / (1.0f + expf(-score));
  if (threadIdx.x == 0) {
    scores[b] = score;
    if (escalate) escalate[b] = !(score <= tau);
  }
}

arb_status launch_pool_route(const float *tok_dot, const int32_t *cu_step_lens, int batch, float b_head, int pool,
                             int probability, float tau, float *scores, uint8_t *escalate, hipStream_t st) {
  if (batch == 0) return ARB_OK;
  hipLaunchKernelGGL(pool_route_kernel, dim3(batch), dim3(64), 0, st, tok_dot, cu_step_lens, b_head, pool, probability,
                     tau, scores, escalate);
  ARB_CHECK_LAUNCH("pool_route");
  return ARB_OK;
}

__global__ void route_kernel(const float *__restrict__ scores, int n, float tau, int sense,
                             uint8_t *__restrict__ escalate) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float s = scores[i];
  escalate[i] = sense == ARB_ACCEPT_IF_GT ? !(s > tau) : !(s <= tau);
}

arb_status launch_route(const float *scores, int n, float tau, int sense, uint8_t *escalate, hipStream_t st) {
  if (n == 0) return ARB_OK;
  hipLaunchKernelGGL(route_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, scores, n, tau, sense, escalate);
  ARB_CHECK_LAUNCH("route");
  return ARB_OK;
}

// ------------------------------------------------------------- advantage routing

// Definitions 4.1 and 4.2, Eq. 4.4: delta = s_t - s_d; escalate iff not (delta <= tau), the same
// comparison as route_kernel; realized score = s_t where escalated, s_d elsewhere.
__global__ void advantage_route_kernel(const float *__restrict__ s_t, const float *__restrict__ s_d, int n, float tau,
                                    const float *__restrict__ tau_device, float *__restrict__ delta,
                                    uint8_t *__restrict__ escalate, float *__restrict__ realized) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float t = tau_device ? *tau_device : tau;
  const float a = s_t[i], b = s_d[i], d = a - b;
  const bool esc = !(d <= t);
  if (delta) delta[i] = d;
  if (escalate) escalate[i] = esc;
  if (realized) realized[i] = esc ? a : b;
}

arb_status launch_advantage_route(const float *s_t, const float *s_d, int n, float tau, const float *tau_device,
                               float *delta, uint8_t *escalate, float *realized, hipStream_t st) {
  if (n == 0) return ARB_OK;
  hipLaunchKernelGGL(advantage_route_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, s_t, s_d, n, tau, tau_device, delta,
                     escalate, realized);
  ARB_CHECK_LAUNCH("advantage_route");
  return ARB_OK;
}

// Threshold for a budget of escalations (Theorem B.1): tau = max(0, the (budget+1)-th largest delta),
// found by a most-significant-byte-first radix select in one workgroup (n is a number of reasoning
// steps, not of tokens).  Keys order floats as unsigned integers; NaN, which escalates under any tau,
// ranks above every number, and if the selected entry is a NaN the result is +inf.
__device__ __forceinline__ uint32_t order_key(float x) {
  if (x != x) return 0xFFFFFFFFu;
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__global__ __launch_bounds__(256) void budget_threshold_kernel(const float *__restrict__ delta, int n, int budget,
                                                               float *__restrict__ tau_out) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sel_prefix, sel_rank;
  const int tid = threadIdx.x;
  if (budget >= n) {                        // nothing is cut off: every positive advantage may escalate
    if (tid == 0) *tau_out = 0.f;
    return;
  }
  uint32_t prefix = 0, rank = (uint32_t)budget;        // rank from the top among keys matching the prefix
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0;
    __syncthreads();
    const uint32_t mask = shift == 24 ? 0u : 0xFFFFFFFFu << (shift + 8);
    for (int i = tid; i < n; i += 256) {
      const uint32_t k = order_key(delta[i]);
      if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (tid == 0) {
      uint32_t r = rank;
      int b = 255;
      for (; b > 0; --b) {
        if (r < hist[b]) break;
        r -= hist[b];
      }
      sel_prefix = prefix | ((uint32_t)b << shift);
      sel_rank = r;
    }
    __syncthreads();
    prefix = sel_prefix;
    rank = sel_rank;
    __syncthreads();
  }
  if (tid == 0) {
    float t;
    if (prefix == 0xFFFFFFFFu) {
      t = __uint_as_float(0x7F800000u);                 // the NaNs alone exceed the budget
    } else {
      const uint32_t u = (prefix & 0x80000000u) ? (prefix & 0x7FFFFFFFu) : ~prefix;
      t = __uint_as_float(u);
      t = t > 0.f ? t : 0.f;
    }
    *tau_out = t;
  }
}

arb_status launch_budget_threshold(const float *delta, int n, int budget, float *tau_out, hipStream_t st) {
  hipLaunchKernelGGL(budget_threshold_kernel, dim3(1), dim3(256), 0, st, delta, n, budget, tau_out);
  ARB_CHECK_LAUNCH("budget_threshold");
  return ARB_OK;
}

// ------------------------------------------------------- next-token choice (LM head)

// Rows rows[i] of a bf16 [*, d] matrix, copied to a dense [n, d] matrix (the last step token of each
// sequence, as input of the LM head GEMM).
__global__ void gather_rows_kernel(const bf16 *__restrict__ src, const int32_t *__restrict__ rows, int d,
                                   bf16 *__restrict__ dst) {
  const int i = blockIdx.x;
  const bf16 *s = src + (size_t)rows[i] * d;
  for (int c = threadIdx.x * 8; c < d; c += blockDim.x * 8) *(bf16x8 *)(dst + (size_t)i * d + c) = *(const bf16x8 *)(s + c);
}

arb_status launch_gather_rows(const bf16 *src, const int32_t *rows, int n, int d, bf16 *dst, hipStream_t st) {
  if (n == 0) return ARB_OK;
  if (d % 8 != 0) return arb_fail(ARB_EUNSUPPORTED, "gather_rows: width %d is not a multiple of 8", d);
  hipLaunchKernelGGL(gather_rows_kernel, dim3(n), dim3(256), 0, st, src, rows, d, dst);
  ARB_CHECK_LAUNCH("gather_rows");
  return ARB_OK;
}

// Choice of one token per row of fp32 logits [n, V], in two launches.  Greedy (temperature <= 0): the smallest
// index of the maximum.  Otherwise the token is drawn from softmax(logits / temperature) by inversion with the
// caller's uniform u in [0, 1): the smallest k with sum_{i<=k} w_i >= u * sum_i w_i, w_i = exp((l_i - max) / temperature);
// every sum has a fixed order, so a call is reproducible.  For u > 0 a token whose weight is 0 in fp32 is never drawn: a
// chunk, then a thread's range in it, claims the target only if its cumulative weight crosses it, and where sums of the same
// weights in another order end short of the target the last token with a weight is taken.
//
// The logits are read once at memory speed: a row is cut into chunks, a workgroup reduces one chunk with
// 16-byte loads of neighbouring lanes to (maximum, its smallest index, sum of exp relative to the chunk's maximum),
// and one workgroup per row joins the chunks; only when sampling it reads the one chunk that holds the target again.
// (One workgroup per row, each thread walking its own contiguous range, took 195 us for 16 rows of 151936: a 4-byte
// load per cache line and lane and 16 of 256 CUs at work.  The two launches take 6.)
struct ChoiceChunk { float max, sum; int arg, unused; };
constexpr int kChoiceChunk = 4096;        // least elements per chunk: 4 loads of 16 bytes per thread

// (v, i) ordered by larger v, then smaller i; NaN never wins
__device__ __forceinline__ void take_better(float &v, int &i, float v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
}

// Best (value, index) over a block of 256 threads; every thread gets it.
__device__ __forceinline__ void block_best_256(float &v, int &i, float *lds_v, int *lds_i) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) take_better(v, i, __shfl_xor(v, o, 64), __shfl_xor(i, o, 64));
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { lds_v[w] = v; lds_i[w] = i; }
  __syncthreads();
  v = lds_v[0]; i = lds_i[0];
#pragma unroll
  for (int k = 1; k < 4; ++k) take_better(v, i, lds_v[k], lds_i[k]);
}

__global__ __launch_bounds__(256) void choice_chunk_kernel(const float *__restrict__ logits, int V, int chunk_len,
                                                           float temperature, ChoiceChunk *__restrict__ chunks) {
  __shared__ float red_v[4];
  __shared__ int red_i[4];
  const int tid = threadIdx.x, lo = blockIdx.x * chunk_len, hi = min(lo + chunk_len, V);
  const float *l = logits + (size_t)blockIdx.y * V;
  float best = -INFINITY;
  int arg = V;
  for (int i = lo + tid * 4; i < hi; i += 1024) {            // V is a multiple of 4: a load is whole or not there
    const f32x4 x = *(const f32x4 *)(l + i);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (x[e] > best) { best = x[e]; arg = i + e; }
  }
  block_best_256(best, arg, red_v, red_i);
  float sum = 0.f;
  if (temperature > 0.f && arg < V) {
    const float inv_t = 1.0f / temperature;
    for (int i = lo + tid * 4; i < hi; i += 1024) {
      const f32x4 x = *(const f32x4 *)(l + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) sum += expf((x[e] - best) * inv_t);
    }
    sum = block_sum_256(sum, red_v);
  }
  if (tid == 0) chunks[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = ChoiceChunk{best, sum, arg, 0};
}

__global__ __launch_bounds__(256) void choice_join_kernel(const float *__restrict__ logits, int V, int chunk_len,
                                                          int n_chunks, float temperature,
                                                          const float *__restrict__ uniforms,
                                                          const ChoiceChunk *__restrict__ chunks,
                                                          int32_t *__restrict__ token, float *__restrict__ chosen) {
  __shared__ float red_v[256];
  __shared__ int red_i[256];
  const int row = blockIdx.x, tid = threadIdx.x;
  const float *l = logits + (size_t)row * V;
  const ChoiceChunk mine = tid < n_chunks ? chunks[(size_t)row * n_chunks + tid] : ChoiceChunk{-INFINITY, 0.f, V, 0};
  float mx = mine.max;
  int arg = mine.arg;
  block_best_256(mx, arg, red_v, red_i);
  const int amax = arg < V ? arg : 0;                    // a row of NaNs or -inf picks token 0
  if (!(temperature > 0.f)) {
    if (tid == 0) {
      token[row] = amax;
      if (chosen) chosen[row] = l[amax];
    }
    return;
  }
  const float inv_t = 1.0f / temperature;
  // the chunk that contains the target: the first whose cumulative weight reaches it
  __shared__ float before_s, target_s;
  __shared__ int chunk_s, pick_s, last_s;                // last_s: last token of the chunk with a weight (else its largest logit)
  __syncthreads();
  red_v[tid] = mine.arg < V ? mine.sum * expf((mine.max - mx) * inv_t) : 0.f;
  __syncthreads();
  if (tid == 0) {
    float total = 0.f;
    for (int t = 0; t < n_chunks; ++t) total += red_v[t];
    const float target = uniforms[row] * total;
    float run = 0.f;
    int c = -1;
    for (int t = 0; t < n_chunks && c < 0; ++t) {
      if (target <= run + red_v[t]) c = t; else run += red_v[t];
    }
    before_s = run;
    target_s = target;
    chunk_s = arg < V ? c : -1;                           // -1: no chunk claims the target (NaN, or rounding at the very end)
    pick_s = V;
  }
  __syncthreads();
  const int c = chunk_s;
  if (tid == c) last_s = mine.arg;
  __syncthreads();
  int k = amax;                                           // ... then the mode
  if (c >= 0) {
    const int lo = c * chunk_len, hi = min(lo + chunk_len, V), per = (hi - lo + 255) / 256;
    const int a = min(lo + tid * per, hi), b = min(a + per, hi);
    float part = 0.f;
    int last = -1;
    for (int i = a; i < b; ++i) {
      const float w = expf((l[i] - mx) * inv_t);
      part += w;
      if (w > 0.f) last = i;
    }
    atomicMax(&last_s, last);
    red_v[tid] = part;
    __syncthreads();
    if (tid == 0) {
      float run = before_s;
      for (int t = 0; t < 256; ++t) {
        const float p = red_v[t];
        red_v[t] = run;
        run += p;
      }
    }
    __syncthreads();
    // the range that contains the target: before < target <= before + part (the row's first range also takes target == 0)
    const float before = red_v[tid];
    if (a < b && (target_s > before || (c == 0 && tid == 0)) && target_s <= before + part) {
      float run = before;
      int pick = last < 0 ? a : last;                     // rounding in the re-summation cannot leave the range
      for (int i = a; i < b; ++i) {
        run += expf((l[i] - mx) * inv_t);
        if (run >= target_s) { pick = i; break; }
      }
      atomicMin(&pick_s, pick);
    }
    __syncthreads();
    k = pick_s < V ? pick_s : last_s;                     // ... nor the chunk
  }
  if (tid == 0) {
    token[row] = k;
    if (chosen) chosen[row] = l[k];
  }
}

// scratch: device memory of at least scratch_bytes >= n * 16 bytes (more lets a row be cut into more chunks)
arb_status launch_sample_token(const float *logits, int n, int V, float temperature, const float *uniforms,
                               int32_t *token, float *chosen, void *scratch, size_t scratch_bytes, hipStream_t st) {
  if (n == 0) return ARB_OK;
  size_t most = scratch_bytes / ((size_t)n * sizeof(ChoiceChunk));
  if (most < 1) return arb_fail(ARB_ECAPACITY, "sample_token: scratch of %zu bytes for %d rows", scratch_bytes, n);
  if (most > 256) most = 256;                             // a thread of the joining workgroup per chunk
  int chunk_len = kChoiceChunk;
  if ((size_t)ceil_div(V, chunk_len) > most) chunk_len = ceil_div(ceil_div(V, (int)most), 1024) * 1024;
  const int n_chunks = ceil_div(V, chunk_len);
  ChoiceChunk *chunks = (ChoiceChunk *)scratch;
  for (int r = 0; r < n; r += 65535) {                    // grid.y limit
    const int m = n - r < 65535 ? n - r : 65535;
    hipLaunchKernelGGL(choice_chunk_kernel, dim3(n_chunks, m), dim3(256), 0, st, logits + (size_t)r * V, V, chunk_len,
                       temperature, chunks + (size_t)r * n_chunks);
  }
  ARB_CHECK_LAUNCH("choice_chunk");
  hipLaunchKernelGGL(choice_join_kernel, dim3(n), dim3(256), 0, st, logits, V, chunk_len, n_chunks, temperature, uniforms,
                     chunks, token, chosen);
  ARB_CHECK_LAUNCH("choice_join");
  return ARB_OK;
}

// Length of a generated step (Alg. 1: tokens up to and including the first separator or
// end-of-sequence token) for each row of tokens [n, S]; S if neither occurs.
__global__ void first_stop_kernel(const int32_t *__restrict__ tokens, int n, int S, int sep, int eos,
                                  int32_t *__restrict__ len, uint8_t *__restrict__ ended) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n) return;
  int L = S;
  uint8_t e = 0;
  for (int i = 0; i < S; ++i) {
    const int t = tokens[(size_t)b * S + i];
    if (t == sep || t == eos) { L = i + 1; e = t == eos; break; }
  }
  len[b] = L;
  if (ended) ended[b] = e;
}

arb_status launch_first_stop(const int32_t *tokens, int n, int S, int sep, int eos, int32_t *len, uint8_t *ended,
                             hipStream_t st) {
  if (n == 0) return ARB_OK;
  hipLaunchKernelGGL(first_stop_kernel, dim3(ceil_div(n, 64)), dim3(64), 0, st, tokens, n, S, sep, eos, len, ended);
  ARB_CHECK_LAUNCH("first_stop");
  return ARB_OK;
}

// One decoding iteration of steps that are generated token by token (Alg. 1: a step ends with its first
// separator or end-of-sequence token, or at S tokens).  Row r = open_rows[j] was fed this iteration and chose
// chosen[j]: the token is appended, len and done are updated, and the rows that stay open are written in
// order to next_rows with their tokens in next_ids (the ids of the next iteration).  One workgroup walks the
// open rows 256 at a time; the order-preserving compaction is a ballot per wave plus a scan over the waves.
__global__ __launch_bounds__(256) void step_advance_kernel(const int32_t *__restrict__ open_rows,
                                                           const int32_t *__restrict__ chosen, int n_open, int S, int sep,
                                                           int eos, int32_t *__restrict__ steps, int32_t *__restrict__ len,
                                                           uint8_t *__restrict__ done, int32_t *__restrict__ next_rows,
                                                           int32_t *__restrict__ next_ids, int32_t *__restrict__ n_next) {
  __shared__ int wave_count[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int base = 0;                                  // rows kept by the chunks before this one
  for (int j0 = 0; j0 < n_open; j0 += 256) {
    const int j = j0 + threadIdx.x;
    bool keep = false;
    int r = 0, t = 0;
    if (j < n_open) {
      r = open_rows[j];
      t = chosen[j];
      const int l = len[r];
      steps[(size_t)r * S + l] = t;
      len[r] = l + 1;
      const bool stop = t == sep || t == eos || l + 1 >= S;
      done[r] = stop ? (t == eos ? 2 : 1) : 0;
      keep = !stop;
    }
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(keep);
    if (lane == 0) wave_count[wave] = __builtin_popcountll(mask);
    __syncthreads();
    int before = base;
    for (int w = 0; w < wave; ++w) before += wave_count[w];
    if (keep) {
      const int pos = before + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
      next_rows[pos] = r;
      next_ids[pos] = t;
    }
    base += wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
    __syncthreads();
  }
  if (threadIdx.x == 0) *n_next = base;
}

arb_status launch_step_advance(const int32_t *open_rows, const int32_t *chosen, int n_open, int S, int sep, int eos,
                               int32_t *steps, int32_t *len, uint8_t *done, int32_t *next_rows, int32_t *next_ids,
                               int32_t *n_next, hipStream_t st) {
  hipLaunchKernelGGL(step_advance_kernel, dim3(1), dim3(256), 0, st, open_rows, chosen, n_open, S, sep, eos, steps, len,
                     done, next_rows, next_ids, n_next);
  ARB_CHECK_LAUNCH("step_advance");
  return ARB_OK;
}

// ids[cu[j] + i] = steps[rows[j]][i] for i < cu[j+1] - cu[j]: the steps of the listed rows as one ragged token list
__global__ __launch_bounds__(256) void pack_steps_kernel(const int32_t *__restrict__ steps, int S,
                                                         const int32_t *__restrict__ rows, const int32_t *__restrict__ cu,
                                                         int n_rows, int32_t *__restrict__ ids) {
  const int j = blockIdx.x;
  if (j >= n_rows) return;
  const int r = rows[j], begin = cu[j], n = min(cu[j + 1] - begin, S);
  for (int i = threadIdx.x; i < n; i += blockDim.x) ids[begin + i] = steps[(size_t)r * S + i];
}

arb_status launch_pack_steps(const int32_t *steps, int S, const int32_t *rows, const int32_t *cu, int n_rows, int32_t *ids,
                             hipStream_t st) {
  if (n_rows == 0) return ARB_OK;
  hipLaunchKernelGGL(pack_steps_kernel, dim3(n_rows), dim3(256), 0, st, steps, S, rows, cu, n_rows, ids);
  ARB_CHECK_LAUNCH("pack_steps");
  return ARB_OK;
}

