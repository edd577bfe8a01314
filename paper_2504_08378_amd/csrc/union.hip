// Small-batch decode over the union of the tokens' active sets (extension of Section 4's
// operation C from one token to B <= 8 tokens; the paper itself decodes one token at a time).
//
//   Y[b][o] = sum_{j in idx_b[b]} Wt[j][o] * X[b][j]
//
// Step 1 (two small launches): every token's kept channels as bits in device memory (the batched decoder
// layer does this inside its selection launch); per 256 channels, turn the tokens' bits into
// Xm[j][b] = X[b][j] if token b keeps channel j else 0 (fp16, 8 tokens per row) and into that part of the
// ascending union U, whose place follows from the bits of all lower channels.
// Step 2: the gathered product over U on the matrix cores; every weight row of the union is read
// once for all tokens.
#include "af_internal.h"

#define UB_THREADS 1024
#define UB_RANGE 256   // channels per workgroup of the builder

struct UnionBuildParams {
  const half_t* X;         // [B][in]
  const int32_t* idx_b;    // [B][idx_stride], k entries used
  unsigned char* kept;     // [B][af_kept_stride(in)]
  int32_t* union_idx;      // [in]
  int32_t* union_n;        // [1]
  half_t* Xm;              // [in][8]
  int B, k, in, idx_stride;
  int* tickets;            // the device error word lies behind them
};

// Builder, first launch: workgroup b turns token b's list into bits, put together in LDS.  An entry
// outside [0, in) is dropped and reported.
__global__ __launch_bounds__(UB_THREADS) void union_mark_kernel(UnionBuildParams p) {
  extern __shared__ __align__(16) unsigned s_kept[];  // af_kept_stride(in) bytes
  const int b = blockIdx.x, words = af_kept_stride(p.in) / 4;
  const int kb = p.k;
  const int32_t* list = p.idx_b + (size_t)b * p.idx_stride;
  int j[4];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) j[u] = t0 + u * UB_THREADS < kb ? list[t0 + u * UB_THREADS] : -1;
  };
  fetch(threadIdx.x);  // on the way while the bits are cleared
  for (int i = threadIdx.x; i < words; i += UB_THREADS) s_kept[i] = 0;
  __syncthreads();
  for (int t0 = threadIdx.x; t0 < kb; t0 += 4 * UB_THREADS) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if ((unsigned)j[u] < (unsigned)p.in)
        atomicOr(&s_kept[j[u] >> 4], 1u << ((j[u] >> 2 & 3) * 8 + (j[u] & 3)));
      else if (t0 + u * UB_THREADS < kb)
        af_report_bad_index(p.tickets);  // broken precondition
    }
    if (t0 + 4 * UB_THREADS < kb) fetch(t0 + 4 * UB_THREADS);
  }
  __syncthreads();
  unsigned* out = reinterpret_cast<unsigned*>(p.kept + (size_t)b * af_kept_stride(p.in));
  for (int i = threadIdx.x; i < words; i += UB_THREADS) out[i] = s_kept[i];
}

// Builder, second launch: workgroup r owns the channels [r * UB_RANGE, (r + 1) * UB_RANGE).  It writes
// their masked, transposed token values and its part of the ascending union, behind the channels of
// all lower ranges, which it counts itself (16 bytes of bits hold 64 channels of a token).  The builder this
// replaces set the bits by atomics in device memory, had a launch of its own to move the parts into place,
// and in the batched layer read the selection's lists back: 70B-shape layer, eight tokens 354 -> 340 us,
// gate|up over four tokens 132 -> 130 us.
__global__ __launch_bounds__(UB_RANGE) void union_gather_kernel(UnionBuildParams p) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  constexpr int WAVES = UB_RANGE / AF_WAVE;
  __shared__ unsigned s_wtot[WAVES], s_below[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = blockIdx.x, stride = af_kept_stride(p.in);
  const int j = r * UB_RANGE + tid;
  // All loads without a branch between them (a token behind the last is read as the last one): each would
  // otherwise be waited for before the next.
  const int jr = min(j, p.in - 1);
  unsigned char kb[8];
  half_t x[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const size_t t = (size_t)min(b, p.B - 1);
    kb[b] = p.kept[t * stride + (jr >> 2)];
    x[b] = p.X[t * p.in + jr];
  }
  unsigned below = 0;
  for (int q = tid; q < r * (UB_RANGE / 64); q += UB_RANGE) {
    u32x4 piece[8];
#pragma unroll
    for (int b = 0; b < 8; ++b)
      piece[b] = *reinterpret_cast<const u32x4*>(p.kept + (size_t)min(b, p.B - 1) * stride + q * 16);
#pragma unroll
    for (int b = 1; b < 8; ++b) piece[0] |= piece[b];
#pragma unroll
    for (int c = 0; c < 4; ++c) below += (unsigned)__popc(piece[0][c]);
  }
  unsigned m = 0;
  half8 v;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const unsigned bit = b < p.B && j < p.in ? kb[b] >> (j & 3) & 1u : 0u;
    m |= bit;
    v[b] = bit ? x[b] : (half_t)0;
  }
  if (j < p.in) *reinterpret_cast<half8*>(p.Xm + (size_t)j * 8) = v;
  below = af_wave_sum(below);
  const unsigned inc = af_wave_incl_scan(m);
  if (lane == 63) {
    s_wtot[wave] = inc;
    s_below[wave] = below;
  }
  __syncthreads();
  unsigned base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    base += s_below[w] + (w < wave ? s_wtot[w] : 0u);
    total += s_below[w] + s_wtot[w];
  }
  if (m) p.union_idx[base + inc - 1] = j;
  if (r == (int)gridDim.x - 1 && tid == 0) *p.union_n = (int)total;
}

#define UG_THREADS 1024
#define UG_CHUNK 2048  // rows staged at a time

struct UnionGemvParams {
  const half_t* W;
  const half_t* Xm;        // [in][8]
  const int32_t* idx;      // union
  const int32_t* nidx_dev;
  float* partials;         // [S][B][out_pad]
  int* tickets;
  void* Y;                 // [B][out]
  const half_t* residual;  // [B][out] added to the product, or null
  int out, ld, nidx_host, y_kind, out_pad, B;
};

// Workgroup (tile, split): sixteen waves, CW of them side by side across a tile of 128 * CW columns,
// the others on different rows.  In a wave 16 lanes span 128 columns (16 bytes each) and its four
// lane groups take eight rows each, so a step is 32 rows: the lane that has loaded eight rows holds,
// for each of its eight columns, the eight consecutive contraction elements that a lane supplies to
// the 16x16x32 matrix instruction, four byte permutations away.  Eight of those (one per column; the
// tokens in the rows of the result, half of which stay unused) take the place of 64 B multiply-adds
// per row pair, add up the lane groups on the way and need 32 accumulators where eight tokens
// needed 64.  The kernel streams the union (4.6 to 6.4 TB/s at the 70B shape).
// One such workgroup per compute unit: 256-thread workgroups needed 38 to 48 splits to fill the
// chip, and the last one of a tile then added up 48 x 2048 partial sums on its own.  us with the
// builder, 50 % of the channels kept, 1 / 4 / 8 tokens, before (vector unit, 256 threads) and now:
//   8192 -> 10240  32.3 / 49.1 / 56.2   25.7 / 37.7 / 41.2     8192 -> 57344  87.4 / 157.6 / 171.8   79.5 / 137.9 / 147.3
//   8192 -> 8192   31.1 / 46.5 / 53.9   24.0 / 33.7 / 35.9     28672 -> 8192  52.5 / 96.5 / 105.9    50.5 / 81.3 / 86.6
//   4096 -> 4096   25.4 / 49.7 / 54.8   18.3 / 18.7 / 19.9     11008 -> 4096  41.3 / 56.0 / 61.3     20.8 / 27.4 / 29.4
// (the same large workgroups on the vector unit: 8192 -> 57344 80.9 / 139.5 / 155.9, 28672 -> 8192
// 49.1 / 81.5 / 92.5; two 512-thread workgroups per unit: within 1 % of one of 1024).
template <int CW>
__global__ __launch_bounds__(UG_THREADS) void gemv_union_kernel(UnionGemvParams p) {
  typedef float float4v __attribute__((ext_vector_type(4)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  constexpr int THREADS = UG_THREADS;
  constexpr int TW = 128 * CW, RW = UG_THREADS / AF_WAVE / CW;
  constexpr int XLD = UG_CHUNK + 8;  // 16 bytes further per token: another bank group
  constexpr int STAGE_BYTES = 8 * XLD * 2 + UG_CHUNK * 4, RED_BYTES = RW * 4 * TW * 4;
  __shared__ __align__(16) char s_mem[STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES];
  half_t* s_x = reinterpret_cast<half_t*>(s_mem);  // [token][staged row]
  int* s_idx = reinterpret_cast<int*>(s_mem + 8 * XLD * 2);
  float(*s_red)[4][TW] = reinterpret_cast<float(*)[4][TW]>(s_mem);  // behind the row loop
  __shared__ int s_last;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lx = lane & 15, g = lane >> 4;
  const int cw = wave % CW, rw = wave / CW;
  const int tile0 = blockIdx.x * TW;
  const int col = tile0 + cw * 128 + lx * 8;
  const int col_ld = col < p.out ? col : 0;
  const int S = gridDim.y, s = blockIdx.y;

  const int nidx = min(*p.nidx_dev, p.nidx_host);
  const int R = af_ceil_div_small(nidx, S);
  const int r0 = min(s * R, nidx), r1 = min(r0 + R, nidx);

  float4v acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = float4v{0.f, 0.f, 0.f, 0.f};
  const half_t* wcol = p.W + col_ld;

  auto multiply = [&](const u32x4 (&w)[8], int pos) __attribute__((always_inline)) {
    const half8 a = *reinterpret_cast<const half8*>(s_x + (lane & 7) * XLD + pos);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4 b;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        b[i] = __builtin_amdgcn_perm(w[2 * i + 1][c / 2], w[2 * i][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
      // The step's sum starts from zero and joins the others in a rounded addition: with the running
      // sum as the instruction's addend the error against 64 bits grew with the number of steps
      // (8192 -> 57344, four tokens: 2.07e-7; 1.25e-7 this way, 1.30e-7 on the vector unit).
      acc[c] += __builtin_amdgcn_mfma_f32_16x16x32_f16(a, __builtin_bit_cast(half8, b), float4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
  };

  for (int base = r0; base < r1; base += UG_CHUNK) {
    const int cnt = min(UG_CHUNK, r1 - base);
    __syncthreads();
    for (int i = tid; i < (cnt + 31) / 32 * 32; i += THREADS) {  // whole steps: zeros behind the end
      const int j = i < cnt ? p.idx[base + i] : 0;
      half8 x = *reinterpret_cast<const half8*>(p.Xm + (size_t)j * 8);
      s_idx[i] = j;
#pragma unroll
      for (int b = 0; b < 8; ++b) s_x[b * XLD + i] = i < cnt ? x[b] : (half_t)0;
    }
    __syncthreads();
    int i = rw * 32;
    for (; i + 32 <= cnt; i += RW * 32) {
      u32x4 w[8];
      int j[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) j[u] = s_idx[i + g * 8 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        w[u] = af_load_once(reinterpret_cast<const u32x4*>(wcol + (size_t)j[u] * p.ld));
      __builtin_amdgcn_sched_barrier(0);
      multiply(w, i + g * 8);
    }
    if (i < cnt) {  // the last step of the list: its missing rows are zero
      u32x4 w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        w[u] = u32x4{0u, 0u, 0u, 0u};
        if (i + g * 8 + u < cnt)
          w[u] = af_load_once(reinterpret_cast<const u32x4*>(wcol + (size_t)s_idx[i + g * 8 + u] * p.ld));
      }
      multiply(w, i + g * 8);
    }
  }

  auto store = [&](int b, int colg, float v) {
    if (colg < p.out) {
      if (p.residual) v += (float)p.residual[(size_t)b * p.out + colg];
      if (p.y_kind == AF_F16)
        reinterpret_cast<half_t*>(p.Y)[(size_t)b * p.out + colg] = (half_t)v;
      else
        reinterpret_cast<float*>(p.Y)[(size_t)b * p.out + colg] = v;
    }
  };
  // Lane group h holds tokens 4 h .. 4 h + 3: added up over the waves one group at a time.
  float* mine = p.partials + (size_t)s * p.B * p.out_pad;
  for (int h = 0; h * 4 < p.B; ++h) {
    __syncthreads();  // the staged rows, or the sums of the tokens before, have been read
    if (g == h) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) s_red[rw][r][cw * 128 + lx * 8 + c] = acc[c][r];
    }
    __syncthreads();
    const int nb = min(4, p.B - h * 4);
    for (int e = tid; e < nb * TW; e += THREADS) {
      const int b = e / TW, c = e % TW;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < RW; ++w) v += s_red[w][b][c];
      if (S == 1)
        store(h * 4 + b, tile0 + c, v);
      else
        af_store_agent(mine + (size_t)(h * 4 + b) * p.out_pad + tile0 + c, v);
    }
  }
  if (S == 1) return;
  af_stores_done();
  __syncthreads();
  if (tid == 0) {
    int old = af_ticket_take(&p.tickets[af_ticket_of(blockIdx.x)]);
    s_last = (old == S - 1);
  }
  __syncthreads();
  if (!s_last) return;
  for (int e = tid; e < p.B * TW; e += THREADS) {
    const int b = e / TW, c = e % TW;
    store(b, tile0 + c,
          af_sum_partials(p.partials + (size_t)b * p.out_pad + tile0 + c, (size_t)p.B * p.out_pad, S));
  }
  if (tid == 0) af_ticket_reset(&p.tickets[af_ticket_of(blockIdx.x)]);
}

int af_launch_union_f16(af_ctx* ctx, const af_union_args& u) {
  const int in = u.in, out = u.out, B = u.B, k = u.k;
  UnionBuildParams bp;
  bp.X = u.X;
  bp.idx_b = u.idx_b;
  bp.union_idx = u.union_idx;
  bp.union_n = u.union_n;
  bp.Xm = (half_t*)(ctx->ws + ctx->lay.union_x);
  bp.B = B;
  bp.k = k;
  bp.in = in;
  bp.idx_stride = u.idx_stride;
  bp.tickets = (int*)(ctx->ws + ctx->lay.tickets);
  bp.kept = (unsigned char*)(ctx->ws + ctx->lay.union_kept);
  if (!u.marked) {
    hipLaunchKernelGGL(union_mark_kernel, dim3(B), dim3(UB_THREADS), af_kept_stride(in), ctx->stream, bp);
    AF_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(union_gather_kernel, dim3((in + UB_RANGE - 1) / UB_RANGE), dim3(UB_RANGE), 0, ctx->stream, bp);
  AF_LAUNCH_CHECK();

  // Tile width: narrow outputs fill the chip with 128 columns and few splits (8192 -> 8192, eight
  // tokens: 35.9 us with 128 columns and 4 splits, 38.4 with 256 and 8; 11008 -> 4096 29.4 / 31.0);
  // from there on longer pieces of a row count for more (8192 -> 10240 41.4 / 41.2, 8192 -> 57344
  // 164.7 / 147.1; 512 columns 151.9).  512 columns where the 256-column tiles leave compute units without
  // one and the wider ones fill a third more (129 to 170 tiles of 256; us for 1 / 4 / 8 tokens on the vector unit,
  // 256 and 512 columns): 8192 -> 33024 56.5 / 101.1 / 111.6, 61.2 / 107.0 / 114.9 and 50.9 / 87.6 / 94.8;
  // 4096 -> 40960 38.4 / 69.0 / 75.9, 36.4 / 60.1 / 64.9 and 34.8 / 57.5 / 64.0.  On the other side of the line
  // 4096 -> 24576 (192 and 240 workgroups) 29.2 / 49.1 / 54.7, 25.7 / 39.7 / 43.5 and 25.3 / 39.6 / 44.8, and with
  // as many of either 8192 -> 49152 77.1 / 139.7 / 144.9, 70.0 / 121.1 / 129.5 and 70.0 / 122.9 / 133.8.
  int cw = out <= 8192 ? 1 : 2;
  auto workgroups = [&](int width) { const int t = (out + width - 1) / width; return t >= ctx->n_cu ? t : ctx->n_cu / t * t; };
  if (cw == 2 && workgroups(512) <= ctx->n_cu && 3 * workgroups(512) >= 4 * workgroups(256)) cw = 4;
  if (ctx->tune_lx == 16) cw = 1;
  if (ctx->tune_lx == 32) cw = 2;
  if (ctx->tune_lx == 64) cw = 4;
  const int tw = cw * 128;
  const int tiles = (out + tw - 1) / tw;
  const int out_pad = tiles * tw;
  if (tiles > AF_TICKET_ATTN) return AF_ESHAPE;
  const int nidx_max = (long long)B * k < in ? B * k : in;
  int S = ctx->n_cu / tiles;  // one workgroup per compute unit
  if (ctx->tune_split > 0) S = ctx->tune_split;
  int max_s = (nidx_max + 31) / 32;
  if (max_s < 1) max_s = 1;
  if (S > max_s) S = max_s;
  if (S > 256) S = 256;
  if (S < 1) S = 1;
  while (S > 1 && (size_t)S * B * out_pad > ctx->lay.partial_floats) --S;

  UnionGemvParams p;
  p.W = (const half_t*)u.Wt;
  p.Xm = bp.Xm;
  p.idx = u.union_idx;
  p.nidx_dev = u.union_n;
  p.partials = (float*)(ctx->ws + ctx->lay.partials);
  p.tickets = (int*)(ctx->ws + ctx->lay.tickets);
  p.Y = u.Y;
  p.residual = u.residual;
  p.out = out;
  p.ld = u.ld;
  p.nidx_host = nidx_max;
  p.y_kind = u.y_kind;
  p.out_pad = out_pad;
  p.B = B;
  dim3 grid(tiles, S);
  if (cw == 1)
    hipLaunchKernelGGL(gemv_union_kernel<1>, grid, dim3(UG_THREADS), 0, ctx->stream, p);
  else if (cw == 4)
    hipLaunchKernelGGL(gemv_union_kernel<4>, grid, dim3(UG_THREADS), 0, ctx->stream, p);
  else
    hipLaunchKernelGGL(gemv_union_kernel<2>, grid, dim3(UG_THREADS), 0, ctx->stream, p);
  AF_LAUNCH_CHECK();
  return AF_OK;
}

extern "C" int af_sparse_gemv_union_f16(af_ctx* ctx, const void* Wt, int in, int out, int ld,
                                        const void* X_f16, int B, const int32_t* idx_b, int k,
                                        int32_t* union_idx, int32_t* union_n, void* Y, int y_kind) {
  if (!ctx || !Wt || !X_f16 || !union_idx || !union_n || !Y || (!idx_b && k > 0)) return AF_ENULL;
  if (in <= 0 || out <= 0 || in > AF_MAX_N || B < 1 || B > AF_MAX_BATCH || k < 0 || k > in)
    return AF_EINVAL;
  if (out % 8 || ld % 8 || ld < out) return AF_ESHAPE;
  if (y_kind != AF_F16 && y_kind != AF_F32) return AF_EINVAL;
  if (!ctx->ws) return AF_EWORKSPACE;
  if (in > ctx->max_in || out > ctx->max_out || B > ctx->max_batch) return AF_EWORKSPACE;
  if (ctx->validate)
    for (int b = 0; b < B; ++b) {
      const int rc = af_validate_idx(ctx, idx_b + (size_t)b * k, k, nullptr, in);
      if (rc) return rc;
    }
  af_union_args u{};
  u.Wt = Wt;
  u.in = in;
  u.out = out;
  u.ld = ld;
  u.X = (const half_t*)X_f16;
  u.B = B;
  u.idx_b = idx_b;
  u.idx_stride = k;
  u.k = k;
  u.union_idx = union_idx;
  u.union_n = union_n;
  u.Y = Y;
  u.y_kind = y_kind;
  return af_launch_union_f16(ctx, u);
}
