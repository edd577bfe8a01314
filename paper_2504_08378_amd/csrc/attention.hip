// Decode attention of one token (or of one token each of B sequences): rotary embedding of the new
// q and k, append to the KV cache, softmax attention over the cache and the new token.
//
// Workgroup (key head and up to 8 of the query heads that share it, key split): every key and
// value row is read once for all of those heads.  A wave takes 32 keys at a time through the matrix
// cores and keeps a running softmax of its own; nothing is exchanged between the waves before each
// of them has gone through its keys, so a workgroup has one barrier up to its sums, and the first
// key / value rows are requested together with q.
//   scores   D[key][head] = K Q^T, 16 keys x 16 heads per instruction: a lane supplies eight
//            consecutive dimensions of one key row, which is the load it has made, and gets four
//            keys of one head, so the softmax of a head runs along the registers of four lanes;
//   values   D[dim][head] = V^T P^T: a lane supplies eight keys of one dimension.  Which keys is
//            free as long as both operands agree, so it takes the eight whose probabilities it
//            has already (no transposition of P), loads those eight rows of V and picks the
//            columns by byte permutation.
// q and the probabilities are fp32 values.  Each enters the instructions as three fp16 values, the rounded one
// and two of what that leaves: all 24 bits of q, and of every weight above 2^-16 of the largest (smaller ones
// to 2^-40 of it).  The products of the parts are added outside of the instructions, and those of a score's
// dimensions as well.  Error of the fp32 results (before their rounding) against 64 bits, 32 heads on 32, scores of
// 0.4 rms, with the vector unit / with two parts, 2^15 in the exponent and all parts in one running sum / now:
// 16 keys 0.80 / 2.06 / 0.73e-7, 64 keys 1.01 / 2.48 / 0.75e-7, 6001 keys 1.38 / 2.98 / 1.11e-7; scores of 2.4 rms,
// 64 keys 1.67 / 1.85 / 1.53e-7.
// What bounds it: latency at short contexts (load, scores, softmax, values, partial sums to the last
// workgroup of a head), the read of the cache at long ones.  With one workgroup per query head, which
// read the rows of a key head once for each of its query heads, us per layer (attention and short
// GEMVs: 512 channels), before / now: 64 heads on 8 key heads, 512 keys 45.3 / 41.6, 2000 keys 54.1 / 43.3, 6001 keys
// 76.1 / 49.6; 32 on 8, 512 keys 41.9 / 39.3, 4000 keys 51.7 / 43.5; 32 on 32, 512 keys 42.2 / 40.4, 3000 keys 49.2 / 47.8,
// 8000 keys 61.5 / 58.8 (1 to 2 us of that by the GEMVs' tickets).  Caches of fewer than 128 keys: attn_short_kernel.
// A first version that rotated q in every lane, 300 instructions of one wave, was 2 us slower throughout.  The error of the fp16 result against 64 bits is that
// of the rounding alone (2.0942e-4 at 32 heads and 512 keys, before and now).
#include <math.h>

#include "attention.h"

#define ATT_THREADS 256
#define ATT_WAVES (ATT_THREADS / AF_WAVE)
#define ATT_HEADS 8        // query heads of one workgroup, at most
#define ATT_STEP 32        // keys of a wave per step
#define ATT_MAX_KEYS 2048  // cache keys per key split
// Workgroups that a compute unit holds (the batched launch has more of them than there are units).
#define ATT_WAVES_PER_SIMD(hd) ((hd) == 128 ? 2 : 3)

typedef float att_f4 __attribute__((ext_vector_type(4)));
typedef half_t att_h2 __attribute__((ext_vector_type(2)));
typedef half_t att_h4 __attribute__((ext_vector_type(4)));
typedef unsigned short att_us2 __attribute__((ext_vector_type(2)));

// The product with a factor's rests, to be added to the one with its rounded value.  An infinite key or value
// times the zero that a rest may be is NaN: then the other product has the infinity, and the NaN is put aside
// (the median ignores it).  The rounded value is zero for a factor of zero only: one that would round to zero
// takes the smallest fp16 of its sign, and the rests what that is too much.
__device__ __forceinline__ float att_rest(float r) { return __builtin_amdgcn_fmed3f(r, -3.0e38f, 3.0e38f); }

// a * b + c rounded to fp16 once, the last step of a rotated key.  With a conversion of an fp32
// fma in its place, which is what the compiler makes of other surroundings, some elements of the cache
// differ in their last bit.
__device__ __forceinline__ half_t att_fma_half(half_t a, float b, float c) {
  unsigned d;
  asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]"
      : "=v"(d)
      : "v"((unsigned)__builtin_bit_cast(unsigned short, a)), "v"(b), "v"(c));
  return __builtin_bit_cast(half_t, (unsigned short)d);
}

// cs / sn: the rotary table of the token's position.  bx: number of the (key head, head group).
template <int HD>
__device__ __forceinline__ void attn_decode_body(const AttnParams& p, const float* cs_tab, const float* sn_tab,
                                                 const int bx, const int s, const int KS) {
  constexpr int TT = HD / 32;   // contraction steps of the scores
  constexpr int VC = HD / 16;   // value columns of a lane
  constexpr int QLD = HD + 8;
  typedef half_t vrow __attribute__((ext_vector_type(VC)));
  typedef unsigned vwords __attribute__((ext_vector_type(VC / 2)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) half_t s_q[3][ATT_HEADS][QLD];  // rotated queries: rounded, 2^11 and 2^22 times the rests
  __shared__ __align__(16) half_t s_kn[HD], s_vn[HD];      // the new token's row
  __shared__ __align__(16) float s_acc[ATT_WAVES][ATT_HEADS][HD + 4];
  __shared__ float2 s_ml[ATT_WAVES][ATT_HEADS];
  __shared__ int s_last;

  af_prof_begin(p.prof);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int rep = p.n_heads / p.n_kv, gh = p.group_heads, groups = (rep + gh - 1) / gh;
  const int kvh = groups == 1 ? bx : bx / groups, grp = bx - kvh * groups;
  const int heads = min(gh, rep - grp * gh), h0 = kvh * rep + grp * gh;
  const int T = p.kv_len;  // the new token's place
  // cached keys of a split, in whole steps; the last split has the new token as well
  const int KP = (af_ceil_div_small(T, KS) + ATT_STEP - 1) / ATT_STEP * ATT_STEP;
  const bool owns_new = s == KS - 1;
  const int t0 = min(s * KP, T), t1 = owns_new ? T + 1 : min(t0 + KP, T);

  // Four rotated pairs per thread: of a query head's, or of the new key's, which is the last "head".
  const int rh = tid / (HD / 8), ri = tid % (HD / 8) * 4;
  const half_t* vn = p.qkv + (size_t)(p.n_heads + p.n_kv + kvh) * HD;
  const half_t* rsrc = rh < heads ? p.qkv + (size_t)(h0 + rh) * HD : p.qkv + (size_t)(p.n_heads + kvh) * HD;
  const att_h4 ra = *reinterpret_cast<const att_h4*>(rsrc + ri), rb = *reinterpret_cast<const att_h4*>(rsrc + ri + HD / 2);
  att_f4 rc, rs;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    rc[j] = cs_tab[ri + j];
    rs[j] = sn_tab[ri + j];
  }
  const half8 vnew = *reinterpret_cast<const half8*>(vn + tid % (HD / 8) * 8);

  const half_t* Kc = p.k_cache + (size_t)kvh * p.kv_cap * HD;
  const half_t* Vc = p.v_cache + (size_t)kvh * p.kv_cap * HD;
  // Rows of a step; what lies behind the cache is read as its last row and replaced or masked.
  half8 kr[2][TT];
  vrow vr[8];
  const int last = max(min(t1, T) - 1, 0);
  auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned o = (unsigned)min(k0 + i * 16 + n, last) * HD + g * 8;
#pragma unroll
      for (int t = 0; t < TT; ++t) kr[i][t] = af_load_once(reinterpret_cast<const half8*>(Kc + o + t * 32));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned o = (unsigned)min(k0 + (j >> 2) * 16 + g * 4 + (j & 3), last) * HD + n * VC;
      vr[j] = af_load_once(reinterpret_cast<const vrow*>(Vc + o));
    }
  };
  int k0 = t0 + wave * ATT_STEP;
  if (k0 < t1) fetch(k0);
  __builtin_amdgcn_sched_barrier(0);

  if (rh <= heads) {
    att_h4 h[2], mid[2], lo[2];
    // the exponentials below are powers of two
    const float scale = 1.44269504088896340736f / sqrtf((float)HD);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = (float)ra[j], b = (float)rb[j];
      const float x[2] = {__builtin_fmaf(a, rc[j], -(b * rs[j])), __builtin_fmaf(b, rc[j], a * rs[j])};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float q = x[e] * scale;
        h[e][j] = (half_t)q;
        if (h[e][j] == (half_t)0 && q != 0.f) h[e][j] = (half_t)__builtin_copysignf(0x1p-24f, q);
        const float rest = (q - (float)h[e][j]) * 2048.0f;
        mid[e][j] = (half_t)rest;
        lo[e][j] = (half_t)((rest - (float)mid[e][j]) * 2048.0f);
      }
      if (rh == heads) {
        h[0][j] = att_fma_half(ra[j], rc[j], -(b * rs[j]));
        h[1][j] = att_fma_half(rb[j], rc[j], a * rs[j]);
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (rh < heads) {
        *reinterpret_cast<att_h4*>(&s_q[0][rh][ri + e * (HD / 2)]) = h[e];
        *reinterpret_cast<att_h4*>(&s_q[1][rh][ri + e * (HD / 2)]) = mid[e];
        *reinterpret_cast<att_h4*>(&s_q[2][rh][ri + e * (HD / 2)]) = lo[e];
      } else {
        *reinterpret_cast<att_h4*>(&s_kn[ri + e * (HD / 2)]) = h[e];  // fp16, as in the cache
        if (owns_new && grp == 0)
          *reinterpret_cast<att_h4*>(const_cast<half_t*>(Kc) + (size_t)T * HD + ri + e * (HD / 2)) = h[e];
      }
    }
  }
  if (tid < HD / 8) {
    *reinterpret_cast<half8*>(&s_vn[tid * 8]) = vnew;
    if (owns_new && grp == 0) *reinterpret_cast<half8*>(const_cast<half_t*>(Vc) + (size_t)T * HD + tid * 8) = vnew;
  }
  __syncthreads();

  float m = -INFINITY, l = 0.f;  // of head n: maximum (uniform over the lane groups), this lane's sum
  // Dimensions (4 g + r) VC + c of head n: with the weights' rounded values, and with their rests.  These sums run
  // through the instructions (at most sixteen steps; 2000 keys a split: 1.37e-7, additions outside 1.15e-7,
  // fp32 on the vector unit 1.82e-7; the additions cost 0.2 us).
  att_f4 acc[VC], low[VC];
  const att_f4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < VC; ++c) acc[c] = low[c] = zero4;
  const int hn = min(n, heads - 1);  // the rest of the result's columns repeat the last head
  while (k0 < t1) {
    const bool edge = k0 + ATT_STEP > min(t1, T);
    if (edge) {  // the new token's row
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (k0 + i * 16 + n == T) {
#pragma unroll
          for (int t = 0; t < TT; ++t) kr[i][t] = *reinterpret_cast<const half8*>(&s_kn[t * 32 + g * 8]);
        }
    }
    // scores of keys k0 + 16 i + 4 g + r, head n
    float sc[8];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      auto part = [&](int which, int t, att_f4 c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(
            kr[i][t], *reinterpret_cast<const half8*>(&s_q[which][hn][t * 32 + g * 8]), c, 0, 0, 0);
      };
      att_f4 mid = zero4, lo = zero4;
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        lo = part(2, t, lo);
        mid = part(1, t, mid);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) mid[r] = att_rest(mid[r] + lo[r] * (1.0f / 2048.0f)) * (1.0f / 2048.0f);
      att_f4 d = part(0, 0, mid) + part(0, 1, zero4);
      if constexpr (TT == 4) d += part(0, 2, zero4) + part(0, 3, zero4);
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[i * 4 + r] = d[r];
    }
    vwords vw[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) vw[j] = __builtin_bit_cast(vwords, vr[j]);
    if (edge) {
      const vwords vnw = __builtin_bit_cast(vwords, *reinterpret_cast<const vrow*>(&s_vn[n * VC]));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int key = k0 + (j >> 2) * 16 + g * 4 + (j & 3);
        if (key == T) vw[j] = vnw;
        if (key >= t1) {  // behind the split's end: no weight, and no value
          sc[j] = -INFINITY;
#pragma unroll
          for (int c = 0; c < VC / 2; ++c) vw[j][c] = 0u;
        }
      }
    }
    // running softmax
    float mx = sc[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sc[j]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, AF_WAVE));
    mx = fmaxf(mx, __shfl_xor(mx, 32, AF_WAVE));
    mx = fmaxf(mx, m);
    const float safe = mx == -INFINITY ? 0.f : mx;  // nothing but keys without weight so far
    if (__any(m != mx) && k0 >= t0 + ATT_WAVES * ATT_STEP) {
      const float corr = __builtin_amdgcn_exp2f(m - safe);
      l *= corr;
#pragma unroll
      for (int c = 0; c < VC; ++c) {
        acc[c] *= corr;
        low[c] *= corr;
      }
    }
    m = mx;
    // Weights times 2^15 (in the range of fp16; the factor joins behind the exponential, whose argument it
    // would round) as a rounded down value and two rests.
    u32x4 ph, pm, pl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e0 = __builtin_amdgcn_exp2f(sc[2 * i] - safe) * 32768.f, e1 = __builtin_amdgcn_exp2f(sc[2 * i + 1] - safe) * 32768.f;
      l += e0 + e1;
      // no zero for a weight that is not: with the bits of a float or 1, whichever is less
      const att_us2 some = {(unsigned short)min(__builtin_bit_cast(unsigned, e0), 1u), (unsigned short)min(__builtin_bit_cast(unsigned, e1), 1u)};
      const att_h2 hi = __builtin_bit_cast(att_h2, __builtin_elementwise_max(__builtin_bit_cast(att_us2, __builtin_amdgcn_cvt_pkrtz(e0, e1)), some));
      const float r0 = e0 - (float)hi[0], r1 = e1 - (float)hi[1];
      const att_h2 mid = {(half_t)r0, (half_t)r1};
      const att_h2 lo = {(half_t)(r0 - (float)mid[0]), (half_t)(r1 - (float)mid[1])};
      ph[i] = __builtin_bit_cast(unsigned, hi);
      pm[i] = __builtin_bit_cast(unsigned, mid);
      pl[i] = __builtin_bit_cast(unsigned, lo);
    }
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      u32x4 a;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i] = __builtin_amdgcn_perm(vw[2 * i + 1][c / 2], vw[2 * i][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
      const half8 a8 = __builtin_bit_cast(half8, a);
      low[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a8, __builtin_bit_cast(half8, pl), low[c], 0, 0, 0);
      low[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a8, __builtin_bit_cast(half8, pm), low[c], 0, 0, 0);
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a8, __builtin_bit_cast(half8, ph), acc[c], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);  // with the products and the next rows' addresses mixed, registers spill
    k0 += ATT_WAVES * ATT_STEP;
    if (k0 < t1) fetch(k0);
  }
  l += __shfl_xor(l, 16, AF_WAVE);
  l += __shfl_xor(l, 32, AF_WAVE);

  // the waves' sums
  if (n < heads) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < VC; ++c) s_acc[wave][n][(g * 4 + r) * VC + c] = acc[c][r] + att_rest(low[c][r]);
    if (g == 0) s_ml[wave][n] = make_float2(m, l);
  }
  __syncthreads();
  const int d = lane * 2;  // two dimensions per lane, a head per wave
  for (int hh = wave; hh < heads; hh += ATT_WAVES) {
    float M = -INFINITY, L = 0.f, v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int w = 0; w < ATT_WAVES; ++w) M = fmaxf(M, s_ml[w][hh].x);
    const float safe = M == -INFINITY ? 0.f : M;
#pragma unroll
    for (int w = 0; w < ATT_WAVES; ++w) {
      const float f = __builtin_amdgcn_exp2f(s_ml[w][hh].x - safe);
      L += f * s_ml[w][hh].y;
      if (d < HD) {
        v0 += f * s_acc[w][hh][d];
        v1 += f * s_acc[w][hh][d + 1];
      }
    }
    float* mine = p.part + ((size_t)(h0 + hh) * KS + s) * (HD + 2);
    if (d < HD) {
      if (KS == 1)
        *reinterpret_cast<half2v*>(p.out + (size_t)(h0 + hh) * HD + d) = half2v{(half_t)(v0 / L), (half_t)(v1 / L)};
      else
        af_store_agent2(mine + 2 + d, v0, v1);
    }
    if (KS > 1 && lane == 0) af_store_agent2(mine, M, L);
  }
  if (KS == 1) {
    af_prof_end(p.prof);
    return;
  }
  af_stores_done();
  __syncthreads();
  if (tid == 0) {
    int old = af_ticket_take(&p.tickets[af_ticket_of(p.ticket0 + bx)]);
    s_last = (old == KS - 1);
  }
  __syncthreads();
  if (!s_last) {
    af_prof_end(p.prof);
    return;
  }
  // The splits of each head, in split order.  Lane q has the maximum and the weight of split q (KS <= 64); the
  // partials come from other XCDs, so they are fetched sixteen at a time, the first together with those.
  for (int hh = wave; hh < heads; hh += ATT_WAVES) {
    const float* part = p.part + (size_t)(h0 + hh) * KS * (HD + 2);
    const af_float2 ml = af_load_agent2(part + min(lane, KS - 1) * (HD + 2));
    float v0 = 0.f, v1 = 0.f, f = 0.f, L = 1.f;
    for (int q0 = 0; q0 < KS; q0 += 16) {
      af_float2 av[16];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        av[u] = af_load_agent2(part + min(q0 + u, KS - 1) * (HD + 2) + 2 + (d < HD ? d : 0));
      if (q0 == 0) {
        float M = lane < KS ? ml[0] : -INFINITY;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, AF_WAVE));
        f = lane < KS ? __builtin_amdgcn_exp2f(ml[0] - (M == -INFINITY ? 0.f : M)) : 0.f;
        L = af_wave_sum(lane < KS ? f * ml[1] : 0.f);
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (q0 + u < KS) {
          const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f), q0 + u));
          v0 += w * av[u][0];
          v1 += w * av[u][1];
        }
      }
    }
    if (d < HD)
      *reinterpret_cast<half2v*>(p.out + (size_t)(h0 + hh) * HD + d) = half2v{(half_t)(v0 / L), (half_t)(v1 / L)};
  }
  if (tid == 0) af_ticket_reset(&p.tickets[af_ticket_of(p.ticket0 + bx)]);
  af_prof_end(p.prof);
}

template <int HD>
__global__ __launch_bounds__(ATT_THREADS, ATT_WAVES_PER_SIMD(HD)) void attn_decode_kernel(AttnParams p) {
  attn_decode_body<HD>(p, p.cs, p.sn, blockIdx.x, blockIdx.y, gridDim.y);
}

// Caches of fewer than 128 keys, one token: a workgroup per query head on the vector unit, in fp32.  All keys and
// values are requested at once, a wave holds every score (one or two per lane) and forms the softmax for itself, and
// nothing is split over workgroups.  At this size the launch is a chain of dependent steps, and that of the matrix-core
// form is longer whatever the number of keys (us per layer of 512 channels, heads/key heads, keys, matrix cores / this;
// head width 128): 4/2, 17 33.6 / 32.2; 4/2, 90 34.2 / 33.5; 32/32, 60 38.1 / 36.4; 32/32, 64 38.3 / 37.4; 64/8, 64 39.9 /
// 39.6; 64/8, 100 40.2 / 39.7; width 64, 16/4, 64 34.3 / 33.3.  The launch itself: 4/2, 17 5.1 / 4.2.  From 64 keys on the
// second eight rows a lane and the second score cost 0.6 to 1 us (32/32, 63 and 64: 36.4, 37.4).
// KEYS: at most, with the new token's.
template <int HD, int KEYS>
__global__ __launch_bounds__(ATT_THREADS) void attn_short_kernel(AttnParams p) {
  constexpr int LPK = HD / 8;                  // lanes per key (16 bytes each)
  constexpr int KPB = ATT_THREADS / LPK;       // keys of the workgroup at a time
  constexpr int NB = KEYS / KPB, P = KEYS / AF_WAVE;
  __shared__ __align__(16) float s_q[HD], s_kn[HD], s_vn[HD];
  __shared__ float s_sc[KEYS];
  __shared__ __align__(16) float s_pv[KPB][HD];

  af_prof_begin(p.prof);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x, rep = p.n_heads / p.n_kv, kvh = h / rep, T = p.kv_len;
  const half_t* q = p.qkv + (size_t)h * HD;
  const half_t* kn = p.qkv + (size_t)(p.n_heads + kvh) * HD;
  const half_t* vn = p.qkv + (size_t)(p.n_heads + p.n_kv + kvh) * HD;
  half_t* Kc = p.k_cache + (size_t)kvh * p.kv_cap * HD;
  half_t* Vc = p.v_cache + (size_t)kvh * p.kv_cap * HD;
  const int lk = tid % LPK, kq = tid / LPK;

  // q (first wave), the new k (second) and v (the others), and behind them the rows: loads return in order.  A row
  // behind the cache is read as the last one (or as the one that the new token goes to) and not used.
  const half_t* src = wave == 0 ? q : (wave == 1 ? kn : vn);
  const int i = wave < 2 ? lane % (HD / 2) : (tid - 128) % HD;
  const half_t a = src[i], b = src[wave < 2 ? i + HD / 2 : i];
  const float cs = p.cs[lane % (HD / 2)], sn = p.sn[lane % (HD / 2)];
  half8 kr[NB], vr[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const unsigned o = (unsigned)min(kq + u * KPB, max(T - 1, 0)) * HD + lk * 8;
    kr[u] = af_load_once(reinterpret_cast<const half8*>(Kc + o));
    vr[u] = af_load_once(reinterpret_cast<const half8*>(Vc + o));
  }
  __builtin_amdgcn_sched_barrier(0);

  if (wave == 0) {
    if (lane < HD / 2) {
      const float scale = 1.0f / sqrtf((float)HD);
      s_q[i] = __builtin_fmaf((float)a, cs, -((float)b * sn)) * scale;
      s_q[i + HD / 2] = __builtin_fmaf((float)b, cs, (float)a * sn) * scale;
    }
  } else if (wave == 1) {
    if (lane < HD / 2) {
      const half_t ha = att_fma_half(a, cs, -((float)b * sn)), hb = att_fma_half(b, cs, (float)a * sn);
      s_kn[i] = (float)ha;  // fp16, as in the cache
      s_kn[i + HD / 2] = (float)hb;
      if (h % rep == 0) {
        Kc[(size_t)T * HD + i] = ha;
        Kc[(size_t)T * HD + i + HD / 2] = hb;
      }
    }
  } else if (tid - 128 < HD) {
    s_vn[i] = (float)a;
    if (h % rep == 0) Vc[(size_t)T * HD + i] = a;
  }
  __syncthreads();

  float qr[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) qr[c] = s_q[lk * 8 + c];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int key = kq + u * KPB;
    float d = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) d += (float)kr[u][c] * qr[c];
    if (key == T) {
      d = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) d += s_kn[lk * 8 + c] * qr[c];
    }
#pragma unroll
    for (int off = 1; off < LPK; off <<= 1) d += __shfl_xor(d, off, AF_WAVE);
    if (lk == 0) s_sc[key] = key <= T ? d : -INFINITY;
  }
  __syncthreads();

  float e[P], m = -INFINITY, l = 0.f;  // of keys lane, lane + 64
#pragma unroll
  for (int j = 0; j < P; ++j) {
    e[j] = s_sc[j * AF_WAVE + lane];
    m = fmaxf(m, e[j]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, AF_WAVE));
#pragma unroll
  for (int j = 0; j < P; ++j) {
    e[j] = j * AF_WAVE + lane <= T ? expf(e[j] - m) : 0.f;
    l += e[j];
  }
  l = af_wave_sum(l);
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int key = kq + u * KPB;
    const float w = __shfl(e[u * KPB / AF_WAVE], key % AF_WAVE, AF_WAVE);
    if (key < T) {
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] += w * (float)vr[u][c];
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) s_pv[kq][lk * 8 + c] = acc[c];
  __syncthreads();
  if (tid < HD) {
    float v[4] = {__shfl(P > 1 && T >= AF_WAVE ? e[P - 1] : e[0], T % AF_WAVE, AF_WAVE) * s_vn[tid], 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < KPB; ++g) v[g & 3] += s_pv[g][tid];
    p.out[(size_t)h * HD + tid] = (half_t)(((v[0] + v[1]) + (v[2] + v[3])) / l);
  }
  af_prof_end(p.prof);
}

// The same for B tokens in one launch (af_decode_layer_batch): grid (key heads x head groups, key splits, tokens);
// every token has its own caches, length, position and number of key splits.  The rotary table
// of a token is formed here, in fp64 like the host does for the single-token launch
// (angle = pos * theta^(-2i/HD) with the host's theta^(-2i/HD)).
struct AttnBatchParams {
  AttnParams base;          // token 0's qkv / out, the shared sizes; cs / sn unused
  half_t* k_caches[AF_MAX_BATCH];
  half_t* v_caches[AF_MAX_BATCH];
  int kv_lens[AF_MAX_BATCH];
  int poss[AF_MAX_BATCH];
  int splits[AF_MAX_BATCH];  // key splits of each token
  double inv_freq[64];
  long long qkv_stride, out_stride, part_stride;  // elements between the tokens
};

template <int HD>
__global__ __launch_bounds__(ATT_THREADS, ATT_WAVES_PER_SIMD(HD)) void attn_decode_batch_kernel(AttnBatchParams bp) {
  __shared__ float s_cs[HD / 2], s_sn[HD / 2];
  const int b = blockIdx.z;
  const int KS = bp.splits[b];
  if ((int)blockIdx.y >= KS) return;  // uniform for the workgroup: this token has fewer splits
  AttnParams p = bp.base;
  p.qkv += (size_t)b * bp.qkv_stride;
  p.out += (size_t)b * bp.out_stride;
  p.part += (size_t)b * bp.part_stride;
  p.ticket0 = b * p.n_heads;
  p.k_cache = bp.k_caches[b];
  p.v_cache = bp.v_caches[b];
  p.kv_len = bp.kv_lens[b];
  if (threadIdx.x < HD / 2) {
    const double ang = (double)bp.poss[b] * bp.inv_freq[threadIdx.x];
    s_cs[threadIdx.x] = (float)cos(ang);
    s_sn[threadIdx.x] = (float)sin(ang);
  }
  __syncthreads();
  attn_decode_body<HD>(p, s_cs, s_sn, blockIdx.x, blockIdx.y, KS);
}

static int attn_groups(const af_layer_cfg* cfg, int gh) {  // workgroups side by side: key heads x groups of query heads
  const int rep = cfg->n_heads / cfg->n_kv_heads;
  return cfg->n_kv_heads * ((rep + gh - 1) / gh);
}

// Query heads of a workgroup, for one token.  With four, a wave has one head's splits to add up and not two, one
// after the other; with eight the rows of eight query heads are read once and not twice, which only
// caches of more than 3 M key elements notice (us per layer, attention and short GEMVs, 8 / 4; heads/key heads,
// keys): 8/1, 300 35.4 / 34.4; 64/8, 300 40.0 / 39.6; 64/8, 3000 43.5 / 43.6; 64/8, 6001 47.5 / 47.9.  Batches
// fill the chip and take eight (64/8, eight tokens of 512 keys, a layer with short GEMVs 133.7 / 142.4).
static int attn_group_heads(const af_layer_cfg* cfg, int kv_len) {
  return (long long)cfg->n_kv_heads * kv_len * cfg->head_dim <= 3 << 20 ? ATT_HEADS / 2 : ATT_HEADS;
}

// Key splits of one token, 0 if the partial results of enough splits do not fit.  One while the four waves take the
// keys in one step (batches), or in two with a head width of 64, where the step is half as long: no partial results, no
// ticket (one token, when it took this form at any length; one per 64 keys / one; 32/32, 100: 37.1 / 36.1; 64/8, 100:
// 40.1 / 38.2; 8/1, 100: 35.8 / 33.8; width 64, 16/4,
// 200: 34.2 / 33.5, and 256: 34.6 / 35.0).  Beyond that one per 32 keys, a wave's step, and one for the new token,
// up to one workgroup per compute unit and sixteen splits; more only lengthen the sum over them (one per 64 keys /
// this; 16/4, 128: 35.8 / 35.1; 32/32, 200: 37.1 / 36.8; 8/1, 400: 35.8 / 35.5; at 8 / 16 / 32 splits 32/32,
// 695: 38.4 / 39.7 / 43.0; 16/1, 1500: 39.8 / 37.4 / 38.5).  Where that leaves more than 512 keys to a split, twice as
// many (32/32, 3000: 8 splits 45.2, 16 44.2).  Batches: one per 64 keys (64/8, eight tokens of 512 keys 129.8, one
// per 32 133.7).
// `tuned`: the number asked for by option (0: none).  The option is the single-token launch's.
static int attn_splits(const af_ctx* ctx, const af_layer_cfg* cfg, int gh, bool batch, int kv_len, size_t floats, int tuned) {
  int KS = batch ? (kv_len + 63) / 64 : (kv_len + ATT_STEP - 1) / ATT_STEP + 1;
  if (kv_len < (cfg->head_dim == 64 ? 2 : 1) * ATT_WAVES * ATT_STEP) KS = 1;
  int cap = ctx->n_cu / attn_groups(cfg, gh);
  if (cap > 16) cap = 16;
  if (cap < 1) cap = 1;
  if (kv_len > 512 * cap) cap *= 2;
  if (KS > cap) KS = cap;
  if (KS < (kv_len + ATT_MAX_KEYS - 1) / ATT_MAX_KEYS) KS = (kv_len + ATT_MAX_KEYS - 1) / ATT_MAX_KEYS;  // very long caches
  if (tuned > 0) KS = tuned;
  if (KS < 1) KS = 1;
  if (KS > 64) KS = 64;
  while (KS > 1 && (size_t)cfg->n_heads * KS * (cfg->head_dim + 2) > floats) --KS;
  return (kv_len + KS - 1) / KS > ATT_MAX_KEYS ? 0 : KS;
}

int af_launch_attention(af_ctx* ctx, const af_layer_cfg* cfg, const half_t* qkv, void* kc, void* vc,
                        int kv_len, int kv_cap, int pos, half_t* out) {
  const int gh = attn_group_heads(cfg, kv_len);
  const int KS = attn_splits(ctx, cfg, gh, false, kv_len, ctx->lay.attn_floats, ctx->tune_attn_splits);
  if (KS == 0) return AF_EINVAL;
  AttnParams p;
  p.qkv = qkv;
  p.k_cache = (half_t*)kc;
  p.v_cache = (half_t*)vc;
  p.out = out;
  p.part = (float*)(ctx->ws + ctx->lay.attn_part);
  p.tickets = (int*)(ctx->ws + ctx->lay.tickets) + AF_TICKET_ATTN;
  p.ticket0 = 0;
  p.group_heads = gh;
  p.n_heads = cfg->n_heads;
  p.n_kv = cfg->n_kv_heads;
  p.kv_len = kv_len;
  p.kv_cap = kv_cap;
  p.head_dim = cfg->head_dim;
  p.prof = af_prof_take(ctx);
  for (int i = 0; i < cfg->head_dim / 2; ++i) {
    const double ang = (double)pos * pow((double)cfg->rope_theta, -2.0 * (double)i / (double)cfg->head_dim);
    p.cs[i] = (float)cos(ang);
    p.sn[i] = (float)sin(ang);
  }
  if (kv_len < 128 && ctx->tune_attn_splits == 0) {
    const dim3 grid(cfg->n_heads), threads(ATT_THREADS);
    if (cfg->head_dim == 128 && kv_len < 64)
      hipLaunchKernelGGL((attn_short_kernel<128, 64>), grid, threads, 0, ctx->stream, p);
    else if (cfg->head_dim == 128)
      hipLaunchKernelGGL((attn_short_kernel<128, 128>), grid, threads, 0, ctx->stream, p);
    else if (kv_len < 64)
      hipLaunchKernelGGL((attn_short_kernel<64, 64>), grid, threads, 0, ctx->stream, p);
    else
      hipLaunchKernelGGL((attn_short_kernel<64, 128>), grid, threads, 0, ctx->stream, p);
    AF_LAUNCH_CHECK();
    return AF_OK;
  }
  dim3 grid(attn_groups(cfg, p.group_heads), KS);
  if (cfg->head_dim == 128)
    hipLaunchKernelGGL(attn_decode_kernel<128>, grid, dim3(ATT_THREADS), 0, ctx->stream, p);
  else
    hipLaunchKernelGGL(attn_decode_kernel<64>, grid, dim3(ATT_THREADS), 0, ctx->stream, p);
  AF_LAUNCH_CHECK();
  return AF_OK;
}

int af_launch_attention_batch(af_ctx* ctx, const af_layer_cfg* cfg, int B, const half_t* qkv,
                              long long qkv_stride, void* const* kcs, void* const* vcs, const int* kv_len,
                              int kv_cap, const int* pos, half_t* out, long long out_stride) {
  AttnBatchParams bp{};
  AttnParams& p = bp.base;
  int ks_max = 1;
  const size_t per_split = (size_t)cfg->n_heads * (cfg->head_dim + 2);
  for (int b = 0; b < B; ++b) {
    const int KS = attn_splits(ctx, cfg, ATT_HEADS, true, kv_len[b], ctx->lay.attn_floats / B, 0);
    if (KS == 0) return AF_EINVAL;
    bp.splits[b] = KS;
    if (KS > ks_max) ks_max = KS;
    bp.k_caches[b] = (half_t*)kcs[b];
    bp.v_caches[b] = (half_t*)vcs[b];
    bp.kv_lens[b] = kv_len[b];
    bp.poss[b] = pos[b];
  }
  if ((size_t)B * ks_max * per_split > ctx->lay.attn_floats) return AF_EWORKSPACE;
  p.qkv = qkv;
  p.out = out;
  p.part = (float*)(ctx->ws + ctx->lay.attn_part);
  p.tickets = (int*)(ctx->ws + ctx->lay.tickets) + AF_TICKET_ATTN;
  p.ticket0 = 0;
  p.group_heads = ATT_HEADS;
  p.n_heads = cfg->n_heads;
  p.n_kv = cfg->n_kv_heads;
  p.kv_cap = kv_cap;
  p.head_dim = cfg->head_dim;
  p.prof = nullptr;
  for (int i = 0; i < cfg->head_dim / 2; ++i)
    bp.inv_freq[i] = pow((double)cfg->rope_theta, -2.0 * (double)i / (double)cfg->head_dim);
  bp.qkv_stride = qkv_stride;
  bp.out_stride = out_stride;
  bp.part_stride = (long long)ks_max * (long long)per_split;
  dim3 grid(attn_groups(cfg, p.group_heads), ks_max, B);
  if (cfg->head_dim == 128)
    hipLaunchKernelGGL(attn_decode_batch_kernel<128>, grid, dim3(ATT_THREADS), 0, ctx->stream, bp);
  else
    hipLaunchKernelGGL(attn_decode_batch_kernel<64>, grid, dim3(ATT_THREADS), 0, ctx->stream, bp);
  AF_LAUNCH_CHECK();
  return AF_OK;
}
