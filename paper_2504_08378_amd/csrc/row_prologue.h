// Workgroup-local front end of the fused GEMV kernels: produce the operator's input vector in
// LDS (plain copy, RMSNorm, or SiLU(gate)*up) and, when asked, run the activation selection
// (Section 2.1 Top-K sparsity / Section 6 threshold form; Section 4 operation T) right there,
// so that operation T needs no kernel of its own: every workgroup of the GEMV repeats the
// cheap O(n) selection on its own copy of the vector and keeps only its split of the
// ascending index list.  The arithmetic is the same as in select.hip (exact two-digit radix
// select on the 15-bit magnitude key, ties to the lower index).
#pragma once
#include "af_internal.h"

// Replicas of the digit histograms.  Measured 1 / 2 / 4 / 8 / 16 on the synthetic activations:
// 2.360 / 2.364 / 2.367 / 2.378 / 2.411 ms per 7B token (zeroing and merging the replicas cost
// more than the atomic conflicts they avoid); 4 keeps a vector of equal magnitudes, which sends
// every lane to one bin, at a quarter of the serialisation a single table would see.
#ifndef RP_HIST_COPIES
#define RP_HIST_COPIES 4
#endif
#define RP_SCRATCH_WORDS (384 * RP_HIST_COPIES)  // both digit tables; reused by the caller afterwards
// Elements per LDS / global access of the element passes.  With 4 a 4096-wide input gives every
// one of 1024 threads one vector; with 8 half of the threads would idle while the others walk
// twice as many elements one after the other, and those serial walks are what the front end
// spends its time in.
#ifndef RP_EV
#define RP_EV 4
#endif
typedef _Float16 rp_half __attribute__((ext_vector_type(RP_EV)));
typedef unsigned short rp_u16 __attribute__((ext_vector_type(RP_EV)));

// Class of a wave's share of a split's channels (1024-thread workgroups): up to 64, 128, 256 channels, more.
static inline int gemv_range_class(int n, int S) {
  const int share = ((n / RP_EV + S - 1) / S * RP_EV + 15) / 16;
  return share <= 64 ? 0 : (share <= 128 ? 1 : (share <= 256 ? 2 : 3));
}

template <int THREADS>
struct RowPrologue {
  static constexpr int WAVES = THREADS / AF_WAVE;

  struct Smem {
    unsigned wave_tot[WAVES];
    float red[WAVES];
    unsigned digit, above;
    // router of a mixture-of-experts block run inside the gate|up launch
    float rpart[WAVES][AF_MOE_MAX_EXPERTS];
    float logit[AF_MOE_MAX_EXPERTS];
    int experts[AF_MOE_MAX_TOP];
    float weights[AF_MOE_MAX_TOP];
  };

  // Histogram scratch: RP_HIST_COPIES replicas, replica-major (replica r of bin b at
  // r * 256 + b): lanes of one replica that hit different bins hit different banks, and the
  // merge reads 256 consecutive words per replica.  First 256-bin table at word 0, the
  // 128-bin table of the second digit behind it.
  static constexpr int H1 = 0;
  static constexpr int H2 = 256 * RP_HIST_COPIES;

  static __device__ __forceinline__ void zero_hist(unsigned* hist) {
    for (int i = threadIdx.x; i < RP_SCRATCH_WORDS; i += THREADS) hist[i] = 0;
  }

  // first-digit counts of one vector into this lane's replica
  static __device__ __forceinline__ void count_digit1(unsigned* hist, const rp_half& h) {
    const rp_u16 b = __builtin_bit_cast(rp_u16, h);
    const int rep = threadIdx.x & (RP_HIST_COPIES - 1);
#pragma unroll
    for (int c = 0; c < RP_EV; ++c) atomicAdd(&hist[H1 + rep * 256 + ((b[c] & 0x7FFFu) >> 7)], 1u);
  }

  // Fill xs[0..n) with the fp16 bits of the operator input (n % 8 == 0).  Global reads are
  // RP_EV-element vectors issued four at a time, so a thread waits for memory once per batch and
  // not once per element.
  // `hist`, when given (top-k selection follows), receives the histogram of the first radix
  // digit on the way: the values are counted while they are still in registers, which saves
  // the selection a pass over LDS and two barriers (select_split is told so).
  static __device__ __forceinline__ void produce(const af_row_src& r, unsigned short* xs, Smem& sm,
                                                 bool store_x, int store_phase, int store_stride,
                                                 unsigned* hist = nullptr) {
    // RMSNorm of a vector of at most one access per thread (n <= RP_EV * THREADS: 4096 channels
    // for the 1024-thread kernels) takes the copy of the code without the batch of four and its
    // masks: the front end is bound by the instructions its waves issue, and that copy issues
    // fewer (4096 -> 12288 15.7 -> 15.4 us, 4096 -> 22016 21.2 -> 20.8 us, when these went through
    // here; with early rows they take produce_raw, and what is left is short streams, the router's
    // launches, given rows and the whole-layer kernel).  The other two producers measured no better
    // with a second copy, so they keep the one.
    if (r.pro == AF_PRO_RMSNORM && r.n <= RP_EV * THREADS)
      produce_batched<1>(r, xs, sm, store_x, store_phase, store_stride, hist);
    else
      produce_batched<4>(r, xs, sm, store_x, store_phase, store_stride, hist);
  }

  template <int B>
  static __device__ __forceinline__ void produce_batched(const af_row_src& r, unsigned short* xs, Smem& sm,
                                                         bool store_x, int store_phase, int store_stride,
                                                         unsigned* hist) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = r.n, nvec = n / RP_EV;
    rp_half* xv = reinterpret_cast<rp_half*>(xs);
    const rp_half* src = reinterpret_cast<const rp_half*>(r.src);
    rp_half zero;
#pragma unroll
    for (int c = 0; c < RP_EV; ++c) zero[c] = (half_t)0;
    if (hist != nullptr) {
      zero_hist(hist);
      if (r.pro != AF_PRO_RMSNORM) __syncthreads();  // the norm has a barrier of its own before it counts
    }
    if (r.pro == AF_PRO_NONE) {
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = (v0 + u * THREADS < nvec) ? src[v0 + u * THREADS] : zero;
#pragma unroll
        for (int u = 0; u < B; ++u)
          if (v0 + u * THREADS < nvec) {
            xv[v0 + u * THREADS] = t[u];
            if (hist != nullptr) count_digit1(hist, t[u]);
          }
      }
    } else if (r.pro == AF_PRO_RMSNORM) {
      const rp_half* gain = reinterpret_cast<const rp_half*>(r.gain);
      // When one batch per thread covers the vector (the usual case) the gains are fetched
      // together with the source, so the sum-of-squares reduction does not sit between two
      // dependent global round trips.
      const bool single = nvec <= B * THREADS;
      rp_half g[B];
      float ss = 0.f;
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = (v0 + u * THREADS < nvec) ? src[v0 + u * THREADS] : zero;
        if (single) {
#pragma unroll
          for (int u = 0; u < B; ++u) g[u] = (v0 + u * THREADS < nvec) ? gain[v0 + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
#pragma unroll
          for (int c = 0; c < RP_EV; ++c) ss += (float)t[u][c] * (float)t[u][c];
          if (v0 + u * THREADS < nvec) xv[v0 + u * THREADS] = t[u];  // raw; normalised below
        }
      }
      ss = af_wave_sum(ss);
      if (lane == 0) sm.red[wave] = ss;
      __syncthreads();
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += sm.red[w];
      const float scale = 1.0f / sqrtf(tot / (float)n + r.eps);
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        if (!single) {
#pragma unroll
          for (int u = 0; u < B; ++u) g[u] = (v0 + u * THREADS < nvec) ? gain[v0 + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (v0 + u * THREADS < nvec) {
            rp_half h = xv[v0 + u * THREADS];   // each thread revisits the vectors it wrote
#pragma unroll
            for (int c = 0; c < RP_EV; ++c) h[c] = (half_t)((float)h[c] * scale * (float)g[u][c]);
            xv[v0 + u * THREADS] = h;
            if (hist != nullptr) count_digit1(hist, h);
          }
        }
      }
    } else {  // AF_PRO_SILUMUL: src = gate[n] | up[n]
      const rp_half* up = reinterpret_cast<const rp_half*>(r.src + n);
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        rp_half g[B], u8[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const bool ok = v0 + u * THREADS < nvec;
          g[u] = ok ? src[v0 + u * THREADS] : zero;
          u8[u] = ok ? up[v0 + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (v0 + u * THREADS < nvec) {
            rp_half h;
#pragma unroll
            for (int c = 0; c < RP_EV; ++c) {
              const float gg = (float)g[u][c];
              h[c] = (half_t)(gg * __builtin_amdgcn_rcpf(1.0f + __expf(-gg)) * (float)u8[u][c]);
            }
            xv[v0 + u * THREADS] = h;
            if (hist != nullptr) count_digit1(hist, h);
          }
        }
      }
    }
    __syncthreads();
    if (store_x && r.x_out != nullptr) {
      rp_half* dst = reinterpret_cast<rp_half*>(r.x_out);
      for (int v = store_phase * THREADS + tid; v < nvec; v += store_stride * THREADS) dst[v] = xv[v];
    }
  }

  // digit d with count(digit > d) < want <= count(digit >= d); result in sm.digit / sm.above
  static __device__ __forceinline__ void find_digit(const unsigned* hist, Smem& sm, int nbins,
                                                    unsigned want) {
    // The first wave sums the replicas itself, four neighbouring bins per lane and 16 bytes
    // per LDS read, and scans them; the others only wait for the answer (one barrier).
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x;
    if (tid < AF_WAVE) {
      unsigned cnt[4] = {0u, 0u, 0u, 0u};
      if (4 * tid < nbins) {
#pragma unroll
        for (int c = 0; c < RP_HIST_COPIES; ++c) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(hist + c * nbins + 4 * tid);
          cnt[0] += v[0];
          cnt[1] += v[1];
          cnt[2] += v[2];
          cnt[3] += v[3];
        }
      }
      const unsigned mine = cnt[0] + cnt[1] + cnt[2] + cnt[3];
      const unsigned pre = af_wave_incl_scan(mine);                       // bins of lanes <= mine
      const unsigned all = (unsigned)__builtin_amdgcn_readlane((int)pre, 63);
      unsigned above = all - pre;                                         // bins of higher lanes
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        if (above < want && want <= above + cnt[q]) {
          sm.digit = 4 * tid + q;
          sm.above = above;
        }
        above += cnt[q];
      }
    }
    __syncthreads();
  }

  // exclusive prefix over the workgroup in thread order; *total gets the sum over all threads.
  // sm.wave_tot must not be rewritten before the next barrier of the caller.
  static __device__ __forceinline__ unsigned excl_scan(unsigned v, Smem& sm, unsigned* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned inc = af_wave_incl_scan(v);
    if (lane == 63) sm.wave_tot[wave] = inc;
    __syncthreads();
    unsigned base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const unsigned t = sm.wave_tot[w];
      if (w < wave) base += t;
      tot += t;
    }
    *total = tot;
    return base + inc - v;
  }

  // |x| > t as an integer test on the magnitude key: key > bits(largest fp16 <= t) for t >= 0;
  // -1 lets every key pass for t < 0.  (NaN is kept out by the separate key <= 0x7C00 test.)
  static __device__ __forceinline__ int threshold_key(float t) {
    if (t < 0.f) return -1;
    typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
    const fp16x2 h = __builtin_amdgcn_cvt_pkrtz(t, 0.f);  // toward zero = downward for t >= 0
    return (int)(__builtin_bit_cast(unsigned, h) & 0x7FFFu);
  }

  // Threshold selection without an index list for the whole vector (Section 6: a channel is
  // active iff its magnitude passes the preloaded threshold, which needs no look at any other
  // channel).  The channels are cut into S contiguous ranges of whole RP_EV-element vectors;
  // workgroup s builds x only for its range, in xs[0 .. RP_EV * vectors of the range), and lists
  // the channels of that range that pass, as (index << 16 | fp16 bits).  RMSNorm still reads
  // the whole source once for the sum of squares.  Returns the number of list entries.
  // The caller guarantees RP_EV * ceil(n / RP_EV / S) <= capacity of `list` (8 * ceil(n / 8 / S)
  // is at least that).
  static __device__ __forceinline__ int threshold_range(const af_row_src& r, unsigned short* xs,
                                                        Smem& sm, unsigned* list, int S, int s,
                                                        bool store_x) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = r.n, nvec = n / RP_EV;
    const int V = af_ceil_div_small(nvec, S);
    const int vs0 = min(s * V, nvec), vs1 = min(vs0 + V, nvec), nv = vs1 - vs0;
    constexpr int B = 4;
    rp_half* xv = reinterpret_cast<rp_half*>(xs);
    const rp_half* src = reinterpret_cast<const rp_half*>(r.src);
    rp_half zero;
#pragma unroll
    for (int c = 0; c < RP_EV; ++c) zero[c] = (half_t)0;

    if (r.pro == AF_PRO_NONE) {
      for (int i0 = tid; i0 < nv; i0 += B * THREADS) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = (i0 + u * THREADS < nv) ? src[vs0 + i0 + u * THREADS] : zero;
#pragma unroll
        for (int u = 0; u < B; ++u)
          if (i0 + u * THREADS < nv) xv[i0 + u * THREADS] = t[u];
      }
    } else if (r.pro == AF_PRO_SILUMUL) {
      const rp_half* up = reinterpret_cast<const rp_half*>(r.src + n);
      for (int i0 = tid; i0 < nv; i0 += B * THREADS) {
        rp_half g[B], u8[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const bool ok = i0 + u * THREADS < nv;
          g[u] = ok ? src[vs0 + i0 + u * THREADS] : zero;
          u8[u] = ok ? up[vs0 + i0 + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (i0 + u * THREADS < nv) {
            rp_half h;
#pragma unroll
            for (int c = 0; c < RP_EV; ++c) {
              const float gg = (float)g[u][c];
              h[c] = (half_t)(gg * __builtin_amdgcn_rcpf(1.0f + __expf(-gg)) * (float)u8[u][c]);
            }
            xv[i0 + u * THREADS] = h;
          }
        }
      }
    } else {  // AF_PRO_RMSNORM
      const rp_half* gain = reinterpret_cast<const rp_half*>(r.gain);
      // the range's own vectors (raw) and their gains travel with the first batch of the
      // full pass, so there is one global round trip before the reduction
      const bool single = nv <= B * THREADS;
      rp_half g[B];
      if (single) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const bool ok = tid + u * THREADS < nv;
          t[u] = ok ? src[vs0 + tid + u * THREADS] : zero;
          g[u] = ok ? gain[vs0 + tid + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
          if (tid + u * THREADS < nv) xv[tid + u * THREADS] = t[u];
      } else {
        for (int i = tid; i < nv; i += THREADS) xv[i] = src[vs0 + i];
      }
      float ss = 0.f;
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = (v0 + u * THREADS < nvec) ? src[v0 + u * THREADS] : zero;
#pragma unroll
        for (int u = 0; u < B; ++u) {
#pragma unroll
          for (int c = 0; c < RP_EV; ++c) ss += (float)t[u][c] * (float)t[u][c];
        }
      }
      ss = af_wave_sum(ss);
      if (lane == 0) sm.red[wave] = ss;
      __syncthreads();
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += sm.red[w];
      const float scale = 1.0f / sqrtf(tot / (float)n + r.eps);
      for (int i0 = tid; i0 < nv; i0 += B * THREADS) {
        if (!single) {
#pragma unroll
          for (int u = 0; u < B; ++u) g[u] = (i0 + u * THREADS < nv) ? gain[vs0 + i0 + u * THREADS] : zero;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (i0 + u * THREADS < nv) {
            rp_half h = xv[i0 + u * THREADS];   // each thread revisits the vectors it wrote
#pragma unroll
            for (int c = 0; c < RP_EV; ++c) h[c] = (half_t)((float)h[c] * scale * (float)g[u][c]);
            xv[i0 + u * THREADS] = h;
          }
        }
      }
    }
    __syncthreads();
    if (store_x && r.x_out != nullptr) {
      rp_half* dst = reinterpret_cast<rp_half*>(r.x_out);
      for (int i = tid; i < nv; i += THREADS) dst[vs0 + i] = xv[i];
    }

    return range_list(r, xs, sm, list, vs0, nv);
  }

  // Threshold compare, scan and list over nv vectors of x that lie in LDS at xs; the first of
  // them is vector vs0 of the operator input.  Every thread owns a contiguous run.
  static __device__ __forceinline__ int range_list(const af_row_src& r, const unsigned short* xs,
                                                   Smem& sm, unsigned* list, int vs0, int nv) {
    const int tid = threadIdx.x;
    const int T = threshold_key(r.t);
    const int cv = (nv + THREADS - 1) / THREADS;
    const int v0 = min(tid * cv, nv), v1 = min(v0 + cv, nv);
    const rp_u16* xb = reinterpret_cast<const rp_u16*>(xs);
    unsigned gt = 0;
    for (int v = v0; v < v1; ++v) {
      const rp_u16 b = xb[v];
#pragma unroll
      for (int c = 0; c < RP_EV; ++c) {
        const unsigned key = b[c] & 0x7FFFu;
        gt += ((int)key > T) & (key <= 0x7C00u);
      }
    }
    unsigned tot;
    unsigned pos = excl_scan(gt, sm, &tot);
    if (gt != 0) {
      for (int v = v0; v < v1; ++v) {
        const rp_u16 b = xb[v];
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) {
          const unsigned bits = b[c];
          const unsigned key = bits & 0x7FFFu;
          if (((int)key > T) & (key <= 0x7C00u)) {
            list[pos] = ((unsigned)((vs0 + v) * RP_EV + c) << 16) | bits;
            ++pos;
          }
        }
      }
    }
    __syncthreads();
    return (int)tot;
  }

  // Threshold selection of split s's channel range when the whole x already lies in LDS (the
  // router below needs all of it): the compare / scan / list part of threshold_range alone.
  static __device__ __forceinline__ int threshold_range_of_full(const af_row_src& r,
                                                                const unsigned short* xs, Smem& sm,
                                                                unsigned* list, int S, int s) {
    const int nvec = r.n / RP_EV;
    const int V = af_ceil_div_small(nvec, S);
    const int vs0 = min(s * V, nvec), vs1 = min(vs0 + V, nvec);
    return range_list(r, xs + (size_t)vs0 * RP_EV, sm, list, vs0, vs1 - vs0);
  }

  // The `top` largest of E logits (ties to the lower expert, slot 0 the largest) and the
  // softmax over them; one thread.
  static __device__ __forceinline__ void router_pick(const float* logit, int E, int top, int* experts,
                                                     float* weights) {
    unsigned taken = 0;
    float z0 = 0.f, den = 0.f;
    for (int s = 0; s < top; ++s) {
      int best = -1;
      for (int e = 0; e < E; ++e)
        if (!((taken >> e) & 1u) && (best < 0 || logit[e] > logit[best])) best = e;
      taken |= 1u << best;
      experts[s] = best;
      if (s == 0) z0 = logit[best];
      weights[s] = expf(logit[best] - z0);
      den += weights[s];
    }
    for (int s = 0; s < top; ++s) weights[s] /= den;
  }

  // Router of a mixture-of-experts block inside the GEMV's front end: logits[e] = Wr[e] . x over
  // the x in LDS (n <= 8 * THREADS; wr[e] holds this thread's 8 router weights of expert e,
  // fetched by the caller before x was built), reduced lanes -> waves -> one lane per expert in a
  // fixed order, then the pick.  Leaves sm.experts / sm.weights / sm.logit for every thread.
  template <int E_MAX>
  static __device__ __forceinline__ void router_in_lds(const unsigned short* xs, int n, Smem& sm,
                                                       const half8 (&wr)[E_MAX], int E, int top) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const half8* xv = reinterpret_cast<const half8*>(xs);
    float acc[E_MAX];
#pragma unroll
    for (int e = 0; e < E_MAX; ++e) acc[e] = 0.f;
    if (tid < (n >> 3)) {
      const half8 x8 = xv[tid];
#pragma unroll
      for (int e = 0; e < E_MAX; ++e)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[e] += (float)wr[e][c] * (float)x8[c];
    }
#pragma unroll
    for (int e = 0; e < E_MAX; ++e) {
      const float t = af_wave_sum(acc[e]);
      if (lane == 0) sm.rpart[wave][e] = t;
    }
    __syncthreads();
    if (tid < E) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) t += sm.rpart[w][tid];
      sm.logit[tid] = t;
    }
    __syncthreads();
    if (tid == 0) router_pick(sm.logit, E, top, sm.experts, sm.weights);
    __syncthreads();
  }

  // ---- early rows ---------------------------------------------------------------------------
  // A top-k front end is some 4 us in which memory is idle.  Most of the rows it will keep are
  // obvious before it has run: a wave looks at (up to 64, one per lane) channels of its own, takes
  // the largest of them and requests their rows before the front end starts, so that they arrive
  // behind it.  A row taken early that the exact selection then does not keep is dropped (its
  // products are not formed); the selection lists the rows that were not taken.  A wave has to know
  // its channels beforehand, so the channels and not the list are cut into splits: they are dealt
  // out in small groups (af_dealt_channel), because what is kept may lie together (whole heads
  // at the o projection).  With one contiguous range per split, half of the vector 6 times the other
  // took 26.1 us for 4096 -> 22016 and 54.6 for 28672 -> 8192, where even inputs take 21.2 and 50.5.
  // Wave w of every split has its groups in the same sixteenth of the vector, its stretch; it counts
  // the ties of all of that for their ranks, so what it took stays in its own registers.
  struct Early {
    uint2 tot[WAVES];  // per-wave counts of the selection
    unsigned ties[WAVES];
    int last_tie;  // the last channel of the whole vector that is kept with the k-th magnitude
    int done;      // waves that have streamed their rows
  };
  struct EarlyWave {            // uniform over the wave, but for ch
    int cycles, q0, q1;         // of the deal, and the wave's
    int S, s;                   // splits, and the workgroup's own
    int ch, ch1;                // this lane's channels of the wave's first 64 and of its next, -1: none
    unsigned long long taken;   // bit l: lane l's channel was taken
    unsigned long long kept;    // bit l: lane l's channel is kept by the selection
    int T;                      // the k-th magnitude's key, and how many channels are kept with it
    unsigned quota;
  };
  template <int B>
  struct Raw {  // one thread's share of the operator's source: NONE x; RMSNORM hidden, gain; SILUMUL gate, up
    rp_half a[B], b[B];
  };

  static __device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  // This lane's channel of pass i over the wave's channels, -1: none.
  static __device__ __forceinline__ int early_channel(const EarlyWave& ew, int i, int n) {
    const int l = i << 6 | (int)(threadIdx.x & 63);
    const int j = af_dealt_channel(ew.q0, ew.S, ew.s, wave_id(), l);
    return l < own_channels(ew) && j < n ? j : -1;
  }
  static __device__ __forceinline__ int own_channels(const EarlyWave& ew) { return (ew.q1 - ew.q0) * AF_DEAL; }
  // cycles: af_dealt_cycles(n, S)
  static __device__ __forceinline__ EarlyWave early_block(int n, int S, int s, int cycles) {
    EarlyWave ew;
    ew.cycles = cycles;
    ew.q0 = af_dealt_cycle(cycles, wave_id(), WAVES);
    ew.q1 = af_dealt_cycle(cycles, wave_id() + 1, WAVES);
    ew.S = S;
    ew.s = s;
    ew.ch = early_channel(ew, 0, n);
    ew.ch1 = -1;
    ew.taken = ew.kept = 0;
    return ew;
  }
  // Wave w's stretch in groups of 8 channels (n % 8 == 0), and the pieces (of 32
  // groups) of the longest stretch.
  static constexpr int GROUP = 8;
  static __device__ __forceinline__ int stretch_begin(const EarlyWave& ew, int w, int n) {
    return min(af_dealt_cycle(ew.cycles, w, WAVES) * ew.S * (AF_DEAL / GROUP), n / GROUP);
  }
  static __device__ __forceinline__ int stretch_pieces(const EarlyWave& ew) {
    return ((ew.cycles + WAVES - 1) / WAVES * ew.S * (AF_DEAL / GROUP) + 31) / 32;
  }
  // Does workgroup j of the launch write any piece of the index list?
  static __device__ __forceinline__ bool early_lists(const af_row_src& r, const EarlyWave& ew, int j) {
    return r.idx_out != nullptr && j < stretch_pieces(ew) * WAVES;
  }
  // Of a group's magnitude keys, how many are T / lie above T: two keys to a word, whose sums with
  // what is missing to 0x8000 carry into the sign bits (a compare and an addition for every key made
  // the look at the stretch the longest part of the selection).
  typedef unsigned group_keys __attribute__((ext_vector_type(GROUP / 2)));
  static __device__ __forceinline__ unsigned group_at(const group_keys b, int T) {
    const unsigned t2 = (unsigned)T | (unsigned)T << 16;
    unsigned other = 0;
#pragma unroll
    for (int c = 0; c < GROUP / 2; ++c)
      other += (unsigned)__popc((((b[c] ^ t2) & 0x7FFF7FFFu) + 0x7FFF7FFFu) & 0x80008000u);
    return GROUP - other;
  }
  static __device__ __forceinline__ unsigned group_above(const group_keys b, int T) {
    const unsigned m = 0x7FFFu - (unsigned)min(T, 0x7FFF), m2 = m | m << 16;
    unsigned n = 0;
#pragma unroll
    for (int c = 0; c < GROUP / 2; ++c) n += (unsigned)__popc(((b[c] & 0x7FFF7FFFu) + m2) & 0x80008000u);
    return n;
  }

  static __device__ __forceinline__ float silu_mul(float g, float u) {
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
  }

  // All of the thread's source loads, in flight together (n <= RP_EV * B * THREADS).
  template <int B>
  static __device__ __forceinline__ void load_raw(const af_row_src& r, Raw<B>& raw) {
    const int nvec = r.n / RP_EV;
    const rp_half* a = reinterpret_cast<const rp_half*>(r.src);
    const rp_half* b = reinterpret_cast<const rp_half*>(r.pro == AF_PRO_RMSNORM ? r.gain : r.src + r.n);
    rp_half zero;
#pragma unroll
    for (int c = 0; c < RP_EV; ++c) zero[c] = (half_t)0;
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int v = threadIdx.x + u * THREADS;
      raw.a[u] = v < nvec ? a[v] : zero;
      if (r.pro != AF_PRO_NONE) raw.b[u] = v < nvec ? b[v] : zero;
    }
  }

  // x into xs and (unless null) the first digit's histogram into `hist` (zeroed by the caller), from the loaded
  // source; the arithmetic is produce()'s.  The caller barriers between zeroing and this call.
  template <int B>
  static __device__ __forceinline__ void produce_raw(const af_row_src& r, Raw<B>& raw, unsigned short* xs,
                                                     Smem& sm, bool store_x, int store_phase,
                                                     int store_stride, unsigned* hist) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nvec = r.n / RP_EV;
    rp_half* xv = reinterpret_cast<rp_half*>(xs);
    float scale = 1.f;
    if (r.pro == AF_PRO_RMSNORM) {
      float ss = 0.f;
#pragma unroll
      for (int u = 0; u < B; ++u)
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) ss += (float)raw.a[u][c] * (float)raw.a[u][c];
      ss = af_wave_sum(ss);
      if (lane == 0) sm.red[wave] = ss;
    }
    __syncthreads();  // the norm's partial sums, and the zeroed histogram
    if (r.pro == AF_PRO_RMSNORM) {
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += sm.red[w];
      scale = 1.0f / sqrtf(tot / (float)r.n + r.eps);
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int v = tid + u * THREADS;
      if (v < nvec) {
        rp_half h = raw.a[u];
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) {
          if (r.pro == AF_PRO_RMSNORM) h[c] = (half_t)((float)h[c] * scale * (float)raw.b[u][c]);
          if (r.pro == AF_PRO_SILUMUL) h[c] = (half_t)silu_mul((float)h[c], (float)raw.b[u][c]);
        }
        xv[v] = h;
        if (hist != nullptr) count_digit1(hist, h);
      }
    }
    __syncthreads();
    if (store_x && r.x_out != nullptr) {
      rp_half* dst = reinterpret_cast<rp_half*>(r.x_out);
      for (int v = store_phase * THREADS + tid; v < nvec; v += store_stride * THREADS) dst[v] = xv[v];
    }
  }

  // The two source values of this lane's channel.
  static __device__ __forceinline__ void early_load(const af_row_src& r, const EarlyWave& ew, half_t* a,
                                                    half_t* b) {
    const int j = max(ew.ch, 0);
    *a = r.src[j];
    *b = r.pro == AF_PRO_NONE ? (half_t)1 : (r.pro == AF_PRO_RMSNORM ? r.gain[j] : r.src[r.n + j]);
  }

  // Choose at most CAP of the wave's first 64 channels; row[0..count) gets (lane << 16 | channel).  The
  // magnitude is the producer's up to the norm's common factor.  The cut is the largest value of
  // the key's exponent and first mantissa bit that at least `want` of the channels reach: one
  // compare, ballot and population count per bit.  want is at most 3/4 of the channels that are
  // kept on average, so that what the cut lets in lies above the k-th magnitude almost always.
  // The cut resolves half an octave, so more than `want` can reach it, and up to CAP of them are
  // taken: with magnitudes that are all alike, some that are dropped.  Stopping at `want` instead
  // saves those 0.1-0.3 us and costs spread magnitudes as much (80 %: 28672 -> 8192 29.8 -> 30.3 us,
  // 8192 -> 10240 15.8 -> 15.9); so does taking none where the cut lets in twice the average.
  template <int CAP>
  static __device__ __forceinline__ int early_pick(const af_row_src& r, EarlyWave& ew, unsigned* row, half_t a,
                                                   half_t b) {
    const int lane = threadIdx.x & 63;
    const float x = r.pro == AF_PRO_SILUMUL ? silu_mul((float)a, (float)b) : (float)a * (float)b;
    const int looked = __popcll(__ballot(ew.ch >= 0));
    const unsigned key = ew.ch >= 0 ? __builtin_bit_cast(unsigned short, (half_t)x) & 0x7FFFu : 0u;
    const int share = (int)((float)looked * 0.75f * (float)r.k * __builtin_amdgcn_rcpf((float)r.n));
    const int want = min(CAP, share);
    unsigned T = 0;
#pragma unroll
    for (int bit = 14; bit >= 9; --bit) {
      const unsigned t = T | (1u << bit);
      if (__popcll(__ballot(key >= t)) >= want) T = t;
    }
    const unsigned long long cand = want > 0 ? __ballot(key >= T && ew.ch >= 0) : 0ull;
    const int rank = (int)lanes_below(cand);
    const bool mine = ((cand >> lane) & 1ull) && rank < CAP;
    ew.taken = __ballot(mine);
    if (mine) row[rank] = (unsigned)(lane << 16 | ew.ch);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // row[] is read by the other lanes of this wave
    __builtin_amdgcn_wave_barrier();
    return __popcll(ew.taken);
  }

  // Exact top-k over xs (first digit already counted in `hist`), restricted to the channels dealt to
  // this split: list[] gets those that are kept and were not taken early, first those above the
  // k-th magnitude, then the ties, each in ascending order; returns their number.  ew.kept tells
  // which of the wave's first 64 channels are kept.  j: the workgroup's number in the launch.
  static __device__ __forceinline__ int select_dealt(const af_row_src& r, const unsigned short* xs,
                                                     unsigned* hist, Smem& sm, Early& el, EarlyWave& ew,
                                                     unsigned* list, int j) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = wave_id();
    const int nvec = r.n / RP_EV;
    const rp_u16* xv = reinterpret_cast<const rp_u16*>(xs);
    const int rep = lane & (RP_HIST_COPIES - 1);
    int T = 0x8000;
    unsigned quota = 0;
    if (r.k > 0) {
      find_digit(hist + H1, sm, 256, (unsigned)r.k);
      const unsigned d1 = sm.digit, above1 = sm.above;
      for (int v = tid; v < nvec; v += THREADS) {
        const rp_u16 b = xv[v];
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) {
          const unsigned key = b[c] & 0x7FFFu;
          if ((key >> 7) == d1) atomicAdd(&hist[H2 + rep * 128 + (key & 127u)], 1u);
        }
      }
      __syncthreads();
      find_digit(hist + H2, sm, 128, (unsigned)r.k - above1);
      T = (int)((d1 << 7) | sm.digit);
      quota = (unsigned)r.k - above1 - sm.above;
    }
    // Everything that is looked at comes into registers together: the wave's own channels (up to
    // 128 of them; wider shares go on in loops) and its stretch.
    const int passes = (own_channels(ew) + AF_WAVE - 1) / AF_WAVE;
    const int g_lo = stretch_begin(ew, wave, r.n), g_hi = stretch_begin(ew, wave + 1, r.n);
    const group_keys* xg = reinterpret_cast<const group_keys*>(xs);
    const unsigned bits0 = xs[max(ew.ch, 0)], bits1 = xs[max(ew.ch1, 0)];
    const group_keys b0 = xg[max(min(g_lo + lane, g_hi - 1), 0)], b1 = xg[max(min(g_lo + AF_WAVE + lane, g_hi - 1), 0)];
    __builtin_amdgcn_sched_barrier(0);
    const bool lists = early_lists(r, ew, j);
    struct Look {
      unsigned long long gt, eq;  // lanes above T / at T
    };
    auto look = [&](int ch, unsigned bits) {
      const int key = ch >= 0 ? (int)(bits & 0x7FFFu) : -1;
      return Look{__ballot(key > T), __ballot(key == T)};
    };
    const Look l0 = look(ew.ch, bits0);
    Look l1 = {0ull, 0ull};
    unsigned open_n = counts(l0.gt & ~ew.taken, l0.eq & ~ew.taken);  // as (above T | at T << 16)
    if (passes > 1) {
      l1 = look(ew.ch1, bits1);
      open_n += counts(l1.gt, l1.eq);
    }
    for (int i = 2; i < passes; ++i) {
      const int ch = early_channel(ew, i, r.n);
      const Look l = look(ch, xs[max(ch, 0)]);
      open_n += counts(l.gt, l.eq);
    }
    // of the stretch: its ties, and where the index list is written also what lies above T
    auto stretch = [&](int g, const group_keys& b) {
      unsigned c = group_at(b, T) << 16;
      if (lists) c += group_above(b, T);
      return g < g_hi ? c : 0u;
    };
    unsigned all_n = stretch(g_lo + lane, b0);
    if (g_lo + AF_WAVE < g_hi) all_n += stretch(g_lo + AF_WAVE + lane, b1);
    for (int g0 = g_lo + 2 * AF_WAVE; g0 < g_hi; g0 += AF_WAVE) all_n += stretch(g0 + lane, xg[min(g0 + lane, g_hi - 1)]);
    all_n = __ballot(all_n != 0) != 0 ? af_wave_sum(all_n) : 0u;
    if (lane == 0) el.tot[wave] = make_uint2(all_n, open_n);
    if (tid == 0) {
      el.last_tie = r.n;
      el.done = 0;
    }
    __syncthreads();
    // every wave scans the (at most 16) wave counts on its own lanes
    static_assert(WAVES <= 16, "one row of lanes");
    const uint2 wt = el.tot[lane % WAVES];
    const unsigned all_s = af_row_incl_scan(wt.x), open_s = af_row_incl_scan(wt.y);
    const unsigned all_pre = (unsigned)__builtin_amdgcn_readlane((int)all_s, wave) - all_n;
    const unsigned open_pre = (unsigned)__builtin_amdgcn_readlane((int)open_s, wave) - open_n;
    const unsigned n_gt = (unsigned)__builtin_amdgcn_readlane((int)open_s, WAVES - 1) & 0xFFFFu;  // ties are listed behind these
    // The first `quota` ties of the whole vector are kept; the one stretch in which they run out
    // looks up the last of them.
    const unsigned eq_pre = all_pre >> 16;
    int last_tie = eq_pre < quota ? r.n : -1;
    if (eq_pre < quota && eq_pre + (all_n >> 16) > quota) {
      unsigned seen = eq_pre;
      for (int g0 = g_lo; g0 < g_hi && last_tie == r.n; g0 += AF_WAVE) {
        const group_keys b = xg[min(g0 + lane, g_hi - 1)];
        const unsigned mine_n = g0 + lane < g_hi ? group_at(b, T) : 0u;
        const unsigned up_to = af_wave_incl_scan(mine_n);
        unsigned rank = seen + up_to - mine_n;
        const unsigned long long found = __ballot(rank < quota && rank + mine_n >= quota);
        if (found != 0) {
          int mine = 0;
#pragma unroll
          for (int c = 0; c < GROUP; ++c)
            if ((int)(b[c / 2] >> (c % 2 * 16) & 0x7FFFu) == T && ++rank == quota) mine = (g0 + lane) * GROUP + c;
          last_tie = __builtin_amdgcn_readlane(mine, (int)__builtin_ctzll(found));
          if (lane == 0) el.last_tie = last_tie;
        }
        seen += (unsigned)__builtin_amdgcn_readlane((int)up_to, AF_WAVE - 1);
      }
    }
    unsigned gt_pos = open_pre & 0xFFFFu, eq_pos = n_gt + (open_pre >> 16), ties = 0;
    auto put = [&](int ch, unsigned bits, const Look& l, unsigned long long free) {
      const unsigned long long keq = l.eq != 0 ? l.eq & __ballot(ch <= last_tie) : 0ull;
      const unsigned entry = ((unsigned)ch << 16) | bits;
      if (((l.gt & free) >> lane) & 1ull) list[gt_pos + lanes_below(l.gt & free)] = entry;
      gt_pos += (unsigned)__popcll(l.gt & free);
      if (keq != 0) {
        if (((keq & free) >> lane) & 1ull) list[eq_pos + lanes_below(keq & free)] = entry;
        eq_pos += (unsigned)__popcll(keq & free);
        ties += (unsigned)__popcll(keq & free);
      }
      return l.gt | keq;
    };
    ew.kept = put(ew.ch, bits0, l0, ~ew.taken);
    if (passes > 1) put(ew.ch1, bits1, l1, ~0ull);
    for (int i = 2; i < passes; ++i) {
      const int ch = early_channel(ew, i, r.n);
      const unsigned bits = xs[max(ch, 0)];
      put(ch, bits, look(ch, bits), ~0ull);
    }
    if (lane == 0) el.ties[wave] = ties;
    if (j == 0 && r.count_out != nullptr && tid == 0) *r.count_out = r.k;
    __syncthreads();
    ew.T = T;
    ew.quota = quota;
    const unsigned all_ties = (unsigned)__builtin_amdgcn_readlane(
        (int)af_row_incl_scan(el.ties[lane % WAVES]), WAVES - 1);
    return (int)(n_gt + all_ties);
  }

  // Workgroup j's part of the ascending index list of the whole vector: pieces j, j + J, ... of the
  // launch's J workgroups, piece p being number p / WAVES of stretch p % WAVES.  Called by every wave
  // when it has streamed its rows: the first one does it, while it would wait for the others (they end
  // 2 us apart; 7B step 2.215 ms, 2.222 with every stretch written by its own wave beside the partial
  // sums or ahead of the rows, 2.203 without the list).
  static __device__ __forceinline__ void early_write_list(const af_row_src& r, const unsigned short* xs,
                                                          Early& el, const EarlyWave& ew, int j, int J) {
    if (!early_lists(r, ew, j)) return;
    int before = 0;
    if ((threadIdx.x & 63) == 0) before = atomicAdd(&el.done, 1);
    if (__builtin_amdgcn_readfirstlane(before) != 0) return;
    const int lane = threadIdx.x & 63, pieces = stretch_pieces(ew) * WAVES;
    const group_keys* xg = reinterpret_cast<const group_keys*>(xs);
    typedef unsigned short half_group __attribute__((ext_vector_type(GROUP / 2)));
    const half_group* xh = reinterpret_cast<const half_group*>(xs);
    const unsigned all_s = af_row_incl_scan(el.tot[lane % WAVES].x);
    for (int p = j; p < pieces; p += J) {
      const int w = p % WAVES, i = p / WAVES;
      const int g_lo = stretch_begin(ew, w, r.n), g_hi = stretch_begin(ew, w + 1, r.n), g_p = g_lo + i * 32;
      if (g_p >= g_hi) continue;
      // the channels in front of the piece, above T | at T << 16
      unsigned front = 0;
      for (int g0 = g_lo; g0 < g_p; g0 += AF_WAVE) {
        const group_keys b = xg[min(g0 + lane, g_p - 1)];
        front += g0 + lane < g_p ? group_above(b, ew.T) + (group_at(b, ew.T) << 16) : 0u;
      }
      if (i > 0) front = af_wave_sum(front);
      const unsigned pre = w > 0 ? (unsigned)__builtin_amdgcn_readlane((int)all_s, w - 1) : 0u;
      front += pre;
      const int last_tie = (pre >> 16) < ew.quota ? el.last_tie : -1;  // the ties of later stretches are not kept
      const int h = g_p * 2 + lane;  // half a group per lane
      const half_group b = xh[min(h, g_hi * 2 - 1)];
      unsigned keep = 0;
#pragma unroll
      for (int c = 0; c < GROUP / 2; ++c) {
        const int key = (int)(b[c] & 0x7FFFu);
        keep |= (unsigned)(h < g_hi * 2 && (key > ew.T || (key == ew.T && h * (GROUP / 2) + c <= last_tie))) << c;
      }
      unsigned pos = (front & 0xFFFFu) + min(front >> 16, ew.quota) + af_wave_incl_scan((unsigned)__popc(keep)) -
                     (unsigned)__popc(keep);
#pragma unroll
      for (int c = 0; c < GROUP / 2; ++c)
        if ((keep >> c) & 1u) r.idx_out[pos++] = h * (GROUP / 2) + c;
    }
  }

  // ---- threshold form, one wave's channels in registers ---------------------------------------
  // A threshold decides a channel without a look at any other, so a wave can decide its own: lane l has
  // channels first + l, first + 64 + l, ... of the split's contiguous range (at most 64 P per wave), and what is
  // kept is a mask per 64 of them.  The rows of the first are requested at once; the others' places in the
  // split's list follow from population counts.  x goes through LDS nowhere.  (threshold_range, for wider
  // shares and the in-kernel router, builds x in LDS and counts, scans and lists it there.)  us before / now:
  //   7B step at 50 % 2056 / 1916, its layers at 30 % 75.7 / 71.4, at 80 % 45.6 / 42.6; 4-bit (the list alone,
  //   no rows early) 52.0 / 50.5 and at 80 % 43.1 / 41.6; 70B-shape layers at 50 % 165.1 / 159.8
  //   4096 -> 12288 behind the norm at 40 % 14.39 / 12.85; 11008 -> 4096 behind SiLU 12.17 / 11.42, at 80 %
  //   7.21 / 6.90; 1000 -> 30000 10.17 / 9.28; 16384 -> 32768 (wide shares, the LDS form) 98.6 / 99.1
  template <int P>
  struct RangeWave {
    int first;                   // the wave's first channel
    unsigned bits[P];            // fp16 bits of x
    unsigned long long kept[P];  // and whether the channel passes, per lane
  };
  template <int P>
  static __device__ __forceinline__ void threshold_wave(const af_row_src& r, Smem& sm, int S, int s, bool store_x,
                                                        RangeWave<P>& rw) {
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int n = r.n, nvec = n / RP_EV;
    const int V = af_ceil_div_small(nvec, S);
    const int c0 = min(s * V, nvec) * RP_EV, c1 = min(min(s * V, nvec) + V, nvec) * RP_EV;
    const int share = (c1 - c0 + WAVES - 1) / WAVES;
    rw.first = c0 + wave * share;
    const int end = min(rw.first + share, c1);
    half_t a[P], b[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int j = min(rw.first + i * AF_WAVE + lane, n - 1);
      a[i] = r.src[j];
      b[i] = r.pro == AF_PRO_NONE ? (half_t)0 : (r.pro == AF_PRO_RMSNORM ? r.gain[j] : r.src[n + j]);
    }
    float scale = 1.f;
    if (r.pro == AF_PRO_RMSNORM) {  // the sum of squares as in threshold_range
      const rp_half* src = reinterpret_cast<const rp_half*>(r.src);
      rp_half zero;
#pragma unroll
      for (int c = 0; c < RP_EV; ++c) zero[c] = (half_t)0;
      float ss = 0.f;
      constexpr int B = 2;
      for (int v0 = tid; v0 < nvec; v0 += B * THREADS) {
        rp_half t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = (v0 + u * THREADS < nvec) ? src[v0 + u * THREADS] : zero;
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
          for (int c = 0; c < RP_EV; ++c) ss += (float)t[u][c] * (float)t[u][c];
      }
      ss = af_wave_sum(ss);
      if (lane == 0) sm.red[wave] = ss;
      __syncthreads();
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += sm.red[w];
      scale = 1.0f / sqrtf(tot / (float)n + r.eps);
    }
    const int T = threshold_key(r.t);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int j = rw.first + i * AF_WAVE + lane;
      half_t x = a[i];
      if (r.pro != AF_PRO_NONE) {
        // The product is rounded to fp32 first, as in the other forms of the front end, which work on vectors:
        // for one element the compiler would take an instruction that rounds it to fp16 at once.
        float v = r.pro == AF_PRO_RMSNORM ? (float)x * scale * (float)b[i] : silu_mul((float)x, (float)b[i]);
        asm("" : "+v"(v));
        x = (half_t)v;
      }
      rw.bits[i] = __builtin_bit_cast(unsigned short, x);
      const unsigned key = rw.bits[i] & 0x7FFFu;
      rw.kept[i] = __ballot(j < end && (int)key > T && key <= 0x7C00u);
      if (store_x && r.x_out != nullptr && j < end) r.x_out[j] = x;
    }
  }
  // The kept channels but the first `taken` of the wave's first 64 into the split's list, ascending; returns
  // their number.
  template <int P>
  static __device__ __forceinline__ int threshold_list(const RangeWave<P>& rw, int taken, Smem& sm, unsigned* list) {
    const int lane = threadIdx.x & 63, wave = wave_id();
    static_assert(WAVES <= 16, "one row of lanes");
    unsigned mine = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) mine += (unsigned)__popcll(rw.kept[i]);
    mine -= (unsigned)taken;
    if (lane == 0) sm.wave_tot[wave] = mine;
    __syncthreads();
    const unsigned scan = af_row_incl_scan(sm.wave_tot[lane % WAVES]);
    int pos = __builtin_amdgcn_readlane((int)scan, wave) - (int)mine - taken;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int rank = (int)lanes_below(rw.kept[i]);
      if (((rw.kept[i] >> lane) & 1ull) && (i > 0 || rank >= taken))
        list[pos + rank] = (unsigned)(rw.first + i * AF_WAVE + lane) << 16 | rw.bits[i];
      pos += __popcll(rw.kept[i]);
    }
    __syncthreads();
    return __builtin_amdgcn_readlane((int)scan, WAVES - 1);
  }

  static __device__ __forceinline__ unsigned counts(unsigned long long gt, unsigned long long eq) {
    return (unsigned)__popcll(gt) + ((unsigned)__popcll(eq) << 16);
  }
  // number of set bits of m below this lane
  static __device__ __forceinline__ unsigned lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
  }

  // Select on xs[0..n) (n % 8 == 0) and keep the entries of split s of S in list[] as
  // (index << 16 | fp16 bits).  Returns the number of entries kept by this workgroup;
  // *nidx_total is the size of the whole index set.  `hist` is RP_SCRATCH_WORDS words of LDS.
  // `list` may be null (only idx_out / count_out are wanted).
  // Every thread owns a contiguous run of RP_EV-element vectors, read from LDS one vector at a
  // time in each pass; the thread order is therefore the index order.
  // `kept_bits`, when given (S == 1 only): bit c of byte v tells whether channel 4 v + c is kept.
  static __device__ __forceinline__ int select_split(const af_row_src& r, const unsigned short* xs,
                                                     unsigned* hist, Smem& sm, unsigned* list,
                                                     int S, int s, bool store_idx, bool store_count,
                                                     int* nidx_total, bool digit1_counted = false,
                                                     unsigned char* kept_bits = nullptr) {
    static_assert(RP_EV == 4, "a byte of kept_bits is one vector");
    const int tid = threadIdx.x, lane = tid & 63;
    const int nvec = r.n / RP_EV;
    const int cv = (nvec + THREADS - 1) / THREADS;  // vectors per thread
    const int v0 = min(tid * cv, nvec), v1 = min(v0 + cv, nvec);
    const rp_u16* xv = reinterpret_cast<const rp_u16*>(xs);
    const int rep = lane & (RP_HIST_COPIES - 1);
    // Both selection rules become integer tests on the magnitude key:
    //   kept outright  <=>  (int)key > T  and  key <= kmax
    //   tie candidates <=>  key == T, kept while the quota lasts (top-k only)
    // top-k: T from the radix select below, kmax = 0x7FFF.  threshold: |x| > t  <=>  key >
    // bits(largest fp16 <= t) for t >= 0 (T = -1 passes everything for t < 0); kmax = 0x7C00
    // keeps NaN out, quota = 0.
    int T = 0x8000;
    unsigned quota = 0, kmax = 0x7FFFu;
    const bool topk = r.sel == AF_SEL_TOPK;
    if (!topk) {
      kmax = 0x7C00u;
      T = threshold_key(r.t);
    }
    if (topk && r.k > 0) {
      if (!digit1_counted) {
        zero_hist(hist);
        __syncthreads();
        for (int v = v0; v < v1; ++v) {
          const rp_u16 b = xv[v];
#pragma unroll
          for (int c = 0; c < RP_EV; ++c)
            atomicAdd(&hist[H1 + rep * 256 + ((b[c] & 0x7FFFu) >> 7)], 1u);
        }
        __syncthreads();
      }
      find_digit(hist + H1, sm, 256, (unsigned)r.k);
      const unsigned d1 = sm.digit, above1 = sm.above;
      for (int v = v0; v < v1; ++v) {
        const rp_u16 b = xv[v];
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) {
          const unsigned key = b[c] & 0x7FFFu;
          if ((key >> 7) == d1) atomicAdd(&hist[H2 + rep * 128 + (key & 127u)], 1u);
        }
      }
      __syncthreads();
      find_digit(hist + H2, sm, 128, (unsigned)r.k - above1);
      T = (int)((d1 << 7) | sm.digit);
      quota = (unsigned)r.k - above1 - sm.above;
    }
    unsigned gt = 0, eq = 0;
    for (int v = v0; v < v1; ++v) {
      const rp_u16 b = xv[v];
#pragma unroll
      for (int c = 0; c < RP_EV; ++c) {
        const unsigned key = b[c] & 0x7FFFu;
        gt += ((int)key > T) & (key <= kmax);
        eq += (int)key == T;
      }
    }
    unsigned tot;
    const unsigned pre = excl_scan(gt | (eq << 16), sm, &tot);
    const int nidx = (int)((tot & 0xFFFFu) + min(tot >> 16, quota));
    *nidx_total = nidx;
    const int R = af_ceil_div_small(nidx, S);
    const int r0 = min(s * R, nidx), r1 = min(r0 + R, nidx);
    unsigned pos = (pre & 0xFFFFu) + min(pre >> 16, quota);
    unsigned eq_seen = pre >> 16;
    // only threads whose run overlaps the split's positions need the second look
    const unsigned my_kept = gt + (min(eq_seen + eq, quota) - min(eq_seen, quota));
    if (((int)(pos + my_kept) > r0 && (int)pos < r1) || kept_bits != nullptr) {
      const bool to_mem = store_idx && r.idx_out != nullptr;
      for (int v = v0; v < v1; ++v) {
        const rp_u16 b = xv[v];
        unsigned bits_v = 0;
#pragma unroll
        for (int c = 0; c < RP_EV; ++c) {
          const unsigned bits = b[c];
          const unsigned key = bits & 0x7FFFu;
          const bool is_eq = (int)key == T;
          const bool keep = (((int)key > T) & (key <= kmax)) | (is_eq & (eq_seen < quota));
          eq_seen += is_eq;
          if (keep & ((int)pos >= r0) & ((int)pos < r1)) {
            const int j = v * RP_EV + c;
            if (list != nullptr) list[pos - r0] = ((unsigned)j << 16) | bits;
            if (to_mem) r.idx_out[pos] = j;
          }
          pos += keep;
          bits_v |= (unsigned)keep << c;
        }
        if (kept_bits != nullptr) kept_bits[v] = (unsigned char)bits_v;
      }
    }
    if (store_count && r.count_out != nullptr && tid == 0) *r.count_out = nidx;
    __syncthreads();
    return r1 - r0;
  }
};
