// Body of the gathered-row sparse GEMV over an input-channel-major fp16 matrix (Section 4,
// operation C), shared by the stand-alone kernel (gemv_f16.hip) and the whole-layer kernel
// (layer.hip).  See gemv_f16.hip for the decomposition.
#pragma once
#include <type_traits>

#include "af_internal.h"
#include "row_prologue.h"

#define GEMV_LIST 2048  // rows given by the caller are staged this many at a time

struct GemvParams {
  const half_t* W;
  af_row_src rows;
  float* partials;
  int* tickets;
  void* y;
  const half_t* residual;
  // The argument block stays within 248 bytes: launches of this kernel were measured 0.3-0.4 us
  // slower once it grew to 280 bytes (the launch itself does not care: near-empty kernels take
  // the same time with 16 bytes or 1 KB of arguments; the cost was in this kernel's start-up).
  // Hence the flag word.
  int out, ld, out_pad;
  int flags;  // GEMV_F_*
  int list_off;   // byte offset of the staged-row list in dynamic LDS (behind x)
  // Output columns come in `slots` of cols_per_slot columns, each covered by tiles_per_slot
  // tiles.  A plain GEMV has one slot.  With w_sel, slot s multiplies by the matrix
  // W + w_sel[s] * w_stride (leading dimension ld), so the experts a router picked on the
  // device are reached without a host round trip.  y_scale (device, one float) scales the
  // product before the residual is added.
  int cols_per_slot, tiles_per_slot;
  union {
    int done_total;    // see `done` below
    int early_cycles;  // launches with early rows (never part of a whole layer): af_dealt_cycles
  };
  const int* w_sel;
  long long w_stride;
  const float* y_scale;
  // Router of a mixture-of-experts block run in this launch's front end (gate|up): every
  // workgroup works out the experts itself from x and uses them for its slot; workgroup
  // (0, 0) publishes them for the launches that follow.  Null router_Wr: no router.
  const half_t* router_Wr;  // [router_E][in]
  int router_E, router_top;
  int32_t* router_experts;
  float* router_weights;
  float* router_logits;
  long long* prof;  // time stamps of this launch (af_profile_set), or null
  // Whole-layer kernel only (null otherwise): the operator is one phase of a kernel whose
  // workgroups go on to the next operator.  Results are then stored through to memory (agent
  // scope) and every workgroup that has finished a tile adds one to *done; the workgroup that
  // brings it to done_total clears *done_prev, the counter of the phase before (all of its
  // waiters have passed it by then).
  // GEMV_F_DONE_PREV: the counter of the phase before is done[-1]; GEMV_F_DONE_LAST: the
  // kernel's last phase, nobody waits on *done and it is cleared as well.
  int* done;
  __host__ __device__ bool f32_out() const { return flags & 1; }
  __host__ __device__ bool use_lds_x() const { return flags & 2; }
  __host__ __device__ bool range_sel() const { return flags & 4; }
};
enum { GEMV_F_F32 = 1, GEMV_F_LDS_X = 2, GEMV_F_RANGE_SEL = 4, GEMV_F_DONE_PREV = 8, GEMV_F_DONE_LAST = 16 };
static_assert(sizeof(GemvParams) <= 248, "keep the kernel argument block small (see above)");

// One finished tile of a whole-layer phase: the results are acknowledged, then counted.
__device__ __forceinline__ void gemv_phase_signal(const GemvParams& p) {
  af_stores_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    const int old = __hip_atomic_fetch_add(p.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == p.done_total - 1) {
      if (p.flags & GEMV_F_DONE_PREV) __hip_atomic_store(p.done - 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (p.flags & GEMV_F_DONE_LAST) __hip_atomic_store(p.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Whole-layer kernel: the finished tile is read by other workgroups of the same launch, so it
// is written through to memory (agent scope).  Two-byte write-through stores would each cost a
// read-modify-write in the memory controller; the tile is therefore put together in LDS
// (`stage`, free at this point) and leaves as 8-byte stores of neighbouring lanes.
// valid % 8 == 0, (y + out0) 8-byte aligned.  v_of(c) yields the sum of column c.
template <int THREADS, typename F>
__device__ __forceinline__ void store_tile_through(const GemvParams& p, int out0, int valid,
                                                   unsigned short* stage, F v_of) {
  const float scale = p.y_scale ? *p.y_scale : 1.0f;
  if (!p.f32_out()) {
    for (int c = threadIdx.x; c < valid; c += THREADS) {
      float v = v_of(c) * scale;
      if (p.residual) v += (float)p.residual[out0 + c];
      stage[c] = __builtin_bit_cast(unsigned short, (half_t)v);
    }
    __syncthreads();
    unsigned long long* dst = reinterpret_cast<unsigned long long*>(reinterpret_cast<half_t*>(p.y) + out0);
    const unsigned long long* src = reinterpret_cast<const unsigned long long*>(stage);
    for (int q = threadIdx.x; q < (valid >> 2); q += THREADS)
      __hip_atomic_store(dst + q, src[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    for (int c = threadIdx.x; c < valid; c += THREADS) {
      float v = v_of(c) * scale;
      if (p.residual) v += (float)p.residual[out0 + c];
      af_store_agent(reinterpret_cast<float*>(p.y) + out0 + c, v);
    }
  }
}

// What store_out adds to column `col`; fetched by its callers before they wait for the sums.
__device__ __forceinline__ float residual_of(const GemvParams& p, int col) {
  return p.residual ? (float)p.residual[col] : 0.f;
}
__device__ __forceinline__ void store_out(const GemvParams& p, int col, float v, float residual) {
  if (p.y_scale) v *= *p.y_scale;
  if (p.residual) v += residual;
  if (!p.f32_out())
    reinterpret_cast<half_t*>(p.y)[col] = (half_t)v;
  else
    reinterpret_cast<float*>(p.y)[col] = v;
}

// Launch shape and parameters of one fp16 GEMV as the host plans it: tiles x S workgroups of
// nw waves, lx lanes across a tile, `lds` bytes of dynamic LDS.
struct GemvPlan {
  GemvParams p;
  int tiles, S, lx, nw;
  int early;  // gemv_early_class (top-k), gemv_range_class (thresholds) or gemv_given_class (rows given) of the launch
  size_t lds;
};
// whole_layer: the operator runs as a phase of the whole-layer kernel (1024-thread workgroups,
// at most one per compute unit).  Defined in gemv_f16.hip.
int af_plan_gemv_f16(af_ctx* ctx, const af_gemv_args& a, bool whole_layer, GemvPlan* plan);

// Virtual launch position of a workgroup: the stand-alone kernel passes blockIdx / gridDim, the
// whole-layer kernel the position it has given the workgroup in the current operator.
struct GemvPos {
  int bx, by, gx, gy;
};
// LDS of one workgroup that the GEMV bodies need besides the dynamic region: declared once by
// the kernel and shared by all the operators it runs.
template <int NW, int TWMAX = 512>
struct GemvLds {
  static constexpr int SCRATCH = RP_SCRATCH_WORDS > NW * TWMAX ? RP_SCRATCH_WORDS : NW * TWMAX;
  __align__(16) unsigned scratch[SCRATCH];  // histograms, later the wave sums
  typename RowPrologue<NW * AF_WAVE>::Smem rp;
  int last;
};
// ... and the kernels that request rows early
template <int NW, int TWMAX, int CAP>
struct GemvEarlyLds : GemvLds<NW, TWMAX> {
  typename RowPrologue<NW * AF_WAVE>::Early early;
  unsigned early_row[NW][CAP];
};

// PHASE: the operator is a phase of the whole-layer kernel (p.done is set).
// PAIR: the launch multiplies two inputs by two device-picked matrices and adds both products to the
// residual stream, the first one rounded to fp16 before the second joins it (the down projections
// of the two experts of a mixture-of-experts block).  Workgroups are (tile, split of input `pair`);
// the tile's last workgroup adds up both.
// EARLY (top-k launches of 1024-thread workgroups): the rows whose selection is obvious are
// requested before the front end runs (RowPrologue, "early rows").  EARLY is the number of
// vectors of the operator's source that one thread holds (1, 4 or 8; 0: no early rows).
// GIVEN (1024-thread launches behind a producer whose rows are known, and their number on the host): the
// rows of a lane's first U steps are requested before x is built.  GIVEN is the number of source vectors
// of a thread, as for EARLY.
// RANGE (threshold launches of 1024-thread workgroups without an index list): passes of 64 channels
// that a wave decides in registers (RowPrologue, threshold_wave), requesting its first rows at once; 0: the
// form that builds x in LDS.
template <int LX, int U, int NW, bool ROUTED, bool PHASE, int EARLY, bool PAIR = false, int RANGE = 0, int GIVEN = 0, typename LDS_T>
__device__ __forceinline__ void gemv_f16_body(const GemvParams& p, const GemvPos vb,
                                              unsigned short* xs, LDS_T& lds, const int pair = 0) {
  constexpr int GEMV_THREADS = NW * AF_WAVE;
  constexpr int GEMV_WAVES = NW;
  constexpr int LY = AF_WAVE / LX;
  constexpr int TW = LX * 8;
  constexpr int STEP = GEMV_WAVES * LY;  // rows taken per workgroup iteration
  typedef RowPrologue<GEMV_THREADS> RP;
  unsigned* s_scratch = lds.scratch;
  typename RP::Smem& s_rp = lds.rp;
  int& s_last = lds.last;
  float(*s_red)[TW] = reinterpret_cast<float(*)[TW]>(s_scratch);
  // staged rows, (index << 16 | fp16 bits of x)
  unsigned* s_list = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(xs) + p.list_off);

  af_prof_begin(p.prof);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lx = lane % LX, ly = lane / LX;
  // one slot (a plain GEMV): no division
  const int slot = p.tiles_per_slot >= vb.gx ? 0 : vb.bx / p.tiles_per_slot;
  const int tile_in = vb.bx - slot * p.tiles_per_slot;   // tile inside the slot
  const int col = tile_in * TW + lx * 8;                       // column inside the slot
  // lanes past the slot's edge read the tile's first column and are dropped at the store
  const int col_ld = col < p.cols_per_slot ? col : tile_in * TW;
  const int S = vb.gy, s = vb.by;
  const af_row_src& r = p.rows;

  // Rows given and their number known on the host: fetch this thread's share of the first
  // staging pass now, so that the index round trip overlaps the construction of x.
  constexpr int PF = GEMV_LIST / GEMV_THREADS;
  int pre[PF];
  const bool prefetched = r.sel == AF_ROWS_GIVEN && r.idx != nullptr && r.nidx_dev == nullptr;
  if (prefetched) {
    const int R = af_ceil_div_small(r.nidx_host, S);
    const int r0 = min(s * R, r.nidx_host), r1 = min(r0 + R, r.nidx_host);
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int i = r0 + tid + u * GEMV_THREADS;
      pre[u] = i < r1 ? r.idx[i] : 0;
    }
  }

  constexpr int RE = 8;  // experts the in-kernel router handles
  constexpr bool routed = ROUTED;
  half8 wr[routed ? RE : 1];
  if constexpr (routed) {  // this thread's router weights do not depend on x: fetch them before x is built
#pragma unroll
    for (int e = 0; e < RE; ++e) {
#pragma unroll
      for (int c = 0; c < 8; ++c) wr[e][c] = (half_t)0;
      if (e < p.router_E && tid < (r.n >> 3))
        wr[e] = *reinterpret_cast<const half8*>(p.router_Wr + (size_t)e * r.n + (size_t)tid * 8);
    }
  }
  if constexpr (!EARLY && !GIVEN) {
    if (p.use_lds_x() && (!p.range_sel() || routed))
      RP::produce(r, xs, s_rp, s == 0, vb.bx, vb.gx, r.sel == AF_SEL_TOPK ? s_scratch : nullptr);
  }
  if constexpr (routed) {
    RP::template router_in_lds<RE>(xs, r.n, s_rp, wr, p.router_E, p.router_top);
    if (vb.bx == 0 && s == 0) {
      if (tid < p.router_top) {
        p.router_experts[tid] = s_rp.experts[tid];
        p.router_weights[tid] = s_rp.weights[tid];
      }
      if (tid < p.router_E) p.router_logits[tid] = s_rp.logit[tid];
    }
  }

  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  const half_t* wcol = p.W + col_ld;
  if (routed)
    wcol += (size_t)s_rp.experts[slot] * (size_t)p.w_stride;
  else if (p.w_sel)
    wcol += (size_t)p.w_sel[slot] * (size_t)p.w_stride;

  // Early rows: UE batches of LY rows per wave, half of them requested behind the loads of the
  // operator's source and before anything waits for the front end, half once x is in LDS.  Four
  // batches are 64 KB per compute unit, about what it can have in flight: with all eight at the
  // head the waves stalled on the requests themselves (q|k|v of the 7B shape: the last wave got
  // its eighth request out 2.3 us after its first) and held up the front end.
  // The narrowest tiles (four rows a batch) get by with four.
  constexpr int UE = EARLY || RANGE ? (LX == 16 ? 4 : 8) : (GIVEN ? U : 1);
  half8 ew[UE];
#pragma unroll
  for (int u = 0; u < UE; ++u)
#pragma unroll
    for (int c = 0; c < 8; ++c) ew[u][c] = (half_t)0;
  int early_n = 0;
  bool early_pending = false;
  typename RP::EarlyWave early;
  typename RP::template RangeWave<RANGE ? RANGE : 1> range;
  // Batches U0 .. U0 + 3 of the early rows.  A missing row is read as the wave's last one, or as row 0:
  // no branch around the loads.
  auto request_of = [&](auto from, auto channel_of) __attribute__((always_inline)) {
    if constexpr (EARLY || RANGE) {
      constexpr int U0 = decltype(from)::value;
      const unsigned* row = lds.early_row[wave];
      unsigned e[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) e[u] = row[max(min((U0 + u) * LY + ly, early_n - 1), 0)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned j = early_n > 0 ? channel_of(e[u]) : 0u;
        ew[U0 + u] = af_load_once(reinterpret_cast<const half8*>(wcol + (size_t)j * p.ld));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if constexpr (RANGE) {
    RP::template threshold_wave<RANGE>(r, s_rp, S, s, vb.bx == 0, range);
    early_n = min(__popcll(range.kept[0]), UE * LY);
    const int rank = (int)RP::lanes_below(range.kept[0]);
    if (((range.kept[0] >> lane) & 1ull) && rank < early_n)
      lds.early_row[wave][rank] = (unsigned)(range.first + lane) << 16 | range.bits[0];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // read by the other lanes of this wave
    __builtin_amdgcn_wave_barrier();
    auto channel_of = [](unsigned e) { return e >> 16; };
    request_of(std::integral_constant<int, 0>{}, channel_of);
    if constexpr (UE == 8) {
      if (early_n > 4 * LY) request_of(std::integral_constant<int, 4>{}, channel_of);
    }
    early_pending = true;
  }
  unsigned given[GIVEN ? UE : 1];  // channels of the rows of the lane's first U steps
  int given_n = 0;                 // rows of the split's first staging pass
  if constexpr (GIVEN) {
    const int R = af_ceil_div_small(r.nidx_host, S), r0 = min(s * R, r.nidx_host);
    given_n = min(min(r0 + R, r.nidx_host) - r0, GEMV_LIST);
#pragma unroll
    for (int u = 0; u < UE; ++u) {  // a missing row is read as the split's last one, or as row 0
      const int i = r0 + max(min(u * STEP + wave * LY + ly, given_n - 1), 0);
      given[u] = given_n == 0 ? 0u : (r.idx ? (unsigned)r.idx[i] : (unsigned)i);
    }
    typename RP::template Raw<GIVEN> raw;
    RP::template load_raw<GIVEN>(r, raw);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): see EARLY
    auto request = [&](int u0, int u1) __attribute__((always_inline)) {
#pragma unroll
      for (int u = u0; u < u1; ++u) {
        const unsigned j = given[u] < (unsigned)r.n ? given[u] : 0u;
        ew[u] = af_load_once(reinterpret_cast<const half8*>(wcol + (size_t)j * p.ld));
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    request(0, UE / 2);
    RP::template produce_raw<GIVEN>(r, raw, xs, s_rp, s == 0, vb.bx, vb.gx, nullptr);
    request(UE / 2, UE);
    early_pending = true;
  }
  if constexpr (EARLY) {
    early = RP::early_block(r.n, S, s, p.early_cycles);
    half_t ea, eb;
    RP::early_load(r, early, &ea, &eb);
    typename RP::template Raw<EARLY> raw;
    RP::template load_raw<EARLY>(r, raw);
    RP::zero_hist(s_scratch);
    if (RP::own_channels(early) > AF_WAVE) early.ch1 = RP::early_channel(early, 1, r.n);
    // The source is in registers before the first row load goes out: otherwise the compiler,
    // which tracks the masked loads above with one counter, would make the front end wait for
    // the rows as well.  (For the same reason the number of vectors is a template argument and
    // not a branch.)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    unsigned* row = lds.early_row[wave];
    early_n = RP::template early_pick<UE * LY>(r, early, row, ea, eb);
    auto request = [&](auto from) __attribute__((always_inline)) {
      request_of(from, [](unsigned e) { return e & 0xFFFFu; });
    };
    request(std::integral_constant<int, 0>{});
    RP::template produce_raw<EARLY>(r, raw, xs, s_rp, s == 0, vb.bx, vb.gx, s_scratch);
    if constexpr (UE == 8) {
      if (early_n > 4 * LY) request(std::integral_constant<int, 4>{});
    }
    early_pending = true;
  }
  // Products of the early rows; called with the first batch of listed rows already requested.  They
  // have sums of their own that join the others at the end: these are the largest of x, and with
  // them at the head of one running sum everything behind was rounded at their size (error against
  // 64 bits, 4096 -> 22016 at 30 %: 1.48e-7 against 1.29e-7 of a sum in index order).
  float early_acc[EARLY ? 8 : 1] = {};
  auto take_early = [&]() __attribute__((always_inline)) {
    if constexpr (GIVEN) {
      early_pending = false;
#pragma unroll
      for (int u = 0; u < UE; ++u) {
        if (u * STEP + wave * LY + ly < given_n) {
          if (given[u] < (unsigned)r.n) {
            const float xv = (float)__builtin_bit_cast(half_t, xs[given[u]]);
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] += (float)ew[u][c] * xv;
          } else if (lx == 0) {  // broken precondition: nothing is added, and the error word
            af_report_bad_index(p.tickets);
          }
        }
      }
    }
    if constexpr (RANGE) {  // the first channels, not the largest: into the running sums
      early_pending = false;
#pragma unroll
      for (int u = 0; u < UE; ++u) {
        const int i = u * LY + ly;
        if (i < early_n) {
          const float xv = (float)__builtin_bit_cast(half_t, (unsigned short)(lds.early_row[wave][i] & 0xFFFFu));
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[c] += (float)ew[u][c] * xv;
        }
      }
    }
    if constexpr (EARLY) {
      early_pending = false;
#pragma unroll
      for (int u = 0; u < UE; ++u) {
        const int i = u * LY + ly;
        const unsigned e = early_n > 0 ? lds.early_row[wave][min(i, early_n - 1)] : 0u;
        if (i < early_n && (early.kept >> (e >> 16)) & 1ull) {
          const float xv = (float)__builtin_bit_cast(half_t, xs[e & 0xFFFFu]);
#pragma unroll
          for (int c = 0; c < 8; ++c) early_acc[c] += (float)ew[u][c] * xv;
        }
      }
    }
  };

  // One pass over `cnt` staged rows of s_list.
  auto stream = [&](int cnt, int from = 0) {
    int i = from + wave * LY + ly;
    for (; i + (U - 1) * STEP < cnt; i += U * STEP) {
      half8 w[U];
      unsigned e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        e[u] = s_list[i + u * STEP];
        w[u] = af_load_once(reinterpret_cast<const half8*>(wcol + (size_t)(e[u] >> 16) * p.ld));
      }
      // All U loads are issued before the first product: without this fence the instruction
      // scheduler has, in some instantiations, paired every load with its own wait (one row in
      // flight instead of U), which halves the streaming rate.
      __builtin_amdgcn_sched_barrier(0);
      if ((EARLY || RANGE || GIVEN) && early_pending) take_early();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float xv = (float)__builtin_bit_cast(half_t, (unsigned short)(e[u] & 0xFFFFu));
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += (float)w[u][c] * xv;
      }
    }
    // Ragged end: one more batch of the same depth with the missing rows masked off, so its
    // loads are all in flight together (a row-at-a-time loop would pay one memory round trip
    // per row, up to U - 1 of them in a row).
    if (i < cnt) {
      half8 w[U];
      unsigned e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = i + u * STEP < cnt;
        e[u] = ok ? s_list[i + u * STEP] : 0u;
        if (ok) {
          w[u] = af_load_once(reinterpret_cast<const half8*>(wcol + (size_t)(e[u] >> 16) * p.ld));
        } else {
#pragma unroll
          for (int c = 0; c < 8; ++c) w[u][c] = (half_t)0;
        }
      }
      if ((EARLY || RANGE || GIVEN) && early_pending) take_early();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float xv = (float)__builtin_bit_cast(half_t, (unsigned short)(e[u] & 0xFFFFu));
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += (float)w[u][c] * xv;
      }
    }
  };

  if constexpr (EARLY) {
    stream(RP::select_dealt(r, xs, s_scratch, s_rp, lds.early, early, s_list, s * vb.gx + vb.bx));
    if (early_pending) take_early();
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += early_acc[c];
    RP::early_write_list(r, xs, lds.early, early, s * vb.gx + vb.bx, vb.gx * S);
  } else if constexpr (RANGE) {
    stream(RP::template threshold_list<RANGE>(range, early_n, s_rp, s_list));
    if (early_pending) take_early();
  } else if (p.range_sel()) {
    stream(routed ? RP::threshold_range_of_full(r, xs, s_rp, s_list, S, s)
                  : RP::threshold_range(r, xs, s_rp, s_list, S, s, vb.bx == 0));
  } else if (r.sel != AF_ROWS_GIVEN) {
    int nidx_total;
    const int cnt = RP::select_split(r, xs, s_scratch, s_rp, s_list, S, s, vb.bx == 0,
                                     vb.bx == 0 && s == 0, &nidx_total, p.use_lds_x());
    stream(cnt);
  } else {
    int nidx = r.nidx_host;
    if (r.nidx_dev) nidx = min(*r.nidx_dev, nidx);
    const int R = af_ceil_div_small(nidx, S);
    const int r0 = min(s * R, nidx), r1 = min(r0 + R, nidx);
    const unsigned short* xg = reinterpret_cast<const unsigned short*>(r.src);
    for (int base = r0; base < r1; base += GEMV_LIST) {
      const int cnt = min(GEMV_LIST, r1 - base);
      const int from = GIVEN && base == r0 ? U * STEP : 0;  // the rows in front have been requested
      __syncthreads();
      if (prefetched && base == r0) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          const int i = tid + u * GEMV_THREADS;
          if (i < cnt && i >= from) {
            const int j = pre[u];
            if ((unsigned)j < (unsigned)r.n) {
              const unsigned bits = p.use_lds_x() ? xs[j] : xg[j];
              s_list[i] = ((unsigned)j << 16) | bits;
            } else {  // broken precondition: row 0 times zero, and the error word
              s_list[i] = 0u;
              af_report_bad_index(p.tickets);
            }
          }
        }
      } else {
        for (int i = from + tid; i < cnt; i += GEMV_THREADS) {
          const int j = r.idx ? r.idx[base + i] : base + i;
          if ((unsigned)j < (unsigned)r.n) {
            const unsigned bits = p.use_lds_x() ? xs[j] : xg[j];
            s_list[i] = ((unsigned)j << 16) | bits;
          } else {
            s_list[i] = 0u;
            af_report_bad_index(p.tickets);
          }
        }
      }
      __syncthreads();
      stream(cnt, from);
    }
    if (GIVEN && early_pending) take_early();
  }
  __syncthreads();  // s_scratch changes its role: histograms -> wave sums

  // lane groups -> one row of sums per wave
  const int first = af_sum_lane_groups<LX>(acc);
#pragma unroll
  for (int c = 0; c < LX / 8; ++c) s_red[wave][lx * 8 + first + c] = acc[c];
  __syncthreads();

  const int tile0 = vb.bx * TW;                      // in the padded column space
  const int out0 = slot * p.cols_per_slot + tile_in * TW;  // first output column of the tile
  const int valid = min(TW, p.cols_per_slot - tile_in * TW);
  if (S == 1 && !PAIR) {
    if constexpr (PHASE) {
      store_tile_through<GEMV_THREADS>(p, out0, valid, xs, [&](int c) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < GEMV_WAVES; ++w) v += s_red[w][c];
        return v;
      });
      gemv_phase_signal(p);
    } else {
      for (int c = tid; c < valid; c += GEMV_THREADS) {
        const float res = residual_of(p, out0 + c);
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < GEMV_WAVES; ++w) v += s_red[w][c];
        store_out(p, out0 + c, v, res);
      }
    }
    af_prof_end(p.prof);
    return;
  }

  float* mine = p.partials + (size_t)s * p.out_pad;
  for (int c = tid; c < TW; c += GEMV_THREADS) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < GEMV_WAVES; ++w) v += s_red[w][c];
    af_store_agent(mine + tile0 + c, v);  // out_pad covers whole tiles
  }
  af_stores_done();
  __syncthreads();
  if (tid == 0) {
    int old = af_ticket_take(&p.tickets[af_ticket_of(vb.bx)]);
    s_last = (old == (PAIR ? 2 * S : S) - 1);
  }
  __syncthreads();
  if (!s_last) {
    af_prof_end(p.prof);
    return;
  }
  if constexpr (PAIR) {
    const size_t n = (size_t)S * p.out_pad;
    const float* first = p.partials - pair * n + tile0;
    const float* scale = p.y_scale - pair;
    for (int c = tid; c < valid; c += GEMV_THREADS) {
      const float res = residual_of(p, out0 + c);
      const float a = af_sum_partials(first + c, p.out_pad, S), b = af_sum_partials(first + n + c, p.out_pad, S);
      const half_t h = (half_t)(a * scale[0] + res);
      reinterpret_cast<half_t*>(p.y)[out0 + c] = (half_t)(b * scale[1] + (float)h);
    }
  } else if constexpr (PHASE) {
    store_tile_through<GEMV_THREADS>(p, out0, valid, xs, [&](int c) {
      return af_sum_partials(p.partials + tile0 + c, p.out_pad, S);
    });
  } else {
    for (int c = tid; c < valid; c += GEMV_THREADS) {
      const float res = residual_of(p, out0 + c);
      store_out(p, out0 + c, af_sum_partials(p.partials + tile0 + c, p.out_pad, S), res);
    }
  }
  if (tid == 0) af_ticket_reset(&p.tickets[af_ticket_of(vb.bx)]);  // ready for the next launch
  if constexpr (PHASE) gemv_phase_signal(p);
  af_prof_end(p.prof);
}

// GEMV_MODE(pro, kind): the producer and the way the rows are found as compile-time constants
// (kind: 0 rows given, 1 top-k, 2 threshold with an index list, 3 threshold per channel range).
// A kernel instantiated for one mode carries none of the other modes' code and branches, which
// measured 0.4-0.5 us per launch (q|k|v 16.7 -> 16.3 us, gate|up 23.5 -> 23.0 us); mode -1 is
// the generic kernel that reads both from its arguments.  Top-k modes carry the width class of
// their input (gemv_early_class) in bits 4 and 5, threshold modes per channel range the class of a wave's share.
#define GEMV_MODE(pro, kind) ((pro) | ((kind) << 2))
template <int MODE>
__device__ __forceinline__ GemvParams gemv_fix_mode(const GemvParams& p) {
  GemvParams q = p;
  if constexpr (MODE >= 0) {
    constexpr int pro = MODE & 3, kind = (MODE >> 2) & 3;
    q.rows.pro = pro;
    q.rows.sel = kind == 0 ? (int)AF_ROWS_GIVEN : (kind == 1 ? (int)AF_SEL_TOPK : (int)AF_SEL_THRESHOLD);
    q.flags = (p.flags & ~(GEMV_F_LDS_X | GEMV_F_RANGE_SEL)) |
              ((pro != AF_PRO_NONE || kind != 0) ? GEMV_F_LDS_X : 0) | (kind == 3 ? GEMV_F_RANGE_SEL : 0);
  }
  return q;
}
// The mode the generic kernel would find in these arguments.
static inline int gemv_mode_of(const GemvParams& p) {
  const int kind = p.rows.sel == AF_ROWS_GIVEN ? 0 : (p.rows.sel == AF_SEL_TOPK ? 1 : (p.range_sel() ? 3 : 2));
  return GEMV_MODE(p.rows.pro, kind);
}

// Do the launches of this instantiation request rows early?  (A router's launch does not know its
// matrix before its front end has run.)
constexpr int gemv_early(int mode, int nw, bool routed) {
  constexpr int vectors[4] = {1, 4, 8, 0};
  return mode >= 0 && ((mode >> 2) & 3) == 1 && nw == 16 && !routed ? vectors[mode >> 4] : 0;
}
// Passes of the threshold launches that decide their channels in registers: shares of up to 64, 128
// and 256 channels per wave.  Wider ones (class GEMV_EARLY_NONE) build x in LDS.
constexpr int gemv_range(int mode, int nw, bool routed) {
  constexpr int passes[4] = {1, 2, 4, 0};
  return mode >= 0 && ((mode >> 2) & 3) == 3 && nw == 16 && !routed ? passes[mode >> 4] : 0;
}
// Source vectors of a thread in the launches that request given rows ahead of x.
constexpr int gemv_given(int mode, int nw, bool routed) {
  constexpr int vectors[4] = {1, 4, 8, 0};
  return mode >= 0 && ((mode >> 2) & 3) == 0 && (mode & 3) != AF_PRO_NONE && nw == 16 && !routed ? vectors[mode >> 4] : 0;
}
enum { GEMV_EARLY_NONE = 3 };
// Rows that a wave of a launch with LX lanes across a tile can take.
constexpr int gemv_early_cap(int lx) { return (lx == 16 ? 4 : 8) * AF_WAVE / lx; }
// Which of them: inputs of up to 4096, 16384 and AF_MAX_N channels.
static inline int gemv_width_class(int n) { return n <= RP_EV * 1024 ? 0 : (n <= 4 * RP_EV * 1024 ? 1 : 2); }
// ... and whether at all: not where early rows cost more than they hide.  The look for the rows is
// 0.5-1 us of front end.  Up to 4096 channels it pays from a stream of 100, 132 (up to 3584 channels 120) and 150 KB
// a workgroup on, by the width of the tile (us without / with, index list written; 50 % unless stated):
//   128 columns: 4096 -> 4096 (85 KB) 10.45 / 10.67         2048 -> 6144 at 30 % (90 KB) 10.10 / 10.32
//                4096 -> 6144 (102 KB) 11.57 / 11.40        4096 -> 6144 at 30 % (143 KB) 13.62 / 12.70
//   256 columns: 2048 -> 12288 (102 KB) 10.71 / 11.23       4096 -> 8192 (128 KB) 12.44 / 12.96, behind SiLU 12.18 / 12.45
//                3072 -> 8192 at 30 % (134 KB) 12.38 / 11.86    2048 -> 12288 at 30 % (143 KB) 12.67 / 11.96
//                2200 -> 10128 at 30 % (128 KB) 13.20 / 11.79   3056 -> 10128 (127 KB) 13.19 / 12.36
//                3496 -> 9208 (124 KB) 13.21 / 12.94            2800 -> 8136 at 30 % (122 KB) 12.79 / 12.15
//                2800 -> 10128 (116 KB) 12.15 / 11.94, behind SiLU 11.88 / 12.16    4000 -> 8136 (125 KB) 13.17 / 13.71
//                4096 -> 6400 at 30 % (143 KB) 13.61 / 12.46    3072 -> 12288 (154 KB) 13.22 / 12.34
//   512 columns: 4096 -> 14336 at 80 % (136 KB) 11.38 / 11.85   3072 -> 14336 at 70 % (153 KB) 12.00 / 11.67
//                3072 -> 22016 at 80 % (153 KB) 11.98 / 12.03   4096 -> 22016 (409 KB) 21.28 / 19.69
// Wider inputs have a longer front end to hide behind: from 48 KB on, or from 72 KB where few
// channels are kept and so less than 48 KB can be taken early,
//   10672 -> 920 (55 KB) 12.82 / 12.36      12632 -> 616 at 30 % (58 KB) 15.33 / 14.36    14456 -> 1536 at 70 % (67 KB) 13.83 / 12.89
//   5120 -> 4096 at 80 % (42 KB) 9.75 / 9.69    8192 -> 4096 at 80 % (68 KB) 10.91 / 11.16    11008 -> 4096 at 80 % (91 KB) 13.21 / 13.05
// but there the look also grows with the channels that a wave owns, of which it takes from the first
// 64 only, so what is taken has to be worth it: 1 KB for the workgroup to 6 of a wave's channels, to
// 3.5 behind the SiLU producer (channels : KB; * SiLU):
//   17856 -> 3408 at 80 % (124 : 36) 18.91 / 16.87    28304 -> 3152 at 80 % (177 : 36) 23.50 / 21.87
//   19888 -> 6472 at 90 % (138 : 32) 18.05 / 17.29    28672 -> 8192 at 90 % (224 : 32) 22.43 / 21.66
//   *11008 -> 6144 (137 : 64) 21.42 / 20.10           *28672 -> 4096 (224 : 64) 34.30 / 34.06
//   *28672 -> 6144 (358 : 64) 44.74 / 45.77           *28672 -> 10240 at 80 % (299 : 72) 32.53 / 31.92
static inline int gemv_early_class(int pro, int n, int k, int S, int lx) {
  const long long row = lx * 16, bytes = k / S * row;
  const int share = (int)((long long)k * 48 / n), cap = gemv_early_cap(lx);
  const long long early = (share < cap ? share : cap) * 16 * row;  // taken by the workgroup's waves
  const int line = lx == 16 ? 100 : (lx == 32 ? (n <= 3584 ? 120 : 132) : 150);
  const bool pays = n <= 4096 ? bytes >= line * 1024
                              : bytes >= (early >= 48 * 1024 ? 48 : 72) * 1024 &&
                                    n / S / 16 * 2 * 1024 <= (pro == AF_PRO_SILUMUL ? 7 : 12) * early;
  return pays ? gemv_width_class(n) : (int)GEMV_EARLY_NONE;
}
// Given rows ahead of x.  A list has to be in registers first, which the plain form fetches in the shadow of
// the norm; that costs short streams more than the rows' head start gives (us per layer, three of four
// layers reusing two of four lists, plain / ahead; KB of rows per workgroup in q|k|v and gate|up):
//   4096 channels, tiles of 256 and 512 columns: 102, 205 KB 51.6 / 52.1    205, 409 KB 67.9 / 67.2    286, 573 KB 78.9 / 78.1
//   3072, 128 and 512: 90, 268 KB 57.3 / 57.4    2048, 128 and 256: 45, 179 KB 45.6 / 46.3    512, 128: 4, 8 KB 34.4 / 36.1
//   5120: 170, 256 KB 61.1 / 60.4    320, 640 KB 86.2 / 84.8      8192: 341, 2048 KB 168.6 / 167.4
// All rows (no list): 2048 -> 8192 (128 KB) 11.74 / 11.46 but 2048 -> 7936 (127 KB) 10.59 / 10.77, 3072 -> 6400 (154 KB)
// 12.16 / 11.96, 2048 -> 10240 (170 KB) 12.02 / 11.71; 512 columns: 1024 -> 16384 (170 KB) 10.71 / 10.69, 2048 -> 14336
// (227 KB) 14.36 / 13.73; 128 columns: 4096 -> 4096 (128 KB) 11.69 / 11.66, behind SiLU 11.27 / 11.52; 256, behind SiLU:
// 4096 -> 6400 (204 KB) 13.47 / 13.38.  Behind SiLU, beyond 24576 channels, both halves of the source fill the registers:
// 24000 -> 4096 36.67 / 36.45, 25000 -> 4096 38.20 / 38.32, 28672 -> 5120 52.9 / 53.6.
static inline int gemv_given_class(int pro, bool dense, int n, int nidx, int S, int lx) {
  const long long bytes = (long long)(nidx / S) * lx * 16;
  if (pro == AF_PRO_SILUMUL && n > 24576) return GEMV_EARLY_NONE;
  const int narrow = lx == 16 || (lx == 64 && !dense) ? 320 : (lx == 32 && dense && pro == AF_PRO_RMSNORM ? 150 : 200);
  return bytes >= (n <= RP_EV * 1024 ? narrow : 160) * 1024 ? gemv_width_class(n) : (int)GEMV_EARLY_NONE;
}
static_assert(8 * RP_EV * 1024 >= AF_MAX_N, "the widest input fits the largest class");

// ROUTED: the instantiation that runs a mixture-of-experts router in its front end (kept apart
// so that the plain launches do not carry its registers).
template <int LX, int U, int NW, bool ROUTED, int MODE = -1>
__global__ __launch_bounds__(NW * AF_WAVE) void gemv_f16_kernel(GemvParams p) {
  extern __shared__ __align__(16) unsigned short xs[];  // the operator input, when built here
  constexpr int EARLY = gemv_early(MODE, NW, ROUTED), RANGE = gemv_range(MODE, NW, ROUTED);
  constexpr int GIVEN = gemv_given(MODE, NW, ROUTED);
  __shared__ std::conditional_t<(EARLY + RANGE > 0), GemvEarlyLds<NW, LX * 8, gemv_early_cap(LX)>, GemvLds<NW, LX * 8>> lds;
  const GemvPos vb = {(int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x, (int)gridDim.y};
  if constexpr (MODE >= 0) {
    const GemvParams q = gemv_fix_mode<MODE>(p);
    gemv_f16_body<LX, U, NW, ROUTED, false, EARLY, false, RANGE, GIVEN>(q, vb, xs, lds);
  } else {
    gemv_f16_body<LX, U, NW, ROUTED, false, EARLY>(p, vb, xs, lds);
  }
}

// The second input of a launch with two (see PAIR); everything else is in `p`, whose partials and
// matrix choices lie in front of the second input's.
struct GemvPairParams {
  GemvParams p;
  const half_t* src;
  half_t* x_out;
  int32_t* idx_out;
  int32_t* count_out;
};
template <int LX, int U, int MODE>
__global__ __launch_bounds__(16 * AF_WAVE) void gemv_f16_pair_kernel(GemvPairParams d) {
  constexpr int NW = 16;
  extern __shared__ __align__(16) unsigned short xs[];
  constexpr int EARLY = gemv_early(MODE, NW, false), RANGE = gemv_range(MODE, NW, false);
  __shared__ std::conditional_t<(EARLY + RANGE > 0), GemvEarlyLds<NW, LX * 8, gemv_early_cap(LX)>, GemvLds<NW, LX * 8>> lds;
  const int S = (int)gridDim.y >> 1, pair = (int)blockIdx.y >= S;
  const GemvPos vb = {(int)blockIdx.x, (int)blockIdx.y - pair * S, (int)gridDim.x, S};
  GemvParams q = gemv_fix_mode<MODE>(d.p);
  if (pair) {
    q.rows.src = d.src;
    q.rows.x_out = d.x_out;
    q.rows.idx_out = d.idx_out;
    q.rows.count_out = d.count_out;
    q.w_sel += 1;
    q.y_scale += 1;
    q.partials += (size_t)S * q.out_pad;
  }
  gemv_f16_body<LX, U, NW, false, false, EARLY, true, RANGE>(q, vb, xs, lds, pair);
}
