// Host side of the C ABI declared in include/river.h: workspace layout, launches,
// bookkeeping.  All arithmetic of the decode step lives in river_device.h.
#include "river.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "river_device.h"
#include "river_prefill.h"

using namespace river;

// ------------------------------------------------------------------ kernels
//
// All kernels take the device descriptor by pointer (it lives in the workspace and is read
// with scalar loads) and the per-step arguments by value.

// One-kernel-per-phase mode.  The exit state travels between the kernels of a token in
// DevState: the QKV kernel of block l derives it (every workgroup identically), workgroup 0
// stores it in slot l & 1, the other kernels of the block read that slot.
__device__ __forceinline__ Ctl load_ctl(DevRef D, int l) {
  Ctl c;
  c.river = D.st->slot_river[l & 1] != 0;
  c.exit_pos = D.st->slot_exit[l & 1];
  return c;
}

template <int DT, int V>
__global__ __launch_bounds__(kBlock) void k_qkv(const Dev *Dp, StepArgs A, int l) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  Ctl ctl;
  if (l == 0) {
    ctl = ctl_init(D, A);
    record_init(D, A);
  } else {
    ctl = load_ctl(D, l - 1);
  }
  Pre<DT, V> pre;
  const bool guess = l == 0 ? ctl.river : guess_river_after(A, ctl, l);
  prefetch_phase<DT>(D, l, PH_QKV, guess, pre);
  phase_qkv<DT>(D, A, l, guess, ctl, lds, pre);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    D.st->slot_river[l & 1] = ctl.river;
    D.st->slot_exit[l & 1] = ctl.exit_pos;
  }
}
// F16: the 16-bit KV cache of a bf16 model holds IEEE half values (a kernel of its own per
// cache type, so that no kernel carries both conversions)
template <int DT, bool F16>
__global__ __launch_bounds__(kBlock) void k_attn(const Dev *Dp, StepArgs A, int l) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  phase_attn<DT, F16, 0>(D, A, l, load_ctl(D, l), lds, [] {}, [] {});
}
template <int DT, int V>
__global__ __launch_bounds__(kBlock) void k_oproj(const Dev *Dp, StepArgs A, int l) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  const Ctl ctl = load_ctl(D, l);
  Pre<DT, V> pre;
  prefetch_phase<DT>(D, l, PH_O, ctl.river, pre);
  phase_oproj<DT>(D, A, l, ctl.river, lds, pre);
}
template <int DT, int V>
__global__ __launch_bounds__(kBlock) void k_gateup(const Dev *Dp, StepArgs A, int l) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  const Ctl ctl = load_ctl(D, l);
  Pre<DT, V> pre;
  prefetch_phase<DT>(D, l, PH_GU, ctl.river, pre);
  phase_gateup<DT>(D, A, l, ctl.river, lds, pre);
}
template <int DT, int V>
__global__ __launch_bounds__(kBlock) void k_down(const Dev *Dp, StepArgs A, int l) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  const Ctl ctl = load_ctl(D, l);
  Pre<DT, V> pre;
  prefetch_phase<DT>(D, l, PH_DOWN, ctl.river, pre);
  phase_down<DT>(D, A, l, ctl.river, lds, pre);
}
template <int DT>
__global__ __launch_bounds__(kBlock) void k_head(const Dev *Dp, StepArgs A) {
  constexpr int V = 0;
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  const Ctl ctl = load_ctl(D, D.L - 1);
  Pre<DT, V> pre;
  prefetch_head<DT>(D, pre);
  phase_head<DT>(D, A, ctl, lds, pre);
}

// The end of a prefill on the matrix cores (bf16): h(L) of the last position completed from the sums of the last GEMM, final
// norm, LM head, token, and the state a new sequence starts from.  One launch for what were five (reset, last sums, head, copy of the
// logits, token of the batched sequence), 3 to 5 us each with nothing to do: four 8B blocks, 77 tokens 561 -> 547 us, four 1B
// blocks, 255 tokens 407 -> 400 (there the last sums still have their launch, 5 us: see launch_prefill_head).  Bound by the stream of the head behind 10 us of launch, staging and hand-over (30 us for 131 MB).
// n_part >= 0: h(L) = h_row + n_part planes part + j * stride, added in order, d_model of at most kPfHeadCols columns; < 0: it lies in
// Dev::hidden already.  The weight prefetch is issued in front of it, as in a decode step.
constexpr int kPfHeadCols = kNormRuns * kBlock * 8, kPfHeadPlanes = 8;
__global__ __launch_bounds__(kBlock) void k_pf_head(const Dev *Dp, const float *h_row, const float *part, size_t stride, int n_part,
                                                    float *out_logits, int *host_row, int *batch_token) {
  constexpr int V = 0;
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  float *const h = D.hidden + (size_t)D.L * D.d;
  Pre<1, V> pre;
  prefetch_head<1>(D, pre);
  NormIn<1> in;
  float ss[1] = {0.f};
  if (n_part >= 0) {
#pragma unroll
    for (int k = 0; k < kNormRuns; ++k) {
      const int i = (k * kBlock + in.tid) * 8;
      if (i >= D.d) continue;
      pf::Run8 x = pf::ld_run8(h_row + i);
#pragma unroll
      for (int e = 0; e < 8; ++e) in.g[k][e] = Store<1>::ld(D.final_norm, i + e);
      pf::add_planes(part + i, stride, n_part, [&](const float *p, bool ok) {
        const pf::Run8 q = pf::ld_run8(p);
#pragma unroll
        for (int e = 0; e < 8; ++e) x.v[e] += ok ? q.v[e] : 0.f;
      });
      if (blockIdx.x == 0) pf::st_run8(h + i, x);
      in.v[k][0] = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
      in.v[k][1] = make_float4(x.v[4], x.v[5], x.v[6], x.v[7]);
      float q2[2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        q2[q] = (in.v[k][q].x * in.v[k][q].x + in.v[k][q].y * in.v[k][q].y) + (in.v[k][q].z * in.v[k][q].z + in.v[k][q].w * in.v[k][q].w);
      ss[0] += q2[0] + q2[1];
    }
  } else {
    ss[0] = in.fetch<true>(h, D.final_norm, D.d);
  }
  block_sum_k<1, true>(ss, lds_red(D, lds));
  in.put<true>(h, D.final_norm, D.d, 1.0f / sqrtf(ss[0] / (float)D.d + D.eps), run_log2<1, V>(false, D.d), lds, lds_half(D, lds));
  lds_barrier();
  // the rows and the token, as in phase_head (a function that both share costs the step kernel 0.8 % at the 1B shape)
  float *const red = lds_red(D, lds);
  const int lane = pre.lane;
  float best = -INFINITY;
  int besti = 0x7fffffff;
  auto rows_of = [&](int t, Rows<kRD> &rw) { head_rows<1>(D, t, rw); };
  auto epi = [&](int t, float (&acc)[kRD]) {
#pragma unroll
    for (int r = 0; r < kRD; ++r) {
      const int row = t * kRD + r;
      if (row < D.vocab) {
        if (lane == 0) {
          D.logits[row] = acc[r];
          if (out_logits) out_logits[row] = acc[r];
        }
        argmax_take(best, besti, acc[r], row);
      }
    }
  };
  stream_tasks<Dense<1, kRD, kUD>, 1, kRD>((D.vocab + kRD - 1) / kRD, D.d, D.group, lds, pre, rows_of, epi);
  block_argmax(best, besti, red);
  if (threadIdx.x == 0) {
    pub(D.amax_val + blockIdx.x, best);
    pub((float *)D.amax_idx + blockIdx.x, __int_as_float(besti));
  }
  if (!last_arriver(&D.st->head_cnt, gridDim.x, lds_flag(D, lds))) return;
  float top = -INFINITY;
  int token = 0x7fffffff;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += blockDim.x)
    argmax_take(top, token, sub(D.amax_val + i), __float_as_int(sub((const float *)D.amax_idx + i)));
  block_argmax(top, token, red);
  if (threadIdx.x < kBarCounters) *bar_counter(D.bar, threadIdx.x) = 0;
  if (threadIdx.x == 0) {
    *bar_error(D.bar) = 0;
    *D.st = DevState{};
    D.st->cur_token = token;
    if (batch_token) *batch_token = token;
    if (host_row) { host_store(host_row, token); host_store(host_row + 1, 0); }
  }
}

#ifdef RIVER_TRACE
// diagnostics build: every workgroup stamps the 100 MHz wall clock when it arrives at and
// when it is released from each device-wide barrier of the last launch
#define TRACE_ARRIVE() if (threadIdx.x == 0) D.trace[((k - A.bar_base - 1) * 2 + 0) * gridDim.x + blockIdx.x] = wall_clock64()
#define TRACE_RELEASE() if (threadIdx.x == 0) D.trace[((k - A.bar_base - 1) * 2 + 1) * gridDim.x + blockIdx.x] = wall_clock64()
#else
#define TRACE_ARRIVE()
#define TRACE_RELEASE()
#endif

// Persistent mode: one launch per token.  The phase functions are inlined into one loop body
// (as separate functions every call saved and restored ~100 registers per lane).  The
// device-wide barrier that PRECEDES a phase is executed inside that phase's function, and
// the phase's first weight loads are issued between arriving at and waiting on it, so they
// are in flight while the workgroups synchronise.  k is the index of that barrier (0: none,
// first phase of the launch).
#ifndef RIVER_PSTEP_INLINE
#define RIVER_PSTEP_INLINE __forceinline__
#endif
__device__ __forceinline__ int pack_ctl(const Ctl &c) { return (c.exit_pos << 1) | (c.river ? 1 : 0); }
__device__ __forceinline__ Ctl unpack_ctl(int v) { Ctl c; c.river = v & 1; c.exit_pos = v >> 1; return c; }

template <int DT, int V>
__device__ RIVER_PSTEP_INLINE int pstep_qkv(const Dev *Dp, StepArgs A, int l, int ctl_packed,
                                      unsigned long long k, float *lds) {
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  Ctl ctl = unpack_ctl(ctl_packed);
  Pre<DT, V> pre;
  // block l (1-based) has just run: what will block l + 1 run as, as far as known now
  const bool guess = (l == 0) ? ctl.river : guess_river_after(A, ctl, l);
  if (l > 0) { barrier_arrive(D.bar, k); TRACE_ARRIVE(); }
  prefetch_phase<DT>(D, l, PH_QKV, guess, pre);
  if (l > 0) { barrier_wait(D.bar, k, D.spin_limit, D.bar_vector_poll); TRACE_RELEASE(); }
  phase_qkv<DT>(D, A, l, guess, ctl, lds, pre);
  return pack_ctl(ctl);
}
template <int DT, bool F16, int HD>
__device__ RIVER_PSTEP_INLINE void pstep_attn(const Dev *Dp, StepArgs A, int l, int ctl_packed, unsigned long long k,
                                        float *lds) {
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  phase_attn<DT, F16, HD>(D, A, l, unpack_ctl(ctl_packed), lds, [&] { barrier_arrive(D.bar, k); TRACE_ARRIVE(); },
                 [&] { barrier_wait(D.bar, k, D.spin_limit, D.bar_vector_poll); TRACE_RELEASE(); });
}
template <int DT, int PH, int V>
__device__ RIVER_PSTEP_INLINE void pstep_gemv(const Dev *Dp, StepArgs A, int l, bool river, unsigned long long k,
                                        float *lds) {
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  Pre<DT, V> pre;
  barrier_arrive(D.bar, k); TRACE_ARRIVE();
  prefetch_phase<DT>(D, l, PH, river, pre);
  barrier_wait(D.bar, k, D.spin_limit, D.bar_vector_poll); TRACE_RELEASE();
  if (PH == PH_O) phase_oproj<DT>(D, A, l, river, lds, pre);
  else if (PH == PH_GU) phase_gateup<DT>(D, A, l, river, lds, pre);
  else phase_down<DT>(D, A, l, river, lds, pre);
}
template <int DT, int V>
__device__ RIVER_PSTEP_INLINE void pstep_head(const Dev *Dp, StepArgs A, int ctl_packed, unsigned long long k,
                                        float *lds) {
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  const Ctl ctl = unpack_ctl(ctl_packed);
  Pre<DT, V> pre;
  barrier_arrive(D.bar, k); TRACE_ARRIVE();
  prefetch_head<DT>(D, pre);
  barrier_wait(D.bar, k, D.spin_limit, D.bar_vector_poll); TRACE_RELEASE();
  phase_head<DT>(D, A, ctl, lds, pre);
}

// The number of barriers (5 L - 1, one more with the head) is the same for every workgroup
// whatever the exit state.
template <int DT, bool F16, int V, int HD>
__global__ __launch_bounds__(kBlock) void k_step_persistent(const Dev *Dp, StepArgs A) {
  extern __shared__ float lds[];
  DevRef D = *RIVER_CONSTANT(Dev, Dp);
  unsigned long long k = A.bar_base;
  const int L = D.L;
  record_init(D, A);
  int ctl = pack_ctl(ctl_init(D, A));
  for (int l = 0; l < L; ++l) {
    ctl = pstep_qkv<DT, V>(Dp, A, l, ctl, l ? ++k : 0, lds);
    const bool river = ctl & 1;
    pstep_attn<DT, F16, HD>(Dp, A, l, ctl, ++k, lds);
    pstep_gemv<DT, PH_O, V>(Dp, A, l, river, ++k, lds);
    pstep_gemv<DT, PH_GU, V>(Dp, A, l, river, ++k, lds);
    pstep_gemv<DT, PH_DOWN, V>(Dp, A, l, river, ++k, lds);
  }
  if (A.want_head) pstep_head<DT, V>(Dp, A, ctl, ++k, lds);
}

// Interleaves the river's scale and zero arrays into one (scale, zero) pair per group,
// so that a lane fetches both with one load.
template <int DT>
__global__ void k_pack_sz(const void *scale, const void *zero, void *out, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n)
    ((typename Store<DT>::SZ *)out)[i] = Store<DT>::pack(Store<DT>::ld(scale, i), Store<DT>::ld(zero, i));
}

// River construction.  The floor is the stream (weights read once, half a byte per weight written:
// 0.15 GB for a 14336 x 4096 bf16 matrix); what the kernel must not do is give a lane a whole group,
// whose elements then come one at a time from addresses a group apart.  A lane owns runs of 16
// consecutive elements (one or two 16-byte loads per eight of them, one 8-byte store of codes), the
// `1 << lg_log2` lanes of a group are neighbours and agree on minimum and maximum by lane exchange.
// The host picks the lanes per group as the power of two that covers the group's runs (at most a
// wavefront; longer groups take several rounds, and lanes beyond the group's last run repeat its
// first one, which changes neither extreme).  slots = groups per row << lg_log2 lanes serve a row.
// WIDE: w is 16-byte and codes 8-byte aligned (every row then is too: cols % 16 == 0); otherwise the
// same runs go element by element.  14336 x 4096 bf16, group 64: 1531 us as one lane per group with
// scalar loads, 42 us now (3.7 TB/s; a large copy reaches 4.7).
template <int DT, bool WIDE>
__device__ __forceinline__ void quant_load16(const void *w, size_t i, float (&v)[16]) {
  if constexpr (WIDE) {
    constexpr int EPL = Store<DT>::EPL;
#pragma unroll
    for (int k = 0; k < 16 / EPL; ++k) {
      float f[EPL];
      Store<DT>::unpack(ld_stream16((const char *)w + (i + k * EPL) * sizeof(typename Store<DT>::T)), f);
#pragma unroll
      for (int e = 0; e < EPL; ++e) v[k * EPL + e] = f[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = Store<DT>::ld(w, i + e);
  }
}
template <int DT, bool WIDE>
__global__ __launch_bounds__(256) void k_quantize_w4(const void *w, long long rows, int cols, int group, int gpr,
                                                     int lg_log2, uint8_t *codes, void *scale, void *zero) {
  // workgroup -> its first lane's (row, slot): a uniform division; the lane's own is a 32-bit one
  const unsigned slots = (unsigned)gpr << lg_log2;
  const unsigned long long first = ((unsigned long long)blockIdx.y * gridDim.x + blockIdx.x) * 256u;
  const unsigned in_row = (unsigned)(first % slots) + threadIdx.x;
  const long long r = (long long)(first / slots) + in_row / slots;
  if (r >= rows) return;                               // (whole groups of lanes: 256 and slots are multiples of one)
  const unsigned slot = in_row % slots;
  const int g = (int)(slot >> lg_log2), li = (int)slot & ((1 << lg_log2) - 1);
  const int c0 = g * group, runs = min(group, cols - c0) >> 4;
  const size_t base = (size_t)r * cols + c0;
  const int stride = 1 << lg_log2, my = li < runs ? li : 0;
  float v[16];
  quant_load16<DT, WIDE>(w, base + my * 16, v);
  float mn = v[0], mx = v[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) { mn = fminf(mn, v[e]); mx = fmaxf(mx, v[e]); }
  for (int q = my + stride; q < runs; q += stride) {
    float u[16];
    quant_load16<DT, WIDE>(w, base + q * 16, u);
#pragma unroll
    for (int e = 0; e < 16; ++e) { mn = fminf(mn, u[e]); mx = fmaxf(mx, u[e]); }
  }
  for (int o = 1; o < stride; o <<= 1) { mn = fminf(mn, __shfl_xor(mn, o)); mx = fmaxf(mx, __shfl_xor(mx, o)); }
  // the stored (rounded) scale and zero point define the grid
  const float s = Store<DT>::rnd((mx > mn) ? (mx - mn) / 15.0f : 1.0f);
  const float z = Store<DT>::rnd(-mn / s);
  if (li == 0) {
    const size_t idx = (size_t)r * gpr + g;
    Store<DT>::st(scale, idx, s);
    Store<DT>::st(zero, idx, z);
  }
  auto encode = [&](const float (&x)[16], int q) {
    uint32_t word[2] = {0u, 0u};
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float t = rintf(x[e] / s + z);
      const int c = t < 0.f ? 0 : (t > 15.f ? 15 : (int)t);
      word[e >> 3] |= (uint32_t)c << (4 * (e & 7));
    }
    uint8_t *dst = codes + ((base + (size_t)q * 16) >> 1);
    if constexpr (WIDE) {
      *(u32x2 *)dst = u32x2{word[0], word[1]};
    } else {
#pragma unroll
      for (int b = 0; b < 8; ++b) dst[b] = (uint8_t)(word[b >> 2] >> (8 * (b & 3)));
    }
  };
  if (li < runs) encode(v, li);
  for (int q = li + stride; q < runs; q += stride) {
    quant_load16<DT, WIDE>(w, base + q * 16, v);
    encode(v, q);
  }
}

// A new sequence: the token state and the barrier's counters and error flag start at zero.  One workgroup of 64.
__global__ void k_reset(DevState *st, unsigned long long *bar) {
  if (threadIdx.x == 0) { *st = DevState{}; *bar_error(bar) = 0; }
  if (threadIdx.x < kBarCounters) *bar_counter(bar, threadIdx.x) = 0;
}

__global__ void k_fill_bytes(uint4 *p, size_t n16, uint32_t word) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = make_uint4(word, word, word, word);
}

// ------------------------------------------------------------------ context

struct Layout {
  size_t kcache, vcache, rope, hidden, qbuf, obuf, kvcur, h1, abuf, logits, part_o, part_ml, cos_part,
      amax_val, amax_idx, state, rec, layers, dev, trace, qsz, total;
  size_t cache_bytes, qsz_bytes;
  size_t bd_partial;                     // [kBdKSplit][32][d_model] partial sums of the K-sliced GEMMs
  size_t bd_ssq;
  size_t bd_stream, bd_stream_bytes;     // batched contexts: the GEMM weights a second time, in stream order (bd::BdB)
  // activation buffers of the GEMM prefill (pf_rows rows each; 0 rows: that path is not offered)
  size_t pf_tok, pf_h, pf_x16, pf_q16, pf_a16, pf_big, pf_big_bytes;
  int pf_rows;
  // batched contexts (max_batch > 1): per-sequence state, step buffers, records
  size_t bd_state, bd_hprev, bd_part_o, bd_part_ml, bd_tickets, bd_logits, bd_hist, bd_rec;
};


// Barrier blocks that are polled with scalar loads live in uncached device memory, which is
// allocated once per device and process and never freed (freeing uncached memory that a
// kernel has read is not safe on all systems); contexts take and return slots of it.
namespace {
constexpr int kBarSlots = 64, kBarDevices = 16;
std::mutex g_bar_mu;
char *g_bar_pool[kBarDevices];
unsigned long long g_bar_used[kBarDevices];
}
// Static scratch for river_create_static: the step-transient part of the workspace
// (activations, partial results, counters, records, descriptor tables) and the barrier
// block, for callers that must not allocate.  Each device holds its own copy of the array;
// host code uses the per-device address from hipGetSymbolAddress, never the array's name.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes + kBarBytes];
namespace {
char *g_static_ptr[kBarDevices];          // device address of g_static_scratch, per device
bool g_static_live[kBarDevices];          // a live context uses the device's scratch
}
// Address of the current device's copy of the static scratch (looked up once per device).
static int static_scratch_ptr(int dev, char **ptr, std::string *why) {
  std::lock_guard<std::mutex> lk(g_bar_mu);
  if (dev < 0 || dev >= kBarDevices) { *why = "device index too large for the static scratch table"; return RIVER_EINVAL; }
  if (!g_static_ptr[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch));
    if (e != hipSuccess || !p) {
      *why = std::string("hipGetSymbolAddress(static scratch): ") + hipGetErrorString(e);
      return RIVER_EHIP;
    }
    g_static_ptr[dev] = (char *)p;
  }
  *ptr = g_static_ptr[dev];
  return RIVER_OK;
}

static int bar_acquire(int dev, int *slot, char **ptr, std::string *why) {
  std::lock_guard<std::mutex> lk(g_bar_mu);
  if (dev < 0 || dev >= kBarDevices) { *why = "device index too large for the barrier pool"; return RIVER_EINVAL; }
  if (!g_bar_pool[dev]) {
    void *p = nullptr;
    const hipError_t e = hipExtMallocWithFlags(&p, (size_t)kBarSlots * kBarBytes, hipDeviceMallocUncached);
    if (e != hipSuccess) { *why = std::string("uncached barrier pool: ") + hipGetErrorString(e); return RIVER_EHIP; }
    g_bar_pool[dev] = (char *)p;
  }
  for (int i = 0; i < kBarSlots; ++i)
    if (!(g_bar_used[dev] >> i & 1ull)) {
      g_bar_used[dev] |= 1ull << i;
      *slot = i;
      *ptr = g_bar_pool[dev] + (size_t)i * kBarBytes;
      return RIVER_OK;
    }
  *why = "more than 64 live contexts on one device";
  return RIVER_ENOSPC;
}
static void bar_release(int dev, int slot) {
  std::lock_guard<std::mutex> lk(g_bar_mu);
  if (slot >= 0) g_bar_used[dev] &= ~(1ull << slot);
}

// Pinned host memory of a context, beside its barrier slot (64 slots, allocated with the first context of
// a device and kept): the last kernel of a synchronous call writes the record there, so that the call
// waits for the stream and nothing else, and the first kernel of a short prefill reads its tokens there.
// (A pageable copy and the wait for it take 19 us, a kernel's store and the wait 11.)  A record that does
// not fit, and contexts without a barrier slot, use copies.
constexpr int kHostRec = 4096, kHostTok = 512;
struct HostSlot { int32_t rec[kHostRec], tok[kHostTok]; };
namespace { HostSlot *g_host_pool[kBarDevices]; }
static HostSlot *host_slot(int dev, int slot) {             // null: no pinned memory to be had
  std::lock_guard<std::mutex> lk(g_bar_mu);
  if (!g_host_pool[dev]) {
    void *p = nullptr;
    if (hipHostMalloc(&p, sizeof(HostSlot) * kBarSlots, hipHostMallocCoherent) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_host_pool[dev] = (HostSlot *)p;
  }
  return g_host_pool[dev] + slot;
}

struct river_ctx {
  river_config cfg;
  Dev dev;              // host copy of the descriptor
  const Dev *dev_d;     // the same in the workspace
  Layout lay;
  char *ws;
  hipStream_t stream;
  int pos;              // positions in the cache
  bool have_token;      // DevState::cur_token is valid
  bool have_river;
  long long steps;      // decode steps recorded so far
  unsigned long long bar_total;
  int bar_slot = -1;    // slot of the process-wide barrier pool
  int bar_device = 0;
  HostSlot *host = nullptr;   // pinned memory of this context (null: copies)
  bool is_static = false; // activations and barrier block live in the device's static scratch
  ~river_ctx() {
    bar_release(bar_device, bar_slot);
    if (is_static) {
      std::lock_guard<std::mutex> lk(g_bar_mu);
      g_static_live[bar_device] = false;
    }
  }
  int grid_persist, grid_gemv, block;
  size_t lds_bytes;
  bool broken;
  std::string err;
  std::vector<DevLayer> layers_h;   // host copy of the per-block pointer table (GEMM prefill launches)
  std::vector<bd::BdB> bd_dense_h, bd_twin_h;   // [L][4] stream-order weights of the QKV / O / gate-up / down GEMMs
  bd::BdB bd_head;                  // (batched contexts; a twin that was not given: null)
  std::vector<int32_t> rec_h;       // host copy of a step's record
  std::vector<int> pos_b;           // batched contexts: positions in the cache, per sequence
  long long steps_b = 0;            // batched decode steps recorded so far
  int last_n = 0;                   // sequences of the last batched step
  bd::SeqState st_b{};
};

static thread_local std::string g_create_err;

// Rows of d_model and n_q * head_dim columns of at most four 1 KiB granules (see Shape).  Sections of four bf16
// blocks of head size 64, d_model 512 / 1024 / 1536 / 2048 / 2304 / 2560 / 3072 / 4096, us per step with the
// narrow shapes and without: backbone 108 / 119 / 142 / 168 / 207 / 228 / 262 / 368 and 108 / 123 / 145 / 171 / 200 / 218 /
// 257 / 360, river 110 / 115 / 124 / 132 / 163 / 185 / 199 / 231 and 114 / 122 / 130 / 140 / 166 / 177 / 190 / 223.
static bool narrow_model(const river_config &c) {
  return std::max(c.d_model, c.n_q_heads * c.head_dim) * (c.dtype == RIVER_BF16 ? 2 : 4) <= 4096;
}
// The one-launch step kernel of a configuration (bf16), by cache type, head size and variant (see Pre)
typedef void (*StepKernel)(const Dev *, StepArgs);
template <bool F16, int HD>
static StepKernel step_kernel_of(const river_config &c) {
  const bool cols32 = c.d_model % 32 == 0 && c.d_ffn % 32 == 0 && c.n_q_heads * c.head_dim % 32 == 0;
  if (!cols32) return k_step_persistent<1, F16, 0, HD>;
  return narrow_model(c) ? k_step_persistent<1, F16, V_NARROW | V_COLS32, HD> : k_step_persistent<1, F16, V_COLS32, HD>;
}
static StepKernel step_kernel(const river_ctx *x) {
  const river_config &c = x->cfg;
  const bool f16 = c.kv_dtype == RIVER_KV_F16;
  return c.head_dim == 128 ? (f16 ? step_kernel_of<true, 128>(c) : step_kernel_of<false, 128>(c))
                           : (f16 ? step_kernel_of<true, 64>(c) : step_kernel_of<false, 64>(c));
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Shapes the GEMM prefill handles: bf16 storage, every contraction length a multiple of the
// 64-column K tile, quantisation groups made of whole K tiles.
static bool gemm_prefill_ok(const river_config *c) {
  return c->dtype == RIVER_BF16 && c->d_model % 64 == 0 && c->d_ffn % 64 == 0 &&
         (c->n_q_heads * c->head_dim) % 64 == 0 && c->river_group % 64 == 0 && c->prefill_gemm_min_tokens >= 0;
}

static bool valid_cfg(const river_config *c, std::string *why) {
  auto bad = [&](const char *m) { if (why) *why = m; return false; };
  if (!c) return bad("null config");
  if (c->n_layers < 1 || c->d_model < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->d_ffn < 1 ||
      c->vocab < 1 || c->max_seq < 1)
    return bad("non-positive dimension");
  if (c->dtype != RIVER_F32 && c->dtype != RIVER_BF16) return bad("dtype must be RIVER_F32 or RIVER_BF16");
  if (c->max_batch < 1 || c->max_batch > bd::kRows) return bad("max_batch must be in [1, 32]");
  if (c->batch_exit_rule != 0 && c->batch_exit_rule != 1) return bad("batch_exit_rule must be 0 or 1");
  if (c->river_bits != 4) return bad("river_bits must be 4");
  if (c->river_group < 32 || c->river_group % 32) return bad("river_group must be a multiple of 32");
  if (c->n_q_heads % c->n_kv_heads) return bad("n_q_heads must be a multiple of n_kv_heads");
  const int hd = c->head_dim;
  if (hd != 64 && hd != 128) return bad("head_dim must be 64 or 128");
  if (c->d_model % 16 || c->d_ffn % 16) return bad("d_model and d_ffn must be multiples of 16");
  if (c->vocab % 2) return bad("vocab must be even");
  if (c->min_exit_layer < 0 || c->min_exit_layer > c->n_layers) return bad("min_exit_layer out of range");
  if (c->exec_mode != RIVER_EXEC_KERNELS && c->exec_mode != RIVER_EXEC_PERSISTENT) return bad("bad exec_mode");
  if (c->exec_mode == RIVER_EXEC_PERSISTENT && c->dtype != RIVER_BF16)
    return bad("RIVER_EXEC_PERSISTENT is available for RIVER_BF16 only; use RIVER_EXEC_KERNELS for RIVER_F32");
  if (c->spin_limit < 0) return bad("negative spin_limit");
  if (c->kv_dtype != RIVER_KV_SAME && c->kv_dtype != RIVER_KV_F16) return bad("bad kv_dtype");
  if (c->kv_dtype == RIVER_KV_F16 && c->dtype != RIVER_BF16) return bad("RIVER_KV_F16 needs RIVER_BF16 weights");
  if (!(c->rope_base > 0.f) || !(c->rms_eps >= 0.f)) return bad("bad rope_base / rms_eps");
  if (c->max_batch > 1) {
    if (!gemm_prefill_ok(c))
      return bad("max_batch > 1 needs RIVER_BF16 with d_model, d_ffn and river_group multiples of 64 and the GEMM "
                 "prefill enabled");
  }
  return true;
}


static int x_capacity(const river_config *c) {
  int cap = c->d_model;
  cap = std::max(cap, c->n_q_heads * c->head_dim);
  cap = std::max(cap, c->d_ffn);
  cap = std::max(cap, attn_lds_floats(c->head_dim));
  // the staged vector is stored granule-wise (64 lanes x up to 32 columns): whole granules
  return (int)align_up(cap, 2048);
}

// [rows, cols] of block matrix m (wq wk wv wo w_gate w_up w_down)
static void matrix_shape(const river_config *c, int m, long long *rows, long long *cols) {
  const long long q = (long long)c->n_q_heads * c->head_dim, kv = (long long)c->n_kv_heads * c->head_dim;
  const long long d = c->d_model, f = c->d_ffn;
  const long long R[7] = {q, kv, kv, d, f, f, d}, C[7] = {d, d, d, q, d, d, f};
  *rows = R[m];
  *cols = C[m];
}
static size_t qsz_matrix_bytes(const river_config *c, int m) {
  long long rows, cols;
  matrix_shape(c, m, &rows, &cols);
  const long long gpr = (cols + c->river_group - 1) / c->river_group;
  return (size_t)(rows * gpr) * (c->dtype == RIVER_BF16 ? 4 : 8);
}

// The four GEMMs of a block in a batched step: matrices (stacked along N, or interleaved), N, K
struct BdGemmShape { int ms[3], nm, interleaved, N, K; };
static BdGemmShape bd_gemm_shape(const river_config *c, int g) {
  const int q = c->n_q_heads * c->head_dim, kv = c->n_kv_heads * c->head_dim, d = c->d_model, f = c->d_ffn;
  switch (g) {
    case 0: return {{M_WQ, M_WK, M_WV}, 3, 0, q + 2 * kv, d};
    case 1: return {{M_WO, M_WO, M_WO}, 1, 0, d, q};
    case 2: return {{M_GATE, M_UP, M_UP}, 2, 1, 2 * f, d};
    default: return {{M_DOWN, M_DOWN, M_DOWN}, 1, 0, d, f};
  }
}
static size_t bd_stream_bytes_of(const river_config *c) {
  size_t per_block = 0;
  for (int g = 0; g < 4; ++g) {
    const BdGemmShape sh = bd_gemm_shape(c, g);
    per_block += align_up(bd::bd_dense_bytes(sh.N, sh.K), 256) + align_up(bd::bd_codes_bytes(sh.N, sh.K), 256) +
                 align_up(bd::bd_pairs_bytes(sh.N, sh.K), 256);
  }
  return per_block * (size_t)c->n_layers + align_up(bd::bd_dense_bytes(c->vocab, c->d_model), 256);
}

static Layout make_layout(const river_config *c) {
  Layout y{};
  const size_t es = c->dtype == RIVER_BF16 ? 2 : 4;
  const size_t kvd = (size_t)c->n_kv_heads * c->head_dim;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  y.cache_bytes = (size_t)c->n_layers * c->max_seq * kvd * es;      // one sequence
  y.kcache = take(y.cache_bytes * c->max_batch);
  y.vcache = take(y.cache_bytes * c->max_batch);
  y.rope = take((size_t)c->max_seq * (c->head_dim / 2) * sizeof(float2));
  y.hidden = take((size_t)(c->n_layers + 1) * c->d_model * 4);
  y.qbuf = take((size_t)c->n_q_heads * c->head_dim * 4);
  y.obuf = take((size_t)c->n_q_heads * c->head_dim * 4);
  y.kvcur = take((size_t)2 * kvd * 4);
  y.h1 = take((size_t)c->d_model * 4);
  y.abuf = take((size_t)c->d_ffn * 4);
  y.logits = take((size_t)c->vocab * 4);
  y.part_o = take((size_t)c->n_q_heads * kMaxSplits * c->head_dim * 4);
  y.part_ml = take((size_t)c->n_q_heads * kMaxSplits * 4 * 4);
  y.cos_part = take((size_t)kMaxGrid * 4 * 4);
  y.amax_val = take((size_t)kMaxGrid * 4);
  y.amax_idx = take((size_t)kMaxGrid * 4);
  y.state = take(sizeof(DevState));
  y.rec = take((size_t)kRecords * (kRecHead + c->n_layers) * 4);
  y.layers = take((size_t)c->n_layers * sizeof(DevLayer));
  y.dev = take(sizeof(Dev));
  y.trace = take(((size_t)5 * c->n_layers * 2 * kMaxGrid + 64) * 8);
  // packed (scale, zero) pairs of every river matrix of every block
  y.qsz_bytes = 0;
  for (int m = 0; m < 7; ++m) y.qsz_bytes += align_up(qsz_matrix_bytes(c, m), 256);
  y.qsz_bytes *= (size_t)c->n_layers;
  y.qsz = take(y.qsz_bytes);
  y.pf_rows = 0;
  if (gemm_prefill_ok(c)) {
    const size_t qd = (size_t)c->n_q_heads * c->head_dim;
    // (the GEMMs address their fp16 input with 31-bit offsets: fewer rows for matrices wider than 262000)
    const size_t widest = std::max({(size_t)c->d_model, (size_t)c->d_ffn, qd}) * 2;
    const size_t most = std::max((size_t)128, std::min((size_t)pf::kChunk, (size_t)0x7fff0000 / widest / 128 * 128));
    const size_t rows = std::min(align_up((size_t)c->max_seq, 128), most);
    y.pf_rows = (int)rows;
    y.pf_tok = take(rows * 4);
    y.pf_h = take(rows * c->d_model * 4);
    y.pf_x16 = take(rows * std::max((size_t)c->d_model, qd) * 2);
    y.pf_q16 = take(rows * qd * 2);
    y.pf_a16 = take(rows * c->d_ffn * 2);
    // fp32 planes of the QKV, O and down GEMMs: one of all rows, or several K slices of fewer
    y.pf_big_bytes = std::max(rows, std::min((size_t)pf::kChunk, 16 * rows)) * std::max((size_t)c->d_model, qd + 2 * kvd) * 4;
    y.pf_big = take(y.pf_big_bytes);
  }
  if (c->max_batch > 1) {
    const size_t B = c->max_batch, qd = (size_t)c->n_q_heads * c->head_dim;
    y.bd_state = take(6 * B * 4);
    y.bd_hprev = take((size_t)bd::kRows * c->d_model * 4);
    y.bd_part_o = take((size_t)bd::kRows * qd * bd::kBdAttnMaxSplits * 4);      // attention split partials
    y.bd_part_ml = take((size_t)bd::kRows * std::max(c->n_q_heads * bd::kBdAttnMaxSplits, bd::kBdArgmaxChunks) * 2 * 4);  // (also the argmax partials)
    y.bd_tickets = take((size_t)bd::kRows * c->n_q_heads * 4);
    y.bd_logits = take(B * c->vocab * 4);
    y.bd_hist = take((size_t)(c->n_layers + 1) * B * c->d_model * 4);
    y.bd_rec = take((size_t)bd::kRecordsB * B * (2 + c->n_layers) * 4);         // a step's row: tokens, exits, similarities
    y.bd_partial = take((size_t)bd::kBdKSplit * bd::kRows * c->d_model * 4);
    y.bd_ssq = take((size_t)kMaxGrid * bd::kRows * 4);                          // sums of squares per GEMM workgroup and row
    y.bd_stream_bytes = bd_stream_bytes_of(c);
    y.bd_stream = take(y.bd_stream_bytes);
  }
  y.total = off;
  return y;
}

#define HIP_TRY(ctx, expr)                                                              \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) {                                                             \
      (ctx)->err = std::string(#expr) + ": " + hipGetErrorString(e_);                   \
      (ctx)->broken = true;                                                             \
      return RIVER_EHIP;                                                                \
    }                                                                                   \
  } while (0)

extern "C" size_t river_workspace_bytes(const river_config *cfg) {
  if (!valid_cfg(cfg, nullptr)) return 0;
  return make_layout(cfg).total;
}

extern "C" int river_quantize_w4(const void *w, int64_t rows, int64_t cols, int32_t group,
                                 int32_t dtype, void *codes, void *scale, void *zero,
                                 void *hip_stream) {
  if (!w || !codes || !scale || !zero || rows < 1 || cols < 16 || cols % 16 || group < 32 ||
      group % 32 || cols > (1 << 30) || (dtype != RIVER_F32 && dtype != RIVER_BF16))
    return RIVER_EINVAL;
  const long long gpr = (cols + group - 1) / group;
  int lg = 0;                                              // log2 of the lanes per group
  while (lg < 6 && (16 << lg) < std::min<long long>(group, cols)) ++lg;
  const long long slots = gpr << lg;                       // lanes per row
  if (rows > (0x7fffffffLL << 8) / slots) return RIVER_EINVAL;
  // two grid dimensions: one holds fewer than 2^32 threads (a larger launch is cut off without an error)
  const long long wgs = (rows * slots + 255) / 256, most = 1 << 23;
  const dim3 grid((unsigned)std::min(wgs, most), (unsigned)((wgs + most - 1) / most)), blk(256);
  const bool wide = ((uintptr_t)w) % 16 == 0 && ((uintptr_t)codes) % 8 == 0;
  hipStream_t st = (hipStream_t)hip_stream;
  auto k = dtype == RIVER_BF16 ? (wide ? k_quantize_w4<1, true> : k_quantize_w4<1, false>)
                               : (wide ? k_quantize_w4<0, true> : k_quantize_w4<0, false>);
  k<<<grid, blk, 0, st>>>(w, rows, (int)cols, group, (int)gpr, lg, (uint8_t *)codes, scale, zero);
  return hipGetLastError() == hipSuccess ? RIVER_OK : RIVER_EHIP;
}

static int reset_state(river_ctx *x) {
  k_reset<<<dim3(1), dim3(64), 0, x->stream>>>(x->dev.st, x->dev.bar);
  HIP_TRY(x, hipGetLastError());
  x->bar_total = 0;
  return RIVER_OK;
}

static int create_impl(const river_config *cfg, const river_weights *w, const river_qweights *q,
                       void *workspace, size_t workspace_bytes, void *hip_stream, river_ctx **out,
                       bool use_static) {
  std::string why;
  if (!out) { g_create_err = "null out"; return RIVER_EINVAL; }
  *out = nullptr;
  if (!valid_cfg(cfg, &why)) { g_create_err = why; return RIVER_EINVAL; }
  if (!w || !workspace) { g_create_err = "null weights or workspace"; return RIVER_EINVAL; }
  if (((uintptr_t)workspace) % 256) { g_create_err = "workspace must be 256-byte aligned"; return RIVER_EINVAL; }
  if (!w->tok_emb || !w->final_norm || !w->lm_head || !w->attn_norm || !w->wq || !w->wk || !w->wv ||
      !w->wo || !w->ffn_norm || !w->w_gate || !w->w_up || !w->w_down) {
    g_create_err = "null weight table";
    return RIVER_EINVAL;
  }
  const int L = cfg->n_layers;
  const void *const *tabs[9] = {w->attn_norm, w->ffn_norm, w->wq, w->wk, w->wv, w->wo,
                                w->w_gate, w->w_up, w->w_down};
  for (int l = 0; l < L; ++l)
    for (int t = 0; t < 9; ++t)
      if (!tabs[t][l] || ((uintptr_t)tabs[t][l]) % 16) {
        g_create_err = "null or misaligned (16 B) layer weight";
        return RIVER_EINVAL;
      }
  Layout lay = make_layout(cfg);
  if (workspace_bytes < lay.total) { g_create_err = "workspace too small"; return RIVER_ENOSPC; }

  river_ctx *x = new river_ctx();
  x->cfg = *cfg;
  x->lay = lay;
  x->ws = (char *)workspace;
  x->stream = (hipStream_t)hip_stream;
  x->pos = 0;
  x->have_token = false;
  x->steps = 0;
  x->bar_total = 0;
  x->broken = false;
  x->block = kBlock;

  // river twins: a block's twin is usable only if all its 21 pointers are given
  std::vector<DevLayer> hl(L);
  std::vector<const void *> hqs((size_t)L * 7, nullptr), hqz((size_t)L * 7, nullptr);
  x->have_river = q != nullptr;
  for (int l = 0; l < L; ++l) {
    DevLayer &d = hl[l];
    d.attn_norm = w->attn_norm[l];
    d.ffn_norm = w->ffn_norm[l];
    d.w[0] = w->wq[l]; d.w[1] = w->wk[l]; d.w[2] = w->wv[l]; d.w[3] = w->wo[l];
    d.w[4] = w->w_gate[l]; d.w[5] = w->w_up[l]; d.w[6] = w->w_down[l];
    for (int m = 0; m < 7; ++m) {
      d.qc[m] = nullptr; d.qsz[m] = nullptr;
      if (q && q->codes[m] && q->scale[m] && q->zero[m]) {
        d.qc[m] = (const uint8_t *)q->codes[m][l];
        hqs[(size_t)l * 7 + m] = q->scale[m][l];
        hqz[(size_t)l * 7 + m] = q->zero[m][l];
        if (((uintptr_t)d.qc[m]) % 16) {
          g_create_err = "misaligned (16 B) river codes";
          delete x;
          return RIVER_EINVAL;
        }
      }
    }
  }
  // blocks above L_s must have a complete twin if a river is given at all
  if (q)
    for (int l = std::max(cfg->min_exit_layer, 0); l < L; ++l)
      for (int m = 0; m < 7; ++m)
        if (!hl[l].qc[m] || !hqs[(size_t)l * 7 + m] || !hqz[(size_t)l * 7 + m]) {
          g_create_err = "river twin missing for a block above min_exit_layer";
          delete x;
          return RIVER_EINVAL;
        }

  int dev_id = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev_id) != hipSuccess || hipGetDeviceProperties(&prop, dev_id) != hipSuccess) {
    g_create_err = "no HIP device";
    delete x;
    return RIVER_EHIP;
  }
  const int cus = prop.multiProcessorCount;
  // one workgroup per CU, a multiple of 8 (the XCDs)
  x->grid_persist = std::max(8, std::min(cus, kMaxGrid) / 8 * 8);
  // One launch per phase: no more workgroups than the widest phase has tasks for (a task is one or two
  // rows per wavefront; attention: a query head and split), a multiple of 8.  Small models only: the
  // tiny fp32 shape runs 88 workgroups instead of 256.
  {
    const int qkv = (cfg->n_q_heads + 2 * cfg->n_kv_heads) * cfg->head_dim, splits = std::min(kMaxSplits, (cfg->max_seq + 255) / 256);
    const int tasks = std::max({qkv, cfg->d_model, cfg->d_ffn, (cfg->vocab + 1) / 2, kWaves * cfg->n_q_heads * splits});
    x->grid_gemv = std::min(x->grid_persist, (tasks + 8 * kWaves - 1) / (8 * kWaves) * 8);
  }

  // Where the step-transient part of the layout [hidden, qsz) lives: in the workspace, or in
  // the device's static scratch followed by the barrier block (`act + lay.X` addresses member
  // X of that part in both cases).
  char *act = x->ws;
  char *static_bar = nullptr;
  if (use_static) {
    const size_t need = lay.qsz - lay.hidden;
    if (need > kStaticScratchBytes) {
      g_create_err = "configuration needs " + std::to_string(need) + " bytes of scratch; the static scratch of "
                     "river_create_static holds " + std::to_string(kStaticScratchBytes) + " (use river_create)";
      delete x;
      return RIVER_ENOSPC;
    }
    char *sp = nullptr;
    std::string why2;
    const int rc = static_scratch_ptr(dev_id, &sp, &why2);
    if (rc != RIVER_OK) { g_create_err = why2; delete x; return rc; }
    bool busy;
    {
      std::lock_guard<std::mutex> lk(g_bar_mu);
      busy = g_static_live[dev_id];
      if (!busy) g_static_live[dev_id] = true;
    }
    if (busy) {                 // (the context's destructor takes the same lock)
      g_create_err = "the static scratch of this device is in use by a live context";
      delete x;
      return RIVER_ESTATE;
    }
    x->is_static = true;
    x->bar_device = dev_id;
    act = sp - lay.hidden;
    static_bar = sp + (lay.qsz - lay.hidden);
  }

  Dev &D = x->dev;
  D.L = L; D.d = cfg->d_model; D.nq = cfg->n_q_heads; D.nkv = cfg->n_kv_heads; D.hd = cfg->head_dim;
  D.ffn = cfg->d_ffn; D.vocab = cfg->vocab; D.max_seq = cfg->max_seq; D.min_exit = cfg->min_exit_layer;
  D.group = cfg->river_group;
  D.kv_f16 = cfg->kv_dtype == RIVER_KV_F16 ? 1 : 0;
  D.spin_limit = cfg->spin_limit > 0 ? cfg->spin_limit : (1 << 22);
  D.xcap = x_capacity(cfg);
  D.eps = cfg->rms_eps; D.tau = cfg->tau;
  D.tok_emb = w->tok_emb; D.final_norm = w->final_norm; D.lm_head = w->lm_head;
  char *ws = x->ws;
  D.layers = (const DevLayer *)(act + lay.layers);
  D.kcache = ws + lay.kcache; D.vcache = ws + lay.vcache;
  D.rope = (const float2 *)(ws + lay.rope);
  D.hidden = (float *)(act + lay.hidden);
  D.qbuf = (float *)(act + lay.qbuf); D.obuf = (float *)(act + lay.obuf);
  D.kvcur = (float *)(act + lay.kvcur);
  D.h1 = (float *)(act + lay.h1); D.abuf = (float *)(act + lay.abuf);
  D.logits = (float *)(act + lay.logits);
  D.part_o = (float *)(act + lay.part_o); D.part_ml = (float *)(act + lay.part_ml);
  D.cos_part = (float *)(act + lay.cos_part);
  D.amax_val = (float *)(act + lay.amax_val); D.amax_idx = (int *)(act + lay.amax_idx);
  D.st = (DevState *)(act + lay.state);
  if (use_static) {
    // ordinary device memory: polled with device-coherent vector loads (see barrier_wait)
    D.bar = (unsigned long long *)static_bar;
    D.bar_vector_poll = 1;
  } else {
    char *bp = nullptr;
    std::string why2;
    x->bar_device = dev_id;
    const int rc = bar_acquire(dev_id, &x->bar_slot, &bp, &why2);
    if (rc != RIVER_OK) { g_create_err = why2; delete x; return rc; }
    D.bar = (unsigned long long *)bp;
    D.bar_vector_poll = 0;
    const size_t words = cfg->max_batch > 1 ? (size_t)cfg->max_batch * (2 + L) : (size_t)kRecHead + L;
    if (words <= kHostRec) x->host = host_slot(dev_id, x->bar_slot);
  }
  D.rec = (int *)(act + lay.rec);
  D.trace = (unsigned long long *)(act + lay.trace);
  x->lds_bytes = ((size_t)D.xcap + lds_half_floats(D.xcap) + 64) * sizeof(float);

  // RoPE table in double precision: angle = pos * base^(-2i/hd)
  const int half = cfg->head_dim / 2;
  std::vector<float2> rope((size_t)cfg->max_seq * half);
  for (int i = 0; i < half; ++i) {
    const double th = std::pow((double)cfg->rope_base, -2.0 * i / cfg->head_dim);
    for (int p = 0; p < cfg->max_seq; ++p) {
      const double a = (double)p * th;
      rope[(size_t)p * half + i] = make_float2((float)std::cos(a), (float)std::sin(a));
    }
  }
  auto fail = [&](const char *what, hipError_t e) {
    g_create_err = std::string(what) + ": " + hipGetErrorString(e);
    delete x;
    return RIVER_EHIP;
  };
  hipError_t e;
  if ((e = hipMemcpyAsync(ws + lay.rope, rope.data(), rope.size() * sizeof(float2),
                          hipMemcpyHostToDevice, x->stream)) != hipSuccess)
    return fail("rope upload", e);
  x->dev_d = (const Dev *)(act + lay.dev);
  if ((e = hipMemcpyAsync(act + lay.dev, &x->dev, sizeof(Dev), hipMemcpyHostToDevice, x->stream)) != hipSuccess)
    return fail("descriptor upload", e);
  // pack (scale, zero) pairs of every river matrix that was given into the workspace
  {
    size_t off = lay.qsz;
    for (int l = 0; l < L; ++l)
      for (int m = 0; m < 7; ++m) {
        const size_t bytes = qsz_matrix_bytes(cfg, m);
        if (hl[l].qc[m] && hqs[(size_t)l * 7 + m] && hqz[(size_t)l * 7 + m]) {
          const long long n = (long long)(bytes / (cfg->dtype == RIVER_BF16 ? 4 : 8));
          const unsigned nb = (unsigned)((n + 255) / 256);
          if (cfg->dtype == RIVER_BF16)
            k_pack_sz<1><<<dim3(nb), dim3(256), 0, x->stream>>>(hqs[(size_t)l * 7 + m], hqz[(size_t)l * 7 + m], ws + off, n);
          else
            k_pack_sz<0><<<dim3(nb), dim3(256), 0, x->stream>>>(hqs[(size_t)l * 7 + m], hqz[(size_t)l * 7 + m], ws + off, n);
          hl[l].qsz[m] = ws + off;
        }
        off += align_up(bytes, 256);
      }
    if ((e = hipGetLastError()) != hipSuccess) return fail("river (scale, zero) packing", e);
  }
  // batched contexts: the GEMM weights a second time, in the order the batched GEMM streams them
  x->bd_dense_h.assign((size_t)L * 4, bd::BdB{nullptr, nullptr});
  x->bd_twin_h.assign((size_t)L * 4, bd::BdB{nullptr, nullptr});
  x->bd_head = bd::BdB{nullptr, nullptr};
  if (cfg->max_batch > 1) {
    size_t off = lay.bd_stream;
    auto blocks_of = [](size_t pieces) { return dim3((unsigned)((pieces + 255) / 256)); };
    for (int l = 0; l <= L; ++l)
      for (int g = 0; g < (l < L ? 4 : 1); ++g) {
        pf::GemmB Bw{}, Bc{}, Bs{};
        BdGemmShape sh = bd_gemm_shape(cfg, g);
        bool twin = l < L;
        if (l == L) {                                         // the LM head
          sh = BdGemmShape{{0, 0, 0}, 1, 0, cfg->vocab, cfg->d_model};
          Bw.w[0] = Bw.w[1] = Bw.w[2] = w->lm_head;
          Bw.rows[0] = cfg->vocab;
        } else {
          for (int i = 0; i < 3; ++i) {
            const int m = sh.ms[i < sh.nm ? i : 0];
            long long r, cc;
            matrix_shape(cfg, m, &r, &cc);
            Bw.w[i] = hl[l].w[m];
            Bc.w[i] = hl[l].qc[m];
            Bs.w[i] = hqs[(size_t)l * 7 + m];
            Bs.sz[i] = hqz[(size_t)l * 7 + m];
            Bw.rows[i] = Bc.rows[i] = Bs.rows[i] = i < sh.nm ? (int)r : 0;
            twin = twin && Bc.w[i] && Bs.w[i] && Bs.sz[i];
          }
        }
        const size_t units = bd::bd_units(sh.N);
        bd::k_bd_pack_dense<<<blocks_of(units * (sh.K / 64) * 64), dim3(256), 0, x->stream>>>(
            Bw, sh.interleaved, sh.N, sh.K, (uint4 *)(ws + off));
        bd::BdB dense{ws + off, nullptr};
        off += align_up(bd::bd_dense_bytes(sh.N, sh.K), 256);
        if (l == L) { x->bd_head = dense; break; }
        x->bd_dense_h[(size_t)l * 4 + g] = dense;
        const size_t cb = align_up(bd::bd_codes_bytes(sh.N, sh.K), 256), pb = align_up(bd::bd_pairs_bytes(sh.N, sh.K), 256);
        if (twin) {
          const size_t nkt = (size_t)(sh.K + 127) / 128;
          bd::k_bd_pack_codes<<<blocks_of(units * nkt * 32), dim3(256), 0, x->stream>>>(
              Bc, sh.interleaved, sh.N, sh.K, (uint4 *)(ws + off));
          bd::k_bd_pack_pairs<<<blocks_of(units * nkt * 16), dim3(256), 0, x->stream>>>(
              Bs, sh.interleaved, sh.N, sh.K, cfg->river_group, (uint32_t *)(ws + off + cb));
          x->bd_twin_h[(size_t)l * 4 + g] = bd::BdB{ws + off, ws + off + cb};
        }
        off += cb + pb;
      }
    if ((e = hipGetLastError()) != hipSuccess) return fail("stream-order weight packing", e);
  }
  x->layers_h = hl;
  x->pos_b.assign(cfg->max_batch, 0);
  if (cfg->max_batch > 1) {
    int *sp = (int *)(ws + lay.bd_state);
    const int B = cfg->max_batch;
    x->st_b.pos = sp; x->st_b.token = sp + B; x->st_b.river = sp + 2 * B; x->st_b.exit_pos = sp + 3 * B;
    x->st_b.forced = sp + 4 * B;
    if ((e = hipMemsetAsync(ws + lay.bd_state, 0, (size_t)6 * B * 4, x->stream)) != hipSuccess)
      return fail("sequence state clear", e);
    if ((e = hipMemsetAsync(ws + lay.bd_tickets, 0, (size_t)bd::kRows * cfg->n_q_heads * 4, x->stream)) != hipSuccess)
      return fail("attention ticket clear", e);
  }
  if ((e = hipMemcpyAsync(act + lay.layers, hl.data(), hl.size() * sizeof(DevLayer),
                          hipMemcpyHostToDevice, x->stream)) != hipSuccess)
    return fail("layer table upload", e);
  // everything after the caches starts at zero (state, counters, records, activations); the
  // static scratch keeps the previous context's contents, so this clear is what resets it
  if ((e = hipMemsetAsync(act + lay.hidden, 0, lay.layers - lay.hidden, x->stream)) != hipSuccess)
    return fail("workspace clear", e);
  if (use_static && (e = hipMemsetAsync(static_bar, 0, kBarBytes, x->stream)) != hipSuccess)
    return fail("barrier block clear", e);
  if ((e = hipMemsetAsync(ws + lay.kcache, 0, lay.vcache - lay.kcache + align_up(lay.cache_bytes * cfg->max_batch, 256),
                          x->stream)) != hipSuccess)
    return fail("cache clear", e);
  if ((e = hipStreamSynchronize(x->stream)) != hipSuccess) return fail("create sync", e);

  {
    const int lb = (int)x->lds_bytes;
    const void *fns[] = {
        (const void *)k_qkv<0, 0>, (const void *)k_qkv<0, V_NARROW>, (const void *)k_qkv<1, 0>,
        (const void *)k_attn<0, false>, (const void *)k_attn<1, false>, (const void *)k_attn<1, true>,
        (const void *)k_oproj<0, 0>, (const void *)k_oproj<0, V_NARROW>, (const void *)k_oproj<1, 0>,
        (const void *)k_gateup<0, 0>, (const void *)k_gateup<0, V_NARROW>, (const void *)k_gateup<1, 0>,
        (const void *)k_down<0, 0>, (const void *)k_down<0, V_NARROW>, (const void *)k_down<1, 0>,
        (const void *)k_head<0>, (const void *)k_head<1>, (const void *)k_pf_head, (const void *)step_kernel(x)};
    for (const void *f : fns)
      if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lb)) != hipSuccess)
        return fail("hipFuncSetAttribute(max dynamic LDS)", e);
    if (gemm_prefill_ok(cfg)) {
      std::vector<std::pair<const void *, int>> pfg = {
          {(const void *)pf::k_pf_gemm<pf::TileM, false, pf::PF_STORE>, pf::TileM::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileM, false, pf::PF_SWIGLU>, pf::TileM::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileM, true, pf::PF_STORE>, pf::TileM::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileM, true, pf::PF_SWIGLU>, pf::TileM::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileN, false, pf::PF_STORE>, pf::TileN::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileN, false, pf::PF_SWIGLU>, pf::TileN::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileN, true, pf::PF_STORE>, pf::TileN::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileN, true, pf::PF_SWIGLU>, pf::TileN::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileL, false, pf::PF_STORE>, pf::TileL::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileL, false, pf::PF_SWIGLU>, pf::TileL::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileL, true, pf::PF_STORE>, pf::TileL::LDS_BYTES},
          {(const void *)pf::k_pf_gemm<pf::TileL, true, pf::PF_SWIGLU>, pf::TileL::LDS_BYTES}};
      auto rows = [&](auto mb) {
        constexpr int MB = decltype(mb)::value;
        const int dense = pf::RowsTile<MB, false>::LDS_BYTES, codes = pf::RowsTile<MB, true>::LDS_BYTES;
        pfg.push_back({(const void *)pf::k_pf_gemm_rows<MB, false, pf::PF_STORE, false>, dense});
        pfg.push_back({(const void *)pf::k_pf_gemm_rows<MB, false, pf::PF_SWIGLU, false>, dense});
        pfg.push_back({(const void *)pf::k_pf_gemm_rows<MB, true, pf::PF_STORE, false>, codes});
        pfg.push_back({(const void *)pf::k_pf_gemm_rows<MB, true, pf::PF_SWIGLU, false>, codes});
      };
      rows(IC<1>{}); rows(IC<2>{}); rows(IC<3>{}); rows(IC<4>{});
      auto attn = [&](auto hd) {
        constexpr int HD = decltype(hd)::value;
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 1, 1>, pf::attn_lds_bytes(HD, 1)});
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 2, 1>, pf::attn_lds_bytes(HD, 1)});
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 4, 1>, pf::attn_lds_bytes(HD, 1)});
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 1, 2>, pf::attn_lds_bytes(HD, 2)});
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 2, 2>, pf::attn_lds_bytes(HD, 2)});
        pfg.push_back({(const void *)pf::k_pf_attn<HD, 4, 2>, pf::attn_lds_bytes(HD, 2)});
      };
      attn(IC<64>{}); attn(IC<128>{});
      pfg.push_back({(const void *)pf::k_pf_gemm_rows<3, false, pf::PF_STORE, true>, pf::RowsTile<3, false>::LDS_BYTES});
      pfg.push_back({(const void *)pf::k_pf_gemm_rows<1, true, pf::PF_STORE, true>, pf::RowsTile<1, true>::LDS_BYTES});
      for (const auto &f : pfg)
        if ((e = hipFuncSetAttribute(f.first, hipFuncAttributeMaxDynamicSharedMemorySize, f.second)) != hipSuccess)
          return fail("hipFuncSetAttribute(prefill GEMM LDS)", e);
    }
    if (cfg->max_batch > 1) {
      // the widest batched GEMMs keep 64 KiB of partial tiles beside their static LDS
      if ((e = hipFuncSetAttribute((const void *)bd::k_bd_gemm<1, 8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bd::bd_gemm_lds_bytes(8, 1))) != hipSuccess ||
          (e = hipFuncSetAttribute((const void *)bd::k_bd_gemm<2, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bd::bd_gemm_lds_bytes(4, 2))) != hipSuccess)
        return fail("hipFuncSetAttribute(batched GEMM LDS)", e);
    }
  }
  *out = x;
  return RIVER_OK;
}

extern "C" int river_create(const river_config *cfg, const river_weights *w, const river_qweights *q,
                            void *workspace, size_t workspace_bytes, void *hip_stream,
                            river_ctx **out) {
  return create_impl(cfg, w, q, workspace, workspace_bytes, hip_stream, out, false);
}

extern "C" int river_create_static(const river_config *cfg, const river_weights *w, const river_qweights *q,
                                   void *workspace, size_t workspace_bytes, void *hip_stream,
                                   river_ctx **out) {
  return create_impl(cfg, w, q, workspace, workspace_bytes, hip_stream, out, true);
}

// Enqueue one token (prompt position or decode step).  V: see Pre.
template <int DT, int V>
static int launch_step(river_ctx *x, const StepArgs &A0) {
  StepArgs A = A0;
  const Dev &D = x->dev;
  const Dev *Dp = x->dev_d;
  const dim3 blk(x->block);
  const size_t lds = x->lds_bytes;
  hipStream_t s = x->stream;
  if (x->cfg.exec_mode == RIVER_EXEC_PERSISTENT) {
    // bf16 only (river_create refuses the combination with fp32)
    if constexpr (DT == 1) {
      A.bar_base = x->bar_total;
      step_kernel(x)<<<dim3(x->grid_persist), blk, lds, s>>>(Dp, A);
      x->bar_total += 5ull * D.L - 1 + (A.want_head ? 1 : 0);
    } else {
      x->err = "RIVER_EXEC_PERSISTENT is available for RIVER_BF16 only";
      return RIVER_EINVAL;
    }
  } else {
    const dim3 gg(x->grid_gemv);
    for (int l = 0; l < D.L; ++l) {
      k_qkv<DT, V><<<gg, blk, lds, s>>>(Dp, A, l);
      if (DT == 1 && D.kv_f16) k_attn<DT, DT == 1><<<gg, blk, lds, s>>>(Dp, A, l);
      else k_attn<DT, false><<<gg, blk, lds, s>>>(Dp, A, l);
      k_oproj<DT, V><<<gg, blk, lds, s>>>(Dp, A, l);
      k_gateup<DT, V><<<gg, blk, lds, s>>>(Dp, A, l);
      k_down<DT, V><<<gg, blk, lds, s>>>(Dp, A, l);
    }
    if (A.want_head) k_head<DT><<<gg, blk, lds, s>>>(Dp, A);
  }
  HIP_TRY(x, hipGetLastError());
  return RIVER_OK;
}

static int enqueue(river_ctx *x, int token, int forced_e, int want_head, int rec_slot, bool to_host) {
  StepArgs A{};
  A.pos = x->pos;
  A.token = token;
  A.forced_e = forced_e;
  A.want_head = want_head;
  A.rec_slot = rec_slot;
  A.host_row = to_host && x->host ? x->host->rec : nullptr;
  const int T = x->pos + 1;
  // one workgroup per (query head, split); splits as far as there are workgroups for them
  const int max_splits = std::max(1, std::min(kMaxSplits, x->grid_persist / x->cfg.n_q_heads));
  // One split per kAttnPosPerSplit positions up to four splits; every further split costs each
  // consumer another read of all partial outputs, so beyond that a workgroup first takes
  // twice the positions (measured at contexts 768 .. 4096).
  int S = (T + kAttnPosPerSplit - 1) / kAttnPosPerSplit;
  if (S > 4) S = std::max(4, (T + 2 * kAttnPosPerSplit - 1) / (2 * kAttnPosPerSplit));
  A.n_splits = std::max(1, std::min(max_splits, S));
  A.bar_base = 0;
  const bool bf16 = x->cfg.dtype == RIVER_BF16, narrow = !bf16 && narrow_model(x->cfg);
  // (bf16: the one-launch kernel, see step_kernel; its launch-per-phase mode is for debugging)
  const int rc = bf16 ? launch_step<1, 0>(x, A)
                      : (narrow ? launch_step<0, V_NARROW>(x, A) : launch_step<0, 0>(x, A));
  if (rc == RIVER_OK) x->pos += 1;
  return rc;
}

static int device_wait_gave_up(river_ctx *x) {
  x->err = "a device-wide barrier wait exceeded spin_limit; results of the step are invalid";
  x->broken = true;
  return RIVER_EHIP;
}
// Waits for the stream: did a bounded device wait give up?
static int check_device_error(river_ctx *x) {
  int err = 0;
  HIP_TRY(x, hipMemcpyAsync(&err, (char *)x->dev.bar + kBarErrorByte, sizeof(int),
                            hipMemcpyDeviceToHost, x->stream));
  HIP_TRY(x, hipStreamSynchronize(x->stream));
  return err ? device_wait_gave_up(x) : RIVER_OK;
}

#define CHECK_CTX(x)                                   \
  do {                                                 \
    if (!(x)) return RIVER_EINVAL;                     \
    if ((x)->broken) return RIVER_EHIP;                \
  } while (0)

// Tile and number of K slices of a prefill GEMM.  A workgroup's time is its K tiles times what one
// takes, which grows with the share of the chip that is at work (clock, caches): TileM (128 x 128)
// 0.5 .. 0.67 us, and as much again for every further one of its CU; TileN (256 x 128) 0.85 .. 1.15 and
// TileL (256 x 256) 1.4 .. 2.05 us, one workgroup per CU.  K slices cost the write and the read of their
// planes of partial sums (4 MB per us); the one plane of an unsliced matrix is not counted, so slices have
// to win by more than a plane.  The rule takes the least of that over the tiles and up to 16 slices of at
// least four K tiles.  (us measured, the kernel by itself, its planes not yet read, best K slices of
// TileM / TileN / TileL: N 3072 K 2048, 255 rows 10 / 12 / 15; N 6144 K 4096, 512 rows 40 / 36 / 36, and 41
// for TileM unsliced, which the rule takes: 44 in a prefill; N 4096 K 14336, 512 rows 75 / 64 / 64, one
// slice 132 / 187 / 272; N 28672 K 4096, 512 rows 147 / 132 / 114, 4096 rows 1199 / 1144 / 903.)
// Up to kRowsMost rows the tiles are k_pf_gemm_rows', with TileM's count of slices, which is the best one there too (us
// by slices, 77 rows: N 6144 K 4096 3 / 4 / 5 / 6 / 8 of them 17.8 / 15.6 / 14.5 / 21.7 / 20.1; N 4096 K 4096 4 / 6 / 8 / 9
// 15.1 / 12.8 / 13.4 / 17.4; N 4096 K 14336 35.9 / 29.6 / 24.0 / 36.6; taken 5, 8 and 8).  Four blocks of the 8B shape, half of them river, 77
// tokens: 624 us with TileM, 563 with it.  Beyond 128 rows it would take two tiles of rows (us in a prefill, the tiles
// above / two of it): N 3072 K 2048, 255 rows 12.9 / 13.1, N 16384 28.4 / 28.6; N 6144 K 4096, 200 rows 26.9 / 27.2, N 28672
// 72 / 95; with 2 x 96 rows, N 16384 K 2048, 160 rows 26.9 / 23.6, which has not been built.
struct PfTile { int tm, tn; double alone, full; };
constexpr PfTile kPfTiles[3] = {{pf::TileM::TM, pf::TileM::TN, 0.5, 0.67},
                                {pf::TileN::TM, pf::TileN::TN, 0.85, 1.15},
                                {pf::TileL::TM, pf::TileL::TN, 1.4, 2.05}};
struct PfPlan { int tile, split; };
static PfPlan pf_plan(const river_ctx *x, int N, int K, int m, bool may_split) {
  PfPlan best{0, 1};
  double best_us = 1e30;
  const int nk = K / pf::TK, cus = x->grid_persist;
  const bool rows = m <= pf::kRowsMost;
  for (int i = 0; i < (rows ? 1 : 3); ++i) {
    const PfTile &t = kPfTiles[i];
    const long long tiles = (long long)((N + t.tn - 1) / t.tn) * ((m + t.tm - 1) / t.tm);
    for (int sp = 1; sp <= (may_split ? 16 : 1); ++sp) {
      if (sp > 1 && (nk / sp < 4 || (size_t)sp * m * N * 4 > x->lay.pf_big_bytes)) break;
      const double load = (double)(tiles * sp) / cus, whole = std::floor(load), part = load - whole;
      const double k_tile_us = whole * t.full + (part > 0.0 ? t.alone + (t.full - t.alone) * part : 0.0);
      const double us = (nk + sp - 1) / sp * k_tile_us + (sp > 1 ? 2.0 * sp * m * N * 4 / 4e6 : 0.0);
      if (us < best_us) { best_us = us; best = PfPlan{rows ? 3 : i, sp}; }
    }
  }
  return best;
}

// GEMM of the prefill over the stacked matrices ms[0..nm) of block l: fp32 planes of partial sums in
// C (returns how many), or with EPI = PF_SWIGLU the fp16 activation of the down projection.
template <class T, bool W4, int EPI>
static void launch_gemm_t(river_ctx *x, const pf::GemmB &B, int N, const _Float16 *A, int K, void *C, int ldc, int m, int split) {
  const int n_tiles = (N + T::TN - 1) / T::TN, m_tiles = (m + T::TM - 1) / T::TM;
  const dim3 grid((n_tiles * split + 7) / 8 * 8 * m_tiles);      // (see the kernel's workgroup -> tile mapping)
  pf::k_pf_gemm<T, W4, EPI><<<grid, dim3(T::NT), T::LDS_BYTES, x->stream>>>(A, K, B, N, K, x->cfg.river_group, C, ldc, m, m_tiles, split);
}
template <int MB, bool W4, int EPI, bool EXACT = false>
static void launch_rows_t(river_ctx *x, const pf::GemmB &B, int N, const _Float16 *A, int K, void *C, int ldc, int m, int split, int rows32 = 32) {
  typedef pf::RowsTile<MB, W4> T;
  const int n_tiles = (N + T::TN - 1) / T::TN;
  const int stages = (K + T::COLS - 1) / T::COLS;
  const pf::RowsDeal deal{rows32, n_tiles, split, (uint32_t)(((1ull << 32) + split - 1) / split), stages / split, stages % split};
  const dim3 grid((n_tiles * split + 7) / 8 * 8);
  pf::k_pf_gemm_rows<MB, W4, EPI, EXACT><<<grid, dim3(T::NT), T::LDS_BYTES, x->stream>>>(A, K, B, N, K, x->cfg.river_group, C, ldc, m, deal);
}
// the stacked matrices ms[0..nm) of block l; returns their rows
static int gemm_operand(const river_ctx *x, int l, bool w4, const int *ms, int nm, pf::GemmB *B) {
  int N = 0;
  for (int i = 0; i < nm; ++i) {
    long long r, c;
    matrix_shape(&x->cfg, ms[i], &r, &c);
    B->w[i] = w4 ? (const void *)x->layers_h[l].qc[ms[i]] : x->layers_h[l].w[ms[i]];
    B->sz[i] = x->layers_h[l].qsz[ms[i]];
    B->rows[i] = (int)r;
    N += (int)r;
  }
  for (int i = nm; i < 3; ++i) { B->w[i] = B->w[0]; B->sz[i] = B->sz[0]; B->rows[i] = 0; }
  return N;
}
template <int EPI>
static int launch_gemm(river_ctx *x, int l, bool w4, const int *ms, int nm, const _Float16 *A, int K, void *C, int m) {
  pf::GemmB B{};
  const int N = gemm_operand(x, l, w4, ms, nm, &B);
  const PfPlan p = pf_plan(x, N, K, m, EPI == pf::PF_STORE);
  const int ldc = EPI == pf::PF_SWIGLU ? B.rows[0] : N;
  auto launch = [&](auto tile) {
    typedef decltype(tile) T;
    if (w4) launch_gemm_t<T, true, EPI>(x, B, N, A, K, C, ldc, m, p.split);
    else launch_gemm_t<T, false, EPI>(x, B, N, A, K, C, ldc, m, p.split);
  };
  auto rows = [&](auto mb) {
    constexpr int MB = decltype(mb)::value;
    if (w4) launch_rows_t<MB, true, EPI>(x, B, N, A, K, C, ldc, m, p.split);
    else launch_rows_t<MB, false, EPI>(x, B, N, A, K, C, ldc, m, p.split);
  };
  if (p.tile == 3) {
    const int mb = (m + 31) / 32;
    if (mb == 1) rows(IC<1>{});
    else if (mb == 2) rows(IC<2>{});
    else if (mb == 3) rows(IC<3>{});
    else rows(IC<4>{});
  } else if (p.tile == 0) launch(pf::TileM{});
  else if (p.tile == 1) launch(pf::TileN{});
  else launch(pf::TileL{});
  return p.split;
}

// GEMM of a pass over a short prompt (EXACT, see pf::k_pf_gemm_rows): planes of kShort rows in C; returns how many.
static int launch_gemm_exact(river_ctx *x, int l, bool w4, const int *ms, int nm, const _Float16 *A, int K, float *C, int m) {
  pf::GemmB B{};
  const int N = gemm_operand(x, l, w4, ms, nm, &B), M = w4 ? pf::kShort : 3 * pf::kShort;
  const int split = pf_plan(x, N, K, M, true).split;
  if (w4) launch_rows_t<1, true, pf::PF_STORE, true>(x, B, N, A, K, C, N, M, split, m);
  else launch_rows_t<3, false, pf::PF_STORE, true>(x, B, N, A, K, C, N, M, split, m);
  return split * (w4 ? 1 : 3);
}

// Original final norm + LM head + argmax on the last prompt position, the call's results and the new sequence's state (k_pf_head).
// h_row: the position's residual row, parts planes of plane_rows rows behind each other with its sums in row `row`.  More planes than
// kPfHeadPlanes (the single row of a down projection to 2048 columns has up to 16) and wider rows are added up by k_pf_norm in front.
static void launch_prefill_head(river_ctx *x, const float *h_row, const float *planes, int parts, int plane_rows, int row, float *out_logits,
                                int *batch_token) {
  const river_config &c = x->cfg;
  const int d = c.d_model;
  int n_part = parts;
  if (parts > kPfHeadPlanes || d > kPfHeadCols) {               // (every workgroup reads the planes: 16 KB each at the 8B shape)
    // (the norm kernel takes rows that the planes hold from their row 0 on)
    pf::k_pf_norm<false><<<dim3(1), dim3(512), 0, x->stream>>>((float *)h_row, nullptr, x->dev.tok_emb, planes + (size_t)row * d, parts, plane_rows,
                                                               nullptr, d, c.rms_eps, nullptr, x->dev.hidden + (size_t)c.n_layers * d, 0, 0);
    n_part = -1;
  }
  k_pf_head<<<dim3(x->grid_gemv), dim3(x->block), x->lds_bytes, x->stream>>>(x->dev_d, h_row, planes + (size_t)row * d, (size_t)plane_rows * d, n_part,
                                                                             out_logits, x->host ? x->host->rec : nullptr, batch_token);
  x->bar_total = 0;
}

// Short prompts (see river_prefill.h): passes of up to kShort positions, from kShortMin positions on, for models with
// blocks of at least kShortBlockBytes.  us per prompt of 2 / 3 / 31 tokens through the decode kernels, and of
// 3 / 31 in a pass: four 8B blocks, backbone 702 / 1030 / 10317 and 564 / 630, river 426 / 618 / 6036 and 379 / 419;
// three blocks of 72 MB 199 / 287 / 2763 and 233 / 267 (with 128 x 128 tiles 242 / 256), river 166 / 237 / 2246 and 175 / 189; three of 23 MB, by
// 128 x 128 tiles,
// 166 / 237 / 2257 and 202 / 220, river 164 / 235 / 2222 and 184 / 193.  So a pass costs two to three positions at
// every size, and the line in block size is not where passes begin to pay: below it a prompt equals,
// bit for bit, that of a context that never uses GEMMs (prefill_gemm_min_tokens < 0), and only that holds it there.
constexpr int kShortMin = 3;
constexpr size_t kShortBlockBytes = (size_t)64 << 20;
static bool prefill_short_ok(const river_ctx *x, int n) {
  const river_config &c = x->cfg;
  if (x->lay.pf_rows == 0 || n < kShortMin) return false;
  size_t block = 0;
  for (int m = 0; m < 7; ++m) {
    long long r, k;
    matrix_shape(&c, m, &r, &k);
    block += (size_t)(r * k) * 2;
  }
  // (the gate/up GEMM's planes are the largest: three of kShort rows)
  return block >= kShortBlockBytes && (size_t)3 * pf::kShort * 2 * c.d_ffn * 4 <= x->lay.pf_big_bytes;
}
static int prefill_short(river_ctx *x, const int32_t *tokens, int n, int ep, float *out_logits) {
  const river_config &c = x->cfg;
  const Dev &D = x->dev;
  const Layout &y = x->lay;
  hipStream_t s = x->stream;
  const int L = c.n_layers, d = c.d_model, qd = c.n_q_heads * c.head_dim, ffn = c.d_ffn;
  int *tok = (int *)(x->ws + y.pf_tok);
  float *h = (float *)(x->ws + y.pf_h), *big = (float *)(x->ws + y.pf_big);
  _Float16 *x16 = (_Float16 *)(x->ws + y.pf_x16), *q32 = (_Float16 *)(x->ws + y.pf_q16), *a16 = (_Float16 *)(x->ws + y.pf_a16);
  const int m_qkv[3] = {M_WQ, M_WK, M_WV}, m_o[1] = {M_WO}, m_gu[2] = {M_GATE, M_UP}, m_d[1] = {M_DOWN};
  const int rope_wgs = ((c.n_q_heads + c.n_kv_heads) * (c.head_dim / 8) + c.n_kv_heads * c.head_dim / 4 + 255) / 256;   // (see k_pf_rope_store)
  const dim3 blk(512);
  auto attn = c.head_dim == 128 ? pf::k_pf_attn_rows<128> : pf::k_pf_attn_rows<64>;
  for (int c0 = 0; c0 < n; c0 += pf::kShort) {
    const int m = std::min(pf::kShort, n - c0), last = c0 + m == n ? m - 1 : -1;
    const int *tok_src = tok;
    if (x->host && n <= kHostTok) {
      std::memcpy(x->host->tok + c0, tokens + c0, (size_t)m * 4);
      tok_src = x->host->tok + c0;
    } else {
      HIP_TRY(x, hipMemcpyAsync(tok, tokens + c0, (size_t)m * 4, hipMemcpyHostToDevice, s));
    }
    int parts = 0;
    auto norm = [&](bool river, const int *tk, const void *gain, float *row_out, int row) {
      (river ? pf::k_pf_norm<false> : pf::k_pf_norm<true>)<<<dim3(m), blk, 0, s>>>(
          h, tk, D.tok_emb, big, parts, pf::kShort, gain, d, c.rms_eps, gain ? x16 : nullptr, row_out, row, 0);
    };
    for (int l = 0; l < L; ++l) {
      const bool river = l >= ep;
      const DevLayer &W = x->layers_h[l];
      norm(river, l ? nullptr : tok_src, W.attn_norm, D.hidden + (size_t)l * d, last);
      parts = launch_gemm_exact(x, l, river, m_qkv, 3, x16, d, big, m);
      pf::k_pf_rope_store<true><<<dim3(m, rope_wgs), dim3(256), 0, s>>>(big, parts, pf::kShort, D.rope, c.n_q_heads, c.n_kv_heads, c.head_dim, c0, l,
                                                        c.max_seq, D.kcache, D.vcache, D.kv_f16, q32);
      if (l == L - 1 && last < 0) break;                     // (a pass before the last: its keys and values are all that is read)
      attn<<<dim3((c.n_q_heads + 3) / 4, m), dim3(256), 0, s>>>((const float *)q32, D.kcache, D.vcache, D.kv_f16, c.n_q_heads,
                                                                 c.n_kv_heads, l, c.max_seq, c0, !river, x16);
      parts = launch_gemm_exact(x, l, river, m_o, 1, x16, qd, big, m);
      norm(river, nullptr, W.ffn_norm, nullptr, -1);
      parts = launch_gemm_exact(x, l, river, m_gu, 2, x16, d, big, m);
      pf::k_pf_swiglu_rows<<<dim3((ffn + 2047) / 2048, m), dim3(256), 0, s>>>(big, parts, ffn, !river, a16);
      parts = launch_gemm_exact(x, l, river, m_d, 1, a16, ffn, big, m);
    }
    if (last >= 0) launch_prefill_head(x, h + (size_t)last * d, big, parts, pf::kShort, last, out_logits, nullptr);
    HIP_TRY(x, hipGetLastError());
  }
  HIP_TRY(x, hipGetLastError());
  x->pos = n;
  return RIVER_OK;
}

// Attention of a chunk's queries: as many query heads of a kv head per workgroup (4, 2 or 1) as divide them, two tiles of
// keys a step where one a step makes no more workgroups than there are CUs (us in a prefill, one / two tiles, 32 heads on 8 of head
// size 128: 77 rows 10.6 / 9.7, 512 28.9 / 20.2, 1024 46 / 33, 2048 89 / 69, beyond the line 2560 98 to 113 / 106 to
// 109; 8 on 2: 3072 rows 110 / 74, a prompt of 8300 in three chunks and two blocks as a whole 1025 / 856).  Keys and values of the
// next block are as far from 64 bits either way: 1.77e-3 of 3072 positions, 1.70e-3 of 8300 (their rounding to bf16).
template <int HD, int HG>
static void launch_attn_t(river_ctx *x, int l, const void *kc, const void *vc, int c0, int m, const _Float16 *q16, _Float16 *o16) {
  const river_config &c = x->cfg;
  auto go = [&](auto ks) {
    constexpr int KS = decltype(ks)::value, QT = 256 / HG / KS;
    pf::k_pf_attn<HD, HG, KS><<<dim3(c.n_q_heads / HG, (m + QT - 1) / QT), dim3(512), pf::attn_lds_bytes(HD, KS), x->stream>>>(
        q16, kc, vc, x->dev.kv_f16, c.n_q_heads, c.n_kv_heads, l, c.max_seq, c0, m, o16);
  };
  const int wgs = c.n_q_heads / HG * ((m + 256 / HG - 1) / (256 / HG));
  if (wgs <= x->grid_persist) go(IC<2>{});
  else go(IC<1>{});
}
static int heads_per_group(const river_config &c) {
  const int rep = c.n_q_heads / c.n_kv_heads;
  return rep % 4 == 0 ? 4 : rep % 2 == 0 ? 2 : 1;
}
static void launch_attn(river_ctx *x, int l, const void *kc, const void *vc, int c0, int m, const _Float16 *q16, _Float16 *o16) {
  const int hg = heads_per_group(x->cfg);
  auto f = x->cfg.head_dim == 128 ? (hg == 4 ? launch_attn_t<128, 4> : hg == 2 ? launch_attn_t<128, 2> : launch_attn_t<128, 1>)
                                  : (hg == 4 ? launch_attn_t<64, 4> : hg == 2 ? launch_attn_t<64, 2> : launch_attn_t<64, 1>);
  f(x, l, kc, vc, c0, m, q16, o16);
}
// ... and of the last position P alone, in splits of at least 128 positions
static void launch_attn_last(river_ctx *x, int l, const void *kc, const void *vc, int P, const _Float16 *q16, _Float16 *o16) {
  const river_config &c = x->cfg;
  const int hg = heads_per_group(c), splits = std::min(kMaxSplits, (P + 128) / 128);
  auto k = c.head_dim == 128 ? (hg == 4 ? pf::k_pf_attn_last<128, 4> : hg == 2 ? pf::k_pf_attn_last<128, 2> : pf::k_pf_attn_last<128, 1>)
                             : (hg == 4 ? pf::k_pf_attn_last<64, 4> : hg == 2 ? pf::k_pf_attn_last<64, 2> : pf::k_pf_attn_last<64, 1>);
  k<<<dim3(c.n_q_heads / hg, splits), dim3(256 * hg), 0, x->stream>>>(q16, kc, vc, x->dev.kv_f16, c.n_q_heads, c.n_kv_heads, l, c.max_seq, P,
                                                                splits, x->dev.part_o, x->dev.part_ml, o16);
}

// Prefill phase on the matrix cores: the prompt in equal chunks of up to pf_rows tokens, every block
// as MFMA GEMMs over the chunk (see river_prefill.h); blocks above ep run as river twins.
static int prefill_gemm(river_ctx *x, int seq, const int32_t *tokens, int n, int ep, float *out_logits) {
  const river_config &c = x->cfg;
  const Dev &D = x->dev;
  const Layout &y = x->lay;
  hipStream_t s = x->stream;
  const int L = c.n_layers, d = c.d_model, qd = c.n_q_heads * c.head_dim, ffn = c.d_ffn;
  int *tok = (int *)(x->ws + y.pf_tok);
  float *h = (float *)(x->ws + y.pf_h), *big = (float *)(x->ws + y.pf_big);
  _Float16 *x16 = (_Float16 *)(x->ws + y.pf_x16), *q16 = (_Float16 *)(x->ws + y.pf_q16);
  _Float16 *a16 = (_Float16 *)(x->ws + y.pf_a16);
  char *kc = (char *)D.kcache + (size_t)seq * y.cache_bytes, *vc = (char *)D.vcache + (size_t)seq * y.cache_bytes;
  const int m_qkv[3] = {M_WQ, M_WK, M_WV}, m_o[1] = {M_WO}, m_gu[2] = {M_GATE, M_UP}, m_d[1] = {M_DOWN};
  const int rope_wgs = ((c.n_q_heads + c.n_kv_heads) * (c.head_dim / 8) + c.n_kv_heads * c.head_dim / 4 + 255) / 256;   // (see k_pf_rope_store)
  const int chunks = (n + y.pf_rows - 1) / y.pf_rows, step = std::min(y.pf_rows, ((n + chunks - 1) / chunks + 255) / 256 * 256);
  for (int c0 = 0; c0 < n; c0 += step) {
    const int m = std::min(step, n - c0);
    const int last = c0 + m == n ? m - 1 : -1;              // the row whose h(0..L) is kept
    const int *tok_src = tok;
    if (x->host && n <= kHostTok) {      // (the call waits for the stream: the slot is free)
      std::memcpy(x->host->tok + c0, tokens + c0, (size_t)m * 4);
      tok_src = x->host->tok + c0;
    } else {
      HIP_TRY(x, hipMemcpyAsync(tok, tokens + c0, (size_t)m * 4, hipMemcpyHostToDevice, s));
    }
    const dim3 rowwise(m <= 2 * x->grid_persist ? 512 : 256);
    int parts = 0;                                           // partial sums waiting to be added into h
    for (int l = 0; l < L; ++l) {
      const bool river = l >= ep;
      const DevLayer &W = x->layers_h[l];
      pf::k_pf_norm<false><<<dim3(m), rowwise, 0, s>>>(h, l ? nullptr : tok_src, D.tok_emb, big, parts, m, W.attn_norm, d, c.rms_eps, x16,
                                                D.hidden + (size_t)l * d, last, 0);
      parts = launch_gemm<pf::PF_STORE>(x, l, river, m_qkv, 3, x16, d, big, m);
      pf::k_pf_rope_store<false><<<dim3(m, rope_wgs), dim3(256), 0, s>>>(big, parts, m, D.rope, c.n_q_heads, c.n_kv_heads, c.head_dim, c0, l,
                                                      c.max_seq, kc, vc, D.kv_f16, q16);
      // Behind the last block's keys and values only the last prompt position goes on (its h(L) is the
      // head's input, nobody reads the others'): from there on the last block is one row of the last
      // chunk -- unless the chunk is one row tile anyway, which a single row does not make faster.  One of
      // four blocks at the 8B shape, 4096 tokens: 1.4 ms of GEMMs become 0.1 ms (77 tokens: 3 % slower).
      const bool tail = l == L - 1 && m > pf::TileM::TM;
      if (l == L - 1 && last < 0) break;
      const int t0 = tail ? last : 0, rows = tail ? 1 : m;
      if (tail) launch_attn_last(x, l, kc, vc, c0 + last, q16 + (size_t)last * qd, x16 + (size_t)last * qd);
      else launch_attn(x, l, kc, vc, c0, m, q16, x16);
      parts = launch_gemm<pf::PF_STORE>(x, l, river, m_o, 1, x16 + (size_t)t0 * qd, qd, big, rows);
      pf::k_pf_norm<false><<<dim3(rows), rowwise, 0, s>>>(h, nullptr, nullptr, big, parts, rows, W.ffn_norm, d, c.rms_eps, x16, nullptr, -1, t0);
      (void)launch_gemm<pf::PF_SWIGLU>(x, l, river, m_gu, 2, x16 + (size_t)t0 * d, d, a16, rows);
      parts = launch_gemm<pf::PF_STORE>(x, l, river, m_d, 1, a16, ffn, big, rows);
    }
    if (last >= 0) {
      const bool tail = m > pf::TileM::TM;
      launch_prefill_head(x, h + (size_t)last * d, big, parts, tail ? 1 : m, tail ? 0 : last, out_logits, c.max_batch > 1 ? x->st_b.token + seq : nullptr);
    }
    HIP_TRY(x, hipGetLastError());
  }
  if (c.max_batch > 1) x->pos_b[seq] = n;
  else x->pos = n;
  return RIVER_OK;
}

// Are `bytes` bytes from p memory of the current device that one allocation holds?
static bool device_memory(const void *p, size_t bytes) {
  hipPointerAttribute_t at;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice || at.device != dev ||
      hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess)
    return false;
  const size_t before = (size_t)((const char *)p - (const char *)base);
  return before <= size && bytes <= size - before;
}

extern "C" int river_prefill(river_ctx *x, int32_t seq, const int32_t *tokens, int32_t n_tokens,
                             int32_t prefill_exit_layer, int32_t *out_token, float *out_logits) {
  if (!x) return RIVER_EINVAL;
  if (seq < 0 || seq >= x->cfg.max_batch || !tokens || n_tokens < 1) {
    x->err = "bad prefill arguments";
    return RIVER_EINVAL;
  }
  if (n_tokens > x->cfg.max_seq) { x->err = "prompt longer than max_seq"; return RIVER_ENOSPC; }
  for (int i = 0; i < n_tokens; ++i)
    if (tokens[i] < 0 || tokens[i] >= x->cfg.vocab) { x->err = "token id out of range"; return RIVER_EINVAL; }
  const int L = x->cfg.n_layers;
  const int ep = prefill_exit_layer < 0 ? L : prefill_exit_layer;
  if (ep != L && (ep < x->cfg.min_exit_layer || ep > L)) {
    x->err = "prefill exit layer outside [L_s, L]";
    return RIVER_EINVAL;
  }
  if (ep < L && !x->have_river) { x->err = "prefill below full depth needs river weights"; return RIVER_ESTATE; }
  // a new sequence also clears a previous device-side time-out
  x->broken = false;
  int rc;
  x->pos = 0;
  x->have_token = false;
  const int min_gemm = x->cfg.prefill_gemm_min_tokens > 0 ? x->cfg.prefill_gemm_min_tokens : 32;
  // the head's kernel stores the logits where the caller wants them if all of that is this device's memory (else a copy, which
  // refuses what it cannot write; a kernel would fault)
  float *direct = nullptr;
  if (out_logits) {
    const hipError_t pending = hipPeekAtLastError();
    if (device_memory(out_logits, (size_t)x->cfg.vocab * 4) && (uintptr_t)out_logits % 4 == 0) direct = out_logits;
    else if (pending == hipSuccess) (void)hipGetLastError();     // (the look's own error, not one that was there before)
  }
  if (x->lay.pf_rows > 0 && (n_tokens >= min_gemm || x->cfg.max_batch > 1)) {
    rc = prefill_gemm(x, seq, tokens, n_tokens, ep, direct);
    if (rc) return rc;
  } else if (prefill_short_ok(x, n_tokens)) {
    rc = prefill_short(x, tokens, n_tokens, ep, direct);
    if (rc) return rc;
  } else {
    // one or two tokens, fp32 models and shapes the GEMM path does not take: the decode kernels,
    // one prompt position after the other
    direct = nullptr;
    rc = reset_state(x);
    if (rc) return rc;
    for (int i = 0; i < n_tokens; ++i) {
      rc = enqueue(x, tokens[i], ep, i == n_tokens - 1, -1, i == n_tokens - 1);
      if (rc) return rc;
    }
  }
  if (out_logits && !direct)
    HIP_TRY(x, hipMemcpyAsync(out_logits, x->dev.logits, (size_t)x->cfg.vocab * 4, hipMemcpyDeviceToDevice,
                              x->stream));
  if (x->host) {
    HIP_TRY(x, hipStreamSynchronize(x->stream));
    if (x->host->rec[1] & kRecErrorBit) return device_wait_gave_up(x);
    x->have_token = true;
    if (out_token) *out_token = x->host->rec[0];
    return RIVER_OK;
  }
  rc = check_device_error(x);
  if (rc) return rc;
  x->have_token = true;
  if (out_token) {
    HIP_TRY(x, hipMemcpyAsync(out_token, (char *)x->dev.st + offsetof(DevState, cur_token), sizeof(int),
                              hipMemcpyDeviceToHost, x->stream));
    HIP_TRY(x, hipStreamSynchronize(x->stream));
  }
  return RIVER_OK;
}

extern "C" int river_decode_step(river_ctx *x, const int32_t *in_token, const int32_t *forced_exit,
                                 int32_t *out_token, int32_t *out_exit_layer, float *out_sims) {
  CHECK_CTX(x);
  if (x->cfg.max_batch > 1) { x->err = "a batched context decodes with river_decode_batch"; return RIVER_ESTATE; }
  if (!x->have_token && !in_token) { x->err = "decode before prefill"; return RIVER_ESTATE; }
  if (x->pos < 1) { x->err = "decode before prefill"; return RIVER_ESTATE; }
  if (x->pos >= x->cfg.max_seq) { x->err = "KV cache full"; return RIVER_ENOSPC; }
  const int L = x->cfg.n_layers;
  int tok = -1, fe = -1;
  if (in_token) {
    tok = *in_token;
    if (tok < 0 || tok >= x->cfg.vocab) { x->err = "token id out of range"; return RIVER_EINVAL; }
  }
  if (forced_exit) {
    fe = *forced_exit;
    const bool ok = fe == L || (fe >= x->cfg.min_exit_layer && fe <= L && fe >= 0);
    if (!ok) { x->err = "forced exit position outside [L_s, L]"; return RIVER_EINVAL; }
  }
  if ((fe >= 0 && fe < L) || (fe < 0 && x->cfg.tau < 1.0f)) {
    if (!x->have_river) { x->err = "an exit is possible but no river weights were given"; return RIVER_ESTATE; }
  }
  if (!out_token && (out_exit_layer || out_sims)) {
    x->err = "out_token is NULL but other outputs are not";
    return RIVER_EINVAL;
  }
  const int slot = (int)(x->steps % kRecords);
  int rc = enqueue(x, tok, fe, 1, slot, out_token != nullptr);
  if (rc) return rc;
  x->steps += 1;
  x->have_token = true;
  if (!out_token) return RIVER_OK;
  // the step's record, the device's error flag with it: written to the host by the step, or in one copy
  const size_t row = (size_t)kRecHead + L;
  const int32_t *rec;
  if (x->host) {
    rec = x->host->rec;
  } else {
    x->rec_h.resize(row);
    HIP_TRY(x, hipMemcpyAsync(x->rec_h.data(), x->dev.rec + slot * row, row * 4, hipMemcpyDeviceToHost, x->stream));
    rec = x->rec_h.data();
  }
  HIP_TRY(x, hipStreamSynchronize(x->stream));
  *out_token = rec[0];
  if (out_exit_layer) *out_exit_layer = rec[1] & ~kRecErrorBit;
  if (out_sims) std::memcpy(out_sims, rec + kRecHead, (size_t)L * 4);
  return rec[1] & kRecErrorBit ? device_wait_gave_up(x) : RIVER_OK;
}

// GEMM g (QKV, O, gate/up, down) of block l of a batched decode step, or the LM head (Bq null,
// sides = kSideDense): bf16 matrices for the rows in the backbone, 4-bit twins for the others (see
// bd::k_bd_gemm).  The rows of B are dealt out to one workgroup per CU, eight at a time.
static int launch_bd_gemm_b(river_ctx *x, const bd::BdB &Bd, const bd::BdB &Bq, int N, const _Float16 *Af, int K,
                            void *C, int ldc, int epi, int sides, int n, bd::BdNorm nrm = bd::BdNorm{},
                            int *grid_out = nullptr) {
  // A matrix with at most 16 rows per CU (the down projection; the output projection, which also
  // prepares the next norm, stays whole) would have every workgroup
  // read the whole activation tile for a single row block; it is dealt out as K slices of four
  // times the rows instead, and the kernel that consumes the sum adds the partial sums up.
  int k_split = 1;
  if (epi == bd::EPI_ADD && N <= 16 * x->grid_persist && K >= 4096 && ldc == x->cfg.d_model) k_split = bd::kBdKSplit;
  // (the consumer of a fused norm adds up at most 16 * kSsqLoads partial sums per row)
  const int cus = epi == bd::EPI_ADD_NORM ? std::min(x->grid_persist, 16 * bd::kSsqLoads) : x->grid_persist;
  const int per_cu = (N * k_split + cus - 1) / cus;
  const int rows_per_wg = std::max(8, (per_cu + 7) / 8 * 8);
  const int blocks = (rows_per_wg + 15) / 16;
  const dim3 grid((N + rows_per_wg - 1) / rows_per_wg * k_split), blk(512);
  if (grid_out) *grid_out = (int)grid.x;
  hipStream_t s = x->stream;
  const int *rv = x->st_b.river;
  if (k_split > 1) { C = x->ws + x->lay.bd_partial; epi = bd::EPI_STORE; }
#define RIVER_BD_LAUNCH(MB, RBW)                                                                               \
  bd::k_bd_gemm<MB, RBW><<<grid, blk, bd::bd_gemm_lds_bytes(RBW, MB), s>>>(Af, Bd, Bq, N, K, C, ldc, epi, rv, \
                                                                          sides, n, rows_per_wg, k_split, nrm)
  if (n <= 16) {
    if (blocks <= 1) RIVER_BD_LAUNCH(1, 1);
    else if (blocks <= 2) RIVER_BD_LAUNCH(1, 2);
    else if (blocks <= 4) RIVER_BD_LAUNCH(1, 4);
    else RIVER_BD_LAUNCH(1, 8);
  } else {
    if (blocks <= 1) RIVER_BD_LAUNCH(2, 1);
    else if (blocks <= 2) RIVER_BD_LAUNCH(2, 2);
    else RIVER_BD_LAUNCH(2, 4);
  }
#undef RIVER_BD_LAUNCH
  return k_split > 1 ? k_split : 0;          // partial sums the consumer has to add
}
static int launch_bd_gemm(river_ctx *x, int l, int g, int sides, const _Float16 *Af, void *C, int ldc, int epi, int n,
                          bd::BdNorm nrm = bd::BdNorm{}, int *grid_out = nullptr) {
  const BdGemmShape sh = bd_gemm_shape(&x->cfg, g);
  return launch_bd_gemm_b(x, x->bd_dense_h[(size_t)l * 4 + g], x->bd_twin_h[(size_t)l * 4 + g], sh.N, Af, sh.K, C, ldc,
                          epi, sides, n, nrm, grid_out);
}

extern "C" int river_decode_batch(river_ctx *x, int32_t n_seq, const int32_t *in_tokens, const int32_t *forced_exit,
                                  int32_t *out_tokens, int32_t *out_exit_layers, float *out_sims) {
  CHECK_CTX(x);
  const river_config &c = x->cfg;
  if (c.max_batch < 2) { x->err = "river_decode_batch needs a context created with max_batch > 1"; return RIVER_ESTATE; }
  if (n_seq < 1 || n_seq > c.max_batch) { x->err = "n_seq outside [1, max_batch]"; return RIVER_EINVAL; }
  if (!out_tokens && (out_exit_layers || out_sims)) {
    x->err = "out_tokens is NULL but other outputs are not";
    return RIVER_EINVAL;
  }
  const int L = c.n_layers, n = n_seq;
  bd::StepIn in{};
  int *const fe = in.forced;
  for (int b = 0; b < n; ++b) {
    in.pos[b] = x->pos_b[b];
    in.token[b] = in_tokens ? in_tokens[b] : -1;
    fe[b] = -1;
    if (x->pos_b[b] < 1) { x->err = "decode before prefill of every sequence"; return RIVER_ESTATE; }
    if (x->pos_b[b] >= c.max_seq) { x->err = "KV cache full"; return RIVER_ENOSPC; }
    if (in_tokens && (in_tokens[b] < 0 || in_tokens[b] >= c.vocab)) { x->err = "token id out of range"; return RIVER_EINVAL; }
    if (forced_exit) {
      fe[b] = forced_exit[b];
      const bool ok = fe[b] < 0 || fe[b] == L || (fe[b] >= c.min_exit_layer && fe[b] <= L);
      if (!ok) { x->err = "forced exit position outside [L_s, L]"; return RIVER_EINVAL; }
    }
    if (((fe[b] >= 0 && fe[b] < L) || (fe[b] < 0 && c.tau < 1.0f)) && !x->have_river) {
      x->err = "an exit is possible but no river weights were given";
      return RIVER_ESTATE;
    }
  }
  const Dev &D = x->dev;
  const Layout &y = x->lay;
  hipStream_t s = x->stream;
  const int d = c.d_model, qd = c.n_q_heads * c.head_dim, ffn = c.d_ffn;
  float *h = (float *)(x->ws + y.pf_h), *big = (float *)(x->ws + y.pf_big);
  float *hprev = (float *)(x->ws + y.bd_hprev);
  float *part_o = (float *)(x->ws + y.bd_part_o), *part_ml = (float *)(x->ws + y.bd_part_ml);
  unsigned int *tickets = (unsigned int *)(x->ws + y.bd_tickets);
  const float *partial = (const float *)(x->ws + y.bd_partial);
  float *logits = (float *)(x->ws + y.bd_logits), *hist = (float *)(x->ws + y.bd_hist);
  _Float16 *x16 = (_Float16 *)(x->ws + y.pf_x16), *o16 = (_Float16 *)(x->ws + y.pf_q16);
  _Float16 *a16 = (_Float16 *)(x->ws + y.pf_a16);
  const int slot = (int)(x->steps_b % bd::kRecordsB);
  const size_t B = c.max_batch;
  int *const rec_token = (int *)(x->ws + y.bd_rec) + (size_t)slot * B * (2 + L), *const rec_exit = rec_token + B;
  float *const rec_sims = (float *)(rec_exit + B);
  const bd::SeqState st = x->st_b;
  float *s_of = (float *)(st.forced + B);                    // [max_batch] similarities of the current block
  // the sequences' state, h(0), and the norm in front of block 1's QKV GEMM (the other norms: the
  // previous block's last kernel)
  bd::k_bd_begin<<<dim3(n), dim3(256), 0, s>>>(in, st, D.tok_emb, d, c.vocab, L, h, hprev, hist, rec_sims,
                                               x->layers_h[0].attn_norm, c.rms_eps, x16);
  const size_t seq_stride = y.cache_bytes / 2;               // elements (bf16)
  // attention: one workgroup per (sequence, kv head, group of query heads, split of the positions);
  // splits so that every CU has two workgroups (measured best) of at least 128 positions, or 256 where half the
  // CUs have one without: a split more is a merge behind another workgroup's publication, about as long as two
  // batches of 64 positions (128 / 256, 8 steps of four blocks: 8B, 32 sequences at 200 positions 4249 / 4154 us; 1B, 16
  // at 400 2428 / 2400; mid-size shape, 8 at 200, 16 workgroups unsplit: 1669 / 1692)
  const int rep = c.n_q_heads / c.n_kv_heads, arep = rep % 4 == 0 ? 4 : 1;
  int t_max = 1;
  for (int b = 0; b < n; ++b) t_max = std::max(t_max, x->pos_b[b] + 1);
  const int hgs = rep / arep, groups = n * c.n_kv_heads * hgs;
  const int per_split = 2 * groups >= x->grid_persist ? 256 : 128;
  int n_splits = (2 * x->grid_persist + groups - 1) / groups;
  n_splits = std::max(1, std::min({n_splits, bd::kBdAttnMaxSplits, (t_max + per_split - 1) / per_split}));
  const size_t attn_lds = bd::bd_attn_lds_bytes(arep, c.head_dim);
  const int qkv_ld = qd + 2 * c.n_kv_heads * c.head_dim;
  for (int l = 0; l < L; ++l) {
    const DevLayer &W = x->layers_h[l];
    // Which weight sets have rows in this block, where it does not depend on the step's similarities:
    // forced exits, thresholds that never fire, blocks in front of the first exit test (else 0).  The
    // GEMMs then start their weight stream without looking at the rows' flags first (1.4 us each).
    int sides = 0;
    for (int b = 0; b < n && sides >= 0; ++b) {
      if (fe[b] >= 0) sides |= l >= fe[b] ? bd::kSideTwin : bd::kSideDense;
      else if (c.tau >= 1.0f || l < std::max(c.min_exit_layer, 1)) sides |= bd::kSideDense;
      else sides = -1;
    }
    sides = std::max(sides, 0);
    launch_bd_gemm(x, l, 0, sides, x16, big, qkv_ld, bd::EPI_STORE, n);
    {
      const dim3 ga((n * c.n_kv_heads * n_splits + 7) / 8 * 8 * hgs);
      auto attn = c.head_dim == 128
                      ? (arep == 4 ? (D.kv_f16 ? bd::k_bd_attn<128, true, 4> : bd::k_bd_attn<128, false, 4>)
                                   : (D.kv_f16 ? bd::k_bd_attn<128, true, 1> : bd::k_bd_attn<128, false, 1>))
                      : (arep == 4 ? (D.kv_f16 ? bd::k_bd_attn<64, true, 4> : bd::k_bd_attn<64, false, 4>)
                                   : (D.kv_f16 ? bd::k_bd_attn<64, true, 1> : bd::k_bd_attn<64, false, 1>));
      attn<<<ga, dim3(256), attn_lds, s>>>(big, D.rope, D.kcache, D.vcache, c.n_q_heads, c.n_kv_heads, n, l, c.max_seq,
                                           seq_stride, st.pos, n_splits, part_o, part_ml, tickets, o16);
    }
    // The output projection completes h; the norm in front of gate/up rides on the two GEMMs:
    // fp16(h * gain) and the rows' partial sums of squares from the first, 1 / rms applied by the
    // second (see bd::BdNorm).
    float *ssq = (float *)(x->ws + y.bd_ssq);
    int o_grid = 0;
    launch_bd_gemm(x, l, 1, sides, o16, h, d, bd::EPI_ADD_NORM, n, bd::BdNorm{W.ffn_norm, x16, ssq, nullptr, 0, 0, 0.f}, &o_grid);
    // gate and up rows interleaved, SwiGLU in the epilogue: the down projection's input as fp16
    launch_bd_gemm(x, l, 2, sides, x16, a16, ffn, bd::EPI_SWIGLU, n, bd::BdNorm{nullptr, nullptr, nullptr, ssq, o_grid, d, c.rms_eps});
    const int pd = launch_bd_gemm(x, l, 3, sides, a16, h, d, bd::EPI_ADD, n);
    // similarity, the sequences' own exit decisions, and the norm in front of the next GEMM
    const bool may_exit = l + 1 >= c.min_exit_layer && l + 1 < L;
    const bool batch_rule = c.batch_exit_rule == 1;
    bd::k_bd_block_end<<<dim3(n), dim3(512), 0, s>>>(hprev, h, d, l + 1, L, st, s_of, rec_sims,
                                                     hist + (size_t)(l + 1) * B * d, may_exit && !batch_rule, c.tau,
                                                     l + 1 < L ? x->layers_h[l + 1].attn_norm : D.final_norm,
                                                     c.rms_eps, x16, partial, pd);
    if (may_exit && batch_rule)
      bd::k_bd_decide<<<dim3(1), dim3(64), 0, s>>>(n, l + 1, L, c.min_exit_layer, c.tau, c.batch_exit_rule, st, s_of);
  }
  // the original LM head (its input is already normalised), greedy token per sequence
  launch_bd_gemm_b(x, x->bd_head, x->bd_head, c.vocab, x16, d, logits, c.vocab, bd::EPI_STORE, bd::kSideDense, n);
  // (the attention kernels are done with their partial-result area and tickets)
  bd::k_bd_argmax<<<dim3(n * bd::kBdArgmaxChunks), dim3(256), 0, s>>>(logits, c.vocab, st, rec_token, rec_exit, part_ml, tickets,
                                                                               out_tokens && x->host ? x->host->rec : nullptr, (int)B, rec_sims, L);
  HIP_TRY(x, hipGetLastError());
  for (int b = 0; b < n; ++b) x->pos_b[b] += 1;
  x->steps_b += 1;
  x->last_n = n;
  if (!out_tokens) return RIVER_OK;
  const int32_t *rec;
  if (x->host) {
    rec = x->host->rec;
  } else {
    x->rec_h.resize(B * (2 + L));
    HIP_TRY(x, hipMemcpyAsync(x->rec_h.data(), rec_token, (out_sims ? B * 2 + (size_t)n * L : B + n) * 4, hipMemcpyDeviceToHost, s));
    rec = x->rec_h.data();
  }
  HIP_TRY(x, hipStreamSynchronize(s));
  std::memcpy(out_tokens, rec, (size_t)n * 4);
  if (out_exit_layers) std::memcpy(out_exit_layers, rec + B, (size_t)n * 4);
  if (out_sims) std::memcpy(out_sims, rec + 2 * B, (size_t)n * L * 4);
  return RIVER_OK;
}

extern "C" int river_read_batch_records(river_ctx *x, int32_t n_steps, int32_t n_seq, int32_t *tokens,
                                        int32_t *exit_layers) {
  CHECK_CTX(x);
  if (x->cfg.max_batch < 2 || n_steps < 0 || n_steps > bd::kRecordsB || n_steps > x->steps_b || n_seq < 1 ||
      n_seq > x->cfg.max_batch || (n_steps > 0 && (!tokens || !exit_layers))) {
    x->err = "bad batch record request";
    return RIVER_EINVAL;
  }
  const size_t B = x->cfg.max_batch, row = B * (2 + (size_t)x->cfg.n_layers);
  std::vector<int32_t> rows(2 * B * (size_t)n_steps);         // tokens and exits of a step are neighbours
  for (int i = 0; i < n_steps; ++i) {
    const size_t slot = (size_t)((x->steps_b - n_steps + i) % bd::kRecordsB);
    HIP_TRY(x, hipMemcpyAsync(rows.data() + 2 * B * i, (int *)(x->ws + x->lay.bd_rec) + slot * row, 2 * B * 4,
                              hipMemcpyDeviceToHost, x->stream));
  }
  HIP_TRY(x, hipStreamSynchronize(x->stream));
  for (int i = 0; i < n_steps; ++i) {
    std::memcpy(tokens + (size_t)i * n_seq, rows.data() + 2 * B * i, (size_t)n_seq * 4);
    std::memcpy(exit_layers + (size_t)i * n_seq, rows.data() + 2 * B * i + B, (size_t)n_seq * 4);
  }
  return RIVER_OK;
}

extern "C" int river_read_records(river_ctx *x, int32_t n, int32_t *tokens, int32_t *exit_layers,
                                  float *sims) {
  CHECK_CTX(x);
  if (n < 0 || n > kRecords || n > x->steps || (n > 0 && (!tokens || !exit_layers))) {
    x->err = "bad record count";
    return RIVER_EINVAL;
  }
  int rc = check_device_error(x);
  if (rc) return rc;
  // the ring's rows in at most two copies
  const size_t row = (size_t)kRecHead + x->cfg.n_layers;
  std::vector<int32_t> rows(row * (size_t)n);
  const int first = n ? (int)((x->steps - n) % kRecords) : 0, n0 = std::min(n, kRecords - first);
  if (n0 > 0) HIP_TRY(x, hipMemcpyAsync(rows.data(), x->dev.rec + first * row, n0 * row * 4, hipMemcpyDeviceToHost, x->stream));
  if (n > n0) HIP_TRY(x, hipMemcpyAsync(rows.data() + n0 * row, x->dev.rec, (n - n0) * row * 4, hipMemcpyDeviceToHost, x->stream));
  HIP_TRY(x, hipStreamSynchronize(x->stream));
  for (int i = 0; i < n; ++i) {
    tokens[i] = rows[i * row];
    exit_layers[i] = rows[i * row + 1] & ~kRecErrorBit;
    if (sims) std::memcpy(sims + (size_t)i * x->cfg.n_layers, rows.data() + i * row + kRecHead, (size_t)x->cfg.n_layers * 4);
  }
  return RIVER_OK;
}

extern "C" int river_rewind(river_ctx *x, int32_t seq, int32_t new_len) {
  CHECK_CTX(x);
  if (x->cfg.max_batch > 1) {
    if (seq < 0 || seq >= x->cfg.max_batch || new_len < 0 || new_len > x->pos_b[seq]) {
      x->err = "bad rewind length";
      return RIVER_EINVAL;
    }
    x->pos_b[seq] = new_len;                                  // (the next step is told)
    return RIVER_OK;
  }
  if (seq != 0 || new_len < 0 || new_len > x->pos) { x->err = "bad rewind length"; return RIVER_EINVAL; }
  x->pos = new_len;
  return RIVER_OK;
}

extern "C" int river_position(const river_ctx *x) { return x ? x->pos : RIVER_EINVAL; }
extern "C" int river_seq_position(const river_ctx *x, int32_t seq) {
  if (!x || seq < 0 || seq >= x->cfg.max_batch) return RIVER_EINVAL;
  return x->cfg.max_batch > 1 ? x->pos_b[seq] : x->pos;
}

extern "C" int river_get_debug(river_ctx *x, int32_t what, void *dst, size_t bytes) {
  if (!x || !dst) return RIVER_EINVAL;
  const char *src = nullptr;
  size_t n = 0;
  switch (what) {
    case RIVER_DBG_HIDDEN: src = (const char *)x->dev.hidden; n = (size_t)(x->cfg.n_layers + 1) * x->cfg.d_model * 4; break;
    case RIVER_DBG_LOGITS: src = (const char *)x->dev.logits; n = (size_t)x->cfg.vocab * 4; break;
    case RIVER_DBG_KCACHE: src = (const char *)x->dev.kcache; n = x->lay.cache_bytes * x->cfg.max_batch; break;
    case RIVER_DBG_VCACHE: src = (const char *)x->dev.vcache; n = x->lay.cache_bytes * x->cfg.max_batch; break;
    case RIVER_DBG_BATCH_HIDDEN:
      if (x->cfg.max_batch < 2) { x->err = "not a batched context"; return RIVER_EINVAL; }
      src = x->ws + x->lay.bd_hist;
      n = (size_t)(x->cfg.n_layers + 1) * x->cfg.max_batch * x->cfg.d_model * 4;
      break;
    case RIVER_DBG_BATCH_LOGITS:
      if (x->cfg.max_batch < 2) { x->err = "not a batched context"; return RIVER_EINVAL; }
      src = x->ws + x->lay.bd_logits;
      n = (size_t)x->cfg.max_batch * x->cfg.vocab * 4;
      break;
    case RIVER_DBG_TRACE: src = (const char *)x->dev.trace; n = ((size_t)5 * x->cfg.n_layers * 2 * x->grid_persist + 64) * 8; break;
    default: x->err = "unknown debug buffer"; return RIVER_EINVAL;
  }
  if (bytes != n) { x->err = "debug buffer size mismatch"; return RIVER_EINVAL; }
  HIP_TRY(x, hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, x->stream));
  HIP_TRY(x, hipStreamSynchronize(x->stream));
  return RIVER_OK;
}

extern "C" int river_fill_cache(river_ctx *x, int32_t value) {
  CHECK_CTX(x);
  const uint32_t b = (uint32_t)value & 0xffu;
  const uint32_t word = b | (b << 8) | (b << 16) | (b << 24);
  const size_t n16 = (x->lay.vcache - x->lay.kcache + align_up(x->lay.cache_bytes * x->cfg.max_batch, 256)) / 16;
  k_fill_bytes<<<dim3(1024), dim3(256), 0, x->stream>>>((uint4 *)x->dev.kcache, n16, word);
  HIP_TRY(x, hipGetLastError());
  return RIVER_OK;
}

extern "C" const char *river_last_error(const river_ctx *x) {
  return x ? x->err.c_str() : g_create_err.c_str();
}

extern "C" int river_destroy(river_ctx *x) {
  if (!x) return RIVER_OK;
  (void)hipStreamSynchronize(x->stream);
  delete x;
  return RIVER_OK;
}
