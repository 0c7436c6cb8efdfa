// libblink: host side of the C ABI (provisioning, ring producer, token reader, loop launcher) and the
// kernel entry points. See include/blink.h for the contract of every exported function.
#include "../../include/blink.h"
#include "blink_device.h"
#include "phase_kernels.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

// ================================================================================================
// kernels
// ================================================================================================
__global__ void __launch_bounds__(BLK_THREADS) k_sched(DevCtx c) {
  __shared__ SchedShared sh;
  sched_step(c, sh);
}

// speculative decoding: the drafts of the running greedy requests, ahead of the scheduler step that feeds them
__global__ void __launch_bounds__(BLK_THREADS) k_spec_draft(DevCtx c) { spec_draft(c, blockIdx.x, gridDim.x); }

typedef void (*phase_kernel_t)(DevCtx, u32);
static phase_kernel_t phase_kernel(int ph, bool f32) {
  if (f32) {
    switch (ph) {
      case PH_EMBED: return k_embed_f32;
      case PH_QKV: return k_qkv_f32;
      case PH_ATTN: return k_attention_f32;
      case PH_OPROJ: return k_oproj_f32;
      case PH_GATEUP: return k_gateup_f32;
      case PH_DOWN: return k_down_f32;
      case PH_LM_HEAD: return k_lm_head_f32;
      default: return k_sample_publish_f32;
    }
  }
  switch (ph) {
    case PH_EMBED: return k_embed;
    case PH_QKV: return k_qkv;
    case PH_ATTN: return k_attention;
    case PH_OPROJ: return k_oproj;
    case PH_GATEUP: return k_gateup;
    case PH_DOWN: return k_down;
    case PH_LM_HEAD: return k_lm_head;
    case PH_ATTN_COMBINE: return k_attention_combine;
    case PH_ROUTER: return k_moe_router;
    case PH_ROUTE: return k_moe_route;
    case PH_MOE_GATEUP: return k_moe_gateup;
    case PH_MOE_DOWN: return k_moe_down;
    case PH_MOE_COMBINE: return k_moe_combine;
    case PH_MOE_PERMUTE: return k_moe_permute;
    default: return k_sample_publish;
  }
}

// (cos, sin) of pos * theta^(-2i/hd), evaluated in fp64 and rounded once
__global__ void k_rope_table(float2* tab, u32 max_pos, u32 half, double theta) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (u64)max_pos * half) return;
  const u32 p = (u32)(i / half), j = (u32)(i % half);
  const double ang = (double)p * pow(theta, -2.0 * (double)j / (double)(2 * half));
  tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}

__global__ void __launch_bounds__(BLK_THREADS) k_pack_weights(const bf16_t* src, f16_t* dst, u32 N, u32 K, u32 pair_rows, u32 perm_hd) {
  pack_weights(src, dst, N, K, pair_rows, perm_hd, (u64)blockIdx.x * blockDim.x + threadIdx.x, (u64)gridDim.x * blockDim.x);
}

// plain copy of `n16` 16-byte words: the known-size kernel that calibrates the HBM traffic counters
__global__ void __launch_bounds__(BLK_THREADS) k_copy_calibration(const uint4* src, uint4* dst, u64 n16) {
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (u64)gridDim.x * blockDim.x) dst[i] = src[i];
}

// plain read of `n16` 16-byte words, eight non-temporal loads in flight per lane: what a kernel that only reads (the decode
// attention's KV stream, a decode GEMM's weight stream) can reach. The sum is written only if it equals a value it never takes.
__global__ void __launch_bounds__(BLK_THREADS) k_read_calibration(const uint4* src, u32* dst, u64 n16) {
  typedef u32 u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t* p = (const u32x4_t*)src;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  u32 acc = 0;
  for (; i + 7 * stride < n16; i += 8 * stride) {
    u32x4_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(p + i + u * stride);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u][0] ^ v[u][1] ^ v[u][2] ^ v[u][3];
  }
  for (; i < n16; i += stride) { const u32x4_t v = p[i]; acc ^= v[0] ^ v[1] ^ v[2] ^ v[3]; }
  if (acc == 0x9E3779B9u) dst[(u64)blockIdx.x * blockDim.x + threadIdx.x] = acc;     // (the buffer holds zeros)
}

// register-only MFMA loop (sixteen independent 16x16x32 bf16 products per round and wave): the rate the matrix cores
// sustain on this chip at its clocks, beside which the GEMM kernels' rates are read
__global__ void __launch_bounds__(BLK_THREADS) k_mfma_calibration(float* dst, u32 rounds) {
  const u32 lane = threadIdx.x & 63;
  bf16x8_t x, y;
#pragma unroll
  for (int i = 0; i < 8; ++i) { x[i] = (__bf16)(0.001f * (float)((lane + i) & 7)); y[i] = (__bf16)(0.002f * (float)((lane * 3 + i) & 7)); }
  floatx4_t acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  for (u32 r = 0; r < rounds; ++r) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc[i], 0, 0, 0);
  }
  floatx4_t s = acc[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) s += acc[i];
  dst[(u64)blockIdx.x * blockDim.x + threadIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ void __launch_bounds__(BLK_THREADS) k_sample_rows(const float* logits, u32 n_rows, u32 V, const SampleRowParams* params,
                                                             const u32* token_index, i32* tokens) {
  __shared__ SamplerShared sh;
  sample_rows(logits, n_rows, V, params, token_index, tokens, sh);
}

// the device clock, written to pinned host memory (blink_clock_sync)
__global__ void k_clock_probe(HostMirror* m) {
  __hip_atomic_store(&m->clock_probe, dev_now_ns(), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One request into its ring slot (the frontend's write of section 4.4): payload first, then, behind a system-scope fence, the state
// word. Reads the staged descriptor and prompt from pinned host memory (16 bytes a load, four of them in flight per thread: the time of the
// call is that of the reads over the bus); one workgroup.
__global__ void __launch_bounds__(BLK_THREADS) k_ring_write(const SlotDesc* desc_in, const i32* prompt_in, u32 n_prompt, SlotStatus st, SlotDesc* desc, i32* prompt,
                                                            SlotStatus* status) {
  const u32 quads = (n_prompt + 3) / 4;                            // (the staging buffer is padded to whole ones; a slot's prompt is not)
  for (u32 i0 = threadIdx.x; i0 < quads; i0 += 4 * BLK_THREADS) {
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = ((const int4*)prompt_in)[min(i0 + u * BLK_THREADS, quads - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const u32 t = 4 * (i0 + u * BLK_THREADS);
      if (t < n_prompt) prompt[t] = v[u].x;
      if (t + 1 < n_prompt) prompt[t + 1] = v[u].y;
      if (t + 2 < n_prompt) prompt[t + 2] = v[u].z;
      if (t + 3 < n_prompt) prompt[t + 3] = v[u].w;
    }
  }
  if (threadIdx.x < sizeof(SlotDesc) / 4) ((u32*)desc)[threadIdx.x] = ((const u32*)desc_in)[threadIdx.x];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) {
    status->gen_count = st.gen_count; status->ticket_lo = st.ticket_lo; status->flags = st.flags;
    __hip_atomic_store(&status->state, st.state, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// The token reader (section 4.4) in one launch and one wait: the slots' metadata against what the host has had of every slot, the new records
// of all of them into one pinned array (slot ascending, at most `room` in all), a description of each, and a slot whose
// last record this is back to EMPTY behind them. One workgroup, small enough (32 registers) to run beside the GEMMs. The host
// reads nothing of it in between: as a copy of the metadata, a decision there and a fetch a poll waited for the device twice.
// Where 256 slots have more than POLL_HERE new records between them, their records are left to k_fetch_outputs, a second launch and
// wait: one workgroup takes 512 records to the host in 2.3 us and more. 512 slots with 8 / 16 / 64 / 120 records each, us a poll: all of it here
// 46 / 62 / 160 / 288, with the second launch 43 / 52 / 84 / 138 (the metadata copied and then one fetch, as it once was: 59 / 65 / 91 / 178).
#define POLL_HERE 2048u
struct OutPick { u32 slot, from, n : 30, left : 1, completed : 1, at; };
static_assert(sizeof(OutPick) == 16, "written as one store");
struct OutWant { u32 slot, ticket_lo, have, pad; };       // a slot with a request, slot ascending, written by the host
__global__ void __launch_bounds__(BLK_THREADS) __attribute__((amdgpu_num_vgpr(16))) k_poll_outputs(const OutWant* want, u32 n_want, SlotStatus* status, const OutRec* out_arena, u32 max_seq_len, u32 room,
                                                             OutRec* to, OutPick* picks, u32* n_picks) {
  __shared__ u32 part[BLK_THREADS / WAVE], s_slot[BLK_THREADS], s_from[BLK_THREADS], s_n[BLK_THREADS], s_at[BLK_THREADS];
  const u32 lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  u32 staged = 0, listed = 0;
  for (u32 base = 0; base < n_want && staged < room; base += BLK_THREADS) {
    u32 slot = 0, n = 0, have = 0;
    bool done = false;
    if (base + threadIdx.x < n_want) {
      const uint4 q = *(const uint4*)(want + base + threadIdx.x);
      slot = q.x;
      const SlotStatus* st = status + slot;
      // state and count in one word, as they are published, behind the records (which are read past the caches too)
      const u64 word = __hip_atomic_load((const u64*)st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      if (__hip_atomic_load(&st->ticket_lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == q.y) {
        have = q.z;
        done = (u32)word == BLINK_SLOT_DECODE_COMPLETED;
        n = (u32)(word >> 32) > have ? (u32)(word >> 32) - have : 0u;
      }
    }
    // records and slots before this thread's
    u32 inc = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const u32 t = __shfl_up(inc, o); if (lane >= (u32)o) inc += t; }
    __syncthreads();
    if (lane == 63u) part[w] = inc;
    __syncthreads();
    u32 at = inc - n, sum = 0;
    for (u32 i = 0; i < BLK_THREADS / WAVE; ++i) { if (i < w) at += part[i]; sum += part[i]; }
    const u32 left = room - staged, full = n;
    const bool left_over = min(sum, left) > POLL_HERE;
    n = at >= left ? 0u : min(n, left - at);
    const unsigned long long some = __ballot(n != 0);
    u32 place = (u32)__popcll(some & ((1ull << lane) - 1ull));
    __syncthreads();
    if (lane == 0) part[w] = (u32)__popcll(some);
    __syncthreads();
    u32 strip = 0;
    for (u32 i = 0; i < BLK_THREADS / WAVE; ++i) { if (i < w) place += part[i]; strip += part[i]; }
    if (n) {
      s_slot[place] = slot; s_from[place] = have; s_n[place] = n; s_at[place] = staged + at;
      OutPick p;
      p.slot = slot; p.from = have; p.n = n; p.left = left_over; p.completed = done && n == full; p.at = staged + at;
      *(uint4*)(picks + listed + place) = *(const uint4*)&p;
    }
    __syncthreads();
    const u32 n_recs = strip ? s_at[strip - 1] + s_n[strip - 1] - staged : 0u, n_here = left_over ? 0u : n_recs;
    for (u32 r0 = 0; r0 < n_here; r0 += 2 * BLK_THREADS) {      // a thread per record, two on their way
      u64 v[2][2];
#pragma unroll
      for (u32 u = 0; u < 2; ++u) {
        const u32 r = staged + min(r0 + u * BLK_THREADS + threadIdx.x, n_recs - 1);
        u32 lo = 0, hi = strip;                                  // its slot: the last k with s_at[k] <= r
        while (hi - lo > 1) {
          const u32 mid = (lo + hi) / 2;
          if (s_at[mid] <= r) lo = mid; else hi = mid;
        }
        const u64* src = (const u64*)(out_arena + (u64)s_slot[lo] * max_seq_len + s_from[lo] + (r - s_at[lo]));
#pragma unroll
        for (u32 h = 0; h < 2; ++h) v[u][h] = __hip_atomic_load(src + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
#pragma unroll
      for (u32 u = 0; u < 2; ++u) {
        const u32 r = r0 + u * BLK_THREADS + threadIdx.x;
        if (r < n_recs) *(ulonglong2*)(to + staged + r) = make_ulonglong2(v[u][0], v[u][1]);
      }
    }
    staged += n_recs;
    listed += strip;
    __syncthreads();                                             // (every record of the strip has been read)
    if (done && n && n == full && !left_over) {
      SlotStatus* st = status + slot;
      st->gen_count = 0; st->ticket_lo = 0; st->flags = 0;
      __hip_atomic_store(&st->state, (u32)BLINK_SLOT_EMPTY, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  if (threadIdx.x == 0) *n_picks = listed;
}

// The records that k_poll_outputs has left, a workgroup per FETCH_PIECE records of a slot (`pieces` of them per slot; the host waits
// for the launch before the slot can be taken again, so it is EMPTY whichever piece ends last).
#define FETCH_PIECE 1024u
__global__ void __launch_bounds__(BLK_THREADS) __attribute__((amdgpu_num_vgpr(16))) k_fetch_outputs(const OutPick* picks, u32 pieces, SlotStatus* status, const OutRec* out_arena, u32 max_seq_len, OutRec* to) {
  const OutPick p = picks[blockIdx.x / pieces];
  const u32 first = blockIdx.x % pieces * FETCH_PIECE;
  if (!p.left || first >= p.n) return;
  const u32 last = min(p.n, first + FETCH_PIECE) - 1;
  const u64* const src = (const u64*)(out_arena + (u64)p.slot * max_seq_len + p.from);
  for (u32 r0 = first; r0 <= last; r0 += 2 * BLK_THREADS) {
    u64 v[2][2];
#pragma unroll
    for (u32 u = 0; u < 2; ++u)
#pragma unroll
      for (u32 h = 0; h < 2; ++h) v[u][h] = __hip_atomic_load(src + 2 * (u64)min(r0 + u * BLK_THREADS + threadIdx.x, last) + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
#pragma unroll
    for (u32 u = 0; u < 2; ++u) {
      const u32 r = r0 + u * BLK_THREADS + threadIdx.x;
      if (r <= last) *(ulonglong2*)(to + p.at + r) = make_ulonglong2(v[u][0], v[u][1]);
    }
  }
  if (p.completed && first == 0 && threadIdx.x == 0) {
    SlotStatus* st = status + p.slot;
    st->gen_count = 0; st->ticket_lo = 0; st->flags = 0;
    __hip_atomic_store(&st->state, (u32)BLINK_SLOT_EMPTY, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ void k_open_window(SchedState* ss, u64 iter_limit) {
  ss->stopped = 0;
  ss->iter_limit = iter_limit;
}

// ================================================================================================
// host
// ================================================================================================
static thread_local std::string g_err;
static int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}
#define HIPCHK(x)                                                                                   \
  do {                                                                                              \
    hipError_t e_ = (x);                                                                            \
    if (e_ != hipSuccess) return fail(BLINK_ERR_DEVICE, "%s: %s (%s:%d)", #x, hipGetErrorString(e_), __FILE__, __LINE__); \
  } while (0)

// staging of blink_debug_read, 4 MB: the two descriptions, then DBG_SLOTS pieces of the result for each thread that copies them out (one on
// its way while the other is copied)
#define DBG_PIECE (512u << 10)
#define DBG_THREADS 4u
#define DBG_SLOTS 2u
#define DBG_AHEAD (256u << 10)

struct blink_engine {
  blink_config cfg{};
  DevCtx ctx{};
  int n_cu = 256;
  u32 grid = 512;
  hipStream_t compute = nullptr, s_in = nullptr, s_out = nullptr;
  std::vector<void*> dev_allocs;
  std::vector<void*> host_allocs;
  HostCtrl* hctrl = nullptr;
  HostMirror* hmirror = nullptr;
  // producer side
  u64 next_ticket = 0;
  char* stage_in = nullptr;       // pinned: descriptor + status + prompt
  // reader side
  std::vector<std::atomic<u32>> shadow_state;   // host view: 0 empty, 1 in flight
  std::vector<u32> delivered;
  std::vector<u64> slot_ticket;
  OutWant* stage_want = nullptr;       // pinned [ring_slots]
  u32* stage_n_picks = nullptr;        // pinned
  OutRec* stage_out = nullptr;         // pinned
  u64 stage_out_cap = 0;
  OutPick* stage_picks = nullptr;      // pinned [ring_slots]
  u64 iter_limit = 0;                  // of the current window (0: none)
  u64 iter_before = 0;                 // iterations and chains run before the current window
  u32 chains_before = 0;
  char* stage_dbg = nullptr;           // pinned: staging of blink_debug_read (one call at a time: dbg_mu)
  hipEvent_t dbg_ev[DBG_THREADS * DBG_SLOTS] = {};
  std::mutex dbg_mu;
  // loop
  std::thread launcher;
  hipGraphExec_t iter_graph[3] = {};          // the kernel chains of one iteration (Chain)
  bool whole_chain_ok = false, merge_in_ok = false;   // which of the shorter chains exist for this engine
  char *host_step_h = nullptr, *host_step_d = nullptr;   // BLINK_FLAG_HOST_STEP: pinned and device ends of the per-step copies
  u64 host_step_bytes = 0;
  int timed_phase = -1;                 // phase whose launches are bracketed by HIP events (-1: none)
  std::vector<hipEvent_t> phase_ev;     // [depth][n_layers][2]
  std::vector<char> phase_rec;          // [depth][n_layers]: the pair has been recorded and not yet read
  std::vector<float> phase_ms;          // per enqueued iteration of the current window: summed duration
  std::vector<hipEvent_t> events;
  std::atomic<bool> loop_active{false};
  std::atomic<int> loop_rc{0};
  std::atomic<u32> windows{0};
  bool shut = false;
  char *calib_src = nullptr, *calib_dst = nullptr;   // buffers of blink_calibration_copy
  u64 calib_bytes = 64ull << 20;
  u64 weight_bytes = 0, kv_bytes = 0, ring_bytes = 0;
  std::mutex dev_mu;   // serialises hipSetDevice-dependent host calls that allocate nothing

  explicit blink_engine(u32 slots) : shadow_state(slots) {}
};

// Launches a kernel and returns the launch's own result. (hipGetLastError also reports what any earlier HIP call of the same thread
// has left behind, the caller's own included.)
template <typename... P, typename... A>
static hipError_t launch(void (*kernel)(P...), u32 grid, u32 block, hipStream_t st, A... args) {
  std::tuple<P...> as_declared(args...);
  return std::apply([&](auto&... a) {
    void* argv[] = {(void*)&a...};
    return hipLaunchKernel((const void*)kernel, dim3(grid), dim3(block), argv, 0, st);
  }, as_declared);
}

template <typename T>
static int dalloc(blink_engine* e, T** p, u64 count, bool zero = true) {
  void* q = nullptr;
  const u64 bytes = count * sizeof(T) > 0 ? count * sizeof(T) : 16;
  HIPCHK(hipMalloc(&q, bytes));
  e->dev_allocs.push_back(q);
  if (zero) HIPCHK(hipMemset(q, 0, bytes));
  *p = (T*)q;
  return 0;
}
template <typename T>
static int halloc(blink_engine* e, T** p, u64 count) {
  void* q = nullptr;
  HIPCHK(hipHostMalloc(&q, count * sizeof(T) > 0 ? count * sizeof(T) : 16, hipHostMallocMapped));
  memset(q, 0, count * sizeof(T));
  e->host_allocs.push_back(q);
  *p = (T*)q;
  return 0;
}

static u64 expected_weight_bytes(const blink_config* c) {
  const u64 es = c->dtype == 1 ? 2 : 4;
  const u64 d = c->d_model, hd = c->head_dim, nq = c->n_q_heads, nkv = c->n_kv_heads, F = c->d_ffn, V = c->vocab;
  const u64 E = c->n_experts;
  const u64 ffn = E ? E * d + E * 3 * F * d : 3 * F * d;   // router and E experts, or the one dense FFN
  const u64 per_layer = 4 * d + 4 * d + es * ((nq + 2 * nkv) * hd * d + d * nq * hd + ffn);
  return es * V * d * 2 + c->n_layers * per_layer + 4 * d;
}

static void free_all(blink_engine* e) {
  for (hipGraphExec_t g : e->iter_graph) if (g) (void)hipGraphExecDestroy(g);
  for (hipEvent_t ev : e->events) (void)hipEventDestroy(ev);
  for (hipEvent_t ev : e->phase_ev) (void)hipEventDestroy(ev);
  for (hipEvent_t ev : e->dbg_ev) if (ev) (void)hipEventDestroy(ev);
  for (void* p : e->dev_allocs) (void)hipFree(p);
  for (void* p : e->host_allocs) (void)hipHostFree(p);
  if (e->compute) (void)hipStreamDestroy(e->compute);
  if (e->s_in) (void)hipStreamDestroy(e->s_in);
  if (e->s_out) (void)hipStreamDestroy(e->s_out);
  delete e;
}

static int build_graph(blink_engine* e);

static int init_impl(const blink_config* cfg, blink_engine* e) {
  HIPCHK(hipSetDevice(cfg->device));
  hipDeviceProp_t prop;
  HIPCHK(hipGetDeviceProperties(&prop, cfg->device));
  e->n_cu = prop.multiProcessorCount;
  e->ctx.n_cu = (u32)e->n_cu;
  e->grid = (u32)e->n_cu * 2;
  HIPCHK(hipStreamCreateWithFlags(&e->compute, hipStreamNonBlocking));
  HIPCHK(hipStreamCreateWithFlags(&e->s_in, hipStreamNonBlocking));
  HIPCHK(hipStreamCreateWithFlags(&e->s_out, hipStreamNonBlocking));
  DevCtx& c = e->ctx;
  c.n_layers = cfg->n_layers; c.d = cfg->d_model; c.nq = cfg->n_q_heads; c.nkv = cfg->n_kv_heads; c.hd = cfg->head_dim;
  c.F = cfg->d_ffn; c.V = cfg->vocab; c.dtype = cfg->dtype; c.eps = cfg->rms_eps; c.theta = cfg->rope_theta;
  c.bs = cfg->kv_block_size; c.n_blocks = cfg->kv_num_blocks; c.max_batch = cfg->max_batch; c.max_seq_len = cfg->max_seq_len;
  c.max_prefill_tokens = cfg->max_prefill_tokens; c.ring_slots = cfg->ring_slots;
  c.max_blocks_per_seq = (cfg->max_seq_len + cfg->kv_block_size - 1) / cfg->kv_block_size;
  // a prefill iteration holds at most max_prefill_tokens, except that its first request is exempt
  c.maxT = std::max(std::max(cfg->max_prefill_tokens, cfg->max_seq_len), cfg->max_batch);
  c.eos = cfg->eos_token_id; c.flags = cfg->flags; c.trace_cap = cfg->trace_capacity ? cfg->trace_capacity : 65536u;
  c.qkv_n = (c.nq + 2 * c.nkv) * c.hd;
  c.n_experts = cfg->n_experts; c.n_active = cfg->n_experts ? cfg->n_active : 0;
  // speculative decoding: a decoding sequence feeds up to 1 + spec_k tokens and has a logits row for each of them
  c.spec_k = (cfg->flags & BLINK_FLAG_SPECULATIVE) ? cfg->spec_tokens : 0u;
  const u64 rows_cap = (u64)c.max_batch * (c.spec_k + 1);
  c.maxT = std::max<u32>(c.maxT, (u32)rows_cap);
  const u64 es = c.dtype == 1 ? 2 : 4;

  // ---- ring ----
  SlotStatus* status; SlotDesc* desc; i32* in_arena; OutRec* out_arena;
  if (int rc = dalloc(e, &status, c.ring_slots)) return rc;
  if (int rc = dalloc(e, &desc, c.ring_slots)) return rc;
  if (int rc = dalloc(e, &in_arena, (u64)c.ring_slots * c.max_seq_len, false)) return rc;
  if (int rc = dalloc(e, &out_arena, (u64)c.ring_slots * c.max_seq_len, false)) return rc;
  c.status = status; c.desc = desc; c.in_arena = in_arena; c.out_arena = out_arena;
  e->ring_bytes = (u64)c.ring_slots * (sizeof(SlotStatus) + sizeof(SlotDesc) + (u64)c.max_seq_len * (4 + sizeof(OutRec)));
  if (int rc = halloc(e, &e->hctrl, 1)) return rc;
  if (int rc = halloc(e, &e->hmirror, 1)) return rc;
  c.hctrl = e->hctrl; c.hmirror = e->hmirror;
  if (int rc = halloc(e, &e->stage_in, sizeof(SlotDesc) + sizeof(SlotStatus) + ((u64)c.max_seq_len + 3) / 4 * 16)) return rc;
  if (int rc = halloc(e, &e->stage_want, c.ring_slots)) return rc;
  if (int rc = halloc(e, &e->stage_n_picks, 1)) return rc;
  e->stage_out_cap = 1u << 16;
  if (int rc = halloc(e, &e->stage_out, e->stage_out_cap)) return rc;
  if (int rc = halloc(e, &e->stage_picks, c.ring_slots)) return rc;
  {
    void* q = nullptr;
    HIPCHK(hipHostMalloc(&q, 1024 + (u64)DBG_PIECE * DBG_THREADS * DBG_SLOTS, hipHostMallocMapped));
    e->host_allocs.push_back(q);
    e->stage_dbg = (char*)q;
  }
  for (auto& ev : e->dbg_ev) HIPCHK(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
  e->delivered.assign(c.ring_slots, 0);
  e->slot_ticket.assign(c.ring_slots, 0);
  for (auto& s : e->shadow_state) s.store(0);

  // ---- scheduler state ----
  if (int rc = dalloc(e, &c.ss, 1)) return rc;
  if (int rc = dalloc(e, &c.run, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.preq, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.block_tables, (u64)c.max_batch * c.max_blocks_per_seq)) return rc;
  {
    u32 cap = 1;
    while (cap < c.n_blocks) cap <<= 1;
    c.fs_mask = cap - 1;
    if (int rc = dalloc(e, &c.free_stack, cap)) return rc;
    if (cfg->flags & BLINK_FLAG_PREFIX_CACHE) {
      c.pc_bmask = 2 * cap - 1;
      if (int rc = dalloc(e, &c.pc_ref, c.n_blocks)) return rc;
      if (int rc = dalloc(e, &c.pc_key, c.n_blocks)) return rc;
      if (int rc = dalloc(e, &c.pc_flags, c.n_blocks)) return rc;
      if (int rc = dalloc(e, &c.pc_next, c.n_blocks)) return rc;
      if (int rc = dalloc(e, &c.pc_pos, c.n_blocks)) return rc;
      if (int rc = dalloc(e, &c.pc_bucket, 2ull * cap, false)) return rc;
      HIPCHK(hipMemset(c.pc_bucket, 0xFF, 2ull * cap * 4));     // ~0u: empty chain
    }
  }
  if (int rc = dalloc(e, &c.meta, 1)) return rc;
  if (int rc = dalloc(e, &c.seq_bslot, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.seq_len, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.cu_seqlens, c.max_batch + 1)) return rc;
  if (int rc = dalloc(e, &c.last_idx, rows_cap)) return rc;
  if (c.spec_k) {
    if (int rc = dalloc(e, &c.spec_len, c.max_batch)) return rc;
    if (int rc = dalloc(e, &c.spec_tok, (u64)c.max_batch * SPEC_MAX_DRAFTS)) return rc;
    if (int rc = dalloc(e, &c.sample_row0, c.max_batch)) return rc;
    if (int rc = dalloc(e, &c.sample_nrow, c.max_batch)) return rc;
    if (int rc = dalloc(e, &c.sample_tok0, c.max_batch)) return rc;
  }
  if (int rc = dalloc(e, &c.sample_bslot, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.seq_pos0, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.seq_ring, c.max_batch)) return rc;
  if (int rc = dalloc(e, &c.cu_qtiles, c.max_batch + 1)) return rc;
  if (int rc = dalloc(e, &c.cu_chunks, c.max_batch + 1)) return rc;
  if (int rc = dalloc(e, &c.input_ids, c.maxT)) return rc;
  if (int rc = dalloc(e, &c.positions, c.maxT)) return rc;
  if (int rc = dalloc(e, &c.slot_mapping, c.maxT)) return rc;
  if (int rc = dalloc(e, &c.tok_bslot, c.maxT)) return rc;
  if (int rc = dalloc(e, &c.trace, c.trace_cap)) return rc;
  {
    std::vector<u32> fs(c.n_blocks);
    for (u32 i = 0; i < c.n_blocks; ++i) fs[i] = c.n_blocks - 1 - i;   // first pops return 0, 1, 2, ...
    HIPCHK(hipMemcpy(c.free_stack, fs.data(), (u64)c.n_blocks * 4, hipMemcpyHostToDevice));
    SchedState s0{};
    s0.free_top = c.n_blocks;
    s0.stopped = 1;
    HIPCHK(hipMemcpy(c.ss, &s0, sizeof s0, hipMemcpyHostToDevice));
  }

  // ---- weights ----
  // fp32 model: the blob is uploaded as is and the matrices are used in their [out][in] layout.
  // bf16 model: the embedding table and the gains are kept as they come; every other matrix goes through a staging
  // buffer into its packed form (MFMA operand order) and the row-major copy is not kept.
  c.tune_nw = cfg->tune;
  {
    std::vector<LayerW> lw(c.n_layers);
    const u64 d = c.d, hd = c.hd, nq = c.nq, nkv = c.nkv, F = c.F, V = c.V;
    const char* hsrc = (const char*)cfg->weights;
    u64 off = 0;
    if (c.dtype == 0) {
      char* wdev;
      if (int rc = dalloc(e, &wdev, cfg->weights_bytes, false)) return rc;
      HIPCHK(hipMemcpy(wdev, hsrc, cfg->weights_bytes, hipMemcpyHostToDevice));
      e->weight_bytes = cfg->weights_bytes;
      c.embed = wdev + off; off += es * V * d;
      for (u32 l = 0; l < c.n_layers; ++l) {
        lw[l].g1 = (const float*)(wdev + off); off += 4 * d;
        lw[l].wqkv = wdev + off; off += es * (nq + 2 * nkv) * hd * d;
        lw[l].wo = wdev + off; off += es * d * nq * hd;
        lw[l].g2 = (const float*)(wdev + off); off += 4 * d;
        lw[l].wgu = wdev + off; off += es * 2 * F * d;
        lw[l].wd = wdev + off; off += es * d * F;
      }
      c.gf = (const float*)(wdev + off); off += 4 * d;
      c.lm = wdev + off; off += es * V * d;
    } else {
      std::vector<LayerWP> lp(c.n_layers);
      const u64 stage_bytes = 2 * std::max(std::max(std::max(V * d, 2 * F * d), (u64)c.n_experts * d), std::max((nq + 2 * nkv) * hd * d, d * nq * hd));
      char *stage = nullptr, *embed = nullptr;
      float* gains = nullptr;
      HIPCHK(hipMalloc((void**)&stage, stage_bytes));     // freed at the end of this block, on every path
      // src_off2 != 0: the second half of the rows is stored there (an expert's up matrix lies apart from its gate matrix)
      auto pack_to = [&](f16_t* p, u64 src_off, u64 src_off2, u32 N, u32 K, u32 pair_rows, u32 perm_hd) -> int {
        if (src_off2) {
          HIPCHK(hipMemcpy(stage, hsrc + src_off, (u64)N * K, hipMemcpyHostToDevice));
          HIPCHK(hipMemcpy(stage + (u64)N * K, hsrc + src_off2, (u64)N * K, hipMemcpyHostToDevice));
        } else {
          HIPCHK(hipMemcpy(stage, hsrc + src_off, (u64)N * K * 2, hipMemcpyHostToDevice));
        }
        HIPCHK(launch(k_pack_weights, 2048, BLK_THREADS, e->compute, (const bf16_t*)stage, p, N, K, pair_rows, perm_hd));
        HIPCHK(hipStreamSynchronize(e->compute));          // the staging buffer is reused by the next matrix
        return 0;
      };
      auto pack = [&](u64 src_off, u32 N, u32 K, u32 pair_rows, u32 perm_hd, const f16_t** dst) -> int {
        f16_t* p;
        const u64 elems = (u64)((N + 15) / 16) * gemm_k_tiles(K) * 512;
        if (int rc = dalloc(e, &p, elems, false)) return rc;
        if (int rc = pack_to(p, src_off, 0, N, K, pair_rows, perm_hd)) return rc;
        *dst = p;
        e->weight_bytes += elems * 2;
        return 0;
      };
      // the experts of one layer: packed one after the other (2F x d gate/up pairs, then d x F down matrices)
      auto pack_experts = [&](u64 off_g, u64 off_u, u64 off_d, LayerWP& lp_l) -> int {
        const u64 E = c.n_experts, gu = (2 * F / 16) * gemm_k_tiles(c.d) * 512, dn = (d / 16) * gemm_k_tiles(c.F) * 512;   // elements of one expert
        f16_t *pgu, *pd;
        if (int rc = dalloc(e, &pgu, E * gu, false)) return rc;
        if (int rc = dalloc(e, &pd, E * dn, false)) return rc;
        for (u64 x = 0; x < E; ++x) {
          if (int rc = pack_to(pgu + x * gu, off_g + x * 2 * F * d, off_u + x * 2 * F * d, 2 * c.F, c.d, c.F, 0)) return rc;
          if (int rc = pack_to(pd + x * dn, off_d + x * 2 * d * F, 0, c.d, c.F, 0, 0)) return rc;
        }
        lp_l.wgu = pgu; lp_l.wd = pd;
        e->weight_bytes += E * (gu + dn) * 2;
        return 0;
      };
      auto all = [&]() -> int {
        if (int rc = dalloc(e, &embed, 2 * V * d, false)) return rc;
        if (int rc = dalloc(e, &gains, (2 * (u64)c.n_layers + 1) * d, false)) return rc;
        HIPCHK(hipMemcpy(embed, hsrc + off, 2 * V * d, hipMemcpyHostToDevice));
        c.embed = embed; off += 2 * V * d;
        e->weight_bytes = 2 * V * d + (2 * (u64)c.n_layers + 1) * d * 4;
        for (u32 l = 0; l < c.n_layers; ++l) {
          float* g1 = gains + (2 * (u64)l) * d;
          float* g2 = g1 + d;
          HIPCHK(hipMemcpy(g1, hsrc + off, 4 * d, hipMemcpyHostToDevice)); off += 4 * d;
          if (int rc = pack(off, c.qkv_n, c.d, 0, c.hd, &lp[l].wqkv)) return rc;
          off += 2 * (nq + 2 * nkv) * hd * d;
          if (int rc = pack(off, c.d, c.nq * c.hd, 0, 0, &lp[l].wo)) return rc;
          off += 2 * d * nq * hd;
          HIPCHK(hipMemcpy(g2, hsrc + off, 4 * d, hipMemcpyHostToDevice)); off += 4 * d;
          if (c.n_experts) {
            const u64 E = c.n_experts;
            if (int rc = pack(off, c.n_experts, c.d, 0, 0, &lp[l].wr)) return rc;
            off += 2 * E * d;
            if (int rc = pack_experts(off, off + 2 * E * F * d, off + 4 * E * F * d, lp[l])) return rc;
            off += 2 * 3 * E * F * d;
          } else {
            if (int rc = pack(off, 2 * c.F, c.d, c.F, 0, &lp[l].wgu)) return rc;
            off += 2 * 2 * F * d;
            if (int rc = pack(off, c.d, c.F, 0, 0, &lp[l].wd)) return rc;
            off += 2 * d * F;
          }
          lw[l].g1 = g1; lw[l].g2 = g2; lw[l].wqkv = lw[l].wo = lw[l].wgu = lw[l].wd = nullptr;
        }
        float* gf = gains + 2 * (u64)c.n_layers * d;
        HIPCHK(hipMemcpy(gf, hsrc + off, 4 * d, hipMemcpyHostToDevice)); off += 4 * d;
        c.gf = gf;
        if (int rc = pack(off, c.V, c.d, 0, 0, &c.lm_p)) return rc;
        off += 2 * V * d;
        c.lm = nullptr;
        return 0;
      };
      const int rc = all();
      const std::string keep = g_err;
      (void)hipFree(stage);
      g_err = keep;
      if (rc) return rc;
      LayerWP* dp;
      if (int rc2 = dalloc(e, &dp, c.n_layers)) return rc2;
      HIPCHK(hipMemcpy(dp, lp.data(), sizeof(LayerWP) * c.n_layers, hipMemcpyHostToDevice));
      c.players = dp;
    }
    if (off != cfg->weights_bytes) return fail(BLINK_ERR_INVAL, "internal: weight layout %llu != %llu", (unsigned long long)off, (unsigned long long)cfg->weights_bytes);
    LayerW* dl;
    if (int rc = dalloc(e, &dl, c.n_layers)) return rc;
    HIPCHK(hipMemcpy(dl, lw.data(), sizeof(LayerW) * c.n_layers, hipMemcpyHostToDevice));
    c.layers = dl;
  }
  {
    float2* tab;
    if (int rc = dalloc(e, &tab, (u64)c.max_seq_len * (c.hd / 2), false)) return rc;
    const u64 n = (u64)c.max_seq_len * (c.hd / 2);
    HIPCHK(launch(k_rope_table, (u32)((n + 255) / 256), 256, e->compute, tab, c.max_seq_len, c.hd / 2, (double)c.theta));
    c.rope_tab = tab;
  }
  // ---- bf16 model: packed activation operands between the GEMMs, decode attention partials ----
  c.TBS = ((c.maxT + 255) / 256) * 16;   // whole 256-token workgroup tiles
  if (c.dtype == 1) {
    const u64 tile_tokens = (u64)c.TBS * 16;
    auto k_pad = [](u32 K) { return (u64)gemm_k_tiles(K) * 32; };      // (the padding stays zero)
    if (int rc = dalloc(e, &c.xq, tile_tokens * k_pad(c.d))) return rc;
    if (int rc = dalloc(e, &c.aq, tile_tokens * k_pad(c.nq * c.hd))) return rc;
    if (c.n_experts) {
      // every (token, selected expert) pair is a column of the grouped GEMMs; the columns of one expert start at a
      // multiple of 16, and a workgroup tile may read up to 255 columns past the last one
      const u64 cols = (u64)c.maxT * c.n_active + 16ull * c.n_experts + 256 + 16;
      c.moe_TBS = (u32)((cols + 15) / 16);
      if (int rc = dalloc(e, &c.hq_moe, (u64)c.moe_TBS * 16 * k_pad(c.F))) return rc;
      if (int rc = dalloc(e, &c.xq_moe, (u64)c.moe_TBS * 16 * k_pad(c.d))) return rc;
      if (int rc = dalloc(e, &c.y_moe, (u64)c.moe_TBS * 16 * c.d, false)) return rc;
      if (int rc = dalloc(e, &c.moe_logits, (u64)c.maxT * c.n_experts, false)) return rc;
      if (int rc = dalloc(e, &c.moe_count, (u64)c.n_experts * MOE_COUNT_STRIDE)) return rc;
      if (int rc = dalloc(e, &c.moe_list, (u64)c.n_experts * c.maxT)) return rc;
      if (int rc = dalloc(e, &c.moe_sel, (u64)c.n_layers * c.maxT * c.n_active)) return rc;
      if (int rc = dalloc(e, &c.moe_pos, (u64)c.maxT * c.n_active)) return rc;
      if (int rc = dalloc(e, &c.moe_w, (u64)c.maxT * c.n_active)) return rc;
      if (int rc = dalloc(e, &c.moe_rstd, c.maxT)) return rc;
    } else if (int rc = dalloc(e, &c.hq, tile_tokens * k_pad(c.F))) return rc;
    if (int rc = dalloc(e, &c.ssq, tile_tokens * (c.d / 16))) return rc;
    {
      const std::vector<GemmPlan> plan = gemm_plan_table(c.maxT, c.qkv_n, c.d, c.nq * c.hd, c.F, c.V, c.n_experts != 0, (u32)e->n_cu, cfg->tune);
      u64* dev;
      static_assert(sizeof(GemmPlan) == 8, "an entry is one word");
      if (int rc = dalloc(e, &dev, plan.size())) return rc;
      HIPCHK(hipMemcpy(dev, plan.data(), plan.size() * sizeof(GemmPlan), hipMemcpyHostToDevice));
      c.gemm_plan = dev;
      bool cut = false;                          // (K in slices: not in a mixture of experts, nor in matrices that are large enough)
      for (const GemmPlan& p : plan) cut = cut || p.qkv >> 3 || p.oproj >> 3 || p.down >> 3;
      if (cut) {
        if (int rc = dalloc(e, &c.gemm_part, (u64)e->n_cu * (256 * 128 / 2), false)) return rc;
        if (int rc = dalloc(e, &c.gemm_part_count, (u64)e->n_cu)) return rc;
      }
    }
    if (int rc = dalloc(e, &c.qbuf, ((u64)c.maxT + 16) * c.nq * c.hd)) return rc;   // (and x: 16 rows for the tokens that fill up a tile)
    {
      c.chunk_cap = c.max_batch * ((c.max_seq_len + ATTN_CHUNK_TOKENS - 1) / ATTN_CHUNK_TOKENS);
      if (int rc = dalloc(e, &c.chunk_rec, 2ull * c.chunk_cap)) return rc;
      if (int rc = dalloc(e, &c.attn_ctr, 2ull * c.n_layers)) return rc;
    }
    {
      const u64 chunks = (u64)c.max_batch * ((c.max_seq_len + ATTN_CHUNK_TOKENS - 1) / ATTN_CHUNK_TOKENS), G = c.nq / c.nkv;
      if (int rc = dalloc(e, &c.attn_part_o, chunks * c.nkv * G * c.hd)) return rc;
      if (int rc = dalloc(e, &c.attn_part_ml, chunks * c.nkv * G * 2)) return rc;
      if (int rc = dalloc(e, &c.attn_merge_ctr, (u64)c.max_batch * c.nkv)) return rc;
    }
  }
  if (int rc = dalloc(e, &e->calib_src, e->calib_bytes)) return rc;
  if (int rc = dalloc(e, &e->calib_dst, e->calib_bytes)) return rc;
  // ---- KV pool ----
  c.kv_kv_stride = (u64)c.n_blocks * c.nkv * c.bs * c.hd;
  c.kv_layer_stride = 2 * c.kv_kv_stride;
  e->kv_bytes = (u64)c.n_layers * c.kv_layer_stride * es;
  char* kv;
  if (int rc = dalloc(e, &kv, e->kv_bytes, true)) return rc;   // zeroed: masked keys multiply cached values by 0
  c.kv = kv;
  // ---- activations ----
  if (int rc = dalloc(e, &c.x, ((u64)c.maxT + 16) * c.d)) return rc;
  if (c.dtype == 0) {
    if (int rc = dalloc(e, &c.qkv, (u64)c.maxT * c.qkv_n)) return rc;
    if (int rc = dalloc(e, &c.attn, (u64)c.maxT * c.nq * c.hd)) return rc;
    if (int rc = dalloc(e, &c.gu, (u64)c.maxT * c.F)) return rc;
  }
  if (int rc = dalloc(e, &c.logits, rows_cap * c.V)) return rc;
  HIPCHK(hipStreamSynchronize(e->compute));
  HIPCHK(hipDeviceSynchronize());
  c.idle_poll_ns = 1000ull * (cfg->idle_poll_us ? cfg->idle_poll_us : 2000u);
  e->hctrl->exit_when_idle = (cfg->flags & BLINK_FLAG_EXIT_WHEN_IDLE) ? 1u : 0u;
  {
    u32 depth = cfg->pump_depth ? cfg->pump_depth : 8u;
    if (depth > 1024) depth = 1024;
    if (cfg->flags & BLINK_FLAG_HOST_STEP) {
      depth = 1;
      e->host_step_bytes = 32ull * c.max_batch;
      if (int rc = halloc(e, &e->host_step_h, e->host_step_bytes)) return rc;
      if (int rc = dalloc(e, &e->host_step_d, e->host_step_bytes)) return rc;
    }
    e->events.resize(depth);
    for (u32 i = 0; i < depth; ++i) HIPCHK(hipEventCreateWithFlags(&e->events[i], hipEventDisableTiming));
    e->phase_ev.resize((u64)depth * c.n_layers * 2);
    for (auto& ev : e->phase_ev) HIPCHK(hipEventCreate(&ev));
    e->phase_rec.assign((u64)depth * c.n_layers, 0);
  }
  if (int rc = build_graph(e)) return rc;
  return 0;
}

extern "C" int blink_init(const blink_config* cfg, blink_engine** out) {
  g_err.clear();
  if (!cfg || !out) return fail(BLINK_ERR_INVAL, "null argument");
  *out = nullptr;
  if (!cfg->weights) return fail(BLINK_ERR_INVAL, "weights is null");
  if (cfg->dtype > 1) return fail(BLINK_ERR_INVAL, "dtype must be 0 (fp32) or 1 (bf16)");
  if (!cfg->n_layers || !cfg->d_model || !cfg->n_q_heads || !cfg->n_kv_heads || !cfg->d_ffn || !cfg->vocab)
    return fail(BLINK_ERR_INVAL, "zero model dimension");
  if (cfg->head_dim != 64 && cfg->head_dim != 128) return fail(BLINK_ERR_INVAL, "head_dim must be 64 or 128");
  if (cfg->n_q_heads % cfg->n_kv_heads || cfg->n_q_heads / cfg->n_kv_heads > ATT_MAX_G)
    return fail(BLINK_ERR_INVAL, "n_q_heads must be a multiple (at most %d) of n_kv_heads", ATT_MAX_G);
  if (cfg->d_model % 32 || cfg->d_ffn % 32 || (cfg->n_q_heads * cfg->head_dim) % 32)
    return fail(BLINK_ERR_INVAL, "d_model, d_ffn and n_q_heads*head_dim must be multiples of 32");
  if (cfg->dtype == 1) {
    const u32 G = cfg->n_q_heads / cfg->n_kv_heads;
    if (!(G == 1 || G == 2 || G == 3 || G == 4 || G == 6 || G == 8))
      return fail(BLINK_ERR_INVAL, "bf16 path: n_q_heads / n_kv_heads must be 1, 2, 3, 4, 6 or 8");
  }
  if (cfg->n_experts) {
    if (cfg->dtype != 1) return fail(BLINK_ERR_INVAL, "mixture-of-experts models are built for dtype 1 (bf16 weights) only");
    if (cfg->n_experts > MOE_MAX_EXPERTS || !cfg->n_active || cfg->n_active > MOE_MAX_ACTIVE || cfg->n_active > cfg->n_experts)
      return fail(BLINK_ERR_INVAL, "n_experts must be at most %d and n_active in [1, min(%d, n_experts)]", MOE_MAX_EXPERTS, MOE_MAX_ACTIVE);
  }
  if (cfg->vocab >= (1u << 24)) return fail(BLINK_ERR_INVAL, "vocab must be below 2^24");
  if (cfg->kv_block_size != 16) return fail(BLINK_ERR_INVAL, "kv_block_size must be 16");
  if (!cfg->kv_num_blocks || !cfg->max_batch || cfg->max_batch > SCHED_MAX_BATCH)
    return fail(BLINK_ERR_INVAL, "kv_num_blocks must be positive and max_batch in [1, %d]", SCHED_MAX_BATCH);
  if (cfg->dtype == 1 && cfg->max_batch > ATTN_META_MAX)
    return fail(BLINK_ERR_INVAL, "bf16 models take at most %d batch slots (attention keeps the batch metadata in LDS)", ATTN_META_MAX);
  if (!cfg->max_seq_len || !cfg->max_prefill_tokens) return fail(BLINK_ERR_INVAL, "max_seq_len and max_prefill_tokens must be positive");
  if (cfg->max_seq_len >= (1u << 22)) return fail(BLINK_ERR_INVAL, "max_seq_len must be below 2^22 (the scheduler sorts contexts by a 32-bit key)");
  if ((cfg->flags & BLINK_FLAG_CHUNKED_PREFILL) && (cfg->flags & BLINK_FLAG_PREEMPTION))
    return fail(BLINK_ERR_INVAL, "preemption is built for the plain (pause-and-resume) mode, not together with chunked prefill");
  if ((cfg->flags & BLINK_FLAG_PREFIX_CACHE) && (cfg->flags & (BLINK_FLAG_CHUNKED_PREFILL | BLINK_FLAG_PREEMPTION)))
    return fail(BLINK_ERR_INVAL, "prefix caching is built for the plain mode, not together with chunked prefill or preemption");
  if ((cfg->flags & BLINK_FLAG_CHUNKED_PREFILL) && cfg->max_prefill_tokens <= cfg->max_batch)
    return fail(BLINK_ERR_INVAL, "chunked prefill: max_prefill_tokens (the token budget of an iteration) must exceed max_batch");
  if (cfg->flags & BLINK_FLAG_SPECULATIVE) {
    if (cfg->flags & (BLINK_FLAG_CHUNKED_PREFILL | BLINK_FLAG_PREEMPTION | BLINK_FLAG_PREFIX_CACHE))
      return fail(BLINK_ERR_INVAL, "speculative decoding is built for the plain mode, not together with chunked prefill, preemption or prefix caching");
    if (cfg->spec_tokens < 1 || cfg->spec_tokens >= SPEC_MAX_DRAFTS)
      return fail(BLINK_ERR_INVAL, "speculative decoding: spec_tokens must be in [1, %u]", SPEC_MAX_DRAFTS - 1);
  }
  if (!cfg->ring_slots || (cfg->ring_slots & (cfg->ring_slots - 1))) return fail(BLINK_ERR_INVAL, "ring_slots must be a power of two");
  if (cfg->weights_bytes != expected_weight_bytes(cfg))
    return fail(BLINK_ERR_INVAL, "weights_bytes is %llu, the model needs %llu", (unsigned long long)cfg->weights_bytes,
                (unsigned long long)expected_weight_bytes(cfg));
  int n_dev = 0;
  if (hipGetDeviceCount(&n_dev) != hipSuccess || n_dev <= 0) return fail(BLINK_ERR_DEVICE, "no HIP device available");
  if (cfg->device < 0 || cfg->device >= n_dev) return fail(BLINK_ERR_INVAL, "device %d out of range", cfg->device);
  blink_engine* e = new blink_engine(cfg->ring_slots);
  e->cfg = *cfg;
  e->cfg.weights = nullptr;
  const int rc = init_impl(cfg, e);
  if (rc) {
    const std::string keep = g_err;
    free_all(e);
    g_err = keep;
    return rc;
  }
  *out = e;
  return BLINK_OK;
}

extern "C" int blink_submit(blink_engine* e, const int32_t* prompt, uint32_t n_prompt, uint32_t max_new_tokens,
                            const blink_sampling* sp, uint64_t* request_id_out) {
  g_err.clear();
  if (!e || !prompt || !sp) return fail(BLINK_ERR_INVAL, "null argument");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  const DevCtx& c = e->ctx;
  if (n_prompt == 0 || max_new_tokens == 0) return fail(BLINK_ERR_INVAL, "empty prompt or max_new_tokens == 0");
  if (!(sp->temperature >= 0.f) || !(sp->top_p > 0.f && sp->top_p <= 1.f)) return fail(BLINK_ERR_INVAL, "temperature must be >= 0 and top_p in (0,1]");
  if (sp->temperature > 0.f && (sp->top_k == 0 || sp->top_k > SAMPLER_MAX_K) && c.V > SAMPLER_MAX_K)
    return fail(BLINK_ERR_INVAL, "sampling needs top_k in [1, %d] when vocab exceeds %d", SAMPLER_MAX_K, SAMPLER_MAX_K);
  if ((u64)n_prompt + max_new_tokens > c.max_seq_len) return fail(BLINK_ERR_TOO_LARGE, "prompt + max_new_tokens exceeds max_seq_len");
  const u64 need = std::max<u64>(1, ((u64)n_prompt + max_new_tokens - 1 + c.bs - 1) / c.bs);
  if (need > c.n_blocks) return fail(BLINK_ERR_TOO_LARGE, "KV reservation of %llu blocks exceeds the pool", (unsigned long long)need);
  for (u32 i = 0; i < n_prompt; ++i)
    if (prompt[i] < 0 || (u32)prompt[i] >= c.V) return fail(BLINK_ERR_INVAL, "token id %d at %u outside the vocabulary", prompt[i], i);
  const u64 t = e->next_ticket;
  const u32 slot = (u32)(t & (c.ring_slots - 1));
  if (e->shadow_state[slot].load(std::memory_order_acquire) != 0) return fail(BLINK_ERR_FULL, "ring slot %u still in use", slot);
  HIPCHK(hipSetDevice(e->cfg.device));
  // payload first: prompt tokens and descriptor; then the state word (section 4.4 "RDMA datapath")
  SlotDesc* d = (SlotDesc*)e->stage_in;
  SlotStatus* st = (SlotStatus*)(e->stage_in + sizeof(SlotDesc));
  i32* ptoks = (i32*)(e->stage_in + sizeof(SlotDesc) + sizeof(SlotStatus));
  memset(d, 0, sizeof *d);
  d->ticket = t; d->n_prompt = n_prompt; d->max_new = max_new_tokens; d->temperature = sp->temperature; d->top_k = sp->top_k;
  d->top_p = sp->top_p; d->seed = sp->seed;
  memcpy(ptoks, prompt, (u64)n_prompt * 4);
  st->state = BLINK_SLOT_PREFILL_PENDING; st->gen_count = 0; st->ticket_lo = (u32)t; st->flags = 0;
  e->slot_ticket[slot] = t;
  e->delivered[slot] = 0;
  e->shadow_state[slot].store(1, std::memory_order_release);
  // one small kernel and one wait: 20 us a call on an idle engine, 26 with a prompt of 4000 tokens (read 4 bytes a load: 44), 30 beside
  // prefill iterations of 8000 tokens (three copies and one wait: 23 / 28 / 37; and a second wait: 33 / 38)
  const hipError_t launched = launch(k_ring_write, 1, BLK_THREADS, e->s_in, d, ptoks, n_prompt, *st, c.desc + slot, c.in_arena + (u64)slot * c.max_seq_len, c.status + slot);
  if (launched != hipSuccess) e->shadow_state[slot].store(0, std::memory_order_release);
  HIPCHK(launched);
  HIPCHK(hipStreamSynchronize(e->s_in));
  e->next_ticket = t + 1;
  if (request_id_out) *request_id_out = t;
  return BLINK_OK;
}

// ---- loop launcher -----------------------------------------------------------------------------------------
// The host thread is a pump: it enqueues the fixed kernel chain of one iteration, several iterations ahead,
// and never reads a result the device waits for. Every decision (what runs, on which shapes, when the window
// ends) is taken on the device; an iteration enqueued after the window has ended costs a few empty kernels.
static bool phase_per_layer(int ph) { return (ph >= PH_LAYER_FIRST && ph <= PH_LAYER_LAST) || ph >= PH_ATTN_COMBINE; }

static int launch_phase(blink_engine* e, const DevCtx& ctx, hipStream_t st, int ph, u32 layer, u64 enq_index) {
  const bool timed = e->timed_phase == ph && enq_index != ~0ull;
  hipEvent_t a = nullptr, b = nullptr;
  if (timed) {
    const u64 slot = (enq_index % e->events.size()) * e->ctx.n_layers + (phase_per_layer(ph) ? layer : 0);
    a = e->phase_ev[2 * slot];
    b = e->phase_ev[2 * slot + 1];
    e->phase_rec[slot] = 1;
    HIPCHK(hipEventRecord(a, st));
  }
  // the GEMMs of a bf16 model run one eight-wave workgroup per compute unit, and so does the down projection of an fp32 model
  const bool gemm = ph == PH_QKV || ph == PH_OPROJ || ph == PH_GATEUP || ph == PH_DOWN || ph == PH_LM_HEAD || ph == PH_MOE_GATEUP || ph == PH_MOE_DOWN;
  const bool bf16 = e->ctx.dtype == 1;
  const bool down_f32 = !bf16 && ph == PH_DOWN;
  const u32 threads = down_f32 ? 64u * F32_DOWN_WAVES : bf16 && (gemm || ph == PH_ATTN) ? 512u : (u32)BLK_THREADS;
  HIPCHK(launch(phase_kernel(ph, !bf16), (bf16 && gemm) || down_f32 ? (u32)e->n_cu : e->grid, threads, st, ctx, layer));
  if (timed) HIPCHK(hipEventRecord(b, st));
  return 0;
}

// The kernel chains of one iteration. The merge kernel behind every attention launch (32 per iteration of a 32-layer model; an empty
// kernel costs 4-5 us here, the gap before the next one 2-3 us) is there in the first only.
// CHAIN_WHOLE: for iterations whose decode attention takes whole contexts as its items. The scheduler step of this chain is told to
// make them so whatever the batch (bit 22 of its tuning word), and no item leaves a partial result.
// CHAIN_MERGE_IN: the attention kernel merges the chunks of a context itself (bit 4).
enum Chain { CHAIN_MERGE_KERNEL, CHAIN_WHOLE, CHAIN_MERGE_IN };
static int enqueue_iteration_kernels(blink_engine* e, hipStream_t st, u64 enq_index, Chain kind) {
  DevCtx c = e->ctx;
  if (kind == CHAIN_WHOLE) c.tune_nw |= 0x400000u;
  if (kind == CHAIN_MERGE_IN) c.tune_nw |= 0x10u;
  if (c.spec_k) HIPCHK(launch(k_spec_draft, (c.max_batch + 3) / 4, BLK_THREADS, st, c));
  HIPCHK(launch(k_sched, 1, BLK_THREADS, st, c));
  if (int rc = launch_phase(e, c, st, PH_EMBED, 0, enq_index)) return rc;
  // the phases of a layer; the norms and the rotary step have no kernels of their own
  static const int dense[] = {PH_QKV, PH_ATTN, PH_ATTN_COMBINE, PH_OPROJ, PH_GATEUP, PH_DOWN};
  static const int experts[] = {PH_QKV, PH_ATTN, PH_ATTN_COMBINE, PH_OPROJ, PH_ROUTER, PH_ROUTE, PH_MOE_PERMUTE, PH_MOE_GATEUP, PH_MOE_DOWN, PH_MOE_COMBINE};
  const int *const chain = c.n_experts ? experts : dense, n = (int)(c.n_experts ? sizeof experts : sizeof dense) / (int)sizeof(int);
  for (u32 l = 0; l < c.n_layers; ++l)
    for (int i = 0; i < n; ++i) {
      if (chain[i] == PH_ATTN_COMBINE && (c.dtype == 0 || kind != CHAIN_MERGE_KERNEL)) continue;
      if (int rc = launch_phase(e, c, st, chain[i], l, enq_index)) return rc;
    }
  if (int rc = launch_phase(e, c, st, PH_LM_HEAD, 0, enq_index)) return rc;
  return launch_phase(e, c, st, PH_SAMPLE, 0, enq_index);
}

static int capture_chain(blink_engine* e, Chain kind, hipGraphExec_t* out) {
  hipGraph_t g = nullptr;
  HIPCHK(hipStreamBeginCapture(e->compute, hipStreamCaptureModeThreadLocal));
  const int rc = enqueue_iteration_kernels(e, e->compute, ~0ull, kind);
  hipError_t er = hipStreamEndCapture(e->compute, &g);
  if (rc) return rc;
  HIPCHK(er);
  HIPCHK(hipGraphInstantiate(out, g, nullptr, nullptr, 0));
  HIPCHK(hipGraphDestroy(g));
  return 0;
}

static int build_graph(blink_engine* e) {
  // The chain for whole contexts exists where the scheduler can make whole contexts the items of every decode iteration: bf16
  // models in the plain mode, unless the tuning word forces chunk items or the static kernel (bits 15, 23) or rules
  // the chain out (bit 5). The one that merges in the attention kernel exists in every mode (not with bits 5 and 23).
  const u32 ext = BLINK_FLAG_CHUNKED_PREFILL | BLINK_FLAG_PREEMPTION | BLINK_FLAG_PREFIX_CACHE | BLINK_FLAG_SPECULATIVE;
  e->whole_chain_ok = e->ctx.dtype == 1 && e->ctx.chunk_rec && !(e->cfg.flags & ext) && !(e->cfg.tune & 0x808020u);
  e->merge_in_ok = e->ctx.dtype == 1 && e->ctx.chunk_rec && !(e->cfg.tune & 0x800020u);
  if (e->cfg.flags & BLINK_FLAG_NO_GRAPH) return 0;
  // (the one with the merge kernel is never taken where the attention kernel merges whatever the number of items)
  if (!e->merge_in_ok || !((e->cfg.tune & 0x8u) || merge_in_attention(~0u, e->ctx.hd, (u32)e->n_cu)))
    if (int rc = capture_chain(e, CHAIN_MERGE_KERNEL, &e->iter_graph[CHAIN_MERGE_KERNEL])) return rc;
  if (e->whole_chain_ok)
    if (int rc = capture_chain(e, CHAIN_WHOLE, &e->iter_graph[CHAIN_WHOLE])) return rc;
  if (e->merge_in_ok)
    if (int rc = capture_chain(e, CHAIN_MERGE_IN, &e->iter_graph[CHAIN_MERGE_IN])) return rc;
  return 0;
}

// Which chain the next iteration runs is the launcher's choice, and the only one it makes: from the number of running
// sequences and of the attention items ahead that the scheduler step last mirrored to the host (plain reads of pinned memory, several iterations old,
// hints and nothing more) it takes the chain for whole contexts when the device would make those the items anyway (the same
// threshold), and the one that merges in the attention kernel where that is cheaper (merge_in_attention). Any chain is correct
// for any iteration; a stale hint costs a few iterations with the other one.
static Chain pick_chain(const blink_engine* e) {
  const u32 nrun = *(volatile const u32*)&e->hmirror->n_running, items = *(volatile const u32*)&e->hmirror->attn_items;
  if (e->whole_chain_ok && ((e->cfg.tune & 0x80u) || (u64)nrun * e->ctx.nkv >= WHOLE_CONTEXT_PAIRS_PER_CU * (u64)e->ctx.n_cu)) return CHAIN_WHOLE;
  if (e->merge_in_ok && ((e->cfg.tune & 0x8u) || merge_in_attention(items, e->ctx.hd, (u32)e->ctx.n_cu))) return CHAIN_MERGE_IN;
  return CHAIN_MERGE_KERNEL;
}

static int enqueue_iteration(blink_engine* e, u64 enq_index) {
  const Chain kind = pick_chain(e);
  if (e->iter_graph[kind] && e->timed_phase < 0) {
    HIPCHK(hipGraphLaunch(e->iter_graph[kind], e->compute));
    return 0;
  }
  return enqueue_iteration_kernels(e, e->compute, enq_index, kind);
}

// durations of the timed phase for the iteration enqueued at enq_index (its events have completed). A phase without kernels in
// that iteration's chain counts as 0: its events are not asked (the error of an event that was never recorded would stay behind
// for the next launch's check, which then ends the loop).
static void harvest_phase_times(blink_engine* e, u64 enq_index) {
  if (e->timed_phase < 0) return;
  const bool per_layer = phase_per_layer(e->timed_phase);
  const u32 n = per_layer ? e->ctx.n_layers : 1;
  float sum = 0.f;
  for (u32 l = 0; l < n; ++l) {
    const u64 slot = (enq_index % e->events.size()) * e->ctx.n_layers + l;
    float ms = 0.f;
    if (!e->phase_rec[slot]) continue;
    e->phase_rec[slot] = 0;
    if (hipEventElapsedTime(&ms, e->phase_ev[2 * slot], e->phase_ev[2 * slot + 1]) == hipSuccess) sum += ms;
  }
  e->phase_ms.push_back(sum);
}

static void pump_loop(blink_engine* e) {
  int rc = 0;
  if (hipSetDevice(e->cfg.device) != hipSuccess) rc = BLINK_ERR_DEVICE;
  const u32 depth = (u32)e->events.size();
  u64 enq = 0, done = 0;                         // iterations enqueued, and waited for
  while (rc == 0) {
    // `depth` iterations in flight, but no more than the window still lacks: behind its last iteration a chain is a row of
    // empty kernels (60-500 us for the eight of them) that the end of the window would wait for. What it lacks are the
    // iterations that have not begun, and what is on its way to them are the chains whose scheduler step has not run: the device
    // mirrors both counts in one word. (Chains not waited for are one more, the one that runs: counted like that,
    // the last chain was enqueued only behind the end of the one before it.)
    const u64 limit = e->iter_limit, progress = *(volatile const u64*)&e->hmirror->progress;
    const u64 lacking = limit - e->iter_before - ((u32)progress - (u32)e->iter_before);
    const u32 coming = (u32)enq - ((u32)(progress >> 32) - e->chains_before);
    const bool enough = limit != 0 && coming >= lacking;
    if (enq - done >= depth || (enough && enq > done)) {   // wait for the oldest one
      if (hipEventSynchronize(e->events[done % depth]) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
      harvest_phase_times(e, done);
      ++done;
      if (e->hmirror->error) { rc = BLINK_ERR_DEVICE; break; }
      if (__atomic_load_n(&e->hmirror->stopped, __ATOMIC_ACQUIRE)) break;
      if (e->host_step_bytes) {   // the previous iteration has ended: its tokens to the host, a batch description back
        const u64 tok_bytes = sizeof(i32) * (u64)e->ctx.max_batch;
        if (hipMemcpyAsync(e->host_step_h, e->ctx.input_ids, tok_bytes, hipMemcpyDeviceToHost, e->compute) != hipSuccess ||
            hipStreamSynchronize(e->compute) != hipSuccess ||
            hipMemcpyAsync(e->host_step_d, e->host_step_h, e->host_step_bytes, hipMemcpyHostToDevice, e->compute) != hipSuccess) {
          rc = BLINK_ERR_DEVICE;
          break;
        }
      }
      continue;
    }
    if (enough) break;                           // the window's iterations have run
    rc = enqueue_iteration(e, enq);
    if (rc == 0 && hipEventRecord(e->events[enq % depth], e->compute) != hipSuccess) rc = BLINK_ERR_DEVICE;
    ++enq;
  }
  if (hipStreamSynchronize(e->compute) != hipSuccess && rc == 0) rc = BLINK_ERR_DEVICE;
  if (rc == 0) for (u64 i = done; i < enq; ++i) harvest_phase_times(e, i);
  if (rc == 0 && e->hmirror->error) rc = BLINK_ERR_DEVICE;
  e->loop_rc.store(rc);
  e->loop_active.store(false, std::memory_order_release);
}

extern "C" int blink_run(blink_engine* e, uint64_t max_iterations) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  if (e->loop_active.load(std::memory_order_acquire)) return fail(BLINK_ERR_STATE, "the loop is already running");
  if (e->launcher.joinable()) e->launcher.join();
  HIPCHK(hipSetDevice(e->cfg.device));
  if (e->hmirror->error) return fail(BLINK_ERR_DEVICE, "device loop error %u", e->hmirror->error);
  e->iter_before = e->hmirror->iteration;
  const u64 iter_limit = max_iterations ? e->iter_before + max_iterations : 0;
  e->iter_limit = iter_limit;
  e->chains_before = (u32)(e->hmirror->progress >> 32);
  e->hmirror->stopped = 0;
  HIPCHK(launch(k_open_window, 1, 1, e->compute, e->ctx.ss, iter_limit));
  e->loop_active.store(true, std::memory_order_release);
  e->loop_rc.store(0);
  e->windows.fetch_add(1);
  e->phase_ms.clear();
  e->launcher = std::thread(pump_loop, e);
  return BLINK_OK;
}

extern "C" int blink_set_exit_when_idle(blink_engine* e, uint32_t on) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  if (e->loop_active.load(std::memory_order_acquire)) return fail(BLINK_ERR_STATE, "stop the loop first");
  __atomic_store_n(&e->hctrl->exit_when_idle, on ? 1u : 0u, __ATOMIC_RELEASE);
  return BLINK_OK;
}

extern "C" int blink_wait(blink_engine* e) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->launcher.joinable()) e->launcher.join();
  const int rc = e->loop_rc.load();
  if (rc) return fail(rc, "the loop ended with an error (device error %u)", e->hmirror ? e->hmirror->error : 0u);
  return BLINK_OK;
}

extern "C" int blink_poll_outputs(blink_engine* e, blink_event* buf, uint32_t cap, uint32_t* n_out) {
  g_err.clear();
  if (!e || !n_out || (!buf && cap)) return fail(BLINK_ERR_INVAL, "null argument");
  *n_out = 0;
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  const DevCtx& c = e->ctx;
  HIPCHK(hipSetDevice(e->cfg.device));
  u32 n_want = 0;
  for (u32 slot = 0; slot < c.ring_slots; ++slot)
    if (e->shadow_state[slot].load(std::memory_order_acquire) != 0) e->stage_want[n_want++] = OutWant{slot, (u32)e->slot_ticket[slot], e->delivered[slot], 0};
  if (n_want == 0 || cap == 0) return BLINK_OK;  // (no request is under way)
  HIPCHK(launch(k_poll_outputs, 1, BLK_THREADS, e->s_out, e->stage_want, n_want, c.status, c.out_arena, c.max_seq_len,
                (u32)std::min<u64>(cap, e->stage_out_cap), e->stage_out, e->stage_picks, e->stage_n_picks));
  HIPCHK(hipStreamSynchronize(e->s_out));
  const u32 n_picks = *e->stage_n_picks;
  u32 longest = 0;                               // of the slots whose records are still there
  for (u32 k = 0; k < n_picks; ++k)
    if (e->stage_picks[k].left) longest = std::max<u32>(longest, e->stage_picks[k].n);
  if (longest) {
    const u32 pieces = (longest + FETCH_PIECE - 1) / FETCH_PIECE;
    HIPCHK(launch(k_fetch_outputs, n_picks * pieces, BLK_THREADS, e->s_out, e->stage_picks, pieces, c.status, c.out_arena, c.max_seq_len, e->stage_out));
    HIPCHK(hipStreamSynchronize(e->s_out));
  }
  // events across requests ordered by (iteration, ring slot); per request by index
  u32 w = 0;
  for (u32 k = 0; k < n_picks; ++k) {
    const OutPick p = e->stage_picks[k];
    for (u32 i = 0; i < p.n; ++i) {
      const OutRec& r = e->stage_out[w];         // (the slots' records follow each other)
      blink_event& ev = buf[w++];
      ev.request_id = e->slot_ticket[p.slot];
      ev.index = p.from + i;
      ev.token = r.token;
      ev.flags = (ev.index == 0 ? BLINK_EVENT_FIRST : 0u) | ((p.completed && i + 1 == p.n) ? BLINK_EVENT_LAST : 0u);
      ev.iteration = r.iteration;
      ev.device_ns = r.device_ns;
    }
    e->delivered[p.slot] = p.from + p.n;
  }
  // completed slots are EMPTY on the device now, and become reusable here
  for (u32 k = 0; k < n_picks; ++k)
    if (e->stage_picks[k].completed) e->shadow_state[e->stage_picks[k].slot].store(0, std::memory_order_release);
  *n_out = w;
  return BLINK_OK;
}

extern "C" int blink_stop(blink_engine* e) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  __atomic_store_n(&e->hctrl->stop, 1u, __ATOMIC_RELEASE);
  if (e->launcher.joinable()) e->launcher.join();
  __atomic_store_n(&e->hctrl->stop, 0u, __ATOMIC_RELEASE);
  const int rc = e->loop_rc.load();
  if (rc) return fail(rc, "the loop ended with an error (device error %u)", e->hmirror->error);
  return BLINK_OK;
}

extern "C" int blink_shutdown(blink_engine* e) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  (void)hipSetDevice(e->cfg.device);
  e->shut = true;
  if (e->hctrl) __atomic_store_n(&e->hctrl->stop, 1u, __ATOMIC_RELEASE);
  if (e->launcher.joinable()) e->launcher.join();
  (void)hipDeviceSynchronize();
  free_all(e);
  return BLINK_OK;
}

// the most recent min(cap_records, records kept) trace records, oldest of them first
extern "C" int blink_get_trace(blink_engine* e, blink_trace_record* buf, uint64_t cap_records, uint64_t* n_out) {
  g_err.clear();
  if (!e || !n_out || (!buf && cap_records)) return fail(BLINK_ERR_INVAL, "null argument");
  static_assert(sizeof(blink_trace_record) == sizeof(TraceRec), "trace record layout");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop before reading the trace");
  HIPCHK(hipSetDevice(e->cfg.device));
  const u64 iters = e->hmirror->iteration;
  const u64 have = std::min<u64>(iters, e->ctx.trace_cap);
  const u64 n = std::min<u64>(have, cap_records);
  const u64 first = iters - n;
  for (u64 i = 0; i < n; ++i) {
    const u64 idx = (first + i) % e->ctx.trace_cap;
    const u64 run = std::min<u64>(n - i, e->ctx.trace_cap - idx);
    HIPCHK(hipMemcpy(buf + i, e->ctx.trace + idx, run * sizeof(TraceRec), hipMemcpyDeviceToHost));
    i += run - 1;
  }
  *n_out = n;
  return BLINK_OK;
}

extern "C" int blink_get_stats(blink_engine* e, blink_stats* out) {
  g_err.clear();
  if (!e || !out) return fail(BLINK_ERR_INVAL, "null argument");
  memset(out, 0, sizeof *out);
  out->running = e->loop_active.load() ? 1u : 0u;
  out->windows = e->windows.load();
  out->kv_bytes = e->kv_bytes; out->weight_bytes = e->weight_bytes; out->ring_bytes = e->ring_bytes;
  if (out->running) {   // only the host mirror is read while the loop is active
    out->iterations = e->hmirror->iteration;
    out->tokens_out = e->hmirror->tokens_out;
    out->n_running = e->hmirror->n_running;
    out->device_error = e->hmirror->error;
    return BLINK_OK;
  }
  HIPCHK(hipSetDevice(e->cfg.device));
  SchedState s;
  HIPCHK(hipMemcpy(&s, e->ctx.ss, sizeof s, hipMemcpyDeviceToHost));
  out->iterations = s.iteration; out->prefill_iterations = s.prefill_iterations; out->tokens_out = s.tokens_out;
  out->tokens_prefilled = s.tokens_prefilled; out->next_ticket = s.next_ticket; out->n_running = s.n_running;
  out->free_blocks = s.free_top - s.free_lo; out->committed_blocks = s.committed; out->device_error = s.error;
  out->prefix_hit_blocks = s.cache_hits; out->prefix_evictions = s.evictions; out->pinned_blocks = s.pinned; out->pad1 = 0;
  out->spec_drafted = s.drafted; out->spec_accepted = s.accepted;
  return BLINK_OK;
}

// Device memory into a caller's (pageable) buffer, in pieces through pinned memory: a piece is on its way over the bus while others are
// copied out of the staging buffer, by up to four threads where there is much of it, because most of the time is the first touch of the
// caller's pages. Each thread has its own places of the buffer and fills them again as it has copied them out, so that any size goes
// through the same few megabytes. Into new pages, as one hipMemcpy / like this: 8 MB .80 / .46 ms, 16.8 MB 3.4 / .87, 33 MB 5.9 / 1.6, 131 MB
// 21.8 / 6.1.
static hipError_t read_back(blink_engine* e, char* to, const char* from, u64 n) {
  const u32 pieces = (u32)((n + DBG_PIECE - 1) / DBG_PIECE), threads = std::min(DBG_THREADS, (pieces + 3) / 4), ahead = threads * DBG_SLOTS;
  auto slot = [=](u32 i) { return i % threads * DBG_SLOTS + i / threads % DBG_SLOTS; };
  auto place = [=](u32 i) { return e->stage_dbg + 1024 + (u64)slot(i) * DBG_PIECE; };
  auto bytes = [=](u32 i) { return std::min<u64>(DBG_PIECE, n - (u64)i * DBG_PIECE); };
  auto ask = [=](u32 i) -> hipError_t {
    const hipError_t er = hipMemcpyAsync(place(i), from + (u64)i * DBG_PIECE, bytes(i), hipMemcpyDeviceToHost, e->s_out);
    return er != hipSuccess ? er : hipEventRecord(e->dbg_ev[slot(i)], e->s_out);
  };
  auto part = [=](u32 t) -> hipError_t {         // pieces t, t + threads, .., of which the first DBG_SLOTS have been asked for
    hipError_t er = hipSetDevice(e->cfg.device);
    for (u32 i = t; i < pieces && er == hipSuccess; i += threads) {
      er = hipEventSynchronize(e->dbg_ev[slot(i)]);
      if (er != hipSuccess) break;
      memcpy(to + (u64)i * DBG_PIECE, place(i), bytes(i));
      if (i + ahead < pieces) er = ask(i + ahead);
    }
    return er;
  };
  hipError_t result[DBG_THREADS] = {};
  for (u32 i = 0; i < std::min(pieces, ahead) && result[0] == hipSuccess; ++i) result[0] = ask(i);
  if (result[0] == hipSuccess) {
    std::thread helpers[DBG_THREADS];
    for (u32 t = 1; t < threads; ++t) {
      try { helpers[t] = std::thread([&result, &part, t]() { result[t] = part(t); }); } catch (...) {}   // (no thread to be had: below)
    }
    result[0] = part(0);
    for (u32 t = 1; t < threads; ++t) {
      if (helpers[t].joinable()) helpers[t].join();
      else result[t] = part(t);
    }
  }
  for (hipError_t er : result)
    if (er != hipSuccess) { (void)hipStreamSynchronize(e->s_out); return er; }      // (nothing on its way into the staging buffer any more)
  return hipSuccess;
}

extern "C" int blink_debug_read(blink_engine* e, uint32_t what, void* buf, uint64_t cap_bytes, uint64_t* n_bytes) {
  g_err.clear();
  if (!e || !buf || !n_bytes) return fail(BLINK_ERR_INVAL, "null argument");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop before reading device state");
  HIPCHK(hipSetDevice(e->cfg.device));
  const DevCtx& c = e->ctx;
  std::lock_guard<std::mutex> lock(e->dbg_mu);
  // Both descriptions and, for the logits, the first rows come with one wait: a small result needs no other.
  IterMeta& m = *(IterMeta*)e->stage_dbg;
  SchedState& s = *(SchedState*)(e->stage_dbg + 512);
  static_assert(sizeof(IterMeta) <= 512 && sizeof(SchedState) <= 512, "staging layout");
  char* const data = e->stage_dbg + 1024;
  HIPCHK(hipMemcpyAsync(&m, c.meta, sizeof m, hipMemcpyDeviceToHost, e->s_out));
  HIPCHK(hipMemcpyAsync(&s, c.ss, sizeof s, hipMemcpyDeviceToHost, e->s_out));
  const u64 ahead = what == BLINK_DBG_LOGITS ? std::min<u64>(std::min<u64>(cap_bytes, DBG_AHEAD), (u64)c.max_batch * (c.spec_k + 1) * c.V * 4) : 0;
  if (ahead) HIPCHK(hipMemcpyAsync(data, c.logits, ahead, hipMemcpyDeviceToHost, e->s_out));
  HIPCHK(hipStreamSynchronize(e->s_out));
  const void* src = nullptr;
  u64 n = 0;
  switch (what) {
    case BLINK_DBG_LOGITS: src = c.logits; n = (u64)m.n_samples * c.V * 4; break;
    case BLINK_DBG_FREE_STACK: {
      const u32 count = s.free_top - s.free_lo;
      n = 4 + (u64)count * 4;
      if (n > cap_bytes) return fail(BLINK_ERR_INVAL, "buffer too small: need %llu bytes", (unsigned long long)n);
      memcpy(buf, &count, 4);
      std::vector<u32> ring((u64)c.fs_mask + 1);
      HIPCHK(hipMemcpy(ring.data(), c.free_stack, ring.size() * 4, hipMemcpyDeviceToHost));
      for (u32 i = 0; i < count; ++i) ((u32*)buf)[1 + i] = ring[(s.free_lo + i) & c.fs_mask];
      *n_bytes = n;
      return BLINK_OK;
    }
    case BLINK_DBG_INPUT_IDS: src = c.input_ids; n = (u64)m.n_tokens * 4; break;
    case BLINK_DBG_POSITIONS: src = c.positions; n = (u64)m.n_tokens * 4; break;
    case BLINK_DBG_SLOT_MAPPING: src = c.slot_mapping; n = (u64)m.n_tokens * 4; break;
    case BLINK_DBG_SEQ_BATCH_SLOT: src = c.seq_bslot; n = (u64)m.n_seqs * 4; break;
    case BLINK_DBG_BLOCK_TABLES: src = c.block_tables; n = (u64)c.max_batch * c.max_blocks_per_seq * 4; break;
    case BLINK_DBG_SEQ_LENS: src = c.seq_len; n = (u64)m.n_seqs * 4; break;
    case BLINK_DBG_CU_SEQLENS: src = c.cu_seqlens; n = ((u64)m.n_seqs + 1) * 4; break;
    case BLINK_DBG_SLOT_STATES: {
      n = (u64)c.ring_slots * 4;
      if (n > cap_bytes) return fail(BLINK_ERR_INVAL, "buffer too small: need %llu bytes", (unsigned long long)n);
      std::vector<SlotStatus> st(c.ring_slots);
      HIPCHK(hipMemcpy(st.data(), c.status, sizeof(SlotStatus) * c.ring_slots, hipMemcpyDeviceToHost));
      for (u32 i = 0; i < c.ring_slots; ++i) ((u32*)buf)[i] = st[i].state;
      *n_bytes = n;
      return BLINK_OK;
    }
    case BLINK_DBG_HIDDEN: src = c.x; n = (u64)m.n_tokens * c.d * 4; break;
    case BLINK_DBG_ROUTING: {
      if (!c.n_experts) return fail(BLINK_ERR_INVAL, "not a mixture-of-experts model");
      const u64 row = (u64)m.n_tokens * c.n_active * 4;
      n = row * c.n_layers;
      if (n > cap_bytes) return fail(BLINK_ERR_INVAL, "buffer too small: need %llu bytes", (unsigned long long)n);
      for (u32 l = 0; l < c.n_layers && row; ++l)
        HIPCHK(hipMemcpy((char*)buf + l * row, c.moe_sel + (u64)l * c.maxT * c.n_active, row, hipMemcpyDeviceToHost));
      *n_bytes = n;
      return BLINK_OK;
    }
    case BLINK_DBG_ATTN_ITEMS: {
      if (!c.chunk_rec) return fail(BLINK_ERR_INVAL, "not a bf16 model");
      static_assert(sizeof(ChunkRec) == 32, "work list record layout");
      n = (u64)m.n_chunks * sizeof(ChunkRec);
      if (n > cap_bytes) return fail(BLINK_ERR_INVAL, "buffer too small: need %llu bytes", (unsigned long long)n);
      const u64 n_first = (u64)m.n_full_chunks * sizeof(ChunkRec);
      if (n_first) HIPCHK(hipMemcpy(buf, c.chunk_rec, n_first, hipMemcpyDeviceToHost));
      if (n > n_first) HIPCHK(hipMemcpy((char*)buf + n_first, c.chunk_rec + c.chunk_cap, n - n_first, hipMemcpyDeviceToHost));
      *n_bytes = n;
      return BLINK_OK;
    }
    default: return fail(BLINK_ERR_INVAL, "unknown selector %u", what);
  }
  if (n > cap_bytes) return fail(BLINK_ERR_INVAL, "buffer too small: need %llu bytes", (unsigned long long)n);
  if (n && n <= ahead) memcpy(buf, data, n);
  else if (n) HIPCHK(read_back(e, (char*)buf, (const char*)src, n));
  *n_bytes = n;
  return BLINK_OK;
}

extern "C" int blink_time_phase(blink_engine* e, int32_t phase) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop first");
  if (phase < -1 || phase > PH_MOE_PERMUTE) return fail(BLINK_ERR_INVAL, "phase out of range");
  e->timed_phase = phase;
  return BLINK_OK;
}

extern "C" int blink_get_phase_times(blink_engine* e, float* ms_per_iteration, uint64_t cap, uint64_t* n_out) {
  g_err.clear();
  if (!e || !n_out || (!ms_per_iteration && cap)) return fail(BLINK_ERR_INVAL, "null argument");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop first");
  const u64 n = std::min<u64>(cap, e->phase_ms.size());
  for (u64 i = 0; i < n; ++i) ms_per_iteration[i] = e->phase_ms[i];
  *n_out = n;
  return BLINK_OK;
}

extern "C" int blink_calibration_copy(blink_engine* e, uint64_t bytes) {
  g_err.clear();
  if (!e) return fail(BLINK_ERR_INVAL, "null engine");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop first");
  void* src = e->calib_src;
  void* dst = e->calib_dst;
  const u64 cap = e->calib_bytes;
  if (bytes == 0 || bytes > cap || (bytes & 15)) return fail(BLINK_ERR_INVAL, "bytes must be a multiple of 16 in (0, %llu]", (unsigned long long)cap);
  HIPCHK(hipSetDevice(e->cfg.device));
  HIPCHK(launch(k_copy_calibration, e->grid * 4, BLK_THREADS, e->compute, (const uint4*)src, (uint4*)dst, bytes / 16));
  HIPCHK(hipStreamSynchronize(e->compute));
  return BLINK_OK;
}

extern "C" int blink_calibration_rates(blink_engine* e, double* copy_gbs, double* mfma_bf16_tflops, double* read_gbs) {
  g_err.clear();
  if (!e || !copy_gbs || !mfma_bf16_tflops || !read_gbs) return fail(BLINK_ERR_INVAL, "null argument");
  if (e->loop_active.load()) return fail(BLINK_ERR_STATE, "stop the loop first");
  HIPCHK(hipSetDevice(e->cfg.device));
  hipEvent_t t0, t1;
  HIPCHK(hipEventCreate(&t0));
  HIPCHK(hipEventCreate(&t1));
  // copy buffers of 1 GiB each, held only during this call: far larger than the 256 MB last-level cache, so the rate is HBM's
  const u64 copy_bytes = 1ull << 30, n16 = copy_bytes / 16;
  char *src = nullptr, *dst = nullptr;
  if (hipMalloc((void**)&src, copy_bytes) != hipSuccess || hipMalloc((void**)&dst, copy_bytes) != hipSuccess) {
    if (src) (void)hipFree(src);
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    (void)hipGetLastError();             // (the caller's next look must not find this one)
    return fail(BLINK_ERR_DEVICE, "no room for the two 1 GiB copy buffers");
  }
  const u32 rounds = 4096, wgs = e->grid * 2;        // the MFMA loop writes one float per lane: 1 MiB of the 64 MiB buffer
  float best_copy = 0.f, best_mfma = 0.f, best_read = 0.f;
  int rc = hipMemsetAsync(src, 0, copy_bytes, e->compute) == hipSuccess ? BLINK_OK : BLINK_ERR_DEVICE;
  for (int rep = 0; rep < 4 && rc == BLINK_OK; ++rep) {   // the first repetition warms up; the best of the rest counts
    float ms = 0.f;
    if (hipEventRecord(t0, e->compute) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (launch(k_copy_calibration, e->grid * 4, BLK_THREADS, e->compute, (const uint4*)src, (uint4*)dst, n16) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (hipEventRecord(t1, e->compute) != hipSuccess || hipEventSynchronize(t1) != hipSuccess || hipEventElapsedTime(&ms, t0, t1) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (rep && (best_copy == 0.f || ms < best_copy)) best_copy = ms;
    if (hipEventRecord(t0, e->compute) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (launch(k_mfma_calibration, wgs, BLK_THREADS, e->compute, (float*)e->calib_dst, rounds) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (hipEventRecord(t1, e->compute) != hipSuccess || hipEventSynchronize(t1) != hipSuccess || hipEventElapsedTime(&ms, t0, t1) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (rep && (best_mfma == 0.f || ms < best_mfma)) best_mfma = ms;
    if (hipEventRecord(t0, e->compute) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (launch(k_read_calibration, e->grid, BLK_THREADS, e->compute, (const uint4*)src, (u32*)e->calib_dst, n16) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (hipEventRecord(t1, e->compute) != hipSuccess || hipEventSynchronize(t1) != hipSuccess || hipEventElapsedTime(&ms, t0, t1) != hipSuccess) { rc = BLINK_ERR_DEVICE; break; }
    if (rep && (best_read == 0.f || ms < best_read)) best_read = ms;
  }
  (void)hipStreamSynchronize(e->compute);
  (void)hipFree(src);
  (void)hipFree(dst);
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  if (rc != BLINK_OK) return fail(BLINK_ERR_DEVICE, "calibration kernels failed");
  *copy_gbs = 2.0 * (double)(n16 * 16) / ((double)best_copy * 1e-3) / 1e9;   // bytes read + bytes written
  *read_gbs = (double)(n16 * 16) / ((double)best_read * 1e-3) / 1e9;
  *mfma_bf16_tflops = (double)wgs * (BLK_THREADS / 64) * rounds * 16.0 * (2.0 * 16 * 16 * 32) / ((double)best_mfma * 1e-3) / 1e12;
  return BLINK_OK;
}

static u64 host_now_ns() {
  return (u64)std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

extern "C" int blink_clock_sync(blink_engine* e, uint64_t* device_ns, uint64_t* host_ns, uint64_t* uncertainty_ns) {
  g_err.clear();
  if (!e || !device_ns || !host_ns || !uncertainty_ns) return fail(BLINK_ERR_INVAL, "null argument");
  if (e->shut) return fail(BLINK_ERR_STATE, "engine is shut down");
  std::lock_guard<std::mutex> lk(e->dev_mu);
  HIPCHK(hipSetDevice(e->cfg.device));
  u64 best_span = ~0ull;
  for (int rep = 0; rep < 8; ++rep) {
    __atomic_store_n(&e->hmirror->clock_probe, 0ull, __ATOMIC_RELEASE);
    const u64 h0 = host_now_ns();
    HIPCHK(launch(k_clock_probe, 1, 1, e->s_in, e->hmirror));   // not the compute stream: the loop may be running there
    u64 dv = 0, h1 = h0;
    while ((dv = __atomic_load_n(&e->hmirror->clock_probe, __ATOMIC_ACQUIRE)) == 0) {
      h1 = host_now_ns();
      if (h1 - h0 > 2000000000ull) return fail(BLINK_ERR_DEVICE, "the clock probe kernel did not run within 2 s");
    }
    h1 = host_now_ns();
    HIPCHK(hipStreamSynchronize(e->s_in));
    // the device read its clock somewhere between h0 and h1; the launch takes most of that span, so the read is
    // placed at its end, and the whole span is reported as the uncertainty
    if (h1 - h0 < best_span) { best_span = h1 - h0; *device_ns = dv; *host_ns = h1; *uncertainty_ns = h1 - h0; }
  }
  return BLINK_OK;
}

// ---- stand-alone sampler ------------------------------------------------------------------------------------
static int sample_rows_check(const float* logits, uint32_t n_rows, uint32_t vocab, const blink_sampling* params,
                             const uint32_t* token_index, int32_t* tokens_out) {
  if (!logits || !params || !token_index || !tokens_out) return fail(BLINK_ERR_INVAL, "null argument");
  if (n_rows == 0 || vocab == 0 || vocab >= (1u << 24)) return fail(BLINK_ERR_INVAL, "n_rows must be positive and vocab in [1, 2^24)");
  for (u32 r = 0; r < n_rows; ++r) {
    const blink_sampling& sp = params[r];
    if (!(sp.temperature >= 0.f) || !(sp.top_p > 0.f && sp.top_p <= 1.f)) return fail(BLINK_ERR_INVAL, "row %u: temperature must be >= 0 and top_p in (0,1]", r);
    if (sp.temperature > 0.f && (sp.top_k == 0 || sp.top_k > SAMPLER_MAX_K) && vocab > SAMPLER_MAX_K)
      return fail(BLINK_ERR_INVAL, "row %u: sampling needs top_k in [1, %d] when vocab exceeds %d", r, SAMPLER_MAX_K, SAMPLER_MAX_K);
  }
  return BLINK_OK;
}

// Device staging of one call, 256-byte aligned parts: logits rows, parameters, output indices, tokens.
struct SampleStaging { u64 params, index, tokens, total; };
static SampleStaging sample_staging(uint32_t n_rows, uint32_t vocab) {
  auto pad = [](u64 b) { return (b + 255) & ~255ull; };
  SampleStaging s;
  s.params = pad((u64)n_rows * vocab * 4);
  s.index = s.params + pad((u64)n_rows * sizeof(blink_sampling));
  s.tokens = s.index + pad((u64)n_rows * 4);
  s.total = s.tokens + pad((u64)n_rows * 4);
  return s;
}

// copies the rows and their parameters into the staging memory at `dev`, samples, copies the tokens back
static int sample_rows_on(char* dev, hipStream_t st, const float* logits, uint32_t n_rows, uint32_t vocab, const blink_sampling* params,
                          const uint32_t* token_index, int32_t* tokens_out) {
  static_assert(sizeof(blink_sampling) == sizeof(SampleRowParams), "the kernel reads blink_sampling as it is");
  const SampleStaging s = sample_staging(n_rows, vocab);
  HIPCHK(hipMemcpyAsync(dev, logits, (u64)n_rows * vocab * 4, hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(dev + s.params, params, (u64)n_rows * sizeof(blink_sampling), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(dev + s.index, token_index, (u64)n_rows * 4, hipMemcpyHostToDevice, st));
  HIPCHK(launch(k_sample_rows, std::min<u32>(n_rows, 1024u), BLK_THREADS, st, (const float*)dev, n_rows, vocab,
                (const SampleRowParams*)(dev + s.params), (const u32*)(dev + s.index), (i32*)(dev + s.tokens)));
  HIPCHK(hipMemcpyAsync(tokens_out, dev + s.tokens, (u64)n_rows * 4, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  return BLINK_OK;
}

extern "C" int blink_sample_rows(int32_t device, const float* logits, uint32_t n_rows, uint32_t vocab, const blink_sampling* params,
                                 const uint32_t* token_index, int32_t* tokens_out) {
  g_err.clear();
  if (int rc = sample_rows_check(logits, n_rows, vocab, params, token_index, tokens_out)) return rc;
  int n_dev = 0;
  if (hipGetDeviceCount(&n_dev) != hipSuccess || n_dev <= 0) return fail(BLINK_ERR_DEVICE, "no HIP device available");
  if (device < 0 || device >= n_dev) return fail(BLINK_ERR_INVAL, "device %d out of range", device);
  HIPCHK(hipSetDevice(device));
  char* dev = nullptr;
  HIPCHK(hipMalloc((void**)&dev, sample_staging(n_rows, vocab).total));
  const int rc = sample_rows_on(dev, nullptr, logits, n_rows, vocab, params, token_index, tokens_out);
  const std::string keep = g_err;
  (void)hipFree(dev);
  g_err = keep;
  return rc;
}

// ---- the same without any allocation: the staging lives in a static device array ------------------------------------
#define SAMPLE_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[SAMPLE_SCRATCH_BYTES];
#define SAMPLE_MAX_DEVICES 64
static std::mutex g_scratch_mu;                          // one call at a time per process: the calls share the array
static char* g_scratch_ptr[SAMPLE_MAX_DEVICES] = {};     // device address of `scratch` on every device used so far

extern "C" int blink_sample_rows_static(int32_t device, const float* logits, uint32_t n_rows, uint32_t vocab, const blink_sampling* params,
                                        const uint32_t* token_index, int32_t* tokens_out) {
  g_err.clear();
  if (int rc = sample_rows_check(logits, n_rows, vocab, params, token_index, tokens_out)) return rc;
  const u64 need = sample_staging(n_rows, vocab).total;
  if (need > SAMPLE_SCRATCH_BYTES)
    return fail(BLINK_ERR_TOO_LARGE, "%u rows of %u logits need %llu bytes of staging, the static buffer holds %u", n_rows, vocab,
                (unsigned long long)need, (unsigned)SAMPLE_SCRATCH_BYTES);
  int n_dev = 0;
  if (hipGetDeviceCount(&n_dev) != hipSuccess || n_dev <= 0) return fail(BLINK_ERR_DEVICE, "no HIP device available");
  if (device < 0 || device >= n_dev || device >= SAMPLE_MAX_DEVICES) return fail(BLINK_ERR_INVAL, "device %d out of range", device);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  HIPCHK(hipSetDevice(device));
  if (!g_scratch_ptr[device]) {   // every device holds its own copy of the array at its own address
    char* p = nullptr;
    HIPCHK(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(BLINK_ERR_DEVICE, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[device] = p;
  }
  return sample_rows_on(g_scratch_ptr[device], nullptr, logits, n_rows, vocab, params, token_index, tokens_out);
}

extern "C" const char* blink_last_error(void) { return g_err.c_str(); }
