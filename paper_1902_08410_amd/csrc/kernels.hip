// HIP kernels of libdpsnn for gfx950 (64-lane wavefronts).
//
//  k_gen      one wavefront per source row: draws the K_out synapses of the
//             source from Philox (blocks of synapses per target population,
//             Eq. 1 targets, uniform delay, quantile-table efficacy), sorts
//             them by (delay, target, draw index) in LDS and writes the row
//             and the start of each delay's segment.  The delay index rides
//             in the top 6 bits of each target word.
//  k_init     initial membrane potentials, fatigue and refractory counters.
//  k_rows     rows back in reading order, (target, delay, draw index).
//  k_neuron   one step of dt for a tile of 1024 neurons (4 per thread): the
//             tile's inbox summed in LDS, the input slot read and cleared
//             where marked, external Poisson drive, Eq. 2 update, threshold,
//             5 ms population counts; the tile's spikes are listed for the log
//             and their row segments entered in the lists of their arrival
//             steps.
//  k_deliver  the events that arrive in the next step: blocks share the pieces
//             of the list that is due evenly, sort their events by target tile
//             (an LDS hash, one returning atomic per tile) and store them in
//             the target tiles' inboxes.  Other blocks append the spike log
//             and, for plastic networks, register the activations (without
//             inboxes: add the events into the slots).
//  k_step     fused schedule, one launch per step: some blocks deliver the list
//             that is due while the others update two tiles each.
//  k_persist  the split schedule's work for many steps in one cooperative launch.
//  k_tick     the step counter after a run, and the log of its last fused step.
//  k_drain    folds pending events into the slots (inspection, and before
//             the efficacies of a plastic network change).
//  k_stdp_update  the periodic efficacy update of plastic networks.
//
// Events are delivered when they arrive, not when they are emitted: rows are
// sorted by (delay, target), a spike enters its row's segments, cut into
// pieces, in the lists of the steps they arrive in, and at step t the list of
// step t + 1 is written into the inboxes read at t + 1.  An event moves
// once (row -> inbox -> sum) and its inbox entry needs no delay.  Events
// that find an inbox full are added into the slot of the next step with an
// atomic, pieces that find a list full into the slot of their arrival, and the
// (tile, slot) is marked so that the update reads that slot.
// Every path sums integers, so the result does not depend on the path or
// the order.
//
// Inboxes have two parities, so that in the fused schedule the deliveries of
// step t fill one while the updates of step t empty the other; the kernel
// boundary orders consecutive steps.  The step index is read on the device
// (t = *t_base + t_off) so that launches can be captured in a graph.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "dpsnn_internal.h"
#include "philox.h"

namespace dpsnn {

// ------------------------------------------------------------------------
// LDS written by some lanes of a wavefront and read by others: the hardware
// performs one wavefront's LDS operations in order, so only the compiler
// must not move them across this point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix of v over the wavefront's lanes, by cross-lane moves in the
// vector unit (rows of 16 lanes, then across the rows).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Clang vector type for the non-temporal loads and stores.
typedef float NtF4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS only: global loads and stores issued
// before it stay in flight (a full __syncthreads waits for all of them).
// Used where threads share data through LDS alone.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Step index and residues of the launch for step t_base + o.t_off: one
// 16-byte uniform load, then conditional subtractions (each residue sum is
// below twice its modulus; the bin sum below 2 cap + 1).
__device__ __forceinline__ StepTime step_time(const StepArgs& a, const StepOff& o) {
  const uint4 c = *reinterpret_cast<const uint4*>(a.t_base);
  StepTime T;
  T.t = c.x + o.t_off;
  uint32_t sl = c.y + o.d_slot;
  if (sl >= (uint32_t)a.D) sl -= (uint32_t)a.D;
  T.slot = sl;
  const uint32_t carry = c.z + o.d_phase >= (uint32_t)a.rate_bin_steps ? 1u : 0u;
  uint32_t b = c.w + o.d_bin + carry;
  if (b >= (uint32_t)a.rate_bins_cap) b -= (uint32_t)a.rate_bins_cap;
  if (b >= (uint32_t)a.rate_bins_cap) b -= (uint32_t)a.rate_bins_cap;
  T.bin = b;
  return T;
}

// Module and population of global neuron id.
__device__ __forceinline__ void module_pop(const StepArgs& a, int32_t id, int32_t* mod,
                                           int* pop) {
  const NetDev& nd = a.nets[a.tile_net[id >> 10]];
  const uint32_t local = (uint32_t)(id - (int32_t)nd.base);
  const uint32_t m = module_of(nd, local);
  *mod = nd.mbase + (int32_t)m;
  const int32_t l = (int32_t)(local - m * (uint32_t)nd.K);
  *pop = (l >= nd.pop_hi[0]) + (l >= nd.pop_hi[1]) + (l >= nd.pop_hi[2]);
}

// Population of neuron id of tile `tile` (uniform: its network's constants come
// by scalar loads).
__device__ __forceinline__ uint32_t pop_in_tile(const StepArgs& a, int tile, int32_t id) {
  const NetDev& nd = a.nets[__builtin_amdgcn_readfirstlane(a.tile_net[tile])];
  const uint32_t local = (uint32_t)(id - (int32_t)nd.base);
  const int32_t l = (int32_t)(local - module_of(nd, local) * (uint32_t)nd.K);
  return (uint32_t)((l >= nd.pop_hi[0]) + (l >= nd.pop_hi[1]) + (l >= nd.pop_hi[2]));
}

// ------------------------------------------------------------------------
// Connectivity generation
__host__ __device__ inline int gen_pow2(int Ko) {
  int P = 64;
  while (P < Ko) P <<= 1;
  return P;
}
__host__ __device__ inline int gen_stage_bytes(int Ko) {
  // sort keys (8 per slot of the power-of-two sort) + efficacy index (2) +
  // block (1) + a counter per delay
  return gen_pow2(Ko) * 8 + ((3 * Ko + 15) / 16) * 16 + 64 * 4;
}

// Bitonic sort of P (a power of two) keys in LDS by NT threads (one wavefront,
// or a block), ascending.
template <int NT>
__device__ __forceinline__ void lds_sort(uint64_t* key, int P, int tid) {
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int q = tid; q < P / 2; q += NT) {
        const int lo = 2 * q - (q & (stride - 1));
        const int hi = lo + stride;
        const uint64_t x = key[lo], y = key[hi];
        if ((x > y) == ((lo & size) == 0)) {
          key[lo] = y;
          key[hi] = x;
        }
      }
      if (NT == 64)
        wave_lds_sync();
      else
        __syncthreads();
    }
  }
}

template <int WDT>
__global__ void __launch_bounds__(256) k_gen(GenArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wpb = blockDim.x >> 6;
  const int64_t s = (int64_t)blockIdx.x * wpb + wave;
  if (s >= a.N) return;  // whole wavefronts only: no block barrier below
  const int Ko = a.K_out;
  const int P = gen_pow2(Ko);

  unsigned char* base = smem + (size_t)wave * gen_stage_bytes(Ko);
  uint64_t* st_key = reinterpret_cast<uint64_t*>(base);
  uint16_t* st_w = reinterpret_cast<uint16_t*>(base + (size_t)P * 8);
  uint8_t* st_b = reinterpret_cast<uint8_t*>(st_w + Ko);
  uint32_t* st_cnt = reinterpret_cast<uint32_t*>(base + gen_stage_bytes(Ko)) - 64;  // by delay

  const int32_t ls = (int32_t)(s % a.K);
  const int32_t ms = (int32_t)(s / a.K);
  const int pop = (ls >= a.pop_hi[0]) + (ls >= a.pop_hi[1]) + (ls >= a.pop_hi[2]);
  const int xs = ms % a.W, ys = ms / a.W;

  // The keys are sorted by (target, delay, j) where the sums of |efficacy| per
  // target are taken (int32 inputs), so that neighbouring lanes add to
  // neighbouring targets, and the row is then written in (delay, target, j)
  // order by a stable counting sort on the delay (48x48, two networks of
  // 2.88 G synapses: build 275 ms, and 313 with the keys in row order); else
  // the keys are in row order and written as they stand (96x96, int8: 316 ms,
  // and 352 by the counting sort).
  const int tgt_sh = a.absum ? 18 : 12, del_sh = a.absum ? 12 : 38;

  // draw synapse j of block b
  for (int j = lane; j < P; j += 64) {
    uint64_t key = ~0ull;
    if (j < Ko) {
      int b = 0;
      while (b + 1 < a.n_blk[pop] && j >= a.blk_end[pop][b]) ++b;
      const int lo = a.blk_lo[pop][b], size = a.blk_hi[pop][b] - lo;
      const int rule = a.blk_rule[pop][b];
      uint4 u;
      int32_t mt = ms;
      uint32_t nu;  // the word that picks the neuron
      if (rule == kRuleOwn) {
        u = philox10(make_uint4((uint32_t)s, (uint32_t)j, 0u, kTagSyn), a.key0, a.key1);
        nu = u.x;
      } else {
        // Eq. 1: module offset from word 0; with open edges a draw that
        // leaves the grid is repeated with counter word 2 = attempt
        for (uint32_t att = 0;; ++att) {
          u = philox10(make_uint4((uint32_t)s, (uint32_t)j, att, kTagSyn), a.key0, a.key1);
          int lo2 = 0, hi2 = a.n_off - 1;  // first threshold above u.x
          while (lo2 < hi2) {
            const int mid = (lo2 + hi2) >> 1;
            if (a.off_thr[mid] <= u.x)
              lo2 = mid + 1;
            else
              hi2 = mid;
          }
          int xt = xs + a.off_xy[2 * lo2];
          int yt = ys + a.off_xy[2 * lo2 + 1];
          if (!a.open) {
            if (xt >= a.W) xt -= a.W;
            if (yt >= a.H) yt -= a.H;
          }
          if (xt >= 0 && xt < a.W && yt >= 0 && yt < a.H) {
            mt = yt * a.W + xt;
            break;
          }
          if (att + 1 == (uint32_t)kMaxAttempts) break;  // own module
        }
        nu = u.y;
      }
      uint32_t r;
      if (mt == ms && ls >= lo && ls < lo + size) {  // no autapse
        r = scale32(nu, (uint32_t)(size - 1));
        r += r >= (uint32_t)(ls - lo) ? 1u : 0u;
      } else {
        r = scale32(nu, (uint32_t)size);
      }
      const int32_t tg = mt * a.K + lo + (int32_t)r;
      const uint32_t k = scale32(u.z, (uint32_t)a.n_del);
      st_w[j] = (uint16_t)(u.w >> 16);
      st_b[j] = (uint8_t)b;
      key = ((uint64_t)(uint32_t)tg << tgt_sh) | ((uint64_t)k << del_sh) | (uint64_t)j;
    }
    st_key[j] = key;
  }
  st_cnt[lane] = 0;
  wave_lds_sync();
  // the keys are distinct; the padding keys sort last
  lds_sort<64>(st_key, P, lane);
  if (a.absum) {
    for (int pos = lane; pos < Ko; pos += 64)
      atomicAdd(&st_cnt[(st_key[pos] >> del_sh) & 63u], 1u);
    wave_lds_sync();
    const uint32_t own = st_cnt[lane];
    uint32_t incl = own;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t x = __shfl_up(incl, off);
      if (lane >= off) incl += x;
    }
    wave_lds_sync();
    st_cnt[lane] = incl - own;
  } else {
    int l = 0, h = Ko;  // first key of delay index >= lane
    while (l < h) {
      const int mid = (l + h) >> 1;
      if ((int)((st_key[mid] >> del_sh) & 63u) < lane)
        l = mid + 1;
      else
        h = mid;
    }
    st_cnt[lane] = (uint32_t)l;
  }
  wave_lds_sync();
  // first synapse of each delay
  for (int k = lane; k <= a.n_del; k += 64)
    a.row_off[s * (a.n_del + 1) + k] = (uint16_t)(k < 64 ? st_cnt[k] : (uint32_t)Ko);
  const int64_t rb = s * a.row_stride;
  for (int p0 = 0; p0 < Ko; p0 += 64) {
    const int pos = p0 + lane;
    const bool on = pos < Ko;
    const uint64_t key = on ? st_key[pos] : 0ull;
    const int32_t tg = (int32_t)((key >> tgt_sh) & (uint64_t)kTargetMask);
    const int k = (int)((key >> del_sh) & 63u);
    int64_t o = rb + pos;
    if (a.absum) {
      // lanes with the same delay
      unsigned long long same = __ballot(on);
      for (int bit = 0; bit < 6; ++bit) {
        const unsigned long long set = __ballot((k >> bit) & 1);
        same &= (k >> bit) & 1 ? set : ~set;
      }
      const int rank = __popcll(same & ((1ull << lane) - 1));
      o = rb + (on ? st_cnt[k] : 0u) + rank;
      wave_lds_sync();
      if (on && rank == 0) st_cnt[k] += (uint32_t)__popcll(same);
      wave_lds_sync();
    }
    if (!on) continue;
    const uint16_t wi = st_w[key & 4095u];
    const int b = st_b[key & 4095u];
    const int32_t gt = tg + (int32_t)a.tgt_base;  // global target index
    a.tgt[o] = gt | (k << kDelayShift);
    if (WDT == DPSNN_W_F32)
      static_cast<float*>(a.w)[o] = static_cast<const float*>(a.wtab[pop][b])[wi];
    else if (WDT == DPSNN_W_F16)
      static_cast<uint16_t*>(a.w)[o] = static_cast<const uint16_t*>(a.wtab[pop][b])[wi];
    else
      static_cast<int8_t*>(a.w)[o] = static_cast<const int8_t*>(a.wtab[pop][b])[wi];
    if (a.absum) {
      const int64_t f = a.wfix_tab[pop][b][wi];
      atomicAdd(&a.absum[gt], (unsigned long long)(f < 0 ? -f : f));
    }
  }
  for (int j = Ko + lane; j < a.row_stride; j += 64) {
    a.tgt[rb + j] = 0;
    if (WDT == DPSNN_W_F32)
      static_cast<float*>(a.w)[rb + j] = 0.f;
    else if (WDT == DPSNN_W_F16)
      static_cast<uint16_t*>(a.w)[rb + j] = 0;
    else
      static_cast<int8_t*>(a.w)[rb + j] = 0;
  }
}

// Rows in the order they are read in, (target, delay, draw index): a block per
// row sorts the row's words in LDS (they are stored by (delay, target, draw
// index), so equal words keep their order by place) and copies the word and
// one value per synapse, of 1, 2 or 4 bytes.  (One row of 1000 synapses read
// back: 79 us with one wavefront a row, 45 so.)
constexpr int kRowThreads = 256;
template <typename T>
__global__ void __launch_bounds__(kRowThreads) k_rows(const int32_t* tgt, const T* val,
                                                      int row_stride, int Ko, int32_t* out_tgt,
                                                      T* out_val) {
  extern __shared__ __align__(16) uint64_t s_key[];
  const int P = gen_pow2(Ko);
  const int64_t rb = (int64_t)blockIdx.x * row_stride, ob = (int64_t)blockIdx.x * Ko;
  for (int j = threadIdx.x; j < P; j += kRowThreads) {
    const int32_t w = j < Ko ? tgt[rb + j] : 0;
    s_key[j] = j < Ko ? (uint64_t)(w & kTargetMask) << 18 |
                            (uint64_t)((uint32_t)w >> kDelayShift) << 12 | (uint64_t)j
                      : ~0ull;
  }
  __syncthreads();
  lds_sort<kRowThreads>(s_key, P, threadIdx.x);
  for (int j = threadIdx.x; j < Ko; j += kRowThreads) {
    const uint64_t key = s_key[j];
    out_tgt[ob + j] = (int32_t)(key >> 18) | (int32_t)((uint32_t)(key >> 12 & 63u) << kDelayShift);
    if (val) out_val[ob + j] = val[rb + (int)(key & 4095u)];
  }
}

__global__ void k_absum_max(const unsigned long long* v, int64_t n,
                            unsigned long long* out) {
  unsigned long long m = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    m = v[i] > m ? v[i] : m;
  atomicMax(out, m);
}

// ------------------------------------------------------------------------
// Initial state: V uniform on [E, V_th) from (i, 0, 0, INIT), c = 0, ref = 0.
__global__ void k_init(InitArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.N_pad) return;
  float V = 0.f;
  if (i < a.N) {
    const int l = (int)(i % a.K);
    const int q = (l >= a.pop_hi[0]) + (l >= a.pop_hi[1]) + (l >= a.pop_hi[2]);
    const uint4 u = philox10(make_uint4((uint32_t)i, 0u, 0u, kTagInit), a.key0, a.key1);
    const float f = (float)(u.x >> 8) * 0x1p-24f;
    V = a.E[q] + (a.Vth[q] - a.E[q]) * f;
  }
  a.V[i] = V;
  a.c[i] = 0.f;
  a.ref[i] = 0;
}

// ------------------------------------------------------------------------
// Fixed-point helpers

// Input sum in mV: one rounding of I * 2^-Q to binary32 (an int64 sum below
// 2^53 converts to binary64 exactly first).
__device__ __forceinline__ float fix_to_f32(int32_t v) { return (float)v; }
__device__ __forceinline__ float fix_to_f32(int64_t v) { return (float)(double)v; }

template <typename Acc>
__device__ __forceinline__ void atomic_add_fix(Acc* p, Acc v);
template <>
__device__ __forceinline__ void atomic_add_fix<int32_t>(int32_t* p, int32_t v) {
  atomicAdd(p, v);
}
template <>
__device__ __forceinline__ void atomic_add_fix<int64_t>(int64_t* p, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v);
}

template <typename Acc>
__device__ __forceinline__ void lds_add(Acc* p, Acc v);
template <>
__device__ __forceinline__ void lds_add<int32_t>(int32_t* p, int32_t v) {
  atomicAdd(p, v);
}
template <>
__device__ __forceinline__ void lds_add<int64_t>(int64_t* p, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v);
}

// Fixed-point efficacy of a code entry, computed as delivery computes it
// from the stored code (same conversions, same int8 scale).
template <typename Acc>
struct CodeDec {
  float two_q;
  int f16;
  Acc sc[kMaxPops];  // int8 scale of each source population of the network
  __device__ __forceinline__ Acc operator()(uint32_t e) const {
    const uint32_t code = e >> kCodeShift;
    if (f16) {
      __half_raw r;
      r.x = (unsigned short)code;
      return (Acc)__builtin_rintf(__half2float(__half(r)) * two_q);
    }
    const Acc q = (Acc)(int8_t)(uint8_t)(code & 0xFFu);
    const uint32_t pop = (code >> 8) & 3u;
    const Acc s = pop == 0u ? sc[0] : pop == 1u ? sc[1] : pop == 2u ? sc[2] : sc[3];
    return q * s;
  }
};

// Decoder for the entries of tile `tile` (uniform loads).
template <typename Acc>
__device__ __forceinline__ CodeDec<Acc> code_dec(const StepArgs& a, int tile) {
  CodeDec<Acc> d;
  d.two_q = a.two_q;
  d.f16 = a.q_code == kCodeF16;
#pragma unroll
  for (int q = 0; q < kMaxPops; ++q) d.sc[q] = 0;
  if (a.q_code == kCodeI8) {
    const int64_t b = (int64_t)a.P * a.nets[a.tile_net[tile]].mbase;
#pragma unroll
    for (int q = 0; q < kMaxPops; ++q)
      if (q < a.P) d.sc[q] = (Acc)a.sfix[b + q];
  }
  return d;
}

// Entry views: the in-tile index (x) and the fixed-point efficacy (w) of
// each format.
struct PackedEntry {
  uint32_t v;
};
struct CodeEntry {
  uint32_t v;
};
template <typename Acc>
__device__ __forceinline__ uint32_t ent_x(const QEntry<Acc>& e) { return e.x(); }
__device__ __forceinline__ uint32_t ent_x(PackedEntry e) { return e.v & 1023u; }
__device__ __forceinline__ uint32_t ent_x(CodeEntry e) { return e.v & 0xFFFFu; }
template <typename Acc>
__device__ __forceinline__ Acc ent_w(const QEntry<Acc>& e, const CodeDec<Acc>&) {
  return e.w();
}
template <typename Acc>
__device__ __forceinline__ Acc ent_w(PackedEntry e, const CodeDec<Acc>&) {
  return (Acc)((int32_t)e.v >> 10);
}
template <typename Acc>
__device__ __forceinline__ Acc ent_w(CodeEntry e, const CodeDec<Acc>& d) {
  return d(e.v);
}

// The update takes 256 threads per tile; a block of the fused schedule updates
// two tiles.
__device__ __forceinline__ int tile_tid() { return (int)threadIdx.x & 255; }

// The inbox of one tile.  The update of step t sums the events that arrive
// at t from the tile's inbox of parity t & 1, which the deliveries of step
// t - 1 filled, and empties it.  Entries are loaded kQBatch per thread at a
// time before any is used, so that their memory latency is paid once.
constexpr int kQBatch = 8;

// Packed entry (int32 inputs whose efficacies all fit 21 bits): fixed-point
// efficacy << 10 | in-tile index.
__device__ __forceinline__ uint32_t pack_entry(int32_t w, uint32_t idx) {
  return ((uint32_t)w << 10) | idx;
}

// Entry formats of the inboxes, fixed per kernel instance: QEntry, packed
// entries or code entries.
constexpr int kFmtWide = 0;
constexpr int kFmtPacked = 1;
constexpr int kFmtCode = 2;

template <typename Acc, typename E>
__device__ __forceinline__ void gather_batches(const E* iq, uint32_t n_in, Acc* s_in,
                                               const CodeDec<Acc>& dec) {
  const int tid = tile_tid(), nth = 256;
  for (uint32_t r0 = 0; r0 < n_in; r0 += (uint32_t)nth * kQBatch) {
    E e[kQBatch];
#pragma unroll
    for (int u = 0; u < kQBatch; ++u) {
      const uint32_t k = r0 + (uint32_t)(u * nth + tid);
      if (k < n_in) e[u] = iq[k];
    }
#pragma unroll
    for (int u = 0; u < kQBatch; ++u) {
      const uint32_t k = r0 + (uint32_t)(u * nth + tid);
      if (k < n_in) lds_add<Acc>(&s_in[ent_x(e[u]) & 1023u], ent_w<Acc>(e[u], dec));
    }
  }
}

template <typename Acc, int FMT>
__device__ __forceinline__ void gather_now(const StepArgs& a, int tile, const StepTime& T,
                                           Acc* s_in) {
  const int tid = tile_tid(), nth = 256;
  const int64_t box = (int64_t)(T.t & 1u) * a.n_tiles + tile;
  const uint32_t got = a.in_cnt[box * kInboxStride];
  const uint32_t n_in = got < (uint32_t)a.in_cap ? got : (uint32_t)a.in_cap;
  for (int k = tid; k < 1024; k += nth) s_in[k] = 0;
  lds_barrier();
  const int64_t io = box * a.in_stride;
  if constexpr (FMT == kFmtCode) {
    gather_batches<Acc>(static_cast<const CodeEntry*>(a.in_q) + io, n_in, s_in,
                        code_dec<Acc>(a, tile));
  } else {
    const CodeDec<Acc> none{};
    if constexpr (FMT == kFmtPacked)
      gather_batches<Acc>(static_cast<const PackedEntry*>(a.in_q) + io, n_in, s_in, none);
    else
      gather_batches<Acc>(static_cast<const QEntry<Acc>*>(a.in_q) + io, n_in, s_in, none);
  }
  lds_barrier();
  // every thread has used the count and the slot mark: the inbox is empty
  // and the slot cleared now
  if (tid == 0) {
    a.in_cnt[box * kInboxStride] = 0;
    a.s_dirty[(int64_t)tile * a.D + T.slot] = 0u;
  }
}


// Entry q of a four-entry array of uniform values, without indexing; the
// update is compiled for NP = 2 populations (q in 0..1) or up to 4.
template <int NP, typename T>
__device__ __forceinline__ T sel(const T (&v)[kMaxPops], int q) {
  if (NP == 2) return q ? v[1] : v[0];
  return q == 0 ? v[0] : q == 1 ? v[1] : q == 2 ? v[2] : v[3];
}

// Population of module-local index l from the ends h[0..2] of the first
// three populations.
template <int NP>
__device__ __forceinline__ int pop_index(int l, int h0, int h1, int h2) {
  if (NP == 2) return l >= h0 ? 1 : 0;
  return (l >= h0) + (l >= h1) + (l >= h2);
}

// ------------------------------------------------------------------------
// Neuron update of the 4 neurons i0..i0+3 (global indices) of one thread at
// step t; nd is the tile's network.  neuron_load reads and clears the input
// slot, reads the state and adds the external drive; neuron_finish adds the
// inbox sums (s_in, may be null), integrates Eq. 2 and returns the
// spiking neurons as a mask (compact_spikes lists them).  Counters of the random draws
// use the network's own neuron indices, so a network in a batch draws what
// it draws alone.
template <typename Acc>
struct NeuronRegs {
  Acc I[4];
  float V[4], c[4];
  uint32_t r4;
};

// Where the four neurons of a thread sit: global index i0 of the first,
// its network-local index il0 (a multiple of 4), and the module and
// module-local index of il0.
struct NeuronPos {
  uint32_t i0, il0, m0;
  int l0;
};

__device__ __forceinline__ NeuronPos neuron_pos(const NetDev& nd, int tile, int tid) {
  NeuronPos P;
  P.i0 = ((uint32_t)tile * 256u + (uint32_t)tid) * 4u;
  P.il0 = P.i0 - (uint32_t)nd.base;
  P.m0 = module_of(nd, P.il0);
  P.l0 = (int)(P.il0 - P.m0 * (uint32_t)nd.K);
  return P;
}

template <typename Acc, int NP>
__device__ __forceinline__ void neuron_load(const StepArgs& a, const NetDev& nd, int net,
                                            const NeuronPos& P, const StepTime& T,
                                            NeuronRegs<Acc>& R) {
  const uint32_t i0 = P.i0, t = T.t;
  Acc* sl = static_cast<Acc*>(a.slots) + ((size_t)T.slot * (size_t)a.N_pad + i0);
  // with inboxes the slot holds input only where an event found a list or inbox
  // full (marked per tile and slot); gather_now clears the mark
  const bool marked = a.q_cap == 0 || a.s_dirty[(i0 >> 10) * (uint32_t)a.D + T.slot] != 0u;
  if (!marked) {
#pragma unroll
    for (int j = 0; j < 4; ++j) R.I[j] = 0;
  } else if (sizeof(Acc) == 4) {
    const int4 v = *reinterpret_cast<const int4*>(sl);
    R.I[0] = v.x; R.I[1] = v.y; R.I[2] = v.z; R.I[3] = v.w;
    *reinterpret_cast<int4*>(sl) = make_int4(0, 0, 0, 0);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      R.I[j] = sl[j];
      sl[j] = 0;
    }
  }
  // the state streams through once per step: non-temporal loads and
  // stores keep it from displacing the tables and entries in L2
  const NtF4 V4 = __builtin_nontemporal_load(reinterpret_cast<const NtF4*>(a.V + i0));
  const NtF4 c4 = __builtin_nontemporal_load(reinterpret_cast<const NtF4*>(a.c + i0));
  R.r4 = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(a.ref + i0));
  R.V[0] = V4.x; R.V[1] = V4.y; R.V[2] = V4.z; R.V[3] = V4.w;
  R.c[0] = c4.x; R.c[1] = c4.y; R.c[2] = c4.z; R.c[3] = c4.w;

  // external Poisson drive generated on the fly: counts from word j of
  // (il0/4, t, EXT); efficacies 2b and 2b+1 of neuron j from word j of
  // (il0/4, t, EXTJ | b << 8), high half then low half
  const uint32_t g = P.il0 >> 2;
  const uint4 u = philox10(make_uint4(g, t, 0u, kTagExt), nd.key0, nd.key1);
  const uint32_t uu[4] = {u.x, u.y, u.z, u.w};
  int q[4], k[4], npj[4];
  const int h0 = nd.pop_hi[0], h1 = nd.pop_hi[1], h2 = nd.pop_hi[2];
  const int np[kMaxPops] = {nd.n_pois[0], nd.n_pois[1], NP > 2 ? nd.n_pois[2] : 0,
                            NP > 2 ? nd.n_pois[3] : 0};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int lj = P.l0 + j;
    if (lj >= nd.K) lj -= nd.K;
    q[j] = pop_index<NP>(lj, h0, h1, h2);
    k[j] = 0;
    npj[j] = sel<NP>(np, q[j]);
  }
  // Poisson counts: the number of thresholds (increasing, uniform over the
  // block) not above the draw; the scan of a neuron stops at its first
  // threshold above the draw, the wavefront's once no lane goes on (most
  // counts are 0 or 1)
  bool on[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) on[j] = true;
  for (int x = 0; x < kMaxPois; ++x) {
    const uint32_t th[kMaxPops] = {nd.pois[0][x], nd.pois[1][x],
                                   NP > 2 ? nd.pois[2][x] : 0u, NP > 2 ? nd.pois[3][x] : 0u};
    bool any = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      on[j] = on[j] && x < npj[j] && uu[j] >= sel<NP>(th, q[j]);
      k[j] += on[j] ? 1 : 0;
      any |= on[j];
    }
    if (!__any(any)) break;
  }
  int kmax = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) kmax = k[j] > kmax ? k[j] : kmax;
  const Acc* jx = static_cast<const Acc*>(a.jx) + (size_t)net * kMaxPops * kQuantN;
  for (int b = 0; 2 * b < kmax; ++b) {
    const uint4 v = philox10(make_uint4(g, t, 0u, kTagExtJ | ((uint32_t)b << 8)), nd.key0, nd.key1);
    const uint32_t vv[4] = {v.x, v.y, v.z, v.w};
    Acc e0[4], e1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // issue the table loads before any is used
      e0[j] = 2 * b < k[j] ? jx[q[j] * kQuantN + (vv[j] >> 16)] : (Acc)0;
      e1[j] = 2 * b + 1 < k[j] ? jx[q[j] * kQuantN + (vv[j] & 0xFFFFu)] : (Acc)0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) R.I[j] += e0[j] + e1[j];
  }
}

template <typename Acc, int NP>
__device__ __forceinline__ uint32_t neuron_finish(const StepArgs& a, const NetDev& nd,
                                                  const NeuronPos& P, const StepTime& T,
                                                  NeuronRegs<Acc>& R, const Acc* s_in) {
  if (s_in) {  // this thread's four entries of the tile's inbox sums
#pragma unroll
    for (int j = 0; j < 4; ++j) R.I[j] += s_in[4 * tile_tid() + j];
  }
  const uint32_t i0 = P.i0;
  const int l0 = P.l0;
  // per-population constants: uniform loads, selected per lane.  NP = 3:
  // up to four populations whose constants form two classes (entry 1 holds
  // those of population cls_rep, where class 1 begins), selected two-way
  constexpr int NS = NP == 3 ? 2 : NP;
  const int r1 = NP == 3 ? nd.cls_rep : 1;
  const float Pm[kMaxPops] = {nd.Pm[0], nd.Pm[r1], nd.Pm[2], nd.Pm[3]};
  const float Pc[kMaxPops] = {nd.Pc[0], nd.Pc[r1], nd.Pc[2], nd.Pc[3]};
  const float PVc[kMaxPops] = {nd.PVc[0], nd.PVc[r1], nd.PVc[2], nd.PVc[3]};
  const float It[kMaxPops] = {nd.Iterm[0], nd.Iterm[r1], nd.Iterm[2], nd.Iterm[3]};
  const float E[kMaxPops] = {nd.E[0], nd.E[r1], nd.E[2], nd.E[3]};
  const float Vth[kMaxPops] = {nd.Vth[0], nd.Vth[r1], nd.Vth[2], nd.Vth[3]};
  const float Vr[kMaxPops] = {nd.Vr[0], nd.Vr[r1], nd.Vr[2], nd.Vr[3]};
  const float al[kMaxPops] = {nd.alpha[0], nd.alpha[r1], nd.alpha[2], nd.alpha[3]};
  const int na[kMaxPops] = {nd.n_arp[0], nd.n_arp[r1], nd.n_arp[2], nd.n_arp[3]};
  const int h0 = nd.pop_hi[0], h1 = nd.pop_hi[1], h2 = nd.pop_hi[2];
  const int c_hi = NP == 3 ? nd.cls_hi : 0;
  uint32_t r_out = 0, mask = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int lj = l0 + j;
    if (lj >= nd.K) lj -= nd.K;
    const int qq = pop_index<NP>(lj, h0, h1, h2);
    const int qs = NP == 3 ? (lj >= c_hi ? 1 : 0) : qq;  // constants' entry
    uint32_t rj = (R.r4 >> (8 * j)) & 0xFFu;
    if ((int64_t)P.il0 + j < nd.N) {
      const float dv = fix_to_f32(R.I[j]) * a.inv2q;
      float Vj = R.V[j], cj = R.c[j];
      const float Pcq = sel<NS>(Pc, qs), Eq = sel<NS>(E, qs);
      bool spk = false;
      if (rj > 0) {
        rj -= 1;
        cj = cj * Pcq;
      } else {
        float vv = Vj - Eq;
        vv = vv * sel<NS>(Pm, qs);
        vv = Eq + vv;
        const float cc = cj * sel<NS>(PVc, qs);
        vv = vv - cc;
        vv = vv + sel<NS>(It, qs);
        vv = vv + dv;
        cj = cj * Pcq;
        if (vv > sel<NS>(Vth, qs)) {
          spk = true;
          vv = sel<NS>(Vr, qs);
          cj = cj + sel<NS>(al, qs);
          rj = (uint32_t)sel<NS>(na, qs);
        }
        Vj = vv;
      }
      R.V[j] = Vj;
      R.c[j] = cj;
      if (spk) {
        mask |= 1u << j;
        if (a.t_post) a.t_post[i0 + j] = (int32_t)T.t;  // plastic networks
        // population count of the rate bin (Sec. 2.3)
        const uint32_t mod = (uint32_t)nd.mbase + P.m0 + (l0 + j >= nd.K ? 1u : 0u);
        atomicAdd(&a.rates[((size_t)T.bin * (uint32_t)a.M + mod) * (uint32_t)a.P + qq], 1u);
      }
    }
    r_out |= rj << (8 * j);
  }
  __builtin_nontemporal_store(NtF4{R.V[0], R.V[1], R.V[2], R.V[3]},
                              reinterpret_cast<NtF4*>(a.V + i0));
  __builtin_nontemporal_store(NtF4{R.c[0], R.c[1], R.c[2], R.c[3]},
                              reinterpret_cast<NtF4*>(a.c + i0));
  __builtin_nontemporal_store(r_out, reinterpret_cast<uint32_t*>(a.ref + i0));
  return mask;
}

// Spikes of a tile in neuron order: each thread holds up to four (bit j of
// mask: neuron i0 + j); the prefix within a wavefront comes from three
// ballots of the per-thread counts, the wavefront totals are exchanged in
// LDS (s_wt, one per wavefront).  Writes the ids in increasing order to
// s_spk and returns the block's count (the same in every thread); s_spk is
// read by other threads only after the next barrier.
__device__ __forceinline__ int compact_spikes(uint32_t mask, uint32_t i0, int32_t* s_spk,
                                              int* s_wt) {
  const int tid = tile_tid(), lane = tid & 63, wave = tid >> 6;
  const uint32_t c = (uint32_t)__popc(mask);
  const unsigned long long b0 = __ballot(c & 1u), b1 = __ballot(c & 2u), b2 = __ballot(c & 4u);
  const unsigned long long lt = (1ull << lane) - 1ull;
  const int pre = __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt);
  if (lane == 0) s_wt[wave] = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
  lds_barrier();
  int base = 0, total = 0;
  for (int w = 0; w < 4; ++w) {
    const int v = s_wt[w];
    base += w < wave ? v : 0;
    total += v;
  }
  int k = base + pre;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if ((mask >> j) & 1u) s_spk[k++] = (int32_t)(i0 + j);
  return total;
}

// Plasticity event of one synapse (Sec. 2.1): source spike at step ta,
// target's last spike tp; t_act and y are the synapse's state (the rule is
// documented with dpsnn_params; binary32, no contraction).
__device__ __forceinline__ void stdp_event(const StepArgs& a, int32_t ta, int32_t tp,
                                           int32_t& t_act, float& y) {
  const int32_t L = a.stdp_L;
  const float* Ep = a.stdp_tab;
  const float* Em = Ep + L;
  const float* Dy = Em + L;
  const int32_t tl = t_act;
  y = (tl >= 0 && ta - tl < L) ? y * Dy[ta - tl] : 0.0f;
  if (tl >= 0 && tp > tl && tp - tl < L && ta - tp < L) y = y + Ep[tp - tl] * Dy[ta - tp];
  if (tp >= 0 && ta - tp < L) y = y - Em[ta - tp];
  t_act = ta;
}

__device__ __forceinline__ void record_spike(const StepArgs& a, int32_t id, uint32_t t,
                                             unsigned long long pos) {
  if (pos < (unsigned long long)a.spike_log_cap) a.log[pos] = make_int2((int)t, id);
}

// Plasticity events of the 256 synapses from p0 of the row of spiking
// source s: when the source is excitatory its synapses register the
// activation (4 per lane, 16-byte accesses).
__device__ __forceinline__ void row_plasticity(const StepArgs& a, int32_t s, int p0, uint32_t t,
                                               int lane) {
  const int64_t rb = (int64_t)s * a.row_stride;
  const int p = p0 + lane * 4;
  int32_t ms;
  int q;
  module_pop(a, s, &ms, &q);
  if (a.nets[a.tile_net[s >> 10]].exc[q] && p < a.K_out) {
    const int4 tg = *reinterpret_cast<const int4*>(a.tgt + rb + p);
    const int4 ta4 = *reinterpret_cast<const int4*>(a.syn_t + rb + p);
    const float4 y4 = *reinterpret_cast<const float4*>(a.syn_y + rb + p);
    const int32_t tgv[4] = {tg.x, tg.y, tg.z, tg.w};
    int32_t tav[4] = {ta4.x, ta4.y, ta4.z, ta4.w};
    float yv[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (p + j < a.K_out)
        stdp_event(a, (int32_t)t, a.t_post[tgv[j] & kTargetMask], tav[j], yv[j]);
    *reinterpret_cast<int4*>(a.syn_t + rb + p) = make_int4(tav[0], tav[1], tav[2], tav[3]);
    *reinterpret_cast<float4*>(a.syn_y + rb + p) = make_float4(yv[0], yv[1], yv[2], yv[3]);
  }
}

// Target word and stored efficacy (binary32 bits or code) of synapse x + k,
// x uniform: a scalar base and a 32-bit lane offset.  Non-temporal loads: a
// segment is read once per spike, and the inboxes written now and read in
// the next step stay in L2 (24x24: the update 18.0 us against 19.9 with
// ordinary loads).
__device__ __forceinline__ int32_t load_target(const StepArgs& a, int64_t x, uint32_t k) {
  const int32_t* p = a.tgt + x;
  return __builtin_nontemporal_load(p + k);
}
template <int WDT>
__device__ __forceinline__ uint32_t load_code(const StepArgs& a, int64_t x, uint32_t k) {
  if constexpr (WDT == DPSNN_W_F32) {
    const uint32_t* p = static_cast<const uint32_t*>(a.w) + x;
    return __builtin_nontemporal_load(p + k);
  } else if constexpr (WDT == DPSNN_W_F16) {
    const uint16_t* p = static_cast<const uint16_t*>(a.w) + x;
    return __builtin_nontemporal_load(p + k);
  } else {
    const uint8_t* p = static_cast<const uint8_t*>(a.w) + x;
    return __builtin_nontemporal_load(p + k);
  }
}

// Fixed-point value of a stored efficacy (int8: code | source population
// << 8, dec holding the scales of the source's network).
template <typename Acc, int WDT>
__device__ __forceinline__ Acc fix_of(const StepArgs& a, uint32_t code, const CodeDec<Acc>& dec) {
  if constexpr (WDT == DPSNN_W_F32)
    return (Acc)__builtin_rintf(__uint_as_float(code) * a.two_q);
  else
    return dec(code << kCodeShift);
}

// Handles without inboxes: the events of synapses p0 .. p0 + 255 of the row of
// a spike of this step are added into the slots of their arrival, by one
// wavefront, all loads before the first addition (a row at a time, load by
// load: 2x2 modules 19.4 us per step in the split schedule, 11.3 so).
template <typename Acc, int WDT>
__device__ __forceinline__ void row_to_slots(const StepArgs& a, int32_t s, int p0,
                                             const StepTime& T, int lane) {
  const CodeDec<Acc> dec = code_dec<Acc>(a, s >> 10);
  uint32_t pop = 0;
  if (WDT == DPSNN_W_I8) {
    int32_t ms;
    int q;
    module_pop(a, s, &ms, &q);
    pop = (uint32_t)q << 8;
  }
  Acc* slots = static_cast<Acc*>(a.slots);
  int slot0 = (int)T.slot + a.d_min;  // slot of arrival at t + d_min
  if (slot0 >= a.D) slot0 -= a.D;
  const int64_t rb = (int64_t)s * a.row_stride;
  int32_t tv[4];
  uint32_t cv[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {  // (lanes past the row read its last synapse)
    const int p = p0 + 64 * u + lane < a.K_out ? p0 + 64 * u + lane : a.K_out - 1;
    tv[u] = load_target(a, rb, (uint32_t)p);
    cv[u] = load_code<WDT>(a, rb, (uint32_t)p);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (p0 + 64 * u + lane >= a.K_out) continue;
    int sl = slot0 + (int)((uint32_t)tv[u] >> kDelayShift);
    if (sl >= a.D) sl -= a.D;
    atomic_add_fix<Acc>(slots + (int64_t)sl * a.N_pad + (tv[u] & kTargetMask),
                        fix_of<Acc, WDT>(a, cv[u] | pop, dec));
  }
}

// Delivery of the events that arrive at step t + 1.  Rows are sorted by
// (delay, target), so the events of a spike that arrive in one step are one
// contiguous segment of its row.  When a neuron spikes, its segments are cut
// into pieces of at most 64 synapses (8 where the segments are short), and
// each piece is entered in the list of its arrival step (push_pieces); a step
// reads the list that is due and writes every event once, into the inbox its
// target tile sums in the next step.  The list of a step is kept in parts by groups of tiles that are
// neighbours on the grid (delivery order), so consecutive pieces reach the
// same tiles.
//
// A block takes slices of NW x R consecutive pieces, R per wavefront, one
// lane per synapse (short pieces: 64 per wavefront, their synapses one after
// the other in R rows of lanes), and sorts their events by target tile in LDS: the first
// lane of each run of one tile claims the tile's entry of a hash table and
// adds the run there, which gives the run its rank; a prefix over the table
// gives each tile's first position, and one returning atomic per distinct
// tile reserves the tile's events in its inbox; the events are then placed
// in LDS and copied out in that order, so that consecutive lanes write
// consecutive entries.
// Pieces per wavefront of the delivery kernel, and of its plastic form, whose
// blocks share the CUs with those of the emission pass (24x24 plastic: 39 us
// per step with 8, 45 with 16; 48x48 delivery 62 and 63 us, 96x96 126 and 116)
// or with 8-byte entries, whose LDS would leave one block per CU, or with
// short pieces (8 rows hold the synapses of 64); of the fused and persistent
// schedules.
constexpr int kDlvR = 16, kDlvRSmall = 8, kFusedR = 8, kPersistR = 8;
// Table entries (bits): more than the distinct target tiles of a slice, which
// grow with lambda (48x48: about 250 at lambda 1, over 1000 at 4; a table of
// 1024 entries costs 2 us less there and 4 us more here).
constexpr int kDlvHash = 11, kFusedHash = 11, kPersistHash = 10;
constexpr int kMinR = 4;        // a slice has at least this many pieces per wavefront
constexpr int kProbes = 8;      // past these a run makes a reservation of its own
constexpr uint32_t kTabEmpty = 0xFFFF0000u;  // no tile has index 65535

// A piece: first synapse (global) << 9 | synapses << 2 | source population.
__device__ __forceinline__ unsigned long long piece_make(int64_t first, int n, uint32_t pop) {
  return (unsigned long long)first << 9 | (unsigned long long)n << 2 | pop;
}

template <typename Acc, bool WIDE>
struct InboxEntry {
  typedef uint32_t type;
};
template <typename Acc>
struct InboxEntry<Acc, true> {
  typedef unsigned long long type;
};

template <typename Ent, int BS, int R, int HB>
struct DeliverLds {
  uint32_t part[kPartMax];      // inclusive prefix of the parts' pieces
  uint32_t tab[1 << HB];        // tile << 16 | events, then first position
  uint32_t dst[1 << HB];        // inbox entry of the tile's first event, minus that position
  union {
    struct {
      Ent ent[BS * R];          // the slice's events by target tile
      uint16_t key[BS * R];     // their table entries
    };
    struct {                    // before: heads of the runs of each piece, and
      uint8_t scr[BS / 64][R][68];    // inbox positions of runs outside the table
      uint32_t lone[BS / 64][64];
      uint8_t own[BS / 64][64 * kShortPiece];  // piece of each synapse (short pieces)
    };
  };
  uint32_t wsum[BS / 64];
  uint32_t full;                // some inbox ends within the slice's events
};

// Inclusive prefix of v over the block (every thread takes part); *total is
// the block's sum.  s_w: one word per wavefront, not read since a barrier.
template <int BS>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* s_w, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t x = __shfl_up(incl, off);
    if (lane >= off) incl += x;
  }
  if (lane == 63) s_w[wave] = incl;
  lds_barrier();
  uint32_t all = 0;
#pragma unroll
  for (int w = 0; w < BS / 64; ++w) {
    const uint32_t x = s_w[w];
    incl += w < wave ? x : 0u;
    all += x;
  }
  *total = all;
  return incl;
}

template <typename Acc, int WDT, bool PACKED>
__device__ __forceinline__ typename InboxEntry<Acc, WDT == DPSNN_W_F32 && !PACKED>::type make_entry(
    const StepArgs& a, uint32_t code, uint32_t idx) {
  if constexpr (WDT != DPSNN_W_F32) {
    return code_entry(code, idx);
  } else {
    const Acc w = (Acc)__builtin_rintf(__uint_as_float(code) * a.two_q);
    if constexpr (PACKED) {
      return pack_entry((int32_t)w, idx);
    } else {
      const QEntry<Acc> e = QEntry<Acc>::make(idx, w);
      return *reinterpret_cast<const unsigned long long*>(&e);
    }
  }
}

// An entry that found the inbox of its tile full: into slot `slot` of its
// arrival, which is marked for the update.
template <typename Acc, int WDT, bool PACKED, typename Ent>
__device__ __forceinline__ void entry_to_slot(const StepArgs& a, Ent e, int tile, int slot) {
  Acc w;
  uint32_t idx;
  if constexpr (WDT != DPSNN_W_F32) {
    const CodeDec<Acc> dec = code_dec<Acc>(a, tile);
    w = ent_w<Acc>(CodeEntry{(uint32_t)e}, dec);
    idx = (uint32_t)e & 1023u;
  } else if constexpr (PACKED) {
    w = (Acc)((int32_t)e >> 10);
    idx = (uint32_t)e & 1023u;
  } else {
    const QEntry<Acc> q = *reinterpret_cast<const QEntry<Acc>*>(&e);
    w = q.w();
    idx = q.x() & 1023u;
  }
  atomic_add_fix<Acc>(
      static_cast<Acc*>(a.slots) + (int64_t)slot * a.N_pad + (int64_t)tile * 1024 + idx, w);
  a.s_dirty[(int64_t)tile * a.D + slot] = 1u;
}

// The events of a piece added into slot `slot`, marked for the updates (one
// wavefront).
template <typename Acc, int WDT>
__device__ __forceinline__ void piece_to_slot(const StepArgs& a, unsigned long long piece, int slot,
                                              int lane) {
  const int n = (int)(piece >> 2 & 127u);
  const int64_t x = (int64_t)(piece >> 9) + lane;
  if (lane >= n) return;
  const int32_t target = a.tgt[x] & kTargetMask;
  uint32_t code = load_code<WDT>(a, x, 0u);
  if (WDT == DPSNN_W_I8) code |= (uint32_t)(piece & 3u) << 8;
  const CodeDec<Acc> dec = code_dec<Acc>(a, target >> 10);
  atomic_add_fix<Acc>(static_cast<Acc*>(a.slots) + (int64_t)slot * a.N_pad + target,
                      fix_of<Acc, WDT>(a, code, dec));
  a.s_dirty[(int64_t)(target >> 10) * a.D + slot] = 1u;
}

// Table entry of a tile: an odd multiple, so that neighbouring tiles neither
// collide nor share a thread's part of the table.
template <int HB>
__device__ __forceinline__ uint32_t tab_hash(uint32_t tile) {
  return __umul24(tile, 421u) & ((1u << HB) - 1u);
}

// Inclusive prefix over the parts of a list (counts `cnt`, at most `cap`
// each) into L.part, and the total; ends with the writes, not with a barrier.
template <int BS, typename Lds>
__device__ __forceinline__ uint32_t part_prefix(const uint32_t* cnt, int nparts, uint32_t cap,
                                                Lds& L) {
  const int tid = threadIdx.x;
  const int per = (nparts + BS - 1) / BS;  // consecutive parts per thread
  uint32_t mine = 0;
  for (int k = 0; k < per; ++k) {
    const int c = tid * per + k;
    const uint32_t v = c < nparts ? cnt[c * kPieceStride] : 0u;
    mine += v < cap ? v : cap;
    if (c < nparts) L.part[c] = mine;
  }
  uint32_t S;
  const uint32_t pre = block_scan<BS>(mine, L.wsum, &S) - mine;
  for (int k = 0; k < per; ++k)
    if (tid * per + k < nparts) L.part[tid * per + k] += pre;
  return S;
}

// Part of entry s of a list (the first whose prefix exceeds s), and the
// entry's place in it.
template <typename Lds>
__device__ __forceinline__ int part_of(const Lds& L, int nparts, uint32_t s, uint32_t* at) {
  int l = 0, h = nparts - 1;
  while (l < h) {
    const int mid = (l + h) >> 1;
    if (L.part[mid] > s)
      h = mid;
    else
      l = mid + 1;
  }
  *at = s - (l ? L.part[l - 1] : 0u);
  return l;
}

// The pieces that are due in slot `slot` (the slot of step t + 1, whose
// inboxes have parity `par`), shared among nb blocks of which this is b.
template <typename Acc, int WDT, bool PACKED, int BS, int R, int HB, bool SHORT, typename Lds>
__device__ __forceinline__ void deliver_slices(const StepArgs& a, int slot, uint32_t par, int b,
                                               int nb, Lds& L) {
  typedef typename InboxEntry<Acc, WDT == DPSNN_W_F32 && !PACKED>::type Ent;
  constexpr int NW = BS / 64;
  constexpr int HN = 1 << HB;
  constexpr int PT = HN / BS;  // table entries per thread
  constexpr int WP = SHORT ? 64 : R;  // pieces of a wavefront in a slice
  static_assert(PT >= 1 && BS * R <= 65536 && R <= 64 && (!SHORT || R == kShortPiece), "");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nparts = a.n_parts;
  for (int h = tid; h < HN; h += BS) L.tab[h] = kTabEmpty;
  if (tid == 0) L.full = 0;
  const uint32_t S = part_prefix<BS>(a.piece_n + (int64_t)slot * nparts * kPieceStride, nparts,
                                     (uint32_t)a.piece_cap, L);
  // every block takes `rounds` slices of P pieces: as few as a slice of NW WP
  // pieces allows, all of one size, so that no block works on while the
  // others have ended; never less than NW WP / 4 pieces (long ones: NW kMinR),
  // to share reservations
  const uint32_t rounds = (S + (uint32_t)(nb * NW * WP) - 1u) / (uint32_t)(nb * NW * WP);
  if (rounds == 0) return;
  constexpr uint32_t kMinP = NW * (SHORT ? WP / 4 : kMinR);
  uint32_t P = (S + (uint32_t)nb * rounds - 1u) / ((uint32_t)nb * rounds);
  if (P < kMinP) P = kMinP;
  // consecutive blocks go to the eight XCDs in turn: those of one XCD take
  // consecutive pieces, so that the inboxes they share meet in its L2
  const int g = nb % 8 == 0 ? (b & 7) * (nb >> 3) + (b >> 3) : b;
  uint32_t s0 = (uint32_t)g * rounds * P;
  if (s0 >= S) return;
  const uint32_t s_end = s0 + rounds * P < S ? s0 + rounds * P : S;
  lds_barrier();
  const unsigned long long* pieces = a.pieces + (int64_t)slot * nparts * a.piece_cap;
  uint32_t* in_cnt = a.in_cnt + (int64_t)par * a.n_tiles * kInboxStride;
  Ent* in_q = static_cast<Ent*>(a.in_q) + (int64_t)par * a.n_tiles * a.in_stride;
  // lane p holds piece p of the wavefront
  auto records = [&](uint32_t from) -> unsigned long long {
    const uint32_t k = (uint32_t)(lane * NW + wave), s = from + k;
    if (lane >= WP || k >= P || s >= s_end) return 0ull;
    uint32_t at;
    const int l = part_of(L, nparts, s, &at);
    return pieces[(int64_t)l * a.piece_cap + at];
  };
  int32_t tv[R];   // target words
  uint32_t cv[R];  // stored efficacies
  int T = 0;       // events of the wavefront (SHORT)
  auto load = [&](unsigned long long rec) {
    if constexpr (SHORT) {
      // the pieces' synapses one after the other, 64 to a row: each finds its
      // piece by its place in the wavefront's scratch
      const uint32_t n = (uint32_t)rec >> 2 & 127u;
      const uint32_t incl = wave_scan(n);
      T = __builtin_amdgcn_readlane((int)incl, 63);
      for (uint32_t j = 0; j < n; ++j) L.own[wave][incl - n + j] = (uint8_t)lane;
      wave_lds_sync();
      const unsigned long long from = (rec >> 9) - (incl - n);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        tv[r] = 0;
        cv[r] = 0;
        if (r * 64 >= T) continue;  // uniform
        // lanes past the last synapse read it
        const int e = r * 64 + lane < T ? r * 64 + lane : T - 1;
        const int p = L.own[wave][e];
        const unsigned long long x =
            ((unsigned long long)__shfl((uint32_t)(from >> 32), p) << 32 |
             __shfl((uint32_t)from, p)) + (uint32_t)e;
        tv[r] = load_target(a, (int64_t)x, 0u);
        cv[r] = load_code<WDT>(a, (int64_t)x, 0u);
        if (WDT == DPSNN_W_I8) cv[r] |= (__shfl((uint32_t)rec, p) & 3u) << 8;
      }
      return;
    }
    const uint32_t rec_lo = (uint32_t)rec, rec_hi = (uint32_t)(rec >> 32);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t lo = __builtin_amdgcn_readlane(rec_lo, r);
      const uint32_t hi = __builtin_amdgcn_readlane(rec_hi, r);
      const int64_t x0 = (int64_t)(((unsigned long long)hi << 32 | lo) >> 9);
      const uint32_t n = lo >> 2 & 127u;
      // lanes past the piece read its last synapse (of row 0 if there is none)
      const uint32_t end = n ? n - 1u : 0u;
      const uint32_t k = (uint32_t)lane < end ? (uint32_t)lane : end;
      tv[r] = load_target(a, x0, k);
      cv[r] = load_code<WDT>(a, x0, k);
    }
  };
  unsigned long long rec = records(s0);
  for (;;) {
    const bool more = s0 + P < s_end;
    load(rec);
    uint32_t rec_lo = (uint32_t)rec;
    auto len = [&](int r) -> int {
      if constexpr (SHORT) return T - 64 * r < 0 ? 0 : T - 64 * r < 64 ? T - 64 * r : 64;
      return (int)(__builtin_amdgcn_readlane(rec_lo, r) >> 2 & 127u);
    };
    Ent en[R];
    uint32_t tl[R];  // target tile
#pragma unroll
    for (int r = 0; r < R; ++r) {
      uint32_t c = cv[r];
      if (WDT == DPSNN_W_I8 && !SHORT) c |= (__builtin_amdgcn_readlane(rec_lo, r) & 3u) << 8;
      en[r] = make_entry<Acc, WDT, PACKED>(a, c, (uint32_t)tv[r] & 1023u);
      tl[r] = (uint32_t)(tv[r] & kTargetMask) >> 10;
    }
    // the hashes and masks are recomputed past this point and the next such
    // one: cheaper than the registers that carrying them over takes
    asm volatile("" : "+v"(rec_lo));
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(tl[r]));
    // the first lane of each run of one tile claims the tile's table entry
    uint32_t at[R];  // the claim, then table entry << 16 | rank
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int prev = __builtin_amdgcn_update_dpp(-1, (int)tl[r], 0x138, 0xf, 0xf, false);
      const bool head = lane < len(r) && prev != (int)tl[r];
      at[r] = kTabEmpty;
      if (head) at[r] = atomicCAS(&L.tab[tab_hash<HB>(tl[r])], kTabEmpty, tl[r] << 16);
    }
    asm volatile("" : "+v"(rec_lo));
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(tl[r]));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int n = len(r);
      if (n == 0) {  // uniform
        at[r] = ~0u;
        continue;
      }
      const int prev = __builtin_amdgcn_update_dpp(-1, (int)tl[r], 0x138, 0xf, 0xf, false);
      const bool head = lane < n && prev != (int)tl[r];
      const unsigned long long heads = __ballot(head);
      // the head of this lane's run and the end of the run, through the
      // wavefront's scratch, indexed by the number of heads below
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(heads >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u));
      uint8_t* scr = L.scr[wave][r];
      if (head) scr[below] = (uint8_t)lane;
      if (lane == 0) scr[__popcll(heads)] = (uint8_t)n;
      wave_lds_sync();
      const uint32_t k = head ? below : below - 1u;  // (lane 0 is a head)
      const uint32_t from = scr[k], end = scr[k + 1];
      uint32_t h = tab_hash<HB>(tl[r]), v = 0;
      const bool lost = at[r] != kTabEmpty && at[r] >> 16 != tl[r];
      if (__any(lost)) {  // another tile holds an entry: probe the next ones
        bool found = !lost;
        for (int x = 1; x < kProbes && !found; ++x) {
          h = (h + 1) & (HN - 1);
          const uint32_t old = atomicCAS(&L.tab[h], kTabEmpty, tl[r] << 16);
          found = old == kTabEmpty || old >> 16 == tl[r];
        }
        if (!found) {  // a reservation of its own for the run
          uint32_t pos = atomicAdd(&in_cnt[(int64_t)tl[r] * kInboxStride], end - from);
          for (uint32_t x = from; x < end; ++x) L.lone[wave][x] = pos++;
        }
        wave_lds_sync();
        // lanes of such runs store their events now
        const bool lone = __shfl((int)!found, (int)from) && lane < n;
        if (lone) {
          const uint32_t pos = L.lone[wave][lane];
          if (pos < (uint32_t)a.in_cap)
            in_q[(int64_t)tl[r] * a.in_stride + pos] = en[r];
          else
            entry_to_slot<Acc, WDT, PACKED>(a, en[r], (int)tl[r], slot);
        }
        if (head && found) v = (h << 16) | (atomicAdd(&L.tab[h], end - from) & 0xFFFFu);
        at[r] = lone ? ~0u : __shfl(v, (int)from) + (uint32_t)lane - from;
        wave_lds_sync();
      } else {
        if (head) v = (h << 16) | (atomicAdd(&L.tab[h], end - from) & 0xFFFFu);
        at[r] = __shfl(v, (int)from) + (uint32_t)lane - from;
      }
      if (lane >= n) at[r] = ~0u;
    }
    lds_barrier();
    // prefix over the table and the reservations
    uint32_t te[PT], tb[PT], sum = 0;
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      te[j] = L.tab[tid * PT + j];
      const uint32_t n = te[j] & 0xFFFFu;
      tb[j] = 0;
      if (n) tb[j] = atomicAdd(&in_cnt[(int64_t)(te[j] >> 16) * kInboxStride], n);
      sum += n;
    }
    uint32_t total;
    uint32_t pre = block_scan<BS>(sum, L.wsum, &total) - sum;
    {
      uint32_t p = pre;
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const uint32_t n = te[j] & 0xFFFFu;
        if (n) L.tab[tid * PT + j] = (te[j] & 0xFFFF0000u) | p;
        p += n;
      }
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (at[r] != ~0u) {
        const uint32_t h = at[r] >> 16;
        const uint32_t p = (L.tab[h] & 0xFFFFu) + (at[r] & 0xFFFFu);
        L.ent[p] = en[r];
        L.key[p] = (uint16_t)h;
      }
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const uint32_t n = te[j] & 0xFFFFu;
      if (n) {
        L.dst[tid * PT + j] = (te[j] >> 16) * (uint32_t)a.in_stride + tb[j] - pre;
        if (tb[j] + n > (uint32_t)a.in_cap) L.full = 1;
      }
      pre += n;
    }
    lds_barrier();
    // copy out
    if (!L.full) {
      for (uint32_t p0 = tid; p0 < total; p0 += 4 * BS) {
        uint32_t to[4];
        Ent v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t p = p0 + (uint32_t)(u * BS);
          if (p < total) {
            to[u] = L.dst[L.key[p]] + p;
            v[u] = L.ent[p];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (p0 + (uint32_t)(u * BS) < total) in_q[to[u]] = v[u];
      }
    } else {
      for (uint32_t p = tid; p < total; p += BS) {
        const uint32_t to = L.dst[L.key[p]] + p;
        const uint32_t tile = L.tab[L.key[p]] >> 16;
        if (to - tile * (uint32_t)a.in_stride < (uint32_t)a.in_cap)
          in_q[to] = L.ent[p];
        else
          entry_to_slot<Acc, WDT, PACKED>(a, L.ent[p], (int)tile, slot);
      }
    }
    if (!more) break;
    s0 += P;
    rec = records(s0);
    lds_barrier();  // the table is emptied, the events' space written again
    for (int h = tid; h < HN; h += BS) L.tab[h] = kTabEmpty;
    if (tid == 0) L.full = 0;
    lds_barrier();
  }
}

// Enters the spikes s_spk[0 .. n) of tile `tile` (slot `now` = t mod D) in the
// lists of their arrival steps, delays of index l0 and more; by the tile's
// threads.  Pieces that find a list full go into the slots, a
// wavefront per piece (48x48 with a single delay, 16 pieces a spike, 7 % of the
// neurons in the largest step: update 1341 us when lists held a piece per
// neuron and the lane that found one full added its synapses alone, 64 now).
//
// Lanes take (delay, spike) pairs, delay first: the lanes of one delay follow
// each other, so a prefix over the wavefront and one returning atomic per
// delay give every pair its place (48x48: update 30.1 us with an atomic per
// pair, 28.7 so; with 100 synapses a neuron and 96 Hz 70 and 36).
template <typename Acc, int WDT>
__device__ __forceinline__ void push_pieces(const StepArgs& a, int tile, int now, int l0, int n,
                                            const int32_t* s_spk) {
  const int place = a.tile_place[tile];
  const int nl = a.n_del - l0, lane = threadIdx.x & 63, items = n * nl;
  const int plen = a.piece_len;
  // (from the last wavefront on: the first ones deliver the events of delay 1
  // meanwhile in the fused schedule: 24x24 population model 16.9 -> 16.1 us)
  for (int i0 = __builtin_amdgcn_readfirstlane((tile_tid() & 192) ^ 192); i0 < items; i0 += 256) {
    const int i = i0 + lane;
    int len = 0, slot = 0, head = 0, tail = 0;
    int32_t s = 0;
    uint32_t pop = 0, np = 0, lost = 0;
    int64_t first = 0;
    if (i < items) {
      const int d = i / n, l = l0 + d;
      s = s_spk[i - d * n];
      const uint16_t* ro = a.row_off + (int64_t)s * (a.n_del + 1) + l;
      const int o0 = ro[0];
      len = (int)ro[1] - o0;
      slot = now + a.d_min + l;
      if (slot >= a.D) slot -= a.D;
      first = (int64_t)s * a.row_stride + o0;
      np = (uint32_t)(len + plen - 1) / (uint32_t)plen;
      // first and last lane of the delay
      head = d * n - i0 > 0 ? d * n - i0 : 0;
      tail = (d + 1) * n - i0 < 64 ? (d + 1) * n - i0 - 1 : 63;
    }
    const uint32_t incl = wave_scan(np);
    const uint32_t before = __shfl(incl - np, head), all = __shfl(incl, tail) - before;
    const int64_t part = (int64_t)slot * a.n_parts + (place >> a.part_shift);
    uint32_t at = 0;
    if (i < items && lane == head && all) at = atomicAdd(&a.piece_n[part * kPieceStride], all);
    if (WDT == DPSNN_W_I8) pop = pop_in_tile(a, tile, s);
    at = __shfl(at, head) + incl - np - before;
    int o = 0;
    for (; o < len && at < (uint32_t)a.piece_cap; o += plen, ++at)
      a.pieces[part * a.piece_cap + at] = piece_make(first + o, len - o < plen ? len - o : plen, pop);
    lost = o < len ? (uint32_t)(len - o) : 0u;
    for (unsigned long long over = __ballot(lost > 0); over; over &= over - 1) {
      const int from = __ffsll(over) - 1;
      const int m = __shfl((int)lost, from), to = __shfl(slot, from);
      const int64_t x = __shfl((long long)(first + len - (int)lost), from);
      const uint32_t q = __shfl(pop, from);
      for (int p = 0; p < m; p += 64)
        piece_to_slot<Acc, WDT>(a, piece_make(x + p, m - p < 64 ? m - p : 64, q), to, lane);
    }
  }
}

// Work done when a spike is emitted (plastic networks: the activations of
// its synapses; handles without inboxes: its events into the slots), for the
// listed spikes of this step, one wavefront per 256 synapses: wavefront w of
// nw takes items w, w + nw, ...
template <typename Acc, int WDT, bool PLAST, int BS, typename Lds>
__device__ __forceinline__ void emission_items(const StepArgs& a, const StepTime& T, int b, int nb,
                                               Lds& L) {
  const int lane = threadIdx.x & 63;
  const uint32_t n = part_prefix<BS>(a.emit_n + (T.t & 1u) * (uint32_t)(a.n_parts * kPieceStride),
                                     a.n_parts, ~0u, L);
  lds_barrier();
  const uint32_t cpr = (uint32_t)(a.K_out + 255) / 256u;  // at most 16, of 2^26 spikes
  const uint32_t items = n * cpr;
  for (uint32_t it = __builtin_amdgcn_readfirstlane(b * (BS / 64) + (int)(threadIdx.x >> 6));
       it < items; it += (uint32_t)(nb * (BS / 64))) {
    const uint32_t k = it / cpr;
    uint32_t at;
    const int part = part_of(L, a.n_parts, k, &at);
    const int32_t s = __builtin_amdgcn_readfirstlane(
        a.emit_id[((int64_t)part << (a.part_shift + 10)) + at]);
    const int p0 = (int)(it - k * cpr) * 256;
    if (PLAST) row_plasticity(a, s, p0, T.t, lane);
    if (!a.q_cap) row_to_slots<Acc, WDT>(a, s, p0, T, lane);
  }
}

// The spikes of step t into the spike log, in (step, neuron) order: part of
// nparts takes a range of tiles, its first position the counts of the tiles
// before them; the last part advances the log bases and the spike total.
template <int BS>
__device__ __forceinline__ void log_step(const StepArgs& a, uint32_t t, int part, int nparts,
                                         uint32_t* s_w) {
  constexpr int NW = BS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (a.n_tiles + nparts - 1) / nparts;
  const int lo = part * per < a.n_tiles ? part * per : a.n_tiles;
  const int hi = lo + per < a.n_tiles ? lo + per : a.n_tiles;
  const unsigned long long log0 = a.log_base[t & 1u];
  const int32_t* cnt = a.blk_cnt + (t & 1u) * (uint32_t)a.n_tiles;
  const uint16_t* spk = a.spk + (t & 1u) * a.N_pad;
  uint32_t acc = 0;
  for (int b = tid; b < lo; b += BS) acc += (uint32_t)cnt[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) s_w[wave] = acc;
  lds_barrier();
  uint32_t run = 0;  // spikes of the tiles before the next chunk
  for (int w = 0; w < NW; ++w) run += s_w[w];
  for (int b0 = lo; b0 < hi; b0 += BS) {
    const int b = b0 + tid;
    const uint32_t c = b < hi ? (uint32_t)cnt[b] : 0u;
    uint32_t incl = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    lds_barrier();
    if (lane == 63) s_w[wave] = incl;
    lds_barrier();
    uint32_t at = run + incl - c;
    for (int w = 0; w < NW; ++w) {
      const uint32_t v = s_w[w];
      at += w < wave ? v : 0u;
      run += v;
    }
    if (a.spike_log_cap > 0 && c > 0) {
      const uint16_t* ids = spk + (int64_t)b * 1024;
      for (uint32_t k = 0; k < c; ++k)
        record_spike(a, b * 1024 + (int32_t)ids[k], t, log0 + at + k);
    }
  }
  if (part == nparts - 1 && tid == 0) {
    a.log_base[(t + 1u) & 1u] = log0 + run;
    a.n_spikes[0] += run;
  }
}

// ------------------------------------------------------------------------
// Update of one tile of 1024 neurons by 256 threads (whole wavefronts of a
// block, all of which pass its four barriers); lists its
// spikes (ids in increasing order, s_spk) and returns their number.
template <typename Acc, int NP, int FMT>
__device__ __forceinline__ int update_tile(const StepArgs& a, const StepTime& T, int tile,
                                           int32_t* s_spk, Acc* s_in, int* s_wt) {
  const int tid = tile_tid();
  const int net = __builtin_amdgcn_readfirstlane(a.tile_net[tile]);
  const NetDev& nd = a.nets[net];
  const NeuronPos P = neuron_pos(nd, tile, tid);
  NeuronRegs<Acc> R;
  neuron_load<Acc, NP>(a, nd, net, P, T, R);
  if (a.q_cap)
    gather_now<Acc, FMT>(a, tile, T, s_in);
  else
    lds_barrier();
  const uint32_t mask = neuron_finish<Acc, NP>(a, nd, P, T, R, a.q_cap ? s_in : nullptr);
  const int n = compact_spikes(mask, P.i0, s_spk, s_wt);
  lds_barrier();
  return n;
}

// The spikes of a tile listed for the log, by step parity.
__device__ __forceinline__ void list_for_log(const StepArgs& a, const StepTime& T, int tile, int n,
                                             const int32_t* s_spk) {
  const int tid = tile_tid();
  const uint32_t par = T.t & 1u;
  if (tid == 0) a.blk_cnt[par * (uint32_t)a.n_tiles + (uint32_t)tile] = n;
  uint16_t* out = a.spk + par * a.N_pad + (int64_t)tile * 1024;
  for (int k = tid; k < n; k += 256) out[k] = (uint16_t)(s_spk[k] & 1023);
}

// The same, listed also for the emission pass, and entered in the lists of
// their arrival steps (split and persistent schedules).
template <typename Acc, int WDT>
__device__ __forceinline__ void list_spikes(const StepArgs& a, const StepTime& T, int tile, int n,
                                            const int32_t* s_spk, int* s_wt) {
  const int tid = threadIdx.x;
  list_for_log(a, T, tile, n, s_spk);
  if (n == 0) return;
  if (a.emit_id) {
    const int part = a.tile_place[tile] >> a.part_shift;
    if (tid == 0)
      s_wt[0] = (int)atomicAdd(
          &a.emit_n[((T.t & 1u) * (uint32_t)a.n_parts + (uint32_t)part) * kPieceStride],
          (uint32_t)n);
    lds_barrier();
    int32_t* out = a.emit_id + ((int64_t)part << (a.part_shift + 10)) + s_wt[0];
    for (int k = tid; k < n; k += 256) out[k] = s_spk[k];
  }
  if (a.q_cap) push_pieces<Acc, WDT>(a, tile, (int)T.slot, 0, n, s_spk);
}

template <typename Acc, int NP, int FMT, int WDT>
__global__ void __launch_bounds__(256) k_neuron(StepArgs a, StepOff o) {
  __shared__ int32_t s_spk[1024];
  __shared__ Acc s_in[1024];
  __shared__ int s_wt[4];
  const StepTime T = step_time(a, o);
  const int tile = (int)blockIdx.x;
  const int n = update_tile<Acc, NP, FMT>(a, T, tile, s_spk, s_in, s_wt);
  list_spikes<Acc, WDT>(a, T, tile, n, s_spk, s_wt);
}

// Counters that start from zero in the next step (nothing else uses them in
// this one): the list of this step's arrivals, which the previous step
// delivered, and the next step's emission list.
__device__ __forceinline__ void clear_counters(const StepArgs& a, const StepTime& T) {
  uint32_t* cnt = a.piece_n + (int64_t)T.slot * a.n_parts * kPieceStride;
  if (a.q_cap)
    for (int c = threadIdx.x; c < a.n_parts; c += blockDim.x) cnt[c * kPieceStride] = 0u;
  if (a.emit_id)
    for (int c = threadIdx.x; c < a.n_parts; c += blockDim.x)
      a.emit_n[(((T.t + 1u) & 1u) * (uint32_t)a.n_parts + (uint32_t)c) * kPieceStride] = 0u;
}

template <typename Acc, int WDT, bool PLAST, bool PACKED, bool SHORT>
__global__ void __launch_bounds__(kDlvThreads, PLAST || SHORT ? 6 : 4)
    k_deliver(StepArgs a, StepOff o) {
  typedef typename InboxEntry<Acc, WDT == DPSNN_W_F32 && !PACKED>::type Ent;
  constexpr int R = PLAST || SHORT || sizeof(Ent) == 8 ? kDlvRSmall : kDlvR;
  __shared__ DeliverLds<Ent, kDlvThreads, R, kDlvHash> L;
  const StepTime T = step_time(a, o);
  if ((int)blockIdx.x < a.log_blocks) {
    if (blockIdx.x == 0) clear_counters(a, T);
    log_step<kDlvThreads>(a, T.t, blockIdx.x, a.log_blocks, L.wsum);
    return;
  }
  int b = (int)blockIdx.x - a.log_blocks;
  if ((PLAST || !a.q_cap) && b < a.emit_blocks) {
    emission_items<Acc, WDT, PLAST, kDlvThreads>(a, T, b, a.emit_blocks, L);
    return;
  }
  if (PLAST || !a.q_cap) b -= a.emit_blocks;
  const int nb = a.deliver_grid;
  const int next = (int)T.slot + 1 < a.D ? (int)T.slot + 1 : 0;
  if (a.q_cap)
    deliver_slices<Acc, WDT, PACKED, kDlvThreads, R, kDlvHash, SHORT>(a, next, (T.t + 1u) & 1u, b,
                                                                     nb, L);
}

// The events that arrive one step after the spikes s_spk[0 .. n) (d_min = 1:
// the first segment of their rows), straight into the inboxes of step t + 1:
// one returning atomic per run of one target tile; a wavefront per spike, or 16
// lanes per spike where the segments are short (24x24 modules of 125 neurons at
// 92 Hz, 6 synapses per delay: 18.9 us per step with a wavefront per spike, 14.8
// so; 24x24 with 100 synapses a neuron at 95 Hz: 39.7 and 34.4).
template <typename Acc, int WDT, bool PACKED, bool SHORT>
__device__ __forceinline__ void deliver_first(const StepArgs& a, const StepTime& T, int tile,
                                              int n, const int32_t* s_spk) {
  typedef typename InboxEntry<Acc, WDT == DPSNN_W_F32 && !PACKED>::type Ent;
  constexpr int LG = SHORT ? 16 : 64, GS = 64 / LG;  // lanes per spike, spikes at a time
  const int lane = threadIdx.x & 63, wave = tile_tid() >> 6, sub = lane & (LG - 1);
  const uint32_t par = (T.t + 1u) & 1u;
  const int slot = (int)T.slot + 1 < a.D ? (int)T.slot + 1 : 0;
  uint32_t* in_cnt = a.in_cnt + (int64_t)par * a.n_tiles * kInboxStride;
  Ent* in_q = static_cast<Ent*>(a.in_q) + (int64_t)par * a.n_tiles * a.in_stride;
  for (int k0 = wave * GS; k0 < n; k0 += 4 * GS) {
    const int k = k0 + lane / LG;
    int32_t s = s_spk[k < n ? k : n - 1];
    int end = k < n ? (int)a.row_off[(int64_t)s * (a.n_del + 1) + 1] : 0;
    if (!SHORT) {
      s = __builtin_amdgcn_readfirstlane(s);
      end = __builtin_amdgcn_readfirstlane(end);
    }
    const uint32_t pop = WDT == DPSNN_W_I8 ? pop_in_tile(a, tile, s) << 8 : 0u;
    const int64_t rb = (int64_t)s * a.row_stride;
    for (int o = 0; SHORT ? (bool)__any(o < end) : o < end; o += LG) {
      const int left = end - o < 0 ? 0 : end - o, m = left < LG ? left : LG;
      // (lanes past the segment read its last synapse, or the row's first)
      const int64_t x = m ? rb + o + (sub < m ? sub : m - 1) : rb;
      const int32_t target = a.tgt[x] & kTargetMask;
      const Ent e = make_entry<Acc, WDT, PACKED>(a, load_code<WDT>(a, x, 0u) | pop,
                                                 (uint32_t)target & 1023u);
      const int tl = target >> 10;
      const int prev = __builtin_amdgcn_update_dpp(-1, tl, 0x138, 0xf, 0xf, false);
      const bool head = sub < m && (prev != tl || (SHORT && sub == 0));
      const unsigned long long heads = __ballot(head);
      const unsigned long long after = heads >> lane >> 1;
      // the run ends with the segment or at the next head
      const int to_head = after ? __ffsll(after) : 64, to_end = m - sub;
      uint32_t v = 0;
      if (head)
        v = atomicAdd(&in_cnt[(int64_t)tl * kInboxStride],
                      (uint32_t)(to_head < to_end ? to_head : to_end)) -
            (uint32_t)lane;
      const unsigned long long upto = heads & ((2ull << lane) - 1ull);
      const uint32_t pos = __shfl(v, upto ? 63 - __clzll((long long)upto) : 0) + (uint32_t)lane;
      if (sub < m) {
        if (pos < (uint32_t)a.in_cap)
          in_q[(int64_t)tl * a.in_stride + pos] = e;
        else
          entry_to_slot<Acc, WDT, PACKED>(a, e, tl, slot);
      }
    }
  }
}

// Fused schedule: one launch per step.  The first log_blocks blocks append
// the log of the previous step of this run (the tick after a run appends that
// of its last), the next n_dlv deliver the pieces that are due at t + 1, all
// of them emitted before this step; the others update two tiles each, list
// their spikes for later steps and deliver their events of delay 1 themselves.
template <typename Acc, int WDT, int NP, int FMT, bool SHORT>
__global__ void __launch_bounds__(kDlvThreads, 6) k_step(StepArgs a, StepOff o, int n_dlv) {
  constexpr bool PACKED = FMT == kFmtPacked;
  __shared__ union {
    struct {
      int32_t spk[2][1024];
      Acc in[2][1024];
      int wt[2][4];
    } u;
    DeliverLds<typename InboxEntry<Acc, FMT == kFmtWide>::type, kDlvThreads, kFusedR, kFusedHash> d;
  } L;
  const StepTime T = step_time(a, o);
  const int next = (int)T.slot + 1 < a.D ? (int)T.slot + 1 : 0;
  int b = (int)blockIdx.x;
  if (b < a.log_blocks) {
    if (b == 0) clear_counters(a, T);
    if (o.t_off > 0) log_step<kDlvThreads>(a, T.t - 1u, b, a.log_blocks, L.d.wsum);
    return;
  }
  b -= a.log_blocks;
  if (b < n_dlv) {
    if (a.q_cap)
      deliver_slices<Acc, WDT, PACKED, kDlvThreads, kFusedR, kFusedHash, SHORT>(
          a, next, (T.t + 1u) & 1u, b, n_dlv, L.d);
    return;
  }
  const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8), tid = tile_tid();
  const int tile = (b - n_dlv) * 2 + half;
  if (tile >= a.n_tiles) {  // (an odd number of tiles) the barriers of the other's update
    lds_barrier();
    if (a.q_cap) lds_barrier();
    lds_barrier();
    lds_barrier();
    return;
  }
  const int32_t* spk = L.u.spk[half];
  const int n = update_tile<Acc, NP, FMT>(a, T, tile, L.u.spk[half], L.u.in[half], L.u.wt[half]);
  list_for_log(a, T, tile, n, spk);
  if (n == 0) return;
  if (a.q_cap) {
    push_pieces<Acc, WDT>(a, tile, (int)T.slot, a.d_min == 1 ? 1 : 0, n, spk);
    if (a.d_min == 1) deliver_first<Acc, WDT, PACKED, SHORT>(a, T, tile, n, spk);
  } else {
    for (int k = tid >> 6; k < n; k += 4) {
      const int32_t id = __builtin_amdgcn_readfirstlane(spk[k]);
      for (int p0 = 0; p0 < a.K_out; p0 += 256) row_to_slots<Acc, WDT>(a, id, p0, T, tid & 63);
    }
  }
}

// Residues of step t_base + t_off computed on the device (the persistent
// schedule's steps inside one launch).
__device__ __forceinline__ StepOff step_off_dev(const StepArgs& a, uint32_t t_off) {
  StepOff o;
  o.t_off = t_off;
  o.d_slot = t_off % (uint32_t)a.D;
  o.d_phase = t_off % (uint32_t)a.rate_bin_steps;
  o.d_bin = (t_off / (uint32_t)a.rate_bin_steps) % (uint32_t)a.rate_bins_cap;
  return o;
}

// Persistent schedule: n_steps steps in one cooperative launch of blocks
// that are all resident at once (G of them).  Each step: block b updates
// tiles b, b + G, ...; the grid synchronises; block 0 appends the spike log,
// and all blocks share the list of pieces that is due; the grid synchronises.
// This is the split schedule's sequence of work, so the results are the same.
template <typename Acc, int WDT, int NP, int FMT>
__global__ void __launch_bounds__(256) k_persist(StepArgs a, StepOff o, uint32_t n_steps) {
  __shared__ union {
    struct {
      int32_t spk[1024];
      Acc in[1024];
      int wt[4];
    } u;
    DeliverLds<typename InboxEntry<Acc, FMT == kFmtWide>::type, 256, kPersistR, kPersistHash> d;
  } L;
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const int G = (int)gridDim.x;
  for (uint32_t k = 0; k < n_steps; ++k) {
    const StepTime T = step_time(a, step_off_dev(a, o.t_off + k));
    for (int tile = (int)blockIdx.x; tile < a.n_tiles; tile += G) {
      const int n = update_tile<Acc, NP, FMT>(a, T, tile, L.u.spk, L.u.in, L.u.wt);
      list_spikes<Acc, WDT>(a, T, tile, n, L.u.spk, L.u.wt);
      lds_barrier();  // the tile's LDS is reused by the next one
    }
    grid.sync();
    if (blockIdx.x == 0) {
      clear_counters(a, T);
      log_step<256>(a, T.t, 0, 1, L.d.wsum);
      lds_barrier();
    }
    if (!a.q_cap)
      emission_items<Acc, WDT, false, 256>(a, T, (int)blockIdx.x, G, L.d);
    const int next = (int)T.slot + 1 < a.D ? (int)T.slot + 1 : 0;
    if (a.q_cap && a.piece_len == kShortPiece)
      deliver_slices<Acc, WDT, FMT == kFmtPacked, 256, kShortPiece, kPersistHash, true>(
          a, next, (T.t + 1u) & 1u, (int)blockIdx.x, G, L.d);
    else if (a.q_cap)
      deliver_slices<Acc, WDT, FMT == kFmtPacked, 256, kPersistR, kPersistHash, false>(
          a, next, (T.t + 1u) & 1u, (int)blockIdx.x, G, L.d);
    grid.sync();
  }
}

// A thread per tile, as far as one block goes (24x24, a step at a time with
// the log on: 32.5 us per step with 256 threads, 29.3 with 1024).
constexpr int kTickThreads = 1024;

// Advance the device step counter after `n` steps; after a run of the fused
// schedule (log_last) append the log of its last step first.
__global__ void __launch_bounds__(kTickThreads) k_tick(StepArgs a, uint32_t n, int log_last) {
  __shared__ uint32_t s_w[kTickThreads / 64];
  const uint32_t t1 = a.t_base[0] + n;
  if (log_last) log_step<kTickThreads>(a, t1 - 1u, 0, 1, s_w);
  __syncthreads();  // every thread has read the counter
  if (threadIdx.x == 0) {
    // the counter and the residues the step kernels start from
    a.t_base[0] = t1;
    a.t_base[1] = t1 % (uint32_t)a.D;
    a.t_base[2] = t1 % (uint32_t)a.rate_bin_steps;
    a.t_base[3] = (t1 / (uint32_t)a.rate_bin_steps) % (uint32_t)a.rate_bins_cap;
  }
  // the emission lists of the next step start empty whatever the schedule
  if (a.emit_id)
    for (int c = threadIdx.x; c < 2 * a.n_parts; c += kTickThreads)
      a.emit_n[c * kPieceStride] = 0u;
}

// Folds the events that are still to arrive after t steps into the slots: the
// inboxes (arriving at t) and the lists of the later steps; all are left empty
// and the slots that got something marked.  Block b < n_tiles takes the inbox
// of tile b, the others a list each, `share` of them one list (2x2 modules
// with an efficacy update every 10 steps: 26.1 us per step when the tiles'
// blocks took the lists too and marked every slot, 18.3 so).
template <typename Acc, typename E>
__device__ __forceinline__ void drain_inbox(const StepArgs& a, int tile, uint32_t t,
                                            const CodeDec<Acc>& dec) {
  const int64_t box = (int64_t)(t & 1u) * a.n_tiles + tile;
  const uint32_t got = a.in_cnt[box * kInboxStride];
  const uint32_t n_in = got < (uint32_t)a.in_cap ? got : (uint32_t)a.in_cap;
  const E* iq = static_cast<const E*>(a.in_q) + box * a.in_stride;
  Acc* sl = static_cast<Acc*>(a.slots) + (int64_t)(t % (uint32_t)a.D) * a.N_pad +
            (int64_t)tile * 1024;
  for (uint32_t e = threadIdx.x; e < n_in; e += blockDim.x)
    atomic_add_fix<Acc>(sl + (ent_x(iq[e]) & 1023u), ent_w<Acc>(iq[e], dec));
  __syncthreads();  // every thread has read the count
  if (threadIdx.x == 0 && got) {
    a.in_cnt[box * kInboxStride] = 0;
    a.s_dirty[(int64_t)tile * a.D + t % (uint32_t)a.D] = 1u;
  }
}

template <typename Acc, int WDT>
__global__ void __launch_bounds__(256) k_drain(StepArgs a, uint32_t t, int share) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((int)blockIdx.x < a.n_tiles) {
    const int tile = (int)blockIdx.x;
    const CodeDec<Acc> dec = code_dec<Acc>(a, tile);
    if (a.q_code)
      drain_inbox<Acc, CodeEntry>(a, tile, t, dec);
    else if (sizeof(Acc) == 4 && a.q_packed)
      drain_inbox<Acc, PackedEntry>(a, tile, t, dec);
    else
      drain_inbox<Acc, QEntry<Acc>>(a, tile, t, dec);
    return;
  }
  const int now = (int)(t % (uint32_t)a.D);  // the list of t is delivered already
  const int y = (int)blockIdx.x - a.n_tiles, x = y / share;
  const int slot = x / a.n_parts;
  uint32_t* cnt = a.piece_n + (int64_t)x * kPieceStride;
  const uint32_t got = cnt[0];
  const uint32_t n = slot == now ? 0u : got < (uint32_t)a.piece_cap ? got : (uint32_t)a.piece_cap;
  const unsigned long long* p = a.pieces + (int64_t)x * a.piece_cap;
  for (uint32_t k = (uint32_t)((y - x * share) * 4 + wave); k < n; k += (uint32_t)(4 * share))
    piece_to_slot<Acc, WDT>(a, p[k], slot, lane);
  __syncthreads();  // every thread has read the count
  // the last of the list's blocks empties it (the word after the count, which
  // nothing else uses, tells them apart)
  if (threadIdx.x == 0 && (share == 1 || atomicAdd(cnt + 1, 1u) == (uint32_t)share - 1u)) {
    cnt[0] = 0;
    cnt[1] = 0;
  }
}

// ------------------------------------------------------------------------

// The launch for step t_base + t_off: t_off and its residues.
static StepOff step_off(const StepArgs& a, uint32_t t_off) {
  StepOff o;
  o.t_off = t_off;
  o.d_slot = t_off % (uint32_t)a.D;
  o.d_phase = t_off % (uint32_t)a.rate_bin_steps;
  o.d_bin = (t_off / (uint32_t)a.rate_bin_steps) % (uint32_t)a.rate_bins_cap;
  return o;
}

hipError_t launch_gen(const GenArgs& a, int wdt, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  const int per_wave = gen_stage_bytes(a.K_out);
  int wpb = 60000 / per_wave;
  wpb = wpb < 1 ? 1 : (wpb > 4 ? 4 : wpb);
  const int64_t blocks = (a.N + wpb - 1) / wpb;
  const size_t lds = (size_t)wpb * per_wave;
  if (wdt == DPSNN_W_F32)
    hipLaunchKernelGGL(k_gen<DPSNN_W_F32>, dim3((unsigned)blocks), dim3(64 * wpb), lds, st, a);
  else if (wdt == DPSNN_W_F16)
    hipLaunchKernelGGL(k_gen<DPSNN_W_F16>, dim3((unsigned)blocks), dim3(64 * wpb), lds, st, a);
  else
    hipLaunchKernelGGL(k_gen<DPSNN_W_I8>, dim3((unsigned)blocks), dim3(64 * wpb), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_rows(const int32_t* tgt, const void* val, int val_bytes, int row_stride, int Ko,
                       int64_t rows, int32_t* out_tgt, void* out_val, hipStream_t st) {
  if (rows == 0 || Ko == 0) return hipSuccess;
  const dim3 grid((unsigned)rows), block(kRowThreads);
  const size_t lds = (size_t)gen_pow2(Ko) * 8;
  if (val_bytes == 4)
    hipLaunchKernelGGL(k_rows<uint32_t>, grid, block, lds, st, tgt,
                       static_cast<const uint32_t*>(val), row_stride, Ko, out_tgt,
                       static_cast<uint32_t*>(out_val));
  else if (val_bytes == 2)
    hipLaunchKernelGGL(k_rows<uint16_t>, grid, block, lds, st, tgt,
                       static_cast<const uint16_t*>(val), row_stride, Ko, out_tgt,
                       static_cast<uint16_t*>(out_val));
  else
    hipLaunchKernelGGL(k_rows<uint8_t>, grid, block, lds, st, tgt,
                       static_cast<const uint8_t*>(val), row_stride, Ko, out_tgt,
                       static_cast<uint8_t*>(out_val));
  return hipGetLastError();
}

hipError_t launch_absum_max(const unsigned long long* absum, int64_t n,
                            unsigned long long* out, hipStream_t st) {
  hipLaunchKernelGGL(k_absum_max, dim3(1024), dim3(256), 0, st, absum, n, out);
  return hipGetLastError();
}

hipError_t launch_init(const InitArgs& a, hipStream_t st) {
  const int64_t blocks = (a.N_pad + 255) / 256;
  hipLaunchKernelGGL(k_init, dim3((unsigned)blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <typename Acc, int FMT, int WDT>
static void launch_neuron_fmt(const StepArgs& a, uint32_t t_off, hipStream_t st) {
  const dim3 tiles((unsigned)a.n_tiles), block(256);
  const StepOff o = step_off(a, t_off);
  if (a.P <= 2)
    hipLaunchKernelGGL((k_neuron<Acc, 2, FMT, WDT>), tiles, block, 0, st, a, o);
  else if (a.two_cls)
    hipLaunchKernelGGL((k_neuron<Acc, 3, FMT, WDT>), tiles, block, 0, st, a, o);
  else
    hipLaunchKernelGGL((k_neuron<Acc, 4, FMT, WDT>), tiles, block, 0, st, a, o);
}

template <typename Acc>
static void launch_neuron(const StepArgs& a, uint32_t t_off, hipStream_t st) {
  if (a.q_code == kCodeF16) {
    launch_neuron_fmt<Acc, kFmtCode, DPSNN_W_F16>(a, t_off, st);
    return;
  }
  if (a.q_code == kCodeI8) {
    launch_neuron_fmt<Acc, kFmtCode, DPSNN_W_I8>(a, t_off, st);
    return;
  }
  if constexpr (sizeof(Acc) == 4) {
    if (a.q_packed) {
      launch_neuron_fmt<Acc, kFmtPacked, DPSNN_W_F32>(a, t_off, st);
      return;
    }
  }
  launch_neuron_fmt<Acc, kFmtWide, DPSNN_W_F32>(a, t_off, st);
}

template <typename Acc, bool SHORT>
static void launch_deliver_len(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  const dim3 block(kDlvThreads);
  const dim3 grid((unsigned)(a.log_blocks + a.emit_blocks + (a.q_cap ? a.deliver_grid : 0)));
  const StepOff o = step_off(a, t_off);
  const bool packed = sizeof(Acc) == 4 && a.q_packed;
  constexpr bool P4 = sizeof(Acc) == 4;
  if (a.plastic && packed)
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_F32, true, P4, SHORT>), grid, block, 0, st, a, o);
  else if (a.plastic)
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_F32, true, false, SHORT>), grid, block, 0, st, a, o);
  else if (wdt == DPSNN_W_F32 && packed)
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_F32, false, P4, SHORT>), grid, block, 0, st, a, o);
  else if (wdt == DPSNN_W_F32)
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_F32, false, false, SHORT>), grid, block, 0, st, a, o);
  else if (wdt == DPSNN_W_F16)
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_F16, false, false, SHORT>), grid, block, 0, st, a, o);
  else
    hipLaunchKernelGGL((k_deliver<Acc, DPSNN_W_I8, false, false, SHORT>), grid, block, 0, st, a, o);
}

template <typename Acc>
static void launch_deliver(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  if (a.piece_len == kShortPiece)
    launch_deliver_len<Acc, true>(a, wdt, t_off, st);
  else
    launch_deliver_len<Acc, false>(a, wdt, t_off, st);
}

template <typename Acc>
static void launch_split(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  launch_neuron<Acc>(a, t_off, st);
  launch_deliver<Acc>(a, wdt, t_off, st);
}

template <typename Acc, int NP, bool SHORT>
static void launch_fused_len(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  const int nd = a.fused_dlv;
  const dim3 grid((unsigned)(a.log_blocks + nd + (a.n_tiles + 1) / 2)), block(kDlvThreads);
  const StepOff o = step_off(a, t_off);
  if (wdt == DPSNN_W_F16) {
    hipLaunchKernelGGL((k_step<Acc, DPSNN_W_F16, NP, kFmtCode, SHORT>), grid, block, 0, st, a, o, nd);
    return;
  }
  if (wdt == DPSNN_W_I8) {
    hipLaunchKernelGGL((k_step<Acc, DPSNN_W_I8, NP, kFmtCode, SHORT>), grid, block, 0, st, a, o, nd);
    return;
  }
  if constexpr (sizeof(Acc) == 4) {
    if (a.q_packed) {
      hipLaunchKernelGGL((k_step<Acc, DPSNN_W_F32, NP, kFmtPacked, SHORT>), grid, block, 0, st, a, o,
                         nd);
      return;
    }
  }
  hipLaunchKernelGGL((k_step<Acc, DPSNN_W_F32, NP, kFmtWide, SHORT>), grid, block, 0, st, a, o, nd);
}

template <typename Acc, int NP>
static void launch_fused_np(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  if (a.piece_len == kShortPiece)
    launch_fused_len<Acc, NP, true>(a, wdt, t_off, st);
  else
    launch_fused_len<Acc, NP, false>(a, wdt, t_off, st);
}

template <typename Acc>
static void launch_fused(const StepArgs& a, int wdt, uint32_t t_off, hipStream_t st) {
  if (a.P <= 2)
    launch_fused_np<Acc, 2>(a, wdt, t_off, st);
  else if (a.two_cls)
    launch_fused_np<Acc, 3>(a, wdt, t_off, st);
  else
    launch_fused_np<Acc, 4>(a, wdt, t_off, st);
}

template <typename Acc, int WDT, int NP, int FMT>
static hipError_t launch_persist_t(const StepArgs& a, uint32_t t_off, uint32_t n,
                                   hipStream_t st) {
  const void* fn = reinterpret_cast<const void*>(&k_persist<Acc, WDT, NP, FMT>);
  const size_t lds = 0;
  int per_cu = 0, dev = 0, cus = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, &k_persist<Acc, WDT, NP, FMT>, 256, lds);
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (per_cu < 1 || cus < 1) return hipErrorLaunchFailure;
  StepArgs aa = a;
  StepOff o = step_off(a, t_off);
  uint32_t nn = n;
  void* args[] = {&aa, &o, &nn};
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)(per_cu * cus)), dim3(256), args,
                                    (unsigned)lds, st);
}

template <typename Acc, int NP>
static hipError_t launch_persist_np(const StepArgs& a, int wdt, uint32_t t_off, uint32_t n,
                                    hipStream_t st) {
  if (wdt == DPSNN_W_F16) return launch_persist_t<Acc, DPSNN_W_F16, NP, kFmtCode>(a, t_off, n, st);
  if (wdt == DPSNN_W_I8) return launch_persist_t<Acc, DPSNN_W_I8, NP, kFmtCode>(a, t_off, n, st);
  if constexpr (sizeof(Acc) == 4)
    if (a.q_packed) return launch_persist_t<Acc, DPSNN_W_F32, NP, kFmtPacked>(a, t_off, n, st);
  return launch_persist_t<Acc, DPSNN_W_F32, NP, kFmtWide>(a, t_off, n, st);
}

hipError_t launch_persist(const StepArgs& a, int wdt, int acc_bits, uint32_t t_off, uint32_t n,
                          hipStream_t st) {
  if (acc_bits == 32)
    return a.P <= 2 ? launch_persist_np<int32_t, 2>(a, wdt, t_off, n, st)
                    : launch_persist_np<int32_t, 4>(a, wdt, t_off, n, st);
  return a.P <= 2 ? launch_persist_np<int64_t, 2>(a, wdt, t_off, n, st)
                  : launch_persist_np<int64_t, 4>(a, wdt, t_off, n, st);
}

hipError_t launch_step(const StepArgs& a, int wdt, int acc_bits, int sched, uint32_t t_off,
                       hipStream_t st) {
  if (sched == DPSNN_SCHED_PERSIST) return launch_persist(a, wdt, acc_bits, t_off, 1, st);
  if (sched == DPSNN_SCHED_SPLIT) {
    if (acc_bits == 32)
      launch_split<int32_t>(a, wdt, t_off, st);
    else
      launch_split<int64_t>(a, wdt, t_off, st);
  } else {
    if (acc_bits == 32)
      launch_fused<int32_t>(a, wdt, t_off, st);
    else
      launch_fused<int64_t>(a, wdt, t_off, st);
  }
  return hipGetLastError();
}

// One phase of the split schedule on its own (0 = neuron update, 1 = delivery).
hipError_t launch_phase(const StepArgs& a, int wdt, int acc_bits, int phase, uint32_t t_off,
                        hipStream_t st) {
  if (phase == 0) {
    if (acc_bits == 32)
      launch_neuron<int32_t>(a, t_off, st);
    else
      launch_neuron<int64_t>(a, t_off, st);
  } else {
    if (acc_bits == 32)
      launch_deliver<int32_t>(a, wdt, t_off, st);
    else
      launch_deliver<int64_t>(a, wdt, t_off, st);
  }
  return hipGetLastError();
}

// Update of a tile: spike ids, input sums, totals of its wavefronts.
template <typename Acc>
static constexpr size_t update_lds() {
  return 1024 * 4 + 1024 * sizeof(Acc) + 4 * 4;
}

template <typename Acc, typename Ent>
static size_t step_lds(const StepArgs& a, int sched) {
  if (sched == DPSNN_SCHED_FUSED)
    return std::max(2 * update_lds<Acc>(), sizeof(DeliverLds<Ent, kDlvThreads, kFusedR, kFusedHash>));
  if (sched == DPSNN_SCHED_PERSIST)
    return std::max(update_lds<Acc>(), sizeof(DeliverLds<Ent, 256, kPersistR, kPersistHash>));
  const bool small = a.plastic || a.piece_len == kShortPiece || sizeof(Ent) == 8;
  return std::max(update_lds<Acc>(),
                  small ? sizeof(DeliverLds<Ent, kDlvThreads, kDlvRSmall, kDlvHash>)
                        : sizeof(DeliverLds<Ent, kDlvThreads, kDlvR, kDlvHash>));
}

size_t step_lds_bytes(const StepArgs& a, int wdt, int acc_bits, int sched) {
  const bool four = wdt != DPSNN_W_F32 || a.q_packed;
  if (acc_bits == 32)
    return four ? step_lds<int32_t, uint32_t>(a, sched)
                : step_lds<int32_t, unsigned long long>(a, sched);
  return four ? step_lds<int64_t, uint32_t>(a, sched)
              : step_lds<int64_t, unsigned long long>(a, sched);
}

hipError_t launch_drain(const StepArgs& a, int wdt, int acc_bits, uint32_t t, hipStream_t st) {
  if (a.q_cap == 0 || a.n_tiles == 0) return hipSuccess;
  const int lists = a.D * a.n_parts, share = std::max(1, std::min(16, 1024 / lists));
  const dim3 grid((unsigned)(a.n_tiles + lists * share)), block(256);
  if (acc_bits == 32) {
    if (wdt == DPSNN_W_F32)
      hipLaunchKernelGGL((k_drain<int32_t, DPSNN_W_F32>), grid, block, 0, st, a, t, share);
    else if (wdt == DPSNN_W_F16)
      hipLaunchKernelGGL((k_drain<int32_t, DPSNN_W_F16>), grid, block, 0, st, a, t, share);
    else
      hipLaunchKernelGGL((k_drain<int32_t, DPSNN_W_I8>), grid, block, 0, st, a, t, share);
  } else {
    if (wdt == DPSNN_W_F32)
      hipLaunchKernelGGL((k_drain<int64_t, DPSNN_W_F32>), grid, block, 0, st, a, t, share);
    else if (wdt == DPSNN_W_F16)
      hipLaunchKernelGGL((k_drain<int64_t, DPSNN_W_F16>), grid, block, 0, st, a, t, share);
    else
      hipLaunchKernelGGL((k_drain<int64_t, DPSNN_W_I8>), grid, block, 0, st, a, t, share);
  }
  return hipGetLastError();
}

// Periodic efficacy update of every plastic synapse after T steps (Sec. 2.1:
// the synapses apply their integrated plasticity signal once per period):
// w = clip(w + eta (y Dy(T - t_act)), 0, w_max), y = 0.
__global__ void __launch_bounds__(256) k_stdp_update(StepArgs a, int32_t T) {
  const int64_t total = a.N_pad * a.row_stride;
  const int32_t L = a.stdp_L;
  const float* Dy = a.stdp_tab + 2 * L;
  float* w = static_cast<float*>(const_cast<void*>(a.w));  // plastic efficacies
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = x / a.row_stride;
    const int j = (int)(x - s * a.row_stride);
    if (j >= a.K_out) continue;
    const NetDev& nd = a.nets[a.tile_net[s >> 10]];
    const int64_t il = s - nd.base;
    if (il >= nd.N) continue;  // padding
    const int l = (int)((uint32_t)il - module_of(nd, (uint32_t)il) * (uint32_t)nd.K);
    const int q = (l >= nd.pop_hi[0]) + (l >= nd.pop_hi[1]) + (l >= nd.pop_hi[2]);
    if (!nd.exc[q]) continue;
    const int32_t tl = a.syn_t[x];
    if (tl >= 0 && T - tl < L) {
      float v = w[x] + a.stdp_eta * (a.syn_y[x] * Dy[T - tl]);
      v = v < 0.0f ? 0.0f : (v > a.stdp_wmax ? a.stdp_wmax : v);
      w[x] = v;
    }
    a.syn_y[x] = 0.0f;
  }
}

hipError_t launch_stdp_update(const StepArgs& a, int32_t T, hipStream_t st) {
  const int64_t total = a.N_pad * a.row_stride;
  const int64_t blocks = std::min<int64_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_stdp_update, dim3((unsigned)blocks), dim3(256), 0, st, a, T);
  return hipGetLastError();
}

hipError_t launch_tick(const StepArgs& a, uint32_t n, int sched, hipStream_t st) {
  hipLaunchKernelGGL(k_tick, dim3(1), dim3(kTickThreads), 0, st, a, n, sched == DPSNN_SCHED_FUSED ? 1 : 0);
  return hipGetLastError();
}

}  // namespace dpsnn
