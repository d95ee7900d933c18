// Device code of the decode step for gfx950 (CDNA4), included by the
// translation units that instantiate the step kernel (kl_step_*.hip).
//
// One kernel, kl_step_kernel, runs any contiguous run of the step's phases:
//   embed | for each layer: qkv, attn, oproj, gateup, down | head
// The three schedules differ only in how many launches cover the run:
//   looped     one cooperative launch for everything (kernel looping, Sec. 2
//              and Sec. 3.2 of arXiv 2410.23668: the L chained layer calls
//              become one call with an outer loop; kernel boundaries become
//              tagged words and device-scope counters),
//   per-layer  one launch per layer (the fused-layer kernel K0 of Sec. 2),
//   per-op     one launch per phase.
// The work partition depends only on StepParams::nwg, so every schedule
// performs the same arithmetic in the same order: results are bit-identical.
//
// Pipelining across phases (the "pipelined outer loop" of Sec. 3.2): a phase
// issues the first loads of its weight tiles before it waits for its input
// activations, so HBM keeps streaming while the grid synchronises.  Data that crosses workgroups (activations, partials,
// the new KV slot) is written and read with device-coherent (agent-scope)
// accesses, so a barrier needs no cache write-back or invalidation: only the
// completion of the stores before the arrival.
//
// Weights are pre-packed into 1 KiB tiles of 8 rows x 64 columns (bf16,
// row-major inside the tile); the tiles of one 8-row group are contiguous
// along K.  A wave reads one tile per 16-byte-per-lane load: lane l holds row
// l/8, columns 8*(l%8) .. +7.  Activations are fp32 in LDS; accumulation is
// fp32 with a fixed order.

#pragma once

#include <type_traits>

#include "kl_internal.h"
#include "kl_shares.h"
#include "kl.h"

namespace kl {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- helpers

// The thread's index in its workgroup, opaque to the compiler at each use:
// values derived from it are formed where they are used instead of being
// hoisted out of the layer loop and kept live (or spilled) across the kernel.
__device__ __forceinline__ unsigned kl_tid() {
    unsigned t = __builtin_amdgcn_workitem_id_x();
    asm volatile("" : "+v"(t));
    return t;
}

__device__ __forceinline__ float bf_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((unsigned)h << 16); }

// fp32 -> bf16, round to nearest even (one conversion instruction on gfx950).
__device__ __forceinline__ uint16_t f2bf(float f) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

// The two bf16 terms of a matrix-core activation: hi = bf16(x), lo =
// bf16(x - hi) (x - hi is exact in fp32), so hi + lo = x (1 + O(2^-17)).
__device__ __forceinline__ void split_bf16(float x, uint16_t &hi, uint16_t &lo) {
    hi = f2bf(x);
    lo = f2bf(x - bf2f(hi));
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 CTRL, 0xF, 0xF, false));
}
// DPP controls: quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E,
// row_half_mirror = 0x141, row_mirror = 0x140.
// Sum over aligned groups of 8 lanes; every lane of the group gets the sum.
__device__ __forceinline__ float sum8(float v) {
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    return v;
}
__device__ __forceinline__ float sum16(float v) { v = sum8(v); return v + dpp<0x140>(v); }

// op(v, v of lane ^ 16) and op(v, v of lane ^ 32) by the row and half swaps
// of gfx950.  (The shuffle built on the lane index keeps that index live across
// the whole kernel; spilled, its reload in a staging step waits for every
// load in flight, the weight ring included.)
template <class Op>
__device__ __forceinline__ float xor16(float v, Op &&op) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float xor32(float v, Op &&op) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_16_32(float v) {
    const auto add = [](float a, float b) { return a + b; };
    return xor32(xor16(v, add), add);
}
__device__ __forceinline__ float max_16_32(float v) {
    const auto mx = [](float a, float b) { return fmaxf(a, b); };
    return xor32(xor16(v, mx), mx);
}
__device__ __forceinline__ float wave_sum(float v) { return sum_16_32(sum16(v)); }
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<0xB1>(v));
    v = fmaxf(v, dpp<0x4E>(v));
    v = fmaxf(v, dpp<0x141>(v));
    v = fmaxf(v, dpp<0x140>(v));
    return max_16_32(v);
}
// the value of another lane
__device__ __forceinline__ int from_lane(int v, int lane) {
    return __builtin_amdgcn_ds_bpermute(lane * 4, v);
}
__device__ __forceinline__ float from_lane(float v, int lane) {
    return __int_as_float(from_lane(__float_as_int(v), lane));
}

// Sum over the workgroup; every thread gets the same value (fixed order).
__device__ __forceinline__ float block_sum(float v, float *sm) {
    v = wave_sum(v);
    const int wid = kl_tid() >> 6;
    if ((kl_tid() & 63) == 0) sm[wid] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += sm[w];
    __syncthreads();
    return t;
}

__device__ __forceinline__ void split_range(int n, int parts, int i, int &a, int &b) {
    a = (int)((long long)n * i / parts);
    b = (int)((long long)n * (i + 1) / parts);
}

// The same for the rows of a long weight stream, 4 % more to the workgroups
// on even XCDs (workgroup w runs on XCD w % 8) and 4 % less to those on odd
// ones.  Under a full read stream the odd XCD of each pair gets 8 to 10 % less
// of the bandwidth: with equal shares the 70B shape's gate/up product ended
// after 128 us on even XCDs and 140 us on odd ones, the 8B shape's LM head
// after 140 and 152.  (Bounds are rounded down: with part 0 on an even XCD,
// shares of a few rows come out equal; with part 0 on an odd one, as some FFN
// column blocks of an odd number of workgroups, a share below 25 rows that
// divides evenly leans by a row, 44 rows in 11 parts as 3 and 5 in turn.
// Rounding it to equal shares was measured level: hidden 1024, ffn 1472, 8
// layers 277 us either way.)
__device__ __forceinline__ void split_rows(int n, int parts, int i, int &a, int &b) {
    const int odd = (blockIdx.x - i) & 1;   // XCD parity of part 0
    const auto bound = [&](int k) {
        const long long skew = (k & 1) ? (odd ? -1 : 1) : 0;   // in 1/25 of a share
        return k == parts ? n : (int)(n * (25ll * k + skew) / (25ll * parts));
    };
    a = bound(i);
    b = bound(i + 1);
}

// A sequence whose token or position is out of range still runs through the
// step with clamped values (every read stays in bounds), but writes nothing
// the caller owns except NaN logits and hidden state: its K/V slots are left
// untouched.  The embedding phase raises the matching error bits.
// Greedy sampling (the Sampling block, Sec. 2, Fig. 3) reduces each
// candidate logit to a 64-bit key, (order-preserving bits of the logit << 32)
// | (0xFFFFFFFF - index): the largest key is the largest logit and, among equal
// logits, the lowest index.  NaN logits (a skipped sequence) are no
// candidates; key 0 means none and decodes to token -1 (out of range).
__device__ __forceinline__ unsigned long long argmax_key(float v, int idx) {
    const unsigned u = __float_as_uint(v);
    const unsigned ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)ord << 32) | (0xFFFFFFFFu - (unsigned)idx);
}
__device__ __forceinline__ int key_token(unsigned long long k) {
    return k ? (int)(0xFFFFFFFFu - (unsigned)k) : -1;
}
__device__ __forceinline__ int raw_tok(const StepParams &P, int b) {
    if (P.tok_keys)
        return key_token(__hip_atomic_load(const_cast<unsigned long long *>(P.tok_keys + b),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return P.tokens[b];
}
__device__ __forceinline__ int raw_pos(const StepParams &P, int b) {
    return P.positions[b] + P.pos_add;
}

__device__ __forceinline__ int eff_pos(const StepParams &P, int b) {
    const int p = raw_pos(P, b);
    const int lim = min(P.cap, P.max_seq);
    return p < 0 ? 0 : (p >= lim ? lim - 1 : p);
}
__device__ __forceinline__ int eff_tok(const StepParams &P, int b) {
    const int t = raw_tok(P, b);
    return (t < 0 || t >= P.V) ? 0 : t;
}
__device__ __forceinline__ bool seq_ok(const StepParams &P, int b) {
    const int t = raw_tok(P, b), p = raw_pos(P, b);
    return t >= 0 && t < P.V && p >= 0 && p < min(P.cap, P.max_seq);
}
// On the per-sequence path (at most kMfmaBatch - 1 sequences) both are read once per launch
// into LDS (bar_init), so that no phase starts with a dependent memory round
// trip for them.
__device__ __forceinline__ int *seq_table(const StepParams &P);
template <bool PS>
__device__ __forceinline__ int pos_of(const StepParams &P, int b) {
    if constexpr (PS) return seq_table(P)[b];
    else return eff_pos(P, b);
}
template <bool PS>
__device__ __forceinline__ bool ok_of(const StepParams &P, int b) {
    if constexpr (PS) return seq_table(P)[kMfmaBatch + b] != 0;
    else return seq_ok(P, b);
}

__device__ __forceinline__ size_t kv_row(const StepParams &P, int l, int b, int g) {
    return (((size_t)l * P.kv_batch + b) * P.nkv + g) * (size_t)P.cap;
}

// ---------------------------------------------------------------- coherent accesses
//
// Relaxed agent-scope atomic loads and stores compile to ordinary vector
// memory instructions with the device-coherence bit (sc1): they see, and are
// seen by, every XCD without flushing or invalidating the XCD-private L2.

__device__ __forceinline__ void st_dev(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev_u16(uint16_t *p, uint16_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev_u32(unsigned *p, unsigned v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The residual stream is kept in fixed point: int64 in units of 2^-32.  Every
// contribution (the embedding, each O-projection partial, each
// down-projection partial) is rounded once to that grid and added with an
// integer atomic, so the sum is exact and independent of the order in which
// workgroups add: results are reproducible however the work is split.  The
// range (+-2^31) and resolution (2^-32) are far beyond fp32 activations'.
constexpr double kFixScale = 4294967296.0;   // 2^32
__device__ __forceinline__ long long to_fix(double v) { return __double2ll_rn(v * kFixScale); }
__device__ __forceinline__ float from_fix(long long v) {
    return (float)v * (1.0f / 4294967296.0f);
}
__device__ __forceinline__ void st_dev_u64(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_dev(const float *p) {
    return __hip_atomic_load(const_cast<float *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_dev_u64(const void *p) {
    return __hip_atomic_load(reinterpret_cast<unsigned long long *>(const_cast<void *>(p)),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32x4 ld_stream_16B(const void *p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}

// Block barrier for LDS hand-offs only: the wave's LDS operations complete,
// then s_barrier; unlike __syncthreads (whose workgroup release fence also
// waits for every outstanding memory load), loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// s_waitcnt vmcnt(0): this wave's stores have completed at their coherence point.
__device__ __forceinline__ void wait_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// ---------------------------------------------------------------- grid barrier
//
// Arrival counting on monotonically increasing 64-bit counters, one per
// group of workgroups: workgroup w arrives on counter w % ng (one atomic
// add), and a waiter's wave 0 polls all ng counters at once, one per lane.
// Spreading arrivals over ng counters keeps the atomics on any one address
// few; polling them directly saves a second atomic hop.  The counters are
// never reset: every launch ends with counter g at E * size_g, E being the
// number of barriers completed so far, and at launch start each workgroup
// recovers E from its own group's counter.  Barrier k of a launch is complete
// when counter g reaches base_g + (k + 1) * size_g for every group g.  The
// wait is bounded by a poll count: past it, KL_DEVERR_BARRIER is raised and every
// later wait returns at once, so a broken barrier ends the kernel instead of
// hanging it.
constexpr int kSpinLimit = 1 << 22;   // polls before a wait gives up (well over a second)

// The per-group bases of the current launch live in the dynamic LDS area (a
// fixed slot after everything else; see lds_layout), which every phase
// function addresses the same way.
extern __shared__ __align__(16) char kl_smem[];
__device__ __forceinline__ unsigned long long *bar_bases(const StepParams &P);

__device__ __forceinline__ int bar_groups(const StepParams &P) { return bar_group_count(P.nwg); }
__device__ __forceinline__ unsigned bar_gsize(const StepParams &P, int ng, int g) {
    return bar_group_size(P.nwg, ng, g);
}
__device__ __forceinline__ unsigned long long *bar_counter(const StepParams &P, int g) {
    return P.bar + 32 * (g + 1);   // 256 bytes apart
}

// At launch start: the barrier bases of this launch and the step's first tag
// of the tagged hand-offs, into LDS (before any wait; any wave may do it).
__device__ __forceinline__ unsigned *launch_epoch(const StepParams &P);
__device__ __forceinline__ void seg_init(const StepParams &P, int lane);
struct OwnRows { int first, count; };
__device__ __forceinline__ OwnRows own_rows(const StepParams &P);
__device__ __forceinline__ long long *own_x(const StepParams &P);
__device__ __forceinline__ void bar_init(const StepParams &P) {
    // Only this workgroup's own group counter is read: that group cannot
    // complete barrier 0 before this workgroup arrives, so the value rounds
    // down to the number E of whole barriers done by earlier launches.  Any
    // other group may already be one barrier further, so its base is E times
    // its size, not its current value rounded down.
    const int ng = bar_groups(P);
    const unsigned t = kl_tid();
    if (t < (unsigned)ng) {
        const int own = blockIdx.x % ng;
        const unsigned long long c = ld_dev_u64(bar_counter(P, own));
        bar_bases(P)[t] = bar_launch_base(c, P.nwg, ng, own, (int)t);
    } else if (t == 64) {
        *launch_epoch(P) = __hip_atomic_load(P.epoch_ptr, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    } else if (t >= 128 && t < 192) {
        seg_init(P, (int)t - 128);
    } else if (t >= 96 && t < 96 + kMfmaBatch && !P.batched) {
        const int b = (int)t - 96;
        if (b < P.B) {
            seq_table(P)[b] = eff_pos(P, b);
            seq_table(P)[kMfmaBatch + b] = seq_ok(P, b) ? 1 : 0;
        }
    }
    if (!P.batched) {   // the residual as the launch before left it
        const OwnRows R = own_rows(P);
        for (int i = (int)t; i < P.B * R.count; i += kThreads)
            own_x(P)[(i / R.count) * P.own_max + i % R.count] = (long long)ld_dev_u64(
                P.xf + (size_t)(i / R.count) * P.Hp + R.first + i % R.count);
    }
    __syncthreads();
}

// Optional timeline: the control wave of every workgroup stamps
// (s_memrealtime, 100 MHz) the end of phase i of the launch (slot 0), the
// start and end of phase i's wait for its inputs (slots 1, 2) and the moment
// its inputs are staged (slot 3: the GEMV path's first activation vector in
// LDS, the batched path's normalised activations written by the whole grid,
// an attention phase's last chunk result published).
__device__ __forceinline__ void trace_stamp(const StepParams &P, int i, int what) {
    if (P.trace && i >= 0 && i < P.trace_max)
        P.trace[((size_t)i * P.nwg + blockIdx.x) * 4 + what] = wall_clock64();
}

// The control wave (kCtlWave) does all of a workgroup's barrier traffic.  It
// never has weight or KV loads in flight, so its polls are not queued behind
// the compute waves' prefetches (a wave's loads complete in issue order).
__device__ __forceinline__ bool is_ctl_lane0() { return kl_tid() == kCtlWave * 64; }

// Every wave drains its stores (they must be visible before the signal),
// then the control wave signals.
__device__ __forceinline__ void drain_all() {
    wait_stores();
    __syncthreads();
}

// Arrival on grid barrier k after phase ti.
// (the phase's end is stamped once every wave of the workgroup is done)
__device__ __forceinline__ void bar_arrive(const StepParams &P, int k, int ti) {
    drain_all();
    if (is_ctl_lane0()) {
        trace_stamp(P, ti, 0);
        __hip_atomic_fetch_add(bar_counter(P, blockIdx.x % bar_groups(P)), 1ull,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Arrival on a local counter (one add per arriving workgroup) after phase ti.
__device__ __forceinline__ void local_arrive(const StepParams &P, unsigned *cnt, int ti) {
    drain_all();
    if (is_ctl_lane0()) {
        trace_stamp(P, ti, 0);
        __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Spin until *flag_fn() says done; gives up (raising KL_DEVERR_BARRIER) after
// kSpinLimit polls or as soon as another wait has given up.
template <class Done>
__device__ __forceinline__ void spin_until(const StepParams &P, Done &&done) {
    for (int spins = 1;; ++spins) {
        if (done()) return;
        if ((spins & 63) == 0 &&
            (__hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
             KL_DEVERR_BARRIER))
            return;
        if (spins >= kSpinLimit) {
            __hip_atomic_fetch_or(P.err, KL_DEVERR_BARRIER, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
    }
}

__device__ __forceinline__ void bar_wait(const StepParams &P, int k, int ti) {
    if ((kl_tid() >> 6) == kCtlWave) {
        const int lane = kl_tid() & 63, ng = bar_groups(P);
        const bool mine = lane < ng;
        const unsigned long long target =
            mine ? bar_target(bar_bases(P)[lane], k, P.nwg, ng, lane) : 0ull;
        if (lane == 0) trace_stamp(P, ti, 1);
        spin_until(P, [&]() {
            const bool d = !mine || bar_reached(ld_dev_u64(bar_counter(P, lane)), target);
            return __all(d) != 0;
        });
        if (lane == 0) trace_stamp(P, ti, 2);
    }
    __syncthreads();
}

// ---------------------------------------------------------------- tagged hand-offs
//
// On the per-sequence path, values that cross workgroups inside a layer (the
// rotated queries and the new key and value for the attention, the chunk
// results for the O projection, the SwiGLU output for the down projection)
// travel as tagged words: one 8-byte word holds the 32-bit value and the tag
// of the step and layer that wrote it, written and read as one
// device-coherent access.  A reader polls the words themselves and takes a
// value once its tag is the current one.  The writer therefore needs no
// drain of its stores and no counter, and the reader no separate wait before
// loading: a hand-off costs the time for the stores to land plus one load
// round trip, instead of store drain, counter atomic, counter poll and data
// load one after the other.  Tags are epoch + layer, each step using a fresh
// range of tags that never includes 0 (cleared memory); the epoch is read at
// launch start and advanced by the step's last phase once every workgroup has
// read it (ll_next_epoch, epoch_last_arrival).
__device__ __forceinline__ unsigned ll_tag(const StepParams &P, int l) {
    return *launch_epoch(P) + (unsigned)l;
}
__device__ __forceinline__ void st_ll(unsigned long long *p, unsigned v, unsigned tag) {
    st_dev_u64(p, ll_word(v, tag));
}
__device__ __forceinline__ void st_ll_f(unsigned long long *p, float v, unsigned tag) {
    st_ll(p, __float_as_uint(v), tag);
}

// Threads tid = 0 .. nt - 1 (the caller's numbering) gather n tagged words:
// word i (address addr(i)) goes to put(i, value) once it carries 'tag'.  Each
// thread takes words tid, tid + nt, ... in rounds of W, issuing a round's
// loads together (from in-range addresses, masked when used) and reloading
// the round until every word of it is current.  A round gives up after
// kSpinLimit polls, raising KL_DEVERR_BARRIER, so a missing writer ends the
// kernel instead of hanging it.
template <int W, class Addr, class Put>
__device__ __forceinline__ void ll_gather(const StepParams &P, int n, unsigned tag, int tid,
                                          int nt, Addr &&addr, Put &&put) {
    for (int base = 0; base < n; base += W * nt) {
        unsigned long long v[W];
        for (int spins = 1;; ++spins) {
#pragma unroll
            for (int k = 0; k < W; ++k) v[k] = ld_dev_u64(addr(min(base + tid + k * nt, n - 1)));
            bool ok = true;
#pragma unroll
            for (int k = 0; k < W; ++k) ok = ok && (base + tid + k * nt >= n || ll_current(v[k], tag));
            if (ok) break;
            if ((spins & 63) == 0 &&
                (__hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
                 KL_DEVERR_BARRIER))
                break;
            if (spins >= kSpinLimit) {
                __hip_atomic_fetch_or(P.err, KL_DEVERR_BARRIER, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
#pragma unroll
        for (int k = 0; k < W; ++k)
            if (base + tid + k * nt < n) put(base + tid + k * nt, ll_value(v[k]));
    }
}

// ---------------------------------------------------------------- params
//
// The step kernel is one function per (head_dim, group size), with every
// phase inlined (no calls: a call would save and restore callee-saved
// registers through scratch memory on every phase).  Each phase reads the
// step parameters from the kernel-argument segment itself, through an
// address the compiler cannot see through, so the loads stay inside the
// phase instead of being hoisted out of the layer loop, where the values of
// all phases together would exhaust the registers.
#define KL_KARG __attribute__((address_space(4)))

typedef uint64_t KArg;

__device__ __forceinline__ KArg kernarg_address() {
#if defined(__HIP_DEVICE_COMPILE__)
    return (KArg)(const KL_KARG char *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    return 0;
#endif
}

__device__ __forceinline__ StepParams load_params(KArg ka) {
#if defined(__HIP_DEVICE_COMPILE__)
    unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)ka);
    unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(ka >> 32));
    asm volatile("" : "+s"(lo), "+s"(hi));
    const KL_KARG StepParams *p = (const KL_KARG StepParams *)(((KArg)hi << 32) | lo);
    return *p;
#else
    return StepParams{};   // the host pass only type-checks device code
#endif
}

// ---------------------------------------------------------------- LDS layout

// Offsets (in floats) come from the host, which sizes the allocation.

struct Lds {
    float *a;     // activation vector (max K extent); aliased by the attention area
    float *attn;  // attention scratch (same storage as a)
    float *red;   // [kWaves][kRgBatch][kTileRows] GEMV partial sums
    float *sm;    // small reductions and flags (64 floats)
    unsigned long long *bar;   // [kBarGroups] barrier bases of this launch
};

__device__ __forceinline__ Lds lds_layout(char *smem, const StepParams &P) {
    Lds s;
    float *f = reinterpret_cast<float *>(smem);
    s.a = f;
    s.attn = f;
    s.red = f + P.lds_red;
    s.sm = f + P.lds_sm;
    s.bar = reinterpret_cast<unsigned long long *>(f + P.lds_bar);
    return s;
}
__device__ __forceinline__ uint8_t *mm_slots(const StepParams &P, const Lds &S) {
    return P.multi == 2 ? reinterpret_cast<uint8_t *>(S.a + P.lds_mm) : nullptr;
}
// P.multi = 2: the pass runs on the matrix cores; a staged vector is three
// bf16 terms (all 24 bits), column 4 t + b of the B operand being term t of
// sequence b, in rows of mm_stride(K) elements.
constexpr int kMmCols = 3 * kMultiSeq;
__device__ __forceinline__ constexpr int mm_stride(int K) { return K + 8; }   // (bank spread)
__device__ __forceinline__ uint16_t *mm_act(const Lds &S) {
    return reinterpret_cast<uint16_t *>(S.a);
}
__device__ __forceinline__ void mm_put(uint16_t *x, int stride, int b, int i, float v) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const uint16_t h = f2bf(v);
        x[(4 * t + b) * stride + i] = h;
        v -= bf2f(h);
    }
}
// Per-sequence path: with P.multi the B sequences share each GEMV pass, their
// staged vectors one after the other in the activation area (sequence b's wave
// sums of squares b kSmSeq floats into sm); otherwise every sequence is staged
// at the start of the area in turn.
__device__ __forceinline__ float *seq_sm(const StepParams &P, const Lds &S, int b);
// The Q/K/V phase's staged RoPE row (cos, sin) of sequence b: after the
// activation vectors.
__device__ __forceinline__ float *rope_row(const StepParams &P, const Lds &S, int b) {
    if (P.multi == 2) return S.a + kMmCols * mm_stride(P.Hp) / 2 + b * P.d;
    return S.a + (P.multi ? kMultiSeq * P.Hp + b * P.d : P.Hp);
}

__device__ __forceinline__ unsigned long long *bar_bases(const StepParams &P) {
    return lds_layout(kl_smem, P).bar;
}
// (after the barrier bases)
__device__ __forceinline__ unsigned *launch_epoch(const StepParams &P) {
    return reinterpret_cast<unsigned *>(lds_layout(kl_smem, P).bar + kBarGroups);
}
// (after the epoch: position and validity of each sequence, per-sequence path)
__device__ __forceinline__ int *seq_table(const StepParams &P) {
    return reinterpret_cast<int *>(lds_layout(kl_smem, P).bar + kBarGroups) + 4;
}
// (then, mixture of experts: per sequence, its two experts and their
// weights (float bits), chosen in the gate/up phase, used by the down phase)
__device__ __forceinline__ int *route_table(const StepParams &P) {
    return seq_table(P) + 2 * kMfmaBatch;
}

// (then: the workgroup's share of the attention, see seg_init)
__device__ __forceinline__ int *seg_table(const StepParams &P) {
    return route_table(P) + 4 * kMfmaBatch;
}
// (then: the head's argmax keys of up to kMfmaBatch or, on the matrix-core
// path, kGemmBatch sequences)
__device__ __forceinline__ unsigned long long *amax_slots(const StepParams &P) {
    return reinterpret_cast<unsigned long long *>(seg_table(P) + 8);
}
// (then, per-sequence path: the residual rows this workgroup owns, int64
// fixed point [sequence][own_max])
__device__ __forceinline__ long long *own_x(const StepParams &P) {
    return reinterpret_cast<long long *>(amax_slots(P) + kMfmaBatch);
}

// ---------------------------------------------------------------- activations

// Cache-policy bits (sc1, device-coherent) of the copies from device memory
// straight to LDS (global_load_lds, 16 bytes per lane), and the wait for a
// wave's copies.
constexpr int kLdsCoherent = 16;
__device__ __forceinline__ void ctl_copy_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Activation staging: loads are issued in batches of kStageBatch per thread
// before any is used.
constexpr int kStageBatch = 8;
// a[i] = x[i] * rsqrt(mean(x^2) + eps) * gain[i] for i < n, 0 up to npad,
// x read from the fixed-point residual stream.  The gain is loaded in the
// same batch as x (a dependent second batch would cost a second memory round
// trip, ~2 us when HBM is saturated), and so are the ne floats of an optional
// extra vector (esrc -> edst in LDS), e.g. the RoPE row the epilogue needs.
// RMSNorm staging for the GEMV path, with the normalisation deferred: the
// weight product is linear, so W (x r g) = r (W (x g)) with the per-sequence
// scale r = 1 / sqrt(mean(x^2) + eps) applied in the epilogue (rms_scale).
// Stages a = x g (zero padding) and leaves each wave's partial sum of x^2
// in sm[wave]; the weight stream starts as soon as a is in LDS, without
// waiting for a block-wide reduction.  x arrives as tagged words (xw, tag),
// which the threads poll themselves: the hand-off costs the words' stores and
// one load round trip, where a grid barrier cost the drain of the adds, its
// counters' round trip and then the load's.
__device__ __forceinline__ bool give_up(const StepParams &P, int spins) {
    if ((spins & 63) == 0 &&
        (__hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & KL_DEVERR_BARRIER))
        return true;
    if (spins < kSpinLimit) return false;
    __hip_atomic_fetch_or(P.err, KL_DEVERR_BARRIER, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}
__device__ __forceinline__ void stage_rms_deferred(const StepParams &P,
                                                   const unsigned long long *__restrict__ xw,
                                                   unsigned tag, const float *__restrict__ gain,
                                                   int n, int npad, float *a, float *sm,
                                                   const float *esrc = nullptr,
                                                   float *edst = nullptr, int ne = 0) {
    float ss = 0.f;
    for (int i0 = kl_tid(); i0 < npad; i0 += kStageBatch * kThreads) {
        unsigned long long v[kStageBatch];
        float gv[kStageBatch];
        float ev = 0.f;
        const bool first = i0 == (int)kl_tid();
        // (every load is unconditional, from a clamped address, and masked
        // when used: a conditional device-coherent load becomes a branch that
        // waits for its load before the next one is issued)
#pragma unroll
        for (int k = 0; k < kStageBatch; ++k) {
            const int i = i0 + k * kThreads;
            const float g = gain[min(i, n - 1)];
            gv[k] = i < n ? g : 0.f;
        }
        if (first && (int)kl_tid() < ne) ev = esrc[kl_tid()];
        for (int spins = 1;; ++spins) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < kStageBatch; ++k) v[k] = ld_dev_u64(xw + min(i0 + k * kThreads, n - 1));
#pragma unroll
            for (int k = 0; k < kStageBatch; ++k) ok = ok && ll_current(v[k], tag);
            if (ok || give_up(P, spins)) break;
        }
#pragma unroll
        for (int k = 0; k < kStageBatch; ++k) {
            const int i = i0 + k * kThreads;
            const float x = i < n ? __uint_as_float(ll_value(v[k])) : 0.f;
            ss = fmaf(x, x, ss);
            if (i < npad) a[i] = x * gv[k];
        }
        if (first && (int)kl_tid() < ne) edst[kl_tid()] = ev;
    }
    ss = wave_sum(ss);
    if ((kl_tid() & 63) == 0) sm[kl_tid() >> 6] = ss;
    lds_barrier();
}
// The same for sequences 0 .. nb - 1 (nb <= kMultiSeq) together, their loads
// issued in one batch: sequence b's words at xw + b xstride, its
// staged vector at a + b astride, its wave sums at sm + b kSmSeq, and the ne
// floats esrc(b) -> edst(b).  (Loads for b >= nb repeat sequence nb - 1's
// and are dropped: every load stays unconditional.)  Half the batch per
// sequence keeps the loads in flight within the registers the weight ring
// leaves.  The sum of a thread's terms is taken in the order of
// stage_rms_deferred, so the values are the same.
constexpr int kSmSeq = kThreads / 64;   // floats between sequences' wave sums
constexpr int kStageMulti = 4;          // loads per thread and sequence per batch
struct NoExtra {   // stage_rms_multi without an extra vector
    __device__ float *operator()(int) const { return nullptr; }
};
template <class ESrc, class EDst>
__device__ __forceinline__ void stage_rms_multi(const StepParams &P,
                                                const unsigned long long *__restrict__ xw,
                                                int xstride, unsigned tag,
                                                const float *__restrict__ gain, int n, int npad,
                                                int nb, float *a, int astride, float *sm,
                                                ESrc &&esrc, EDst &&edst, int ne) {
    float ss[kMultiSeq];
#pragma unroll
    for (int bb = 0; bb < kMultiSeq; ++bb) ss[bb] = 0.f;
    for (int i0 = kl_tid(); i0 < npad; i0 += kStageMulti * kThreads) {
        unsigned long long v[kMultiSeq][kStageMulti];
        float gv[kStageMulti], ev[kMultiSeq];
        const bool first = i0 == (int)kl_tid();
#pragma unroll
        for (int k = 0; k < kStageMulti; ++k) {
            const int i = i0 + k * kThreads;
            const float g = gain[min(i, n - 1)];
            gv[k] = i < n ? g : 0.f;
        }
        if (first && (int)kl_tid() < ne) {
#pragma unroll
            for (int bb = 0; bb < kMultiSeq; ++bb) ev[bb] = esrc(min(bb, nb - 1))[kl_tid()];
        }
        for (int spins = 1;; ++spins) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < kStageMulti; ++k)
#pragma unroll
                for (int bb = 0; bb < kMultiSeq; ++bb)
                    v[bb][k] = ld_dev_u64(xw + (size_t)min(bb, nb - 1) * xstride +
                                          min(i0 + k * kThreads, n - 1));
#pragma unroll
            for (int k = 0; k < kStageMulti; ++k)
#pragma unroll
                for (int bb = 0; bb < kMultiSeq; ++bb) ok = ok && ll_current(v[bb][k], tag);
            if (ok || give_up(P, spins)) break;
        }
#pragma unroll
        for (int bb = 0; bb < kMultiSeq; ++bb) {
            if (bb < nb) {
#pragma unroll
                for (int k = 0; k < kStageMulti; ++k) {
                    const int i = i0 + k * kThreads;
                    const float x = i < n ? __uint_as_float(ll_value(v[bb][k])) : 0.f;
                    ss[bb] = fmaf(x, x, ss[bb]);
                    if (i < npad) {
                        if (P.multi == 2)
                            mm_put(reinterpret_cast<uint16_t *>(a), mm_stride(npad), bb, i, x * gv[k]);
                        else
                            a[bb * astride + i] = x * gv[k];
                    }
                }
                if (first && (int)kl_tid() < ne) edst(bb)[kl_tid()] = ev[bb];
            }
        }
    }
#pragma unroll
    for (int bb = 0; bb < kMultiSeq; ++bb) {
        if (bb < nb) {
            const float t = wave_sum(ss[bb]);
            if ((kl_tid() & 63) == 0) sm[bb * kSmSeq + (kl_tid() >> 6)] = t;
        }
    }
    lds_barrier();
}
// The scale r of the sequence staged last by stage_rms_deferred (the wave
// partials are added in wave order: the same value in every thread).
__device__ __forceinline__ float rms_scale(const float *sm, int n, float eps) {
    float ss = 0.f;
#pragma unroll
    for (int w = 0; w < kSmSeq; ++w) ss += sm[w];
    return 1.0f / sqrtf(ss / (float)n + eps);
}
__device__ __forceinline__ float *seq_sm(const StepParams &P, const Lds &S, int b) {
    return S.sm + (P.multi ? b * kSmSeq : 0);
}

// ---------------------------------------------------------------- GEMV engine
//
// y_b[r] = sum_k W[r][k] a_b[k] for the rows of the row groups a workgroup owns in a
// packed matrix with KT k-tiles per row group, for each sequence b.  Each
// wave takes a fixed slice of the k-tiles of every row group (split-K inside
// the workgroup), keeps U tile loads in flight, and reduces its partial dot
// products over the 8 lanes of a row with DPP.  The slices are summed in wave
// order through LDS, and epi(b, r, y_r, y_r+1) is called once per row pair.
// Row groups are processed in batches of kRgBatch.  The first loads are
// issued before wait() (whatever precedes the staging of the activations) and
// before stage(b) (which fills a with sequence b's activation vector); each
// next batch's first loads are issued before the previous batch's reduction.
// Tile loads in flight per wave (8 KiB; 16 MB over the chip, 2.5 us of HBM).
// Twice as many stream no faster, and what a phase waits for at its start
// (tagged words, activations) queues behind the first ring: 8B shape, batch
// 1, 2980 us a step against 3129 with 16.
constexpr int kGemvDepth = 8;
constexpr int kGemmDepth = 16;   // matrix-core path
// one sequence's GEMV partial sums in the reduction area (either row sharing)
constexpr int kRedStride = kWaves * kRgBatch * kTileRows;

// The ring of tile loads must stay in flight across loop iterations, the
// grid barrier and the activation staging, and the compiler only places a
// precise "wait for the oldest load" (vmcnt(U-1)) when every path issues the
// same loads.  So the ring is refilled unconditionally: once the batch's real
// tiles are exhausted, a slot is refilled from a 16-byte dummy line that all
// lanes share (one cache line per wave), and only the consumption of a slot
// is conditional.
//
// A workgroup owns the row groups first .. first + count - 1 (a strided
// assignment, stride = grid size, was measured no faster).
struct RgRange { int first, count; };
template <bool BAT>
__device__ __forceinline__ RgRange own_rgs(int nrg, const StepParams &P) {
    int a, b;
    if (BAT) split_range(nrg, P.nwg, blockIdx.x, a, b);
    else split_rows(nrg, P.nwg, blockIdx.x, a, b);
    return RgRange{a, b - a};
}

// Two ways to share a row group's tiles among the waves:
//   split-K   (long rows, KT >= 2 kWaves): wave w takes the k-tiles
//             [w KT / kWaves, (w + 1) KT / kWaves) of every row group; the
//             wave partial sums are added in wave order through LDS;
//   row-split (short rows): wave w takes whole row groups w, w + kWaves, ...
//             of the batch and needs no cross-wave sum.
// Both orders are fixed by the partition alone.
// The first ring of loads is issued before wait() and stage(0), overlapping
// their latency.
// The waves' sums are added in 64 bits.  (A long K range of several packed
// matrices, KTG > 0: each matrix's products are summed apart as well, so that
// the O projection over all heads rounds no more than its sums by head did.)
// KTG > 0: the K range spans several packed matrices of KTG k-tiles per row
// group each, gstride tiles apart (k-tile kt of row group r is tile
// (kt / KTG) gstride + r KTG + kt % KTG); 0: one matrix of KT.
template <bool RowSplit, int KTG, class Wait, class Stage, class Epi>
__device__ __forceinline__ void gemv_rows(const uint8_t *__restrict__ W, int KT, int first,
                                          int count, int B, const float *__restrict__ a,
                                          float *red, const uint8_t *dummy, Wait &&wait,
                                          Stage &&stage, Epi &&epi, int gstride = 0) {
    constexpr int U = kGemvDepth;
    constexpr int BATCH = RowSplit ? kWaves * kRgBatch : kRgBatch;   // row groups per LDS round
    // wave-uniform values live in scalar registers, so every branch below is
    // a scalar branch
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63;
    const int row = lane >> 3, sub = lane & 7;
    const int kt0 = RowSplit ? 0 : (wid * KT) / kWaves;
    const int nk = RowSplit ? KT : ((wid + 1) * KT) / kWaves - kt0;
    const int rstep = RowSplit ? kWaves : 1;   // a wave's next row group, in batch items
    const uint8_t *base = W + (size_t)lane * 16;
    const float *abase = a + sub * 8;
    u32x4 buf[U];
    int n = 0, ltile = 0, lk = 0, left = 0;   // batch items; next tile, its k index; tiles left

    // from a wave's last tile of one row group to its first of the next, and
    // (KTG) from the last tile of one packed matrix to the first of the next
    const int ktr = KTG ? KTG : KT;   // tiles between row groups
    const int kg0 = KTG ? kt0 / ktr : 0, kr0 = KTG ? kt0 % ktr : kt0;
    const int jump = KTG ? 0 : (rstep - 1) * KT + (KT - nk) + 1;
    int lrg = 0, kr = 0, kg = 0;
    // load the next tile of the batch, or the dummy line (branch-free)
    auto load_next = [&]() {
        const bool real = left > 0;
        if constexpr (KTG != 0) {
            const int t = __builtin_amdgcn_readfirstlane(kg * gstride + lrg * ktr + kr);
            const u32x4 v = ld_stream_16B(real ? base + (size_t)t * kTileBytes : dummy);
            const bool wrap = lk + 1 == nk, over = kr + 1 == ktr;
            lk = wrap ? 0 : lk + 1;
            lrg = wrap ? lrg + rstep : lrg;
            kg = wrap ? kg0 : (over ? kg + 1 : kg);
            kr = wrap ? kr0 : (over ? 0 : kr + 1);
            left = real ? left - 1 : left;
            return v;
        } else {
            const int t = __builtin_amdgcn_readfirstlane(ltile);
            const u32x4 v = ld_stream_16B(real ? base + (size_t)t * kTileBytes : dummy);
            const bool wrap = lk + 1 == nk;
            ltile = real ? ltile + (wrap ? jump : 1) : ltile;
            lk = real ? (wrap ? 0 : lk + 1) : lk;
            left = real ? left - 1 : left;
            return v;
        }
    };
    auto start = [&](int ib) {   // batch of row groups ib .. ib + BATCH - 1
        const int nb = min(BATCH, count - ib);
        const int mine = RowSplit ? (nb > wid ? (nb - wid + kWaves - 1) / kWaves : 0) : nb;
        n = nk * mine;
        left = n;
        lrg = first + ib + (RowSplit ? wid : 0);
        ltile = lrg * KT + kt0;
        lk = 0;
        kg = kg0;
        kr = kr0;
#pragma unroll
        for (int s = 0; s < U; ++s) buf[s] = load_next();
    };

    // the control wave takes part in the staging and the epilogue only
    const bool compute = wid < kWaves;
    const bool has_rows = count > 0;
    if (has_rows && compute) start(0);
    wait();
    if (!has_rows) return;
    for (int b = 0; b < B; ++b) {
        for (int ib = 0; ib < count; ib += BATCH) {
            if ((b > 0 || ib > 0) && compute) start(ib);
            if (ib == 0) stage(b);
            const int nrg = min(BATCH, count - ib);
            int cr = RowSplit ? wid : 0, ck = 0;   // batch item of the row group in progress
            float acc = 0.f, tot = 0.f;   // (KTG: of the packed matrix in progress, of those before)
            int cg = 0;
            // item i sits in slot i % U and is refilled with item i + U (or
            // the dummy line) right after it is consumed
            if (compute)
            for (int i0 = 0; i0 < n; i0 += U) {
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    if (i0 + s < n) {
                        const u32x4 wv = buf[s];
                        const float *ap = abase + (kt0 + ck) * kTileK;
                        const float4 a0 = *reinterpret_cast<const float4 *>(ap);
                        const float4 a1 = *reinterpret_cast<const float4 *>(ap + 4);
                        acc = fmaf(bf_lo(wv.x), a0.x, acc);
                        acc = fmaf(bf_hi(wv.x), a0.y, acc);
                        acc = fmaf(bf_lo(wv.y), a0.z, acc);
                        acc = fmaf(bf_hi(wv.y), a0.w, acc);
                        acc = fmaf(bf_lo(wv.z), a1.x, acc);
                        acc = fmaf(bf_hi(wv.z), a1.y, acc);
                        acc = fmaf(bf_lo(wv.w), a1.z, acc);
                        acc = fmaf(bf_hi(wv.w), a1.w, acc);
                        if (KTG && ++cg == KTG) {
                            tot += acc;
                            acc = 0.f;
                            cg = 0;
                        }
                        if (++ck == nk) {
                            const float t = sum8(tot + acc);
                            if (sub == 0) {
                                if (RowSplit) red[cr * kTileRows + row] = t;
                                else red[(wid * kRgBatch + cr) * kTileRows + row] = t;
                            }
                            acc = tot = 0.f;
                            ck = cg = 0;
                            cr += rstep;
                        }
                    }
                    buf[s] = load_next();
                }
            }
            lds_barrier();
            for (int t = kl_tid(); t < nrg * (kTileRows / 2); t += kThreads) {
                const int rgi = t / (kTileRows / 2), pr = (t % (kTileRows / 2)) * 2;
                double y0 = 0, y1 = 0;
                if (RowSplit) {
                    y0 = red[rgi * kTileRows + pr];
                    y1 = red[rgi * kTileRows + pr + 1];
                } else {
                    for (int w = 0; w < kWaves; ++w) {
                        if (((w + 1) * KT) / kWaves == (w * KT) / kWaves) continue;   // empty slice
                        y0 += red[(w * kRgBatch + rgi) * kTileRows + pr];
                        y1 += red[(w * kRgBatch + rgi) * kTileRows + pr + 1];
                    }
                }
                epi(b, (first + ib + rgi) * kTileRows + pr, y0, y1);
            }
            lds_barrier();
        }
    }
}

// Several sequences per pass (B <= kMultiSeq): every tile is applied to all
// B staged vectors (astride floats apart; their partial sums kRedStride
// floats apart in red), so the weights stream once for all of them.  The
// activation reads from LDS then bound the pass, so a wave takes its row
// groups kMultiRg at a time, interleaved tile by tile at each k (tiles
// (r, k), (r + 1, k), ..., (r, k + 1), ...): one read of the B vectors at k
// serves kMultiRg tiles.  A group short of kMultiRg real row groups is padded
// with spare loads of the dummy line, whose products are dropped.  Every row
// group's sums are taken in the same order as in gemv_rows, so the results
// are those of B passes of one sequence.  With U a multiple of kMultiRg, a
// group's tiles sit in consecutive ring slots, known at compile time in the
// unrolled loop.
constexpr int kMultiRg = 4;
template <bool RowSplit, int KTG, class Wait, class Stage, class Epi>
__device__ __forceinline__ void gemv_rows_multi(const uint8_t *__restrict__ W, int KT, int first,
                                                int count, int B, const float *__restrict__ a,
                                                int astride, float *red, const uint8_t *dummy,
                                                Wait &&wait, Stage &&stage, Epi &&epi,
                                                int gstride) {
    constexpr int U = kGemvDepth, NP = kMultiRg;
    static_assert(U % NP == 0, "a ring slot's place in its group must be fixed");
    constexpr int BATCH = RowSplit ? kWaves * kRgBatch : kRgBatch;
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63;
    const int row = lane >> 3, sub = lane & 7;
    const int kt0 = RowSplit ? 0 : (wid * KT) / kWaves;
    const int nk = RowSplit ? KT : ((wid + 1) * KT) / kWaves - kt0;
    // tiles between a wave's row groups, and (KTG) from one packed matrix's
    // last tile of a row group to the next one's first
    const int ktr = KTG ? KTG : KT, rsz = (RowSplit ? kWaves : 1) * ktr;
    const int kover = KTG ? gstride - ktr + 1 : 1;
    const uint8_t *base = W + (size_t)lane * 16;
    const float *abase = a + sub * 8;
    u32x4 buf[U];
    // loads: the wave's row groups gi .. gi + NP - 1 of the batch (mine of
    // them), at k index lk; tile0 = the first row group's first tile
    int n = 0, mine = 0, tile0 = 0, gi = 0, lk = 0, lt = 0, kr = 0;   // (lt: tiles from k index 0)
    auto load_h = [&](int h) {
        const bool real = gi + h < mine;
        const int t = __builtin_amdgcn_readfirstlane(tile0 + (gi + h) * rsz + lt);
        const u32x4 v = ld_stream_16B(real ? base + (size_t)t * kTileBytes : dummy);
        if (h == NP - 1) {
            const bool wrap = lk + 1 == nk, over = KTG && kr + 1 == ktr;
            lk = wrap ? 0 : lk + 1;
            lt = wrap ? 0 : lt + (over ? kover : 1);
            kr = wrap ? (KTG ? kt0 % ktr : 0) : (over ? 0 : kr + 1);
            gi = wrap ? gi + NP : gi;
        }
        return v;
    };
    auto start = [&](int ib) {
        const int nb = min(BATCH, count - ib);
        mine = RowSplit ? (nb > wid ? (nb - wid + kWaves - 1) / kWaves : 0) : nb;
        n = nk * NP * ((mine + NP - 1) / NP);
        tile0 = (first + ib + (RowSplit ? wid : 0)) * ktr +
                (KTG ? (kt0 / ktr) * gstride + kt0 % ktr : kt0);
        gi = lk = lt = 0;
        kr = KTG ? kt0 % ktr : 0;
#pragma unroll
        for (int s = 0; s < U; ++s) buf[s] = load_h(s % NP);
    };
    const bool compute = wid < kWaves;
    const bool has_rows = count > 0;
    if (has_rows && compute) start(0);
    wait();
    if (!has_rows) return;
    for (int ib = 0; ib < count; ib += BATCH) {
        if (ib > 0 && compute) start(ib);
        if (ib == 0)
            for (int bb = 0; bb < B; ++bb) stage(bb);
        const int nrg = min(BATCH, count - ib);
        int cr = 0, ck = 0;   // the group in progress (its first row group), its k index
        float acc[NP][kMultiSeq], tot[KTG ? NP : 1][KTG ? kMultiSeq : 1];
        int cg = 0;
#pragma unroll
        for (int h = 0; h < NP; ++h)
#pragma unroll
            for (int bb = 0; bb < kMultiSeq; ++bb) {
                acc[h][bb] = 0.f;
                if (KTG) tot[h][bb] = 0.f;
            }
        // a group's NP tiles sit in slots s .. s + NP - 1; they are consumed
        // together (each sequence's vector read once for all of them), then
        // refilled in order
        if (compute)
        for (int i0 = 0; i0 < n; i0 += U) {
#pragma unroll
            for (int s = 0; s < U; s += NP) {
                if (i0 + s < n) {
                    float wf[NP][8];
#pragma unroll
                    for (int h = 0; h < NP; ++h) {
                        const u32x4 wv = buf[s + h];
                        wf[h][0] = bf_lo(wv.x); wf[h][1] = bf_hi(wv.x);
                        wf[h][2] = bf_lo(wv.y); wf[h][3] = bf_hi(wv.y);
                        wf[h][4] = bf_lo(wv.z); wf[h][5] = bf_hi(wv.z);
                        wf[h][6] = bf_lo(wv.w); wf[h][7] = bf_hi(wv.w);
                    }
#pragma unroll
                    for (int bb = 0; bb < kMultiSeq; ++bb) {
                        if (bb < B) {
                            const float *ap = abase + bb * astride + (kt0 + ck) * kTileK;
                            const float4 a0 = *reinterpret_cast<const float4 *>(ap);
                            const float4 a1 = *reinterpret_cast<const float4 *>(ap + 4);
                            const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
                            for (int h = 0; h < NP; ++h) {
                                float v = acc[h][bb];
#pragma unroll
                                for (int e = 0; e < 8; ++e) v = fmaf(wf[h][e], av[e], v);
                                acc[h][bb] = v;
                            }
                        }
                    }
                    if (KTG && ++cg == KTG) {
#pragma unroll
                        for (int hh = 0; hh < NP; ++hh)
#pragma unroll
                            for (int bb = 0; bb < kMultiSeq; ++bb) {
                                tot[hh][bb] += acc[hh][bb];
                                acc[hh][bb] = 0.f;
                            }
                        cg = 0;
                    }
                    if (++ck == nk) {   // the group's row groups are done
#pragma unroll
                        for (int hh = 0; hh < NP; ++hh) {
                            const int c = cr + hh;   // the wave's c-th row group of the batch
                            const int ri = RowSplit ? (wid + c * kWaves) * kTileRows + row
                                                    : (wid * kRgBatch + c) * kTileRows + row;
#pragma unroll
                            for (int bb = 0; bb < kMultiSeq; ++bb) {
                                if (bb < B) {
                                    const float t = sum8(KTG ? tot[hh][bb] + acc[hh][bb] : acc[hh][bb]);
                                    if (c < mine && sub == 0) red[bb * kRedStride + ri] = t;
                                }
                                acc[hh][bb] = 0.f;
                                if (KTG) tot[hh][bb] = 0.f;
                            }
                        }
                        ck = cg = 0;
                        cr += NP;
                    }
                }
#pragma unroll
                for (int h = 0; h < NP; ++h) buf[s + h] = load_h(h);
            }
        }
        lds_barrier();
        for (int t = kl_tid(); t < B * nrg * (kTileRows / 2); t += kThreads) {
            const int bb = t / (nrg * (kTileRows / 2)), tt = t - bb * (nrg * (kTileRows / 2));
            const int rgi = tt / (kTileRows / 2), pr = (tt % (kTileRows / 2)) * 2;
            const float *rd = red + bb * kRedStride;
            double y0 = 0, y1 = 0;
            if (RowSplit) {
                y0 = rd[rgi * kTileRows + pr];
                y1 = rd[rgi * kTileRows + pr + 1];
            } else {
                for (int w = 0; w < kWaves; ++w) {
                    if (((w + 1) * KT) / kWaves == (w * KT) / kWaves) continue;   // empty slice
                    y0 += rd[(w * kRgBatch + rgi) * kTileRows + pr];
                    y1 += rd[(w * kRgBatch + rgi) * kTileRows + pr + 1];
                }
            }
            epi(bb, (first + ib + rgi) * kTileRows + pr, y0, y1);
        }
        lds_barrier();
    }
}

// The same on the matrix cores (P.multi = 2): row groups in pairs (16-row
// blocks), each tile pair re-laid out through a per-wave LDS slot as in the
// batched engine, one product per 32 columns for all sequences' three terms.
// Two accumulators (the halves of a tile) keep the sums short.  The vector-unit
// form is bound by its 8 multiplies per tile and sequence and the reads of the
// vectors; here the cost does not grow with the sequences.  8 layers of the 8B
// shape, batch 3 1067 -> 1043 us, batch 4 1195 -> 1162; the error against 64
// bits is 0.8 times the vector-unit form's.  (P.multi = 1 stays where three
// terms of the vectors do not fit in LDS, as at the 70B shape.)
template <bool RowSplit, int KTG, class Wait, class Stage, class Epi>
__device__ __forceinline__ void gemv_rows_mm(const uint8_t *__restrict__ W, int KT, int first,
                                             int count, int B, const uint16_t *X, int xs,
                                             uint8_t *slots, float *red, const uint8_t *dummy,
                                             Wait &&wait, Stage &&stage, Epi &&epi, int gstride) {
    constexpr int U = kGemvDepth, NP = 2;
    constexpr int BATCH = RowSplit ? kWaves * kRgBatch : kRgBatch;
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63;
    const int kt0 = RowSplit ? 0 : (wid * KT) / kWaves;
    const int nk = RowSplit ? KT : ((wid + 1) * KT) / kWaves - kt0;
    const int ktr = KTG ? KTG : KT, rsz = (RowSplit ? kWaves : 1) * ktr;
    const int kover = KTG ? gstride - ktr + 1 : 1;
    const uint8_t *base = W + (size_t)lane * 16;
    uint8_t *ws = slots + min(wid, kWaves - 1) * 2048;
    const uint16_t *xb = X + min(lane & 15, kMmCols - 1) * xs + 8 * (lane >> 4);
    u32x4 buf[U];
    int n = 0, mine = 0, tile0 = 0, gi = 0, lk = 0, lt = 0, kr = 0;
    auto load_h = [&](int h) {
        const bool real = gi + h < mine;
        const int t = __builtin_amdgcn_readfirstlane(tile0 + (gi + h) * rsz + lt);
        const u32x4 v = ld_stream_16B(real ? base + (size_t)t * kTileBytes : dummy);
        if (h == NP - 1) {
            const bool wrap = lk + 1 == nk, over = KTG && kr + 1 == ktr;
            lk = wrap ? 0 : lk + 1;
            lt = wrap ? 0 : lt + (over ? kover : 1);
            kr = wrap ? (KTG ? kt0 % ktr : 0) : (over ? 0 : kr + 1);
            gi = wrap ? gi + NP : gi;
        }
        return v;
    };
    auto start = [&](int ib) {
        const int nb = min(BATCH, count - ib);
        mine = RowSplit ? (nb > wid ? (nb - wid + kWaves - 1) / kWaves : 0) : nb;
        n = nk * NP * ((mine + NP - 1) / NP);
        tile0 = (first + ib + (RowSplit ? wid : 0)) * ktr +
                (KTG ? (kt0 / ktr) * gstride + kt0 % ktr : kt0);
        gi = lk = lt = 0;
        kr = KTG ? kt0 % ktr : 0;
#pragma unroll
        for (int s = 0; s < U; ++s) buf[s] = load_h(s % NP);
    };
    const bool compute = wid < kWaves;
    const bool has_rows = count > 0;
    if (has_rows && compute) start(0);
    wait();
    if (!has_rows) return;
    for (int ib = 0; ib < count; ib += BATCH) {
        if (ib > 0 && compute) start(ib);
        if (ib == 0)
            for (int bb = 0; bb < B; ++bb) stage(bb);
        const int nrg = min(BATCH, count - ib);
        int cr = 0, ck = 0, cg = 0;
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        f32x4 tot = {0.f, 0.f, 0.f, 0.f};
        if (compute)
        for (int i0 = 0; i0 < n; i0 += U) {
#pragma unroll
            for (int s = 0; s < U; s += NP) {
                if (i0 + s < n) {
                    const int wr = lane >> 3, wc = lane & 7;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        *reinterpret_cast<u32x4 *>(
                            ws + t * 1024 + (wr * 8 + (wc ^ ((wr + t) & 7))) * 16) = buf[s + t];
#pragma unroll
                    for (int st = 0; st < 2; ++st) {
                        const int r16 = lane & 15, ko = 4 * st + (lane >> 4);
                        const int at = r16 >> 3, ar = r16 & 7;
                        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
                            ws + at * 1024 + (ar * 8 + (ko ^ ((ar + at) & 7))) * 16);
                        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(
                            xb + (kt0 + ck) * kTileK + 32 * st);
                        acc[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x, acc[st], 0, 0, 0);
                    }
                    if (KTG && ++cg == KTG) {
                        tot += acc[0] + acc[1];
                        acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
                        cg = 0;
                    }
                    if (++ck == nk) {   // the pair's row groups are done
                        const f32x4 y = tot + (acc[0] + acc[1]);
                        const int b = lane & 15;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            // the terms: columns b, b + 4, b + 8
                            const float t = y[v] + (dpp<0x12C>(y[v]) + dpp<0x128>(y[v]));
                            const int r16 = 4 * (lane >> 4) + v, c = cr + (r16 >> 3);
                            const int ri = (RowSplit ? (wid + c * kWaves) * kTileRows
                                                     : (wid * kRgBatch + c) * kTileRows) + (r16 & 7);
                            if (b < B && c < mine) red[b * kRedStride + ri] = t;
                        }
                        acc[0] = acc[1] = tot = f32x4{0.f, 0.f, 0.f, 0.f};
                        ck = cg = 0;
                        cr += NP;
                    }
                }
#pragma unroll
                for (int h = 0; h < NP; ++h) buf[s + h] = load_h(h);
            }
        }
        lds_barrier();
        for (int t = kl_tid(); t < B * nrg * (kTileRows / 2); t += kThreads) {
            const int bb = t / (nrg * (kTileRows / 2)), tt = t - bb * (nrg * (kTileRows / 2));
            const int rgi = tt / (kTileRows / 2), pr = (tt % (kTileRows / 2)) * 2;
            const float *rd = red + bb * kRedStride;
            double y0 = 0, y1 = 0;
            if (RowSplit) {
                y0 = rd[rgi * kTileRows + pr];
                y1 = rd[rgi * kTileRows + pr + 1];
            } else {
                for (int w = 0; w < kWaves; ++w) {
                    if (((w + 1) * KT) / kWaves == (w * KT) / kWaves) continue;   // empty slice
                    y0 += rd[(w * kRgBatch + rgi) * kTileRows + pr];
                    y1 += rd[(w * kRgBatch + rgi) * kTileRows + pr + 1];
                }
            }
            epi(bb, (first + ib + rgi) * kTileRows + pr, y0, y1);
        }
        lds_barrier();
    }
}

// Row groups are shared split-K when they are long enough for every wave to
// hold two or more tiles, else row-split.  Multi: the B sequences share each
// pass (gemv_rows_multi).
template <bool Multi = false, int KTG = 0, class Wait, class Stage, class Epi>
__device__ __forceinline__ void gemv_phase(const uint8_t *__restrict__ W, int KT, int first,
                                           int count, int B, const float *__restrict__ a,
                                           float *red, const uint8_t *dummy, Wait &&wait,
                                           Stage &&stage, Epi &&epi, int astride = 0,
                                           int gstride = 0, uint8_t *mm_slots = nullptr) {
    if constexpr (Multi) {
        if (mm_slots) {
            const uint16_t *X = reinterpret_cast<const uint16_t *>(a);
            if (KT >= 2 * kWaves)
                gemv_rows_mm<false, KTG>(W, KT, first, count, B, X, mm_stride(astride), mm_slots, red,
                                         dummy, wait, stage, epi, gstride);
            else
                gemv_rows_mm<true, KTG>(W, KT, first, count, B, X, mm_stride(astride), mm_slots, red,
                                        dummy, wait, stage, epi, gstride);
            return;
        }
        if (KT >= 2 * kWaves)
            gemv_rows_multi<false, KTG>(W, KT, first, count, B, a, astride, red, dummy, wait, stage,
                                        epi, gstride);
        else
            gemv_rows_multi<true, KTG>(W, KT, first, count, B, a, astride, red, dummy, wait, stage,
                                       epi, gstride);
    } else if (KT >= 2 * kWaves) {
        gemv_rows<false, KTG>(W, KT, first, count, B, a, red, dummy, wait, stage, epi, gstride);
    } else {
        gemv_rows<true, KTG>(W, KT, first, count, B, a, red, dummy, wait, stage, epi, gstride);
    }
}

// ---------------------------------------------------------------- batched engine
//
// Y[r][b] = sum_k W[r][k] X[b][k] on the matrix cores (v_mfma_f32_16x16x32_bf16:
// D[16x16] += A[16x32] B[32x16]) for the row groups first .. first + count - 1
// and up to kGemmBatch sequences b0 .. b0 + nb - 1.  A block is 16 weight
// rows (2 row groups); A = W[16 rows][32 k], B = X[32 k][16 sequences], two
// products per 32 columns cover 32 sequences, each product taken for both
// bf16 terms of X (hi, then lo, into the same accumulators).  Operand layouts:
// A lane l holds A[l % 16][8 (l / 16) .. +7], B lane l holds
// B[8 (l / 16) .. +7][l % 16], D lane l holds D[4 (l / 16) + v][l % 16].
// Weight tiles arrive through the same kind of ring of 16-byte loads as the
// GEMV path and are re-laid out through a per-wave LDS slot (2 KiB: the two
// tiles of a block at one k-tile; the slots follow the two activation chunk
// buffers).  X is staged in LDS in chunks of kGemmChunkK columns (kActStride
// bf16 per row; the hi rows, then kLoOff elements further the lo rows), in
// two chunk buffers: stage(c, buf) fills chunk c.

constexpr int kLoOff = kGemmBatch * kActStride;   // elements from a chunk's hi rows to its lo rows

struct GemmLds {
    uint16_t *act[2];   // [2 terms][kGemmBatch][kActStride] bf16
};

__device__ __forceinline__ GemmLds gemm_lds(char *smem) {
    GemmLds g;
    g.act[0] = reinterpret_cast<uint16_t *>(smem);
    g.act[1] = reinterpret_cast<uint16_t *>(smem + 2 * kGemmActBytes);
    return g;
}

//
// A workgroup's products cover the row groups first .. first + count - 1 and
// the K range of W (KT k-tiles).  The K range may span several packed
// matrices of ktg k-tiles each, gstride tiles apart: k-tile kt of row group
// r is tile (kt / ktg) gstride + r ktg + kt % ktg.
//
// Work split: wave w owns the 16-row blocks w, w + kWaves, ... and takes
// them in groups of up to kGemmMaxBlk; for each group it runs through the
// chunks of K, and within a chunk through its blocks, one ring pass (U = 16
// tile loads: the 8 k-tiles of the chunk x the block's 2 row groups) per
// block.  Slot s of a pass is always (k-tile s / 2, row group s % 2), so
// that the consuming code is the same straight-line code for every pass; the
// loads run ahead through the same sequence across blocks, chunks and
// groups, and every slot is refilled unconditionally (with the zero tile
// once the wave's work is exhausted, or for a row group or k-tile past the
// range), so the compiler keeps the whole ring in flight.
//
// Activations: with up to two chunks (1024 columns) the whole K range is
// staged once and stays resident, and the waves then run without any
// workgroup barrier; longer K ranges stream through the two chunk buffers
// (the control wave copies chunk f + 1 while the compute waves work on chunk
// f; one barrier per chunk, every wave taking part in every chunk's
// barrier).  stage(c, buf) fills chunk c with the control wave's
// memory-to-LDS copies (a no-op in the other waves).
//
// Each block's products go straight from the accumulators to epi(b, r,
// y_r, y_r+1), for its row pairs and sequences b < nb.
//
// pre() runs once, after the first ring of weight loads is issued (so the
// weight stream overlaps whatever pre() waits for), before anything touches
// the activation buffers; it runs even when there are no rows.
//
// Memory-to-LDS copies issued inside the compute loop would make the
// compiler wait for all outstanding loads before each of the loop's LDS
// accesses (draining the ring once per pass), so the two modes are separate
// instances and the streaming copies run in a loop of the control wave's own.
// ready(c) (control wave) waits until chunk c's inputs are complete;
// all_ready() (control wave) runs once all of them are, before the first
// products reach epi.
template <bool resident, class Pre, class Ready, class AllReady, class Stage, class Epi>
__device__ __forceinline__ void gemm_rows_mode(const uint8_t *__restrict__ W, int KT, int first,
                                               int count, int ktg, size_t gstride, int b0,
                                               int nb, const uint8_t *dummy, const GemmLds &L,
                                               Pre &&pre, Ready &&ready, AllReady &&all_ready,
                                               Stage &&stage, Epi &&epi) {
    constexpr int U = kGemmDepth;
    constexpr int CT = kGemmChunkK / kTileK;   // k-tiles per chunk
    constexpr int MB = kGemmMaxBlk;
    static_assert(U == 2 * CT, "a ring pass is one chunk of one 16-row block");
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63;
    const bool compute = wid < kWaves;
    const int nkc = resident ? min((KT + CT - 1) / CT, 2) : (KT + CT - 1) / CT;
    const int nblk = (count + 1) / 2;
    const int mine = (compute && nblk > wid) ? (nblk - wid + kWaves - 1) / kWaves : 0;
    const int ngrp = (mine + MB - 1) / MB;
    const int ngrp_wg = ((nblk + kWaves - 1) / kWaves + MB - 1) / MB;   // wave 0's
    const int last_rg = first + count;
    // (LDS addresses are formed from the shared array itself: a pointer taken
    // out of GemmLds by a run-time index is a generic pointer, and generic
    // loads would make every wait for an operand a wait for the whole ring)
    uint8_t *ws = reinterpret_cast<uint8_t *>(kl_smem + 4 * kGemmActBytes + wid * 2048);
    const int lo16 = lane * 16;

    // load generator: group gi, chunk gc, block gb of the group, slot gs;
    // (kg, kr) = (k-tile / ktg, k-tile % ktg) of the next load, and (kg0,
    // kr0) of the current chunk's first k-tile (wave-uniform scalars,
    // advanced by selects)
    int gi = 0, gc = 0, gb = 0, gs = 0, kg = 0, kr = 0, kg0 = 0, kr0 = 0;
    auto load_next = [&]() {
        const int blk = wid + kWaves * (MB * gi + gb);
        const int rg = first + 2 * blk + (gs & 1);
        const int kt = gc * CT + (gs >> 1);
        const bool inb = gi < ngrp && rg < last_rg && kt < KT;
        const size_t tile = (size_t)kg * gstride + (size_t)rg * ktg + kr;
        const uint8_t *src = inb ? W + tile * kTileBytes : dummy;
        const u32x4 v = ld_stream_16B(src + lo16);
        int nkr = kr + (gs & 1), nkg = kg;
        nkg = nkr == ktg ? nkg + 1 : nkg;
        nkr = nkr == ktg ? 0 : nkr;
        const bool pass_end = gs == U - 1;
        const bool blk_next = pass_end && gb + 1 < min(MB, mine - MB * gi);
        const bool chunk_end = pass_end && !blk_next;
        const bool grp_end = chunk_end && gc + 1 >= nkc;
        gs = pass_end ? 0 : gs + 1;
        gb = blk_next ? gb + 1 : (chunk_end ? 0 : gb);
        gc = grp_end ? 0 : (chunk_end ? gc + 1 : gc);
        gi = grp_end ? gi + 1 : gi;
        kg = grp_end ? 0 : (blk_next ? kg0 : nkg);
        kr = grp_end ? 0 : (blk_next ? kr0 : nkr);
        kg0 = grp_end ? 0 : (chunk_end ? nkg : kg0);
        kr0 = grp_end ? 0 : (chunk_end ? nkr : kr0);
        return v;
    };

    // (padding sequences: their rows of the activation buffers hold copies of
    // finite values; a product's columns are independent, and the outputs of
    // padding sequences are never stored)
    u32x4 buf[U];
    if (compute) {   // (the control wave keeps its load queue empty)
#pragma unroll
        for (int s = 0; s < U; ++s) buf[s] = load_next();
    }
    pre();
    if (count <= 0) return;
    // The first chunk (resident: both) is copied by all nine waves, whose
    // rings are full by now: copied by the control wave alone it took three
    // round trips, as one wave has at most 63 memory operations in flight.
    if (!compute) {
        ready(0);
        if (resident && nkc > 1) ready(1);
    }
    __syncthreads();   // (the buffers may still hold the previous sequence group)
    stage(0, L.act[0], true);
    if (resident && nkc > 1) stage(1, L.act[1], true);
    if (resident && !compute) all_ready();
    ctl_copy_wait();
    __syncthreads();

    if constexpr (!resident) {
        if (!compute) {
            // chunk f + 1 into buffer (f + 1) % 2 while the compute waves work on chunk f
            const int total = ngrp_wg * nkc;
            for (int f = 0; f < total; ++f) {
                if (f + 1 < total) {
                    if (f + 1 < nkc) ready(f + 1);
                    stage((f + 1) % nkc, L.act[(f + 1) & 1], false);
                    ctl_copy_wait();
                }
                if (f == nkc - 1) all_ready();
                __syncthreads();
            }
            return;
        }
    }
    f32x4 acc[MB][2];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ngl = resident ? ngrp : ngrp_wg;
    int f = 0;   // chunks consumed (streaming: chunk f sits in buffer f % 2)
    for (int g = 0; g < ngl; ++g) {
        const int nbg = min(MB, mine - MB * g);
        for (int c = 0; c < nkc; ++c, ++f) {
            const uint16_t *act = reinterpret_cast<const uint16_t *>(
                kl_smem + ((resident ? c : f) & 1) * (2 * kGemmActBytes));
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                if (i >= nbg) continue;   // (uniform)
#pragma unroll
                for (int s = 0; s < U; ++s) {
                    // tile (s % 2) of the block -> the wave's slot; the 16-byte
                    // column c of row r of tile t sits at column c ^ ((r + t) & 7),
                    // so that both these writes and the operand reads below (16
                    // rows at a time) are free of LDS bank conflicts
                    {
                        const int wr = lane >> 3, wc = lane & 7, tt = s & 1;
                        *reinterpret_cast<u32x4 *>(
                            ws + tt * 1024 + (wr * 8 + (wc ^ ((wr + tt) & 7))) * 16) = buf[s];
                    }
                    if (s & 1) {
                        const int ktl = s >> 1;
#pragma unroll
                        for (int st = 0; st < 2; ++st) {
                            const int r16 = lane & 15, ko = 4 * st + (lane >> 4);
                            const int at = r16 >> 3, ar = r16 & 7;
                            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
                                ws + at * 1024 + (ar * 8 + (ko ^ ((ar + at) & 7))) * 16);
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const int b = h * 16 + (lane & 15);
                                const int k = ktl * kTileK + 32 * st + 8 * (lane >> 4);
                                const bf16x8 x = *reinterpret_cast<const bf16x8 *>(
                                    act + b * kActStride + k);
                                const bf16x8 xl = *reinterpret_cast<const bf16x8 *>(
                                    act + kLoOff + b * kActStride + k);
                                acc[i][h] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x, acc[i][h], 0, 0, 0);
                                acc[i][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, xl, acc[i][h],
                                                                                   0, 0, 0);
                            }
                        }
                    }
                    buf[s] = load_next();
                }
            }
            // chunk f consumed by every wave; f + 1 staged (by the control wave,
            // which waits for its copies; the ring stays in flight)
            if (!resident) lds_barrier();
        }
        // the group's products: lane l holds rows 4 (l / 16) .. + 3 of the
        // block for sequence h 16 + l % 16
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            if (i >= nbg) continue;   // (uniform)
            const int blk = wid + kWaves * (MB * g + i);
            const int r4 = 4 * (lane >> 4);
            const bool rv = first + 2 * blk + (r4 >> 3) < last_rg;
            const int r = (first + 2 * blk) * kTileRows + r4;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int b = h * 16 + (lane & 15);
                if (rv && b < nb) {
                    epi(b0 + b, r, acc[i][h][0], acc[i][h][1]);
                    epi(b0 + b, r + 2, acc[i][h][2], acc[i][h][3]);
                }
                acc[i][h] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
}

template <class Pre, class Ready, class AllReady, class Stage, class Epi>
__device__ __forceinline__ void gemm_rows(const uint8_t *__restrict__ W, int KT, int first,
                                          int count, int ktg, size_t gstride, int b0, int nb,
                                          const uint8_t *dummy, const GemmLds &L, Pre &&pre,
                                          Ready &&ready, AllReady &&all_ready, Stage &&stage,
                                          Epi &&epi) {
    if (KT <= 2 * (kGemmChunkK / kTileK))
        gemm_rows_mode<true>(W, KT, first, count, ktg, gstride, b0, nb, dummy, L, pre, ready,
                             all_ready, stage, epi);
    else
        gemm_rows_mode<false>(W, KT, first, count, ktg, gstride, b0, nb, dummy, L, pre, ready,
                              all_ready, stage, epi);
}


// ---------------------------------------------------------------- phases
//
// Synchronization between the phases of a layer (l):
//   per-sequence path   tagged words throughout: q, k, v -> attention; the
//                  attention's parts -> merge -> O projection; residual
//                  (owners) -> gate/up; SwiGLU -> down; down's partial sums ->
//                  owners -> residual -> next layer.  A writer of layer l + 1
//                  has transitively waited for every reader of layer l's words,
//                  because a workgroup reads words only in phases in which it
//                  has rows.
//   matrix-core path:
//   grid barrier   after embed, the q/k/v product, attn, oproj, gateup and
//                  down (and the SwiGLU fold, with several gate/up K slices).
//   cnt_qkv[g]     qkv -> attn: KV head g's workgroups fold exactly the q/k/v
//                  rows of that head, so the attention of head g waits only
//                  for them (Sg arrivals per layer).
//   norm_cnt[c]    RMSNorm slices -> products (norm_batched).
// Local counters grow monotonically within a step (zeroed by the embedding
// phase); their targets are (l + 1) times the arrivals per layer.
// Every workgroup arrives on, and waits on, every grid barrier.

// ---------------------------------------------------------------- batched phases
//
// A weight phase runs the GEMV engine on the per-sequence path and the
// matrix-core engine otherwise (sequences in groups of kGemmBatch; the
// weights stream once per group).  In the batched path every input is staged
// as bf16 chunks: prep() runs once after wait(), both once the first weight
// loads are in flight; ready(c) (control wave) waits for chunk c's inputs;
// stageb(c, b0, nb, buf, all) fills chunk c for sequences b0 .. b0 + nb - 1
// (memory-to-LDS copies, by all waves or by the control wave).
// (done(b0, nb) runs in every thread after the matrix-core path's group of
// sequences b0 .. b0 + nb - 1)
struct NoGroupDone {
    __device__ void operator()(int, int) const {}
};
// Per-sequence path: with P.multi, the sequences' vectors sit astride floats
// apart and share each pass (stage1(b) is called for every b before the
// pass; stage1(0) may stage them all).
struct NoReady {   // weight_phase whose inputs are complete after prep()
    __device__ void operator()(int) const {}
};
struct NoAllReady {
    __device__ void operator()(int, int) const {}
};
template <bool BAT, class Wait, class Prep, class Stage1, class StageB, class Epi,
          class Done = NoGroupDone, class Ready = NoReady, class AllReady = NoAllReady>
__device__ __forceinline__ void weight_phase(const StepParams &P, const Lds &S,
                                             const uint8_t *W, int KT, int first, int count,
                                             Wait &&wait, Prep &&prep, Stage1 &&stage1,
                                             StageB &&stageb, Epi &&epi, int ktg = 0,
                                             size_t gstride = 0, Done done = Done(),
                                             int astride = 0, Ready ready = Ready(),
                                             AllReady all_ready = AllReady()) {
    if constexpr (!BAT) {
        if (P.multi)
            gemv_phase<true>(W, KT, first, count, P.B, S.a, S.red, P.dummy, wait, stage1, epi,
                             astride, 0, mm_slots(P, S));
        else
            gemv_phase(W, KT, first, count, P.B, S.a, S.red, P.dummy, wait, stage1, epi);
        return;
    }
    const GemmLds L = gemm_lds(kl_smem);
    for (int b0 = 0; b0 < P.B; b0 += kGemmBatch) {
        const int nb = min(kGemmBatch, P.B - b0);
        gemm_rows(W, KT, first, count, ktg ? ktg : KT, gstride, b0, nb, P.dummy, L,
                  [&]() {   // (first group only: the inputs' wait and the grid-wide prologue)
                      if (b0 == 0) {
                          wait();
                          prep();
                      }
                  },
                  [&](int c) { if (b0 == 0) ready(c); }, [&]() { all_ready(b0, nb); },
                  [&](int c, uint16_t *buf, bool all) { stageb(c, b0, nb, buf, all); }, epi);
        done(b0, nb);
    }
}

// Batched RMSNorm (Sec. 2), deferred scale.  The K-slice partial sums of
// the last O or down projection (nparts of them) are first folded into the
// residual, x = x_in + sum_s fix(part_s) (exact integer adds, so the order is
// immaterial), and x is written to x_out; act / act_lo = the two bf16 terms
// of x gain, and the row's sum of squares goes to P.ssp per kGemmChunkK
// columns.  The consumers apply r = 1 / rms(x) to the products (rms_r).
// Items (sequence, kGemmChunkK-column slice) are spread over the grid, one
// column per thread.  Each item arrives on its slice's counter (norm_cnt,
// B arrivals per slice per RMSNorm step); a product waits only for the
// slices it stages (norm_wait) instead of on a grid barrier.  The counters
// sit kNormCntStride words apart: on one shared line, the polls of every
// control wave and the items' atomics contend (measured slower than the
// grid barrier).
__device__ __forceinline__ unsigned *norm_cnt(const StepParams &P) {
    return P.cnt + P.nkv;
}
__device__ __forceinline__ void norm_batched(const StepParams &P, const Lds &S,
                                             const float *gain, const long long *xin,
                                             long long *xout, int nparts) {
    static_assert(kGemmChunkK <= kThreads, "one column per thread");
    const int ns = (P.Hp + kGemmChunkK - 1) / kGemmChunkK;
    const int plast = max(nparts - 1, 0);
    for (int it = blockIdx.x; it < P.B * ns; it += P.nwg) {
        const int b = it / ns, sl = it % ns;
        const int i = sl * kGemmChunkK + (int)kl_tid();
        const bool live = (int)kl_tid() < kGemmChunkK && i < P.Hp;
        const int ic = min(i, P.Hp - 1);
        // (unconditional loads from in-range addresses, masked when used)
        long long x = (long long)ld_dev_u64(xin + (size_t)b * P.Hp + ic);
        const float *pr = P.xpart + (size_t)b * P.Hp + ic;
        float pv[kMaxKSlices];
#pragma unroll
        for (int q = 0; q < kMaxKSlices; ++q)
            pv[q] = ld_dev(pr + (size_t)min(q, plast) * P.xpart_stride);
#pragma unroll
        for (int q = 0; q < kMaxKSlices; ++q)
            if (q < nparts) x += to_fix(pv[q]);
        float ss = 0.f;
        if (live) {
            const float xv = from_fix(x);
            ss = xv * xv;   // (padding columns hold zero)
            if (nparts > 0)
                st_dev_u64(reinterpret_cast<unsigned long long *>(xout + (size_t)b * P.Hp + i),
                           (unsigned long long)x);
            uint16_t hi, lo;
            split_bf16(xv * gain[i], hi, lo);
            st_dev_u16(P.act + (size_t)b * P.Hp + i, hi);
            st_dev_u16(P.act_lo + (size_t)b * P.Hp + i, lo);
        }
        ss = block_sum(ss, S.sm);
        if (kl_tid() == 0) st_dev(P.ssp + (size_t)b * ns + sl, ss);
        drain_all();   // (also: S.sm is reused by the next item)
        if (is_ctl_lane0())
            __hip_atomic_fetch_add(norm_cnt(P) + kNormCntStride * sl, 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The control wave waits until the slices R of RMSNorm step inst (numbered
// within the step: 2 l for layer l's attention norm, 2 l + 1 for its FFN norm,
// 2 L for the final norm) are complete.  No workgroup barrier:
// the control wave then copies those slices (the other waves meet it at the
// barrier after the copies).
__device__ __forceinline__ void norm_wait(const StepParams &P, int inst, SliceRange R) {
    if (is_ctl_lane0()) {
        const unsigned target = (unsigned)(inst + 1) * (unsigned)P.B;
        for (int c = R.first; c < R.end; ++c)
            spin_until(P, [&]() {
                return (int)(__hip_atomic_load(norm_cnt(P) + kNormCntStride * c, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) - target) >= 0;
            });
    }
}

// (the steps that apply the scales keep those of sequences below
// kRScaleTable in LDS, in the area of the GEMV partial sums, which the
// batched path does not use)
constexpr int kRScaleTable = kWaves * kRgBatch * kTileRows;

// 1 / rms of sequence b's row normalised by the last batched RMSNorm step
// (its column-slice sums of squares, added in slice order).
__device__ __forceinline__ float rms_r(const StepParams &P, int b) {
    const int ns = (P.Hp + kGemmChunkK - 1) / kGemmChunkK;
    float ss = 0.f;
    for (int s0 = 0; s0 < ns; s0 += 16) {
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = ld_dev(P.ssp + (size_t)b * ns + min(s0 + j, ns - 1));
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (s0 + j < ns) ss += v[j];
    }
    return 1.0f / sqrtf(ss / (float)P.H + P.eps);
}

// The scales rms_r of sequences below kRScaleTable, in LDS (S.red), for
// the steps that fold a batched product's partials; ends with a workgroup
// barrier.
__device__ __forceinline__ void rms_table(const StepParams &P, const Lds &S) {
    for (int t = kl_tid(); t < min(P.B, kRScaleTable); t += kThreads) S.red[t] = rms_r(P, t);
    __syncthreads();
}
__device__ __forceinline__ float rms_of(const StepParams &P, const Lds &S, int b) {
    return b < kRScaleTable ? S.red[b] : rms_r(P, b);
}

// Chunk c of the normalised activations (control wave: memory-to-LDS copies).
//
// Rows k0 .. k0 + kc - 1 (kc <= kGemmChunkK: one 16-byte copy per lane and row)
// of both terms of sequences b0 .. b0 + nb - 1 of a two-term bf16 matrix with
// row stride ld.  The copies are straight-line code without branches: a
// branch or loop between two copies makes the compiler wait for the first
// before issuing the second (it cannot tell that their LDS ranges are
// disjoint).  Lanes past kc copy a clamped in-row address, and padding rows (b
// >= nb) are left as they are (or receive a copy of row nb - 1): the
// matrix-core loop's columns are independent, outputs of padding sequences
// are discarded, and columns past kc are never consumed.
//
// NR rows first, first + step, ...
template <int NR>
__device__ __forceinline__ void copy_rows(const uint16_t *hi, const uint16_t *lo, int ld, int k0,
                                          int kc, int b0, int nb, uint16_t *buf, int first,
                                          int step) {
    const int lane = kl_tid() & 63;
    const uint64_t col = (uint64_t)(k0 + min(lane * 8, kc - 8));
    // (the row offset is opaque to the compiler at each step, so that the
    // addresses are formed right before their copies instead of all at once)
    uint64_t row = (uint64_t)(b0 + first) * ld;
    const uint64_t last = (uint64_t)(b0 + nb - 1) * ld;
    uint16_t *d = buf + first * kActStride;
#pragma unroll
    for (int b = 0; b < NR; ++b) {
        const uint64_t o = min(row, last) + col;
        __builtin_amdgcn_global_load_lds(hi + o, d + b * step * kActStride, 16, 0, kLdsCoherent);
        __builtin_amdgcn_global_load_lds(lo + o, d + kLoOff + b * step * kActStride, 16, 0,
                                         kLdsCoherent);
        row += (uint64_t)step * ld;
        asm volatile("" : "+v"(row));
    }
}
// All waves (wave w the rows w, w + kWaves + 1, ...) or the control wave; the
// caller waits for the copies.
__device__ __forceinline__ void copy_chunk(const uint16_t *hi, const uint16_t *lo, int ld, int k0,
                                           int kc, int b0, int nb, uint16_t *buf, bool all) {
    constexpr int NW = kWaves + 1;
    static_assert(kGemmBatch <= 4 * NW, "rows per wave");
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    if (all) {
        const int n = nb > wid ? (nb - wid + NW - 1) / NW : 0;
        if (n == 1) copy_rows<1>(hi, lo, ld, k0, kc, b0, nb, buf, wid, NW);
        else if (n == 2) copy_rows<2>(hi, lo, ld, k0, kc, b0, nb, buf, wid, NW);
        else if (n == 3) copy_rows<3>(hi, lo, ld, k0, kc, b0, nb, buf, wid, NW);
        else if (n == 4) copy_rows<4>(hi, lo, ld, k0, kc, b0, nb, buf, wid, NW);
    } else if (wid == kCtlWave) {
        if (nb <= 8) copy_rows<8>(hi, lo, ld, k0, kc, b0, nb, buf, 0, 1);
        else if (nb <= 16) copy_rows<16>(hi, lo, ld, k0, kc, b0, nb, buf, 0, 1);
        else copy_rows<kGemmBatch>(hi, lo, ld, k0, kc, b0, nb, buf, 0, 1);
    }
}

__device__ __forceinline__ void stage_act_chunk(const StepParams &P, int c, int b0, int nb,
                                                uint16_t *buf, bool all) {
    const int k0 = c * kGemmChunkK;
    copy_chunk(P.act, P.act_lo, P.Hp, k0, min(kGemmChunkK, P.Hp - k0), b0, nb, buf, all);
}

// Chunk c of a two-term bf16 matrix src / src_lo [b][ld] with K columns
// (control wave: memory-to-LDS copies, so the compute waves keep working on
// the previous chunk).
__device__ __forceinline__ void stage_bf16_chunk(const uint16_t *src, const uint16_t *src_lo,
                                                 int ld, int K, int c, int b0, int nb,
                                                 uint16_t *buf, bool all) {
    const int k0 = c * kGemmChunkK;
    copy_chunk(src, src_lo, ld, k0, min(kGemmChunkK, K - k0), b0, nb, buf, all);
}

// Per-sequence path: the residual has one owner per row, the workgroup that
// has the row's O projection (own_rows), which keeps it in LDS (own_x; a copy
// in memory for later launches) and publishes each new value as the float
// that the next RMSNorm reads, as tagged words.  The down projection's
// partial sums come to the owner as tagged words too, one per FFN column
// block (and expert slot), each rounded to the fixed-point grid and added:
// the same exact sum as by atomics, without their traffic (one 8-byte
// read-modify-write per partial at memory) and without the drain and the
// grid barrier that a sum by many writers needs before it can be read.
__device__ __forceinline__ OwnRows own_rows(const StepParams &P) {
    int a, b;
    split_range(P.o_rg, P.nwg, blockIdx.x, a, b);
    return OwnRows{a * kTileRows, (b - a) * kTileRows};
}
// row r of this workgroup's (sequence b) := x, published in 'words' with 'tag'
__device__ __forceinline__ void put_x(const StepParams &P, int b, int r, const OwnRows &R,
                                      long long x, unsigned long long *words, unsigned tag) {
    const size_t i = (size_t)b * P.Hp + R.first + r;
    own_x(P)[b * P.own_max + r] = x;
    st_ll_f(words + i, from_fix(x), tag);
    st_dev_u64(reinterpret_cast<unsigned long long *>(P.xf + i), (unsigned long long)x);
}
// Control wave, after layer l's down projection: the owned rows' partial sums
// (nj per row and sequence), the new residual.
__device__ __forceinline__ void gather_down(const StepParams &P, int l, int nj) {
    const OwnRows R = own_rows(P);
    const int n = nj * R.count, lane = kl_tid() & 63;
    if (n == 0) return;
    // (a sequence at a time, in rounds of as many loads as the 8B shape needs:
    // larger rounds, or all sequences in one, measured no faster)
    for (int b = 0; b < P.B; ++b) {
        const unsigned long long *src = P.dp_ll + (size_t)b * nj * P.Hp + R.first;
        unsigned long long *own = reinterpret_cast<unsigned long long *>(own_x(P) + b * P.own_max);
        ll_gather<8>(
            P, n, ll_tag(P, l), lane, 64,
            [&](int i) { return src + (size_t)(i / R.count) * P.Hp + i % R.count; },
            [&](int i, unsigned v) {
                __hip_atomic_fetch_add(own + i % R.count,
                                       (unsigned long long)to_fix(__uint_as_float(v)),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            });
    }
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < P.B * R.count; i += 64) {
        const int b = i / R.count, r = i % R.count;
        put_x(P, b, r, R, own_x(P)[b * P.own_max + r], P.xb_ll, ll_tag(P, l + 1));
    }
}

// Before the threads poll for the residual after a down projection: this
// workgroup's own rows have arrived at their owner (the control wave comes
// here from gather_down), so the others' are about to.  Without it every
// workgroup that is early polls the whole residual over and over, 8 MB a round
// across the chip, and the words the others wait for queue behind that.
__device__ __forceinline__ void owners_wait(const StepParams &P, int ti) {
    lds_barrier();
    if (is_ctl_lane0()) trace_stamp(P, ti, 1);
}

// Embedding block (Sec. 2): x = E[token] (exact in fixed point).  Workgroup 0
// records bad token ids and positions, and zeroes the local counters.
__device__ __forceinline__ void phase_embed(KArg ka, int gwait, int garrive, int ti) {
    const StepParams P = load_params(ka);
    if (gwait >= 0) bar_wait(P, gwait, ti);
    if (blockIdx.x == 0) {
        for (int b = kl_tid(); b < P.B; b += kThreads) {
            const int t = raw_tok(P, b), p = raw_pos(P, b);
            int bits = 0;
            if (t < 0 || t >= P.V) bits |= KL_DEVERR_TOKEN;
            if (p < 0 || p >= P.cap || p >= P.max_seq) bits |= KL_DEVERR_POSITION;
            if (bits) atomicOr(P.err, bits);
            // token loop: record the token taken, clear the next step's argmax
            // (this step's is in use as soon as some workgroup's head is done,
            // which nothing here precedes)
            if (P.tok_emit) P.tok_emit[b] = t;
            if (P.amax) st_dev_u64(P.amax_next + b, 0ull);
        }
        const int nc = P.nkv + kNormCntStride * ((P.Hp + kGemmChunkK - 1) / kGemmChunkK);
        if (P.batched)   // (the local counters are used by batched steps only)
            for (int i = kl_tid(); i < nc; i += kThreads)
                __hip_atomic_store(P.cnt + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!P.batched) {   // every workgroup its own residual rows, published as layer 0's input
        const OwnRows R = own_rows(P);
        for (int i = kl_tid(); i < P.B * R.count; i += kThreads) {
            const int b = i / R.count, r = i % R.count;
            put_x(P, b, r, R, to_fix(bf2f(P.embed[(size_t)eff_tok(P, b) * P.H + R.first + r])),
                  P.xb_ll, ll_tag(P, 0));
        }
        lds_barrier();
        if (is_ctl_lane0()) trace_stamp(P, ti, 0);
        return;
    }
    const int total = P.B * P.Hp;
    for (int idx = blockIdx.x * kThreads + kl_tid(); idx < total; idx += P.nwg * kThreads) {
        const int b = idx / P.Hp, i = idx % P.Hp;
        const float e = (i < P.H) ? bf2f(P.embed[(size_t)eff_tok(P, b) * P.H + i]) : 0.f;
        st_dev_u64(reinterpret_cast<unsigned long long *>(P.xf + idx),
                   (unsigned long long)to_fix(e));
    }
    if (garrive >= 0) bar_arrive(P, garrive, ti);
}

// One rotation pair (rows lr, lr + 1 of KV head g's block, lr even) of the
// q/k/v projection of sequence b: RoPE (Sec. 2) on query and key rows with
// cs = (cos, sin) of the pair's angle at the sequence's position, then the
// key and value to the KV cache at that position, and the query (and the new
// key and value, for the attention) to the attention's inputs: tagged words
// (LL, the per-sequence path, tag 'tag') or plain device-coherent stores.
template <bool LL, class Rope>
__device__ __forceinline__ void qkv_store(const StepParams &P, int l, int b, int g, int lr,
                                          float y0, float y1, Rope &&rope, unsigned tag = 0) {
    const int d = P.d, half = P.d / 2, G = P.group;
    const int p = pos_of<LL>(P, b);
    const bool ok = ok_of<LL>(P, b);
    unsigned long long *kvl = LL ? P.kv_ll + ((size_t)b * P.nkv + g) * d : nullptr;
    if (lr < (G + 1) * d) {
        const int i = (lr % d) >> 1;
        const float2 cs = rope(p, i);
        const float u0 = y0 * cs.x - y1 * cs.y;
        const float u1 = y0 * cs.y + y1 * cs.x;
        if (lr < G * d) {
            const size_t qo = (size_t)b * P.nq * d + (size_t)(g * G + lr / d) * d;
            if (LL) {
                st_ll_f(P.q_ll + qo + i, u0, tag);
                st_ll_f(P.q_ll + qo + i + half, u1, tag);
            } else {
                st_dev(P.q + qo + i, u0);
                st_dev(P.q + qo + i + half, u1);
            }
        } else {
            const uint16_t k0 = f2bf(u0), k1 = f2bf(u1);
            if (ok) {
                uint16_t *kk = P.kc + (kv_row(P, l, b, g) + p) * d;
                st_dev_u16(kk + i, k0);
                st_dev_u16(kk + i + half, k1);
            }
            if (LL) st_ll(kvl + i, (unsigned)k0 | ((unsigned)k1 << 16), tag);
        }
    } else {
        const int j = lr - (G + 1) * d;
        const unsigned v01 = (unsigned)f2bf(y0) | ((unsigned)f2bf(y1) << 16);
        if (ok) {
            uint16_t *vv = P.vc + (kv_row(P, l, b, g) + p) * d;
            st_dev_u32(reinterpret_cast<unsigned *>(vv + j), v01);
        }
        if (LL) st_ll(kvl + half + j / 2, v01, tag);
    }
}

// Batched path: KV head g's q/k/v rows from the K-slice partials (sums in
// slice order), through qkv_store, by head g's workgroups (part of Sg).
__device__ __forceinline__ void fold_qkv(const StepParams &P, const Lds &S, int l, int g,
                                         int part) {
    const int hrows = P.qkv_rg * kTileRows, rows = P.nkv * hrows, KS = P.KSq;
    rms_table(P, S);
    const int npair = hrows / 2, total = P.B * npair, half = P.d / 2;
    for (int e = part * kThreads + kl_tid(); e < total; e += P.Sg * kThreads) {
        const int b = e / npair, lr = 2 * (e % npair);
        const float *src = P.gpart + (size_t)b * rows + g * hrows + lr;
        float y0 = 0.f, y1 = 0.f;
        for (int q0 = 0; q0 < KS; q0 += 4) {
            // (unconditional loads from in-range addresses, masked when used)
            unsigned long long v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = ld_dev_u64(src + (size_t)min(q0 + j, KS - 1) * P.qpart_stride);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (q0 + j < KS) {
                    y0 += __uint_as_float((unsigned)v[j]);
                    y1 += __uint_as_float((unsigned)(v[j] >> 32));
                }
            }
        }
        const float r = rms_of(P, S, b);   // the deferred RMSNorm scale
        y0 *= r;
        y1 *= r;
        if (P.qkv_bias) {   // (packed row order)
            const float *bias = reinterpret_cast<const float *>(
                P.arena + (size_t)l * P.layer_stride + P.off_qkv_bias);
            y0 += bias[g * hrows + lr];
            y1 += bias[g * hrows + lr + 1];
        }
        qkv_store<false>(P, l, b, g, lr, y0, y1,
                         [&](int p, int i) { return P.rope[(size_t)p * half + i]; });
    }
}

// RMSNorm + Q/K/V projection of KV head g + RoPE + KV-cache append.  The rows
// of head g's block are: its G query heads, then its key, then its value
// head; query and key rows are packed in rotation pairs (dims i, i + d/2).
// Batched path: a 2-D partition (KSq K slices x row groups of all heads)
// writes K-slice partials; after grid barrier qbar head g's workgroups fold
// them (fold_qkv).
template <bool BAT>
__device__ __forceinline__ void phase_qkv(KArg ka, int l, int gwait, int qbar, int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    const int g = blockIdx.x / P.Sg, part = blockIdx.x % P.Sg;
    const bool member = g < P.nkv;
    const uint8_t *Lb = P.arena + (size_t)l * P.layer_stride;
    const float *gain = reinterpret_cast<const float *>(Lb + P.off_attn_norm);
    const int half = P.d / 2;
    if constexpr (BAT) {
        const int KS = P.KSq, RB = P.nwg / KS, KT = P.Hp / kTileK, KTs = KT / KS;
        const int ks = blockIdx.x / RB, rb = blockIdx.x % RB, ksc = min(ks, KS - 1);
        const int nrg = P.nkv * P.qkv_rg, rows = nrg * kTileRows;
        int a0 = 0, a1 = 0;
        if (ks < KS) split_range(nrg, RB, rb, a0, a1);
        const int col0 = ksc * KTs * kTileK;
        float *pp = P.gpart + (size_t)ksc * P.qpart_stride;
        weight_phase<true>(
            P, S, Lb + P.off_qkv + (size_t)ksc * KTs * kTileBytes, KTs, a0, a1 - a0,
            [&]() { if (gwait >= 0) bar_wait(P, gwait, ti); },
            // (layer 0 reads the embedding; later layers fold the down
            // projection's partials, x: xf2 -> xf)
            [&]() {
                norm_batched(P, S, gain, l == 0 ? P.xf : P.xf2, P.xf, l == 0 ? 0 : P.KSd);
                if (is_ctl_lane0()) trace_stamp(P, ti, 3);
            },
            [&](int) {},
            [&](int c, int b0, int nb, uint16_t *buf, bool all) {
                stage_bf16_chunk(P.act + col0, P.act_lo + col0, P.Hp, KTs * kTileK, c, b0, nb, buf, all);
            },
            [&](int b, int r, float y0, float y1) {
                st_dev(pp + (size_t)b * rows + r, y0);
                st_dev(pp + (size_t)b * rows + r + 1, y1);
            },
            KT, 0, NoGroupDone(), 0,
            [&](int c) { norm_wait(P, 2 * l, staged_slices(col0, KTs * kTileK, c, kGemmChunkK)); });
        bar_arrive(P, qbar, -1);
        bar_wait(P, qbar, -1);
        if (member) {
            fold_qkv(P, S, l, g, part);
            local_arrive(P, P.cnt + g, ti);
        }
        return;
    }
    int a0 = 0, a1 = 0;
    if (member) split_range(P.qkv_rg, P.Sg, part, a0, a1);
    const int row0 = g * P.qkv_rg * kTileRows;   // first packed row of head g's block
    weight_phase<false>(
        P, S, Lb + P.off_qkv, P.Hp / kTileK, g * P.qkv_rg + a0, a1 - a0,
        [&]() { owners_wait(P, ti); }, [&]() {},
        [&](int b) {
            // the RoPE row of the sequence's position rides along (rope_row)
            auto rsrc = [&](int bb) {
                return reinterpret_cast<const float *>(P.rope +
                                                       (size_t)pos_of<true>(P, bb) * half);
            };
            if (P.multi) {
                if (b == 0)
                    stage_rms_multi(P, P.xb_ll, P.Hp, ll_tag(P, l), gain, P.H, P.Hp, P.B, S.a, P.Hp,
                                    S.sm, rsrc,
                                    [&](int bb) { return rope_row(P, S, bb); }, 2 * half);
            } else {
                stage_rms_deferred(P, P.xb_ll + (size_t)b * P.Hp, ll_tag(P, l), gain, P.H, P.Hp, S.a,
                                   S.sm, rsrc(b), rope_row(P, S, b), 2 * half);
            }
            if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
        },
        [&](int, int, int, uint16_t *, bool) {},
        [&](int b, int r, float y0, float y1) {
            // the deferred RMSNorm scale
            const float rs = rms_scale(seq_sm(P, S, b), P.H, P.eps);
            y0 *= rs;
            y1 *= rs;
            if (P.qkv_bias) {   // (packed row order)
                const float *bias = reinterpret_cast<const float *>(Lb + P.off_qkv_bias);
                y0 += bias[r];
                y1 += bias[r + 1];
            }
            qkv_store<true>(P, l, b, g, r - row0, y0, y1, [&](int, int i) {
                return reinterpret_cast<const float2 *>(rope_row(P, S, b))[i];
            }, ll_tag(P, l));
        },
        0, 0, NoGroupDone(), P.Hp);
    // (the attention polls the tagged words: no drain, no counter)
    if (is_ctl_lane0()) trace_stamp(P, ti, 0);
}

// ---------------------------------------------------------------- attention
//
// Split-K flash decoding over the whole batch at once.  The cached positions
// of a sequence are cut into units (attn_unit<D>() positions: 4 KiB of keys
// and 4 KiB of values), a sequence of position p has p / unit + 1 of them
// (the last holds the new position), and the units of all sequences, one
// sequence after the other, are dealt in equal contiguous shares to the
// workgroups of a KV head.  A share is one or more segments (a run of units
// of one sequence); its start is found once per launch (seg_init).  A share
// that starts inside a sequence hands its part of that sequence over as
// tagged words; the share with the sequence's first units, which is its last
// segment, merges them (matrix-core path; on the per-sequence path every
// segment is handed over and the O projection merges, merge_parts).  No
// barrier separates a share's segments: the waves go on to the next one while
// the control wave merges and stages.  Equal
// shares matter where contexts differ or the batch does not divide the
// workgroups: with one item per (sequence, chunk) the phase lasted as long as
// the longest item (8B shape, batch 32, contexts 2048 to 4096: ends spread
// from 49 to 86 us).
//
// A compute wave takes every kWaves-th unit of a segment and keeps the loads
// of two units' keys in flight, and of one or two units' values (VD in
// attn_units; 12 or 16 KiB, 96 or 128 KiB per workgroup, across segments).
// Both products run on the matrix cores, in layouts that need no exchange
// between lanes:
//   scores  v_mfma_f32_16x16x32_bf16, A = 16 key rows (16 bytes of a row per
//           lane), B = the queries (scaled, log2 units) as two bf16 terms
//           (three on the per-sequence path and at D = 64: their 24 bits,
//           as fp32 queries on the vector units have); column n is
//           head n & 7 (zero past G).  Tile row 4 k + v is the
//           position that the value product below wants from lane (k, n) in
//           its register v.
//   values  v_mfma_f32_16x16x4_f32 (fp32 probabilities, bf16 values exact in
//           fp32): A_e = element e of each lane's 16 bytes of a value row
//           (one load per lane covers a slab of 1024 / (2 D) positions), B =
//           the slab's probabilities as they came out of the score tile.
//           D = 64: a slab has 8 positions, 2 k and 2 k + 1 in lane group k;
//           rows and columns 0-7 are the even ones' product, 8-15 the odd
//           ones' (the other two quarters are never read).
// All heads of the group share one pass over K and V, up to 8 of them at the
// cost of one: per unit 32 fp32 products of 32 cycles against about 3000
// cycles that its 8 KiB take from HBM (a SIMD's share): bound by HBM, 6.4 TB/s
// at the 8B shape, batch 32.  The running maximum
// moves only when a score passes it by 2^8 (the exponentials stay below 2^8
// and exact sums are unaffected), so the loop has no cross-lane step.
// Measured, per layer: 70B shape (8 heads a group), batch 32, 4096 cached: 88
// us for 537 MB, against 166 with two head teams that each streamed the chunk
// and multiplied on the vector units; 8B shape, batch 16, 8192 cached: 95
// against 132; batch 1, 4096 cached: 7.1 against 8.5, 32768 cached: 26 against
// 35.
template <int D> __device__ __forceinline__ constexpr int attn_unit() { return 2048 / D; }
__device__ __forceinline__ int attn_units_of(int pnew, int up) { return pnew / up + 1; }

// A workgroup's share, in LDS (seg_table): first sequence, its first unit,
// units of the share, units of the whole batch, workgroups that have shares,
// whether the shares keep to a sequence each (seg_by_sequence, kl_shares.h).
// (one wave, once per launch, before the launch's first barrier)
__device__ __forceinline__ void seg_init(const StepParams &P, int lane) {
    const int up = 2048 / P.d;
    int T = 0;
    for (int b0 = 0; b0 < P.B; b0 += 64) {
        int u = b0 + lane < P.B ? attn_units_of(eff_pos(P, b0 + lane), up) : 0;
        for (int off = 1; off < 64; off <<= 1) u += from_lane(u, lane ^ off);
        T += u;
    }
    const int part = blockIdx.x % P.Sg;
    int *t = seg_table(P);
    if (lane == 0) t[5] = 0;
    if (!P.batched && P.B > 1 && seg_short(P.Sg, P.B, T)) {   // (B <= kMfmaBatch: a lane a sequence)
        const int u = lane < P.B ? attn_units_of(eff_pos(P, lane), up) : 0;
        int before = u;   // inclusive sum
        for (int off = 1; off < kMfmaBatch; off <<= 1) {
            const int o = from_lane(before, max(lane - off, 0));
            before += lane >= off ? o : 0;
        }
        before -= u;
        const SeqParts q = seq_parts(P.Sg, P.B, lane, before, u, T);
        int most = lane < P.B ? (u + q.count - 1) / q.count : 0;   // the largest share
        for (int off = 1; off < kMfmaBatch; off <<= 1) most = max(most, from_lane(most, lane ^ off));
        if (seg_by_sequence(P.Sg, T, __builtin_amdgcn_readfirstlane(most))) {
            if (lane < P.B && part >= q.first && part < q.first + q.span) {
                int x0 = 0, x1 = 0;
                if (part - q.first < q.count) split_range(u, q.count, part - q.first, x0, x1);
                t[0] = lane;
                t[1] = x0;
                t[2] = x1 - x0;
            }
            if (lane == 0) {
                t[3] = T;
                t[4] = P.Sg;   // (not used)
                t[5] = 1;
            }
            return;
        }
    }
    const int np = min(P.Sg, T);
    int a = 0, e = 0;
    if (part < np) split_range(T, np, part, a, e);
    if (lane == 0) {
        t[0] = t[1] = 0;
        t[2] = e - a;
        t[3] = T;
        t[4] = np;
    }
    // the sequence that holds unit a
    int before = 0;
    for (int b0 = 0; b0 < P.B; b0 += 64) {
        const int own = b0 + lane < P.B ? attn_units_of(eff_pos(P, b0 + lane), up) : 0;
        int s = own;   // inclusive sum
        for (int off = 1; off < 64; off <<= 1) {
            const int o = from_lane(s, max(lane - off, 0));
            s += lane >= off ? o : 0;
        }
        const int s0 = before + s - own;
        if (own > 0 && s0 <= a && a < s0 + own) {
            t[0] = b0 + lane;
            t[1] = a - s0;
        }
        before += __builtin_amdgcn_readlane(s, 63);
    }
}
template <int D, int G, bool LL>
__device__ __forceinline__ void attn_units(KArg ka, int l, int g, int part, int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    constexpr int UP = attn_unit<D>();              // positions per unit
    constexpr int PP = 512 / D;                     // positions per value slab
    constexpr int HS = D + 4;                       // floats between heads' wave outputs (banks)
    constexpr int WS = G * HS;                      // floats per wave
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63, k4 = lane >> 4, n = lane & 15;
    // two sets, alternating by segment: while a segment's units run, the
    // control wave merges the waves of the one before and stages the queries
    // of the one after
    constexpr int NT = LL || D == 64 ? 3 : 2, QS = D + 8;      // query terms; bf16 per row (banks)
    uint16_t *const qs0 = reinterpret_cast<uint16_t *>(S.attn);   // [2][NT][G][QS] scaled queries
    float *const wm0 = S.attn + 2 * NT * G * QS / 2;   // [2][kWaves][G] wave maxima (log2 units)
    float *const wl0 = wm0 + 2 * kWaves * G;        // [2][kWaves][G] wave sums
    float *const wa0 = wl0 + 2 * kWaves * G;        // [2][kWaves][G][HS] wave outputs
    uint16_t *const kn0 = reinterpret_cast<uint16_t *>(wa0 + 2 * kWaves * WS);   // [2][D] new key
    uint16_t *const vn0 = kn0 + 2 * D;                                           // [2][D] new value
    // waves done with the set's segments so far [2]; segments with staged queries
    int *const flags = reinterpret_cast<int *>(vn0 + 2 * D);
    auto flag = [&](int i) {
        return __hip_atomic_load(flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const int *tab = seg_table(P);
    int b = __builtin_amdgcn_readfirstlane(tab[0]), u0 = __builtin_amdgcn_readfirstlane(tab[1]);
    int left = __builtin_amdgcn_readfirstlane(tab[2]);
    if (left <= 0) return;
    int pnew = __builtin_amdgcn_readfirstlane(pos_of<LL>(P, b));
    const unsigned tag = ll_tag(P, l);

    // the merged (max, sum, unnormalised output) of the waves of set z, for
    // output t of the G D
    auto merge_waves = [&](int z, int t, float &M, float &L, float &O) {
        const float *wm = wm0 + z * kWaves * G, *wl = wl0 + z * kWaves * G;
        const int h = t / D, dd = t % D;
        M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, wm[w * G + h]);
        O = 0.f, L = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = wm[w * G + h];
            const float a = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
            L = fmaf(wl[w * G + h], a, L);
            O = fmaf(wa0[(z * kWaves + w) * WS + h * HS + dd], a, O);
        }
    };
    // output t of sequence sb
    auto finish = [&](int sb, int t, float L, float O) {
        uint16_t hi, lo;
        split_bf16(O / L, hi, lo);
        const size_t o = (size_t)sb * P.nq * D + (size_t)g * G * D + t;
        st_dev_u16(P.acto + o, hi);
        st_dev_u16(P.acto_lo + o, lo);
    };
    // a share that starts inside a sequence hands its part of it to the
    // workgroup that has the sequence's first units, as tagged words [head]
    // [D outputs, max, sum]
    // (slot: the workgroup's part; per-sequence path: part + sequence, since
    // every segment is handed over)
    unsigned long long *const parts = P.po_ll + (size_t)g * (LL ? P.Sg + P.B : P.Sg) * G * (D + 2);
    auto hand_over = [&](int sb, int t, float M, float L, float O) {
        unsigned long long *w = parts + ((size_t)(LL ? part + sb : part) * G + t / D) * (D + 2);
        st_ll_f(w + t % D, O, tag);
        if (t % D == 0) {
            st_ll_f(w + D, M, tag);
            st_ll_f(w + D + 1, L, tag);
        }
    };

    if (wid < kWaves) {
        // tile row l % 16 of this lane: its position in the unit (D = 64: in
        // the unit's first half), and the lane's position in a value slab
        const int kp = D == 128 ? (n & 3) * 4 + (n >> 2) : 8 * ((n & 3) >> 1) + 2 * (n >> 2) + (n & 1);
        const int vp = lane / (D / 8), kcol = 8 * k4, vcol = 8 * (lane % (D / 8));
        // position of score register s (0 .. 3): D = 128: slab s, position k;
        // D = 64: slab s, position 2 k (columns 0-7) or 2 k + 1 (columns 8-15)
        const int sp = D == 128 ? k4 : 2 * k4 + (n >> 3);
        // units whose values are in flight: one where two spilled inside the
        // unit loop, and the reloads of spilled registers waited for the rings
        // (per-sequence path; D = 64, with the queries' third term: 8 layers
        // of hidden 2048, 32 heads of 64 on 8 KV heads, batch 8, contexts 2000
        // 691 -> 667 us, batch 32 961 -> 927; 4 layers with 32 KV heads, batch
        // 8, 4000 565 -> 517, batch 32, 2000 828 -> 746)
        constexpr int VD = LL || D == 64 ? 1 : 2;
        u32x4 kr[2][4], vr[VD][4];
        const uint16_t *kb = nullptr, *vb = nullptr;
        // the current segment: its sequence's units, its end and the end of
        // its units with cached positions; the wave's units, its first one's
        // position, the last cached position
        int U = 0, u1 = 0, uc = 0, mine = 0, base = 0, last = 0, rot = 0;
        // The wave's i-th unit is its (i + rot) mod mine -th in memory: the
        // workgroups start at different places of their shares.  Shares are
        // often whole powers of two apart, and in step they met in the same
        // HBM banks (8B shape, batch 16, 8192 cached positions: 121 -> 95 us
        // per layer; batch 32, contexts 2048-4096: 86 -> 81; batch 32, 4096:
        // 90-93 either way).  Past the last unit: past the context.
        auto place = [&](int i) {
            const int x = i + rot;
            return i >= mine ? (1 << 16) : (x >= mine ? x - mine : x);
        };
        // (loads of unit i of the wave; positions past the cached ones take
        // the last cached one's, in range and masked when used)
        auto issue_k = [&](int j, int i) {
            const int p0 = base + place(i) * kWaves * UP + kp;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int t = D == 128 ? 0 : x >> 1, ks = D == 128 ? x : x & 1;
                kr[j][x] = ld_stream_16B(kb + (size_t)min(p0 + 16 * t, last) * D + 32 * ks);
            }
        };
        auto issue_v = [&](int j, int i) {
            const int p0 = base + place(i) * kWaves * UP + vp;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                vr[j % VD][x] = ld_stream_16B(vb + (size_t)min(p0 + x * PP, last) * D);
        };
        // units of the segments so far (the waves take the share's units in
        // turn, across its segments)
        int taken = 0;
        auto enter = [&]() {   // the segment (b, u0): addresses and the first two units' loads
            const size_t row0 = kv_row(P, l, b, g);
            kb = P.kc + row0 * D + kcol;
            vb = P.vc + row0 * D + vcol;
            last = max(pnew - 1, 0);
            U = attn_units_of(pnew, UP);
            u1 = u0 + min(left, U - u0);
            uc = min(u1, (pnew + UP - 1) / UP);
            const int f = u0 + ((wid - taken) & (kWaves - 1));
            base = f * UP;
            mine = f < uc ? (uc - f + kWaves - 1) / kWaves : 0;
            rot = mine > 0 ? (int)(blockIdx.x * 5u) % mine : 0;
            issue_k(0, 0);
            issue_v(0, 0);
            issue_k(1, 1);
            if (VD > 1) issue_v(1, 1);
        };
        enter();
        lds_barrier();
        // query operands: D = 128: 4 column blocks with two terms in one, then
        // 4 with the third; D = 64: 2 column blocks per term
        for (int seg = 0;; ++seg) {
            const int z = seg & 1;
            left -= u1 - u0;
            const int pnext = left > 0 ? __builtin_amdgcn_readfirstlane(pos_of<LL>(P, b + 1)) : 0;
            if (seg >= 2)   // (the first two were staged before the barrier)
                while (flag(2) <= seg) __builtin_amdgcn_s_sleep(1);
            asm volatile("" ::: "memory");

            // (operand x: the terms past the second stay in LDS and are read for
            // each unit, which keeps their registers free)
            const uint16_t *qs = qs0 + z * NT * G * QS;
            auto query = [&](int x, int lq) {
                const int h = lq & 7, ks = D == 128 ? x & 3 : x & 1;
                const int term = D == 128 ? 2 * (x >> 2) + ((lq >> 3) & 1) : x >> 1;
                const bool live = h < G && term < NT;
                const u32x4 w = *reinterpret_cast<const u32x4 *>(
                    qs + ((live ? term : 0) * G + (live ? h : 0)) * QS + 32 * ks + 8 * (lq >> 4));
                return __builtin_bit_cast(bf16x8, live ? w : u32x4{0u, 0u, 0u, 0u});
            };
            bf16x8 qb[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) qb[x] = query(x, kl_tid() & 63);
            f32x4 acc[8];
            float m = -INFINITY, lsum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
            // one unit whose first position is p0, cached positions below
            // lim: keys kq, values vq; kdone() / vdone() refill the ring
            auto unit = [&](u32x4 *kq, u32x4 *vq, int p0, int lim, auto &&kdone, auto &&vdone) {
                float s[4];
                if constexpr (D == 128) {
                    const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
                    auto dot = [&](int x, const f32x4 &c) {
                        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, kq[x & 3]), x < 4 ? qb[x & 3] : query(x, lane), c,
                            0, 0, 0);
                    };
                    if constexpr (LL) {
                        // (the column blocks' sums and the third terms' on their
                        // own, added as a tree: in one accumulator the scores'
                        // rounding grew the step's error by a half)
                        f32x4 a = dot(0, z4) + dot(1, z4);
                        a += dot(2, z4) + dot(3, z4);
                        const f32x4 c = dot(7, dot(6, dot(5, dot(4, z4))));
#pragma unroll
                        for (int v = 0; v < 4; ++v) s[v] = a[v] + (dpp<0x128>(a[v]) + c[v]);
                    } else {
                        const f32x4 a = dot(3, dot(2, dot(1, dot(0, z4))));
#pragma unroll
                        for (int v = 0; v < 4; ++v) s[v] = a[v] + dpp<0x128>(a[v]);   // both terms
                    }
                } else {
                    f32x4 t[2];
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
                        auto dot = [&](int x, const f32x4 &c) {
                            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, kq[2 * y + (x & 1)]),
                                x < 4 ? qb[x & 3] : query(x, lane), c, 0, 0, 0);
                        };
                        t[y] = (dot(0, z4) + dot(1, z4)) + dot(5, dot(4, dot(3, dot(2, z4))));
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        s[v] = n < 8 ? t[v >> 1][2 * (v & 1)] : t[v >> 1][2 * (v & 1) + 1];
                }
                kdone();
                if (p0 + UP > lim) {   // (uniform: the context's last unit)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (p0 + v * PP + sp >= lim) s[v] = -INFINITY;
                        if (p0 + v * PP + vp >= lim) vq[v] = u32x4{0u, 0u, 0u, 0u};
                    }
                }
                float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
                if (__any(mx > m + 8.f)) {
                    if constexpr (D == 64) mx = fmaxf(mx, dpp<0x128>(mx));
                    mx = max_16_32(mx);
                    const float mn = fmaxf(m, mx);
                    const float al = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
                    m = mn;
                    lsum *= al;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] *= al;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[v] = s[v] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s[v] - m);
                    lsum += s[v];
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const u32x4 w = vq[v];
                    const float vf[8] = {bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y),
                                         bf_lo(w.z), bf_hi(w.z), bf_lo(w.w), bf_hi(w.w)};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e], s[v], acc[e], 0, 0, 0);
                }
                vdone();
            };
            for (int i = 0; i < mine; i += 2) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int p0 = base + place(i + j) * kWaves * UP;
                    if (i + j < mine) {
                        unit(kr[j], vr[j % VD], p0, pnew, [&]() { issue_k(j, i + j + 2); },
                             [&]() { issue_v(j, i + j + VD); });
                    } else {
                        issue_k(j, i + j + 2);
                        issue_v(j, i + j + VD);
                    }
                }
            }
            if (u1 == U && ((wid - taken - (uc - u0)) & (kWaves - 1)) == 0) {
                // the new position, from LDS (by the wave whose turn it is)
                u32x4 kq[4], vq[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int ks = D == 128 ? x : x & 1;
                    const bool mk = n == 0 && (D == 128 || x < 2);
                    kq[x] = *reinterpret_cast<const u32x4 *>(kn0 + z * D + 32 * ks + kcol);
                    vq[x] = *reinterpret_cast<const u32x4 *>(vn0 + z * D + vcol);
                    if (!mk) kq[x] = u32x4{0u, 0u, 0u, 0u};
                }
                unit(kq, vq, 0, 1, []() {}, []() {});
            }
            taken += uc - u0;
            ++b;
            u0 = 0;
            pnew = pnext;
            if (left > 0) enter();
            // this wave's (max, sum, output) into set z
            lsum = sum_16_32(lsum);
            if constexpr (D == 64) {
                lsum += dpp<0x128>(lsum);
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[e][r] += from_lane(acc[e][r], ((kl_tid() & 63) + 40) & 63);
            }
            const int le = kl_tid() & 63, ke = le >> 4, ne = le & 15;
            if (ne < G && ke < D / 32) {
                float *o = wa0 + (z * kWaves + wid) * WS + ne * HS + 32 * ke;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    *reinterpret_cast<float4 *>(o + 8 * r) =
                        make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
                    *reinterpret_cast<float4 *>(o + 8 * r + 4) =
                        make_float4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
                }
                if (ke == 0) {
                    wm0[(z * kWaves + wid) * G + ne] = m;
                    wl0[(z * kWaves + wid) * G + ne] = lsum;
                }
            }
            if (left <= 0) break;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (le == 0)
                __hip_atomic_fetch_add(flags + z, 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    } else {
        // the control wave: the queries and the new key and value of sequence
        // sb, position spos, into set z
        // queries in log2 units: softmax weights are 2^(s log2(e) - max)
        const float scale = 1.4426950408889634f / sqrtf((float)D);
        auto put_q = [&](int z, int i, float q) {   // its bf16 terms
            uint16_t *d = qs0 + (z * NT * G + i / D) * QS + i % D;
            float x = q * scale;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint16_t h = f2bf(x);
                d[t * G * QS] = h;
                x -= bf2f(h);
            }
        };
        auto stage_q = [&](int sb, int spos, int z) {
            if constexpr (LL) {   // (tagged words)
                const size_t qo = (size_t)sb * P.nq * D + (size_t)g * G * D;
                const unsigned long long *kvl = P.kv_ll + ((size_t)sb * P.nkv + g) * D;
                uint16_t *kn = kn0 + z * D, *vn = vn0 + z * D;
                ll_gather<(G * D + D + 63) / 64>(
                    P, G * D + D, tag, lane, 64,
                    [&](int i) { return i < G * D ? P.q_ll + qo + i : kvl + (i - G * D); },
                    [&](int i, unsigned v) {
                        if (i < G * D) {
                            put_q(z, i, __uint_as_float(v));
                        } else if (i < G * D + D / 2) {   // key dims j and j + D/2
                            const int j = i - G * D;
                            kn[j] = (uint16_t)v;
                            kn[j + D / 2] = (uint16_t)(v >> 16);
                        } else {                           // value dims 2j and 2j + 1
                            reinterpret_cast<unsigned *>(vn)[i - G * D - D / 2] = v;
                        }
                    });
                return;
            }
            constexpr int N2 = G * D / 2, NQ = (N2 + 63) / 64;   // pairs; per lane
            const float *src = P.q + (size_t)sb * P.nq * D + (size_t)g * G * D;
            const size_t o = (kv_row(P, l, sb, g) + spos) * D + (lane % (D / 4)) * 4;
            unsigned long long qv[NQ];
#pragma unroll
            for (int k = 0; k < NQ; ++k) qv[k] = ld_dev_u64(src + 2 * min(lane + 64 * k, N2 - 1));
            const unsigned long long kv = ld_dev_u64((lane < 32 ? P.kc : P.vc) + o);
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                if (N2 % 64 == 0 || lane + 64 * k < N2) {
                    put_q(z, 2 * (lane + 64 * k), __uint_as_float((unsigned)qv[k]));
                    put_q(z, 2 * (lane + 64 * k) + 1, __uint_as_float((unsigned)(qv[k] >> 32)));
                }
            }
            if (lane % 32 < D / 4)
                reinterpret_cast<unsigned long long *>((lane < 32 ? kn0 : vn0) + z * D)[lane % 32] = kv;
        };
        // (pn[i % 3]: the position of the share's segment i's sequence, b + i)
        auto pos_at = [&](int i) { return __builtin_amdgcn_readfirstlane(pos_of<LL>(P, b + i)); };
        auto units_at = [&](int p) { return attn_units_of(p, UP); };
        int rest = left - min(left, units_at(pnew) - u0);   // units after this segment
        int pn1 = rest > 0 ? pos_at(1) : 0;
        if (lane == 0) {
            trace_stamp(P, ti, 1);
            flags[0] = flags[1] = 0;
            flags[2] = 2;
            if (!LL)
                spin_until(P, [&]() {
                    return (int)(__hip_atomic_load(P.cnt + g, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT) -
                                 (unsigned)(l + 1) * (unsigned)P.Sg) >= 0;
                });
        }
        __builtin_amdgcn_wave_barrier();
        stage_q(b, pnew, 0);
        if (rest > 0) stage_q(b + 1, pn1, 1);
        if (lane == 0) trace_stamp(P, ti, 2);
        lds_barrier();
        for (int seg = 0; rest > 0; ++seg) {
            // (segment seg is not the share's last: it ends its sequence)
            const int z = seg & 1, done = kWaves * (seg / 2 + 1);
            const int rest1 = rest - min(rest, units_at(pn1));   // after the next segment
            const int pn2 = rest1 > 0 ? pos_at(2) : 0;
            while (flag(z) < done) __builtin_amdgcn_s_sleep(1);
            asm volatile("" ::: "memory");
            for (int t = kl_tid() & 63; t < G * D; t += 64) {
                float M, L, O;
                merge_waves(z, t, M, L, O);
                if (!LL && u0 == 0) finish(b, t, L, O);
                else hand_over(b, t, M, L, O);
            }
            if (rest1 > 0) {
                stage_q(b + 2, pn2, z);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if ((kl_tid() & 63) == 0)
                    __hip_atomic_store(flags + 2, seg + 3, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            ++b;
            u0 = 0;
            left = rest;
            rest = rest1;
            pnew = pn1;
            pn1 = pn2;
        }
    }
    lds_barrier();
    // the share's last segment, by every thread: set and segment as the
    // walks above left them, found again from the share
    {
        int nb = __builtin_amdgcn_readfirstlane(tab[0]), nu = __builtin_amdgcn_readfirstlane(tab[1]);
        int nl = __builtin_amdgcn_readfirstlane(tab[2]), z = 0, U;
        const int T = __builtin_amdgcn_readfirstlane(tab[3]);
        const int np = __builtin_amdgcn_readfirstlane(tab[4]);
        int seq0, e0;
        split_range(T, np, part, seq0, e0);
        seq0 -= nu;   // the sequence's first unit, counted over the batch
        for (;;) {
            U = attn_units_of(__builtin_amdgcn_readfirstlane(pos_of<LL>(P, nb)), UP);
            if (nl <= U - nu) break;
            nl -= U - nu;
            seq0 += U;
            ++nb;
            nu = 0;
            z ^= 1;
        }
        // (the shares f + 1 .. e hold the rest of a sequence that starts here)
        const int e = (int)(((long long)(seq0 + U) * np - 1) / T);
        const int more = nu == 0 ? e - part : 0;
        constexpr int NB = 8;   // shares whose words are loaded together
        for (int t = kl_tid(); t < G * D; t += kThreads) {
            float M, L, O;
            merge_waves(z, t, M, L, O);
            if (LL || nu > 0) {
                hand_over(nb, t, M, L, O);
                continue;
            }
            for (int q0 = 0; q0 < more; q0 += NB) {
                unsigned long long v[NB][3];
                spin_until(P, [&]() {
                    bool ok = true;
#pragma unroll
                    for (int q = 0; q < NB; ++q) {
                        const unsigned long long *w =
                            parts + ((size_t)(part + 1 + min(q0 + q, more - 1)) * G + t / D) * (D + 2);
                        v[q][0] = ld_dev_u64(w + t % D);
                        v[q][1] = ld_dev_u64(w + D);
                        v[q][2] = ld_dev_u64(w + D + 1);
                    }
#pragma unroll
                    for (int q = 0; q < NB; ++q)
#pragma unroll
                        for (int i = 0; i < 3; ++i) ok = ok && ll_current(v[q][i], tag);
                    return ok;
                });
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    if (q0 + q < more) {
                        const float mq = __uint_as_float(ll_value(v[q][1]));
                        const float mn = fmaxf(M, mq);
                        const float a = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - mn);
                        const float c = mq == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mq - mn);
                        L = L * a + __uint_as_float(ll_value(v[q][2])) * c;
                        O = O * a + __uint_as_float(ll_value(v[q][0])) * c;
                        M = mn;
                    }
                }
            }
            finish(nb, t, L, O);
        }
    }
    if (is_ctl_lane0()) trace_stamp(P, ti, 3);
    lds_barrier();   // (the attention area is the next phase's)
}

// Query head h's merged outputs of sequence b.  The O projection stages them
// P.o_heads heads at a time: the words of such a part, of all sequences, are
// contiguous.
__device__ __forceinline__ unsigned long long *o_words(const StepParams &P, int b, int h, int d) {
    int h0 = 0;
    while (h - h0 >= P.o_heads) h0 += P.o_heads;
    const int n = min(P.o_heads, P.nq - h0);
    return P.o_ll + ((size_t)P.B * h0 + (size_t)b * n + (h - h0)) * d;
}

// Per-sequence path, one wave: the merged attention outputs of sequence b that
// this workgroup hands on, o = sum_c w_c A_c / sum_c w_c L_c with w_c = 2^(M_c - M),
// M the largest of the parts' maxima (A_c, M_c, L_c the parts' unnormalised
// outputs, maxima in log2 units and sums).  Items of 16 outputs of one query
// head and sequence are spread over the grid (8B shape, batch 1: one per
// workgroup), so that every part is read once, where a merge by every
// workgroup that needs a head's outputs read all of its parts in each of
// them.  Lane 16 c + j takes output j of parts c, c + 4, ..., lane c the
// maximum and sum of part c.
template <int D, int G>
__device__ __forceinline__ void merge_parts(const StepParams &P, int l, int b) {
    constexpr int MD = 16, WD = D + 2, NB = 8;   // outputs per item; loads per lane and round
    const int lane = kl_tid() & 63, j = lane & 15, cl = lane >> 4;
    const unsigned tag = ll_tag(P, l);
    const int T = __builtin_amdgcn_readfirstlane(seg_table(P)[3]);
    const int np = __builtin_amdgcn_readfirstlane(seg_table(P)[4]);
    const int items = P.nq * (D / MD);
    const auto units = [&](int q) {
        return attn_units_of(__builtin_amdgcn_readfirstlane(pos_of<true>(P, q)), 2048 / D);
    };
    int seq0 = 0;   // sequence b's first unit, counted over the batch
    for (int q = 0; q < b; ++q) seq0 += units(q);
    {
        int f, nc;
        if (__builtin_amdgcn_readfirstlane(seg_table(P)[5])) {
            const SeqParts q = seq_parts(P.Sg, P.B, b, seq0, units(b), T);
            f = q.first;
            nc = q.count;
        } else {
            f = (int)(((long long)(seq0 + 1) * np - 1) / T);
            nc = (int)(((long long)(seq0 + units(b)) * np - 1) / T) - f + 1;
        }
        for (int it = blockIdx.x; it < items; it += P.nwg) {
            const int h = it / (D / MD), d0 = it % (D / MD) * MD, g = h / G;
            const unsigned long long *src =
                P.po_ll + (((size_t)g * (P.Sg + P.B) + f + b) * G + h % G) * WD;
            float M = -INFINITY, L = 0.f, O = 0.f;
            for (int c0 = 0; c0 < nc; c0 += 4 * NB) {
                const int n = min(4 * NB, nc - c0);
                unsigned long long v[NB], vm, vl;
                for (int spins = 1;; ++spins) {
                    bool ok = true;
                    const unsigned long long *q = src + (size_t)(c0 + min(lane, n - 1)) * G * WD + D;
                    vm = ld_dev_u64(q);
                    vl = ld_dev_u64(q + 1);
#pragma unroll
                    for (int k = 0; k < NB; ++k)
                        v[k] = ld_dev_u64(src + (size_t)(c0 + min(cl + 4 * k, n - 1)) * G * WD + d0 + j);
#pragma unroll
                    for (int k = 0; k < NB; ++k) ok = ok && ll_current(v[k], tag);
                    ok = ok && ll_current(vm, tag) && ll_current(vl, tag);
                    if (__all(ok) || give_up(P, spins)) break;
                }
                const float mc = lane < n ? __uint_as_float(ll_value(vm)) : -INFINITY;
                const float mn = fmaxf(M, wave_max(mc));
                const float al = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - mn);
                const float w = mc == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc - mn);
                L = L * al + wave_sum(w * (lane < n ? __uint_as_float(ll_value(vl)) : 0.f));
                float o = 0.f;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const float wk = from_lane(w, cl + 4 * k);   // (zero past n)
                    o = fmaf(cl + 4 * k < n ? __uint_as_float(ll_value(v[k])) : 0.f, wk, o);
                }
                o = sum_16_32(o);
                O = O * al + o;
                M = mn;
            }
            if (lane < MD) st_ll_f(o_words(P, b, h, D) + d0 + j, O / L, tag);
        }
    }
}

// Attention of KV head g, by units (attn_units).  Per-sequence path: the
// segments' results leave as tagged words; batched path: the merged outputs
// are published before a grid barrier.
template <int D, int G, bool BAT>
__device__ __forceinline__ void phase_attn(KArg ka, int l, int garrive, int ti) {
    const StepParams P = load_params(ka);
    const int g = blockIdx.x / P.Sg, part = blockIdx.x % P.Sg;
    if (g < P.nkv) {
        attn_units<D, G, !BAT>(ka, l, g, part, ti);
    }
    if (garrive >= 0) bar_arrive(P, garrive, ti);
    else if (is_ctl_lane0()) trace_stamp(P, ti, 0);
}

// O projection: x += Wo o.  Per-sequence path: each workgroup for the rows it
// owns, over all of K (the packed matrices of all query heads): the weight
// ring starts at once (8B shape: it holds the whole share, 128 KiB), the
// control wave merges its items of the attention meanwhile, and every thread
// then gathers the merged outputs; the sums are complete, so the epilogue adds
// them to the owned residual and publishes it.  (By query head, with the
// merge of a head's parts in each of its workgroups and the partial products
// added by atomics before a grid barrier, the phase and the hand-off to the
// gate/up product took 16.4 us at the 8B shape, batch 1; now 14.3.)
template <int D, int G, bool BAT>
__device__ __forceinline__ void phase_oproj(KArg ka, int l, int gwait, int garrive, int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    const uint8_t *Wo = P.arena + (size_t)l * P.layer_stride + P.off_o;
    if constexpr (BAT) {
        const int KTO = G * D / kTileK;
        // 2-D partition: KSo K slices (the columns of nkv / KSo KV heads
        // each) x row groups; a workgroup writes its slice's partial sums,
        // which the next RMSNorm step folds into the residual.  Every wave
        // gets whole 16-row blocks and the activation staging is one slice.
        // (The O projection is packed per query head, D / kTileK k-tiles per
        // row group: a slice spans gps G packed matrices.)
        const int KS = P.KSo, RB = P.nwg / KS;
        const int ks = blockIdx.x / RB, rb = blockIdx.x % RB, ksc = min(ks, KS - 1);
        const int gps = P.nkv / KS, width = gps * G * D;   // KV heads and columns per slice
        int a0 = 0, a1 = 0;
        if (ks < KS) split_range(P.o_rg, RB, rb, a0, a1);
        const int col0 = ksc * width;
        float *part = P.xpart + (size_t)ksc * P.xpart_stride;
        weight_phase<true>(
            P, S, Wo + (size_t)ksc * gps * P.o_rg * KTO * kTileBytes, gps * KTO, a0, a1 - a0,
            [&]() { if (gwait >= 0) bar_wait(P, gwait, ti); },
            [&]() {}, [&](int) {},
            [&](int c, int b0, int nb, uint16_t *buf, bool all) {
                stage_bf16_chunk(P.acto + col0, P.acto_lo + col0, P.nq * D, width, c, b0, nb, buf, all);
            },
            [&](int b, int r, float y0, float y1) {
                st_dev(part + (size_t)b * P.Hp + r, y0);
                st_dev(part + (size_t)b * P.Hp + r + 1, y1);
            },
            D / kTileK, (size_t)P.o_rg * (D / kTileK));
    } else {
        const OwnRows R = own_rows(P);
        constexpr int KTq = D / kTileK;
        const int K = P.nq * D, KT = P.nq * KTq;
        const unsigned tag = ll_tag(P, l);
        auto wait = [&]() {
            // (sequence 0 by the control wave, whose loads do not queue behind
            // a ring; the others by a compute wave each, beside it)
            const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
            const int b = wid == kCtlWave ? 0 : wid + 1;
            if (is_ctl_lane0()) trace_stamp(P, ti, 1);
            if (b < P.B) merge_parts<D, G>(P, l, b);
            if (is_ctl_lane0()) trace_stamp(P, ti, 2);
            lds_barrier();   // (as in owners_wait)
        };
        auto epi = [&](int b, int r, double y0, double y1) {
            const long long *x = own_x(P) + b * P.own_max + (r - R.first);
            put_x(P, b, r - R.first, R, x[0] + to_fix(y0), P.xa_ll, tag);
            put_x(P, b, r + 1 - R.first, R, x[1] + to_fix(y1), P.xa_ll, tag);
        };
        if (P.multi) {
            // (a part of the heads at a time, where LDS cannot hold the
            // outputs of all: the sums of the parts but the last are added to
            // the owned residual without publishing it)
            for (int h0 = 0; h0 < P.nq; h0 += P.o_heads) {
                const int nh = min(P.o_heads, P.nq - h0), Kp = nh * D;
                gemv_phase<true, KTq>(
                    Wo + (size_t)h0 * P.o_rg * KTq * kTileBytes, nh * KTq,
                    R.first / kTileRows, R.count / kTileRows, P.B, S.a, S.red, P.dummy,
                    [&]() { if (h0 == 0) wait(); },
                    [&](int b) {
                        // (the control wave leaves the gather to the others,
                        // whose rings are done by then; all sequences'
                        // outputs, b Kp floats apart)
                        if (b == 0)
                            ll_gather<16>(
                                P, P.B * Kp, tag, kl_tid(), kThreads,
                                [&](int i) { return P.o_ll + (size_t)P.B * h0 * D + i; },
                                [&](int i, unsigned v) {
                                    if (P.multi == 2) {
                                        const int q = (i >= K) + (i >= 2 * K) + (i >= 3 * K);
                                        mm_put(mm_act(S), mm_stride(K), q, i - q * K,
                                               __uint_as_float(v));
                                    } else {
                                        S.a[i] = __uint_as_float(v);
                                    }
                                });
                        if (b == P.B - 1) lds_barrier();
                        if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
                    },
                    [&](int b, int r, double y0, double y1) {
                        if (h0 + nh == P.nq) return epi(b, r, y0, y1);
                        long long *x = own_x(P) + b * P.own_max + (r - R.first);
                        x[0] += to_fix(y0);
                        x[1] += to_fix(y1);
                    },
                    Kp, P.o_rg * KTq, mm_slots(P, S));
            }
        } else {
            gemv_phase<false, KTq>(
                Wo, KT, R.first / kTileRows, R.count / kTileRows, P.B, S.a, S.red, P.dummy, wait,
                [&](int b) {
                    ll_gather<8>(P, K, tag, kl_tid(), kThreads,
                                 [&](int i) { return P.o_ll + (size_t)b * K + i; },
                                 [&](int i, unsigned v) { S.a[i] = __uint_as_float(v); });
                    lds_barrier();
                    if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
                },
                epi, 0, P.o_rg * KTq);
        }
        if (is_ctl_lane0()) trace_stamp(P, ti, 0);
    }
    if (garrive >= 0) bar_arrive(P, garrive, ti);
}


// ---------------------------------------------------------------- mixture of experts
//
// Per-sequence path (the Mixtral variant of Table 2).  Each of a token's
// top_k expert slots has nwg / top_k workgroups, laid out like the dense
// FFN's (column block j = w / Rc of the slot's expert).  Every workgroup
// computes the router logits of every sequence itself (same data, same
// order: the same values everywhere), so no hand-off is needed, and keeps
// the chosen experts in LDS for the down phase of the same launch.

// Router logits of sequence b from the staged activation (a = x gain, the
// RMSNorm scale deferred as in the gate/up product): the packed router (one
// row group of E <= 8 rows) split over the compute waves by k-tiles, the
// wave partials added in wave order; then the top_k experts (the lowest index
// first among equal logits) and the softmax of their logits.
__device__ __forceinline__ void route_experts(const StepParams &P, const Lds &S,
                                              const uint8_t *Lb, int b) {
    const int wid = __builtin_amdgcn_readfirstlane(kl_tid() >> 6);
    const int lane = kl_tid() & 63, row = lane >> 3, sub = lane & 7;
    const int KT = P.Hp / kTileK;
    if (wid < kWaves) {
        const uint8_t *R = Lb + P.off_router + (size_t)lane * 16;
        float acc = 0.f;
        for (int kt = (wid * KT) / kWaves; kt < ((wid + 1) * KT) / kWaves; ++kt) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(R + (size_t)kt * kTileBytes);
            const float *ap = S.a + kt * kTileK + sub * 8;
            const float4 a0 = *reinterpret_cast<const float4 *>(ap);
            const float4 a1 = *reinterpret_cast<const float4 *>(ap + 4);
            acc = fmaf(bf_lo(w.x), a0.x, acc);
            acc = fmaf(bf_hi(w.x), a0.y, acc);
            acc = fmaf(bf_lo(w.y), a0.z, acc);
            acc = fmaf(bf_hi(w.y), a0.w, acc);
            acc = fmaf(bf_lo(w.z), a1.x, acc);
            acc = fmaf(bf_hi(w.z), a1.y, acc);
            acc = fmaf(bf_lo(w.w), a1.z, acc);
            acc = fmaf(bf_hi(w.w), a1.w, acc);
        }
        acc = sum8(acc);
        if (sub == 0) S.red[wid * kTileRows + row] = acc;
    }
    lds_barrier();
    float *logit = S.red + kWaves * kTileRows;
    if (kl_tid() < kTileRows) {
        float t = 0.f;
        for (int w = 0; w < kWaves; ++w) t += S.red[w * kTileRows + kl_tid()];
        logit[kl_tid()] = t * rms_scale(S.sm, P.H, P.eps);
    }
    lds_barrier();
    if (kl_tid() == 0) {
        int e0 = 0;
        for (int e = 1; e < P.E; ++e)
            if (logit[e] > logit[e0]) e0 = e;
        int e1 = e0;
        float w0 = 1.f, w1 = 0.f;
        if (P.topk == 2) {
            e1 = -1;
            for (int e = 0; e < P.E; ++e)
                if (e != e0 && (e1 < 0 || logit[e] > logit[e1])) e1 = e;
            const float t = expf(logit[e1] - logit[e0]);   // softmax of the two logits
            w0 = 1.f / (1.f + t);
            w1 = t / (1.f + t);
        }
        int *rt = route_table(P) + 4 * b;
        rt[0] = e0;
        rt[1] = e1;
        rt[2] = __float_as_int(w0);
        rt[3] = __float_as_int(w1);
    }
    lds_barrier();
}

// The expert slot, FFN column block and part of this workgroup (slot >= topk
// or j >= Sc: no FFN rows).
struct MoeShare { int slot, j, part; };
__device__ __forceinline__ MoeShare moe_share(const StepParams &P) {
    const int nwk = P.nwg / P.topk, loc = blockIdx.x % nwk;
    return MoeShare{(int)blockIdx.x / nwk, loc / P.Rc, loc % P.Rc};
}

// RMSNorm, router, and the gate/up product + SwiGLU of this workgroup's
// expert slot for each sequence: m[b][slot] as tagged words.
__device__ __forceinline__ void moe_gateup(const StepParams &P, const Lds &S, int l, int ti) {
    const uint8_t *Lb = P.arena + (size_t)l * P.layer_stride;
    const float *gain = reinterpret_cast<const float *>(Lb + P.off_ffn_norm);
    const MoeShare ms = moe_share(P);
    const bool member = ms.slot < P.topk && ms.j < P.Sc;
    int first = 0, count = 0;
    if (member) {   // as the dense FFN: block j covers SwiGLU outputs [j KTc 64, + KTc 64)
        const int r0 = min(P.gu_rg, ms.j * P.KTc * 2 * kTileK / kTileRows);
        const int r1 = min(P.gu_rg, (ms.j + 1) * P.KTc * 2 * kTileK / kTileRows);
        int a0, a1;
        split_rows(r1 - r0, P.Rc, ms.part, a0, a1);
        first = r0 + a0;
        count = a1 - a0;
    }
    // (a workgroup without rows in either product reads nothing: nothing it
    // hands on would hold the residual's owners back from overwriting the
    // words)
    if (!member) return;
    {
        int a0, a1;
        split_rows(P.down_rg, P.Rc, ms.part, a0, a1);
        if (count == 0 && a0 == a1) return;
    }
    if (is_ctl_lane0()) trace_stamp(P, ti, 1);
    for (int b = 0; b < P.B; ++b) {
        stage_rms_deferred(P, P.xa_ll + (size_t)b * P.Hp, ll_tag(P, l), gain, P.H, P.Hp, S.a, S.sm);
        route_experts(P, S, Lb, b);
        if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
        const int e = route_table(P)[4 * b + ms.slot];
        gemv_phase(
            Lb + P.off_gu + (size_t)e * P.gu_estride, P.Hp / kTileK, first, count, 1, S.a,
            S.red, P.dummy, [&]() {}, [&](int) {},
            [&](int, int r, float gt, float up) {
                const float rs = rms_scale(S.sm, P.H, P.eps);
                gt *= rs;
                up *= rs;
                st_ll_f(P.m_ll + ((size_t)b * P.topk + ms.slot) * P.Fp + (r >> 1),
                        gt / (1.0f + expf(-gt)) * up, ll_tag(P, l));
            });
    }
}

// Down product of this workgroup's expert slot for each sequence, weighted
// by the slot's router weight, added into the residual.
__device__ __forceinline__ void moe_down(const StepParams &P, const Lds &S, int l, int ti) {
    const MoeShare ms = moe_share(P);
    if (ms.slot >= P.topk || ms.j >= P.Sc) return;
    int a0, a1;
    split_rows(P.down_rg, P.Rc, ms.part, a0, a1);
    if (a0 == a1) return;
    const int kw = P.KTc * kTileK, c0 = ms.j * kw, nreal = max(0, min(kw, P.F - c0));
    const int nj = P.topk * P.Sc;
    for (int b = 0; b < P.B; ++b) {
        const int *rt = route_table(P) + 4 * b;
        const int e = rt[ms.slot];
        const float we = __int_as_float(rt[2 + ms.slot]);
        gemv_phase(
            P.arena + (size_t)l * P.layer_stride + P.off_down + (size_t)e * P.down_estride +
                (size_t)ms.j * P.down_rg * P.KTc * kTileBytes,
            P.KTc, a0, a1 - a0, 1, S.a, S.red, P.dummy, [&]() {},
            [&](int) {
                if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 1);
                if ((kl_tid() >> 6) == kCtlWave)
                    ll_gather<kDownGather>(
                        P, nreal, ll_tag(P, l), kl_tid() & 63, 64,
                        [&](int i) {
                            return P.m_ll + ((size_t)b * P.topk + ms.slot) * P.Fp + c0 + i;
                        },
                        [&](int i, unsigned v) { S.a[i] = __uint_as_float(v); });
                for (int i = nreal + kl_tid(); i < kw; i += kThreads) S.a[i] = 0.f;
                lds_barrier();
                if (b == 0 && is_ctl_lane0()) {
                    trace_stamp(P, ti, 2);
                    trace_stamp(P, ti, 3);
                }
            },
            [&](int, int r, float y0, float y1) {
                unsigned long long *w = P.dp_ll + ((size_t)b * nj + ms.slot * P.Sc + ms.j) * P.Hp + r;
                st_ll_f(w, we * y0, ll_tag(P, l));
                st_ll_f(w + 1, we * y1, ll_tag(P, l));
            });
    }
}

// RMSNorm + gate/up projection + SwiGLU for FFN column block j = w / Rc:
// m = silu(Wg u) * (Wu u).  Packed rows alternate gate i, up i.
template <bool BAT>
__device__ __forceinline__ void phase_gateup(KArg ka, int l, int gwait, int garrive, int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    const uint8_t *Lb = P.arena + (size_t)l * P.layer_stride;
    const float *gain = reinterpret_cast<const float *>(Lb + P.off_ffn_norm);
    if constexpr (BAT) {
        // 2-D partition: KSg K slices (of Hp / KSg columns, one chunk or a
        // few) x row groups, so a workgroup's load ring streams through all
        // of its blocks within few chunks; the gate and up partial sums go
        // to the slice's partial buffer, and the SwiGLU is applied when the
        // down phase folds them (fold_swiglu); with one slice (see the host's
        // choice) it is applied in the epilogue
        const int KS = P.KSg, RB = P.nwg / KS, KT = P.Hp / kTileK, KTs = KT / KS;
        const int ks = blockIdx.x / RB, rb = blockIdx.x % RB, ksc = min(ks, KS - 1);
        int a0 = 0, a1 = 0;
        if (ks < KS) split_range(P.gu_rg, RB, rb, a0, a1);
        const int col0 = ksc * KTs * kTileK;
        float *part = P.gpart + (size_t)ksc * P.gpart_stride;
        const int grow = P.gu_rg * kTileRows;
        weight_phase<true>(
            P, S, Lb + P.off_gu + (size_t)ksc * KTs * kTileBytes, KTs, a0, a1 - a0,
            [&]() { if (gwait >= 0) bar_wait(P, gwait, ti); },
            // (folds the O projection's partials, x: xf -> xf2)
            [&]() {
                norm_batched(P, S, gain, P.xf, P.xf2, P.KSo);
                if (is_ctl_lane0()) trace_stamp(P, ti, 3);
            },
            [&](int) {},
            [&](int c, int b0, int nb, uint16_t *buf, bool all) {
                stage_bf16_chunk(P.act + col0, P.act_lo + col0, P.Hp, KTs * kTileK, c, b0, nb, buf, all);
            },
            [&](int b, int r, float gt, float up) {
                if (KS > 1) {
                    st_dev(part + (size_t)b * grow + r, gt);
                    st_dev(part + (size_t)b * grow + r + 1, up);
                    return;
                }
                // one slice: the sums are complete, and the SwiGLU is applied here
                const float rs = rms_of(P, S, b), g = gt * rs;
                uint16_t hi, lo;
                split_bf16(g / (1.0f + expf(-g)) * (up * rs), hi, lo);
                const size_t o = (size_t)b * P.Fp + (r >> 1);
                st_dev_u16(P.actm + o, hi);
                st_dev_u16(P.actm_lo + o, lo);
            },
            KT, 0, NoGroupDone(), 0,
            [&](int c) {
                norm_wait(P, 2 * l + 1, staged_slices(col0, KTs * kTileK, c, kGemmChunkK));
            },
            // (the sequences' RMSNorm scales for the epilogue: every slice is complete)
            [&](int b0, int nb) {
                const int b = b0 + (int)(kl_tid() & 63);
                if (KS == 1 && (int)(kl_tid() & 63) < nb && b < kRScaleTable) S.red[b] = rms_r(P, b);
            });
        if (garrive >= 0) bar_arrive(P, garrive, ti);
        return;
    }
    if (P.E > 1) {
        moe_gateup(P, S, l, ti);
        if (is_ctl_lane0()) trace_stamp(P, ti, 0);
        return;
    }
    const int j = blockIdx.x / P.Rc, part = blockIdx.x % P.Rc;
    const bool member = j < P.Sc;
    int first = 0, count = 0;
    if (member) {
        // block j covers SwiGLU outputs [j KTc 64, (j + 1) KTc 64): 2 packed rows each
        const int r0 = min(P.gu_rg, j * P.KTc * 2 * kTileK / kTileRows);
        const int r1 = min(P.gu_rg, (j + 1) * P.KTc * 2 * kTileK / kTileRows);
        int a0, a1;
        split_rows(r1 - r0, P.Rc, part, a0, a1);
        first = r0 + a0;
        count = a1 - a0;
    }
    weight_phase<false>(
        P, S, Lb + P.off_gu, P.Hp / kTileK, first, count,
        [&]() { if (is_ctl_lane0()) trace_stamp(P, ti, 1); }, [&]() {},
        [&](int b) {
            if (P.multi) {
                if (b == 0)
                    stage_rms_multi(P, P.xa_ll, P.Hp, ll_tag(P, l), gain, P.H, P.Hp, P.B, S.a, P.Hp,
                                    S.sm, NoExtra(), NoExtra(), 0);
            } else {
                stage_rms_deferred(P, P.xa_ll + (size_t)b * P.Hp, ll_tag(P, l), gain, P.H, P.Hp, S.a,
                                   S.sm);
            }
            if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
        },
        [&](int, int, int, uint16_t *, bool) {},
        [&](int b, int r, float gt, float up) {
            // the deferred RMSNorm scale
            const float rs = rms_scale(seq_sm(P, S, b), P.H, P.eps);
            gt *= rs;
            up *= rs;
            st_ll_f(P.m_ll + (size_t)b * P.Fp + (r >> 1), gt / (1.0f + expf(-gt)) * up,
                    ll_tag(P, l));
        },
        0, 0, NoGroupDone(), P.Hp);
    // (the down projection polls the tagged words: no drain, no counter)
    if (is_ctl_lane0()) trace_stamp(P, ti, 0);
}

// Batched path: the SwiGLU of the gate/up K-slice partials, m = silu(g) u with
// g, u the fixed-order sums over the slices, as the two bf16 terms the down
// projection stages; the (sequence, FFN column) elements are spread over the
// grid.  Ends with grid barrier k.
__device__ __forceinline__ void fold_swiglu(const StepParams &P, const Lds &S, int k) {
    const int F = P.F, grow = P.gu_rg * kTileRows, KS = P.KSg;
    rms_table(P, S);
    const int total = P.B * F, stride = P.nwg * kThreads;
    // a thread's elements e0 + k stride, k < FE, are loaded together (one
    // memory round trip per KS / 4 slices instead of one per element)
    constexpr int FE = 4;
    for (int e0 = blockIdx.x * kThreads + kl_tid(); e0 - (int)kl_tid() < total;
         e0 += FE * stride) {
        float gs[FE], us[FE];
#pragma unroll
        for (int k = 0; k < FE; ++k) gs[k] = us[k] = 0.f;
        for (int q0 = 0; q0 < KS; q0 += 4) {
            // (unconditional loads from in-range addresses, masked when used)
            unsigned long long v[FE][4];
#pragma unroll
            for (int k = 0; k < FE; ++k) {
                const int ec = min(e0 + k * stride, total - 1), b = ec / F, f = ec % F;
                const float *src = P.gpart + (size_t)b * grow + 2 * f;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[k][j] = ld_dev_u64(src + (size_t)min(q0 + j, KS - 1) * P.gpart_stride);
            }
#pragma unroll
            for (int k = 0; k < FE; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (q0 + j < KS) {
                        gs[k] += __uint_as_float((unsigned)v[k][j]);
                        us[k] += __uint_as_float((unsigned)(v[k][j] >> 32));
                    }
                }
        }
#pragma unroll
        for (int k = 0; k < FE; ++k) {
            const int e = e0 + k * stride;
            if (e < total) {
                const int b = e / F, f = e % F;
                const float r = rms_of(P, S, b);   // the deferred RMSNorm scale
                const float g = gs[k] * r, u = us[k] * r;
                uint16_t hi, lo;
                split_bf16(g / (1.0f + expf(-g)) * u, hi, lo);
                st_dev_u16(P.actm + (size_t)b * P.Fp + f, hi);
                st_dev_u16(P.actm_lo + (size_t)b * P.Fp + f, lo);
            }
        }
    }
    bar_arrive(P, k, -1);
    bar_wait(P, k, -1);
}

// Down projection of FFN column block j: x += Wd[:, block j] m[block j], for
// the rows this workgroup owns among block j's workgroups.
template <bool BAT>
__device__ __forceinline__ void phase_down(KArg ka, int l, int gwait, int xbar, int garrive,
                                           int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    const uint8_t *Wd = P.arena + (size_t)l * P.layer_stride + P.off_down;
    if constexpr (BAT) {
        // 2-D partition: KSd K slices (Sc / KSd FFN column blocks each) x row
        // groups, partial sums folded by the next RMSNorm step (as for the O
        // projection)
        const int KS = P.KSd, RB = P.nwg / KS;
        const int ks = blockIdx.x / RB, rb = blockIdx.x % RB, ksc = min(ks, KS - 1);
        const int gps = P.Sc / KS, width = gps * P.KTc * kTileK;
        int a0 = 0, a1 = 0;
        if (ks < KS) split_range(P.down_rg, RB, rb, a0, a1);
        const size_t col0 = (size_t)ksc * width;
        float *part = P.xpart + (size_t)ksc * P.xpart_stride;
        weight_phase<true>(
            P, S, Wd + (size_t)ksc * gps * P.down_rg * P.KTc * kTileBytes, gps * P.KTc, a0,
            a1 - a0, [&]() { if (gwait >= 0) bar_wait(P, gwait, ti); },
            [&]() {
                if (xbar >= 0) fold_swiglu(P, S, xbar);
                if (is_ctl_lane0()) trace_stamp(P, ti, 3);
            },
            [&](int) {},
            [&](int c, int b0, int nb, uint16_t *buf, bool all) {
                stage_bf16_chunk(P.actm + col0, P.actm_lo + col0, P.Fp, width, c, b0, nb, buf, all);
            },
            [&](int b, int r, float y0, float y1) {
                st_dev(part + (size_t)b * P.Hp + r, y0);
                st_dev(part + (size_t)b * P.Hp + r + 1, y1);
            },
            P.KTc, (size_t)P.down_rg * P.KTc);
    } else if (P.E > 1) {
        moe_down(P, S, l, ti);
        if ((kl_tid() >> 6) == kCtlWave) gather_down(P, l, P.topk * P.Sc);
        if (is_ctl_lane0()) trace_stamp(P, ti, 0);
    } else {
        const int j = blockIdx.x / P.Rc, part = blockIdx.x % P.Rc;
        // (the partial products to the rows' owners, gather_down)
        auto epi = [&](int b, int r, float y0, float y1) {
            unsigned long long *w = P.dp_ll + ((size_t)b * P.Sc + j) * P.Hp + r;
            st_ll_f(w, y0, ll_tag(P, l));
            st_ll_f(w + 1, y1, ll_tag(P, l));
        };
        if (j < P.Sc) {
            int a0, a1;
            split_rows(P.down_rg, P.Rc, part, a0, a1);
            const int kw = P.KTc * kTileK, c0 = j * kw, nreal = max(0, min(kw, P.F - c0));
            weight_phase<false>(
                P, S, Wd + (size_t)j * P.down_rg * P.KTc * kTileBytes, P.KTc, a0, a1 - a0,
                [&]() {}, [&]() {},
                [&](int b) {
                    // block j of the SwiGLU output as tagged words, gathered
                    // by the control wave (its loads are not queued behind
                    // the weight ring); padding columns are zero.  With
                    // P.multi the first call gathers every sequence's block
                    // (block of sequence bb at a + bb kw).
                    if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 1);
                    if (P.multi) {
                        if (b > 0) return;
                        if ((kl_tid() >> 6) == kCtlWave)
                            ll_gather<kDownGather>(
                                P, P.B * nreal, ll_tag(P, l), kl_tid() & 63, 64,
                                [&](int i) {
                                    const int bb = i / nreal;
                                    return P.m_ll + (size_t)bb * P.Fp + c0 + (i - bb * nreal);
                                },
                                [&](int i, unsigned v) {
                                    const int bb = i / nreal;
                                    if (P.multi == 2)
                                        mm_put(mm_act(S), mm_stride(kw), bb, i - bb * nreal,
                                               __uint_as_float(v));
                                    else
                                        S.a[bb * kw + (i - bb * nreal)] = __uint_as_float(v);
                                });
                        for (int i = kl_tid(); i < P.B * (kw - nreal); i += kThreads) {
                            const int bb = i / (kw - nreal);
                            const int k = nreal + (i - bb * (kw - nreal));
                            if (P.multi == 2) mm_put(mm_act(S), mm_stride(kw), bb, k, 0.f);
                            else S.a[bb * kw + k] = 0.f;
                        }
                    } else {
                        if ((kl_tid() >> 6) == kCtlWave)
                            ll_gather<kDownGather>(
                                P, nreal, ll_tag(P, l), kl_tid() & 63, 64,
                                [&](int i) { return P.m_ll + (size_t)b * P.Fp + c0 + i; },
                                [&](int i, unsigned v) { S.a[i] = __uint_as_float(v); });
                        for (int i = nreal + kl_tid(); i < kw; i += kThreads) S.a[i] = 0.f;
                    }
                    lds_barrier();
                    if (b == 0 && is_ctl_lane0()) {
                        trace_stamp(P, ti, 2);
                        trace_stamp(P, ti, 3);
                    }
                },
                [&](int, int, int, uint16_t *, bool) {}, epi, 0, 0, NoGroupDone(), kw);
        }
        if ((kl_tid() >> 6) == kCtlWave) gather_down(P, l, P.Sc);
        if (is_ctl_lane0()) trace_stamp(P, ti, 0);
    }
    if (garrive >= 0) bar_arrive(P, garrive, ti);
}

// Batched path: the final residual stream -> hidden_out (fp32), elements
// spread over the grid.  (One memory round trip; by one workgroup alone the
// copy is a chain of B H / kThreads of them, which ended 130 us after the rest
// of the head at the 8B shape and batch 32, 280 us at the 70B shape.)
__device__ __forceinline__ void copy_hidden(const StepParams &P) {
    for (int idx = blockIdx.x * kThreads + kl_tid(); idx < P.B * P.H; idx += P.nwg * kThreads) {
        const int b = idx / P.H;
        const float x = from_fix((long long)ld_dev_u64(P.xf + (size_t)b * P.Hp + idx % P.H));
        P.hidden_out[idx] = seq_ok(P, b) ? x : __builtin_nanf("");
    }
}

// Classifier block (Sec. 2): final RMSNorm + LM head -> fp32 logits.
template <bool BAT>
__device__ __forceinline__ void phase_head(KArg ka, int gwait, int ti) {
    const StepParams P = load_params(ka);
    const Lds S = lds_layout(kl_smem, P);
    const RgRange R = own_rgs<BAT>(P.head_rg, P);
    const int V = P.V;
    // greedy sampling: this workgroup's best key per sequence (LDS atomics),
    // then one device-scope atomic per sequence into P.amax
    unsigned long long *best = amax_slots(P);
    const bool sample = P.amax != nullptr;
    if (sample && kl_tid() < (BAT ? kGemmBatch : kMfmaBatch))
        best[kl_tid()] = 0ull;   // (staging barriers follow)
    // per-sequence path: this workgroup has read the epoch (bar_init); the
    // answer is used at the end of the phase
    unsigned arrivals = 0;
    auto epoch_arrive = [&]() {
        if (!BAT && is_ctl_lane0())
            arrivals = __hip_atomic_fetch_add(P.epoch_arrivals, 1u, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
    };
    auto flush = [&](int b0, int nb) {
        if (!sample) return;
        __syncthreads();
        const int t = kl_tid();
        if (t < nb) {
            const unsigned long long k = best[t];
            if (k) __hip_atomic_fetch_max(P.amax + b0 + t, k, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
            best[t] = 0ull;
        }
        __syncthreads();
    };
    weight_phase<BAT>(
        P, S, reinterpret_cast<const uint8_t *>(P.lm_head), P.Hp / kTileK, R.first, R.count,
        [&]() {
            if (gwait >= 0) bar_wait(P, gwait, ti);
            if (!BAT) owners_wait(P, ti);
        },
        [&]() {
            // (folds the last down projection's partials, x: xf2 -> xf), and
            // the sequences' RMSNorm scales for the epilogue
            norm_batched(P, S, P.final_norm, P.xf2, P.xf, P.KSd);
            norm_wait(P, 2 * P.L, SliceRange{0, (P.Hp + kGemmChunkK - 1) / kGemmChunkK});
            __syncthreads();
            rms_table(P, S);
            if (is_ctl_lane0()) trace_stamp(P, ti, 3);
            if (P.hidden_out) copy_hidden(P);
        },
        [&](int b) {
            if (P.multi) {
                if (b == 0)
                    stage_rms_multi(P, P.xb_ll, P.Hp, ll_tag(P, P.L), P.final_norm, P.H, P.Hp, P.B,
                                    S.a, P.Hp, S.sm, NoExtra(), NoExtra(), 0);
            } else {
                stage_rms_deferred(P, P.xb_ll + (size_t)b * P.Hp, ll_tag(P, P.L), P.final_norm, P.H,
                                   P.Hp, S.a, S.sm);
            }
            // (behind the staging's loads, beside the products)
            if (b == 0) epoch_arrive();
            if (b == 0 && is_ctl_lane0()) trace_stamp(P, ti, 3);
        },
        [&](int c, int b0, int nb, uint16_t *buf, bool all) { stage_act_chunk(P, c, b0, nb, buf, all); },
        [&](int b, int r, float y0, float y1) {
            // the deferred RMSNorm scale
            const float rs = !BAT ? rms_scale(seq_sm(P, S, b), P.H, P.eps) : rms_of(P, S, b);
            y0 *= rs;
            y1 *= rs;
            const bool ok = ok_of<!BAT>(P, b);
            if (!ok) y0 = y1 = __builtin_nanf("");
            float *lg = P.logits + (size_t)b * V;
            if (r < V) lg[r] = y0;
            if (r + 1 < V) lg[r + 1] = y1;
            if (sample && ok) {
                unsigned long long k = (r < V) ? argmax_key(y0, r) : 0ull;
                if (r + 1 < V) k = max(k, argmax_key(y1, r + 1));
                __hip_atomic_fetch_max(best + (BAT ? b % kGemmBatch : b), k, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        },
        0, 0, [&](int b0, int nb) { flush(b0, nb); }, P.Hp);
    if constexpr (!BAT) {
        if (R.count == 0) epoch_arrive();   // (nothing was staged)
        flush(0, P.B);
        // the hidden state: every workgroup its own rows (each row's last
        // value was put by the control wave or before the launch)
        if (P.hidden_out && (kl_tid() >> 6) == kCtlWave) {
            const OwnRows O = own_rows(P);
            for (int i = kl_tid() & 63; i < P.B * O.count; i += 64) {
                const int b = i / O.count, r = i % O.count;
                P.hidden_out[(size_t)b * P.H + O.first + r] =
                    ok_of<true>(P, b) ? from_fix(own_x(P)[b * P.own_max + r]) : __builtin_nanf("");
            }
        }
    }
    // the step's last phase: the next step's tags.  Per-sequence path: by the
    // last workgroup that has read this step's (a launch of the head alone
    // polls for tags of this step, and nothing else of it orders a workgroup
    // that starts late before one that is done; in the looped launch likewise
    // a workgroup without work in the layers).  Matrix-core path: the head
    // uses no tags, and a launch with layers has had every workgroup in its
    // grid barriers.
    const bool last = BAT ? blockIdx.x == 0 : epoch_last_arrival(arrivals, P.nwg);
    if (last && is_ctl_lane0()) {
        if (!BAT)
            __hip_atomic_store(P.epoch_arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(P.epoch_ptr, ll_next_epoch(*launch_epoch(P), P.L + 1), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (is_ctl_lane0()) trace_stamp(P, ti, 0);
}

// ---------------------------------------------------------------- kernels

// Runs the phases selected by 'phases' for layers [l0, l1) in order:
// embed, (qkv, attn, oproj, gateup, down) per layer, head.  Grid barrier k is
// the k-th arrival of the launch; a phase that needs the residual stream waits
// on the latest one, and an arriving phase arrives only if a later phase of
// the same launch waits (a launch boundary already orders the rest).
template <int D, int G, bool BAT>
__global__ __launch_bounds__(kThreads) void kl_step_kernel(StepParams P, int l0, int l1,
                                                          int phases) {
    (void)P;   // read through the kernel-argument segment (see load_params)
    const KArg ka = kernarg_address();
    const bool has_qkv = phases & kPhQkv, has_gu = phases & kPhGateUp, has_head = phases & kPhHead;
    const int nlay = (phases & kPhLayer) ? l1 - l0 : 0;
    // batched steps add grid barriers of their own: after the q/k/v product
    // (its fold) and in the SwiGLU fold (their RMSNorm steps hand over through
    // slice counters instead)
    constexpr bool batched = BAT;
    bar_init(load_params(ka));
    int na = 0, ti = 0;   // grid arrivals so far; phase index (for the trace)
    auto gw = [&]() { return na - 1; };                 // barrier to wait on (-1: none)
    auto ga = [&](bool waited_later) { return waited_later ? na++ : -1; };
    auto xb = [&]() { return batched ? na++ : -1; };    // the phase's own barrier
    const bool has_attn = phases & kPhAttn, has_op = phases & kPhOproj;
    const bool has_down = phases & kPhDown;
    // (the per-sequence path has no grid barriers: tagged words throughout)
    if (phases & kPhEmbed) {
        phase_embed(ka, -1, BAT ? ga((has_qkv && nlay > 0) || has_head) : -1, ti++);
    }
    for (int l = l0; l < l1; ++l) {
        // batched steps: attn -> oproj and gateup -> down are grid barriers
        // too (full-K products with one writer per output)
        if (phases & kPhQkv) {
            const int w = gw(), q = xb();
            phase_qkv<BAT>(ka, l, w, q, ti++);
        }
        if (phases & kPhAttn) phase_attn<D, G, BAT>(ka, l, BAT ? ga(has_op) : -1, ti++);
        if (phases & kPhOproj) {
            const int w = BAT && has_attn ? gw() : -1, a = BAT ? ga(has_gu) : -1;
            phase_oproj<D, G, BAT>(ka, l, w, a, ti++);
        }
        if (phases & kPhGateUp) {
            const int w = gw(), a = BAT ? ga(has_down) : -1;
            phase_gateup<BAT>(ka, l, w, a, ti++);
        }
        if (phases & kPhDown) {
            // (batched: the SwiGLU fold of the gate/up partials, with several K
            // slices, ends with a grid barrier of its own)
            const int w = BAT && has_gu ? gw() : -1;
            const int x = BAT && load_params(ka).KSg > 1 ? na++ : -1;
            phase_down<BAT>(ka, l, w, x, BAT ? ga((has_qkv && l + 1 < l1) || has_head) : -1, ti++);
        }
    }
    if (has_head) {
        phase_head<BAT>(ka, gw(), ti++);
    }
}

}  // namespace kl
