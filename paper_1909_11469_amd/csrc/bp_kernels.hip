// HIP kernels of libbp for gfx950 (CDNA4, wave64).
//
// One iteration of Alg. 1 is one launch of an evaluation kernel (plus the top-k
// selection kernels for frontier residual BP).
//
// Evaluation kernel (Eq. (2) + Eq. (4) + frontier rule + commit, fused):
// messages are stored grouped by source node (CSR by source), so slot e holds
// m_{i->k}, the message the thread of slot e recomputes, and the outgoing
// messages of a run of source nodes form one contiguous slot range.  A block
// owns such a tile of nodes:
//   phase 1  coalesced loads of the tile's own slots (old value, reverse index,
//            coupling, target id) and of the incoming messages m_{k->i} at the
//            reverse slots (the one gather per message);
//   phase 2  one thread per node (per node-state for K > 2) sums the incoming
//            logs with the log unary into A_i = log psi_i + sum_k log m_{k->i};
//   phase 3  one thread per slot computes m_{i->k} from the cavity
//            A_i - log m_{k->i} (Eq. (2) excludes exactly that message),
//            normalises it, forms the L-infinity residual against the old value,
//            applies the frontier rule and writes the next buffer at its own
//            slot (coalesced).
// Every slot of the next buffer is written exactly once per iteration, so the
// update is synchronous (Jacobi) with no atomics on message values.
//
// Randomized BP chooses p_t from n_t, which is only known once every block of
// iteration t has counted its residuals.  The kernel therefore writes the
// committed state under both keep thresholds (two output buffers); the next
// launch computes p_t from the finished counters in its prologue and reads the
// matching buffer.  No pass over the messages is needed between iterations.
#include <type_traits>

#include "bp_internal.h"

namespace bp {
namespace {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  The random filter of
// Sec. IV-A for the message i -> j, j the neighbour of rank r of i (slots of a
// source are ordered by target, so r is the slot's offset in the source's
// range), uses word r mod 4 of the output for counter (i, r div 4, t, 0): one
// call serves four messages of one source.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4(unsigned int c0, unsigned int c1, unsigned int c2,
                                         unsigned int k0, unsigned int k1) {
    unsigned int c3 = 0u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // full 64-bit products: one v_mad_u64_u32 each instead of a hi/lo pair
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * c0;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * c2;
        const unsigned int n0 = (unsigned int)(p1 >> 32) ^ c1 ^ k0;
        const unsigned int n2 = (unsigned int)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0;
        c1 = (unsigned int)p1;
        c2 = n2;
        c3 = (unsigned int)p0;
    }
    return make_uint4(c0, c1, c2, c3);
}

// The 24-bit uniform of the message of rank r of source i at iteration t.
__device__ __forceinline__ unsigned int draw24(const EvalArgs& a, int i, int r) {
    const uint4 w = philox4((unsigned int)i, (unsigned int)r >> 2, a.t, a.key0, a.key1);
    const int k = r & 3;
    const unsigned int x = k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
    return x >> 8;
}

// Hardware exp2 / log2 / reciprocal (v_exp_f32, v_log_f32, v_rcp_f32, about 1 ulp)
// where the argument range needs none of the library's fix-ups: exp2 may
// underflow to zero or overflow to +inf, both harmless where it is used below;
// log2 is only taken of values in [1, 2]; rcp only of values in [1, +inf].
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float log2_hw(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float rcp_hw(float x) { return __builtin_amdgcn_rcpf(x); }

// Short forms of logf and expf, for a normal finite x > 0 and for -100 <= x <= 0: the
// same bits without the denormal, infinity and underflow handling (6 and 4 of about
// 12 instructions).  A wave takes the short form or the library's by a vote over its
// lanes (log_batch, exp_batch), and other kernels call the library, so a result that
// does not depend on its neighbours rests on the bits being equal:
// bp_check_short_math compares every float of both ranges.
//
// The steps and the two-float constants are those of the LLVM AMDGPU backend's expansion
// of llvm.log.f32 and llvm.exp.f32 (open source) with contraction.  log x = y ln 2 with
// y = log2 x and ln 2 = hi + lo: e collects y lo and the rounding error of y hi; the
// last step, contracted, multiplies again without rounding, so that error enters
// twice (at most half an ulp).  exp x = 2^(x log2 e): the product as the sum p + q
// of two floats, whose integer part goes to the exponent.
__device__ __forceinline__ float log_normal(float x) {
#pragma clang fp contract(off)
    constexpr float hi = 0x1.62e42ep-1f, lo = 0x1.efa39ep-25f;
    const float y = __builtin_amdgcn_logf(x);
    const float e = fmaf(y, lo, fmaf(y, hi, -(y * hi)));
    return fmaf(y, hi, e);
}
__device__ __forceinline__ float exp_reduced(float x) {
#pragma clang fp contract(off)
    constexpr float hi = 0x1.715476p+0f, lo = 0x1.4ae0bep-26f;
    const float p = x * hi;
    const float q = fmaf(x, lo, fmaf(x, hi, -p));
    const float n = rintf(p);
    return ldexpf(__builtin_amdgcn_exp2f((p - n) + q), (int)n);
}
// log and exp of N values per lane: the short forms when every lane of the wave
// is in their range, else the library's.  exp: every value <= 0 (or NaN).
template <int N>
__device__ __forceinline__ void log_batch(float* v) {
    float mn = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) mn = fminf(mn, v[i]);
    if (__all(mn >= 1.17549435e-38f)) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = log_normal(v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = logf(v[i]);
    }
}
template <int N>
__device__ __forceinline__ void exp_batch(float* v) {
    float mn = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) mn = fminf(mn, v[i]);
    if (__all(mn >= -100.0f)) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = exp_reduced(v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = expf(v[i]);
    }
}

// The floats of each range whose short form differs from the library's: diff[0] log,
// diff[1] exp.
constexpr unsigned int kLogFirst = 0x00800000u, kLogLast = 0x7F7FFFFFu;  // normal, positive
constexpr unsigned int kExpFirst = 0x80000000u, kExpLast = 0xC2C80000u;  // -0 ... -100
__global__ __launch_bounds__(kBlock) void k_check_short_math(unsigned long long* diff) {
    const unsigned int id = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock;
    unsigned int dl = 0, de = 0;
    for (unsigned long long b = kLogFirst + (unsigned long long)id; b <= kLogLast; b += stride) {
        const float x = __uint_as_float((unsigned int)b);
        dl += __float_as_uint(log_normal(x)) != __float_as_uint(logf(x));
    }
    for (unsigned long long b = kExpFirst + (unsigned long long)id; b <= kExpLast; b += stride) {
        const float x = __uint_as_float((unsigned int)b);
        de += __float_as_uint(exp_reduced(x)) != __float_as_uint(expf(x));
    }
    if (id == 0) de += __float_as_uint(exp_reduced(0.0f)) != __float_as_uint(expf(0.0f));
    if (dl) atomicAdd(&diff[0], (unsigned long long)dl);
    if (de) atomicAdd(&diff[1], (unsigned long long)de);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// 1 / (1 + e^{-x}); e^{-x} overflows to +inf for x < -88 and gives 0.
__device__ __forceinline__ float sigmoid_fast(float x) {
    return rcp_hw(1.0f + exp2_hw(-kLog2e * x));
}

// Workgroup barrier for LDS hand-offs only: waits for this wave's LDS
// operations and meets the other waves, without the release/acquire fences of
// __syncthreads(), which would also wait for every outstanding global load
// (the prefetched next tile).  No global memory written in a launch is read
// back by another wave of the same block.
__device__ __forceinline__ void lds_barrier() {
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wave reductions on the vector units: lane 63 collects the wave through DPP row
// shifts and row broadcasts, six dependent instructions instead of six trips
// through the LDS crossbar (ds_bpermute).  A lane without a source adds `id`.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int dpp_or(unsigned int id, unsigned int v) {
    return (unsigned int)__builtin_amdgcn_update_dpp((int)id, (int)v, CTRL, ROWS, 0xF, false);
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
// Sum over the wave, valid in lane 63.
__device__ __forceinline__ unsigned int dpp_sum_last(unsigned int v) {
    v += dpp_or<kRowShr1, 0xF>(0u, v);
    v += dpp_or<kRowShr2, 0xF>(0u, v);
    v += dpp_or<kRowShr4, 0xF>(0u, v);
    v += dpp_or<kRowShr8, 0xF>(0u, v);
    v += dpp_or<kRowBcast15, 0xA>(0u, v);
    v += dpp_or<kRowBcast31, 0xC>(0u, v);
    return v;
}
__device__ __forceinline__ unsigned int dpp_max_last(unsigned int v) {
    v = max(v, dpp_or<kRowShr1, 0xF>(0u, v));
    v = max(v, dpp_or<kRowShr2, 0xF>(0u, v));
    v = max(v, dpp_or<kRowShr4, 0xF>(0u, v));
    v = max(v, dpp_or<kRowShr8, 0xF>(0u, v));
    v = max(v, dpp_or<kRowBcast15, 0xA>(0u, v));
    v = max(v, dpp_or<kRowBcast31, 0xC>(0u, v));
    return v;
}
// The same, in every lane (a scalar).
__device__ __forceinline__ unsigned int wave_sum32(unsigned int v) {
    return (unsigned int)__builtin_amdgcn_readlane((int)dpp_sum_last(v), 63);
}
__device__ __forceinline__ unsigned int wave_max32(unsigned int v) {
    return (unsigned int)__builtin_amdgcn_readlane((int)dpp_max_last(v), 63);
}

struct RedScratch {
    float rmax[kBlock / 64];
    unsigned int act[kBlock / 64];
    unsigned int sa[kBlock / 64];
    unsigned int sb[kBlock / 64];
};

// Block-wide reduction of the per-thread residual max and counts, then one
// atomic per quantity per block into the block's counter copy (integer adds and
// an ordered max on the FP32 bit pattern of a non-negative float: both order
// independent, so the totals are deterministic).
__device__ __forceinline__ void block_accumulate(RedScratch* red, CounterLine* ctr, unsigned int t,
                                                 float rmax, unsigned int act, unsigned int sa,
                                                 unsigned int sb) {
    // (residuals are non-negative, so their bit patterns order as integers)
    const unsigned int rm = dpp_max_last(__float_as_uint(rmax));
    act = dpp_sum_last(act);
    sa = dpp_sum_last(sa);
    sb = dpp_sum_last(sb);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) {
        red->rmax[w] = __uint_as_float(rm);
        red->act[w] = act;
        red->sa[w] = sa;
        red->sb[w] = sb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = red->rmax[0];
        unsigned int A = red->act[0], SA = red->sa[0], SB = red->sb[0];
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
            r = fmaxf(r, red->rmax[i]);
            A += red->act[i];
            SA += red->sa[i];
            SB += red->sb[i];
        }
        CounterLine* c = ctr + (t & 3u) * kCounterCopies + (blockIdx.x & (kCounterCopies - 1));
        if (A) atomicAdd(&c->active, (unsigned long long)A);
        if (SA) atomicAdd(&c->sel_a, (unsigned long long)SA);
        if (SB) atomicAdd(&c->sel_b, (unsigned long long)SB);
        if (r > 0.0f) atomicMax(&c->rmax, __float_as_uint(r));
    }
}

__device__ __forceinline__ int tile_of_block(const EvalArgs& a) {
    // Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous
    // range of tiles so neighbouring tiles share that XCD's L2.
    const int b = blockIdx.x;
    return (b & 7) * a.tiles_per_xcd + (b >> 3);
}

// Which of the two committed outcomes iteration t - 1 kept: p_{t-1} is the low
// setting when EdgeRatio = n_{t-1} / n_{t-2} exceeds the threshold (Sec. IV-A).
__device__ __forceinline__ int select_outcome(const EvalArgs& a, unsigned long long n1, long long n2) {
    if (a.sched != kModeRnBP || !a.two_outputs) return 0;
    const bool p_low = !a.dynamic_p || (n2 > 0 && ((double)n1 / (double)n2 > a.ratio_threshold));
    return (p_low == (a.low_is_a != 0)) ? 0 : 1;
}

// Tell the host how many evaluations of the run are closed and whether the last of
// them converged: one word of pinned memory, so that the host can follow the run
// (and stop launching) without a readback that leaves the device idle.  The store
// crosses the bus while the block waits for it (about 2 us of its launch), so only
// every kReportEvery-th count is reported, and convergence at once.
__device__ __forceinline__ void report_progress(const EvalArgs& a, unsigned long long closed,
                                                bool converged) {
    if (a.prog && (converged || closed % kReportEvery == 0))
        __hip_atomic_store(a.prog, closed << 1 | (converged ? 1ull : 0ull), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// The counter lines the prologue needs, loaded by the 64 lanes of one wave
// (lane c reads copy c): n of iterations t - 1 and t - 2, and for the block that
// closes iteration t - 1 also its frontier sizes and max residual.
struct CtrLoad {
    unsigned int n1, n2, sa, sb, rm, done;
};

__device__ __forceinline__ void ctr_load(const EvalArgs& a, bool lead, CtrLoad& c) {
    const int lane = threadIdx.x & 63;
    const CounterLine* c1 = a.ctr + ((a.t - 1u) & 3u) * kCounterCopies + lane;
    c.done = a.st->done;
    c.n1 = (unsigned int)c1->active;
    c.n2 = a.it >= 2 ? (unsigned int)a.ctr[((a.t - 2u) & 3u) * kCounterCopies + lane].active : 0u;
    c.sa = lead ? (unsigned int)c1->sel_a : 0u;
    c.sb = lead ? (unsigned int)c1->sel_b : 0u;
    c.rm = lead ? c1->rmax : 0u;
}

// Run by the 64 lanes of one wave after ctr_load: sum the counter copies of
// iteration t - 1 (and t - 2), and, when `close` is set, record iteration
// t - 1 (IsConverged, statistics, the buffer p_{t-1} selects) and clear the
// copies of t + 1.  The statistics are updated with stores and no-return
// atomics, so nothing waits.  Returns n_{t-1} and n_{t-2} (the host's value
// when t - 2 precedes the run).
__device__ __forceinline__ void wave_close(const EvalArgs& a, bool close, const CtrLoad& c,
                           unsigned long long& n1_out, long long& n2_out) {
    const int lane = threadIdx.x & 63;
    // (counts of a launch are at most the number of messages, below 2^31)
    const unsigned long long n1 = wave_sum32(c.n1);
    const unsigned long long n2 = wave_sum32(c.n2);
    const long long n2s = a.it >= 2 ? (long long)n2 : a.prev_active_host;
    n1_out = n1;
    n2_out = n2s;
    if (!close) return;
    const unsigned long long sa = wave_sum32(c.sa);
    const unsigned long long sb = wave_sum32(c.sb);
    const unsigned int rm = wave_max32(c.rm);
    CounterLine* z = a.ctr + ((a.t + 1u) & 3u) * kCounterCopies + lane;
    z->active = 0ull;
    z->sel_a = 0ull;
    z->sel_b = 0ull;
    z->rmax = 0u;
    if (lane != 0) return;
    DevState* st = a.st;
    report_progress(a, (unsigned long long)a.it, n1 == 0ull);
    const unsigned int tp = a.t - 1u;
    const int sel = select_outcome(a, n1, n2s);
    atomicAdd(&st->evaluated, a.num_messages);
    atomicAdd(&st->evals, 1ull);
    st->last_t = (long long)tp;
    st->last_active = n1;
    st->last_rmax = rm;
    st->last_prev = n2s;
    if (n1 == 0ull) {
        st->done = 1u;
        st->conv_t = (long long)tp;
    } else if (!a.after_final) {
        unsigned long long cm;
        if (a.sched == kModeLBP)
            cm = a.num_messages;
        else if (a.sched == kModeRBP)
            cm = a.rbp_k;
        else if (a.sched == kModeRS)
            cm = 0ull;  // the splash kernels count their commits
        else
            cm = sel ? sb : sa;
        if (cm) atomicAdd(&st->committed, cm);
        atomicAdd(&st->iterations, 1ull);
        st->in_sel[a.t & 3u] = (unsigned int)sel;
    }
}

// Start of iteration t, in two parts so that a kernel can issue other loads
// between them: prologue_issue loads the counters (wave 0), prologue_finish
// (all threads of the block) returns the buffer holding m^t, or nullptr when
// an earlier evaluation found no residual above eps (the block then exits).
// The previous launch wrote the outcome under both keep thresholds, so
// choosing p_{t-1} is choosing a buffer.  The lead block (one per graph and
// launch) also closes iteration t - 1.
__device__ __forceinline__ void prologue_issue(const EvalArgs& a, CtrLoad& c, bool lead) {
    if (a.it != 0 && threadIdx.x < 64) ctr_load(a, lead, c);
}

// VALUES: both buffers are read and one taken, not an indexed one read, so that a local
// copy of the arguments (the batched launch's) stays in registers.  The other kernels
// index their kernel arguments: with VALUES the K = 2 kernel waits for its prefetched
// loads earlier (2000 x 2000 LBP, 30 sweeps: 2,459 us; 1,931 indexed).
template <bool VALUES = false>
__device__ __forceinline__ const float* prologue_finish(const EvalArgs& a, const CtrLoad& c,
                                                        unsigned long long* s_red,
                                                        bool lead) {
    const float* const buf0 = VALUES ? a.in_buf[0] : nullptr;
    const float* const buf1 = VALUES ? a.in_buf[1] : nullptr;
    if (a.it == 0) {
        if (lead && threadIdx.x < 64) {
            CounterLine* z = a.ctr + ((a.t + 1u) & 3u) * kCounterCopies + threadIdx.x;
            z->active = 0ull;
            z->sel_a = 0ull;
            z->sel_b = 0ull;
            z->rmax = 0u;
            if (threadIdx.x == 0) a.st->in_sel[a.t & 3u] = (unsigned int)a.sel0;
        }
        return a.in_buf[0];
    }
    if (threadIdx.x < 64) {
        unsigned long long n1;
        long long n2;
        wave_close(a, lead && !c.done, c, n1, n2);
        if (threadIdx.x == 0) {
            s_red[0] = c.done ? 0ull : n1;
            s_red[1] = (unsigned long long)n2;
        }
    }
    lds_barrier();
    const unsigned long long n1 = s_red[0];
    if (n1 == 0ull) return nullptr;
    const int sel = select_outcome(a, n1, (long long)s_red[1]);
    if (VALUES) return sel ? buf1 : buf0;
    return a.in_buf[sel];
}

template <bool VALUES = false>
__device__ __forceinline__ const float* iteration_prologue(const EvalArgs& a,
                                                           unsigned long long* s_red, bool lead) {
    CtrLoad c;
    prologue_issue(a, c, lead);
    return prologue_finish<VALUES>(a, c, s_red, lead);
}

// ---------------------------------------------------------------------------
// K = 2 Ising, one log-odds value per message: lambda = log(m(1) / m(0)).
// Aggregate L_i = u_i + sum_k lambda_{k->i} with u_i = log psi_i(1) - log psi_i(0).
// With H = (L_i - lambda_{k->i}) / 2 the outgoing message of Eq. (2) for
// psi = exp(J s_i s_k) has log-odds log cosh(J + H) - log cosh(J - H) (the sum
// over x_i in closed form; normalisation included).
// The slot e of m_{i->k} gives e as the output index, its own old value, and
// lambda_{k->i} at rev[e].
// ---------------------------------------------------------------------------
// log(1 + e^{-2|x|}), in (0, log 2]: log2 is taken of a value in (1, 2].
__device__ __forceinline__ float logcosh_tail(float x) {
    return kLn2 * log2_hw(1.0f + exp2_hw(-2.0f * kLog2e * fabsf(x)));
}

// Array access with a 32-bit byte offset from a wave-uniform base: the
// compiler emits the global_load/store form that adds a 32-bit VGPR offset to a
// 64-bit SGPR base, so per-lane accesses need no 64-bit address arithmetic.
// Every array the K = 2 kernel touches holds fewer than 2^30 four-byte elements
// (checked at graph creation).
template <class T>
__device__ __forceinline__ T ld32(const T* base, int i) {
    return *(const T*)((const char*)base + (unsigned int)i * 4u);
}
template <class T>
__device__ __forceinline__ void st32(T* base, int i, T v) {
    *(T*)((char*)base + (unsigned int)i * 4u) = v;
}
// A pointer the compiler cannot prove uniform (chosen from LDS data), made uniform.
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)v);
    const unsigned int hi = __builtin_amdgcn_readfirstlane((unsigned int)(v >> 32));
    return (T*)(((unsigned long long)hi << 32) | lo);
}

// Where one slot's results go: plain pointers, or buffer resources.
struct OutPtr {
    const EvalArgs& a;
    __device__ void out0(int e, float v) const { a.out_buf[0][e] = v; }
    __device__ void out1(int e, float v) const { a.out_buf[1][e] = v; }
    __device__ void cand(int e, float v) const { a.cand[e] = v; }
    __device__ void key(int e, float r) const { a.keys[e] = __float_as_uint(r); }
};
struct OutOff {
    float* o0;
    float* o1;
    float* c;
    unsigned int* k;
    __device__ void out0(int e, float v) const { st32(o0, e, v); }
    __device__ void out1(int e, float v) const { st32(o1, e, v); }
    __device__ void cand(int e, float v) const { st32(c, e, v); }
    __device__ void key(int e, float r) const { st32(k, e, __float_as_uint(r)); }
};

// Eq. (2), Eq. (4) and the frontier rule for one slot; returns the residual.
// log cosh(J + H) - log cosh(J - H) is evaluated as
// 2 sgn(J H) min(|J|, |H|) + tail(J + H) - tail(J - H): the identity
// |J + H| - |J - H| = 2 sgn(J H) min(|J|, |H|) keeps it exact in the leading term
// for any finite J and H (no cancellation of two large magnitudes, no overflow),
// and the tails are bounded by log 2.
__device__ __forceinline__ float logodds_update(float L, float lam_in, float J) {
    const float H = 0.5f * (L - lam_in);
    const float lead = copysignf(2.0f * fminf(fabsf(J), fabsf(H)), J * H);
    return lead + logcosh_tail(J + H) - logcosh_tail(J - H);
}

template <int MODE, class Out>
__device__ __forceinline__ float logodds_slot(const EvalArgs& a, const Out& out, float L,
                                              float lam_in, float J, float lam_old, int e,
                                              unsigned int u24, unsigned int& act,
                                              unsigned int& sa, unsigned int& sb) {
    const float lam_new = logodds_update(L, lam_in, J);
    const float r = fabsf(sigmoid_fast(lam_new) - sigmoid_fast(lam_old));
    const bool active = r > a.eps;
    act += active;
    if (MODE == kModeLBP) {
        out.out0(e, lam_new);
    } else if (MODE == kModeRnBP) {
        bool ka = false, kb = false;
        if (active) {
            ka = u24 < a.thr_a;
            kb = u24 < a.thr_b;
        }
        sa += ka;
        sb += kb;
        out.out0(e, ka ? lam_new : lam_old);
        if (a.two_outputs) out.out1(e, kb ? lam_new : lam_old);
    } else if (MODE == kModeRBP) {
        out.cand(e, lam_new);
        out.key(e, r);
    }
    return r;
}

constexpr int kPP = kTileSlotsLogOdds / kBlockLO;              // slots per thread per tile
constexpr int kPJ = (kTileNodesLogOdds + kBlockLO) / kBlockLO;    // node entries (TN + 1) per thread

// The per-thread share of one tile: node bounds and unaries, and the slots'
// own old values, reverse indices and couplings.
struct TileRegs {
    int n0, nn, s0, ns;
    int ptr[kPJ];
    float u[kPJ];
    float old[kPP];
    int rev[kPP];
    float J[kPP];
};

// Issue every load of a tile (indices clamped into the tile, so there is no
// per-lane branch and the loads are not ordered behind one another): the graph
// constants, then the tile's own old messages.  R16: the reverse slots are
// read as 16-bit offsets from the slot (EvalArgs.rev16).
template <class T>
__device__ __forceinline__ T ld16(const T* base, int i) {
    return *(const T*)((const char*)base + (unsigned int)i * 2u);
}
template <int MODE, bool R16 = false>
__device__ __forceinline__ void tile_load_const(TileRegs& d, const EvalArgs& a, int4 b) {
    const int tid = threadIdx.x;
    d.n0 = b.x;
    d.nn = b.y - b.x;
    d.s0 = b.z;
    d.ns = b.w - b.z;
#pragma unroll
    for (int j = 0; j < kPJ; ++j) {
        const int v = tid + j * kBlockLO;
        d.ptr[j] = ld32(a.node_ptr, d.n0 + min(v, d.nn));
        d.u[j] = ld32(a.unary, d.n0 + min(v, max(d.nn - 1, 0)));
    }
    // a tile without slots reads slot 0 (its own s0 may be one past the last
    // slot, and what lies there is no slot to gather from)
#pragma unroll
    for (int k = 0; k < kPP; ++k) {
        const int s = d.ns > 0 ? d.s0 + min(tid + k * kBlockLO, d.ns - 1) : 0;
        d.rev[k] = R16 ? s + (int)ld16(a.rev16, s) : ld32(a.rev, s);
        d.J[k] = ld32(a.coupling, s);
    }
}

__device__ __forceinline__ void tile_load_msgs(TileRegs& d, const float* m_in) {
#pragma unroll
    for (int k = 0; k < kPP; ++k)
        d.old[k] = ld32(m_in, d.ns > 0 ? d.s0 + min((int)threadIdx.x + k * kBlockLO, d.ns - 1) : 0);
}

template <int MODE, bool R16 = false>
__device__ __forceinline__ void tile_load(TileRegs& d, const EvalArgs& a, const float* m_in,
                                          int4 b) {
    tile_load_const<MODE, R16>(d, a, b);
    tile_load_msgs(d, m_in);
}

// Tile w + j * W of this block's XCD range (tiles are dealt to XCDs in
// contiguous ranges so that neighbouring tiles share an L2), or -1.
__device__ __forceinline__ int block_tile(const EvalArgs& a, int j) {
    const int w = (int)(blockIdx.x >> 3) + j * (int)(gridDim.x >> 3);
    if (w >= a.tiles_per_xcd) return -1;
    const int t = (int)(blockIdx.x & 7) * a.tiles_per_xcd + w;
    return t < a.num_tiles ? t : -1;
}

// Add 1 to LDS bin `bin` for every lane with `on`.  Residual keys share
// their leading digits, so most lanes of a wave hit one bin: the lanes whose
// bin equals the first active lane's are counted by a ballot and one atomic,
// the rest add individually.
__device__ __forceinline__ void lds_count(unsigned int* h, unsigned int bin, bool on) {
    const unsigned long long act = __ballot(on);
    if (!act) return;
    const int lead = __ffsll((long long)act) - 1;
    const unsigned int lb = (unsigned int)__shfl((int)bin, lead, 64);
    const bool same = on && bin == lb;
    const unsigned long long sm = __ballot(same);
    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&h[lb], (unsigned int)__popcll(sm));
    if (on && !same) atomicAdd(&h[bin], 1u);
}

// LDS of the K = 2 tile loop.
struct LogoddsLds {
    float lam[kTileSlotsLogOdds];
    unsigned short owner[kTileSlotsLogOdds];
    unsigned int u[kTileSlotsLogOdds];  // 24-bit uniforms of the slots (RnBP)
    unsigned short ptr[kTileNodesLogOdds + 1];
    float L[kTileNodesLogOdds];
    unsigned int hist[256];             // frontier RBP: first radix digit of the keys
};

// The software-pipelined tile loop of the K = 2 kernel over a sequence of
// tiles (seq.valid(j), seq.bounds(j)): while tile j is computed, the loads of
// tile j + 1 are in flight, so the math of Eq. (2), the residual and the random
// filter overlap the memory traffic instead of following it.  `cur` holds the
// graph constants of tile 0 (issued by the caller); iteration j issues the
// loads of tile j + 1, aggregates tile j (LDS), issues the gathers of tile
// j + 1, computes and stores tile j, then stages tile j + 1 into LDS, so every
// wait falls on loads that had a whole phase to complete.
template <int MODE, class Seq, bool R16 = false>
__device__ __forceinline__ void logodds_tile_loop(const EvalArgs& a, const float* __restrict__ m_in,
                                                  const Seq& seq, TileRegs& cur, int4 bnext,
                                                  LogoddsLds& l, float& rmax, unsigned int& act,
                                                  unsigned int& sa, unsigned int& sb) {
    const OutOff out{a.out_buf[0], a.out_buf[1], a.cand, a.keys};
    const int tid = threadIdx.x;
    TileRegs nxt;
    float lin[kPP];
    tile_load_msgs(cur, m_in);
#pragma unroll
    for (int k = 0; k < kPP; ++k) lin[k] = ld32(m_in, cur.rev[k]);
    // stage tile 0
#pragma unroll
    for (int jj = 0; jj < kPJ; ++jj) {
        const int v = tid + jj * kBlockLO;
        if (v <= cur.nn) l.ptr[v] = (unsigned short)(cur.ptr[jj] - cur.s0);
        if (v < cur.nn) l.L[v] = cur.u[jj];
    }
#pragma unroll
    for (int k = 0; k < kPP; ++k) {
        const int q = tid + k * kBlockLO;
        if (q < cur.ns) l.lam[q] = lin[k];
    }
    for (int j = 0;; ++j) {
        const bool has_next = seq.valid(j + 1);
        const int4 bnext2 = seq.valid(j + 2) ? seq.bounds(j + 2) : make_int4(0, 0, 0, 0);
        if (has_next) tile_load<MODE, R16>(nxt, a, m_in, bnext);
        lds_barrier();
        // node aggregates of tile j, incoming messages in slot order; for
        // RnBP also the draws of the node's messages, four per Philox call
        for (int v = tid; v < cur.nn; v += kBlockLO) {
            const int q0 = l.ptr[v], q1 = l.ptr[v + 1];
            float L = l.L[v];
            for (int q = q0; q < q1; ++q) {
                L += l.lam[q];
                l.owner[q] = (unsigned short)v;
            }
            l.L[v] = L;
            if (MODE == kModeRnBP) {
                for (int q = q0; q < q1; q += 4) {
                    const uint4 w = philox4((unsigned int)(cur.n0 + v), (unsigned int)(q - q0) >> 2,
                                            a.t, a.key0, a.key1);
                    l.u[q] = w.x >> 8;
                    if (q + 1 < q1) l.u[q + 1] = w.y >> 8;
                    if (q + 2 < q1) l.u[q + 2] = w.z >> 8;
                    if (q + 3 < q1) l.u[q + 3] = w.w >> 8;
                }
            }
        }
        lds_barrier();
        float lin_n[kPP];
        if (has_next) {
#pragma unroll
            for (int k = 0; k < kPP; ++k) lin_n[k] = ld32(m_in, nxt.rev[k]);
        }
        // outgoing messages of tile j, written at their own slots
#pragma unroll
        for (int k = 0; k < kPP; ++k) {
            const int q = tid + k * kBlockLO;
            float r = 0.0f;
            if (q < cur.ns) {
                const int v = l.owner[q];
                const unsigned int u24 = MODE == kModeRnBP ? l.u[q] : 0u;
                r = logodds_slot<MODE>(a, out, l.L[v], lin[k], cur.J[k], cur.old[k],
                                       cur.s0 + q, u24, act, sa, sb);
                rmax = fmaxf(rmax, r);
            }
            // frontier RBP: the first radix digit of the key (top 8 bits)
            if (MODE == kModeRBP && a.hist0) lds_count(l.hist, __float_as_uint(r) >> 24, q < cur.ns);
        }
        if (!has_next) break;
        lds_barrier();  // tile j's LDS reads are done
        cur = nxt;
#pragma unroll
        for (int k = 0; k < kPP; ++k) lin[k] = lin_n[k];
#pragma unroll
        for (int jj = 0; jj < kPJ; ++jj) {
            const int v = tid + jj * kBlockLO;
            if (v <= cur.nn) l.ptr[v] = (unsigned short)(cur.ptr[jj] - cur.s0);
            if (v < cur.nn) l.L[v] = cur.u[jj];
        }
#pragma unroll
        for (int k = 0; k < kPP; ++k) {
            const int q = tid + k * kBlockLO;
            if (q < cur.ns) l.lam[q] = lin[k];
        }
        bnext = bnext2;
    }
}

// The tiles of this block's XCD range (tiles are dealt to XCDs in contiguous
// ranges so that neighbouring tiles share an L2).
struct XcdTiles {
    const EvalArgs& a;
    const int4* tiles;
    __device__ bool valid(int j) const { return block_tile(a, j) >= 0; }
    __device__ int4 bounds(int j) const { return tiles[block_tile(a, j)]; }
};

// K = 2 evaluation kernel.  A persistent grid (as many blocks as are resident)
// walks the tiles with the pipelined tile loop.
template <int MODE, bool R16>
__global__ __launch_bounds__(kBlockLO) void k_eval_logodds(EvalArgs a) {
    __shared__ LogoddsLds l;
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];

    const int4* __restrict__ tiles = (const int4*)a.tiles4;
    const int t0 = block_tile(a, 0), t1 = block_tile(a, 1);
    // a block without tiles loads tile 0 and computes nothing, so that the
    // first loads are unconditional
    int4 bcur = tiles[t0 >= 0 ? t0 : 0];
    int4 bnext = t1 >= 0 ? tiles[t1] : make_int4(0, 0, 0, 0);
    // the counters are loaded first and the first tile's graph constants next,
    // so that the two latencies overlap (loads complete in issue order)
    CtrLoad cl;
    prologue_issue(a, cl, blockIdx.x == 0);
    TileRegs cur;
    tile_load_const<MODE, R16>(cur, a, bcur);
    __builtin_amdgcn_sched_barrier(0);
    const float* m_sel = prologue_finish(a, cl, s_red, blockIdx.x == 0);
    if (!m_sel) return;
    const float* __restrict__ m_in = uniform_ptr(m_sel);
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    const bool hist = MODE == kModeRBP && a.hist0;
    if (hist)
        for (int i = threadIdx.x; i < 256; i += kBlockLO) l.hist[i] = 0u;  // seen after the loop's barriers
    if (t0 >= 0)
        logodds_tile_loop<MODE, XcdTiles, R16>(a, m_in, XcdTiles{a, tiles}, cur, bnext, l, rmax, act,
                                              sa, sb);
    if (hist) {
        // the block's digit counts into one of the copies of the global histogram
        lds_barrier();
        unsigned int* gh = a.st->hist[0][blockIdx.x & (kHistCopies - 1)];
        for (int i = threadIdx.x; i < 256; i += kBlockLO)
            if (l.hist[i]) atomicAdd(&gh[i], l.hist[i]);
    }
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// A node whose degree exceeds a tile: one block, aggregate by a block
// reduction of the gathered incoming messages, then stream the slots.
template <int MODE>
__device__ __forceinline__ void logodds_big_node(const EvalArgs& a, const float* __restrict__ m_in,
                                                 int4 b, float* s_part, float& rmax,
                                                 unsigned int& act, unsigned int& sa,
                                                 unsigned int& sb) {
    const int tid = threadIdx.x;
    const int n0 = b.x, s0 = b.z, ns = b.w - b.z;
    float part = 0.0f;
    const int nt = (int)blockDim.x;
    for (int q = tid; q < ns; q += nt) part += m_in[a.rev[s0 + q]];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if ((tid & 63) == 0) s_part[tid >> 6] = part;
    __syncthreads();
    float L = a.unary[n0];
#pragma unroll
    for (int i = 0; i < nt / 64; ++i) L += s_part[i];
    for (int q = tid; q < ns; q += nt) {
        const int s = s0 + q;
        const unsigned int u24 = MODE == kModeRnBP ? draw24(a, n0, q) : 0u;
        const float r = logodds_slot<MODE>(a, OutPtr{a}, L, m_in[a.rev[s]], a.coupling[s], m_in[s], s,
                                           u24, act, sa, sb);
        rmax = fmaxf(rmax, r);
    }
}

// Nodes whose degree exceeds a tile, one block each.  Runs after k_eval_logodds
// in the same iteration (same prologue, no bookkeeping).
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_eval_logodds_big(EvalArgs a) {
    __shared__ RedScratch red;
    __shared__ float s_part[kBlock / 64];
    __shared__ unsigned long long s_red[2];
    const int4 b = ((const int4*)a.big4)[blockIdx.x];
    const float* __restrict__ m_in = iteration_prologue(a, s_red, false);
    if (!m_in) return;
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    logodds_big_node<MODE>(a, m_in, b, s_part, rmax, act, sa, sb);
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// ---------------------------------------------------------------------------
// Batched evaluation for serving: one launch evaluates one iteration of every
// graph of a batch.  The graph's arguments live in device memory and its
// iteration number is the launch index minus the launch of its first
// evaluation, so graphs admitted at different times advance independently,
// each exactly as bp_run would advance it alone (same tiles, same per-slot
// arithmetic, per-graph counters and random keys).  The launch index is a
// device counter (BatchCtl), so a sequence of launches can be recorded once in
// a HIP graph and replayed.
//
// The grid is persistent: block b takes a contiguous range of the tile list
// (entries of one graph are contiguous, regular tiles first), splits it into
// runs of one graph, and runs each graph's regular tiles through the same
// software-pipelined tile loop as bp_run's kernel, then its oversized nodes.
// ---------------------------------------------------------------------------

// The arguments of graph G for the launch with index `launch`: its per-launch fields
// as bp_run sets them for its iteration it = launch - G.first.  (A kernel of its own
// that stored them before every launch took 4.7 us of the launch's 32.)
__device__ __forceinline__ EvalArgs batch_args(const BatchGraph& G, long long it) {
    EvalArgs a = G.a;
    a.it = it;
    a.t = (unsigned int)it;
    a.after_final = 0;
    a.prog = nullptr;
    const int pin = (int)(it & 1);
    a.in_buf[0] = it == 0 ? G.msg[0] : G.msg[2 * pin];
    a.in_buf[1] = it == 0 ? G.msg[0] : G.msg[2 * pin + 1];
    a.out_buf[0] = G.msg[2 * (pin ^ 1)];
    a.out_buf[1] = G.msg[2 * (pin ^ 1) + 1];
    return a;
}

// The regular tiles of one graph's run of list entries.
struct ListTiles {
    const int4* tiles;
    const int4* list;
    int e0, n;
    __device__ bool valid(int j) const { return j < n; }
    __device__ int4 bounds(int j) const { return tiles[list[e0 + j].y]; }
};

template <int MODE>
__device__ __forceinline__ void batch_run(const EvalArgs& a, const float* __restrict__ m_in,
                                          const int4* __restrict__ list, int e0, int nreg, int e1,
                                          LogoddsLds& l, float* s_part, float& rmax,
                                          unsigned int& act, unsigned int& sa, unsigned int& sb) {
    if (nreg > 0) {
        const ListTiles seq{(const int4*)a.tiles4, list, e0, nreg};
        TileRegs cur;
        tile_load_const<MODE>(cur, a, seq.bounds(0));
        const int4 bnext = nreg > 1 ? seq.bounds(1) : make_int4(0, 0, 0, 0);
        logodds_tile_loop<MODE>(a, m_in, seq, cur, bnext, l, rmax, act, sa, sb);
    }
    for (int e = e0 + nreg; e < e1; ++e) {
        const int4 b = ((const int4*)a.big4)[list[e].y];
        logodds_big_node<MODE>(a, m_in, b, s_part, rmax, act, sa, sb);
    }
}

__global__ __launch_bounds__(kBlockLO) void k_eval_batch(const BatchGraph* __restrict__ graphs,
                                                       const int4* __restrict__ list,
                                                       const BatchCtl* __restrict__ ctl,
                                                       int step) {
    __shared__ LogoddsLds l;
    __shared__ float s_part[kBlock / 64];
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    // `step`: the launch's number among those since the counter last advanced
    const long long launch = ctl->launch + step;
    const int n = ctl->entries;
    const int per = (n + (int)gridDim.x - 1) / (int)gridDim.x;
    int e = (int)blockIdx.x * per;
    const int e_end = min(n, e + per);
    while (e < e_end) {
        const int4 ent = list[e];  // {graph slot, tile, oversized node?, 0}
        int f = e + 1;
        while (f < e_end && list[f].x == ent.x) ++f;
        int r1 = e;
        while (r1 < f && list[r1].z == 0) ++r1;
        // (uniform, so that the graph's arguments are scalar loads)
        const BatchGraph& G = graphs[__builtin_amdgcn_readfirstlane(ent.x)];
        const long long it = launch - G.first, last = G.max_iters;
        if (it >= 0 && it <= last) {  // admitted and not finished
            const EvalArgs a = batch_args(G, it);
            // the block holding the graph's first tile closes its previous iteration
            // (requesting the first tile's constants ahead of the counters took 24 more
            // registers and no time off)
            const float* m_sel = iteration_prologue<true>(a, s_red, ent.z == 0 && ent.y == 0);
            if (m_sel) {
                const float* __restrict__ m_in = uniform_ptr(m_sel);
                float rmax = 0.0f;
                unsigned int act = 0, sa = 0, sb = 0;
                const int mode = it == last ? kModeEvalOnly : G.mode;
                if (mode == kModeLBP)
                    batch_run<kModeLBP>(a, m_in, list, e, r1 - e, f, l, s_part, rmax, act, sa, sb);
                else if (mode == kModeRnBP)
                    batch_run<kModeRnBP>(a, m_in, list, e, r1 - e, f, l, s_part, rmax, act, sa, sb);
                else
                    batch_run<kModeEvalOnly>(a, m_in, list, e, r1 - e, f, l, s_part, rmax, act,
                                             sa, sb);
                block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
            }
        }
        lds_barrier();  // the run's LDS (and s_red) is free for the next run
        e = f;
    }
}

// ---------------------------------------------------------------------------
// Generic layout: [E][K] normalised FP32 probabilities, K <= KP.
// ---------------------------------------------------------------------------
// Lanes of one group of R = 2 or 4 consecutive lanes (R aligned) exchanging
// values with DPP quad permutations (no LDS).
__device__ __forceinline__ float dpp_xor1(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ float dpp_xor2(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));
}
__device__ __forceinline__ float dpp_xor3(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x1B, 0xF, 0xF, false));
}
template <int R>
__device__ __forceinline__ float group_max(float v) {
    v = fmaxf(v, dpp_xor1(v));
    if (R == 4) v = fmaxf(v, dpp_xor2(v));
    return v;
}
// Sum over the group in a fixed order (part 0 + part 1 [+ part 2 + part 3]),
// the same in every lane of the group.
template <int R>
__device__ __forceinline__ float group_sum(float v, int h) {
    if (R == 2) {
        const float o = dpp_xor1(v);
        return h == 0 ? v + o : o + v;
    }
    const float o1 = dpp_xor1(v), o2 = dpp_xor2(v), o3 = dpp_xor3(v);
    float p[4];
    p[0] = h == 0 ? v : h == 1 ? o1 : h == 2 ? o2 : o3;
    p[1] = h == 1 ? v : h == 0 ? o1 : h == 3 ? o2 : o3;
    p[2] = h == 2 ? v : h == 3 ? o1 : h == 0 ? o2 : o3;
    p[3] = h == 3 ? v : h == 2 ? o1 : h == 1 ? o2 : o3;
    return (p[0] + p[1]) + (p[2] + p[3]);
}
// Lane pp of each group, read by every lane of the group (DPP quad_perm
// broadcast; for R = 2 the quad holds two groups).
template <int R, int PP>
__device__ __forceinline__ float group_bcast(float v) {
    constexpr int sel = R == 4 ? PP * 0x55 : (PP | PP << 2 | (2 + PP) << 4 | (2 + PP) << 6);
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), sel, 0xF, 0xF, false));
}
template <int R>
__device__ __forceinline__ float group_bcast(float v, int pp) {
    return pp == 0 ? group_bcast<R, 0>(v)
                   : pp == 1 ? group_bcast<R, 1>(v)
                             : pp == 2 ? group_bcast<R, 2 % R>(v) : group_bcast<R, 3 % R>(v);
}

// Outcome flags of [E][K] rows (EvalArgs.row_flags).  A launch under dynamic p
// writes whole rows of one outcome (the one its prologue chose for the previous
// iteration: a prediction) and the other outcome's row only where the two keep
// decisions differ, marked by the sign bit of the whole row's first entry
// (messages are non-negative).  The next launch reads whole rows from `p` (the
// buffer of the predicted outcome); if it chose the other outcome, flagged rows
// come from `alt`.  `on` is 0 for rows written without flags.
struct FlagRows {
    const float* p;
    const float* alt;   // nullptr: the prediction held
    int on;
};

// Entry x of the row starting at `row` (x == 0 loses the flag bit).
__device__ __forceinline__ float flag_entry(const FlagRows& f, long long row, int x) {
    float v = f.p[row + x];
    if (f.on) {
        if (f.alt && (__float_as_uint(f.p[row]) >> 31)) v = f.alt[row + x];
        if (x == 0) v = fabsf(v);
    }
    return v;
}

// Where a launch writes: whole rows of outcome `prim`, the other outcome's
// rows where the decisions differ.  (In this layout two outcomes always come with
// flags: a launch without them has one.)
__device__ __forceinline__ float flag_first(float v, bool diff) {
    return diff ? __uint_as_float(__float_as_uint(v) | 0x80000000u) : v;
}

// The input rows of a launch and the outcome its own rows are written for:
// sel = the outcome its prologue chose (m_sel = in_buf[sel]); with flags the
// previous launch wrote whole rows of outcome in_sel[t - 1].
__device__ __forceinline__ FlagRows flag_inputs(const EvalArgs& a, const float* m_sel,
                                                int& p_out) {
    const int sel = (a.it >= 1 && m_sel == a.in_buf[1]) ? 1 : 0;
    p_out = a.it == 0 ? a.sel0 : sel;
    FlagRows f{m_sel, nullptr, 0};
    if (a.row_flags && a.it >= 1) {
        const int p_in = (int)a.st->in_sel[(a.t - 1u) & 3u];
        f.p = a.in_buf[p_in];
        f.alt = p_in != sel ? a.in_buf[p_in ^ 1] : nullptr;
        f.on = 1;
    }
    return f;
}

// Eq. (2) for one slot split over a group of R lanes (KP = K states, each lane
// owns KR = K / R of them): the lane computes its part of the cavity
// distribution g, and each lane forms its KR outputs c(y) = sum_x psi(x, y) g(x)
// from the shared table in LDS, taking g(x) of the other parts from their lanes
// one value at a time (a lane never holds all of g).  Messages that use the
// transposed table read psi^T, staged beside psi, so that both sum over x in
// ascending order with the same row reads.  The normalisation and the residual
// are reduced over the group.
template <int KP, int R, int MODE>
__device__ __forceinline__ void slot_update_split(const EvalArgs& a, const FlagRows& fr,
                                                  const float* s_logm, const float* s_A,
                                                  const float* s_psi, const float* s_psiT,
                                                  const unsigned short* s_owner, int s0, int n0,
                                                  int ns, float& rmax, unsigned int& act,
                                                  unsigned int& sa, unsigned int& sb, int p_out) {
    const float* __restrict__ m_in = fr.p;
    constexpr int KR = KP / R;
    constexpr int KS = KP + 1;
    const int tid = threadIdx.x;
    const int q = tid / R, h = tid % R;
    if (q >= ns) return;  // the R lanes of a slot leave together
    const int s = s0 + q;
    const int v = s_owner[q];
    float gp[KR];
    float mx = -3.402823466e38f;
#pragma unroll
    for (int i = 0; i < KR; ++i) {
        const int x = h * KR + i;
        gp[i] = s_A[v * KS + x] - s_logm[q * KS + x];
        mx = fmaxf(mx, gp[i]);
    }
    mx = group_max<R>(mx);
#pragma unroll
    for (int i = 0; i < KR; ++i) gp[i] -= mx;
    exp_batch<KR>(gp);
    const float* tab =
        a.pair_kind == kPairSharedAsym && a.orient[s] ? s_psiT : s_psi;
    float c[KR];
#pragma unroll
    for (int j = 0; j < KR; ++j) c[j] = 0.0f;
#pragma unroll
    for (int pp = 0; pp < R; ++pp) {
#pragma unroll
        for (int i = 0; i < KR; ++i) {
            const float gx = group_bcast<R>(gp[i], pp);  // g(x), x = pp KR + i
            const float4* row = (const float4*)(tab + (pp * KR + i) * KP + h * KR);
#pragma unroll
            for (int j4 = 0; j4 < KR / 4; ++j4) {
                const float4 p4 = row[j4];
                c[4 * j4] = fmaf(p4.x, gx, c[4 * j4]);
                c[4 * j4 + 1] = fmaf(p4.y, gx, c[4 * j4 + 1]);
                c[4 * j4 + 2] = fmaf(p4.z, gx, c[4 * j4 + 2]);
                c[4 * j4 + 3] = fmaf(p4.w, gx, c[4 * j4 + 3]);
            }
        }
    }
    float z = 0.0f;
#pragma unroll
    for (int j = 0; j < KR; ++j) z += c[j];
    z = group_sum<R>(z, h);
    const float inv = 1.0f / z;
    const long long eo = (long long)s * KP + h * KR;
    float old[KR];
    float r = 0.0f;
#pragma unroll
    for (int j4 = 0; j4 < KR / 4; ++j4) {
        const float4 o4 = *(const float4*)(m_in + eo + 4 * j4);
        old[4 * j4] = o4.x;
        old[4 * j4 + 1] = o4.y;
        old[4 * j4 + 2] = o4.z;
        old[4 * j4 + 3] = o4.w;
    }
    if (fr.on) {
        // the flag is the sign of the row's first entry (lane h = 0 holds it)
        const long long row = (long long)s * KP;
        if (fr.alt && (__float_as_uint(m_in[row]) >> 31)) {
#pragma unroll
            for (int j4 = 0; j4 < KR / 4; ++j4) {
                const float4 o4 = *(const float4*)(fr.alt + eo + 4 * j4);
                old[4 * j4] = o4.x;
                old[4 * j4 + 1] = o4.y;
                old[4 * j4 + 2] = o4.z;
                old[4 * j4 + 3] = o4.w;
            }
        }
        if (h == 0) old[0] = fabsf(old[0]);
    }
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        c[j] *= inv;
        r = fmaxf(r, fabsf(c[j] - old[j]));
    }
    r = group_max<R>(r);
    const bool active = r > a.eps;
    const bool lead = h == 0;  // counts once per slot
    rmax = fmaxf(rmax, r);
    act += active && lead;
    if (MODE == kModeLBP) {
#pragma unroll
        for (int j = 0; j < KR; ++j) a.out_buf[0][eo + j] = c[j];
    } else if (MODE == kModeRnBP) {
        bool ka = false, kb = false;
        if (active) {
            const int node = n0 + v;
            const unsigned int u24 = draw24(a, node, s - a.node_ptr[node]);
            ka = u24 < a.thr_a;
            kb = u24 < a.thr_b;
        }
        sa += ka && lead;
        sb += kb && lead;
        if (a.row_flags) {
            const bool kp = p_out == 0 ? ka : kb, ko = p_out == 0 ? kb : ka;
            const bool diff = ka != kb;
            float* op = a.out_buf[p_out] + eo;
#pragma unroll
            for (int j = 0; j < KR; ++j)
                op[j] = (j == 0 && h == 0) ? flag_first(kp ? c[0] : old[0], diff) : (kp ? c[j] : old[j]);
            if (diff) {
                float* os = a.out_buf[p_out ^ 1] + eo;
#pragma unroll
                for (int j = 0; j < KR; ++j) os[j] = ko ? c[j] : old[j];
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < KR; ++j) a.out_buf[0][eo + j] = ka ? c[j] : old[j];
    } else if (MODE == kModeRBP) {
#pragma unroll
        for (int j = 0; j < KR; ++j) a.cand[eo + j] = c[j];
        if (lead) a.keys[s] = __float_as_uint(r);
    }
}

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16 bit pattern, round to nearest even (finite inputs).
__device__ __forceinline__ short bf16_rne(float f) {
    const unsigned int b = __float_as_uint(f);
    return (short)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}

// Eq. (2) for K = 32 with one symmetric shared table on the matrix cores.  Each
// wave takes 32 slots of the tile; the products c = g P of its slots are one
// 32 x 32 x 32 matrix product, 16 v_mfma_f32_32x32x2f32 steps with FP32 inputs
// and FP32 accumulation.  Operand layout of that instruction: lane l supplies
// A[l % 32][l / 32] and B[l / 32][l % 32] of each 32 x 2 / 2 x 32 step, and
// holds D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] in accumulator r = 0..15.
// So lane (m = l % 32, h = l / 32) computes the cavity values g(x) of slot m
// for the states x = 2 s + h, holds column m of the table for those states,
// and after the product the tile goes through LDS (rows of 33 floats) back to
// one slot per lane pair, each lane with 16 consecutive states of its slot.
// BF16: the same product with BF16 operands (v_mfma_f32_32x32x8_bf16, FP32
// accumulation): 4 steps of 8 states, lane (m, h) supplying the states
// 8 s + 4 h .. 8 s + 4 h + 3; g and the table are rounded to 8-bit mantissas.
// The lane's operand entry st of the product covers state mfma32_state(st).
template <bool BF16>
__device__ __forceinline__ int mfma32_state(int st, int h) {
    return BF16 ? 8 * (st >> 2) + 4 * h + (st & 3) : 2 * st + h;
}

// B operand of the lane: P[x][m] for its 16 states (loaded once per block).
template <bool BF16>
__device__ __forceinline__ void mfma32_table(const EvalArgs& a, float* pb) {
    const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
#pragma unroll
    for (int st = 0; st < 16; ++st) pb[st] = a.pair[mfma32_state<BF16>(st, h) * 32 + m];
}

// Position of state x in an LDS row of k_eval_mfma32: the 16 states of half h
// (mfma32_state) are consecutive at 16 h, so a lane reads its operands as four
// 16-byte words.
constexpr int kMfmaStride = 36;  // floats per row: 16-byte aligned, 8 rows span the 32 banks

// p_out (row_flags): the outcome whose rows are written whole.  ns >= 1: a lane past the
// tile's slots reads the last one's row.
template <int MODE, bool BF16 = false>
__device__ __forceinline__ void slot_update_mfma32(const EvalArgs& a, const FlagRows& fr,
                                                   float* s_logm, const float* s_A,
                                                   const unsigned short* s_owner,
                                                   const int* s_ptr, int s0, int n0, int ns,
                                                   float& rmax, unsigned int& act,
                                                   unsigned int& sa, unsigned int& sb, int p_out) {
    constexpr int K = 32, KS = kMfmaStride;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 31, h = lane >> 5;
    const int q = 32 * w + m;  // slot of the tile
    const bool valid = q < ns;
    // A operand: the cavity distribution of slot q at the lane's states
    const int v = valid ? s_owner[q] : 0;
    float gv[16];
    float mx = -3.402823466e38f;
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const float4 A4 = *(const float4*)(s_A + v * KS + 16 * h + 4 * t4);
        const float4 l4 = *(const float4*)(s_logm + q * KS + 16 * h + 4 * t4);
        // (nothing reads the product of a row past the tile's slots)
        gv[4 * t4] = A4.x - l4.x;
        gv[4 * t4 + 1] = A4.y - l4.y;
        gv[4 * t4 + 2] = A4.z - l4.z;
        gv[4 * t4 + 3] = A4.w - l4.w;
    }
#pragma unroll
    for (int st = 0; st < 16; ++st) mx = fmaxf(mx, gv[st]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
    for (int st = 0; st < 16; ++st) gv[st] -= mx;
    exp_batch<16>(gv);
    // (held back, here and for the lane's own row below, so that the registers of
    // one phase are not live through the others: 56 instead of 123, and LDS, not
    // registers, sets the resident blocks)
    __builtin_amdgcn_sched_barrier(0);
    float pb[16];
    mfma32_table<BF16>(a, pb);
    floatx16 d;
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = 0.0f;
    if (BF16) {
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const shortx4 ga = {bf16_rne(gv[4 * st]), bf16_rne(gv[4 * st + 1]), bf16_rne(gv[4 * st + 2]),
                                bf16_rne(gv[4 * st + 3])};
            const shortx4 pbb = {bf16_rne(pb[4 * st]), bf16_rne(pb[4 * st + 1]), bf16_rne(pb[4 * st + 2]),
                                 bf16_rne(pb[4 * st + 3])};
            d = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(ga, pbb, d, 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int st = 0; st < 16; ++st)
            d = __builtin_amdgcn_mfma_f32_32x32x2f32(gv[st], pb[st], d, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the lane's own row: states 16 h .. of slot m (after the product, so that
    // its registers are not held through it; requested before the LDS round trip)
    const int sl = s0 + q;
    const long long eo = (long long)min(sl, s0 + ns - 1) * K + 16 * h;
    float old[16];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const float4 o4 = *(const float4*)(fr.p + eo + 4 * t4);
        old[4 * t4] = o4.x;
        old[4 * t4 + 1] = o4.y;
        old[4 * t4 + 2] = o4.z;
        old[4 * t4 + 3] = o4.w;
    }
    // D[i][m] -> LDS row 32 w + i (the wave's own rows of the log buffer, which
    // its lanes have finished reading: LDS operations of a wave run in order)
    float* rows = s_logm + (32 * w) * KS;
#pragma unroll
    for (int r = 0; r < 16; ++r) rows[(8 * (r >> 2) + 4 * h + (r & 3)) * KS + m] = d[r];
    // back as slot m, states 16 h .. 16 h + 15
    float c[16];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const float4 c4 = *(const float4*)(rows + m * KS + 16 * h + 4 * t4);
        c[4 * t4] = c4.x;
        c[4 * t4 + 1] = c4.y;
        c[4 * t4 + 2] = c4.z;
        c[4 * t4 + 3] = c4.w;
    }
    if (fr.on) {
        // the flag is the sign of the row's first entry (lane h = 0 holds it)
        if (fr.alt && __shfl((int)(__float_as_uint(old[0]) >> 31), m, 64)) {
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {
                const float4 o4 = *(const float4*)(fr.alt + eo + 4 * t4);
                old[4 * t4] = o4.x;
                old[4 * t4 + 1] = o4.y;
                old[4 * t4 + 2] = o4.z;
                old[4 * t4 + 3] = o4.w;
            }
        }
        if (h == 0) old[0] = fabsf(old[0]);
    }
    float z = 0.0f;
#pragma unroll
    for (int t = 0; t < 16; ++t) z += c[t];
    const float zo = __shfl_xor(z, 32, 64);
    z = h == 0 ? z + zo : zo + z;
    const float inv = 1.0f / z;
    float r = 0.0f;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        c[t] *= inv;
        r = fmaxf(r, fabsf(c[t] - old[t]));
    }
    r = fmaxf(r, __shfl_xor(r, 32, 64));
    const bool active = valid && r > a.eps;
    const bool lead = h == 0;  // counts once per slot
    if (valid) rmax = fmaxf(rmax, r);
    act += active && lead;
    if (MODE == kModeEvalOnly) return;
    // What is stored whole goes back through the wave's LDS rows, so that eight lanes
    // write the 128 bytes of a row in one request: from the lane pair's registers every
    // store would be 16 bytes of 64 rows, four requests for each 64 bytes.
    float* dst;
    if (MODE == kModeLBP) {
        dst = a.out_buf[0];
    } else if (MODE == kModeRBP) {
        dst = a.cand;
        if (lead && valid) a.keys[sl] = __float_as_uint(r);
    } else {
        bool ka = false, kb = false;
        if (active) {
            const unsigned int u24 = draw24(a, n0 + v, q - s_ptr[v]);
            ka = u24 < a.thr_a;
            kb = u24 < a.thr_b;
        }
        sa += ka && lead;
        sb += kb && lead;
        // the whole row of outcome p_out; with two outcomes (row_flags) its first
        // entry's sign bit set where they differ, the other outcome's row only there
        bool kp = ka;
        dst = a.out_buf[0];
        if (a.row_flags) {
            const bool ko = p_out == 0 ? kb : ka, diff = ka != kb;
            kp = p_out == 0 ? ka : kb;
            dst = a.out_buf[p_out];
            if (diff) {
                float4* os = (float4*)(a.out_buf[p_out ^ 1] + eo);
#pragma unroll
                for (int t4 = 0; t4 < 4; ++t4)
                    os[t4] = ko ? make_float4(c[4 * t4], c[4 * t4 + 1], c[4 * t4 + 2], c[4 * t4 + 3])
                                : make_float4(old[4 * t4], old[4 * t4 + 1], old[4 * t4 + 2],
                                              old[4 * t4 + 3]);
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) c[t] = kp ? c[t] : old[t];
            if (h == 0) c[0] = flag_first(c[0], diff);
        } else {
#pragma unroll
            for (int t = 0; t < 16; ++t) c[t] = kp ? c[t] : old[t];
        }
    }
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4)
        *(float4*)(rows + m * KS + 16 * h + 4 * t4) =
            make_float4(c[4 * t4], c[4 * t4 + 1], c[4 * t4 + 2], c[4 * t4 + 3]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = (lane >> 3) + 8 * j, x = 4 * (lane & 7);
        const float4 v4 = *(const float4*)(rows + i * KS + x);
        if (32 * w + i < ns) *(float4*)(dst + (long long)(s0 + 32 * w + i) * K + x) = v4;
    }
}

// A shared K x K table seen through the constant address space: with K known
// at compile time its entries are wave-uniform scalar loads (s_load into SGPRs
// that the multiply-adds read directly), not one LDS read per multiply-add.
typedef const __attribute__((address_space(4))) float* ConstF;

// c(y) += sum_x P[x][y] g(x) (T: P[y][x]) for a uniform table P.
template <int K, bool T>
__device__ __forceinline__ void matvec_uniform(ConstF P, const float* g, float* c) {
#pragma unroll
    for (int x = 0; x < K; ++x) {
        const float gx = g[x];
#pragma unroll
        for (int y = 0; y < K; ++y) c[y] = fmaf(T ? P[y * K + x] : P[x * K + y], gx, c[y]);
    }
}

// LDS of the [E][K] kernels: rows of K + 1 floats (a thread per slot reads its
// own row, and an odd stride puts the rows of neighbouring lanes in different
// banks).  Node rows are sized by the largest node count of a tile.
struct GenericLds {
    float* logm;             // [TS][KS] logs of the incoming messages
    float* A;                // [TN][KS] node aggregates
    float* psi;              // [K][K] shared table (paths that read it from LDS)
    float* psiT;             // [K][K] its transpose (asymmetric tables), else psi
    int* rev;                // [TS]
    int* ptr;                // [TN + 1] local slot offsets of the nodes
    unsigned short* owner;   // [TS]
};

// tables: the number of K x K tables reserved (0; 1, psi; 2, psi and psi^T);
// the launch sizes the LDS the same way
__device__ __forceinline__ GenericLds generic_lds(float* smem, int K, int TS, int TN,
                                                  int tables) {
    GenericLds l;
    const int KS = K + 1;
    l.logm = smem;
    l.A = l.logm + TS * KS;
    l.psi = l.A + ((TN * KS + 3) & ~3);  // 16-byte aligned: read as float4 rows
    l.psiT = tables == 2 ? l.psi + K * K : l.psi;
    l.rev = (int*)(l.psi + tables * K * K);
    l.ptr = l.rev + TS;
    l.owner = (unsigned short*)(l.ptr + TN + 1);
    return l;
}

// Phase 1 of a tile whose slots fit (ns <= TS): gather the incoming rows
// m_{k->i} (K consecutive threads per row; a tile holds at most
// kTileFloatsGeneric values, kPer per thread, and a thread issues all of its
// loads before using the first), take logs of K * m (the constant cancels in
// the cavity and the normalisation, and it keeps the node aggregate near zero
// for messages near uniform, where FP32 rounding of a large aggregate would
// dominate), and sum them per node with the unary: A_i(x) of Eq. (2)/(3).
// Ends with a barrier.
// Rows written with outcome flags (EvalArgs.row_flags): m_in is the buffer of
// full rows; the sign bit of a row's first entry marks a message whose other
// outcome is in m_alt.  m_alt == nullptr: the full rows hold the chosen
// outcome, and only the flag bit is cleared (a no-op on unflagged rows).
__device__ __forceinline__ void generic_phase1(const EvalArgs& a, const float* __restrict__ m_in,
                                               const GenericLds& l, int K, int n0, int nn,
                                               int s0, int ns, const float* m_alt = nullptr) {
    const int tid = threadIdx.x;
    const int KS = K + 1;
    const float fK = (float)K;
    for (int q = tid; q < ns; q += kBlock) l.rev[q] = a.rev[s0 + q];
    for (int v = tid; v <= nn; v += kBlock) l.ptr[v] = a.node_ptr[n0 + v] - s0;
    __syncthreads();
    constexpr int kPer = kTileFloatsGeneric / kBlock;
    float gat[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid + j * kBlock;
        const int q = i / K, x = i - q * K;
        gat[j] = q < ns ? m_in[(long long)l.rev[q] * K + x] : 1.0f;
    }
    if (m_alt) {
        // the other outcome was chosen: flagged rows come from m_alt
        unsigned int f[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = tid + j * kBlock;
            const int q = i / K;
            f[j] = q < ns ? __float_as_uint(m_in[(long long)l.rev[q] * K]) >> 31 : 0u;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = tid + j * kBlock;
            const int q = i / K, x = i - q * K;
            if (f[j]) gat[j] = m_alt[(long long)l.rev[q] * K + x];
        }
    }
    // (the flag bit is the sign of a row's first entry; messages are non-negative)
#pragma unroll
    for (int j = 0; j < kPer; ++j) gat[j] = fK * fabsf(gat[j]);
    log_batch<kPer>(gat);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid + j * kBlock;
        const int q = i / K, x = i - q * K;
        if (q < ns) l.logm[q * KS + x] = gat[j];
    }
    // the nodes' unaries (loads first), then the aggregates
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid + j * kBlock;
        const int v = i / K, x = i - v * K;
        gat[j] = v < nn ? a.unary[(long long)(n0 + v) * K + x] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid + j * kBlock;
        const int v = i / K, x = i - v * K;
        if (v < nn) {
            const int q0 = l.ptr[v], q1 = l.ptr[v + 1];
            float acc = gat[j];
            for (int q = q0; q < q1; ++q) acc += l.logm[q * KS + x];
            l.A[v * KS + x] = acc;
            if (x == 0)
                for (int q = q0; q < q1; ++q) l.owner[q] = (unsigned short)v;
        }
    }
    __syncthreads();
}

// K = 32 with a symmetric shared table and no oversized node: Eq. (2) on the
// matrix cores (slot_update_mfma32).  A kernel of its own, so that its register
// count (and hence its occupancy) is not set by the paths it does not take.
//
// What bounds it: the messages past L2 (500 x 500 grid, RnBP: 407 MB in 100 us, 4.05
// TB/s against 4.7 of a large copy; the own row and the gathered one are both read, the
// other outcome's rows written and read back), once the latency is covered: a tile
// is a chain of dependent loads (counters -> buffer choice; tile bounds -> reverse
// slots -> incoming rows), and a CU holds a handful of blocks.  So the counters, the tile's bounds, reverse slots and node
// bounds are requested together, then the incoming rows, the lane's own row and
// the unaries; only LDS barriers separate the phases, so no request is waited
// for before its value is used.  (Several tiles per block, the next one's
// constants prefetched, ran slower: 949 and 1,003 us a solve for three and six
// tiles against 935 for one.)
struct Mfma32Lds {
    float* logm;             // [128][kMfmaStride]
    float* A;                // [TN][kMfmaStride]
    int* rev;                // [128]
    int* ptr;                // [TN + 1]
    unsigned short* owner;   // [128]
};
constexpr int kMfmaSlots = kTileFloatsGeneric / 32;
__host__ __device__ inline size_t mfma32_lds_bytes(int TN) {
    return sizeof(float) * (size_t)kMfmaStride * (kMfmaSlots + TN) +
           sizeof(int) * (size_t)(kMfmaSlots + TN + 1) + sizeof(unsigned short) * kMfmaSlots;
}

template <int MODE, bool BF16>
__global__ __launch_bounds__(kBlock) void k_eval_mfma32(
    EvalArgs a) {
    extern __shared__ float4 smem4[];
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    constexpr int K = 32, KS = kMfmaStride;
    const int tid = threadIdx.x, lane = tid & 63;
    const int TN = a.tile_nodes_max;
    Mfma32Lds l;
    l.logm = (float*)smem4;
    l.A = l.logm + kMfmaSlots * KS;
    l.rev = (int*)(l.A + TN * KS);
    l.ptr = l.rev + kMfmaSlots;
    l.owner = (unsigned short*)(l.ptr + TN + 1);

    CtrLoad cl;
    prologue_issue(a, cl, blockIdx.x == 0);
    const int tile = tile_of_block(a);
    const bool has = tile < a.num_tiles;
    const int n0 = has ? a.tile_start[tile] : 0, n1 = has ? a.tile_start[tile + 1] : 0;
    const int s0 = has ? a.tile_slot[tile] : 0, s1 = has ? a.tile_slot[tile + 1] : 0;
    const int nn = n1 - n0, ns = s1 - s0;
    if (tid < ns) l.rev[tid] = a.rev[s0 + tid];
    if (tid <= nn && has) l.ptr[tid] = a.node_ptr[n0 + tid] - s0;
    const float* m_sel = prologue_finish(a, cl, s_red, blockIdx.x == 0);
    // (a tile without slots has no message to write and no row that its lanes could
    // read in place of one: the buffers may start behind it, or hold nothing)
    if (!m_sel || ns == 0) return;
    int p_out;
    const FlagRows fr = flag_inputs(a, m_sel, p_out);
    const float* __restrict__ m_in = fr.p;
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    lds_barrier();
    // incoming rows: eight lanes per row, four rows per thread
    float4 g4[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = tid + u * kBlock, q = i >> 3;
        g4[u] = *(const float4*)(m_in + (long long)l.rev[min(q, ns - 1)] * K +
                                 4 * (i & 7));
    }
    // unaries of node v (this thread's four positions p4 ..)
    auto load_unary = [&](int v, int p4) {
        const float* un = a.unary + (long long)(n0 + min(v, nn - 1)) * K;
        const int h = p4 >> 4, st = p4 & 15;
        return make_float4(un[mfma32_state<BF16>(st, h)], un[mfma32_state<BF16>(st + 1, h)],
                           un[mfma32_state<BF16>(st + 2, h)], un[mfma32_state<BF16>(st + 3, h)]);
    };
    float4 acc = load_unary(tid >> 3, 4 * (tid & 7));
    if (fr.alt) {
        // the other outcome was chosen: flagged rows (the sign of a row's
        // first entry) come from alt
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = tid + u * kBlock, q = i >> 3;
            const int f = __shfl((int)(__float_as_uint(g4[u].x) >> 31), lane & ~7, 64);
            if (f && q < ns)
                g4[u] = *(const float4*)(fr.alt + (long long)l.rev[q] * K + 4 * (i & 7));
        }
    }
    // logs of K m (as generic_phase1)
    constexpr float fK = (float)K;
    float lg[16];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        lg[4 * u] = fK * fabsf(g4[u].x);
        lg[4 * u + 1] = fK * g4[u].y;
        lg[4 * u + 2] = fK * g4[u].z;
        lg[4 * u + 3] = fK * g4[u].w;
    }
    log_batch<16>(lg);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = tid + u * kBlock, q = i >> 3, x4 = i & 7;
        float* row = l.logm + q * KS;
        if (BF16) {
            *(float4*)(row + 16 * (x4 & 1) + 4 * (x4 >> 1)) =
                make_float4(lg[4 * u], lg[4 * u + 1], lg[4 * u + 2], lg[4 * u + 3]);
        } else {
            *(float2*)(row + 2 * x4) = make_float2(lg[4 * u], lg[4 * u + 2]);
            *(float2*)(row + 16 + 2 * x4) = make_float2(lg[4 * u + 1], lg[4 * u + 3]);
        }
    }
    // node aggregates: a thread per node and four positions
    for (int i0 = 0; i0 < 8 * nn; i0 += kBlock) {
        const int i = i0 + tid, v = i >> 3, p4 = 4 * (i & 7);
        if (i0) acc = load_unary(v, p4);
        if (i0 == 0) lds_barrier();  // the logs are in LDS
        if (v < nn) {
            const int q0 = l.ptr[v], q1 = l.ptr[v + 1];
            for (int q = q0; q < q1; ++q) {
                const float4 t = *(const float4*)(l.logm + q * KS + p4);
                acc.x += t.x;
                acc.y += t.y;
                acc.z += t.z;
                acc.w += t.w;
                if (p4 == 0) l.owner[q] = (unsigned short)v;
            }
            *(float4*)(l.A + v * KS + p4) = acc;
        }
    }
    lds_barrier();
    slot_update_mfma32<MODE, BF16>(a, fr, l.logm, l.A, l.owner, l.ptr, s0, n0, ns, rmax, act, sa, sb,
                                   p_out);
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// Shared tables with K = 32 or 64: each slot is split over R = 2 or 4 lanes,
// which read the table from LDS (the lanes of a wave need different columns).
// Graphs with a node over the tile limit take k_eval_pairs.
template <int KP, int MODE>
__global__ __launch_bounds__(kBlock) void k_eval_split(EvalArgs a) {
    extern __shared__ float smem[];
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    const float* m_sel = iteration_prologue(a, s_red, blockIdx.x == 0);
    if (!m_sel) return;
    int p_out;
    const FlagRows fr = flag_inputs(a, m_sel, p_out);
    const int tile = tile_of_block(a);
    if (tile >= a.num_tiles) return;
    constexpr int TS = kTileFloatsGeneric / KP;  // slots per tile
    constexpr int R = KP * kBlock / kTileFloatsGeneric;
    static_assert(R == 2 || R == 4, "lane groups of 2 or 4");
    const bool asym = a.pair_kind == kPairSharedAsym;
    const GenericLds l = generic_lds(smem, KP, TS, a.tile_nodes_max, asym ? 2 : 1);
    const int n0 = a.tile_start[tile], n1 = a.tile_start[tile + 1];
    const int s0 = a.tile_slot[tile], s1 = a.tile_slot[tile + 1];
    const int ns = s1 - s0, nn = n1 - n0;
    for (int i = threadIdx.x; i < KP * KP; i += kBlock) l.psi[i] = a.pair[i];
    if (asym)
        for (int i = threadIdx.x; i < KP * KP; i += kBlock) l.psiT[i] = a.pair[(i % KP) * KP + i / KP];
    generic_phase1(a, fr.p, l, KP, n0, nn, s0, ns, fr.alt);
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    slot_update_split<KP, R, MODE>(a, fr, l.logm, l.A, l.psi, l.psiT, l.owner, s0, n0, ns, rmax, act,
                                   sa, sb, p_out);
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// K up to 16 (shared tables; K = 2 also Ising and per-slot tables): a thread per
// slot, every K compiled, so that the products are K * K multiply-adds that take
// the table from scalar registers.  (One width per power of two, the states past K
// predicated away, took 428 us for ten RnBP sweeps of a 300 x 300 grid with
// K = 5 and 616 us for nine LBP sweeps with K = 13.)
template <int KP, int MODE>
__global__ __launch_bounds__(kBlock) void k_eval_generic(EvalArgs a) {
    extern __shared__ float smem[];
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    const float* m_sel = iteration_prologue(a, s_red, blockIdx.x == 0);
    if (!m_sel) return;
    int p_out;
    const FlagRows fr = flag_inputs(a, m_sel, p_out);
    const float* __restrict__ m_in = fr.p;
    const int tile = tile_of_block(a);
    if (tile >= a.num_tiles) return;
    constexpr int K = KP;
    const int TS = kTileFloatsGeneric / K;  // slots per tile
    const int KS = K + 1;
    const GenericLds l = generic_lds(smem, K, TS, a.tile_nodes_max, 0);
    float* s_logm = l.logm;
    float* s_A = l.A;
    unsigned short* s_owner = l.owner;

    const int n0 = a.tile_start[tile], n1 = a.tile_start[tile + 1];
    const int s0 = a.tile_slot[tile], s1 = a.tile_slot[tile + 1];
    const int ns = s1 - s0, nn = n1 - n0;
    const int tid = threadIdx.x;
    const bool big = ns > TS;
    const float fK = (float)K;

    if (!big) {
        generic_phase1(a, m_in, l, K, n0, nn, s0, ns, fr.alt);
    } else {
        // single node with degree > TS: aggregate each state with a strided sum
        for (int x = 0; x < K; ++x) {
            float part = 0.0f;
            for (int q = tid; q < ns; q += kBlock)
                part += logf(fK * flag_entry(fr, (long long)a.rev[s0 + q] * K, x));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
            if ((tid & 63) == 0) red.rmax[tid >> 6] = part;
            __syncthreads();
            if (tid == 0) {
                float acc = a.unary[(long long)n0 * K + x];
                for (int i = 0; i < kBlock / 64; ++i) acc += red.rmax[i];
                s_A[x] = acc;
            }
            __syncthreads();
        }
    }
    __syncthreads();

    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    for (int q = tid; q < ns; q += kBlock) {
        const int s = s0 + q;
        const int v = big ? 0 : s_owner[q];
        const int node = n0 + v;
        const long long rin = big ? (long long)a.rev[s] * K : 0;
        float g[KP];
        float mx = -3.402823466e38f;
#pragma unroll
        for (int x = 0; x < KP; ++x) {
            const float lm = big ? logf(fK * flag_entry(fr, rin, x)) : s_logm[q * KS + x];
            g[x] = s_A[v * KS + x] - lm;
            mx = fmaxf(mx, g[x]);
        }
#pragma unroll
        for (int x = 0; x < KP; ++x) g[x] -= mx;
        exp_batch<KP>(g);
        float c[KP];
#pragma unroll
        for (int y = 0; y < KP; ++y) c[y] = 0.0f;
        // (Ising and per-slot tables: K = 2 only; wider tables of their own take
        // k_eval_pairs)
        if (KP == 2 && a.pair_kind == kPairIsing) {
            // exp(J s_i s_k) scaled by exp(-|J|): one entry is 1, the other exp(-2|J|)
            const float J = a.coupling[s];
            const float ep = expf(J - fabsf(J)), em = expf(-J - fabsf(J));
            c[0] = ep * g[0] + em * g[1];
            c[1] = em * g[0] + ep * g[1];
        } else if (KP > 2 || a.pair_kind != kPairDense) {
            const ConstF P4 = (ConstF)(uintptr_t)a.pair;
            if (a.pair_kind == kPairSharedAsym && a.orient[s])
                matvec_uniform<KP, true>(P4, g, c);
            else
                matvec_uniform<KP, false>(P4, g, c);
        } else {
            const float* P = a.pair + (long long)s * K * K;
#pragma unroll
            for (int x = 0; x < K; ++x)
#pragma unroll
                for (int y = 0; y < K; ++y) c[y] = fmaf(P[x * K + y], g[x], c[y]);
        }
        float z = 0.0f;
#pragma unroll
        for (int y = 0; y < KP; ++y) z += c[y];
        const float inv = 1.0f / z;
        const long long eo = (long long)s * K;
        float r = 0.0f;
        float old[KP];
#pragma unroll
        for (int y = 0; y < KP; ++y) {
            c[y] *= inv;
            old[y] = flag_entry(fr, eo, y);
            r = fmaxf(r, fabsf(c[y] - old[y]));
        }
        const bool active = r > a.eps;
        rmax = fmaxf(rmax, r);
        act += active;
        if (MODE == kModeLBP) {
#pragma unroll
            for (int y = 0; y < KP; ++y) a.out_buf[0][eo + y] = c[y];
        } else if (MODE == kModeRnBP) {
            bool ka = false, kb = false;
            if (active) {
                const unsigned int u24 = draw24(a, node, s - a.node_ptr[node]);
                ka = u24 < a.thr_a;
                kb = u24 < a.thr_b;
            }
            sa += ka;
            sb += kb;
            if (a.row_flags) {
                // the whole row of outcome p_out, the other where they differ
                const bool kp = p_out == 0 ? ka : kb, ko = p_out == 0 ? kb : ka;
                const bool diff = ka != kb;
                float* op = a.out_buf[p_out] + eo;
#pragma unroll
                for (int y = 0; y < KP; ++y) op[y] = y == 0 ? flag_first(kp ? c[0] : old[0], diff) : (kp ? c[y] : old[y]);
                if (diff) {
                    float* os = a.out_buf[p_out ^ 1] + eo;
#pragma unroll
                    for (int y = 0; y < KP; ++y) os[y] = ko ? c[y] : old[y];
                }
            } else {
#pragma unroll
                for (int y = 0; y < KP; ++y) a.out_buf[0][eo + y] = ka ? c[y] : old[y];
            }
        } else if (MODE == kModeRBP) {
#pragma unroll
            for (int y = 0; y < KP; ++y) a.cand[eo + y] = c[y];
            a.keys[s] = __float_as_uint(r);
        }
    }
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// ---------------------------------------------------------------------------
// [E][K] layout, a lane per (slot, target state) pair: tables of their own per
// slot (K > 2), and shared tables with a K over 16 that is not 32 or 64.
//
// With a thread per slot a per-slot table is read K * K floats apart by
// neighbouring lanes, and a wide odd K needs K padded to 32 or 64 with every
// product predicated (1,024 or 4,096 of them, unrolled).  Here the outputs of the
// tile's slots are dealt to lanes pair by pair: consecutive lanes read
// consecutive entries of a table row, the outputs are stored coalesced, and the
// code does not depend on K.  Bound by the chain of phases, whose waves wait more than
// half of the time: 89 MB past L2 in 32 us for 20,000 edges with K = 21 tables of
// their own (2.8 TB/s, the vector units issue 27 % of it); 32 MB in 43 us for the
// 203 x 197 grid with one table (issue 46 %).  Every sum runs in the order the per-slot
// path takes (source states and target states ascending), so both round alike.
// Against a thread per slot, per solve: 20,000 edges with K = 21 tables of their
// own, seven LBP sweeps, 1,166 -> 341 us; 203 x 197 Potts grid, K = 21, six LBP
// sweeps, 763 -> 410 us; 300 x 300, K = 48, six RnBP sweeps, 10,722 -> 2,135 us.
//
//   1  incoming rows gathered and logged into LDS, node aggregates (as
//      generic_phase1)
//   2  cavity distributions g of every slot: a group of W lanes per slot (W = K
//      rounded up to a power of two), the maximum by shuffles, g in LDS
//   3  products c(y) = sum_x psi(x, y) g(x): per-slot tables from global memory
//      (four pairs per lane, eight rows each in flight), shared tables from LDS,
//      and symmetric shared tables as 32-row tiles on the matrix cores
//      (v_mfma_f32_32x32x2f32; states past K contribute products with 0)
//   4  a lane per slot: normalisation; pairs: |change|; a lane per slot:
//      residual and frontier decision; pairs: stores
// ---------------------------------------------------------------------------
enum PairTable : int { kTabDense = 0, kTabShared = 1, kTabMfma = 2 };

struct PairsLds {
    float* G;                // [TS][KS] logs of the incoming messages, then g, then |change|
    float* C;                // [TS][KS] outputs
    float* A;                // [TN][KS] node aggregates
    float* inv;              // [TS] 1 / z
    float* psi;              // [K][K] shared table
    int* rev;                // [TS]
    int* ptr;                // [TN + 1]
    unsigned int* keep;      // [TS]
    unsigned short* owner;   // [TS]
};

__host__ __device__ inline size_t pairs_lds_bytes(int K, int TS, int TN, int tables) {
    const int KS = K | 1;
    return sizeof(float) * ((size_t)2 * TS * KS + (size_t)TN * KS + TS + (size_t)tables * K * K) +
           sizeof(int) * ((size_t)TS + TN + 1 + TS) + sizeof(unsigned short) * (size_t)TS;
}

__device__ __forceinline__ PairsLds pairs_lds(float* smem, int K, int TS, int TN, int tables) {
    const int KS = K | 1;
    PairsLds l;
    l.G = smem;
    l.C = l.G + TS * KS;
    l.A = l.C + TS * KS;
    l.inv = l.A + TN * KS;
    l.psi = l.inv + TS;
    l.rev = (int*)(l.psi + tables * K * K);
    l.ptr = l.rev + TS;
    l.keep = (unsigned int*)(l.ptr + TN + 1);
    l.owner = (unsigned short*)(l.keep + TS);
    return l;
}

template <int MODE, int TAB>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(
    TAB == kTabShared ? 5 : 1))) void k_eval_pairs(EvalArgs a) {
    extern __shared__ float smem[];
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    // entries per lane in flight (eight cost the matrix-core variant a wave per
    // SIMD: 465 instead of 386 us for six sweeps of the 203 x 197 grid, K = 21)
    constexpr int U = kPairsUnroll;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int K = a.num_states, KS = K | 1;
    const int TS = a.tile_slots_max, TN = a.tile_nodes_max;
    const PairsLds l = pairs_lds(smem, K, TS, TN, TAB == kTabDense ? 0 : 1);
    const unsigned int magic = a.k_magic;
    auto row_of = [&](int i) { return (int)(((unsigned int)i * magic) >> 20); };  // i / K
    // the counters and the tile's graph constants are in flight together
    CtrLoad cl;
    prologue_issue(a, cl, blockIdx.x == 0);
    const int tile = tile_of_block(a);
    const bool has = tile < a.num_tiles;
    const int n0 = has ? a.tile_start[tile] : 0, n1 = has ? a.tile_start[tile + 1] : 0;
    const int s0 = has ? a.tile_slot[tile] : 0, s1 = has ? a.tile_slot[tile + 1] : 0;
    const int nn = n1 - n0, node_slots = s1 - s0;
    // a node over the tile limit: its slots are taken TS at a time
    const bool big = node_slots > TS;
    const int ns0 = big ? TS : node_slots;
    for (int q = tid; q < ns0; q += kBlock) l.rev[q] = a.rev[s0 + q];
    for (int v = tid; v <= nn && has; v += kBlock) l.ptr[v] = a.node_ptr[n0 + v] - s0;
    if (TAB != kTabDense) {
        for (int i = tid; i < K * K; i += kBlock) l.psi[i] = a.pair[i];
    }
    const float* m_sel = prologue_finish(a, cl, s_red, blockIdx.x == 0);
    if (!m_sel || !has) return;
    int p_out;
    const FlagRows fr = flag_inputs(a, m_sel, p_out);
    const float* __restrict__ m_in = fr.p;
    const float fK = (float)K;
    if (big) {
        // aggregate each state over all of the node's slots with a strided sum
        for (int x = 0; x < K; ++x) {
            float part = 0.0f;
            for (int q = tid; q < node_slots; q += kBlock)
                part += logf(fK * flag_entry(fr, (long long)a.rev[s0 + q] * K, x));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
            if (lane == 0) red.rmax[w] = part;
            __syncthreads();
            if (tid == 0) {
                float acc = a.unary[(long long)n0 * K + x];
                for (int i = 0; i < kBlock / 64; ++i) acc += red.rmax[i];
                l.A[x] = acc;
            }
            __syncthreads();
        }
    }
    __syncthreads();
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    for (int base = 0; base < node_slots; base += TS) {
        const int sc = s0 + base, ns = min(TS, node_slots - base), P = ns * K;
        if (base) {
            __syncthreads();  // the LDS rows of the previous slots are free
            for (int q = tid; q < ns; q += kBlock) l.rev[q] = a.rev[sc + q];
            __syncthreads();
        }
        // 1. logs of K m (as generic_phase1) and the node aggregates
        for (int c0 = 0; c0 < P; c0 += U * kBlock) {
            float v[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = c0 + tid + j * kBlock;
                const int q = row_of(i);
                v[j] = i < P ? m_in[(long long)l.rev[q] * K + (i - q * K)] : 1.0f;
            }
            if (fr.alt) {
                // the other outcome was chosen: flagged rows come from alt
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const int i = c0 + tid + j * kBlock;
                    const int q = row_of(i);
                    if (i < P) {
                        const long long r = (long long)l.rev[q] * K;
                        if (__float_as_uint(m_in[r]) >> 31) v[j] = fr.alt[r + (i - q * K)];
                    }
                }
            }
            // a flag is the sign of a row's first entry (messages are non-negative)
#pragma unroll
            for (int j = 0; j < U; ++j) v[j] = fK * fabsf(v[j]);
            log_batch<U>(v);
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = c0 + tid + j * kBlock;
                const int q = row_of(i);
                if (i < P) l.G[q * KS + (i - q * K)] = v[j];
            }
        }
        const int NK = big ? 0 : nn * K;
        if (big)
            for (int q = tid; q < ns; q += kBlock) l.owner[q] = 0;
        for (int c0 = 0; c0 < NK; c0 += 4 * kBlock) {
            float u[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = c0 + tid + j * kBlock;
                u[j] = i < NK ? a.unary[(long long)n0 * K + i] : 0.0f;
            }
            if (c0 == 0) __syncthreads();  // the logs are in LDS
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = c0 + tid + j * kBlock;
                if (i < NK) {
                    const int v = row_of(i), x = i - v * K;
                    const int q0 = l.ptr[v], q1 = l.ptr[v + 1];
                    float acc = u[j];
                    for (int q = q0; q < q1; ++q) acc += l.G[q * KS + x];
                    l.A[v * KS + x] = acc;
                    if (x == 0)
                        for (int q = q0; q < q1; ++q) l.owner[q] = (unsigned short)v;
                }
            }
        }
        __syncthreads();

        // 2. cavity distributions
        {
            const int wl = a.k_wlog, W = 1 << wl;
            const int x = tid & (W - 1);
            for (int q = tid >> wl; q < ns; q += kBlock >> wl) {
                float c = -3.402823466e38f;
                if (x < K) c = l.A[l.owner[q] * KS + x] - l.G[q * KS + x];
                float mx = fmaxf(c, -3.402823466e38f);
                for (int o = W >> 1; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
                if (x < K) l.G[q * KS + x] = expf(c - mx);
            }
        }
        __syncthreads();

        // 3. products
        if (TAB == kTabMfma) {
            const int m = lane & 31, h = lane >> 5;
            for (int r0 = 32 * w; r0 < ns; r0 += 32 * (kBlock / 64)) {
                const float* g = l.G + min(r0 + m, ns - 1) * KS;
                for (int y0 = 0; y0 < K; y0 += 32) {
                    const bool col = y0 + m < K;
                    floatx16 d;
#pragma unroll
                    for (int r = 0; r < 16; ++r) d[r] = 0.0f;
                    for (int xs = 0; xs < K; xs += 8) {
                        float ga[4], pb[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int x = xs + 2 * u + h;
                            ga[u] = x < K ? g[x] : 0.0f;
                            pb[u] = x < K && col ? l.psi[x * K + y0 + m] : 0.0f;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            d = __builtin_amdgcn_mfma_f32_32x32x2f32(ga[u], pb[u], d, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int q = r0 + 8 * (r >> 2) + 4 * h + (r & 3);
                        if (q < ns && col) l.C[q * KS + y0 + m] = d[r];
                    }
                }
            }
        } else {
            for (int c0 = 0; c0 < P; c0 += 4 * kBlock) {
                const float* T[4];
                const float* g[4];
                int o[4], sx[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = min(c0 + tid + j * kBlock, P - 1);
                    const int q = row_of(i), y = i - q * K;
                    g[j] = l.G + q * KS;
                    o[j] = q * KS + y;
                    // element (x, y) at T[x * sx]; transposed for the other
                    // direction of an asymmetric shared table
                    T[j] = TAB == kTabDense ? a.pair + (long long)(sc + q) * K * K + y : l.psi + y;
                    sx[j] = K;
                    if (TAB == kTabShared && a.pair_kind == kPairSharedAsym && a.orient[sc + q]) {
                        T[j] = l.psi + y * K;
                        sx[j] = 1;
                    }
                }
                float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                int x = 0;
                for (; x + 8 <= K; x += 8) {
                    float tv[4][8];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int u = 0; u < 8; ++u) tv[j][u] = T[j][(x + u) * sx[j]];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int u = 0; u < 8; ++u) acc[j] = fmaf(tv[j][u], g[j][x + u], acc[j]);
                }
                if (x < K) {
                    // the last states in one predicated step
                    float tv[4][8];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int u = 0; u < 8; ++u) tv[j][u] = x + u < K ? T[j][(x + u) * sx[j]] : 0.0f;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (x + u >= K) break;
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[j] = fmaf(tv[j][u], g[j][x + u], acc[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c0 + tid + j * kBlock < P) l.C[o[j]] = acc[j];
            }
        }
        __syncthreads();

        // 4. normalisation, residual, frontier decision, stores
        for (int q = tid; q < ns; q += kBlock) {
            const float* c = l.C + q * KS;
            float z = 0.0f;
            for (int y = 0; y < K; ++y) z += c[y];
            l.inv[q] = 1.0f / z;
        }
        const long long e0 = (long long)sc * K;  // the tile's rows are contiguous
        // entry i of the tile's own rows (row q)
        auto old_entry = [&](int i, int q) {
            float v = m_in[e0 + i];
            if (fr.on) {
                if (fr.alt && (__float_as_uint(m_in[e0 + q * K]) >> 31)) v = fr.alt[e0 + i];
                v = fabsf(v);
            }
            return v;
        };
        __syncthreads();
        for (int c0 = 0; c0 < P; c0 += U * kBlock) {
            float old[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = min(c0 + tid + j * kBlock, P - 1);
                old[j] = old_entry(i, row_of(i));
            }
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = c0 + tid + j * kBlock;
                if (i >= P) continue;
                const int q = row_of(i), o = q * KS + (i - q * K);
                const float v = l.C[o] * l.inv[q];
                l.C[o] = v;
                l.G[o] = fabsf(v - old[j]);
            }
        }
        __syncthreads();
        for (int q = tid; q < ns; q += kBlock) {
            const float* d = l.G + q * KS;
            float r = 0.0f;
            for (int y = 0; y < K; ++y) r = fmaxf(r, d[y]);
            const bool active = r > a.eps;
            rmax = fmaxf(rmax, r);
            act += active;
            if (MODE == kModeRnBP) {
                bool ka = false, kb = false;
                if (active) {
                    const int v = l.owner[q];
                    const unsigned int u24 = draw24(a, n0 + v, base + q - l.ptr[v]);
                    ka = u24 < a.thr_a;
                    kb = u24 < a.thr_b;
                }
                sa += ka;
                sb += kb;
                l.keep[q] = (ka ? 1u : 0u) | (kb ? 2u : 0u);
            }
            if (MODE == kModeRBP) a.keys[sc + q] = __float_as_uint(r);
        }
        if (MODE == kModeRnBP) __syncthreads();
        if (MODE != kModeEvalOnly) {
            for (int c0 = 0; c0 < P; c0 += U * kBlock) {
                float old[U];
                if (MODE == kModeRnBP) {
#pragma unroll
                    for (int j = 0; j < U; ++j) {
                        const int i = min(c0 + tid + j * kBlock, P - 1);
                        old[j] = old_entry(i, row_of(i));
                    }
                }
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const int i = c0 + tid + j * kBlock;
                    if (i >= P) continue;
                    const int q = row_of(i), y = i - q * K;
                    const float v = l.C[q * KS + y];
                    if (MODE == kModeLBP) {
                        a.out_buf[0][e0 + i] = v;
                    } else if (MODE == kModeRBP) {
                        a.cand[e0 + i] = v;
                    } else {
                        const unsigned int kp2 = l.keep[q];
                        const bool ka = kp2 & 1u, kb = kp2 & 2u;
                        if (a.row_flags) {
                            // the whole row of outcome p_out, the other where they differ
                            const bool kp = p_out == 0 ? ka : kb, ko = p_out == 0 ? kb : ka;
                            const bool diff = ka != kb;
                            const float f = kp ? v : old[j];
                            a.out_buf[p_out][e0 + i] = y == 0 ? flag_first(f, diff) : f;
                            if (diff) a.out_buf[p_out ^ 1][e0 + i] = ko ? v : old[j];
                        } else {
                            a.out_buf[0][e0 + i] = ka ? v : old[j];
                        }
                    }
                }
            }
        }
    }
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// Closes the last evaluation of a run (one wave): the same bookkeeping the
// next evaluation's prologue would do.  With `host` (pinned memory) it also copies
// the state's leading words there, which a readback would take a launch for.
__global__ void k_close_run(EvalArgs a, unsigned int* host, int words) {
    if (!a.st->done) {
        CtrLoad c;
        ctr_load(a, true, c);
        unsigned long long n1;
        long long n2;
        wave_close(a, true, c, n1, n2);
    }
    if (!host) return;
    __threadfence();  // lane 0's stores and adds, before the lanes read them from L2
    const unsigned int* st = (const unsigned int*)a.st;
    for (int i = threadIdx.x; i < words; i += 64)
        host[i] = __hip_atomic_load(&st[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_init_state(DevState* st, int nw, CounterLine* ctr) {
    unsigned int* w = (unsigned int*)st;
    for (int i = threadIdx.x; i < nw; i += blockDim.x) w[i] = 0u;
    unsigned int* c = (unsigned int*)ctr;
    const int nc = (int)(4 * kCounterCopies * sizeof(CounterLine) / sizeof(unsigned int));
    for (int i = threadIdx.x; i < nc; i += blockDim.x) c[i] = 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        st->conv_t = -1;
        st->last_prev = -1;
    }
}

__global__ void k_fill(float* p, float v, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Eq. (3): beliefs from the node aggregate.
// ---------------------------------------------------------------------------
__global__ void k_marginals_logodds(const int* node_ptr, const int* rev, const float* unary,
                                    const float* lam, float* out, int N) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float L = unary[n];
    for (int s = node_ptr[n]; s < node_ptr[n + 1]; ++s) L += lam[rev[s]];
    out[2 * (long long)n + 1] = 1.0f / (1.0f + expf(-L));
    out[2 * (long long)n + 0] = 1.0f / (1.0f + expf(L));
}

// Wave-wide max and sum (every lane gets the result).
__device__ __forceinline__ float wave_max_f(float v) {
    const int id = __float_as_int(-INFINITY);
    auto step = [&](float x, int moved) { return fmaxf(x, __int_as_float(moved)); };
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowShr1, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowShr2, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowShr4, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowShr8, 0xF, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowBcast15, 0xA, 0xF, false));
    v = step(v, __builtin_amdgcn_update_dpp(id, __float_as_int(v), kRowBcast31, 0xC, 0xF, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Eq. (3) for the [E][K] layout: a group of W lanes per variable, V states per lane
// (V = 4 and 16-byte loads where K is a multiple of four, else 1; W = K / V rounded
// up to a power of two, 64 / W variables per wave); the logs of K m are summed in
// slot order, as the evaluation kernels sum them, four rows in flight.  Bound by
// the instructions around the logs: with a state per lane, eight rows per round
// (a grid has four) and the row numbers by shuffles it took 71 us on a 500 x 500
// grid with K = 32, now 30 us.  Shuffles stay inside the group, whose lanes run
// the same loop trips.
template <int V>
__global__ void k_marginals_generic(const int* node_ptr, const int* rev, const float* unary,
                                    const float* m, float* out, int N, int K, int wl) {
    constexpr int kRows = 4;
    const int lane = threadIdx.x & 63;
    const int W = 1 << wl;
    const int G = 64 >> wl;  // variables per wave
    const int x = (lane & (W - 1)) * V;
    const bool on = x < K;
    const int xc = on ? x : 0;
    const float fK = (float)K;
    const long long waves = (long long)gridDim.x * (blockDim.x >> 6);
    const long long w0 = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    auto load = [&](const float* p, float* v) {
        if (V == 4) {
            const float4 t = *(const float4*)p;
            v[0] = t.x;
            v[V > 1 ? 1 : 0] = t.y;
            v[V > 2 ? 2 : 0] = t.z;
            v[V > 3 ? 3 : 0] = t.w;
        } else {
            v[0] = *p;
        }
    };
    for (long long n0 = w0 * G; n0 < N; n0 += waves * G) {
        const int n = (int)(n0 + (lane >> wl));
        if (n < N) {
            float acc[V];
            load(unary + (long long)n * K + xc, acc);
            const int s0 = node_ptr[n], s1 = node_ptr[n + 1];
            for (int c = s0; c < s1; c += kRows) {
                int r[kRows];
                float v[kRows * V];
#pragma unroll
                for (int u = 0; u < kRows; ++u) r[u] = rev[min(c + u, s1 - 1)];
#pragma unroll
                for (int u = 0; u < kRows; ++u) load(m + (long long)r[u] * K + xc, v + u * V);
#pragma unroll
                for (int u = 0; u < kRows * V; ++u) v[u] *= fK;
                log_batch<kRows * V>(v);
#pragma unroll
                for (int u = 0; u < kRows; ++u)
                    if (c + u < s1) {
#pragma unroll
                        for (int i = 0; i < V; ++i) acc[i] += v[u * V + i];
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < V; ++i) mx = fmaxf(mx, on ? acc[i] : -INFINITY);
            for (int o = W >> 1; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
            float e[V];
#pragma unroll
            for (int i = 0; i < V; ++i) e[i] = on ? expf(acc[i] - mx) : 0.0f;
            // the sum in one order whatever V: states 1 apart are added last, as the
            // halving shuffles over single states add them
            float z = 0.0f;
            if (V == 4) {
                float p[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    p[i] = e[i];
                    for (int o = W >> 1; o > 0; o >>= 1) p[i] += __shfl_xor(p[i], o, 64);
                }
                z = (p[0] + p[V > 2 ? 2 : 0]) + (p[V > 1 ? 1 : 0] + p[V > 3 ? 3 : 0]);
            } else {
                z = e[0];
                for (int o = W >> 1; o > 0; o >>= 1) z += __shfl_xor(z, o, 64);
            }
            if (on) {
                float* po = out + (long long)n * K + x;
                if (V == 4)
                    *(float4*)po = make_float4(e[0] / z, e[V > 1 ? 1 : 0] / z, e[V > 2 ? 2 : 0] / z,
                                               e[V > 3 ? 3 : 0] / z);
                else
                    *po = e[0] / z;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Variables with their own numbers of states (ragged layout, Sec. II-A with
// K_i states per variable, as in the side-chain models of Sec. IV-E): the
// message i -> j holds K_j floats at moff[slot], the table of slot i -> j is
// K_i x K_j (x_i major) at toff[slot], the unary of i is K_i floats at uoff[i].
// Every slot has its own table, so Eq. (2) is a vector-matrix product whose
// table entries are each used once per iteration: 2 flops per 4-byte table
// entry, far below the ridge of the matrix cores and of the vector units, so
// the vector units take it and the kernel is bound by the table traffic.
//
// One wave per source variable (grid-stride over records ordered by work, the
// largest first): lane x holds the aggregate of states x and x + 64 (K_i <= 128);
// the cavity of each outgoing slot, g(x_i) = exp(A(x_i) - log m_{j->i}(x_i) - max),
// goes to LDS.  Then every (slot, target state) pair of the variable gets a lane,
// which takes the product with its slot's table as a chain of fused multiply-adds
// over the source states (the table entries of consecutive lanes are contiguous; a
// lane runs four pairs together, 32 loads in flight); a lane per slot forms the
// normalisation and the frontier decision, the pair lanes the change and the
// committed values.
//
// What bounds a wave is its chain of dependent steps, so: everything a variable
// needs to know comes in one record and its slots' offsets in one load each (row
// of the incoming message, table, outputs); the first table entries, which depend
// on no message, are requested before the incoming rows; the slot of a pair is one
// LDS byte; maxima over the wave go through DPP; a slot's sum reads eight outputs
// at a time; its largest change is an LDS integer maximum.  8,000 variables, mean
// degree 8, 2..81 states: 106 -> 46 us per sweep (116 MB of tables: 25 us at
// the rate of a large copy, 15 at that of one the Infinity Cache holds).  A heavy variable (slots over the wave's LDS, or much product
// work: ragged_flat) gives each of its slots a wave of its own (ragged_slot),
// taken before the other variables, so the launch is not held up by one wave that
// runs a long chain of table loads.
// ---------------------------------------------------------------------------

// Wave-local LDS hand-off: this wave's LDS stores are complete and visible to
// its other lanes (a wave executes its LDS operations in order).
__device__ __forceinline__ void wave_lds_sync() { __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int MODE>
__device__ __forceinline__ void ragged_commit(const EvalArgs& a, int q, float v, float old, bool ka,
                                              bool kb) {
    if (MODE == kModeLBP) {
        a.out_buf[0][q] = v;
    } else if (MODE == kModeRnBP) {
        a.out_buf[0][q] = ka ? v : old;
        if (a.two_outputs) a.out_buf[1][q] = kb ? v : old;
    } else if (MODE == kModeRBP) {
        a.cand[q] = v;
    }
}

// One slot i -> j of a heavy variable on one wave: the aggregate of i over all
// its incoming rows (lanes over source states, rows eight at a time, summed in
// slot order as the flat path sums them), the cavity of j's row, then the
// product with the slot's table.  For K_j <= 64 the wave covers R = 64 / K_j
// table rows per step: lane r K_j + y reads entry (step R + r) K_j + y, so each
// load is one contiguous run of the table, eight steps in flight, and the R
// partial sums of each target state are added through LDS.  For larger K_j,
// lanes take target states y and y + 64 over all source states.
template <int MODE>
__device__ __forceinline__ void ragged_slot(const EvalArgs& a, const float* __restrict__ m_in, int s,
                                            int i, float* G, float* Cv, float& rmax,
                                            unsigned int& act, unsigned int& sa, unsigned int& sb) {
    const int lane = threadIdx.x & 63;
    const int Ki = a.kv[i];
    const int s0 = a.node_ptr[i], s1 = a.node_ptr[i + 1];
    const float fK = (float)Ki;
    const bool x0 = lane < Ki, x1 = lane + 64 < Ki;
    const float* U = a.unary + a.uoff[i];
    const int mo = a.moff[s], Kj = a.moff[s + 1] - mo;
    const float* __restrict__ T = a.pair + a.toff[s];
    const int rj = a.rin[s];
    const bool y0 = lane < Kj, y1 = lane + 64 < Kj;
    const float old0 = y0 ? m_in[mo + lane] : 0.0f;
    const float old1 = y1 ? m_in[mo + lane + 64] : 0.0f;
    float A0 = x0 ? U[lane] : 0.0f, A1 = x1 ? U[lane + 64] : 0.0f;
    for (int b = s0; b < s1; b += 64) {
        const int nb = min(64, s1 - b);
        const int my_rin = lane < nb ? a.rin[b + lane] : 0;
        for (int k0 = 0; k0 < nb; k0 += 8) {
            float v0[8], v1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int rin = __shfl(my_rin, min(k0 + j, nb - 1), 64);
                v0[j] = x0 ? m_in[rin + lane] : 1.0f;
                v1[j] = x1 ? m_in[rin + lane + 64] : 1.0f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) v0[j] *= fK;
            log_batch<8>(v0);
            if (Ki > 64) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v1[j] *= fK;
                log_batch<8>(v1);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (k0 + j >= nb) break;
                if (x0) A0 += v0[j];
                if (x1) A1 += v1[j];
            }
        }
    }
    const float c0 = x0 ? A0 - logf(fK * m_in[rj + lane]) : -INFINITY;
    const float c1 = x1 ? A1 - logf(fK * m_in[rj + lane + 64]) : -INFINITY;
    const float mx = wave_max_f(fmaxf(c0, c1));
    if (x0) G[lane] = expf(c0 - mx);
    if (x1) G[lane + 64] = expf(c1 - mx);
    wave_lds_sync();
    float o0 = 0.0f, o1 = 0.0f;
    if (Kj <= 64) {
        const int R = 64 / Kj;
        const int r = lane / Kj;
        const int RK = R * Kj;
        const int steps = (Ki + R - 1) / R;
        float acc = 0.0f;
        int st = 0;
        for (; st + 16 <= steps; st += 16) {
            float tv[16], gv[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int x = (st + u) * R + r;
                const bool ok = lane < RK && x < Ki;
                tv[u] = ok ? T[(st + u) * RK + lane] : 0.0f;
                gv[u] = ok ? G[x] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) acc = fmaf(tv[u], gv[u], acc);
        }
        for (; st < steps; st += 8) {
            // the remaining steps, predicated, eight loads together
            float tv[8], gv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int x = (st + u) * R + r;
                const bool ok = st + u < steps && lane < RK && x < Ki;
                tv[u] = ok ? T[(st + u) * RK + lane] : 0.0f;
                gv[u] = ok ? G[x] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(tv[u], gv[u], acc);
        }
        Cv[lane] = acc;
        wave_lds_sync();
        if (y0)
            for (int q = 0; q < R; ++q) o0 += Cv[q * Kj + lane];
    } else {
        int x = 0;
        for (; x + 8 <= Ki; x += 8) {
            float t0[8], t1[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                t0[u] = T[(x + u) * Kj + lane];
                t1[u] = y1 ? T[(x + u) * Kj + lane + 64] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float gx = G[x + u];
                o0 = fmaf(t0[u], gx, o0);
                o1 = fmaf(t1[u], gx, o1);
            }
        }
        if (x < Ki) {
            float t0[8], t1[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool ok = x + u < Ki;
                t0[u] = ok ? T[(x + u) * Kj + lane] : 0.0f;
                t1[u] = ok && y1 ? T[(x + u) * Kj + lane + 64] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (x + u >= Ki) break;
                const float gx = G[x + u];
                o0 = fmaf(t0[u], gx, o0);
                o1 = fmaf(t1[u], gx, o1);
            }
        }
    }
    const float z = wave_sum_f(o0 + o1);
    o0 /= z;
    o1 /= z;
    const float res = wave_max_f(fmaxf(y0 ? fabsf(o0 - old0) : 0.0f, y1 ? fabsf(o1 - old1) : 0.0f));
    const bool active = res > a.eps;
    bool ka = false, kb = false;
    if (MODE == kModeRnBP && active) {
        const unsigned int u24 = draw24(a, i, s - s0);
        ka = u24 < a.thr_a;
        kb = u24 < a.thr_b;
    }
    if (y0) ragged_commit<MODE>(a, mo + lane, o0, old0, ka, kb);
    if (y1) ragged_commit<MODE>(a, mo + lane + 64, o1, old1, ka, kb);
    if (lane == 0) {
        if (MODE == kModeRBP) a.keys[s] = __float_as_uint(res);
        act += active;
        sa += ka;
        sb += kb;
        rmax = fmaxf(rmax, res);
    }
    wave_lds_sync();  // G and Cv are free for the wave's next slot
}

// The LDS of one wave of the flat path (four blocks of four waves per CU).
struct RaggedLds {
    float G[kRaggedFlat];                  // logs, then cavity vectors, slot-major; then old values
    float C[kRaggedFlat];                  // aggregate; then outputs of the variable's slots
    unsigned char slot[kRaggedFlat];       // slot of an output
    int toff[kRaggedMaxDeg];               // table of the slot
    union {
        int rin[kRaggedMaxDeg];            // row of the message into the variable
        float inv[kRaggedMaxDeg];          // 1 / z
    };
    unsigned int r[kRaggedMaxDeg];         // residual bits, then the keep decisions
    unsigned short off[kRaggedMaxDeg + 1]; // first output of the slot
};
static_assert(kRaggedMaxDeg <= 64, "a lane per slot");

// Largest value of each row of 16 lanes, in all of them.
__device__ __forceinline__ float row_max_f(float v) {
    auto ror = [](float x, auto ctrl) {
        return __int_as_float(
            __builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    v = fmaxf(v, ror(v, std::integral_constant<int, 0x128>{}));  // row_ror 8, 4, 2, 1
    v = fmaxf(v, ror(v, std::integral_constant<int, 0x124>{}));
    v = fmaxf(v, ror(v, std::integral_constant<int, 0x122>{}));
    return fmaxf(v, ror(v, std::integral_constant<int, 0x121>{}));
}

// One variable (record f) on NW waves: a wave of its own, or the whole block.
template <int MODE, int NW>
__device__ __forceinline__ void ragged_var(const EvalArgs& a, const float* __restrict__ m_in, int f,
                                           RaggedLds& l, float& rmax, unsigned int& act,
                                           unsigned int& sa, unsigned int& sb) {
    constexpr int NT = 64 * NW;
    constexpr int PJ = NW == 1 ? 4 : 2, XS = 32 / PJ;  // pairs of a lane, states per step
    const int lane = threadIdx.x & 63;
    const int wv = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lid = 64 * wv + lane;  // lane of the group
    auto sync = [&]() {
        if (NW == 1)
            wave_lds_sync();
        else
            lds_barrier();
    };
    const int4 va = ((const int4*)a.vrec)[2 * f], vb = ((const int4*)a.vrec)[2 * f + 1];
    const int s0 = __builtin_amdgcn_readfirstlane(va.x), deg = __builtin_amdgcn_readfirstlane(va.y);
    const int Ki = __builtin_amdgcn_readfirstlane(va.z), uo = __builtin_amdgcn_readfirstlane(va.w);
    const int mo0 = __builtin_amdgcn_readfirstlane(vb.x), P = __builtin_amdgcn_readfirstlane(vb.y);
    const int i = __builtin_amdgcn_readfirstlane(vb.z);
    const unsigned int magic = (unsigned int)__builtin_amdgcn_readfirstlane(vb.w);
    if (deg == 0) return;
    const float* U = a.unary + uo;
    const float fK = (float)Ki;  // log(K_i m) keeps the aggregate near zero
    const bool x0 = lane < Ki, x1 = lane + 64 < Ki;
    // a lane per slot: the row of the message into the variable, the table,
    // the first output
    const int sl = s0 + min(lane, deg - 1);
    const int rin_k = a.rin[sl];
    const int to_k = a.toff[sl];
    const int off_k = lane < deg ? a.moff[sl] - mo0 : P;
    float A0 = x0 ? U[lane] : 0.0f, A1 = x1 ? U[lane + 64] : 0.0f;
    if (lid <= deg && lid < 64) l.off[lid] = (unsigned short)off_k;
    if (lid == 0) l.off[deg] = (unsigned short)P;
    if (lid < deg) {
        l.rin[lid] = rin_k;
        l.toff[lid] = to_k;
        l.r[lid] = 0u;
    }
    for (int k = wv; k < deg; k += NW) {
        const int o = __builtin_amdgcn_readlane(off_k, k);
        const int e = k + 1 < deg ? __builtin_amdgcn_readlane(off_k, min(k + 1, 63)) : P;
        for (int q = o + lane; q < e; q += 64) l.slot[q] = (unsigned char)k;
    }
    sync();
    // the pairs of a lane: PJ, NT apart, of each PJ NT (a wave skips what lies past P)
    const float* T[PJ];
    const float* g[PJ];
    int Kj[PJ];
    float tv[PJ][XS];
    auto pairs = [&](int pb) {
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
            const int pp = min(pb + lid + NT * j, P - 1);
            const int k = l.slot[pp];
            const int o = l.off[k];
            Kj[j] = l.off[k + 1] - o;
            T[j] = a.pair + l.toff[k] + (pp - o);
            g[j] = l.G + k * Ki;
        }
    };
    // table rows x .. x + XS - 1 of every pair (rows past the last: the last again)
    auto load_tables = [&](int pb, int x) {
        if (x + XS <= Ki) {
#pragma unroll
            for (int j = 0; j < PJ; ++j) {
                if (pb + 64 * wv + NT * j >= P) break;
                const float* t = T[j] + x * Kj[j];
#pragma unroll
                for (int u = 0; u < XS; ++u) {
                    tv[j][u] = *t;
                    t += Kj[j];
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < PJ; ++j) {
                if (pb + 64 * wv + NT * j >= P) break;
#pragma unroll
                for (int u = 0; u < XS; ++u) tv[j][u] = T[j][min(x + u, Ki - 1) * Kj[j]];
            }
        }
    };
    pairs(0);
    load_tables(0, 0);
    // logs of the incoming rows, lane by entry: slot q = e / K_i, state e - q K_i
    const int DK = deg * Ki;
    constexpr int RU = NW == 1 ? 4 : 2;
    for (int e0 = 0; e0 < DK; e0 += RU * NT) {
        float v[RU];
#pragma unroll
        for (int j = 0; j < RU; ++j) {
            const int e = min(e0 + lid + NT * j, DK - 1);
            const int q = (int)(((unsigned int)e * magic) >> 20);
            v[j] = m_in[l.rin[q] + (e - q * Ki)];
        }
#pragma unroll
        for (int j = 0; j < RU; ++j) v[j] *= fK;
        log_batch<RU>(v);
#pragma unroll
        for (int j = 0; j < RU; ++j) {
            const int e = e0 + lid + NT * j;
            if (e < DK) l.G[e] = v[j];
        }
    }
    sync();
    // the aggregate, in slot order
    if (wv == 0) {
        for (int k0 = 0; k0 < deg; k0 += 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = l.G[min(k0 + j, deg - 1) * Ki + min(lane, Ki - 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k0 + j < deg) A0 += v[j];
            if (Ki > 64) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    v[j] = l.G[min(k0 + j, deg - 1) * Ki + min(lane + 64, Ki - 1)];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k0 + j < deg) A1 += v[j];
            }
        }
        if (x0) l.C[lane] = A0;
        if (x1) l.C[lane + 64] = A1;
    }
    sync();
    // the cavities, W lanes per slot (K_i rounded up to 16, 32 or 64)
    {
        const int wl = Ki <= 16 ? 4 : Ki <= 32 ? 5 : 6;
        const int x = lid & ((1 << wl) - 1);
        for (int k = lid >> wl; k < deg; k += NT >> wl) {
            float* G = l.G + k * Ki;
            const float c0 = x < Ki ? l.C[x] - G[x] : -INFINITY;
            const float c1 = Ki > 64 && x + 64 < Ki ? l.C[x + 64] - G[x + 64] : -INFINITY;
            float mx = row_max_f(fmaxf(c0, c1));
            if (wl > 4) mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            if (wl > 5) mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (x < Ki) G[x] = expf(c0 - mx);
            if (Ki > 64 && x + 64 < Ki) G[x + 64] = expf(c1 - mx);
        }
    }
    sync();
    for (int pb = 0; pb < P; pb += PJ * NT) {
        if (pb) {
            pairs(pb);
            load_tables(pb, 0);
        }
        float acc[PJ];
#pragma unroll
        for (int j = 0; j < PJ; ++j) acc[j] = 0.0f;
        // XS source states per step, the last step cut short
        for (int x = 0; x < Ki; x += XS) {
            if (x) load_tables(pb, x);
            if (x + XS <= Ki) {
#pragma unroll
                for (int j = 0; j < PJ; ++j) {
                    if (pb + 64 * wv + NT * j >= P) break;
#pragma unroll
                    for (int u = 0; u < XS; ++u) acc[j] = fmaf(tv[j][u], g[j][x + u], acc[j]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < XS - 1; ++u) {
                    if (x + u >= Ki) break;
#pragma unroll
                    for (int j = 0; j < PJ; ++j) acc[j] = fmaf(tv[j][u], g[j][x + u], acc[j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < PJ; ++j)
            if (pb + lid + NT * j < P) l.C[pb + lid + NT * j] = acc[j];
    }
    sync();
    if (lid < deg) {
        const int o = l.off[lid], n = l.off[lid + 1] - o;
        float z = 0.0f;
        for (int q = 0; q < n; q += 8) {
            float c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = l.C[o + min(q + u, n - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) z += q + u < n ? c[u] : 0.0f;
        }
        l.inv[lid] = 1.0f / z;
    }
    sync();
    // normalised outputs back into C, old values into G (the cavities are
    // done), the largest change of each slot
    for (int pb = 0; pb < P; pb += PJ * NT) {
        float old[PJ];
#pragma unroll
        for (int j = 0; j < PJ; ++j) old[j] = m_in[mo0 + min(pb + lid + NT * j, P - 1)];
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
            const int p = pb + lid + NT * j;
            if (p >= P) continue;
            const int k = l.slot[p];
            const float v = l.C[p] * l.inv[k];
            l.C[p] = v;
            const float d = fabsf(v - old[j]);
            if (d > 0.0f) atomicMax(&l.r[k], __float_as_uint(d));  // (not for NaN)
            if (MODE == kModeRnBP) l.G[p] = old[j];
        }
    }
    sync();
    if (lid < deg) {
        const float r = __uint_as_float(l.r[lid]);
        const bool active = r > a.eps;
        bool ka = false, kb = false;
        if (MODE == kModeRnBP && active) {
            const unsigned int u24 = draw24(a, i, lid);
            ka = u24 < a.thr_a;
            kb = u24 < a.thr_b;
        }
        if (MODE == kModeRBP) a.keys[s0 + lid] = __float_as_uint(r);
        l.r[lid] = (ka ? 1u : 0u) | (kb ? 2u : 0u);
        act += active;
        sa += ka;
        sb += kb;
        rmax = fmaxf(rmax, r);
    }
    if (MODE == kModeRnBP) sync();
    if (MODE != kModeEvalOnly) {
        for (int p = lid; p < P; p += NT) {
            const unsigned int kp = MODE == kModeRnBP ? l.r[l.slot[p]] : 0u;
            ragged_commit<MODE>(a, mo0 + p, l.C[p], MODE == kModeRnBP ? l.G[p] : 0.0f, kp & 1u,
                                kp & 2u);
        }
    }
    sync();  // the LDS is free for the next variable
}

template <int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_ragged(
    EvalArgs a) {
    __shared__ RedScratch red;
    __shared__ unsigned long long s_red[2];
    __shared__ RaggedLds s_l[kBlock / 64];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const float* __restrict__ m_in = iteration_prologue(a, s_red, blockIdx.x == 0);
    if (!m_in) return;
    float rmax = 0.0f;
    unsigned int act = 0, sa = 0, sb = 0;
    // work items in turn over the blocks: four heavy slots, or one wide variable, or
    // four other variables
    constexpr int W = kBlock / 64;
    const int nh = (a.num_heavy + W - 1) / W, nw = a.num_wide;
    const int items = nh + nw + (a.num_flat - nw + W - 1) / W;
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        if (it < nh) {
            const int h = it * W + w;
            if (h < a.num_heavy)
                ragged_slot<MODE>(a, m_in, a.heavy[2 * h], a.heavy[2 * h + 1], s_l[w].G, s_l[w].C,
                                  rmax, act, sa, sb);
        } else if (it < nh + nw) {
            lds_barrier();  // the waves of the block leave their own variables
            ragged_var<MODE, W>(a, m_in, it - nh, s_l[0], rmax, act, sa, sb);
        } else {
            const int f = nw + (it - nh - nw) * W + w;
            if (f < a.num_flat) ragged_var<MODE, 1>(a, m_in, f, s_l[w], rmax, act, sa, sb);
        }
    }
    block_accumulate(&red, a.ctr, a.t, rmax, act, sa, sb);
}

// Eq. (3) for the ragged layout: one wave per variable.
__global__ __launch_bounds__(kBlock) void k_marginals_ragged(EvalArgs a, float* out) {
    const float* __restrict__ m = a.in_buf[0];
    const int lane = threadIdx.x & 63;
    const int waves = (int)(gridDim.x * (blockDim.x >> 6));
    for (int i = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); i < a.num_nodes;
         i += waves) {
        const int Ki = a.kv[i];
        const float* U = a.unary + a.uoff[i];
        const float fK = (float)Ki;
        const bool x0 = lane < Ki, x1 = lane + 64 < Ki;
        float A0 = x0 ? U[lane] : -INFINITY, A1 = x1 ? U[lane + 64] : -INFINITY;
        for (int s = a.node_ptr[i]; s < a.node_ptr[i + 1]; ++s) {
            const int rin = a.rin[s];
            if (x0) A0 += logf(fK * m[rin + lane]);
            if (x1) A1 += logf(fK * m[rin + lane + 64]);
        }
        const float mx = wave_max_f(fmaxf(A0, A1));
        const float e0 = x0 ? expf(A0 - mx) : 0.0f, e1 = x1 ? expf(A1 - mx) : 0.0f;
        const float z = wave_sum_f(e0 + e1);
        if (x0) out[a.uoff[i] + lane] = e0 / z;
        if (x1) out[a.uoff[i] + lane + 64] = e1 / z;
    }
}

// The uniform start state: 1 / K_j in every entry of message i -> j.
__global__ void k_fill_ragged(float* m, const int* moff, int E) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < E; e += gridDim.x * blockDim.x) {
        const int q0 = moff[e], q1 = moff[e + 1];
        const float v = 1.0f / (float)(q1 - q0);
        for (int q = q0; q < q1; ++q) m[q] = v;
    }
}

// ---------------------------------------------------------------------------
// Sparse re-evaluation (K = 2 log-odds layout, RnBP), messages committed in
// place.  The candidate of Eq. (2) for i -> j depends only on the messages into
// i (and on i's own old value for the residual), so after a commit only the
// messages out of nodes that received a committed message ("dirty" nodes) can
// change.  Every other stored candidate and residual is, bit for bit, what a
// full evaluation would compute again: the same arithmetic on the same inputs,
// and a committed message whose source is clean has candidate = message and
// residual 0.
//
// n_t is carried as a running count: the evaluation adds, per re-evaluated
// slot, (new residual > eps) - (old residual > eps), and the commit subtracts
// the committed slots; both add into counter set t & 3 of the iteration whose
// count they change, and the commit of iteration t reads
// n_t = n_{t-1} + (sum of set t & 3).  R_t is only reported for the last
// evaluation of a run, so it is taken once, over the stored residuals, after
// the run.  A node flag records whether any of the node's slots is active, so
// the commit visits only such nodes.
// ---------------------------------------------------------------------------
constexpr int kSparseChunk = 4;  // slots per group of loads (= words of one Philox call)
constexpr int kSparseGridMax = 1024;  // blocks of the residual-max pass

__device__ __forceinline__ int sparse_grid_stride() { return (int)(gridDim.x * blockDim.x); }

// Block sum of a signed and an unsigned per-thread count, added into counter
// copy (blockIdx & 63) of set `set`: the signed one into its active count
// (wrapping modulo 2^64), the unsigned one into sel_a (evaluated slots) or,
// with `committed`, into sel_b.
__device__ __forceinline__ void sparse_accumulate(CounterLine* ctr, unsigned int set, int d,
                                                  unsigned int ev, int* s_d, unsigned int* s_ev,
                                                  bool committed) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        d += __shfl_xor(d, o, 64);
        ev += __shfl_xor(ev, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_d[threadIdx.x >> 6] = d;
        s_ev[threadIdx.x >> 6] = ev;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        long long D = 0;
        unsigned long long EV = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            D += s_d[w];
            EV += s_ev[w];
        }
        CounterLine* c = ctr + (set & 3u) * kCounterCopies + (blockIdx.x & (kCounterCopies - 1));
        if (D) atomicAdd(&c->active, (unsigned long long)D);
        if (EV) atomicAdd(committed ? &c->sel_b : &c->sel_a, EV);
    }
}

// Operands of up to four consecutive slots c .. c+3 of a node ending at s1
// (indices clamped into the node, so the loads are unconditional).
struct SparseChunk {
    float lin[kSparseChunk], J[kSparseChunk], old[kSparseChunk];
    unsigned int key[kSparseChunk];
};

__device__ __forceinline__ void sparse_load_lin(const EvalArgs& a, const float* m, int c, int s1,
                                                float* lin) {
#pragma unroll
    for (int k = 0; k < kSparseChunk; ++k) lin[k] = m[a.rev[min(c + k, s1 - 1)]];
}

__device__ __forceinline__ void sparse_load_chunk(const EvalArgs& a, const float* m, int c, int s1,
                                                  SparseChunk& d) {
#pragma unroll
    for (int k = 0; k < kSparseChunk; ++k) {
        const int e = min(c + k, s1 - 1);
        d.lin[k] = m[a.rev[e]];
        d.J[k] = a.coupling[e];
        d.old[k] = m[e];
        d.key[k] = a.keys[e];
    }
}

__device__ __forceinline__ void sparse_eval_chunk(const EvalArgs& a, float L, int c, int s1,
                                                  const SparseChunk& d, unsigned int& act,
                                                  unsigned int& old_act) {
    unsigned int unused = 0;
#pragma unroll
    for (int k = 0; k < kSparseChunk; ++k) {
        if (c + k >= s1) break;
        old_act += (!a.sp_first && __uint_as_float(d.key[k]) > a.eps) ? 1u : 0u;
        logodds_slot<kModeRBP>(a, OutPtr{a}, L, d.lin[k], d.J[k], d.old[k], c + k, 0u, act, unused,
                               unused);
    }
}

// Iteration t, evaluation: the slots of every dirty node are evaluated again
// (the incoming messages are summed in slot order, as the tiled kernel sums
// them; operands are loaded four slots at a time, and a node of at most four
// slots is evaluated from one set of loads).  sp_first: the first sparse
// iteration of a run, whose stored residuals are not yet valid (counted as 0).
__global__ __launch_bounds__(kBlock) void k_sparse_eval(EvalArgs a) {
    __shared__ int s_d[kBlock / 64];
    __shared__ unsigned int s_ev[kBlock / 64];
    // (the flag, the slot range and the unary are requested together, and the done
    // flag with them: a node's chain is then three round trips, not five)
    const unsigned int done = a.st->done;
    const float* __restrict__ m = a.in_buf[0];
    int delta = 0;
    unsigned int ev = 0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < a.num_nodes; i += sparse_grid_stride()) {
        const unsigned char dirty = a.dirty[i];
        const int s0 = a.node_ptr[i], s1 = a.node_ptr[i + 1];
        const float u = a.unary[i];
        __builtin_amdgcn_sched_barrier(0);
        if (done || !dirty) continue;
        a.dirty[i] = 0;
        unsigned int act = 0, old_act = 0;
        if (s1 > s0) {
            SparseChunk d;
            sparse_load_chunk(a, m, s0, s1, d);
            float L = u;
#pragma unroll
            for (int k = 0; k < kSparseChunk; ++k)
                if (s0 + k < s1) L += d.lin[k];
            for (int c = s0 + kSparseChunk; c < s1; c += kSparseChunk) {
                float lin[kSparseChunk];
                sparse_load_lin(a, m, c, s1, lin);
#pragma unroll
                for (int k = 0; k < kSparseChunk; ++k)
                    if (c + k < s1) L += lin[k];
            }
            sparse_eval_chunk(a, L, s0, s1, d, act, old_act);
            for (int c = s0 + kSparseChunk; c < s1; c += kSparseChunk) {
                sparse_load_chunk(a, m, c, s1, d);
                sparse_eval_chunk(a, L, c, s1, d, act, old_act);
            }
        }
        a.hasact[i] = act ? 1 : 0;
        delta += (int)act - (int)old_act;
        ev += (unsigned int)(s1 - s0);
    }
    if (done) return;
    sparse_accumulate(a.ctr, a.t, delta, ev, s_d, s_ev, false);
}

// Iteration t, commit.  Every block forms n_t and n_{t-1} and takes p_t from
// EdgeRatio = n_t / n_{t-1} (Sec. IV-A); block 0 also closes evaluation t
// (IsConverged, statistics including the commits of iteration t - 1, n_t kept
// for the next iteration) and clears counter set t + 2.  Then the active slots of flagged nodes are drawn (the
// same Philox words as the tiled kernel, one call per four slots) and the kept
// ones committed in place; their targets are marked dirty.  After the last
// allowed commit (after_final) the evaluation is closed and nothing committed.
// Each thread takes one node; its flag, slot range and first four residuals
// are loaded before the counters are summed, so the two latencies overlap.
__global__ __launch_bounds__(kBlock) void k_sparse_commit(EvalArgs a) {
    __shared__ unsigned long long s_n[3];
    __shared__ int s_d[kBlock / 64];
    __shared__ unsigned int s_ev[kBlock / 64];
    // (the node's flag and slot range are requested together)
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int ic = min(i, max(a.num_nodes - 1, 0));
    const unsigned char flag = a.hasact[ic];
    int s0 = a.node_ptr[ic], s1 = a.node_ptr[ic + 1];
    __builtin_amdgcn_sched_barrier(0);
    const bool mine = i < a.num_nodes && flag;
    unsigned int key[kSparseChunk] = {0u, 0u, 0u, 0u};
    if (mine) {
#pragma unroll
        for (int k = 0; k < kSparseChunk; ++k) key[k] = a.keys[min(s0 + k, s1 - 1)];
    }
    // wave 0 reads the done flag once for the block (block 0 may set it during
    // this launch, so the other waves must not read it themselves)
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const unsigned int done = a.st->done;
        const CounterLine* c0 = a.ctr + (a.t & 3u) * kCounterCopies + lane;
        // (a signed change, at most the number of messages either way: below 2^31)
        const long long d = (int)wave_sum32((unsigned int)c0->active);
        const long long base = a.sp_first ? 0ll : (long long)a.st->sp_n[(a.t - 1u) & 3u];
        const unsigned long long n1 = (unsigned long long)(base + d);
        long long n2;
        if (!a.sp_first)
            n2 = (long long)a.st->sp_n[(a.t - 1u) & 3u];
        else if (a.it >= 1)  // switched from the full evaluation: its count of t - 1
            n2 = (long long)wave_sum32((unsigned int)a.ctr[((a.t - 1u) & 3u) * kCounterCopies + lane].active);
        else
            n2 = a.prev_active_host;
        if (blockIdx.x == 0 && !done) {
            const unsigned long long ev = wave_sum32((unsigned int)c0->sel_a);
            // messages committed by iteration t - 1 (none on the first sparse iteration)
            const unsigned long long cm_prev = a.sp_first ? 0ull : wave_sum32((unsigned int)c0->sel_b);
            CounterLine* z = a.ctr + ((a.t + 2u) & 3u) * kCounterCopies + lane;
            z->active = 0ull;
            z->sel_a = 0ull;
            z->sel_b = 0ull;
            z->rmax = 0u;
            if (lane == 0) {
                DevState* st = a.st;
                report_progress(a, (unsigned long long)a.it + 1ull, n1 == 0ull);
                atomicAdd(&st->evaluated, ev);
                atomicAdd(&st->evals, 1ull);
                if (cm_prev) atomicAdd(&st->committed, cm_prev);
                st->sp_n[a.t & 3u] = n1;
                st->last_t = (long long)a.t;
                st->last_active = n1;
                st->last_rmax = 0u;  // taken after the run
                st->last_prev = n2;
                if (n1 == 0ull) {
                    st->done = 1u;
                    st->conv_t = (long long)a.t;
                } else if (!a.after_final) {
                    atomicAdd(&st->iterations, 1ull);
                }
            }
        }
        if (lane == 0) {
            s_n[0] = n1;
            s_n[1] = (unsigned long long)n2;
            s_n[2] = done;
        }
    }
    __syncthreads();
    const unsigned long long n1 = s_n[0];
    if (s_n[2] || n1 == 0ull || a.after_final) return;
    const unsigned int thr = select_outcome(a, n1, (long long)s_n[1]) ? a.thr_b : a.thr_a;
    float* __restrict__ m = a.out_buf[0];
    unsigned int cm = 0;
    if (mine) {
        unsigned int left = 0;
        for (int c = s0; c < s1; c += kSparseChunk) {
            if (c != s0) {
#pragma unroll
                for (int k = 0; k < kSparseChunk; ++k) key[k] = a.keys[min(c + k, s1 - 1)];
            }
            bool any = false;
#pragma unroll
            for (int k = 0; k < kSparseChunk; ++k)
                any |= c + k < s1 && __uint_as_float(key[k]) > a.eps;
            if (!any) continue;
            const uint4 w = philox4((unsigned int)i, (unsigned int)(c - s0) >> 2, a.t, a.key0, a.key1);
            const unsigned int u[kSparseChunk] = {w.x >> 8, w.y >> 8, w.z >> 8, w.w >> 8};
            bool take[kSparseChunk];
            float cv[kSparseChunk];
            int dv[kSparseChunk];
#pragma unroll
            for (int k = 0; k < kSparseChunk; ++k) {
                const bool act = c + k < s1 && __uint_as_float(key[k]) > a.eps;
                take[k] = act && u[k] < thr;
                left += act && !take[k];
                if (take[k]) {
                    cv[k] = a.cand[c + k];
                    dv[k] = a.dst[c + k];
                }
            }
#pragma unroll
            for (int k = 0; k < kSparseChunk; ++k) {
                if (!take[k]) continue;
                m[c + k] = cv[k];
                a.keys[c + k] = 0u;
                a.dirty[dv[k]] = 1;
                ++cm;
            }
        }
        if (!left) a.hasact[i] = 0;
    }
    // the committed slots leave the count of iteration t + 1; their number is
    // added to the statistics when iteration t + 1 is closed
    sparse_accumulate(a.ctr, a.t + 1u, -(int)cm, cm, s_d, s_ev, true);
}

// Per-graph setup: the target of each slot (slot rev[e] carries the reverse
// message, whose target is the source of e), then every node dirty.
__global__ __launch_bounds__(kBlock) void k_sparse_setup(EvalArgs a, int build_dst) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= a.num_nodes) return;
    if (build_dst) {
        for (int e = a.node_ptr[i]; e < a.node_ptr[i + 1]; ++e) a.dst[a.rev[e]] = i;
    }
    a.dirty[i] = 1;
}

// After a sparse run: R_t of its last evaluation, the largest stored residual
// (no commit followed that evaluation, so the stored residuals are its own).
// One atomic per block.
__global__ __launch_bounds__(kBlock) void k_sparse_rmax(EvalArgs a) {
    __shared__ unsigned int s_r[kBlock / 64];
    unsigned int r = 0;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < (long long)a.num_messages;
         e += (long long)gridDim.x * kBlock)
        r = max(r, a.keys[e]);
    r = wave_max32(r);
    if ((threadIdx.x & 63) == 0) s_r[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) r = max(r, s_r[w]);
        if (r) atomicMax(&a.st->last_rmax, r);
    }
}

// ---------------------------------------------------------------------------
// Greedy top-k for frontier residual BP: most-significant-digit radix select
// over the FP32 bit patterns of the residuals (monotone for values >= 0),
// 4 passes of 8 bits, then a commit that takes every key above the threshold
// and the lowest-slot keys equal to it (slots are ordered by (target, source)).
// ---------------------------------------------------------------------------
constexpr int kSelBlock = 256;
constexpr int kCommitChunk = 4096;

// IsConverged for the top-k step: nothing is selected or committed when the
// evaluation of iteration t found no residual above eps.
__global__ void k_rbp_gate(DevState* st, const CounterLine* ctr, int slot) {
    const unsigned int n = wave_sum32((unsigned int)ctr[slot * kCounterCopies + threadIdx.x].active);
    if (threadIdx.x == 0) st->rbp_skip = (st->done || n == 0u) ? 1u : 0u;
}

// Keys per thread of a histogram pass and positions per thread of the tie
// count and the commit: loaded as four 16-byte vectors, so that a thread's
// loads are all in flight at once.
constexpr int kSelPer = 16;
constexpr int kHistGrid = 1024;  // most blocks of a histogram pass
static_assert(kCommitChunk == kSelBlock * kSelPer, "one commit chunk per block");

// The keys (or slot indices) base[q0 .. q0+15], clamped to n (entries past n
// are left unchanged).  base is 16-byte aligned (arena offsets are multiples
// of 256 bytes).
template <class T>
__device__ __forceinline__ void sel_load16(const T* base, long long q0, long long n, T* v) {
    if (q0 + kSelPer <= n) {
        const uint4* p = (const uint4*)(base + q0);
#pragma unroll
        for (int j = 0; j < kSelPer / 4; ++j) {
            const uint4 w = p[j];
            v[4 * j + 0] = (T)w.x;
            v[4 * j + 1] = (T)w.y;
            v[4 * j + 2] = (T)w.z;
            v[4 * j + 3] = (T)w.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (q0 + j < n) v[j] = base[q0 + j];
    }
}

// What the passes of the select have fixed after the digit of pass `pass`, as
// every block of the next launch works it out for itself from the histogram of
// that pass (a launch of one block between two passes took 3.3 us, most of it
// launch latency; 256 sums of kHistCopies words are in flight together here).
// Digit b is the largest whose suffix count S(b) (keys with digit >= b) reaches the
// number still to take, 0 if none.  Called by all kSelBlock threads; block 0
// records the result for the launches after the next.
struct SelShared {
    unsigned int tot[kSelBlock / 64];
    SelPick pick;
};
// The loads of the pick, issued ahead of what else a launch waits for.
struct SelLoad {
    unsigned int h[kHistCopies];
    SelPick before;
};
__device__ __forceinline__ SelLoad sel_load(const DevState* st, int pass, unsigned int k) {
    SelLoad l;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) l.h[c] = st->hist[pass][c][threadIdx.x];
    l.before = SelPick{0u, 0u, k, 0u};
    if (pass) l.before = st->sel[pass - 1];
    return l;
}
__device__ __forceinline__ SelPick sel_pick(DevState* st, int pass, const SelLoad& l,
                                            SelShared& s) {
    const int b = threadIdx.x, lane = b & 63, w = b >> 6;
    unsigned int hb = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) hb += l.h[c];
    SelPick p = l.before;
    // suffix sums: within the wave by shuffles, then the totals of the waves above
    unsigned int S = hb;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = (unsigned int)__shfl_down((int)S, o, 64);
        if (lane + o < 64) S += y;
    }
    if (lane == 0) s.tot[w] = S;
    __syncthreads();
    for (int i = w + 1; i < kSelBlock / 64; ++i) S += s.tot[i];
    const unsigned int S1 = S - hb;
    if (b == 0 ? S1 < p.krem : (S >= p.krem && S1 < p.krem)) {
        const int shift = 24 - 8 * pass;
        p.prefix |= (unsigned int)b << shift;
        p.mask |= 0xFFu << shift;
        p.krem -= S1;
        p.rank = pass == 3 && hb != p.krem ? 1u : 0u;
        s.pick = p;
        if (blockIdx.x == 0) st->sel[pass] = p;
    }
    __syncthreads();
    return s.pick;
}

// Clear the histogram of a pass that no block of this launch reads or adds to.
__device__ __forceinline__ void sel_clear(DevState* st, int pass) {
    unsigned int* h = &st->hist[pass][0][0];
    for (int i = blockIdx.x * kSelBlock + threadIdx.x; i < kHistCopies * 256; i += gridDim.x * kSelBlock)
        h[i] = 0u;
}

// Digit histogram of pass `pass` (8 bits from the top) of the keys matching
// the prefix fixed by the passes before (picked here, see sel_pick), over the
// chunks of kCommitChunk keys this block takes (grid-stride), added into one of
// kHistCopies copies (by block index) so that blocks do not queue on one address.
// With gate_ctr (the first launch after an evaluation that counted digit 0) it is
// also IsConverged for the top-k: nothing is selected or committed when that
// evaluation found no residual above eps.  The histogram of pass p is read in
// the launch after it, and cleared in the one after that (pass 3's in the next
// iteration's pass 1).
__global__ __launch_bounds__(kSelBlock) void k_rbp_hist(DevState* st, const unsigned int* keys,
                                                        int E, int pass, unsigned int k,
                                                        const CounterLine* gate_ctr) {
    __shared__ unsigned int h[256];
    __shared__ SelShared ss;
    __shared__ unsigned int s_skip;
    // the gate, the histogram of the pass before and the block's first keys are all
    // requested before the first of them is waited for
    const int chunks = (E + kCommitChunk - 1) / kCommitChunk;
    int c = blockIdx.x;
    unsigned int v[kSelPer];
    auto load_keys = [&]() {
        sel_load16(keys, (long long)c * kCommitChunk + (long long)threadIdx.x * kSelPer, (long long)E, v);
    };
    SelLoad sl;
    if (pass) sl = sel_load(st, pass - 1, k);
    if (c < chunks) load_keys();
    if (gate_ctr) {
        if (threadIdx.x < 64) {
            const unsigned int n = wave_sum32((unsigned int)gate_ctr[threadIdx.x].active);
            if (threadIdx.x == 0) {
                s_skip = (st->done || n == 0u) ? 1u : 0u;
                if (blockIdx.x == 0) st->rbp_skip = s_skip;
            }
        }
    } else if (threadIdx.x == 0) {
        s_skip = st->rbp_skip;
    }
    h[threadIdx.x] = 0u;
    __syncthreads();
    if (s_skip) return;
    SelPick p{0u, 0u, k, 0u};
    if (pass) {
        p = sel_pick(st, pass - 1, sl, ss);
        sel_clear(st, pass >= 2 ? pass - 2 : 3);
    }
    const int shift = 24 - 8 * pass;
    while (c < chunks) {
        const long long q0 = (long long)c * kCommitChunk + (long long)threadIdx.x * kSelPer;
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            lds_count(h, (v[j] >> shift) & 255u, q0 + j < E && (v[j] & p.mask) == p.prefix);
        c += gridDim.x;
        if (c < chunks) load_keys();
    }
    __syncthreads();
    if (h[threadIdx.x])
        atomicAdd(&st->hist[pass][blockIdx.x & (kHistCopies - 1)][threadIdx.x], h[threadIdx.x]);
}

// Ties at the threshold key are taken in (target, source) order.  Slots are
// ordered by (source, target), so position p visits the message in slot rev[p],
// whose (target, source) is the (source, target) of slot p: walking positions
// in order walks tied messages in (target, source) order.  Without rev the
// positions are the keys' indices (residual splash ranks tied variables by id).
// The last digit is picked here (block 0 records it); when the threshold key has more
// ties than are still to take, each block counts the ties among its kCommitChunk
// positions.
__global__ __launch_bounds__(kSelBlock) void k_rbp_tiecount(DevState* st, const unsigned int* keys,
                                                            const int* rev, int E,
                                                            unsigned int* block_ties) {
    __shared__ unsigned int part[kSelBlock / 64];
    __shared__ SelShared ss;
    const SelLoad sl = sel_load(st, 3, 0u);
    if (st->rbp_skip) return;
    const SelPick pk = sel_pick(st, 3, sl, ss);
    sel_clear(st, 2);
    if (!pk.rank) return;
    const unsigned int T = pk.prefix;
    const long long q0 = (long long)blockIdx.x * kCommitChunk + (long long)threadIdx.x * kSelPer;
    unsigned int c = 0;
    if (rev) {
        int e[kSelPer];
        sel_load16(rev, q0, (long long)E, e);
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (q0 + j < E) c += keys[e[j]] == T;
    } else {
        // positions are the keys' own indices (variables of residual splash)
        unsigned int kv[kSelPer];
        sel_load16(keys, q0, (long long)E, kv);
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (q0 + j < E) c += kv[j] == T;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int sum = 0;
        for (int i = 0; i < kSelBlock / 64; ++i) sum += part[i];
        block_ties[blockIdx.x] = sum;
    }
}

// Exclusive prefix sums of the nb block tie counts, in place (one block: each
// thread takes a contiguous run, the run totals are scanned in LDS).  Only for more
// than kTieScanBlocks blocks: up to there a committing block adds up the counts
// before its own itself, one load per thread and 256 blocks (a launch saved,
// 1.4 us of it latency).
constexpr int kTieScanBlocks = 2048;
__global__ __launch_bounds__(kSelBlock) void k_rbp_tiescan(DevState* st, unsigned int* block_ties,
                                                           int nb) {
    __shared__ unsigned int part[kSelBlock];
    if (st->rbp_skip || !st->sel[3].rank) return;
    const int per = (nb + kSelBlock - 1) / kSelBlock;
    const int r0 = threadIdx.x * per, r1 = min(nb, r0 + per);
    unsigned int run = 0;
    for (int i = r0; i < r1; ++i) run += block_ties[i];
    part[threadIdx.x] = run;
    __syncthreads();
    for (int o = 1; o < kSelBlock; o <<= 1) {
        const unsigned int add = threadIdx.x >= (unsigned)o ? part[threadIdx.x - o] : 0u;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned int acc = part[threadIdx.x] - run;
    for (int i = r0; i < r1; ++i) {
        const unsigned int v = block_ties[i];
        block_ties[i] = acc;
        acc += v;
    }
}

// Ties before block blockIdx.x (called by all kSelBlock threads).
__device__ __forceinline__ unsigned int ties_before(const unsigned int* block_ties, bool scanned,
                                                    unsigned int* s_w) {
    if (scanned) return block_ties[blockIdx.x];
    unsigned int c = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kSelBlock) c += block_ties[i];
    c = wave_sum32(c);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    c = 0;
    for (int i = 0; i < kSelBlock / 64; ++i) c += s_w[i];
    return c;
}

// Commit the frontier: every key above the threshold, and among keys equal to
// it the first sel_krem in position order (ranked ties) or all of them.  A
// thread takes kSelPer consecutive positions; the ties before it come from an
// exclusive scan over the block's threads plus the block's offset.
__global__ __launch_bounds__(kSelBlock) void k_rbp_commit(DevState* st, unsigned int* keys,
                                                          const int* rev, const float* cand,
                                                          float* m, int E, int row, int all,
                                                          const unsigned int* block_ties,
                                                          RbpSparse sp, const int* moff,
                                                          int scanned) {
    __shared__ unsigned int part[kSelBlock / 64];
    __shared__ unsigned int s_cm[kSelBlock / 64];
    if (st->rbp_skip) return;
    const unsigned int T = st->sel[3].prefix;
    const bool rank = !all && st->sel[3].rank;
    const unsigned int krem = st->sel[3].krem;
    const long long q0 = (long long)blockIdx.x * kCommitChunk + (long long)threadIdx.x * kSelPer;
    int e[kSelPer];
    if (rank) {
        sel_load16(rev, q0, (long long)E, e);
    } else {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j) e[j] = (int)(q0 + j);
    }
    unsigned int take = 0, tie = 0;  // bit j: position q0 + j
    unsigned int kv[kSelPer];
    if (all) {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (q0 + j < E) take |= 1u << j;
        if (sp.on) sel_load16(keys, q0, (long long)E, kv);
    } else {
        if (rank) {
#pragma unroll
            for (int j = 0; j < kSelPer; ++j) kv[j] = q0 + j < E ? keys[e[j]] : 0u;
        } else {
            sel_load16(keys, q0, (long long)E, kv);  // positions are slots: contiguous
        }
#pragma unroll
        for (int j = 0; j < kSelPer; ++j) {
            if (q0 + j >= E) continue;
            if (kv[j] > T) take |= 1u << j;
            if (kv[j] == T) tie |= 1u << j;
        }
        if (!rank) take |= tie;
    }
    if (rank) {
        // ties before this thread: inclusive scan within the wave, then the
        // totals of the lower waves
        const unsigned int c = (unsigned int)__popc(tie);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        unsigned int x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = (unsigned int)__shfl_up((int)x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) part[w] = x;
        __syncthreads();
        unsigned int before = ties_before(block_ties, scanned, s_cm) + x - c;
        for (int i = 0; i < w; ++i) before += part[i];
#pragma unroll
        for (int j = 0; j < kSelPer; ++j) {
            if (!(tie >> j & 1u)) continue;
            if (before < krem) take |= 1u << j;
            ++before;
        }
        __syncthreads();  // s_cm is reused below
    }
    unsigned int cm = 0;  // committed messages whose residual was above eps
    if (take && row == 1) {
        float cv[kSelPer];
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (take >> j & 1u) cv[j] = cand[e[j]];
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (take >> j & 1u) m[e[j]] = cv[j];
        if (sp.on) {
            // sparse re-evaluation: the committed message's residual is 0 until
            // its source is evaluated again; its target is evaluated again
            int dv[kSelPer];
#pragma unroll
            for (int j = 0; j < kSelPer; ++j)
                if (take >> j & 1u) dv[j] = sp.dst[e[j]];
#pragma unroll
            for (int j = 0; j < kSelPer; ++j) {
                if (!(take >> j & 1u)) continue;
                cm += __uint_as_float(kv[j]) > sp.eps ? 1u : 0u;
                keys[e[j]] = 0u;
                sp.dirty[dv[j]] = 1;
            }
        }
    } else if (take && moff) {
        // ragged rows: slot e's K_j values at moff[e]
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (take >> j & 1u)
                for (int q = moff[e[j]]; q < moff[e[j] + 1]; ++q) m[q] = cand[q];
    } else if (take) {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (take >> j & 1u)
                for (int x = 0; x < row; ++x)
                    m[(long long)e[j] * row + x] = cand[(long long)e[j] * row + x];
    }
    if (sp.on) {
        // the committed active messages leave the running count of the next iteration
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cm += __shfl_xor(cm, o, 64);
        if ((threadIdx.x & 63) == 0) s_cm[threadIdx.x >> 6] = cm;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned int c = 0;
            for (int w = 0; w < kSelBlock / 64; ++w) c += s_cm[w];
            CounterLine* z = sp.ctr + (unsigned)sp.set * kCounterCopies +
                             (blockIdx.x & (kCounterCopies - 1));
            if (c) atomicAdd(&z->active, (unsigned long long)(-(long long)c));
        }
    }
}

// Frontier residual BP with sparse re-evaluation: close evaluation t after
// k_sparse_eval (one wave).  n_t = n_{t-1} + the running-count changes of
// counter set t & 3; statistics as the full path records them (k messages
// committed per committing iteration); the top-k kernels run only when n_t > 0
// and t is not the evaluation after the last allowed commit.  Clears counter
// set t + 2.
__global__ void k_sparse_rbp_close(EvalArgs a) {
    const int lane = threadIdx.x;
    DevState* st = a.st;
    const unsigned int done = st->done;
    const CounterLine* c0 = a.ctr + (a.t & 3u) * kCounterCopies + lane;
    const long long d = (int)wave_sum32((unsigned int)c0->active);
    const long long base = a.sp_first ? 0ll : (long long)st->sp_n[(a.t - 1u) & 3u];
    const unsigned long long n1 = (unsigned long long)(base + d);
    long long n2;
    if (!a.sp_first)
        n2 = (long long)st->sp_n[(a.t - 1u) & 3u];
    else if (a.it >= 1)  // switched from the full evaluation: its count of t - 1
        n2 = (long long)wave_sum32((unsigned int)a.ctr[((a.t - 1u) & 3u) * kCounterCopies + lane].active);
    else
        n2 = a.prev_active_host;
    const unsigned long long ev = wave_sum32((unsigned int)c0->sel_a);
    if (done) {
        if (lane == 0) st->rbp_skip = 1u;
        return;
    }
    CounterLine* z = a.ctr + ((a.t + 2u) & 3u) * kCounterCopies + lane;
    z->active = 0ull;
    z->sel_a = 0ull;
    z->sel_b = 0ull;
    z->rmax = 0u;
    if (lane != 0) return;
    report_progress(a, (unsigned long long)a.it + 1ull, n1 == 0ull);
    atomicAdd(&st->evaluated, ev);
    atomicAdd(&st->evals, 1ull);
    st->sp_n[a.t & 3u] = n1;
    st->last_t = (long long)a.t;
    st->last_active = n1;
    st->last_rmax = 0u;  // taken after the run
    st->last_prev = n2;
    if (n1 == 0ull) {
        st->done = 1u;
        st->conv_t = (long long)a.t;
        st->rbp_skip = 1u;
    } else if (a.after_final) {
        st->rbp_skip = 1u;
    } else {
        atomicAdd(&st->iterations, 1ull);
        atomicAdd(&st->committed, a.rbp_k);
        st->rbp_skip = 0u;
    }
}

// ---------------------------------------------------------------------------
// Whole runs of small K = 2 graphs in one block: at most kSmallPer messages and
// variables per thread, every array of the iteration in LDS or registers.
//
// A launch per iteration costs such a graph 5 us (32 us with the top-k's six
// launches) whatever its size: the launch, the counters and the messages from
// memory, each a latency of its own.  Here an iteration is three barriers
// (a few more for the top-k), and n_t is known before the commit, so only the
// outcome that p_t chooses is written.  The arithmetic per message is the tiled
// kernel's, the incoming messages are summed in slot order as it sums them, the
// draws are the same words: the results are bit for bit the same.
//
// LDS: in[s] holds the message into the source of slot s (that of slot rev[s]),
// so a commit of slot s writes in[rev[s]].  A launch takes up to max_commits
// commits (the run's bound, cut so that one launch stays short), closes with an
// evaluation and leaves the messages in memory.
// ---------------------------------------------------------------------------
template <int NT>
struct SmallLds {
    float in[NT * kSmallPer];
    float L[NT * kSmallPer];             // node aggregates
    unsigned int u[NT * kSmallPer];      // 24-bit uniforms (RnBP)
    unsigned short ptr[NT * kSmallPer + 1];
    unsigned int hist[256];              // top-k
    unsigned int ties[NT * kSmallPer / 32];
    unsigned int pick[4];
    unsigned int n[2][NT / 64], rm[2][NT / 64];
    unsigned int tot[4];
    unsigned long long cm[NT / 64];
};

// The rbp_k largest residual keys of the block's slots, ties by position (see
// k_rbp_tiecount: slot e is at position rev[e]); bit k of the result: the
// thread's slot tid + k NT is taken.
template <int NT>
__device__ __forceinline__ unsigned int small_topk(SmallLds<NT>& l, int E, unsigned int k,
                                                   const float* r, const int* rev) {
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned int prefix = 0, mask = 0, krem = k, ties = 0;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) l.hist[tid] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSmallPer; ++j) {
            const unsigned int key = __float_as_uint(r[j]);
            lds_count(l.hist, (key >> shift) & 255u, tid + j * NT < E && (key & mask) == prefix);
        }
        __syncthreads();
        // the pick (as sel_pick), four digits per lane of one wave
        if (tid < 64) {
            unsigned int h[4], S = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = l.hist[4 * lane + i];
                S += h[i];
            }
            const unsigned int own = S;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned int y = (unsigned int)__shfl_down((int)S, o, 64);
                if (lane + o < 64) S += y;
            }
            unsigned int above = S - own;  // keys with a digit of a higher lane
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                const unsigned int Sb = above + h[i];
                if (4 * lane + i == 0 ? above < krem : (Sb >= krem && above < krem)) {
                    l.pick[0] = (unsigned int)(4 * lane + i);
                    l.pick[1] = krem - above;
                    l.pick[2] = h[i];
                }
                above = Sb;
            }
        }
        __syncthreads();
        prefix |= l.pick[0] << shift;
        mask |= 0xFFu << shift;
        krem = l.pick[1];
        ties = l.pick[2];
    }
    const bool rank = ties != krem;
    if (rank) {
        for (int i = tid; i < NT * kSmallPer / 32; i += NT) l.ties[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSmallPer; ++j)
            if (tid + j * NT < E && __float_as_uint(r[j]) == prefix)
                atomicOr(&l.ties[rev[j] >> 5], 1u << (rev[j] & 31));
        __syncthreads();
    }
    unsigned int take = 0;
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (tid + j * NT >= E) continue;
        const unsigned int key = __float_as_uint(r[j]);
        bool t = key > prefix;
        if (key == prefix) {
            t = true;
            if (rank) {
                unsigned int before = __popc(l.ties[rev[j] >> 5] & ((1u << (rev[j] & 31)) - 1u));
                for (int i = 0; i < rev[j] >> 5; ++i) before += __popc(l.ties[i]);
                t = before < krem;
            }
        }
        take |= (t ? 1u : 0u) << j;
    }
    return take;
}

template <int MODE, int NT>
__global__ __launch_bounds__(NT) void k_solve_small(EvalArgs a, float* msg, int fresh,
                                                    long long max_commits, SmallState* out) {
    __shared__ SmallLds<NT> l;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int E = (int)a.num_messages, N = a.num_nodes;
    // the thread's slots tid + k NT and nodes tid + k NT
    float J[kSmallPer], old[kSmallPer], u[kSmallPer];
    int rev[kSmallPer], owner[kSmallPer];
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k) {
        const int s = tid + k * NT, v = tid + k * NT;
        rev[k] = 0;
        J[k] = old[k] = u[k] = 0.0f;
        if (s < E) {
            rev[k] = a.rev[s];
            J[k] = a.coupling[s];
            old[k] = fresh ? 0.0f : msg[s];
            l.in[s] = fresh ? 0.0f : msg[rev[k]];
        }
        if (v < N) {
            u[k] = a.unary[v];
            const int p0 = a.node_ptr[v], p1 = a.node_ptr[v + 1];
            l.ptr[v] = (unsigned short)p0;
            if (v == N - 1) l.ptr[N] = (unsigned short)p1;
            // l.u holds the owners until they are in registers
            for (int q = p0; q < p1; ++q) l.u[q] = (unsigned int)v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k) owner[k] = tid + k * NT < E ? (int)l.u[tid + k * NT] : 0;
    __syncthreads();
    long long n_prev = a.prev_active_host;
    unsigned int t = a.t;
    unsigned long long committed = 0;  // per thread
    long long commits = 0;
    unsigned int n_last, rm_last;
    long long prev_last;
    bool done = false;
    for (;;) {
        // node aggregates, incoming messages in slot order; RnBP: the draws
#pragma unroll
        for (int k = 0; k < kSmallPer; ++k) {
            const int v = tid + k * NT;
            if (v >= N) break;
            const int q0 = l.ptr[v], q1 = l.ptr[v + 1];
            float L = u[k];
            for (int q = q0; q < q1; ++q) L += l.in[q];
            l.L[v] = L;
            if (MODE == kModeRnBP) {
                for (int q = q0; q < q1; q += 4) {
                    const uint4 x = philox4((unsigned int)v, (unsigned int)(q - q0) >> 2, t, a.key0,
                                            a.key1);
                    l.u[q] = x.x >> 8;
                    if (q + 1 < q1) l.u[q + 1] = x.y >> 8;
                    if (q + 2 < q1) l.u[q + 2] = x.z >> 8;
                    if (q + 3 < q1) l.u[q + 3] = x.w >> 8;
                }
            }
        }
        __syncthreads();
        float cand[kSmallPer], r[kSmallPer];
        unsigned int act = 0, acts = 0;  // bit k: slot k active; their number
        float rmax = 0.0f;
#pragma unroll
        for (int k = 0; k < kSmallPer; ++k) {
            const int s = tid + k * NT;
            cand[k] = r[k] = 0.0f;
            if (s < E) {
                cand[k] = logodds_update(l.L[owner[k]], l.in[s], J[k]);
                r[k] = fabsf(sigmoid_fast(cand[k]) - sigmoid_fast(old[k]));
                rmax = fmaxf(rmax, r[k]);
                if (r[k] > a.eps) {
                    act |= 1u << k;
                    ++acts;
                }
            }
        }
        // n_t and R_t (two sets in turn, so that one barrier separates them)
        const int par = (int)(t & 1u);
        const unsigned int wn = dpp_sum_last(acts), wr = dpp_max_last(__float_as_uint(rmax));
        if (lane == 63) {
            l.n[par][w] = wn;
            l.rm[par][w] = wr;
        }
        __syncthreads();
        unsigned int n = 0, rm = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) {
            n += l.n[par][i];
            rm = max(rm, l.rm[par][i]);
        }
        n_last = n;
        rm_last = rm;
        prev_last = n_prev;
        done = n == 0u;
        if (done || commits == max_commits) break;
        unsigned int take;  // bit k: slot k is committed
        if (MODE == kModeLBP) {
            take = ~0u;
        } else if (MODE == kModeRnBP) {
            const unsigned int thr =
                select_outcome(a, (unsigned long long)n, n_prev) ? a.thr_b : a.thr_a;
            take = 0u;
#pragma unroll
            for (int k = 0; k < kSmallPer; ++k)
                if ((act >> k & 1u) && l.u[tid + k * NT] < thr) take |= 1u << k;
            committed += __popc(take);
        } else {
            take = a.rbp_k >= (unsigned long long)E
                       ? ~0u
                       : small_topk<NT>(l, E, (unsigned int)a.rbp_k, r, rev);
        }
#pragma unroll
        for (int k = 0; k < kSmallPer; ++k) {
            if (tid + k * NT < E && (take >> k & 1u)) {
                old[k] = cand[k];
                l.in[rev[k]] = cand[k];
            }
        }
        ++commits;
        ++t;
        n_prev = (long long)n;
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k)
        if (tid + k * NT < E) msg[tid + k * NT] = old[k];
    if (MODE == kModeRnBP) {
        // at most kSmallPer commits per thread and iteration: below 2^32 per launch
        const unsigned int c = dpp_sum_last((unsigned int)committed);
        if (lane == 63) l.cm[w] = c;
        __syncthreads();
    }
    if (tid == 0) {
        unsigned long long cm = 0;
        if (MODE == kModeRnBP)
            for (int i = 0; i < NT / 64; ++i) cm += l.cm[i];
        else
            cm = (unsigned long long)commits * (MODE == kModeLBP ? (unsigned long long)E : a.rbp_k);
        out->done = done ? 1u : 0u;
        out->rmax = rm_last;
        out->t = (long long)t;
        out->n = (long long)n_last;
        out->prev = prev_last;
        out->commits = commits;
        out->committed = cm;
    }
}

// ---------------------------------------------------------------------------
// Residual splash (Sec. II-B, Sec. III-A) in frontier form, K = 2 log-odds
// layout, messages committed in place.  After the evaluation of iteration t
// (the candidate and residual key of every message, as for frontier RBP):
//   1. the residual of variable v is the largest residual of the messages into
//      v (for each slot s of v, slot rev[s] holds the message into v);
//   2. the k variables of largest residual are the roots: the radix select of
//      frontier RBP over the variable keys, tied variables taken by id;
//   3. level d holds every variable at distance exactly d from some root: a
//      thread per root marks its neighbours (d = 1) and their neighbours that
//      are neither the root nor adjacent to it (d = 2) with the iteration's tag;
//   4. the marked variables of each level are compacted into a list (wave
//      ballot and lane prefix counts, a block prefix sum in LDS, one atomic per
//      block);
//   5. the levels are updated in the order h, ..., 0, ..., h with two launches
//      each: the candidates of every message out of the level's variables,
//      computed from the messages as they stand, then their commit.
// The list order depends on the order in which blocks append; no result does
// (every message of a level is computed from the state the level starts from).
// ---------------------------------------------------------------------------
constexpr int kRsGrid = 512;  // blocks of the grid-stride splash kernels

// IsConverged for the splash: nothing is selected or updated when the
// evaluation of iteration t found no residual above eps; the level lists of
// iteration t start empty.
__global__ void k_rs_gate(DevState* st, const CounterLine* ctr, int slot) {
    const unsigned int n = wave_sum32((unsigned int)ctr[slot * kCounterCopies + threadIdx.x].active);
    if (threadIdx.x == 0) st->rbp_skip = (st->done || n == 0u) ? 1u : 0u;
    if (threadIdx.x <= kSplashMaxDepth) st->rs_count[threadIdx.x] = 0u;
}

// Block-wide exclusive prefix of the per-thread item counts c (lane prefix by
// shuffles, wave totals in LDS) and one atomic per block on *count; returns the
// list position of the thread's first item.  Called by every thread of the
// block; s_w holds kBlock / 64 + 1 words.
__device__ __forceinline__ unsigned int block_append(unsigned int c, unsigned int* count,
                                                     unsigned int* s_w) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned int x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = (unsigned int)__shfl_up((int)x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int tot = 0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
            const unsigned int v = s_w[i];
            s_w[i] = tot;
            tot += v;
        }
        s_w[kBlock / 64] = tot ? atomicAdd(count, tot) : 0u;
    }
    __syncthreads();
    const unsigned int pos = s_w[kBlock / 64] + s_w[w] + x - c;
    __syncthreads();  // s_w is reused by the next call
    return pos;
}


// 1. Variable residual keys (FP32 bit patterns of non-negative residuals order
// as unsigned integers).
__global__ __launch_bounds__(kBlock) void k_rs_vkeys(RsArgs r) {
    if (r.st->rbp_skip) return;
    for (int v = blockIdx.x * kBlock + threadIdx.x; v < r.num_nodes; v += gridDim.x * kBlock) {
        const int s0 = r.node_ptr[v], s1 = r.node_ptr[v + 1];
        unsigned int k = 0u;
        for (int s = s0; s < s1; ++s) k = max(k, r.keys[r.rev[s]]);
        r.vkey[v] = k;
    }
}

// 2. The roots: every variable whose key is above the selected threshold, and
// among the variables equal to it the first sel_krem by id (all of them when
// `all`); each is marked in level 0 and appended to list 0.  Same chunking as
// the tie count (kSelPer consecutive variables per thread).
__global__ __launch_bounds__(kSelBlock) void k_rs_roots(RsArgs r, int all,
                                                        const unsigned int* block_ties,
                                                        int scanned) {
    __shared__ unsigned int part[kSelBlock / 64];
    __shared__ unsigned int s_tb[kSelBlock / 64];
    __shared__ unsigned int s_w[kBlock / 64 + 1];
    static_assert(kSelBlock == kBlock, "block_append assumes kBlock threads");
    const DevState* st = r.st;
    if (st->rbp_skip) return;
    const int N = r.num_nodes;
    const unsigned int T = st->sel[3].prefix;
    const bool rank = !all && st->sel[3].rank;
    const unsigned int krem = st->sel[3].krem;
    const long long q0 = (long long)blockIdx.x * kCommitChunk + (long long)threadIdx.x * kSelPer;
    unsigned int take = 0, tie = 0;
    if (all) {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
            if (q0 + j < N) take |= 1u << j;
    } else {
        unsigned int kv[kSelPer];
        sel_load16(r.vkey, q0, (long long)N, kv);
#pragma unroll
        for (int j = 0; j < kSelPer; ++j) {
            if (q0 + j >= N) continue;
            if (kv[j] > T) take |= 1u << j;
            if (kv[j] == T) tie |= 1u << j;
        }
        if (!rank) take |= tie;
    }
    if (rank) {
        const unsigned int c = (unsigned int)__popc(tie);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        unsigned int x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = (unsigned int)__shfl_up((int)x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) part[w] = x;
        __syncthreads();
        unsigned int before = ties_before(block_ties, scanned, s_tb) + x - c;
        for (int i = 0; i < w; ++i) before += part[i];
#pragma unroll
        for (int j = 0; j < kSelPer; ++j) {
            if (!(tie >> j & 1u)) continue;
            if (before < krem) take |= 1u << j;
            ++before;
        }
    }
    unsigned int pos = block_append((unsigned int)__popc(take), &r.st->rs_count[0], s_w);
#pragma unroll
    for (int j = 0; j < kSelPer; ++j) {
        if (!(take >> j & 1u)) continue;
        const int v = (int)(q0 + j);
        r.mark[v] = r.tag;
        r.list[pos++] = v;
    }
}

// Whether w is among the targets dst[s0 .. s1) (ascending: the slots of a
// source are ordered by target).
__device__ __forceinline__ bool rs_adjacent(const int* dst, int s0, int s1, int w) {
    int lo = s0, hi = s1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (dst[mid] < w)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo < s1 && dst[lo] == w;
}

// 3. Levels 1 and 2 of every root's splash: a variable at distance exactly 1 is
// a neighbour of the root; one at distance exactly 2 is a neighbour of a
// neighbour that is neither the root nor one of its neighbours.  Marks are
// plain stores of the iteration's tag (several roots may store the same word).
__global__ __launch_bounds__(kBlock) void k_rs_bfs(RsArgs r) {
    if (r.st->rbp_skip) return;
    const unsigned int nr = r.st->rs_count[0];
    const size_t N = (size_t)r.num_nodes;
    unsigned int* m1 = r.mark + N;
    unsigned int* m2 = r.mark + 2 * N;
    for (unsigned int i = blockIdx.x * kBlock + threadIdx.x; i < nr; i += gridDim.x * kBlock) {
        const int root = r.list[i];
        const int s0 = r.node_ptr[root], s1 = r.node_ptr[root + 1];
        for (int s = s0; s < s1; ++s) {
            const int u = r.dst[s];
            m1[u] = r.tag;
            if (r.depth < 2) continue;
            const int u0 = r.node_ptr[u], u1 = r.node_ptr[u + 1];
            for (int q = u0; q < u1; ++q) {
                const int w = r.dst[q];
                if (w == root || rs_adjacent(r.dst, s0, s1, w)) continue;
                m2[w] = r.tag;
            }
        }
    }
}

// 4. The lists of levels 1 .. h.  Each block takes a contiguous range of the
// variables: it counts its marked variables of a level (block sum), reserves
// their places with one atomic, then writes them in order, a chunk of 256 at a
// time (wave ballot, the lane's rank among the flagged lanes of its wave
// (mbcnt), the wave offsets from a prefix sum in LDS).  A small grid keeps the
// atomics on the level counters few (one per block and level).
constexpr int kRsListGrid = 128;
__global__ __launch_bounds__(kBlock) void k_rs_lists(RsArgs r) {
    __shared__ unsigned int s_w[kBlock / 64];
    __shared__ unsigned int s_base;
    if (r.st->rbp_skip) return;
    const int N = r.num_nodes;
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int per = ((N + (int)gridDim.x - 1) / (int)gridDim.x + kBlock - 1) / kBlock * kBlock;
    const int v0 = (int)blockIdx.x * per, v1 = min(N, v0 + per);
    for (int d = 1; d <= r.depth; ++d) {
        const unsigned int* mk = r.mark + (size_t)d * N;
        int* L = r.list + (size_t)d * N;
        unsigned int c = 0;
        for (int v = v0 + tid; v < v1; v += kBlock) c += mk[v] == r.tag ? 1u : 0u;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c += (unsigned int)__shfl_xor((int)c, o, 64);
        if (lane == 0) s_w[w] = c;
        __syncthreads();
        if (tid == 0) {
            unsigned int tot = 0;
            for (int i = 0; i < kBlock / 64; ++i) tot += s_w[i];
            s_base = tot ? atomicAdd(&r.st->rs_count[d], tot) : 0u;
        }
        __syncthreads();
        unsigned int off = s_base;
        for (int vb = v0; vb < v1; vb += kBlock) {
            const int v = vb + tid;
            const bool f = v < v1 && mk[v] == r.tag;
            const unsigned long long b = __ballot(f);
            const unsigned int before = __builtin_amdgcn_mbcnt_hi(
                (unsigned int)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)b, 0u));
            __syncthreads();  // s_w of the previous chunk has been read
            if (lane == 0) s_w[w] = (unsigned int)__popcll(b);
            __syncthreads();
            unsigned int wpre = 0, tot = 0;
            for (int i = 0; i < kBlock / 64; ++i) {
                const unsigned int x = s_w[i];
                if (i < w) wpre += x;
                tot += x;
            }
            if (f) L[off + wpre + before] = v;
            off += tot;
        }
        __syncthreads();  // s_w and s_base are reused by the next level
    }
}

// 5a. Eq. (2) for every message out of the variables of level d, from the
// messages as they stand (the incoming log-odds summed in slot order with the
// unary, as the tiled kernel sums them).
__global__ __launch_bounds__(kBlock) void k_rs_level_eval(RsArgs r, int d) {
    if (r.st->rbp_skip) return;
    const unsigned int n = r.st->rs_count[d];
    const int* L = r.list + (size_t)d * r.num_nodes;
    for (unsigned int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const int v = L[i];
        const int s0 = r.node_ptr[v], s1 = r.node_ptr[v + 1];
        float agg = r.unary[v];
        for (int s = s0; s < s1; ++s) agg += r.m[r.rev[s]];
        for (int s = s0; s < s1; ++s) r.cand[s] = logodds_update(agg, r.m[r.rev[s]], r.coupling[s]);
    }
}

// 5b. Commit level d's candidates; the committed messages are added to the
// run's commit and evaluation counts (one atomic per block).
__global__ __launch_bounds__(kBlock) void k_rs_level_commit(RsArgs r, int d) {
    __shared__ unsigned int s_c[kBlock / 64];
    if (r.st->rbp_skip) return;
    const unsigned int n = r.st->rs_count[d];
    const int* L = r.list + (size_t)d * r.num_nodes;
    unsigned int c = 0;
    for (unsigned int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const int v = L[i];
        const int s0 = r.node_ptr[v], s1 = r.node_ptr[v + 1];
        for (int s = s0; s < s1; ++s) r.m[s] = r.cand[s];
        c += (unsigned int)(s1 - s0);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long C = 0;
        for (int w = 0; w < kBlock / 64; ++w) C += s_c[w];
        if (C) {
            atomicAdd(&r.st->committed, C);
            atomicAdd(&r.st->evaluated, C);
        }
    }
}

__global__ void k_fill_u32(unsigned int* p, unsigned int v, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launch wrappers
// ---------------------------------------------------------------------------
hipError_t launch_init_state(DevState* st, size_t bytes, CounterLine* ctr, hipStream_t s) {
    k_init_state<<<1, 256, 0, s>>>(st, (int)(bytes / sizeof(unsigned int)), ctr);
    return hipGetLastError();
}

hipError_t launch_check_short_math(unsigned long long* diff, hipStream_t s) {
    k_check_short_math<<<4096, kBlock, 0, s>>>(diff);
    return hipGetLastError();
}

hipError_t launch_fill(float* p, float v, long long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_fill<<<(int)blocks, 256, 0, s>>>(p, v, n);
    return hipGetLastError();
}

template <int KP>
static hipError_t launch_generic(int mode, const EvalArgs& a, int grid, size_t shm,
                                 hipStream_t s) {
    switch (mode) {
    case kModeLBP: k_eval_generic<KP, kModeLBP><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRnBP: k_eval_generic<KP, kModeRnBP><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRBP: k_eval_generic<KP, kModeRBP><<<grid, kBlock, shm, s>>>(a); break;
    default: k_eval_generic<KP, kModeEvalOnly><<<grid, kBlock, shm, s>>>(a); break;
    }
    return hipGetLastError();
}

template <int KP>
static hipError_t launch_split(int mode, const EvalArgs& a, int grid, size_t shm, hipStream_t s) {
    switch (mode) {
    case kModeLBP: k_eval_split<KP, kModeLBP><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRnBP: k_eval_split<KP, kModeRnBP><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRBP: k_eval_split<KP, kModeRBP><<<grid, kBlock, shm, s>>>(a); break;
    default: k_eval_split<KP, kModeEvalOnly><<<grid, kBlock, shm, s>>>(a); break;
    }
    return hipGetLastError();
}

template <int TAB>
static hipError_t launch_pairs(int mode, const EvalArgs& a, int grid, size_t shm, hipStream_t s) {
    switch (mode) {
    case kModeLBP: k_eval_pairs<kModeLBP, TAB><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRnBP: k_eval_pairs<kModeRnBP, TAB><<<grid, kBlock, shm, s>>>(a); break;
    case kModeRBP: k_eval_pairs<kModeRBP, TAB><<<grid, kBlock, shm, s>>>(a); break;
    default: k_eval_pairs<kModeEvalOnly, TAB><<<grid, kBlock, shm, s>>>(a); break;
    }
    return hipGetLastError();
}

hipError_t launch_eval(int layout, int mode, const EvalArgs& a, hipStream_t s) {
    const int grid = 8 * a.tiles_per_xcd;
    if (grid <= 0) return hipSuccess;
    if (layout == kLayoutLogOdds) {
        const int g = a.pipe_grid;
        if (a.rev16) {
            switch (mode) {
            case kModeLBP: k_eval_logodds<kModeLBP, true><<<g, kBlockLO, 0, s>>>(a); break;
            case kModeRnBP: k_eval_logodds<kModeRnBP, true><<<g, kBlockLO, 0, s>>>(a); break;
            case kModeRBP: k_eval_logodds<kModeRBP, true><<<g, kBlockLO, 0, s>>>(a); break;
            default: k_eval_logodds<kModeEvalOnly, true><<<g, kBlockLO, 0, s>>>(a); break;
            }
        } else {
            switch (mode) {
            case kModeLBP: k_eval_logodds<kModeLBP, false><<<g, kBlockLO, 0, s>>>(a); break;
            case kModeRnBP: k_eval_logodds<kModeRnBP, false><<<g, kBlockLO, 0, s>>>(a); break;
            case kModeRBP: k_eval_logodds<kModeRBP, false><<<g, kBlockLO, 0, s>>>(a); break;
            default: k_eval_logodds<kModeEvalOnly, false><<<g, kBlockLO, 0, s>>>(a); break;
            }
        }
        if (a.num_big > 0) {
            switch (mode) {
            case kModeLBP: k_eval_logodds_big<kModeLBP><<<a.num_big, kBlock, 0, s>>>(a); break;
            case kModeRnBP: k_eval_logodds_big<kModeRnBP><<<a.num_big, kBlock, 0, s>>>(a); break;
            case kModeRBP: k_eval_logodds_big<kModeRBP><<<a.num_big, kBlock, 0, s>>>(a); break;
            default: k_eval_logodds_big<kModeEvalOnly><<<a.num_big, kBlock, 0, s>>>(a); break;
            }
        }
        return hipGetLastError();
    }
    if (layout == kLayoutRagged) {
        const int g = a.pipe_grid;
        switch (mode) {
        case kModeLBP: k_eval_ragged<kModeLBP><<<g, kBlock, 0, s>>>(a); break;
        case kModeRnBP: k_eval_ragged<kModeRnBP><<<g, kBlock, 0, s>>>(a); break;
        case kModeRBP: k_eval_ragged<kModeRBP><<<g, kBlock, 0, s>>>(a); break;
        default: k_eval_ragged<kModeEvalOnly><<<g, kBlock, 0, s>>>(a); break;
        }
        return hipGetLastError();
    }
    const int K = a.num_states;
    const int TN = a.tile_nodes_max;
    if (K == 32 && a.pair_kind == kPairShared && !a.tile_big && !a.no_mfma) {
        const size_t shm = mfma32_lds_bytes(TN);
        if (a.mfma_bf16) {
            switch (mode) {
            case kModeLBP: k_eval_mfma32<kModeLBP, true><<<grid, kBlock, shm, s>>>(a); break;
            case kModeRnBP: k_eval_mfma32<kModeRnBP, true><<<grid, kBlock, shm, s>>>(a); break;
            case kModeRBP: k_eval_mfma32<kModeRBP, true><<<grid, kBlock, shm, s>>>(a); break;
            default: k_eval_mfma32<kModeEvalOnly, true><<<grid, kBlock, shm, s>>>(a); break;
            }
        } else {
            switch (mode) {
            case kModeLBP: k_eval_mfma32<kModeLBP, false><<<grid, kBlock, shm, s>>>(a); break;
            case kModeRnBP: k_eval_mfma32<kModeRnBP, false><<<grid, kBlock, shm, s>>>(a); break;
            case kModeRBP: k_eval_mfma32<kModeRBP, false><<<grid, kBlock, shm, s>>>(a); break;
            default: k_eval_mfma32<kModeEvalOnly, false><<<grid, kBlock, shm, s>>>(a); break;
            }
        }
        return hipGetLastError();
    }
    if (a.pairs_route) {
        const size_t shm =
            pairs_lds_bytes(K, a.tile_slots_max, TN, a.pair_kind == kPairDense ? 0 : 1);
        if (a.pair_kind == kPairDense) return launch_pairs<kTabDense>(mode, a, grid, shm, s);
        // 32-wide matrix tiles for the symmetric tables
        if (a.pair_kind == kPairShared && !a.no_mfma)
            return launch_pairs<kTabMfma>(mode, a, grid, shm, s);
        return launch_pairs<kTabShared>(mode, a, grid, shm, s);
    }
    const int TS = kTileFloatsGeneric / K;
    const int tables = K <= 16 ? 0 : a.pair_kind == kPairSharedAsym ? 2 : 1;
    const size_t shm =
        sizeof(float) * (size_t)(TS * (K + 1) + ((TN * (K + 1) + 3) & ~3) + tables * K * K) +
        sizeof(int) * (size_t)(TS + TN + 1) + sizeof(unsigned short) * (size_t)TS;
    switch (K) {
    case 2: return launch_generic<2>(mode, a, grid, shm, s);
    case 3: return launch_generic<3>(mode, a, grid, shm, s);
    case 4: return launch_generic<4>(mode, a, grid, shm, s);
    case 5: return launch_generic<5>(mode, a, grid, shm, s);
    case 6: return launch_generic<6>(mode, a, grid, shm, s);
    case 7: return launch_generic<7>(mode, a, grid, shm, s);
    case 8: return launch_generic<8>(mode, a, grid, shm, s);
    case 9: return launch_generic<9>(mode, a, grid, shm, s);
    case 10: return launch_generic<10>(mode, a, grid, shm, s);
    case 11: return launch_generic<11>(mode, a, grid, shm, s);
    case 12: return launch_generic<12>(mode, a, grid, shm, s);
    case 13: return launch_generic<13>(mode, a, grid, shm, s);
    case 14: return launch_generic<14>(mode, a, grid, shm, s);
    case 15: return launch_generic<15>(mode, a, grid, shm, s);
    case 16: return launch_generic<16>(mode, a, grid, shm, s);
    case 32: return launch_split<32>(mode, a, grid, shm, s);
    case 64: return launch_split<64>(mode, a, grid, shm, s);
    default: return hipErrorInvalidValue;
    }
}

int logodds_blocks_per_cu(int mode) {
    int n = 0;
    hipError_t e;
    switch (mode) {
    case kModeLBP:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k_eval_logodds<kModeLBP, true>, kBlockLO, 0);
        break;
    case kModeRnBP:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k_eval_logodds<kModeRnBP, true>, kBlockLO, 0);
        break;
    case kModeRBP:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k_eval_logodds<kModeRBP, true>, kBlockLO, 0);
        break;
    default:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)k_eval_logodds<kModeEvalOnly, true>, kBlockLO, 0);
        break;
    }
    return e == hipSuccess ? n : 0;
}

// After a step: the done flag of every graph, gathered for one readback, and the
// launch counter advanced by the step's launches.
__global__ void k_batch_status(const BatchGraph* graphs, int num_graphs, unsigned int* done,
                               BatchCtl* ctl, int launches) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g == 0) ctl->launch += launches;
    if (g >= num_graphs) return;
    const DevState* st = graphs[g].a.st;
    done[g] = st ? st->done : 0u;
}

hipError_t launch_batch_status(const BatchGraph* graphs, int num_graphs, unsigned int* done,
                               BatchCtl* ctl, int launches, hipStream_t s) {
    k_batch_status<<<(num_graphs + 255) / 256, 256, 0, s>>>(graphs, num_graphs, done, ctl, launches);
    return hipGetLastError();
}

hipError_t launch_eval_batch(const BatchGraph* graphs, const int* list, const BatchCtl* ctl,
                             int step, int grid, hipStream_t s) {
    k_eval_batch<<<grid, kBlockLO, 0, s>>>(graphs, (const int4*)list, ctl, step);
    return hipGetLastError();
}

hipError_t batch_graph_nodes(const BatchGraph* graphs, const int* list, const BatchCtl* ctl,
                             int grid, int launches, hipGraph_t* out) {
    hipGraph_t gr = nullptr;
    hipError_t e = hipGraphCreate(&gr, 0);
    if (e != hipSuccess) return e;
    const int4* lst = (const int4*)list;
    int step = 0;
    void* args[4] = {(void*)&graphs, (void*)&lst, (void*)&ctl, (void*)&step};
    hipKernelNodeParams p{};
    p.func = (void*)k_eval_batch;
    p.gridDim = dim3((unsigned)grid);
    p.blockDim = dim3(kBlockLO);
    p.kernelParams = args;
    hipGraphNode_t prev = nullptr;
    // (adding a node copies its arguments)
    for (; step < launches && e == hipSuccess; ++step) {
        hipGraphNode_t node = nullptr;
        e = hipGraphAddKernelNode(&node, gr, prev ? &prev : nullptr, prev ? 1 : 0, &p);
        prev = node;
    }
    if (e != hipSuccess) {
        (void)hipGraphDestroy(gr);
        return e;
    }
    *out = gr;
    return hipSuccess;
}

template <int NT>
static hipError_t launch_small_nt(int mode, const EvalArgs& a, float* msg, int fresh,
                                  long long max_commits, SmallState* out, hipStream_t s) {
    switch (mode) {
    case kModeLBP: k_solve_small<kModeLBP, NT><<<1, NT, 0, s>>>(a, msg, fresh, max_commits, out); break;
    case kModeRnBP: k_solve_small<kModeRnBP, NT><<<1, NT, 0, s>>>(a, msg, fresh, max_commits, out); break;
    default: k_solve_small<kModeRBP, NT><<<1, NT, 0, s>>>(a, msg, fresh, max_commits, out); break;
    }
    return hipGetLastError();
}

hipError_t launch_solve_small(int mode, const EvalArgs& a, float* msg, int fresh,
                              long long max_commits, SmallState* out, hipStream_t s) {
    // the fewest waves that hold the graph: fewer to meet at each barrier
    const long long most = std::max<long long>((long long)a.num_messages, a.num_nodes);
    if (most <= 256 * kSmallPer)
        return launch_small_nt<256>(mode, a, msg, fresh, max_commits, out, s);
    if (most <= 512 * kSmallPer)
        return launch_small_nt<512>(mode, a, msg, fresh, max_commits, out, s);
    return launch_small_nt<1024>(mode, a, msg, fresh, max_commits, out, s);
}

hipError_t launch_close_run(const EvalArgs& a, void* host, size_t bytes, hipStream_t s) {
    k_close_run<<<1, 64, 0, s>>>(a, (unsigned int*)host, (int)(bytes / sizeof(unsigned int)));
    return hipGetLastError();
}

hipError_t launch_marginals(int layout, const int* node_ptr, const int* rev,
                            const float* unary, const float* m, float* out, int N, int K,
                            hipStream_t s) {
    if (N <= 0) return hipSuccess;
    const int grid = (N + 255) / 256;
    if (layout == kLayoutLogOdds)
        k_marginals_logodds<<<grid, 256, 0, s>>>(node_ptr, rev, unary, m, out, N);
    else {
        // 16-byte stores need the caller's buffer aligned (its rows then are)
        const bool v4 = K % 4 == 0 && (uintptr_t)out % 16 == 0;
        const int L = v4 ? K / 4 : K;
        int wl = 0;
        while ((1 << wl) < L) ++wl;
        const long long per_block = 4ll * (64 >> wl);  // four waves
        const int g = (int)std::min<long long>((N + per_block - 1) / per_block, 65536);
        if (v4)
            k_marginals_generic<4><<<g, 256, 0, s>>>(node_ptr, rev, unary, m, out, N, K, wl);
        else
            k_marginals_generic<1><<<g, 256, 0, s>>>(node_ptr, rev, unary, m, out, N, K, wl);
    }
    return hipGetLastError();
}

hipError_t launch_marginals_ragged(const EvalArgs& a, float* out, hipStream_t s) {
    if (a.num_nodes <= 0) return hipSuccess;
    const int waves = kBlock / 64;
    long long g = ((long long)a.num_nodes + waves - 1) / waves;
    if (g > 8192) g = 8192;
    k_marginals_ragged<<<(int)g, kBlock, 0, s>>>(a, out);
    return hipGetLastError();
}

hipError_t launch_fill_ragged(float* m, const int* moff, int E, hipStream_t s) {
    if (E <= 0) return hipSuccess;
    long long g = ((long long)E + 255) / 256;
    if (g > 8192) g = 8192;
    k_fill_ragged<<<(int)g, 256, 0, s>>>(m, moff, E);
    return hipGetLastError();
}

hipError_t launch_sparse_iteration(const EvalArgs& a, hipStream_t s) {
    // at least one block, so that a graph without slots still closes its
    // evaluation (n_t = 0)
    const int grid = a.num_nodes > 0 ? (a.num_nodes + kBlock - 1) / kBlock : 1;
    k_sparse_eval<<<grid, kBlock, 0, s>>>(a);
    k_sparse_commit<<<grid, kBlock, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_sparse_rbp_eval(const EvalArgs& a, hipStream_t s) {
    const int grid = a.num_nodes > 0 ? (a.num_nodes + kBlock - 1) / kBlock : 1;
    k_sparse_eval<<<grid, kBlock, 0, s>>>(a);
    k_sparse_rbp_close<<<1, 64, 0, s>>>(a);
    return hipGetLastError();
}

// After a run with outcome flags: rows of `prim` whose first entry carries the
// flag take the other outcome's row (when the last choice was the other
// outcome) or just lose the flag.
__global__ void k_resolve_rows(float* prim, const float* other, int take_other, long long E,
                               int K) {
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < E;
         e += (long long)gridDim.x * blockDim.x) {
        float* r = prim + e * K;
        const float v0 = r[0];
        if (!(__float_as_uint(v0) >> 31)) continue;
        if (take_other) {
            for (int x = 0; x < K; ++x) r[x] = other[e * K + x];
        } else {
            r[0] = fabsf(v0);
        }
    }
}

hipError_t launch_resolve_rows(float* const* pair_bufs, int prim, int sel, long long E, int K,
                               hipStream_t s) {
    if (E <= 0) return hipSuccess;
    long long g = (E + 255) / 256;
    if (g > 4096) g = 4096;
    k_resolve_rows<<<(int)g, 256, 0, s>>>(pair_bufs[prim], pair_bufs[prim ^ 1], sel != prim ? 1 : 0,
                                          E, K);
    return hipGetLastError();
}

hipError_t launch_sparse_rmax(const EvalArgs& a, hipStream_t s) {
    long long g = ((long long)a.num_messages + kBlock - 1) / kBlock;
    const int grid = g < 1 ? 1 : g > kSparseGridMax ? kSparseGridMax : (int)g;
    k_sparse_rmax<<<grid, kBlock, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_sparse_setup(const EvalArgs& a, int build_dst, hipStream_t s) {
    const int grid = (a.num_nodes + kBlock - 1) / kBlock;
    if (grid <= 0) return hipSuccess;
    k_sparse_setup<<<grid, kBlock, 0, s>>>(a, build_dst);
    return hipGetLastError();
}

hipError_t launch_rbp_gate(DevState* st, const CounterLine* ctr, int slot_idx, hipStream_t s) {
    k_rbp_gate<<<1, 64, 0, s>>>(st, ctr, slot_idx);
    return hipGetLastError();
}

hipError_t launch_rbp_select(DevState* st, const unsigned int* keys, const int* rev, int E,
                             unsigned int k, const CounterLine* gate_ctr, int hist0_done,
                             unsigned int* block_ties, hipStream_t s) {
    const int nb = (E + kCommitChunk - 1) / kCommitChunk;
    const int grid = nb > 0 ? nb : 1;
    // few enough blocks that their adds to one histogram word stay short
    const int hgrid = std::min(grid, kHistGrid);
    const CounterLine* gate = gate_ctr;  // the first launch
    for (int pass = hist0_done ? 1 : 0; pass < 4; ++pass) {
        k_rbp_hist<<<hgrid, kSelBlock, 0, s>>>(st, keys, E, pass, k, gate);
        gate = nullptr;
    }
    k_rbp_tiecount<<<grid, kSelBlock, 0, s>>>(st, keys, rev, E, block_ties);
    if (nb > kTieScanBlocks) k_rbp_tiescan<<<1, kSelBlock, 0, s>>>(st, block_ties, nb);
    return hipGetLastError();
}

hipError_t launch_rbp_commit(DevState* st, unsigned int* keys, const int* rev,
                             const float* cand, float* m, int E, int row, int all, int slot_idx,
                             const unsigned int* block_ties, const RbpSparse& sp,
                             const int* moff, hipStream_t s) {
    (void)slot_idx;
    const int nb = (E + kCommitChunk - 1) / kCommitChunk;
    if (nb <= 0) return hipSuccess;
    k_rbp_commit<<<nb, kSelBlock, 0, s>>>(st, keys, rev, cand, m, E, row, all, block_ties, sp,
                                         moff, nb > kTieScanBlocks ? 1 : 0);
    return hipGetLastError();
}

size_t splash_bytes(int num_nodes) {
    const size_t n = (size_t)(num_nodes > 0 ? num_nodes : 0);
    const size_t part = (sizeof(unsigned int) * n + 255) & ~size_t(255);
    const size_t lv = (sizeof(unsigned int) * n * (kSplashMaxDepth + 1) + 255) & ~size_t(255);
    return part + 2 * lv;
}

static int rs_grid(long long items) {
    const long long g = (items + kBlock - 1) / kBlock;
    return g < 1 ? 1 : g > kRsGrid ? kRsGrid : (int)g;
}

hipError_t launch_rs_gate(DevState* st, const CounterLine* ctr, int slot_idx, hipStream_t s) {
    k_rs_gate<<<1, 64, 0, s>>>(st, ctr, slot_idx);
    return hipGetLastError();
}

hipError_t launch_rs_select(const RsArgs& r, unsigned int k, int all, unsigned int* block_ties,
                            hipStream_t s) {
    const int N = r.num_nodes;
    if (N <= 0) return hipSuccess;
    k_rs_vkeys<<<rs_grid(N), kBlock, 0, s>>>(r);
    if (!all) {
        hipError_t e = launch_rbp_select(r.st, r.vkey, nullptr, N, k, nullptr, 0, block_ties, s);
        if (e != hipSuccess) return e;
    }
    const int nb = (N + kCommitChunk - 1) / kCommitChunk;
    k_rs_roots<<<nb, kSelBlock, 0, s>>>(r, all, block_ties, nb > kTieScanBlocks ? 1 : 0);
    if (r.depth >= 1) {
        k_rs_bfs<<<rs_grid(N), kBlock, 0, s>>>(r);
        k_rs_lists<<<kRsListGrid, kBlock, 0, s>>>(r);
    }
    return hipGetLastError();
}

hipError_t launch_rs_level(const RsArgs& r, int d, hipStream_t s) {
    if (r.num_nodes <= 0) return hipSuccess;
    k_rs_level_eval<<<rs_grid(r.num_nodes), kBlock, 0, s>>>(r, d);
    k_rs_level_commit<<<rs_grid(r.num_nodes), kBlock, 0, s>>>(r, d);
    return hipGetLastError();
}

hipError_t launch_fill_u32(unsigned int* p, unsigned int v, long long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_fill_u32<<<(int)blocks, 256, 0, s>>>(p, v, n);
    return hipGetLastError();
}

}  // namespace bp

// ---------------------------------------------------------------------------
// bp_run_noalloc: bp_run with its per-run scratch (iteration state, counters,
// top-k tie counts) in a file-scope device array instead of the graph's
// memory.  Each GPU holds its own copy of the array; its device address is
// looked up once per device, with that device current, and only that address
// is handed to kernels (the array's name is a host-side stand-in).
// ---------------------------------------------------------------------------
#include <mutex>

namespace {
constexpr size_t kNoAllocScratchBytes = (size_t(1) << 20) + (size_t(1) << 15);  // graphs up to ~10^9 messages
constexpr int kNoAllocMaxDevices = 64;
std::mutex g_noalloc_mu;
char* g_noalloc_ptr[kNoAllocMaxDevices];
}  // namespace

static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

extern "C" int bp_run_noalloc(bp_graph* g, int schedule, double eps, double p, uint64_t seed,
                              const bp_run_opts* opts, bp_run_stats* stats) {
    if (!g) return bp::report_error(BP_EINVAL, "graph is NULL");
    const int dev = bp::graph_device(g);
    if (dev < 0 || dev >= kNoAllocMaxDevices)
        return bp::report_error(BP_EDEVICE, "device index out of the static scratch table");
    char* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        ptr = g_noalloc_ptr[dev];
        if (!ptr) {
            int prev = -1;
            if (hipGetDevice(&prev) != hipSuccess)
                return bp::report_error(BP_EDEVICE, "hipGetDevice failed");
            if (prev != dev && hipSetDevice(dev) != hipSuccess)
                return bp::report_error(BP_EDEVICE, "hipSetDevice failed");
            void* addr = nullptr;
            const hipError_t e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
            if (prev != dev) (void)hipSetDevice(prev);
            if (e != hipSuccess || !addr)
                return bp::report_error(BP_EDEVICE, "hipGetSymbolAddress(scratch) failed");
            ptr = (char*)addr;
            g_noalloc_ptr[dev] = ptr;
        }
    }
    return bp::run_with_scratch(g, schedule, eps, p, seed, opts, stats, ptr,
                                kNoAllocScratchBytes);
}
