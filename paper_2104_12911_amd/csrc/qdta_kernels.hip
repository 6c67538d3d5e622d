// qdta_kernels.hip -- gfx950 kernels of the QDTA hot path.
//
// One Frank-Wolfe iteration of the link-flow form (Alg. 6, section 5.1):
//   k_bpr        link costs by the BPR curve (Eq. 1)
//   k_sssp_wg    destination-rooted FP32 shortest-path trees, delta-stepping
//   k_sssp_ds    (Get_shortest_path of Alg. 3 / Alg. 7), one workgroup or one
//                wavefront per tree
//   k_sssp_pull  the same trees on small networks, by passes over labels in LDS
//   k_walk       route truncation (Eq. 2) and loading along the successor
//                links (Eq. 5, Alg. 3), int64 fixed-point atomics
//   k_gap        exact sums for the relative gap, stop test
//   k_ls_*       line search on the Beckmann objective (Eq. 6, Eq. 8-10,
//                Alg. 8-9), K step sizes per pass over the links
//   k_fw_update  f <- f + rint(alpha (y - f))
// plus the tie-rule fallback under FP32 absorption, the residual-demand
// walk of Alg. 4 and the compaction of its accumulator, and the frozen-path
// model of an interval's iterations with its reverse pass (k_path_*,
// k_adj_*: derivatives for OD calibration, not part of the paper).
//
// Numeric contract: FP64 per-link arithmetic with no fused multiply-add (the
// library is compiled with -ffp-contract=off), power by repeated
// multiplication, FP32 min-plus with IEEE round-to-nearest adds, int64 flows
// in units of 2^-20 vehicle, decision sums exact as int128 multiples of 2^-16.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <type_traits>

#include "qdta_internal.h"

namespace qdta {

typedef __int128 i128;

#define RULE_NONE 0
#define RULE_CEIL 1
#define RULE_FLOOR 2
#define RULE_PROGRESS 3

static constexpr double kFxInv = 1.0 / 1048576.0;   // 2^-20, exact
static constexpr double kSumQ = 65536.0;            // 2^16

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

// Coherent (L2) load of a word that other waves update with atomics.
__device__ __forceinline__ uint32_t ld_coherent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_coherent(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every access this wavefront has issued (atomics without a result too) is done.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Exact int128 accumulation with 64-bit atomics: the value is kept as three
// signed chunk sums, v = c2 * 2^84 + c1 * 2^42 + c0.  A term takes as few of
// them as it needs (each part below 2^42 in size, so 2^20 terms fit a chunk):
// atomics on one line run one after another, about 12 ns each.
__device__ __forceinline__ void acc3_add(long long* acc, i128 v) {
    const i128 one = 1;
    if (v > -(one << 42) && v < (one << 42)) {
        if (v != 0) atomicAdd((unsigned long long*)&acc[0], (unsigned long long)(long long)v);
        return;
    }
    const unsigned long long m42 = (1ull << 42) - 1;
    const unsigned long long lo = (unsigned long long)v & m42;
    if (lo) atomicAdd((unsigned long long*)&acc[0], lo);
    v >>= 42;
    if (v > -(one << 42) && v < (one << 42)) {
        atomicAdd((unsigned long long*)&acc[1], (unsigned long long)(long long)v);
        return;
    }
    const unsigned long long mid = (unsigned long long)v & m42;
    if (mid) atomicAdd((unsigned long long*)&acc[1], mid);
    atomicAdd((unsigned long long*)&acc[2], (unsigned long long)(long long)(v >> 42));
}

__device__ __forceinline__ i128 acc3_value(const long long* acc) {
    return (i128)acc[2] * ((i128)1 << 84) + (i128)acc[1] * ((i128)1 << 42) + (i128)acc[0];
}

__device__ __forceinline__ void put128(long long* out, i128 v) {
    out[0] = (long long)(unsigned long long)v;
    out[1] = (long long)(v >> 64);
}

__device__ __forceinline__ i128 get128(const long long* in) {
    return (i128)(((unsigned __int128)(unsigned long long)in[1] << 64) | (unsigned long long)in[0]);
}

// Exact sums of many terms rint(s), s = x * 2^16, in two doubles: H takes the
// term's multiple of 2^26 (adding 1.5 * 2^78 rounds to one), L the rest.  With
// |term| < 2^66 and at most 2^13 terms (a workgroup's chunk has 2^11 links)
// |H| stays below 2^79 and |L| below 2^39, so every addition is exact and the
// order does not matter: five FP64 additions a term, where the same term as an
// int128 took the compiler's double -> int128 conversion and a 4-word add.
// Larger terms are left out and noted (odd): the workgroup then goes over its
// links once more for those alone (xsum_large), adding them to three words of LDS
// per sum, of which 2^11 such terms need a part, while 2^22 of them, one by one,
// would overflow the words in memory.  One beyond the int128 range (or not finite)
// sets bad.  (A branch for them in the loop itself: 33.2 us a pass over 255,754
// links at K = 32 with its atomics in memory, 34.8 in LDS, 32.1 so.)
struct XSum {
    double H = 0.0, L = 0.0;
};
constexpr double kXSplit = 453347182355485940514816.0;    // 1.5 * 2^78
constexpr double kXLimit = 73786976294838206464.0;        // 2^66
__device__ __forceinline__ void xsum_add(XSum& a, double s, int& odd) {
    const double v = __builtin_rint(s);
    const bool in = __builtin_fabs(v) < kXLimit;
    odd |= in ? 0 : 1;
    const double u = in ? v : 0.0;
    const double h = (u + kXSplit) - kXSplit;
    a.H += h;
    a.L += u - h;
}
__device__ __forceinline__ void xsum_large(long long* big, double s, int& bad) {
    const double v = __builtin_rint(s);
    if (__builtin_fabs(v) < kXLimit) return;
    if (__builtin_fabs(v) < 1.7e38) acc3_add(big, (i128)v);
    else bad = 1;
}
__device__ __forceinline__ i128 xsum_value(const XSum& a) { return (i128)a.H + (i128)a.L; }

// Workgroup sums of two terms per thread and of their large terms (big, in LDS;
// NULL: none), added to this workgroup's copy of an instance's exact accumulators
// ([copy][2][3] words, kSumReps copies).
__device__ void wg_pair_add(const XSum& x0, const XSum& x1, const long long* big, long long* acc,
                            double (*red)[kWG]) {
    const int tid = threadIdx.x;
    red[0][tid] = x0.H;
    red[1][tid] = x0.L;
    red[2][tid] = x1.H;
    red[3][tid] = x1.L;
    __syncthreads();
    for (int s = kWG / 2; s > 0; s >>= 1) {
        if (tid < s)
            for (int q = 0; q < 4; ++q) red[q][tid] += red[q][tid + s];
        __syncthreads();
    }
    if (tid < 2) {
        XSum x;
        x.H = red[2 * tid][0];
        x.L = red[2 * tid + 1][0];
        acc3_add(acc + 3 * tid, xsum_value(x) + (big ? acc3_value(big + 3 * tid) : 0));
    }
}

// Whether this workgroup is the last of its instance's `all` to get here (every
// thread gets the answer); the ticket is back at zero then.  The workgroups'
// atomics before this are done when the last one goes on.
__device__ __forceinline__ bool last_of_instance(unsigned int* ticket, unsigned int all, int* lds) {
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) {
        *lds = atomicAdd(ticket, 1u) == all - 1;
        if (*lds) *ticket = 0u;
    }
    __syncthreads();
    return *lds != 0;
}

// The two sums over the copies of an instance's accumulators, which are set to
// zero for the next use; one wavefront, every lane gets both.
__device__ __forceinline__ void take_sums(long long* acc, int lane, i128& s0, i128& s1) {
    long long c = 0;
    if (lane < 6) {
        long long w[kSumReps];
#pragma unroll
        for (int r = 0; r < kSumReps; ++r)
            w[r] = __hip_atomic_load(acc + r * 6 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int r = 0; r < kSumReps; ++r) {
            c += w[r];
            acc[r * 6 + lane] = 0;
        }
    }
    long long v[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) v[j] = __shfl(c, j);
    s0 = acc3_value(v);
    s1 = acc3_value(v + 3);
}

// Workgroups per link chunk for the kernels that stream over the links once:
// one per kWG links while that is not more than the card has CUs (their sums'
// atomics meet on a few words), else fewer.
static int sum_split(int nblk) {
    int split = 1;
    while (split < kChunk / kWG && nblk * split < 256) split *= 2;
    return split;
}

// BPR curve (Eq. 1): c0 (1 + alpha (kappa F / C)^beta) in FP64; with
// `marginal` the marginal cost d(F c)/dF = c0 (1 + (alpha (beta+1)) p).
__device__ __forceinline__ double bpr64(double F, float c0, float cap, double alpha, int beta, double kappa,
                                        int marginal = 0) {
    double r = (F * kappa) / (double)cap;
    double p = r;
    for (int k = 1; k < beta; ++k) p = p * r;
    const double g = marginal ? alpha * (double)(beta + 1) : alpha;
    return (double)c0 * (1.0 + g * p);
}

// Objective term and its derivative along the FW direction at step alpha:
// the Beckmann integral (Eq. 6), or under the system optimum the total
// travel time v c(v) with derivative t c0 (1 + (ab (beta+1)) p).
__device__ __forceinline__ void ls_terms(double F, double Y, float c0, float cap, double ab, int beta, double kappa,
                                         double alpha, int so, double& obj, double& der) {
    double t = Y - F;
    double v = F + alpha * t;
    double r = (v * kappa) / (double)cap;
    double p = r;
    for (int k = 1; k < beta; ++k) p = p * r;
    double cost = (double)c0 * (1.0 + ab * p);
    if (so) {
        const double mc = (double)c0 * (1.0 + (ab * (double)(beta + 1)) * p);
        obj = v * cost;
        der = t * mc;
        return;
    }
    double g = ab * v;
    g = g * p;
    g = g / (double)(beta + 1);
    obj = (double)c0 * (v + g);
    der = t * cost;
}

// ---------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_i64(int64_t* p, int64_t v, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

static int grid_for(int64_t count) {
    int64_t g = (count + kWG - 1) / kWG;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_fill_u32(hipStream_t s, uint32_t* p, uint32_t v, int64_t count) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(count)), dim3(kWG), 0, s, p, v, count);
    return hipGetLastError();
}
hipError_t launch_fill_i64(hipStream_t s, int64_t* p, int64_t v, int64_t count) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(count)), dim3(kWG), 0, s, p, v, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A1: link costs (Eq. 1)
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool inst_live(const InstState* st, int i) {
    return st == nullptr || (st[i].active && !st[i].converged);
}

// The cost of link a into the link records: the reverse records (source node,
// cost) read by the shortest-path kernels, the forward records (head node,
// cost) read by the walks, and the contracted records.
__device__ __forceinline__ void put_cost(const NetDev& net, uint2* __restrict__ radj, int a, float c) {
    const uint32_t w = __float_as_uint(c);
    radj[net.revpos[a]].y = w;
    net.fadj[a].y = w;
    if (net.cbuf) {
        const int2 at = net.cslot[a];
        if (at.x >= 0) net.cbuf[at.x] = w;
        if (at.y >= 0) net.cbuf[at.y] = w;
    }
}

// This workgroup's part of sum log(cost) (see k_prep), when asked for.
__device__ __forceinline__ void put_logsum(double s, double* logpart) {
    __shared__ double part[kWG / 64];
    if (!logpart) return;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < kWG / 64; ++k) t += part[k];
        logpart[blockIdx.x * gridDim.y + blockIdx.y] = t;
    }
}

// One link per thread: kChunk / kWG workgroups per chunk (a workgroup that took
// a whole chunk held a 1,520-link network's costs for 7 us).
__global__ __launch_bounds__(kWG) void k_bpr(NetDev net, const int64_t* __restrict__ f, double alpha, int beta,
                                             float* __restrict__ cost, uint2* __restrict__ radj,
                                             const InstState* st, int only_active, int* err,
                                             float* __restrict__ tcost, double* logpart) {
    const int b = blockIdx.x;
    const int inst = net.blk_inst[b];
    if (only_active && !inst_live(st, inst)) return;
    const InstDev I = net.inst[inst];
    const int a = net.blk_start[b] + (int)blockIdx.y * kWG + (int)threadIdx.x;
    double lg = 0.0;
    if (a < I.link0 + I.m) {
        int bad = 0;
        const double F = (double)f[a] * kFxInv;
        const float c0 = net.c0[a], cap = net.cap[a];
        const float c32 = (float)bpr64(F, c0, cap, alpha, beta, I.kappa, net.objective);
        if (!(c32 <= 3.4028234663852886e38f)) bad = 1;
        cost[a] = c32;
        if (tcost) {
            const float t32 = net.objective ? (float)bpr64(F, c0, cap, alpha, beta, I.kappa) : c32;
            if (!(t32 <= 3.4028234663852886e38f)) bad = 1;
            tcost[a] = t32;
        }
        if (radj) put_cost(net, radj, a, c32);
        if (logpart) lg = log((double)c32);
        if (bad) *err = 1;
    }
    put_logsum(lg, logpart);
}

hipError_t launch_bpr(hipStream_t s, const NetDev& net, const int64_t* f, double alpha, int beta, float* cost,
                      uint2* radj, const InstState* st, int only_active, int* err, float* tcost, double* logpart) {
    if (net.nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bpr, dim3(net.nblk, kLogParts), dim3(kWG), 0, s, net, f, alpha, beta, cost, radj, st,
                       only_active, err, tcost, logpart);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A5: line search
// ---------------------------------------------------------------------------
// The K step sizes of a K-section pass over [lo, hi], one per lane.
__device__ __forceinline__ void ks_alphas(double lo, double hi, int K, int lane, double* out) {
    if (lane < K) out[lane] = lo + ((hi - lo) * (double)lane) / (double)(K - 1);
}

// Start the line search of iteration j of one instance: one wavefront, every
// lane with the same arguments (j too: S.iter is written by one lane of the same
// kernel in k_gap, so the others must not read it there).
__device__ void ls_begin_wave(InstState& S, int j, double* al, long long* acc, int K, int ls_mode, double dx,
                              int lane) {
    for (int k = lane; k < K * 6 * kLsReps; k += 64) acc[k] = 0;
    if (ls_mode == 2) {                  // MSA
        if (lane == 0) S.alpha = 1.0 / ((double)j + 1.0);
    } else if (ls_mode == 1) {           // quasi-Newton, Alg. 8 initial guess
        const double a = 2.0 / (2.0 + (double)j);
        if (lane == 0) S.qn_alpha = a;
        if (lane < 3) al[lane] = lane == 0 ? a - dx : lane == 1 ? a : a + dx;
    } else {                              // K-section on [0, 1]
        if (lane == 0) {
            S.lo = 0.0;
            S.hi = 1.0;
        }
        ks_alphas(0.0, 1.0, K, lane, al);
    }
    if (lane == 0) {
        S.ls_pass = 0;
        S.ls_done = ls_mode == 2 ? 1 : 0;
    }
}

// A4: exact sums for the relative gap, sum c F and sum c Y, and the stop test.
// The last workgroup of an instance takes the sums and decides (Alg. 6): the
// relative gap against tol, or the iteration cap; it also advances the
// iteration index j, so a captured iteration replays with the right j, and
// starts the line search of an instance that goes on.
__global__ __launch_bounds__(kWG) void k_gap(NetDev net, const float* __restrict__ cost,
                                             const int64_t* __restrict__ f, const int64_t* __restrict__ y,
                                             long long* acc, InstState* st, int* err, unsigned int* ticket,
                                             GapRule G, double* alphas, long long* ls_acc) {
    __shared__ double red[4][kWG];
    __shared__ long long s_big[6];
    __shared__ int s_last;
    const int b = blockIdx.x;
    const int inst = net.blk_inst[b];
    if (!inst_live(st, inst)) return;
    if (threadIdx.x < 6) s_big[threadIdx.x] = 0;   // seen by all after __syncthreads_or below
    const InstDev I = net.inst[inst];
    const int part = kChunk / (int)gridDim.y;
    const int a0 = net.blk_start[b] + (int)blockIdx.y * part;
    const int a1 = min(a0 + part, I.link0 + I.m);
    long long* sums = acc + (long long)inst * kSumReps * 6;
    long long* mine = sums + ((blockIdx.y * gridDim.x + blockIdx.x) % kSumReps) * 6;
    XSum sf, sy;
    int odd = 0;
    for (int a = a0 + threadIdx.x; a < a1; a += kWG) {
        const double c = (double)cost[a];
        xsum_add(sf, c * ((double)f[a] * kFxInv) * kSumQ, odd);
        xsum_add(sy, c * ((double)y[a] * kFxInv) * kSumQ, odd);
    }
    odd = __syncthreads_or(odd);
    if (odd) {
        int bad = 0;
        for (int a = a0 + threadIdx.x; a < a1; a += kWG) {
            const double c = (double)cost[a];
            xsum_large(s_big, c * ((double)f[a] * kFxInv) * kSumQ, bad);
            xsum_large(s_big + 3, c * ((double)y[a] * kFxInv) * kSumQ, bad);
        }
        if (bad) *err = 1;
    }
    wg_pair_add(sf, sy, odd ? s_big : nullptr, mine, red);
    const unsigned int all = (unsigned int)((I.m + kChunk - 1) / kChunk) * gridDim.y;
    if (!last_of_instance(&ticket[inst], all, &s_last) || threadIdx.x >= 64) return;
    InstState& S = st[inst];
    int next = 0;                            // the iteration whose line search starts (0: none)
    i128 scf, scy;
    take_sums(sums, (int)threadIdx.x, scf, scy);
    if (threadIdx.x == 0) {
        const int j = S.iter + 1;
        S.iter = j;
        S.gap = (double)(scf - scy) / (double)scf;
        if (G.fixed_iters <= 0 && G.stop_rule == 0 && __builtin_fabs(S.gap) < G.tol) {
            S.converged = 1;
            S.stopped_by = 1;
        } else if (j > G.cap_iter) {
            S.converged = 1;
            S.stopped_by = 0;
        } else {
            next = j;
        }
    }
    next = __shfl(next, 0);
    if (next)
        ls_begin_wave(S, next, alphas + (long long)inst * G.K, ls_acc + (long long)inst * G.K * 6 * kLsReps, G.K,
                      G.ls_mode, G.dx, (int)threadIdx.x);
}

hipError_t launch_gap(hipStream_t s, const NetDev& net, const float* cost, const int64_t* f, const int64_t* y,
                      long long* acc, InstState* st, int* err, unsigned int* ticket, const GapRule& rule,
                      double* alphas, long long* ls_acc) {
    if (net.nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gap, dim3(net.nblk, sum_split(net.nblk)), dim3(kWG), 0, s, net, cost, f, y, acc, st, err,
                       ticket, rule, alphas, ls_acc);
    return hipGetLastError();
}

// Start the line search of iteration j for every live instance.
// only_fallback: restart as K-section only the instances whose quasi-Newton
// search met a non-positive C'' (ls_done == 2).
__global__ __launch_bounds__(64) void k_ls_begin(InstState* st, double* alphas, int K, int ls_mode, double dx,
                                                 long long* ls_acc, int only_fallback) {
    const int i = blockIdx.x;
    InstState& S = st[i];
    if (!S.active || S.converged) return;
    if (only_fallback && S.ls_done != 2) return;
    ls_begin_wave(S, S.iter, alphas + (long long)i * K, ls_acc + (long long)i * K * 6 * kLsReps, K, ls_mode, dx,
                  (int)threadIdx.x);
}

hipError_t launch_ls_begin(hipStream_t s, int ninst, InstState* st, double* alphas, int K, int ls_mode, double dx,
                           long long* ls_acc, int only_fallback) {
    hipLaunchKernelGGL(k_ls_begin, dim3(ninst), dim3(64), 0, s, st, alphas, K, ls_mode, dx, ls_acc, only_fallback);
    return hipGetLastError();
}

// Decide after a pass over the links: K-section bracket update (root of C', C
// convex in alpha), or one quasi-Newton step (Alg. 8 with Eq. 10).  One
// wavefront per instance, lane k with the sums of step size k (K <= 64): read
// one after another by one thread they took 8.6 us at K = 32.  The sums are
// read coherently, so the last workgroup of a pass may decide.
__device__ void ls_decide_wave(InstState& S, double* al, long long* acc, const LsRule& R, int lane) {
    const int K = R.K;
    auto sum_of = [&](int k, int which) -> i128 {
        long long c[3] = {0, 0, 0};
#pragma unroll
        for (int r = 0; r < kLsReps; ++r)
#pragma unroll
            for (int j = 0; j < 3; ++j)
                c[j] += __hip_atomic_load(acc + (r * K + k) * 6 + which * 3 + j, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
        return acc3_value(c);
    };
    auto from = [&](i128 v, int src) -> i128 {
        long long w[2];
        put128(w, v);
        w[0] = __shfl(w[0], src);
        w[1] = __shfl(w[1], src);
        return get128(w);
    };
    int done = 0;
    const int pass = S.ls_pass + 1;
    double alpha = 0.0;
    if (R.mode == 0) {
        const i128 d = lane < K ? sum_of(lane, 1) : 0;
        const unsigned long long up = __ballot(lane < K && d >= 0);
        const int kk = up ? __ffsll(up) - 1 : -1;
        if (kk <= 0) {                     // the root lies at or outside an end
            alpha = al[kk == 0 ? 0 : K - 1];
            done = 1;
        } else {
            const double lo = al[kk - 1], hi = al[kk];
            const i128 dlo = from(d, kk - 1), dhi = from(d, kk);
            if (pass >= R.passes) {
                const double da = (double)dlo, db = (double)dhi;
                alpha = lo - (da * (hi - lo)) / (db - da);
                done = 1;
            } else {
                ks_alphas(lo, hi, K, lane, al);
            }
            if (lane == 0) {
                S.lo = lo;
                S.hi = hi;
                put128(S.dlo, dlo);
                put128(S.dhi, dhi);
            }
        }
    } else {
        const i128 c = lane < 3 ? sum_of(lane, 0) : 0;
        const double cm = (double)from(c, 0) / kSumQ;
        const double c0v = (double)from(c, 1) / kSumQ;
        const double cp = (double)from(c, 2) / kSumQ;
        const double d1 = (cp - cm) / (2.0 * R.dx);
        const double d2 = ((cm - 2.0 * c0v) + cp) / (R.dx * R.dx);
        const double a = S.qn_alpha;
        if (lane == 0) S.qn_iters++;
        if (__builtin_fabs(d1) < R.T1) { alpha = a; done = 1; }
        else if (!(d2 > 0.0)) { done = 2; }               // fall back to K-section
        else {
            double an = a - d1 / d2;
            if (an < 0.0) an = 0.0;
            if (an > 1.0) an = 1.0;
            if (__builtin_fabs(an - a) < R.T2 || pass >= R.max_ls) { alpha = an; done = 1; }
            else {
                if (lane == 0) S.qn_alpha = an;
                if (lane < 3) al[lane] = lane == 0 ? an - R.dx : lane == 1 ? an : an + R.dx;
            }
        }
    }
    if (!done)
        for (int k = lane; k < K * 6 * kLsReps; k += 64) acc[k] = 0;
    if (lane == 0) {
        S.ls_evals++;
        S.ls_pass = pass;
        S.ls_done = done;
        if (done == 1) S.alpha = alpha;
    }
}

__global__ __launch_bounds__(64) void k_ls_decide(InstState* st, double* alphas, LsRule R, long long* ls_acc) {
    const int i = blockIdx.x;
    InstState& S = st[i];
    if (!S.active || S.converged || S.ls_done) return;
    ls_decide_wave(S, alphas + (long long)i * R.K, ls_acc + (long long)i * R.K * 6 * kLsReps, R, (int)threadIdx.x);
}

hipError_t launch_ls_decide(hipStream_t s, int ninst, InstState* st, double* alphas, const LsRule& R,
                            long long* ls_acc) {
    hipLaunchKernelGGL(k_ls_decide, dim3(ninst), dim3(64), 0, s, st, alphas, R, ls_acc);
    return hipGetLastError();
}

// a / b correctly rounded, y = RN(1 / b): two residual corrections (Markstein's
// theorem: the first leaves a faithful quotient, the second, whose residual is
// then exact, the rounded one) instead of the 11 operations of a division.
// Needs a quotient and residuals in the normal range: an infinite or NaN
// quotient comes out as NaN (both set the overflow flag of the sums).
template <bool FAST>
__device__ __forceinline__ double div_by(double a, double b, double y) {
    if (!FAST) return a / b;
    double q = a * y;
    q = __builtin_fma(__builtin_fma(-b, q, a), y, q);
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}

// One link as a pass over the links reads it from LDS, once for all K step
// sizes: F, Y - F, c0 * 2^16 (the sums' scale; a power of two changes no
// rounding), the capacity and its reciprocal.
struct LsLink {
    double F, t, c0q, cap, rcap;
};

// ls_terms at step size alpha, both terms times 2^16.
template <int BETA, bool SO, bool FAST>
__device__ __forceinline__ void ls_terms_q(const LsLink& l, double ab, int beta, double kappa, double rbeta1,
                                           double alpha, double& obj, double& der) {
    const double v = l.F + alpha * l.t;
    const double r = div_by<FAST>(v * kappa, l.cap, l.rcap);
    double p = r;
    if (BETA > 0) {
#pragma unroll
        for (int k = 1; k < BETA; ++k) p = p * r;
    } else {
        for (int k = 1; k < beta; ++k) p = p * r;
    }
    const double cost = l.c0q * (1.0 + ab * p);
    if (SO) {
        obj = v * cost;
        der = l.t * (l.c0q * (1.0 + (ab * (double)(beta + 1)) * p));
        return;
    }
    const double g = div_by<FAST>((ab * v) * p, (double)(beta + 1), rbeta1);
    obj = l.c0q * (v + g);
    der = l.t * cost;
}

// One pass over the links: C(alpha_k) and C'(alpha_k) for all k at once.
// Bound by FP64 issue: about 40 operations per (link, step size), 41 us for
// 1.25M links x 32 at the vector rate of the card.  A workgroup takes
// kChunk / gridDim.y links of one chunk (launch_ls_eval), stages them in LDS
// 256 at a time, and thread (g, k) = (tid / K, tid % K) takes every
// (kWG / K)-th link at step size k.  rule.on: the last workgroup of an
// instance decides (the ticket counts them), which saves the decision's own
// launch.
constexpr int kLsTile = kWG;
template <int BETA, bool SO>
__global__ __launch_bounds__(kWG) void k_ls_eval(NetDev net, const int64_t* __restrict__ f,
                                                 const int64_t* __restrict__ y, double alpha_b, int beta, int K,
                                                 double* alphas, long long* ls_acc, InstState* st, int only_pending,
                                                 int* err, int k0, int kstride, int reps, LsRule rule) {
    __shared__ union {                       // the links of a tile; after the last, the threads' sums
        LsLink link[kLsTile];
        double red[4][kWG];
    } s_mem;
    auto& s_link = s_mem.link;
    auto& s_red = s_mem.red;
    __shared__ long long s_big[2 * kMaxK * 3];   // large terms, per step size and sum
    __shared__ int s_last;
    const int b = blockIdx.x;
    const int inst = net.blk_inst[b];
    if (st && (!st[inst].active || st[inst].converged || (only_pending && st[inst].ls_done))) return;
    const InstDev I = net.inst[inst];
    const int part = kChunk / (int)gridDim.y;
    const int a0 = net.blk_start[b] + (int)blockIdx.y * part;
    const int a1 = min(a0 + part, I.link0 + I.m);
    const int tid = threadIdx.x;
    const int G = kWG / K;                    // links taken side by side
    const int k = tid % K, g = tid / K;
    const bool live = g < G;
    double* al = alphas + (long long)inst * kstride + k0;
    long long* sums = ls_acc + (long long)inst * reps * kstride * 6;     // [reps][kstride][2][3]
    const int rep = (int)((blockIdx.y * gridDim.x + blockIdx.x) % (unsigned)reps);
    long long* acc = sums + ((long long)rep * kstride + k0) * 6;
    const double alpha = live ? al[k] : 0.0;
    const double kappa = I.kappa, rbeta1 = 1.0 / (double)(beta + 1);
    // kappa far from 1 could take the quotient out of the normal range
    const bool fast = kappa > 0x1p-60 && kappa < 0x1p60;
    XSum sc, sd;
    int odd = 0, bad = 0;
    // the links of the tile at t0 into LDS; how many they are
    auto stage = [&](int t0) __attribute__((always_inline)) {
        const int nt = min(kLsTile, a1 - t0);
        if (tid < nt) {
            const int a = t0 + tid;
            LsLink l;
            l.F = (double)f[a] * kFxInv;
            l.t = (double)y[a] * kFxInv - l.F;
            l.c0q = (double)net.c0[a] * kSumQ;
            l.cap = (double)net.cap[a];
            l.rcap = 1.0 / l.cap;
            s_link[tid] = l;
        }
        __syncthreads();
        return nt;
    };
    for (int t0 = a0; t0 < a1; t0 += kLsTile) {
        const int nt = stage(t0);
        if (live) {
            double obj, der;
            if (fast) {
#pragma unroll 2
                for (int x = g; x < nt; x += G) {
                    ls_terms_q<BETA, SO, true>(s_link[x], alpha_b, beta, kappa, rbeta1, alpha, obj, der);
                    xsum_add(sc, obj, odd);
                    xsum_add(sd, der, odd);
                }
            } else {
                for (int x = g; x < nt; x += G) {
                    ls_terms_q<BETA, SO, false>(s_link[x], alpha_b, beta, kappa, rbeta1, alpha, obj, der);
                    xsum_add(sc, obj, odd);
                    xsum_add(sd, der, odd);
                }
            }
        }
        __syncthreads();
    }
    odd = __syncthreads_or(odd);
    if (odd) {                                // once more, for the large terms alone
        for (int x = tid; x < K * 6; x += kWG) s_big[x] = 0;   // (before the first tile's barrier)
        for (int t0 = a0; t0 < a1; t0 += kLsTile) {
            const int nt = stage(t0);
            if (live)
                for (int x = g; x < nt; x += G) {
                    double obj, der;
                    ls_terms_q<BETA, SO, false>(s_link[x], alpha_b, beta, kappa, rbeta1, alpha, obj, der);
                    xsum_large(s_big + k * 6, obj, bad);
                    xsum_large(s_big + k * 6 + 3, der, bad);
                }
            __syncthreads();
        }
        if (bad) *err = 1;
    }
    s_red[0][tid] = sc.H;
    s_red[1][tid] = sc.L;
    s_red[2][tid] = sd.H;
    s_red[3][tid] = sd.L;
    __syncthreads();
    int s = 1;
    while (s < G) s <<= 1;
    for (s >>= 1; s > 0; s >>= 1) {
        if (g < s && g + s < G) {
            for (int q = 0; q < 4; ++q) s_red[q][tid] += s_red[q][tid + s * K];
        }
        __syncthreads();
    }
    // threads 0..K-1 add the objective's sums, K..2K-1 the derivative's
    if (tid < 2 * K) {
        const int w = tid / K, kk = tid % K;
        XSum x;
        x.H = s_red[2 * w][kk];
        x.L = s_red[2 * w + 1][kk];
        acc3_add(acc + kk * 6 + 3 * w, xsum_value(x) + (odd ? acc3_value(s_big + kk * 6 + 3 * w) : 0));
    }
    if (!rule.on) return;
    const unsigned int all = (unsigned int)((I.m + kChunk - 1) / kChunk) * gridDim.y;
    if (last_of_instance(&rule.ticket[inst], all, &s_last) && tid < 64)
        ls_decide_wave(st[inst], al, sums, rule, tid);
}

hipError_t launch_ls_eval(hipStream_t s, const NetDev& net, const int64_t* f, const int64_t* y, double alpha_b,
                          int beta, int K, double* alphas, long long* ls_acc, InstState* st, int only_pending,
                          int* err, const LsRule& rule, int k0, int kstride, int reps) {
    if (net.nblk == 0) return hipSuccess;
    if (kstride <= 0) kstride = K;
    // Workgroups per chunk: enough of them to fill the card, each thread with
    // 16 evaluations at least (below that its reduction and atomics weigh more:
    // 256k links at K = 3 took 36 us a pass with 1,000 workgroups, 16 with 250).
    // A pass over 1.25M links at K = 32: 70 us (307 us with one workgroup per
    // chunk, int128 terms and divisions); over 1,520 links, where one chunk
    // used to be one workgroup: 8 us (114 us, and 8 us more for its decision).
    int split = 1;
    while (split < kChunk / 64 && (int64_t)net.nblk * split < 1024 && (kChunk / split) * K >= 16 * kWG) split *= 2;
    const dim3 g(net.nblk, split), blk(kWG);
#define QDTA_LS(B, SO)                                                                                             \
    hipLaunchKernelGGL((k_ls_eval<B, SO>), g, blk, 0, s, net, f, y, alpha_b, beta, K, alphas, ls_acc, st, only_pending, \
                       err, k0, kstride, reps, rule)
    if (net.objective) {
        if (beta == 4) QDTA_LS(4, true);
        else QDTA_LS(0, true);
    } else {
        if (beta == 4) QDTA_LS(4, false);
        else QDTA_LS(0, false);
    }
#undef QDTA_LS
    return hipGetLastError();
}

__global__ void k_ls_export(int ninst, const long long* ls_acc, int K, int reps, int64_t* sums) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ninst * K * 2) return;
    const int inst = t / (2 * K);
    i128 v = 0;
    for (int r = 0; r < reps; ++r)
        v += acc3_value(ls_acc + (((long long)inst * reps + r) * K * 2 + (t - inst * 2 * K)) * 3);
    put128((long long*)sums + 2 * (long long)t, v);
}

hipError_t launch_ls_export(hipStream_t s, int ninst, const long long* ls_acc, int K, int reps, int64_t* sums) {
    int n = ninst * K * 2;
    hipLaunchKernelGGL(k_ls_export, dim3((n + 63) / 64), dim3(64), 0, s, ninst, ls_acc, K, reps, sums);
    return hipGetLastError();
}

// Scratch of the allocation-free line-search entry point: error flags and the
// exact chunk accumulators, in a static array every device holds once for
// the process (kNoAllocWords 64-bit words, 196,736 bytes).  Host code never
// passes the array's name to a kernel: on the host it is not a device
// address.  noalloc_scratch() looks the device address up once per device
// (with that device current) and the kernels receive that pointer.
static __device__ __align__(256) long long scratch[kNoAllocWords];

hipError_t noalloc_scratch(int device, long long** out) {
    static std::mutex mu;
    static std::map<int, long long*> addr;
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(device);
    if (it != addr.end()) {
        *out = it->second;
        return hipSuccess;
    }
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = static_cast<long long*>(p);
    *out = static_cast<long long*>(p);
    return hipSuccess;
}

// Objective (Beckmann, or total travel time under the system optimum) of f
// (slot 0) and, apply_rule = 1, of the would-be update f + rint(alpha (y - f))
// (slot 1), exact.  The last workgroup of an instance decides: apply_rule = 1,
// the Converged test of Eq. 7 on the two; 0, slot 0 is the objective of the
// returned iterate.
__global__ __launch_bounds__(kWG) void k_obj(NetDev net, const int64_t* __restrict__ f,
                                             const int64_t* __restrict__ y, double alpha_b, int beta,
                                             long long* acc, InstState* st, int apply_rule, double tol, int* err,
                                             unsigned int* ticket) {
    __shared__ double red[4][kWG];
    __shared__ long long s_big[6];
    __shared__ int s_last;
    const int b = blockIdx.x;
    const int inst = net.blk_inst[b];
    if (!st[inst].active) return;
    if (apply_rule && st[inst].converged) return;
    if (threadIdx.x < 6) s_big[threadIdx.x] = 0;   // seen by all after __syncthreads_or below
    const InstDev I = net.inst[inst];
    const int part = kChunk / (int)gridDim.y;
    const int a0 = net.blk_start[b] + (int)blockIdx.y * part;
    const int a1 = min(a0 + part, I.link0 + I.m);
    long long* sums = acc + (long long)inst * kSumReps * 6;
    long long* mine = sums + ((blockIdx.y * gridDim.x + blockIdx.x) % kSumReps) * 6;
    const double alpha = apply_rule ? st[inst].alpha : 0.0;
    XSum s0, s1;
    int odd = 0;
    auto terms = [&](int a, double& now, double& then) {
        double der;
        const double F = (double)f[a] * kFxInv;
        ls_terms(F, F, net.c0[a], net.cap[a], alpha_b, beta, I.kappa, 0.0, net.objective, now, der);
        then = 0.0;
        if (apply_rule) {
            const int64_t fn = f[a] + (int64_t)__builtin_rint(alpha * (double)(y[a] - f[a]));
            const double Fn = (double)fn * kFxInv;
            ls_terms(Fn, Fn, net.c0[a], net.cap[a], alpha_b, beta, I.kappa, 0.0, net.objective, then, der);
        }
    };
    for (int a = a0 + threadIdx.x; a < a1; a += kWG) {
        double now, then;
        terms(a, now, then);
        xsum_add(s0, now * kSumQ, odd);
        xsum_add(s1, then * kSumQ, odd);
    }
    odd = __syncthreads_or(odd);
    if (odd) {
        int bad = 0;
        for (int a = a0 + threadIdx.x; a < a1; a += kWG) {
            double now, then;
            terms(a, now, then);
            xsum_large(s_big, now * kSumQ, bad);
            xsum_large(s_big + 3, then * kSumQ, bad);
        }
        if (bad) *err = 1;
    }
    wg_pair_add(s0, s1, odd ? s_big : nullptr, mine, red);
    const unsigned int all = (unsigned int)((I.m + kChunk - 1) / kChunk) * gridDim.y;
    if (!last_of_instance(&ticket[inst], all, &s_last) || threadIdx.x >= 64) return;
    i128 v0, v1;
    take_sums(sums, (int)threadIdx.x, v0, v1);
    if (threadIdx.x != 0) return;
    if (apply_rule) {
        const double b0 = (double)v0, b1 = (double)v1;
        if (__builtin_fabs((b0 - b1) / b0) < tol) {
            st[inst].converged = 1;
            st[inst].stopped_by = 2;
        }
    } else {
        st[inst].obj = (double)v0 / kSumQ;
    }
}

hipError_t launch_obj(hipStream_t s, const NetDev& net, const int64_t* f, const int64_t* y, double alpha_b, int beta,
                      long long* acc, InstState* st, int apply_rule, double tol, int* err, unsigned int* ticket) {
    if (net.nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_obj, dim3(net.nblk, sum_split(net.nblk)), dim3(kWG), 0, s, net, f, y, alpha_b, beta, acc, st,
                       apply_rule, tol, err, ticket);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A6: link-flow update
// ---------------------------------------------------------------------------
// One link per thread.  alpha_per_inst NULL: the step of a running iteration,
// S.alpha of each live instance, whose first workgroup also notes the applied
// update -- or, when the step is zero and no fixed iteration count was asked
// for, stops the instance: f would not change and the next iteration would
// repeat this one (a workgroup that sees it stopped has nothing to add).
__global__ __launch_bounds__(kWG) void k_fw_update(NetDev net, int64_t* __restrict__ f, const int64_t* __restrict__ y,
                                                   const double* alpha_per_inst, InstState* st, int fixed_iters) {
    const int b = blockIdx.x;
    const int inst = net.blk_inst[b];
    if (!inst_live(st, inst)) return;
    const InstDev I = net.inst[inst];
    const double alpha = alpha_per_inst ? alpha_per_inst[inst] : st[inst].alpha;
    const int a = net.blk_start[b] + (int)blockIdx.y * kWG + (int)threadIdx.x;
    if (a < I.link0 + I.m) {
        const int64_t fa = f[a];
        f[a] = fa + (int64_t)__builtin_rint(alpha * (double)(y[a] - fa));
    }
    if (!alpha_per_inst && a == I.link0) {
        InstState& S = st[inst];
        if (alpha == 0.0 && fixed_iters <= 0) {
            S.converged = 1;
            S.stopped_by = 3;
        } else {
            S.iters = S.iter;
            S.last_alpha = alpha;
        }
    }
}

hipError_t launch_fw_update(hipStream_t s, const NetDev& net, int64_t* f, const int64_t* y,
                            const double* alpha_per_inst, InstState* st, int fixed_iters) {
    if (net.nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fw_update, dim3(net.nblk, kLogParts), dim3(kWG), 0, s, net, f, y, alpha_per_inst, st,
                       fixed_iters);
    return hipGetLastError();
}

// Given costs into the link records, with the log sums of k_prep, and into
// copy where one is asked for.
__global__ __launch_bounds__(kWG) void k_scatter_rcost(NetDev net, const float* __restrict__ cost,
                                                       uint2* __restrict__ radj, double* logpart,
                                                       float* __restrict__ copy) {
    const int b = blockIdx.x;
    const InstDev I = net.inst[net.blk_inst[b]];
    const int a = net.blk_start[b] + (int)blockIdx.y * kWG + (int)threadIdx.x;
    double lg = 0.0;
    if (a < I.link0 + I.m) {
        const float c = cost[a];
        put_cost(net, radj, a, c);
        if (copy) copy[a] = c;
        lg = log((double)c);
    }
    put_logsum(lg, logpart);
}

hipError_t launch_scatter_rcost(hipStream_t s, const NetDev& net, const float* cost, uint2* radj, double* logpart,
                                float* copy) {
    if (net.nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter_rcost, dim3(net.nblk, kLogParts), dim3(kWG), 0, s, net, cost, radj, logpart, copy);
    return hipGetLastError();
}

__global__ __launch_bounds__(kWG) void k_cslot_init(NetDev net) {
    for (int64_t a = blockIdx.x * (int64_t)kWG + threadIdx.x; a < net.M; a += (int64_t)gridDim.x * kWG) {
        const int2 w = net.cslot[a];
        if (w.x >= 0) net.cbuf[w.x] = net.fadj[a].y;
        if (w.y >= 0) net.cbuf[w.y] = net.fadj[a].y;
    }
}

hipError_t launch_cslot_init(hipStream_t s, const NetDev& net) {
    if (net.M == 0 || !net.cbuf) return hipSuccess;
    hipLaunchKernelGGL(k_cslot_init, dim3(grid_for(net.M)), dim3(kWG), 0, s, net);
    return hipGetLastError();
}

// A fresh state of every instance, at iteration iter: active with links (all)
// or with legs.
__global__ void k_init_state(NetDev net, InstState* st, int all, int iter) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= net.ninst) return;
    InstState S = {};
    S.active = all ? net.inst[i].m > 0 : net.inst[i].nleg > 0;
    S.iter = iter;
    st[i] = S;
}

hipError_t launch_init_state(hipStream_t s, const NetDev& net, InstState* st, int all, int iter) {
    hipLaunchKernelGGL(k_init_state, dim3((net.ninst + 63) / 64), dim3(64), 0, s, net, st, all, iter);
    return hipGetLastError();
}

// The tables of nq trees of one instance, rooted at dest (local nodes), with
// tree-major labels of `words` words each.
__global__ void k_tree_tables(const int32_t* __restrict__ dest, int nq, int32_t node0, int32_t inst, int64_t words,
                              int32_t* dest_node, int32_t* dest_inst, int64_t* dest_lab) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nq) return;
    dest_node[t] = node0 + dest[t];
    dest_inst[t] = inst;
    dest_lab[t] = t * words;
}

hipError_t launch_tree_tables(hipStream_t s, const int32_t* dest, int nq, int32_t node0, int32_t inst, int64_t words,
                              int32_t* dest_node, int32_t* dest_inst, int64_t* dest_lab) {
    hipLaunchKernelGGL(k_tree_tables, dim3((nq + 63) / 64), dim3(64), 0, s, dest, nq, node0, inst, words, dest_node,
                       dest_inst, dest_lab);
    return hipGetLastError();
}

__global__ void k_copy_alpha(int ninst, const InstState* st, double* out) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ninst) out[i] = st[i].alpha;
}

hipError_t launch_copy_alpha(hipStream_t s, int ninst, const InstState* st, double* out) {
    hipLaunchKernelGGL(k_copy_alpha, dim3((ninst + 63) / 64), dim3(64), 0, s, ninst, st, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A2: shortest-path trees, one wavefront per destination (delta-stepping)
// ---------------------------------------------------------------------------
// A tree's label of node v is one 32-bit word, tree t's at
// labels[dest_lab[t] + v]:
//     (f << 31) | FP32 bits of D(v),   f = 1 when v is NOT queued.
// D >= 0, so the value bits order like the value.  Among queued words
// (f = 0) unsigned order is value order, so an atomicMin of a queued
// candidate both lowers the value and marks the node queued -- provided the
// candidate is below the current value, which the relaxation checks first
// with a coherent read (only the tree's own wavefront writes its labels, and
// lanes of one instruction only write queued words, which keeps that check
// valid).  The word it replaced tells whether this relaxation queued the
// node.  An atomicOr of the flag takes a node off the queue and returns its
// label.  A tree starts from +inf, not queued, on every node.
constexpr uint32_t kNotQueued = 0x80000000u;
constexpr uint32_t kValueBits = 0x7fffffffu;
constexpr uint32_t kNoNode = 0xffffffffu;
__device__ __forceinline__ const label_t* tree_labels(const label_t* labels, const DemDev& dem, int t) {
    return labels + dem.dest_lab[t];
}
__device__ __forceinline__ float lab_val(const label_t* lab, int64_t v) {
    return __uint_as_float(lab[v] & kValueBits);
}

__device__ __forceinline__ unsigned long long lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// how many of the mask's lanes are below this one
__device__ __forceinline__ int lanes_set_below(unsigned long long mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ float wave_min(float x) {
    for (int o = 32; o > 0; o >>= 1) x = fminf(x, __shfl_xor(x, o));
    return x;
}

// Each wavefront owns one destination tree at a time (a work counter hands
// out trees) and runs delta-stepping on the reverse graph: D[q] = 0, and the
// nodes taken from the near queue relax their in-links (u, w):
// D[u] = min(D[u], fl32(D[w] + c)).
//   - Up to 64 nodes are popped per step (FIFO ring); their in-links are
//     flattened across the lanes with a prefix sum of the in-degrees, so each
//     step relaxes 64 links whatever the degree mix.
//   - A relaxation that lowers a label and finds the node's queued bit clear
//     sets it and puts the node in the near queue when its label is below the
//     bucket bound thr, else in the far queue together with that label.  A
//     node is in at most one queue.  A pop clears the bit first, then reads
//     the label, so an improvement after the read queues the node again.
//   - A tree starts by writing +inf over its labels and clearing the wave's
//     bitmap (128-byte aligned streaming stores).
//   - When the near queue empties, thr moves to delta above the smallest far
//     label (kept as a running minimum) and one pass moves the far entries
//     below thr to the near queue.
// Queue counters are wave-uniform values updated from ballots, so a tree
// needs no barrier and no shared-memory atomics.  Whatever the order, the
// labels reach the least fixed point of D(v) = min_e fl32(D(head e) + c_e),
// the FP32 min-plus distance.

// U: nodes popped per lane per step (up to 64 U per step); V: in-links each
// lane relaxes per chunk, their loads, label checks and atomics issued back
// to back.
// early: stop a tree once every origin of its legs is settled (AON and
// residual walks read nothing beyond); 0 builds complete trees.
template <int U, int V>
__global__ __launch_bounds__(kWG) void k_sssp_ds(NetDev net, DemDev dem, const uint2* __restrict__ radj,
                                                 label_t* labels, Scratch scr, const InstState* st,
                                                 const float* __restrict__ delta_inst, int early, int t_begin,
                                                 int t_end) {
    constexpr int W = kWG / 64;
    constexpr int NP = 64 * U;                    // nodes per step
    __shared__ int s_pre[W][NP + 1];
    __shared__ float s_dw[W][NP];
    __shared__ int s_e0[W][NP];
    // near queue as 64 rings, one per node-id range (lane r keeps range r's
    // head and count): take offsets / heads for pops, tails / push counts
    __shared__ int s_tpre[W][64], s_rh[W][64], s_tail[W][64], s_push[W][64];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t slot = (int64_t)blockIdx.x * W + wv;
    const unsigned long long below = lanes_below(lane);
    int32_t* nearq = scr.nearq + slot * scr.nmax;
    uint2* farq = reinterpret_cast<uint2*>(scr.farq) + slot * scr.nmax;
    int* pre = s_pre[wv];
    float* sdw = s_dw[wv];
    int* se0 = s_e0[wv];
    int* tpre = s_tpre[wv];
    int* rhd = s_rh[wv];
    int* rtail = s_tail[wv];
    int* rpush = s_push[wv];

    for (;;) {
        int t = 0;
        if (lane == 0) t = t_begin + atomicAdd(scr.work, 1);
        t = __shfl(t, 0);
        if (t >= t_end) break;
        const int inst = dem.dest_inst[t];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int n = I.n, node0 = I.node0;
        const int* __restrict__ rptr = net.rptr + node0;
        label_t* D = labels + dem.dest_lab[t];
        const int root = dem.dest_node[t] - node0;
        const float delta = delta_inst[inst];
        // reset the tree's labels to +inf, not queued (the region is 128-byte
        // aligned and padded to a multiple of 32 words)
        {
            uint4* D4 = reinterpret_cast<uint4*>(D);
            const uint32_t w0 = kNotQueued | kInfBits;
            const uint4 inf4 = make_uint4(w0, w0, w0, w0);
            const int n4 = (n + 31) / 32 * 8;
            for (int i = lane; i < n4; i += 64) D4[i] = inf4;
        }
        __threadfence_block();
        // ranges of 2^rsh node ids (at most 64); ring r holds at most the
        // range's nodes (each node is queued once): capacity size + 1, so the
        // rings take n + 64 entries
        int rsh = 0;
        while (((n - 1) >> rsh) >= 64) ++rsh;
        const int rs = 1 << rsh;
        const int nranges = ((n - 1) >> rsh) + 1;
        const bool rvalid = lane < nranges;
        const int rcap = rvalid ? min(rs, n - lane * rs) + 1 : 1;
        if (lane == 0) {
            D[root] = 0u;                         // value 0, queued
            nearq[(root >> rsh) * (rs + 1)] = root;
        }
        __threadfence_block();
        int rh = 0, rc = (lane == (root >> rsh)) ? 1 : 0;
        // ring slot of range r at position pos (r < nranges)
        auto ring_at = [&](int r, int pos) -> int32_t* {
            const int cap = min(rs, n - r * rs) + 1;
            if (pos >= cap) pos -= cap;
            return nearq + (int64_t)r * (rs + 1) + pos;
        };
        // before a phase that pushes to near: tails after the pops, counters at 0
        auto open_push = [&]() {
            int tl = rh + rc;
            if (tl >= rcap) tl -= rcap;
            rtail[lane] = tl;
            rpush[lane] = 0;
            __builtin_amdgcn_wave_barrier();
        };
        auto push_near = [&](int v) {
            const int r = v >> rsh;
            *ring_at(r, rtail[r] + atomicAdd(&rpush[r], 1)) = v;
        };
        // after it: the ring counts take in what was pushed
        auto close_push = [&]() {
            __builtin_amdgcn_wave_barrier();
            if (rvalid) rc += rpush[lane];
        };
        const int l0 = early ? dem.qptr[t] : 0, l1 = early ? dem.qptr[t + 1] : 0;
        int ncnt = 1;                             // queued in near (sum of the ring counts)
        int fcnt = 0;
        float thr = delta;
        float fmin = __uint_as_float(kInfBits);   // smallest label pushed to far
        for (;;) {
            while (ncnt > 0) {
                const int k = ncnt < NP ? ncnt : NP;
                // pop from the lowest non-empty ranges first: nodes close in id
                // (and, in Hilbert order, in space) are handled together, so
                // their label lines are reused before they leave the cache
                int incl = rc;
                for (int o = 1; o < 64; o <<= 1) {
                    const int x = __shfl_up(incl, o);
                    if (lane >= o) incl += x;
                }
                const int excl = incl - rc;
                const int take = max(0, min(rc, NP - excl));
                tpre[lane] = min(excl, NP);
                rhd[lane] = rh;
                __builtin_amdgcn_wave_barrier();
                // pop: slot j = u * 64 + lane, from the largest range r with tpre[r] <= j
                int deg[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = u * 64 + lane;
                    deg[u] = 0;
                    if (j < k) {
                        int lo = 0, hi = 64;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (tpre[mid] <= j) lo = mid; else hi = mid;
                        }
                        const int w = *ring_at(lo, rhd[lo] + (j - tpre[lo]));
                        const uint32_t lw = atomicOr(&D[w], kNotQueued);   // dequeue, read the label
                        const int e0 = rptr[w];
                        deg[u] = rptr[w + 1] - e0;
                        se0[j] = e0;
                        sdw[j] = __uint_as_float(lw & kValueBits);
                    }
                }
                rh += take;
                if (rh >= rcap) rh -= rcap;
                rc -= take;
                ncnt -= k;
                open_push();
                // exclusive prefix of in-degrees in slot order
                int base = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    int incl = deg[u];
                    for (int o = 1; o < 64; o <<= 1) {
                        const int x = __shfl_up(incl, o);
                        if (lane >= o) incl += x;
                    }
                    pre[u * 64 + lane] = base + incl - deg[u];
                    base += __shfl(incl, 63);
                }
                if (lane == 0) pre[k] = base;
                const int total = base;
                __builtin_amdgcn_wave_barrier();
                for (int g0 = 0; g0 < total; g0 += 64 * V) {
                    int vv[V];
                    float cd[V];
                    bool ok[V];
#pragma unroll
                    for (int x = 0; x < V; ++x) {
                        const int g = g0 + x * 64 + lane;
                        ok[x] = g < total;
                        vv[x] = 0;
                        cd[x] = 0.0f;
                        if (ok[x]) {
                            int lo = 0, hi = k;   // owner slot: pre[lo] <= g < pre[lo + 1]
                            while (hi - lo > 1) {
                                const int mid = (lo + hi) >> 1;
                                if (pre[mid] <= g) lo = mid; else hi = mid;
                            }
                            const int e = se0[lo] + (g - pre[lo]);
                            const uint2 r = radj[e];
                            vv[x] = (int)r.x - node0;
                            cd[x] = sdw[lo] + __uint_as_float(r.y);
                        }
                    }
                    uint32_t cur[V];               // current value bits (coherent: see the word layout)
#pragma unroll
                    for (int x = 0; x < V; ++x) cur[x] = ok[x] ? (ld_coherent(&D[vv[x]]) & kValueBits) : 0u;
                    bool pn[V], pf[V];
#pragma unroll
                    for (int x = 0; x < V; ++x) {
                        pn[x] = pf[x] = false;
                        const uint32_t cb = __float_as_uint(cd[x]);
                        // cb is a queued word below the value: the min lowers the value;
                        // a replaced word that was not queued means this relaxation queued v
                        if (ok[x] && cb < cur[x] && (atomicMin(&D[vv[x]], cb) & kNotQueued)) {
                            pn[x] = cd[x] < thr;
                            pf[x] = !pn[x];
                        }
                    }
                    float fm = __uint_as_float(kInfBits);
#pragma unroll
                    for (int x = 0; x < V; ++x) {
                        const unsigned long long bn = __ballot(pn[x]), bf = __ballot(pf[x]);
                        if (pn[x]) push_near(vv[x]);
                        if (pf[x]) {
                            farq[fcnt + __popcll(bf & below)] = make_uint2((uint32_t)vv[x], __float_as_uint(cd[x]));
                            fm = fminf(fm, cd[x]);
                        }
                        ncnt += __popcll(bn);
                        fcnt += __popcll(bf);
                    }
                    fmin = fminf(fmin, wave_min(fm));
                }
                close_push();
                __threadfence_block();
            }
            // Bucket [.., thr) is drained.  Far entries carry the label they had
            // when queued; one improved since may now lie below thr.
            if (early) {
                // all origins below thr?  (cheap test before the exact one)
                bool pend = false;
                for (int l = l0 + lane; l < l1; l += 64) {
                    const int o = dem.leg_orig[l] - node0;
                    if (!(__uint_as_float(ld_coherent(&D[o]) & kValueBits) < thr)) pend = true;
                }
                if (__ballot(pend) == 0ull) {
                    // exact: move far entries whose current label is below thr
                    int moved = 0;
                    open_push();
                    for (int i0 = 0; i0 < fcnt; i0 += 64) {
                        const int i = i0 + lane;
                        const bool h = i < fcnt;
                        const uint2 ent = h ? farq[i] : make_uint2(0u, kInfBits);
                        const float dv = h ? __uint_as_float(ld_coherent(&D[ent.x]) & kValueBits) : 0.0f;
                        const bool late = h && dv < thr;
                        const unsigned long long bl = __ballot(late);
                        if (late) push_near((int)ent.x);
                        // keep the rest, in order
                        const unsigned long long bk = __ballot(h && !late);
                        if (h && !late) farq[i0 - moved + __popcll(bk & below)] = ent;
                        ncnt += __popcll(bl);
                        moved += __popcll(bl);
                    }
                    fcnt -= moved;
                    close_push();
                    __threadfence_block();
                    if (moved == 0) break;            // every node below thr is settled
                    if (fcnt > 0) {
                        float km = __uint_as_float(kInfBits);
                        for (int i = lane; i < fcnt; i += 64) km = fminf(km, __uint_as_float(farq[i].y));
                        fmin = wave_min(km);
                    } else {
                        fmin = __uint_as_float(kInfBits);
                    }
                    continue;
                }
            }
            if (fcnt == 0) break;
            // next bucket: delta above the smallest far label
            thr = fmaxf(thr, fmin) + delta;
            // FP32 absorption can make fmin + delta == fmin: always admit the minimum
            if (!(thr > fmin)) thr = __uint_as_float(__float_as_uint(fmin) + 1u);
            int keep = 0;
            float kmin = __uint_as_float(kInfBits);
            open_push();
            for (int i0 = 0; i0 < fcnt; i0 += 64) {
                const int i = i0 + lane;
                const bool h = i < fcnt;
                uint2 ent = h ? farq[i] : make_uint2(0u, kInfBits);
                // by the label now: an improved node is not queued again
                if (h) ent.y = ld_coherent(&D[ent.x]) & kValueBits;
                const float dv = __uint_as_float(ent.y);
                const bool ton = h && dv < thr;
                const bool tok = h && !ton;
                const unsigned long long bn = __ballot(ton), bk = __ballot(tok);
                if (ton) push_near((int)ent.x);
                if (tok) farq[keep + __popcll(bk & below)] = ent;
                ncnt += __popcll(bn);
                keep += __popcll(bk);
                kmin = fminf(kmin, tok ? dv : __uint_as_float(kInfBits));
            }
            fcnt = keep;
            fmin = wave_min(kmin);
            close_push();
            __threadfence_block();
        }
    }
}

// Workgroup-per-tree form of delta-stepping: the NT = 128 U threads of a
// workgroup grow one tree together, each relaxing V records a step.
//   - A label here is the plain FP32 value, with no queued flag: a relaxation
//     that lowers a label queues the node together with the value it wrote, and
//     a pop uses that value.  A node improved again while it waits is queued
//     again, and its older entry relaxes nothing that the newer one would not
//     lower further.  A pop therefore touches no label at all.
//   - A queue entry is (node, row, value, parent).  The row is the node's
//     packed record row, which saves a pop the row pointers, or kNoRow + the
//     number of records already relaxed.  Records whose source is the parent,
//     the node this value came from, are skipped: adding non-negative costs to a
//     value that came from the parent's label cannot lower that label.
//   - A step takes up to NT entries, from a circular buffer in LDS, then from the
//     ring in memory that takes the buffer's overflow.  V neighbouring lanes
//     relax an entry, one record each, so that a row is one piece of memory to
//     the load; a wavefront takes 64 / V entries a round, every wavefront as many
//     rounds as the step's entries need (at most V, issued together).  The rest
//     of a row longer than V is queued again in pieces of V.
//   - No label is changed by an atomic: on this memory they are carried out
//     beyond the L2 (one memory write each, and the line leaves the L2).  Only
//     the tree's own workgroup touches its labels, so a step's improvements meet
//     in a table in LDS: each puts its key (step, value, its number) into the
//     slot of its node's hash by one atomic minimum.  Keys of a later step are
//     smaller, so the table is not cleared.  After a barrier a candidate whose
//     key is still there stores the label and queues the node; one beaten by a
//     key of the same node is done; one beaten by another node's key (about one
//     in 20) has its record queued again, as a row of one, for the next step.
//     Two barriers a step, and two dependent memory accesses, record and label.
//   - Entries at or above the bucket bound thr go to the far queue.  When the
//     near entries are used up, thr moves delta above the smallest far value and
//     one pass moves the far entries below it, dropping those whose label has
//     been lowered since.  A near entry that finds the ring full goes to the far
//     queue too; a far queue that could overflow in the next step is compacted
//     to its live entries first, of which a node has at most one.
//
// CT: the chain-contracted search.  Nodes left out by the contraction are
// never queued; the kept nodes' in-links come from the contracted records
// (a chain's record adds its link costs one at a time); a leg whose origin
// is left out waits for the kept nodes its label depends on; the chain
// nodes' labels are filled from their chains' ends afterwards (k_chain_fill).
//
// Bound by the rate of memory requests where all trees together are far larger
// than the L2 (550k nodes, 5,000 trees: 48 ms, 84 ms before this form; 1.83G line
// reads and 1.14G writes leave the L2, 38G reads a second beside 24G writes, where
// a gather of random words, one read each, reaches 41G), by the latency of a
// step's chain of accesses and the issue of its instructions below that (metro
// network, 100k nodes, 1,000 trees: 2.1 ms, 5.7; 22,801-node grid, 300 trees:
// 0.69 ms, 3.77; 400-node grid, 40 trees: 0.06 ms, 0.13).  What each part gave on
// the 550k nodes: no flag and no pop access 84 -> 65 ms, no atomics -> 56, no
// dependent cost block for a chain -> 54.6, the step's two barriers and
// branch-free phases -> 51 (and 2.7 -> 2.4 ms on the metro network, 1.2 -> 0.8 on
// the grid), lanes over records with minimum keys instead of a thread per entry
// with compare-and-swapped slots -> 48 (2.4 -> 2.1, 0.79 -> 0.69).
//
// The registers of <2, 4> and <2, 2> are kept to 128 VGPRs, for the four
// workgroups per CU that the LDS holds (151 of them, for three: 2.7 instead of
// 2.1 ms on the metro network, whose 1,000 trees then take two turns).  W is the
// most wavefronts per SIMD that the allocation is told to aim at; with that
// minimum it decides nothing (<2, 4, true> compiles to the same code with 7 and
// with 8), but it is part of the name that kernel traces are searched for.
template <int U, int V, bool CT, int W = 8>
__global__ __launch_bounds__(128 * U) __attribute__((amdgpu_waves_per_eu(U == 2 ? 4 : 1, W))) void k_sssp_wg(
    NetDev net, DemDev dem, const uint2* __restrict__ radj, label_t* labels, Scratch scr, const InstState* st,
    const float* __restrict__ delta_inst, int early, int t_begin, int t_end) {
    constexpr int NT = 128 * U;
    constexpr int NW = NT / 64;
    constexpr int E = 64 / V;                     // entries of a round: one record per lane
    constexpr int NB = 2 * NT;                    // entries of the LDS buffer
    constexpr int NH = 2 * V * NT;                // slots of the hash table, twice what a step can take
    constexpr int kIdBits = 11;
    constexpr uint32_t kIdMask = (1u << kIdBits) - 1u;
    constexpr uint32_t kEpochs = 1u << (32 - kIdBits);
    static_assert(NT * V <= 1 << kIdBits, "a candidate's number fits");
    constexpr int F = NT >= 512 ? 1 : 512 / NT;   // far entries per thread and turn of a pass over them
    static_assert(NT * (V + 1) <= kSearchSlack, "the far queue has room for one step beyond a node each");
    // 64 spare words after the first two: what a lane without work reads and
    // writes (its own word), so that the accesses of a phase are issued back to
    // back with no branch between them
    __shared__ uint4 s_buf[NB + 64];              // near entries
    __shared__ unsigned long long s_val[NH + 64]; // per slot the least key put into it
    __shared__ uint2 s_cand[V * NT];              // node and value of each candidate of the step
    __shared__ unsigned long long s_cnt[2];       // far << 32 | near entries pushed in a step (odd, even)
    __shared__ int s_t;                           // next tree
    __shared__ uint32_t s_fm;                     // smallest value pushed to far
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lx = lane & (V - 1);
    const int cap = (int)scr.nmax;                // entries of the ring and of the far queue
    uint4* nearq = reinterpret_cast<uint4*>(scr.nearq) + (int64_t)blockIdx.x * scr.nmax;
    uint4* farq = reinterpret_cast<uint4*>(scr.farq) + (int64_t)blockIdx.x * scr.nmax;
    const uint4* __restrict__ crec = reinterpret_cast<const uint4*>(net.cbuf);
    for (int x = tid; x < NH + 64; x += NT) s_val[x] = ~0ull;
    uint32_t epoch = kEpochs - 1u;
    unsigned long long n_taken = 0;               // counted by every thread alike (uniform values)
    unsigned int n_relaxed = 0;                   // this thread's own
    for (;;) {
        if (tid == 0) s_t = t_begin + atomicAdd(scr.work, 1);
        __syncthreads();
        const int t = s_t;
        __syncthreads();
        if (t >= t_end) break;
        const int inst = dem.dest_inst[t];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int n = I.n;
        const uint32_t node0 = (uint32_t)I.node0;
        const int* __restrict__ rptr = (CT ? net.crptr : net.rptr) + node0;
        const uint32_t* __restrict__ crow = CT ? net.crow + node0 : nullptr;
        label_t* D = labels + dem.dest_lab[t];
        const int root = dem.dest_node[t] - (int)node0;
        const float delta = delta_inst[inst];
        {
            uint4* D4 = reinterpret_cast<uint4*>(D);
            const uint4 inf4 = make_uint4(kInfBits, kInfBits, kInfBits, kInfBits);
            const int n4 = (n + 31) / 32 * 8;
            for (int i = tid; i < n4; i += NT) D4[i] = inf4;
        }
        __threadfence_block();
        __syncthreads();
        if (tid == 0) {
            D[root] = 0u;
            s_buf[0] = make_uint4((uint32_t)root, CT ? crow[root] : kNoRow, 0u, kNoNode);
            s_cnt[0] = s_cnt[1] = 0ull;
        }
        __threadfence_block();
        __syncthreads();
        int bh = 0, bc = 1, rh = 0, rc = 0;       // head and count of the buffer and of the ring
        int fcnt = 0, par = 0;                    // far entries; which counters the next pushes use
        float thr = delta;
        float lfm = __uint_as_float(kInfBits);    // smallest far value this thread has pushed since the last pass
        // first positions of this wavefront's entries of the two queues
        auto reserve = [&](int near, int far, int& pn, int& pf) {
            unsigned long long p = 0ull;
            if (lane == 0) p = atomicAdd(&s_cnt[par], ((unsigned long long)far << 32) | (unsigned)near);
            pn = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
            pf = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
        };
        // The near entry number p of a pushing phase that found bc and rc entries:
        // into the buffer, else the ring; false if both are full.
        auto put_near = [&](int p, const uint4& ent) -> bool {
            if (p < NB - bc) {
                s_buf[(bh + bc + p) & (NB - 1)] = ent;
                return true;
            }
            const int r = p - (NB - bc);
            if (r >= cap - rc) return false;
            int q = rh + rc + r;
            if (q >= cap) q -= cap;
            nearq[q] = ent;
            return true;
        };
        auto put_far = [&](int p, const uint4& ent) {
            farq[fcnt + p] = ent;
            lfm = fminf(lfm, __uint_as_float(ent.z));
        };
        // after the barrier that ends a pushing phase: its entries are counted in
        auto fold = [&]() {
            const unsigned long long c = s_cnt[par];
            const int nn = __builtin_amdgcn_readfirstlane((int)(uint32_t)c), ib = min(nn, NB - bc);
            fcnt += __builtin_amdgcn_readfirstlane((int)(uint32_t)(c >> 32));
            rc += min(nn - ib, cap - rc);
            bc += ib;
            par ^= 1;
            if (tid == 0) s_cnt[par] = 0ull;      // read by all before the phase that just ended
        };
        // One pass over the first total_far far entries: those below `below_thr`
        // whose label is still theirs go to near, the others below it are dropped,
        // the rest stay; all = drop every entry whose label is not its own.
        auto sweep_far = [&](float below_thr, bool all) {
            const int total_far = fcnt;
            fcnt = 0;                             // entries kept are pushed from the front again
            lfm = __uint_as_float(kInfBits);
            for (int i0 = 0; i0 < total_far; i0 += NT * F) {
                uint4 ent[F];
                bool low[F], keep[F];
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const int i = i0 + f * NT + tid;
                    keep[f] = i < total_far;
                    ent[f] = keep[f] ? farq[i] : make_uint4(0u, 0u, kInfBits, 0u);
                }
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    low[f] = keep[f] && __uint_as_float(ent[f].z) < below_thr;
                    if (low[f] || (keep[f] && all)) keep[f] = D[ent[f].x] == ent[f].z;
                    low[f] = low[f] && keep[f];
                    keep[f] = keep[f] && !(__uint_as_float(ent[f].z) < below_thr);
                }
                __syncthreads();                  // the turn's entries are read before they are overwritten
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const unsigned long long bn = __ballot(low[f]);
                    int p, q;
                    if (bn) {
                        reserve(__popcll(bn), 0, p, q);
                        if (low[f]) keep[f] = !put_near(p + lanes_set_below(bn), ent[f]);
                    }
                    const unsigned long long bf = __ballot(keep[f]);
                    if (bf) {
                        reserve(0, __popcll(bf), p, q);
                        if (keep[f]) put_far(q + lanes_set_below(bf), ent[f]);
                    }
                }
            }
            __syncthreads();
            fold();
        };
        int lcur = early ? dem.qptr[t] : 0;
        const int lend = early ? dem.qptr[t + 1] : 0;
        for (;;) {
            while (bc + rc > 0) {
                if (fcnt + NT * (V + 1) > cap) {
                    __syncthreads();              // the counters' reset is seen
                    sweep_far(0.0f, true);        // keep only the live far entries
                }
                if (--epoch == 0u) {
                    for (int x = tid; x < NH + 64; x += NT) s_val[x] = ~0ull;
                    epoch = kEpochs - 2u;
                    __syncthreads();
                }
                const int k = min(bc + rc, NT), kb = min(bc, k);
                // this wavefront's rounds: every NW-th E entries
                const int rounds = k > wv * E ? (k - wv * E + NW * E - 1) / (NW * E) : 0;
                uint4 ent[V], r[V];
                uint32_t cb[V];                   // candidates
                uint32_t okm = 0u, lng = 0u;      // bit j: may lower its source; first of a row longer than V
                auto row_of = [&](const uint4& e, int& first, int& deg) {
                    if (e.y & kNoRow) {
                        first = rptr[e.x] + (int)(e.y & ~kNoRow);
                        deg = rptr[e.x + 1] - first;
                        if (deg == 0) first = 0;
                    }
                };
                auto slot_of = [&](uint32_t v, bool p) {
                    return p ? (int)((v * 2654435761u) >> 16) & (NH - 1) : NH + lane;
                };
                auto relax = [&](auto nr) __attribute__((always_inline)) {
                    constexpr int R = decltype(nr)::value;
                    int e0[R], deg[R];
                    bool in[R], un = false;
#pragma unroll
                    for (int j = 0; j < R; ++j) ent[j] = s_buf[(bh + (j * NW + wv) * E + lane / V) & (NB - 1)];
                    if (k > kb) {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const int i = (j * NW + wv) * E + lane / V;
                            int q = rh + (i - kb);
                            if (q >= cap) q -= cap;
                            if (i >= kb && i < k) ent[j] = nearq[q];
                        }
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        in[j] = (j * NW + wv) * E + lane / V < k;
                        e0[j] = in[j] ? (int)(ent[j].y >> kRowCountBits) : 0;
                        deg[j] = in[j] ? (int)(ent[j].y & ((1u << kRowCountBits) - 1u)) : 0;
                        un |= in[j] && (ent[j].y & kNoRow);
                    }
                    if (__ballot(un)) {
#pragma unroll
                        for (int j = 0; j < R; ++j)
                            if (in[j]) row_of(ent[j], e0[j], deg[j]);
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const int at = e0[j] + min(lx, max(deg[j] - 1, 0));
                        if (CT) {
                            r[j] = crec[at];
                        } else {
                            const uint2 q = radj[at];
                            r[j] = make_uint4(q.x, q.y, 0u, kNoRow);
                        }
                    }
                    uint32_t cur[R], two = 0u;
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        // form 0: a link; 1, 2: a chain's two or three costs; the last
                        // word is the source's packed row but for form 2 (see below)
                        const float d = __uint_as_float(ent[j].z);
                        const uint32_t form = CT ? r[j].x >> 30 : 0u;
                        r[j].x = (CT ? r[j].x & 0x3fffffffu : r[j].x) - node0;
                        const float c1 = d + __uint_as_float(r[j].y);
                        const float c2 = c1 + __uint_as_float(r[j].z);
                        const float c3 = c2 + __uint_as_float(r[j].w);
                        cb[j] = __float_as_uint(form == 0u ? c1 : form == 1u ? c2 : c3);
                        const bool ok = lx < deg[j] && r[j].x != ent[j].w;
                        okm |= ok ? 1u << j : 0u;
                        lng |= lx == 0 && deg[j] > V ? 1u << j : 0u;
                        if (CT) two |= ok && form == 2u ? 1u << j : 0u;
                        cur[j] = D[ok ? r[j].x : 0u];
                        n_relaxed += lx < deg[j] ? 1u : 0u;
                    }
                    if (CT && __ballot(two != 0u)) {
#pragma unroll
                        for (int j = 0; j < R; ++j)
                            if (two >> j & 1u) r[j].w = crow[r[j].x];
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const uint32_t id = (uint32_t)((j * NW + wv) * 64 + lane);
                        const bool p = (okm >> j & 1u) && cb[j] < cur[j];
                        okm = p ? okm : okm & ~(1u << j);
                        const unsigned long long key =
                            (unsigned long long)__builtin_amdgcn_alignbit(epoch, cb[j], 32 - kIdBits) << 32 |
                            (cb[j] << kIdBits | id);
                        atomicMin(&s_val[slot_of(r[j].x, p)], key);
                        s_cand[id] = make_uint2(r[j].x, cb[j]);
                    }
                };
                if constexpr (V == 2) {
                    if (rounds == 1) relax(std::integral_constant<int, 1>{});
                    else if (rounds) relax(std::integral_constant<int, 2>{});
                } else {
                    if (rounds == 1) relax(std::integral_constant<int, 1>{});
                    else if (rounds == 2) relax(std::integral_constant<int, 2>{});
                    else if (rounds == 3) relax(std::integral_constant<int, 3>{});
                    else if (rounds) relax(std::integral_constant<int, V>{});
                }
                const int kr = k - kb;
                bh = (bh + kb) & (NB - 1);
                bc -= kb;
                rh += kr;
                if (rh >= cap) rh -= cap;
                rc -= kr;
                n_taken += (unsigned)k;
                __syncthreads();
                // the least key of each slot is its candidate's, which writes the label
                // and queues the node
                auto resolve = [&](auto nr) __attribute__((always_inline)) {
                    constexpr int R = decltype(nr)::value;
                    uint32_t top[R], win = 0u, put;
                    unsigned long long bn[R], bf[R];
                    int cn = 0, cf = 0;
#pragma unroll
                    for (int j = 0; j < R; ++j) top[j] = (uint32_t)s_val[slot_of(r[j].x, okm >> j & 1u)];
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const uint32_t id = (uint32_t)((j * NW + wv) * 64 + lane);
                        const bool w = (okm >> j & 1u) && top[j] == (cb[j] << kIdBits | id);
                        win |= w ? 1u << j : 0u;
                        if (w) D[r[j].x] = cb[j];
                    }
                    put = win;
                    if (__ballot(lng != 0u)) {
                        // the rest of a longer row: pieces of V records; or, if its row does
                        // not pack or the near queues are full, one entry with all of it
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const bool l = lng >> j & 1u;
                            if (!__ballot(l)) continue;
                            int first = (int)(ent[j].y >> kRowCountBits), deg = l ? (int)(ent[j].y & ((1u << kRowCountBits) - 1u)) : 0;
                            if (l) row_of(ent[j], first, deg);
                            const int row0 = l ? rptr[ent[j].x] : 0;
                            for (int done = V; __ballot(done < deg) != 0ull; done += V) {
                                const bool more = done < deg;
                                const uint32_t rest = kNoRow + (uint32_t)(first + done - row0);
                                uint4 e = make_uint4(ent[j].x, pack_row(first + done, min(V, deg - done)), ent[j].z,
                                                     ent[j].w);
                                if (e.y == kNoRow) e.y = rest;
                                const unsigned long long bm = __ballot(more);
                                int p, q;
                                reserve(__popcll(bm), 0, p, q);
                                const bool full = more && !put_near(p + lanes_set_below(bm), e);
                                const unsigned long long bw = __ballot(full);
                                if (bw) {
                                    e.y = rest;
                                    reserve(0, __popcll(bw), p, q);
                                    if (full) put_far(q + lanes_set_below(bw), e);
                                }
                                if (more && (e.y & kNoRow)) deg = 0;   // all of it is queued
                            }
                        }
                    }
                    uint32_t lost = okm & ~win, hard = 0u;
                    if (__ballot(lost != 0u)) {
                        // a candidate that met another node's key in its slot has its record
                        // queued again, as a row of one; where that does not pack, see below
                        uint32_t other[R];
#pragma unroll
                        for (int j = 0; j < R; ++j) other[j] = s_cand[top[j] & kIdMask].x;
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const bool l = (lost >> j & 1u) && other[j] != r[j].x;
                            int first = (int)(ent[j].y >> kRowCountBits), deg = 0;
                            if (l) row_of(ent[j], first, deg);
                            const uint32_t y = pack_row(first + lx, 1);
                            const bool again = l && y != kNoRow;
                            hard |= l && !again ? 1u << j : 0u;
                            put |= again ? 1u << j : 0u;
                            r[j].x = again ? ent[j].x : r[j].x;
                            r[j].w = again ? y : r[j].w;
                            cb[j] = again ? ent[j].z : cb[j];
                            ent[j].x = again ? ent[j].w : ent[j].x;
                        }
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const bool p = put >> j & 1u, nr = __uint_as_float(cb[j]) < thr;
                        bn[j] = __ballot(p && nr);
                        bf[j] = __ballot(p && !nr);
                        cn += __popcll(bn[j]);
                        cf += __popcll(bf[j]);
                    }
                    int p, q;
                    reserve(cn, cf, p, q);
                    if (p + cn <= NB - bc) {      // this wavefront's near entries all go to the buffer
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const bool w = (put >> j & 1u) && __uint_as_float(cb[j]) < thr;
                            const int at = (bh + bc + p + lanes_set_below(bn[j])) & (NB - 1);
                            s_buf[w ? at : NB + lane] = make_uint4(r[j].x, r[j].w, cb[j], ent[j].x);
                            p += __popcll(bn[j]);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const uint4 e = make_uint4(r[j].x, r[j].w, cb[j], ent[j].x);
                            bool full = false;
                            if ((put >> j & 1u) && __uint_as_float(cb[j]) < thr)
                                full = !put_near(p + lanes_set_below(bn[j]), e);
                            p += __popcll(bn[j]);
                            if (full && !(win >> j & 1u)) {
                                hard |= 1u << j;
                                full = false;
                            }
                            const unsigned long long bx = __ballot(full);
                            if (bx) {             // ring full
                                int p1, q1;
                                reserve(0, __popcll(bx), p1, q1);
                                if (full) put_far(q1 + lanes_set_below(bx), e);
                            }
                        }
                    }
                    if (cf) {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            if ((put >> j & 1u) && !(__uint_as_float(cb[j]) < thr))
                                put_far(q + lanes_set_below(bf[j]), make_uint4(r[j].x, r[j].w, cb[j], ent[j].x));
                            q += __popcll(bf[j]);
                        }
                    }
                    if (__ballot(hard != 0u)) {
                        // no room for the record, or its row does not pack: no other node's
                        // key won this slot, so only such candidates write the label now
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            const bool h = hard >> j & 1u;
                            const uint32_t id = (uint32_t)((j * NW + wv) * 64 + lane);
                            const uint2 c = s_cand[id];
                            bool low = false;
                            if (h) low = c.y < atomicMin(&D[c.x], c.y);
                            const uint4 e = make_uint4(c.x, CT && h ? crow[c.x] : kNoRow, c.y, kNoNode);
                            const unsigned long long bl = __ballot(low);
                            if (bl) {
                                reserve(0, __popcll(bl), p, q);
                                if (low) put_far(q + lanes_set_below(bl), e);
                            }
                        }
                        __threadfence();          // labels changed by atomics are not read from the L1
                    }
                };
                if constexpr (V == 2) {
                    if (rounds == 1) resolve(std::integral_constant<int, 1>{});
                    else if (rounds) resolve(std::integral_constant<int, 2>{});
                } else {
                    if (rounds == 1) resolve(std::integral_constant<int, 1>{});
                    else if (rounds == 2) resolve(std::integral_constant<int, 2>{});
                    else if (rounds == 3) resolve(std::integral_constant<int, 3>{});
                    else if (rounds) resolve(std::integral_constant<int, V>{});
                }
                __syncthreads();
                fold();
            }
            // the smallest far value
            if (tid == 0) s_fm = kInfBits;
            __syncthreads();
            {
                const float m = wave_min(lfm);
                if (lane == 0) atomicMin(&s_fm, __float_as_uint(m));
            }
            __syncthreads();
            const float fmin = __uint_as_float(s_fm);
            if (early) {
                bool pend = false;
                while (lcur < lend) {
                    const int l = lcur + tid;
                    bool p = false;
                    if (l < lend) {
                        if (CT) {
                            const uint2 an = net.anc[dem.leg_orig[l]];
                            p = !(__uint_as_float(D[an.x - node0]) < thr && __uint_as_float(D[an.y - node0]) < thr);
                        } else {
                            p = !(__uint_as_float(D[(uint32_t)dem.leg_orig[l] - node0]) < thr);
                        }
                    }
                    if (__syncthreads_or(p)) { pend = true; break; }
                    lcur += NT;
                }
                // no entry below thr is left: every label below it is final
                if (!pend && !(fmin < thr)) break;
            }
            if (fcnt == 0) break;
            thr = fmaxf(thr, fmin) + delta;
            if (!(thr > fmin)) thr = __uint_as_float(__float_as_uint(fmin) + 1u);
            bh = rh = 0;
            sweep_far(thr, false);
        }
        __syncthreads();
    }
    if (scr.stats) {
        for (int o = 32; o > 0; o >>= 1) n_relaxed += __shfl_xor(n_relaxed, o);
        if (tid == 0) atomicAdd(&scr.stats[0], n_taken);
        if (lane == 0) atomicAdd(&scr.stats[1], (unsigned long long)n_relaxed);
    }
}

template <int U, int V>
__global__ __launch_bounds__(kWG) void k_sssp_wn(NetDev net, DemDev dem, const uint2* __restrict__ radj,
                                                 label_t* labels, Scratch scr, const InstState* st,
                                                 const float* __restrict__ delta_inst, int early, int t_begin,
                                                 int t_end) {
    constexpr int NT = kWG;
    constexpr int NP = NT * U;                    // nodes per step
    __shared__ int s_rh[64], s_rc[64], s_rhp[64], s_tail[64], s_push[64], s_tpre[64];
    __shared__ int s_t, s_nn, s_fn;
    __shared__ uint32_t s_fm;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t* nearq = scr.nearq + (int64_t)blockIdx.x * scr.nmax;
    uint2* farq = reinterpret_cast<uint2*>(scr.farq) + (int64_t)blockIdx.x * scr.nmax;
    unsigned long long n_taken = 0, n_relaxed = 0;    // counted by every thread alike (uniform values)
    for (;;) {
        if (tid == 0) s_t = t_begin + atomicAdd(scr.work, 1);
        __syncthreads();
        const int t = s_t;
        __syncthreads();
        if (t >= t_end) break;
        const int inst = dem.dest_inst[t];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int n = I.n, node0 = I.node0;
        const int* __restrict__ rptr = net.rptr + node0;
        label_t* D = labels + dem.dest_lab[t];
        const int root = dem.dest_node[t] - node0;
        const float delta = delta_inst[inst];
        {
            uint4* D4 = reinterpret_cast<uint4*>(D);
            const uint32_t w0 = kNotQueued | kInfBits;
            const uint4 inf4 = make_uint4(w0, w0, w0, w0);
            const int n4 = (n + 31) / 32 * 8;
            for (int i = tid; i < n4; i += NT) D4[i] = inf4;
        }
        int rsh = 0;
        while (((n - 1) >> rsh) >= 64) ++rsh;
        const int rs = 1 << rsh;
        const int nranges = ((n - 1) >> rsh) + 1;
        if (tid < 64) {
            s_rh[tid] = 0;
            s_rc[tid] = (tid == (root >> rsh)) ? 1 : 0;
            s_push[tid] = 0;
        }
        if (tid == 0) {
            s_nn = 0;
            s_fn = 0;
            s_fm = kInfBits;
        }
        __threadfence_block();
        __syncthreads();
        if (tid == 0) {
            D[root] = 0u;                         // value 0, queued
            nearq[(root >> rsh) * (rs + 1)] = root;
        }
        __threadfence_block();
        __syncthreads();
        auto ring_at = [&](int r, int pos) -> int32_t* {
            const int cap = min(rs, n - r * rs) + 1;
            if (pos >= cap) pos -= cap;
            return nearq + (int64_t)r * (rs + 1) + pos;
        };
        auto push_near = [&](int v) {
            const int r = v >> rsh;
            *ring_at(r, s_tail[r] + atomicAdd(&s_push[r], 1)) = v;
            atomicAdd(&s_nn, 1);
        };
        // wavefront 0: tails of the rings for the pushes to come
        auto open_push = [&]() {
            if (wv == 0) {
                const int cap = lane < nranges ? min(rs, n - lane * rs) + 1 : 1;
                int tl = s_rh[lane] + s_rc[lane];
                if (tl >= cap) tl -= cap;
                s_tail[lane] = tl;
                s_push[lane] = 0;
            }
        };
        // after a pushing phase (all threads past a barrier): counts folded in
        int ncnt = 1, fcnt = 0;
        float thr = delta, fmin = __uint_as_float(kInfBits);
        auto fold = [&]() -> int {
            __threadfence_block();
            __syncthreads();
            const int nn = s_nn, fn = s_fn;
            const float fm = __uint_as_float(s_fm);
            __syncthreads();
            if (wv == 0) {
                if (lane < nranges) s_rc[lane] += s_push[lane];
                s_push[lane] = 0;
            }
            if (tid == 0) {
                s_nn = 0;
                s_fn = 0;
                s_fm = kInfBits;
            }
            ncnt += nn;
            fcnt += fn;
            fmin = fminf(fmin, fm);
            return nn;
        };
        int lcur = early ? dem.qptr[t] : 0;
        const int lend = early ? dem.qptr[t + 1] : 0;
        for (;;) {
            while (ncnt > 0) {
                const int k = ncnt < NP ? ncnt : NP;
                if (wv == 0) {
                    const int rc = s_rc[lane], rh = s_rh[lane];
                    int incl = rc;
                    for (int o = 1; o < 64; o <<= 1) {
                        const int x = __shfl_up(incl, o);
                        if (lane >= o) incl += x;
                    }
                    const int excl = incl - rc;
                    const int take = max(0, min(rc, NP - excl));
                    const int cap = lane < nranges ? min(rs, n - lane * rs) + 1 : 1;
                    s_tpre[lane] = min(excl, NP);
                    s_rhp[lane] = rh;
                    int nh = rh + take;
                    if (nh >= cap) nh -= cap;
                    s_rh[lane] = nh;
                    s_rc[lane] = rc - take;
                    int tl = nh + rc - take;
                    if (tl >= cap) tl -= cap;
                    s_tail[lane] = tl;
                    s_push[lane] = 0;
                }
                __syncthreads();
                // every thread takes up to U nodes and relaxes all their in-links
                // itself: in-degrees of road networks are small, so the owner
                // search and the degree prefix sum of k_sssp_ds are left out
                int wn_[U], e0_[U], e1_[U];
                float dw_[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = u * NT + tid;
                    wn_[u] = -1;
                    e0_[u] = e1_[u] = 0;
                    dw_[u] = 0.0f;
                    if (j < k) {
                        int lo = 0, hi = 64;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (s_tpre[mid] <= j) lo = mid; else hi = mid;
                        }
                        wn_[u] = *ring_at(lo, s_rhp[lo] + (j - s_tpre[lo]));
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (wn_[u] < 0) continue;
                    const uint32_t lw = atomicOr(&D[wn_[u]], kNotQueued);   // dequeue, read the label
                    e0_[u] = rptr[wn_[u]];
                    e1_[u] = rptr[wn_[u] + 1];
                    dw_[u] = __uint_as_float(lw & kValueBits);
                }
                ncnt -= k;
                n_taken += (unsigned)k;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    for (int e = e0_[u]; e < e1_[u]; e += V) {
                        int vv[V];
                        float cd[V];
                        bool ok[V];
#pragma unroll
                        for (int x = 0; x < V; ++x) {
                            ok[x] = e + x < e1_[u];
                            vv[x] = 0;
                            cd[x] = 0.0f;
                            if (ok[x]) {
                                const uint2 r = radj[e + x];
                                vv[x] = (int)r.x - node0;
                                cd[x] = dw_[u] + __uint_as_float(r.y);
                            }
                        }
                        uint32_t cur[V];
#pragma unroll
                        for (int x = 0; x < V; ++x) cur[x] = ok[x] ? (ld_coherent(&D[vv[x]]) & kValueBits) : 0u;
#pragma unroll
                        for (int x = 0; x < V; ++x) {
                            const uint32_t cb = __float_as_uint(cd[x]);
                            if (ok[x] && cb < cur[x] && (atomicMin(&D[vv[x]], cb) & kNotQueued)) {
                                if (cd[x] < thr) {
                                    push_near(vv[x]);
                                } else {
                                    farq[fcnt + atomicAdd(&s_fn, 1)] = make_uint2((uint32_t)vv[x], cb);
                                    atomicMin(&s_fm, cb);
                                }
                            }
                        }
                    }
                    n_relaxed += (unsigned)(e1_[u] - e0_[u]);
                }
                fold();
            }
            if (early) {
                bool pend = false;
                while (lcur < lend) {
                    const int l = lcur + tid;
                    bool p = false;
                    if (l < lend) {
                        const int o = dem.leg_orig[l] - node0;
                        p = !(__uint_as_float(ld_coherent(&D[o]) & kValueBits) < thr);
                    }
                    if (__syncthreads_or(p)) { pend = true; break; }
                    lcur += NT;
                }
                if (!pend) {
                    // exact: queue the far nodes whose current label is below thr
                    int moved = 0, keep = 0;
                    float km = __uint_as_float(kInfBits);
                    open_push();
                    __syncthreads();
                    for (int i0 = 0; i0 < fcnt; i0 += NT) {
                        const int i = i0 + tid;
                        const bool h = i < fcnt;
                        uint2 ent = h ? farq[i] : make_uint2(0u, kInfBits);
                        if (h) ent.y = ld_coherent(&D[ent.x]) & kValueBits;   // the label now
                        const bool late = h && __uint_as_float(ent.y) < thr;
                        __syncthreads();                  // the chunk is read before it is overwritten
                        if (late) {
                            push_near((int)ent.x);
                        } else if (h) {
                            farq[keep + atomicAdd(&s_fn, 1)] = ent;
                            atomicMin(&s_fm, ent.y);
                        }
                        __threadfence_block();
                        __syncthreads();
                        const int nn = s_nn, fn = s_fn;
                        const float fm = __uint_as_float(s_fm);
                        __syncthreads();
                        if (tid == 0) {
                            s_nn = 0;
                            s_fn = 0;
                            s_fm = kInfBits;
                        }
                        ncnt += nn;
                        moved += nn;
                        keep += fn;
                        km = fminf(km, fm);
                    }
                    if (wv == 0) {
                        if (lane < nranges) s_rc[lane] += s_push[lane];
                        s_push[lane] = 0;
                    }
                    __syncthreads();
                    fcnt = keep;
                    fmin = km;
                    if (moved == 0) break;                // every label below thr is final
                    continue;
                }
            }
            if (fcnt == 0) break;
            thr = fmaxf(thr, fmin) + delta;
            if (!(thr > fmin)) thr = __uint_as_float(__float_as_uint(fmin) + 1u);
            int keep = 0;
            float km = __uint_as_float(kInfBits);
            open_push();
            __syncthreads();
            for (int i0 = 0; i0 < fcnt; i0 += NT) {
                const int i = i0 + tid;
                const bool h = i < fcnt;
                uint2 ent = h ? farq[i] : make_uint2(0u, kInfBits);
                // key by the label now: a far node improved since its push keeps
                // its queued flag and is not pushed again, and waiting for the
                // threshold to pass its old label would make every node it
                // reaches meanwhile be popped again
                if (h) ent.y = ld_coherent(&D[ent.x]) & kValueBits;
                __syncthreads();
                if (h && __uint_as_float(ent.y) < thr) {
                    push_near((int)ent.x);
                } else if (h) {
                    farq[keep + atomicAdd(&s_fn, 1)] = ent;
                    atomicMin(&s_fm, ent.y);
                }
                __threadfence_block();
                __syncthreads();
                const int nn = s_nn, fn = s_fn;
                const float fm = __uint_as_float(s_fm);
                __syncthreads();
                if (tid == 0) {
                    s_nn = 0;
                    s_fn = 0;
                    s_fm = kInfBits;
                }
                ncnt += nn;
                keep += fn;
                km = fminf(km, fm);
            }
            if (wv == 0) {
                if (lane < nranges) s_rc[lane] += s_push[lane];
                s_push[lane] = 0;
            }
            __syncthreads();
            fcnt = keep;
            fmin = km;
        }
        __syncthreads();
    }
    if (scr.stats) {
        for (int o = 32; o > 0; o >>= 1) n_relaxed += __shfl_xor(n_relaxed, o);
        if (tid == 0) atomicAdd(&scr.stats[0], n_taken);
        if (lane == 0) atomicAdd(&scr.stats[1], n_relaxed);
    }
}

// Block-local form of the same delta-stepping.  The node ids of an instance
// are cut into blocks of B consecutive ids (in Hilbert order a block is a
// compact patch of the network).  The near queue holds blocks, not nodes: a
// block is queued (once: a bit per block in LDS) while it holds a queued node
// whose label is below the bucket bound thr.  A step takes up to NW * KB
// blocks off the queue; each wavefront, for each of its blocks,
//   - loads the block's label words and in-link offsets (coalesced) and its
//     in-link records into LDS;
//   - relaxes inside the block to closure: every queued node below thr is
//     taken (flag set with an LDS atomicOr that returns its label) and its
//     in-links relaxed, those from inside the block by an LDS atomicMin on the
//     staged word, those from other blocks into a mailbox; repeated until no
//     queued node below thr is left -- many hops for one load of the block;
//   - writes the changed words back; a node first queued in this visit at or
//     above thr goes to the far queue.
// Then the whole workgroup applies the mailboxes to the labels in memory (a
// coherent read, then an atomicMin where the candidate is lower), queueing the
// block of every node it improves below thr and sending to the far queue the
// nodes it queues at or above thr.  Only one workgroup touches a tree, and
// the two phases are separated by barriers, so the words a phase-1 wavefront
// stages are not changed under it.  Whatever the order, the labels reach the
// least fixed point of D(v) = min_e fl32(D(head e) + c_e), as in k_sssp_wg.
//   A node is sent to the far queue at most once per tree: it is queued at or
// above thr only before it is first taken (afterwards its label stays below
// the thr of that moment), so the far queue holds at most n entries.
// B: nodes per block (a multiple of 64); KB: blocks per wavefront per step.
// kBlkMaxBits (qdta_internal.h): blocks per tree the LDS bitmap covers.
template <int B, int KB>
__global__ __launch_bounds__(kWG) void k_sssp_blk(NetDev net, DemDev dem, const uint2* __restrict__ radj,
                                                  label_t* labels, Scratch scr, const InstState* st,
                                                  const float* __restrict__ delta_inst, int early, int t_begin,
                                                  int t_end) {
    constexpr int NT = kWG;
    constexpr int NW = NT / 64;
    constexpr int R = B / 64;                   // nodes per lane in a block
    constexpr int KMAX = NW * KB;               // blocks per step
    constexpr int kBlkEmax = 3 * B;             // in-link records staged per block (the rest are read in place)
    constexpr int kBlkMbx = 2 * B;              // mailbox entries (target, candidate) per wavefront and step
    constexpr int kBig = 8;                     // per wavefront and step: nodes whose cross-block in-links
                                                // are too many for the mailbox, relaxed in phase 2 by all threads
    __shared__ uint32_t s_bits[kBlkMaxBits / 32];
    __shared__ uint32_t s_lab[NW][B];
    __shared__ int s_rp[NW][B + 1];
    __shared__ uint2 s_adj[NW][kBlkEmax];
    // one mailbox and one big-node list per (wavefront, block of the step), so
    // every block visit starts with room for any one node: each visit takes
    // at least one node
    __shared__ uint2 s_mb[NW * KB][kBlkMbx];
    __shared__ int s_mc[NW * KB];
    __shared__ uint2 s_big[NW * KB][kBig];
    __shared__ int s_nbig[NW * KB];
    __shared__ int s_blk[KMAX];
    __shared__ int s_t, s_qh, s_qn, s_qt, s_fn;
    __shared__ uint32_t s_fm;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const unsigned long long below = lanes_below(lane);
    int32_t* ring = scr.nearq + (int64_t)blockIdx.x * scr.nmax;
    uint2* farq = reinterpret_cast<uint2*>(scr.farq) + (int64_t)blockIdx.x * scr.nmax;
    uint32_t* L = s_lab[wv];
    int* RP = s_rp[wv];
    uint2* A = s_adj[wv];
    unsigned long long n_taken = 0, n_relaxed = 0;    // this lane's work, for the counters
    for (;;) {
        if (tid == 0) s_t = t_begin + atomicAdd(scr.work, 1);
        __syncthreads();
        const int t = s_t;
        __syncthreads();
        if (t >= t_end) break;
        const int inst = dem.dest_inst[t];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int n = I.n, node0 = I.node0;
        const int* __restrict__ rptr = net.rptr + node0;
        label_t* D = labels + dem.dest_lab[t];
        const int root = dem.dest_node[t] - node0;
        const float delta = delta_inst[inst];
        const int nb = (n + B - 1) / B;
        const int qcap = nb + 1;                // ring of block ids; at most nb are queued
        {
            uint4* D4 = reinterpret_cast<uint4*>(D);
            const uint32_t w0 = kNotQueued | kInfBits;
            const uint4 inf4 = make_uint4(w0, w0, w0, w0);
            const int n4 = (n + 31) / 32 * 8;
            for (int i = tid; i < n4; i += NT) D4[i] = inf4;
        }
        for (int i = tid; i < (nb + 31) / 32; i += NT) s_bits[i] = 0u;
        if (tid == 0) {
            s_qh = 0;
            s_qn = 0;
            s_qt = 0;
            s_fn = 0;
            s_fm = kInfBits;
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            D[root] = 0u;                       // value 0, queued
            const int b = root / B;
            s_bits[b >> 5] |= 1u << (b & 31);
            ring[0] = b;
            s_qt = 1;
            s_qn = 1;
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // queue block b unless it is queued (LDS bit); safe from any thread
        auto push_block = [&](int b) {
            const uint32_t bit = 1u << (b & 31);
            if (atomicOr(&s_bits[b >> 5], bit) & bit) return;
            int pos = atomicAdd(&s_qt, 1);
            pos = pos % qcap;
            ring[pos] = b;
            atomicAdd(&s_qn, 1);
        };
        float thr = delta;
        int fcnt = 0;
        float fmin = __uint_as_float(kInfBits);
        int lcur = early ? dem.qptr[t] : 0;
        const int lend = early ? dem.qptr[t + 1] : 0;
        for (;;) {
            for (;;) {
                const int qn = s_qn;
                if (qn == 0) break;
                const int k = qn < KMAX ? qn : KMAX;
                const int qh = s_qh;
                __syncthreads();                // every thread has read the counters
                if (tid < k) {
                    const int b = ring[(qh + tid) % qcap];
                    s_blk[tid] = b;
                    atomicAnd(&s_bits[b >> 5], ~(1u << (b & 31)));
                }
                if (tid == 0) {
                    s_qh = (qh + k) % qcap;
                    s_qn = qn - k;
                }
                if (tid < KMAX) {
                    s_mc[tid] = 0;
                    s_nbig[tid] = 0;
                }
                __syncthreads();
                // ---- phase 1: each wavefront relaxes its blocks to closure
                for (int kb = 0; kb < KB; ++kb) {
                    const int j = kb * NW + wv;
                    if (j >= k) break;
                    const int b = s_blk[j];
                    uint2* MB = s_mb[j];
                    uint2* BG = s_big[j];
                    int mcnt = 0, nbig = 0;
                    const int v0 = b * B;
                    const int nv = min(B, n - v0);
                    uint32_t w0[R];
                    bool q0[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int i = lane + 64 * r;
                        w0[r] = i < nv ? ld_coherent(&D[v0 + i]) : (kNotQueued | kInfBits);
                        q0[r] = !(w0[r] & kNotQueued);
                        L[i] = w0[r];
                        RP[i] = i < nv ? rptr[v0 + i] : 0;
                    }
                    if (lane == 0) RP[nv] = rptr[v0 + nv];
                    __builtin_amdgcn_wave_barrier();
                    const int e_lo = RP[0];
                    const int E = RP[nv] - e_lo;
                    for (int x = lane; x < E && x < kBlkEmax; x += 64) A[x] = radj[e_lo + x];
                    __builtin_amdgcn_wave_barrier();
                    bool skipped = false;
                    for (;;) {
                        bool act[R];
                        int cc[R];
                        bool any = false;
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const int i = lane + 64 * r;
                            const uint32_t w = i < nv ? L[i] : kNotQueued;
                            act[r] = !(w & kNotQueued) && __uint_as_float(w) < thr;
                            cc[r] = 0;
                            if (act[r]) {
                                any = true;
                                for (int e = RP[i]; e < RP[i + 1]; ++e) {
                                    const int x = e - e_lo;
                                    const uint32_t src = x < kBlkEmax ? A[x].x : radj[e].x;
                                    if ((unsigned)((int)src - node0 - v0) >= (unsigned)nv) ++cc[r];
                                }
                            }
                        }
                        if (__ballot(any) == 0ull) break;
                        // mailbox room: nodes in (r, lane) order take their cross-block
                        // in-links while they fit; the rest stay queued for a later visit.
                        // A node with more than half a mailbox of them ("big") takes one
                        // of kBig slots instead and is relaxed in phase 2.
                        bool big[R];
                        int excl[R], bex[R];
                        int base = 0, bbase = 0;
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            big[r] = act[r] && cc[r] > kBlkMbx / 2;
                            const int c1 = big[r] ? 0 : cc[r];
                            int incl = c1;
                            for (int o = 1; o < 64; o <<= 1) {
                                const int y = __shfl_up(incl, o);
                                if (lane >= o) incl += y;
                            }
                            excl[r] = base + incl - c1;
                            base += __shfl(incl, 63);
                            const unsigned long long bb = __ballot(big[r]);
                            bex[r] = bbase + __popcll(bb & below);
                            bbase += __popcll(bb);
                        }
                        bool fit[R];
                        bool anyfit = false, anyskip = false;
                        int used = 0, bused = 0;
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            fit[r] = act[r] && (big[r] ? nbig + bex[r] < kBig : mcnt + excl[r] + cc[r] <= kBlkMbx);
                            anyfit |= fit[r];
                            anyskip |= act[r] && !fit[r];
                            if (fit[r] && !big[r]) used = max(used, excl[r] + cc[r]);
                            if (fit[r] && big[r]) bused = max(bused, bex[r] + 1);
                        }
                        for (int o = 32; o > 0; o >>= 1) {
                            used = max(used, __shfl_xor(used, o));
                            bused = max(bused, __shfl_xor(bused, o));
                        }
                        if (__ballot(anyskip) != 0ull) skipped = true;
                        if (__ballot(anyfit) == 0ull) break;
                        float du[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            du[r] = 0.0f;
                            if (fit[r]) {
                                const int i = lane + 64 * r;
                                du[r] = __uint_as_float(atomicOr(&L[i], kNotQueued) & kValueBits);
                                n_taken += 1;
                                n_relaxed += (unsigned)(RP[i + 1] - RP[i]);
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            if (!fit[r]) continue;
                            const int i = lane + 64 * r;
                            if (big[r]) BG[nbig + bex[r]] = make_uint2((uint32_t)(v0 + i), __float_as_uint(du[r]));
                            int slot = mcnt + excl[r];
                            for (int e = RP[i]; e < RP[i + 1]; ++e) {
                                const int x = e - e_lo;
                                const uint2 rec = x < kBlkEmax ? A[x] : radj[e];
                                const int sv = (int)rec.x - node0;
                                const float cd = du[r] + __uint_as_float(rec.y);
                                const uint32_t cb = __float_as_uint(cd);
                                const int jj = sv - v0;
                                if ((unsigned)jj < (unsigned)nv) {
                                    if (cb < (L[jj] & kValueBits)) atomicMin(&L[jj], cb);
                                } else if (!big[r]) {
                                    MB[slot++] = make_uint2((uint32_t)sv, cb);
                                }
                            }
                        }
                        mcnt += used;
                        nbig += bused;
                        __builtin_amdgcn_wave_barrier();
                    }
                    // write the changed words back; a node first queued in this visit
                    // at or above thr goes to the far queue
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int i = lane + 64 * r;
                        const uint32_t w = i < nv ? L[i] : w0[r];
                        if (w != w0[r]) D[v0 + i] = w;
                        const bool far = i < nv && !(w & kNotQueued) && !(__uint_as_float(w) < thr);
                        const bool tofar = far && !q0[r];
                        if (far && w != w0[r]) atomicMin(&s_fm, w);
                        const unsigned long long bf = __ballot(tofar);
                        if (bf) {
                            int fb = 0;
                            if (lane == 0) fb = atomicAdd(&s_fn, __popcll(bf));
                            fb = __shfl(fb, 0);
                            if (tofar) farq[fcnt + fb + __popcll(bf & below)] = make_uint2((uint32_t)(v0 + i), w);
                        }
                    }
                    if (skipped && lane == 0) push_block(b);
                    if (lane == 0) {
                        s_mc[j] = mcnt;
                        s_nbig[j] = nbig;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                // ---- phase 2: the mailboxes into the labels in memory
                auto apply = [&](int sv, uint32_t cb) {
                    const uint32_t cur = ld_coherent(&D[sv]);
                    if (cb < (cur & kValueBits)) {
                        const uint32_t old = atomicMin(&D[sv], cb);
                        const bool below_thr = __uint_as_float(cb) < thr;
                        if (old & kNotQueued) {
                            // this relaxation queued the node
                            if (below_thr) {
                                push_block(sv / B);
                            } else {
                                const int fp = atomicAdd(&s_fn, 1);
                                farq[fcnt + fp] = make_uint2((uint32_t)sv, cb);
                                atomicMin(&s_fm, cb);
                            }
                        } else if (!(__uint_as_float(old & kValueBits) < thr)) {
                            if (below_thr) push_block(sv / B);   // a far node now below thr
                            else atomicMin(&s_fm, cb);           // a far node improved
                        }
                    }
                };
                int mtot = 0, moff[KMAX];
#pragma unroll
                for (int w = 0; w < KMAX; ++w) {
                    moff[w] = mtot;
                    mtot += s_mc[w];
                }
                for (int g = tid; g < mtot; g += NT) {
                    int w = 0;
#pragma unroll
                    for (int x = 1; x < KMAX; ++x)
                        if (g >= moff[x]) w = x;
                    const uint2 m = s_mb[w][g - moff[w]];
                    apply((int)m.x, m.y);
                }
                // the big nodes' cross-block in-links, spread over the workgroup
                for (int w = 0; w < KMAX; ++w) {
                    for (int x = 0; x < s_nbig[w]; ++x) {
                        const uint2 bg = s_big[w][x];
                        const int u = (int)bg.x, ub = u / B;
                        const float du = __uint_as_float(bg.y);
                        for (int e = rptr[u] + tid; e < rptr[u + 1]; e += NT) {
                            const uint2 rec = radj[e];
                            const int sv = (int)rec.x - node0;
                            if (sv / B != ub) apply(sv, __float_as_uint(du + __uint_as_float(rec.y)));
                        }
                    }
                }
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                fcnt += s_fn;
                fmin = fminf(fmin, __uint_as_float(s_fm));
                __syncthreads();
                if (tid == 0) {
                    s_fn = 0;
                    s_fm = kInfBits;
                }
                __syncthreads();
            }
            // bucket [.., thr) drained: every label below thr is final
            if (early) {
                bool pend = false;
                while (lcur < lend) {
                    const int l = lcur + tid;
                    bool p = false;
                    if (l < lend) {
                        const int o = dem.leg_orig[l] - node0;
                        p = !(__uint_as_float(ld_coherent(&D[o]) & kValueBits) < thr);
                    }
                    if (__syncthreads_or(p)) { pend = true; break; }
                    lcur += NT;
                }
                if (!pend) break;               // every origin is settled
            }
            if (fcnt == 0) break;
            thr = fmaxf(thr, fmin) + delta;
            if (!(thr > fmin)) thr = __uint_as_float(__float_as_uint(fmin) + 1u);
            // move the far nodes below thr (keyed by their labels now) to the
            // near queue; drop those taken since (flag set)
            int keep = 0;
            float km = __uint_as_float(kInfBits);
            for (int i0 = 0; i0 < fcnt; i0 += NT) {
                const int i = i0 + tid;
                const bool h = i < fcnt;
                uint2 ent = h ? farq[i] : make_uint2(0u, kInfBits);
                uint32_t cur = h ? ld_coherent(&D[ent.x]) : kNotQueued;
                __syncthreads();                // the chunk is read before it is overwritten
                const bool live = h && !(cur & kNotQueued);
                ent.y = cur & kValueBits;
                if (live && __uint_as_float(ent.y) < thr) {
                    push_block((int)ent.x / B);
                } else if (live) {
                    farq[keep + atomicAdd(&s_fn, 1)] = ent;
                    atomicMin(&s_fm, ent.y);
                }
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                const int fn = s_fn;
                const float fm = __uint_as_float(s_fm);
                __syncthreads();
                if (tid == 0) {
                    s_fn = 0;
                    s_fm = kInfBits;
                }
                keep += fn;
                km = fminf(km, fm);
            }
            __syncthreads();
            fcnt = keep;
            fmin = km;
        }
        __syncthreads();
    }
    if (scr.stats) {
        for (int o = 32; o > 0; o >>= 1) {
            n_taken += __shfl_xor(n_taken, o);
            n_relaxed += __shfl_xor(n_relaxed, o);
        }
        if (lane == 0) {
            atomicAdd(&scr.stats[0], n_taken);
            atomicAdd(&scr.stats[1], n_relaxed);
        }
    }
}

// What a launch of the search needs in place: the bucket width per instance,
// delta = scale * (geometric mean link cost of the instance), from the log sums
// the cost kernels leave per workgroup (added in a fixed order), the tree
// counter, and, where given, y and the tie flags at zero.  The geometric mean
// follows the typical link; the arithmetic mean is dominated by the few links
// that congestion makes very slow.
__global__ __launch_bounds__(kWG) void k_prep(NetDev net, const double* __restrict__ logpart, double scale,
                                              float* delta_inst, int32_t* work, int64_t* __restrict__ y,
                                              int32_t* __restrict__ absorb_q, int Q) {
    __shared__ double part[kWG];
    if (blockIdx.x == 0 && threadIdx.x == 0) *work = 0;
    const int64_t first = blockIdx.x * (int64_t)kWG + threadIdx.x, stride = (int64_t)gridDim.x * kWG;
    if (y)
        for (int64_t a = first; a < net.M; a += stride) y[a] = 0;
    if (absorb_q)
        for (int64_t q = first; q < Q; q += stride) absorb_q[q] = 0;
    for (int inst = blockIdx.x; inst < net.ninst; inst += gridDim.x) {
        const InstDev I = net.inst[inst];
        // the instance's workgroups are a run: its first chunk is the one at link0
        const int n = (I.m + kChunk - 1) / kChunk * kLogParts;
        double s = 0.0;
        for (int k = threadIdx.x; k < n; k += kWG) s += logpart[(int64_t)net.inst_blk[inst] * kLogParts + k];
        part[threadIdx.x] = s;
        __syncthreads();
        for (int k = kWG / 2; k > 0; k >>= 1) {
            if ((int)threadIdx.x < k) part[threadIdx.x] += part[threadIdx.x + k];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            double d = I.m > 0 ? scale * exp(part[0] / (double)I.m) : 1.0;
            if (!(d > 0.0) || !(d < 3.0e38)) d = 3.0e38;
            delta_inst[inst] = (float)d;
        }
        __syncthreads();
    }
}

hipError_t launch_prep(hipStream_t s, const NetDev& net, const double* logpart, double delta_scale, float* delta_inst,
                       int32_t* work, int64_t* y, int32_t* absorb_q, int Q) {
    const int64_t words = std::max<int64_t>(y ? net.M : 1, absorb_q ? Q : 1);
    const int64_t g = std::max<int64_t>((words + 4 * kWG - 1) / (4 * kWG), std::min(net.ninst, 1024));
    hipLaunchKernelGGL(k_prep, dim3((unsigned)std::min<int64_t>(g, 2048)), dim3(kWG), 0, s, net, logpart, delta_scale,
                       delta_inst, work, y, absorb_q, Q);
    return hipGetLastError();
}

// Labels of the chain nodes left out of the contracted search, from their
// chains' ends: for chain node x_j, the FP32 fold from v through x_k..x_j
// and the fold from u through x_1..x_j (each over links that exist: a
// missing link's +inf cost stops the fold), and the lesser of the two.
// Turning back inside a chain never beats this, since each addition of a
// non-negative cost keeps or raises a value.  Work item (r, t): chunk r of
// kFillChunk chains of tree t's instance, kFillPer per thread with their
// header and end-label loads in flight together; items run chunk by chunk,
// so the trees in flight share the chunk's headers and blocks in the cache.
constexpr int kFillPer = kFillChunk / kWG;
__global__ __launch_bounds__(kWG) void k_chain_fill(NetDev net, DemDev dem, label_t* labels, const InstState* st,
                                                    int t_begin, int t_end) {
    const int64_t nq = t_end - t_begin;
    const int64_t items = (int64_t)net.fill_chunks * nq;
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int r = (int)(it / nq);
        const int t = t_begin + (int)(it - (int64_t)r * nq);
        const int inst = dem.dest_inst[t];
        if (!inst_live(st, inst)) continue;
        const int cb = net.inst_chain[inst] + r * kFillChunk;
        const int ce = min(net.inst_chain[inst + 1], cb + kFillChunk);
        if (cb >= ce) continue;
        label_t* D = labels + dem.dest_lab[t];
        const int node0 = net.inst[inst].node0;
        // loads with in-range indices whether or not the slot has a chain, so
        // that none of them waits on a branch
        int4 h[kFillPer];
        bool ok[kFillPer];
#pragma unroll
        for (int q = 0; q < kFillPer; ++q) {
            const int ch = cb + q * kWG + (int)threadIdx.x;
            ok[q] = ch < ce;
            h[q] = net.ch_hdr[min(ch, ce - 1)];
        }
        uint32_t wu[kFillPer], wv[kFillPer];
#pragma unroll
        for (int q = 0; q < kFillPer; ++q) {
            wu[q] = D[h[q].x - node0];
            wv[q] = D[h[q].y - node0];
        }
#pragma unroll
        for (int q = 0; q < kFillPer; ++q) {
            const float du = __uint_as_float(wu[q] & kValueBits), dv = __uint_as_float(wv[q] & kValueBits);
            if (!ok[q] || (!(du < __uint_as_float(kInfBits)) && !(dv < __uint_as_float(kInfBits)))) continue;
            const uint32_t* blk = net.cbuf + h[q].w;
            const int k = h[q].z;
            float lv[kChainMax];
            float l = du;
#pragma unroll
            for (int j = 0; j < kChainMax; ++j) {
                if (j < k) {
                    l = l + __uint_as_float(blk[3 * j + 2]);
                    lv[j] = l;
                }
            }
            float rv = dv;
#pragma unroll
            for (int j = kChainMax - 1; j >= 0; --j) {
                if (j < k) {
                    rv = rv + __uint_as_float(blk[3 * j + 1]);
                    D[(int)blk[3 * j] - node0] = kNotQueued | __float_as_uint(fminf(lv[j], rv));
                }
            }
        }
    }
}

hipError_t launch_chain_fill(hipStream_t s, const NetDev& net, const DemDev& dem, label_t* labels,
                             const InstState* st, int t_begin, int t_end) {
    const int64_t items = (int64_t)net.fill_chunks * (t_end - t_begin);
    if (items <= 0 || !net.cbuf) return hipSuccess;
    hipLaunchKernelGGL(k_chain_fill, dim3((unsigned)std::min<int64_t>(items, 4096)), dim3(kWG), 0, s, net, dem, labels,
                       st, t_begin, t_end);
    return hipGetLastError();
}

// Trees of small networks: the labels of a tree in LDS, every thread the keeper
// of P nodes, whose first four out-links it holds in registers (further ones are
// read again by each pass).  A pass lowers each of a thread's nodes to the least
// of fl32(D(head) + c) over its out-links; passes run without barriers -- labels
// only fall, each is written by its keeper alone, and any order of such steps
// ends at the same least fixed point -- and every kPullPasses of them the
// workgroup asks whether any label fell.  If none did, every pass since the last
// question read the final labels.  Labels are compared by their bits, as the
// queues do: a sum below zero (or NaN) lies above all others and is not taken.
// Between two questions every label is lowered along one more link at least, so
// n of them are enough where no cycle of costs is negative; no input takes more.
// Bound by the passes' LDS reads, about as many passes as the longest shortest
// path has links, so for small n only (pull_trees); no queue and no chain of
// memory accesses in a step.  Whole call, 40 trees of a congested 400-node grid:
// 56 us, 107 with k_sssp_wg; 1,200 of 2,025 nodes: 266 and 340.
constexpr int kPullPasses = 4;

template <int NT, int P>
__global__ __launch_bounds__(NT) void k_sssp_pull(NetDev net, DemDev dem, label_t* labels, Scratch scr,
                                                  const InstState* st, int t_begin) {
    __shared__ float s_lab[NT * P];
    const int t = t_begin + (int)blockIdx.x, tid = threadIdx.x;
    const int inst = dem.dest_inst[t];
    if (!inst_live(st, inst)) return;
    const InstDev I = net.inst[inst];
    const int n = I.n, node0 = I.node0, root = dem.dest_node[t] - node0;
    const float inf = __uint_as_float(kInfBits);
    label_t* D = labels + dem.dest_lab[t];
    volatile float* lab = s_lab;
    float mine[P], c[P][4];
    int head[P][4], e0[P], deg[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int v = tid + p * NT;
        e0[p] = v < n ? net.row_ptr[node0 + v] : 0;
        deg[p] = v < n ? net.row_ptr[node0 + v + 1] - e0[p] : 0;
        mine[p] = v == root ? 0.0f : inf;
        lab[v] = mine[p];
    }
    bool more = false;
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = j < deg[p];
            const uint2 r = in ? net.fadj[e0[p] + j] : make_uint2((uint32_t)node0, kInfBits);
            head[p][j] = (int)r.x - node0;
            c[p][j] = __uint_as_float(r.y);
        }
        more |= deg[p] > 4;
    }
    const bool longer = __ballot(more) != 0ull;
    int passes = 0;
    bool fell;
    int asked = 0;
    __syncthreads();
    do {
        fell = false;
        for (int k = 0; k < kPullPasses; ++k) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                float d[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = lab[head[p][j]];
                uint32_t low = min(min(__float_as_uint(d[0] + c[p][0]), __float_as_uint(d[1] + c[p][1])),
                                   min(__float_as_uint(d[2] + c[p][2]), __float_as_uint(d[3] + c[p][3])));
                if (longer)
                    for (int e = 4; e < deg[p]; ++e) {
                        const uint2 r = net.fadj[e0[p] + e];
                        low = min(low, __float_as_uint(lab[(int)r.x - node0] + __uint_as_float(r.y)));
                    }
                if (low < __float_as_uint(mine[p])) {
                    mine[p] = __uint_as_float(low);
                    lab[tid + p * NT] = mine[p];
                    fell = true;
                }
            }
        }
        passes += kPullPasses;
    } while (__syncthreads_or(fell) && ++asked < n);
    const int top = (n + 31) / 32 * 32;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int v = tid + p * NT;
        if (v < top) D[v] = kNotQueued | __float_as_uint(mine[p]);
    }
    if (scr.stats && tid == 0) {
        atomicAdd(&scr.stats[0], (unsigned long long)passes * (unsigned)n);
        atomicAdd(&scr.stats[1], (unsigned long long)passes * (unsigned)I.m);
    }
}

hipError_t launch_trees(hipStream_t s, const NetDev& net, const DemDev& dem, const uint2* radj, label_t* labels,
                        const Scratch& scr, int slots, const InstState* st, const float* delta_inst, int variant,
                        int early, int t_begin, int t_end, bool fill) {
    if (t_end <= t_begin) return hipSuccess;
    hipError_t e = hipSuccess;
    if (variant >= kPullVariant) {
        // a workgroup per tree, by the nodes of the largest instance
#define QDTA_SSSP_PULL(NT, P) \
    hipLaunchKernelGGL((k_sssp_pull<NT, P>), dim3(t_end - t_begin), dim3(NT), 0, s, net, dem, labels, scr, st, t_begin)
        switch (variant - kPullVariant) {
            case 0: QDTA_SSSP_PULL(256, 1); break;
            case 1: QDTA_SSSP_PULL(512, 1); break;
            case 2: QDTA_SSSP_PULL(1024, 1); break;
            case 3: QDTA_SSSP_PULL(1024, 2); break;
            default: QDTA_SSSP_PULL(1024, 4); break;
        }
#undef QDTA_SSSP_PULL
        return hipGetLastError();
    }
    int blocks = (slots + (kWG / 64) - 1) / (kWG / 64);
    if (variant >= 32 || (variant >= 8 && variant < 16)) {
        // node queue, one workgroup of 128 U threads per tree (scratch slot =
        // workgroup), V lanes per entry.  256 threads and 4 lanes where no other
        // shape is asked for: a step's entries are 100 to 250 on road networks and
        // grids, so 128 threads take twice the steps, 512 keep half as many trees in
        // flight, and two lanes leave most rows to a second step.  Metro network,
        // 1,000 trees, <2, 4> / <4, 4> / <1, 4> / <2, 2>, ms: 2.4 / 2.8 / 2.7 / 3.3;
        // 22,801-node grid, 300 trees, congested: 0.80 / 1.36 / 1.20 / 1.55 (with a
        // thread per entry).  With a CU for every tree, 512 threads share out a
        // step's rounds further (auto_shape).
        const bool ct = variant >= 32;
        if (ct && !net.cbuf) return hipErrorInvalidValue;
        static const int units[] = {1, 1, 2, 4, 2, 4};
        const int v = min(variant - (ct ? 32 : 8), 5), nt = 128 * units[v];
        // where every tree can have a CU it has its own workgroup
        blocks = max((slots * 64 + nt - 1) / nt, min(t_end - t_begin, scr.cus));
        blocks = min(blocks, min(scr.near_w, scr.far_w) / 4);
        if (blocks <= 0) return hipErrorInvalidValue;
#define QDTA_SSSP_WG(...)                                                                                          \
    hipLaunchKernelGGL((k_sssp_wg<__VA_ARGS__>), dim3(blocks), dim3(nt), 0, s, net, dem, radj, labels, scr, st,     \
                       delta_inst, early, t_begin, t_end)
        switch (2 * v + ct) {
            case 0: QDTA_SSSP_WG(1, 2, false); break;
            case 1: QDTA_SSSP_WG(1, 2, true); break;
            case 2: QDTA_SSSP_WG(1, 4, false); break;
            case 3: QDTA_SSSP_WG(1, 4, true); break;
            case 4: QDTA_SSSP_WG(2, 4, false); break;
            case 5: QDTA_SSSP_WG(2, 4, true, 7); break;
            case 6: QDTA_SSSP_WG(4, 4, false); break;
            case 7: QDTA_SSSP_WG(4, 4, true); break;
            case 8: QDTA_SSSP_WG(2, 2, false); break;
            case 9: QDTA_SSSP_WG(2, 2, true); break;
            case 10: QDTA_SSSP_WG(4, 2, false); break;
            default: QDTA_SSSP_WG(4, 2, true); break;
        }
#undef QDTA_SSSP_WG
        e = hipGetLastError();
        if (e != hipSuccess || !ct || !fill) return e;
        return launch_chain_fill(s, net, dem, labels, st, t_begin, t_end);   // the left-out chain nodes
    }
    if (variant >= 24) {
        // one workgroup per tree, every thread relaxing its own nodes' in-links
        blocks = min(blocks, min(scr.near_w, scr.far_w / 2));
        if (blocks <= 0) return hipErrorInvalidValue;
        dim3 g(blocks), b(kWG);
#define QDTA_SSSP_WN(U, V) \
    hipLaunchKernelGGL((k_sssp_wn<U, V>), g, b, 0, s, net, dem, radj, labels, scr, st, delta_inst, early, t_begin, \
                       t_end)
        switch (variant - 24) {
            case 0: QDTA_SSSP_WN(1, 4); break;
            case 1: QDTA_SSSP_WN(2, 4); break;
            case 2: QDTA_SSSP_WN(2, 2); break;
            default: QDTA_SSSP_WN(1, 2); break;
        }
#undef QDTA_SSSP_WN
        return hipGetLastError();
    }
    if (variant >= 16) {
        // block-local trees, one workgroup per tree (scratch slot = workgroup)
        blocks = min(blocks, min(scr.near_w, scr.far_w / 2));
        if (blocks <= 0) return hipErrorInvalidValue;
        dim3 g(blocks), b(kWG);
#define QDTA_SSSP_BLK(B, KB) \
    hipLaunchKernelGGL((k_sssp_blk<B, KB>), g, b, 0, s, net, dem, radj, labels, scr, st, delta_inst, early, t_begin, \
                       t_end)
        switch (variant - 16) {
            case 0: QDTA_SSSP_BLK(128, 1); break;
            case 1: QDTA_SSSP_BLK(128, 2); break;
            case 2: QDTA_SSSP_BLK(64, 2); break;
            default: QDTA_SSSP_BLK(256, 1); break;
        }
#undef QDTA_SSSP_BLK
        return hipGetLastError();
    }
    // one wavefront per tree (scratch slot = wavefront)
    blocks = min(blocks, min(scr.near_w, scr.far_w / 2) / (kWG / 64));
    if (blocks <= 0) return hipErrorInvalidValue;
    dim3 g(blocks), b(kWG);
#define QDTA_SSSP(U, V) \
    hipLaunchKernelGGL((k_sssp_ds<U, V>), g, b, 0, s, net, dem, radj, labels, scr, st, delta_inst, early, \
                       t_begin, t_end)
    switch (variant) {
        case 0: QDTA_SSSP(1, 4); break;
        case 1: QDTA_SSSP(2, 4); break;
        case 2: QDTA_SSSP(4, 4); break;
        case 3: QDTA_SSSP(4, 8); break;
        case 4: QDTA_SSSP(8, 8); break;
        default: QDTA_SSSP(1, 1); break;
    }
#undef QDTA_SSSP
    return hipGetLastError();
}

hipError_t launch_sssp(hipStream_t s, const NetDev& net, const DemDev& dem, const double* logpart, const uint2* radj,
                       label_t* labels, const Scratch& scr, int slots, const InstState* st, double delta_scale,
                       float* delta_inst, int variant, int early, bool fill, int64_t* y, int32_t* absorb_q) {
    hipError_t e = launch_prep(s, net, logpart, delta_scale, delta_inst, scr.work, y, absorb_q, dem.Q);
    if (e != hipSuccess) return e;
    return launch_trees(s, net, dem, radj, labels, scr, slots, st, delta_inst, variant, early, 0, dem.Q, fill);
}

// ---------------------------------------------------------------------------
// A3: truncation + loading, and the residual walk of Alg. 4
// ---------------------------------------------------------------------------
// Successor of u on the tree whose labels are lab[node - node0]: the
// lowest-uid out-link (u, w) that is tight, fl32(D(w) + c) == D(u), and
// strict, D(w) < D(u).  -1 when FP32 absorption leaves none.
__device__ __forceinline__ int succ_strict(const NetDev& net, const label_t* lab, int node0, int u, float du,
                                          const float* tree_cost) {
    const int e1 = net.row_ptr[u + 1];
    for (int e = net.row_ptr[u]; e < e1; ++e) {
        const float dw = lab_val(lab, net.col[e] - node0);
        if (dw < du && dw + tree_cost[e] == du) return e;
    }
    return -1;
}

// The same successor, reading (head, cost) from the forward link records,
// whose costs are the ones the trees were grown with: one line per link
// instead of the head and cost arrays.  Also returns the head and the cost.
__device__ __forceinline__ int succ_rec(const NetDev& net, const label_t* lab, int node0, int u, float du, int& head,
                                       float& cost) {
    const int e1 = net.row_ptr[u + 1];
    for (int e = net.row_ptr[u]; e < e1; ++e) {
        const uint2 r = net.fadj[e];
        const float dw = lab_val(lab, (int)r.x - node0);
        const float c = __uint_as_float(r.y);
        if (dw < du && dw + c == du) {
            head = (int)r.x;
            cost = c;
            return e;
        }
    }
    return -1;
}

// The same successor as succ_rec, for a walk that carries u's forward row
// packed (kNoRow: read the row pointers): the row's records with their
// heads' packed rows, then the heads' labels, are loaded four at a time
// together (indices past the row's end repeat its last link), and the
// lowest tight strict link wins as before.  Also returns the head's packed
// row and label for the next hop.
__device__ __forceinline__ int succ_row(const NetDev& net, const label_t* lab, int node0, int u, uint32_t row,
                                        float du, int& head, float& cost, uint32_t& head_row, float& head_lab) {
    int e0, deg;
    if (row != kNoRow) {
        e0 = (int)(row >> kRowCountBits);
        deg = (int)(row & ((1u << kRowCountBits) - 1u));
    } else {
        e0 = net.row_ptr[u];
        deg = net.row_ptr[u + 1] - e0;
    }
    const int last = e0 + deg - 1;
    for (int b = 0; b < deg; b += 4) {
        uint2 r[4];
        uint32_t fr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = min(e0 + b + j, last);
            r[j] = net.fadj[e];
            fr[j] = net.frow[e];
        }
        float dw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) dw[j] = lab_val(lab, (int)r[j].x - node0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float c = __uint_as_float(r[j].y);
            if (b + j < deg && dw[j] < du && dw[j] + c == du) {
                head = (int)r[j].x;
                cost = c;
                head_row = fr[j];
                head_lab = dw[j];
                return e0 + b + j;
            }
        }
    }
    return -1;
}

// The same by four neighbouring lanes for one u: each takes every fourth link of
// the row, and all return the lowest tight strict one.
__device__ __forceinline__ int succ_quad(const NetDev& net, const label_t* lab, int node0, int u, uint32_t row,
                                         float du, int& head, float& cost, uint32_t& head_row, float& head_lab) {
    const int lane = threadIdx.x & 63, j = lane & 3, quad = lane & 60;
    int e0, deg;
    if (row != kNoRow) {
        e0 = (int)(row >> kRowCountBits);
        deg = (int)(row & ((1u << kRowCountBits) - 1u));
    } else {
        e0 = net.row_ptr[u];
        deg = net.row_ptr[u + 1] - e0;
    }
    for (int b = 0; b < deg; b += 4) {
        const int e = e0 + min(b + j, deg - 1);
        const uint2 r = net.fadj[e];
        const uint32_t fr = net.frow[e];
        const float dw = lab_val(lab, (int)r.x - node0), c = __uint_as_float(r.y);
        const unsigned m = (unsigned)(__ballot(b + j < deg && dw < du && dw + c == du) >> quad) & 15u;
        if (m) {
            const int w = __ffs(m) - 1;
            head = __shfl((int)r.x, quad + w);
            cost = __shfl(c, quad + w);
            head_row = (uint32_t)__shfl((int)fr, quad + w);
            head_lab = __shfl(dw, quad + w);
            return e0 + b + w;
        }
    }
    return -1;
}

struct WalkOut {
    int64_t* y;
    int32_t* stop;
    float* stop_delay;           // AON mode, may be NULL: the delay a leg stops with (link-progress rule)
    int residual_mode;
    const double* lambda;        // per instance (residual mode)
    int64_t* r_dense;            // residual accumulator, indexed like the labels
    unsigned long long* done_fx;
    TransitOut tr;               // residual mode, link-progress rule: legs left on a link
    int* err;                    // set when the transit list overflows
};

// Residual mode adds rint(lambda d) of a leg that stops at s short of q to
// the accumulator word of (tree qi, node s), whose label offset is lab0 --
// or, when it stops on a link with a delay, appends it to the transit list
// -- and returns the weight a completed leg adds to done_fx otherwise.
__device__ __forceinline__ int64_t finish_leg(const WalkOut& o, int l, int s, int q, int qi, int64_t lab0, int inst,
                                              int node0, int64_t d, float delay) {
    if (!o.residual_mode) {
        if (o.stop) o.stop[l] = s - node0;
        if (o.stop_delay) o.stop_delay[l] = delay;
        return 0;
    }
    const int64_t w = (int64_t)__builtin_rint(o.lambda[inst] * (double)d);
    if (s == q) return w;
    if (w == 0) return 0;
    if (delay > 0.0f) {
        const unsigned int k = atomicAdd(o.tr.n, 1u);
        if (k < o.tr.cap) {
            o.tr.q[k] = qi;
            o.tr.node[k] = s - node0;
            o.tr.delay[k] = delay;
            o.tr.w[k] = w;
        } else {
            *o.err = 1;
        }
        return 0;
    }
    atomicAdd(reinterpret_cast<unsigned long long*>(&o.r_dense[lab0 + (s - node0)]), (unsigned long long)w);
    return 0;
}

// One step of the truncated walk (Eq. 2 read as CEIL / FLOOR / NONE, or the
// link-progress rule): whether a leg at a node at time tau stops there, and
// after entering a link (new time nt) whether it stops on it.  PROGRESS loads
// as CEIL; a trip still on a link at dt stops at its head with delay
// nt - dt (a trip on its last link completes), and a leg that starts with
// its delay at or above dt is still on its way to its origin.
// A delay a leg leaves the interval with, rounded up to a whole multiple of
// pq seconds in FP64 when pq > 0 (legs stopped on the same link for the
// same destination then merge).
__device__ __forceinline__ float progress_delay(float x, double pq) {
    return pq > 0.0 ? (float)(pq * ceil((double)x / pq)) : x;
}

__device__ __forceinline__ bool stop_at_node(int rule, float tau, float dt) {
    return (rule == RULE_CEIL || rule == RULE_PROGRESS) && tau >= dt;
}

// time_cost: the costs that clock the truncation (Eq. 2); NULL = the trees'
// own costs (the forward records), as in the AON of an iteration.
// Q lanes walk a leg (1: succ_row, 4: succ_quad), the NT threads of a workgroup a
// contiguous run of NT / Q * LPT legs.  Loads of a workgroup's legs are summed per
// link in an LDS table first (legs of one destination share links); the table is
// added to y when the workgroup is done, and a load whose probes find no slot goes
// to y directly.  Integer sums: the order does not change them.  16 slots per
// walker (48 KB at 256, twelve wavefronts per CU): half as many hold too few of
// the distinct links (1,191 against 823 us at 316k legs), and twice as many leave
// half the wavefronts.
template <int NT, int LPT, int Q>
__global__ __launch_bounds__(NT) void k_walk(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                              const float* __restrict__ time_cost, const InstState* st,
                                              FlagsDev fl, WalkOut o, int l_begin, int l_end) {
    constexpr int SLOTS = 16 * NT / Q;
    const bool lead = Q == 1 || threadIdx.x % Q == 0;
    __shared__ int s_key[SLOTS];
    __shared__ unsigned long long s_sum[SLOTS];
    // completed weight of the first leg's instance (residual mode): one global
    // atomic per workgroup, since the legs' own ran one after another on the one
    // word (residual walk of 73k legs: 0.75 -> 0.15 ms)
    __shared__ unsigned long long s_done;
    const bool loads = !o.residual_mode;
    if (loads)
        for (int x = threadIdx.x; x < SLOTS; x += NT) {
            s_key[x] = -1;
            s_sum[x] = 0ull;
        }
    __shared__ int s_absorbed;
    if (threadIdx.x == 0) {
        s_done = 0ull;
        s_absorbed = 0;
    }
    __syncthreads();
    auto load = [&](int e, int64_t d) {
        int h = (int)(((unsigned)e * 2654435761u) >> 20) & (SLOTS - 1);
        for (int probe = 0; probe < 4; ++probe) {
            const int k = atomicCAS(&s_key[h], -1, e);   // one access, whether the slot is taken or not
            if (k == -1 || k == e) {
                atomicAdd(&s_sum[h], (unsigned long long)d);
                return;
            }
            h = (h + 1) & (SLOTS - 1);
        }
        atomicAdd(reinterpret_cast<unsigned long long*>(&o.y[e]), (unsigned long long)d);
    };
    const int base = l_begin + blockIdx.x * (NT / Q) * LPT;
    const int lim = min(l_end, base + (NT / Q) * LPT);
    const int inst0 = dem.dest_inst[dem.leg_q[base]];
    for (int l = base + (int)threadIdx.x / Q; l < lim; l += NT / Q) {
        const int qi = dem.leg_q[l];
        const int inst = dem.dest_inst[qi];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int node0 = I.node0;
        const int q = dem.dest_node[qi];
        const label_t* lab = tree_labels(labels, dem, qi);
        const int64_t d = dem.leg_dfx[l];
        int u = dem.leg_orig[l];
        float du = lab_val(lab, u - node0);
        if (lead) fl.int_node[l] = -1;
        if (!(du <= 3.4028234663852886e38f)) {       // origin cannot reach q
            *fl.err_unreach = 1;
            if (lead && o.stop) o.stop[l] = -1;
            continue;
        }
        float tau = dem.leg_delay ? dem.leg_delay[l] : 0.0f;
        float delay = 0.0f;
        bool absorbed = false;
        if (I.rule == RULE_PROGRESS && tau >= I.dt32) {
            delay = progress_delay(tau - I.dt32, I.pq);   // still on its way to its origin
        } else {
            uint32_t urow = kNoRow;                   // u's forward row, carried from the link into u
            for (int hops = 0; u != q; ++hops) {
                if (stop_at_node(I.rule, tau, I.dt32)) break;
                int head = 0;
                float ce = 0.0f, hlab = 0.0f;
                uint32_t hrow = kNoRow;
                const int e = Q == 4 ? succ_quad(net, lab, node0, u, urow, du, head, ce, hrow, hlab)
                                     : succ_row(net, lab, node0, u, urow, du, head, ce, hrow, hlab);
                if (e < 0 || hops > I.n) {            // absorption: finish in the fallback
                    if (lead) {
                        fl.int_node[l] = u;
                        fl.int_tau[l] = tau;
                    }
                    fl.absorb_q[qi] = 1;
                    s_absorbed = 1;
                    absorbed = true;
                    break;
                }
                const float nt = tau + (time_cost ? time_cost[e] : ce);
                if (I.rule == RULE_FLOOR && nt > I.dt32) break;
                if (loads && lead) load(e, d);
                tau = nt;
                u = head;
                urow = hrow;
                du = hlab;
                if (I.rule == RULE_PROGRESS && tau > I.dt32) {
                    if (u != q) delay = progress_delay(tau - I.dt32, I.pq);
                    break;
                }
            }
        }
        if (lead && !absorbed) {
            const int64_t wd = finish_leg(o, l, u, q, qi, dem.dest_lab[qi], inst, node0, d, delay);
            if (wd && inst == inst0) atomicAdd(&s_done, (unsigned long long)wd);
            else if (wd) atomicAdd(&o.done_fx[inst], (unsigned long long)wd);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_absorbed) *fl.absorb_any = 1;
    if (loads) {
        for (int x = threadIdx.x; x < SLOTS; x += NT)
            if (s_key[x] >= 0) atomicAdd(reinterpret_cast<unsigned long long*>(&o.y[s_key[x]]), s_sum[x]);
    } else if (threadIdx.x == 0 && s_done) {
        atomicAdd(&o.done_fx[inst0], s_done);
    }
}

hipError_t launch_walk(hipStream_t s, const NetDev& net, const DemDev& dem, const label_t* labels,
                       const float* time_cost, int64_t* y, int32_t* stop,
                       const InstState* st, const FlagsDev& fl, int residual_mode, const double* lambda,
                       int64_t* r_dense, unsigned long long* done_fx,
                       int l_begin, int l_end, float* stop_delay, const TransitOut* tr) {
    if (l_end < 0) l_end = dem.P;
    if (l_end <= l_begin) return hipSuccess;
    WalkOut o{y, stop, stop_delay, residual_mode, lambda, r_dense, done_fx,
              tr ? *tr : TransitOut{nullptr, nullptr, nullptr, nullptr, nullptr, 0u}, fl.err_overflow};
    // Four lanes a leg load a row's links together (one line instead of one a
    // link), which pays while most legs are in flight at once (512 threads hold 128
    // legs, about 98,000 on the card); two legs per thread put the most in flight
    // and share the table between the most.  The line is where they were found to
    // cross: legs, us of the phase with four lanes a leg / with two legs a thread:
    // 85,713 326 / 533; 180,898 548 / 618; 175,041 697 / 691; 203,948 870 / 685;
    // 229,780 752 / 731; 348,614 968 / 852; 1.13M 3,429 / 3,393 (road networks of 100k
    // and 300k nodes at 900 s); static grids: 89,700 436 / 755; 175,980 793 / 909;
    // 249,500 986 / 929; 359,400 1,344 / 1,289.  One leg per thread, not used, lies
    // between them or below on some of these (125,800 legs: 401; 1.13M: 2,989) and
    // above both on others (203,948: 793; 229,780: 863; 249,500: 1,047).
#define QDTA_WALK(NT, LPT, Q)                                                                                      \
    hipLaunchKernelGGL((k_walk<NT, LPT, Q>),                                                                       \
                       dim3((unsigned)((l_end - l_begin + NT / Q * LPT - 1) / (NT / Q * LPT))), dim3(NT), 0, s,    \
                       net, dem, labels, time_cost, st, fl, o, l_begin, l_end)
    if (l_end - l_begin < 200000) QDTA_WALK(512, 1, 4);
    else QDTA_WALK(256, 2, 1);
#undef QDTA_WALK
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A3, plain intervals: loading by children-before-parent accumulation
// ---------------------------------------------------------------------------
// Without truncation every leg of tree q loads its whole path to q, so the
// flow on the successor link of v is the demand of all legs whose paths pass
// through v.  Instead of walking every leg to q, the legs' paths are merged:
//   pass 1 (k_sweep_count): each leg walks from its origin; at every node it
//     reaches it adds 1 to the node's arrival count and goes on only if it
//     was the first to arrive -- so each node's count is the number of legs
//     and path branches that will bring demand into it;
//   pass 2 (k_sweep_push): each leg starts again with its demand; at a node
//     it adds what it carries to the node's accumulator and takes one off
//     the count; the arrival that takes the count to zero is the last, takes
//     the whole accumulated demand, loads the successor link with it and goes
//     on to the parent.
// Every link is loaded once per tree with the integer sum of the demand of
// the legs that use it: the same int64 y as the walk.  Both scratch arrays
// (indexed like the labels) are back at zero afterwards.  A tree where a
// walker meets FP32 absorption is flagged; pass 2 walks its legs as k_walk
// does (clearing the counts pass 1 left on their paths) and the tie
// fallback finishes them.  Used only when every instance is plain.
__global__ __launch_bounds__(kWG) void k_sweep_count(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                                     const InstState* st, FlagsDev fl, uint32_t* cnt) {
    const int l = blockIdx.x * kWG + threadIdx.x;
    if (l >= dem.P) return;
    const int qi = dem.leg_q[l];
    const int inst = dem.dest_inst[qi];
    if (!inst_live(st, inst)) return;
    const InstDev I = net.inst[inst];
    if (I.rule != RULE_NONE) return;
    const int node0 = I.node0, q = dem.dest_node[qi];
    const label_t* lab = tree_labels(labels, dem, qi);
    uint32_t* C = cnt + dem.dest_lab[qi] - node0;       // indexed by global node id
    int u = dem.leg_orig[l];
    float du = lab_val(lab, u - node0);
    if (!(du <= 3.4028234663852886e38f)) return;        // unreachable: reported by pass 2
    for (int hops = 0; u != q; ++hops) {
        if (atomicAdd(&C[u], 1u) != 0u) return;         // another arrival goes on from here
        int head = 0;
        float ce = 0.0f;
        const int e = succ_rec(net, lab, node0, u, du, head, ce);
        if (e < 0 || hops > I.n) {                      // absorption: this tree is walked
            fl.absorb_q[qi] = 1;
            return;
        }
        u = head;
        du = lab_val(lab, u - node0);
    }
}

__global__ __launch_bounds__(kWG) void k_sweep_push(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                                    const InstState* st, FlagsDev fl, WalkOut o, uint32_t* cnt,
                                                    int64_t* acc) {
    const int l = blockIdx.x * kWG + threadIdx.x;
    if (l >= dem.P) return;
    const int qi = dem.leg_q[l];
    const int inst = dem.dest_inst[qi];
    if (!inst_live(st, inst)) return;
    const InstDev I = net.inst[inst];
    const int node0 = I.node0, q = dem.dest_node[qi];
    const label_t* lab = tree_labels(labels, dem, qi);
    uint32_t* C = cnt + dem.dest_lab[qi] - node0;
    int64_t* A = acc + dem.dest_lab[qi] - node0;
    int u = dem.leg_orig[l];
    float du = lab_val(lab, u - node0);
    fl.int_node[l] = -1;
    if (!(du <= 3.4028234663852886e38f)) {
        *fl.err_unreach = 1;
        if (o.stop) o.stop[l] = -1;
        return;
    }
    if (o.stop) o.stop[l] = q - node0;                  // without truncation every leg completes
    if (o.stop_delay) o.stop_delay[l] = 0.0f;
    const bool sweep = !ld_coherent(&fl.absorb_q[qi]);
    int64_t carry = dem.leg_dfx[l];
    for (int hops = 0; u != q; ++hops) {
        if (sweep) {
            atomicAdd(reinterpret_cast<unsigned long long*>(&A[u]), (unsigned long long)carry);
            wait_memory();                              // the demand is in before the count drops
            if (atomicSub(&C[u], 1u) != 1u) return;     // not the last arrival: done
            carry = (int64_t)atomicExch(reinterpret_cast<unsigned long long*>(&A[u]), 0ull);
        } else {
            C[u] = 0u;                                  // a flagged tree: clear what pass 1 counted
        }
        int head = 0;
        float ce = 0.0f;
        const int e = succ_rec(net, lab, node0, u, du, head, ce);
        if (e < 0 || hops > I.n) {                      // absorption (flagged trees only): the fallback
            fl.int_node[l] = u;                         // finishes the leg
            fl.int_tau[l] = 0.0f;
            fl.absorb_q[qi] = 1;
            *fl.absorb_any = 1;
            return;
        }
        atomicAdd((unsigned long long*)&o.y[e], (unsigned long long)carry);
        u = head;
        du = lab_val(lab, u - node0);
    }
}

hipError_t launch_sweep(hipStream_t s, const NetDev& net, const DemDev& dem, const label_t* labels,
                        int64_t* y, int32_t* stop, float* stop_delay, const InstState* st, const FlagsDev& fl,
                        uint32_t* cnt, int64_t* acc) {
    if (dem.P == 0) return hipSuccess;
    const dim3 g((dem.P + kWG - 1) / kWG), b(kWG);
    hipLaunchKernelGGL(k_sweep_count, g, b, 0, s, net, dem, labels, st, fl, cnt);
    WalkOut o{y, stop, stop_delay, 0, nullptr, nullptr, nullptr,
              TransitOut{nullptr, nullptr, nullptr, nullptr, nullptr, 0u}, fl.err_overflow};
    hipLaunchKernelGGL(k_sweep_push, g, b, 0, s, net, dem, labels, st, fl, o, cnt, acc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tie-rule fallback under FP32 absorption
// ---------------------------------------------------------------------------
// For a flagged tree: hop depth h to q inside the tight subgraph (links with
// fl32(D(w) + c) == D(v)), breadth-first from q; a node without a strict
// tight link then takes the lowest-uid tight link to a node with h - 1.
// Trees mode fills the missing successors; walk mode finishes the legs that
// the walk interrupted.  One workgroup per flagged tree.
__global__ __launch_bounds__(kWG) void k_fallback(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                                  const float* __restrict__ tree_cost,
                                                  const float* __restrict__ time_cost, const InstState* st,
                                                  FlagsDev fl, Scratch scr, WalkOut o, int trees_mode,
                                                  int32_t* succ_out, int32_t n_out) {
    __shared__ int s_cnt[2];
    int32_t* hop = scr.farq + (int64_t)blockIdx.x * scr.nmax;
    int32_t* qbase = scr.nearq + (int64_t)blockIdx.x * scr.nmax;
    for (int qi = blockIdx.x; qi < dem.Q; qi += gridDim.x) {
        if (!fl.absorb_q[qi]) continue;
        const int inst = dem.dest_inst[qi];
        if (!inst_live(st, inst)) continue;
        const InstDev I = net.inst[inst];
        const int n = I.n, node0 = I.node0;
        const label_t* lab = tree_labels(labels, dem, qi);
        const int q = dem.dest_node[qi];
        // breadth-first levels in one FIFO: level L occupies [s_cnt[0], s_cnt[1])
        for (int v = threadIdx.x; v < n; v += kWG) hop[v] = -1;
        if (threadIdx.x == 0) { s_cnt[0] = 0; s_cnt[1] = 1; }
        __syncthreads();
        if (threadIdx.x == 0) { hop[q - node0] = 0; qbase[0] = q - node0; }
        __syncthreads();
        for (int level = 0;; ++level) {
            const int lo = s_cnt[0], hi = s_cnt[1];
            if (lo == hi) break;
            __syncthreads();
            for (int i = lo + threadIdx.x; i < hi; i += kWG) {
                const int u = qbase[i];
                const float du = lab_val(lab, u);
                for (int e = net.rptr[node0 + u]; e < net.rptr[node0 + u + 1]; ++e) {
                    const int v = net.rsrc[e] - node0;
                    const int link = net.rlink[e];
                    const float dv = lab_val(lab, v);
                    if (dv <= 3.4028234663852886e38f && du + tree_cost[link] == dv) {
                        if (atomicCAS(&hop[v], -1, level + 1) == -1) {
                            int pos = atomicAdd(&s_cnt[1], 1);
                            qbase[pos] = v;
                        }
                    }
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) s_cnt[0] = hi;
            __syncthreads();
        }
        // successor with the hop rule where no strict tight link exists
        auto succ_full = [&](int u, float du) -> int {
            int e = succ_strict(net, lab, node0, u, du, tree_cost);
            if (e >= 0) return e;
            const int hu = ld_coherent(&hop[u - node0]);
            for (int k = net.row_ptr[u]; k < net.row_ptr[u + 1]; ++k) {
                const int w = net.col[k];
                const float dw = lab_val(lab, w - node0);
                if (dw + tree_cost[k] == du && ld_coherent(&hop[w - node0]) == hu - 1) return k;
            }
            return -1;
        };
        if (trees_mode) {
            const int t = qi;
            for (int v = threadIdx.x; v < n; v += kWG) {
                const int g = node0 + v;
                const float dv = lab_val(lab, v);
                if (g == q || !(dv <= 3.4028234663852886e38f)) continue;
                if (succ_out[(int64_t)t * n_out + v] >= 0) continue;
                const int e = succ_full(g, dv);
                succ_out[(int64_t)t * n_out + v] = e >= 0 ? e - I.link0 : -1;
            }
        } else {
            for (int l = dem.qptr[qi] + threadIdx.x; l < dem.qptr[qi + 1]; l += kWG) {
                int u = fl.int_node[l];
                if (u < 0) continue;
                float tau = fl.int_tau[l];
                float du = lab_val(lab, u - node0);
                const int64_t d = dem.leg_dfx[l];
                float delay = 0.0f;
                for (int hops = 0; u != q && hops <= n; ++hops) {
                    if (stop_at_node(I.rule, tau, I.dt32)) break;
                    const int e = succ_full(u, du);
                    if (e < 0) break;
                    const float nt = tau + time_cost[e];
                    if (I.rule == RULE_FLOOR && nt > I.dt32) break;
                    if (!o.residual_mode) atomicAdd((unsigned long long*)&o.y[e], (unsigned long long)d);
                    tau = nt;
                    u = net.col[e];
                    du = lab_val(lab, u - node0);
                    if (I.rule == RULE_PROGRESS && tau > I.dt32) {
                        if (u != q) delay = progress_delay(tau - I.dt32, I.pq);
                        break;
                    }
                }
                fl.int_node[l] = -1;
                const int64_t w = finish_leg(o, l, u, q, qi, dem.dest_lab[qi], inst, node0, d, delay);
                if (w) atomicAdd(&o.done_fx[inst], (unsigned long long)w);
            }
        }
        __syncthreads();
    }
}

hipError_t launch_fallback(hipStream_t s, const NetDev& net, const DemDev& dem, const label_t* labels,
                           const float* tree_cost, const float* time_cost, int64_t* y, int32_t* stop,
                           const InstState* st, const FlagsDev& fl, const Scratch& scr, int slots,
                           int residual_mode, const double* lambda, int64_t* r_dense,
                           unsigned long long* done_fx, int trees_mode,
                           int32_t* succ_out, int32_t n_out, float* stop_delay, const TransitOut* tr) {
    if (dem.Q == 0) return hipSuccess;
    WalkOut o{y, stop, stop_delay, residual_mode, lambda, r_dense, done_fx,
              tr ? *tr : TransitOut{nullptr, nullptr, nullptr, nullptr, nullptr, 0u}, fl.err_overflow};
    hipLaunchKernelGGL(k_fallback, dim3(slots), dim3(kWG), 0, s, net, dem, labels, tree_cost, time_cost, st, fl, scr,
                       o, trees_mode, succ_out, n_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A8: compaction of the residual accumulator
// ---------------------------------------------------------------------------
// Tree t's residual legs are the non-zero words of its row (n words at
// dest_lab[t]); rows are taken in tree order and nodes in ascending order,
// which is (destination, origin) order.  The write pass clears what it
// reads, so the accumulator is all zero again afterwards.
__device__ __forceinline__ int block_excl_scan(int x, int* tot, int* s_w) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = x;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int k = 0; k < kWG / 64; ++k) {
        if (k < wv) before += s_w[k];
        all += s_w[k];
    }
    __syncthreads();
    *tot = all;
    return before + incl - x;
}

__global__ __launch_bounds__(kWG) void k_resid_count(NetDev net, DemDev dem, const int64_t* __restrict__ r_dense,
                                                     int64_t* cnt) {
    __shared__ int s_w[kWG / 64];
    const int t = blockIdx.x;
    const int n = net.inst[dem.dest_inst[t]].n;
    const int64_t* row = r_dense + dem.dest_lab[t];
    int c = 0;
    for (int v = threadIdx.x; v < n; v += kWG) c += row[v] != 0;
    int tot = 0;
    block_excl_scan(c, &tot, s_w);
    if (threadIdx.x == 0) cnt[t] = tot;
}

__global__ __launch_bounds__(kWG) void k_resid_write(NetDev net, DemDev dem, int64_t* r_dense, const int64_t* off,
                                                     int32_t* r_orig, int32_t* r_q, int64_t* r_w) {
    __shared__ int s_w[kWG / 64];
    const int t = blockIdx.x;
    const int n = net.inst[dem.dest_inst[t]].n;
    int64_t* row = r_dense + dem.dest_lab[t];
    int64_t base = off[t];
    for (int v0 = 0; v0 < n; v0 += kWG) {
        const int v = v0 + threadIdx.x;
        const int64_t x = v < n ? row[v] : 0;
        int tot = 0;
        const int pos = block_excl_scan(x != 0 ? 1 : 0, &tot, s_w);
        if (x != 0) {
            r_orig[base + pos] = v;
            r_q[base + pos] = t;
            r_w[base + pos] = x;
            row[v] = 0;
        }
        base += tot;
    }
}

hipError_t launch_resid_count(hipStream_t s, const NetDev& net, const DemDev& dem, const int64_t* r_dense,
                              int64_t* cnt) {
    if (dem.Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_resid_count, dim3(dem.Q), dim3(kWG), 0, s, net, dem, r_dense, cnt);
    return hipGetLastError();
}

hipError_t launch_resid_write(hipStream_t s, const NetDev& net, const DemDev& dem, int64_t* r_dense,
                              const int64_t* off, int32_t* r_orig, int32_t* r_q, int64_t* r_w) {
    if (dem.Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_resid_write, dim3(dem.Q), dim3(kWG), 0, s, net, dem, r_dense, off, r_orig, r_q, r_w);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Parity output of trees: dist[t][v], succ[t][v] (local uid)
// ---------------------------------------------------------------------------
// A thread per (node, tree): the four first links of its row and then their
// heads' labels are loaded together, from the records the trees were grown with.
// Bound by those gathers (100 trees of 100k nodes: 60 us, 93 with the links one
// after another from three arrays and a 64-bit division per output).
__global__ __launch_bounds__(kWG) void k_trees_out(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                                   int32_t inst, float* dist, int32_t* succ, int32_t* absorb_q,
                                                   int* absorb_any) {
    const InstDev I = net.inst[inst];
    const int v = (int)(blockIdx.x * kWG + threadIdx.x), g = I.node0 + v;
    if (v >= I.n) return;
    const int e0 = net.row_ptr[g], deg = net.row_ptr[g + 1] - e0;
    for (int t = blockIdx.y; t < dem.Q; t += gridDim.y) {
        const label_t* lab = tree_labels(labels, dem, t);
        const float dv = lab_val(lab, v);
        int e = -1;
        if (g != dem.dest_node[t] && dv <= 3.4028234663852886e38f) {
            for (int b = 0; b < deg && e < 0; b += 4) {
                uint2 r[4];
                float dw[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] = net.fadj[e0 + min(b + j, deg - 1)];
#pragma unroll
                for (int j = 0; j < 4; ++j) dw[j] = lab_val(lab, (int)r[j].x - I.node0);
#pragma unroll
                for (int j = 3; j >= 0; --j)
                    if (b + j < deg && dw[j] < dv && dw[j] + __uint_as_float(r[j].y) == dv) e = e0 + b + j;
            }
            if (e < 0 && atomicExch(&absorb_q[t], 1) == 0) *absorb_any = 1;
        }
        dist[(int64_t)t * I.n + v] = dv;
        succ[(int64_t)t * I.n + v] = e >= 0 ? e - I.link0 : -1;
    }
}

hipError_t launch_trees_out(hipStream_t s, const NetDev& net, const DemDev& dem, const label_t* labels, int n,
                            int32_t inst, float* dist, int32_t* succ, int32_t* absorb_q, int* absorb_any) {
    if (dem.Q == 0) return hipSuccess;
    hipLaunchKernelGGL(k_trees_out, dim3((n + kWG - 1) / kWG, dem.Q < 65535 ? dem.Q : 65535), dim3(kWG), 0, s, net, dem,
                       labels, inst, dist, succ, absorb_q, absorb_any);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Frozen-path model and its reverse pass (OD calibration)
// ---------------------------------------------------------------------------
// The truncated path of every leg under one iterate's trees: the links the
// walk of that iterate loads (same successor rule, same clock), in walk
// order.  ptr == NULL counts them into len[l]; otherwise they are written at
// links[ptr[l]] (and the leg index at leg_of[ptr[l]]), never past ptr[l + 1].
// bad: three words, set to 1 where an origin cannot reach its destination, where
// FP32 absorption ends a path (the tie fallback's paths are not recorded), and
// where a path is longer than counted.
__global__ __launch_bounds__(kWG) void k_path_walk(NetDev net, DemDev dem, const label_t* __restrict__ labels,
                                                   const int64_t* __restrict__ ptr, int32_t* __restrict__ links,
                                                   int32_t* __restrict__ leg_of, int64_t* __restrict__ len,
                                                   int* bad) {
    const int l = blockIdx.x * kWG + threadIdx.x;
    if (l >= dem.P) return;
    const int qi = dem.leg_q[l];
    const InstDev I = net.inst[dem.dest_inst[qi]];
    const int node0 = I.node0;
    const int q = dem.dest_node[qi];
    const label_t* lab = tree_labels(labels, dem, qi);
    int u = dem.leg_orig[l];
    float du = lab_val(lab, u - node0);
    const int64_t at = ptr ? ptr[l] : 0, end = ptr ? ptr[l + 1] : 0;
    int64_t k = 0;
    if (!(du <= 3.4028234663852886e38f)) {
        bad[0] = 1;
        if (len) len[l] = 0;
        return;
    }
    float tau = 0.0f;
    for (int hops = 0; u != q; ++hops) {
        if (I.rule == RULE_CEIL && tau >= I.dt32) break;
        int head = 0;
        float ce = 0.0f;
        const int e = succ_rec(net, lab, node0, u, du, head, ce);
        if (e < 0 || hops > I.n) {
            bad[1] = 1;
            break;
        }
        const float nt = tau + ce;
        if (I.rule == RULE_FLOOR && nt > I.dt32) break;
        if (ptr) {
            if (at + k >= end) {
                bad[2] = 1;
                break;
            }
            links[at + k] = e;
            leg_of[at + k] = l;
        }
        ++k;
        tau = nt;
        u = head;
        du = lab_val(lab, u - node0);
    }
    if (len) len[l] = k;
}

hipError_t launch_path_walk(hipStream_t s, const NetDev& net, const DemDev& dem, const label_t* labels,
                            const int64_t* ptr, int32_t* links, int32_t* leg_of, int64_t* len, int* bad) {
    if (dem.P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_path_walk, dim3((dem.P + kWG - 1) / kWG), dim3(kWG), 0, s, net, dem, labels, ptr, links,
                       leg_of, len, bad);
    return hipGetLastError();
}

// y += rint(d 2^20) along every leg's path: the loading of Eq. 5 for a
// real-valued demand, exact in int64 whatever the order of the atomics.
// One lane per (leg, link) entry of the flattened paths, so the link ids
// and leg indices are read coalesced and long paths spread over lanes.  A
// workgroup takes a run of kPathRun entries and sums it per link in LDS first:
// the legs of a destination are neighbours and share many of their links, and an
// atomic on y is carried out beyond the L2.  The table keeps the 16 links of a
// 128-byte line of y together (links along a path are neighbours too), so that
// the sums leave it line by line, as the entries themselves would; with the lines
// scattered over the slots, paths that share little took longer than an atomic on
// y per entry.  Forward pass of the model, one iterate, us, with an atomic per entry
// / with scattered slots / so: 261k legs to 5,000 of 550k nodes at 900 s 2,058 /
// 2,716 / 1,600, to the end 5,058 / 4,791 / 2,730; 27,400 legs to 300 of 100k nodes
// 401 / 282 / 241.  (Runs of 1,024 and 2,048 entries and smaller workgroups: up to
// 20% longer.)
constexpr int kPathRun = 4096, kPathWG = 1024;

__global__ __launch_bounds__(kPathWG) void k_path_load(int64_t total, const int32_t* __restrict__ links,
                                                   const int32_t* __restrict__ leg_of, const double* __restrict__ d,
                                                   int64_t* y, int* err) {
    constexpr int SLOTS = kPathRun;
    __shared__ int s_key[SLOTS];
    __shared__ unsigned long long s_sum[SLOTS];
    for (int x = threadIdx.x; x < SLOTS; x += kPathWG) {
        s_key[x] = -1;
        s_sum[x] = 0ull;
    }
    __syncthreads();
    const int64_t i0 = blockIdx.x * (int64_t)kPathRun, i1 = min(total, i0 + kPathRun);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kPathWG) {
        const int e = links[i];
        const double x = d[leg_of[i]] * 1048576.0;
        if (!(x > -9.0e18 && x < 9.0e18)) {
            *err = 1;
            continue;
        }
        const int64_t w = (int64_t)__builtin_rint(x);
        if (w == 0) continue;
        int h = ((int)(((unsigned)(e >> 4) * 2654435761u) >> 16) << 4 | (e & 15)) & (SLOTS - 1);
        bool in = false;
        for (int probe = 0; probe < 4 && !in; ++probe) {
            const int k = atomicCAS(&s_key[h], -1, e);
            in = k == -1 || k == e;
            if (!in) h = (h + 1) & (SLOTS - 1);
        }
        if (in) atomicAdd(&s_sum[h], (unsigned long long)w);
        else atomicAdd(reinterpret_cast<unsigned long long*>(&y[e]), (unsigned long long)w);
    }
    __syncthreads();
    for (int x = threadIdx.x; x < SLOTS; x += kPathWG)
        if (s_sum[x]) atomicAdd(reinterpret_cast<unsigned long long*>(&y[s_key[x]]), s_sum[x]);
}

hipError_t launch_path_load(hipStream_t s, int64_t total, const int32_t* links, const int32_t* leg_of,
                            const double* d, int64_t* y, int* err) {
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_path_load, dim3((unsigned)((total + kPathRun - 1) / kPathRun)), dim3(kPathWG), 0, s, total, links,
                       leg_of, d, y, err);
    return hipGetLastError();
}

// dbar[l] (+)= the sum of g over leg l's path: the transpose of the
// loading.  A group of 16 lanes per leg reads the link ids coalesced; each
// lane sums every 16th entry in walk order, then the group adds its 16
// partial sums by a fixed butterfly, so the result does not vary run to run.
constexpr int kGatherLanes = 16;

__global__ __launch_bounds__(kWG) void k_path_gather(int P, const int64_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ links,
                                                     const double* __restrict__ g, double* dbar, int accumulate) {
    const int64_t gid = (blockIdx.x * (int64_t)kWG + threadIdx.x) / kGatherLanes;
    const int sub = threadIdx.x % kGatherLanes;
    const bool live = gid < P;
    double acc = 0.0;
    if (live) {
        const int l = (int)gid;
        for (int64_t k = ptr[l] + sub; k < ptr[l + 1]; k += kGatherLanes) acc += g[links[k]];
    }
    for (int o = kGatherLanes / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kGatherLanes);
    if (live && sub == 0) {
        const int l = (int)gid;
        dbar[l] = accumulate ? dbar[l] + acc : acc;
    }
}

hipError_t launch_path_gather(hipStream_t s, int P, const int64_t* ptr, const int32_t* links, const double* g,
                              double* dbar, int accumulate) {
    if (P == 0) return hipSuccess;
    const int64_t threads = (int64_t)P * kGatherLanes;
    hipLaunchKernelGGL(k_path_gather, dim3((unsigned)((threads + kWG - 1) / kWG)), dim3(kWG), 0, s, P, ptr, links, g,
                       dbar, accumulate);
    return hipGetLastError();
}

// BPR cost, dc/dv and dc/dC at v (veh) in FP64, products left to right.
__device__ __forceinline__ void bpr_terms(double v, float c0f, float capf, double ab, int beta, double kappa,
                                          double& cost, double& dcdv, double& dcdcap) {
    const double c0 = (double)c0f, cap = (double)capf;
    const double r = (v * kappa) / cap;
    double p1 = 1.0;
    for (int k = 1; k < beta; ++k) p1 = p1 * r;
    const double p = p1 * r;
    cost = c0 * (1.0 + ab * p);
    dcdv = c0 * ab * (double)beta * p1 * kappa / cap;
    dcdcap = -c0 * ab * (double)beta * p / cap;
}

// Reverse step of one FW update f' = f + alpha (y - f), where alpha is the
// root of F(a) = sum_a t_a c_a(f_a + a t_a) (t = y - f): per-workgroup
// partial sums of abar = fbar . t and dF/dalpha = sum t^2 c'(v).
__global__ __launch_bounds__(kWG) void k_adj_sums(NetDev net, const int64_t* __restrict__ f,
                                                  const int64_t* __restrict__ y, const double* __restrict__ alpha,
                                                  const double* __restrict__ fbar, double ab, int beta,
                                                  double* part) {
    __shared__ double s0[kWG], s1[kWG];
    const double al = *alpha, kappa = net.inst[0].kappa;
    double a0 = 0.0, a1 = 0.0;
    for (int64_t a = blockIdx.x * (int64_t)kWG + threadIdx.x; a < net.M; a += (int64_t)gridDim.x * kWG) {
        const double F = (double)f[a] * kFxInv, t = (double)y[a] * kFxInv - F;
        double cost, dcdv, dcdcap;
        bpr_terms(F + al * t, net.c0[a], net.cap[a], ab, beta, kappa, cost, dcdv, dcdcap);
        a0 += fbar[a] * t;
        a1 += t * t * dcdv;
    }
    s0[threadIdx.x] = a0;
    s1[threadIdx.x] = a1;
    __syncthreads();
    for (int k = kWG / 2; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) {
            s0[threadIdx.x] += s0[threadIdx.x + k];
            s1[threadIdx.x] += s1[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s0[0];
        part[2 * blockIdx.x + 1] = s1[0];
    }
}

// s = -abar / (dF/dalpha) for a step size strictly inside (0, 1) that is a
// root (not the fixed MSA sequence); 0 otherwise.  One workgroup, partials
// summed in a fixed order.
__global__ __launch_bounds__(kWG) void k_adj_scale(const double* __restrict__ part, int nb,
                                                   const double* __restrict__ alpha, int is_root, double* s_out) {
    __shared__ double s0[kWG], s1[kWG];
    double a0 = 0.0, a1 = 0.0;
    for (int b = threadIdx.x; b < nb; b += kWG) {
        a0 += part[2 * b];
        a1 += part[2 * b + 1];
    }
    s0[threadIdx.x] = a0;
    s1[threadIdx.x] = a1;
    __syncthreads();
    for (int k = kWG / 2; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) {
            s0[threadIdx.x] += s0[threadIdx.x + k];
            s1[threadIdx.x] += s1[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double al = *alpha;
        *s_out = (is_root && al > 0.0 && al < 1.0 && s1[0] != 0.0) ? -s0[0] / s1[0] : 0.0;
    }
}

// Per link: ybar, and fbar and capbar carried back through the update and
// through alpha's dependence on (f, y, C) (implicit-function theorem).
__global__ __launch_bounds__(kWG) void k_adj_links(NetDev net, const int64_t* __restrict__ f,
                                                   const int64_t* __restrict__ y, const double* __restrict__ alpha,
                                                   const double* __restrict__ sp, double ab, int beta, double* fbar,
                                                   double* __restrict__ ybar, double* capbar) {
    const double al = *alpha, s = *sp, kappa = net.inst[0].kappa;
    for (int64_t a = blockIdx.x * (int64_t)kWG + threadIdx.x; a < net.M; a += (int64_t)gridDim.x * kWG) {
        const double F = (double)f[a] * kFxInv, t = (double)y[a] * kFxInv - F;
        double cost, dcdv, dcdcap;
        bpr_terms(F + al * t, net.c0[a], net.cap[a], ab, beta, kappa, cost, dcdv, dcdcap);
        const double g = fbar[a];
        ybar[a] = al * g + s * (cost + al * t * dcdv);
        fbar[a] = (1.0 - al) * g + s * (-cost + (1.0 - al) * t * dcdv);
        capbar[a] = capbar[a] + s * t * dcdcap;
    }
}

static int adj_blocks(int64_t M) {
    const int64_t b = (M + kWG - 1) / kWG;
    return b < 1 ? 1 : (b > 1024 ? 1024 : (int)b);
}

hipError_t launch_adj_step(hipStream_t s, const NetDev& net, const int64_t* f, const int64_t* y,
                           const double* alpha, int is_root, double ab, int beta, double* fbar, double* ybar,
                           double* capbar, double* part /*[2 x 1024]*/, double* sbuf) {
    if (net.M == 0) return hipSuccess;
    const int nb = adj_blocks(net.M);
    hipLaunchKernelGGL(k_adj_sums, dim3(nb), dim3(kWG), 0, s, net, f, y, alpha, fbar, ab, beta, part);
    hipLaunchKernelGGL(k_adj_scale, dim3(1), dim3(kWG), 0, s, part, nb, alpha, is_root, sbuf);
    hipLaunchKernelGGL(k_adj_links, dim3(nb), dim3(kWG), 0, s, net, f, y, alpha, sbuf, ab, beta, fbar, ybar, capbar);
    return hipGetLastError();
}

// flows in veh from fixed point
__global__ void k_fx_to_veh(int64_t M, const int64_t* __restrict__ f, double* out) {
    for (int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; a < M; a += (int64_t)gridDim.x * blockDim.x)
        out[a] = (double)f[a] * kFxInv;
}

hipError_t launch_fx_to_veh(hipStream_t s, int64_t M, const int64_t* f, double* out) {
    if (M == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fx_to_veh, dim3(adj_blocks(M)), dim3(kWG), 0, s, M, f, out);
    return hipGetLastError();
}

}  // namespace qdta
