// slice.hip -- slice sampling along a random direction (Neal 2003: stepping
// out and shrinkage, Sec. 4; a random line through x, Sec. 5.1) as the
// five-state FSM of Sec. 3.1's slice panel: INIT E, EXPAND, INIT S, SHRINK,
// DONE.  The transition function slice_next() is generated by fsmgen from
// the program "initE W[expand]{ expand } initS W[shrink]{ shrink } done"
// (slice_fsm.inc); this file supplies the five blocks and the two loop
// conditions.
//
// Draw t from x (l = log pi):
//   INIT E  ln u; d = z / |z|; L = -w u', R = L + w; evaluate both ends
//   EXPAND  step out the left end by w if it is inside the slice, else the
//           right end; evaluate it                      (while an end is inside)
//   INIT S  t ~ U(L, R), x' = x + t d, evaluate
//   SHRINK  t < 0 ? L = t : R = t; draw again, evaluate (while x' is outside)
//   DONE    x = x', emit
// A point is inside the slice when l(p) - l(x) > ln u (the difference form
// of l(p) > l(x) + ln u: the sum can round onto l(x) in FP32, and a bracket
// collapsing onto x would then never be accepted).  The loop count N_ij is
// the number of density evaluations.  Guard: after 10^4 evaluations the
// draw ends with x kept (counted; expected never).
//
// One lane per chain (D <= 16): x, d and the scalars live in registers; state
// in HBM is [field][d][chain] / [field][chain].  One FSM step runs the chain's
// block and follows the generated transition, with DONE bundled into the step
// that accepts (it is cheap).  EXPAND, INIT S and SHRINK share one body (choose
// a position on the line, evaluate it, update): lanes in different ones of
// these states run together instead of one after another.
//
// What a draw needs that depends on (chain, draw) only -- its direction, ln u,
// the first interval's and the first point's uniforms -- is drawn ahead for a
// window of W draws of every chain by a kernel of its own (sl_dir_kernel, all
// lanes active) and read from there; only SHRINK draws its angles in the loop.
// Both runtimes read the same window, so they give the same bits.  The FSM
// runtime runs the chains window by window (a chain stops at the end of its
// window; the next window starts from every chain's own draw index).
//
// What bounds the FSM kernel: the serial chain of a step (position, point,
// density, comparison: about 300 vector instructions) and chains that wait for
// the slowest one of their wave.  Against one chain per lane with a body per
// state, all draws in the loop and windows of 32 draws: 1024 chains x 500 draws
// at D = 10 25.3 -> 6.9 ms.
#include "dr_device.h"
#include "slice_fsm.inc"

namespace fsmmc {

struct SlK {
    DrK pd;  // density parameters (target, D, prec) and the counters
    int m, n, D;
    uint32_t tstop;
    uint64_t seed;
    float w;
    float* x;              // [d][chain]
    float *lx, *L, *R, *tt;  // [chain]
    int32_t *k, *flags, *evals, *ns, *ne;
    uint32_t* t;
    int64_t* budget;
    float* out;
    int32_t* counts;
    unsigned long long* ctr;
    int32_t* maxN;  // [2][n]: largest expansion and shrink counts of each draw
    int32_t* ecur;  // [chain]: expansions of the draw just finished (synchronized runtime)
    float* sink;
    float* dirw;            // [chain][W][D + 3]: draws tsnap .. tsnap + W - 1 (SlAhead)
    const uint32_t* tsnap;  // [chain]: first draw of the chain's window
    int W;
    int lpw;  // chains per wave of the FSM kernel (lanes lpw .. 63 idle)
};

// The chain of this thread in the FSM kernel, blocks of one wave (m: none).
__device__ __forceinline__ int lane_chain(int lpw, int m)
{
    const int lane = threadIdx.x, c = (int)blockIdx.x * lpw + lane;
    return lane < lpw && c < m ? c : m;
}

enum SliceFlags { SF_INL = 1, SF_INR = 2, SF_ACC = 4, SF_GUARD = 8 };

template <int NM>
struct SlLane {
    float x[NM], dir[NM];
    float lx, lnu, L, R, tt, u1;
    int k, fl, evals, s, e;
    uint32_t t;
    // the loop conditions the generated transition function asks for
    __device__ bool expand() const { return (fl & (SF_INL | SF_INR)) && !(fl & SF_GUARD); }
    __device__ bool shrink() const { return !(fl & SF_ACC) && !(fl & SF_GUARD); }
};

// What a draw reads from the window: direction, then ln u, the interval's
// uniform, the first point's uniform.
template <int NM>
struct SlAhead {
    float dir[NM], lnu, u0, u1;
};

template <int NM>
__device__ __forceinline__ void sl_ahead(const SlK& a, int c, uint32_t t, uint32_t tsnap, SlAhead<NM>& A)
{
    // past the window's last draw nothing is used of it
    const float* p = a.dirw + ((size_t)c * a.W + min(t - tsnap, (uint32_t)(a.W - 1))) * (a.D + 3);
#pragma unroll
    for (int d = 0; d < NM; ++d) A.dir[d] = d < a.D ? p[d] : 0.0f;
    A.lnu = p[a.D];
    A.u0 = p[a.D + 1];
    A.u1 = p[a.D + 2];
}

template <int NM>
__device__ __forceinline__ void sl_take(const SlAhead<NM>& A, SlLane<NM>& L)
{
#pragma unroll
    for (int d = 0; d < NM; ++d) L.dir[d] = A.dir[d];
    L.lnu = A.lnu;
    L.u1 = A.u1;
}

// The chain's state; the draw in progress, if any, reads its part of the
// window again (A), and the next INIT E the same.
template <int NM>
__device__ __forceinline__ void sl_load(const SlK& a, int c, SlLane<NM>& L, SlAhead<NM>& A)
{
#pragma unroll
    for (int d = 0; d < NM; ++d) L.x[d] = d < a.D ? a.x[(size_t)d * a.m + c] : 0.0f;
    L.lx = a.lx[c];
    L.L = a.L[c];
    L.R = a.R[c];
    L.tt = a.tt[c];
    L.k = a.k[c];
    L.fl = a.flags[c];
    L.evals = a.evals[c];
    L.s = a.ns[c];
    L.e = a.ne[c];
    L.t = a.t[c];
    sl_ahead<NM>(a, c, L.t, a.tsnap[c], A);
    sl_take<NM>(A, L);
    if (L.k != SLICE_INITE) sl_ahead<NM>(a, c, L.t + 1, a.tsnap[c], A);
}

template <int NM>
__device__ __forceinline__ void sl_store(const SlK& a, int c, const SlLane<NM>& L)
{
#pragma unroll
    for (int d = 0; d < NM; ++d)
        if (d < a.D) a.x[(size_t)d * a.m + c] = L.x[d];
    a.lx[c] = L.lx;
    a.L[c] = L.L;
    a.R[c] = L.R;
    a.tt[c] = L.tt;
    a.k[c] = L.k;
    a.flags[c] = L.fl;
    a.evals[c] = L.evals;
    a.ns[c] = L.s;
    a.ne[c] = L.e;
    a.t[c] = L.t;
}

// l(x + s d) into v, returned; one density evaluation.
template <int NM>
__device__ __forceinline__ float sl_eval(const SlK& a, const SlLane<NM>& L, float s, float* v)
{
#pragma unroll
    for (int d = 0; d < NM; ++d) v[d] = d < a.D ? L.x[d] + s * L.dir[d] : 0.0f;
    return dr_logpdf<NM>(a.pd, v);
}

template <int NM>
__device__ __forceinline__ bool sl_inside(const SlK& a, const SlLane<NM>& L, float s)
{
    float v[NM];
    return sl_eval<NM>(a, L, s, v) - L.lx > L.lnu;
}

// The random direction of draw t of chain c: z / |z|, z = D normals of the NU
// stream (written to out[0 .. D)).
template <int NM>
__device__ __forceinline__ void sl_direction(uint64_t seed, int D, int c, uint32_t t, float* out)
{
    float v[NM];
#pragma unroll
    for (int b = 0; b < NM / 4; ++b) {
        float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (4 * b < D) normals4<float>(seed, (uint32_t)c, t, ROLE_NU, 0, (uint32_t)b, z);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int d = 4 * b + i;
            v[d] = d < D ? z[i] : 0.0f;
        }
    }
    float nn = 0.0f;
#pragma unroll
    for (int d = 0; d < NM; ++d) nn += v[d] * v[d];
    const float inv = 1.0f / sqrtf(nn);
#pragma unroll
    for (int d = 0; d < NM; ++d)
        if (d < D) out[d] = v[d] * inv;
}

// INIT E, and the loads of the next draw's part of the window.
template <int NM>
__device__ __forceinline__ void sl_init_e(const SlK& a, int c, uint32_t tsnap, SlLane<NM>& L, SlAhead<NM>& A)
{
    sl_take<NM>(A, L);
    L.L = -a.w * A.u0;
    L.R = L.L + a.w;
    sl_ahead<NM>(a, c, L.t + 1, tsnap, A);
    L.fl = (sl_inside<NM>(a, L, L.L) ? SF_INL : 0) | (sl_inside<NM>(a, L, L.R) ? SF_INR : 0);
    L.evals = 2;
    L.s = 0;
    L.e = 0;
    L.k = slice_next(SLICE_INITE, L);
}

template <int NM>
__device__ __forceinline__ void sl_done(const SlK& a, int c, SlLane<NM>& L, const float* xb, float lp)
{
    if (!(L.fl & SF_GUARD)) {
#pragma unroll
        for (int d = 0; d < NM; ++d) L.x[d] = xb[d];
        L.lx = lp;
    }
    float* o = a.out + ((size_t)c * a.n + L.t) * a.D;
#pragma unroll
    for (int d = 0; d < NM; ++d)
        if (d < a.D) o[d] = L.x[d];
    a.counts[(size_t)c * a.n + L.t] = L.evals;
    L.t += 1;
}

// EXPAND (step the left end out if it is inside the slice, else the right
// end), INIT S or SHRINK (a point on [L, R]): a position, its density, the
// update.  A step that reaches DONE runs it too.  Returns 1 when the step
// ended a draw (and sets *guard if the evaluation guard stopped it).
template <int NM>
__device__ __forceinline__ int sl_walk(const SlK& a, int c, SlLane<NM>& L, int* guard)
{
    const bool grow = L.k == SLICE_EXPAND, shrink = L.k == SLICE_SHRINK;
    const bool left = grow ? (L.fl & SF_INL) != 0 : shrink && L.tt < 0.0f;  // the end that moves
    const bool stop = L.evals >= kEssMaxEvals;
    if (shrink) {
        L.L = left ? L.tt : L.L;
        L.R = left ? L.R : L.tt;
        L.s += 1;
    }
    float pos;
    if (grow) {
        pos = left ? L.L - a.w : L.R + a.w;
        if (!stop) {
            L.L = left ? pos : L.L;
            L.R = left ? L.R : pos;
        }
    } else {
        float u = L.u1;
        if (shrink) u = uniform<float>(a.seed, (uint32_t)c, L.t, ROLE_ANGLE, (uint32_t)(1 + L.s));
        pos = L.L + (L.R - L.L) * u;
        if (!stop) L.tt = pos;
    }
    float v[NM];
    const float lp = sl_eval<NM>(a, L, pos, v);
    const int bit = grow ? (left ? SF_INL : SF_INR) : SF_ACC;
    const int hit = lp - L.lx > L.lnu ? bit : 0;
    L.fl = stop ? L.fl | SF_GUARD : (L.fl & ~bit) | hit;
    L.evals += stop ? 0 : 1;
    L.e += grow && !stop ? 1 : 0;
    L.k = slice_next(L.k, L);
    if (L.k != SLICE_DONE) return 0;
    *guard = (L.fl & SF_GUARD) ? 1 : 0;
    sl_done<NM>(a, c, L, v, lp);
    L.k = slice_next(SLICE_DONE, L);
    return 1;
}

// One FSM step: the chain's block, then the generated transition.
template <int NM>
__device__ __forceinline__ int sl_step(const SlK& a, int c, uint32_t tsnap, SlLane<NM>& L, SlAhead<NM>& A, int* guard)
{
    if (L.k == SLICE_INITE) {
        sl_init_e<NM>(a, c, tsnap, L, A);
        return 0;
    }
    return sl_walk<NM>(a, c, L, guard);
}

// The window's entries of the next W draws of every chain (thread per chain and slot);
// the window starts at the chain's current draw index, recorded in tsnap.
template <int NM>
__global__ __launch_bounds__(256) void sl_dir_kernel(SlK a, uint32_t* tsnap)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)a.m * a.W) return;
    const int c = (int)(i / a.W), w = (int)(i % a.W);
    const uint32_t t0 = a.t[c];
    if (w == 0) tsnap[c] = t0;
    const uint32_t t = t0 + (uint32_t)w;
    if (t >= (uint32_t)a.n) return;
    float* o = a.dirw + i * (a.D + 3);
    sl_direction<NM>(a.seed, a.D, c, t, o);
    o[a.D] = logf(uniform<float>(a.seed, (uint32_t)c, t, ROLE_THRESH, 0));
    o[a.D + 1] = uniform<float>(a.seed, (uint32_t)c, t, ROLE_ANGLE, 0);
    o[a.D + 2] = uniform<float>(a.seed, (uint32_t)c, t, ROLE_ANGLE, 1);
}

// FSM runtime, one window: every lane runs its chain to the end of its
// window (or n, or its budget).  ctr[3] counts chains that can go on (short
// of n with budget left), ctr[4] chains short of n.
template <int D>
__global__ __launch_bounds__(64) void sl_fsm_kernel(SlK a)
{
    constexpr int NM = D;  // the dimension itself: no masks, no idle elements
    a.D = a.pd.D = D;
    __shared__ unsigned long long s_sum;
    const int c = lane_chain(a.lpw, a.m);
    uint32_t steps = 0, live = 0, guards = 0, more = 0, iters = 0;
    if (c < a.m) {
        SlLane<NM> L;
        SlAhead<NM> A;
        sl_load<NM>(a, c, L, A);
        int64_t budget = a.budget[c];
        const uint32_t tsnap = a.tsnap[c];
        const uint32_t stop = min(min(a.tstop, (uint32_t)a.n), tsnap + (uint32_t)a.W);
        for (;;) {
            // the body most chains of the wave wait for (INIT E or the walk)
            const bool go = L.t < stop && budget > 0;
            const int ni = __popcll(__ballot(go && L.k == SLICE_INITE)), nw = __popcll(__ballot(go && L.k != SLICE_INITE));
            if (ni + nw == 0) break;
            ++iters;
            if (ni >= nw) {
                if (go && L.k == SLICE_INITE) {
                    sl_init_e<NM>(a, c, tsnap, L, A);
                    ++steps;
                    --budget;
                }
            } else if (go && L.k != SLICE_INITE) {
                int g = 0;
                (void)sl_walk<NM>(a, c, L, &g);
                guards += (uint32_t)g;
                ++steps;
                --budget;
            }
        }
        sl_store<NM>(a, c, L);
        a.budget[c] = budget;
        live = L.t < (uint32_t)a.n ? 1u : 0u;
        more = (L.t < min(a.tstop, (uint32_t)a.n) && budget > 0) ? 1u : 0u;
    }
    const unsigned long long st = block_sum_u64(wave_sum_u64(steps), &s_sum);
    if (threadIdx.x == 0 && st) atomicAdd(&a.ctr[0], st);
    const unsigned long long lv = block_sum_u64(wave_sum_u64(live), &s_sum);
    if (threadIdx.x == 0 && lv) atomicAdd(&a.ctr[4], lv);
    const unsigned long long mo = block_sum_u64(wave_sum_u64(more), &s_sum);
    if (threadIdx.x == 0 && mo) atomicAdd(&a.ctr[3], mo);
    const unsigned long long gd = block_sum_u64(wave_sum_u64(guards), &s_sum);
    if (threadIdx.x == 0 && gd) atomicAdd(&a.ctr[2], gd);
    dr_count_lanes(a.pd, steps, iters, &s_sum);
}

// Synchronized runtime: draw `draw` of every chain; the draw's largest
// expansion and shrink counts go to maxN[0][draw] and maxN[1][draw], the
// chain's own expansion count to ecur.
template <int NM>
__global__ __launch_bounds__(256) void sl_sync_kernel(SlK a, uint32_t draw)
{
    __shared__ unsigned long long s_sum;
    __shared__ int s_max;
    const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    uint32_t steps = 0, guards = 0;
    int ne = 0, ns = 0;
    if (c < a.m) {
        SlLane<NM> L;
        SlAhead<NM> A;
        sl_load<NM>(a, c, L, A);
        const uint32_t tsnap = a.tsnap[c];
        while (L.t <= draw) {
            int g = 0;
            if (sl_step<NM>(a, c, tsnap, L, A, &g)) {
                ne = L.e;
                ns = L.s;
            }
            guards += (uint32_t)g;
            ++steps;
        }
        sl_store<NM>(a, c, L);
        a.ecur[c] = ne;
    }
    const int me = block_max_i32(wave_max_i32(ne), &s_max);
    if (threadIdx.x == 0) atomicMax(&a.maxN[draw], me);
    const int ms = block_max_i32(wave_max_i32(ns), &s_max);
    if (threadIdx.x == 0) atomicMax(&a.maxN[a.n + draw], ms);
    const unsigned long long st = block_sum_u64(wave_sum_u64(steps), &s_sum);
    if (threadIdx.x == 0 && st) atomicAdd(&a.ctr[0], st);
    const unsigned long long gd = block_sum_u64(wave_sum_u64(guards), &s_sum);
    if (threadIdx.x == 0 && gd) atomicAdd(&a.ctr[2], gd);
    dr_count_lanes(a.pd, steps, steps, &s_sum);
}

// vmap padding of draw `draw`: the two batched while loops run max_j e_j
// expansions and max_j s_j shrinks; chain c computes and discards the
// (max e - e_c) + (max s - s_c) density evaluations it would have been masked
// through.
template <int NM>
__global__ __launch_bounds__(256) void sl_pad_kernel(SlK a, uint32_t draw)
{
    __shared__ unsigned long long s_sum;
    const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    int extra = 0;
    if (c < a.m) {
        const int e = a.ecur[c];
        const int s = a.counts[(size_t)c * a.n + draw] - 3 - e;  // evaluations = 2 + e + 1 + s
        extra = max(a.maxN[draw] - e, 0) + max(a.maxN[a.n + draw] - s, 0);
        if (extra > 0) {
            SlLane<NM> L;
            SlAhead<NM> A;
            sl_load<NM>(a, c, L, A);
            float v[NM], acc = 0.0f;
            for (int i = 0; i < extra; ++i) acc += sl_eval<NM>(a, L, L.R + (float)i * a.w, v);
            a.sink[c] = acc;
        }
    }
    const unsigned long long tot = block_sum_u64(wave_sum_u64((unsigned long long)extra), &s_sum);
    if (threadIdx.x == 0 && tot) atomicAdd(&a.ctr[1], tot);
    dr_count_lanes(a.pd, 0u, (uint32_t)extra, &s_sum);
}

// ------------------------------------------------------------ host side
// Chains per wave of the FSM kernel: the smallest power of two, up to 64, that
// leaves at most 256 waves, one per CU -- with fewer chains a wave waits less for its
// slowest one and skips more bodies, but waves that share a CU mostly slow each
// other down.  The rule gives the best column of each row but the third, where it
// takes 16 chains (5.76): one chain a wave, 16 waves a CU, is faster there and was not
// measured at other sizes, nor is it known why 4 is slower than both.  ms a job, D =
// 10, by chains per wave:
//   chains x draws    64     16     4      1
//    256 x 500       7.85   7.08   6.26   5.39
//   1024 x 500       8.42   8.05   6.78   8.20
//   4096 x 300       6.10   5.76   6.73   5.04
//   65536 x 200 (D = 16)  8.09  10.7  18.0
static int sl_chains_per_wave(int m)
{
    int l = 1;
    while (l < 64 && (m + l - 1) / l > 256) l *= 2;
    return l;
}

static SlK sl_view(const JobDev& j)
{
    SlK a;
    a.pd = dr_view(j);
    a.m = j.m;
    a.n = j.n;
    a.D = j.D;
    a.tstop = j.tstop;
    a.seed = j.seed;
    a.w = (float)j.scales[0];
    a.x = (float*)j.x;
    a.lx = (float*)j.lx;
    a.L = (float*)j.tmin;
    a.R = (float*)j.tmax;
    a.tt = (float*)j.theta;
    a.k = j.k;
    a.flags = j.flags;
    a.evals = j.evals;
    a.ns = j.nn;
    a.ne = j.jd;
    a.t = j.t;
    a.budget = j.budget;
    a.out = (float*)j.out;
    a.counts = j.counts;
    a.ctr = j.ctr;
    a.maxN = j.maxN;
    a.ecur = j.vdir;
    a.sink = (float*)j.sink;
    a.dirw = (float*)j.nu;
    a.tsnap = j.tsnap;
    a.W = j.W;
    a.lpw = sl_chains_per_wave(j.m);
    return a;
}

hipError_t sl_init_state(const JobDev& j, const void* x0, hipStream_t s)
{
    // x in [d][chain] and log pi(x) (funnel: exact draw; otherwise N(0, I)); k = INIT E
    return dr_init_state(j, x0, s);
}

#define FSMMC_SL_DISPATCH(KERNEL, D_, ...)                                           \
    if ((D_) <= 4)                                                                 \
        hipLaunchKernelGGL(KERNEL<4>, __VA_ARGS__);                                \
    else if ((D_) <= 8)                                                            \
        hipLaunchKernelGGL(KERNEL<8>, __VA_ARGS__);                                \
    else if ((D_) <= 12)                                                           \
        hipLaunchKernelGGL(KERNEL<12>, __VA_ARGS__);                               \
    else                                                                           \
        hipLaunchKernelGGL(KERNEL<16>, __VA_ARGS__);

hipError_t sl_dir_window(const JobDev& j, hipStream_t s)
{
    const SlK a = sl_view(j);
    const size_t tot = (size_t)j.m * j.W;
    FSMMC_SL_DISPATCH(sl_dir_kernel, j.D, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, a, j.tsnap)
    return hipGetLastError();
}

hipError_t sl_fsm_round(const JobDev& j, hipStream_t s)
{
    const SlK a = sl_view(j);
#define FSMMC_SL_FSM(D) \
    case D: hipLaunchKernelGGL(sl_fsm_kernel<D>, dim3((j.m + a.lpw - 1) / a.lpw), dim3(64), 0, s, a); break;
    switch (j.D) {
        FSMMC_SL_FSM(1) FSMMC_SL_FSM(2) FSMMC_SL_FSM(3) FSMMC_SL_FSM(4) FSMMC_SL_FSM(5) FSMMC_SL_FSM(6)
        FSMMC_SL_FSM(7) FSMMC_SL_FSM(8) FSMMC_SL_FSM(9) FSMMC_SL_FSM(10) FSMMC_SL_FSM(11) FSMMC_SL_FSM(12)
        FSMMC_SL_FSM(13) FSMMC_SL_FSM(14) FSMMC_SL_FSM(15) FSMMC_SL_FSM(16)
    default: return hipErrorInvalidValue;
    }
#undef FSMMC_SL_FSM
    return hipGetLastError();
}

hipError_t sl_sync_draw(const JobDev& j, uint32_t draw, hipStream_t s)
{
    const SlK a = sl_view(j);
    FSMMC_SL_DISPATCH(sl_sync_kernel, j.D, dim3((j.m + 255) / 256), dim3(256), 0, s, a, draw)
    return hipGetLastError();
}

hipError_t sl_pad_draw(const JobDev& j, uint32_t draw, hipStream_t s)
{
    const SlK a = sl_view(j);
    FSMMC_SL_DISPATCH(sl_pad_kernel, j.D, dim3((j.m + 255) / 256), dim3(256), 0, s, a, draw)
    return hipGetLastError();
}

}  // namespace fsmmc
