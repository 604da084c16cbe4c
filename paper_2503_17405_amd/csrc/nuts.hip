// nuts.hip -- the no-U-turn sampler (Hoffman & Gelman 2014) as an FSM
// (Sec. 3.1, Fig. "Finite state machines ...", HMC-NUTS panel: INIT, DOUBLE,
// INTEGRATE, CHECK, DONE; Sec. 7.3: iterative form, an outer doubling loop
// and an inner integration loop), for Bayesian logistic regression.
//
// One runtime step for every chain:
//   1. nuts_fsm_step_kernel (one wavefront per chain): add up the row-slice
//      partials of the gradient that just arrived, in slice order
//      (grad U = theta - X^T r, U = |theta|^2 / 2 - loglik), finish that
//      leapfrog (second half-kick, multinomial leaf choice, U-turn
//      checkpoints), then run the cheap states back to back (CHECK, DONE,
//      INIT, DOUBLE) until the chain needs the next gradient, and issue the
//      first half of that leapfrog (Appendix, Alg. "bundled step as input to
//      amortized step").  Each block appends its requesters to the step's list.
//   2. logreg_grad_bf16_kernel: eta = X Theta, r = y - sigmoid(eta), X^T r
//      and the log-likelihood, fused for a tile of 128 listed chains and a
//      slice of rows on the bf16 matrix cores (exact three-piece splits of
//      the FP32 operands, FP32 results); eta never leaves registers.
// The synchronized runtime runs the same step (nuts_step_kernel) and lists its
// requesters in chain order with a kernel of their own (nuts_compact_kernel); a
// chain that finishes a draw waits until every chain has finished it
// (device-side barrier), and in vmap mode the gradient phase then covers every
// chain.
// Readings: multinomial leaf sampling inside a subtree, biased progressive
// merge of subtrees, generalized U-turn criterion on every aligned sub-span,
// divergence when H - H0 > 1000, identity mass.
#include "nuts_block.h"
#include <algorithm>

namespace fsmmc {

// FSM runtime: NW chains per block, their requests appended to the list (slot
// step mod 3; the next step's slot is cleared here).  Bound by latency at few
// chains (one round trip for the state, then a serial chain of vector work) and
// by the state's bytes at many.  A list built by a kernel of its own cost 2.1 us
// and a launch gap per step at 16 chains, 5.2 us at 4096: 16 chains (N = 1000,
// D = 10, 200 draws, depth 10) 31.6 -> 27.8 ms, 4096 chains (N = 10^4, D = 100)
// 4.5% faster.
template <int EPL, int NW, bool AHEAD>
__global__ __launch_bounds__(64 * NW) void nuts_fsm_step_kernel(NutsK a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = (int)(blockIdx.x * NW) + wave;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.rcnt[(a.step + 1) % 3] = 0u;
    int bits = 0;
    if (c < a.m) bits = nuts_chain_step<EPL, AHEAD>(a, c, lane);
    nuts_append<NW>(a, c, wave, bits, (int)(a.step % 3));
}

template <int EPL>
__global__ __launch_bounds__(256) void nuts_step_kernel(NutsK a)
{
    const int lane = threadIdx.x & 63;
    const int c = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.wctr[(a.step + 1) % 3] = 0u;
        a.wctr[3 + (a.step + 1) % 3] = 0u;
    }
    int bits = 0;
    if (c < a.m) bits = nuts_chain_step<EPL>(a, SliceGrad{a}, c, lane);
    // chains alive / still inside their draw, one atomic per block
    __shared__ unsigned s_alive, s_indraw;
    if (threadIdx.x == 0) {
        s_alive = 0;
        s_indraw = 0;
    }
    __syncthreads();
    if (lane == 0 && bits) {
        atomicAdd(&s_alive, (bits & NC_ALIVE) ? 1u : 0u);
        atomicAdd(&s_indraw, (bits & NC_INDRAW) ? 1u : 0u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_alive) atomicAdd(&a.wctr[3 + a.step % 3], s_alive);
        if (s_indraw) atomicAdd(&a.wctr[a.step % 3], s_indraw);
    }
}

// Finishes the leapfrogs that wait for their gradient, as the next step would, and
// asks for none: the chains stop before their next leapfrog.
template <int EPL>
__global__ __launch_bounds__(256) void nuts_settle_kernel(NutsK a)
{
    const int lane = threadIdx.x & 63, c = uni((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (c >= a.m) return;
    NutsScal S = nuts_load(a, c, uni(a.t[c]));
    if (S.t >= a.tstop || !(S.fl & NF_PENDING)) return;
    float* Vc = a.V + (size_t)c * a.nvec * a.Dp;
    NutsBox<EPL, BOX_MEMORY> box(Vc, a.Dp, lane, Vc + (size_t)V_FIXED * a.Dp);
    const int64_t budget = S.budget;
    S.budget = 0;
    (void)nuts_chain_body<EPL, SliceGrad>(a, SliceGrad{a}, c, lane, S, box);
    S.budget = budget;
    nuts_store(a, c, S, 0, lane);
}

__global__ __launch_bounds__(1024) void nuts_compact_kernel(const int32_t* req, int m, int vmap, int32_t* list,
                                                            int32_t* count, unsigned long long* ctr)
{
    nuts_compact_block<1024>(req, m, vmap, list, count, ctr);
}

// Default start: theta0 ~ N(0, I) from the INIT stream (into both buffers).
__global__ void nuts_normal_init_kernel(float* thp, int vstride, float* thq, int m, int D, int Dp, uint64_t seed)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)m * Dp) return;
    const int c = (int)(i / Dp), d = (int)(i % Dp);
    const float z = d < D ? normal_at<float>(seed, (uint32_t)c, 0, ROLE_INIT, 0, (uint32_t)d) : 0.0f;
    thp[(size_t)c * vstride + d] = z;
    thq[(size_t)c * Dp + d] = z;
}

// ------------------------------------------------------------ host side
int nuts_nvec(int max_depth) { return V_FIXED + 2 * max_depth; }

hipError_t nuts_init_state(const JobDev& j, const void* x0, hipStream_t s)
{
    float* thp = (float*)j.V + (size_t)V_THP * j.Dp;
    const int vstride = j.nvec * j.Dp;
    if (x0) {
        hipError_t e = hipMemcpy2DAsync(thp, (size_t)vstride * 4, x0, (size_t)j.D * 4, (size_t)j.D * 4, j.m,
                                        hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        e = hipMemcpy2DAsync(j.Thq, (size_t)j.Dp * 4, x0, (size_t)j.D * 4, (size_t)j.D * 4, j.m,
                             hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    } else {
        const size_t tot = (size_t)j.m * j.Dp;
        hipLaunchKernelGGL(nuts_normal_init_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, thp,
                           vstride, (float*)j.Thq, j.m, j.D, j.Dp, j.seed);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // grad U and U at the start, straight into the proposal slots (gP, UP)
    float* gp = (float*)j.V + (size_t)V_GP * j.Dp;
    return nuts_gradient_dense(j, j.m, gp, (float*)j.lx, vstride, j.Dp, s);
}

template <int EPL, int NW, bool AHEAD>
static void fsm_step_launch(const NutsK& a, hipStream_t s)
{
    hipLaunchKernelGGL((nuts_fsm_step_kernel<EPL, NW, AHEAD>), dim3((a.m + NW - 1) / NW), dim3(64 * NW), 0, s, a);
}

// Four chains per block up to 1024 chains (every block has a CU to itself),
// eight above, where the blocks' atomics on the one count cost more than the
// wait for a block's slowest chain.  Vectors and 32 slices ahead up to 2048
// chains: 46 chains, N = 8000, D = 50 (250 slices) 6.0 -> 4.8 ms, N = 5379, D = 83
// (169 slices) 47 -> 40 ms; at 65536 chains the vectors' extra reads cost 16.0 ->
// 16.6 ms at D = 20, 42.2 -> 50.2 at D = 100.
template <int EPL>
static void fsm_step(const NutsK& a, hipStream_t s)
{
    if (a.m <= 1024)
        fsm_step_launch<EPL, 4, true>(a, s);
    else if (a.m <= 2048)
        fsm_step_launch<EPL, 8, true>(a, s);
    else
        fsm_step_launch<EPL, 8, false>(a, s);
}

template <int NK32, int NT, int R>
__global__ __launch_bounds__(64 * kNutsBlockWaves) void nuts_block_kernel(NutsK a, GradK g, int G, int K)
{
    extern __shared__ __align__(16) unsigned char lds[];
    if (blockIdx.x == 0 && threadIdx.x == 0) a.rcnt[(a.step + 1) % 3] = 0u;
    nuts_block_run<NK32, NT, R>(a, g, (int)blockIdx.x * G, G, K, lds, a.rcnt + a.step % 3);
}

// Chains per block of the block kernel, or 0: the job runs a launch per step.
// `chains` compete for the 256 compute units: as few per block as give every unit
// one, at most 8, then several rounds of blocks.  A step's cost in cycles is the
// transition (6000) and per 32-row chunk the 6 k-step and 3 d-tile KiB that each
// unit reads at 64 bytes a cycle, against 20 us or so for a step of two launches.
// Below the line at 40000: 16 chains, N = 1000, D = 10 (one round, 10600): 6.1 ->
// 1.8 ms for 40 draws; 4096 chains, N = 2000, D = 20 (two rounds, 36200): 3.9 ->
// 2.8; 4096, N = 1000, D = 50 (36600): 6.3 -> 5.5.  Above: N = 8000, D = 20 (54000):
// 16 chains 5.9 -> 4.8 but 256 chains 2.75 -> 3.2; N = 4000, D = 50 (54000): 8.4 ->
// 9.9; 16384 chains, N = 1000, D = 10 (eight rounds, 85000): 4.3 -> 7.5.
int nuts_block_chains(const JobDev& j, int64_t chains)
{
    if (j.EPL != 1) return 0;
    const int nt = nuts_block_class(j.D), nk32 = (nt + 1) / 2, chunks = (j.N + 31) / 32;
    const int64_t G = std::min<int64_t>(kNutsBlockWaves, (chains + 255) / 256);
    const int64_t rounds = (chains + 256 * G - 1) / (256 * G);
    if (rounds * (6000 + (int64_t)chunks * 48 * (2 * nk32 + nt)) > 40000) return 0;
    return nuts_block_lds((int)G, j.nslices, nt, j.max_depth).bytes <= kNutsBlockLds ? (int)G : 0;
}

constexpr int kNutsHeld = 4;
// Whether the waves' shares of X fit their registers.
static bool nuts_block_held(const JobDev& j, int G)
{
    int lgp = 0;
    while ((1 << lgp) < G) ++lgp;
    const int per = (j.nslices + kNutsBlockWaves - 1) / kNutsBlockWaves;
    return j.slice_rows == 32 && per <= kNutsHeld && per <= (16 >> lgp);
}

template <int NK32, int NT, int R>
static hipError_t block_launch(const JobDev& j, const NutsK& a, int G, int K, hipStream_t s, bool setup)
{
    const void* f = (const void*)nuts_block_kernel<NK32, NT, R>;
    if (setup) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kNutsBlockLds);
    hipLaunchKernelGGL((nuts_block_kernel<NK32, NT, R>), dim3((j.m + G - 1) / G), dim3(64 * kNutsBlockWaves),
                       nuts_block_lds(G, j.nslices, NT, j.max_depth).bytes, s, a, grad_view(j, 0), G, K);
    return hipGetLastError();
}

static hipError_t block_dispatch(const JobDev& j, const NutsK& a, int G, int K, hipStream_t s, bool setup)
{
    switch (nuts_block_class(j.D)) {
    case 1:
        if (nuts_block_held(j, G)) return block_launch<1, 1, kNutsHeld>(j, a, G, K, s, setup);
        return block_launch<1, 1, 0>(j, a, G, K, s, setup);
    case 2: return block_launch<1, 2, 0>(j, a, G, K, s, setup);
    case 3: return block_launch<2, 3, 0>(j, a, G, K, s, setup);
    default: return block_launch<2, 4, 0>(j, a, G, K, s, setup);
    }
}

hipError_t nuts_block_setup(const JobDev& j) { return block_dispatch(j, NutsK{}, nuts_block_chains(j, j.m), 0, nullptr, true); }

hipError_t nuts_block_steps(const JobDev& j, int G, int K, uint32_t step, hipStream_t s)
{
    return block_dispatch(j, nuts_view(j, 0, step), G, K, s, false);
}

hipError_t nuts_settle(const JobDev& j, hipStream_t s)
{
    const NutsK a = nuts_view(j, 0, 0);
    const dim3 grid((j.m + 3) / 4), block(256);
    if (j.Dp <= 64)
        hipLaunchKernelGGL(nuts_settle_kernel<1>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(nuts_settle_kernel<2>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t nuts_transition(const JobDev& j, int mode, uint32_t step, hipStream_t s)
{
    NutsK a = nuts_view(j, mode, step);
    if (mode == 0) {
        if (j.Dp <= 64)
            fsm_step<1>(a, s);
        else
            fsm_step<2>(a, s);
        return hipGetLastError();
    }
    const dim3 grid((j.m + 3) / 4), block(256);
    if (j.Dp <= 64)
        hipLaunchKernelGGL(nuts_step_kernel<1>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(nuts_step_kernel<2>, grid, block, 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(nuts_compact_kernel, dim3(1), dim3(1024), 0, s, j.req, j.m, mode == 1 ? 1 : 0, j.list, j.count,
                       j.ctr);
    return hipGetLastError();
}

}  // namespace fsmmc
