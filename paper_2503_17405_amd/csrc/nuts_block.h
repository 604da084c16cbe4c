// nuts_block.h -- NUTS on Bayesian logistic regression with a block's chains kept
// in its wavefronts and their gradients computed by the block itself, for jobs
// whose rows one compute unit goes through quickly (nuts_block_chains in nuts.hip).
// Shared by the single-job kernel (nuts.hip) and the grouped one (batch.hip).
//
// One block of 8 waves holds G <= 8 chains, chain g in the registers of wave g.
// A step is the transition of nuts_device.h (waves g < G), the positions' bf16
// pieces into LDS, a barrier, the gradient over all rows of the job by the 8
// waves, a barrier.  Against one launch per transition and one per gradient this
// takes out the launches, the state's round trips through memory and the wait
// of every chain for the slowest block.  16 chains, N = 1000, D = 10: 19.5 -> 4.8 us
// per step (200 draws: 27.7 -> 7.1 ms); a mixed batch with 128 chains, N = 2000,
// D = 20: 16.0 -> 13.4 ms.  A step is now the transition, one wave's serial vector
// work (2.3 us), and the gradient, bound by the reads of X (64 bytes a cycle) or,
// with X held, by the matrix cores and the residuals (2 us).
//
// The gradient gives logreg_grad_tile's bits.  There a column of a matrix-core
// tile is a chain and a block a row slice; a column's result depends on that
// column alone.  Here the 16 columns are Gp = 2^ceil(log2 G) chains times 16 / Gp
// row slices: a wave takes `spw` slices at once, keeps of each slice's product the
// slice's own columns, and so forms the residuals of all its slices in one
// pass of vector work.  Within a slice the chunks, the k steps
// and the piece products keep their order, and the transition adds the slices in
// slice order.
//
// State between launches is that of the launch-per-step path (a pending chain's
// slice partials in Gpart and Upart, its position in Thq), so a job may go from
// one to the other between any two launches.
#pragma once
#include "logreg_device.h"
#include "nuts_device.h"

namespace fsmmc {

constexpr int kNutsBlockWaves = 8;
constexpr int kNutsBlockLds = 150 * 1024;  // at most

// Kernel class of a dimension up to 64: d tiles of 16 (the k steps of 32 follow).
__host__ __device__ inline int nuts_block_class(int D) { return (D + 15) / 16; }

// LDS of a block (bytes), Dp = 64: position pieces [3][8][64], request flags,
// slice sums [G][nslices rounded up to 8][16 NT + 4] (X^T r, loglik) and eight rows
// more (BlockGrad reads ahead), checkpoints [G][2 J][64].
__host__ __device__ inline int nuts_block_rows(int nslices) { return (nslices + 7) & ~7; }
struct NutsBlockLds {
    int G, ck, bytes;
};
__host__ __device__ inline NutsBlockLds nuts_block_lds(int G, int nslices, int NT, int J)
{
    NutsBlockLds l;
    l.G = 3 * kNutsBlockWaves * 128 + 64;
    l.ck = l.G + (G * nuts_block_rows(nslices) + 8) * (16 * NT + 4) * 4;
    l.bytes = l.ck + G * 2 * J * 256;
    return l;
}

// The gradient of a chain from its slice sums in LDS, added in slice order: lane d
// adds component d, and lane 16 NT the log-likelihoods (a lane of its own while
// NT < 4; with all 64 taken every lane adds them).
template <int NT>
struct BlockGrad {
    const float* G;  // slice rows of ST floats: X^T r, then loglik
    int nslices;
    __device__ __forceinline__ void operator()(int, const WaveVec<1>& th, int lane, WaveVec<1>& g, float& Un) const
    {
        constexpr int ST = 16 * NT + 4, L = 16 * NT;
        WaveVec<1> gs;
        gs.r[0] = 0.0f;
        float ll = 0.0f;
        const float* gp = G + (lane < ST ? lane : 0);
        // eight slices' reads in flight while the eight before them are added; the
        // rows past the last slice are zero (read ahead by eight more, unused)
        float v[8], u[8];
        auto fetch = [&](int s0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = gp[(s0 + i) * ST];
                if constexpr (NT == 4) u[i] = G[(s0 + i) * ST + L];
            }
        };
        fetch(0);
#pragma unroll 2
        for (int s0 = 0; s0 < nslices; s0 += 8) {
            float w[8], x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                w[i] = v[i];
                if constexpr (NT == 4) x[i] = u[i];
            }
            fetch(s0 + 8);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                gs.r[0] += w[i];
                if constexpr (NT == 4) ll += x[i];
            }
        }
        if constexpr (NT < 4) {
            ll = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gs.r[0]), L));
            if (lane >= L) gs.r[0] = 0.0f;
        }
        slice_finish<1>(th, gs, ll, g, Un);
    }
};

// Rows 16 rt + 4 q4 .. + 3 of both row tiles (two packed words each) into the
// B operand's order, rows 8 q4 .. + 7 of the chunk, by exchanges across the
// rows of 16 lanes.
__device__ __forceinline__ uint4 rows_to_operand(uint2 t0, uint2 t1)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 a = __builtin_amdgcn_permlane32_swap(t0.x, t1.x, false, false);
    const u2 b = __builtin_amdgcn_permlane32_swap(t0.y, t1.y, false, false);
    const u2 x = __builtin_amdgcn_permlane16_swap(a.x, a.y, false, false);
    const u2 y = __builtin_amdgcn_permlane16_swap(b.x, b.y, false, false);
    return make_uint4(x.x, y.x, x.y, y.y);
}

// X operands of one chunk.  With one d tile (D <= 16) only the first 16 of the 32 k
// slots are used: one load then brings both row tiles (lanes 0-31 row tile 0, in
// the first 16 slots, 32-63 row tile 1, in the others), and Theta's pieces stand
// in the first slots for the one (zero in the others) and in the last for the
// other.
template <int NK32, int NT>
struct ChunkX {
    static constexpr int NR = NT == 1 ? 1 : 2;
    uint4 x[NK32][NR][3];
    __device__ __forceinline__ void load(const unsigned char* chunk, int lane)
    {
        const unsigned char* src = chunk + (NT == 1 ? 2048 * (lane >> 5) + 16 * (lane & 31) : 16 * lane);
#pragma unroll
        for (int kk = 0; kk < NK32; ++kk)
#pragma unroll
            for (int rt = 0; rt < NR; ++rt)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    x[kk][rt][p] = *reinterpret_cast<const uint4*>(src + p * 4096 + rt * 2048 + kk * 1024);
    }
    // eta = X Theta of both row tiles (b: Theta's pieces, per row tile if they differ)
    __device__ __forceinline__ void eta(const uint4 (&b)[2][3], floatx4 (&en)[2]) const
    {
        en[0] = en[1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kk = 0; kk < NK32; ++kk)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                en[rt] = mfma_bf16x6(x[kk][NT == 1 ? 0 : rt], b[NT == 1 ? rt : kk], en[rt]);
    }
};

template <int NT>
struct ChunkD {
    uint4 x[NT][3];
    __device__ __forceinline__ void load(const unsigned char* chunk, int lane)
    {
        const unsigned char* src = chunk + GradB<2>::XRB + 16 * lane;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int p = 0; p < 3; ++p) x[t][p] = *reinterpret_cast<const uint4*>(src + p * 4096 + t * 1024);
    }
    __device__ __forceinline__ void xtr(const uint4 (&b)[3], floatx4 (&acc)[NT]) const
    {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16x6(x[t], b, acc[t]);
    }
};

// Operands of R chunks kept in registers from step to step (R = 0: none).
template <int NK32, int NT, int R>
struct HeldX {
    ChunkX<NK32, NT> x[R > 0 ? R : 1];
    ChunkD<NT> d[R > 0 ? R : 1];
};

// Slice sums of all slices for the block's chains (positions' pieces in Tp), into
// Gs.  lgp: log2 of the chains' columns; spw: slices a wave takes at once.  R > 0: the
// slices are chunks, and the wave's, at most R, are held in H.
template <int NK32, int NT, int R>
__device__ __forceinline__ void nuts_block_gradient(const GradK& a, int G, int lgp, int spw, const uint16_t* Tp,
                                                    float* Gs, const HeldX<NK32, NT, R>& H)
{
    using S = GradB<2>;
    constexpr float kLn2 = 0.693147180559945309f;
    constexpr int ST = 16 * NT + 4;
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int l16 = lane & 15, q4 = lane >> 4;
    const int mychain = l16 & ((1 << lgp) - 1), mygrp = l16 >> lgp;
    const int cps = R > 0 ? 1 : a.slice_rows >> 5;  // chunks per slice (the last slice may hold fewer)
    const int nlast = (a.N - (a.nslices - 1) * a.slice_rows + 31) >> 5;
    const unsigned char* Xb = reinterpret_cast<const unsigned char*>(a.Xb);
    uint4 th[2][3];  // by k step, or (one d tile) by row tile
#pragma unroll
    for (int i = 0; i < (NT == 1 ? 2 : NK32); ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
            th[i][p] = *reinterpret_cast<const uint4*>(Tp + (p * kNutsBlockWaves + mychain) * 64 +
                                                       (NT == 1 ? (16 * i + 8 * q4) & 31 : 32 * i + 8 * q4));

    for (int set = wave * spw; set < a.nslices; set += kNutsBlockWaves * spw) {
        const int nset = min(spw, a.nslices - set);
        const bool ends = set + nset == a.nslices;  // holds the job's last slice
        const int nch0 = ends && nset == 1 ? nlast : cps;
        const bool ok = mygrp < nset;
        const int rb = ok ? (set + mygrp) * a.slice_rows : 0;
        const int re = min(rb + a.slice_rows, a.N);
        const int nch = ok ? (re - rb + 31) >> 5 : 0;
        floatx4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        float uacc = 0.0f;
        for (int c = 0; c < nch0; ++c) {
            const int na = ends && c >= nlast ? nset - 1 : nset;  // slices that have a chunk c
            const unsigned char* src0 = Xb + (size_t)(set * cps + c) * S::CHUNK;
            const size_t sstep = (size_t)cps * S::CHUNK;
            const float* yp = a.y + rb + (ok ? 32 * c : 0) + 4 * q4;
            const float4 y0 = *reinterpret_cast<const float4*>(yp), y1 = *reinterpret_cast<const float4*>(yp + 16);
            floatx4 en[2];
            en[0] = en[1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            auto eta = [&](const ChunkX<NK32, NT>& x, int s) {
                floatx4 e[2];
                x.eta(th, e);
                en[0] = mygrp == s ? e[0] : en[0];
                en[1] = mygrp == s ? e[1] : en[1];
            };
            ChunkD<NT> xd;
            if constexpr (R > 0) {
#pragma unroll
                for (int s = 0; s < R; ++s)
                    if (s < na) eta(H.x[s], s);
            } else {
                ChunkX<NK32, NT> xa, xn;
                xa.load(src0, lane);
#pragma unroll 2
                for (int s = 0; s < na; ++s) {
                    xn.load(src0 + min(s + 1, na - 1) * sstep, lane);
                    eta(xa, s);
                    xa = xn;
                }
                xd.load(src0, lane);
            }
            // residuals and log-likelihood, the terms of logreg_grad_tile in its order
            const float yv[2][4] = {{y0.x, y0.y, y0.z, y0.w}, {y1.x, y1.y, y1.z, y1.w}};
            float lin = 0.0f, prod[2] = {1.0f, 1.0f};
            uint2 rp[2][3];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                uint32_t ph[4], pm[4], pl[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = en[rt][i], y = yv[rt][i];
                    const bool pos = v >= 0.0f;
                    const float ex = __expf(-fabsf(v));
                    const float inv = __builtin_amdgcn_rcpf(1.0f + ex);
                    const float sig = pos ? inv : ex * inv;
                    lin = fmaf(pos ? y - 1.0f : y, v, lin);
                    prod[rt] *= 1.0f + ex;
                    split_bf16x3(y - sig, ph[i], pm[i], pl[i]);
                }
                rp[rt][0] = make_uint2(ph[0] | (ph[1] << 16), ph[2] | (ph[3] << 16));
                rp[rt][1] = make_uint2(pm[0] | (pm[1] << 16), pm[2] | (pm[3] << 16));
                rp[rt][2] = make_uint2(pl[0] | (pl[1] << 16), pl[2] | (pl[3] << 16));
            }
            const float term = lin - kLn2 * (__builtin_amdgcn_logf(prod[0]) + __builtin_amdgcn_logf(prod[1]));
            if (c < nch) uacc += term;
            uint4 rb3[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) rb3[p] = rows_to_operand(rp[0][p], rp[1][p]);
            floatx4 acc0[NT];  // at the chunk's start: the slices' products do not wait for each other
#pragma unroll
            for (int t = 0; t < NT; ++t) acc0[t] = acc[t];
            auto xtr = [&](const ChunkD<NT>& x, int s) {
                floatx4 o[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) o[t] = acc0[t];
                x.xtr(rb3, o);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mygrp == s ? o[t] : acc[t];
            };
            if constexpr (R > 0) {
#pragma unroll
                for (int s = 0; s < R; ++s)
                    if (s < na) xtr(H.d[s], s);
            } else {
                ChunkD<NT> xe;
#pragma unroll 2
                for (int s = 0; s < na; ++s) {
                    xe.load(src0 + min(s + 1, na - 1) * sstep, lane);
                    xtr(xd, s);
                    xd = xe;
                }
            }
        }
        if (nch > 0) {  // ln 2 per padding row of this lane's rows (the slice's last chunk)
            float npad = 0.0f;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                const int rowl = rb + 32 * (nch - 1) + 16 * rt + 4 * q4;
                npad += (float)min(4, max(0, rowl + 4 - re));
            }
            uacc += npad * kLn2;
        }
        uacc += __shfl_xor(uacc, 16, 64);
        uacc += __shfl_xor(uacc, 32, 64);
        if (ok && mychain < G) {
            float* row = Gs + (mychain * nuts_block_rows(a.nslices) + set + mygrp) * ST;
#pragma unroll
            for (int t = 0; t < NT; ++t) *reinterpret_cast<floatx4*>(row + 16 * t + 4 * q4) = acc[t];
            if (q4 == 0) row[16 * NT] = uacc;
        }
    }
}

// Up to K steps of chains first .. first + G - 1 (one block; lds: nuts_block_lds
// bytes).  Pending chains at the end are counted in rcnt (if given).
template <int NK32, int NT, int R>
__device__ __forceinline__ void nuts_block_run(const NutsK& a, const GradK& gk, int first, int G, int K,
                                               unsigned char* lds, uint32_t* rcnt)
{
    constexpr int ST = 16 * NT + 4;
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const NutsBlockLds L = nuts_block_lds(G, a.nslices, NT, a.J);
    uint16_t* Tp = reinterpret_cast<uint16_t*>(lds);
    int* flag = reinterpret_cast<int*>(lds + 3 * kNutsBlockWaves * 128);
    float* Gs = reinterpret_cast<float*>(lds + L.G);
    int lgp = 0;
    while ((1 << lgp) < G) ++lgp;
    const int spw = min(16 >> lgp, (a.nslices + kNutsBlockWaves - 1) / kNutsBlockWaves);
    HeldX<NK32, NT, R> H;
    if constexpr (R > 0) {
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const int sl = min(wave * spw + s, a.nslices - 1);
            const unsigned char* src = reinterpret_cast<const unsigned char*>(gk.Xb) + (size_t)sl * GradB<2>::CHUNK;
            H.x[s].load(src, lane);
            H.d[s].load(src, lane);
        }
    }

    const int c = first + wave;
    bool live = wave < G && c < a.m;
    uint32_t t0 = 0;
    if (live) {
        t0 = uni(a.t[c]);
        live = t0 < a.tstop;
    }
    const bool mine = live;
    const int cl = mine ? c : 0;
    float* ck = reinterpret_cast<float*>(lds + L.ck) + (size_t)(mine ? wave : 0) * 2 * a.J * 64;
    NutsBox<1, BOX_HELD> box(a.V + (size_t)cl * a.nvec * 64, 64, lane, ck);
    NutsScal Sc = nuts_load(a, cl, t0);
    const int rows = nuts_block_rows(a.nslices);
    float* Gw = Gs + wave * rows * ST;
    if (mine) {
        for (int s = a.nslices; s < rows; ++s) {
            Gw[s * ST + min(lane, ST - 1)] = 0.0f;
            if constexpr (ST > 64) Gw[s * ST + 64] = 0.0f;
        }
        const float* cm = box.Vc + V_FIXED * 64;
        for (int i = 0; i < 2 * a.J; ++i) ck[i * 64 + lane] = cm[i * 64 + lane];
        if (Sc.fl & NF_PENDING) {
            for (int s = 0; s < a.nslices; ++s) {
                if (lane < 16 * NT) Gw[s * ST + lane] = gk.Gpart[((size_t)s * a.m + c) * 64 + lane];
                if (lane == 0) Gw[s * ST + 16 * NT] = gk.Upart[(size_t)s * a.m + c];
            }
        }
    }
    const BlockGrad<NT> grad{Gw, a.nslices};
    unsigned long long steps = 0;
    int req = 0;
    for (int it = 0; it < K; ++it) {
        req = 0;
        if (live) {
            req = nuts_chain_body<1, BlockGrad<NT>, false, BOX_HELD>(a, grad, c, lane, Sc, box) & NC_REQ ? 1 : 0;
            if (req) {
                WaveVec<1> th;
                box.template get<V_THR, V_THL>(Sc.v > 0, th);
                uint32_t h, m, l;
                split_bf16x3(th.r[0], h, m, l);
                Tp[wave * 64 + lane] = (uint16_t)h;
                Tp[(kNutsBlockWaves + wave) * 64 + lane] = (uint16_t)m;
                Tp[(2 * kNutsBlockWaves + wave) * 64 + lane] = (uint16_t)l;
                ++steps;
            }
            live = req != 0;
        }
        if (lane == 0) flag[wave] = req;
        __syncthreads();
        const int4 f0 = *reinterpret_cast<const int4*>(flag), f1 = *reinterpret_cast<const int4*>(flag + 4);
        if (uni(f0.x | f0.y | f0.z | f0.w | f1.x | f1.y | f1.z | f1.w) == 0) break;
        nuts_block_gradient<NK32, NT, R>(gk, G, lgp, spw, Tp, Gs, H);
        __syncthreads();
    }
    if (!mine) return;
    box.write_back();
    float* cm = box.Vc + V_FIXED * 64;
    for (int i = 0; i < 2 * a.J; ++i) cm[i * 64 + lane] = ck[i * 64 + lane];
    if (req) {  // K steps done: the state the launch-per-step path leaves after its gradient
        WaveVec<1> th;
        box.template get<V_THR, V_THL>(Sc.v > 0, th);
        th.store(a.Thq + (size_t)c * 64, lane);
        for (int s = 0; s < a.nslices; ++s) {
            gk.Gpart[((size_t)s * a.m + c) * 64 + lane] = lane < 16 * NT ? Gw[s * ST + lane] : 0.0f;
            if (lane == 0) gk.Upart[(size_t)s * a.m + c] = Gw[s * ST + 16 * NT];
        }
    }
    nuts_store(a, c, Sc, req, lane);
    if (lane == 0) {
        if (steps) atomicAdd(&a.ctr[0], steps);
        if (req && rcnt) atomicAdd(rcnt, 1u);
    }
}

}  // namespace fsmmc
