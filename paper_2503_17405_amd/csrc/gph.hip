// gph.hip -- elliptical slice sampling of GP-regression hyperparameters
// (Sec. 7.2): theta = (tau, lambda, sigma) with the N(0, I) prior, and the
// marginal likelihood
//   y ~ N(0, C),  C = tau^2 exp(-lambda^2 |x_i - x_k|^2) + (sigma^2 + jitter) I,
//   log L = -y^T C^-1 y / 2 - log det C / 2,
// an O(n^3) Cholesky factorisation inside every loop iteration: the regime
// where the log-density dominates each transition and the FSM gain tracks R(m).
//
// Persistent kernel: a block of NW waves takes chains from a device ticket
// counter and runs each one's ESS FSM (INIT, SHRINK, DONE; every step = one
// proposal and one likelihood) to its draw budget, so no chain waits for
// another.  The likelihood is computed by the block in FP64 (kernel matrices
// of smooth kernels are badly conditioned; the 3-D chain state is FP64 too) on
// the matrix cores, from 16 x 16 tiles held in registers (gph_loglik below).
// The squared distances |x_i - x_k|^2 do not depend on theta: they are formed
// once per job (gph_dist_kernel), laid out tile by tile as the lanes read them
// (but for small jobs under an HBM budget, gph_keeps_dist).
// The library builds with contraction off, so the updates are written as
// explicit FMAs (one instruction and one rounding per term).
// The synchronized runtime launches the kernel once per draw (tstop =
// draw + 1); in vmap mode a second launch evaluates the max_j N_j - N_j
// likelihoods a batched while loop would compute and discard.
#include "fsmmc_device.h"
#include "fsmmc_internal.h"

#include <utility>

namespace fsmmc {

constexpr int kGphMaxN = 512;  // observations
constexpr int kGphMaxP = 16;   // input dimension
constexpr int kGphTile = 256;  // doubles of a 16 x 16 tile

struct GphK {
    int m, n, N, p;
    uint32_t tstop;
    uint64_t seed;
    double jitter;
    const double* y;   // N outputs
    const double* X;   // N x p inputs
    const double* r2;  // squared distances, tile (I, J <= I) at I (I + 1) / 2 + J (gph_dist_kernel), or NULL
    double *th, *nu;  // [chain][3]
    double *lx, *phi, *pmin, *pmax, *logu;
    int32_t *k, *evals;
    uint32_t* t;
    int64_t* budget;
    double* out;  // m x n x 3
    int32_t* counts;
    unsigned long long* ctr;
    int32_t* maxN;
    double* sink;
    double* slots;  // N >= 256: finished tiles of the leading columns, slot_tiles per block
    int slot_tiles;
};

__device__ __forceinline__ double rl(double v, int l)
{
    const int64_t b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// ------------------------------------------------------------ likelihood
// log L(th) by a block of NW waves.  The matrix is C with y as one more row (row
// n), so that the factorisation's row n is the forward solve z = L^-1 y; it is
// cut into 16 x 16 tiles, T tile columns and R tile rows (R = T, or T + 1 when
// 16 divides n).
//
// Tile layout ("fragments"): lane (q, i) = (lane / 16, lane % 16) holds row i,
// columns q, q + 4, q + 8, q + 12.  For v_mfma_f64_16x16x4_f64 this is the
// operand layout of A and of B^T (k step s: column 4 s + q) and, with the
// product taken transposed, the layout of the result: a finished tile is the
// next product's operand with no data movement.  Registers hold minus the
// remaining matrix, so every update is a plain accumulation.
//
// Right-looking over the tile columns t.  The wave that owns row t factors the
// diagonal tile (gph_factor) and publishes minus its inverse in LDS; every wave
// then takes its rows' tiles of column t to L_It = A_It L_tt^-T (four MFMAs),
// publishes them in LDS and updates its remaining tiles with L_It L_ct^T (four
// MFMAs each, L_ct from LDS).  Two barriers per tile column; the next diagonal
// tile is factored beside the other waves' updates.  Wave w owns rows
// w and 2 NW - 1 - w: 2 NW + 1 tiles whatever w, all in registers (position p:
// column p of the first row for p <= w, column 2 NW - p of the second above).
//
// LEAD (n >= 256, more than 16 tile rows): the leading R - 16 tile columns go
// first, in panels of four columns (rows dealt to the waves in turn, up to five
// each); their finished tiles go to the block's slot in memory, and the
// panels after them and the trailing 16 rows start from C minus the products
// of those tiles.
//
// What bounds it: the FP64 matrix and vector units have the same rate (one
// MFMA = 64 cycles of its SIMD = 16 FMAs), but an FMA form needs its operands
// broadcast through LDS (four times the LDS bytes per flop) or by lane reads;
// what is left is the serial chain of the diagonal tiles (about 3600 cycles
// each alone) and, with several blocks per CU, the issue slots that the
// diagonal tiles, the exponentials and the updates share.
// Measured against the factorisations this replaced (n <= 96: the wave's own
// rows in LDS; above: a global work matrix, 32-column panels), whole jobs:
//   n =  25, 1024 chains x 100 draws:  24.9 ->  5.2 ms
//   n =  63,  512 chains x  60 draws:  70.4 ->  7.7 ms
//   n = 100, 1024 chains x  60 draws: 325   -> 23.6 ms
//   n = 191, 1024 chains x   8 draws (8 waves a block -> 6): 17.1 -> 15.2 ms
//   n = 414,  512 chains x  16 draws: 401   -> 80.3 ms
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

// A tile in memory: doubles [half][lane][2], so a lane's four values are two
// 16-byte accesses that fill whole lines.
__device__ __forceinline__ d4 tile_load(const double* t, int lane)
{
    const double2 u = reinterpret_cast<const double2*>(t)[lane];
    const double2 v = reinterpret_cast<const double2*>(t)[64 + lane];
    return d4{u.x, u.y, v.x, v.y};
}

__device__ __forceinline__ void tile_store(double* t, int lane, const d4& v)
{
    reinterpret_cast<double2*>(t)[lane] = make_double2(v[0], v[1]);
    reinterpret_cast<double2*>(t)[64 + lane] = make_double2(v[2], v[3]);
}

// c ? a : b by selects (a branch would give the product two homes and copies between)
__device__ __forceinline__ d4 choose(bool c, const d4& a, const d4& b)
{
    return d4{c ? a[0] : b[0], c ? a[1] : b[1], c ? a[2] : b[2], c ? a[3] : b[3]};
}

// acc + (a b^T)^T, a and b tiles as fragments
__device__ __forceinline__ d4 tile_mac(const d4& a, const d4& b, d4 acc)
{
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
    return acc;
}

// v[k] / v[k] = x for a wave-uniform k known at run time only (registers have no
// index: a chain of uniform branches).  With these the tile loops are loops:
// copies of their bodies per tile made 150 KiB of code (now 50) and spilled.
// Every index into a register tile array is a template constant (each):
// with unrolled loops the branches are merged into one indexed access before
// the loops unroll, and the array ends up in scratch memory.
#define FSMMC_INLINE __attribute__((always_inline))
template <int... I, typename F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, const F& f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(const F& f)
{
    each_of(std::make_integer_sequence<int, N>{}, f);
}
template <int N>
__device__ __forceinline__ d4 pick(const d4 (&v)[N], int k)
{
    d4 x = v[0];
    each<N>([&](auto i) FSMMC_INLINE {
        if (i == k) x = v[i];
    });
    return x;
}
template <int N>
__device__ __forceinline__ void put(d4 (&v)[N], int k, const d4& x)
{
    each<N>([&](auto i) FSMMC_INLINE {
        if (i == k) v[i] = x;
    });
}

// What a wave gathers along the way: the pivots of its diagonal tiles as a
// mantissa product and an exponent sum (factors in [1/2, 1), 16 a tile: two trailing
// tiles and, for n >= 256, one in each panel of four leading columns, so 112 at n =
// 512 and a product of at least 2^-112), and |z|^2 (the lanes of row n).  A pivot that is not positive makes its column,
// and with it z, NaN.
struct GphSum {
    double pm = 1.0, zz = 0.0;
    int pe = 0;
};

// The diagonal tile: acc = minus the remaining tile.  Lanes 0-15 take the
// tile's rows whole, lanes 16-31 the identity's: eliminating the columns
// leaves L in the former and L^-T in the latter, and minus L^-1 goes to inv as
// a tile.  Only the first nc columns exist (the last tile; what the others
// hold goes nowhere).  yrow: the tile's row that is row n of the matrix, or -1.
__device__ __forceinline__ void gph_factor(const d4& acc, int nc, int yrow, int lane, double* inv, GphSum& G)
{
    __builtin_amdgcn_s_setprio(3);  // every other wave of the block waits for this one
    int i = lane & 15;
    asm volatile("" : "+v"(i));
    const bool unit = (lane & 16) != 0;
    double W[16];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double a, b, c[4];
        lane_pair<16>(-acc[r], a, b);  // a: rows 0 and 2 of 16 lanes, b: rows 1 and 3
        lane_pair<32>(a, c[0], c[2]);
        lane_pair<32>(b, c[1], c[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q) W[4 * r + q] = unit ? (4 * r + q == i ? 1.0 : 0.0) : c[q];
    }
    auto pivot = [&](double ajj, int j) {
        G.pm *= j < nc ? __builtin_amdgcn_frexp_mant(ajj) : 1.0;
        G.pe += j < nc ? __builtin_amdgcn_frexp_exp(ajj) : 0;
        // 1 / sqrt(ajj): the hardware estimate (about 2^-26) and one
        // third-order step, y + y e (1/2 + 3/8 e), e = 1 - a y^2
        const double y0 = __builtin_amdgcn_rsq(ajj);
        const double e = fma(-(ajj * y0), y0, 1.0);
        return fma(y0 * e, fma(0.375, e, 0.5), y0);
    };
    double r = pivot(rl(W[0], 0), 0);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        W[j] *= r;
        if (j < 15) {  // the next pivot first: its reciprocal root runs under the other updates
            W[j + 1] = fma(-W[j], rl(W[j], j + 1), W[j + 1]);
            r = pivot(rl(W[j + 1], j + 1), j + 1);
        }
#pragma unroll
        for (int u = j + 2; u < 16; ++u) W[u] = fma(-W[j], rl(W[j], u), W[u]);
        __builtin_amdgcn_sched_barrier(0);  // one column's lane reads in scalar registers at a time
    }
    if (lane == yrow) {
#pragma unroll
        for (int j = 0; j < 16; ++j) G.zz = j < nc ? fma(W[j], W[j], G.zz) : G.zz;
    }
    if (unit && lane < 32) {  // lane 16 + i: column i of L^-1, element u at (row u, column i)
#pragma unroll
        for (int u = 0; u < 16; ++u) inv[((i >> 3) * 64 + (i & 3) * 16 + u) * 2 + ((i >> 2) & 1)] = -W[u];
    }
    __builtin_amdgcn_s_setprio(0);
}

// The squared distance of inputs i and k (0 past the last).
__device__ __forceinline__ double gph_dist2(const double* X, int N, int p, int i, int k)
{
    double s = 0.0;
    if (i < N && k < N)
        for (int d = 0; d < p; ++d) {
            const double e = X[i * p + d] - X[k * p + d];
            s = fma(e, e, s);
        }
    return s;
}

// Minus tile (I, J) of C (with y as row n).  KEPT: the job holds the squared distances.
template <bool KEPT>
__device__ __forceinline__ d4 gph_tile_of_c(const GphK& a, double tau2, double lam2, double s2, int I, int J, int lane)
{
    const int row = 16 * I + (lane & 15), col0 = 16 * J + (lane >> 4);
    d4 v, r2;
    if constexpr (KEPT) {
        r2 = tile_load(a.r2 + (size_t)(I * (I + 1) / 2 + J) * kGphTile, lane);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) r2[r] = gph_dist2(a.X, a.N, a.p, row, col0 + 4 * r);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = -(tau2 * exp(-lam2 * r2[r]) + (row == col0 + 4 * r ? s2 : 0.0));
    if (16 * I + 16 > a.N) {  // the tile row that holds row n and the padding below it
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = col0 + 4 * r;
            if (row >= a.N) v[r] = row == a.N && col < a.N ? -a.y[col] : 0.0;
        }
    }
    return v;
}

// LDS doubles: one published column (2 NW tiles; two for 8 waves), the inverse, two
// sums per wave
template <int NW>
constexpr int gph_lds_doubles() { return ((NW >= 8 ? 4 : 2) * NW + 1) * kGphTile + 2 * NW; }

// Waves a SIMD holds at the registers of the class: 2 NW + 1 tiles of 8 and
// about 60 more (4 waves: 128, 3: 168, 2: 256).
constexpr int gph_waves_per_simd(int NW) { return NW >= 8 ? 2 : (NW >= 6 ? 3 : 4); }

template <int NW, bool LEAD, bool KEPT>
__device__ double gph_loglik(const GphK& a, const double* th, double* slot, double* sm)
{
    constexpr int RW = 2 * NW;
    const int n = a.N, T = (n + 15) >> 4, R = (n + 16) >> 4, yrow = n & 15;
    int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    // opaque here and at each phase below: what is derived from them would
    // otherwise be kept across the whole chain loop, and spilled
    asm volatile("" : "+v"(lane), "+s"(wave));
    double* colb = sm;
    constexpr int NB = NW >= 8 ? 2 : 1;  // column buffers
    double* inv = sm + NB * RW * kGphTile;
    double* red = inv + kGphTile;
    const double tau2 = th[0] * th[0], lam2 = th[1] * th[1], s2 = th[2] * th[2] + a.jitter;
    GphSum G;
    // L_It from minus the remaining tile x; its part of |z|^2 if it holds row n
    auto solve = [&](const d4& iv, const d4& x, int I) {
        const d4 L = tile_mac(iv, x, d4{0.0, 0.0, 0.0, 0.0});
        if (I == R - 1 && (lane & 15) == yrow) {
#pragma unroll
            for (int r = 0; r < 4; ++r) G.zz = fma(L[r], L[r], G.zz);
        }
        return L;
    };
    const int base = LEAD ? R - RW : 0;  // rows and columns below go first
    if constexpr (LEAD) {
        constexpr int NS = (kGphMaxN / 16 + 1 + NW - 1) / NW;  // rows per wave, at most
        auto at = [&](int I, int k) { return slot + (size_t)(k * R + I) * kGphTile; };
        for (int P = 0; P < base; P += 4) {
            const int pc = min(4, base - P);
            d4 acc[NS][4];  // [slot s: row P + wave + NW s][column]
            // C's tiles by way of the places in the slot that their L will take
#pragma unroll 1
            for (int v = 0; v < 4 * NS; ++v) {
                const int rel = wave + NW * (v >> 2), c = v & 3;
                if (P + rel < R && c < pc && c <= rel)
                    tile_store(at(P + rel, P + c), lane, gph_tile_of_c<KEPT>(a, tau2, lam2, s2, P + rel, P + c, lane));
            }
            each<4 * NS>([&](auto v) FSMMC_INLINE {
                const int rel = wave + NW * (v >> 2), c = v & 3;
                acc[v >> 2][v & 3] =
                    P + rel < R && c < pc && c <= rel ? tile_load(at(P + rel, P + c), lane) : d4{0.0, 0.0, 0.0, 0.0};
            });
            for (int k = 0; k < P; ++k) {
                d4 A[4];
                each<4>([&](auto c) FSMMC_INLINE { A[c] = tile_load(at(P + min((int)c, pc - 1), k), lane); });
                each<NS>([&](auto s) FSMMC_INLINE {
                    const int I = P + wave + NW * s;
                    if (I < R) {
                        const d4 B = tile_load(at(I, k), lane);
                        each<4>([&](auto c) FSMMC_INLINE { acc[s][c] = tile_mac(A[c], B, acc[s][c]); });
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
#pragma unroll 1
            for (int t = 0; t < pc; ++t) {
                asm volatile("" : "+v"(lane), "+s"(wave));
                if (wave == t) gph_factor(pick(acc[0], t), 16, -1, lane, inv, G);
                __syncthreads();
                const d4 iv = tile_load(inv, lane);
                d4 L[NS];
                each<NS>([&](auto s) FSMMC_INLINE {
                    const int rel = wave + NW * s, I = P + rel;
                    L[s] = d4{0.0, 0.0, 0.0, 0.0};
                    if (rel > t && I < R) {
                        L[s] = solve(iv, pick(acc[s], t), I);
                        tile_store(at(I, P + t), lane, L[s]);
                        if (rel < pc) tile_store(colb + rel * kGphTile, lane, L[s]);
                    }
                });
                __syncthreads();
                each<4>([&](auto u) FSMMC_INLINE {
                    if (u > t && u < pc) {
                        const d4 A = tile_load(colb + u * kGphTile, lane);
                        each<NS>([&](auto s) FSMMC_INLINE {
                            if (wave + NW * s >= u && P + wave + NW * s < R)
                                acc[s][u] = tile_mac(A, L[s], acc[s][u]);
                        });
                    }
                });
            }
        }
    }
    // the trailing rows base .. R - 1, all tiles in registers
    const int ra = wave, rb = RW - 1 - wave;  // this wave's rows, relative to base
    d4 acc[RW + 1];
    each<RW + 1>([&](auto p) FSMMC_INLINE { acc[p] = d4{0.0, 0.0, 0.0, 0.0}; });
#pragma unroll 1
    for (int p = 0; p <= RW; ++p) {
        const bool second = p > wave;
        const int I = base + (second ? rb : ra), J = base + (second ? RW - p : p);
        if (I < R && J < T) put(acc, p, gph_tile_of_c<KEPT>(a, tau2, lam2, s2, I, J, lane));
    }
    if constexpr (LEAD) {
        // minus the leading columns' products: column k of the finished tiles
        // through LDS, the next one's loads in flight
        constexpr int NV = RW * kGphTile / 2 / (64 * NW);  // 16-byte units per thread
        d2 nx[NV];
        auto fetch = [&](int k) {
            const d2* src = reinterpret_cast<const d2*>(slot + (size_t)(k * R + base) * kGphTile);
            each<NV>([&](auto v) FSMMC_INLINE { nx[v] = src[v * 64 * NW + threadIdx.x]; });
        };
        fetch(0);
#pragma unroll 1
        for (int k = 0; k < base; ++k) {
            asm volatile("" : "+v"(lane), "+s"(wave));
            __syncthreads();  // the previous column has been read
            each<NV>([&](auto v) FSMMC_INLINE { reinterpret_cast<d2*>(colb)[v * 64 * NW + threadIdx.x] = nx[v]; });
            __syncthreads();
            if (k + 1 < base) fetch(k + 1);
            const d4 La = tile_load(colb + wave * kGphTile, lane), Lb = tile_load(colb + (RW - 1 - wave) * kGphTile, lane);
            each<RW + 1>([&](auto p) FSMMC_INLINE {
                const bool second = p > wave;
                const d4 A = tile_load(colb + (second ? RW - p : p) * kGphTile, lane);
                acc[p] = tile_mac(A, choose(second, Lb, La), acc[p]);
                if (p % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            });
        }
        __syncthreads();
    }
    // Step t: TRSM of column t, then the updates it allows.  The owner of row
    // t + 1 takes its tiles of column t + 1 first, factors, and leaves its other
    // updates to the next step (column t stays in LDS: two column buffers), so
    // the factorisation runs beside the other waves' updates (n = 414: 93.2 -> 88.2
    // ms for 512 chains x 16 draws; with the up to four blocks per CU of the smaller
    // classes other chains fill that time already, and n = 100 lost 2%).
    constexpr bool kAhead = NW >= 8;
    const int nt = T - base;
    auto owner = [](int t) { return t < NW ? t : RW - 1 - t; };
    bool behind = false;  // this wave has not applied column t - 1 to columns past t
#pragma unroll 1
    for (int t = kAhead ? -1 : 0; t < nt; ++t) {
        asm volatile("" : "+v"(lane), "+s"(wave));
        const int ra = wave, rb = RW - 1 - wave;
        const bool hasa = base + ra < R, hasb = base + rb < R;
        auto factor = [&](int k) {
            gph_factor(pick(acc, k < NW ? wave : wave + 1), min(16, n - 16 * (base + k)), base + k == R - 1 ? yrow : -1,
                       lane, inv, G);
        };
        const bool next = kAhead && t + 1 < nt && wave == owner(t + 1);
        if constexpr (!kAhead)
            if (wave == owner(t)) factor(t);
        if (!kAhead || t >= 0) {
            double* col = colb + (t & (NB - 1)) * RW * kGphTile;
            __syncthreads();
            const d4 iv = tile_load(inv, lane);
            d4 La = d4{0.0, 0.0, 0.0, 0.0}, Lb = La;
            if (ra > t && hasa) {
                La = solve(iv, pick(acc, t), base + ra);
                tile_store(col + ra * kGphTile, lane, La);
            }
            if (rb > t && hasb) {
                Lb = solve(iv, pick(acc, RW - t), base + rb);
                tile_store(col + rb * kGphTile, lane, Lb);
            }
            __syncthreads();
            const int most = next && !behind ? t + 1 : RW;
#pragma unroll 1
            for (int k = behind ? t - 1 : t; k <= t; ++k) {
                const double* ck = colb + (k & (NB - 1)) * RW * kGphTile;
                if constexpr (kAhead) {
                    La = tile_load(ck + ra * kGphTile, lane);
                    Lb = tile_load(ck + rb * kGphTile, lane);
                }
                each<RW + 1>([&](auto p) FSMMC_INLINE {
                    const bool second = p > wave;
                    const int c = second ? RW - p : p;
                    if (c > t && c <= most && base + c < T && (second ? hasb : hasa)) {
                        const d4 A = tile_load(ck + c * kGphTile, lane);
                        if constexpr (NW >= 8) {
                            acc[p] = tile_mac(A, choose(second, Lb, La), acc[p]);
                        } else if (second) {  // no registers to spare for the choice
                            acc[p] = tile_mac(A, Lb, acc[p]);
                        } else {
                            acc[p] = tile_mac(A, La, acc[p]);
                        }
                    }
                });
            }
            behind = kAhead && most == t + 1;
        }
        if (next) factor(t + 1);
    }
    // sums over the lanes, then over the waves in order
    double lg = log(G.pm) + (double)G.pe * 0.69314718055994530942;
    double zz = wave_sum(G.zz);
    if constexpr (NW > 1) {
        if (lane == 0) {
            red[2 * wave] = lg;
            red[2 * wave + 1] = zz;
        }
        __syncthreads();
        lg = zz = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            lg += red[2 * w];
            zz += red[2 * w + 1];
        }
    }
    const double v = -0.5 * zz - 0.5 * lg;
    return v != v ? -INFINITY : v;  // not positive definite
}

// Squared distances of the inputs, one thread per element of a tile; rows and
// columns past N hold 0 (gph_tile_of_c replaces them or nothing reads them).
__global__ __launch_bounds__(256) void gph_dist_kernel(const double* X, int N, int p, double* r2)
{
    int I = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
    while ((I + 1) * (I + 2) / 2 <= (int)blockIdx.x) ++I;
    while (I * (I + 1) / 2 > (int)blockIdx.x) --I;
    const int J = (int)blockIdx.x - I * (I + 1) / 2;
    const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
    r2[(size_t)blockIdx.x * kGphTile + ((r >> 1) * 64 + lane) * 2 + (r & 1)] =
        gph_dist2(X, N, p, 16 * I + (lane & 15), 16 * J + (lane >> 4) + 4 * r);
}

// A chain's state while the block steps it, in LDS: the likelihood needs every
// register, and only wave 0 runs the FSM's own arithmetic.
struct GphState {
    double th[3], nu[3], lx, phi, pmin, pmax, logu;
    double tp[3];  // the proposal of the step in progress
    int64_t budget;
    int k, evals, go;
    uint32_t t;
};

// First half of an FSM step of chain c (ESS: INIT or SHRINK, then the proposal
// into tp); wave 0, lane 0 writes.
__device__ __forceinline__ void gph_propose(const GphK& a, int c, GphState& S, int lane)
{
    double nu[3], phi, pmin, pmax, logu = S.logu;
    int evals;
    const uint64_t seed = (uint64_t)uni((int64_t)a.seed);
    const uint32_t t = uni(S.t);
    if (uni(S.k) == 1) {  // INIT: direction, threshold, first angle and bracket
#pragma unroll
        for (int d = 0; d < 3; ++d) nu[d] = normal_at<double>(seed, (uint32_t)c, t, ROLE_NU, 0, (uint32_t)d);
        logu = log(uniform<double>(seed, (uint32_t)c, t, ROLE_THRESH, 0));
        phi = 2.0 * 3.14159265358979323846 * uniform<double>(seed, (uint32_t)c, t, ROLE_ANGLE, 0);
        pmin = phi - 2.0 * 3.14159265358979323846;
        pmax = phi;
        evals = 0;
    } else {  // SHRINK: the bracket moves to the rejected angle, draw again
#pragma unroll
        for (int d = 0; d < 3; ++d) nu[d] = S.nu[d];
        phi = S.phi;
        pmin = phi < 0.0 ? phi : S.pmin;
        pmax = phi < 0.0 ? S.pmax : phi;
        evals = S.evals;
        phi = pmin + (pmax - pmin) * uniform<double>(seed, (uint32_t)c, t, ROLE_ANGLE, (uint32_t)evals);
    }
    const double cs = cos(phi), sn = sin(phi);
    if (lane == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            S.nu[d] = nu[d];
            S.tp[d] = S.th[d] * cs + nu[d] * sn;
        }
        S.phi = phi;
        S.pmin = pmin;
        S.pmax = pmax;
        S.logu = logu;
        S.evals = evals;
    }
}

// Second half: accept (DONE: emit, then INIT of the next draw) or SHRINK next;
// one lane.  lp = log L(tp).
__device__ __forceinline__ void gph_decide(const GphK& a, int c, GphState& S, double lp, uint32_t* guard)
{
    const int evals = S.evals + 1;
    const bool acc = lp - S.lx > S.logu;
    S.evals = evals;
    S.budget -= 1;
    if (!acc && evals < kEssMaxEvals) {
        S.k = 2;
        return;
    }
    if (acc) {
#pragma unroll
        for (int d = 0; d < 3; ++d) S.th[d] = S.tp[d];
        S.lx = lp;
    } else {
        *guard += 1;
    }
    const uint32_t t = S.t;
#pragma unroll
    for (int d = 0; d < 3; ++d) a.out[((size_t)c * a.n + t) * 3 + d] = S.th[d];
    a.counts[(size_t)c * a.n + t] = evals;
    S.t = t + 1;
    S.k = 1;
}

// One lane.
__device__ __forceinline__ void gph_load(const GphK& a, int c, GphState& S)
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        S.th[d] = a.th[(size_t)c * 3 + d];
        S.nu[d] = a.nu[(size_t)c * 3 + d];
    }
    S.lx = a.lx[c];
    S.phi = a.phi[c];
    S.pmin = a.pmin[c];
    S.pmax = a.pmax[c];
    S.logu = a.logu[c];
    S.budget = a.budget[c];
    S.k = a.k[c];
    S.evals = a.evals[c];
    S.t = a.t[c];
}

__device__ __forceinline__ void gph_store(const GphK& a, int c, const GphState& S)
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        a.th[(size_t)c * 3 + d] = S.th[d];
        a.nu[(size_t)c * 3 + d] = S.nu[d];
    }
    a.lx[c] = S.lx;
    a.phi[c] = S.phi;
    a.pmin[c] = S.pmin;
    a.pmax[c] = S.pmax;
    a.logu[c] = S.logu;
    a.budget[c] = S.budget;
    a.k[c] = S.k;
    a.evals[c] = S.evals;
    a.t[c] = S.t;
}

__device__ __forceinline__ int gph_next_chain(unsigned long long* q, unsigned long long base, int m, int* sh)
{
    __syncthreads();  // the previous chain's reads of *sh are done
    if (threadIdx.x == 0) {
        const unsigned long long off = atomicAdd(q, 1ull) - base;
        *sh = off < (unsigned long long)m ? (int)off : m;
    }
    __syncthreads();
    return uni(*sh);
}

// mode 0: FSM (to tstop or through the budget); mode 1: one draw of the
// synchronized runtime (tstop = draw + 1), recording its largest count;
// mode 2: vmap padding of draw `draw`.
template <int NW, bool LEAD, bool KEPT>
__global__ __launch_bounds__(64 * NW, gph_waves_per_simd(NW)) void gph_kernel(GphK a, unsigned long long* q,
                                                                      unsigned long long base, int mode, uint32_t draw)
{
    __shared__ __align__(16) double sm[gph_lds_doubles<NW>()];
    __shared__ int s_chain;
    __shared__ GphState S;
    // the FSM part reads its arguments from LDS, wave 0 only: kept in scalar
    // registers they would be spilled around every column of gph_factor
    __shared__ GphK sa;
    if (threadIdx.x == 0) sa = a;
    double* slot = LEAD ? a.slots + (size_t)blockIdx.x * a.slot_tiles * kGphTile : nullptr;
    const int tid = threadIdx.x;
    unsigned long long steps = 0;
    uint32_t guard = 0;
    for (;;) {
        const int c = gph_next_chain(q, base, a.m, &s_chain);
        if (c >= a.m) break;
        uint32_t t0 = 0;
        int reps = 0;  // mode 2: likelihoods to discard
        if (tid == 0) {
            gph_load(sa, c, S);
            t0 = S.t;
            if (mode == 2) reps = sa.maxN[draw] - sa.counts[(size_t)c * sa.n + draw];
        }
        double sum = 0.0;
        for (;;) {
            if (tid < 64) {
                if (tid == 0) S.go = mode == 2 ? (reps-- > 0 ? 1 : 0) : (S.t < (mode == 1 ? draw + 1 : sa.tstop) && S.budget > 0 ? 1 : 0);
                if (uni(S.go)) {
                    if (mode != 2)
                        gph_propose(sa, c, S, tid);
                    else if (tid < 3)
                        S.tp[tid] = S.th[tid];
                }
            }
            __syncthreads();
            if (!uni(S.go)) break;
            const double tp[3] = {uni(S.tp[0]), uni(S.tp[1]), uni(S.tp[2])};
            const double lp = gph_loglik<NW, LEAD, KEPT>(a, tp, slot, sm);
            if (tid == 0) {
                ++steps;
                if (mode == 2)
                    sum += lp;
                else
                    gph_decide(sa, c, S, lp, &guard);
            }
        }
        if (tid == 0) {
            if (mode == 2) {
                sa.sink[c] = sum;
            } else if (S.t > t0 || S.budget < sa.budget[c]) {
                gph_store(sa, c, S);
                if (mode == 1 && S.t > t0) atomicMax(&sa.maxN[t0], sa.counts[(size_t)c * sa.n + t0]);
            }
        }
    }
    if (tid == 0) {
        if (steps) atomicAdd(&sa.ctr[mode == 2 ? 1 : 0], steps);
        if (guard) atomicAdd(&sa.ctr[2], (unsigned long long)guard);
    }
}

// Starting state: theta (from x0 or a prior draw N(0, I) on the INIT stream)
// and its log-likelihood, one block per chain.
template <int NW, bool LEAD, bool KEPT>
__global__ __launch_bounds__(64 * NW, gph_waves_per_simd(NW)) void gph_init_kernel(GphK a, int has_x0)
{
    __shared__ __align__(16) double sm[gph_lds_doubles<NW>()];
    double* slot = LEAD ? a.slots + (size_t)blockIdx.x * a.slot_tiles * kGphTile : nullptr;
    for (int c = blockIdx.x; c < a.m; c += gridDim.x) {
        double th[3];
#pragma unroll
        for (int d = 0; d < 3; ++d)
            th[d] = has_x0 ? uni(a.th[(size_t)c * 3 + d]) : normal_at<double>(a.seed, (uint32_t)c, 0, ROLE_INIT, 0, (uint32_t)d);
        const double lx = gph_loglik<NW, LEAD, KEPT>(a, th, slot, sm);
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) a.th[(size_t)c * 3 + d] = th[d];
            a.lx[c] = lx;
            a.k[c] = 1;
        }
    }
}

// ------------------------------------------------------------ host side
// Tiles of a block's slot: the leading R - 16 tile columns, all R rows each.
static int gph_slot_tiles(int N)
{
    const int R = (N + 16) / 16;
    return N < 256 ? 0 : (R - 16) * R;
}

static GphK gph_view(const JobDev& j)
{
    GphK a;
    a.m = j.m;
    a.n = j.n;
    a.N = j.N;
    a.p = j.pdim;
    a.tstop = j.tstop;
    a.seed = j.seed;
    a.jitter = j.noise_sd;
    a.y = (const double*)j.y;
    a.X = (const double*)j.X;
    a.r2 = (const double*)j.L;
    a.th = (double*)j.x;
    a.nu = (double*)j.V;
    a.lx = (double*)j.lx;
    a.phi = (double*)j.theta;
    a.pmin = (double*)j.tmin;
    a.pmax = (double*)j.tmax;
    a.logu = (double*)j.logu;
    a.k = j.k;
    a.evals = j.evals;
    a.t = j.t;
    a.budget = j.budget;
    a.out = (double*)j.out;
    a.counts = j.counts;
    a.ctr = j.ctr;
    a.maxN = j.maxN;
    a.sink = (double*)j.sink;
    a.slots = (double*)j.gslot;
    a.slot_tiles = gph_slot_tiles(j.N);
    return a;
}

int gph_max_obs() { return kGphMaxN; }
int gph_max_inputs() { return kGphMaxP; }

// Waves per block by observations: 2 NW tile rows of 16 must hold them and y's
// row, and the fewer waves (and tiles per wave) the more blocks a CU holds
// (1024 chains: n = 127 with 4 waves 0.51 ms a draw, n = 128 with 6 waves 1.25,
// with 8 waves 1.49; n = 191 1.90 with 6, 2.13 with 8).  8 waves are the most
// whose tiles fit the registers (17 tiles = 136 of 256 per lane); from 256
// observations on the leading columns go through memory.
static int gph_waves(int N) { return N < 32 ? 1 : (N < 64 ? 2 : (N < 128 ? 4 : (N < 192 ? 6 : 8))); }

// Jobs without the squared distances have up to 96 observations or 448 and more
// (gph_keeps_dist).
#define FSMMC_GPH_DISPATCH(N_, KEPT_, CALL)                              \
    switch (gph_waves(N_)) {                                            \
    case 1: if (KEPT_) { CALL(1, false, true); } else { CALL(1, false, false); } break; \
    case 2: if (KEPT_) { CALL(2, false, true); } else { CALL(2, false, false); } break; \
    case 4: if (KEPT_) { CALL(4, false, true); } else { CALL(4, false, false); } break; \
    case 6: CALL(6, false, true); break;                                \
    default:                                                            \
        if ((N_) < 256) {                                               \
            CALL(8, false, true);                                       \
        } else if (KEPT_) {                                             \
            CALL(8, true, true);                                        \
        } else {                                                        \
            CALL(8, true, false);                                       \
        }                                                               \
    }

// Blocks of the persistent kernel: what the chip holds at once, at most one per chain.
static hipError_t gph_blocks(const JobDev& j, int* blocks)
{
    int cus = 256, dev = 0, v = 0, per_cu = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
        cus = v;
    hipError_t e = hipSuccess;
#define FSMMC_GPH_OCC(NW, LEAD, KEPT) \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)gph_kernel<NW, LEAD, KEPT>, 64 * NW, 0)
    FSMMC_GPH_DISPATCH(j.N, true, FSMMC_GPH_OCC)
#undef FSMMC_GPH_OCC
    *blocks = std::max(1, std::min(j.m, cus * std::max(1, per_cu)));
    return e;
}

size_t gph_slot_bytes(const JobDev& j) { return (size_t)j.pblocks * gph_slot_tiles(j.N) * kGphTile * 8; }

size_t gph_dist_bytes(int N)
{
    const size_t R = (size_t)(N + 16) / 16;
    return R * (R + 1) / 2 * kGphTile * 8;
}

// Whether a job keeps the squared distances.  Under an HBM budget only where it then
// holds no more than the vector Cholesky before this one did (a work matrix of n
// rounded up to 32 per block above n = 96, nothing up to there; between 97 and 447 that
// is always enough), so that what fitted a budget still does; the kernels form the distances themselves otherwise
// (6 inputs: n = 25, 1024 chains x 100 draws 4.0 -> 6.1 ms, n = 63, 512 x 60 8.5 ->
// 12.2, n = 96, 1024 x 40 13.9 -> 18.7).
bool gph_keeps_dist(const JobDev& j, bool budget)
{
    const size_t ld = (size_t)(j.N + 31) / 32 * 32;
    const size_t before = j.N > 96 ? (size_t)std::min(j.m, 256) * ld * ld * 8 : 0;
    return !budget || gph_slot_bytes(j) + gph_dist_bytes(j.N) <= before;
}

// Launch shape.
hipError_t gph_setup(JobDev& j)
{
    j.pwpb = gph_waves(j.N);
    return gph_blocks(j, &j.pblocks);
}

// The squared distances (into j.L, after X is in place).
hipError_t gph_dist(const JobDev& j, hipStream_t s)
{
    const int R = (j.N + 16) / 16;
    hipLaunchKernelGGL(gph_dist_kernel, dim3(R * (R + 1) / 2), dim3(256), 0, s, (const double*)j.X, j.N, j.pdim,
                       (double*)j.L);
    return hipGetLastError();
}

hipError_t gph_init_state(const JobDev& j, const void* x0, hipStream_t s)
{
    if (x0) {
        hipError_t e = hipMemcpyAsync(j.x, x0, (size_t)j.m * 3 * 8, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
#define FSMMC_GPH_INIT(NW, LEAD, KEPT) \
    hipLaunchKernelGGL((gph_init_kernel<NW, LEAD, KEPT>), dim3(j.pblocks), dim3(64 * NW), 0, s, gph_view(j), x0 ? 1 : 0)
    FSMMC_GPH_DISPATCH(j.N, j.L != nullptr, FSMMC_GPH_INIT)
#undef FSMMC_GPH_INIT
    return hipGetLastError();
}

hipError_t gph_run(const JobDev& j, int mode, uint32_t draw, unsigned long long* ticket, hipStream_t s)
{
#define FSMMC_GPH_RUN(NW, LEAD, KEPT)                                                                       \
    hipLaunchKernelGGL((gph_kernel<NW, LEAD, KEPT>), dim3(j.pblocks), dim3(64 * NW), 0, s, gph_view(j),     \
                       (unsigned long long*)j.queue, *ticket, mode, draw)
    FSMMC_GPH_DISPATCH(j.N, j.L != nullptr, FSMMC_GPH_RUN)
#undef FSMMC_GPH_RUN
    *ticket += (unsigned long long)j.m + (unsigned long long)j.pblocks;
    return hipGetLastError();
}

}  // namespace fsmmc
