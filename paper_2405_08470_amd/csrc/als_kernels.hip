// CP-ALS dense step on the device, FP64 for every R x R quantity:
// Grams G_w = Y_w^T Y_w, the normal matrix V = Hadamard of the other Grams,
// its Cholesky factorisation and inverse, Y_d = M_d V^-1, column norms
// lambda and the CP fit.  Reductions are two-stage (block partials, then
// one ordered pass), so results do not depend on scheduling.
#include <algorithm>

#include "kernels.hpp"

// Y = M V^-1 on the FP64 matrix cores (1) or with V^-1 in LDS (0); the
// instruction's lane layout used below was measured on the device.
#ifndef SPT_SOLVE_MFMA
#define SPT_SOLVE_MFMA 1
#endif
// Grams of the caller's factors at the start of a sweep on the FP64 matrix
// cores (rank 8: the LDS kernel)
#ifndef SPT_GRAM_MFMA
#define SPT_GRAM_MFMA 1
#endif

namespace spt {

namespace {

constexpr int kGramRows = 32;

template <int R>
__global__ __launch_bounds__(256) void gram_partial_kernel(const float* __restrict__ Y, int64_t rows,
                                                           double* __restrict__ partial) {
    constexpr int E = R * R;
    constexpr int PER = (E + 255) / 256;
    __shared__ float tile[kGramRows][R];
    const int tid = threadIdx.x;
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = std::min<int64_t>(rows, (int64_t)blockIdx.x * chunk);
    const int64_t r1 = std::min<int64_t>(rows, r0 + chunk);
    double acc[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) acc[k] = 0.0;
    for (int64_t base = r0; base < r1; base += kGramRows) {
        const int nr = (int)std::min<int64_t>(kGramRows, r1 - base);
        for (int i = tid; i < kGramRows * R; i += 256) {
            const int rr = i / R, cc = i % R;
            tile[rr][cc] = rr < nr ? Y[(base + rr) * R + cc] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = tid + 256 * k;
            if (e < E) {
                const int r = e / R, c = e % R;
                double s = 0.0;
                for (int i = 0; i < nr; ++i) s += (double)tile[i][r] * (double)tile[i][c];
                acc[k] += s;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = tid + 256 * k;
        if (e < E) partial[(int64_t)blockIdx.x * E + e] = acc[k];
    }
}

// out[e] = sum over b of partial[b][e] for e < E.  Each entry is summed by
// 8 chains (b = c, c+8, ...), each with 4 interleaved accumulators, and the
// chains are combined in a fixed order.
__global__ __launch_bounds__(256) void reduce_partials_kernel(const double* __restrict__ partial,
                                                              int nblocks, int E,
                                                              double* __restrict__ out) {
    __shared__ double red[8][32];
    const int tid = threadIdx.x;
    const int el = tid % 32, c = tid / 32;
    const int e = blockIdx.x * 32 + el;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (e < E) {
        int b = c;
        for (; b + 24 < nblocks; b += 32) {
            s0 += partial[(int64_t)b * E + e];
            s1 += partial[(int64_t)(b + 8) * E + e];
            s2 += partial[(int64_t)(b + 16) * E + e];
            s3 += partial[(int64_t)(b + 24) * E + e];
        }
        for (; b < nblocks; b += 8) s0 += partial[(int64_t)b * E + e];
    }
    red[c][el] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (tid < 32 && e < E) {
        double t = 0.0;
        for (int k = 0; k < 8; ++k) t += red[k][tid];
        out[e] = t;
    }
}

// The threads that hold the R x R normal matrix: a T x T grid of the 256, each
// with P x P entries.
template <int R>
struct NormalShape {
    static constexpr int T = R < 16 ? R : 16;
    static constexpr int P = R / T;
};

// What a pivot of spd_inverse exchanges.
template <int R>
struct NormalLds {
    // the pivot's column (Cholesky), column and row (inverse), of even and odd
    // pivots: the next one is published while this one is still read
    double ccol[2][R], gcol[2][R], grow[2][R];
    double cs[R], gs[R];  // the scaled column and row
    double ridge;
};

// V = Hadamard product of the other modes' Grams; entry (i, j).
template <int R>
__device__ __forceinline__ double normal_entry(const double* __restrict__ grams, int nmodes, int mode, int i, int j) {
    double v = 1.0;
    for (int w = 0; w < nmodes; ++w)
        if (w != mode) v *= grams[(int64_t)w * R * R + i * R + j];
    return v;
}

// Cholesky (the SPD test: every pivot positive) and in-place Gauss-Jordan
// inverse (no pivoting: the pivots are the Schur complements, positive for an
// SPD matrix) of the same matrix, both in one sweep over the pivots.
//
// One workgroup of 256 threads; what bounds it is the chain of R pivots, each
// a square root, two divisions and two exchanges, not arithmetic or memory.
// So both matrices stay in registers, thread (ti, tj) of a T x T grid holding
// the entries (ti + T a, tj + T b), and a pivot exchanges only its column and
// row through LDS: one wave scales the Cholesky column while another scales
// the Gauss-Jordan row, and the threads that own the next column and row
// publish them as they update.  Every entry sees the operations of the plain
// right-looking forms in their order.  R = 64: 60 us against 237 us for
// the two factorisations one after the other with the matrix in LDS, R = 16:
// 8 against 18.8 (MI355X).
// Returns whether every Cholesky pivot was positive; the inverse is in g.
template <int R>
__device__ bool spd_inverse(double (&c)[NormalShape<R>::P * NormalShape<R>::P],
                            double (&g)[NormalShape<R>::P * NormalShape<R>::P], NormalLds<R>& l) {
    constexpr int T = NormalShape<R>::T, P = NormalShape<R>::P;
    const int tid = threadIdx.x;
    const int ti = tid / T, tj = tid % T;
    const bool on = tid < T * T;
    // pivot k = kb T + kk; publishes column k of both matrices and row k of
    // the inverse's
    auto publish = [&](int kb, int kk, int k) {
#pragma unroll
        for (int a = 0; a < P; ++a) {
            if (tj == kk) {
                l.ccol[k & 1][ti + T * a] = c[a * P + kb];
                l.gcol[k & 1][ti + T * a] = g[a * P + kb];
            }
            if (ti == kk) l.grow[k & 1][tj + T * a] = g[kb * P + a];
        }
    };
    if (on) publish(0, 0, 0);
    bool ok = true;
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < P; ++kb)
        for (int kk = 0; kk < T; ++kk) {
            const int k = kb * T + kk;
            // the pivot column of the Cholesky factor (wave 0) and the pivot
            // row of the inverse (wave 1)
            const double *ccol = l.ccol[k & 1], *gcol = l.gcol[k & 1], *grow = l.grow[k & 1];
            double d = ccol[k];
            if (!(d > 0.0)) {
                ok = false;
                d = 1.0;
            }
            if (tid < R) l.cs[tid] = ccol[tid] / sqrt(d);
            const int second = tid - 64;
            if (second >= 0 && second < R) l.gs[second] = (second == k ? 1.0 : grow[second]) / gcol[k];
            __syncthreads();
            if (on) {
                double ci[P], cj[P], gi[P], gj[P];
#pragma unroll
                for (int a = 0; a < P; ++a) {
                    ci[a] = l.cs[ti + T * a];
                    cj[a] = l.cs[tj + T * a];
                    gi[a] = gcol[ti + T * a];
                    gj[a] = l.gs[tj + T * a];
                }
                // Cholesky: entries below and right of the pivot
#pragma unroll
                for (int a = kb; a < P; ++a)
#pragma unroll
                    for (int b = kb; b <= a; ++b)
                        if ((b > kb || tj > kk) && (b < a || tj <= ti)) c[a * P + b] -= ci[a] * cj[b];
                // inverse: every row but the pivot's, whose column restarts from zero
                if (tj == kk)
#pragma unroll
                    for (int a = 0; a < P; ++a) g[a * P + kb] = 0.0;
#pragma unroll
                for (int a = 0; a < P; ++a)
#pragma unroll
                    for (int b = 0; b < P; ++b) g[a * P + b] -= gi[a] * gj[b];
                if (ti == kk)
#pragma unroll
                    for (int b = 0; b < P; ++b) g[kb * P + b] = gj[b];
                if (kk + 1 < T)
                    publish(kb, kk + 1, k + 1);
                else if (kb + 1 < P)
                    publish(kb + 1, 0, k + 1);
            }
            __syncthreads();
        }
    return ok;
}

template <int R>
__global__ __launch_bounds__(256) void normal_inverse_kernel(const double* __restrict__ grams,
                                                              int nmodes, int mode,
                                                              double* __restrict__ Vinv,
                                                              int32_t* __restrict__ status) {
    constexpr int T = NormalShape<R>::T, P = NormalShape<R>::P;
    __shared__ NormalLds<R> l;
    const int tid = threadIdx.x;
    const int ti = tid / T, tj = tid % T;
    const bool on = tid < T * T;
    double v[P * P], c[P * P], g[P * P];
#pragma unroll
    for (int e = 0; e < P * P; ++e) v[e] = on ? normal_entry<R>(grams, nmodes, mode, ti + T * (e / P), tj + T * (e % P)) : 0.0;
    bool ok = false;
    for (int attempt = 0; attempt < 2 && !ok; ++attempt) {
        if (attempt == 1) {
            // one retry with 1e-12 tr(V) / R on the diagonal
            if (on && ti == tj)
#pragma unroll
                for (int a = 0; a < P; ++a) l.cs[ti + T * a] = v[a * P + a];
            __syncthreads();
            if (tid == 0) {
                double tr = 0.0;
                for (int j = 0; j < R; ++j) tr += l.cs[j];
                l.ridge = 1e-12 * tr / R;
            }
            __syncthreads();
            const double ridge = l.ridge;
            if (on && ti == tj)
#pragma unroll
                for (int a = 0; a < P; ++a) v[a * P + a] += ridge;
            __syncthreads();
        }
#pragma unroll
        for (int e = 0; e < P * P; ++e) c[e] = g[e] = v[e];
        ok = spd_inverse<R>(c, g, l);
    }
    // a sweep starts with mode 0
    if (tid == 0) status[0] = (mode == 0 ? 0 : status[0]) | (ok ? 0 : 1);
    if (on)
#pragma unroll
        for (int e = 0; e < P * P; ++e) Vinv[(ti + T * (e / P)) * R + tj + T * (e % P)] = ok ? g[e] : 0.0;
}

// Sums the four waves' Gram tiles (c0 <= c1, register v of lane l: row 4 v +
// l / 16, column l % 16 of the tile) in a fixed order, (0 + 2) + (1 + 3), and
// writes the whole symmetric matrix to dst.  Each wave adds whole registers
// from LDS, every load issued before the first add; the waves adding into one
// LDS matrix in turn was a chain of read-modify-writes that took 18 of a
// workgroup's 34 us at R = 64.
template <int R>
struct GramTiles {
    static constexpr int CT = R / 16;
    static constexpr int NP = CT * (CT + 1) / 2;
    // doubles of LDS: two waves' tiles, then the matrix
    static constexpr int lds = 2 * NP * 256 > R * R ? 2 * NP * 256 : R * R;
};

typedef double v4d __attribute__((ext_vector_type(4)));

template <int R>
__device__ void store_block_gram(v4d (&gacc)[GramTiles<R>::NP], double* buf, double* __restrict__ dst) {
    constexpr int CT = GramTiles<R>::CT, NP = GramTiles<R>::NP;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int rl = lane & 15, q = lane >> 4;
    for (int half = 2; half >= 1; half >>= 1) {
        if (wv >= half && wv < 2 * half) {
            double* const mine = buf + (wv - half) * NP * 256 + lane;
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) mine[(4 * p + v) * 64] = gacc[p][v];
        }
        __syncthreads();
        if (wv < half) {
            const double* const other = buf + wv * NP * 256 + lane;
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) gacc[p][v] += other[(4 * p + v) * 64];
        }
        __syncthreads();
    }
    if (wv == 0) {
        int p = 0;
#pragma unroll
        for (int c0 = 0; c0 < CT; ++c0)
#pragma unroll
            for (int c1 = c0; c1 < CT; ++c1, ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * c0 + 4 * v + q, j = 16 * c1 + rl;
                    buf[i * R + j] = gacc[p][v];
                    if (c1 != c0) buf[j * R + i] = gacc[p][v];
                }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < R * R; e += 256) dst[e] = buf[e];
}

template <int R>
__global__ __launch_bounds__(256) void solve_rows_kernel(const float* __restrict__ M,
                                                          const double* __restrict__ Vinv,
                                                          int64_t rows, float* __restrict__ Y,
                                                          double* __restrict__ gpart,
                                                          double* __restrict__ ipart) {
    constexpr int RB = 256 / R;         // rows per batch
    constexpr int E = R * R;
    constexpr int PER = (E + 255) / 256;
    __shared__ double vinv[R][R];
    __shared__ float mt[RB][R];
    __shared__ float yt[RB][R];
    __shared__ double ired[RB][R];
    const int tid = threadIdx.x;
    const int bi = tid / R, col = tid % R;
    for (int e = tid; e < E; e += 256) vinv[e / R][e % R] = Vinv[e];
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = std::min<int64_t>(rows, (int64_t)blockIdx.x * chunk);
    const int64_t r1 = std::min<int64_t>(rows, r0 + chunk);
    double gacc[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) gacc[k] = 0.0;
    double iacc = 0.0;
    __syncthreads();
    for (int64_t base = r0; base < r1; base += RB) {
        const int nr = (int)std::min<int64_t>(RB, r1 - base);
        const bool valid = bi < nr;
        mt[bi][col] = valid ? M[(base + bi) * R + col] : 0.0f;
        __syncthreads();
        float yf = 0.0f;
        if (valid) {
            double y = 0.0;
#pragma unroll 8
            for (int s = 0; s < R; ++s) y += (double)mt[bi][s] * vinv[s][col];
            yf = (float)y;
            Y[(base + bi) * R + col] = yf;
            iacc += (double)mt[bi][col] * (double)yf;
        }
        yt[bi][col] = yf;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = tid + 256 * k;
            if (e < E) {
                const int r = e / R, c = e % R;
                double s = 0.0;
                for (int i = 0; i < nr; ++i) s += (double)yt[i][r] * (double)yt[i][c];
                gacc[k] += s;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = tid + 256 * k;
        if (e < E) gpart[(int64_t)blockIdx.x * (E + R) + e] = gacc[k];
    }
    ired[bi][col] = iacc;
    __syncthreads();
    if (tid < R) {
        double s = 0.0;
        for (int i = 0; i < RB; ++i) s += ired[i][tid];
        ipart[(int64_t)blockIdx.x * (E + R) + tid] = s;
    }
}

// Y = M V^-1 on the FP64 matrix cores (v_mfma_f64_16x16x4f64), for R a
// multiple of 16.  Each wave takes 16-row tiles.  Operand layout of the
// instruction on gfx950 (wave64, checked on the device): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] of a 16x4 by 4x16 step, and
// register v (0..3) of lane l holds D[4 v + l / 16][l % 16] of the 16x16
// result.  The contraction index k of step s for lane group q = l / 16 is
// k = q R/4 + s, so a lane's A values are R/4 consecutive columns of its row
// of M (vector loads) and its B values are the matching rows of V^-1 (held
// in registers for the whole kernel).  The rounded FP32 result feeds the
// Gram of the unnormalised factor with no data movement: for fixed v, the
// four rows 4 v + q of a tile are the k index of one more step, A = column
// tile c0 and B = column tile c1 of those rows.  <M, Y> per column (for the
// fit) is summed in FP64 per lane.
template <int R>
__global__ __launch_bounds__(256) void solve_rows_mfma_kernel(const float* __restrict__ M,
                                                               const double* __restrict__ Vinv,
                                                               int64_t rows, float* __restrict__ Y,
                                                               double* __restrict__ gpart,
                                                               double* __restrict__ ipart) {
    static_assert(R % 16 == 0, "rank");
    constexpr int CT = R / 16;             // column tiles
    constexpr int KS = R / 4;              // steps of the solve
    constexpr int NP = CT * (CT + 1) / 2;  // Gram tiles c0 <= c1
    constexpr int E = R * R;
    __shared__ double buf[GramTiles<R>::lds];
    __shared__ double ish[4][4][R];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int rl = lane & 15, q = lane >> 4;

    double bv[CT][KS];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int s = 0; s < KS; ++s) bv[ct][s] = Vinv[(q * KS + s) * R + 16 * ct + rl];
    v4d gacc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) gacc[p] = v4d{0.0, 0.0, 0.0, 0.0};
    double iacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) iacc[ct] = 0.0;

    const int64_t tiles = (rows + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t r0 = tile * 16;
        // every load of the tile is issued before any of it is used: the
        // lane's A values, and M at the lane's result positions for <M, Y>
        float av[KS];
        float mv[CT][4];
        const int64_t ra = r0 + rl;
        if (ra < rows) {
            const float4* src = reinterpret_cast<const float4*>(M + ra * R + q * KS);
#pragma unroll
            for (int j = 0; j < KS / 4; ++j) {
                const float4 x = src[j];
                av[4 * j] = x.x;
                av[4 * j + 1] = x.y;
                av[4 * j + 2] = x.z;
                av[4 * j + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < KS; ++j) av[j] = 0.0f;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = r0 + 4 * v + q;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) mv[ct][v] = row < rows ? M[row * R + 16 * ct + rl] : 0.0f;
        }
        v4d acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[s], bv[ct][s], acc[ct], 0, 0, 0);
        double yd[CT][4];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = r0 + 4 * v + q;
                const int col = 16 * ct + rl;
                double y = 0.0;
                if (row < rows) {
                    const float yf = (float)acc[ct][v];
                    Y[row * R + col] = yf;
                    y = (double)yf;
                    iacc[ct] += (double)mv[ct][v] * y;
                }
                yd[ct][v] = y;
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int p = 0;
#pragma unroll
            for (int c0 = 0; c0 < CT; ++c0)
#pragma unroll
                for (int c1 = c0; c1 < CT; ++c1, ++p)
                    gacc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(yd[c0][v], yd[c1][v], gacc[p], 0, 0, 0);
        }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) ish[wv][q][16 * ct + rl] = iacc[ct];
    store_block_gram<R>(gacc, buf, gpart + (int64_t)blockIdx.x * (E + R));
    if (threadIdx.x < R) {
        const int c = threadIdx.x;
        double t = 0.0;
        for (int w = 0; w < 4; ++w)
            for (int g = 0; g < 4; ++g) t += ish[w][g][c];
        ipart[(int64_t)blockIdx.x * (E + R) + c] = t;
    }
}

// Partial Grams Y^T Y on the FP64 matrix cores (R a multiple of 16): each
// wave takes 16-row tiles; lane (rl = lane % 16, q = lane / 16) holds
// Y(r0 + 4v + q, 16c + rl), which is both the A operand (column tile c0 of
// Y^T) and the B operand (column tile c1 of Y) of v_mfma_f64_16x16x4f64 for
// the 4 rows r0 + 4v .. r0 + 4v + 3.  The block writes partial[blockIdx][R*R].
template <int R>
__global__ __launch_bounds__(256) void gram_mfma_kernel(const float* __restrict__ Y, int64_t rows,
                                                         double* __restrict__ partial) {
    static_assert(R % 16 == 0, "rank");
    constexpr int CT = R / 16;
    constexpr int NP = CT * (CT + 1) / 2;
    __shared__ double buf[GramTiles<R>::lds];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int rl = lane & 15, q = lane >> 4;
    v4d gacc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) gacc[p] = v4d{0.0, 0.0, 0.0, 0.0};
    const int64_t tiles = (rows + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t r0 = tile * 16;
        double yd[CT][4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = r0 + 4 * v + q;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) yd[ct][v] = row < rows ? (double)Y[row * R + 16 * ct + rl] : 0.0;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int p = 0;
#pragma unroll
            for (int c0 = 0; c0 < CT; ++c0)
#pragma unroll
                for (int c1 = c0; c1 < CT; ++c1, ++p)
                    gacc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(yd[c0][v], yd[c1][v], gacc[p], 0, 0, 0);
        }
    }
    store_block_gram<R>(gacc, buf, partial + (int64_t)blockIdx.x * R * R);
}

template <int R>
__global__ __launch_bounds__(256) void als_finish_kernel(const double* __restrict__ Gun,
                                                          const double* __restrict__ Isum,
                                                          int nmodes, int mode,
                                                          double* __restrict__ grams,
                                                          double* __restrict__ lambda,
                                                          double normX2, int want_fit,
                                                          double* __restrict__ fit) {
    constexpr int E = R * R;
    __shared__ double lam[R];
    __shared__ double red[256], red16[16], isum[R];
    const int tid = threadIdx.x;
    if (tid < R) {
        isum[tid] = Isum[tid];
        lam[tid] = sqrt(Gun[tid * R + tid]);
        lambda[tid] = lam[tid];
    }
    __syncthreads();
    double* Gm = grams + (int64_t)mode * E;
    for (int e = tid; e < E; e += 256) {
        const int r = e / R, c = e % R;
        const double lr = lam[r], lc = lam[c];
        Gm[e] = (lr > 0.0 && lc > 0.0) ? Gun[e] / (lr * lc) : 0.0;
    }
    if (!want_fit) return;
    __syncthreads();
    // ||Xhat||^2 = lam^T (Hadamard of all Grams) lam, in a fixed order
    double xh = 0.0;
    for (int e = tid; e < E; e += 256) {
        const int r = e / R, c = e % R;
        double h = 1.0;
        for (int w = 0; w < nmodes; ++w) h *= grams[(int64_t)w * E + e];
        xh += lam[r] * h * lam[c];
    }
    red[tid] = xh;
    __syncthreads();
    // 16 sums of 16, then their sum: one chain of 256 dependent LDS reads was
    // most of this kernel's time
    if (tid < 16) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) t += red[16 * tid + i];
        red16[tid] = t;
    }
    __syncthreads();
    if (tid == 0) {
        double x = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) x += red16[i];
        double in = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) in += isum[r];
        double res2 = normX2 + x - 2.0 * in;
        if (res2 < 0.0) res2 = 0.0;
        fit[0] = 1.0 - sqrt(res2) / sqrt(normX2);
    }
}

// Y(i, c) / lambda_c in FP64, rounded once; 4 columns (one 16-byte word) per
// thread, the grid covering the matrix in one sweep where it can.
template <int R>
__global__ void scale_cols_kernel(float* __restrict__ Y, int64_t rows,
                                  const double* __restrict__ lambda) {
    static_assert(R % 4 == 0, "rank");
    const int64_t total4 = rows * (R / 4);
    float4* Y4 = reinterpret_cast<float4*>(Y);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total4;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % (R / 4)) * 4;
        float4 y = Y4[i];
        const double l0 = lambda[c], l1 = lambda[c + 1], l2 = lambda[c + 2], l3 = lambda[c + 3];
        y.x = l0 > 0.0 ? (float)((double)y.x / l0) : 0.0f;
        y.y = l1 > 0.0 ? (float)((double)y.y / l1) : 0.0f;
        y.z = l2 > 0.0 ? (float)((double)y.z / l2) : 0.0f;
        y.w = l3 > 0.0 ? (float)((double)y.w / l3) : 0.0f;
        Y4[i] = y;
    }
}

template <template <int> class K, typename... Args>
void by_rank(int rank, dim3 grid, dim3 block, hipStream_t s, Args... args) {
    switch (rank) {
        case 8: hipLaunchKernelGGL(K<8>::fn, grid, block, 0, s, args...); break;
        case 16: hipLaunchKernelGGL(K<16>::fn, grid, block, 0, s, args...); break;
        case 32: hipLaunchKernelGGL(K<32>::fn, grid, block, 0, s, args...); break;
        case 64: hipLaunchKernelGGL(K<64>::fn, grid, block, 0, s, args...); break;
        default: break;
    }
}

template <int R> struct GramP { static constexpr auto fn = gram_partial_kernel<R>; };
template <int R> struct GramMfma { static constexpr auto fn = gram_mfma_kernel<R>; };
template <> struct GramMfma<8> { static constexpr auto fn = gram_partial_kernel<8>; };
template <int R> struct NormInv { static constexpr auto fn = normal_inverse_kernel<R>; };
template <int R> struct Solve { static constexpr auto fn = solve_rows_kernel<R>; };
template <int R> struct SolveMfma { static constexpr auto fn = solve_rows_mfma_kernel<R>; };
template <> struct SolveMfma<8> { static constexpr auto fn = solve_rows_kernel<8>; };
template <int R> struct Finish { static constexpr auto fn = als_finish_kernel<R>; };
template <int R> struct Scale { static constexpr auto fn = scale_cols_kernel<R>; };

}  // namespace

// One 16-row tile per wave up to 65536 rows: below that the kernels wait on
// latency, not on the partials' reduction (R 64, 12007 rows: 34 us with 4
// tiles per wave, 14 with one).
int gram_blocks(int64_t rows) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(1024, (rows + 63) / 64));
}

void launch_gram_partial(int rank, const float* Y, int64_t rows, double* partial, hipStream_t s) {
#if SPT_GRAM_MFMA
    by_rank<GramMfma>(rank, dim3(gram_blocks(rows)), dim3(256), s, Y, rows, partial);
#else
    by_rank<GramP>(rank, dim3(gram_blocks(rows)), dim3(256), s, Y, rows, partial);
#endif
}

void launch_reduce_partials(const double* partial, int nblocks, int E, double* out, hipStream_t s) {
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((E + 31) / 32), dim3(256), 0, s, partial, nblocks,
                       E, out);
}

void launch_normal_inverse(int rank, int nmodes, int mode, const double* grams, double* Vinv,
                           int32_t* status, hipStream_t s) {
    by_rank<NormInv>(rank, dim3(1), dim3(256), s, grams, nmodes, mode, Vinv, status);
}

int solve_blocks(int64_t rows) { return gram_blocks(rows); }

void launch_solve_rows(int rank, const float* M, const double* Vinv, int64_t rows, float* Y,
                       double* gpart, double* ipart, hipStream_t s) {
#if SPT_SOLVE_MFMA
    by_rank<SolveMfma>(rank, dim3(solve_blocks(rows)), dim3(256), s, M, Vinv, rows, Y, gpart, ipart);
#else
    by_rank<Solve>(rank, dim3(solve_blocks(rows)), dim3(256), s, M, Vinv, rows, Y, gpart, ipart);
#endif
}

void launch_als_finish(int rank, int nmodes, int mode, const double* Gun, const double* Isum,
                       double* grams, double* lambda, double normX2, int want_fit, double* fit,
                       hipStream_t s) {
    by_rank<Finish>(rank, dim3(1), dim3(256), s, Gun, Isum, nmodes, mode, grams, lambda, normX2,
                    want_fit, fit);
}

void launch_scale_cols(int rank, float* Y, int64_t rows, const double* lambda, hipStream_t s) {
    const int64_t total4 = rows * (rank / 4);
    if (total4 == 0) return;
    const int64_t blocks = std::min<int64_t>((total4 + 255) / 256, int64_t(1) << 20);
    by_rank<Scale>(rank, dim3((unsigned)blocks), dim3(256), s, Y, rows, lambda);
}

}  // namespace spt
