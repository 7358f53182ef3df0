// Fused elementwise computation (Alg. 2) and dynamic remapping (Alg. 3) for
// one output mode, mapped to gfx950 wavefronts (the role of Alg. 4).
//
// One workgroup = one partition B_{d,z} of Alg. 1, in S waves of 64 lanes (S
// chosen by the launch: 1 where the partitions alone fill the chip).  A
// nonzero is handled by L = R/4 lanes, each holding 4 consecutive ranks (one
// 16-byte load per gathered factor row per lane, so a row of R FP32 values
// arrives in one request).  The workgroup splits its partition into S*G
// contiguous sub-ranges, G = 64/L, one per lane group; a group walks its
// sub-range in stream order, so runs of equal output row (the stream is
// grouped by row) are summed in registers and each finished row is stored
// once.  A row that crosses a sub-range boundary is finished by a short chain
// combine in LDS at the end.  Rows split across partitions (pieces, see the
// planner) go to a carry slot instead, summed later by the fixup kernel.  No
// atomics.
//
// Records are fetched one step ahead, one per lane (software pipeline),
// which is also where each record is written to its remap position in the
// next mode's stream (Alg. 3).  Each lane decodes the record it fetched into
// its wave's part of LDS once; the gathers of several nonzeros are issued
// before any of them is consumed.  The waves of a workgroup meet only before
// and after their walks.
#pragma once

#include <algorithm>
#include <utility>

#include "kernels.hpp"
#include "record.hpp"

// float4 gathers a lane keeps in flight (register budget of the batch)
#ifndef SPT_GATHER_INFLIGHT
#define SPT_GATHER_INFLIGHT 16
#endif
namespace spt {
namespace {

// Index of mode W in a record (layout kinds of the planner).
template <int W, int RW, int KIND>
__device__ __forceinline__ uint32_t decode(const Rec<RW>& r, const EcArgs& a) {
    if constexpr (KIND == kWord32) {
        return rword<W, RW>(r);
    } else if constexpr (KIND == kHalf16) {
        return (rword<W / 2, RW>(r) >> ((W & 1) * 16)) & 0xFFFFu;
    } else {  // bit fields in the first 64 bits (12-byte record) or 96 bits (16-byte)
        const uint64_t lo = ((uint64_t)rword<1, RW>(r) << 32) | rword<0, RW>(r);
        const int o = a.foff[W];
        if constexpr (RW == 3) {
            return (uint32_t)(lo >> o) & a.fmask[W];
        } else {
            const uint64_t hi = rword<2, RW>(r);
            const uint64_t x = o >= 64 ? (hi >> (o - 64)) : ((lo >> o) | (o ? (hi << (64 - o)) : 0));
            return (uint32_t)x & a.fmask[W];
        }
    }
}

// Orders a wave's LDS accesses before and after it (the waves of a workgroup
// keep their own staging, so no workgroup barrier is needed).  LDS accesses of
// one wave are carried out in order, so this only holds the compiler.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The record's indices into column `at` of the staging rows st[mode].
template <int RW, int KIND, int WIDTH, int... W>
__device__ __forceinline__ void decode_all(const Rec<RW>& r, const EcArgs& a, uint32_t (*st)[WIDTH],
                                           int at, std::integer_sequence<int, W...>) {
    ((st[W][at] = decode<W, RW, KIND>(r, a)), ...);
}

// Carry slot of `row` if it is a split row of this partition, else -1.
__device__ __forceinline__ int split_slot(const EcArgs& a, int sp0, int sp1, int row) {
    int slot = -1;
    for (int j = sp0; j < sp1; ++j)
        if (a.psplit_row[j] == row) slot = a.psplit_slot[j];
    return slot;
}

template <int R>
__device__ __forceinline__ float* row_dst(const EcArgs& a, int row, int slot) {
    return slot >= 0 ? a.carry + (int64_t)slot * R : a.out + (int64_t)row * R;
}

// Factor element types.  A lane loads 16 bytes of a factor row at a time:
// 4 FP32 values, or 8 BF16 values (raw 16-bit patterns, widened exactly).
struct FacF32 {
    static constexpr int kPerLoad = 4;
    static constexpr int kBytes = 4;
};
struct FacBF16 {
    static constexpr int kPerLoad = 8;
    static constexpr int kBytes = 2;
};

template <typename FT>
__device__ __forceinline__ void widen(const uint4& u, float (&f)[FT::kPerLoad]) {
    if constexpr (FT::kPerLoad == 4) {
        f[0] = __uint_as_float(u.x);
        f[1] = __uint_as_float(u.y);
        f[2] = __uint_as_float(u.z);
        f[3] = __uint_as_float(u.w);
    } else {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
}

template <int V>
__device__ __forceinline__ void store_vals(float* dst, const float (&v)[V]) {
#pragma unroll
    for (int i = 0; i < V; i += 4)
        *reinterpret_cast<float4*>(dst + i) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
}

// REUSE: the last gathered mode's row (mode d-1, the second key of mode d's
// stream order, so consecutive nonzeros often share it) is fetched once per
// run of consecutive nonzeros that share it and their output row and kept in
// registers; every nonzero still multiplies it into its product in the same
// order, so both forms give the same bits.  Without REUSE every nonzero
// fetches all its gathered rows.  REUSE costs registers and a branch per
// nonzero; the launch says where it is taken.
//
// What bounds it: with rows in reach of the caches, the 64 bytes a clock each
// CU's L1 returns (74 GB of gathered rows per launch at 4 modes, 1e8 nonzeros,
// R 64, in 2.28-2.49 ms: 30-32 TB/s; 2.40-2.88 ms with one wave per
// workgroup); on the 3-mode 8e7 tensor, line fetches beyond L2 (0.90-0.95 ms,
// before 0.98-1.0); on small tensors, the chain ptr -> record -> gather ->
// store, which more waves per partition shorten (launch choice).
// What a lane group left to the chain combine: a row that starts in it runs on
// past its sub-range; a row from an earlier group ends in it; ... and ends
// before the group's last nonzero (the head partial holds its end).
// (kMoved, during the walk of the ordered form: past the sub-range's first row)
constexpr int kStarts = 1, kEnds = 2, kHead = 4, kMoved = 8;

// Chain combine: a row that runs on past its group's sub-range is summed in
// group order by the threads (one per rank) of the group it starts in, whose
// tail partial opens the chain; a group with no head partial is covered by the
// row as a whole.  Every chain is walked at once, eight groups' flags and
// partials read ahead of their use, so a workgroup of many groups waits for
// its longest row only.
template <int R>
__device__ __forceinline__ void combine_chains(const EcArgs& a, const float* part0, const float* part1,
                                               const int32_t* gflag, const int32_t* prow, const int32_t* pslot,
                                               int groups) {
    for (int i = threadIdx.x; i < groups * R; i += blockDim.x) {
        const int h = i / R, r = i % R;
        if (!(gflag[h] & kStarts)) continue;
        float csum = part1[i];
        bool open = true;
        for (int k = h + 1; open; k += 8) {
            int f[8];
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = k + j < groups ? k + j : groups - 1;
                f[j] = gflag[c];
                v[j] = part1[c * R + r];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (open) {
                    csum += (f[j] & kHead) ? part0[(k + j) * R + r] : v[j];
                    open = !(f[j] & kEnds);
                }
            }
        }
        row_dst<R>(a, prow[h], pslot[h])[r] = csum;
    }
}

template <int N, int R, typename FT>
struct EcShape {
    static constexpr int V = FT::kPerLoad;
    static constexpr int L = R / V;      // lanes per nonzero
    static constexpr int G = 64 / L;     // lane groups of a wave = nonzeros in flight
    static constexpr int SW = N + 2;     // staged words per nonzero: indices in mode order, value, carry slot
};

template <int N, int R, int RW, int KIND, typename FT, bool REUSE, int K>
__global__ __launch_bounds__(64 * kEcMaxWaves) void ec_kernel(const EcArgs a) {
    using Sh = EcShape<N, R, FT>;
    constexpr int V = Sh::V;
    constexpr int L = Sh::L;
    constexpr int G = Sh::G;
    constexpr int NG = N - 1;    // gathered factor rows per nonzero
    constexpr int J = K * L;     // nonzeros per group and step: a lane stages K records
    // nonzeros whose gathers are issued together: the largest power-of-two
    // part of J with at most SPT_GATHER_INFLIGHT float4 gathers in flight per lane
    constexpr int BMAX = (SPT_GATHER_INFLIGHT / NG) > 0 ? SPT_GATHER_INFLIGHT / NG : 1;
    constexpr int B = J <= BMAX ? J : (J / 2 <= BMAX ? J / 2 : (J / 4 <= BMAX ? J / 4 : (J / 8 <= BMAX ? J / 8 : 1)));
    static_assert(R % V == 0 && L >= 1 && 64 % L == 0 && J % B == 0, "rank");
    constexpr int SW = Sh::SW;
    constexpr int MAXSPLIT = kEcMaxSplit;

    const int SG = a.waves * G;  // lane groups of the workgroup
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;

    // LDS, in the order ec_lds_bytes counts it
    HIP_DYNAMIC_SHARED(uint4, smem)
    float* const part0 = reinterpret_cast<float*>(smem);  // head partials of the groups
    float* const part1 = part0 + SG * R;                  // tail partials
    uint32_t(*const stage)[64 * K] = reinterpret_cast<uint32_t(*)[64 * K]>(part1 + SG * R) + wv * SW;
    int32_t* const prow = reinterpret_cast<int32_t*>(part1 + SG * R) + a.waves * SW * 64 * K;  // row of the tail partial
    int32_t* const pslot = prow + SG;        // its carry slot
    int32_t* const gflag = pslot + SG;       // after the walk: kStarts, kEnds, kHead
    uint32_t(*const brow)[2] = reinterpret_cast<uint32_t(*)[2]>(gflag + SG);  // rows before and after a sub-range
    int32_t* const srow = gflag + 3 * SG + wv * 2 * MAXSPLIT;                 // the wave's copy of the split rows
    int32_t* const sslot = srow + MAXSPLIT;

    const int z = blockIdx.x;
    const int gl = lane / L;                 // group within the wave
    const int g = wv * G + gl;
    const int li = lane % L;
    const int64_t s = a.ptr[z];
    const int64_t n = a.ptr[z + 1] - s;
    if (n == 0) return;
    const int sp0 = a.psplit_ptr[z], sp1 = a.psplit_ptr[z + 1];
    const int nsp = sp1 - sp0;
    const bool sp_lds = nsp <= MAXSPLIT;
    const int mode = a.rot[0];
    constexpr auto seq = std::make_integer_sequence<int, N>{};

    const int64_t q = n / SG, rm = n % SG;
    const int64_t gs = s + g * q + (g < rm ? g : rm);
    const int gn = (int)(q + (g < rm ? 1 : 0));
    const int64_t ge = gs + gn;

    // The first records, the rows on either side of the group's sub-range and
    // the split rows are fetched together: one round trip before the walk.
    const bool remap_inline = a.rec_out != nullptr;
    // the records of one step: lane li takes nonzeros li, L + li, ... of its group
    struct Step {
        Rec<RW> rec[K];
        int32_t nxt[K];
    };
    Step sa, sb;
    auto fetch = [&](int step0, Step& to) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (step0 + k * L + li < gn) {
                load_rec<RW>(a.rec_in, gs + step0 + k * L + li, to.rec[k]);
                if (remap_inline) to.nxt[k] = a.nxt[gs + step0 + k * L + li];
            }
    };
    fetch(0, sa);
    if (sp_lds && lane < nsp) {
        srow[lane] = a.psplit_row[sp0 + lane];
        sslot[lane] = a.psplit_slot[sp0 + lane];
    }
    for (int j = li; j < 2; j += L) {
        const int64_t p = j == 0 ? gs - 1 : ge;
        uint32_t row = 0xFFFFFFFFu;
        if (gn > 0 && p >= s && p < s + n) {
            Rec<RW> r;
            load_rec<RW>(a.rec_in, p, r);
            decode_all<RW, KIND>(r, a, stage, lane, seq);
            row = stage[mode][lane];
        }
        brow[g][j] = row;
    }
    if (li == 0) gflag[g] = 0;
    wave_sync();
    const uint32_t before = brow[g][0], after = brow[g][1];

    // acc: the output row's sum so far; ylast (REUSE): the last gathered
    // mode's row of the current run of equal (output row, last gathered row)
    float acc[V], ylast[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        acc[v] = 0.0f;
        ylast[v] = 0.0f;
    }
    int cur_row = -1, cur_slot = -1;
    uint32_t cur_lrow = 0xFFFFFFFFu;  // last gathered mode's row of the current run
    bool first_seg = true;  // still in the sub-range's first row
    const int steps = (int)(q + (rm > 0 ? 1 : 0));

    // carry slot of a row of this partition (-1: not a split row)
    auto slot_of = [&](int row) {
        int slot = -1;
        if (sp_lds) {
            for (int j = 0; j < nsp; ++j)
                if (srow[j] == row) slot = sslot[j];
        } else {
            slot = split_slot(a, sp0, sp1, row);
        }
        return slot;
    };

    // One step: commit the record fetched for this step (remap store,
    // decode), prefetch the next step's record into the other buffer after
    // the first gathers, then run the lane groups over their L nonzeros of
    // this step.  Two record buffers alternate, so a prefetch never
    // overwrites the registers of a remap store still in flight.
    auto step = [&](int step0, Step& cur, Step& next) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (step0 + k * L + li < gn) {
                const int at = k * 64 + lane;
                if (remap_inline) store_rec<RW>(a.rec_out, cur.nxt[k], cur.rec[k]);
                decode_all<RW, KIND>(cur.rec[k], a, stage, at, seq);
                stage[N][at] = rword<RW - 1, RW>(cur.rec[k]);
                stage[N + 1][at] = (uint32_t)slot_of((int)stage[mode][at]);
            }
        wave_sync();
        const int cnt = gn - step0;
        #pragma unroll
        for (int kb = 0; kb < J; kb += B) {
            // the batch's rows first (one LDS wait for all of them), then its
            // gathers back to back; a nonzero past the group's range gathers
            // row 0 (always a valid row) instead of branching around the load
            uint32_t orow[B], rix[B][NG];
            #pragma unroll
            for (int b = 0; b < B; ++b) {
                const int slot = (kb + b) / L * 64 + gl * L + (kb + b) % L;
                orow[b] = stage[mode][slot];
                #pragma unroll
                for (int k = 0; k < NG; ++k) rix[b][k] = stage[a.rot[k + 1]][slot];
            }
            // the last gathered mode's row is fetched only where a run of
            // equal (output row, last gathered row) starts: the same test the
            // accumulation below makes, against the previous nonzero
            bool fresh[B];
            #pragma unroll
            for (int b = 0; b < B; ++b) {
                const uint32_t po = b == 0 ? (uint32_t)cur_row : orow[b - 1];
                const uint32_t pl = b == 0 ? cur_lrow : rix[b - 1][NG - 1];
                fresh[b] = !REUSE || orow[b] != po || rix[b][NG - 1] != pl;
            }
            uint4 y[B][NG];
            #pragma unroll
            for (int b = 0; b < B; ++b) {
                const bool live = kb + b < cnt;
                #pragma unroll
                for (int k = 0; k < NG; ++k) {
                    const uint4* src = reinterpret_cast<const uint4*>(
                        static_cast<const char*>(a.fac[k + 1]) +
                        ((int64_t)(live ? rix[b][k] : 0u) * R + li * V) * FT::kBytes);
                    if (!REUSE || k < NG - 1) {
                        y[b][k] = *src;
                    } else if (live && fresh[b]) {
                        y[b][k] = *src;
                    }
                }
            }
            if (kb == 0) fetch(step0 + J, next);
            #pragma unroll
            for (int b = 0; b < B; ++b) {
                if (kb + b < cnt) {
                    const int slot = (kb + b) / L * 64 + gl * L + (kb + b) % L;
                    const int row = (int)orow[b];
                    if (REUSE && fresh[b]) {
                        widen<FT>(y[b][NG - 1], ylast);
                        cur_lrow = rix[b][NG - 1];
                    }
                    if (row != cur_row) {
                        if (cur_row >= 0) {
                            if (first_seg && before == (uint32_t)cur_row) {
                                store_vals<V>(part0 + g * R + li * V, acc);
                                // (this write also keeps the two stores
                                // apart: merged, they would be one store to
                                // either memory, and every wait for a gather
                                // a wait for all of them)
                                if (li == 0) gflag[g] = kHead;
                            } else {
                                store_vals<V>(row_dst<R>(a, cur_row, cur_slot) + li * V, acc);
                            }
                            first_seg = false;
                        }
                        cur_row = row;
                        cur_slot = (int)stage[N + 1][slot];
                        #pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = 0.0f;
                    }
                    const float val = __uint_as_float(stage[N][slot]);
                    if constexpr (REUSE) {
                        // the product of the gathered rows in mode order, the
                        // last one from the registers of its run
                        float prod[V];
                        if constexpr (NG == 1) {
                            #pragma unroll
                            for (int v = 0; v < V; ++v) prod[v] = ylast[v];
                        } else {
                            widen<FT>(y[b][0], prod);
                            #pragma unroll
                            for (int k = 1; k < NG - 1; ++k) {
                                float f[V];
                                widen<FT>(y[b][k], f);
                                #pragma unroll
                                for (int v = 0; v < V; ++v) prod[v] *= f[v];
                            }
                            #pragma unroll
                            for (int v = 0; v < V; ++v) prod[v] *= ylast[v];
                        }
                        #pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fmaf(prod[v], val, acc[v]);
                    } else {
                        float prod[V];
                        widen<FT>(y[b][0], prod);
                        #pragma unroll
                        for (int k = 1; k < NG; ++k) {
                            float f[V];
                            widen<FT>(y[b][k], f);
                            #pragma unroll
                            for (int v = 0; v < V; ++v) prod[v] *= f[v];
                        }
                        #pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fmaf(prod[v], val, acc[v]);
                    }
                }
            }
        }
        wave_sync();
    };
    for (int t = 0; t < steps; t += 2 * J) {
        step(t, sa, sb);
        if (t + J < steps) step(t + J, sb, sa);
    }

    // the group's last segment
    const bool open_right = cur_row >= 0 && after == (uint32_t)cur_row;
    const bool cont = first_seg && before == (uint32_t)cur_row;  // the whole sub-range inside one longer row
    if (cur_row >= 0) {
        if (open_right || cont) {
            store_vals<V>(part1 + g * R + li * V, acc);
            if (li == 0) {
                prow[g] = cur_row;
                pslot[g] = cur_slot;
            }
        } else {
            store_vals<V>(row_dst<R>(a, cur_row, cur_slot) + li * V, acc);
        }
    }
    if (li == 0) {
        const int head = gflag[g];  // kHead: a row from an earlier group ended inside this one
        gflag[g] = head | (open_right && !cont ? kStarts : 0) | (head || !open_right ? kEnds : 0);
    }
    __syncthreads();

    combine_chains<R>(a, part0, part1, gflag, prow, pslot, SG);
}

// The sums of one wave per partition, bit for bit, with the gathers of `waves`
// waves in flight: the partition is split over the G lane groups as one wave
// splits it, and the waves take turns of B nonzeros per group.  A wave gathers
// its next turn while the others have theirs; at its turn it adds its products
// to the groups' running sums, which pass from wave to wave through LDS, with
// one barrier per turn.  For CP-ALS on tensors whose partitions do not fill the
// chip, where a lone wave's chain of gathers is the kernel.  Plain form, no
// remap inside.
template <int N, int R, int RW, int KIND, typename FT>
__global__ __launch_bounds__(64 * kEcMaxWaves) void ec_ordered_kernel(const EcArgs a) {
    using Sh = EcShape<N, R, FT>;
    constexpr int V = Sh::V, L = Sh::L, G = Sh::G, SW = Sh::SW;
    constexpr int NG = N - 1;
    constexpr int BMAX = (SPT_GATHER_INFLIGHT / NG) > 0 ? SPT_GATHER_INFLIGHT / NG : 1;
    constexpr int B = L <= BMAX ? L : (L / 2 <= BMAX ? L / 2 : (L / 4 <= BMAX ? L / 4 : (L / 8 <= BMAX ? L / 8 : 1)));
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int S = a.waves;

    // LDS, within what ec_lds_bytes counts for the waves' own groups
    HIP_DYNAMIC_SHARED(uint4, smem)
    float* const part0 = reinterpret_cast<float*>(smem);  // head partials of the groups
    float* const part1 = part0 + G * R;                   // tail partials
    float* const sums = part1 + G * R;                    // running sums [64 lanes][V] ...
    int32_t* const prow = reinterpret_cast<int32_t*>(sums + 64 * V);
    int32_t* const pslot = prow + G;
    int32_t* const gflag = pslot + G;
    int32_t* const crow = gflag + G;                      // ... their rows and slots
    int32_t* const cslot = crow + G;
    uint32_t(*const stage)[64] = reinterpret_cast<uint32_t(*)[64]>(cslot + G) + wv * SW;
    int32_t* const srow = cslot + G + S * SW * 64 + wv * 2 * kEcMaxSplit;
    int32_t* const sslot = srow + kEcMaxSplit;

    const int z = blockIdx.x;
    const int g = lane / L;
    const int li = lane % L;
    const int64_t s = a.ptr[z];
    const int64_t n = a.ptr[z + 1] - s;
    if (n == 0) return;
    const int sp0 = a.psplit_ptr[z], sp1 = a.psplit_ptr[z + 1];
    const int nsp = sp1 - sp0;
    const bool sp_lds = nsp <= kEcMaxSplit;
    const int mode = a.rot[0];
    constexpr auto seq = std::make_integer_sequence<int, N>{};

    const int64_t q = n / G, rm = n % G;
    const int64_t gs = s + g * q + (g < rm ? g : rm);
    const int gn = (int)(q + (g < rm ? 1 : 0));
    const int64_t ge = gs + gn;
    const int rounds = (int)((q + (rm > 0 ? 1 : 0) + B * S - 1) / (B * S));

    Rec<RW> rec;
    if (li < B && wv * B + li < gn) load_rec<RW>(a.rec_in, gs + wv * B + li, rec);
    if (sp_lds && lane < nsp) {
        srow[lane] = a.psplit_row[sp0 + lane];
        sslot[lane] = a.psplit_slot[sp0 + lane];
    }
    // the rows before and after the group's sub-range (every wave fetches them)
    uint32_t before = 0xFFFFFFFFu, after = 0xFFFFFFFFu;
    if (gn > 0 && gs > s) {
        Rec<RW> r;
        load_rec<RW>(a.rec_in, gs - 1, r);
        decode_all<RW, KIND>(r, a, stage, lane, seq);
        before = stage[mode][lane];
    }
    if (gn > 0 && ge < s + n) {
        Rec<RW> r;
        load_rec<RW>(a.rec_in, ge, r);
        decode_all<RW, KIND>(r, a, stage, lane, seq);
        after = stage[mode][lane];
    }
    if (wv == 0 && li == 0) {
        gflag[g] = 0;
        crow[g] = -1;
    }
    auto slot_of = [&](int row) {
        int slot = -1;
        if (sp_lds) {
            for (int j = 0; j < nsp; ++j)
                if (srow[j] == row) slot = sslot[j];
        } else {
            slot = split_slot(a, sp0, sp1, row);
        }
        return slot;
    };
    wave_sync();

    // stages the turn whose records are in `rec`, issues its gathers and the
    // next turn's record load
    uint4 y[B][NG];
    auto prepare = [&](int step0) {
        if (li < B && step0 + li < gn) {
            decode_all<RW, KIND>(rec, a, stage, lane, seq);
            stage[N][lane] = rword<RW - 1, RW>(rec);
            stage[N + 1][lane] = (uint32_t)slot_of((int)stage[mode][lane]);
        }
        wave_sync();
        uint32_t rix[B][NG];
        #pragma unroll
        for (int b = 0; b < B; ++b)
            #pragma unroll
            for (int k = 0; k < NG; ++k) rix[b][k] = stage[a.rot[k + 1]][g * L + b];
        #pragma unroll
        for (int b = 0; b < B; ++b)
            #pragma unroll
            for (int k = 0; k < NG; ++k)
                // a nonzero past the group's range gathers row 0
                y[b][k] = *reinterpret_cast<const uint4*>(
                    static_cast<const char*>(a.fac[k + 1]) +
                    ((int64_t)(step0 + b < gn ? rix[b][k] : 0u) * R + li * V) * FT::kBytes);
        if (li < B && step0 + S * B + li < gn) load_rec<RW>(a.rec_in, gs + step0 + S * B + li, rec);
    };
    prepare(wv * B);
    __syncthreads();

    for (int t = 0; t < rounds; ++t) {
        const int step0 = (t * S + wv) * B;
        const int cnt = gn - step0;
        for (int w = 0; w < S; ++w) {
            if (w == wv) {
                int cur_row = crow[g], cur_slot = cslot[g], flags = gflag[g];
                float acc[V];
                #pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = sums[lane * V + v];
                #pragma unroll
                for (int j = 0; j < B; ++j) {
                    if (j < cnt) {
                        const int slot = g * L + j;
                        const int row = (int)stage[mode][slot];
                        if (row != cur_row) {
                            if (cur_row >= 0) {
                                // the sub-range's first row, begun in an earlier group
                                if (!(flags & kMoved) && before == (uint32_t)cur_row) {
                                    store_vals<V>(part0 + g * R + li * V, acc);
                                    flags |= kHead;
                                    if (li == 0) prow[g] = cur_row;  // (keeps the two stores apart)
                                } else {
                                    store_vals<V>(row_dst<R>(a, cur_row, cur_slot) + li * V, acc);
                                }
                                flags |= kMoved;
                            }
                            cur_row = row;
                            cur_slot = (int)stage[N + 1][slot];
                            #pragma unroll
                            for (int v = 0; v < V; ++v) acc[v] = 0.0f;
                        }
                        const float val = __uint_as_float(stage[N][slot]);
                        float prod[V];
                        widen<FT>(y[j][0], prod);
                        #pragma unroll
                        for (int k = 1; k < NG; ++k) {
                            float f[V];
                            widen<FT>(y[j][k], f);
                            #pragma unroll
                            for (int v = 0; v < V; ++v) prod[v] *= f[v];
                        }
                        #pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fmaf(prod[v], val, acc[v]);
                    }
                }
                #pragma unroll
                for (int v = 0; v < V; ++v) sums[lane * V + v] = acc[v];
                wave_sync();
                if (li == 0) {
                    crow[g] = cur_row;
                    cslot[g] = cur_slot;
                    gflag[g] = flags;
                }
            }
            __syncthreads();
            if (w == wv && t + 1 < rounds) prepare(step0 + S * B);
        }
    }

    // the groups' last segments, by the first wave
    if (wv == 0) {
        const int cur_row = crow[g], cur_slot = cslot[g], flags = gflag[g];
        float acc[V];
        #pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = sums[lane * V + v];
        const bool open_right = cur_row >= 0 && after == (uint32_t)cur_row;
        const bool cont = !(flags & kMoved) && before == (uint32_t)cur_row;
        if (cur_row >= 0) {
            if (open_right || cont) {
                store_vals<V>(part1 + g * R + li * V, acc);
                if (li == 0) {
                    prow[g] = cur_row;
                    pslot[g] = cur_slot;
                }
            } else {
                store_vals<V>(row_dst<R>(a, cur_row, cur_slot) + li * V, acc);
            }
        }
        wave_sync();
        if (li == 0) {
            const int head = flags & kHead;
            gflag[g] = head | (open_right && !cont ? kStarts : 0) | (head || !open_right ? kEnds : 0);
        }
    }
    __syncthreads();
    combine_chains<R>(a, part0, part1, gflag, prow, pslot, G);
}

using EcFn = EcFnPtr;

// (where a nonzero has 4 lanes a step takes 2 or 4 records, in the plain form
// also 1; else 1)
template <int N, int R, int RW, int KIND, typename FT, bool REUSE>
EcFn pick_steps(int steps) {
    if constexpr (ec_lanes(R, FT::kBytes == 2) != 4) {
        return ec_kernel<N, R, RW, KIND, FT, REUSE, 1>;
    } else {
        if (steps == 4) return ec_kernel<N, R, RW, KIND, FT, REUSE, 4>;
        if constexpr (!REUSE)
            if (steps == 1) return ec_kernel<N, R, RW, KIND, FT, REUSE, 1>;
        return ec_kernel<N, R, RW, KIND, FT, REUSE, 2>;
    }
}

template <int N, int RW, int KIND, typename FT, bool REUSE>
EcFn pick_rank(int rank, int steps) {
    switch (rank) {
        case 8: return pick_steps<N, 8, RW, KIND, FT, REUSE>(steps);
        case 16: return pick_steps<N, 16, RW, KIND, FT, REUSE>(steps);
        case 32: return pick_steps<N, 32, RW, KIND, FT, REUSE>(steps);
        case 64: return pick_steps<N, 64, RW, KIND, FT, REUSE>(steps);
        case 128: return pick_steps<N, 128, RW, KIND, FT, REUSE>(steps);
        default: return nullptr;
    }
}

template <int N, int RW, int KIND>
EcFn pick_ordered(int rank, int fdtype) {
    switch (rank) {  // the ranks of CP-ALS
        case 8: return fdtype == 0 ? ec_ordered_kernel<N, 8, RW, KIND, FacF32> : ec_ordered_kernel<N, 8, RW, KIND, FacBF16>;
        case 16: return fdtype == 0 ? ec_ordered_kernel<N, 16, RW, KIND, FacF32> : ec_ordered_kernel<N, 16, RW, KIND, FacBF16>;
        case 32: return fdtype == 0 ? ec_ordered_kernel<N, 32, RW, KIND, FacF32> : ec_ordered_kernel<N, 32, RW, KIND, FacBF16>;
        case 64: return fdtype == 0 ? ec_ordered_kernel<N, 64, RW, KIND, FacF32> : ec_ordered_kernel<N, 64, RW, KIND, FacBF16>;
        default: return nullptr;
    }
}

template <int N, int RW, int KIND>
EcFn pick_form(int rank, int fdtype, EcForm form, int steps) {
    if (form == EcForm::kOrdered) {  // for the 12-byte records the library chooses by itself
        if constexpr (RW == 3)
            return pick_ordered<N, RW, KIND>(rank, fdtype);
        else
            return nullptr;
    }
    if (form == EcForm::kReuse)
        return fdtype == 0 ? pick_rank<N, RW, KIND, FacF32, true>(rank, steps)
                           : pick_rank<N, RW, KIND, FacBF16, true>(rank, steps);
    return fdtype == 0 ? pick_rank<N, RW, KIND, FacF32, false>(rank, steps)
                       : pick_rank<N, RW, KIND, FacBF16, false>(rank, steps);
}

// (record words, layout kind) pairs the planner can choose for N modes
template <int N>
EcFn pick_layout(int rank, int fdtype, int words, int kind, EcForm form, int steps) {
    if constexpr (N <= 2) {
        if (words == 3 && kind == kWord32) return pick_form<N, 3, kWord32>(rank, fdtype, form, steps);
        if (words == 4 && kind == kWord32) return pick_form<N, 4, kWord32>(rank, fdtype, form, steps);
    } else if constexpr (N == 3) {
        if (words == 3 && kind == kPacked) return pick_form<N, 3, kPacked>(rank, fdtype, form, steps);
        if (words == 4 && kind == kWord32) return pick_form<N, 4, kWord32>(rank, fdtype, form, steps);
    } else if constexpr (N <= 6) {
        if constexpr (N == 4)
            if (words == 3 && kind == kHalf16) return pick_form<N, 3, kHalf16>(rank, fdtype, form, steps);
        if (words == 3 && kind == kPacked) return pick_form<N, 3, kPacked>(rank, fdtype, form, steps);
        if (words == 4 && kind == kHalf16) return pick_form<N, 4, kHalf16>(rank, fdtype, form, steps);
        if (words == 4 && kind == kPacked) return pick_form<N, 4, kPacked>(rank, fdtype, form, steps);
        if (words == 8 && kind == kWord32) return pick_form<N, 8, kWord32>(rank, fdtype, form, steps);
    } else if constexpr (N == 7) {
        if (words == 3 && kind == kPacked) return pick_form<N, 3, kPacked>(rank, fdtype, form, steps);
        if (words == 8 && kind == kWord32) return pick_form<N, 8, kWord32>(rank, fdtype, form, steps);
    } else {
        if (words == 3 && kind == kPacked) return pick_form<N, 3, kPacked>(rank, fdtype, form, steps);
        if (words == 8 && kind == kHalf16) return pick_form<N, 8, kHalf16>(rank, fdtype, form, steps);
        if (words == 12 && kind == kWord32) return pick_form<N, 12, kWord32>(rank, fdtype, form, steps);
    }
    return nullptr;
}

}  // namespace
}  // namespace spt
