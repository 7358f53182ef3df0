// Launch side of the elementwise kernel (ec_kernel.hpp, instantiated per
// mode count in ec_n2.hip .. ec_n8.hip), the split-row fixup, the BF16 copy
// of the factors and the remap along a chain of next positions.
#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

#include "kernels.hpp"
#include "record.hpp"

namespace spt {

EcFnPtr pick_ec_n2(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n3(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n4(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n5(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n6(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n7(int, int, int, int, EcForm, int);
EcFnPtr pick_ec_n8(int, int, int, int, EcForm, int);

namespace {

// Split rows: one workgroup per row sums its carry slots.  Thread (q, r)
// adds slots q, q + Q, q + 2Q, ... of rank r in four interleaved chains,
// then the Q partials are added in order of q -- a fixed order, so the
// result does not depend on scheduling.  Blocks past the split rows fill
// the rows that have no nonzero with zeros.
template <int R>
__global__ __launch_bounds__(1024) void fixup_kernel(const FixupArgs a, int zero_blocks) {
    constexpr int Q = 1024 / R;
    __shared__ float part[Q][R];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < a.nsplit) {
        const int j = blockIdx.x;
        const int q = tid / R, r = tid % R;
        const int k0 = a.split_ptr[j], k1 = a.split_ptr[j + 1];
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
        int k = k0 + q;
        for (; k + 3 * Q < k1; k += 4 * Q) {
            s0 += a.carry[(int64_t)k * R + r];
            s1 += a.carry[(int64_t)(k + Q) * R + r];
            s2 += a.carry[(int64_t)(k + 2 * Q) * R + r];
            s3 += a.carry[(int64_t)(k + 3 * Q) * R + r];
        }
        for (; k < k1; k += Q) s0 += a.carry[(int64_t)k * R + r];
        part[q][r] = (s0 + s1) + (s2 + s3);
        __syncthreads();
        if (tid < R) {
            float t = 0.f;
            for (int i = 0; i < Q; ++i) t += part[i][tid];
            a.out[(int64_t)a.split_row[j] * R + tid] = t;
        }
        return;
    }
    // zero rows: float4 per thread
    constexpr int R4 = R / 4;
    const int64_t total = (int64_t)a.nempty * R4;
    const int64_t stride = (int64_t)zero_blocks * 1024;
    for (int64_t i = (int64_t)(blockIdx.x - a.nsplit) * 1024 + tid; i < total; i += stride) {
        const int64_t row = a.empty_rows[i / R4];
        reinterpret_cast<float4*>(a.out + row * R)[i % R4] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

struct NxtChain {
    const int32_t* nxt[8];
};

// FP32 -> BF16 by rounding the bit pattern to nearest, ties to even (add
// 0x7FFF plus the lowest kept bit, truncate); NaNs stay quiet NaNs.
__global__ void to_bf16_kernel(const float* __restrict__ src, uint16_t* __restrict__ dst, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t u = __float_as_uint(src[i]);
        if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) {
            dst[i] = (uint16_t)((u >> 16) | 0x0040u);
        } else {
            u += 0x7FFFu + ((u >> 16) & 1u);
            dst[i] = (uint16_t)(u >> 16);
        }
    }
}

template <int RW>
__global__ void remap_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                             int64_t nnz, NxtChain ch, int hops) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < nnz;
         p += (int64_t)gridDim.x * blockDim.x) {
        int64_t d = p;
        for (int h = 0; h < hops; ++h) d = ch.nxt[h][d];
        Rec<RW> r;
        load_rec<RW>(in, p, r);
        store_rec<RW>(out, d, r);
    }
}

EcFnPtr pick_ec(int nmodes, int rank, int fdtype, int words, int kind, EcForm form, int steps = 1) {
    switch (nmodes) {
        case 2: return pick_ec_n2(rank, fdtype, words, kind, form, steps);
        case 3: return pick_ec_n3(rank, fdtype, words, kind, form, steps);
        case 4: return pick_ec_n4(rank, fdtype, words, kind, form, steps);
        case 5: return pick_ec_n5(rank, fdtype, words, kind, form, steps);
        case 6: return pick_ec_n6(rank, fdtype, words, kind, form, steps);
        case 7: return pick_ec_n7(rank, fdtype, words, kind, form, steps);
        case 8: return pick_ec_n8(rank, fdtype, words, kind, form, steps);
        default: return nullptr;
    }
}

// Single-wave workgroups of f one CU holds at once (0 if the query fails).
int resident_blocks(EcFnPtr f, size_t lds) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(f), 64, lds) != hipSuccess)
        return 0;
    return nb;
}

// Whether the form that reuses the last gathered row keeps the occupancy that
// the gathers need: that of the plain form, or 4 waves per SIMD (decided once
// per combination and device).
bool reuse_fits(EcFnPtr plain, EcFnPtr reuse, size_t lds) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    static std::mutex mu;
    static std::map<std::pair<int, EcFnPtr>, bool> fits;
    std::lock_guard<std::mutex> lock(mu);
    auto it = fits.find({dev, plain});
    if (it != fits.end()) return it->second;
    const int occ_plain = resident_blocks(plain, lds), occ_reuse = resident_blocks(reuse, lds);
    return fits[{dev, plain}] = occ_reuse > 0 && occ_reuse >= std::min(occ_plain, 16);
}

// The form of the elementwise kernel, its waves per partition and the records
// its lanes stage per step.
struct EcChoice {
    EcFnPtr f;
    int waves;
    int steps;
};

// Where the lines lie (MI355X, us per launch, plain / reuse form unless said):
// - The reuse form saves a share `repeats` of one of the N-1 gathers and pays
//   with a branch per nonzero.  With N >= 4 that pays or costs nothing at every
//   share measured (4-mode 1e7, R 16, repeats 0.15-0.71: 136-152 / 122-145;
//   4-mode 1e8, R 64: 2692-2861 / 2282-2487; 5-mode 5e7, R 32: 860-901 /
//   721-802; repeats 0.00-0.06: within 1 %), once partitions hold a few hundred
//   nonzeros (8-mode, R 64, 32768 of 8: 570 / 800).  With N = 3 it
//   pays on large skewed tensors (8e7, R 32: 982-1007 / 905-955; 2e7, repeats
//   0.23-0.66: 240-246 / 226-233), not where most rows differ (8e7, repeats
//   0.04-0.20: 1532-2053 / 1564-2106) and not on small tensors, whose rows
//   hit the caches anyway (5e6, R 32, repeats 0.51-0.57: 57-61 / 60-66; 3e5,
//   R 64, 147 partitions: 20-24 / 22-26), unless the rows are long (4e6, R 128,
//   repeats 0.52-0.55: 149-157 / 137-141; 4e6, R 64: 79-80 / 74-75), nor in one
//   wave per partition (1024 partitions of 73, R 128: 67 / 70).  With N = 2 the kept row is the
//   only one, and every nonzero waits for the branch (1e7, R 32, repeats 0.45:
//   89 / 113; R 64: 147 / 235; 3e7, R 64: 376 / 575).
// - Waves per partition: up to 256 partitions leave CUs idle or with one
//   workgroup, so the most waves (1e5 nonzeros, 49 partitions, R 16: 39 us at 1,
//   17 at 4, 14 at 8; 3e5, 147 partitions, R 64: 80 / 32 / 21).  Above that 4:
//   the waves of a workgroup work on neighbouring records and share the rows
//   they gather in L1, and 8 pay more for the combine than they gain (4-mode
//   2e6, R 64: 127 / 72 / 76; 4-mode 1e8, R 64: 2400-2850 / 2280-2490; 1e6, R 8:
//   35 / 23 / 31).  Without rows to share (the plain form) and with enough
//   partitions to fill the chip twice, 1 (8e7, zipf 0.8: 1981-2053 at 1,
//   2042-2120 at 4).
// - More waves pay only while each lane group still has records to walk: with few
//   they cost their start and the combine.  Ratio of 4 waves to 1, all modes:
//   64 partitions, R 16, of 73 nonzeros 1.0, of 146 0.85, R 64, of 36 0.95, of 73
//   0.77 (8 to 4, R 16, of 293 0.98, of 586 0.93; BF16 at R 8, 64 groups a wave,
//   4-mode 3e5, skewed: 8 waves 1.5); 300 partitions, R 32, of 73 0.89, R 16, of
//   146 0.9 to 1.08 (8 modes); 1024 partitions, R 64, of 146 0.8, R 16, of 293 0.92
//   (4 modes), 1.21 (5), of 586 0.91, 1.12; 2048, R 16, skewed, of 700 1.2, of 1030
//   1.1, R 32, of 700 0.75 to 0.95, R 8, of 2047 1.1 to 1.3 (2 to 4 modes), 0.95 (5), 0.74
//   (8), BF16 at R 8, of 2047 1.2 to 1.5.  Beyond 2048 the chip is
//   full with one wave each, and what counts is the rows a group gathers: 4096
//   partitions, R 64, of 700 1.12 (2 and 3 modes), 0.94 (4), 0.87 (8); R 32, of
//   1030 1.17 (3), 1.03 (4), 0.9 (8); R 16, of 1030 1.2 to 1.0; at the default's
//   2048 per partition 0.7 to 1.0.
// - Beyond 1024 partitions, where few nonzeros share rows and these do not fit an
//   XCD's L2 (4 MB; 6 as some of it stays), lines from beyond L2 are the bound and
//   more waves crowd them out (5-mode 1e7, R 64, repeats 0.06, 9 MB: 3600 at 1,
//   3920 at 4; 4-mode 3e7, R 32, 0.03, 10 MB: 3780 / 3970; 2-mode 3e6, R 8, 0.00,
//   8 MB: 104 / 134; against 5-mode 1e7, R 32, 5 MB: 1405 / 1335).
// - CP-ALS feeds its results back, so a change of rounding grows from sweep to
//   sweep: its sums stay those of one wave per partition, bit for bit.  There
//   the reuse form pays only where the partitions fill the chip (4-mode 1e8:
//   2752-3090 / 2396-2853; 1e6, R 8, 611 partitions: 31-43 / 34-47), and below
//   2048 partitions the ordered form takes its place (one wave / ordered:
//   4-mode 2e6, R 64, 977 partitions: 112-147 / 86-115; 1e6, R 8, 611: 35-51 /
//   26-38; 3-mode 3.5e6, R 32, 1710: 50-52 / 47-48; 5e6, 2442: 69-85 / 85-90;
//   eight waves up to 256 partitions, 3e5, R 64, 147: 76 / 63; 1e5, R 16, 49:
//   31 / 26; two above: four gain nothing more at 977 and lose at 1710, 74).

// Waves per partition for kappa partitions of `per` nonzeros, of which one wave's
// G lane groups take per / G each.
int ec_waves(int nmodes, int kappa, int64_t per, int G, bool crowded) {
    if (kappa <= 256) {
        if (G <= 32 && per >= std::min(1024, std::max(256, 32 * G))) return 8;
        return per >= std::min(1024, std::max(32, 8 * G)) ? 4 : 1;
    }
    if (kappa <= 512) return per >= std::min(1024, 10 * G) ? 4 : 1;
    if (kappa <= 1024) return per >= std::min(1024, 40 * G) ? 4 : 1;
    if (crowded) return 1;
    if (kappa <= 2048) return per >= (nmodes >= 5 ? 63 : 70) * G ? 4 : 1;
    if (per >= 2000) return 4;
    const double rows = (double)per * (nmodes - 1);
    return per >= 75 * G && rows * rows >= 1250.0 * 1250.0 * G ? 4 : 1;
}

EcChoice choose_ec(int nmodes, int rank, int fdtype, int words, int kind, int kappa, const EcArgs& a) {
#ifdef SPT_EC_ONE_WAVE  // build option: the order of one wave for every caller
    const bool one_wave = true;
#else
    const bool one_wave = a.one_wave != 0;
#endif
#ifdef SPT_EC_ORDERED  // build option: partitions below which that order takes the ordered form
    constexpr int kOrderedBelow = SPT_EC_ORDERED;
#else
    constexpr int kOrderedBelow = 2048;
#endif
    if (one_wave && !a.rec_out && kappa < kOrderedBelow)
        if (const EcFnPtr ordered = pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kOrdered))
            return {ordered, kappa <= 256 ? 8 : 2, 1};
    const int64_t per = a.nnz / kappa;
    const int lanes = ec_lanes(rank, fdtype != 0);
    const bool crowded = a.repeats < 0.1f && a.gathered > (int64_t(6) << 20);
    // a second record per lane costs more than it hides where lines from beyond L2
    // are the bound and the chip is just full (2-mode 4e6, R 16: 79 us, 75 with one),
    // and on skewed 3-mode tensors with BF16, whose staging is the larger (9e6, R 32:
    // 112 in the reuse form, 92 with one in the plain form; 2e6: 38, 33)
    const bool one = (crowded && kappa > 1024 && kappa <= 2048) || (nmodes == 3 && fdtype != 0 && a.repeats >= 0.1f);
    const int most = ec_step_records(rank, fdtype != 0, per), steps = one && most == 2 ? 1 : most;
    EcChoice c{pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kPlain, steps), 1, steps};
    if (!c.f) return c;
    if (!one_wave) c.waves = ec_waves(nmodes, kappa, per, 64 / lanes, crowded);
#ifdef SPT_EC_FORM  // build option: 0 = always the plain form, 1 = always the reuse form
    const bool want = SPT_EC_FORM != 0;
#else
    const bool long_rows = 16 * lanes >= 256 && kappa > 256;
    bool want = false;
    if (lanes == 4 && steps == 1)
        want = false;  // (that step has no reuse form)
    else if (nmodes >= 4)
        want = one_wave ? kappa >= 4096 : per >= 256;
    else if (nmodes == 3 && a.repeats >= 0.4f)
        want = one_wave ? kappa >= 4096 : c.waves > 1 && (kappa >= 4096 || long_rows);
    if (want) {
        const EcFnPtr reuse = pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kReuse, steps);
        want = reuse && reuse_fits(c.f, reuse, ec_lds_bytes(nmodes, rank, fdtype, 1, steps));
    }
#endif
    if (want) {
        if (lanes == 4) c.steps = std::max(2, steps);
        c.f = pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kReuse, c.steps);
    } else if (kappa >= 8192) {
        c.waves = 1;
    }
#ifdef SPT_EC_WAVES  // build option: waves per partition
    c.waves = SPT_EC_WAVES;
#endif
    return c;
}

}  // namespace

bool pick_ec_exists(int nmodes, int rank, int fdtype, int words, int kind) {
    return pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kPlain) != nullptr;
}

bool launch_ec(int nmodes, int rank, int fdtype, int words, int kind, int kappa, const EcArgs& a,
               hipStream_t s) {
    if (kappa <= 0) return pick_ec(nmodes, rank, fdtype, words, kind, EcForm::kPlain) != nullptr;
    const EcChoice c = choose_ec(nmodes, rank, fdtype, words, kind, kappa, a);
    if (!c.f) return false;
    EcArgs args = a;
    args.waves = c.waves;
    // LDS of one workgroup stays within 64 KB: 4 waves where 8 would need more
    // (70 to 121 KB: steps of 4 records from 4 modes on, with BF16 factors at any
    // number of modes, and there steps of 2 from 5 on; 8 modes at rank 8, BF16)
    while (args.waves > 2 && ec_lds_bytes(nmodes, rank, fdtype, args.waves, c.steps) > 65536) args.waves /= 2;
    hipLaunchKernelGGL(c.f, dim3((unsigned)kappa), dim3((unsigned)(64 * args.waves)),
                       (size_t)ec_lds_bytes(nmodes, rank, fdtype, args.waves, c.steps), s, args);
    return true;
}

void launch_fixup(int rank, const FixupArgs& a, hipStream_t s) {
    const int64_t zero_work = (int64_t)a.nempty * (rank / 4);
    const int zero_blocks = (int)std::min<int64_t>((zero_work + 1023) / 1024, 1024);
    const int blocks = a.nsplit + zero_blocks;
    if (blocks == 0) return;
    switch (rank) {
        case 8: hipLaunchKernelGGL(fixup_kernel<8>, dim3(blocks), dim3(1024), 0, s, a, zero_blocks); break;
        case 16: hipLaunchKernelGGL(fixup_kernel<16>, dim3(blocks), dim3(1024), 0, s, a, zero_blocks); break;
        case 32: hipLaunchKernelGGL(fixup_kernel<32>, dim3(blocks), dim3(1024), 0, s, a, zero_blocks); break;
        case 64: hipLaunchKernelGGL(fixup_kernel<64>, dim3(blocks), dim3(1024), 0, s, a, zero_blocks); break;
        case 128: hipLaunchKernelGGL(fixup_kernel<128>, dim3(blocks), dim3(1024), 0, s, a, zero_blocks); break;
        default: break;
    }
}

void launch_to_bf16(const float* src, uint16_t* dst, int64_t n, hipStream_t s) {
    if (n == 0) return;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src, dst, n);
}

void launch_remap(int words, int64_t nnz, const uint32_t* in, uint32_t* out,
                  const int32_t* const* nxt, int hops, hipStream_t s) {
    if (nnz == 0) return;
    NxtChain ch{};
    for (int h = 0; h < hops; ++h) ch.nxt[h] = nxt[h];
    const int threads = 256;
    const int64_t blocks = std::min<int64_t>((nnz + threads - 1) / threads, 8192);
    if (words == 3)
        hipLaunchKernelGGL((remap_kernel<3>), dim3((unsigned)blocks), dim3(threads), 0, s, in, out,
                           nnz, ch, hops);
    else if (words == 4)
        hipLaunchKernelGGL((remap_kernel<4>), dim3((unsigned)blocks), dim3(threads), 0, s, in, out,
                           nnz, ch, hops);
    else if (words == 8)
        hipLaunchKernelGGL((remap_kernel<8>), dim3((unsigned)blocks), dim3(threads), 0, s, in, out,
                           nnz, ch, hops);
    else
        hipLaunchKernelGGL((remap_kernel<12>), dim3((unsigned)blocks), dim3(threads), 0, s, in, out,
                           nnz, ch, hops);
}

}  // namespace spt
