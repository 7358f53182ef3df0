// Test support for the CPU build of the kernels: stands between the API and
// the launch functions (linked with --wrap, see tests/test_cpu_replay.py).
// Launches can be recorded with their arguments and run again, as a captured
// graph runs them; chosen device allocations can be made to fail; the sum of
// block partials, whose kernel is not in the CPU build, is done here.
#include <functional>
#include <vector>

#include "kernels.hpp"

namespace {
std::vector<std::function<void()>> g_launches;
bool g_record = false;
int g_fail_at = -1;  // the allocation to fail, counted from 0; -1: none

void note(std::function<void()> f) {
    if (g_record) g_launches.push_back(f);
    f();
}
}  // namespace

#define LAUNCH_EC _ZN3spt9launch_ecEiiiiiiRKNS_6EcArgsEP13cpuhip_stream
#define LAUNCH_FIXUP _ZN3spt12launch_fixupEiRKNS_9FixupArgsEP13cpuhip_stream
#define LAUNCH_FORWARD _ZN3spt14launch_forwardEiiiiRKNS_11ForwardArgsEP13cpuhip_stream
#define LAUNCH_REMAP _ZN3spt19launch_remap_stagedEilPKjPjPKiPKtP13cpuhip_stream
#define REDUCE _ZN3spt22launch_reduce_partialsEPKdiiPdP13cpuhip_stream
#define MALLOC _Z9hipMallocPPvm
#define GLUE2(a, b) a##b
#define GLUE(a, b) GLUE2(a, b)
#define WRAP(name) GLUE(__wrap_, name)
#define REAL(name) GLUE(__real_, name)

extern "C" {

bool REAL(LAUNCH_EC)(int, int, int, int, int, int, const spt::EcArgs&, hipStream_t);
bool WRAP(LAUNCH_EC)(int n, int rank, int fdtype, int words, int kind, int kappa, const spt::EcArgs& a, hipStream_t s) {
    bool ok = false;
    note([=, &ok]() { ok = REAL(LAUNCH_EC)(n, rank, fdtype, words, kind, kappa, a, s); });
    if (g_record) g_launches.back() = [=]() { REAL(LAUNCH_EC)(n, rank, fdtype, words, kind, kappa, a, s); };
    return ok;
}

void REAL(LAUNCH_FIXUP)(int, const spt::FixupArgs&, hipStream_t);
void WRAP(LAUNCH_FIXUP)(int rank, const spt::FixupArgs& a, hipStream_t s) {
    note([=]() { REAL(LAUNCH_FIXUP)(rank, a, s); });
}

bool REAL(LAUNCH_FORWARD)(int, int, int, int, const spt::ForwardArgs&, hipStream_t);
bool WRAP(LAUNCH_FORWARD)(int n, int rank, int words, int kind, const spt::ForwardArgs& a, hipStream_t s) {
    bool ok = false;
    note([=, &ok]() { ok = REAL(LAUNCH_FORWARD)(n, rank, words, kind, a, s); });
    if (g_record) g_launches.back() = [=]() { REAL(LAUNCH_FORWARD)(n, rank, words, kind, a, s); };
    return ok;
}

void REAL(LAUNCH_REMAP)(int, int64_t, const uint32_t*, uint32_t*, const int32_t*, const uint16_t*, hipStream_t);
void WRAP(LAUNCH_REMAP)(int words, int64_t nnz, const uint32_t* in, uint32_t* out, const int32_t* ddst,
                        const uint16_t* doff, hipStream_t s) {
    note([=]() { REAL(LAUNCH_REMAP)(words, nnz, in, out, ddst, doff, s); });
}

void WRAP(REDUCE)(const double* partial, int nblocks, int E, double* out, hipStream_t) {
    note([=]() {
        for (int e = 0; e < E; ++e) {
            double t = 0.0;
            for (int b = 0; b < nblocks; ++b) t += partial[(int64_t)b * E + e];
            out[e] = t;
        }
    });
}

hipError_t REAL(MALLOC)(void**, size_t);
hipError_t WRAP(MALLOC)(void** p, size_t bytes) {
    if (g_fail_at >= 0 && g_fail_at-- == 0) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return REAL(MALLOC)(p, bytes);
}

void cpuhip_record(int on) {
    g_record = on != 0;
    if (on) g_launches.clear();
}
int cpuhip_replay() {
    for (auto& f : g_launches) f();
    return (int)g_launches.size();
}
void cpuhip_fail_malloc(int at) { g_fail_at = at; }

}  // extern "C"
