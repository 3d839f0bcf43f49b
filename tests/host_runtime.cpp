// A stand-in for the HIP runtime and the kernel launchers, linked with the library's own host code
// (el_api, el_exec, el_group) into a test library that needs no device: memory is host memory,
// copies happen at once, launches do nothing.  fail_call(n): the n-th runtime call or launch from now
// on fails; fail_new(n): the n-th allocation throws.  n < 0: none.  Both count what they see.
#include <cstdlib>
#include <cstring>
#include <new>

#include "el_impl.h"

namespace {
long long g_call = 0, g_call_fails = -1, g_new = 0, g_new_fails = -1, g_handles = 0;
hipError_t call() { return g_call++ == g_call_fails ? hipErrorUnknown : hipSuccess; }
template <typename H>
hipError_t make(H *h) {
    const hipError_t e = call();
    if (e == hipSuccess) {
        *h = reinterpret_cast<H>(malloc(1));
        ++g_handles;
    }
    return e;
}
template <typename H>
hipError_t drop(H h) {
    free(reinterpret_cast<void *>(h));
    --g_handles;
    return hipSuccess;
}
}  // namespace

void *operator new(size_t n) {
    if (g_new++ == g_new_fails) throw std::bad_alloc();
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void *operator new[](size_t n) { return operator new(n); }
void operator delete(void *p) noexcept { free(p); }
void operator delete[](void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
void operator delete[](void *p, size_t) noexcept { free(p); }

extern "C" {
void fail_call(long long n) { g_call = 0, g_call_fails = n; }
void fail_new(long long n) { g_new = 0, g_new_fails = n; }
long long calls() { return g_call; }
long long news() { return g_new; }
long long handles() { return g_handles; }   // events, streams and graphs not yet released
// what a launch of the plan would take: its block list's entries per XCD, and where it lies
int table_per(el_plan p) { return p->tiles.per; }
int table_of(el_plan p) { return p->tiles.order == p->ws + p->L.tile_order[1] ? 1 : 0; }
int table_inc(el_plan p) { return p->df.incoff == (unsigned)(p->L.inc[1] >> 8) ? 1 : 0; }
int table_rec(el_plan p) {
    return (p->rec.fl == (unsigned char *)p->ws + p->L.rec_fl[1] ? 1 : 0) + (p->rec.pos == (int *)(p->ws + p->L.csr_pos[1]) ? 2 : 0);
}
// entries of the plan's list, as a launch would read them
int table_entries(el_plan p) {
    const auto *e = static_cast<const el::BlockEnt<float> *>(p->tiles.order);
    int n = 0;
    for (int b = 0; b < 8 * p->tiles.per; ++b) n += e[b].flags != 0;
    return n;
}
void set_room(el_plan p, int cap) { p->tiles.cap = cap; }
int room(el_plan p) { return p->tiles.cap; }

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "forced"; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    const hipError_t e = call();
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { return call(); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return call(); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t s) { return drop(s); }
hipError_t hipEventCreate(hipEvent_t *e) { return make(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return drop(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return call(); }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return call(); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return call(); }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return call(); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return make(g); }
hipError_t hipGraphDestroy(hipGraph_t g) { return drop(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) { return make(x); }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return drop(x); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return call(); }
}

namespace el {
hipError_t launch_media_stats(const float *, const float *, const float *, const float *, long long, double, double *stats,
                              double *, hipStream_t) {
    const double ok[kStats] = {1.0, 1.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
    memcpy(stats, ok, sizeof ok);
    return call();
}
hipError_t launch_relax_stats(const float *, int, int, int, int, double *stats, double *, hipStream_t) {
    stats[0] = stats[1] = stats[2] = 0.0;
    return call();
}
hipError_t launch_energy_final(const double *, double *, const double *, int, double *, hipStream_t) { return call(); }
hipError_t launch_eir(const double *, int, const double *, double *, int, int, int, hipStream_t) { return call(); }
hipError_t launch_set_counter(int *, int, hipStream_t) { return call(); }
template <typename T> hipError_t launch_convert_maps(const Dev<T> &, const float *, const float *, const float *, const float *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_zero_state(const Dev<T> &, hipStream_t) { return call(); }
// the middle tile of every other chunk is fluid
template <typename T> hipError_t launch_classify(const Dev<T> &, const Tiles &tl, unsigned char *fast, unsigned char *uni, T *med, unsigned long long *lanes, hipStream_t) {
    for (int q = 0; q < tl.ntiles; ++q) {
        fast[q] = uni[q] = q % 2;
        for (int c = 0; c < 4; ++c) med[4 * (size_t)q + c] = T(c);
    }
    memset(lanes, 0, (size_t)2 * kTileY * tl.ntiles * 8);
    return call();
}
template <typename T> hipError_t launch_inject(const Dev<T> &, const T *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_velocity(const Dev<T> &, const Tiles &, hipStream_t, const Rec *, double *, double *, int *) { return call(); }
template <typename T> hipError_t launch_energy_pot(const Dev<T> &, const Tiles &, double *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_stress(const Dev<T> &, const Tiles &, hipStream_t, int *) { return call(); }
template <typename T> hipError_t launch_gather(const Dev<T> &, const Rec &, double *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_adj_velocity(const Dev<T> &, const Tiles &, hipStream_t, const Rec *, const double *, int *) { return call(); }
template <typename T> hipError_t launch_adj_stress(const Dev<T> &, const Tiles &, hipStream_t, int *) { return call(); }
template <typename T> hipError_t launch_scatter(const Dev<T> &, const Rec &, const double *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_zero_inc(const Dev<T> &, long long, hipStream_t) { return call(); }
template <typename T> hipError_t launch_group_pass(const Grp<T, kGroupMax> &, int, hipStream_t) { return call(); }
template <typename T> hipError_t launch_extract(const Dev<T> &, T *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_fluid_fill(const Dev<T> &, const Tiles &, hipStream_t) { return call(); }
template <typename T> hipError_t launch_dot(const T *, const T *, long long, double *, double *, hipStream_t) { return call(); }
template <typename T> hipError_t launch_relax_setup(const Dev<T> &, const Tiles &, const float *, const Relax<T> &, hipStream_t) { return call(); }
template <typename T> hipError_t launch_relax_compact(const Dev<T> &, const Tiles &, const Relax<T> &, hipStream_t) { return call(); }
template <typename T> hipError_t launch_relax_zero(const Tiles &, const Relax<T> &, hipStream_t) { return call(); }
template <typename T> hipError_t launch_relax(const Dev<T> &, const Tiles &, const Relax<T> &, bool, hipStream_t) { return call(); }
#define HOST_INST(T)                                                                                                              \
    template hipError_t launch_convert_maps<T>(const Dev<T> &, const float *, const float *, const float *, const float *, hipStream_t); \
    template hipError_t launch_zero_state<T>(const Dev<T> &, hipStream_t);                                                        \
    template hipError_t launch_classify<T>(const Dev<T> &, const Tiles &, unsigned char *, unsigned char *, T *, unsigned long long *, hipStream_t); \
    template hipError_t launch_inject<T>(const Dev<T> &, const T *, hipStream_t);                                                 \
    template hipError_t launch_velocity<T>(const Dev<T> &, const Tiles &, hipStream_t, const Rec *, double *, double *, int *);   \
    template hipError_t launch_energy_pot<T>(const Dev<T> &, const Tiles &, double *, hipStream_t);                               \
    template hipError_t launch_stress<T>(const Dev<T> &, const Tiles &, hipStream_t, int *);                                      \
    template hipError_t launch_gather<T>(const Dev<T> &, const Rec &, double *, hipStream_t);                                     \
    template hipError_t launch_adj_velocity<T>(const Dev<T> &, const Tiles &, hipStream_t, const Rec *, const double *, int *);   \
    template hipError_t launch_adj_stress<T>(const Dev<T> &, const Tiles &, hipStream_t, int *);                                  \
    template hipError_t launch_scatter<T>(const Dev<T> &, const Rec &, const double *, hipStream_t);                              \
    template hipError_t launch_zero_inc<T>(const Dev<T> &, long long, hipStream_t);                                               \
    template hipError_t launch_group_pass<T>(const Grp<T, kGroupMax> &, int, hipStream_t);                                        \
    template hipError_t launch_extract<T>(const Dev<T> &, T *, hipStream_t);                                                      \
    template hipError_t launch_fluid_fill<T>(const Dev<T> &, const Tiles &, hipStream_t);                                         \
    template hipError_t launch_dot<T>(const T *, const T *, long long, double *, double *, hipStream_t);                          \
    template hipError_t launch_relax_setup<T>(const Dev<T> &, const Tiles &, const float *, const Relax<T> &, hipStream_t);       \
    template hipError_t launch_relax_compact<T>(const Dev<T> &, const Tiles &, const Relax<T> &, hipStream_t);                    \
    template hipError_t launch_relax_zero<T>(const Tiles &, const Relax<T> &, hipStream_t);                                       \
    template hipError_t launch_relax<T>(const Dev<T> &, const Tiles &, const Relax<T> &, bool, hipStream_t);
HOST_INST(float)
HOST_INST(double)
}  // namespace el
