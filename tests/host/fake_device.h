// Stand-ins for the HIP runtime and for the device side of the library, so
// that the host engine (engine.cpp, included whole by the driver beside this
// file) runs its scheduling on a machine without a GPU: memory is host
// memory, copies happen at once, and a launch plays the slots' state machine
// without any numbers (a solve converges after the iterations and refinement
// trips `dev` asks for).  What is counted: launches, resident launches, waits.
#pragma once

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "resident_shapes.h"

struct Device {
    int iters = 100;          // iterations a solve (FP32 + refinement: a trip) takes
    int trips = 3;            // refinement trips
    int cus = 256;
    int timeouts = 0;         // resident launches from now on that time out
    int refused = 0;          // and those that fail to launch
    // counted
    int actions = 0, resident = 0, waits = 0, graphs = 0;
    void count_from_zero() { actions = resident = waits = graphs = 0; }
};
static Device dev;

extern "C" {
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "ok" : "fake error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { ++dev.waits; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode);
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *);
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = (hipGraphExec_t)1;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t);
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? dev.cus : 1;
    return hipSuccess;
}
}

namespace pcgmi {

// One launch of the tile kernels over the table (which: 2 the second half,
// with the first-half actions too when only second halves are launched; else
// the first half).
inline void play(const BatchHeader *hdr, const Slot *slots, int which)
{
    const bool first = which != 2 || hdr->k2only, second = which == 2;
    for (int s = 0; s < hdr->nslots; ++s) {
        const Slot &S = slots[s];
        SlotState &st = *S.st;
        const int end = st.singular ? (int)K1_MEAN_X : (int)PH_DONE;
        auto go_on = [&](int next) {
            if (st.resident) { st.phase = next; return; }
            st.phase = K2_NONE;
            st.after = next;
        };
        if (first && st.phase < K2_NONE) {
            switch (st.phase) {
            case K1_MEAN_B: go_on(st.after); break;
            case K1_INIT64: st.first = 1; go_on(st.maxit == 0 ? K1_CHECK64 : K1_CG_A); break;
            case K1_CG_A: if (!S.resident) st.phase = K2_CG_B; break;
            case K1_CHECK64:
                if (st.iter >= dev.iters) { st.status = PCG_OK; go_on(end); }
                else if (st.iter >= st.maxit) { st.status = PCG_MAXIT; go_on(end); }
                else go_on(K1_CG_A);
                break;
            case K1_IR_INIT: go_on(K1_IR_RESID); break;
            case K1_IR_RESID:
                st.phase = K2_IR_UPDATE;
                st.outer += 1;
                st.final_upd = st.outer > dev.trips || st.iter >= st.maxit;
                if (st.final_upd) st.status = st.outer > dev.trips ? PCG_OK : PCG_MAXIT;
                break;
            case K1_IR_A: if (!S.resident) st.phase = K2_IR_B; break;
            case K1_MEAN_X: st.phase = K2_SUB_X; break;
            default: break;
            }
        } else if (second && st.phase >= K2_NONE && st.phase < PH_DONE) {
            switch (st.phase) {
            case K2_NONE: st.phase = st.after; break;
            case K2_CG_B:
                st.iter += 1;
                st.phase = st.iter >= dev.iters || st.iter >= st.maxit ? K1_CHECK64 : K1_CG_A;
                break;
            case K2_IR_UPDATE:
                st.inner_iter = 0;
                st.phase = st.final_upd ? end : (int)K1_IR_A;
                break;
            case K2_IR_B:
                st.iter += 1;
                st.inner_iter += 1;
                st.phase = st.inner_iter >= dev.iters || st.iter >= st.maxit ? K1_IR_RESID : K1_IR_A;
                break;
            case K2_SUB_X: st.phase = PH_DONE; break;
            default: break;
            }
        }
    }
}

// Launches issued while a graph is captured, played when it is launched.
struct Recorded { const BatchHeader *hdr; const Slot *slots; int which; };
inline std::vector<Recorded> recorded;
inline bool recording = false;

hipError_t launch_iter(int, int which, int, int, const BatchHeader *hdr, const Slot *slots, hipStream_t)
{
    if (recording) { recorded.push_back({ hdr, slots, which }); return hipSuccess; }
    ++dev.actions;
    play(hdr, slots, which);
    return hipSuccess;
}

hipError_t launch_setup(const double *, const uint8_t *, double *, float *, uint8_t *cls, int64_t, int *,
                        unsigned long long *words, double *, float *, hipStream_t)
{
    if (cls) words[0] = 0x3ff0000000000000ull;   // one density, 1.0
    return hipSuccess;
}
hipError_t launch_copy(const double *, double *, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_mask(const uint8_t *, uint32_t *bits, int, int, int64_t nwords, hipStream_t)
{
    std::memset(bits, 0, (size_t)nwords * 4);
    return hipSuccess;
}
hipError_t launch_triad(double *, const double *, const double *, double, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_check_frac(const double *, const double *, const double *, const double *, const double *,
                             int64_t, int64_t, int64_t, int64_t, int *, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_project(const Slot *, const double *, double, double, const double *const[3],
                          const double *const[3], double *const[3], int, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_rhs(const Slot *, double, double, const double *const[3], const double *const[3], double *,
                      int, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_divnorm(const Slot *, double, const double *, const double *, const double *, double *, int,
                          hipStream_t)
{
    return hipSuccess;
}
hipError_t static_scratch(void **, size_t *) { return hipErrorNoDevice; }

#define PCG_SHAPE(c, p, keep, faces, batch) { c, p, keep, faces, batch },
int resident_shapes(int family, ResidentShape *out, int cap)
{
    static const std::vector<ResidentShape> s[2] = { { PCG_RESIDENT_FP64(PCG_SHAPE) },
                                                     { PCG_RESIDENT_FP32(PCG_SHAPE) } };
    int n = 0;
    for (const ResidentShape &r : s[family == PCG_PREC_FP32_IR])
        if (n < cap) out[n++] = r;
    return n;
}
hipError_t resident_occupancy(int, int, unsigned, int *wgs)
{
    *wgs = 1;
    return hipSuccess;
}

// The resident kernel: `budget` iterations of the solves in their loop.
hipError_t launch_resident(int, int, int, unsigned, const Slot *slots, int s0, int s1, int budget, int, hipStream_t)
{
    if (dev.refused > 0) { --dev.refused; return hipErrorCooperativeLaunchTooLarge; }
    ++dev.resident;
    const bool late = dev.timeouts > 0 && dev.timeouts--;
    for (int s = s0; s < s1; ++s) {
        SlotState &st = *slots[s].st;
        const bool ir = st.phase == K1_IR_A;
        if (!slots[s].resident || st.rfail || (st.phase != K1_CG_A && !ir)) continue;
        if (late) { st.rfail = 1; continue; }
        for (int n = 0; n < budget && (st.phase == K1_CG_A || st.phase == K1_IR_A); ++n) {
            st.iter += 1;
            st.inner_iter += 1;
            st.first = 0;
            if ((ir ? st.inner_iter : st.iter) >= dev.iters || st.iter >= st.maxit)
                st.phase = ir ? K1_IR_RESID : K1_CHECK64;
        }
    }
    return hipSuccess;
}

}  // namespace pcgmi

extern "C" {
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    pcgmi::recorded.clear();
    pcgmi::recording = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    pcgmi::recording = false;
    *g = (hipGraph_t)1;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t)
{
    ++dev.graphs;
    for (const auto &r : pcgmi::recorded) pcgmi::play(r.hdr, r.slots, r.which);
    return hipSuccess;
}
}
