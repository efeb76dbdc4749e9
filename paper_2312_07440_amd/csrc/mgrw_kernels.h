// Kernel templates of libmgrw's QCD processes (one event per lane, several per
// wave, one per wave, programs split over kernels) and their launchers, shared
// by the per-process translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "../../include/mgrw.h"
#include "mgrw_event.h"
#include "mgrw_pool.h"

namespace mgrw {

constexpr int kBlock = 256;
constexpr int kMaxLaunchPoints = MGRW_MAX_POINTS + 1;   // base + new points
// Workgroups of one launch: HIP takes fewer than 2^32 threads in x.
constexpr int64_t kLaunchBlocks = (int64_t(1) << 32) / kBlock - 1;

// Device memory a launch may use for its intermediate buffers instead of
// allocating them.  ptr == nullptr: the launch allocates (stream-ordered).
// Otherwise the buffers are carved from [ptr, ptr + bytes) (ptr 256-byte
// aligned) and the events are processed in chunks whose buffers fit.
struct scratch_span {
    void* ptr;
    size_t bytes;
};

// Events per chunk when each event needs per_event bytes of scratch and the
// chunk a fixed head of head bytes (0 if not even one event fits).
inline int64_t scratch_chunk(const scratch_span& sc, size_t per_event, size_t head) {
    if (sc.bytes <= head || per_event == 0) return 0;
    return int64_t((sc.bytes - head) / per_event);
}

// Round up to the 256-byte alignment of every carved buffer.
constexpr size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Parameters travel by value with each launch (kernel-argument segment), so a
// later mgrw_set_params never races with work already queued.
struct qcd_launch {
    mgrw::qcd_point pts[kMaxLaunchPoints];
    int npts;        // points in pts (base first)
    int mode;        // 0: reweight, 1: |M|^2 of pts[0] only
    double mt;
    int mapping;     // MGRW_MAP_EVENT_PER_LANE or MGRW_MAP_EVENT_PER_WAVE; MGRW_MAP_AUTO: see lanes_faster
    int64_t batch;   // events of the whole call (the launch may be a piece of it)
    int kpoly;       // 1: kappa-polynomial evaluation (one program per helicity for all points)
    double rescue_tau;   // > 0: events with a gluon invariant |2 p_i.p_j|/s below it are redone in FP64
    hipEvent_t t0, t1;   // non-null: recorded around the amplitude kernel(s) of the launch
    int colour_mfma;     // split programs: colour sum on the matrix cores (after the last part)
    scratch_span scratch;   // non-null: caller-provided device scratch (no allocation; events in chunks)
};

struct ew_launch {
    mgrw::ew_point pts[kMaxLaunchPoints];
    int npts;
    int mode;
};

// e+ e- -> n photons: the coupling e = sqrt(4 pi alpha) of every point.
struct qed_launch {
    double e[kMaxLaunchPoints];
    int npts;
    int mode;
    int kpoly;       // 1: one evaluation at e = 1, |M|^2 = e^(2n) |M_1|^2 for every point
    hipEvent_t t0, t1;
    scratch_span scratch;
};

// Device-side timestamps around the amplitude kernel(s) of a launch.
inline void mark(hipEvent_t ev, hipStream_t s) {
    if (ev) (void)hipEventRecord(ev, s);
}

// Library-owned streams of the current device (default priority, created on
// first use, kept until the process ends), on which independent kernels of
// one call run beside the caller's stream.
constexpr int kAuxStreams = 3;
constexpr int kMaxDevices = 64;
inline hipError_t aux_streams(hipStream_t* out) {
    static std::mutex mu;
    static hipStream_t pool[kMaxDevices][kAuxStreams] = {};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < kAuxStreams; ++i) {
        if (!pool[dev][i]) {
            err = hipStreamCreateWithFlags(&pool[dev][i], hipStreamNonBlocking);
            if (err != hipSuccess) {
                pool[dev][i] = nullptr;
                return err;
            }
        }
        out[i] = pool[dev][i];
    }
    return hipSuccess;
}

template <int NEXT>
__device__ __forceinline__ void load_event(const double* __restrict__ mom, int64_t n, int64_t e,
                                           double (&p)[NEXT][4]) {
#pragma unroll
    for (int i = 0; i < NEXT; ++i)
#pragma unroll
        for (int m = 0; m < 4; ++m) p[i][m] = __builtin_nontemporal_load(mom + (int64_t(i) * 4 + m) * n + e);
}

// w_out[k-1][e] = W * (me_k / me_0), NaN where me_0 = 0 (eq. (3)).
__device__ __forceinline__ double reweighted(double w, double me, double me0) {
    return me0 != 0.0 ? w * (me / me0) : __builtin_nan("");
}

// Sum over groups of L consecutive lanes.
template <int L>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
    for (int o = L / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Per-lane LDS slot with an odd number of 32-bit words, so that lanes reading
// the same member hit distinct banks.
template <typename S>
struct lds_slot {
    S v;
    float pad[(sizeof(S) / 4) % 2 == 0 ? 1 : 2];
};

// The reweight loop of one event over the points (one call site, so the
// amplitude program is inlined once).
template <class Proc, typename T, typename KN, typename BS>
__device__ __forceinline__ void run_points(const KN& k, const BS& b, const qcd_launch& a, int64_t n, int64_t e,
                                           const double* __restrict__ w_in, double* __restrict__ out,
                                           double* __restrict__ me0_out) {
    const double w = (a.mode == 0 && w_in) ? w_in[e] : 1.0;
    double me0 = 0.0;
#pragma unroll 1
    for (int kp = 0; kp < a.npts; ++kp) {
        const double me = point_me<Proc, T>(k, b, a.pts[kp]);
        if (kp == 0) {
            me0 = me;
            if (a.mode == 1)
                out[e] = me;
            else if (me0_out)
                me0_out[e] = me;
        } else {
            out[int64_t(kp - 1) * n + e] = reweighted(w, me, me0);
        }
    }
}

// Lanes per workgroup of the one-event-per-lane kernel: in single precision
// each lane owns an LDS slot for its kinematics and bases, and the workgroup
// size is the one of 256, 128, 64 that keeps the most waves resident per CU
// within its 160 KiB of LDS (larger on ties).
constexpr int lane_waves_per_cu(size_t slot, int nb) {
    return slot * nb <= 160 * 1024 ? int((160 * 1024) / (slot * nb)) * (nb / 64) : 0;
}
template <class Proc, typename T>
constexpr int lane_block() {
    if constexpr (sizeof(T) == 4) {
        constexpr size_t slot = sizeof(lds_slot<typename Proc::template kin<T>>) +
                                sizeof(lds_slot<typename Proc::template basis<T>>);
        constexpr int w256 = lane_waves_per_cu(slot, 256), w128 = lane_waves_per_cu(slot, 128),
                      w64 = lane_waves_per_cu(slot, 64);
        return (w256 >= w128 && w256 >= w64) ? 256 : (w128 >= w64 ? 128 : 64);
    } else {
        return kBlock;
    }
}

// One event per lane (where lanes_faster says so, or on request).  In single
// precision the per-lane kinematics and wavefunction bases live in LDS (each
// lane owns a slot; no barriers); in double precision they stay in registers.
// Events 0 .. nb - 1 from the pointers on, whose rows are n apart.
template <class Proc, typename T>
__global__ void __launch_bounds__((lane_block<Proc, T>()))
qcd_kernel(const double* __restrict__ mom, const double* __restrict__ w_in, int64_t n, qcd_launch a,
           double* __restrict__ out, double* __restrict__ me0_out, int64_t nb) {
    constexpr int NB = lane_block<Proc, T>();
    const int64_t e = int64_t(blockIdx.x) * NB + threadIdx.x;
    if (e >= nb) return;   // no barriers below: early exit is safe
    double p[Proc::NEXT][4];
    load_event<Proc::NEXT>(mom, n, e, p);
    using KinT = typename Proc::template kin<T>;
    using BasT = typename Proc::template basis<T>;
    if constexpr (sizeof(T) == 4) {
        __shared__ lds_slot<KinT> ks[NB];
        __shared__ lds_slot<BasT> bs[NB];
        KinT& k = ks[threadIdx.x].v;
        BasT& b = bs[threadIdx.x].v;
        Proc::kinematics(p, a.mt, k);
        Proc::external_basis(p, a.mt, b);
        run_points<Proc, T>(k, b, a, n, e, w_in, out, me0_out);
    } else {
        KinT k;
        BasT b;
        Proc::kinematics(p, a.mt, k);
        Proc::external_basis(p, a.mt, b);
        run_points<Proc, T>(k, b, a, n, e, w_in, out, me0_out);
    }
}

// Several events per wave, one helicity configuration per lane (processes with
// fewer than 64 of them).  The first E lanes of a workgroup form the kinematics
// and bases of its E events in LDS, then every group of NHEL lanes takes an
// event: all points, the helicity sum across the group.  Against one event per
// lane, whose slots in LDS allow seven waves per CU: g g -> t tbar g, base + 16
// points, mixed (150 registers, three waves per SIMD), 262147 events 6.80 ->
// 4.84 ms, 10^6 events 20.5 -> 18.4; and 5000 events, which are 79 waves of the
// other kernel, 2.03 -> 0.15 ms with the re-evaluation.
// nhel = NHEL, as an argument: the loop over a lane's configurations keeps the
// program in a basic block of its own, where it rounds as it does in
// qcd_kernel.
template <class Proc, typename T, int E>
__global__ void __launch_bounds__(kBlock)
qcd_sub_kernel(const double* __restrict__ mom, const double* __restrict__ w_in, int64_t nb, int64_t n, int nhel,
               qcd_launch a, double* __restrict__ out, double* __restrict__ me0_out) {
    constexpr int L = Proc::NHEL;
    static_assert(L < 64 && 64 % L == 0 && E % (kBlock / L) == 0 && E <= kBlock, "whole groups");
    using KinT = typename Proc::template kin<T>;
    using BasT = typename Proc::template basis<T>;
    __shared__ lds_slot<KinT> ks[E];
    __shared__ lds_slot<BasT> bs[E];
    const int64_t first = int64_t(blockIdx.x) * E;
    if (threadIdx.x < E && first + threadIdx.x < nb) {
        double p[Proc::NEXT][4];
        load_event<Proc::NEXT>(mom, n, first + threadIdx.x, p);
        Proc::kinematics(p, a.mt, ks[threadIdx.x].v);
        Proc::external_basis(p, a.mt, bs[threadIdx.x].v);
    }
    __syncthreads();
    const int sub = threadIdx.x % L;
#pragma unroll 1
    for (int i = threadIdx.x / L; i < E; i += kBlock / L) {
        const int64_t e = first + i;
        if (e >= nb) return;   // whole groups of lanes; no barriers below
        const KinT& k = ks[i].v;
        const BasT& b = bs[i].v;
        const double w = (a.mode == 0 && w_in) ? w_in[e] : 1.0;
        double me0 = 0.0;
#pragma unroll 1
        for (int kp = 0; kp < a.npts; ++kp) {
            const qcd_point pt = a.pts[kp];
            double me = group_sum<L>(helicities_me<Proc, T>(k, b, pt, sub, L, nhel)) * Proc::point_norm(pt.gs);
            if (kp == 0) {
                me0 = me;
                if (sub == 0) {
                    if (a.mode == 1)
                        out[e] = me;
                    else if (me0_out)
                        me0_out[e] = me;
                }
            } else if (sub == 0) {
                out[int64_t(kp - 1) * n + e] = reweighted(w, me, me0);
            }
        }
    }
}

// ------------------------------------------------ one event per wave
//
// Lanes carry helicity configurations (h = lane + 64 c); the event's
// kinematics and wavefunctions are wave-uniform, computed once per event by
// qcd_setup_kernel.  The plain kernels and the split programs' in double
// precision stage that record in LDS, one copy per wave; the kappa-polynomial
// kernel and the single-precision parts read it through the scalar cache.  The
// helicity sum is a wave reduction.

#ifndef MGRW_WAVE_WPE
#define MGRW_WAVE_WPE 2
#endif

// Single-precision amplitudes lose digits where diagrams cancel strongly
// against each other: a final-state gluon nearly collinear to a beam gluon or
// to another final-state gluon (small |2 p_i.p_j| / s).  Such events are
// evaluated again in FP64 after the single-precision pass.
template <class Proc>
__device__ __forceinline__ bool ill_conditioned(const double (&p)[Proc::NEXT][4], double tau) {
    const double E = p[0][0] + p[1][0], X = p[0][1] + p[1][1], Y = p[0][2] + p[1][2], Z = p[0][3] + p[1][3];
    const double s = E * E - X * X - Y * Y - Z * Z;
    bool ill = false;
    // gluons: the beams (particles 0 and 1) and the final state (4 ...)
#pragma unroll
    for (int i = 0; i < Proc::NEXT; ++i) {
#pragma unroll
        for (int j = i + 1; j < Proc::NEXT; ++j) {
            const bool gi = i < 2 || i >= 4, gj = j < 2 || j >= 4;
            if (!gi || !gj || (i == 0 && j == 1)) continue;
            const double d = p[i][0] * p[j][0] - p[i][1] * p[j][1] - p[i][2] * p[j][2] - p[i][3] * p[j][3];
            ill = ill || (fabs(2.0 * d) < tau * s);
        }
    }
    return ill;
}

// An event's record: its kinematics and what its consumer makes the external
// wavefunctions from, their table (the kernels that stage the record in LDS) or
// their bases.  With both a g g -> t tbar g g record is 16 % larger.
template <class Proc, typename T>
struct table_record {
    typename Proc::template kin<T> k;
    typename Proc::template ext_table<T> t;
    int skip;   // 1: left to the FP64 re-evaluation
    template <typename P>
    __device__ __forceinline__ void fill(const P& p, double mt) {
        typename Proc::template basis<T> b;
        Proc::kinematics(p, mt, k);
        Proc::external_basis(p, mt, b);
        Proc::external_table(b, t);
    }
};
template <class Proc, typename T>
struct basis_record {
    typename Proc::template kin<T> k;
    typename Proc::template basis<T> b;
    int skip;
    template <typename P>
    __device__ __forceinline__ void fill(const P& p, double mt) {
        Proc::kinematics(p, mt, k);
        Proc::external_basis(p, mt, b);
    }
};

// Kinematics and wavefunction bases of every event; with tau > 0 also lists
// the ill-conditioned events (count, list) and marks them to be skipped.
// Events e0 .. e0 + nb - 1 of the n in mom; record el holds event e0 + el and
// the list holds event numbers.
template <class Proc, class Record>
__global__ void __launch_bounds__(kBlock)
qcd_setup_kernel(const double* __restrict__ mom, int64_t n, int64_t e0, int64_t nb, double mt,
                 Record* __restrict__ ev, double tau, unsigned long long* __restrict__ count,
                 int64_t* __restrict__ list) {
    const int64_t el = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (el >= nb) return;
    const int64_t e = e0 + el;
    double p[Proc::NEXT][4];
    load_event<Proc::NEXT>(mom, n, e, p);
    ev[el].fill(p, mt);
    int skip = 0;
    if (tau > 0.0 && ill_conditioned<Proc>(p, tau)) {
        skip = 1;
        list[atomicAdd(count, 1ull)] = e;
    }
    ev[el].skip = skip;
}

// An event's kinematics record, staged in LDS, as the generated programs
// should read it: each value loaded where the program uses it.  The record is
// wave-uniform; read through its plain address the compiler loads all of it
// ahead of the program and spills (from global memory: into scalar registers,
// then to vector lanes; from LDS: into vector registers, then to scratch).
// An opaque copy of the address keeps each read next to its use, and the
// assumption keeps the reads LDS reads (ds_read) rather than flat loads.  The
// address must be wave-uniform (it is held in scalar registers).
template <class K>
__device__ __forceinline__ const K& lds_near_use(const K& k) {
    const K* p = &k;
    __asm__ volatile("" : "+s"(p));
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_assume(__builtin_amdgcn_is_shared(reinterpret_cast<const void*>(p)));
#endif
    return *p;
}

// The double-precision kernels' record and wavefunctions: every closing group
// reads them through an address of its own.  Through one address for the
// whole program the compiler keeps what several groups read, and the currents
// formed from it, in registers from the first group to the last, and spills.
template <class K>
struct near_kin : K {};
template <class K>
__device__ __forceinline__ const near_kin<K>& near_view(const near_kin<K>& k) {
    MGRW_SCHED_BARRIER();
    return lds_near_use(k);
}
template <class E>
struct near_ext : E {};
struct near_lane {
    template <class V>
    __device__ __forceinline__ const V& operator()(const V& v) const {
        const V* p = &v;
        __asm__ volatile("" : "+v"(p));
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_assume(__builtin_amdgcn_is_shared(reinterpret_cast<const void*>(p)));
#endif
        return *p;
    }
};
template <class E>
__device__ __forceinline__ near_ext<E> near_view(const near_ext<E>& w) {
    return {w.map(near_lane{})};
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Points per pass of the one-event-per-wave kernels (and in double precision
// the accumulators kept in LDS).  The Lorentz chains of a pass hold no
// parameter and are formed once for its points; each point has its own
// closures' couplings, flows, colour sum and helicity sum.  g g -> t tbar g g,
// base + 16 points, amplitude kernel and re-evaluation, 2^20 events in single
// and 20011 in double precision: one point a pass 272 ms and 12.5 ms; two
// 190 ms, two with half of the first point's flows in LDS 213 ms (the LDS
// read-modify-writes cost more than the 98 spilled registers they save), three
// 262 ms (340 spilled); in double precision, bound by its 512 registers at one
// wave per SIMD, two 7.9 ms, three 7.0 ms with 34 of the 72 accumulators in
// LDS (7.8 with 26), four 8.9 ms.
constexpr int kPointsF32 = 2, kPointsF64 = 3, kCellsF64 = 34;
// The same for the split programs in double precision.
constexpr int kPointsSplit64 = 2;
template <typename T, int M>
struct pass_plan {
    static constexpr int NL = sizeof(T) == 4 || M == 1 ? 0 : kCellsF64;
};

// A wave's share of LDS: the event's kinematics, its wavefunctions, and the
// accumulators that the registers do not hold.
template <class Proc, typename T, int M>
struct wave_slot {
    alignas(16) typename Proc::template kin<T> k;
    alignas(16) typename Proc::template ext_table<T> t;
    alignas(16) cx<T> j[64 * pass_plan<T, M>::NL + 1];
};

// Copy an event's record into the wave's slot.
template <class D, class S>
__device__ __forceinline__ void stage_record(const D& ev, S& s, int lane) {
    static_assert(sizeof(s.k) % 4 == 0 && sizeof(s.t) % 4 == 0, "record copied in 32-bit words");
    const uint32_t* src = reinterpret_cast<const uint32_t*>(&ev.k);
    uint32_t* dst = reinterpret_cast<uint32_t*>(&s.k);
    for (int i = lane; i < int(sizeof(s.k) / 4); i += 64) dst[i] = src[i];
    src = reinterpret_cast<const uint32_t*>(&ev.t);
    dst = reinterpret_cast<uint32_t*>(&s.t);
    for (int i = lane; i < int(sizeof(s.t) / 4); i += 64) dst[i] = src[i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// M points of an event evaluated side by side: the flows' accumulators.
// In single precision the first point's are an array, as in a program for one
// point, and the further points' separate members, which are values from the
// start and take no place in the basic block's order of loads and stores
// (see rm).
template <typename T, int K>
struct flow_set {
    flow_set<T, K - 1> lo;
    cx<T> x = {T(0), T(0)};
    template <int I>
    __device__ __forceinline__ cx<T>& at() {
        if constexpr (I == K - 1)
            return x;
        else
            return lo.template at<I>();
    }
};
template <typename T>
struct flow_set<T, 0> {};
template <typename T, int K, int M>
struct point_acc {
    cx<T> J[K];
    flow_set<T, K> more[M > 1 ? M - 1 : 1];
    __device__ __forceinline__ void clear() {
        for (int i = 0; i < K; ++i) J[i] = {T(0), T(0)};
    }
};
template <int I, typename T, int K, int M, int... m>
__device__ __forceinline__ void jadd_more(point_acc<T, K, M>& J, const cm<T, M>& s, std::integer_sequence<int, m...>) {
    ((J.more[m].template at<I>() = J.more[m].template at<I>() + s.v[m + 1]), ...);
}
template <int I, typename T, int K, int M, int... m>
__device__ __forceinline__ void jsub_more(point_acc<T, K, M>& J, const cm<T, M>& s, std::integer_sequence<int, m...>) {
    ((J.more[m].template at<I>() = J.more[m].template at<I>() - s.v[m + 1]), ...);
}
template <int I, typename T, int K, int M>
__device__ __forceinline__ void jadd(point_acc<T, K, M>& J, const cm<T, M>& s) {
    J.J[I] = J.J[I] + s.v[0];
    jadd_more<I>(J, s, points_seq<M - 1>{});
}
template <int I, typename T, int K, int M>
__device__ __forceinline__ void jsub(point_acc<T, K, M>& J, const cm<T, M>& s) {
    J.J[I] = J.J[I] - s.v[0];
    jsub_more<I>(J, s, points_seq<M - 1>{});
}
template <int I, typename T, int K, int KK>
__device__ __forceinline__ void flows_out(flow_set<T, K>& x, cx<T> (&J)[KK]) {
    if constexpr (I < KK) {
        J[I] = x.template at<I>();
        flows_out<I + 1>(x, J);
    }
}
template <class Proc, typename T, int K, int M>
__device__ __forceinline__ void colour_points(point_acc<T, K, M>& J, double (&acc)[M]) {
    acc[0] += double(Proc::colour_sum(J.J));
#pragma unroll
    for (int m = 1; m < M; ++m) {
        cx<T> Jm[K];
        flows_out<0>(J.more[m - 1], Jm);
        acc[m] += double(Proc::colour_sum(Jm));
    }
}

// In double precision: entry q = m K + i (flow i of point m), the first NL of
// them in the lane's LDS column (entry q at lds[64 q]) and the others in
// registers.  The program's indices are constants, so each access resolves to
// one storage at compile time.
// Indices are expanded from packs, not loops: the entries in registers are then
// values from the start, not an array that loops index until late in the
// compilation (which left 2.2 times the spilled registers' worth of code).
template <int K, int M, int NL>
struct point_cells {
    cx<double>* lds;
    cx<double> reg[M * K - NL];
    template <int Q>
    __device__ __forceinline__ cx<double> get() const {
        if constexpr (Q < NL)
            return lds[64 * Q];
        else
            return reg[Q - NL];
    }
    template <int Q>
    __device__ __forceinline__ void set(cx<double> x) {
        if constexpr (Q < NL)
            lds[64 * Q] = x;
        else
            reg[Q - NL] = x;
    }
    template <int... q>
    __device__ __forceinline__ void clear(std::integer_sequence<int, q...>) { (set<q>({0.0, 0.0}), ...); }
    __device__ __forceinline__ void clear() { clear(points_seq<M * K>{}); }
    // point m's flows from / to memory (flow f at p[2 f stride], p[(2 f + 1) stride])
    template <int m, int... f>
    __device__ __forceinline__ void load(const double* p, int stride, std::integer_sequence<int, f...>) {
        (set<m * K + f>({p[2 * f * stride], p[(2 * f + 1) * stride]}), ...);
    }
    template <int m, int... f>
    __device__ __forceinline__ void store(double* p, int stride, std::integer_sequence<int, f...>) const {
        ((p[2 * f * stride] = get<m * K + f>().re, p[(2 * f + 1) * stride] = get<m * K + f>().im), ...);
    }
    template <int m, int... f>
    __device__ __forceinline__ void flows(cx<double>* J, std::integer_sequence<int, f...>) const {
        ((J[f] = get<m * K + f>()), ...);
    }
};
template <int I, int K, int M, int NL, int... m>
__device__ __forceinline__ void jadd_cells(point_cells<K, M, NL>& J, const cm<double, M>& s,
                                           std::integer_sequence<int, m...>) {
    (J.template set<m * K + I>(J.template get<m * K + I>() + s.v[m]), ...);
}
template <int I, int K, int M, int NL, int... m>
__device__ __forceinline__ void jsub_cells(point_cells<K, M, NL>& J, const cm<double, M>& s,
                                           std::integer_sequence<int, m...>) {
    (J.template set<m * K + I>(J.template get<m * K + I>() - s.v[m]), ...);
}
template <int I, int K, int M, int NL>
__device__ __forceinline__ void jadd(point_cells<K, M, NL>& J, const cm<double, M>& s) {
    jadd_cells<I>(J, s, points_seq<M>{});
}
template <int I, int K, int M, int NL>
__device__ __forceinline__ void jsub(point_cells<K, M, NL>& J, const cm<double, M>& s) {
    jsub_cells<I>(J, s, points_seq<M>{});
}
template <class Proc, int m, int K, int M, int NL>
__device__ __forceinline__ double colour_cell(const point_cells<K, M, NL>& J) {
    cx<double> Jm[K];
    J.template flows<m>(Jm, points_seq<K>{});
    return Proc::colour_sum(Jm);
}
template <class Proc, int K, int M, int NL, int... m>
__device__ __forceinline__ void colour_cells(const point_cells<K, M, NL>& J, double (&acc)[M],
                                             std::integer_sequence<int, m...>) {
    ((acc[m] += colour_cell<Proc, m>(J)), ...);
}
template <class Proc, int K, int M, int NL>
__device__ __forceinline__ void colour_points(const point_cells<K, M, NL>& J, double (&acc)[M]) {
    colour_cells<Proc>(J, acc, points_seq<M>{});
}

template <class Proc, typename T, typename W, typename KN, typename C, typename JA>
__device__ __forceinline__ void amplitude_points(const W& w, const KN& k, const C& c, JA& J) {
    J.clear();
    Proc::template program<T>(w, k, c, J);
}

// |M|^2 of one event at points first .. first + M - 1 (of npts), summed over
// the helicity configurations on the wave's lanes; the same value in every
// lane.  s.k and s.t hold the event.
template <class Proc, typename T, int M>
__device__ __forceinline__ void pass_me(wave_slot<Proc, T, M>& s, const qcd_launch& a, int first, int lane,
                                        double (&me)[M]) {
    constexpr int K = Proc::K;
    const auto c = couplings_of<Proc, T, M>(a.pts, first, a.npts);
    double acc[M] = {};
#pragma unroll 1
    for (int hc = 0; hc < Proc::NHEL; hc += 64) {
        __asm__ volatile("" ::: "memory");
        const auto w = Proc::template ext_at<T>(s.t, hc + lane);
        if constexpr (sizeof(T) == 4) {
            point_acc<T, K, M> J;
            amplitude_points<Proc, T>(w, lds_near_use(s.k), c, J);
            colour_points<Proc>(J, acc);
        } else {
            point_cells<K, M, pass_plan<T, M>::NL> J{&s.j[lane], {}};
            amplitude_points<Proc, T>(w, lds_near_use(s.k), c, J);
            colour_points<Proc>(J, acc);
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
        me[m] = wave_sum(acc[m]) * Proc::point_norm(a.pts[first + m < a.npts ? first + m : a.npts - 1].gs);
}

// |M|^2 of point kp of event e: the base point's to me0[i], a new point's to
// its place in out, where reweight_ratio_kernel replaces it by the weight.
__device__ __forceinline__ void store_me(double me, int kp, int64_t e, int64_t i, int64_t n, const qcd_launch& a,
                                         double* __restrict__ out, double* __restrict__ me0) {
    if (kp >= a.npts) return;
    if (kp > 0)
        out[int64_t(kp - 1) * n + e] = me;
    else if (a.mode == 1)
        out[e] = me;
    else
        me0[i] = me;
}

// Eq. (3) for events e0 .. e0 + nb - 1 once their |M|^2 are in out and me0
// (w[i], me0[i]: input weight, if any, and base point of event e0 + i); grid
// (events, new points).
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK)
reweight_ratio_kernel(const double* w, const double* me0, int64_t e0, int64_t nb, int64_t n, double* out) {
    const int64_t i = int64_t(blockIdx.x) * BLOCK + threadIdx.x;
    if (i >= nb) return;
    const int64_t at = int64_t(blockIdx.y) * n + e0 + i;
    out[at] = reweighted(w ? w[i] : 1.0, out[at], me0[i]);
}

// Input weights set aside where out or me0 overlap them: |M|^2 is written there
// before the weights are read.
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) copy_weights_kernel(const double* w, int64_t nb, double* to) {
    const int64_t i = int64_t(blockIdx.x) * BLOCK + threadIdx.x;
    if (i < nb) to[i] = w[i];
}
inline bool overlap(const double* a, int64_t na, const double* b, int64_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + 8 * uintptr_t(nb) && y < x + 8 * uintptr_t(na);
}

// Events from which on a unit of work is a whole event; below, one pass, so
// that a small batch fills the chip (2048 waves in single precision, 1024 in
// double).  1000 events x 17 points: 305 us against 1150 with whole events.  Once
// whole events fill the chip (2048 events) they are faster, as they stage their
// record once: by 1-4 % in single precision at 3, 5, 17 and 65 points, by 3-8 % in
// double at 5 and more; units of one pass are faster where few whole events are
// left for the last round (9000 events in single precision: 1-7 %; 33000: 0.3 %
// at 17 points), the less so the more rounds there are: eight at 16384.
constexpr int64_t kWholeEvents = 16384;

// One wave's unit of work: event e0 + el, passes [u per, (u + 1) per) over its
// points, M points a pass.  Bound by VALU issue: a wave issues at most one
// vector instruction per four cycles and a SIMD takes two, so two waves per
// SIMD (256 registers) are needed and one runs at half rate.
template <class Proc, typename T, int M>
__global__ void __launch_bounds__(kBlock, sizeof(T) == 4 ? MGRW_WAVE_WPE : 1)
qcd_wave_kernel(const table_record<Proc, T>* __restrict__ ev, int64_t e0, int64_t nb, int64_t n, int units, int per,
                qcd_launch a, double* __restrict__ out, double* __restrict__ me0) {
    static_assert(Proc::NHEL % 64 == 0, "helicity configurations must fill whole waves");
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t id = int64_t(blockIdx.x) * (kBlock / 64) + wv;
    const int64_t el = id / units;
    if (el >= nb || ev[el].skip) return;   // whole wave; no barriers below
    const int lane = threadIdx.x & 63;
    // the event's record, staged once per unit in LDS: the program reads the
    // kinematics with broadcast loads, the wavefunctions at the lane's
    // helicities
    using S = wave_slot<Proc, T, M>;
    __shared__ S sl[kBlock / 64];
    S& s = sl[wv];
    stage_record(ev[el], s, lane);
    const int k0 = int(id - el * units) * per * M, k1 = k0 + per * M < a.npts ? k0 + per * M : a.npts;
#pragma unroll 1
    for (int kp = k0; kp < k1; kp += M) {
        double me[M];
        pass_me<Proc, T, M>(s, a, kp, lane, me);
        if (lane == 0)
#pragma unroll
            for (int m = 0; m < M; ++m) store_me(me[m], kp + m, e0 + el, el, n, a, out, me0);
    }
}

// ------------------------------------------------ kappa-polynomial kernels

// Outputs of one event from its helicity-summed B.
template <class Proc>
__device__ __forceinline__ void kpoly_outputs(const double* B, const qcd_launch& a, int64_t n, int64_t e,
                                              double w, double* __restrict__ out, double* __restrict__ me0_out) {
    double me0 = 0.0;
    for (int kp = 0; kp < a.npts; ++kp) {
        const double me = kpoly_me<Proc>(B, a.pts[kp].gs, a.pts[kp].gk / a.pts[kp].gs);
        if (kp == 0) {
            me0 = me;
            if (a.mode == 1)
                out[e] = me;
            else if (me0_out)
                me0_out[e] = me;
        } else {
            out[int64_t(kp - 1) * n + e] = reweighted(w, me, me0);
        }
    }
}

// One event per lane (processes with fewer than 64 helicity configurations).
template <class Proc, typename T>
__global__ void __launch_bounds__(kBlock)
qcd_kpoly_lane_kernel(const double* __restrict__ mom, const double* __restrict__ w_in, int64_t nb, int64_t n,
                      qcd_launch a, double* __restrict__ out, double* __restrict__ me0_out) {
    const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (e >= nb) return;
    double p[Proc::NEXT][4];
    load_event<Proc::NEXT>(mom, n, e, p);
    typename Proc::template kin<T> k;
    typename Proc::template basis<T> b;
    Proc::kinematics(p, a.mt, k);
    Proc::external_basis(p, a.mt, b);
    double B[kpoly_pairs<Proc>()] = {};
#pragma unroll 1
    for (int h = 0; h < Proc::NHEL; ++h) kpoly_helicity<Proc, T>(k, b, h, B);
    kpoly_outputs<Proc>(B, a, n, e, (a.mode == 0 && w_in) ? w_in[e] : 1.0, out, me0_out);
}

// Accumulators of the kappa-polynomial program with the first NL complex
// entries in the lane's LDS column (entry i at lds[i * S]) and the others in
// registers; the program's indices are constants after inlining, so each
// access resolves to one storage at compile time.
template <typename T, int N, int NL, int S>
struct split_acc {
    cx<T>* lds;
    cx<T> reg[N - NL];
    __device__ __forceinline__ cx<T>& operator[](int i) { return i < NL ? lds[i * S] : reg[i - NL]; }
};

// Large single-precision programs (NG K >= 96 accumulators) keep half of
// their kappa-power accumulators in LDS while the program runs.
template <class Proc, typename T>
constexpr bool kpoly_lds_split() {
    return sizeof(T) == 4 && Proc::NG * Proc::K >= 96;
}

// One event per wave, helicity configurations on the lanes.
template <class Proc, typename T>
__global__ void __launch_bounds__(kBlock)
qcd_kpoly_wave_kernel(const basis_record<Proc, T>* __restrict__ ev, int64_t e0, int64_t nb,
                      const double* __restrict__ w_in, int64_t n, qcd_launch a, double* __restrict__ out,
                      double* __restrict__ me0_out) {
    const int64_t el = int64_t(blockIdx.x) * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (el >= nb || ev[el].skip) return;   // whole wave
    const int64_t e = e0 + el;
    const int lane = threadIdx.x & 63;
    double B[kpoly_pairs<Proc>()] = {};
#pragma unroll 1
    for (int hc = 0; hc < Proc::NHEL; hc += 64) {
        __asm__ volatile("" ::: "memory");
        if constexpr (kpoly_lds_split<Proc, T>()) {
            constexpr int N = Proc::NG * Proc::K, NL = N / 2;
            __shared__ cx<T> jl[NL * kBlock];
            split_acc<T, N, NL, kBlock> acc{&jl[threadIdx.x]};
            typename Proc::template ext<T> w;
            typename Proc::template coup<T> c = {T(1), T(1), T(1)};
            Proc::template external<T>(ev[el].b, hc + lane, w);
            Proc::amplitude_kpoly(w, ev[el].k, c, acc);
            cx<T> J[N];
#pragma unroll
            for (int i = 0; i < N; ++i) J[i] = acc[i];
            kpoly_colour<Proc, T>(J, B);
        } else if constexpr (sizeof(T) == 8) {
            // double precision: external wavefunctions in the lane's own LDS
            // slot (10 % faster for g g -> t tbar g g; in single precision
            // registers are faster)
            __shared__ lds_slot<typename Proc::template ext<T>> wfs[kBlock];
            kpoly_helicity<Proc, T>(ev[el].k, ev[el].b, hc + lane, B, wfs[threadIdx.x].v);
        } else {
            kpoly_helicity<Proc, T>(ev[el].k, ev[el].b, hc + lane, B);
        }
    }
#pragma unroll
    for (int i = 0; i < kpoly_pairs<Proc>(); ++i) B[i] = wave_sum(B[i]);
    if (lane == 0) kpoly_outputs<Proc>(B, a, n, e, (a.mode == 0 && w_in) ? w_in[e] : 1.0, out, me0_out);
}

// ------------------------------------- FP64 rescue of ill-conditioned events
//
// In single precision the helicity amplitudes lose digits where diagrams
// cancel strongly against each other: a final-state gluon nearly collinear to
// a beam gluon or to another final-state gluon (small |2 p_i.p_j| / s).  After
// the single-precision pass, events with such an invariant below a threshold
// are listed and evaluated again in double precision, one event per wave,
// overwriting their results.

template <class Proc>
__global__ void rescue_reset_kernel(unsigned long long* count) {
    if (blockIdx.x == 0 && threadIdx.x == 0) count[0] = 0;
}

// Events 0 .. nb - 1 from mom on, whose rows are n apart.
template <class Proc>
__global__ void __launch_bounds__(kBlock)
rescue_flag_kernel(const double* __restrict__ mom, int64_t n, int64_t nb, double tau,
                   unsigned long long* __restrict__ count, int64_t* __restrict__ list) {
    const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (e >= nb) return;
    double p[Proc::NEXT][4];
    load_event<Proc::NEXT>(mom, n, e, p);
    if (ill_conditioned<Proc>(p, tau)) list[atomicAdd(count, 1ull)] = e;
}

// Grid-stride over the listed events; each wave takes one event at a time and
// every wave leaves the loop once the list is exhausted (kappa polynomial).
template <class Proc>
__global__ void __launch_bounds__(kBlock, 1)
qcd_rescue_kpoly_kernel(const double* __restrict__ mom, const int64_t* __restrict__ list,
                        const unsigned long long* __restrict__ count, const double* __restrict__ w_in, int64_t n,
                        qcd_launch a, double* __restrict__ out, double* __restrict__ me0_out) {
    struct event {
        typename Proc::template kin<double> k;
        typename Proc::template basis<double> b;
    };
    __shared__ event sh[kBlock / 64];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t cnt = int64_t(count[0]);
    const int64_t stride = int64_t(gridDim.x) * (kBlock / 64);
    event& d = sh[wv];
#pragma unroll 1
    for (int64_t i = int64_t(blockIdx.x) * (kBlock / 64) + wv; i < cnt; i += stride) {
        const int64_t e = list[i];
        if (lane == 0) {
            double p[Proc::NEXT][4];
            load_event<Proc::NEXT>(mom, n, e, p);
            Proc::kinematics(p, a.mt, d.k);
            Proc::external_basis(p, a.mt, d.b);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const double w = (a.mode == 0 && w_in) ? w_in[e] : 1.0;
        double B[kpoly_pairs<Proc>()] = {};
#pragma unroll 1
        for (int hc = 0; hc < Proc::NHEL; hc += 64)
            if (hc + lane < Proc::NHEL) kpoly_helicity<Proc, double>(d.k, d.b, hc + lane, B);
#pragma unroll
        for (int q = 0; q < kpoly_pairs<Proc>(); ++q) B[q] = wave_sum(B[q]);
        if (lane == 0) kpoly_outputs<Proc>(B, a, n, e, w, out, me0_out);
        // every lane has read the slot before the next event overwrites it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// The same after the kernels that write weights directly: a workgroup deals the
// points of its listed events to groups of as many lanes as there are helicity
// configurations (at most 64), so that all lanes work and a short list's
// latency is that of a few points.  Lists longer than the grid go several
// events at a time, whose kinematics are formed side by side and whose points
// fill the groups also where there are fewer points than groups.  g g -> t tbar
// g: 300 events x 17 points 180 -> 99 us against one wave per event, half of
// its lanes idle, points one by one; 1.5 10^6 events, 2 % of them listed, at one point 862 ->
// 290 us of re-evaluation (one event at a time left seven of eight groups idle;
// one wave per event: 262), two points 755 -> 246.
constexpr int kRedoEvents = 8;
template <class Proc>
__global__ void __launch_bounds__(kBlock, 1)
qcd_rescue_kernel(const double* __restrict__ mom, const int64_t* __restrict__ list,
                  const unsigned long long* __restrict__ count, const double* __restrict__ w_in, int64_t n, int nhel,
                  qcd_launch a, double* __restrict__ out, double* __restrict__ me0_out) {
    constexpr int L = Proc::NHEL < 64 ? Proc::NHEL : 64;
    __shared__ typename Proc::template kin<double> k[kRedoEvents];
    __shared__ typename Proc::template basis<double> b[kRedoEvents];
    __shared__ double mes[kRedoEvents * kMaxLaunchPoints];
    const int64_t cnt = int64_t(count[0]);
    const int64_t share = (cnt + gridDim.x - 1) / gridDim.x;
    const int per = share < kRedoEvents ? int(share) : kRedoEvents;
    const int sub = threadIdx.x % L;
#pragma unroll 1
    for (int64_t i0 = int64_t(blockIdx.x) * per; i0 < cnt; i0 += int64_t(gridDim.x) * per) {   // whole workgroup
        const int m = cnt - i0 < per ? int(cnt - i0) : per;
        if (threadIdx.x < m) {
            double p[Proc::NEXT][4];
            load_event<Proc::NEXT>(mom, n, list[i0 + threadIdx.x], p);
            Proc::kinematics(p, a.mt, k[threadIdx.x]);
            Proc::external_basis(p, a.mt, b[threadIdx.x]);
        }
        __syncthreads();
#pragma unroll 1
        for (int u = threadIdx.x / L; u < m * a.npts; u += kBlock / L) {
            const int i = u / a.npts;
            const qcd_point pt = a.pts[u - i * a.npts];
            const double me = group_sum<L>(helicities_me<Proc, double>(k[i], b[i], pt, sub, L, nhel));
            if (sub == 0) mes[u] = me * Proc::point_norm(pt.gs);
        }
        __syncthreads();
        for (int u = threadIdx.x; u < m * a.npts; u += kBlock) {
            const int i = u / a.npts, kp = u - i * a.npts;
            const int64_t e = list[i0 + i];
            if (kp > 0)
                out[int64_t(kp - 1) * n + e] = reweighted(w_in ? w_in[e] : 1.0, mes[u], mes[i * a.npts]);
            else if (a.mode == 1)
                out[e] = mes[u];
            else if (me0_out)
                me0_out[e] = mes[u];
        }
        __syncthreads();   // the next events overwrite the shared data
    }
}

// The same for the one-event-per-wave pipeline: M points a pass, the listed
// events' points split over waves while the list is short (a unit is then one
// pass), |M|^2 to out and me0 (of event e: me0[e - e0]).
template <class Proc, int M>
__global__ void __launch_bounds__(kBlock, 1)
qcd_redo_kernel(const double* __restrict__ mom, const int64_t* __restrict__ list,
                const unsigned long long* __restrict__ count, int64_t n, int64_t e0, qcd_launch a,
                double* __restrict__ out, double* __restrict__ me0) {
    __shared__ wave_slot<Proc, double, M> sl[kBlock / 64];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t cnt = int64_t(count[0]);
    const int64_t stride = int64_t(gridDim.x) * (kBlock / 64);
    const int passes = (a.npts + M - 1) / M;
    const int units = cnt < kWholeEvents ? passes : 1, per = passes / units;
    wave_slot<Proc, double, M>& s = sl[wv];
#pragma unroll 1
    for (int64_t id = int64_t(blockIdx.x) * (kBlock / 64) + wv; id < cnt * units; id += stride) {
        const int64_t i = id / units;
        const int64_t e = list[i];
        if (lane == 0) {
            double p[Proc::NEXT][4];
            load_event<Proc::NEXT>(mom, n, e, p);
            typename Proc::template basis<double> b;
            Proc::kinematics(p, a.mt, s.k);
            Proc::external_basis(p, a.mt, b);
            Proc::external_table(b, s.t);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int k0 = int(id - i * units) * per * M, k1 = k0 + per * M < a.npts ? k0 + per * M : a.npts;
#pragma unroll 1
        for (int kp = k0; kp < k1; kp += M) {
            double me[M];
            pass_me<Proc, double, M>(s, a, kp, lane, me);
            if (lane == 0)
#pragma unroll
                for (int m = 0; m < M; ++m) store_me(me[m], kp + m, e, e - e0, n, a, out, me0);
        }
        // every lane has read the slot before the next event overwrites it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

constexpr unsigned kRescueBlocks = 1024;

// |M|^2 of events e0 .. e0 + nb - 1 from their records, M points a pass, then
// (list non-null) of the listed ones again in double precision.
template <class Proc, typename T, int M>
void launch_passes(const table_record<Proc, T>* ev, const double* mom, int64_t n, int64_t e0, int64_t nb,
                   const int64_t* list, const unsigned long long* count, const qcd_launch& a, double* out,
                   double* me0, hipStream_t s) {
    const int passes = (a.npts + M - 1) / M;
    const int units = nb < kWholeEvents ? passes : 1, per = passes / units;
    mark(a.t0, s);
    hipLaunchKernelGGL((qcd_wave_kernel<Proc, T, M>), dim3(unsigned((nb * units + kBlock / 64 - 1) / (kBlock / 64))),
                       dim3(kBlock), 0, s, ev, e0, nb, n, units, per, a, out, me0);
    mark(a.t1, s);
    if constexpr (sizeof(T) == 4)
        if (list)
            hipLaunchKernelGGL((qcd_redo_kernel<Proc, M == 1 ? 1 : kPointsF64>), dim3(kRescueBlocks), dim3(kBlock), 0, s, mom, list, count,
                               n, e0, a, out, me0);
}

// One event per wave: per-event data (in single precision with the rescue
// on, also the list of ill-conditioned events, which the amplitude kernel
// skips), the amplitude kernel, the FP64 re-evaluation of the listed events,
// then (plain evaluation) the weights from |M|^2.  KP: kappa-polynomial
// evaluation.  Without a scratch span the buffers are one stream-ordered
// allocation for all n events; with one they are carved from it and the events
// run in chunks whose buffers fit.  Buffers: records, count and list, |M|^2 at
// the base point (where the caller does not want it), input weights set aside.
template <class Proc, typename T, bool KP>
hipError_t launch_wave_pipeline(const double* mom, const double* w_in, int64_t n, const qcd_launch& a, double* out,
                                double* me0, hipStream_t s) {
    const bool rescue = sizeof(T) == 4 && a.rescue_tau > 0.0 && Proc::NEXT > 4;
    const bool base = !KP && a.mode == 0 && !me0;   // room for |M|^2 at the base point
    using ED = std::conditional_t<KP, basis_record<Proc, T>, table_record<Proc, T>>;
    // room for the input weights, where the outputs overlap them
    const bool aside = !KP && a.mode == 0 && (overlap(w_in, n, out, (a.npts - 1) * n) || overlap(w_in, n, me0, n));
    const size_t words = (rescue ? 1 : 0) + (base ? 1 : 0) + (aside ? 1 : 0);
    int64_t chunk = n;
    char* mem = static_cast<char*>(a.scratch.ptr);
    if (mem) {
        chunk = scratch_chunk(a.scratch, sizeof(ED) + words * 8, 1536);
        if (chunk < 1) return hipErrorInvalidValue;
        if (chunk > n) chunk = n;
    } else {
        hipError_t err = work_alloc(reinterpret_cast<void**>(&mem), align256(sizeof(ED) * size_t(n)) + 512 +
                                        words * align256(8 * size_t(n)), s);
        if (err != hipSuccess) return err;
    }
    ED* ev = reinterpret_cast<ED*>(mem);
    char* at = mem + align256(sizeof(ED) * size_t(chunk));
    unsigned long long* count = nullptr;
    int64_t* list = nullptr;
    if (rescue) {
        count = reinterpret_cast<unsigned long long*>(at);
        list = reinterpret_cast<int64_t*>(at + 256);
        at += 256 + align256(8 * size_t(chunk));
    }
    double* m0_buf = reinterpret_cast<double*>(at);
    if (base) at += align256(8 * size_t(chunk));
    double* w_buf = reinterpret_cast<double*>(at);
    hipError_t err = hipSuccess;
    for (int64_t e0 = 0; e0 < n && err == hipSuccess; e0 += chunk) {
        const int64_t nb = n - e0 < chunk ? n - e0 : chunk;
        if (rescue) hipLaunchKernelGGL((rescue_reset_kernel<Proc>), dim3(1), dim3(64), 0, s, count);
        hipLaunchKernelGGL((qcd_setup_kernel<Proc, ED>), dim3(unsigned((nb + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           s, mom, n, e0, nb, a.mt, ev, rescue ? a.rescue_tau : 0.0, count, list);
        if constexpr (KP) {
            mark(a.t0, s);
            hipLaunchKernelGGL((qcd_kpoly_wave_kernel<Proc, T>), dim3(unsigned((nb + kBlock / 64 - 1) / (kBlock / 64))),
                               dim3(kBlock), 0, s, ev, e0, nb, w_in, n, a, out, me0);
            mark(a.t1, s);
            if (rescue)
                hipLaunchKernelGGL((qcd_rescue_kpoly_kernel<Proc>), dim3(kRescueBlocks), dim3(kBlock), 0, s, mom,
                                   list, count, w_in, n, a, out, me0);
        } else {
            double* m0 = base ? m0_buf : (me0 ? me0 + e0 : nullptr);
            const double* w = w_in ? w_in + e0 : nullptr;
            const unsigned blocks = unsigned((nb + kBlock - 1) / kBlock);
            if (aside) {
                hipLaunchKernelGGL((copy_weights_kernel<kBlock>), dim3(blocks), dim3(kBlock), 0, s, w, nb, w_buf);
                w = w_buf;
            }
            constexpr int M = sizeof(T) == 4 ? kPointsF32 : kPointsF64;
            if (a.npts > 1)
                launch_passes<Proc, T, M>(ev, mom, n, e0, nb, list, count, a, out, m0, s);
            else
                launch_passes<Proc, T, 1>(ev, mom, n, e0, nb, list, count, a, out, m0, s);
            if (a.mode == 0 && a.npts > 1)
                hipLaunchKernelGGL((reweight_ratio_kernel<kBlock>), dim3(blocks, unsigned(a.npts - 1)), dim3(kBlock),
                                   0, s, w, m0, e0, nb, n, out);
        }
        err = hipGetLastError();
    }
    if (a.scratch.ptr) return err;
    hipError_t ferr = hipFreeAsync(mem, s);
    return err != hipSuccess ? err : ferr;
}

// ------------------------------------------- programs split over kernels
//
// For the largest process the per-helicity program is split into NCHUNK
// functions (consecutive closing groups); kernel C runs part C for every
// point and helicity of a batch of events, one event per wave with the
// helicity configurations on the lanes.  The colour-flow amplitudes J travel
// between the parts through HBM in a [event][point][component][helicity]
// layout, the helicities in blocks of 64 (consecutive lanes touch consecutive
// words, and one pass's flows are one contiguous piece).  By default the last
// part forms the colour sum (VALU) and the helicity sum (wave reduction), which
// is |M|^2; with the matrix-core colour sum selected it stores J too, and
// qcd_colour_mfma_kernel contracts J with the colour matrix.
// reweight_ratio_kernel forms the weights, after the FP64 re-evaluation.

// Processes whose generated struct provides the bfloat16 split of the colour
// matrix (MFMA_COLOUR) take the matrix-core colour sum.
template <class P, class = void>
struct mfma_colour : std::false_type {};
template <class P>
struct mfma_colour<P, std::void_t<decltype(P::MFMA_COLOUR)>> : std::bool_constant<P::MFMA_COLOUR> {};

#ifndef MGRW_PART_WPE
#define MGRW_PART_WPE 1
#endif

// One wave's unit of work: points [u per, (u + 1) per) of one event.
template <class Proc, typename T, int C, bool STORE_LAST>
__global__ void __launch_bounds__(kBlock, MGRW_PART_WPE)
qcd_part_kernel(const basis_record<Proc, T>* __restrict__ ev, int64_t e0, int64_t nb, T* __restrict__ jbuf, int64_t n,
                int units, int per, qcd_launch a, double* __restrict__ out, double* __restrict__ me0) {
    constexpr int NH = Proc::NHEL, K2 = 2 * Proc::K;
    constexpr bool LAST = C + 1 == Proc::NCHUNK && !STORE_LAST;   // finishes the events here
    static_assert(NH % 64 == 0, "helicity configurations must fill whole waves");
    const int64_t id = int64_t(blockIdx.x) * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t el = id / units;
    if (el >= nb) return;   // whole wave; no barriers below
    const int64_t e = e0 + el;
    if (ev[e].skip) return;   // left to the FP64 re-evaluation
    const int lane = threadIdx.x & 63;
    const typename Proc::template kin<T>& k = ev[e].k;
    const typename Proc::template basis<T>& b = ev[e].b;
    const int k0 = int(id - el * units) * per, k1 = k0 + per < a.npts ? k0 + per : a.npts;
#pragma unroll 1
    for (int kp = k0; kp < k1; ++kp) {
        const qcd_point pt = a.pts[kp];
        const auto c = Proc::template couplings<T>(pt.gs, pt.gs2, pt.gk);
        double acc = 0.0;
#pragma unroll 1
        for (int hc = 0; hc < NH; hc += 64) {
            __asm__ volatile("" ::: "memory");
            __shared__ lds_slot<typename Proc::template ext<T>> wfs[kBlock];
            typename Proc::template ext<T>& wf = wfs[threadIdx.x].v;   // own slot: in registers it would spill
            Proc::template external<T>(b, hc + lane, wf);
            T* jp = jbuf + (el * a.npts + kp) * int64_t(K2) * NH + hc * K2 + lane;
            cx<T> J[Proc::K];
            if constexpr (C == 0) {
#pragma unroll
                for (int f = 0; f < Proc::K; ++f) J[f] = {T(0), T(0)};
            } else {
#pragma unroll
                for (int f = 0; f < Proc::K; ++f) J[f] = {jp[(2 * f) * 64], jp[(2 * f + 1) * 64]};
            }
            Proc::template amplitude_part<C, T>(wf, k, c, J);
            if constexpr (!LAST) {
#pragma unroll
                for (int f = 0; f < Proc::K; ++f) {
                    jp[(2 * f) * 64] = J[f].re;
                    jp[(2 * f + 1) * 64] = J[f].im;
                }
            } else {
                acc += double(Proc::colour_sum(J));
            }
        }
        if constexpr (LAST) {
            const double me = wave_sum(acc) * Proc::point_norm(pt.gs);
            if (lane == 0) store_me(me, kp, e, e, n, a, out, me0);
        }
    }
}

// Waves that run at once at one per SIMD.
constexpr int64_t kWaves1 = 1024;

// Units per event of part C: whole events or single points.  A unit loads and
// stores the flows once per pass either way, but a wave that goes on to its
// event's next point overlaps its stores with that point's work: parts 1-3
// take 13.9 / 16.2 / 21.3 ms for 6001 events x 17 points in whole events
// against 23.0 / 18.5 / 23.1 in points, part 0, which loads no flows, 31.9
// against 23.8.  Whole events, then, for parts that load flows, unless points
// fill the chip so much better that they win in spite of that.
template <int C>
int split_units(int64_t nb, int npts) {
    const int64_t whole = npts * ((nb + kWaves1 - 1) / kWaves1), points = (nb * npts + kWaves1 - 1) / kWaves1;
    return C > 0 && 2 * whole <= 3 * points ? 1 : npts;
}

template <class Proc, typename T, int C>
hipError_t launch_part(const basis_record<Proc, T>* ev, int64_t e0, int64_t nb, T* jbuf, int64_t n, const qcd_launch& a,
                       double* out, double* me0, hipStream_t s) {
    const int units = split_units<C>(nb, a.npts), per = a.npts / units;
    const dim3 grid(unsigned((nb * units + kBlock / 64 - 1) / (kBlock / 64)));
    if constexpr (C + 1 == Proc::NCHUNK && mfma_colour<Proc>::value) {
        if (a.colour_mfma) {
            hipLaunchKernelGGL((qcd_part_kernel<Proc, T, C, true>), grid, dim3(kBlock), 0, s, ev, e0, nb, jbuf, n,
                               units, per, a, out, me0);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((qcd_part_kernel<Proc, T, C, false>), grid, dim3(kBlock), 0, s, ev, e0, nb, jbuf, n, units,
                       per, a, out, me0);
    return hipGetLastError();
}

// ---------------------------------------------- colour sum on the matrix cores
//
// After the last program part, J of every (event, point, helicity) is in HBM
// as X[c][n] (c = 2 flow + re/im, n = helicity; blocks of 64 helicities apart).  Per event and point the
// colour sum over all helicities is
//   sum_h J_h^+ CF J_h = sum_{f, n} X_f[n] (CF X)_f[n],
// with X_f the 2 NHEL real columns (real and imaginary parts) of flow f.
// D = CF X runs on v_mfma_f32_32x32x16_bf16: CF's integer numerators are the
// exact sum of two bfloat16 matrices (CF_BF16_HI + CF_BF16_LO, padded to KP),
// X is split into three bfloat16 terms x1 + x2 + x3 (24 significant bits), and
// the five products with weight above 2^-24 are accumulated in float32; the
// final dot product uses X itself (float32) from HBM.  One workgroup (4 waves)
// per event and point; each wave owns a quarter of D's columns.

typedef __attribute__((ext_vector_type(8))) __bf16 cbf16x8;
typedef __attribute__((ext_vector_type(8))) unsigned short cu16x8;
typedef __attribute__((ext_vector_type(16))) float cf32x16;

__device__ __forceinline__ unsigned short bf16_rne(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<unsigned short>(u >> 16);
}
__device__ __forceinline__ float bf16_float(unsigned short b) { return __uint_as_float(unsigned(b) << 16); }

template <class Proc>
__global__ void __launch_bounds__(kBlock)
qcd_colour_mfma_kernel(const float* __restrict__ jbuf, int64_t e0, int64_t nb, int64_t n, qcd_launch a,
                       double* __restrict__ out, double* __restrict__ me0) {
    constexpr int K = Proc::K, KP = Proc::KP, NH = Proc::NHEL, NCOL = 2 * NH;
    static_assert(KP % 32 == 0 && NCOL % 128 == 0, "tile shapes");
    constexpr int MT = KP / 32, KS = KP / 16, NT_WAVE = NCOL / 32 / (kBlock / 64);
    const int64_t el = blockIdx.x;
    if (el >= nb) return;   // whole block
    const int kp = blockIdx.y;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 31, lh = lane >> 5;
    __shared__ double part[kBlock / 64];
    {
        const float* X = jbuf + (el * a.npts + kp) * int64_t(2 * K) * NH;
        float s = 0.0f;
#pragma unroll 1
        for (int t = 0; t < NT_WAVE; ++t) {
            const int ncol = (wv * NT_WAVE + t) * 32 + lr;   // this lane's column of D
            const int re_im = ncol / NH, h = ncol % NH;
            const auto at = [&](int f) { return (h / 64 * 2 * K + 2 * f + re_im) * 64 + h % 64; };
            // B = X in three bfloat16 terms, all k-steps of this column tile
            cbf16x8 b1[KS], b2[KS], b3[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                cu16x8 u1, u2, u3;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int f = ks * 16 + lh * 8 + r;
                    const float x = f < K ? X[at(f)] : 0.0f;
                    const unsigned short x1 = bf16_rne(x);
                    const float r1 = x - bf16_float(x1);
                    const unsigned short x2 = bf16_rne(r1);
                    const unsigned short x3 = bf16_rne(r1 - bf16_float(x2));
                    u1[r] = x1;
                    u2[r] = x2;
                    u3[r] = x3;
                }
                b1[ks] = __builtin_bit_cast(cbf16x8, u1);
                b2[ks] = __builtin_bit_cast(cbf16x8, u2);
                b3[ks] = __builtin_bit_cast(cbf16x8, u3);
            }
#pragma unroll 1
            for (int mt = 0; mt < MT; ++mt) {
                cf32x16 acc = {};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    cu16x8 hi, lo;
                    const int row = mt * 32 + lr, k0 = ks * 16 + lh * 8;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        hi[r] = Proc::CF_BF16_HI[row * KP + k0 + r];
                        lo[r] = Proc::CF_BF16_LO[row * KP + k0 + r];
                    }
                    const cbf16x8 ah = __builtin_bit_cast(cbf16x8, hi), al = __builtin_bit_cast(cbf16x8, lo);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, b1[ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, b2[ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, b1[ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, b3[ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, b2[ks], acc, 0, 0, 0);
                }
                // D[m][ncol] for m = mt*32 + (r/4)*8 + lh*4 + r%4, dotted with X[m][ncol]
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int f = mt * 32 + (r / 4) * 8 + lh * 4 + r % 4;
                    if (f < K) s += X[at(f)] * acc[r];
                }
            }
        }
        double v = wave_sum(double(s));
        if (lane == 0) part[wv] = v;
        __syncthreads();
        double me = 0.0;
        for (int i = 0; i < kBlock / 64; ++i) me += part[i];
        me *= Proc::point_norm(a.pts[kp].gs);
        if (threadIdx.x == 0) store_me(me, kp, e0 + el, e0 + el, n, a, out, me0);
    }
}

template <class Proc>
hipError_t launch_colour_mfma(const float* jbuf, int64_t e0, int64_t nb, int64_t n, const qcd_launch& a, double* out,
                              double* me0, hipStream_t s) {
    if constexpr (mfma_colour<Proc>::value) {
        if (!a.colour_mfma) return hipSuccess;
        hipLaunchKernelGGL((qcd_colour_mfma_kernel<Proc>), dim3(unsigned(nb), unsigned(a.npts)), dim3(kBlock), 0, s,
                           jbuf, e0, nb, n, a, out, me0);
        return hipGetLastError();
    } else {
        return hipSuccess;
    }
}

// ------------------------------ double-precision instance of the split programs
//
// In double precision the 120 colour-flow amplitudes of g g -> t tbar g g g
// alone would take 480 registers per lane.  The generated program is
// therefore also cut by colour flow: amplitude_fr<C, R> holds the diagrams of
// chunk C of the closing groups that contribute to flow range R (KR flows),
// so only KR amplitudes are live at a time; diagrams with terms in several
// ranges are evaluated once per range.  Kernel (C, R) runs it for a batch of
// events, one event per wave with the helicity configurations on the lanes,
// and passes the range's amplitudes through HBM ([event][point][component]
// [helicity], as the single-precision parts do); qcd_colour64_kernel then
// forms the colour sum from HBM and the helicity sum, which is |M|^2.
//
// The same pipeline re-evaluates the ill-conditioned events of the
// single-precision pass: slots are then positions in the list of those
// events (count on the device), and slots beyond the count exit at once.

// Per-event data of one slot: event e itself, or list[slot].
template <class Proc>
__global__ void __launch_bounds__(kBlock)
qcd_setup64_kernel(const double* __restrict__ mom, int64_t n, double mt, const int64_t* __restrict__ list,
                   const unsigned long long* __restrict__ count, int64_t slots,
                   table_record<Proc, double>* __restrict__ ev) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= slots || (count && i >= int64_t(count[0]))) return;
    const int64_t e = list ? list[i] : i;
    double p[Proc::NEXT][4];
    load_event<Proc::NEXT>(mom, n, e, p);
    ev[i].fill(p, mt);
    ev[i].skip = 0;
}

// M points a pass, as in qcd_wave_kernel, from the record staged in LDS; one
// wave's unit of work is one pass of one slot.  Bound by FP64 issue at one wave
// per SIMD and 512 registers; a diagram with terms in several ranges is
// evaluated in each, so sharing the chains between points pays the more.
// 700 events x 17 points: 42.6 ms with one point a pass, whole events per wave
// and the record read through the scalar cache (874 scalar registers spilled
// to vector lanes), 25.2 ms so.
template <class Proc, int M>
struct fr_plan {
    // accumulators in LDS: what a quarter of the CU's 160 KiB leaves beside the record
    static constexpr size_t record = sizeof(typename Proc::template kin<double>) +
                                     sizeof(typename Proc::template ext_table<double>) + 64;
    static constexpr int room = int((40 * 1024 - record) / 1024);
    static constexpr int NL = M == 1 ? 0 : room;
};
template <class Proc, int M>
struct fr_slot {
    alignas(16) near_kin<typename Proc::template kin<double>> k;
    alignas(16) typename Proc::template ext_table<double> t;
    alignas(16) cx<double> j[64 * fr_plan<Proc, M>::NL + 1];
};
// The flows of M points, `point` values apart.
template <int K, int M, int NL, int... m>
__device__ __forceinline__ void load_points(point_cells<K, M, NL>& J, const double* p, int64_t point, int stride,
                                            std::integer_sequence<int, m...>) {
    (J.template load<m>(p + m * point, stride, points_seq<K>{}), ...);
}
template <int K, int M, int NL, int... m>
__device__ __forceinline__ void store_points(const point_cells<K, M, NL>& J, double* p, int64_t point, int stride,
                                             std::integer_sequence<int, m...>) {
    (J.template store<m>(p + m * point, stride, points_seq<K>{}), ...);
}
// Points of the buffer per slot: whole passes, so that no load or store of a
// pass depends on a point's existence (stores behind a condition put the
// flows across a block boundary, and the register allocator spills ten times
// as much).
__host__ __device__ inline int split64_points(int npts) {
    return npts > 1 ? (npts + kPointsSplit64 - 1) / kPointsSplit64 * kPointsSplit64 : 1;
}
template <class Proc, int C, int R, int M>
__global__ void __launch_bounds__(kBlock, 1)
qcd_fr_kernel(const table_record<Proc, double>* __restrict__ ev, const unsigned long long* __restrict__ count,
              int64_t e0, int64_t nb, double* __restrict__ jbuf, qcd_launch a) {
    constexpr int NH = Proc::NHEL, K2 = 2 * Proc::K, KR = Proc::KR;
    static_assert(NH % 64 == 0, "helicity configurations must fill whole waves");
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t id = int64_t(blockIdx.x) * (kBlock / 64) + wv;
    const int passes = (a.npts + M - 1) / M;
    const int64_t el = id / passes;
    if (el >= nb) return;   // whole wave; no barriers below
    const int64_t i = e0 + el;
    if (count && i >= int64_t(count[0])) return;
    const int lane = threadIdx.x & 63;
    __shared__ fr_slot<Proc, M> sl[kBlock / 64];
    fr_slot<Proc, M>& s = sl[wv];
    stage_record(ev[i], s, lane);
    const int kp = int(id - el * passes) * M;
    const auto c = couplings_of<Proc, double, M>(a.pts, kp, a.npts);
#pragma unroll 1
    for (int hc = 0; hc < NH; hc += 64) {
        __asm__ volatile("" ::: "memory");
        const near_ext<typename Proc::template ext_ref<double>> w = {Proc::template ext_at<double>(s.t, hc + lane)};
        point_cells<KR, M, fr_plan<Proc, M>::NL> J{&s.j[lane], {}};
        double* jp = jbuf + (el * (passes * M) + kp) * int64_t(K2) * NH + hc * K2 + 2 * R * KR * 64 + lane;
        if constexpr (C == 0)
            J.clear();
        else
            load_points(J, jp, int64_t(K2) * NH, 64, points_seq<M>{});
        Proc::template amplitude_fr<C, R, double>(w, s.k, c, J);
        store_points(J, jp, int64_t(K2) * NH, 64, points_seq<M>{});
    }
}

// Flows per block of the streamed colour sum (z = CF J for BS rows at a time).
constexpr int kColourBlock = 40;

// sum_h J_h^+ CF J_h from the amplitudes in HBM: per lane (helicity) and block
// of kColourBlock rows, z_i = sum_t CF[t][i] J_t with J_t streamed from memory
// (CF symmetric, row t of the table contiguous in i, read through the scalar
// cache), then the block's Re(J_i^* z_i); helicity sum by wave reduction.
template <class Proc>
__global__ void __launch_bounds__(kBlock)
qcd_colour64_kernel(const double* __restrict__ jbuf, const int64_t* __restrict__ list,
                    const unsigned long long* __restrict__ count, int64_t e0, int64_t nb, int64_t n, qcd_launch a,
                    double* __restrict__ out, double* __restrict__ me0) {
    constexpr int K = Proc::K, NH = Proc::NHEL, BS = kColourBlock;
    static_assert(K % BS == 0, "colour blocks");
    const int64_t unit = int64_t(blockIdx.x) * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t el = unit / a.npts;   // a unit: one point of one slot
    if (el >= nb) return;   // whole wave
    if (count && e0 + el >= int64_t(count[0])) return;
    const int64_t e = list ? list[e0 + el] : e0 + el;
    const int lane = threadIdx.x & 63;
    const int kp = int(unit - el * a.npts);
    double acc = 0.0;
#pragma unroll 1
    for (int hc = 0; hc < NH; hc += 64) {
        const double* X = jbuf + (el * split64_points(a.npts) + kp) * int64_t(2 * K) * NH + hc * 2 * K + lane;
#pragma unroll 1
        for (int a0 = 0; a0 < K; a0 += BS) {
            double zr[BS], zi[BS];
#pragma unroll
            for (int q = 0; q < BS; ++q) zr[q] = zi[q] = 0.0;
#pragma unroll 2
            for (int t = 0; t < K; ++t) {
                const double jr = X[(2 * t) * 64], ji = X[(2 * t + 1) * 64];
                const double* cf = Proc::CF_DBL + t * K + a0;
#pragma unroll
                for (int q = 0; q < BS; ++q) {
                    zr[q] = fma(cf[q], jr, zr[q]);
                    zi[q] = fma(cf[q], ji, zi[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < BS; ++q)
                acc += zr[q] * X[(2 * (a0 + q)) * 64] + zi[q] * X[(2 * (a0 + q) + 1) * 64];
        }
    }
    const double me = wave_sum(acc) * Proc::point_norm(a.pts[kp].gs);
    if (lane == 0) store_me(me, kp, e, e, n, a, out, me0);
}

template <class Proc, int C, int R>
hipError_t launch_fr(const table_record<Proc, double>* ev, const unsigned long long* count, int64_t e0, int64_t nb,
                     double* jbuf, const qcd_launch& a, hipStream_t s) {
    const int64_t passes = a.npts > 1 ? (a.npts + kPointsSplit64 - 1) / kPointsSplit64 : 1;
    const dim3 grid(unsigned((nb * passes + kBlock / 64 - 1) / (kBlock / 64)));
    if (a.npts > 1)
        hipLaunchKernelGGL((qcd_fr_kernel<Proc, C, R, kPointsSplit64>), grid, dim3(kBlock), 0, s, ev, count, e0, nb,
                           jbuf, a);
    else
        hipLaunchKernelGGL((qcd_fr_kernel<Proc, C, R, 1>), grid, dim3(kBlock), 0, s, ev, count, e0, nb, jbuf, a);
    return hipGetLastError();
}

// Kernel launchers of a split program, one translation unit each.
template <class Proc>
struct split_launchers {
    using part_fn = hipError_t (*)(const basis_record<Proc, float>*, int64_t, int64_t, float*, int64_t,
                                   const qcd_launch&, double*, double*, hipStream_t);
    using fr_fn = hipError_t (*)(const table_record<Proc, double>*, const unsigned long long*, int64_t, int64_t,
                                 double*, const qcd_launch&, hipStream_t);
    part_fn part[Proc::NCHUNK];
    fr_fn fr[Proc::NCHUNK64 * Proc::NFR];
};

// Events per batch of the split programs: the buffer that carries J between
// the parts holds batch x points x 2K x NHEL values of T, about 4.5 GiB at
// most, and a batch of more than one round of waves is a whole number of them
// (17 points: 2048 events in single and 1024 in double precision).
constexpr int64_t kPartBatch = 8192;
constexpr size_t kJBufBytes = size_t(9) << 29;
template <class Proc, typename T>
int64_t part_batch(int64_t n, int npts) {
    const size_t per_event = size_t(npts) * 2 * Proc::K * Proc::NHEL * sizeof(T);
    int64_t b = int64_t(kJBufBytes / per_event);
    b = b > kPartBatch ? kPartBatch : (b < 64 ? 64 : b);
    if (b > kWaves1) b -= b % kWaves1;
    return n < b ? n : b;
}

// Double-precision pipeline over `slots` slots: per-slot data, then batches
// through the (chunk, range) kernels and the colour sum.  list == NULL: slot
// i is event i; otherwise slot i is event list[i] for i < count[0].
template <class Proc>
hipError_t launch_split64(const split_launchers<Proc>& L, const double* mom, int64_t n, const int64_t* list,
                          const unsigned long long* count, int64_t slots, const qcd_launch& a, double* out,
                          double* me0, hipStream_t s, bool timed) {
    using ED = table_record<Proc, double>;
    const int jpts = split64_points(a.npts);
    const int64_t B = part_batch<Proc, double>(slots, jpts);
    ED* ev = nullptr;
    double* jbuf = nullptr;
    hipError_t err = work_alloc(reinterpret_cast<void**>(&ev), sizeof(ED) * size_t(slots), s);
    if (err != hipSuccess) return err;
    err = work_alloc(reinterpret_cast<void**>(&jbuf),
                         sizeof(double) * size_t(B) * jpts * 2 * Proc::K * Proc::NHEL, s);
    if (err != hipSuccess) {
        (void)hipFreeAsync(ev, s);
        return err;
    }
    hipLaunchKernelGGL((qcd_setup64_kernel<Proc>), dim3(unsigned((slots + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       mom, n, a.mt, list, count, slots, ev);
    err = hipGetLastError();
    if (timed) mark(a.t0, s);
    // One (chunk, range) kernel at one wave per SIMD leaves SIMDs idle: with
    // few events per batch (re-evaluating listed events) most of them, and in
    // the last round of waves of a full batch nearly all.  The ranges of a
    // chunk write disjoint parts of jbuf, so they run side by side, range 0
    // on the caller's stream and the others on library streams, joined per
    // chunk.
    constexpr int NFR = Proc::NFR;
    const bool side = NFR - 1 <= kAuxStreams;
    hipStream_t aux[kAuxStreams] = {};
    hipEvent_t fork = nullptr, join[kAuxStreams] = {};
    if (err == hipSuccess && side) {
        err = aux_streams(aux);
        if (err == hipSuccess) err = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
        for (int r = 1; r < NFR && err == hipSuccess; ++r) err = hipEventCreateWithFlags(&join[r - 1], hipEventDisableTiming);
    }
    for (int64_t e0 = 0; e0 < slots && err == hipSuccess; e0 += B) {
        const int64_t nb = slots - e0 < B ? slots - e0 : B;
        for (int c = 0; c < Proc::NCHUNK64 && err == hipSuccess; ++c) {
            if (!side) {
                for (int r = 0; r < NFR && err == hipSuccess; ++r) err = L.fr[c * NFR + r](ev, count, e0, nb, jbuf, a, s);
                continue;
            }
            err = hipEventRecord(fork, s);
            for (int r = 1; r < NFR && err == hipSuccess; ++r) err = hipStreamWaitEvent(aux[r - 1], fork, 0);
            if (err == hipSuccess) err = L.fr[c * NFR](ev, count, e0, nb, jbuf, a, s);
            bool used[kAuxStreams] = {};
            for (int r = 1; r < NFR && err == hipSuccess; ++r) {
                used[r - 1] = true;   // a failed launch may still have queued work
                err = L.fr[c * NFR + r](ev, count, e0, nb, jbuf, a, aux[r - 1]);
            }
            // join every library stream that received work, also after an
            // error, before the buffers are released on the caller's stream
            for (int r = 1; r < NFR; ++r) {
                if (!used[r - 1]) continue;
                hipError_t j = hipEventRecord(join[r - 1], aux[r - 1]);
                if (j == hipSuccess) j = hipStreamWaitEvent(s, join[r - 1], 0);
                if (j != hipSuccess) (void)hipStreamSynchronize(aux[r - 1]);
                if (err == hipSuccess) err = j;
            }
        }
        if (err == hipSuccess) {
            hipLaunchKernelGGL((qcd_colour64_kernel<Proc>),
                               dim3(unsigned((nb * a.npts + kBlock / 64 - 1) / (kBlock / 64))), dim3(kBlock), 0, s,
                               jbuf, list, count, e0, nb, n, a, out, me0);
            err = hipGetLastError();
        }
    }
    if (timed) mark(a.t1, s);
    // the events are released once their pending work has completed
    if (fork) (void)hipEventDestroy(fork);
    for (int r = 0; r < kAuxStreams; ++r)
        if (join[r]) (void)hipEventDestroy(join[r]);
    hipError_t f1 = hipFreeAsync(jbuf, s), f2 = hipFreeAsync(ev, s);
    return err != hipSuccess ? err : (f1 != hipSuccess ? f1 : f2);
}

// |M|^2 of a split program to out and me0 (per event).  FP64 runs the
// double-precision pipeline over all events; mixed precision runs the
// per-event data (listing ill-conditioned events when the re-evaluation is
// on), batches through the single-precision parts (and the matrix-core colour
// sum when selected), then the listed events through the double-precision
// pipeline.
template <class Proc>
hipError_t launch_split_me(const split_launchers<Proc>& L, int fp64, const double* mom, int64_t n, const qcd_launch& a,
                           double* out, double* me0, hipStream_t s) {
    if (fp64) return launch_split64<Proc>(L, mom, n, nullptr, nullptr, n, a, out, me0, s, true);
    using ED = basis_record<Proc, float>;
    const bool rescue = a.rescue_tau > 0.0;
    const int64_t B = part_batch<Proc, float>(n, a.npts);
    ED* ev = nullptr;
    float* jbuf = nullptr;
    int64_t* buf = nullptr;
    hipError_t err = work_alloc(reinterpret_cast<void**>(&ev), sizeof(ED) * size_t(n), s);
    if (err != hipSuccess) return err;
    err = work_alloc(reinterpret_cast<void**>(&jbuf), sizeof(float) * size_t(B) * a.npts * 2 * Proc::K * Proc::NHEL,
                         s);
    if (err == hipSuccess && rescue)
        err = work_alloc(reinterpret_cast<void**>(&buf), sizeof(int64_t) * size_t(n + 1), s);
    if (err != hipSuccess) {
        if (jbuf) (void)hipFreeAsync(jbuf, s);
        (void)hipFreeAsync(ev, s);
        return err;
    }
    unsigned long long* count = rescue ? reinterpret_cast<unsigned long long*>(buf) : nullptr;
    int64_t* list = rescue ? buf + 1 : nullptr;
    if (rescue) hipLaunchKernelGGL((rescue_reset_kernel<Proc>), dim3(1), dim3(64), 0, s, count);
    hipLaunchKernelGGL((qcd_setup_kernel<Proc, ED>), dim3(unsigned((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       mom, n, int64_t(0), n, a.mt, ev, rescue ? a.rescue_tau : 0.0, count, list);
    err = hipGetLastError();
    mark(a.t0, s);
    for (int64_t e0 = 0; e0 < n && err == hipSuccess; e0 += B) {
        const int64_t nb = n - e0 < B ? n - e0 : B;
        for (int c = 0; c < Proc::NCHUNK && err == hipSuccess; ++c)
            err = L.part[c](ev, e0, nb, jbuf, n, a, out, me0, s);
        if (err == hipSuccess) err = launch_colour_mfma<Proc>(jbuf, e0, nb, n, a, out, me0, s);
    }
    mark(a.t1, s);
    hipError_t f1 = hipFreeAsync(jbuf, s), f2 = hipFreeAsync(ev, s);
    if (err == hipSuccess && rescue) err = launch_split64<Proc>(L, mom, n, list, count, n, a, out, me0, s, false);
    hipError_t f3 = rescue ? hipFreeAsync(buf, s) : hipSuccess;
    return err != hipSuccess ? err : (f1 != hipSuccess ? f1 : (f2 != hipSuccess ? f2 : f3));
}

// A split program: |M|^2 of every event and point, then the weights.
template <class Proc>
hipError_t launch_split(const split_launchers<Proc>& L, int fp64, const double* mom, const double* w_in, int64_t n,
                        const qcd_launch& a, double* out, double* me0, hipStream_t s) {
    if (a.scratch.ptr) return hipErrorNotSupported;   // J buffers of MBs per event: always allocated
    const bool weights = a.mode == 0;
    const bool base = weights && !me0;
    const bool aside = weights && (overlap(w_in, n, out, (a.npts - 1) * n) || overlap(w_in, n, me0, n));
    double* buf = nullptr;
    if (base || aside) {
        hipError_t err = work_alloc(reinterpret_cast<void**>(&buf), 16 * size_t(n), s);
        if (err != hipSuccess) return err;
    }
    const unsigned blocks = unsigned((n + kBlock - 1) / kBlock);
    const double* w = w_in;
    if (aside) {
        hipLaunchKernelGGL((copy_weights_kernel<kBlock>), dim3(blocks), dim3(kBlock), 0, s, w_in, n, buf + n);
        w = buf + n;
    }
    double* m0 = base ? buf : me0;
    hipError_t err = launch_split_me<Proc>(L, fp64, mom, n, a, out, m0, s);
    if (err == hipSuccess && weights && a.npts > 1) {
        hipLaunchKernelGGL((reweight_ratio_kernel<kBlock>), dim3(blocks, unsigned(a.npts - 1)), dim3(kBlock), 0, s, w,
                           m0, int64_t(0), n, n, out);
        err = hipGetLastError();
    }
    const hipError_t ferr = buf ? hipFreeAsync(buf, s) : hipSuccess;
    return err != hipSuccess ? err : ferr;
}

// Events of a workgroup of qcd_sub_kernel: 32, so that few lanes wait for the
// kinematics, where that still fills the 768 workgroups that run at once
// several times; below, what the workgroup's lanes hold at once.  Few points
// leave the kinematics more weight: g g -> t tbar g, mixed, 65536 events at one
// point 85 us against 126, at six 418 against 459; at 17, 75000 events, 1419
// against 1339, equal from 200000 on.
constexpr int kSubTile = 32;
constexpr bool sub_tiles(int64_t n, int npts) { return n >= (npts <= 8 ? 65536 : 196608); }
// Whether a batch of a process with fewer than 64 configurations runs one event
// per lane: from both kernels' times, in us and fitted to 0.9-1.1 of what they
// measure at 30000 to 1.5 10^6 events and 1 to 65 points.  A lane's time goes
// in steps, as its kernel adds a wave to every SIMD (g g -> t tbar g in single
// precision: fills the CUs' LDS, seven waves each): first + step points for
// every `events` of the batch, the first of them at least `least` steps.  Several events per
// wave take sub0 + sub1 points ns per event.  For example, times in us of one
// event per lane and of several per wave (both with this rule's tiles):
//   g g -> t tbar, mixed   1 point  95000 events  23.4  22.4   115000  23.3  26.8
//                         17 points 115000 events 303   276    300000  692   675
//   g g -> t tbar, FP64    1 point  55000 events  19.1  27.4   140000  43.4  52.6
//                         17 points 65000 events  247   274    105000  450   441
//   g g -> t tbar g, FP64  1 point  65536 events  140   165    75000   274   205
//                         17 points 65536 events  2274  2408   150000  6992  5536
// and g g -> t tbar g in single precision one per lane only for large batches
// at one point (1.5 10^6 events: 1787 against 1865).
struct lane_cost {
    int64_t events;
    double least, first, step;
    double sub0, sub1, tile0, tile1;   // per workgroup's lanes, and with tiles
};
template <class Proc>
bool lanes_faster(int fp64, int64_t batch, int npts) {
    constexpr lane_cost tt[2] = {{65536, 1.85, 5, 8.50, 0.115, 0.132, 0.050, 0.137},
                                 {65536, 1.08, 5, 13.0, 0.200, 0.235, 0.106, 0.238}};
    constexpr lane_cost ttg[2] = {{114688, 1, 8, 129, 0.88, 1.015, 0.20, 1.03},
                                  {65536, 1, 6, 134, 1.455, 2.083, 0.30, 2.133}};
    static_assert(Proc::NG == 2 || Proc::NG == 3, "measured for g g -> t tbar and g g -> t tbar g");
    const lane_cost& c = Proc::NG == 2 ? tt[fp64 != 0] : ttg[fp64 != 0];
    const double steps = double((batch + c.events - 1) / c.events);
    const double lanes = c.first + c.step * npts * (steps > c.least ? steps : c.least);
    const double per_event = sub_tiles(batch, npts) ? c.tile0 + c.tile1 * npts : c.sub0 + c.sub1 * npts;
    return lanes <= 5.0 + 1e-3 * double(batch) * per_event;
}
// A launch holds kLaunchBlocks E events: 2^29 of g g -> t tbar g.
template <class Proc, int E>
void launch_sub(int fp64, const double* mom, const double* w_in, int64_t nb, int64_t n, const qcd_launch& a,
                double* out, double* me0, hipStream_t s) {
    const auto kernel = fp64 ? qcd_sub_kernel<Proc, double, E> : qcd_sub_kernel<Proc, float, E>;
    for (int64_t e0 = 0; e0 < nb; e0 += kLaunchBlocks * E) {
        const int64_t m = nb - e0 < kLaunchBlocks * E ? nb - e0 : kLaunchBlocks * E;
        hipLaunchKernelGGL(kernel, dim3(unsigned((m + E - 1) / E)), dim3(kBlock), 0, s, mom + e0,
                           w_in ? w_in + e0 : nullptr, m, n, int(Proc::NHEL), a, out + e0, me0 ? me0 + e0 : nullptr);
    }
}

// Events 0 .. nb - 1 from the pointers on, whose rows are n apart: one per lane
// or several per wave.
template <class Proc>
hipError_t launch_lane_kernels(int fp64, const double* mom, const double* w_in, int64_t nb, int64_t n,
                               const qcd_launch& a, double* out, double* me0, hipStream_t s) {
    const dim3 grid(unsigned((nb + kBlock - 1) / kBlock));
    if (a.kpoly) {
        if constexpr (Proc::NHEL % 64 != 0)
            hipLaunchKernelGGL((fp64 ? qcd_kpoly_lane_kernel<Proc, double> : qcd_kpoly_lane_kernel<Proc, float>), grid,
                               dim3(kBlock), 0, s, mom, w_in, nb, n, a, out, me0);
        return hipGetLastError();
    }
    if constexpr (Proc::NHEL < 64) {
        if (a.mapping == MGRW_MAP_AUTO && !lanes_faster<Proc>(fp64, a.batch, a.npts)) {
            constexpr int G = kBlock / Proc::NHEL;   // events a workgroup's lanes hold at once
            if (sub_tiles(nb, a.npts))   // the same weights, whichever
                launch_sub<Proc, kSubTile>(fp64, mom, w_in, nb, n, a, out, me0, s);
            else
                launch_sub<Proc, G>(fp64, mom, w_in, nb, n, a, out, me0, s);
            return hipGetLastError();
        }
    }
    constexpr int NBD = lane_block<Proc, double>(), NBF = lane_block<Proc, float>();
    if (fp64)
        hipLaunchKernelGGL((qcd_kernel<Proc, double>), dim3(unsigned((nb + NBD - 1) / NBD)), dim3(NBD), 0, s, mom,
                           w_in, n, a, out, me0, nb);
    else
        hipLaunchKernelGGL((qcd_kernel<Proc, float>), dim3(unsigned((nb + NBF - 1) / NBF)), dim3(NBF), 0, s, mom,
                           w_in, n, a, out, me0, nb);
    return hipGetLastError();
}

// The kernels that write weights directly, then the FP64 re-evaluation of the
// ill-conditioned events, which reads the input weights a second time: where
// the outputs overlap them they are set aside first.  Buffers: count, list,
// weights.  With a scratch span the events run in chunks whose buffers fit.
template <class Proc>
hipError_t launch_lanes(int fp64, const double* mom, const double* w_in, int64_t n, const qcd_launch& a, double* out,
                        double* me0, hipStream_t s) {
    const bool rescue = !fp64 && a.rescue_tau > 0.0 && Proc::NEXT > 4;   // there is a final-state gluon
    const bool aside =
        rescue && a.mode == 0 && (overlap(w_in, n, out, (a.npts - 1) * n) || overlap(w_in, n, me0, n));
    const size_t words = aside ? 2 : 1;
    int64_t chunk = n;
    char* mem = nullptr;
    if (rescue && a.scratch.ptr) {
        mem = static_cast<char*>(a.scratch.ptr);
        chunk = scratch_chunk(a.scratch, words * 8, 768);
        if (chunk < 1) return hipErrorInvalidValue;
        if (chunk > n) chunk = n;
    } else if (rescue) {
        hipError_t err = work_alloc(reinterpret_cast<void**>(&mem), 256 + words * align256(8 * size_t(n)), s);
        if (err != hipSuccess) return err;
    }
    unsigned long long* count = reinterpret_cast<unsigned long long*>(mem);
    int64_t* list = rescue ? reinterpret_cast<int64_t*>(mem + 256) : nullptr;
    double* w_buf = aside ? reinterpret_cast<double*>(mem + 256 + align256(8 * size_t(chunk))) : nullptr;
    hipError_t err = hipSuccess;
    for (int64_t e0 = 0; e0 < n && err == hipSuccess; e0 += chunk) {
        const int64_t nb = n - e0 < chunk ? n - e0 : chunk;
        const unsigned blocks = unsigned((nb + kBlock - 1) / kBlock);
        const double *p = mom + e0, *w = w_in ? w_in + e0 : nullptr;
        double *o = out + e0, *m0 = me0 ? me0 + e0 : nullptr;
        if (aside) {
            hipLaunchKernelGGL((copy_weights_kernel<kBlock>), dim3(blocks), dim3(kBlock), 0, s, w, nb, w_buf);
            w = w_buf;
        }
        mark(a.t0, s);
        err = launch_lane_kernels<Proc>(fp64, p, w, nb, n, a, o, m0, s);
        mark(a.t1, s);
        if constexpr (Proc::NEXT > 4) {
            if (!rescue || err != hipSuccess) continue;
            hipLaunchKernelGGL((rescue_reset_kernel<Proc>), dim3(1), dim3(64), 0, s, count);
            hipLaunchKernelGGL((rescue_flag_kernel<Proc>), dim3(blocks), dim3(kBlock), 0, s, p, n, nb, a.rescue_tau,
                               count, list);
            if (a.kpoly)
                hipLaunchKernelGGL((qcd_rescue_kpoly_kernel<Proc>), dim3(kRescueBlocks), dim3(kBlock), 0, s, p, list,
                                   count, w, n, a, o, m0);
            else
                hipLaunchKernelGGL((qcd_rescue_kernel<Proc>), dim3(kRescueBlocks), dim3(kBlock), 0, s, p, list, count,
                                   w, n, int(Proc::NHEL), a, o, m0);
            err = hipGetLastError();
        }
    }
    if (!mem || a.scratch.ptr) return err;
    hipError_t ferr = hipFreeAsync(mem, s);
    return err != hipSuccess ? err : ferr;
}

template <class Proc>
hipError_t launch_qcd(int fp64, const double* mom, const double* w_in, int64_t n, const qcd_launch& a,
                      double* out, double* me0, hipStream_t s) {
    if constexpr (Proc::NHEL % 64 == 0) {
        if (a.kpoly)
            return fp64 ? launch_wave_pipeline<Proc, double, true>(mom, w_in, n, a, out, me0, s)
                        : launch_wave_pipeline<Proc, float, true>(mom, w_in, n, a, out, me0, s);
        if (a.mapping == MGRW_MAP_EVENT_PER_WAVE)
            return fp64 ? launch_wave_pipeline<Proc, double, false>(mom, w_in, n, a, out, me0, s)
                        : launch_wave_pipeline<Proc, float, false>(mom, w_in, n, a, out, me0, s);
    } else if (!a.kpoly && a.mapping == MGRW_MAP_EVENT_PER_WAVE) {
        return hipErrorInvalidConfiguration;
    }
    return launch_lanes<Proc>(fp64, mom, w_in, n, a, out, me0, s);
}

}  // namespace mgrw
