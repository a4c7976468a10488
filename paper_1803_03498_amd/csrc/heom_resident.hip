// Resident propagation of small hierarchies: every RK4 step of a run in one
// launch (full density matrices, FP64 or FP32-mixed storage).
//
// A stage of a small hierarchy costs a launch (about 11 us with a replayed
// step graph on 3060 ADOs of 7 x 7, of which the arithmetic is a fraction):
// tables, H and the own elements are fetched again by every launch, and four
// launches follow each other in every step.  Here a workgroup keeps its ADOs
// for the whole run: the elements of the current stage in LDS, y and the
// partial stage combination in registers, H and the link tables in LDS.
// What travels between workgroups is the stage output, through two global
// arrays used in turn, and a grid-wide barrier ends each stage.
//
// Two forms:
//   one workgroup (GRID = false): the hierarchy lives in LDS, the barrier is
//     the workgroup's own.  Dimer (10 ADOs), FP64: 44 -> 4 us per step.
//   a grid (GRID = true): at most 256 workgroups of 256 to 768 threads, group
//     0 for sigma_0 and the observables, the others for the ADOs u >= 1, dealt
//     out one by one (u = 1 + w + g G) so that the ADOs below the top level,
//     which carry the "+" links, spread evenly.
//
// Exchange without cache maintenance.  The eight XCDs have an L2 each, and
// device-scope fences write back and invalidate it: 17 us per barrier of 256
// workgroups.  Instead every exchanged element is stored and loaded at device
// scope, past the L2s; a workgroup waits for its stores, raises its own flag,
// and polls the flags of all the others, one per thread (2.4 us per barrier
// of 256 workgroups with the exchange, against 4.7 us with one shared
// counter).  Nothing exchanged is ever read by a plain load in the same
// launch.  Such loads are slow and a CU has few in flight, so each neighbour
// row is loaded once, by consecutive threads, into LDS, and the elements take
// their coupling terms from there (loading them element by element, each row
// twice: 5.3 against 3.9 us per stage on 3060 ADOs of 7 x 7 in FP32).
//
// Progress.  A launch has at most 256 workgroups, each within half a CU: 80 KiB
// of LDS (the static word included), and 768 threads of 80 registers (six waves
// per SIMD) or 512 of 128 (four).  So two launches of either shape fit the 256
// CUs together, and the host lets at most two run at once (ResidentPermit): every
// workgroup becomes resident.  Should one still be kept out (other processes on the
// GPU), each wait ends after `wait_ticks`, and the workgroups agree through
// one word, by compare and swap, whether the launch commits or aborts.  The
// caller's state is written only after a commit, so the host can run an
// aborted launch's steps by the stage kernels instead.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "heom_device.h"
#include "heom_internal.h"

namespace heom {
namespace {

constexpr int kGridMax = 256;  // workgroups of a launch, sigma_0's included
// dynamic LDS; the kernels' static word takes 16 bytes with its alignment (10
// states of one mode at depth 135 would ask for the full 80 KiB)
constexpr size_t kStaticLds = 16, kGridLds = 80 * 1024 - kStaticLds, kOneLds = 150 * 1024;

// LDS carve-up (bytes): bulk part, and sigma_0 part from its own base.  The
// coupling lines of an element are a list of (element, complex weight)
// entries built once per launch: `links` bounds the entries of a workgroup.
struct ResidentLds {
    size_t h, s, rows, src, id, wt, off, gam, delta, count, bulk;
    size_t h0, s0, rows0, src0, id0, wt0, off0, gam0, delta0, count0, s0part;
};

__host__ __device__ inline int resident_links(int N, int W, int D, int slots, int low) {
    return slots * (D > 0 ? D : 1) * (2 * N - 1) + low * W * (2 * N - 2);
}

// grid: neighbour rows (and columns, for general states) staged in LDS.
__host__ __device__ inline ResidentLds resident_lds(int N, int W, int D, int slots, int low,
                                                    int tsize, bool hc, bool grid, bool herm) {
    const size_t NN = (size_t)N * N, S = slots;
    const size_t per_row = grid ? (size_t)N * (herm ? 1 : 2) : 0;
    const size_t nr = (size_t)slots * (D > 0 ? D : 1) + (size_t)low * W;
    const size_t links = resident_links(N, W, D, slots, low), links0 = (size_t)W * (2 * N - 2);
    ResidentLds L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align16(o + bytes);
        return at;
    };
    L.h = take(NN * (hc ? 2 : 1) * tsize);
    L.s = take(2 * S * NN * tsize);
    L.rows = take(2 * nr * per_row * tsize);
    L.src = take(nr * per_row * 4);
    L.id = take(grid ? nr * 4 : 0);
    L.wt = take(2 * links * tsize);
    L.off = take(links * 4);
    L.gam = take(S * tsize);
    L.delta = take((size_t)N * tsize);
    L.count = take(8);
    L.bulk = o;
    o = 0;
    L.h0 = take(NN * (hc ? 2 : 1) * 8);
    L.s0 = take(2 * NN * 8);
    L.rows0 = take(2 * W * per_row * 8);
    L.src0 = take(W * per_row * 4);
    L.id0 = take(grid ? (size_t)(W + 1) * 4 : 0);
    L.wt0 = take(2 * links0 * 8);
    L.off0 = take(links0 * 4);
    L.gam0 = take(8);
    L.delta0 = take((size_t)N * 8);
    L.count0 = take(8);
    L.s0part = o;
    return L;
}

// An exchanged array: raw buffer accesses that bypass the non-coherent
// caches (aux: the device-scope coherence bit), one per complex element.
constexpr int kDeviceScope = 16;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Exchanged {
    __amdgpu_buffer_rsrc_t r;
    __device__ Exchanged(const void* p, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000)) {}
    template <typename T>
    __device__ __forceinline__ cpx<T> load(uint32_t e) const {
        if constexpr (sizeof(T) == 4) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)(e * 8), 0, kDeviceScope);
            return {__uint_as_float(v.x), __uint_as_float(v.y)};
        } else {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(e * 16), 0, kDeviceScope);
            return {__hiloint2double((int)v.y, (int)v.x), __hiloint2double((int)v.w, (int)v.z)};
        }
    }
    template <typename T>
    __device__ __forceinline__ void store(uint32_t e, cpx<T> a) const {
        if constexpr (sizeof(T) == 4) {
            const u32x2 v = {__float_as_uint(a.re), __float_as_uint(a.im)};
            __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)(e * 8), 0, kDeviceScope);
        } else {
            const u32x4 v = {(uint32_t)__double2loint(a.re), (uint32_t)__double2hiint(a.re),
                             (uint32_t)__double2loint(a.im), (uint32_t)__double2hiint(a.im)};
            __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(e * 16), 0, kDeviceScope);
        }
    }
};

// Grid barrier of one stage.  arrive(): this workgroup's exchanged stores
// are complete and its flag carries `epoch`.  wait(): every workgroup's flag
// does, or the launch was given up (returns false, in all threads alike).
struct GridBarrier {
    const ResidentArgs& A;
    int* dead;  // LDS
    __device__ void arrive(uint32_t epoch) const {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(G(A.flags + kResidentFlagStride * blockIdx.x), epoch, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ uint32_t word() const {
        return __hip_atomic_load(G(A.commit), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // moves the word from "undecided" (A.chunk) to `to`; the decision that stands
    __device__ uint32_t decide(uint32_t to) const {
        uint32_t seen = A.chunk;
        return __hip_atomic_compare_exchange_strong(A.commit, &seen, to, __ATOMIC_RELAXED,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   ? to
                   : seen;
    }
    __device__ bool wait(uint32_t epoch) const {
        if ((int)threadIdx.x < A.members) {
            const gcptr<uint32_t> f = G((const uint32_t*)A.flags + kResidentFlagStride * threadIdx.x);
            const uint64_t t0 = wall_clock64();
            for (uint32_t n = 1;; ++n) {
                const uint32_t v = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((int32_t)(v - epoch) >= 0) break;
                if (n % 64 == 0 || A.wait_ticks == 0) {
                    const bool late = wall_clock64() - t0 >= A.wait_ticks;
                    const uint32_t w = late ? decide(kResidentAborted) : word();
                    if (w == kResidentAborted) *dead = 1;
                    if (w != A.chunk) break;
                }
            }
        }
        __syncthreads();
        return *dead == 0;
    }
};

// Observables of sigma_0 (LDS, interleaved complex128) by one wavefront;
// the same values as the stage kernels' record_sigma0.
__device__ void record_wave(const Job& J, const double* sS, int64_t slot) {
    if (slot < 0 || slot >= J.n_rec_max) return;
    const int N = J.t.N, NN = N * N, lane = threadIdx.x & 63;
    gptr<double> rec = G(J.records) + slot * J.rec_doubles;
    double trr = 0.0, tri = 0.0;
    for (int i = 0; i < N; ++i) {
        trr += sS[2 * (i * N + i)];
        tri += sS[2 * (i * N + i) + 1];
    }
    bool finite = isfinite(trr) && isfinite(tri);
    if (J.rec_kind == 0) {
        double h2 = 0.0;
        for (int e = lane; e < NN; e += 64) {
            const int i = e / N, j = e - i * N;
            const double dr = sS[2 * e] - sS[2 * (j * N + i)];
            const double di = sS[2 * e + 1] + sS[2 * (j * N + i) + 1];
            h2 = fmax(h2, dr * dr + di * di);
        }
        for (int m = 1; m < 64; m *= 2) h2 = fmax(h2, __shfl_xor(h2, m));
        const double herm = sqrt(h2);
        if (lane < N) rec[lane] = sS[2 * (lane * N + lane)];
        if (lane == 0) {
            rec[N] = trr;
            rec[N + 1] = tri;
            rec[N + 2] = herm;
        }
        finite = finite && isfinite(herm);
    } else {
        double pr = 0.0, pi = 0.0;
        for (int a = 0; a < N; ++a) {
            const double m = G(J.mu)[a];
            pr += m * sS[2 * (a * N + J.ground)];
            pi += m * sS[2 * (a * N + J.ground) + 1];
        }
        if (lane == 0) {
            rec[0] = pr;
            rec[1] = pi;
            rec[2] = trr;
            rec[3] = tri;
        }
        finite = finite && isfinite(pr) && isfinite(pi);
    }
    if (!finite && lane == 0) *G(J.status) = 1;
}

// (re, im) pair at LDS index e, one access.
template <typename T>
__device__ __forceinline__ cpx<T> sld(const T* p, int e) {
    const typename vec2<T>::type v = reinterpret_cast<const typename vec2<T>::type*>(p)[e];
    return {v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void sst(T* p, int e, cpx<T> a) {
    typename vec2<T>::type v;
    v.x = a.re;
    v.y = a.im;
    reinterpret_cast<typename vec2<T>::type*>(p)[e] = v;
}

// -i [H, sigma] at (i, j); sigma (S) and H in LDS.
template <typename T, bool HC>
__device__ __forceinline__ cpx<T> commutator(const T* sH, const T* S, int i, int j, int N) {
    T cr = 0, ci = 0;
#pragma unroll 2
    for (int k = 0; k < N; ++k) {
        const cpx<T> x = sld<T>(S, k * N + j), y = sld<T>(S, i * N + k);
        if constexpr (HC) {
            const cpx<T> h = sld<T>(sH, i * N + k), g = sld<T>(sH, k * N + j);
            cr += h.re * x.re - h.im * x.im - (y.re * g.re - y.im * g.im);
            ci += h.re * x.im + h.im * x.re - (y.re * g.im + y.im * g.re);
        } else {
            const T hik = sH[i * N + k], hkj = sH[k * N + j];
            cr += hik * x.re - y.re * hkj;
            ci += hik * x.im - y.im * hkj;
        }
    }
    return {ci, -cr};
}

// Flags of an entry of an element's coupling list, whose other bits are the
// index of the neighbour's element: among the staged rows (GRID), or in the
// LDS state; and of the source of a staged row element (index in the
// exchanged array).
constexpr uint32_t kConj = 0x80000000u;    // take the conjugate (column s of a Hermitian neighbour)
constexpr uint32_t kSigma0 = 0x40000000u;  // an element of sigma_0 (complex128)

// The LDS arrays of one role (bulk or sigma_0).
template <typename TE>
struct Role {
    TE *h, *s, *rows, *wt, *gam, *delta;  // H; stage input; neighbour rows; link weights; ...
    uint32_t *off, *src;                  // list entries; where each row element comes from
    int *id, *count;                      // row of each link; list and row counters
};

// One role's part of the run: EPT elements of type TE per thread, of the
// ADOs u >= 1 (S0 = false; storage type T = TE) or of sigma_0 (S0 = true, TE =
// double).  bulk_s and sigma0_s are the LDS elements of the two roles (the
// neighbours, with one workgroup).  Every __syncthreads is met by both roles.
template <typename TE, typename T, bool HC, bool GRID, bool S0, int EPT>
__device__ __forceinline__ void resident_role(const Job& J, const ResidentArgs& A, const GridBarrier& bar,
                                              const Role<TE>& R, const T* bulk_s, const double* sigma0_s,
                                              int rt, int n_rt) {
    const Tables& t = J.t;
    const int N = t.N, NN = N * N, W = t.W, D = t.D, Dm = D > 0 ? D : 1;
    const bool herm = J.herm != 0;
    const int Gr = GRID ? A.groups : 1, w = GRID ? (int)blockIdx.x - 1 : 0;
    // ADO slots of this workgroup
    const int ns = S0 ? 1 : max(0, (t.n_ado - 2 - w + Gr) / Gr);

    // ---- static tables and the initial state ----
    for (int e = rt; e < NN; e += n_rt) {
        TE re;
        if constexpr (sizeof(TE) == 4) re = G(t.h_re_f32)[e];
        else re = G(t.h_re)[e];
        R.h[HC ? 2 * e : e] = re;
        if constexpr (HC) R.h[2 * e + 1] = (TE)G(t.h_im)[e];
    }
    for (int g = rt; g < ns; g += n_rt) R.gam[g] = S0 ? (TE)0 : (TE)G(t.damping)[1 + w + g * Gr];
    for (int x = rt; x < N; x += n_rt) R.delta[x] = (TE)G(t.delta_state)[x];
    if (rt == 0) R.count[0] = R.count[1] = 0;
    __syncthreads();
    // the neighbour rows: one per link that exists, "-" links first
    const int n_minus = S0 ? 0 : ns * Dm, n_low = S0 ? (D > 0 ? 1 : 0) : min(A.low_slots, ns);
    const int per_row = herm ? N : 2 * N;
    if constexpr (GRID) {
        for (int x = rt; x < n_minus + n_low * W; x += n_rt) {
            int nb, s;
            if (x < n_minus) {
                const int g = x / Dm;
                const size_t at = (size_t)(1 + w + g * Gr) * Dm + (x - g * Dm);
                nb = G(reinterpret_cast<const pair_i*>(t.mlist))[at].x;
                s = nb >= 0 ? G(t.mlist_site)[at] : -1;
            } else {
                const int g = (x - n_minus) / W, l = x - n_minus - g * W;
                nb = G(t.plus)[(S0 ? 0 : (size_t)(1 + w + g * Gr)) * W + l];
                s = nb >= 0 ? G(t.mode_site)[l] : -1;
            }
            if (s < 0) continue;
            const int row = atomicAdd(R.count + 1, 1);
            R.id[x] = row;
            const uint32_t base = (uint32_t)(nb > 0 ? (nb - 1) * NN : 0);
            const uint32_t flag = nb == 0 ? kSigma0 : 0u;
            for (int cc = 0; cc < N; ++cc) {
                R.src[row * per_row + cc] = (base + s * N + cc) | flag;
                if (!herm) R.src[row * per_row + N + cc] = (base + cc * N + s) | flag;
            }
        }
        __syncthreads();
    }
    const int n_src = GRID ? R.count[1] * per_row : 0;
    cpx<TE> y[EPT], c[EPT];  // y and ((Y2 - y) + 2 (Y3 - y))/3 of the step
    // an element's place: slot << 10 | i << 5 | j (N <= 32), -1 without one;
    // its list: begin << 8 | entries; its index in the global arrays
    int place[EPT], list[EPT];
    uint32_t glob[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = rt + n_rt * q;
        y[q] = c[q] = {(TE)0, (TE)0};
        place[q] = -1;
        list[q] = 0;
        glob[q] = 0;
        if (e >= ns * NN) continue;
        const int g = e / NN, ij = e - g * NN, i = ij / N, j = ij - i * N;
        const size_t u = S0 ? 0 : 1 + w + (size_t)g * Gr;
        glob[q] = (uint32_t)(S0 ? ij : (u - 1) * NN + ij);
        y[q] = ld<TE>(S0 ? J.sig0[0] : J.rest[0], glob[q]);
        sst(R.s, e, y[q]);
        // the coupling list: counted, placed, written ("-" links in mode
        // order, then the "+" links of the modes of i and of j)
        const bool plus = i != j && G(t.level)[u] < D;
        const int bi = G(t.state_mode_begin)[i], ni = plus ? G(t.state_mode_begin)[i + 1] - bi : 0;
        const int bj = G(t.state_mode_begin)[j];
        const int np = plus ? ni + G(t.state_mode_begin)[j + 1] - bj : 0;
        int n = np;
        for (int a = 0; a < Dm; ++a) {
            const int s = G(t.mlist_site)[u * Dm + a];
            n += s >= 0 && (s == i || s == j);
        }
        int at = atomicAdd(R.count, n);
        place[q] = g << 10 | i << 5 | j;
        list[q] = at << 8 | n;
        // link x (of the row list), on state i, or on state j (col)
        auto put = [&](int x, int nb, bool col, TE wr, TE wi) {
            const bool cj = herm && col;
            uint32_t o;
            if constexpr (GRID)
                o = (uint32_t)(R.id[x] * per_row + (col ? (herm ? i : N + i) : j));
            else
                o = (uint32_t)(nb == 0 ? 0 : (nb - 1) * NN) + (uint32_t)(cj ? j * N + i : i * N + j) |
                    (nb == 0 ? kSigma0 : 0u);
            R.off[at] = o | (cj ? kConj : 0u);
            sst(R.wt, at++, cpx<TE>{wr, wi});
        };
        for (int a = 0; a < Dm; ++a) {
            const int s = G(t.mlist_site)[u * Dm + a];
            if (s < 0 || (s != i && s != j)) continue;
            TE wl, wc;
            if constexpr (sizeof(TE) == 4) {
                const pair_f v = G(reinterpret_cast<const pair_f*>(t.mlist_w32))[u * Dm + a];
                wl = v.x;
                wc = v.y;
            } else {
                const pair_d v = G(reinterpret_cast<const pair_d*>(t.mlist_w))[u * Dm + a];
                wl = v.x;
                wc = v.y;
            }
            const TE vx = (TE)((i == s) - (j == s)), vo = (TE)((i == s) + (j == s));
            put(g * Dm + a, G(reinterpret_cast<const pair_i*>(t.mlist))[u * Dm + a].x, s != i, wl * vo, wc * vx);
        }
        for (int m = 0; m < np; ++m) {
            const int l = G(t.state_modes)[m < ni ? bi + m : bj + m - ni];
            const TE p = (TE)G(t.plus_w)[u * W + l];
            put(n_minus + g * W + l, G(t.plus)[u * W + l], m >= ni, (TE)0, m < ni ? p : -p);
        }
    }
    __syncthreads();
    const bool rec_wave = S0 && rt < 64;
    if (rec_wave && A.step0 == 0) record_wave(J, sigma0_s, 0);

    const uint32_t x_bytes = (uint32_t)((size_t)(t.n_ado - 1) * NN * 2 * sizeof(T)), s0_bytes = NN * 16u;
    const double dt = J.dt;
    bool ok = true;
    uint32_t epoch = A.epoch0;
    int rec_left = S0 ? J.rec_every - (int)(A.step0 % J.rec_every) : 0;  // steps to the next record
    int64_t rec_slot = S0 ? A.step0 / J.rec_every : 0;
    for (int64_t step = 0; ok && step < A.n_steps; ++step) {
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            const bool first = step == 0 && k == 0, last = step + 1 == A.n_steps && k == 3;
            const double hd = dt * (k < 2 ? 0.5 : k == 2 ? 1.0 : 1.0 / 6.0);
            const TE h = (TE)hd, third = (TE)(1.0 / 3.0), two_thirds = (TE)(2.0 / 3.0);
            // neighbour rows into registers (the first RQ per thread), from
            // the array stage k - 1 wrote, the first stage from the caller's state
            constexpr int RQ = 2;
            const Exchanged xin(first ? J.rest[0] : A.exch[(k + 1) & 1], x_bytes);
            const Exchanged xs0(first ? J.sig0[0] : A.s0x[(k + 1) & 1], s0_bytes);
            auto fetch = [&](uint32_t o) -> cpx<TE> {
                if (!S0 && (o & kSigma0)) {
                    const cpx<double> v = xs0.template load<double>(o & ~kSigma0);
                    return {(TE)v.re, (TE)v.im};
                }
                const cpx<T> v = xin.template load<T>(o);
                return {(TE)v.re, (TE)v.im};
            };
            cpx<TE> rq[RQ];
            if constexpr (GRID) {
#pragma unroll
                for (int q = 0; q < RQ; ++q)
                    if (rt + n_rt * q < n_src) rq[q] = fetch(R.src[rt + n_rt * q]);
            }
            // places and lists pass through an empty asm: addresses derived
            // from them and hoisted out of the loop would hold registers
#pragma unroll
            for (int q = 0; q < EPT; ++q) asm volatile("" : "+v"(place[q]), "+v"(list[q]), "+v"(glob[q]));
            // the stage is y + h f, the last one (-y + Y2 + 2 Y3 + Y4)/3 + dt/6 f
            // = y + ((Y2 - y) + 2 (Y3 - y) + (Y4 - y))/3 + dt/6 f: increments
            // are summed first, so only the last addition rounds at the size
            // of y.  Here the commutator and damping of the increment.
            cpx<TE> out[EPT];
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                out[q] = {(TE)0, (TE)0};
                if (place[q] < 0) continue;
                const int g = place[q] >> 10, i = (place[q] >> 5) & 31, j = place[q] & 31;
                const TE* Sg = R.s + 2 * g * NN;
                cpx<TE> f = commutator<TE, HC>(R.h, Sg, i, j, N);
                const cpx<TE> s = sld<TE>(Sg, i * N + j);
                const TE gm = R.gam[g] + (i != j ? R.delta[i] + R.delta[j] : (TE)0);
                f.re -= gm * s.re;
                f.im -= gm * s.im;
                out[q] = {h * f.re, h * f.im};
                if (k == 3) {
                    out[q].re += c[q].re + third * (s.re - y[q].re);
                    out[q].im += c[q].im + third * (s.im - y[q].im);
                }
            }
            if constexpr (GRID) {
#pragma unroll
                for (int q = 0; q < RQ; ++q)
                    if (rt + n_rt * q < n_src) sst(R.rows, rt + n_rt * q, rq[q]);
#pragma unroll 1
                for (int r = rt + n_rt * RQ; r < n_src; r += n_rt) sst(R.rows, r, fetch(R.src[r]));
                __syncthreads();  // rows in LDS, and every thread has read its stage input
            }
            // the coupling lines
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                if (place[q] < 0) continue;
                const int n = list[q] & 255;
                const uint32_t* loff = R.off + (list[q] >> 8);
                const TE* lwt = R.wt + 2 * (list[q] >> 8);
                cpx<TE> f = {(TE)0, (TE)0};
#pragma unroll 2
                for (int m = 0; m < n; ++m) {
                    const uint32_t o = loff[m];
                    const cpx<TE> wt = sld<TE>(lwt, m);
                    cpx<TE> v;
                    if constexpr (GRID) {
                        v = sld<TE>(R.rows, o & ~kConj);
                    } else if (!S0 && (o & kSigma0)) {
                        const cpx<double> x = sld<double>(sigma0_s, o & ~(kConj | kSigma0));
                        v = {(TE)x.re, (TE)x.im};
                    } else {
                        const cpx<T> x = sld<T>(bulk_s, o & ~kConj);
                        v = {(TE)x.re, (TE)x.im};
                    }
                    if (o & kConj) v.im = -v.im;
                    f.re += wt.re * v.re - wt.im * v.im;
                    f.im += wt.re * v.im + wt.im * v.re;
                }
                out[q].re = y[q].re + (out[q].re + h * f.re);
                out[q].im = y[q].im + (out[q].im + h * f.im);
            }
            if constexpr (!GRID) __syncthreads();  // every thread has read this stage's LDS
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                if (place[q] < 0) continue;
                sst(R.s, rt + n_rt * q, out[q]);
                if constexpr (GRID) {
                    if (!last) {
                        if constexpr (S0) Exchanged(A.s0x[k & 1], s0_bytes).template store<double>(glob[q], out[q]);
                        else Exchanged(A.exch[k & 1], x_bytes).template store<TE>(glob[q], out[q]);
                    }
                }
                const cpx<TE> d = {out[q].re - y[q].re, out[q].im - y[q].im};
                if (k == 0) c[q] = {third * d.re, third * d.im};
                else if (k == 1) c[q] = {c[q].re + two_thirds * d.re, c[q].im + two_thirds * d.im};
                else if (k == 3) y[q] = out[q];
            }
            bool record = false;
            if (S0 && k == 3 && --rec_left == 0) {
                rec_left = J.rec_every;
                ++rec_slot;
                record = true;
            }
            ++epoch;
            if constexpr (GRID) {
                bar.arrive(epoch);
                // the observables while the other workgroups arrive
                if (record && rec_wave) record_wave(J, sigma0_s, rec_slot);
                ok = bar.wait(epoch);
                if (!ok) break;
            } else {
                __syncthreads();
                // sigma_0 changes after the next stage's first barrier, which
                // waits for this wavefront
                if (record && rec_wave) record_wave(J, sigma0_s, rec_slot);
            }
        }
    }
    if constexpr (GRID) {
        // commit or abort, one decision for all workgroups
        if (threadIdx.x == 0 && ok) *bar.dead = bar.decide(A.chunk + 1) == kResidentAborted ? 1 : 0;
        __syncthreads();
        if (!ok || *bar.dead) return;
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q)
        if (place[q] >= 0) st<TE>(S0 ? J.sig0[0] : J.rest[0], glob[q], y[q]);
    if (S0 && rt == 0) {
        *G(J.step) = A.step0 + A.n_steps;
        if (!GRID) *G(A.commit) = A.chunk + 1;
    }
}

// Threads per workgroup and waves per SIMD asked of the register allocator:
// in a grid 768 threads of one element (80 registers) or 512 of more (128),
// so that two workgroups fit a CU; one workgroup alone 1024 threads (128).
template <bool GRID, int EPT>
constexpr int resident_threads() {
    return !GRID ? 1024 : EPT == 1 ? 768 : 512;
}
template <bool GRID, int EPT>
constexpr int resident_waves() {
    return GRID && EPT == 1 ? 6 : 4;
}

template <typename T, bool HC, bool GRID, int EPT>
__global__ __launch_bounds__((resident_threads<GRID, EPT>())) __attribute__((
    amdgpu_waves_per_eu(resident_waves<GRID, EPT>()))) void k_resident(Job J, ResidentArgs A) {
    // 16-byte alignment: the b64 and b128 accesses need it (4 bytes off, the
    // stage took twice as long)
    extern __shared__ __align__(16) char smem[];
    __shared__ __align__(16) int dead;
    const GridBarrier bar{A, &dead};
    if (threadIdx.x == 0) dead = GRID && bar.word() == kResidentAborted ? 1 : 0;
    __syncthreads();
    if (dead) return;
    const ResidentLds L = resident_lds(J.t.N, J.t.W, J.t.D, A.slots, A.low_slots, (int)sizeof(T), HC, GRID, J.herm != 0);
    char* sm0 = smem + (GRID ? 0 : L.bulk);
    auto f64 = [&](size_t at) { return reinterpret_cast<double*>(sm0 + at); };
    auto ft = [&](size_t at) { return reinterpret_cast<T*>(smem + at); };
    const Role<T> rb{ft(L.h), ft(L.s), ft(L.rows), ft(L.wt), ft(L.gam), ft(L.delta),
                     reinterpret_cast<uint32_t*>(smem + L.off), reinterpret_cast<uint32_t*>(smem + L.src),
                     reinterpret_cast<int*>(smem + L.id), reinterpret_cast<int*>(smem + L.count)};
    const Role<double> r0{f64(L.h0), f64(L.s0), f64(L.rows0), f64(L.wt0), f64(L.gam0), f64(L.delta0),
                          reinterpret_cast<uint32_t*>(sm0 + L.off0), reinterpret_cast<uint32_t*>(sm0 + L.src0),
                          reinterpret_cast<int*>(sm0 + L.id0), reinterpret_cast<int*>(sm0 + L.count0)};
    // roles by whole wavefronts
    const int tid = threadIdx.x, n_bulk = GRID ? (int)blockDim.x : A.bulk_threads;
    const bool s0 = GRID ? blockIdx.x == 0 : __builtin_amdgcn_readfirstlane(tid) >= n_bulk;
    if (s0)
        resident_role<double, T, HC, GRID, true, 1>(J, A, bar, r0, rb.s, r0.s, GRID ? tid : tid - n_bulk,
                                                               GRID ? n_bulk : (int)blockDim.x - n_bulk);
    else
        resident_role<T, T, HC, GRID, false, EPT>(J, A, bar, rb, rb.s, r0.s, tid, n_bulk);
}

template <typename T, bool HC, bool GRID, int EPT>
hipError_t launch_t(const Job& J, const ResidentArgs& A, const ResidentPlan& p, hipStream_t stream) {
    const void* fn = reinterpret_cast<const void*>(&k_resident<T, HC, GRID, EPT>);
    {
        static std::once_flag once;
        static hipError_t err = hipSuccess;
        std::call_once(once, [&] {
            err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOneLds);
        });
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL((k_resident<T, HC, GRID, EPT>), dim3(GRID ? p.groups + 1 : 1), dim3(p.threads),
                       p.lds, stream, J, A);
    return hipGetLastError();
}

template <typename T, bool HC>
hipError_t launch_h(const Job& J, const ResidentArgs& A, const ResidentPlan& p, hipStream_t stream) {
    if (p.grid)
        return p.ept == 1   ? launch_t<T, HC, true, 1>(J, A, p, stream)
               : p.ept == 2 ? launch_t<T, HC, true, 2>(J, A, p, stream)
                            : launch_t<T, HC, true, 4>(J, A, p, stream);
    return p.ept == 1 ? launch_t<T, HC, false, 1>(J, A, p, stream)
                      : launch_t<T, HC, false, 2>(J, A, p, stream);
}

// --------------------------------------------------------------------------
// The coherence-block form of an absorption run (heom_propagate_block, see
// k_block_stage for the equations) in one launch: the same two forms, FP64,
// elements (u, a, p), ADO 0 among them.  An element couples to elements of
// the same row and direction only, so nothing is staged: each link is one
// load of the element's own (three directions, 48 bytes, per ADO row).
// Every operation and its order are those of block_stage_elem, so a run
// gives the bits that the server's batched stages give.
// --------------------------------------------------------------------------
struct BlockLds {
    size_t h, s, wt, off, gam, delta, count, total;
};

__host__ __device__ inline BlockLds block_lds(int N, int W, int D, int slots, int low, bool hc) {
    const size_t NN = (size_t)N * N, S = slots;
    // an ADO has at most D "-" rows and W "+" rows, each of three elements
    const size_t links = 3 * (S * (D > 0 ? D : 1) + (size_t)low * W);
    BlockLds L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align16(o + bytes);
        return at;
    };
    L.h = take(NN * (hc ? 16 : 8));
    L.s = take(S * N * 3 * 16);
    L.wt = take(links * 16);
    L.off = take(links * 4);
    L.gam = take(S * 8);
    L.delta = take((size_t)N * 8);
    L.count = take(4);
    L.total = o;
    return L;
}

template <bool HC, bool GRID, int EPT>
__global__ __launch_bounds__((resident_threads<GRID, EPT>())) __attribute__((
    amdgpu_waves_per_eu(resident_waves<GRID, EPT>()))) void k_resident_block(Tables t, ResidentArgs A,
                                                                             BlockRun B, BlockObs obs) {
    extern __shared__ __align__(16) char smem[];
    __shared__ __align__(16) int dead;
    const GridBarrier bar{A, &dead};
    const int tid = threadIdx.x, n_t = blockDim.x;
    if (tid == 0) dead = GRID && bar.word() == kResidentAborted ? 1 : 0;
    __syncthreads();
    if (dead) return;
    const int N = t.N, W = t.W, D = t.D, Dm = D > 0 ? D : 1, R = 3 * N;
    const int Gr = GRID ? A.groups : 1, w = GRID ? (int)blockIdx.x : 0;
    const int ns = max(0, (t.n_ado - 1 - w + Gr) / Gr);
    const BlockLds L = block_lds(N, W, D, A.slots, A.low_slots, HC);
    double* sH = reinterpret_cast<double*>(smem + L.h);
    double* S = reinterpret_cast<double*>(smem + L.s);
    double* sWt = reinterpret_cast<double*>(smem + L.wt);
    uint32_t* sOff = reinterpret_cast<uint32_t*>(smem + L.off);
    double* sGam = reinterpret_cast<double*>(smem + L.gam);
    double* sDelta = reinterpret_cast<double*>(smem + L.delta);
    int* sCount = reinterpret_cast<int*>(smem + L.count);
    for (int e = tid; e < N * N; e += n_t) {
        sH[HC ? 2 * e : e] = G(t.h_re)[e];
        if constexpr (HC) sH[2 * e + 1] = G(t.h_im)[e];
    }
    for (int g = tid; g < ns; g += n_t) sGam[g] = G(t.damping)[w + g * Gr];
    for (int x = tid; x < N; x += n_t) sDelta[x] = G(t.delta_state)[x];
    if (tid == 0) *sCount = 0;
    __syncthreads();
    cpx<double> y[EPT], y2[EPT], y3[EPT];
    int place[EPT], list[EPT];  // slot << 16 | row in the ADO, -1 without one; list begin << 8 | entries
    uint32_t glob[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = tid + n_t * q;
        y[q] = y2[q] = y3[q] = {0.0, 0.0};
        place[q] = -1;
        list[q] = 0;
        glob[q] = 0;
        if (e >= ns * R) continue;
        const int g = e / R, r = e - g * R, a = r / 3;
        const size_t u = w + (size_t)g * Gr;
        glob[q] = (uint32_t)(u * R + r);
        y[q] = ld<double>(B.state, glob[q]);
        sst(S, e, y[q]);
        const int bi = G(t.state_mode_begin)[a];
        const int np = G(t.level)[u] < D ? G(t.state_mode_begin)[a + 1] - bi : 0;
        int n = np;
        for (int k = 0; k < Dm; ++k) n += G(t.mlist_site)[u * Dm + k] == a;
        int at = atomicAdd(sCount, n);
        place[q] = g << 16 | r;
        list[q] = at << 8 | n;
        for (int m = 0; m < np; ++m, ++at) {
            const int l = G(t.state_modes)[bi + m];
            sOff[at] = (uint32_t)(G(t.plus)[u * W + l] * R + r);
            sst(sWt, at, cpx<double>{0.0, G(t.plus_w)[u * W + l]});
        }
        for (int k = 0; k < Dm; ++k) {
            if (G(t.mlist_site)[u * Dm + k] != a) continue;
            const pair_d v = G(reinterpret_cast<const pair_d*>(t.mlist_w))[u * Dm + k];
            sOff[at] = (uint32_t)(G(reinterpret_cast<const pair_i*>(t.mlist))[u * Dm + k].x * R + r);
            sst(sWt, at++, cpx<double>{v.x, v.y});
        }
    }
    __syncthreads();
    // P_p = sum_a obs[p][a] Y_0[a][p] by three threads of ADO 0's workgroup
    auto record = [&](int64_t slot) {
        if (w != 0 || tid >= 3 || slot < 0 || slot >= B.n_rec) return;
        double pr = 0.0, pi = 0.0;
        for (int a = 0; a < N; ++a) {
            const cpx<double> x = sld<double>(S, a * 3 + tid);
            pr = fma(obs.v[tid][a], x.re, pr);
            pi = fma(obs.v[tid][a], x.im, pi);
        }
        G(B.rec)[6 * slot + 2 * tid] = pr;
        G(B.rec)[6 * slot + 2 * tid + 1] = pi;
        if (!(isfinite(pr) && isfinite(pi))) *G(B.status) = 1;
    };
    if (A.step0 == 0) record(0);
    const uint32_t x_bytes = (uint32_t)((size_t)t.n_ado * R * 16);
    bool ok = true;
    uint32_t epoch = A.epoch0;
    int rec_left = B.rec_every - (int)(A.step0 % B.rec_every);
    int64_t rec_slot = A.step0 / B.rec_every;
    for (int64_t step = 0; ok && step < A.n_steps; ++step) {
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            const bool first = step == 0 && k == 0, last = step + 1 == A.n_steps && k == 3;
            const double h = B.dt * (k < 2 ? 0.5 : k == 2 ? 1.0 : 1.0 / 6.0);
            const Exchanged xin(first ? B.state : A.exch[(k + 1) & 1], x_bytes);
            auto fetch = [&](uint32_t o) { return GRID ? xin.template load<double>(o) : sld<double>(S, o); };
#pragma unroll
            for (int q = 0; q < EPT; ++q) asm volatile("" : "+v"(place[q]), "+v"(list[q]), "+v"(glob[q]));
            cpx<double> out[EPT];
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                out[q] = {0.0, 0.0};
                if (place[q] < 0) continue;
                constexpr int KB = 4;  // links in flight
                const int n = list[q] & 255;
                const uint32_t* loff = sOff + (list[q] >> 8);
                const double* lwt = sWt + 2 * (list[q] >> 8);
                cpx<double> xs[KB];
#pragma unroll
                for (int m = 0; m < KB; ++m) {
                    xs[m] = {0.0, 0.0};
                    if (m < n) xs[m] = fetch(loff[m]);
                }
                const int g = place[q] >> 16, r = place[q] & 0xffff, a = r / 3, p = r - 3 * a;
                const double* Sg = S + 2 * g * R;
                const cpx<double> y0 = sld<double>(Sg, r);
                double cr = t.h_shift * y0.re, ci = t.h_shift * y0.im;
#pragma unroll 2
                for (int b = 0; b < N; ++b) {
                    const cpx<double> v = sld<double>(Sg, 3 * b + p);
                    if constexpr (HC) {
                        const cpx<double> hh = sld<double>(sH, a * N + b);
                        cr = fma(hh.re, v.re, fma(-hh.im, v.im, cr));
                        ci = fma(hh.re, v.im, fma(hh.im, v.re, ci));
                    } else {
                        const double hr = sH[a * N + b];
                        cr = fma(hr, v.re, cr);
                        ci = fma(hr, v.im, ci);
                    }
                }
                const double gm = sGam[g] + sDelta[a];
                double fr = fma(-gm, y0.re, ci), fi = fma(-gm, y0.im, -cr);
                auto add = [&](int m, cpx<double> x) {
                    const cpx<double> wt = sld<double>(lwt, m);
                    fr = fma(wt.re, x.re, fma(-wt.im, x.im, fr));
                    fi = fma(wt.re, x.im, fma(wt.im, x.re, fi));
                };
#pragma unroll
                for (int m = 0; m < KB; ++m)
                    if (m < n) add(m, xs[m]);
#pragma unroll 1
                for (int m = KB; m < n; ++m) add(m, fetch(loff[m]));
                const double w_in = k == 0 ? 1.0 : k == 3 ? 1.0 / 3.0 : 0.0;
                double yr = fma(h, fr, w_in * y0.re), yi = fma(h, fi, w_in * y0.im);
                if (k == 1 || k == 2) {
                    yr = fma(1.0, y[q].re, yr);
                    yi = fma(1.0, y[q].im, yi);
                } else if (k == 3) {
                    yr = fma(2.0 / 3.0, y3[q].re, fma(1.0 / 3.0, y2[q].re, fma(-1.0 / 3.0, y[q].re, yr)));
                    yi = fma(2.0 / 3.0, y3[q].im, fma(1.0 / 3.0, y2[q].im, fma(-1.0 / 3.0, y[q].im, yi)));
                }
                out[q] = {yr, yi};
            }
            __syncthreads();  // every thread has read this stage's LDS
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                if (place[q] < 0) continue;
                sst(S, tid + n_t * q, out[q]);
                if constexpr (GRID) {
                    if (!last) Exchanged(A.exch[k & 1], x_bytes).template store<double>(glob[q], out[q]);
                }
                if (k == 0) y2[q] = out[q];
                else if (k == 1) y3[q] = out[q];
                else if (k == 3) y[q] = out[q];
            }
            bool due = false;
            if (k == 3 && --rec_left == 0) {
                rec_left = B.rec_every;
                ++rec_slot;
                due = true;
            }
            ++epoch;
            if constexpr (GRID) {
                bar.arrive(epoch);
                if (due) record(rec_slot);
                ok = bar.wait(epoch);
                if (!ok) break;
            } else {
                __syncthreads();
                if (due) record(rec_slot);
            }
        }
    }
    if constexpr (GRID) {
        if (tid == 0 && ok) dead = bar.decide(A.chunk + 1) == kResidentAborted ? 1 : 0;
        __syncthreads();
        if (!ok || dead) return;
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q)
        if (place[q] >= 0) st<double>(B.state, glob[q], y[q]);
    if (w == 0 && tid == 0) {
        *G(B.step) = A.step0 + A.n_steps;
        if (!GRID) *G(A.commit) = A.chunk + 1;
    }
}

template <bool HC, bool GRID, int EPT>
hipError_t launch_block_t(const Tables& t, const ResidentArgs& A, const BlockRun& B, const BlockObs& obs,
                          const ResidentPlan& p, hipStream_t stream) {
    static std::once_flag once;
    static hipError_t err = hipSuccess;
    std::call_once(once, [&] {
        err = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_resident_block<HC, GRID, EPT>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOneLds);
    });
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL((k_resident_block<HC, GRID, EPT>), dim3(p.groups), dim3(p.threads), p.lds, stream, t, A,
                       B, obs);
    return hipGetLastError();
}

template <bool HC>
hipError_t launch_block_h(const Tables& t, const ResidentArgs& A, const BlockRun& B, const BlockObs& obs,
                          const ResidentPlan& p, hipStream_t stream) {
    if (!p.grid)
        return p.ept == 1 ? launch_block_t<HC, false, 1>(t, A, B, obs, p, stream)
                          : launch_block_t<HC, false, 2>(t, A, B, obs, p, stream);
    return p.ept == 1   ? launch_block_t<HC, true, 1>(t, A, B, obs, p, stream)
           : p.ept == 2 ? launch_block_t<HC, true, 2>(t, A, B, obs, p, stream)
                        : launch_block_t<HC, true, 4>(t, A, B, obs, p, stream);
}

constexpr int round64(int x) { return (x + 63) / 64 * 64; }

}  // namespace

// Which hierarchies run resident.  One workgroup while sigma_0 has a thread
// per element, the other threads hold at most two each, and the LDS holds
// the state; else a grid of up to 255 bulk workgroups, as long as each takes
// one element per thread or 512 threads of four, and 80 KiB of LDS.  N <= 22
// leaves sigma_0 a thread per element in the smallest of these workgroups.
bool resident_plan(const Job& J, int tsize, ResidentPlan* p) {
    const Tables& t = J.t;
    const int N = t.N, NN = N * N, n = t.n_ado - 1;
    if (N > 22 || n < 1 || t.W + t.D > 255) return false;  // a list has at most 255 entries
    const bool hc = t.h_complex != 0;
    const int64_t elements = (int64_t)n * NN;
    *p = ResidentPlan{};
    const int s0_threads = round64(NN), left = 1024 - s0_threads;
    if (left > 0 && elements <= 2 * left) {
        const ResidentLds L = resident_lds(N, t.W, t.D, n, J.n_low, tsize, hc, false, J.herm != 0);
        p->lds = L.bulk + L.s0part;
        if (p->lds <= kOneLds) {
            p->grid = false;
            p->groups = 1;
            p->slots = n;
            p->low_slots = J.n_low;
            p->ept = elements <= left ? 1 : 2;
            p->bulk_threads = round64((int)((elements + p->ept - 1) / p->ept));
            p->threads = p->bulk_threads + s0_threads;
            return true;
        }
    }
    p->grid = true;
    // As many workgroups as there are ADOs, up to 255: a stage's work is divided
    // by their number, its barrier grows with it by little (us per stage with 32 /
    // 64 / 128 / 255: 3060 ADOs of 7 x 7 FP32 11.2 / 11.1 / 7.5 / 4.3, FP64 10.9 /
    // 11.0 / 11.0 / 5.0; 256 of 20 x 20 FP32 5.1 / 4.2 / 4.2 / 4.3; 286 of 5 x 5
    // 3.3 / 3.2 / 3.4 / 3.7; 165 of 4 x 4 3.1 / 3.0 / 3.2 / 3.3).
    p->groups = std::min(n, kGridMax - 1);
    p->slots = (n + p->groups - 1) / p->groups;
    p->low_slots = (J.n_low + p->groups - 1) / p->groups;
    const int per = (int)std::min<int64_t>((int64_t)p->slots * NN, 1 << 20);
    if (per > 4 * 512) return false;
    const ResidentLds L = resident_lds(N, t.W, t.D, p->slots, p->low_slots, tsize, hc, true, J.herm != 0);
    p->lds = std::max(L.bulk, L.s0part);
    p->ept = per <= resident_threads<true, 1>() ? 1 : per <= 2 * resident_threads<true, 2>() ? 2 : 4;
    // at least one thread per flag and per element of sigma_0
    p->threads = std::max({round64((per + p->ept - 1) / p->ept), kGridMax, round64(NN)});
    p->bulk_threads = p->threads;
    return p->lds <= kGridLds;
}

// A workspace has room for three copies of sigma_0 and of the ADOs, and the
// records behind them.  A grid takes two of each and its flags, 64 bytes per
// workgroup: more than the third copies hold where the ADOs are 1 x 1 or 2 x 2
// in FP32 and few enough (481 to 503 of them at 2 x 2, for instance).
bool resident_layout(const ResidentPlan& p, size_t sigma0_bytes, size_t rest_bytes, size_t offset,
                     size_t work_bytes, ResidentLayout* L) {
    *L = ResidentLayout{};
    size_t o = offset;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = (o + bytes + 255) & ~size_t(255);
        return at;
    };
    if (p.grid) {
        L->flag_bytes = (size_t)(p.groups + 1) * kResidentFlagStride * 4;
        L->flags = take(L->flag_bytes);
        for (int k = 0; k < 2; ++k) L->s0x[k] = take(sigma0_bytes);
        for (int k = 0; k < 2; ++k) L->exch[k] = take(rest_bytes);
    }
    L->end = o;
    return o <= work_bytes;
}

hipError_t launch_resident(const Job& J, const ResidentArgs& args, const ResidentPlan& p, int precision,
                           hipStream_t stream) {
    ResidentArgs A = args;
    A.groups = p.groups;
    A.slots = p.slots;
    A.low_slots = p.low_slots;
    A.bulk_threads = p.bulk_threads;
    A.members = p.groups + 1;
    const bool hc = J.t.h_complex != 0;
    if (precision == 0)
        return hc ? launch_h<double, true>(J, A, p, stream) : launch_h<double, false>(J, A, p, stream);
    return hc ? launch_h<float, true>(J, A, p, stream) : launch_h<float, false>(J, A, p, stream);
}

// The same choice for the coherence-block form (elements n_ado * 3 N).
bool resident_block_plan(const Tables& t, int n_low, ResidentPlan* p) {
    const int R = 3 * t.N, n = t.n_ado;
    if (t.W + t.D > 255) return false;
    const int64_t elements = (int64_t)n * R;
    const bool hc = t.h_complex != 0;
    *p = ResidentPlan{};
    if (elements <= 2 * 1024) {
        p->lds = block_lds(t.N, t.W, t.D, n, n_low + 1, hc).total;
        if (p->lds <= kOneLds) {
            p->groups = 1;
            p->slots = n;
            p->low_slots = n_low + 1;
            p->ept = elements <= 1024 ? 1 : 2;
            p->threads = round64((int)((elements + p->ept - 1) / p->ept));
            return true;
        }
    }
    p->grid = true;
    p->groups = std::min(n, kGridMax);
    p->slots = (n + p->groups - 1) / p->groups;
    p->low_slots = (n_low + p->groups) / p->groups;  // of ADOs 0..n_low
    const int per = (int)std::min<int64_t>((int64_t)p->slots * R, 1 << 20);
    if (per > 4 * 512) return false;
    p->lds = block_lds(t.N, t.W, t.D, p->slots, p->low_slots, hc).total;
    p->ept = per <= resident_threads<true, 1>() ? 1 : per <= 2 * resident_threads<true, 2>() ? 2 : 4;
    p->threads = std::max(round64((per + p->ept - 1) / p->ept), kGridMax);
    return p->lds <= kGridLds;
}

hipError_t launch_resident_block(const Tables& t, const ResidentArgs& args, const BlockRun& run,
                                 const BlockObs& obs, const ResidentPlan& p, hipStream_t stream) {
    ResidentArgs A = args;
    A.groups = A.members = p.groups;
    A.slots = p.slots;
    A.low_slots = p.low_slots;
    return t.h_complex != 0 ? launch_block_h<true>(t, A, run, obs, p, stream)
                            : launch_block_h<false>(t, A, run, obs, p, stream);
}

}  // namespace heom
