// Device code shared by the stage kernels: neighbour accesses, the sigma_0
// stage, the matrix-core operations.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "heom_device.h"
#include "heom_internal.h"

namespace heom {
namespace {

// --------------------------------------------------------------------------
// Right-hand side of eq. HEOM for one matrix element (i, j) of ADO u.
// Commutator operands come from LDS (sH: H, sS: sigma_u, both interleaved
// complex, row-major); neighbour elements come from global memory.
//
// Coupling lines for a mode l of state s (V = |s><s|):
//   (V^x A)_ij = ((i==s) - (j==s)) A_ij,  (V^o A)_ij = ((i==s) + (j==s)) A_ij
//   +: i * sign * sqrt((n_l+1)|c_l|) * (V^x sigma_{u+e_l})_ij
//   -: sqrt(n_l/|c_l|) * sign * (i c_l V^x + delta_k0 lambda nu V^o) sigma_{u-e_l}
// Only modes of the states i and j contribute to element (i, j).
// With `herm`, the column s of a neighbour is read as conj(row s).
// --------------------------------------------------------------------------
template <typename T>
struct NbSrc {
    const void* sig0;  // complex128 [N][N] (neighbour index 0)
    const void* rest;  // T [n_ado-1][N][N]
    int N;
};

template <typename T>
__device__ __forceinline__ cpx<T> load_nb(const NbSrc<T>& s, int nb, int r, int c) {
    if (nb == 0) {
        const cpx<double> v = ld<double>(s.sig0, (size_t)r * s.N + c);
        return {(T)v.re, (T)v.im};
    }
    return ld<T>(s.rest, (size_t)(nb - 1) * s.N * s.N + (size_t)r * s.N + c);
}

// Hermitian-packed storage: ADO u >= 1 is the real N x N array
//   P[i][j] = Re sigma(i, j) for i <= j,   P[i][j] = Im sigma(j, i) for i > j,
// half the bytes of the complex form.  With a = min(r, c), b = max(r, c):
//   sigma(r, c) = (P[a][b], +P[b][a]) above the diagonal, (P[a][b], -P[b][a])
//   below it, (P[a][a], 0) on it.
// Packed value P_nb[r][c] of neighbour nb (index 0: the complex128 sigma_0,
// whose upper triangle is taken).
template <typename T>
__device__ __forceinline__ T pk_nb(const NbSrc<T>& s, int nb, int r, int c) {
    if (nb == 0) {
        const cpx<double> v = ld<double>(s.sig0, (size_t)min(r, c) * s.N + max(r, c));
        return (T)(r <= c ? v.re : v.im);
    }
    return G(reinterpret_cast<const T*>(s.rest))[(size_t)(nb - 1) * s.N * s.N + (size_t)r * s.N + c];
}

// Element of row r, column c of ADO u >= 1 where n ADOs lie in tiles of GA
// consecutive ones, [row][ADO][column] (heom_columns.hip).
__device__ __forceinline__ size_t tiled_at(int GA, int N, int u, int r, int c, int n) {
    const int v = u - 1, first = v / GA * GA;
    return (size_t)first * (N * N) + (uint32_t)(r * (min(GA, n - first) * N) + (v - first) * N + c);
}

// Element (r, c) of neighbour nb, from complex (PK false) or packed storage;
// TILE > 0: complex, n ADOs in tiles of TILE.
template <typename T, bool PK, int TILE = 0>
__device__ __forceinline__ cpx<T> nb_get(const NbSrc<T>& s, int nb, int r, int c, int n = 0) {
    if constexpr (TILE > 0) {
        if (nb == 0) return load_nb<T>(s, 0, r, c);
        return ld<T>(s.rest, tiled_at(TILE, s.N, nb, r, c, n));
    } else if constexpr (PK) {
        if (nb == 0) return load_nb<T>(s, 0, r, c);
        const T x = pk_nb(s, nb, min(r, c), max(r, c)), y = pk_nb(s, nb, max(r, c), min(r, c));
        return {x, r < c ? y : (r > c ? -y : (T)0)};
    } else {
        return load_nb<T>(s, nb, r, c);
    }
}

// The job a tile belongs to.  Single-job launches read the descriptor from
// the kernel argument; batched launches from the device job table (found by
// binary search over the jobs' first tiles).  Keeping the two apart lets the
// compiler address each descriptor in its own memory space.
template <bool BATCHED>
struct JobOf;
template <>
struct JobOf<false> {
    static __device__ __forceinline__ const Job& get(const Job& single, const Job*, int, int) {
        return single;
    }
};
template <>
struct JobOf<true> {
    static __device__ __forceinline__ const Job& get(const Job&, const Job* jobs, int n_jobs,
                                                     int tile) {
        int lo = 0, hi = n_jobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].tile_begin <= tile)
                lo = mid;
            else
                hi = mid - 1;
        }
        return jobs[lo];
    }
};

// --------------------------------------------------------------------------
// sigma_0 stage kernel: one workgroup per job, FP64 throughout; reads the
// level-1 ADOs in the bulk precision T.  Also records the observables.
// --------------------------------------------------------------------------
__device__ void record_sigma0(const Job& J, const double* sS, int64_t slot) {
    // sS: interleaved complex128 [N][N] in LDS.  Caller: one thread.
    if (slot < 0 || slot >= J.n_rec_max) return;
    const int N = J.t.N;
    gptr<double> rec = G(J.records) + slot * J.rec_doubles;
    double trr = 0.0, tri = 0.0;
    for (int i = 0; i < N; ++i) {
        trr += sS[2 * (i * N + i)];
        tri += sS[2 * (i * N + i) + 1];
    }
    bool finite = isfinite(trr) && isfinite(tri);
    if (J.rec_kind == 0) {
        double herm = 0.0;
        for (int i = 0; i < N; ++i) {
            rec[i] = sS[2 * (i * N + i)];
            for (int j = 0; j < N; ++j) {
                const double dr = sS[2 * (i * N + j)] - sS[2 * (j * N + i)];
                const double di = sS[2 * (i * N + j) + 1] + sS[2 * (j * N + i) + 1];
                herm = fmax(herm, sqrt(dr * dr + di * di));
            }
        }
        rec[N] = trr;
        rec[N + 1] = tri;
        rec[N + 2] = herm;
        finite = finite && isfinite(herm);
    } else {
        double pr = 0.0, pi = 0.0;
        for (int a = 0; a < N; ++a) {
            pr += G(J.mu)[a] * sS[2 * (a * N + J.ground)];
            pi += G(J.mu)[a] * sS[2 * (a * N + J.ground) + 1];
        }
        rec[0] = pr;
        rec[1] = pi;
        rec[2] = trr;
        rec[3] = tri;
        finite = finite && isfinite(pr) && isfinite(pi);
    }
    if (!finite) *G(J.status) = 1;
}

// LDS plan of the sigma_0 kernel: H and sigma_0 in FP64, per-mode weights,
// per-state tables, and (when they fit) the row s_l (and, for non-Hermitian
// states, the column s_l) of every level-1 ADO e_l.
struct Sigma0Lds {
    size_t h, s, pa, delta, site, begin, modes, rows, cols, total;
    bool rows_in_lds;
};

// cap: the LDS bytes the launch provides (rows are staged only if they fit).
__host__ __device__ inline Sigma0Lds sigma0_lds(int N, int W, int tsize, bool herm, size_t cap) {
    Sigma0Lds L{};
    size_t o = 0;
    const size_t NN = (size_t)N * N;
    L.h = o; o += 16 * NN;
    L.s = o; o += 16 * NN;
    L.pa = o; o += 8 * (size_t)W;
    L.delta = o; o += 8 * (size_t)N;
    L.site = o; o += 4 * (size_t)W;
    L.begin = o; o += 4 * (size_t)(N + 1);
    L.modes = o; o += 4 * (size_t)W;
    o = (o + 15) & ~size_t(15);
    const size_t rows = 2 * (size_t)tsize * W * N;
    L.rows_in_lds = o + rows * (herm ? 1 : 2) <= cap;
    L.rows = o;
    if (L.rows_in_lds) o += rows;
    L.cols = o;
    if (L.rows_in_lds && !herm) o += rows;
    L.total = o;
    return L;
}

// The sigma_0 stage of job `job` by the whole workgroup (any block size):
// the body of k_sigma0, and of the extra workgroups of a bulk launch that
// carries sigma_0 along (lds_cap: the LDS the launch provides).
// HC: the job may have a complex H.  The loops stay rolled: the code also
// runs inside the bulk kernels, whose occupancy its registers would cost.
template <typename T, bool BATCHED, bool HC, bool PK = false, int TILE = 0>
__device__ void sigma0_stage(const Job& single, const Job* jobs, int job, const StageSpec& sp,
                             unsigned lds_cap, char* smem_s0) {
    const Job& J = BATCHED ? jobs[job] : single;
    const Tables& t = J.t;
    const int N = t.N, NN = N * N, W = t.W, D = t.D;
    const bool herm = J.herm != 0;
    const Sigma0Lds L = sigma0_lds(N, W, (int)sizeof(T), herm, lds_cap);
    double* sH = reinterpret_cast<double*>(smem_s0 + L.h);
    double* sS = reinterpret_cast<double*>(smem_s0 + L.s);
    double* sPa = reinterpret_cast<double*>(smem_s0 + L.pa);
    double* sDelta = reinterpret_cast<double*>(smem_s0 + L.delta);
    int* sSite = reinterpret_cast<int*>(smem_s0 + L.site);
    int* sBegin = reinterpret_cast<int*>(smem_s0 + L.begin);
    int* sModes = reinterpret_cast<int*>(smem_s0 + L.modes);
    T* sRows = reinterpret_cast<T*>(smem_s0 + L.rows);  // [W][N] complex
    T* sCols = reinterpret_cast<T*>(smem_s0 + L.cols);  // [W][N] complex
    const int tid = threadIdx.x;
    const bool hc = HC && t.h_complex != 0;
    const NbSrc<T> nbs{J.sig0[sp.in], J.rest[sp.in], N};
    for (int e = tid; e < NN; e += blockDim.x) {
        sH[2 * e] = G(t.h_re)[e];
        sH[2 * e + 1] = hc ? G(t.h_im)[e] : 0.0;
        const cpx<double> v = ld<double>(J.sig0[sp.in], e);
        sS[2 * e] = v.re;
        sS[2 * e + 1] = v.im;
    }
    for (int l = tid; l < W; l += blockDim.x) {
        sPa[l] = (D > 0) ? G(t.plus_coef)[l * (D + 1)] : 0.0;
        sSite[l] = G(t.mode_site)[l];
        sModes[l] = G(t.state_modes)[l];
    }
    for (int x = tid; x <= N; x += blockDim.x) {
        sBegin[x] = G(t.state_mode_begin)[x];
        if (x < N) sDelta[x] = G(t.delta_state)[x];
    }
    if (D > 0 && L.rows_in_lds) {
        for (int idx = tid; idx < W * N; idx += blockDim.x) {
            const int l = idx / N, c = idx - (idx / N) * N;
            const int site = G(t.mode_site)[l];
            const cpx<T> r = nb_get<T, PK, TILE>(nbs, 1 + l, site, c, t.n_ado - 1);
            sRows[2 * idx] = r.re;
            sRows[2 * idx + 1] = r.im;
            if (!herm) {
                const cpx<T> v = load_nb<T>(nbs, 1 + l, c, site);
                sCols[2 * idx] = v.re;
                sCols[2 * idx + 1] = v.im;
            }
        }
    }
    __syncthreads();
    if (sp.record_initial && tid == 0 && *G(J.step) == 0) record_sigma0(J, sS, 0);

    const double h = sp.hmul * J.dt;
#pragma unroll 1
    for (int e = tid; e < NN; e += blockDim.x) {
        const int i = e / N, j = e - (e / N) * N;
        // -i [H, sigma_0] (the damping vanishes at u = 0)
        double cr = 0, ci = 0;
        if (hc) {
#pragma unroll 1
            for (int k = 0; k < N; ++k) {
                const double hr = sH[2 * (i * N + k)], hi = sH[2 * (i * N + k) + 1];
                const double xr = sS[2 * (k * N + j)], xi = sS[2 * (k * N + j) + 1];
                const double yr = sS[2 * (i * N + k)], yi = sS[2 * (i * N + k) + 1];
                const double gr = sH[2 * (k * N + j)], gi = sH[2 * (k * N + j) + 1];
                cr += hr * xr - hi * xi - (yr * gr - yi * gi);
                ci += hr * xi + hi * xr - (yr * gi + yi * gr);
            }
        } else {
#pragma unroll 1
            for (int k = 0; k < N; ++k) {
                const double hik = sH[2 * (i * N + k)], hkj = sH[2 * (k * N + j)];
                cr += hik * sS[2 * (k * N + j)] - sS[2 * (i * N + k)] * hkj;
                ci += hik * sS[2 * (k * N + j) + 1] - sS[2 * (i * N + k) + 1] * hkj;
            }
        }
        const double dl = (i != j) ? sDelta[i] + sDelta[j] : 0.0;
        double fr = ci - dl * sS[2 * e], fi = -cr - dl * sS[2 * e + 1];
        // "+" couplings to the level-1 ADOs e_l (index 1 + l), modes of states i and j
        if (D > 0 && i != j) {
            for (int pass = 0; pass < 2; ++pass) {
                const int s = pass == 0 ? i : j;
                for (int m = sBegin[s]; m < sBegin[s + 1]; ++m) {
                    const int l = sModes[m];
                    cpx<T> x;
                    if (L.rows_in_lds) {
                        if (pass == 0) {
                            x = {sRows[2 * (l * N + j)], sRows[2 * (l * N + j) + 1]};
                        } else if (herm) {
                            x = cconj(cpx<T>{sRows[2 * (l * N + i)], sRows[2 * (l * N + i) + 1]});
                        } else {
                            x = {sCols[2 * (l * N + i)], sCols[2 * (l * N + i) + 1]};
                        }
                    } else {
                        x = (herm && pass == 1) ? cconj(nb_get<T, PK, TILE>(nbs, 1 + l, s, i, t.n_ado - 1))
                                                : nb_get<T, PK, TILE>(nbs, 1 + l, i, j, t.n_ado - 1);
                    }
                    const double pa = pass == 0 ? sPa[l] : -sPa[l];
                    fr -= pa * (double)x.im;
                    fi += pa * (double)x.re;
                }
            }
        }
        // RK4 stage combination in FP64; out may be a base (stage 4), which
        // only this thread reads at element e.
        double yr = sp.w_in * sS[2 * e], yi = sp.w_in * sS[2 * e + 1];
        for (int m = 0; m < sp.nbase; ++m) {
            const cpx<double> bv = ld<double>(J.sig0[sp.base[m]], e);
            yr += sp.wbase[m] * bv.re;
            yi += sp.wbase[m] * bv.im;
        }
        st<double>(J.sig0[sp.out], e, cpx<double>{yr + h * fr, yi + h * fi});
    }
    if (sp.record_after) {
        // the new sigma_0 back into LDS for the observables
        __threadfence();
        __syncthreads();
        for (int e = tid; e < NN; e += blockDim.x) {
            const cpx<double> v = ld<double>(J.sig0[sp.out], e);
            sS[2 * e] = v.re;
            sS[2 * e + 1] = v.im;
        }
        __syncthreads();
        if (tid == 0) {
            const int64_t step = *G(J.step) + 1;
            *G(J.step) = step;
            if (step % J.rec_every == 0) record_sigma0(J, sS, step / J.rec_every);
        }
    }
}

template <typename T>
struct mfma_acc;
template <>
struct mfma_acc<float> {
    typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct mfma_acc<double> {
    typedef double type __attribute__((ext_vector_type(4)));
};

__device__ __forceinline__ mfma_acc<float>::type mfma16(float a, float b,
                                                        mfma_acc<float>::type c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ mfma_acc<double>::type mfma16(double a, double b,
                                                         mfma_acc<double>::type c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Row (inside a 16x16 tile) of output item r held by `lane`.
template <typename T>
__device__ __forceinline__ int mfma_row(int lane, int r);
template <>
__device__ __forceinline__ int mfma_row<float>(int lane, int r) {
    return 4 * (lane >> 4) + r;
}
template <>
__device__ __forceinline__ int mfma_row<double>(int lane, int r) {
    return 4 * r + (lane >> 4);
}

// Wave-uniform value into a scalar register.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ double uniform(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

}  // namespace
}  // namespace heom
