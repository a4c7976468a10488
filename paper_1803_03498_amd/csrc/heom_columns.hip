// Propagation of large Hermitian hierarchies of small systems (real H,
// 2 <= N <= 8, HEOM_FP32_MIXED and HEOM_FP64): eq. HEOM of the section "HEOM
// formalism" of Kramer et al., arXiv:1803.03498, fused with RK4.
//
// A lane holds one column of one ADO: lane (g, c) = (lane / N, lane % N) of a
// wavefront has sigma[k][c] of its g-th ADO, all k.  The product with H is then
// N^2 multiply-adds of registers with scalar registers, a coupling row costs a
// lane one element, and a wavefront's 64 / N ADOs need no barrier.  (The
// kernel of one thread per element, k_stage_small, reads three LDS words per
// multiply-add and waits at barriers.  Seven sites, 12.3 million ADOs, FP32, the
// top level: 3.6 to 5.8 ms per stage there, 2.3 to 4.2 here, 5.3 to 6 TB/s of
// elements, links and rows.)
//
// With Z = -i H sigma + (weighted coupling rows), f = Z + Z^dagger - damping:
// the coupling rows of a column's lane add into its own column of Z, and one
// exchange through LDS (row stride 65 elements: free of bank conflicts both
// ways) brings Z[c][k].
//
// Inside a run the ADOs lie in tiles of 64 / N consecutive ADOs, [k][ADO][c]:
// a wavefront's access to row k is one contiguous piece, lane after lane, and
// so are its coupling rows, because consecutive ADOs mostly couple to the same
// row of consecutive ADOs.  (Row after row of each ADO apart, every 56-byte
// row of seven FP32 states cost a 128-byte line of its own: 13.5 GB fetched
// per stage by the top level and 2.6 ms, and 2.5 ms below it.)  The first step
// reads the caller's order, the last stage of the last step writes it.
//
// A step moves 12 passes over the array instead of 13: stage 2 leaves
// Z = (-y + Y2 + 2 Y3)/3, stage 3 writes Y4 over Y2, stage 4 is
// Y4/3 + Z + dt/6 f(Y4).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "heom_device.h"
#include "heom_internal.h"
#include "heom_stage_common.h"

namespace heom {
namespace {

template <typename T>
struct ColumnsStage {
    const T* in;    // complex [n_ado - 1][N][N], like the others
    T* out;
    const T* base;  // y (stages 2, 3) or Z (stage 4)
    T* z;           // stage 2
    T w_in, h;
    int base_plain, out_plain;  // in the caller's order, not in tiles
};

constexpr int kColStride = 65;  // elements between rows of Z

// LDS of a wavefront: the links of a tile, and in one place its "+" links
// (below the top level) and then Z; of the workgroup: the weights of "-" links
// by mode and n, the states of the modes
template <typename T>
size_t columns_wave_bytes(int N, int W, bool plus) {
    const size_t z = (size_t)N * kColStride * 2 * sizeof(T), n = plus ? (size_t)(64 / N) * W : 0;
    return 64 * 8 + ((std::max(z, n * (4 + sizeof(T))) + 15) & ~size_t(15));
}
template <typename T>
__host__ __device__ inline size_t columns_table_bytes(int W, int D) {
    return ((size_t)W * (D + 1) * 2 * sizeof(T) + (size_t)W * 4 + 15) & ~size_t(15);
}

// PLAIN: `in` is in the caller's order.
template <typename T, int N, bool PLUS, int NBASE, bool ZOUT, bool PLAIN>
__global__ __launch_bounds__(256) void k_columns(Job J, StageSpec sp, ColumnsStage<T> A, int tile_begin,
                                                 int tile_end, int s0_blocks, unsigned wave_bytes,
                                                 unsigned lds_total) {
    extern __shared__ __align__(16) char smem[];
    if constexpr (!PLUS) {
        if ((int)blockIdx.x < s0_blocks) {
            // the first workgroup carries the sigma_0 stage along
            sigma0_stage<T, false, false, false, PLAIN ? 0 : 64 / N>(J, nullptr, 0, sp, lds_total, smem);
            return;
        }
    }
    using C = typename vec2<T>::type;
    constexpr int NN = N * N, GA = 64 / N;
    const Tables& t = J.t;
    const int W = t.W, Dm = t.D, n_rest = t.n_ado - 1;
    const int wave = uniform((int)threadIdx.x >> 6), waves = (int)(blockDim.x >> 6);
    C* sTable = reinterpret_cast<C*>(smem);  // [W][D + 1]
    int* sSite = reinterpret_cast<int*>(sTable + W * (Dm + 1));
    char* mine = smem + columns_table_bytes<T>(W, Dm) + (size_t)wave * wave_bytes;
    pair_i* sLink = reinterpret_cast<pair_i*>(mine);  // (neighbour, weight | state << 16)
    C* Z = reinterpret_cast<C*>(sLink + 64);          // [N][kColStride], [row][lane]
    T* sPlusW = reinterpret_cast<T*>(sLink + 64);     // [GA][W]
    int* sPlus = reinterpret_cast<int*>(sPlusW + (PLUS ? GA * W : 0));
    gcptr<C> in = G(reinterpret_cast<const C*>(A.in));

    const int lane = threadIdx.x & 63;
    const int g = min(lane / N, GA - 1), c = min(lane - g * N, N - 1);
    // one wavefront's LDS accesses are in order; this keeps the compiler's
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    // H (symmetric) and Delta in scalar registers
    T H[N][N], delta[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int j = i; j < N; ++j) {
            T v;
            if constexpr (sizeof(T) == 4) v = G(t.h_re_f32)[i * N + j];
            else v = G(t.h_re)[i * N + j];
            H[i][j] = H[j][i] = uniform(v);
        }
        delta[i] = uniform((T)G(t.delta_state)[i]);
    }
    const T delta_c = (T)G(t.delta_state)[c];

    for (int x = threadIdx.x; x < W * (Dm + 1); x += blockDim.x) {
        const int l = x / (Dm + 1);
        const double m = G(t.minus_coef)[x];
        sTable[x] = C{(T)(m * G(t.mode_lamnu)[l]), (T)(m * G(t.mode_c)[l])};
    }
    for (int l = threadIdx.x; l < W; l += blockDim.x) sSite[l] = G(t.mode_site)[l];
    __syncthreads();

    // each XCD (workgroups go round them) walks a run of tiles of its own
    const int blocks = (int)gridDim.x - s0_blocks, block = (int)blockIdx.x - s0_blocks;
    const int nx = blocks >= 8 ? 8 : 1, xcd = block % nx, slots = blocks / nx + (xcd < blocks % nx);
    const int all = tile_end - tile_begin;
    const int share = all / nx, extra = all % nx;
    const int first_tile = tile_begin + xcd * share + min(xcd, extra);
    const int last_tile = first_tile + share + (xcd < extra);
    const int stride = slots * waves;
    int tl = first_tile + (block / nx) * waves + wave;
    tile_end = last_tile;
    if (tl >= tile_end) return;

    struct Links {
        int nb, code;
        T gam;
    };
    auto count_of = [&](int tile) { return min(GA, n_rest - tile * GA); };
    // element k of this lane's column: at k * step + off of the tile
    auto load = [&](const T* src, int tile, bool plain, C (&v)[N]) {
        const int n = count_of(tile), step = plain ? N : n * N;
        const int off = plain ? min(g, n - 1) * NN + c : min(lane, n * N - 1);
        gcptr<C> at = G(reinterpret_cast<const C*>(src)) + (size_t)tile * (GA * NN);
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = at[(uint32_t)(k * step + off)];
    };
    auto neighbour = [&](int u, int s) {
        return PLAIN ? in[(size_t)(u - 1) * NN + s * N + c] : in[tiled_at(GA, N, u, s, c, n_rest)];
    };
    // lane (g, c): link a0 + c of ADO g
    auto links = [&](int tile, int a0) {
        Links p;
        const int u = 1 + min(tile * GA + g, n_rest - 1);
        const size_t at = (size_t)u * Dm + min(a0 + c, Dm - 1);
        const pair_i v = G(reinterpret_cast<const pair_i*>(t.mlist))[at];
        p.nb = a0 + c < Dm ? v.x : -1;
        p.code = v.y;
        p.gam = (T)G(t.damping)[u];
        return p;
    };

    auto put_links = [&](const Links& p) {
        const int l = p.code & 255;
        sLink[lane] = p.nb < 0 ? pair_i{-1, 0} : pair_i{p.nb, (l * (Dm + 1) + (p.code >> 8)) | sSite[l] << 16};
    };

    // Read ahead by the top level.  Below it the "+" rows are the waits, and
    // registers are wavefronts (2.35 ms per stage with three per SIMD, 2.0 with
    // four, 1.8 with five, 1.6 with six).
    C next[N];
    Links lnext;
    if constexpr (!PLUS) {
        load(A.in, tl, PLAIN, next);
        lnext = links(tl, 0);
    }
    for (; tl < tile_end; tl += stride) {
        C x[N], z[N], bas[N];
        Links p;
        if constexpr (PLUS) {
            load(A.in, tl, PLAIN, x);
            p = links(tl, 0);
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k) x[k] = next[k];
            p = lnext;
        }
        const int n = count_of(tl), ahead = min(tl + stride, tile_end - 1);
        put_links(p);
        fence();
        // the rows of the first N links of each ADO
        C row[N];
        auto rows = [&](int a0) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const pair_i l = sLink[min(g * N + k, 63)];
                row[k] = C{0, 0};
                if (a0 + k < Dm) row[k] = neighbour(max(l.x, 1), l.y >> 16);
            }
        };
        if constexpr (!PLUS) {
            rows(0);
            if constexpr (NBASE > 0) load(A.base, tl, A.base_plain, bas);
        }
        // "+" links of the tile, in the order of the table
        if constexpr (PLUS) {
            const size_t first = (size_t)(1 + tl * GA) * W;
            for (int e = lane; e < n * W; e += 64) {
                sPlus[e] = G(t.plus)[first + e];
                sPlusW[e] = (T)G(t.plus_w)[first + e];
            }
            fence();
        }
        if constexpr (!PLUS) {
            load(A.in, ahead, PLAIN, next);
            lnext = links(ahead, 0);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            T yr = 0, yi = 0;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                yr += H[i][k] * x[k].x;
                yi += H[i][k] * x[k].y;
            }
            z[i] = C{yi, -yr};
        }
        if constexpr (PLUS) {
            // i w sigma_{u+e_l}[i][c], the modes of state i in turn; nothing on
            // the diagonal
            const int* pn = sPlus + min(g, n - 1) * W;
            const T* pw = sPlusW + min(g, n - 1) * W;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int begin = G(t.state_mode_begin)[i], end = G(t.state_mode_begin)[i + 1];
                for (int m = begin; m < end; m += 4) {
                    C y[4];
                    T w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int l = G(t.state_modes)[min(m + q, end - 1)];
                        const int nb = pn[l];
                        const bool on = m + q < end && nb >= 1 && i != c;
                        const T wl = pw[l];
                        w[q] = on ? wl : (T)0;
                        y[q] = neighbour(max(nb, 1), i);
                        if (!on) y[q] = C{0, 0};
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        z[i].x -= w[q] * y[q].y;
                        z[i].y += w[q] * y[q].x;
                    }
                }
            }
        }
        if constexpr (PLUS) {
            __builtin_amdgcn_sched_barrier(0);
            rows(0);
            fence();
        }
#pragma unroll
        for (int k = 0; k < N; ++k) Z[k * kColStride + lane] = z[k];
        for (int a0 = 0;;) {
            // neighbour 0 is sigma_0 (FP64): only the ADOs of the first level
            if (__any(p.nb == 0)) {
#pragma unroll 1
                for (int k = 0; k < N; ++k) {
                    const pair_i l = sLink[min(g * N + k, 63)];
                    if (l.x != 0) continue;
                    const int s = l.y >> 16;
                    const pair_d v = G(reinterpret_cast<const pair_d*>(J.sig0[sp.in]))[s * N + c];
                    const C w = sTable[l.y & 65535];
                    const T vr = (T)v.x, vi = (T)v.y, mc = s == c ? (T)0 : w.y;
                    C* at = Z + s * kColStride + lane;
                    *at = C{at->x + (w.x * vr - mc * vi), at->y + (w.x * vi + mc * vr)};
                }
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if (a0 + k >= Dm) break;
                const pair_i l = sLink[min(g * N + k, 63)];
                const int s = l.y >> 16;
                const C w = sTable[l.y & 65535];
                // (ml + i mc) x, the V^o part alone on the diagonal
                const T mc = s == c ? (T)0 : w.y;
                C* at = Z + s * kColStride + lane;
                if (l.x >= 1)
                    *at = C{at->x + (w.x * row[k].x - mc * row[k].y), at->y + (w.x * row[k].y + mc * row[k].x)};
            }
            a0 += N;
            if (a0 >= Dm) break;
            // more links than states: the next N
            const Links more = links(tl, a0);
            p.nb = more.nb;
            if (!__any(p.nb >= 0)) break;
            fence();
            put_links(more);
            fence();
            rows(a0);
        }
        if constexpr (PLUS) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NBASE > 0) load(A.base, tl, A.base_plain, bas);
        }
        fence();
        const int w = n * N;
        const size_t to = (size_t)tl * (GA * NN);
        const bool mine_out = lane < w;
        const int step = A.out_plain ? N : w, off = A.out_plain ? g * NN + c : lane;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            // w_in sigma + h (Z + Z^dagger - damping) and the stage's base
            const C zk = Z[k * kColStride + lane], zt = Z[c * kColStride + g * N + k];
            const T gm = p.gam + (k == c ? (T)0 : delta[k] + delta_c);
            C o;
            o.x = A.w_in * x[k].x + A.h * (zk.x + zt.x - gm * x[k].x);
            o.y = A.w_in * x[k].y + A.h * (zk.y - zt.y - gm * x[k].y);
            if constexpr (NBASE > 0) o += bas[k];
            if (mine_out) {
                G(reinterpret_cast<C*>(A.out))[to + (uint32_t)(k * step + off)] = o;
                // (-y + Y2 + 2 Y3)/3 by increments on 2/3 y
                if constexpr (ZOUT)
                    G(reinterpret_cast<C*>(A.z))[to + (uint32_t)(k * w + lane)] =
                        (T)(2.0 / 3.0) * bas[k] + (T)(1.0 / 3.0) * ((x[k] - bas[k]) + (T)2 * (o - bas[k]));
            }
        }
        fence();
    }
}

template <typename T, int N, bool PLUS, int NBASE, bool ZOUT, bool PLAIN>
hipError_t launch_part(const Job& J, const StageSpec& sp, const ColumnsStage<T>& A, int tile_begin, int tile_end,
                       hipStream_t stream) {
    const void* fn = reinterpret_cast<const void*>(&k_columns<T, N, PLUS, NBASE, ZOUT, PLAIN>);
    static std::once_flag once;
    static hipError_t err = hipSuccess;
    std::call_once(once, [&] {
        err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    if (err != hipSuccess) return err;
    const size_t wave = columns_wave_bytes<T>(N, J.t.W, PLUS);
    size_t lds = columns_table_bytes<T>(J.t.W, J.t.D) + 4 * wave;
    int extra = 0;
    if (!PLUS) {
        // sigma_0 next to the top level
        lds = std::max(lds, sigma0_lds(N, J.t.W, (int)sizeof(T), true, 40 * 1024).total);
        extra = 1;
    }
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, lds);
    if (e != hipSuccess) return e;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    int groups = std::min((tile_end - tile_begin + 3) / 4, cus * std::max(per_cu, 1));
    if (g_max_workgroups.load() > 0) groups = std::min(groups, g_max_workgroups.load());
    hipLaunchKernelGGL((k_columns<T, N, PLUS, NBASE, ZOUT, PLAIN>), dim3(extra + groups), dim3(256), lds, stream, J, sp, A,
                       tile_begin, tile_end, extra, (unsigned)wave, (unsigned)lds);
    return hipGetLastError();
}

template <typename T, int N, int NBASE, bool ZOUT, bool PLAIN>
hipError_t launch_n(const Job& J, const StageSpec& sp, const ColumnsStage<T>& A, hipStream_t stream) {
    // a tile that holds ADOs of the top level and below takes the "+" form
    const int GA = 64 / N, tiles = (J.t.n_ado - 1 + GA - 1) / GA, low = (J.n_low + GA - 1) / GA;
    if (low > 0) {
        hipError_t e = launch_part<T, N, true, NBASE, ZOUT, PLAIN>(J, sp, A, 0, low, stream);
        if (e != hipSuccess) return e;
    }
    return launch_part<T, N, false, NBASE, ZOUT, PLAIN>(J, sp, A, low, tiles, stream);
}

template <typename T, int N>
hipError_t stage_n(int k, const Job& J, void* z, bool first, bool last, const StageSpec& sp, hipStream_t stream) {
    // slots: y, Y2 and Y4, Y3 (Job::rest 0..3 the same)
    ColumnsStage<T> A{};
    A.in = static_cast<const T*>(J.rest[sp.in]);
    A.out = static_cast<T*>(J.rest[sp.out]);
    A.base = static_cast<const T*>(k == 3 ? z : J.rest[0]);
    A.z = static_cast<T*>(z);
    // w_in and the 2/3 of Z sum to exactly 1
    A.w_in = k == 0 ? (T)1 : k == 3 ? (T)1 - (T)(2.0 / 3.0) : (T)0;
    A.h = (T)(sp.hmul * J.dt);
    A.base_plain = first && k < 3;
    A.out_plain = last && k == 3;
    if (k == 0)
        return first ? launch_n<T, N, 0, false, true>(J, sp, A, stream) : launch_n<T, N, 0, false, false>(J, sp, A, stream);
    if (k == 1) return launch_n<T, N, 1, true, false>(J, sp, A, stream);
    return launch_n<T, N, 1, false, false>(J, sp, A, stream);
}

// f(N) for the compile-time N of the job
template <typename F>
hipError_t with_n(int N, F f) {
    switch (N) {
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool columns_eligible(const Job& J, int precision) {
    const Tables& t = J.t;
    if (precision == 2 || !J.herm || t.h_complex || t.N < 2 || t.N > 8 || t.D < 1 || t.n_ado < 2) return false;
    // two workgroups per CU; 16 bits name a weight
    if (t.W * (t.D + 1) > 65535) return false;
    const size_t lds = precision == 0
                           ? columns_table_bytes<double>(t.W, t.D) + 4 * columns_wave_bytes<double>(t.N, t.W, J.n_low > 0)
                           : columns_table_bytes<float>(t.W, t.D) + 4 * columns_wave_bytes<float>(t.N, t.W, J.n_low > 0);
    return lds <= 80 * 1024;
}

hipError_t columns_stage(int k, const Job& J, void* z, bool first, bool last, int precision, const StageSpec& sp,
                         hipStream_t stream) {
    return with_n(J.t.N, [&](auto n) {
        return precision == 0 ? stage_n<double, n>(k, J, z, first, last, sp, stream)
                              : stage_n<float, n>(k, J, z, first, last, sp, stream);
    });
}

}  // namespace heom
