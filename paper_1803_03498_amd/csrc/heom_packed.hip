// Propagation of Hermitian ADOs in packed form (real H; HEOM_FP32_MIXED and
// HEOM_FP32_HERM with 17 <= N <= 64, HEOM_FP64 with 10 <= N <= 48): eq. HEOM of the section
// "HEOM formalism" of Kramer et al., arXiv:1803.03498, fused with RK4.
//
// A Hermitian matrix is half redundant, and these runs are bound by the bytes
// of the ADO array.  Inside a propagation every ADO u >= 1 is kept as the real
// N x N array P, P[i][j] = Re sigma(i, j) for i <= j and Im sigma(j, i) for
// i > j (the storage of HEOM_FP32_HERM); complex states are packed before the
// first step and unpacked after the last (3 passes over the complex array per
// run).  A step moves 12 passes over P, half the bytes of the complex form
// each:
//   1: Y2 = y + dt/2 f(y)                                    read 1, write 1
//   2: Y3 = y + dt/2 f(Y2), Z = (-y + Y2 + 2 Y3)/3            read 2, write 2
//   3: Y4 = y + dt f(Y3)            (over Y2)                read 2, write 1
//   4: y' = Y4/3 + Z + dt/6 f(Y4)                            read 2, write 1
//
// One wavefront computes one ADO, with no barrier anywhere.  With sigma = A + iB
// (A symmetric, B antisymmetric) and U = H B, V = -H A
//   Re(-i[H, sigma]) = U + U^T,    Im(-i[H, sigma]) = V - V^T,
// 2 N^3 real multiplications per plane and no more.  U[i][j] is added where
// the lane's four rows i are contiguous (P[j][i]), then U[j][i] in place with
// the roles swapped, through the wavefront's LDS tile.  (Without that exchange,
// computing half the 16 x 16 tiles of H B - B H with operands taken from either
// side costs 4/3 as many products, and 48 sites took 1.05 to 1.35 ms per stage
// in FP32 and 2.35 to 2.81 in FP64, against 0.92 to 1.33 and 1.97 to 2.74; 24
// sites 57 to 63 us against 52 to 58.)
//
// Global accesses are linear (P as it lies in memory, 16 bytes per lane): the
// tile goes to this wavefront's own LDS tile, operands and results use that.
// (Operands straight from memory took 2.4 ms per stage at 48 sites: rows 16
// lanes apart do not coalesce, 2200 L1 accesses per plane.)  Lane (g, c) =
// (lane / 16, lane % 16) holds X[16K + 4g + r][16J + c], r = 0..3: the k index
// of a 16x16x4 product is permuted alike in both operands, so that r runs over
// four products, and an element stored transposed is one 16-byte LDS access
// for all r.  The output element (16I + 4g + r, 16J + c) belongs at [j][i],
// again 16 bytes.  (In FP64 the hardware's D rows are 4r + g; columns are
// permuted by the same map.)  The tile's stride 16 NB + 4 keeps both accesses
// free of bank conflicts and makes every offset a constant.
//
// H lies in LDS in operand order, one 16-byte access per block.  FP64 above 32
// states has no room for it next to the tiles of two wavefronts per SIMD, which
// cover each other's waits (one per SIMD: 2.35 ms): it reads the same table
// from memory (L1 and L2; from H itself, rows apart, 2.6 ms).
//
// "-" links ride along as one more product per four links: with E[i][a] =
// (i == s_a) and the weighted rows R_a, E R + (E R)^dagger: E Re R joins U and
// E Im R joins V.  The rows of the
// lower-level neighbours come from mirrors: real and imaginary planes, full
// N x N, of the ADOs below the top level (a few percent), written by every
// stage.  "+" links exist below the top level only; k_packed_plus sums them
// into the output slot of those ADOs first, and the stage adds that.  What it
// reads of a top-level ADO is the row of each of its links; every stage leaves
// those rows side by side ("side" rows), because a row of a Hermitian matrix
// is half a row and half a column of P (48 sites: 0.43 ms per stage without).
//
// Up to 32 states a wavefront's work on one ADO is short, and the chain of
// waits (links, then their rows, then the bases) bounds it: links, tile and
// bases are read ahead, and only as many groups of links are taken as an ADO
// has (14 sites, 237336 ADOs, FP64: 0.60 ms per stage without, 0.38 with; 24
// sites, 20475 ADOs, FP32: 61 and 58 us).
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

// A lane's piece of a P, at element alignment (rows of odd N start anywhere):
// 16 bytes.  32 bytes from lane to lane cost twice the cache and LDS cycles
// (FP64, 14 sites: 0.406 against 0.382 ms per stage).
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct Vec16<double> {
    typedef double type __attribute__((ext_vector_type(2), aligned(8)));
};

template <typename T>
struct PackedStage {
    const T* in;
    T* out;
    const T* base;  // y (stages 2, 3) or Z (stage 4)
    T* z;           // stage 2
    const T *mr_in, *mi_in;  // mirror planes of `in`, [n_low][N][N]
    T *mr_out, *mi_out;      // of `out`
    T* side_out;             // side rows of `out`, complex [top ADO][D][N], or null
    const T* hop;            // H in operand order where LDS has no room for it
    T w_in, h;
};

// Wavefronts per SIMD that registers and LDS allow; one workgroup per CU.
// One row block is FP64 only.
template <typename T, int NB>
constexpr int packed_waves() {
    return sizeof(T) == 4 ? (NB == 2 ? 4 : NB == 3 ? 3 : 2) : (NB == 1 ? 4 : 2);
}
template <typename T, int NB>
constexpr int packed_threads() {
    return 256 * packed_waves<T, NB>();
}
// k-steps of the last K block of `rem` columns (1..16): lane group g takes the
// columns kr g + r, r < kr, so that 8 columns need 2 products, not 4.
__host__ __device__ constexpr int packed_last_steps(int rem) { return (rem + 3) / 4; }
template <typename T, int NB>
constexpr bool packed_h_in_lds() {
    return sizeof(T) == 4 || NB < 3;
}
template <typename T, int NB>
constexpr int packed_stride() {
    return 16 * NB + (packed_h_in_lds<T, NB>() ? 4 : 2);
}
// LDS elements: H in operand order, Delta, one tile per wavefront
template <typename T, int NB>
constexpr size_t packed_lds() {
    return sizeof(T) * ((packed_h_in_lds<T, NB>() ? NB * NB * 256 : 0) + 16 * NB +
                        (size_t)(packed_threads<T, NB>() / 64) * 16 * NB * packed_stride<T, NB>());
}

// H as the A operand of block ik = I NB + K: lane (g, c) holds H[16I + jl][k],
// k = 16K + steps g + r; zero outside N x N, which meets whatever the tile's
// padding holds.
template <typename T>
__device__ __forceinline__ T h_operand(const Tables& t, int NB, int ik, int lane, int r) {
    const int N = t.N, I = ik / NB, K = ik - I * NB;
    const int c = lane & 15, g = lane >> 4, jl = sizeof(T) == 8 ? 4 * (c & 3) + (c >> 2) : c;
    const int steps = K < NB - 1 ? 4 : packed_last_steps(N - 16 * (NB - 1));
    const int row = 16 * I + jl, col = 16 * K + steps * g + r;
    if (r >= steps || row >= N || col >= N) return (T)0;
    if constexpr (sizeof(T) == 4) return G(t.h_re_f32)[row * N + col];
    else return G(t.h_re)[row * N + col];
}

// The same in memory, [block][r / 2][lane][2].
__global__ __launch_bounds__(256) void k_h_operand(Tables t, int NB, double* out) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= NB * NB * 256) return;
    G(out)[x] = h_operand<double>(t, NB, x >> 8, (x >> 1) & 63, 2 * ((x >> 7) & 1) + (x & 1));
}

template <typename T, int NB, bool VA, int NBASE, bool ZOUT>
__global__ __launch_bounds__((packed_threads<T, NB>())) __attribute__((
    amdgpu_waves_per_eu((packed_waves<T, NB>())))) void k_packed(Job J, StageSpec sp, PackedStage<T> A,
                                                                 int s0_blocks, unsigned lds_total) {
    extern __shared__ __align__(16) char smem[];
    if ((int)blockIdx.x < s0_blocks) {
        // the first workgroup carries the sigma_0 stage along
        sigma0_stage<T, false, false, true>(J, nullptr, 0, sp, lds_total, smem);
        return;
    }
    constexpr int PW = 16 / sizeof(T);
    using V = typename Vec16<T>::type;
    typedef T VP __attribute__((ext_vector_type(PW)));  // aligned, in LDS
    typedef T VL __attribute__((ext_vector_type(4)));
    using acc_t = typename mfma_acc<T>::type;
    constexpr int LS = packed_stride<T, NB>(), TILE = 16 * NB * LS;
    constexpr bool kHlds = packed_h_in_lds<T, NB>();
    const Tables& t = J.t;
    const int N = t.N, NN = N * N, Dm = t.D > 0 ? t.D : 1;
    T* sH = reinterpret_cast<T*>(smem);
    T* sDelta = sH + (kHlds ? NB * NB * 256 : 0);
    T* tiles = sDelta + 16 * NB;
    if constexpr (kHlds)
        for (int x = threadIdx.x; x < NB * NB * 256; x += blockDim.x)
            sH[x] = h_operand<T>(t, NB, x >> 8, (x >> 2) & 63, x & 3);
    for (int x = threadIdx.x; x < 16 * NB; x += blockDim.x) sDelta[x] = x < N ? (T)G(t.delta_state)[x] : (T)0;
    // the padding of a tile stays zero
    for (int x = threadIdx.x; x < (int)(blockDim.x / 64) * TILE; x += blockDim.x) tiles[x] = (T)0;
    __syncthreads();

    const int kr = packed_last_steps(N - 16 * (NB - 1));
    const int waves = blockDim.x / 64, wave = uniform((int)threadIdx.x >> 6);
    T* S = tiles + wave * TILE;
    const int first = 1 + ((int)blockIdx.x - s0_blocks) * waves + wave;
    const int stride = ((int)gridDim.x - s0_blocks) * waves;
    int lane = threadIdx.x & 63;

    // linear pieces of P: PW elements at PW (lane + 64 q), q < nq; beyond the
    // end the last ones once more (the same values from several lanes; the
    // loads are not conditional on q, which would keep undefined values live)
    constexpr int Q = NB * NB * 4 / PW;
    int nq = (NN + 64 * PW - 1) / (64 * PW);
    const uint32_t by_n = 0xFFFFFFFFu / (uint32_t)N + 1u;  // e / N = mulhi(e, by_n) for e < 2^16
    struct Pieces {
        V v[Q];
    };
    auto first_of = [&](int q) { return min(PW * (lane + 64 * q), NN - PW); };
    auto load = [&](const T* src, Pieces& p) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            p.v[q] = *reinterpret_cast<gcptr<V>>(G(reinterpret_cast<const char*>(src)) +
                                                     (uint32_t)first_of(q) * (uint32_t)sizeof(T));
    };
    auto store_piece = [&](T* dst, int q, V v) {
        *reinterpret_cast<gptr<V>>(G(reinterpret_cast<char*>(dst)) + (uint32_t)first_of(q) * (uint32_t)sizeof(T)) = v;
    };
    auto lds_at = [&](int e) { return S + (int)__umulhi((uint32_t)e, by_n) * (LS - N) + e; };
    // PW elements from e on: those within `left` in e's row, the rest in the next
    auto lds_row = [&](int e, T*& at, int& left) {
        const int i = (int)__umulhi((uint32_t)e, by_n);
        at = S + i * (LS - N) + e;
        left = N - (e - i * N);
    };
    auto piece_to_lds = [&](int q, V v) {
        if constexpr (VA) {
            *reinterpret_cast<VP*>(lds_at(first_of(q))) = v;
        } else {
            T* at;
            int left;
            lds_row(first_of(q), at, left);
#pragma unroll
            for (int r = 0; r < PW; ++r) at[r < left ? r : r + LS - N] = v[r];
        }
    };
    auto piece_from_lds = [&](int q) -> V {
        V v;
        if constexpr (VA) {
            v = *reinterpret_cast<const VP*>(lds_at(first_of(q)));
        } else {
            T* at;
            int left;
            lds_row(first_of(q), at, left);
#pragma unroll
            for (int r = 0; r < PW; ++r) v[r] = at[r < left ? r : r + LS - N];
        }
        return v;
    };
    // one wavefront's LDS accesses are in order; this keeps the compiler's
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    // the "-" links of an ADO, one per lane, read one ADO ahead, so that
    // rows and tile are a single wait apart
    struct Links {
        int nb, s;
        T ml, mc;
    };
    auto links = [&](int u) {
        Links l;
        const size_t at = (size_t)u * Dm + min(lane, Dm - 1);
        l.nb = G(reinterpret_cast<const pair_i*>(t.mlist))[at].x;
        l.s = G(t.mlist_site)[at];
        if constexpr (sizeof(T) == 4) {
            const pair_f w = G(reinterpret_cast<const pair_f*>(t.mlist_w32))[at];
            l.ml = w.x;
            l.mc = w.y;
        } else {
            const pair_d w = G(reinterpret_cast<const pair_d*>(t.mlist_w))[at];
            l.ml = w.x;
            l.mc = w.y;
        }
        return l;
    };
    // links 4q + g: their rows, columns 16 jb + jl
    struct Rows {
        int s;
        T ml, mc, re[NB], im[NB];
    };
    auto rows = [&](const Links& l, int count, int q) {
        const int c = lane & 15, g = lane >> 4, jl = sizeof(T) == 8 ? 4 * (c & 3) + (c >> 2) : c;
        const int a = 4 * q + g;
        Rows R;
        // every lane takes part: a lane left out would read as 0
        int nb = __shfl(l.nb, a);
        R.s = __shfl(l.s, a);
        R.ml = __shfl(l.ml, a);
        R.mc = __shfl(l.mc, a);
        if (a >= count) nb = -1;
        if (nb < 0) R.s = -1;
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) {
            const int col = min(16 * jb + jl, N - 1);
            R.re[jb] = R.im[jb] = (T)0;
            if (nb > 0) {
                const size_t o = (size_t)(nb - 1) * NN + R.s * N + col;
                R.re[jb] = G(A.mr_in)[o];
                R.im[jb] = G(A.mi_in)[o];
            } else if (nb == 0) {
                const cpx<double> v = ld<double>(J.sig0[sp.in], (size_t)R.s * N + col);
                R.re[jb] = (T)v.re;
                R.im[jb] = (T)v.im;
            }
        }
        return R;
    };

    // The next tile and this one's stage base are read ahead where the
    // registers allow; above 32 states the wavefronts of a SIMD (three in
    // FP32, two in FP64) cover the waits instead, and the bases are read when
    // the accumulators are done with.
    constexpr bool kAhead = NB <= 2;
    // one tile row: also this tile itself and the next four links' rows
    constexpr bool kRoom = NB == 1;
    Pieces pre;
    if constexpr (kAhead) load(A.in + (size_t)(min(first, t.n_ado - 1) - 1) * NN, pre);
    Links ahead = links(min(first, t.n_ado - 1));
    for (int u = first; u < t.n_ado; u += stride) {
        // through an empty asm: addresses and conditions hoisted out of the
        // loop would hold (and spill) a register each
        asm volatile("" : "+v"(lane), "+s"(nq));
        const int c = lane & 15, g = lane >> 4;
        // column (and operand row) of this lane inside a tile
        const int jl = sizeof(T) == 8 ? 4 * (c & 3) + (c >> 2) : c;
        const size_t tile = (size_t)(u - 1) * NN;
        Pieces bas, p;
        const T gam = (T)G(t.damping)[u];
        const Links own_links = ahead;
        // the active links come first
        const int count = __popcll(__ballot(lane < Dm && own_links.s >= 0));
        Rows ra, rb;
        {
            if constexpr (kAhead) p = pre;
            else load(A.in + tile, p);
            if constexpr (kHlds) ra = rows(own_links, count, 0);
            if constexpr (kRoom) rb = rows(own_links, count, 1);
            if constexpr (kAhead) {
                if constexpr (NBASE > 0) load(A.base + tile, bas);
                load(A.in + (size_t)(min(u + stride, t.n_ado - 1) - 1) * NN, pre);
            }
            if constexpr (kRoom) ahead = links(min(u + stride, t.n_ado - 1));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (q < nq) piece_to_lds(q, p.v[q]);
                if (!VA) __builtin_amdgcn_sched_barrier(0);  // four addresses per piece
            }
        }
        fence();
        // U = H B + E R_re and V = -H A + E R_im: the real part is U + U^T, the
        // imaginary one V - V^T
        acc_t accU[NB * NB], accV[NB * NB];
#pragma unroll
        for (int x = 0; x < NB * NB; ++x) accU[x] = accV[x] = acc_t{0, 0, 0, 0};
        auto product = [&](auto imag, acc_t(&W)[NB * NB]) {
#pragma unroll
            for (int K = 0; K < NB; ++K) {
                // the scheduler would otherwise load every K block's operands first
                __builtin_amdgcn_sched_barrier(0);
                const int steps = K < NB - 1 ? 4 : kr, k0 = steps * g;
                const T* Sd = S + (16 * K + k0) * LS + jl;  // direct: [k][jl]
                const T* St = S + jl * LS + 16 * K + k0;    // transposed: [jl][k]
                T X[NB][4], HR[NB][4];
#pragma unroll
                for (int jb = 0; jb < NB; ++jb) {
                    if constexpr (kHlds) {
                        const VL hv = *reinterpret_cast<const VL*>(sH + ((jb * NB + K) * 64 + lane) * 4);
#pragma unroll
                        for (int r = 0; r < 4; ++r) HR[jb][r] = hv[r];
                    } else {
                        // [block][r / PW][lane][PW]: 16 bytes from lane to lane
#pragma unroll
                        for (int r = 0; r < 4; r += PW) {
                            const V hv = *reinterpret_cast<gcptr<V>>(
                                G(A.hop) + (uint32_t)(((jb * NB + K) * 4 + r) * 64 + lane * PW));
#pragma unroll
                            for (int k = 0; k < PW; ++k) HR[jb][r + k] = hv[k];
                        }
                    }
                    // the element as stored, or its mirror
                    T d[4], tr[4];
                    if (K == jb || (imag ? K < jb : K > jb))
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[r] = Sd[r * LS + 16 * jb];
                    if (K == jb || (imag ? K > jb : K < jb)) {
                        if (K < NB - 1) {
                            const VL v = *reinterpret_cast<const VL*>(St + 16 * jb * LS);
#pragma unroll
                            for (int r = 0; r < 4; ++r) tr[r] = v[r];
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r) tr[r] = St[16 * jb * LS + r];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int k = k0 + r;
                        if (K == jb)
                            X[jb][r] = imag ? -(k < jl ? d[r] : tr[r]) : k < jl ? tr[r] : (k > jl ? -d[r] : (T)0);
                        else if (K < jb) X[jb][r] = imag ? -d[r] : tr[r];
                        else X[jb][r] = imag ? -tr[r] : -d[r];
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r >= steps) break;
#pragma unroll
                    for (int a = 0; a < NB; ++a)
#pragma unroll
                        for (int b = 0; b < NB; ++b) W[a * NB + b] = mfma16(HR[a][r], X[b][r], W[a * NB + b]);
                }
            }
        };
        product(std::false_type{}, accU);
        product(std::true_type{}, accV);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kHlds) ra = rows(own_links, count, 0);
        // the rows of four links at a time
        for (int q = 0;;) {
            T E[NB], xr[NB], xi[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                const bool at = 16 * jb + jl == ra.s;
                E[jb] = at ? (T)1 : (T)0;
                // (ml + i mc) x, the V^o part alone on the diagonal
                const T m = at ? (T)0 : ra.mc;
                xr[jb] = ra.ml * ra.re[jb] - m * ra.im[jb];
                xi[jb] = ra.ml * ra.im[jb] + m * ra.re[jb];
            }
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    accU[a * NB + b] = mfma16(E[a], xr[b], accU[a * NB + b]);
                    accV[a * NB + b] = mfma16(E[a], xi[b], accV[a * NB + b]);
                }
            if (4 * ++q >= count) break;
            if constexpr (kRoom) {
                ra = rb;
                rb = rows(own_links, count, q + 1);
            } else {
                ra = rows(own_links, count, q);
            }
        }
        const bool low = u <= J.n_low;
        Pieces plus;
        if constexpr (kRoom)
            if (low) load(A.out + tile, plus);
        if constexpr (!kRoom) ahead = links(min(u + stride, t.n_ado - 1));
        // w_in sigma + h (f - damping) at [j][i], in place of sigma
        fence();
#pragma unroll
        for (int rb = 0; rb < NB; ++rb)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) {
                if (cb == 0) __builtin_amdgcn_sched_barrier(0);
                const int x = cb * NB + rb;  // U, accV[i][j]
                const int j = 16 * rb + jl, i0 = 16 * cb + 4 * g;
                T* at = S + (16 * rb + jl) * LS + 16 * cb + 4 * g;
                const VL s = *reinterpret_cast<const VL*>(at);
                const VL di = *reinterpret_cast<const VL*>(sDelta + i0);
                const T dj = sDelta[j];
                VL o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    T f, gm = gam + di[r] + dj;
                    if (cb > rb) f = accU[x][r];
                    else if (cb < rb) f = accV[x][r];
                    else {
                        f = 4 * g + r >= jl ? accU[x][r] : accV[x][r];
                        if (4 * g + r == jl) gm = gam;
                    }
                    o[r] = A.w_in * s[r] + A.h * (f - gm * s[r]);
                }
                if (cb < NB - 1) {
                    if (j < N) *reinterpret_cast<VL*>(at) = o;
                } else if (VA) {
#pragma unroll
                    for (int r = 0; r < 4; r += PW)
                        if (j < N && i0 + r < N) {
                            VP part;
#pragma unroll
                            for (int k = 0; k < PW; ++k) part[k] = o[r + k];
                            *reinterpret_cast<VP*>(at + r) = part;
                        }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (j < N && i0 + r < N) at[r] = o[r];
                }
            }
        fence();
        // the transposed halves, at [i][j]: U below P's diagonal's row, -V past it
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            __builtin_amdgcn_sched_barrier(0);
            T w[NB][4];
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) w[cb][r] = S[(16 * rb + 4 * g + r) * LS + 16 * cb + jl];
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int x = rb * NB + cb;
                    T f = cb > rb ? accU[x][r] : -accV[x][r];
                    if (cb == rb && jl >= 4 * g + r) f = accU[x][r];
                    const bool inside = (rb < NB - 1 || 16 * rb + 4 * g + r < N) && (cb < NB - 1 || 16 * cb + jl < N);
                    S[(16 * rb + 4 * g + r) * LS + 16 * cb + jl] = inside ? w[cb][r] + A.h * f : (T)0;
                }
        }
        fence();
        // linear again: the bases, and what the next stages need (the pieces'
        // offsets computed anew: kept since the loads they spill)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(lane));
        if constexpr (!kAhead && NBASE > 0) load(A.base + tile, bas);
        if constexpr (ZOUT && !kRoom) load(A.in + tile, p);
        const bool again = low || A.side_out;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= nq) continue;
            V o = piece_from_lds(q);
            if (low) {
                if constexpr (!kRoom)
                    plus.v[q] = *reinterpret_cast<gcptr<V>>(G(reinterpret_cast<const char*>(A.out + tile)) +
                                                            (uint32_t)first_of(q) * (uint32_t)sizeof(T));
                o += A.h * plus.v[q];
            }
            if constexpr (NBASE > 0) o += bas.v[q];
            store_piece(A.out + tile, q, o);
            // (-y + Y2 + 2 Y3)/3 by increments on 2/3 y
            if constexpr (ZOUT)
                store_piece(A.z + tile, q,
                            (T)(2.0 / 3.0) * bas.v[q] +
                                (T)(1.0 / 3.0) * ((p.v[q] - bas.v[q]) + (T)2 * (o - bas.v[q])));
            if (again) piece_to_lds(q, o);
            if (!VA) __builtin_amdgcn_sched_barrier(0);
        }
        if (again) {
            fence();
            if (low) {
                // full planes for the next stage's "-" rows
                for (int e = lane; e < NN; e += 64) {
                    const int i = (int)__umulhi((uint32_t)e, by_n), j = e - i * N;
                    const T up = S[min(i, j) * LS + max(i, j)], lo = S[max(i, j) * LS + min(i, j)];
                    G(A.mr_out)[tile + e] = up;
                    G(A.mi_out)[tile + e] = i < j ? lo : (i > j ? -lo : (T)0);
                }
            } else {
                // the rows that lower levels read of this ADO
                for (int x0 = 0; x0 < count * N; x0 += 64) {
                    const int x = x0 + lane, a = (int)__umulhi((uint32_t)x, by_n), j = x - a * N;
                    const int s = __shfl(own_links.s, a);  // by every lane
                    if (x >= count * N) continue;
                    const T up = S[min(s, j) * LS + max(s, j)], lo = S[max(s, j) * LS + min(s, j)];
                    st<T>(A.side_out, (size_t)(u - 1 - J.n_low) * Dm * N + x,
                          cpx<T>{up, s < j ? lo : (s > j ? -lo : (T)0)});
                }
            }
            fence();
        }
    }
}

// "+" sums of the ADOs 1..n_low (one per workgroup) into F, in P form: with
// S_i[j] = sum over the modes l of state i of w_l sigma_{u+e_l}[i][j],
// i(S_i[j] - conj S_j[i]): Re -(Im S_i[j] + Im S_j[i]), Im Re S_i[j] - Re S_j[i].
template <typename T>
__global__ __launch_bounds__(256) void k_packed_plus(Tables t, int n_low, const T* in, const T* mr, const T* mi,
                                                     const T* side, T* F) {
    extern __shared__ __align__(16) char smem[];
    const int N = t.N, NN = N * N, W = t.W, LS = N + 1;
    T* sA = reinterpret_cast<T*>(smem);
    T* sB = sA + N * LS;
    // per mode, in the order of the states: weight, neighbour, side row
    T* sW = sB + N * LS;
    int* sNb = reinterpret_cast<int*>(sW + W);
    int* sRow = sNb + W;
    int* sBegin = sRow + W;
    const int u = 1 + blockIdx.x, Dm = t.D;
    for (int m = threadIdx.x; m < W; m += 256) {
        const int l = G(t.state_modes)[m], nb = G(t.plus)[(size_t)u * W + l];
        // the link's place among those of u + e_l: the active modes of u before l
        int k = 0;
        for (int a = 0; a < Dm; ++a) {
            const pair_i v = G(reinterpret_cast<const pair_i*>(t.mlist))[(size_t)u * Dm + a];
            k += v.x >= 0 && (v.y & 255) < l;
        }
        sW[m] = (T)G(t.plus_w)[(size_t)u * W + l];
        sNb[m] = nb;
        sRow[m] = (nb - 1 - n_low) * Dm + k;
    }
    for (int x = threadIdx.x; x <= N; x += 256) sBegin[x] = G(t.state_mode_begin)[x];
    __syncthreads();
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N, j = e - i * N;
        T re = 0, im = 0;
#pragma unroll 2
        for (int m = sBegin[i]; m < sBegin[i + 1]; ++m) {
            const T w = sW[m];
            const int nb = sNb[m];
            const size_t at = (size_t)(nb - 1) * NN;
            if (nb <= n_low) {
                re += w * G(mr)[at + e];
                im += w * G(mi)[at + e];
            } else if (side) {
                const cpx<T> v = ld<T>(side, (size_t)sRow[m] * N + j);
                re += w * v.re;
                im += w * v.im;
            } else {
                const T up = G(in)[at + min(i, j) * N + max(i, j)], lo = G(in)[at + max(i, j) * N + min(i, j)];
                re += w * up;
                im += w * (i < j ? lo : -lo);
            }
        }
        sA[i * LS + j] = re;
        sB[i * LS + j] = im;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N, j = e - i * N;
        T f = (T)0;
        if (i < j) f = -(sB[i * LS + j] + sB[j * LS + i]);
        else if (i > j) f = sA[j * LS + i] - sA[i * LS + j];  // Im of (j, i)
        G(F)[(size_t)(u - 1) * NN + e] = f;
    }
}

// Complex ADOs <-> P, one ADO per workgroup; packing also fills the mirror
// planes of the ADOs 1..n_low and the side rows (if any) of the others.
template <typename T>
__global__ __launch_bounds__(256) void k_pack(Tables t, const void* rest, T* P, T* mr, T* mi, T* side, int n_low) {
    extern __shared__ __align__(16) char smem[];
    T* s = reinterpret_cast<T*>(smem);  // [N][N + 1]
    const int N = t.N, NN = N * N;
    const size_t at = (size_t)blockIdx.x * NN;
    const bool low = (int)blockIdx.x < n_low;
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N, j = e - i * N;
        if (j < i) continue;
        const cpx<T> v = ld<T>(rest, at + e);
        s[i * (N + 1) + j] = v.re;
        if (j > i) s[j * (N + 1) + i] = v.im;
        if (low) {
            const T im = j > i ? v.im : (T)0;
            G(mr)[at + e] = G(mr)[at + j * N + i] = v.re;
            G(mi)[at + e] = im;
            if (j > i) G(mi)[at + j * N + i] = -im;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N;
        G(P)[at + e] = s[i * (N + 1) + e - i * N];
    }
    if (low || !side) return;
    const int Dm = t.D;
    for (int x = threadIdx.x; x < Dm * N; x += 256) {
        const int a = x / N, j = x - a * N;
        const int r = G(t.mlist_site)[(size_t)(1 + blockIdx.x) * Dm + a];
        if (r < 0) continue;
        const T up = s[min(r, j) * (N + 1) + max(r, j)], lo = s[max(r, j) * (N + 1) + min(r, j)];
        st<T>(side, ((size_t)((int)blockIdx.x - n_low) * Dm + a) * N + j,
              cpx<T>{up, r < j ? lo : (r > j ? -lo : (T)0)});
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_unpack(const T* P, void* rest, int N) {
    extern __shared__ __align__(16) char smem[];
    T* s = reinterpret_cast<T*>(smem);
    const int NN = N * N;
    const size_t at = (size_t)blockIdx.x * NN;
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N;
        s[i * (N + 1) + e - i * N] = G(P)[at + e];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N, j = e - i * N;
        const T re = s[min(i, j) * (N + 1) + max(i, j)], lo = s[max(i, j) * (N + 1) + min(i, j)];
        st<T>(rest, at + e, cpx<T>{re, i < j ? lo : (i > j ? -lo : (T)0)});
    }
}

// Mirror planes of the packed ADOs 1..n_low.
template <typename T>
__global__ __launch_bounds__(256) void k_mirror(const T* P, T* mr, T* mi, int N) {
    const int NN = N * N;
    const size_t at = (size_t)blockIdx.x * NN;
    for (int e = threadIdx.x; e < NN; e += 256) {
        const int i = e / N, j = e - i * N;
        const T up = G(P)[at + min(i, j) * N + max(i, j)], lo = G(P)[at + max(i, j) * N + min(i, j)];
        G(mr)[at + e] = up;
        G(mi)[at + e] = i < j ? lo : (i > j ? -lo : (T)0);
    }
}

hipError_t full_lds(std::once_flag& once, hipError_t& err, const void* fn) {
    std::call_once(once, [&] {
        err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    return err;
}

template <typename T, int NB, bool VA, int NBASE, bool ZOUT>
hipError_t launch_t(const Job& J, const StageSpec& sp, const PackedStage<T>& A, hipStream_t stream) {
    const void* fn = reinterpret_cast<const void*>(&k_packed<T, NB, VA, NBASE, ZOUT>);
    static std::once_flag once;
    static hipError_t err = hipSuccess;
    if (full_lds(once, err, fn) != hipSuccess) return err;
    constexpr int threads = packed_threads<T, NB>(), waves = threads / 64;
    const int n = J.t.n_ado - 1, N = J.t.N;
    // one workgroup per CU; sigma_0 rides along on a CU of its own when its
    // LDS fits (its rows only if they do)
    size_t lds = packed_lds<T, NB>();
    constexpr size_t budget = 160 * 1024;
    const size_t full = sigma0_lds(N, J.t.W, (int)sizeof(T), true, budget).total;
    const size_t bare = sigma0_lds(N, J.t.W, (int)sizeof(T), true, 0).total;
    int extra = 0;
    hipError_t e;
    if (bare <= budget) {
        lds = std::max(lds, full <= budget ? full : bare);
        extra = 1;
    } else if ((e = launch_sigma0_packed(J, (int)sizeof(T), sp, stream)) != hipSuccess) {
        return e;
    }
    int cus = 256, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 2)
        cus = 256;
    int groups = std::min((n + waves - 1) / waves, cus - extra);
    if (g_max_workgroups.load() > 0) groups = std::min(groups, g_max_workgroups.load());
    hipLaunchKernelGGL((k_packed<T, NB, VA, NBASE, ZOUT>), dim3(extra + groups), dim3(threads), lds, stream, J, sp, A,
                       extra, (unsigned)lds);
    return hipGetLastError();
}

template <typename T, int NB, bool VA>
hipError_t launch_k(int k, const Job& J, const StageSpec& sp, const PackedStage<T>& A, hipStream_t stream) {
    if (k == 0) return launch_t<T, NB, VA, 0, false>(J, sp, A, stream);
    if (k == 1) return launch_t<T, NB, VA, 1, true>(J, sp, A, stream);
    return launch_t<T, NB, VA, 1, false>(J, sp, A, stream);
}

template <typename T>
hipError_t launch_nb(int k, const Job& J, const StageSpec& sp, const PackedStage<T>& A, hipStream_t stream) {
    const bool va = J.t.N % (16 / sizeof(T)) == 0;  // pieces do not cross rows
    switch ((J.t.N + 15) / 16) {
        case 1:
            if constexpr (sizeof(T) == 8)
                return va ? launch_k<T, 1, true>(k, J, sp, A, stream) : launch_k<T, 1, false>(k, J, sp, A, stream);
            return hipErrorInvalidValue;
        case 2: return va ? launch_k<T, 2, true>(k, J, sp, A, stream) : launch_k<T, 2, false>(k, J, sp, A, stream);
        case 3: return va ? launch_k<T, 3, true>(k, J, sp, A, stream) : launch_k<T, 3, false>(k, J, sp, A, stream);
        case 4:
            // FP64 tiles of four wavefronts exceed a CU's LDS
            if constexpr (sizeof(T) == 4)
                return va ? launch_k<T, 4, true>(k, J, sp, A, stream) : launch_k<T, 4, false>(k, J, sp, A, stream);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t stage(int k, const Job& J, const PackedRun& R, const StageSpec& sp, hipStream_t stream) {
    const int N = J.t.N;
    // slot of the bulk arrays: y, Y2 and Y4, Y3 (Job::rest 0..3 the same)
    T* y = static_cast<T*>(J.rest[0]);
    T* a = static_cast<T*>(J.rest[1]);
    T* b = static_cast<T*>(J.rest[2]);
    T* z = static_cast<T*>(R.z);
    PackedStage<T> A{};
    A.in = k == 0 ? y : k == 2 ? b : a;
    A.out = k == 1 ? b : k == 3 ? y : a;
    A.base = k == 3 ? z : y;
    A.z = z;
    A.hop = static_cast<const T*>(R.h);
    const size_t plane = (size_t)J.n_low * N * N;
    T* m[2] = {static_cast<T*>(R.mirror[0]), static_cast<T*>(R.mirror[1])};
    A.mr_in = m[k & 1];
    A.mi_in = m[k & 1] + plane;
    A.mr_out = m[1 - (k & 1)];
    A.mi_out = m[1 - (k & 1)] + plane;
    const T* side_in = static_cast<const T*>(R.side[k & 1]);
    A.side_out = static_cast<T*>(R.side[1 - (k & 1)]);
    // w_in and the 2/3 of Z sum to exactly 1
    A.w_in = k == 0 ? (T)1 : k == 3 ? (T)1 - (T)(2.0 / 3.0) : (T)0;
    A.h = (T)(sp.hmul * J.dt);
    if (J.n_low > 0) {
        static std::once_flag once;
        static hipError_t err = hipSuccess;
        if (full_lds(once, err, reinterpret_cast<const void*>(&k_packed_plus<T>)) != hipSuccess) return err;
        hipLaunchKernelGGL((k_packed_plus<T>), dim3(J.n_low), dim3(256),
                           2 * N * (N + 1) * sizeof(T) + J.t.W * (sizeof(T) + 8) + (N + 1) * 4, stream, J.t, J.n_low,
                           A.in, A.mr_in, A.mi_in, side_in, A.out);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_nb<T>(k, J, sp, A, stream);
}

template <typename T>
hipError_t begin(const Job& J, const PackedRun& R, hipStream_t stream) {
    const int N = J.t.N, n = J.t.n_ado - 1;
    T* mr = static_cast<T*>(R.mirror[0]);
    T* mi = mr + (size_t)J.n_low * N * N;
    if (R.h) {
        const int NB = (N + 15) / 16;
        hipLaunchKernelGGL(k_h_operand, dim3(NB * NB), dim3(256), 0, stream, J.t, NB, static_cast<double*>(R.h));
    }
    if (R.complex_rest)
        hipLaunchKernelGGL((k_pack<T>), dim3(n), dim3(256), N * (N + 1) * sizeof(T), stream, J.t, R.complex_rest,
                           static_cast<T*>(J.rest[0]), mr, mi, static_cast<T*>(R.side[0]), J.n_low);
    else if (J.n_low > 0)
        hipLaunchKernelGGL((k_mirror<T>), dim3(J.n_low), dim3(256), 0, stream, static_cast<const T*>(J.rest[0]), mr,
                           mi, N);
    return hipGetLastError();
}

}  // namespace

// Single jobs over Hermitian ADOs with a real H whose workspace holds the
// packed arrays.  Small matrices pay for padding and for side rows, which do
// not halve: in FP64 10 states still gain (53130 ADOs: 0.38 ms per step against
// 0.41 with the complex kernels; 14 states, 237336 ADOs: 2.1 against 3.2), in
// FP32 up to 16 they do not (16 states, 74613 ADOs: 0.52 against 0.52; 10
// states, 230230 ADOs: 1.22 against 1.11).  A wavefront holds the links of an
// ADO, so at most 64 of them.
bool packed_plan(const Job& J, int precision, size_t sigma0_bytes, size_t work_bytes, size_t offset, PackedLayout* L) {
    const Tables& t = J.t;
    const int64_t n = t.n_ado - 1;
    if (!J.herm || t.h_complex || t.N < (precision == 0 ? 10 : 17) || t.N > (precision == 0 ? 48 : 64) || n < 1 || t.D > 64)
        return false;
    const size_t ts = precision == 0 ? 8 : 4, NN = (size_t)t.N * t.N;
    auto align256 = [](size_t x) { return (x + 255) & ~size_t(255); };
    *L = PackedLayout{};
    size_t o = offset;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align256(std::max<size_t>(bytes, 1));
        return at;
    };
    for (int k = 0; k < 3; ++k) L->sig0[k] = take(sigma0_bytes);
    for (int k = 0; k < 3; ++k) L->array[k] = take((size_t)n * NN * ts);
    for (int k = 0; k < 2; ++k) L->mirror[k] = take(2 * (size_t)J.n_low * NN * ts);
    if (precision != 2) L->y = take((size_t)n * NN * ts);
    if (precision == 0 && t.N > 32) L->h = take(9 * 256 * ts);
    if (o > work_bytes) return false;
    // side rows where they fit too (a packed state leaves no room for them)
    if (precision != 2 && J.n_low > 0 && (n - J.n_low) * t.D < (int64_t(1) << 31)) {
        for (int k = 0; k < 2; ++k) L->side[k] = take(2 * (size_t)(n - J.n_low) * t.D * t.N * ts);
        if (o > work_bytes) L->side[0] = L->side[1] = 0;
    }
    return true;
}

hipError_t packed_begin(const Job& J, const PackedRun& R, int precision, hipStream_t stream) {
    return precision == 0 ? begin<double>(J, R, stream) : begin<float>(J, R, stream);
}

hipError_t packed_stage(int k, const Job& J, const PackedRun& R, int precision, const StageSpec& sp,
                        hipStream_t stream) {
    return precision == 0 ? stage<double>(k, J, R, sp, stream) : stage<float>(k, J, R, sp, stream);
}

hipError_t packed_end(const Job& J, const PackedRun& R, int precision, hipStream_t stream) {
    if (!R.complex_rest) return hipSuccess;
    const int N = J.t.N, n = J.t.n_ado - 1;
    if (precision == 0)
        hipLaunchKernelGGL((k_unpack<double>), dim3(n), dim3(256), N * (N + 1) * 8, stream,
                           static_cast<const double*>(J.rest[0]), R.complex_rest, N);
    else
        hipLaunchKernelGGL((k_unpack<float>), dim3(n), dim3(256), N * (N + 1) * 4, stream,
                           static_cast<const float*>(J.rest[0]), R.complex_rest, N);
    return hipGetLastError();
}

}  // namespace heom
