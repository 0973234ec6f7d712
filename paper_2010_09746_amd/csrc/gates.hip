// Plain-form kernels: one launch per gate (paper, Section 2: gates update
// amplitudes in pairs), the in-place data movement of PermuteQubits and state
// preparation.
//
// Every kernel is bound by HBM traffic.  Threads take consecutive pair indices,
// so for a target position t >= log2(64) a wavefront reads two contiguous
// 64-amplitude runs; for lower t the pairs interleave inside the same cache
// lines and both halves of each line are consumed by the same wavefront.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.cuh"
#include "kernels.h"

namespace qsim {

namespace {

// Amplitude access: non-temporal when every 128-byte line a launch touches is
// read or written whole by one instruction (no qubit below the line size is
// split across instructions), cached otherwise, where the two halves of a line
// arrive from different instructions and the cache merges them.
template <bool NTA, typename C> __device__ __forceinline__ C ld(const C *p)
{
    if constexpr (NTA)
        return ld_stream(p);
    else
        return *p;
}
template <bool NTA, typename C> __device__ __forceinline__ void st(C *p, const C &v)
{
    if constexpr (NTA)
        st_stream(p, v);
    else
        *p = v;
}


constexpr int NT = 256;   // threads per block
constexpr int UNR = 4;    // pairs per thread, loads issued before use

__device__ __forceinline__ uint64_t insert_zero(uint64_t x, int b)
{
    const uint64_t lo = x & ((1ull << b) - 1);
    return ((x >> b) << (b + 1)) | lo;
}

template <typename R>
__global__ __launch_bounds__(NT) void k_set_basis(typename Cx<R>::T *s, uint64_t N, uint64_t x)
{
    using C = typename Cx<R>::T;
    // grid-stride over chunks of NT * UNR items (a launch is capped below 2^31 threads)
    for (uint64_t chunk = (uint64_t)blockIdx.x * NT * UNR; chunk < N; chunk += (uint64_t)gridDim.x * NT * UNR) {
        const uint64_t i0 = chunk + threadIdx.x;
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t i = i0 + (uint64_t)u * NT;
            if (i < N) {
                C v;
                v.x = i == x ? R(1) : R(0);
                v.y = R(0);
                st_stream(&s[i], v);
            }
        }
    }
}

// (a_i, a_j) <- U (a_i, a_j) for j = i | 2^t, optionally only where bit c = 1.
template <typename R, bool CTRL, bool NTA>
__global__ __launch_bounds__(NT) void k_pair_u(typename Cx<R>::T *__restrict__ s, uint64_t npairs,
                                               int t, int c_lo, int c_hi, uint64_t cbit, Mat<R> m)
{
    using C = typename Cx<R>::T;
    // grid-stride over chunks of NT * UNR items (a launch is capped below 2^31 threads)
    for (uint64_t chunk = (uint64_t)blockIdx.x * NT * UNR; chunk < npairs; chunk += (uint64_t)gridDim.x * NT * UNR) {
        const uint64_t p0 = chunk + threadIdx.x;
        C a[UNR], b[UNR];
        uint64_t ii[UNR];
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            uint64_t i;
            if (CTRL)
                i = insert_zero(insert_zero(p, c_lo), c_hi) | cbit;
            else
                i = insert_zero(p, t);
            ii[u] = i;
            if (p < npairs) {
                a[u] = ld<NTA>(&s[i]);
                b[u] = ld<NTA>(&s[i | (1ull << t)]);
            }
        }
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            if (p < npairs) {
                C x = a[u], y = b[u];
                st<NTA>(&s[ii[u]], m.row0(x, y));
                st<NTA>(&s[ii[u] | (1ull << t)], m.row1(x, y));
            }
        }
    }
}

// controlled X: exchange a_i and a_j where bit c = 1
template <typename R, bool NTA>
__global__ __launch_bounds__(NT) void k_cx(typename Cx<R>::T *__restrict__ s, uint64_t nquads, int t,
                                           int lo, int hi, uint64_t cbit)
{
    using C = typename Cx<R>::T;
    // grid-stride over chunks of NT * UNR items (a launch is capped below 2^31 threads)
    for (uint64_t chunk = (uint64_t)blockIdx.x * NT * UNR; chunk < nquads; chunk += (uint64_t)gridDim.x * NT * UNR) {
        const uint64_t p0 = chunk + threadIdx.x;
        C a[UNR], b[UNR];
        uint64_t ii[UNR];
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            ii[u] = insert_zero(insert_zero(p, lo), hi) | cbit;
            if (p < nquads) {
                a[u] = ld<NTA>(&s[ii[u]]);
                b[u] = ld<NTA>(&s[ii[u] | (1ull << t)]);
            }
        }
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            if (p < nquads) {
                st<NTA>(&s[ii[u]], b[u]);
                st<NTA>(&s[ii[u] | (1ull << t)], a[u]);
            }
        }
    }
}

// controlled Z: negate a_i where both bits are 1
template <typename R, bool NTA>
__global__ __launch_bounds__(NT) void k_cz(typename Cx<R>::T *__restrict__ s, uint64_t nquads, int lo,
                                           int hi, uint64_t both)
{
    using C = typename Cx<R>::T;
    // grid-stride over chunks of NT * UNR items (a launch is capped below 2^31 threads)
    for (uint64_t chunk = (uint64_t)blockIdx.x * NT * UNR; chunk < nquads; chunk += (uint64_t)gridDim.x * NT * UNR) {
        const uint64_t p0 = chunk + threadIdx.x;
        C a[UNR];
        uint64_t ii[UNR];
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            ii[u] = insert_zero(insert_zero(p, lo), hi) | both;
            if (p < nquads)
                a[u] = ld<NTA>(&s[ii[u]]);
        }
    #pragma unroll
        for (int u = 0; u < UNR; ++u) {
            uint64_t p = p0 + (uint64_t)u * NT;
            if (p < nquads) {
                C v = a[u];
                v.x = -v.x;
                v.y = -v.y;
                st<NTA>(&s[ii[u]], v);
            }
        }
    }
}

// In-place involution of the index: amplitude x and amplitude J(x) change
// places, where J moves bit p of the index to bit pi[p] and pi[pi[p]] = p.
//
// A tile is the set of amplitudes that share the index bits outside K
// positions closed under pi: the positions inside a 128-byte line, their
// partners, and more pairs and fixed positions up to 2^11 (complex128) or 2^12
// (complex64) amplitudes.  J maps a tile onto a tile, with the index inside it
// permuted, so one workgroup loads a tile and its partner, permutes each
// through LDS and stores it in the other's place.  Every access moves whole
// lines at any pi, and the launch is bound by HBM.  qs_permute_qubits at 29
// qubits: a random placement (two launches) 15.3 -> 7.5 ms complex128 (4.6
// TB/s) and 7.8 -> 4.1 ms complex64, a rotation 23.6 -> 8.9 ms, the reversal
// (one launch; three tile passes before) 10.4 -> 5.3 ms.  Before, one thread
// exchanged one pair wherever its two ends lay, so that a moved line position
// split every line.
struct Involution {
    int K, n_pairs;              // tile bits; exchanged pairs of positions outside the tile
    int inner;                   // the tile's own index is permuted
    uint8_t pos[16], perm[16];   // tile bit b is position pos[b] (ascending), moves to tile bit perm[b]
    uint8_t lo[MAX_QUBITS / 2], hi[MAX_QUBITS / 2];  // those pairs
};

template <typename R> constexpr int INV_BITS = sizeof(R) == 8 ? 11 : 12;  // 32 KiB of LDS

template <typename R> __global__ __launch_bounds__(NT) void k_involution(Cplx<R> *__restrict__ s, Involution J)
{
    using C = Cplx<R>;
    constexpr int NE = (1 << INV_BITS<R>) / NT;
    __shared__ C tile[1 << INV_BITS<R>];
    // the tile's base index, and its partner's (constant bounds: the positions
    // come in a few wide scalar loads, not one at a time)
    uint64_t base = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
#pragma unroll
    for (int b = 0; b < INV_BITS<R>; ++b)
        if (b < J.K)
            base = insert_zero(base, J.pos[b]);
    uint64_t part = base;
#pragma unroll
    for (int k = 0; k < MAX_QUBITS / 2; ++k)
        if (k < J.n_pairs) {
            const uint64_t d = ((base >> J.lo[k]) ^ (base >> J.hi[k])) & 1ull;
            part ^= (d << J.lo[k]) | (d << J.hi[k]);
        }
    if (part < base || (part == base && !J.inner))
        return;  // the partner's workgroup does both, or nothing moves
    const uint32_t tid = threadIdx.x, size = 1u << J.K;
    uint64_t off = 0;   // this thread's part of the index
    uint32_t to = 0;    // where it goes inside the tile
#pragma unroll
    for (int b = 0; b < 8; ++b) {  // threads beyond a smaller tile take no part
        off |= (uint64_t)((tid >> b) & 1u) << J.pos[b];
        to |= ((tid >> b) & 1u) << J.perm[b];
    }
    uint64_t so[NE];
    uint32_t sto[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        so[j] = 0;
        sto[j] = 0;
#pragma unroll
        for (int i = 0; (1 << i) < NE; ++i)
            if ((j >> i) & 1) {
                so[j] |= 1ull << J.pos[8 + i];
                sto[j] |= 1u << J.perm[8 + i];
            }
    }
    auto mine = [&](int j) { return (uint32_t)j * NT + tid < size; };
    const bool two = part != base;
    C va[NE], vb[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j)
        if (mine(j))
            va[j] = ld_stream(&s[base + (off | so[j])]);
    if (two) {
#pragma unroll
        for (int j = 0; j < NE; ++j)
            if (mine(j))
                vb[j] = ld_stream(&s[part + (off | so[j])]);
    }
    auto permute = [&](C(&v)[NE]) {
#pragma unroll
        for (int j = 0; j < NE; ++j)
            if (mine(j))
                tile[lds_swizzle(to | sto[j], J.K)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NE; ++j)
            if (mine(j))
                v[j] = tile[lds_swizzle((uint32_t)j * NT + tid, J.K)];
    };
    if (J.inner)
        permute(va);
#pragma unroll
    for (int j = 0; j < NE; ++j)
        if (mine(j))
            st_stream(&s[part + (off | so[j])], va[j]);
    if (two) {
        if (J.inner) {
            __syncthreads();  // every thread has read its part of the first tile
            permute(vb);
        }
#pragma unroll
        for (int j = 0; j < NE; ++j)
            if (mine(j))
                st_stream(&s[base + (off | so[j])], vb[j]);
    }
}

// blocks for items, at most 2^31 threads per launch (the kernels stride over
// the rest)
inline unsigned blocks_for(uint64_t items)
{
    uint64_t b = (items + (uint64_t)NT * UNR - 1) / ((uint64_t)NT * UNR);
    b = std::min<uint64_t>(b, (1ull << 31) / NT);
    return (unsigned)(b ? b : 1);
}

// qubits below this index split a 128-byte line
template <typename R> constexpr int line_bits() { return sizeof(typename Cx<R>::T) == 16 ? 3 : 4; }

template <typename R, bool NTA>
void plain_gate_nt(typename Cx<R>::T *s, int n, const qs_gate &g, hipStream_t st)
{
    switch (g.kind) {
    case QS_GATE_U: {
        uint64_t np = 1ull << (n - 1);
        hipLaunchKernelGGL((k_pair_u<R, false, NTA>), dim3(blocks_for(np)), dim3(NT), 0, st, s, np, g.q0, 0, 0,
                           0ull, Mat<R>(g.u));
        break;
    }
    case QS_GATE_CU: {
        uint64_t nq = 1ull << (n - 2);
        int lo = g.q0 < g.q1 ? g.q0 : g.q1, hi = g.q0 < g.q1 ? g.q1 : g.q0;
        hipLaunchKernelGGL((k_pair_u<R, true, NTA>), dim3(blocks_for(nq)), dim3(NT), 0, st, s, nq, g.q1, lo, hi,
                           1ull << g.q0, Mat<R>(g.u));
        break;
    }
    case QS_GATE_CX: {
        uint64_t nq = 1ull << (n - 2);
        int lo = g.q0 < g.q1 ? g.q0 : g.q1, hi = g.q0 < g.q1 ? g.q1 : g.q0;
        hipLaunchKernelGGL((k_cx<R, NTA>), dim3(blocks_for(nq)), dim3(NT), 0, st, s, nq, g.q1, lo, hi,
                           1ull << g.q0);
        break;
    }
    case QS_GATE_CZ: {
        uint64_t nq = 1ull << (n - 2);
        int lo = g.q0 < g.q1 ? g.q0 : g.q1, hi = g.q0 < g.q1 ? g.q1 : g.q0;
        hipLaunchKernelGGL((k_cz<R, NTA>), dim3(blocks_for(nq)), dim3(NT), 0, st, s, nq, lo, hi,
                           (1ull << g.q0) | (1ull << g.q1));
        break;
    }
    default:
        fail(QS_ERR_ARG, "unknown gate kind");
    }
    check_launch("plain gate");
}

template <typename R>
void plain_gate_t(void *state, int n, const qs_gate &g, hipStream_t st)
{
    using C = typename Cx<R>::T;
    C *s = reinterpret_cast<C *>(state);
    // the lowest qubit the launch splits on: the target, or the lower of two
    const int low = g.kind == QS_GATE_U ? g.q0 : (g.q0 < g.q1 ? g.q0 : g.q1);
    if (low >= line_bits<R>())
        plain_gate_nt<R, true>(s, n, g, st);
    else
        plain_gate_nt<R, false>(s, n, g, st);
}

}  // namespace

void launch_set_basis(void *state, qs_dtype dt, int n, uint64_t x, hipStream_t st)
{
    uint64_t N = 1ull << n;
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_set_basis<float>, dim3(blocks_for(N)), dim3(NT), 0, st,
                           reinterpret_cast<Cplx<float> *>(state), N, x);
    else
        hipLaunchKernelGGL(k_set_basis<double>, dim3(blocks_for(N)), dim3(NT), 0, st,
                           reinterpret_cast<Cplx<double> *>(state), N, x);
    check_launch("set_basis");
}

void launch_plain_gate(void *state, qs_dtype dt, int n, const qs_gate &g, hipStream_t st)
{
    if (g.kind != QS_GATE_U && n < 2)
        fail(QS_ERR_ARG, "two-qubit gate on a one-qubit state");
    if (dt == QS_C64)
        plain_gate_t<float>(state, n, g, st);
    else
        plain_gate_t<double>(state, n, g, st);
}

template <typename R> static void involution_t(void *state, int n, const std::vector<int> &pi, hipStream_t st)
{
    Involution J{};
    // the tile: line positions and their partners (at most twice the line's
    // bits), then pairs and fixed positions in ascending order while they fit
    std::vector<char> in(n, 0);
    for (int p = 0; p < n && p < line_bits<R>(); ++p)
        in[p] = in[pi[p]] = 1;
    for (int p = 0; p < n; ++p)
        J.K += in[p];
    // Smaller tiles for small states, so that 2^10 of them are in flight: up to
    // 2^20 amplitudes a launch is as long as one workgroup's chain of loads,
    // LDS and stores.  Two moves, 16 qubits complex64: a random placement 51 us
    // with tiles of 2^12, 19 with 2^8, the reversal 24, 13; 20 qubits: 58, 35
    // and 26, 17; complex128, 17 qubits, a rotation 33, 21; 2^11 tiles are
    // slower again (20 qubits complex64, the reversal 38).
    const int most = std::min(INV_BITS<R>, std::max(2 * line_bits<R>(), n - 10));
    for (int p = 0; p < n; ++p) {
        const int need = pi[p] == p ? 1 : 2;
        if (!in[p] && J.K + need <= most) {
            in[p] = in[pi[p]] = 1;
            J.K += need;
        }
    }
    std::vector<int> tb(n, -1);
    for (int p = 0, b = 0; p < n; ++p)
        if (in[p]) {
            tb[p] = b;
            J.pos[b++] = (uint8_t)p;
        }
    for (int b = 0; b < J.K; ++b) {
        J.perm[b] = (uint8_t)tb[pi[J.pos[b]]];
        J.inner |= J.perm[b] != b;
    }
    for (int p = 0; p < n; ++p)
        if (!in[p] && pi[p] > p) {
            J.lo[J.n_pairs] = (uint8_t)p;
            J.hi[J.n_pairs++] = (uint8_t)pi[p];
        }
    // rows of at most 2^22 workgroups (a launch holds fewer than 2^32 threads
    // per dimension)
    const uint64_t tiles = 1ull << (n - J.K), row = std::min<uint64_t>(tiles, 1ull << 22);
    hipLaunchKernelGGL(k_involution<R>, dim3((unsigned)row, (unsigned)(tiles / row)), dim3(NT), 0, st,
                       reinterpret_cast<Cplx<R> *>(state), J);
    check_launch("involution");
}

void launch_involution(void *state, qs_dtype dt, int n, const std::vector<int> &pi, hipStream_t st)
{
    bool moved = false;
    for (int p = 0; p < n; ++p) {
        if (pi[pi[p]] != p)
            fail(QS_ERR_ARG, "internal: position map is not an involution");
        moved |= pi[p] != p;
    }
    if (!moved)
        return;
    if (dt == QS_C64)
        involution_t<float>(state, n, pi, st);
    else
        involution_t<double>(state, n, pi, st);
}

}  // namespace qsim
