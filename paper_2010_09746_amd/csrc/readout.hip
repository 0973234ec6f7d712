// Read-out kernels (paper, Section 2: measurement): norm, <Z_q> for every
// qubit in one read of the state, amplitude gather and the overlap of two
// states.  All sums are accumulated in FP64 and reduced in a fixed order
// (block partials, then one pass over the partials), so results do not depend
// on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.cuh"
#include "kernels.h"

namespace qsim {

namespace {

constexpr int ZT = 256;          // threads per block
constexpr int ZT_BITS = 8;
constexpr int ZCHUNK_BITS = 18;  // largest chunk: 2^18 amplitudes per block

// Sum over the 64 lanes of a wavefront, in a fixed order (every lane gets it).
__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
        x += __shfl_xor(x, d);
    return x;
}

// Amplitudes per block = 2^L.  One block up to 13 qubits (no second launch);
// then blocks of at least 8 loads per thread, about 2^11 blocks (8 per
// compute unit) and at most 2^18 amplitudes each.
template <typename R> int zchunk_bits(int n)
{
    constexpr int vb = sizeof(R) == 4 ? 1 : 0;
    if (n <= 13)
        return n;
    const int lo = ZT_BITS + vb + 3;
    return std::min(std::max(n - 11, lo), ZCHUNK_BITS);
}

// Block b covers physical indices [b 2^L, (b+1) 2^L).  For each position p it
// writes S_p(block) = sum over its indices j with bit p set of |v_j|^2, and
// the block norm: value o (0 the norm, 1 + p position p) at
// part[o * gridDim.x + b].
//
// Bound by the read of the state.  Eight 16-byte loads per thread are in
// flight (one load of a complex64 state holds two amplitudes); the bits of the
// iteration number are summed per thread, the lane bits by the wavefront's
// reduction and the wavefront bits from the four wavefront sums.  qs_expect_z
// as a whole: 28 qubits complex64 703 -> 395 us (5.4 TB/s), complex128 876 ->
// 748 us (5.7 TB/s), 21 qubits complex64 64 -> 28 us, 10 qubits 41 -> 23 us
// (before: one load in flight, at least 2^14 amplitudes per block, and one
// thread adding the 256 terms of an output in turn).
template <typename R>
__global__ __launch_bounds__(ZT) void k_zsum(const Cplx<R> *__restrict__ s, int n, int L, double *part)
{
    constexpr int VB = sizeof(R) == 4 ? 1 : 0;  // index bits inside one 16-byte load
    constexpr int U_BITS = 3, U = 1 << U_BITS;
    constexpr int IT = ZCHUNK_BITS - ZT_BITS;   // iteration bits at most
    constexpr int NV = 1 + 1 + 6 + IT;          // norm, vector bit, lane bits, iteration bits
    __shared__ double red[ZT / 64][NV];
    using Vec = R __attribute__((ext_vector_type(2 << VB)));
    const int tid = threadIdx.x, lane = tid & 63;
    const int nthr = L - VB >= ZT_BITS ? ZT : (1 << (L - VB));
    const int it_bits = L - VB > ZT_BITS ? L - VB - ZT_BITS : 0;
    const uint32_t iters = 1u << it_bits;
    const uint64_t base = (uint64_t)blockIdx.x << L;
    // a wide load at the alignment of one amplitude (a copy, not a cast to the
    // vector type): a server's complex64 request may begin at any of them
    auto load = [&](uint64_t i) {
        Vec x;
        __builtin_memcpy(&x, s + base + (i << VB), sizeof x);
        return x;
    };
    double tot = 0.0, vec = 0.0, acc[IT];
#pragma unroll
    for (int b = 0; b < IT; ++b)
        acc[b] = 0.0;
    if (tid < nthr) {
        for (uint32_t it = 0; it < iters; it += U) {
            Vec v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                v[u] = it + u < iters ? load(((uint64_t)(it + u) << ZT_BITS) + tid) : Vec(R(0));
            double p[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double re = (double)v[u][0], im = (double)v[u][1];
                p[u] = re * re + im * im;
                if constexpr (VB == 1) {
                    const double r1 = (double)v[u][2], i1 = (double)v[u][3], q = r1 * r1 + i1 * i1;
                    vec += q;
                    p[u] += q;
                }
            }
            // sums over the group by its three iteration bits
            const double a01 = p[0] + p[1], a23 = p[2] + p[3], a45 = p[4] + p[5], a67 = p[6] + p[7];
            const double hi = a45 + a67, g = (a01 + a23) + hi;
            acc[0] += (p[1] + p[3]) + (p[5] + p[7]);
            acc[1] += a23 + a67;
            acc[2] += hi;
            tot += g;
#pragma unroll
            for (int b = U_BITS; b < IT; ++b)
                if ((it >> b) & 1)
                    acc[b] += g;
        }
    }
    // lane bits: before lane bit i is added up, the half of the pair whose
    // bit is 1 starts that bit's sum, which then runs over the bits above
    double t = tot;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const double other = __shfl_xor(t, 1 << i);
        double w = ((lane >> i) & 1) ? t : other;
#pragma unroll
        for (int d = i + 1; d < 6; ++d)
            w += __shfl_xor(w, 1 << d);
        if (lane == 0)
            red[tid >> 6][2 + i] = w;
        t += other;
    }
    if (lane == 0)
        red[tid >> 6][0] = t;
    if constexpr (VB == 1) {
        vec = wave_sum(vec);
        if (lane == 0)
            red[tid >> 6][1] = vec;
    }
#pragma unroll
    for (int b = 0; b < IT; ++b)
        if (b < it_bits) {
            const double w = wave_sum(acc[b]);
            if (lane == 0)
                red[tid >> 6][8 + b] = w;
        }
    __syncthreads();
    // one thread per output, the wavefronts in order
    const int outs = n + 1;
    if (tid < outs) {
        const int p = tid - 1;
        int v = 0;                 // which value
        uint32_t waves = 0xfu;     // over which wavefronts
        if (p >= 0) {
            if (p >= L)
                waves = ((base >> p) & 1) ? 0xfu : 0u;
            else if (p < VB)
                v = 1;
            else if (p < VB + 6)
                v = 2 + (p - VB);
            else if (p < VB + ZT_BITS)
                waves = p - VB - 6 == 0 ? 0xau : 0xcu;
            else
                v = 8 + (p - VB - ZT_BITS);
        }
        double r = 0.0;
#pragma unroll
        for (int w = 0; w < ZT / 64; ++w)
            if ((waves >> w) & 1u)
                r += red[w][v];
        part[(uint64_t)tid * gridDim.x + blockIdx.x] = r;
    }
}

// out[o] = sum over blocks of part[o * nblocks + b]: thread t of block o sums
// the blocks b = t (mod 256) in order, then the wavefronts' sums in order.
__global__ __launch_bounds__(256) void k_sum_parts(const double *part, uint64_t nblocks, double *out)
{
    __shared__ double red[4];
    const int o = blockIdx.x;
    double r = 0.0;
    for (uint64_t b = threadIdx.x; b < nblocks; b += 256)
        r += part[(uint64_t)o * nblocks + b];
    r = wave_sum(r);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0)
        out[o] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Fold the per-tile read-out of a tile pass into the sums of k_zsum (see
// ZFoldMap): output 0 is the sum over tiles of T, output 1 + p that of the
// probability of bit p.  Block (s, o) takes slice s of the tiles for output
// o: thread t of the block takes the slice's tiles t (mod 256) in order, the
// 256 sums are added in a fixed tree into work[o * slices + s], and
// k_sum_parts adds the slices in order.
static uint64_t zfold_slices(uint64_t tiles) { return std::min<uint64_t>(256, std::max<uint64_t>(1, tiles >> 10)); }

__global__ __launch_bounds__(256) void k_zfold(const double *parts, uint64_t tiles, uint64_t chunk, ZFoldMap m,
                                               double *work)
{
    __shared__ double red[256];
    const uint64_t s = blockIdx.x;
    const int o = blockIdx.y;
    const int v = o == 0 ? 0 : m.v[o - 1];
    const uint64_t rm = o == 0 ? 0 : m.rm[o - 1];
    const uint64_t t_end = std::min(tiles, (s + 1) * chunk);
    double r = 0.0;
    for (uint64_t t = s * chunk + threadIdx.x; t < t_end; t += 256) {
        const double T = parts[t];
        const bool odd = (__popcll(t & rm) & 1) != 0;
        if (o == 0)
            r += T;
        else if (v >= 1)
            r += odd ? T - parts[(uint64_t)v * tiles + t] : parts[(uint64_t)v * tiles + t];
        else if (odd)
            r += T;
    }
    red[threadIdx.x] = r;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        work[(uint64_t)o * gridDim.x + s] = red[0];
}

template <typename R>
__global__ __launch_bounds__(256) void k_gather(const Cplx<R> *__restrict__ s, const uint64_t *idx, int64_t count,
                                                double *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) {
        const Cplx<R> a = s[idx[i]];
        out[2 * i] = (double)a.x;
        out[2 * i + 1] = (double)a.y;
    }
}

// Amplitudes [i0, i0 + count) in logical order, as FP64: bit q of the logical
// index is position sigma[q].  Four amplitudes per thread; the part of the
// index above the thread id is uniform.  The copy to the host that follows
// bounds the read-out: qs_read_state of 22 qubits complex128 191 -> 7.0 ms
// (9.6 GB/s), 16 qubits 2.4 -> 0.09 ms (before, a host loop over the bits of
// every index).
struct Placement {
    uint8_t sigma[48];
};

template <typename R>
__global__ __launch_bounds__(256) void k_logical(const Cplx<R> *__restrict__ s, int n, Placement pl, uint64_t i0,
                                                 uint64_t count, double *out)
{
    constexpr int U = 4;
    uint64_t lane = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (q < n)
            lane |= (uint64_t)((threadIdx.x >> q) & 1u) << pl.sigma[q];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t at = ((uint64_t)blockIdx.x * U + u) << 8, i = i0 + at;
        uint64_t hi = 0;
        for (int q = 8; q < n; ++q)
            hi |= ((i >> q) & 1ull) << pl.sigma[q];
        const uint64_t k = at + threadIdx.x;
        if (k < count) {
            const Cplx<R> a = s[hi | lane];
            using D2 = double __attribute__((ext_vector_type(2)));
            reinterpret_cast<D2 *>(out)[k] = D2{(double)a.x, (double)a.y};
        }
    }
}

// Enumeration of the amplitude pairs of two states of n qubits: bit i of the
// enumeration index is position pa[i] of a's index and pb[i] of b's.
struct PairMap {
    int n, L;  // 2^L pairs per block
    uint8_t pa[48], pb[48];
};

constexpr int FT = 256, FT_BITS = 8;

inline int fchunk_bits(int n) { return std::min(n, std::min(std::max(n - 12, FT_BITS + 2), 18)); }

__device__ __forceinline__ void deposit(const PairMap &m, int bit, uint64_t x, uint64_t &ja, uint64_t &jb)
{
    ja |= (x & 1ull) << m.pa[bit];
    jb |= (x & 1ull) << m.pb[bit];
}

// partials per block b: value q (re <a|b>, im <a|b>, <a|a>, <b|b>, max |a - b|^2)
// at part[q * gridDim.x + b].
//
// Bound by the reads.  The lowest enumeration bits (the lanes) are the
// positions inside a 128-byte line of a and then those inside a line of b, so
// that whole lines of both states are used by neighbouring lanes at any
// placement; the index parts of a thread and of a block are deposited once,
// and four pairs are in flight.  qs_fidelity as a whole, complex64 against
// complex128 under a random placement: 28 qubits 2986 -> 1192 us (5.4 TB/s), 26
// qubits 509 -> 317 us, 16 qubits 86 -> 27 us (before: a loop over all
// positions, a square root and one load pair in flight for each amplitude,
// lanes in a's order, and one thread adding 256 terms).
template <typename Ra, typename Rb>
__global__ __launch_bounds__(FT) void k_fid(const Cplx<Ra> *__restrict__ a, const Cplx<Rb> *__restrict__ b, PairMap m,
                                            double *part)
{
    constexpr int U_BITS = 2, U = 1 << U_BITS;
    __shared__ double red[FT / 64][5];
    const int tid = threadIdx.x;
    const int nthr = m.L >= FT_BITS ? FT : (1 << m.L);
    uint64_t ta = 0, tb = 0;
    for (int i = 0; i < FT_BITS && i < m.L; ++i)
        deposit(m, i, (uint64_t)tid >> i, ta, tb);
    uint64_t ba = 0, bb = 0;
    for (int i = m.L; i < m.n; ++i)
        deposit(m, i, (uint64_t)blockIdx.x >> (i - m.L), ba, bb);
    const uint32_t iters = 1u << (m.L > FT_BITS ? m.L - FT_BITS : 0);
    double sr = 0, si = 0, na = 0, nb = 0, mx = 0;
    if (tid < nthr) {
        for (uint32_t it = 0; it < iters; it += U) {
            uint64_t ia = 0, ib = 0;
            for (int i = U_BITS; i + FT_BITS < m.L; ++i)
                deposit(m, FT_BITS + i, it >> i, ia, ib);
            Cplx<Ra> x[U];
            Cplx<Rb> y[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                uint64_t ua = 0, ub = 0;
#pragma unroll
                for (int i = 0; i < U_BITS; ++i)
                    if (((u >> i) & 1u) && FT_BITS + i < m.L) {
                        ua |= 1ull << m.pa[FT_BITS + i];
                        ub |= 1ull << m.pb[FT_BITS + i];
                    }
                if (it + u < iters) {
                    x[u] = a[(ba | ia | ua) | ta];
                    y[u] = b[(bb | ib | ub) | tb];
                } else {
                    x[u] = Cplx<Ra>{0, 0};
                    y[u] = Cplx<Rb>{0, 0};
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double xr = x[u].x, xi = x[u].y, yr = y[u].x, yi = y[u].y;
                sr += xr * yr + xi * yi;  // conj(x) * y
                si += xr * yi - xi * yr;
                na += xr * xr + xi * xi;
                nb += yr * yr + yi * yi;
                const double dr = xr - yr, di = xi - yi, d = dr * dr + di * di;
                mx = d > mx ? d : mx;
            }
        }
    }
    sr = wave_sum(sr);
    si = wave_sum(si);
    na = wave_sum(na);
    nb = wave_sum(nb);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double o = __shfl_xor(mx, d);
        mx = o > mx ? o : mx;
    }
    if ((tid & 63) == 0) {
        double *r = red[tid >> 6];
        r[0] = sr;
        r[1] = si;
        r[2] = na;
        r[3] = nb;
        r[4] = mx;
    }
    __syncthreads();
    if (tid < 5) {
        double r = red[0][tid];
        for (int w = 1; w < FT / 64; ++w)
            r = tid == 4 ? (red[w][tid] > r ? red[w][tid] : r) : r + red[w][tid];
        part[(uint64_t)tid * gridDim.x + blockIdx.x] = r;
    }
}

// out[q] over the block partials: block q, thread t takes the blocks
// b = t (mod 256) in order, then a fixed tree over the 256 thread results
// (a sum for q < 4; for q = 4 a maximum, whose square root is the largest
// distance)
__global__ __launch_bounds__(256) void k_fid_final(const double *part, uint64_t nblocks, double *out)
{
    __shared__ double red[256];
    const int q = blockIdx.x;
    double r = 0;
    for (uint64_t b = threadIdx.x; b < nblocks; b += 256) {
        const double v = part[q * nblocks + b];
        r = q == 4 ? (v > r ? v : r) : r + v;
    }
    red[threadIdx.x] = r;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            const double x = red[threadIdx.x], y = red[threadIdx.x + w];
            red[threadIdx.x] = q == 4 ? (y > x ? y : x) : x + y;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        out[q] = q == 4 ? sqrt(red[0]) : red[0];
}

template <typename Ra, typename Rb>
void fid_t(const void *a, const void *b, const PairMap &m, double *work, double *out, hipStream_t st)
{
    const uint64_t nb = 1ull << (m.n - m.L);
    hipLaunchKernelGGL((k_fid<Ra, Rb>), dim3((unsigned)nb), dim3(FT), 0, st, reinterpret_cast<const Cplx<Ra> *>(a),
                       reinterpret_cast<const Cplx<Rb> *>(b), m, work);
    check_launch("fidelity");
    hipLaunchKernelGGL(k_fid_final, dim3(5), dim3(256), 0, st, work, nb, out);
    check_launch("fidelity final");
}

template <typename R> void zsum_t(const void *state, int n, double *work, double *out, hipStream_t st)
{
    const int L = zchunk_bits<R>(n);
    const uint64_t nb = 1ull << (n - L);
    // a single block's values are the result
    hipLaunchKernelGGL(k_zsum<R>, dim3((unsigned)nb), dim3(ZT), 0, st, reinterpret_cast<const Cplx<R> *>(state), n, L,
                       nb == 1 ? out : work);
    check_launch("zsum");
    if (nb > 1) {
        hipLaunchKernelGGL(k_sum_parts, dim3(n + 1), dim3(256), 0, st, work, nb, out);
        check_launch("zsum final");
    }
}

}  // namespace

size_t zsum_work_doubles(int n)
{
    // the smaller blocks (complex128) need more room; not decreasing in n
    return (1ull << (n - zchunk_bits<double>(n))) * (size_t)(n + 1);
}

void launch_zsum(const void *state, qs_dtype dt, int n, double *work, double *out, hipStream_t st)
{
    if (dt == QS_C64)
        zsum_t<float>(state, n, work, out, st);
    else
        zsum_t<double>(state, n, work, out, st);
}

size_t zfold_work_doubles(uint64_t tiles, int n) { return (size_t)zfold_slices(tiles) * (size_t)(n + 1); }

void launch_zfold(const double *parts, uint64_t tiles, int nv, int n, const ZFoldMap &m, double *work_dev,
                  double *out_dev, hipStream_t st)
{
    (void)nv;
    const uint64_t S = zfold_slices(tiles), chunk = (tiles + S - 1) / S;
    hipLaunchKernelGGL(k_zfold, dim3((unsigned)S, (unsigned)(n + 1)), dim3(256), 0, st, parts, tiles, chunk, m,
                       work_dev);
    check_launch("zfold");
    hipLaunchKernelGGL(k_sum_parts, dim3(n + 1), dim3(256), 0, st, work_dev, S, out_dev);
    check_launch("zfold final");
}

void launch_gather(const void *state, qs_dtype dt, const uint64_t *idx, int64_t count, double *out, hipStream_t st)
{
    if (count <= 0)
        return;
    const unsigned nb = (unsigned)((count + 255) / 256);
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_gather<float>, dim3(nb), dim3(256), 0, st, reinterpret_cast<const Cplx<float> *>(state),
                           idx, count, out);
    else
        hipLaunchKernelGGL(k_gather<double>, dim3(nb), dim3(256), 0, st,
                           reinterpret_cast<const Cplx<double> *>(state), idx, count, out);
    check_launch("gather");
}

void launch_logical(const void *state, qs_dtype dt, int n, const std::vector<int> &sigma, uint64_t i0, uint64_t count,
                    double *out, hipStream_t st)
{
    Placement pl{};
    for (int q = 0; q < n; ++q)
        pl.sigma[q] = (uint8_t)sigma[q];
    const unsigned nb = (unsigned)((count + 1023) / 1024);
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_logical<float>, dim3(nb), dim3(256), 0, st, reinterpret_cast<const Cplx<float> *>(state), n,
                           pl, i0, count, out);
    else
        hipLaunchKernelGGL(k_logical<double>, dim3(nb), dim3(256), 0, st,
                           reinterpret_cast<const Cplx<double> *>(state), n, pl, i0, count, out);
    check_launch("logical order");
}

size_t fid_work_doubles(int n) { return (1ull << (n - fchunk_bits(n))) * (size_t)5; }

void launch_fidelity(const void *a, qs_dtype da, const void *b, qs_dtype db, int n, const std::vector<int> &map_b,
                     double *work, double *out, hipStream_t st)
{
    PairMap m{};
    m.n = n;
    m.L = fchunk_bits(n);
    const int la = da == QS_C64 ? 4 : 3, lb = db == QS_C64 ? 4 : 3;  // positions inside a 128-byte line
    int k = 0;
    for (int pass = 0; pass < 3; ++pass)
        for (int p = 0; p < n; ++p) {
            const int rank = p < la ? 0 : map_b[p] < lb ? 1 : 2;
            if (rank != pass)
                continue;
            m.pa[k] = (uint8_t)p;
            m.pb[k++] = (uint8_t)map_b[p];
        }
    if (da == QS_C64 && db == QS_C64)
        fid_t<float, float>(a, b, m, work, out, st);
    else if (da == QS_C64 && db == QS_C128)
        fid_t<float, double>(a, b, m, work, out, st);
    else if (da == QS_C128 && db == QS_C64)
        fid_t<double, float>(a, b, m, work, out, st);
    else
        fid_t<double, double>(a, b, m, work, out, st);
}

}  // namespace qsim
