// Read-out sweeps: marginal probabilities, Pauli expectation values and
// sampling (paper Sec. 2.1 "Measurement and Sampling", shots of Sec. 2.2).
// Each is one read pass over the state; all accumulation is FP64 whatever the
// amplitude precision, with a fixed reduction order (no atomics), so results
// are reproducible run to run.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sv_internal.h"

namespace sv {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxQ = 30;

template <typename R>
struct CT;
template <>
struct CT<float> {
    using C = float2;
};
template <>
struct CT<double> {
    using C = double2;
};

struct Masks {
    uint64_t m[kMaxQ + 1];
    int n;
};

Masks make_masks(std::vector<int> pos)
{
    std::sort(pos.begin(), pos.end());
    Masks im{};
    im.n = int(pos.size());
    for (int j = 0; j < im.n; ++j)
        im.m[j] = (uint64_t(1) << pos[j]) - 1;
    return im;
}

__device__ __forceinline__ uint64_t insert_zeros(uint64_t g, const Masks &im)
{
    for (int j = 0; j < im.n; ++j) {
        const uint64_t lo = im.m[j];
        g = (g & lo) | ((g & ~lo) << 1);
    }
    return g;
}

template <typename C>
__device__ __forceinline__ double prob(C a)
{
    const double x = double(a.x), y = double(a.y);
    return x * x + y * y;
}

// Read-only sweeps read every byte once: loads carry the nontemporal hint
// (a 2 GiB read measured 0.30 ms with it, 0.33 ms without).
typedef float rd_f32x2 __attribute__((ext_vector_type(2)));
typedef float rd_f32x4 __attribute__((ext_vector_type(4)));
typedef double rd_f64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 ldnt(const float2 *p)
{
    const rd_f32x2 q = __builtin_nontemporal_load(reinterpret_cast<const rd_f32x2 *>(p));
    return make_float2(q.x, q.y);
}
__device__ __forceinline__ float4 ldnt(const float4 *p)
{
    const rd_f32x4 q = __builtin_nontemporal_load(reinterpret_cast<const rd_f32x4 *>(p));
    return make_float4(q.x, q.y, q.z, q.w);
}
__device__ __forceinline__ double2 ldnt(const double2 *p)
{
    const rd_f64x2 q = __builtin_nontemporal_load(reinterpret_cast<const rd_f64x2 *>(p));
    return make_double2(q.x, q.y);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Sum over the 256 threads of a block; result valid in every thread.
__device__ __forceinline__ double block_sum(double v, double *sh)
{
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        sh[w] = v;
    __syncthreads();
    const double r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    return r;
}

// Sums of v[0 .. C) over the lanes that differ in bits OFF, OFF / 2, .., 1: with
// each bit a lane keeps the half of the values that its bit names, until one
// is left.
template <int C, int OFF, int NT>
__device__ __forceinline__ void halve_values(double (&v)[NT], int lane)
{
    if constexpr (OFF > 0 && C > 1) {
        const bool hi = (lane & OFF) != 0;
#pragma unroll
        for (int i = 0; i < C / 2; ++i) {
            const double give = hi ? v[i] : v[i + C / 2];
            v[i] = (hi ? v[i + C / 2] : v[i]) + __shfl_xor(give, OFF, 64);
        }
        halve_values<C / 2, OFF / 2>(v, lane);
    } else if constexpr (OFF > 0) {
        v[0] += __shfl_xor(v[0], OFF, 64);
        halve_values<1, OFF / 2>(v, lane);
    }
}

// block_sum of NT values at once (a power of two up to 64), the same sums to
// the bit: each shuffle step hands half of the values still held to the other
// half of the lanes, NT - 1 + 6 - log2(NT) shuffles of a double (32 for NT = 32)
// where one value at a time takes 6 NT (192).  out(t, sum) is called by one
// thread for each value.  sh: 4 NT.
template <int NT, typename F>
__device__ __forceinline__ void block_sums(double (&v)[NT], double *sh, F out)
{
    static_assert(NT >= 1 && NT <= 64 && (NT & (NT - 1)) == 0, "one value per lane");
    constexpr int LT = __builtin_ctz(NT);
    const int lane = threadIdx.x & 63;
    halve_values<NT, 32>(v, lane);
    __syncthreads();
    if ((lane & ((64 >> LT) - 1)) == 0)
        sh[(threadIdx.x >> 6) * NT + (lane >> (6 - LT))] = v[0];
    __syncthreads();
    const int t = threadIdx.x;
    if (t < NT)
        out(t, (sh[t] + sh[NT + t]) + (sh[2 * NT + t] + sh[3 * NT + t]));
}

// ---------------------------------------------------------------------------
// Marginals.  out[x] = sum over rest index r of |a[dep(x, Q) | ins(r)]|^2.
// ---------------------------------------------------------------------------
struct MargArgs {
    uint64_t rest;        // 2^(n-m)
    uint64_t per_chunk;   // rest indices per chunk (multiple of kThreads or rest)
    uint32_t chunks;
    uint32_t nbins;
    int m;
    uint64_t qbit[kMaxQ];
    Masks rest_im;
};

__device__ __forceinline__ uint64_t dep_x(uint64_t x, const MargArgs &a)
{
    uint64_t p = 0;
    for (int b = 0; b < a.m; ++b)
        if ((x >> b) & 1)
            p |= a.qbit[b];
    return p;
}

// Block (chunk, x): one bin, a contiguous range of rest indices (coalesced).
template <typename R>
__global__ __launch_bounds__(kThreads) void k_marg_rmajor(const R *__restrict__ st, double *__restrict__ part,
                                                          const MargArgs a)
{
    using C = typename CT<R>::C;
    __shared__ double sh[4];
    const C *v = reinterpret_cast<const C *>(st);
    const uint64_t x = blockIdx.y;
    const uint64_t xq = dep_x(x, a);
    const uint64_t r0 = uint64_t(blockIdx.x) * a.per_chunk;
    uint64_t r1 = r0 + a.per_chunk;
    if (r1 > a.rest)
        r1 = a.rest;
    double acc = 0.0;
    for (uint64_t r = r0 + threadIdx.x; r < r1; r += kThreads)
        acc += prob(v[xq | insert_zeros(r, a.rest_im)]);
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0)
        part[x * a.chunks + blockIdx.x] = acc;
}

// One thread per bin, sequential over the (few) rest indices.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_marg_xmajor(const R *__restrict__ st, double *__restrict__ out,
                                                          const MargArgs a)
{
    using C = typename CT<R>::C;
    const C *v = reinterpret_cast<const C *>(st);
    const uint64_t stride = uint64_t(gridDim.x) * kThreads;
    for (uint64_t x = uint64_t(blockIdx.x) * kThreads + threadIdx.x; x < a.nbins; x += stride) {
        const uint64_t xq = dep_x(x, a);
        double acc = 0.0;
        for (uint64_t r = 0; r < a.rest; ++r)
            acc += prob(v[xq | insert_zeros(r, a.rest_im)]);
        out[x] = acc;
    }
}

// out[x] = sum_c part[x * chunks + c], ascending c.
__global__ __launch_bounds__(kThreads) void k_sum_rows(const double *__restrict__ part, double *__restrict__ out,
                                                       uint64_t rows, uint32_t cols)
{
    const uint64_t x = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (x >= rows)
        return;
    double acc = 0.0;
    for (uint32_t c = 0; c < cols; ++c)
        acc += part[x * cols + c];
    out[x] = acc;
}

// Wide rows: one workgroup per row, strided partial sums in a fixed order,
// then the fixed block tree.
__global__ __launch_bounds__(kThreads) void k_sum_rows_wide(const double *__restrict__ part, double *__restrict__ out,
                                                            uint32_t cols)
{
    __shared__ double sh[4];
    const double *row = part + uint64_t(blockIdx.x) * cols;
    double acc = 0.0;
    for (uint32_t c = threadIdx.x; c < cols; c += kThreads)
        acc += row[c];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0)
        out[blockIdx.x] = acc;
}

}  // namespace

// out[x] = sum over c of part[x * cols + c], x < rows, in a fixed order.
static hipError_t launch_sum_rows(const double *part, double *out, uint64_t rows, uint32_t cols, hipStream_t s)
{
    if (cols >= kThreads && rows <= (uint64_t(1) << 20)) {
        hipLaunchKernelGGL(k_sum_rows_wide, dim3(uint32_t(rows)), dim3(kThreads), 0, s, part, out, cols);
    } else {
        const uint64_t g = (rows + kThreads - 1) / kThreads;
        hipLaunchKernelGGL(k_sum_rows, dim3(uint32_t(g)), dim3(kThreads), 0, s, part, out, rows, cols);
    }
    return hipGetLastError();
}

namespace {

// ---------------------------------------------------------------------------
// Z-string expectations: sum_i |a_i|^2 (-1)^popcount(i & z_t), up to kFewZ
// strings per pass (more go through the Walsh kernel below: expect_z_batch()).
// part[t * gridDim + block].
//
// A thread visits the indexes h0 + 256 u + threadIdx.x, u < 16, with h0 a
// multiple of 4096 that is the same across the workgroup, so the sign
// factors as (-1)^popcount(h0 & z_t) * (-1)^popcount(u & k_t) *
// (-1)^popcount(threadIdx.x & z_t), k_t = bits 8 .. 11 of z_t.  The first
// factors of all strings form one wave-uniform word per h0: lane t computes
// the parity for string t and a ballot collects them.  The second is folded
// into a Walsh transform of the thread's 16 probabilities over u, so each
// string takes one coefficient, picked by its uniform k_t, per 16
// amplitudes.  The third is applied once at the end.  Per 16 amplitudes
// and string the work is one FP64 FMA with a scalar +-1 operand (the scalar
// unit, shared by a CU's four SIMDs, otherwise bounds the sweep).
// ---------------------------------------------------------------------------
constexpr int kMaxZ = 32;  // strings of one fused read-out
constexpr int kFewZ = 16;
struct ExpZArgs {
    uint64_t nelem;
    int nt;
    uint64_t z[kFewZ];
};

template <typename R, int NZ>
__global__ __launch_bounds__(kThreads) void k_expect_z(const R *__restrict__ st, double *__restrict__ part,
                                                       const ExpZArgs a)
{
    static_assert(NZ <= 64 && NZ <= kFewZ, "one string per lane");
    using C = typename CT<R>::C;
    constexpr int LU = 4, U = 1 << LU;  // amplitudes per thread and step: index bits 8 .. 11
    static_assert(kThreads == 256, "lane and wave bits 0 .. 7");
    __shared__ double sh[4 * NZ];
    const C *v = reinterpret_cast<const C *>(st);
    const int lane = threadIdx.x & 63;
    const uint64_t zl = lane < NZ ? a.z[lane] : 0;  // the string whose parity this lane reports
    double acc[NZ];
#pragma unroll
    for (int t = 0; t < NZ; ++t)
        acc[t] = 0.0;
    const uint64_t chunk = uint64_t(U) * kThreads;
    for (uint64_t h0 = uint64_t(blockIdx.x) * chunk; h0 < a.nelem; h0 += uint64_t(gridDim.x) * chunk) {
        // every load in bounds (past the end: index 0, weight 0) and all of
        // them issued before the first is used
        C x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = h0 + uint64_t(u) * kThreads + threadIdx.x;
            x[u] = ldnt(&v[i < a.nelem ? i : 0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        double w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            w[u] = h0 + uint64_t(u) * kThreads + threadIdx.x < a.nelem ? prob(x[u]) : 0.0;
        // Walsh transform over the step bits: w[k] = sum_u (-1)^popcount(u & k) p_u
#pragma unroll
        for (int b = 1; b < U; b <<= 1)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (!(u & b)) {
                    const double x = w[u], y = w[u | b];
                    w[u] = x + y;
                    w[u | b] = x - y;
                }
        // h0 has bits 0 .. 11 clear: string t's sign is (-1)^popcount(h0 & z_t)
        // (workgroup-uniform, one ballot) times coefficient k = bits 8 .. 11
        // of z_t, times the lane part applied at the end
        const uint64_t sgn = __ballot((__popcll(h0 & zl) & 1) != 0);
#pragma unroll
        for (int t = 0; t < NZ; ++t) {
            const int k = int((a.z[t] >> 8) & (U - 1));
            acc[t] = fma(((sgn >> t) & 1) ? -1.0 : 1.0, w[k], acc[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < NZ; ++t)
        acc[t] = (__popc(threadIdx.x & uint32_t(a.z[t])) & 1) ? -acc[t] : acc[t];
    block_sums<NZ>(acc, sh, [&](int t, double x) {
        if (t < a.nt)
            part[uint64_t(t) * gridDim.x + blockIdx.x] = x;
    });
}

// ---------------------------------------------------------------------------
// General Pauli string, up to the i^(#Y) factor applied on the host:
// S = sum_i conj(a_{i^x}) s(i) a_i,  s(i) = (-1)^popcount(i & yz).  Pairs
// (i, i^x) with bit h (highest bit of x) of i equal to 0 are visited once.
// part[0 * grid + b] = Re, part[1 * grid + b] = Im.
// ---------------------------------------------------------------------------
struct ExpXYArgs {
    uint64_t npairs;
    uint64_t x;
    uint64_t yz;
    uint64_t hmask;  // 2^h - 1
};

template <typename R>
__global__ __launch_bounds__(kThreads) void k_expect_xy(const R *__restrict__ st, double *__restrict__ part,
                                                        const ExpXYArgs a)
{
    using C = typename CT<R>::C;
    __shared__ double sh[4];
    const C *v = reinterpret_cast<const C *>(st);
    double re = 0.0, im = 0.0;
    const uint64_t stride = uint64_t(gridDim.x) * kThreads;
    for (uint64_t g = uint64_t(blockIdx.x) * kThreads + threadIdx.x; g < a.npairs; g += stride) {
        const uint64_t i = (g & a.hmask) | ((g & ~a.hmask) << 1);
        const uint64_t j = i ^ a.x;
        const C ai = v[i], aj = v[j];
        const double si = (__popcll(i & a.yz) & 1) ? -1.0 : 1.0;
        const double sj = (__popcll(j & a.yz) & 1) ? -1.0 : 1.0;
        const double air = ai.x, aii = ai.y, ajr = aj.x, aji = aj.y;
        // conj(aj) * ai * si + conj(ai) * aj * sj
        re += si * (ajr * air + aji * aii) + sj * (air * ajr + aii * aji);
        im += si * (ajr * aii - aji * air) + sj * (air * aji - aii * ajr);
    }
    const double sre = block_sum(re, sh);
    const double sim = block_sum(im, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sre;
        part[uint64_t(gridDim.x) + blockIdx.x] = sim;
    }
}

// ---------------------------------------------------------------------------
// Several general strings from one read: one value per string,
//     V = sum_i s(i) f(a_i, a_{i ^ x}),   s(i) = (-1)^popcount(i & yz),
// f = Re(conj(a_j) a_i) for an even number of Y, Im for an odd one: with
// s(i ^ x) = (-1)^#Y s(i), the other part of S cancels between i and i ^ x
// (S = V, or i V), so only one FP64 product sum is taken per string.
// ---------------------------------------------------------------------------
struct PauliTerm {
    uint64_t x;
    uint64_t yz;
    uint32_t odd;  // number of Y is odd
    uint32_t pad;
};

// (p, q) with f = p b.x + q b.y for the partner amplitude b of a.
template <typename C>
__device__ __forceinline__ void pauli_weights(C a, bool odd, double &p, double &q)
{
    p = odd ? double(a.y) : double(a.x);
    q = odd ? -double(a.x) : double(a.y);
}

// Small states: block (chunk, string), every string reads its chunk of the
// pairs (i, i ^ x) from cache; one launch for all strings, Z strings included
// (x = 0: every amplitude its own partner).  With one chunk part is the result.
constexpr int kMultiTerms = 128;
struct ExpMultiArgs {
    uint64_t per_chunk;  // pairs (amplitudes for x = 0: twice that) per block
    PauliTerm t[kMultiTerms];
};

template <typename R>
__global__ __launch_bounds__(kThreads) void k_expect_multi(const R *__restrict__ st, double *__restrict__ part,
                                                           const ExpMultiArgs a)
{
    using C = typename CT<R>::C;
    __shared__ double sh[4];
    const C *v = reinterpret_cast<const C *>(st);
    const PauliTerm t = a.t[blockIdx.y];
    double acc = 0.0;
    if (t.x == 0) {
        const uint64_t i0 = uint64_t(blockIdx.x) * 2 * a.per_chunk;
        for (uint64_t e = threadIdx.x; e < 2 * a.per_chunk; e += kThreads) {
            const double p = prob(v[i0 + e]);
            acc += (__popcll((i0 + e) & t.yz) & 1) ? -p : p;
        }
    } else {
        const uint64_t hmask = (uint64_t(1) << (63 - __builtin_clzll(t.x))) - 1;
        const uint64_t g0 = uint64_t(blockIdx.x) * a.per_chunk;
        for (uint64_t e = threadIdx.x; e < a.per_chunk; e += kThreads) {
            const uint64_t g = g0 + e;
            const uint64_t i = (g & hmask) | ((g & ~hmask) << 1);
            const C ai = v[i], aj = v[i ^ t.x];
            double p, q;
            pauli_weights(ai, t.odd != 0, p, q);
            const double f = fma(p, double(aj.x), q * double(aj.y));
            acc += (__popcll(i & t.yz) & 1) ? -f : f;
        }
        acc *= 2.0;
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0)
        part[uint64_t(blockIdx.y) * gridDim.x + blockIdx.x] = acc;
}

// Large states: strings whose X and Y positions all lie among the index bits
// of one LDS tile (32 KiB: 2^12 complex64 or 2^11 complex128 amplitudes, the
// lowest bits among them so that runs are whole lines) share one read of the
// state.  A workgroup takes tiles o = block, block + grid, ...; the next
// tile's loads are in flight during the current one's sums.  Per string the
// threads share the tile's pairs of 16-byte vectors (i, i ^ x), both read from
// LDS: 15 vector instructions per four complex64 amplitudes, 8 of them
// conversions to FP64.  They bound the sweep: three reads of 2^27 complex64
// amplitudes with 8..12 strings each take 0.36 ms apiece (0.18 ms a read,
// 0.18 ms per string when every string read the state by itself); complex128,
// without conversions, 0.064 ms per read of 2^24 (0.046 ms per string before).
// Holding every thread's own amplitudes converted instead took 7 instructions
// per amplitude and 229 registers: 0.55 ms per read.
constexpr int kTileTerms = 16;
struct ExpTileArgs {
    uint64_t ntiles;
    uint64_t dep[12];  // physical index bit of tile bit b
    Masks outer;
    int nt;
    uint32_t xl[kTileTerms];   // tile-local X|Y bits
    uint32_t yl[kTileTerms];   // tile-local Y|Z bits
    uint64_t yz[kTileTerms];
    uint32_t odd[kTileTerms];
};

template <typename R>
constexpr int expect_tile_log()
{
    return std::is_same<R, float>::value ? 12 : 11;
}

typedef double f64x16 __attribute__((ext_vector_type(16)));

// Workgroups per CU that the registers of the persistent sweeps leave room
// for; their grids are that many per CU, so that all are resident at once.
template <typename R>
constexpr int tile_per_cu()
{
    return std::is_same<R, float>::value ? 3 : 4;
}
template <typename R>
constexpr int walsh_per_cu()
{
    return std::is_same<R, float>::value ? 4 : 2;
}

template <typename R>
__global__ __launch_bounds__(kThreads, tile_per_cu<R>()) void k_expect_tile(const R *__restrict__ st, double *__restrict__ part,
                                                          const ExpTileArgs a)
{
    constexpr bool F32 = std::is_same<R, float>::value;
    using V = typename std::conditional<F32, float4, double2>::type;  // 16 bytes
    constexpr int LO = F32 ? 1 : 0;   // tile bits inside a vector
    constexpr int NLD = 8;            // vectors per thread: tile bits LO + 8 ..
    __shared__ V tile[NLD * kThreads];
    __shared__ double sh[4];
    const V *v = reinterpret_cast<const V *>(st);
    const int tid = threadIdx.x;
    uint64_t off = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b)
        if ((tid >> b) & 1)
            off |= a.dep[b + LO];
    auto offk = [&](int k) {
        return ((k & 1) ? a.dep[8 + LO] : 0) | ((k & 2) ? a.dep[9 + LO] : 0) | ((k & 4) ? a.dep[10 + LO] : 0);
    };
    f64x16 acc = {};
    V nx[NLD];
    uint64_t base = insert_zeros(blockIdx.x, a.outer);
#pragma unroll
    for (int k = 0; k < NLD; ++k)
        nx[k] = ldnt(&v[(base | off | offk(k)) >> LO]);
    for (uint64_t o = blockIdx.x; o < a.ntiles; o += gridDim.x) {
        const uint64_t cur = base;
#pragma unroll
        for (int k = 0; k < NLD; ++k)
            tile[k * kThreads + tid] = nx[k];
        if (o + gridDim.x < a.ntiles) {
            base = insert_zeros(o + gridDim.x, a.outer);
#pragma unroll
            for (int k = 0; k < NLD; ++k)
                nx[k] = ldnt(&v[(base | off | offk(k)) >> LO]);
        }
        __syncthreads();
        for (int t = 0; t < a.nt; ++t) {
            const uint32_t xl = a.xl[t], yl = a.yl[t], xv = xl >> LO, yv = yl >> LO;
            uint32_t par = 0;  // parity of this thread's part of the signs
            // the number of Y and the swap of a vector's two amplitudes are
            // the same for every thread: a branch, not a selection
            auto sum = [&](auto odd_tag, auto swap_tag) __attribute__((always_inline)) {
                constexpr bool ODD = decltype(odd_tag)::value, SWAP = decltype(swap_tag)::value;
                // f of amplitude a and partner b
                auto f = [](double ar, double ai, double br, double bi) __attribute__((always_inline)) {
                    return ODD ? fma(ai, br, -(ar * bi)) : fma(ai, bi, ar * br);
                };
                double r = 0.0;
                if (!SWAP || xv != 0) {
                    // vectors i (bit h clear, or for h < 4 equal to bit 4, so that
                    // 16 consecutive lanes meet 16 different bank groups) and i ^ xv
                    const int h = 31 - __builtin_clz(xv);
                    const uint32_t hm = (1u << h) - 1u;
                    uint32_t iv = (uint32_t(tid) & hm) | ((uint32_t(tid) & ~hm) << 1);
                    if (h < 4)
                        iv |= ((iv >> 4) & 1u) << h;
                    par = uint32_t(__popc(iv & yv)) & 1u;
                    V p[4], q[4];
                    uint32_t im[4];
#pragma unroll
                    for (uint32_t m = 0; m < 4; ++m) {
                        im[m] = ((m << 8) & hm) | (((m << 8) & ~hm) << 1);
                        p[m] = tile[iv ^ im[m]];
                        q[m] = tile[iv ^ im[m] ^ xv];
                    }
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        double g;
                        if constexpr (F32) {
                            // amplitudes e and e ^ (x & 1), the second with the sign of bit 0
                            const double g1 = SWAP ? f(p[m].z, p[m].w, q[m].x, q[m].y) : f(p[m].z, p[m].w, q[m].z, q[m].w);
                            const double g0 = SWAP ? f(p[m].x, p[m].y, q[m].z, q[m].w) : f(p[m].x, p[m].y, q[m].x, q[m].y);
                            g = fma((yl & 1u) ? -1.0 : 1.0, g1, g0);
                        } else {
                            g = f(p[m].x, p[m].y, q[m].x, q[m].y);
                        }
                        r = fma((__builtin_popcount(im[m] & yv) & 1) ? -1.0 : 1.0, g, r);
                    }
                } else if constexpr (F32) {  // x = 1: the pair inside every vector
                    par = uint32_t(__popc(uint32_t(tid) & yv)) & 1u;
#pragma unroll
                    for (uint32_t k = 0; k < NLD; ++k) {
                        const V p = tile[k * kThreads + tid];
                        r = fma((__builtin_popcount((k << 8) & yv) & 1) ? -1.0 : 1.0, f(p.x, p.y, p.z, p.w), r);
                    }
                }
                return r;
            };
            const bool odd = a.odd[t] != 0, swap = F32 && (xl & 1u) != 0;
            double s;
            if (swap)
                s = odd ? sum(std::true_type{}, std::true_type{}) : sum(std::false_type{}, std::true_type{});
            else
                s = odd ? sum(std::true_type{}, std::false_type{}) : sum(std::false_type{}, std::false_type{});
            // both members of a pair contribute the same
            acc[t] = fma(((__popcll(cur & a.yz[t]) & 1u) ^ par) ? -2.0 : 2.0, s, acc[t]);
        }
        __syncthreads();
    }
    for (int t = 0; t < a.nt; ++t) {
        const double w = block_sum(acc[t], sh);
        if (tid == 0)
            part[uint64_t(t) * gridDim.x + blockIdx.x] = w;
    }
}

// ---------------------------------------------------------------------------
// Many Z strings from one read: a Walsh-Hadamard transform of every 2^12
// segment's probabilities gives sum_i p_i (-1)^popcount(i & k) for all 4096 k
// at once, and a string takes one of them per segment with the sign of its
// high bits: the work per amplitude does not grow with the strings (one per
// thread, up to kWalshTerms per launch).  Three rounds of four index bits in
// registers, exchanged through LDS; the loads of the next segment are in
// flight meanwhile.  Bound by the read: 2^27 complex64 amplitudes in 0.173 ms,
// 2^24 complex128 in 0.048 ms (5.6-6.2 TB/s); 81 strings in three reads of 32
// took 0.56 ms.  Index bits by round: the bits a thread's loads differ in
// (c64 0, 9..11; c128 8..11), 1..4, and the remaining four.
// ---------------------------------------------------------------------------
constexpr int kWalshTerms = 128;
struct ExpWalshArgs {
    uint64_t nseg;
    int nt;
    uint64_t z[kWalshTerms];
};

// LDS slot of index x: bits 6..9 XORed into bits 1..4, so that lanes that
// differ in those bits only use different banks.
__device__ __forceinline__ uint32_t walsh_slot(uint32_t x)
{
    return x ^ ((x >> 5) & 30u);
}

__device__ __forceinline__ void walsh16(f64x16 &w)
{
#pragma unroll
    for (int b = 1; b < 16; b <<= 1)
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (!(u & b)) {
                const double x = w[u], y = w[u | b];
                w[u] = x + y;
                w[u | b] = x - y;
            }
}

template <typename R>
__global__ __launch_bounds__(kThreads, walsh_per_cu<R>()) void k_expect_walsh(const R *__restrict__ st, double *__restrict__ part,
                                                           const ExpWalshArgs a)
{
    constexpr bool F32 = std::is_same<R, float>::value;
    using V = typename std::conditional<F32, float4, double2>::type;  // 16 bytes
    constexpr int SEG = 4096;
    constexpr int NLD = F32 ? 8 : 16;
    __shared__ __align__(16) double w_lds[SEG];
    const V *v = reinterpret_cast<const V *>(st);
    const int tid = threadIdx.x;
    const uint64_t z = tid < a.nt ? a.z[tid] : 0;
    // round 2: index bits 1..4 in registers, the thread gives the others (bit
    // 0 and 5..11); round 3: c64 bits 5..8 in registers, the thread gives
    // 0..4 and 9..11; c128 bits 0 and 5..7, the thread 1..4 and 8..11
    const uint32_t g2 = (tid & 1u) | (uint32_t(tid >> 1) << 5);
    const uint32_t g3 = F32 ? ((tid & 31u) | (uint32_t(tid >> 5) << 9)) : ((tid & 15u) << 1 | uint32_t(tid >> 4) << 8);
    auto r3 = [](uint32_t u) { return F32 ? u << 5 : (u & 1u) | (u >> 1) << 5; };
    double acc = 0.0;
    V nx[NLD];
#pragma unroll
    for (int k = 0; k < NLD; ++k)
        nx[k] = ldnt(&v[uint64_t(blockIdx.x) * (NLD * kThreads) + uint32_t(k * kThreads + tid)]);
    for (uint64_t s = blockIdx.x; s < a.nseg; s += gridDim.x) {
        f64x16 w;
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            if constexpr (F32) {
                w[2 * k] = prob(make_float2(nx[k].x, nx[k].y));
                w[2 * k + 1] = prob(make_float2(nx[k].z, nx[k].w));
            } else {
                w[k] = prob(nx[k]);
            }
        }
        if (s + gridDim.x < a.nseg) {
#pragma unroll
            for (int k = 0; k < NLD; ++k)
                nx[k] = ldnt(&v[(s + gridDim.x) * (NLD * kThreads) + uint32_t(k * kThreads + tid)]);
        }
        walsh16(w);
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            if constexpr (F32)  // the pair of bit 0 stays adjacent
                *reinterpret_cast<double2 *>(&w_lds[walsh_slot(uint32_t(2 * (k * kThreads + tid)))]) =
                    make_double2(w[2 * k], w[2 * k + 1]);
            else
                w_lds[walsh_slot(uint32_t(k * kThreads + tid))] = w[k];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u)
            w[u] = w_lds[walsh_slot(g2 | u << 1)];
        walsh16(w);
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u)
            w_lds[walsh_slot(g2 | u << 1)] = w[u];
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u)
            w[u] = w_lds[walsh_slot(g3 | r3(u))];
        walsh16(w);
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u)
            w_lds[walsh_slot(g3 | r3(u))] = w[u];
        __syncthreads();
        if (tid < a.nt) {
            const double c = w_lds[walsh_slot(uint32_t(z) & (SEG - 1))];
            acc += (__popcll((s << 12) & z) & 1) ? -c : c;
        }
        __syncthreads();
    }
    if (tid < a.nt)
        part[uint64_t(tid) * gridDim.x + blockIdx.x] = acc;
}

// ---------------------------------------------------------------------------
// Sampling.  Stage 1: sums of |a|^2 over blocks of 2^lbs amplitudes.
// ---------------------------------------------------------------------------
// The block is read in steps of 16 16-byte loads per thread, all issued
// before the first is used (indices past the block end: its first vector,
// weight 0).
template <typename R>
__global__ __launch_bounds__(kThreads) void k_block_sums(const R *__restrict__ st, double *__restrict__ bs,
                                                         int lbs)
{
    constexpr bool F32 = std::is_same<R, float>::value;
    using V = typename std::conditional<F32, float4, double2>::type;  // 16 bytes
    constexpr int NL = 16;
    __shared__ double sh[4];
    const uint32_t nv = F32 ? (1u << lbs) >> 1 : (1u << lbs);  // vectors in the block (lbs >= 1)
    const V *v = reinterpret_cast<const V *>(st) + uint64_t(blockIdx.x) * nv;
    double acc = 0.0;
    for (uint32_t e0 = 0; e0 < nv; e0 += NL * kThreads) {
        V x[NL];
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const uint32_t e = e0 + uint32_t(k * kThreads) + threadIdx.x;
            x[k] = ldnt(&v[e < nv ? e : 0]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            double p;
            if constexpr (F32)
                p = prob(make_float2(x[k].x, x[k].y)) + prob(make_float2(x[k].z, x[k].w));
            else
                p = prob(x[k]);
            acc += e0 + uint32_t(k * kThreads) + threadIdx.x < nv ? p : 0.0;
        }
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0)
        bs[blockIdx.x] = acc;
}

// Stage 1b (one workgroup): each shot's block and residual target from the
// block totals, on the device.  Thread c sums the totals of chunk c (nb / 1024
// consecutive blocks, or one block when nb < 1024) in order; running sums over
// the chunks go in groups of 32: within a group, over the groups, and back.
// Shot s targets t = u_s * norm and takes the first block whose running sum
// (chunk start + in-chunk partial sum, added in the same order as the chunk
// total) exceeds t, with residual t minus the running sum before that block.
// Every running sum over chunks is a start plus a sum of nonnegative terms in
// one fixed order, and the next start is that sum at its end, so they never
// decrease.  Where rounding lets a chunk's walk end just short of the next
// chunk's start, the shot takes the chunk's last block of nonzero total, and a
// target at or past the total the last such block of all, each with that total
// as residual.
// (One thread adding up all 1024 chunks took most of 47 us at 2^14 blocks; now
// 16.)
constexpr int kPrepThreads = 1024;
constexpr int kPrepGroup = 32;

__global__ __launch_bounds__(kPrepThreads) void k_sample_prep(const double *__restrict__ bs, uint64_t nb,
                                                              const double *__restrict__ uni, int shots,
                                                              int64_t *__restrict__ blk, double *__restrict__ tgt)
{
    constexpr int NG = kPrepThreads / kPrepGroup;
    __shared__ double csum[kPrepThreads];
    __shared__ double cpre[kPrepThreads + 1];
    __shared__ double gsum[NG];
    __shared__ double gpre[NG + 1];
    __shared__ int64_t cnz[kPrepThreads];
    __shared__ int64_t gnz[NG];
    __shared__ int64_t s_last;
    const int tid = threadIdx.x;
    const uint64_t nchunk = nb < uint64_t(kPrepThreads) ? nb : uint64_t(kPrepThreads);
    const uint64_t cl = nb / nchunk;  // nb is a power of two
    {
        double acc = 0.0;
        int64_t nz = -1;
        if (uint64_t(tid) < nchunk) {
            const double *c = bs + uint64_t(tid) * cl;
            uint64_t b = 0;
            for (; b + 8 <= cl; b += 8) {  // eight loads in flight
                double x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    x[i] = c[b + i];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    acc += x[i];
                    nz = x[i] > 0.0 ? int64_t(uint64_t(tid) * cl + b + i) : nz;
                }
            }
            for (; b < cl; ++b) {
                const double x = c[b];
                acc += x;
                nz = x > 0.0 ? int64_t(uint64_t(tid) * cl + b) : nz;
            }
        }
        csum[tid] = acc;  // chunks past the last one: 0
        cnz[tid] = nz;
    }
    __syncthreads();
    // groups, and chunks of this thread's group, that there are (few states of
    // many qubits fill them: the sums are chains of LDS reads)
    const int ng = int((nchunk + kPrepGroup - 1) / kPrepGroup), in_group = nchunk < kPrepGroup ? int(nchunk) : kPrepGroup;
    if (tid < ng) {
        double run = 0.0;
        int64_t last = -1;
        for (int c = 0; c < in_group; ++c) {
            run += csum[tid * kPrepGroup + c];
            last = cnz[tid * kPrepGroup + c] >= 0 ? cnz[tid * kPrepGroup + c] : last;
        }
        gsum[tid] = run;
        gnz[tid] = last;
    }
    __syncthreads();
    if (tid == 0) {
        double run = 0.0;
        int64_t last = 0;
        for (int c = 0; c < ng; ++c) {
            gpre[c] = run;
            run += gsum[c];
            last = gnz[c] >= 0 ? gnz[c] : last;
        }
        gpre[ng] = run;
        s_last = last;
    }
    __syncthreads();
    if (tid < ng) {
        const double start = gpre[tid];
        double part = 0.0;
        for (int c = 0; c < in_group; ++c) {
            cpre[tid * kPrepGroup + c] = start + part;
            part += csum[tid * kPrepGroup + c];
        }
        if (tid == ng - 1)
            cpre[nchunk] = gpre[ng];
    }
    __syncthreads();
    const double norm = cpre[nchunk];
    for (int sh = tid; sh < shots; sh += kPrepThreads) {
        const double t = uni[sh] * norm;
        uint64_t lo = 0, hi = nchunk;  // first chunk c with cpre[c + 1] > t
        while (lo < hi) {
            const uint64_t mid = (lo + hi) >> 1;
            if (cpre[mid + 1] > t)
                hi = mid;
            else
                lo = mid + 1;
        }
        int64_t b_out = lo < nchunk ? cnz[lo] : s_last;  // a chunk whose sum moved past t holds a nonzero block
        double t_out = bs[b_out];
        if (lo < nchunk) {
            const double start = cpre[lo];
            double part = 0.0;
            bool hit = false;
            for (uint64_t b = lo * cl; b < (lo + 1) * cl && !hit; b += 8) {
                double x[8];  // loads in flight together; past the chunk: 0
#pragma unroll
                for (uint64_t i = 0; i < 8; ++i)
                    x[i] = i < cl ? bs[b + i] : 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const double before = part;
                    part += x[i];
                    if (!hit && start + part > t) {
                        hit = true;
                        b_out = int64_t(b + i);
                        t_out = t - (start + before);
                    }
                }
            }
        }
        blk[sh] = b_out;
        tgt[sh] = t_out;
    }
}

// Stage 2: one workgroup per shot.  The sums of the block's segments of 1024
// amplitudes, ROUND segments at a time with their loads in flight together (0:
// the block is one segment), name the segment to start in; from there the block
// is walked in segments (4 consecutive amplitudes per thread) to the first
// amplitude of nonzero probability whose in-block running sum exceeds the
// residual target.  If rounding leaves none, the last index of nonzero
// probability seen is returned.  (Walking from the block's start, each segment
// waits for memory: 73 us for 1000 shots in 2^14-amplitude blocks at 28 qubits,
// against 31 with eight segments at a time.  Many shots are bound by the bytes
// read: a million at 24 qubits complex128 take 25 ms with four segments at a
// time, 30 with eight, 39 where every segment is summed, 28 by the walk.)  Many
// shots want eight wavefronts per SIMD (with 84 registers a million of an
// 8-qubit complex128 state took 5.6 ms instead of 4.5), few the registers for
// their loads (1000 at 20 qubits complex64: 47 us, 60 with 64 registers).
constexpr int kSearchSegLog = 10;
constexpr int kSearchMaxLog = 16;
constexpr int kSearchMany = 4096;  // shots that keep every CU's memory pipes busy

template <typename R, int ROUND>
__global__ __launch_bounds__(kThreads, ROUND == 8 ? 4 : 8) void k_sample_search(const R *__restrict__ st,
                                                               const int64_t *__restrict__ blocks,
                                                               const double *__restrict__ targets,
                                                               int64_t *__restrict__ out, int lbs)
{
    using C = typename CT<R>::C;
    constexpr int SEG = 1 << kSearchSegLog;
    static_assert(SEG == 4 * kThreads, "four amplitudes per thread");
    __shared__ double wsum[4];
    __shared__ double ssum[1 << (kSearchMaxLog - kSearchSegLog)];
    __shared__ int found;
    __shared__ int lastnz;
    const C *v = reinterpret_cast<const C *>(st);
    const int s = blockIdx.x;
    const uint64_t base = uint64_t(blocks[s]) << lbs;
    const double target = targets[s];
    const int bsz = 1 << lbs;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) {
        found = 0x7fffffff;
        lastnz = -1;
    }
    double running = 0.0;
    int seg0 = 0;
    if constexpr (ROUND > 0) {
        // ROUND segments at a time, up to the first whose end passes the target,
        // else the last of nonzero sum
        const int nseg = bsz >> kSearchSegLog;
        int last = 0;
        double before = 0.0, lastbefore = 0.0;
        bool hit = false;
        for (int g0 = 0; g0 < nseg && !hit; g0 += ROUND) {
            const int g = g0 + w;
            if (g < nseg) {
                const C *va = v + base + (uint64_t(g) << kSearchSegLog);
                const bool two = ROUND > 4 && g + 4 < nseg;
                const C *vb = two ? va + 4 * SEG : va;
                double sa = 0.0, sb = 0.0;
#pragma unroll
                for (int k = 0; k < SEG / 64; ++k) {
                    sa += prob(va[k * 64 + lane]);
                    if constexpr (ROUND > 4)
                        sb += prob(vb[k * 64 + lane]);
                }
                sa = wave_sum(sa);
                if constexpr (ROUND > 4)
                    sb = wave_sum(sb);
                if (lane == 0) {
                    ssum[g] = sa;
                    if (two)
                        ssum[g + 4] = sb;
                }
            }
            __syncthreads();
            for (int i = g0; i < nseg && i < g0 + ROUND && !hit; ++i) {
                const double x = ssum[i];
                if (x > 0.0) {
                    last = i;
                    lastbefore = before;
                }
                before += x;
                hit = before > target;
            }
        }
        seg0 = last << kSearchSegLog;
        running = lastbefore;
    }
    __syncthreads();
    for (int seg = seg0; seg < bsz; seg += SEG) {
        double c[4], pe[4];
        double acc = 0.0;
        int mynz = -1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int off = seg + tid * 4 + e;
            double p = 0.0;
            if (off < bsz)
                p = prob(v[base + off]);
            if (p > 0.0)
                mynz = off;
            acc += p;
            c[e] = acc;
            pe[e] = p;
        }
        // inclusive scan of thread totals within the wave
        double inc = acc;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double o = __shfl_up(inc, d, 64);
            if (lane >= d)
                inc += o;
        }
        if (lane == 63)
            wsum[w] = inc;
        __syncthreads();
        double wprefix = 0.0;
        for (int j = 0; j < w; ++j)
            wprefix += wsum[j];
        const double seg_total = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
        const double excl = running + wprefix + (inc - acc);
        int cand = 0x7fffffff;
#pragma unroll
        for (int e = 3; e >= 0; --e)
            if (excl + c[e] > target && pe[e] > 0.0)
                cand = seg + tid * 4 + e;
        if (cand != 0x7fffffff)
            atomicMin(&found, cand);
        if (mynz >= 0)
            atomicMax(&lastnz, mynz);
        __syncthreads();
        const int f = found;
        if (f != 0x7fffffff) {
            if (tid == 0)
                out[s] = int64_t(base + uint64_t(f));
            return;
        }
        running += seg_total;
        __syncthreads();
    }
    if (tid == 0)
        out[s] = int64_t(base + uint64_t(lastnz >= 0 ? lastnz : bsz - 1));
}

// out[x] = sum over r of p[dep(x, Q') | ins(r, Q')] on a FP64 array of 2^nb values.
__global__ __launch_bounds__(kThreads) void k_marg_doubles(const double *__restrict__ p, double *__restrict__ out,
                                                           const MargArgs a)
{
    const uint64_t stride = uint64_t(gridDim.x) * kThreads;
    for (uint64_t x = uint64_t(blockIdx.x) * kThreads + threadIdx.x; x < a.nbins; x += stride) {
        const uint64_t xq = dep_x(x, a);
        double acc = 0.0;
        for (uint64_t r = 0; r < a.rest; ++r)
            acc += p[xq | insert_zeros(r, a.rest_im)];
        out[x] = acc;
    }
}

// ---------------------------------------------------------------------------
// Marginal, stage 1: fold each 4096-amplitude segment (index bits 0..11) onto
// its 2^lb bins (the bin bits among bits 0..11, none: the segment's sum),
// summing per workgroup the 2^F segments that F index bits above, not bins,
// tell apart (foldmask; the lowest such bits).
// red[(block << lb) | bin] = sum over the workgroup's segments and the
// segment's non-bin bits.  Every thread keeps the sums over the segments of its
// own 16 amplitudes of a segment in registers; they meet in LDS once, after the
// last segment, where each bin is summed by G consecutive lanes over
// interleaved rest indices and combined by a fixed shuffle tree, so the order
// of every sum is fixed.  (Through LDS with two barriers per segment: 486 us
// for 9 low bins with 32 Z strings and block totals at 28 qubits c64, 863 us
// for 10, against 365 and 398.)
// A thread's loads of one segment differ only in the index bits from
// fold_low_bits() up: 9..11 for c64 (a 16-byte load holds the two amplitudes
// of bit 0, the lane gives bits 1..8), 8..11 for c128 (the lane gives bits
// 0..7).  When none of those bits is a bin bit (KSUM), one or two sums per
// thread are enough and the LDS array shrinks to the 2^fold_low_bits() low-bit
// entries (4 or 2 KiB instead of 32), which leaves room for more resident
// workgroups to keep loads in flight.
// ---------------------------------------------------------------------------
constexpr int kSegLog = 12;
struct FoldArgs {
    uint32_t binmask;   // bin bits among the segment's 12 bits
    uint32_t restmask;  // the other segment bits
    int lb;             // popcount(binmask)
    int F;              // log2 segments per workgroup
    uint64_t foldmask;  // the F index bits that tell them apart
    Masks outer;        // inserts zeros there
};

// Index of the first amplitude of segment j of workgroup `block`.
__device__ __forceinline__ uint64_t fold_base(uint64_t block, uint32_t j, const FoldArgs &a)
{
    uint64_t i = insert_zeros(block << kSegLog, a.outer);
    for (uint64_t m = a.foldmask; j != 0; m &= m - 1, j >>= 1)
        if (j & 1)
            i |= m & (~m + 1);
    return i;
}

template <typename R>
constexpr int fold_low_bits()
{
    return std::is_same<R, float>::value ? 9 : 8;
}

// x-th value (ascending) of the integers whose set bits lie in mask.
__device__ __forceinline__ uint32_t deposit(uint32_t x, uint32_t mask)
{
    uint32_t r = 0;
    for (uint32_t m = mask; x && m; m &= m - 1, x >>= 1)
        if (x & 1)
            r |= m & (~m + 1);
    return r;
}

// Optional outputs of the same read (one read of the state for several
// read-outs): NZ > 0, the partial sums of nt <= NZ Z strings (as k_expect_z:
// a Walsh transform over the thread's 16 amplitudes of a segment, indexed by
// the index bits its loads differ in, picks one coefficient per string; the
// segment's higher bits give a workgroup-uniform sign and the lane's bits a
// sign applied once at the end), part[t * grid + block]; TOT, the total
// probability of every 2^tlog consecutive segments in index order (the lowest
// tlog bits of foldmask are bits 12 .. 12 + tlog - 1).
struct ReadoutArgs {
    uint64_t z[kMaxZ];
    int nt;
    int tlog;
    double *zpart;
    double *tot;
};

template <typename R, bool KSUM, int NZ = 0, bool TOT = false>
__global__ __launch_bounds__(kThreads) void k_marg_fold(const R *__restrict__ st, double *__restrict__ red,
                                                        const FoldArgs a, const ReadoutArgs ra)
{
    static_assert(NZ <= kMaxZ && NZ <= 64, "one string per lane");
    constexpr int SEG = 1 << kSegLog;
    constexpr int LOW = fold_low_bits<R>();
    constexpr int PR = KSUM ? (1 << LOW) : SEG;  // LDS entries per segment
    constexpr int MAXB = (PR + kThreads - 1) / kThreads;  // bins per thread when every thread owns whole bins
    constexpr bool F32 = std::is_same<R, float>::value;
    constexpr int NLD = F32 ? SEG / (2 * kThreads) : SEG / kThreads;  // loads per thread per segment
    constexpr int NR = PR / kThreads;  // sums per thread
    __shared__ double pr[PR];
    static_assert(4 * (NZ > 0 ? NZ : 1) <= PR, "the strings' sums reuse pr");
    __shared__ double sh_tot[TOT ? 4 : 1];
    const int tid = threadIdx.x;
    const uint32_t restmask = KSUM ? (a.restmask & uint32_t(PR - 1)) : a.restmask;
    const int B = 1 << a.lb;
    const int E = PR >> a.lb;  // LDS entries per bin
    const int G = B >= kThreads ? 1 : min(64, kThreads / B);
    const int gi = tid % G;
    const int bin0 = tid / G;
    const bool owner_mode = B >= kThreads;
    f64x16 own = 0.0;  // NR of them used
    // Z strings: the lane reports string `lane`'s segment parity by ballot;
    // walsh index of a string: its bits among the loads' varying index bits
    const int lane = tid & 63;
    const uint64_t zl = (NZ > 0 && lane < NZ) ? ra.z[lane] : 0;
    double zacc[NZ > 0 ? NZ : 1];
#pragma unroll
    for (int t = 0; t < (NZ > 0 ? NZ : 1); ++t)
        zacc[t] = 0.0;
    double tsum = 0.0;
    // complex64: the next segment's loads are issued before the current
    // segment's arithmetic (a vector value: registers, not private memory)
    typedef float f32xL __attribute__((ext_vector_type(F32 ? 4 * NLD : 4)));
    f32xL qn;
    if constexpr (F32) {
        const float4 *v4 = reinterpret_cast<const float4 *>(st) + (fold_base(blockIdx.x, 0, a) >> 1);
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const float4 q = ldnt(&v4[tid + k * kThreads]);
            qn[4 * k] = q.x, qn[4 * k + 1] = q.y, qn[4 * k + 2] = q.z, qn[4 * k + 3] = q.w;
        }
    }
    for (uint32_t j = 0; j < (1u << a.F); ++j) {
        const uint64_t base = fold_base(blockIdx.x, j, a);
        // the thread's 16 probabilities, by the index bits its loads differ in
        // (c64: bit 0 and bits 9..11, as 2 k + c; c128: bits 8..11, as k); a
        // vector value, so that picking a string's coefficient by its
        // (uniform) index indexes registers rather than private memory
        f64x16 w;
        if constexpr (F32) {
            const f32xL qc = qn;
            if (j + 1 < (1u << a.F)) {
                const float4 *v4 = reinterpret_cast<const float4 *>(st) + (fold_base(blockIdx.x, j + 1, a) >> 1);
#pragma unroll
                for (int k = 0; k < NLD; ++k) {
                    const float4 q = ldnt(&v4[tid + k * kThreads]);
                    qn[4 * k] = q.x, qn[4 * k + 1] = q.y, qn[4 * k + 2] = q.z, qn[4 * k + 3] = q.w;
                }
            }
#pragma unroll
            for (int k = 0; k < NLD; ++k) {
                const float4 q = make_float4(qc[4 * k], qc[4 * k + 1], qc[4 * k + 2], qc[4 * k + 3]);
                const double p0 = double(q.x) * q.x + double(q.y) * q.y;
                const double p1 = double(q.z) * q.z + double(q.w) * q.w;
                w[2 * k] = p0;
                w[2 * k + 1] = p1;
            }
        } else {
            const double2 *v2 = reinterpret_cast<const double2 *>(st) + base;
#pragma unroll
            for (int k = 0; k < NLD; ++k) {
                const double2 q = ldnt(&v2[tid + k * kThreads]);
                w[k] = q.x * q.x + q.y * q.y;
            }
        }
        // the thread's own sums over the segments: by load (and by bit 0),
        // or over the loads where no bin tells them apart
        double sums[KSUM && F32 ? 2 : 1] = {};
        if constexpr (KSUM || TOT) {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                sums[KSUM && F32 ? k & 1 : 0] += w[k];
        }
        if constexpr (KSUM) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                own[k] += sums[k];
        } else {
            own += w;
        }
        if constexpr (TOT)
            tsum += KSUM && F32 ? sums[0] + sums[KSUM && F32 ? 1 : 0] : sums[0];
        if constexpr (NZ > 0) {
            static_assert(NZ == 0 || NLD * (F32 ? 2 : 1) == 16, "16 probabilities per thread and segment");
            // w[k] <- sum_u (-1)^popcount(u & k) p_u
#pragma unroll
            for (int b = 1; b < 16; b <<= 1)
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    if (!(u & b)) {
                        const double x = w[u], y = w[u | b];
                        w[u] = x + y;
                        w[u | b] = x - y;
                    }
            const uint64_t sgn = __ballot((__popcll(base & zl) & 1) != 0);
#pragma unroll
            for (int t = 0; t < NZ; ++t) {
                const uint64_t zt = ra.z[t];
                const int k = F32 ? int((zt & 1) | (((zt >> 9) & 7) << 1)) : int((zt >> 8) & 15);
                zacc[t] = fma(((sgn >> t) & 1) ? -1.0 : 1.0, w[k], zacc[t]);
            }
        }
        if constexpr (TOT) {
            if (((j + 1) & ((1u << ra.tlog) - 1)) == 0) {
                const double tt = block_sum(tsum, sh_tot);
                if (tid == 0)
                    ra.tot[base >> (kSegLog + ra.tlog)] = tt;
                tsum = 0.0;
            }
        }
    }
    const bool one_bin = KSUM && a.lb == 0;
    if (!one_bin) {
        // thread tid's own[k] is entry 2 tid + 512 (k / 2) + k % 2 (c64) or
        // tid + 256 k (c128)
#pragma unroll
        for (int k = 0; k < NR; ++k)
            pr[F32 ? 2 * tid + 2 * kThreads * (k >> 1) + (k & 1) : tid + kThreads * k] = own[k];
        __syncthreads();
    }
    const uint64_t out0 = uint64_t(blockIdx.x) << a.lb;
    if (one_bin) {
        // no bin below bit 12: the group mode's 64 lanes would walk the 512
        // (256) entries while the rest of the workgroup waits
        double all = own[0];
#pragma unroll
        for (int k = 1; k < (KSUM ? NR : 1); ++k)
            all += own[k];
        all = block_sum(all, pr);
        if (tid == 0)
            red[out0] = all;
    } else if (owner_mode) {
        // bins tid, tid + 256, ...; E <= 16 entries each, ascending
#pragma unroll
        for (int k = 0; k < MAXB; ++k) {
            const int bin = tid + k * kThreads;
            if (bin < B) {
                const uint32_t db = deposit(uint32_t(bin), a.binmask);
                double sacc = 0.0;
                uint32_t x = 0;
                for (int r = 0; r < E; ++r) {
                    sacc += pr[db | x];
                    x = ((x | ~restmask) + 1u) & restmask;
                }
                red[out0 + bin] = sacc;
            }
        }
    } else if (bin0 < B) {
        // the bin's entries x_r = deposit(r, restmask), r = gi, gi + G, ...
        const uint32_t x_step = deposit(uint32_t(G), restmask);
        const uint32_t d_bin0 = deposit(uint32_t(bin0), a.binmask);
        double sacc = 0.0;
        uint32_t x = deposit(uint32_t(gi), restmask);
        for (int r = gi; r < E; r += G) {
            sacc += pr[d_bin0 | x];
            x = ((x | ~restmask) + x_step) & restmask;
        }
        for (int off = 1; off < G; off <<= 1)
            sacc += __shfl_xor(sacc, off, 64);
        if (gi == 0)
            red[out0 + bin0] = sacc;
    }
    if constexpr (NZ > 0) {
        // the lane's index bits: c64 bits 1..8, c128 bits 0..7
        const uint32_t lbits = F32 ? uint32_t(tid) << 1 : uint32_t(tid);
#pragma unroll
        for (int t = 0; t < NZ; ++t)
            zacc[t] = (__popc(lbits & uint32_t(ra.z[t])) & 1) ? -zacc[t] : zacc[t];
        __syncthreads();  // pr is read no more
        block_sums<NZ>(zacc, pr, [&](int t, double x) {
            if (t < ra.nt)
                ra.zpart[uint64_t(t) * gridDim.x + blockIdx.x] = x;
        });
    }
}

// Row-major bin sums over an array of doubles (stage 2 of the folded
// marginal): block (chunk, x) sums one bin over a contiguous rest range.
__global__ __launch_bounds__(kThreads) void k_marg_rmajor_d(const double *__restrict__ p, double *__restrict__ part,
                                                            const MargArgs a)
{
    __shared__ double sh[4];
    const uint64_t x = blockIdx.y;
    const uint64_t xq = dep_x(x, a);
    const uint64_t r0 = uint64_t(blockIdx.x) * a.per_chunk;
    uint64_t r1 = r0 + a.per_chunk;
    if (r1 > a.rest)
        r1 = a.rest;
    double acc = 0.0;
    for (uint64_t r = r0 + threadIdx.x; r < r1; r += kThreads)
        acc += p[xq | insert_zeros(r, a.rest_im)];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0)
        part[x * a.chunks + blockIdx.x] = acc;
}

}  // namespace

// ===========================================================================
// Launchers
// ===========================================================================
namespace {

struct MargPlan {
    bool rmajor;
    uint32_t chunks;
    uint64_t per_chunk;
};

MargPlan marg_plan(int n, int m)
{
    MargPlan p{};
    const uint64_t rest = uint64_t(1) << (n - m);
    const uint64_t nbins = uint64_t(1) << m;
    p.rmajor = rest >= 4096 && m <= 15;
    if (p.rmajor) {
        uint64_t want = std::max<uint64_t>(1, 4096 / nbins);
        uint64_t maxc = std::max<uint64_t>(1, rest / (kThreads * 16));
        uint64_t chunks = std::min(want, maxc);
        p.chunks = uint32_t(chunks);
        p.per_chunk = (rest + chunks - 1) / chunks;
    } else {
        p.chunks = 1;
        p.per_chunk = rest;
    }
    return p;
}

}  // namespace

namespace {

// Route of a marginal: direct (row- or bin-major over the state), or a segment
// fold followed by row- or bin-major sums over the folded array.
struct MargRoute {
    int kind;             // 0 direct, 1 fold
    FoldArgs fold;        // kind 1
    int n2;               // bits of the folded array (kind 1)
    std::vector<int> q2;  // bin positions in the folded array (kind 1)
    MargPlan p2;          // plan over the folded array (kind 1)
    uint64_t red;         // doubles of the folded array
    uint64_t scratch;     // doubles of scratch in all
};

constexpr uint64_t kMaxFolded = uint64_t(1) << 26;  // doubles
constexpr int kFoldGrid = 12;  // log2 workgroups of a fold, where the bins leave enough bits

// The fold route (n >= kSegLog + 2, or kSegLog where no bin is below bit 12; at
// most 10 such bins): as many
// fold bits as bring the workgroups down to 2^kFoldGrid, so that their partial
// sums stay small against the read.
MargRoute fold_route(int n, int m, const int *phys_q)
{
    MargRoute r{};
    uint32_t binmask = 0;
    uint64_t hibins = 0;
    for (int b = 0; b < m; ++b) {
        if (phys_q[b] < kSegLog)
            binmask |= 1u << phys_q[b];
        else
            hibins |= uint64_t(1) << phys_q[b];
    }
    const int lb = __builtin_popcount(binmask);
    std::vector<int> pos;
    for (int p = kSegLog; p < n && int(pos.size()) < std::min(n - kSegLog - kFoldGrid, n - kSegLog - 1); ++p)
        if (!((hibins >> p) & 1)) {
            pos.push_back(p);
            r.fold.foldmask |= uint64_t(1) << p;
        }
    const int F = int(pos.size());
    const int n2 = n - kSegLog - F + lb;
    r.kind = 1;
    r.fold.binmask = binmask;
    r.fold.restmask = ((1u << kSegLog) - 1u) & ~binmask;
    r.fold.lb = lb;
    r.fold.F = F;
    r.fold.outer = make_masks(pos);
    r.n2 = n2;
    r.red = uint64_t(1) << n2;
    r.q2.resize(size_t(m));
    for (int b = 0; b < m; ++b) {
        const int q = phys_q[b];
        const uint64_t below = (uint64_t(1) << q) - 1;
        r.q2[size_t(b)] = q < kSegLog ? __builtin_popcount(binmask & uint32_t(below))
                                      : lb + q - kSegLog - __builtin_popcountll(r.fold.foldmask & below);
    }
    r.p2 = marg_plan(n2, m);
    if (!r.p2.rmajor && m <= 15 && n2 > m) {
        // few rest entries per bin, but not one: still one workgroup per bin (a
        // thread per bin would leave the GPU nearly empty for up to 2^15 bins)
        r.p2.rmajor = true;
        r.p2.chunks = 1;
        r.p2.per_chunk = uint64_t(1) << (n2 - m);
    }
    r.scratch = r.red + (r.p2.rmajor ? (uint64_t(1) << m) * r.p2.chunks : 0);
    return r;
}

MargRoute marg_route(int n, int m, const int *phys_q)
{
    int lb = 0;
    for (int b = 0; b < m; ++b)
        lb += phys_q[b] < kSegLog ? 1 : 0;
    if (n >= kSegLog + (lb > 0 ? 2 : 0) && lb <= 10) {
        MargRoute r = fold_route(n, m, phys_q);
        if (r.red <= kMaxFolded)
            return r;
    }
    MargRoute r{};
    const MargPlan p = marg_plan(n, m);
    r.kind = 0;
    r.scratch = p.rmajor ? (uint64_t(1) << m) * p.chunks : 1;
    return r;
}

}  // namespace

uint64_t marginal_scratch_doubles(int n, int m, const int *phys_q)
{
    return std::max<uint64_t>(1, marg_route(n, m, phys_q).scratch);
}

hipError_t launch_marginal(const void *st, int n, int dtype, const int *phys_q, int m, double *d_scratch,
                           double *d_out, hipStream_t s)
{
    if (m < 0 || m > kMaxQ || m > n)
        return hipErrorInvalidValue;
    const MargRoute route = marg_route(n, m, phys_q);
    if (route.kind == 1) {
        const uint64_t nblk = uint64_t(1) << (n - kSegLog - route.fold.F);
        if (dtype == SV_C64) {
            if ((route.fold.binmask >> fold_low_bits<float>()) == 0)
                hipLaunchKernelGGL((k_marg_fold<float, true>), dim3(uint32_t(nblk)), dim3(kThreads), 0, s,
                                   (const float *)st, d_scratch, route.fold, ReadoutArgs{});
            else
                hipLaunchKernelGGL((k_marg_fold<float, false>), dim3(uint32_t(nblk)), dim3(kThreads), 0, s,
                                   (const float *)st, d_scratch, route.fold, ReadoutArgs{});
        } else {
            if ((route.fold.binmask >> fold_low_bits<double>()) == 0)
                hipLaunchKernelGGL((k_marg_fold<double, true>), dim3(uint32_t(nblk)), dim3(kThreads), 0, s,
                                   (const double *)st, d_scratch, route.fold, ReadoutArgs{});
            else
                hipLaunchKernelGGL((k_marg_fold<double, false>), dim3(uint32_t(nblk)), dim3(kThreads), 0, s,
                                   (const double *)st, d_scratch, route.fold, ReadoutArgs{});
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        MargArgs a2{};
        a2.m = m;
        a2.rest = uint64_t(1) << (route.n2 - m);
        a2.nbins = uint32_t(1u << m);
        for (int b = 0; b < m; ++b)
            a2.qbit[b] = uint64_t(1) << route.q2[size_t(b)];
        a2.rest_im = make_masks(route.q2);
        a2.chunks = route.p2.chunks;
        a2.per_chunk = route.p2.per_chunk;
        const double *red = d_scratch;
        if (route.p2.rmajor) {
            // (the launch that adds up one chunk: 3 us of a call that takes 20 on
            // small states)
            double *part = a2.chunks == 1 ? d_out : d_scratch + route.red;
            hipLaunchKernelGGL(k_marg_rmajor_d, dim3(a2.chunks, a2.nbins), dim3(kThreads), 0, s, red, part, a2);
            e = hipGetLastError();
            if (e != hipSuccess || a2.chunks == 1)
                return e;
            return launch_sum_rows(part, d_out, uint64_t(a2.nbins), a2.chunks, s);
        } else {
            const uint64_t g = std::min<uint64_t>((uint64_t(a2.nbins) + kThreads - 1) / kThreads, 1u << 20);
            hipLaunchKernelGGL(k_marg_doubles, dim3(g), dim3(kThreads), 0, s, red, d_out, a2);
        }
        return hipGetLastError();
    }
    MargArgs a{};
    a.m = m;
    a.rest = uint64_t(1) << (n - m);
    a.nbins = uint32_t(1u << m);
    for (int b = 0; b < m; ++b)
        a.qbit[b] = uint64_t(1) << phys_q[b];
    a.rest_im = make_masks(std::vector<int>(phys_q, phys_q + m));
    MargPlan p = marg_plan(n, m);
    a.chunks = p.chunks;
    a.per_chunk = p.per_chunk;
    if (p.rmajor) {
        dim3 grid(p.chunks, a.nbins);
        if (dtype == SV_C64)
            hipLaunchKernelGGL(k_marg_rmajor<float>, grid, dim3(kThreads), 0, s, (const float *)st, d_scratch, a);
        else
            hipLaunchKernelGGL(k_marg_rmajor<double>, grid, dim3(kThreads), 0, s, (const double *)st, d_scratch, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        return launch_sum_rows(d_scratch, d_out, uint64_t(a.nbins), p.chunks, s);
    } else {
        const uint64_t g = std::min<uint64_t>((uint64_t(a.nbins) + kThreads - 1) / kThreads, 1u << 20);
        if (dtype == SV_C64)
            hipLaunchKernelGGL(k_marg_xmajor<float>, dim3(g), dim3(kThreads), 0, s, (const float *)st, d_out, a);
        else
            hipLaunchKernelGGL(k_marg_xmajor<double>, dim3(g), dim3(kThreads), 0, s, (const double *)st, d_out, a);
    }
    return hipGetLastError();
}

namespace {
constexpr uint32_t kExpGrid = 4096;
uint32_t exp_grid(int n)
{
    const uint64_t need = ((uint64_t(1) << n) + kThreads * 16 - 1) / (kThreads * 16);
    return uint32_t(std::max<uint64_t>(1, std::min<uint64_t>(kExpGrid, need)));
}
}  // namespace

// ---------------------------------------------------------------------------
// Device scratch of the allocation-free expectation entry point
// (sv_expect_pauli_noalloc): the per-workgroup partial sums of one batch of
// strings, then two result doubles per string.  Every device the library
// runs on holds its own copy until the process ends.  In host code the
// name `scratch` is a host-side stand-in, not a device address: the address
// comes from hipGetSymbolAddress, looked up once per device with that device
// current, and only that address is handed to kernels and copies.
// ---------------------------------------------------------------------------
constexpr uint64_t kNoAllocDoubles = uint64_t(kMaxZ) * kExpGrid + 2 * uint64_t(SV_NOALLOC_MAX_TERMS);
static __device__ __align__(256) double scratch[kNoAllocDoubles];

int noalloc_scratch(int device, double **ptr, uint64_t *doubles)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) {
        set_error("device %d outside 0..%d", device, kMaxDevices - 1);
        return SV_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (addr[device] == nullptr) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess || cur != device) {
            set_error("scratch lookup needs device %d current (current %d)", device, cur);
            return SV_EDEVICE;
        }
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            set_error("hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            return SV_EDEVICE;
        }
        addr[device] = static_cast<double *>(p);
    }
    *ptr = addr[device];
    *doubles = kNoAllocDoubles;
    return SV_OK;
}

uint64_t expect_scratch_doubles(int n)
{
    (void)n;
    return uint64_t(kMaxZ) * kExpGrid;
}

// The Walsh kernel's work does not depend on the strings, this sweep's grows
// with them.  Large complex64 states are read faster by the sweep up to 16
// strings (9 / 16 strings, by it and by the Walsh kernel: 2^25 63 / 64 and 65 /
// 66 us, 2^27 174 / 180 and 190, 2^29 631 / 644 and 689); 2^24 amplitudes stay
// in cache (46 / 47 and 44), and complex128 amplitudes bring half the work a
// byte (2^27, nine strings: 348 and 333).
int expect_z_batch(int n, int dtype)
{
    return dtype == SV_C64 && n >= 25 ? kFewZ : 8;
}

hipError_t launch_expect_z(const void *st, int n, int dtype, const uint64_t *zmasks, int nt, double *d_scratch,
                           double *d_out, hipStream_t s)
{
    if (nt < 1 || nt > expect_z_batch(n, dtype))
        return hipErrorInvalidValue;
    ExpZArgs a{};
    a.nelem = uint64_t(1) << n;
    a.nt = nt;
    for (int t = 0; t < nt; ++t)
        a.z[t] = zmasks[t];
    const uint32_t grid = exp_grid(n);
    const dim3 g(grid), b(kThreads);
    if (dtype == SV_C128)
        hipLaunchKernelGGL((k_expect_z<double, 8>), g, b, 0, s, (const double *)st, d_scratch, a);
    else if (nt <= 8)
        hipLaunchKernelGGL((k_expect_z<float, 8>), g, b, 0, s, (const float *)st, d_scratch, a);
    else
        hipLaunchKernelGGL((k_expect_z<float, kFewZ>), g, b, 0, s, (const float *)st, d_scratch, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_sum_rows(d_scratch, d_out, uint64_t(nt), grid, s);
}

hipError_t launch_expect_xy(const void *st, int n, int dtype, uint64_t xmask, uint64_t yzmask, double *d_scratch,
                            double *d_out2, hipStream_t s)
{
    if (xmask == 0)
        return hipErrorInvalidValue;
    ExpXYArgs a{};
    int h = 63 - __builtin_clzll(xmask);
    a.hmask = (uint64_t(1) << h) - 1;
    a.x = xmask;
    a.yz = yzmask;
    a.npairs = uint64_t(1) << (n - 1);
    const uint32_t grid = exp_grid(n - 1);
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_expect_xy<float>, dim3(grid), dim3(kThreads), 0, s, (const float *)st, d_scratch, a);
    else
        hipLaunchKernelGGL(k_expect_xy<double>, dim3(grid), dim3(kThreads), 0, s, (const double *)st, d_scratch, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_sum_rows(d_scratch, d_out2, uint64_t(2), grid, s);
}

int expect_tile_bits(int dtype)
{
    return dtype == SV_C64 ? expect_tile_log<float>() : expect_tile_log<double>();
}

uint64_t expect_tile_low(int dtype)
{
    return dtype == SV_C64 ? 15 : 7;
}

int expect_tile_batch()
{
    return kTileTerms;
}

int expect_multi_batch()
{
    return kMultiTerms;
}

int expect_walsh_batch()
{
    return kWalshTerms;
}

hipError_t launch_expect_multi(const void *st, int n, int dtype, const uint64_t *x, const uint64_t *yz,
                               const int *ny, int nt, double *d_scratch, double *d_out, hipStream_t s)
{
    if (nt < 1 || nt > kMultiTerms || n < 1 || n > kExpectMultiMax)
        return hipErrorInvalidValue;
    ExpMultiArgs a{};
    for (int t = 0; t < nt; ++t)
        a.t[t] = PauliTerm{x[t], yz[t], uint32_t(ny[t] & 1), 0};
    // 2^12 amplitudes (2^11 pairs) per block
    const uint64_t chunks = n > 12 ? uint64_t(1) << (n - 12) : 1;
    a.per_chunk = (uint64_t(1) << (n - 1)) / chunks;
    double *part = chunks == 1 ? d_out : d_scratch;
    const dim3 g{uint32_t(chunks), uint32_t(nt)}, b{uint32_t(kThreads)};
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_expect_multi<float>, g, b, 0, s, (const float *)st, part, a);
    else
        hipLaunchKernelGGL(k_expect_multi<double>, g, b, 0, s, (const double *)st, part, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || chunks == 1)
        return e;
    if (chunks < 32)
        return launch_sum_rows(d_scratch, d_out, uint64_t(nt), uint32_t(chunks), s);
    // (one thread adding up 128 partial sums: 4 us of a call of 28)
    hipLaunchKernelGGL(k_sum_rows_wide, dim3(uint32_t(nt)), dim3(kThreads), 0, s, d_scratch, d_out, uint32_t(chunks));
    return hipGetLastError();
}

// Workgroups of a persistent expectation sweep over nw work items.
static uint32_t persistent_grid(uint64_t nw, int per_cu)
{
    return uint32_t(std::min<uint64_t>(nw, uint64_t(256) * uint64_t(per_cu)));
}

hipError_t launch_expect_tile(const void *st, int n, int dtype, const uint64_t *x, const uint64_t *yz, const int *ny,
                              int nt, double *d_scratch, double *d_out, hipStream_t s)
{
    const int T = expect_tile_bits(dtype);
    if (nt < 1 || nt > kTileTerms || n < T)
        return hipErrorInvalidValue;
    uint64_t bits = expect_tile_low(dtype);
    for (int t = 0; t < nt; ++t)
        bits |= x[t];
    for (int p = 0; p < n && __builtin_popcountll(bits) < T; ++p)
        bits |= uint64_t(1) << p;
    if (__builtin_popcountll(bits) != T || (bits >> n) != 0)
        return hipErrorInvalidValue;
    ExpTileArgs a{};
    a.ntiles = uint64_t(1) << (n - T);
    a.nt = nt;
    int got = 0;
    for (int p = 0; p < n; ++p) {
        if (!((bits >> p) & 1))
            continue;
        a.dep[got] = uint64_t(1) << p;
        a.outer.m[got] = (uint64_t(1) << p) - 1;
        for (int t = 0; t < nt; ++t) {
            a.xl[t] |= uint32_t((x[t] >> p) & 1) << got;
            a.yl[t] |= uint32_t((yz[t] >> p) & 1) << got;
        }
        ++got;
    }
    a.outer.n = T;
    for (int t = 0; t < nt; ++t) {
        a.yz[t] = yz[t];
        a.odd[t] = uint32_t(ny[t] & 1);
    }
    const uint32_t grid = persistent_grid(a.ntiles, dtype == SV_C64 ? tile_per_cu<float>() : tile_per_cu<double>());
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_expect_tile<float>, dim3(grid), dim3(kThreads), 0, s, (const float *)st, d_scratch, a);
    else
        hipLaunchKernelGGL(k_expect_tile<double>, dim3(grid), dim3(kThreads), 0, s, (const double *)st, d_scratch, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_sum_rows(d_scratch, d_out, uint64_t(nt), grid, s);
}

hipError_t launch_expect_walsh(const void *st, int n, int dtype, const uint64_t *zmasks, int nt, double *d_scratch,
                               double *d_out, hipStream_t s)
{
    if (nt < 1 || nt > kWalshTerms || n < 12)
        return hipErrorInvalidValue;
    ExpWalshArgs a{};
    a.nseg = uint64_t(1) << (n - 12);
    a.nt = nt;
    for (int t = 0; t < nt; ++t)
        a.z[t] = zmasks[t];
    const uint32_t grid = persistent_grid(a.nseg, dtype == SV_C64 ? walsh_per_cu<float>() : walsh_per_cu<double>());
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_expect_walsh<float>, dim3(grid), dim3(kThreads), 0, s, (const float *)st, d_scratch, a);
    else
        hipLaunchKernelGGL(k_expect_walsh<double>, dim3(grid), dim3(kThreads), 0, s, (const double *)st, d_scratch, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_sum_rows(d_scratch, d_out, uint64_t(nt), grid, s);
}

int sample_log_block(int n)
{
    return n < 14 ? n : 14;
}

hipError_t launch_block_sums(const void *st, int n, int dtype, double *d_bsums, hipStream_t s)
{
    const int lbs = sample_log_block(n);
    const uint64_t nb = uint64_t(1) << (n - lbs);
    if (dtype == SV_C64)
        hipLaunchKernelGGL(k_block_sums<float>, dim3(uint32_t(nb)), dim3(kThreads), 0, s, (const float *)st, d_bsums, lbs);
    else
        hipLaunchKernelGGL(k_block_sums<double>, dim3(uint32_t(nb)), dim3(kThreads), 0, s, (const double *)st, d_bsums, lbs);
    return hipGetLastError();
}

hipError_t launch_sample_prep(const double *d_bsums, uint64_t nb, const double *d_uniforms, int shots,
                              int64_t *d_blocks, double *d_targets, hipStream_t s)
{
    if (shots <= 0)
        return hipSuccess;
    if (nb == 0 || (nb & (nb - 1)) != 0)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sample_prep, dim3(1), dim3(kPrepThreads), 0, s, d_bsums, nb, d_uniforms, shots, d_blocks,
                       d_targets);
    return hipGetLastError();
}

hipError_t launch_sample_search(const void *st, int n, int dtype, const int64_t *d_blocks, const double *d_targets,
                                int shots, int64_t *d_out, int lbs, hipStream_t s)
{
    if (shots <= 0 || lbs < 1 || lbs > n || lbs > kSearchMaxLog)
        return hipSuccess;
    auto launch = [&](auto r_tag, auto round_tag) {
        using R = decltype(r_tag);
        hipLaunchKernelGGL((k_sample_search<R, decltype(round_tag)::value>), dim3(shots), dim3(kThreads), 0, s,
                           (const R *)st, d_blocks, d_targets, d_out, lbs);
    };
    auto launch_r = [&](auto round_tag) {
        dtype == SV_C64 ? launch(float{}, round_tag) : launch(double{}, round_tag);
    };
    if (lbs <= kSearchSegLog)
        launch_r(std::integral_constant<int, 0>{});
    else if (shots < kSearchMany)
        launch_r(std::integral_constant<int, 8>{});
    else
        launch_r(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused read-out: one k_marg_fold launch over the state gives the marginal's
// fold (when it takes the register-summed fold route), the partial sums of up
// to kMaxZ Z strings and the block totals for sampling; then the marginal's
// second stage and the Z reduction.
// ---------------------------------------------------------------------------
namespace {

// Route of the fused launch; false where the marginal takes another route.
// m = 0: a fold with no bin bits (the total only).
bool fused_route(int n, int m, const int *phys_q, MargRoute &r)
{
    if (n < kSegLog + 2)
        return false;
    r = marg_route(n, m, phys_q);
    return r.kind == 1;
}

// Consecutive segments whose total one workgroup forms (log2, at most 2).
int total_log(const FoldArgs &f)
{
    if (!((f.foldmask >> kSegLog) & 1))
        return 0;
    return ((f.foldmask >> (kSegLog + 1)) & 1) ? 2 : 1;
}

}  // namespace

static_assert(kMaxZ == kReadoutMaxZ, "Z strings of one fused read-out");

bool readout_fusable(int n, int m, const int *phys_q)
{
    MargRoute r;
    return fused_route(n, m, phys_q, r);
}

int readout_log_block(int n, int m, const int *phys_q)
{
    MargRoute r;
    if (!fused_route(n, m, phys_q, r))
        return -1;
    return kSegLog + total_log(r.fold);
}

uint64_t readout_scratch_doubles(int n, int m, const int *phys_q, int nt)
{
    MargRoute r;
    if (!fused_route(n, m, phys_q, r))
        return 0;
    const uint64_t nblk = uint64_t(1) << (n - kSegLog - r.fold.F);
    return r.scratch + uint64_t(nt) * nblk;
}

hipError_t launch_readout(const void *st, int n, int dtype, const int *phys_q, int m, const uint64_t *zmasks,
                          int nt, double *d_scratch, double *d_marg, double *d_z, double *d_tot, hipStream_t s)
{
    MargRoute r;
    if (nt < 0 || nt > kMaxZ || !fused_route(n, m, phys_q, r))
        return hipErrorInvalidValue;
    const uint64_t nblk = uint64_t(1) << (n - kSegLog - r.fold.F);
    ReadoutArgs ra{};
    ra.nt = nt;
    for (int t = 0; t < nt; ++t)
        ra.z[t] = zmasks[t];
    ra.tlog = total_log(r.fold);
    ra.zpart = d_scratch + r.scratch;
    ra.tot = d_tot;
    const dim3 g{uint32_t(nblk)}, b{uint32_t(kThreads)};
    auto launch = [&](auto r_tag, auto ksum_tag) {
        using R = decltype(r_tag);
        constexpr bool KSUM = decltype(ksum_tag)::value;
        const R *p = static_cast<const R *>(st);
        if (nt > 0)
            hipLaunchKernelGGL((k_marg_fold<R, KSUM, kMaxZ, true>), g, b, 0, s, p, d_scratch, r.fold, ra);
        else
            hipLaunchKernelGGL((k_marg_fold<R, KSUM, 0, true>), g, b, 0, s, p, d_scratch, r.fold, ra);
    };
    if (dtype == SV_C64) {
        if ((r.fold.binmask >> fold_low_bits<float>()) == 0)
            launch(float{}, std::true_type{});
        else
            launch(float{}, std::false_type{});
    } else {
        if ((r.fold.binmask >> fold_low_bits<double>()) == 0)
            launch(double{}, std::true_type{});
        else
            launch(double{}, std::false_type{});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (nt > 0) {
        e = launch_sum_rows(ra.zpart, d_z, uint64_t(nt), uint32_t(nblk), s);
        if (e != hipSuccess)
            return e;
    }
    if (m == 0 || !d_marg)
        return hipSuccess;
    MargArgs a2{};
    a2.m = m;
    a2.rest = uint64_t(1) << (r.n2 - m);
    a2.nbins = uint32_t(1u << m);
    for (int b2 = 0; b2 < m; ++b2)
        a2.qbit[b2] = uint64_t(1) << r.q2[size_t(b2)];
    a2.rest_im = make_masks(r.q2);
    a2.chunks = r.p2.chunks;
    a2.per_chunk = r.p2.per_chunk;
    if (r.p2.rmajor) {
        double *part = d_scratch + r.red;
        hipLaunchKernelGGL(k_marg_rmajor_d, dim3(a2.chunks, a2.nbins), dim3(kThreads), 0, s, d_scratch, part, a2);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        return launch_sum_rows(part, d_marg, uint64_t(a2.nbins), a2.chunks, s);
    }
    const uint64_t gg = std::min<uint64_t>((uint64_t(a2.nbins) + kThreads - 1) / kThreads, 1u << 20);
    hipLaunchKernelGGL(k_marg_doubles, dim3(gg), dim3(kThreads), 0, s, d_scratch, d_marg, a2);
    return hipGetLastError();
}

}  // namespace sv
