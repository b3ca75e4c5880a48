// Circuits on small states: one launch, one workgroup, the state in LDS.
//
// A state of at most 2^13 complex64 or 2^12 complex128 amplitudes is 64 KiB: it
// fits the LDS of one CU.  A sweep of it by a launch of its own takes 1.5-5 us
// of kernel and about 4 us of launch, nearly all latency; here the state is
// read once, every gate or fused block is one step over it in LDS (paper Sec.
// 2.1: gate application as sweeps over the amplitudes), and it is written back
// once.  What bounds a step is the chain barrier - LDS read - arithmetic - LDS
// write, so the step records and the matrices are in LDS too, loaded for as
// many steps at a time as fit beside the state.
//
// Measured on MI355X, a circuit per call: 256 gates on 11 qubits complex64
// (one sweep per gate) 105 us against 700-1020 us by launches; 29 blocks of up
// to five qubits on 12 qubits complex128 125 us of kernel against 171 us of
// kernels and 320-350 us by launches.  A one-target step takes 0.27 us at 8
// qubits, where it is a chain of latencies (about 340 cycles to read and
// decode, 430 to address and read the pair, 320 to compute and write, 90 in
// the barrier), 0.40 us at 11 and 0.90 us at 13, where the vector unit of the
// one CU bounds it (at 11 it is busy for 95 % of the cycles).  Workgroups of 256
// and 512 threads were as fast up to 10 qubits and 1.4x and 1.1x slower at 13.
// Applying runs of gates to groups of eight amplitudes in registers (one LDS
// round trip per run) was slower: the uniform dispatch on each gate's target
// and controls took 0.75 us a gate.
//
// Steps use the arithmetic of the per-launch kernels: one-target gates as
// complex 2 x 2 products, blocks of two targets (three below 8 qubits) on the
// vector unit, wider ones on the FP32 / FP64 matrix cores.  A complex product
// is three real ones where the launch of that size takes three (complex64 from
// 12 qubits on, complex128 from 10, for five and six targets from 11); below,
// the launches multiply on the vector unit with four, and the steps take four
// sums, one per product (three products, or the four in two sums, would raise
// the error of a block by a factor of up to 1.4: the vector unit adds the two
// products of a term before it adds them to the sum).
#include <cstring>

#include "sv_device.h"
#include "sv_internal.h"

namespace sv {
namespace {

using namespace dev;

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;

enum : uint32_t {
    kStepGate = 0,    // one target, any controls
    kStepDense2 = 1,  // two targets, one group per thread
    kStepDense3 = 2,
    kStepDense = 3,   // any width, one output per thread: fewer than 16 groups, or many controls
    kStepMfma4 = 4,   // four, five, six targets on the matrix cores, four real products
    kStepMfma5 = 5,
    kStepMfma6 = 6,
    kStepMfma4t = 7,  // the same in three real products
    kStepMfma5t = 8,
    kStepMfma6t = 9,
};

// One step of two or more targets.
struct SmallStep {
    uint32_t ones;      // fixed one bits
    uint32_t ins;       // index bits that the group index leaves out
    uint32_t mat;       // byte offset of its matrix among those in LDS
    uint32_t kind;      // kStep* | targets << 8 | index bits left out << 16
    uint32_t tbits[3];  // index bit of target b, 16 bits each
    uint32_t lo[3];     // up to six index bits left out: their insert masks 2^p - 1, ascending, 16 bits
                        // each (0xffff: none)
    uint32_t load;      // byte offset in the program of the matrices to load into LDS before this step
    uint32_t units;     // 16-byte units of them, 0: this step's matrix is there
};
static_assert(sizeof(SmallStep) == 48, "table layout");

// One one-target step, with its 2 x 2 matrix (u00 u01 u10 u11) behind it.
struct SmallGate {
    uint32_t lo;     // 2^target - 1
    uint32_t ctl;    // control bits
    uint32_t pt;     // LDS byte offset between the two amplitudes of a pair
    uint32_t kind;   // kStepGate | kGate* << 8 | one-target steps from here on in this chunk << 16
    uint32_t pad[8];
};
static_assert(sizeof(SmallGate) == sizeof(SmallStep), "table layout");
constexpr uint32_t kGateDiag = 1;  // diagonal: a pair's amplitudes do not mix
constexpr uint32_t kGateKeep = 2;  // ... and the lower one stays as it is (d0 = 1)

template <typename R>
constexpr uint32_t record_bytes()
{
    return uint32_t(sizeof(SmallStep) + 4 * sizeof(typename CT<R>::C));
}
constexpr uint32_t kChunk = 192;  // step records in LDS at a time
constexpr uint32_t kLdsBytes = 160 << 10;

struct SmallArgs {
    const char *blob;     // records, then large matrices
    uint32_t nsteps;
    uint32_t mbuf_bytes;  // LDS for large matrices
    int n;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
template <typename R>
struct SmallAcc;
template <>
struct SmallAcc<float> {
    using T = floatx4;
};
template <>
struct SmallAcc<double> {
    using T = doublex4;
};
__device__ __forceinline__ floatx4 mma(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mma(double a, double b, doublex4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t uni(uint32_t x)
{
    return uint32_t(__builtin_amdgcn_readfirstlane(int(x)));
}

// U: pairs per thread (2^(n - 1) pairs, at least one).
template <typename R, int U>
__global__ __launch_bounds__(kSmallThreads) void k_small(R *__restrict__ st, const SmallArgs a)
{
    using C = typename CT<R>::C;
    using AccT = typename SmallAcc<R>::T;
    constexpr bool F64 = std::is_same<R, double>::value;
    constexpr uint32_t REC = record_bytes<R>();
    constexpr uint32_t NT = kSmallThreads;
    extern __shared__ __align__(16) unsigned char smem[];
    const int n = a.n;
    const uint32_t npairs = 1u << (n - 1);
    unsigned char *tile = smem;
    unsigned char *mbuf = smem + (sizeof(C) << n);
    unsigned char *tab = mbuf + a.mbuf_bytes;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = uni(tid >> 6), lane = tid & 63;
    auto at = [&](uint32_t off) __attribute__((always_inline)) -> C & { return *reinterpret_cast<C *>(tile + off); };
    // bits 7..11 folded onto bits 1..5: linear over XOR, pairs stay adjacent
    auto slot = [](uint32_t x) __attribute__((always_inline)) { return (x ^ ((x >> 6) & 62u)) * uint32_t(sizeof(C)); };

    const uint32_t nvec = uint32_t(sizeof(C) << n) / 16;
    constexpr uint32_t PERV = 16 / sizeof(C);  // amplitudes per 16-byte vector
    const uint4 *g = reinterpret_cast<const uint4 *>(st);
    for (uint32_t i = tid; i < nvec; i += NT)
        *reinterpret_cast<uint4 *>(tile + slot(i * PERV)) = g[i];
    // (The barrier that ended the step before also ended its reads of the
    // table.)
    auto load_table = [&](uint32_t s) __attribute__((always_inline)) {
        const uint32_t left = a.nsteps - s, m = (left < kChunk ? left : kChunk) * (REC / 16);
        const uint4 *src = reinterpret_cast<const uint4 *>(a.blob + size_t(s) * REC);
        for (uint32_t i = tid; i < m; i += NT)
            reinterpret_cast<uint4 *>(tab)[i] = src[i];
        __syncthreads();
    };
    uint32_t in_chunk = 0;  // steps of the chunk in LDS that are done
    for (uint32_t s = 0; s < a.nsteps;) {
        if (in_chunk == 0)
            load_table(s);
        const unsigned char *rec = tab + in_chunk * REC;
        const u32x4 w0 = *reinterpret_cast<const u32x4 *>(rec);
        const uint32_t kw = uni(w0.w), kind = kw & 255u;
        if (kind == kStepGate) {
            // A run of one-target steps: every pair of the target goes through
            // its matrix, a pair off the controls is written back as read, so
            // a step has no branch; the record and the matrix of the next one
            // are read during the current one.
            const uint32_t run = kw >> 16;
            u32x4 w = w0;
            const C *m = reinterpret_cast<const C *>(rec + sizeof(SmallGate));
            C m00 = m[0], m01 = m[1], m10 = m[2], m11 = m[3];
            for (uint32_t k = 0; k < run; ++k) {
                const u32x4 g = w;
                const C c00 = m00, c01 = m01, c10 = m10, c11 = m11;
                if (k + 1 < run)
                    rec += REC;
                w = *reinterpret_cast<const u32x4 *>(rec);
                m = reinterpret_cast<const C *>(rec + sizeof(SmallGate));
                m00 = m[0], m01 = m[1], m10 = m[2], m11 = m[3];
                if constexpr (U == 1) {
                    if (tid < npairs) {
                        const uint32_t i = (tid & g.x) | ((tid & ~g.x) << 1), o = slot(i);
                        const bool on = (i & g.y) == g.y;
                        const C l = at(o), h = at(o ^ g.z);
                        const bool diag = (g.w >> 8) & kGateDiag, keep = (g.w >> 8) & kGateKeep;
                        const C a0 = cmul(c00, l), a1 = cmul(c10, l), b1 = cmul(c11, h);
                        C y0 = cmad(c01, h, a0), y1 = cmad(c11, h, a1);
                        y0.x = diag ? a0.x : y0.x, y0.y = diag ? a0.y : y0.y;
                        y1.x = diag ? b1.x : y1.x, y1.y = diag ? b1.y : y1.y;
                        const bool on0 = on && !keep;
                        y0.x = on0 ? y0.x : l.x, y0.y = on0 ? y0.y : l.y;
                        y1.x = on ? y1.x : h.x, y1.y = on ? y1.y : h.y;
                        at(o) = y0;
                        at(o ^ g.z) = y1;
                    }
                } else {
                    // several pairs per thread: the arithmetic bounds the step,
                    // so the kinds branch (the same way for every thread)
                    const uint32_t flags = (uni(g.w) >> 8) & 255u;
                    uint32_t o[U];
                    bool on[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t j = tid + uint32_t(u) * NT;
                        const uint32_t i = (j & g.x) | ((j & ~g.x) << 1);
                        on[u] = (i & g.y) == g.y;
                        o[u] = slot(i);
                    }
                    if (flags & kGateDiag) {
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (on[u]) {
                                if (!(flags & kGateKeep))
                                    at(o[u]) = cmul(c00, at(o[u]));
                                at(o[u] ^ g.z) = cmul(c11, at(o[u] ^ g.z));
                            }
                    } else if (uni(g.y) != 0) {
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (on[u]) {
                                const C l = at(o[u]), h = at(o[u] ^ g.z);
                                at(o[u]) = cmad(c01, h, cmul(c00, l));
                                at(o[u] ^ g.z) = cmad(c11, h, cmul(c10, l));
                            }
                    } else {
                        C lo[U], hi[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            lo[u] = at(o[u]);
                            hi[u] = at(o[u] ^ g.z);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            at(o[u]) = cmad(c01, hi[u], cmul(c00, lo[u]));
                            at(o[u] ^ g.z) = cmad(c11, hi[u], cmul(c10, lo[u]));
                        }
                    }
                }
                __syncthreads();
            }
            s += run;
            in_chunk = in_chunk + run == kChunk ? 0 : in_chunk + run;
            continue;
        }
        const u32x4 w1 = reinterpret_cast<const u32x4 *>(rec)[1], w2 = reinterpret_cast<const u32x4 *>(rec)[2];
        const uint32_t nins = kw >> 16;
        const uint32_t ones = uni(w0.x), ins = uni(w0.y);
        const C *M = reinterpret_cast<const C *>(mbuf + uni(w0.z));
        if (const uint32_t units = uni(w2.w)) {
            // (the barrier that ended the step before ended the reads of the
            // matrices that these replace)
            const u32x4 *src = reinterpret_cast<const u32x4 *>(a.blob + uni(w2.z));
#pragma unroll 4
            for (uint32_t i = tid; i < units; i += NT)
                reinterpret_cast<u32x4 *>(mbuf)[i] = src[i];
            __syncthreads();
        }
        const uint32_t tb[3] = {uni(w1.x), uni(w1.y), uni(w1.z)};
        const uint32_t lo[3] = {uni(w1.w), uni(w2.x), uni(w2.y)};
        // index bits of group j (zeros inserted); linear over disjoint bits of
        // j, so a thread deposits its own index once and the parts that are
        // the same for all threads go through the scalar unit
        auto dep = [&](uint32_t j) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const uint32_t m = (lo[i / 2] >> (16 * (i & 1))) & 0xffffu;
                j = (j & m) | ((j & ~m) << 1);
            }
            return j;
        };
        // the same for any number of index bits left out
        auto dep_any = [&](uint32_t j) __attribute__((always_inline)) {
            for (uint32_t m = ins; m != 0; m &= m - 1) {
                const uint32_t l = (m & (0u - m)) - 1u;
                j = (j & l) | ((j & ~l) << 1);
            }
            return j;
        };
        auto target = [&](int b) __attribute__((always_inline)) { return (tb[b / 2] >> (16 * (b & 1))) & 0xffffu; };
        const uint32_t cnt = 1u << (uint32_t(n) - nins);  // groups
        auto small_dense = [&](auto k_tag) __attribute__((always_inline)) {
            constexpr int K = decltype(k_tag)::value, D = 1 << K;
            uint32_t px[D];
#pragma unroll
            for (int e = 0; e < D; ++e) {
                uint32_t x = 0;
#pragma unroll
                for (int b = 0; b < K; ++b)
                    if ((e >> b) & 1)
                        x |= target(b);
                px[e] = slot(x);
            }
            for (uint32_t j = tid; j < cnt; j += NT) {
                const uint32_t o = slot(dep(j) | ones);
                C v[D];
#pragma unroll
                for (int e = 0; e < D; ++e)
                    v[e] = at(o ^ px[e]);
#pragma unroll
                for (int r = 0; r < D; ++r) {
                    if constexpr (K > 2)
                        asm volatile("" ::: "memory");  // a row at a time: 64 entries do not fit the registers
                    C acc = cmul(M[r * D], v[0]);
#pragma unroll
                    for (int c = 1; c < D; ++c)
                        acc = cmad(M[r * D + c], v[c], acc);
                    at(o ^ px[r]) = acc;
                }
            }
        };
        // Matrix cores: item (group set of 16 groups, row block of 16 rows);
        // every wave keeps one row block.  mbuf holds the A operands in the
        // order (row block, k-step, lane): U[16 mt + lane % 16][4 s + lane / 16].
        // Controls are fixed bits of the group index, as in every step.  (With
        // one control, four targets take 2.2 us at 11 qubits and 3.4 at 13, six
        // targets 8.6 at 13; one output per thread on the vector unit took 9,
        // 32 and 120, a launch each 9, 7 and 15.)
        auto mfma_items = [&](auto k_tag, auto p_tag, auto three_tag) __attribute__((always_inline)) {
            constexpr int K = decltype(k_tag)::value, D = 1 << K, NS = D / 4, NMT = D / 16;
            constexpr bool THREE = decltype(three_tag)::value;
            constexpr int PW = decltype(p_tag)::value;  // items per wave
            const uint32_t items = (cnt / 16) * NMT;
            const bool active = wave < items;
            const bool all = PW == 1 || items > kSmallWaves;  // else only the first of a wave's items
            auto dep_c = [&](uint32_t j) __attribute__((always_inline)) { return nins > 6 ? dep_any(j) : dep(j); };
            const uint32_t mt = wave % NMT;
            auto row = [&](uint32_t r) __attribute__((always_inline)) {
                uint32_t x = 0;
#pragma unroll
                for (int b = 0; b < K; ++b)
                    if ((r >> b) & 1)
                        x |= target(b);
                return x;
            };
            const uint32_t q = lane / 16;
            const uint32_t in_lane = slot(((q & 1) ? target(0) : 0u) | ((q & 2) ? target(1) : 0u));
            const uint32_t out_lane = F64 ? in_lane : slot(((q & 1) ? target(2) : 0u) | ((q & 2) ? target(3) : 0u));
            const uint32_t own_j = slot(dep_c(lane % 16) | ones);
            uint32_t go[PW];
            // THREE: sums of ur xr, ui xi, (ur + ui) (xr + xi); else of ur xr, ui xi, ur xi, ui xr
            AccT p1[PW], p2[PW], p3[PW], p4[PW];
            if (active) {
#pragma unroll
                for (int j = 0; j < PW; ++j) {
                    go[j] = own_j ^ slot(dep_c(((wave + uint32_t(kSmallWaves * j)) / NMT) * 16));
                    p1[j] = AccT{};
                    p2[j] = AccT{};
                    p3[j] = AccT{};
                    p4[j] = AccT{};
                }
#pragma unroll 4
                for (int t = 0; t < NS; ++t) {
                    const C u = M[(mt * NS + uint32_t(t)) * 64 + lane];
                    const R us = u.x + u.y;
                    const uint32_t ss = slot(row(uint32_t(4 * t)));
#pragma unroll
                    for (int j = 0; j < PW; ++j) {
                        if (j > 0 && !all)
                            break;
                        const C x = at(go[j] ^ in_lane ^ ss);
                        p1[j] = mma(u.x, x.x, p1[j]);
                        p2[j] = mma(u.y, x.y, p2[j]);
                        if constexpr (THREE) {
                            p3[j] = mma(us, x.x + x.y, p3[j]);
                        } else {
                            p3[j] = mma(u.x, x.y, p3[j]);
                            p4[j] = mma(u.y, x.x, p4[j]);
                        }
                    }
                }
            }
            __syncthreads();  // every row block has read its groups
            if (active) {
#pragma unroll
                for (int j = 0; j < PW; ++j) {
                    if (j > 0 && !all)
                        break;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // accumulator row: 4 (lane / 16) + r (FP32), 4 r + lane / 16 (FP64)
                        const uint32_t rr = slot(row(16 * mt + uint32_t(F64 ? 4 * r : r)));
                        C y;
                        y.x = p1[j][r] - p2[j][r];
                        y.y = THREE ? p3[j][r] - p1[j][r] - p2[j][r] : p3[j][r] + p4[j][r];
                        at(go[j] ^ out_lane ^ rr) = y;
                    }
                }
            }
        };
        // 2^(n - 8 - controls) items: two per wave at 13 qubits without
        // controls, where complex64 takes three products; else at most one
        auto mfma_dense = [&](auto k_tag, auto three_tag) __attribute__((always_inline)) {
            constexpr bool THREE = decltype(three_tag)::value;
            if constexpr (!THREE || F64 || U > 1)  // complex64 below 12 qubits: never three
                mfma_items(k_tag, std::integral_constant<int, U == 4 && THREE ? 2 : 1>{}, three_tag);
        };
        switch (kind) {
        case kStepDense2: small_dense(std::integral_constant<int, 2>{}); break;
        case kStepDense3: small_dense(std::integral_constant<int, 3>{}); break;
        case kStepMfma4: mfma_dense(std::integral_constant<int, 4>{}, std::false_type{}); break;
        case kStepMfma5: mfma_dense(std::integral_constant<int, 5>{}, std::false_type{}); break;
        case kStepMfma6: mfma_dense(std::integral_constant<int, 6>{}, std::false_type{}); break;
        case kStepMfma4t: mfma_dense(std::integral_constant<int, 4>{}, std::true_type{}); break;
        case kStepMfma5t: mfma_dense(std::integral_constant<int, 5>{}, std::true_type{}); break;
        case kStepMfma6t: mfma_dense(std::integral_constant<int, 6>{}, std::true_type{}); break;
        default: {
            // output (group, row) per thread, at most 2^12 / 1024 = 4 of them
            const uint32_t k = (kw >> 8) & 255u, D = 1u << k, outs = cnt << k;
            const C *Mr = M;
            C acc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = tid + uint32_t(u) * NT;
                acc[u] = czero<C>();
                if (j >= outs)
                    continue;
                const uint32_t o = slot(dep_any(j >> k) | ones), r = j & (D - 1);
                for (uint32_t c = 0; c < D; ++c) {
                    uint32_t x = 0;
#pragma unroll
                    for (int b = 0; b < SV_MAX_TARGETS; ++b)
                        if ((c >> b) & 1)
                            x |= target(b);
                    acc[u] = cmad(Mr[r * D + c], at(o ^ slot(x)), acc[u]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = tid + uint32_t(u) * NT;
                if (j >= outs)
                    continue;
                const uint32_t r = j & (D - 1);
                uint32_t x = 0;
#pragma unroll
                for (int b = 0; b < SV_MAX_TARGETS; ++b)
                    if ((r >> b) & 1)
                        x |= target(b);
                at(slot(dep_any(j >> k) | ones) ^ slot(x)) = acc[u];
            }
            break;
        }
        }
        __syncthreads();
        ++s;
        in_chunk = in_chunk + 1 == kChunk ? 0 : in_chunk + 1;
    }
    __syncthreads();  // (nsteps = 0 only)
    uint4 *go = reinterpret_cast<uint4 *>(st);
    for (uint32_t i = tid; i < nvec; i += NT)
        go[i] = *reinterpret_cast<const uint4 *>(tile + slot(i * PERV));
}

uint32_t step_kind(int n, int dtype, const Block &b)
{
    if (b.k == 1)
        return kStepGate;
    if (b.k <= 3 && b.k + b.c <= 6)
        return b.k == 2 ? kStepDense2 : kStepDense3;
    if (b.k < 4 || n - b.k - b.c < 4)
        return kStepDense;
    const bool three = dense_path(n, dtype, b.k, b.c, SV_PREC_NATIVE) == SV_SWEEP_DENSE_MFMA;
    return (three ? kStepMfma4t : kStepMfma4) + uint32_t(b.k - 4);
}

uint64_t large_bytes(int dtype, int k)
{
    const uint64_t amp = dtype == SV_C64 ? 8 : 16;
    return ((amp << (2 * k)) + 15) & ~uint64_t(15);
}

template <typename R>
void put_matrix(char *dst, const Block &b, uint32_t kind)
{
    using C2 = R[2];
    C2 *o = reinterpret_cast<C2 *>(dst);
    const int d = 1 << b.k;
    auto put = [](C2 &x, cd u) {
        x[0] = R(u.real());
        x[1] = R(u.imag());
    };
    if (kind < kStepMfma4) {
        for (int j = 0; j < d * d; ++j)
            put(o[j], b.U[size_t(j)]);
        return;
    }
    for (int mt = 0; mt < d / 16; ++mt)
        for (int s = 0; s < d / 4; ++s)
            for (int lane = 0; lane < 64; ++lane)
                put(o[(mt * (d / 4) + s) * 64 + lane], b.U[size_t(mt * 16 + lane % 16) * d + 4 * s + lane / 16]);
}

uint32_t rec_bytes(int dtype)
{
    return dtype == SV_C64 ? record_bytes<float>() : record_bytes<double>();
}

}  // namespace

bool small_fits(int n, int dtype)
{
    return n <= (dtype == SV_C64 ? 13 : 12);
}

uint64_t small_step_bytes(int dtype, int k)
{
    // (a three-target block may be stored as a four-target one)
    return rec_bytes(dtype) + (k > 1 ? large_bytes(dtype, k == 3 ? 4 : k) : 0);
}

SmallProgram small_begin(char *blob, int n, int dtype, size_t nsteps)
{
    SmallProgram p{};
    p.blob = blob;
    p.n = n;
    p.dtype = dtype;
    p.mat = uint32_t(nsteps * rec_bytes(dtype));
    p.head = -1;
    // beside the state and the table
    const uint32_t table = uint32_t(std::min<size_t>(nsteps, kChunk)) * rec_bytes(dtype);
    p.room = kLdsBytes - uint32_t((dtype == SV_C64 ? 8u : 16u) << n) - table;
    return p;
}

static char *record(const SmallProgram &p, int i)
{
    return p.blob + size_t(i) * rec_bytes(p.dtype);
}

void small_add(SmallProgram &p, const Block &b, const int *pt, const int *pc)
{
    if (b.k == 3 && b.c == 0 && p.n >= 8) {
        // U (x) I on a free index bit: the matrix cores take less time for a
        // 16 x 16 block than the vector unit for an 8 x 8 one
        Block o;
        o.k = 4;
        o.U.assign(256, cd(0.0, 0.0));
        for (int r = 0; r < 16; ++r)
            for (int c = 0; c < 16; ++c)
                if ((r >> 3) == (c >> 3))
                    o.U[size_t(r) * 16 + c] = b.U[size_t(r & 7) * 8 + (c & 7)];
        int free = 0;
        while (free == pt[0] || free == pt[1] || free == pt[2])
            ++free;
        const int pt4[4] = {pt[0], pt[1], pt[2], free};
        small_add(p, o, pt4, pc);
        return;
    }
    uint32_t fixed = 0, bits = 0;
    for (int j = 0; j < b.c; ++j)
        fixed |= 1u << pc[j];
    for (int j = 0; j < b.k; ++j)
        bits |= 1u << pt[j];
    const uint32_t kind = step_kind(p.n, p.dtype, b);
    char *rec = record(p, p.count);
    if (kind == kStepGate) {
        SmallGate g{};
        g.lo = bits - 1;
        g.ctl = fixed;
        const uint32_t amp = p.dtype == SV_C64 ? 8 : 16;
        g.pt = (bits ^ ((bits >> 6) & 62u)) * amp;  // the kernel's slot()
        const uint32_t flags = !b.diag ? 0 : b.U[0] == cd(1.0, 0.0) ? kGateDiag | kGateKeep : kGateDiag;
        g.kind = kStepGate | flags << 8 | 1u << 16;
        std::memcpy(rec, &g, sizeof g);
        if (p.dtype == SV_C64)
            put_matrix<float>(rec + sizeof g, b, kind);
        else
            put_matrix<double>(rec + sizeof g, b, kind);
        ++p.count;
        return;
    }
    SmallStep s{};
    for (int j = 0; j < b.k; ++j)
        s.tbits[j / 2] |= (1u << pt[j]) << (16 * (j & 1));
    s.ins = fixed | bits;
    s.kind = kind | uint32_t(b.k) << 8 | uint32_t(__builtin_popcount(s.ins)) << 16;
    s.ones = fixed;
    s.lo[0] = s.lo[1] = s.lo[2] = 0xffffffffu;
    for (int q = 0, i = 0; q < p.n && i < 6; ++q)
        if ((s.ins >> q) & 1) {
            s.lo[i / 2] ^= (0xffffu ^ ((1u << q) - 1u)) << (16 * (i & 1));
            ++i;
        }
    const uint32_t bytes = uint32_t(large_bytes(p.dtype, b.k));
    if (p.dtype == SV_C64)
        put_matrix<float>(p.blob + p.mat, b, kind);
    else
        put_matrix<double>(p.blob + p.mat, b, kind);
    // matrices go into LDS in groups as large as there is room for; the first
    // step of a group loads it
    if (p.head >= 0) {
        SmallStep *h = reinterpret_cast<SmallStep *>(record(p, p.head));
        if (h->units * 16 + bytes > p.room) {
            p.head = -1;
        } else {
            s.mat = h->units * 16;
            h->units += bytes / 16;
        }
    }
    if (p.head < 0) {
        p.head = p.count;
        s.load = p.mat;
        s.units = bytes / 16;
    }
    p.mat += bytes;
    p.mbuf = std::max(p.mbuf, s.mat + bytes);
    std::memcpy(rec, &s, sizeof s);
    ++p.count;
}

void small_end(SmallProgram &p)
{
    // one-target steps from each one on, within its chunk of the table
    uint32_t run = 0;
    for (int i = p.count - 1; i >= 0; --i) {
        SmallGate *g = reinterpret_cast<SmallGate *>(record(p, i));
        if (uint32_t(i) % kChunk == kChunk - 1)
            run = 0;
        run = (g->kind & 255u) == kStepGate ? run + 1 : 0;
        if (run > 0)
            g->kind = (g->kind & 0xffffu) | run << 16;
    }
}

hipError_t launch_small(void *st, const SmallProgram &p, const void *blob, hipStream_t s)
{
    if (!small_fits(p.n, p.dtype) || p.n < 1)
        return hipErrorInvalidValue;
    SmallArgs a{};
    a.blob = static_cast<const char *>(blob);
    a.nsteps = uint32_t(p.count);
    a.mbuf_bytes = p.mbuf;
    a.n = p.n;
    const size_t amp = p.dtype == SV_C64 ? 8 : 16;
    const size_t lds = (amp << p.n) + p.mbuf + size_t(std::min<uint32_t>(uint32_t(p.count), kChunk)) * rec_bytes(p.dtype);
    const int u = p.n <= 11 ? 1 : p.n == 12 ? 2 : 4;
    auto launch = [&](auto r_tag, auto u_tag) {
        using R = decltype(r_tag);
        constexpr int U = decltype(u_tag)::value;
        if (lds > 65536) {
            // always the most that a program takes: the attribute belongs to the
            // process, and another thread's smaller program must not lower it
            // between this and the launch
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_small<R, U>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsBytes));
            if (e != hipSuccess)
                return e;
        }
        hipLaunchKernelGGL((k_small<R, U>), dim3(1), dim3(kSmallThreads), lds, s, (R *)st, a);
        return hipGetLastError();
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    if (p.dtype == SV_C64)
        return u == 1 ? launch(float{}, One{}) : u == 2 ? launch(float{}, Two{}) : launch(float{}, Four{});
    return u == 1 ? launch(double{}, One{}) : launch(double{}, Two{});
}

}  // namespace sv
