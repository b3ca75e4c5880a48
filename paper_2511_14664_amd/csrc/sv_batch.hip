// Persistent batch kernel: many small circuits in one launch (gfx950).
//
// Workgroups take tasks (circuit, pass, tile) from a global queue in a fixed
// order.  A task loads its tile of 2^lp amplitudes into LDS (or creates
// |0...0> for the first pass), applies the pass's gates in LDS -- each one a
// sweep over the tile, paper Sec. 2.1 -- and either stores the tile or, on the
// last pass, reduces the Z-string expectation values of its amplitudes in
// FP64.  A task of pass p waits until every tile of passes < p of its circuit
// is done; those tasks were dequeued earlier by resident workgroups, so the
// wait always ends.  The wait is still bounded: past the spin limit the task
// raises the error flag, every workgroup drains, and the host reports it.
//
// Cross-workgroup visibility: whatever another workgroup reads (amplitudes,
// partial sums) is stored at device scope (sc1, what a relaxed agent-scope
// atomic store compiles to): the store goes through the XCD's L2 to the memory
// that all XCDs share, and vmcnt counts it until that memory has acknowledged
// it.  Every wave waits for its count to reach zero, then a barrier, then one
// thread raises the count of finished tiles, so whoever reads the raised count
// finds the stores in memory; it passes a barrier, and every thread issues an
// agent-scope acquire fence (its caches' lines of the tile are dropped) before
// loading.  An agent-scope release is this same wait and, before it, the write
// back of L2 lines left dirty by stores of narrower scope; those write nothing
// that another workgroup of the launch reads (results in `out` are read after
// the launch).
#include "sv_batch.h"
#include "sv_device.h"

namespace sv {
namespace {

using namespace dev;

__device__ __forceinline__ uint32_t ins1(uint32_t j, int a)
{
    return (j & ((1u << a) - 1u)) | ((j >> a) << (a + 1));
}

// Insert zeros at tile bits lo < hi.
__device__ __forceinline__ uint32_t ins2(uint32_t j, int lo, int hi)
{
    return ins1(ins1(j, lo), hi);
}

// acc + u * v as four fused multiply-adds (the state arithmetic of the
// in-LDS sweeps; every product is rounded once, into the running sum)
__device__ __forceinline__ float fma_r(float a, float b, float c)
{
    return __builtin_fmaf(a, b, c);
}
__device__ __forceinline__ double fma_r(double a, double b, double c)
{
    return __builtin_fma(a, b, c);
}
template <typename C>
__device__ __forceinline__ C cfma(C u, C v, C acc)
{
    acc.x = fma_r(u.x, v.x, acc.x);
    acc.x = fma_r(-u.y, v.y, acc.x);
    acc.y = fma_r(u.x, v.y, acc.y);
    acc.y = fma_r(u.y, v.x, acc.y);
    return acc;
}

// Element of the LDS tile at byte offset o.  swz() is linear over XOR, so
// the offsets of a group's members are one XOR away from its first one.
template <typename C>
__device__ __forceinline__ C &lds_at(unsigned char *tileb, uint32_t o)
{
    return *reinterpret_cast<C *>(tileb + o);
}

// This wave's device-scope stores are in the memory that all XCDs share (see the
// top of the file).  An agent-scope release fence adds a write-back of the whole
// L2, which holds no dirty line that matters here: 9.5 against 1.8 us per 2^13
// tile.
__device__ __forceinline__ void publish()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // nothing moves below
    __builtin_amdgcn_s_waitcnt(0);                          // vmcnt, expcnt and lgkmcnt all zero
}

// Device-scope store of one amplitude (relaxed atomic 64-bit stores): the
// write goes through the XCD's L2.
template <typename C>
__device__ __forceinline__ void store_dev(C *p, C v)
{
    static_assert(sizeof(C) % 8 == 0, "amplitudes of 8 or 16 bytes");
    uint64_t w[sizeof(C) / 8];
    __builtin_memcpy(w, &v, sizeof(C));
    uint64_t *q = reinterpret_cast<uint64_t *>(p);
#pragma unroll
    for (size_t i = 0; i < sizeof(C) / 8; ++i)
        __hip_atomic_store(q + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same for 16 bytes (there is no 128-bit atomic; nothing needs it in one
// piece).  The wait states keep a later write to v's registers behind the
// store's read of them.
__device__ __forceinline__ void store_dev16(void *p, f32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Register runs.  A thread holds the 2^NR amplitudes of its group in vr, vi.
// Step sweeps through LDS were bound by latency (a read, 16 products and a
// write per amplitude group and a barrier per step, two wavefronts per SIMD:
// vector units 39 % busy on 128 HEA circuits of 10 to 21 qubits); in registers
// the steps of a run follow each other with neither, and the matrix sits in
// scalar registers (the tables are written before the launch, so they are read
// through the constant address space).  The arithmetic of each amplitude is
// the sweeps'.  With 16-byte tile accesses all in flight, strings by
// coefficients and no L2 write-back those circuits take 5.3 ms instead of 9.7:
// per 2^13 tile 41 us in runs (20 steps, vector bound), 15 loading (33 before),
// 6 storing (15), 6 waiting for a task.
// ---------------------------------------------------------------------------
#define SV_CONST __attribute__((address_space(4)))

template <typename T>
__device__ __forceinline__ const SV_CONST T *as_const(const T *p)
{
    return (const SV_CONST T *)(uintptr_t)p;
}

// Dense two-qubit step on register bits A < B; m: row-major re, im pairs.
template <typename R, int NR, int A, int B>
__device__ __forceinline__ void run_two(R (&vr)[1 << NR], R (&vi)[1 << NR], const R (&m)[32])
{
    using C = typename CT<R>::C;
#pragma unroll
    for (int g = 0; g < (1 << NR) / 4; ++g) {
        const int i0 = ((g & ((1 << A) - 1)) | ((g >> A) << (A + 1)));
        const int i = (i0 & ((1 << B) - 1)) | ((i0 >> B) << (B + 1));
        const int e[4] = {i, i | 1 << A, i | 1 << B, i | 1 << A | 1 << B};
        C v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k].x = vr[e[k]];
            v[k].y = vi[e[k]];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            C u;
            u.x = m[8 * r];
            u.y = m[8 * r + 1];
            C acc = cmul(u, v[0]);
#pragma unroll
            for (int c = 1; c < 4; ++c) {
                u.x = m[8 * r + 2 * c];
                u.y = m[8 * r + 2 * c + 1];
                acc = cfma(u, v[c], acc);
            }
            vr[e[r]] = acc.x;
            vi[e[r]] = acc.y;
        }
    }
}

// One-qubit step on register bit A, on the pairs whose first index is in mask.
template <typename R, int NR, int A>
__device__ __forceinline__ void run_one(R (&vr)[1 << NR], R (&vi)[1 << NR], const R (&m)[32], uint32_t mask)
{
    using C = typename CT<R>::C;
    const C m00{m[0], m[1]}, m01{m[2], m[3]}, m10{m[4], m[5]}, m11{m[6], m[7]};
#pragma unroll
    for (int g = 0; g < (1 << NR) / 2; ++g) {
        const int i = (g & ((1 << A) - 1)) | ((g >> A) << (A + 1)), j = i | 1 << A;
        if ((mask >> i) & 1u) {
            const C v0{vr[i], vi[i]}, v1{vr[j], vi[j]};
            const C w0 = cfma(m01, v1, cmul(m00, v0)), w1 = cfma(m11, v1, cmul(m10, v0));
            vr[i] = w0.x;
            vi[i] = w0.y;
            vr[j] = w1.x;
            vi[j] = w1.y;
        }
    }
}

// The pass's runs over the tile in LDS; ends with a barrier.
template <typename R, int NR>
__device__ __forceinline__ void tile_runs(unsigned char *tileb, const BRun *runs, int nruns, const BStep *steps,
                                          const R *mats, int tid)
{
    using C = typename CT<R>::C;
    constexpr uint32_t S = uint32_t(sizeof(C));
    for (int ri = 0; ri < nruns; ++ri) {
        const SV_CONST BRun *run = as_const(runs) + ri;
        uint32_t o = 0;
#pragma unroll
        for (int b = 0; b < kBatchThreadLog; ++b)
            o ^= (swz(1u << run->lane[b]) * S) & uint32_t(-((tid >> b) & 1));
        uint32_t px[NR];
#pragma unroll
        for (int b = 0; b < NR; ++b)
            px[b] = swz(1u << run->reg[b]) * S;
        auto at = [&](int e) __attribute__((always_inline)) {
            uint32_t x = o;
#pragma unroll
            for (int b = 0; b < NR; ++b)
                x ^= ((e >> b) & 1) ? px[b] : 0u;
            return x;
        };
        R vr[1 << NR], vi[1 << NR];
#pragma unroll
        for (int e = 0; e < (1 << NR); ++e) {
            const C v = lds_at<C>(tileb, at(e));
            vr[e] = v.x;
            vi[e] = v.y;
        }
        // The next step's matrix (complex64; complex128 matrices leave no
        // room) and the record after it are read while a step runs.  A matrix
        // is read as 16 elements whatever its size, the buffer is padded for
        // that.
        constexpr bool kAhead = sizeof(R) == 4;
        const int s1 = run->step0 + run->nsteps;
        const SV_CONST BStep *sp = as_const(steps) + run->step0;
        auto matrix = [&](uint32_t mat, R (&m)[32]) __attribute__((always_inline)) {
            const SV_CONST R *M = as_const(mats) + 2 * size_t(mat);
#pragma unroll
            for (int e = 0; e < 32; ++e)
                m[e] = M[e];
        };
        uint32_t mat = sp->mat;
        int type = sp->type, ra = sp->a, rb = sp->b;
        R m[32];
        if constexpr (kAhead)
            matrix(mat, m);
        for (int si = run->step0; si < s1; ++si) {
            // a run has a successor record except at the table's padded end
            ++sp;
            const uint32_t mat_n = sp->mat;
            const int type_n = sp->type, ra_n = sp->a, rb_n = sp->b;
            R mn[32];
            if constexpr (kAhead)
                matrix(mat_n, mn);
            else
                matrix(mat, m);
            if (type == 2) {
                // a < b: index of the pair among them
                switch (ra + rb * (rb - 1) / 2) {
                case 0: run_two<R, NR, 0, 1>(vr, vi, m); break;
                case 1: run_two<R, NR, 0, 2>(vr, vi, m); break;
                case 2: run_two<R, NR, 1, 2>(vr, vi, m); break;
                default:
                    if constexpr (NR >= 4) {
                        switch (ra + rb * (rb - 1) / 2) {
                        case 3: run_two<R, NR, 0, 3>(vr, vi, m); break;
                        case 4: run_two<R, NR, 1, 3>(vr, vi, m); break;
                        case 5: run_two<R, NR, 2, 3>(vr, vi, m); break;
                        default:
                            if constexpr (NR >= 5) {
                                switch (ra) {
                                case 0: run_two<R, NR, 0, 4>(vr, vi, m); break;
                                case 1: run_two<R, NR, 1, 4>(vr, vi, m); break;
                                case 2: run_two<R, NR, 2, 4>(vr, vi, m); break;
                                default: run_two<R, NR, 3, 4>(vr, vi, m); break;
                                }
                            }
                        }
                    }
                }
            } else {
                // register indices with bit rb set
                uint32_t mask = ~0u;
                if (type == 1)
                    mask = rb == 0 ? 0xaaaaaaaau : rb == 1 ? 0xccccccccu : rb == 2 ? 0xf0f0f0f0u
                                                         : rb == 3 ? 0xff00ff00u : 0xffff0000u;
                switch (ra) {
                case 0: run_one<R, NR, 0>(vr, vi, m, mask); break;
                case 1: run_one<R, NR, 1>(vr, vi, m, mask); break;
                case 2: run_one<R, NR, 2>(vr, vi, m, mask); break;
                case 3:
                    if constexpr (NR >= 4)
                        run_one<R, NR, 3>(vr, vi, m, mask);
                    break;
                default:
                    if constexpr (NR >= 5)
                        run_one<R, NR, 4>(vr, vi, m, mask);
                }
            }
            mat = mat_n;
            type = type_n;
            ra = ra_n;
            rb = rb_n;
            if constexpr (kAhead) {
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    m[e] = mn[e];
            }
        }
        // back to the slots this thread read
#pragma unroll
        for (int e = 0; e < (1 << NR); ++e) {
            C v;
            v.x = vr[e];
            v.y = vi[e];
            lds_at<C>(tileb, at(e)) = v;
        }
        __syncthreads();
    }
}

// Global address parts of a tile of 2^(8 + NR) amplitudes moved in 16-byte
// accesses (complex64: pairs; tile bit 0 is then physical bit 0): access s of a
// thread covers tile index (s 256 + tid) << LO.
template <typename R, int NR>
struct RunTile {
    using C = typename CT<R>::C;
    static constexpr int LO = sizeof(C) == 8 ? 1 : 0;
    static constexpr int NV = (1 << NR) >> LO;
    uint64_t lane_off = 0;
    uint64_t hi[NR - LO];
    unsigned char *tileb;
    uint32_t slot0;  // LDS byte offset of access 0 (swz is linear over XOR)

    __device__ __forceinline__ RunTile(const BPass &ps, unsigned char *t, int tid) : tileb(t)
    {
        slot0 = swz(uint32_t(tid) << LO) * uint32_t(sizeof(C));
#pragma unroll
        for (int b = 0; b < kBatchThreadLog; ++b)
            lane_off |= ps.dep[b + LO] & (0 - uint64_t((tid >> b) & 1));
#pragma unroll
        for (int b = 0; b < NR - LO; ++b)
            hi[b] = ps.dep[b + LO + kBatchThreadLog];
    }
    __device__ __forceinline__ uint64_t off(int s) const
    {
        uint64_t o = lane_off;
#pragma unroll
        for (int b = 0; b < NR - LO; ++b)
            o |= ((s >> b) & 1) ? hi[b] : 0;
        return o;
    }
    // the access's one or two amplitudes in the tile
    __device__ __forceinline__ C &slot(int s, int h) const
    {
        return lds_at<C>(tileb, slot0 ^ (swz(uint32_t(((s * kBatchThreads) << LO) + h)) * uint32_t(sizeof(C))));
    }
    // every load in flight before the first LDS store
    __device__ __forceinline__ void load(const C *st) const
    {
        f32x4 v[NV];
#pragma unroll
        for (int s = 0; s < NV; ++s)
            v[s] = *reinterpret_cast<const f32x4 *>(st + off(s));
#pragma unroll
        for (int s = 0; s < NV; ++s) {
            if constexpr (LO) {
                slot(s, 0) = make_float2(v[s].x, v[s].y);
                slot(s, 1) = make_float2(v[s].z, v[s].w);
            } else {
                slot(s, 0) = __builtin_bit_cast(C, v[s]);
            }
        }
    }
    __device__ __forceinline__ void store(C *st) const
    {
#pragma unroll
        for (int s = 0; s < NV; ++s) {
            f32x4 v;
            if constexpr (LO) {
                const float2 x = slot(s, 0), y = slot(s, 1);
                v = f32x4{x.x, x.y, y.x, y.y};
            } else {
                v = __builtin_bit_cast(f32x4, slot(s, 0));
            }
            store_dev16(st + off(s), v);
        }
    }
};

// Z strings of a tile of 2^(8 + NR) amplitudes, out(j, sum) by one thread for
// each.  A Walsh transform over the NR tile bits above the thread's gives, per
// thread, sum_s (-1)^popcount(s & k) p(s, tid) for every k; a string takes the
// coefficient of its upper tile bits, with the parity of its thread bits and of
// its bits outside the tile as sign, so a string costs one LDS read per thread
// instead of one sign and sum per amplitude (147 us for 41 strings of a 2^13
// tile, against 13).  The coefficients take the tile's place in LDS.  Sums in
// FP64; ends with a barrier.
template <typename R, int NR, typename F>
__device__ __forceinline__ void tile_strings(unsigned char *tileb, double *red, const BPass &ps, uint64_t base,
                                             const uint64_t *zm, int nterms, int tid, F out)
{
    using C = typename CT<R>::C;
    __shared__ uint32_t zt[kBatchMaxTerms];  // string's tile bits; bit 31: odd outside the tile
    const int lane = tid & 63, wave = tid >> 6;
    if (tid < nterms) {
        const uint64_t z = zm[tid];
        uint64_t in = 0;
        uint32_t x = 0;
#pragma unroll
        for (int b = 0; b < kBatchThreadLog + NR; ++b) {
            in |= ps.dep[b];
            x |= (z & ps.dep[b]) != 0 ? 1u << b : 0u;
        }
        zt[tid] = x | uint32_t(__popcll(base & z & ~in) & 1) << 31;
    }
    double w[1 << NR];
    const uint32_t slot0 = swz(uint32_t(tid)) * uint32_t(sizeof(C));
#pragma unroll
    for (int s = 0; s < (1 << NR); ++s) {
        const C v = lds_at<C>(tileb, slot0 ^ (swz(uint32_t(s * kBatchThreads)) * uint32_t(sizeof(C))));
        w[s] = double(v.x) * double(v.x) + double(v.y) * double(v.y);
    }
#pragma unroll
    for (int b = 1; b < (1 << NR); b <<= 1)
#pragma unroll
        for (int s = 0; s < (1 << NR); ++s)
            if (!(s & b)) {
                const double x = w[s], y = w[s | b];
                w[s] = x + y;
                w[s | b] = x - y;
            }
    __syncthreads();  // every thread has its amplitudes
    double *coef = reinterpret_cast<double *>(tileb);
#pragma unroll
    for (int s = 0; s < (1 << NR); ++s)
        coef[s * kBatchThreads + tid] = w[s];
    for (int c0 = 0; c0 < nterms; c0 += 16) {
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v[j] = 0.0;
            if (c0 + j < nterms) {
                const uint32_t x = zt[c0 + j];
                const double c = coef[((x >> kBatchThreadLog) & ((1u << NR) - 1)) * kBatchThreads + uint32_t(tid)];
                v[j] = ((__popc(x & uint32_t(kBatchThreads - 1) & uint32_t(tid)) + (x >> 31)) & 1) ? -c : c;
            }
        }
        // halve the values a lane holds at each of four steps, then two more
        // sums: lane l ends with string l / 4
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = ((lane & 32) ? v[i + 8] : v[i]) + __shfl_xor((lane & 32) ? v[i] : v[i + 8], 32, 64);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = ((lane & 16) ? v[i + 4] : v[i]) + __shfl_xor((lane & 16) ? v[i] : v[i + 4], 16, 64);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            v[i] = ((lane & 8) ? v[i + 2] : v[i]) + __shfl_xor((lane & 8) ? v[i] : v[i + 2], 8, 64);
        v[0] = ((lane & 4) ? v[1] : v[0]) + __shfl_xor((lane & 4) ? v[0] : v[1], 4, 64);
        v[0] += __shfl_xor(v[0], 2, 64);
        v[0] += __shfl_xor(v[0], 1, 64);
        if ((lane & 3) == 0)
            red[wave * 16 + (lane >> 2)] = v[0];
        __syncthreads();
        if (tid < 16 && c0 + tid < nterms) {
            double sum = red[tid];
#pragma unroll
            for (int k = 1; k < kBatchThreads / 64; ++k)
                sum += red[16 * k + tid];
            out(c0 + tid, sum);
        }
        __syncthreads();
    }
}

// NRMAX: register index bits of the widest tile's runs (0: none).
template <typename R, int NRMAX>
__global__ __launch_bounds__(kBatchThreads, 2) void k_batch(const BatchArgs a)
{
    using C = typename CT<R>::C;
    // tile amplitudes per thread in flight between global memory and LDS
    constexpr uint32_t kU = 8;
    typedef R VU __attribute__((ext_vector_type(2 * kU)));
    extern __shared__ __align__(16) unsigned char smem[];
    C *tile = reinterpret_cast<C *>(smem);
    unsigned char *tileb = smem;
    double *red = reinterpret_cast<double *>(smem + (sizeof(C) << a.tile_log_max));  // [waves][16]
    C *mcache = reinterpret_cast<C *>(red + (kBatchThreads / 64) * 16);
    BStep *scache = reinterpret_cast<BStep *>(reinterpret_cast<unsigned char *>(mcache) + kBatchMatCacheBytes);
    constexpr uint32_t kMatCap = kBatchMatCacheBytes / sizeof(C);
    __shared__ uint32_t s_task;
    __shared__ int s_flag;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t *head = a.ctr;
    uint32_t *err = a.ctr + 1;
    uint32_t *done = a.ctr + 2;
    uint32_t *fin = a.ctr + 2 + a.ninst;
    C *states = reinterpret_cast<C *>(a.states);
    const C *mats = reinterpret_cast<const C *>(a.mats);

    for (;;) {
        if (tid == 0) {
            uint32_t t = atomicAdd(head, 1u);
            if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
                t = a.ntasks;
            s_task = t;
        }
        __syncthreads();
        const uint32_t t = uint32_t(__builtin_amdgcn_readfirstlane(int(s_task)));
        if (t >= a.ntasks)
            break;
        const BTask tk = a.tasks[t];
        const BInst in = a.inst[tk.inst];
        const BPass &ps = a.pass[in.pass0 + int(tk.pass)];
        const int lp = ps.lp;
        const uint32_t TA = 1u << lp;

        if (tk.pass > 0) {
            if (tid == 0) {
                int ok = 1;
                uint32_t spins = 0;
                while (__hip_atomic_load(&done[tk.inst], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < ps.need) {
                    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                        ++spins > a.spin_limit) {
                        ok = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(8);
                }
                if (!ok)
                    atomicOr(err, 1u);
                s_flag = ok;
            }
            __syncthreads();
            if (!s_flag)
                break;
            // pairs with the producers' release (the count was read relaxed)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }

        // the pass's steps and matrices into LDS (visible after the barrier
        // that ends the tile load; the previous task's last reads of them
        // ended at its final barrier)
        const int nruns = ps.nruns;
        const bool cached = nruns == 0 && ps.nsteps <= kBatchStepCache && ps.nmat <= kMatCap;
        if (cached) {
            for (int i = tid; i < ps.nsteps; i += kBatchThreads)
                scache[i] = a.steps[ps.step0 + i];
            for (uint32_t i = tid; i < ps.nmat; i += kBatchThreads)
                mcache[i] = mats[ps.mat0 + i];
        }

        // tile index -> base, and per-thread low part of the tile offsets
        uint64_t base = tk.tile;
        for (int b = 0; b < lp; ++b) {
            const uint64_t m = ps.ins[b];
            base = (base & m) | ((base & ~m) << 1);
        }
        uint64_t off_lo = 0;
        for (int b = 0; b < kBatchThreadLog && b < lp; ++b)
            if ((tid >> b) & 1)
                off_lo |= ps.dep[b];
        // deposits of the tile bits above the thread bits in registers: the
        // pass table is not re-read after every store of the tile
        constexpr int kHi = kBatchMaxTileLog - kBatchThreadLog;
        uint64_t dep_hi[kHi];
#pragma unroll
        for (int b = 0; b < kHi; ++b)
            dep_hi[b] = b + kBatchThreadLog < lp ? ps.dep[b + kBatchThreadLog] : 0;
        auto off_of = [&](uint32_t s) {
            uint64_t off = off_lo;
#pragma unroll
            for (int b = 0; b < kHi; ++b)
                if ((s >> b) & 1)
                    off |= dep_hi[b];
            return off;
        };
        const uint32_t nsteps_x = TA >= kBatchThreads ? TA / kBatchThreads : 1;
        const bool active = uint32_t(tid) < TA;
        C *st = states + in.state_off;
        // tiles as wide as those of register runs: f(NR) with NR = lp - 8
        auto with_nr = [&](auto f) __attribute__((always_inline)) {
            if constexpr (NRMAX >= 3)
                if (lp == kBatchThreadLog + 3)
                    f(std::integral_constant<int, 3>{});
            if constexpr (NRMAX >= 4)
                if (lp == kBatchThreadLog + 4)
                    f(std::integral_constant<int, 4>{});
            if constexpr (NRMAX >= 5)
                if (lp == kBatchThreadLog + 5)
                    f(std::integral_constant<int, 5>{});
        };
        // opaque per task: what the wide paths derive from the thread index is
        // not kept in registers across tasks
        int tw = tid;
        asm volatile("" : "+v"(tw));
        const bool runs_tile = NRMAX >= kRunMinBits && batch_runs(lp);
        const bool wide = runs_tile && (sizeof(C) == 16 || ps.dep[0] == 1);

        if (tk.pass == 0) {
            for (uint32_t s = 0; s < nsteps_x; ++s) {
                if (!active)
                    break;
                const uint32_t x = s * kBatchThreads + uint32_t(tid);
                C z;
                z.x = (tk.tile == 0 && x == 0) ? R(1) : R(0);
                z.y = R(0);
                tile[swz(x)] = z;
            }
        } else if (wide) {
            with_nr([&](auto nr) { RunTile<R, decltype(nr)::value>(ps, tileb, tw).load(st + base); });
        } else if (nsteps_x >= kU) {
            // kU global loads in flight per thread before the first LDS store
            // (nsteps_x and kU are powers of two: whole chunks)
            for (uint32_t s0 = 0; s0 < nsteps_x; s0 += kU) {
                VU v;  // a vector, not an array: stays in registers
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) {
                    const C x = st[base + off_of(s0 + u)];
                    v[2 * u] = x.x;
                    v[2 * u + 1] = x.y;
                }
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) {
                    C x;
                    x.x = v[2 * u];
                    x.y = v[2 * u + 1];
                    tile[swz((s0 + u) * kBatchThreads + uint32_t(tid))] = x;
                }
            }
        } else {
            for (uint32_t s = 0; s < nsteps_x; ++s) {
                if (!active)
                    break;
                tile[swz(s * kBatchThreads + uint32_t(tid))] = st[base + off_of(s)];
            }
        }
        __syncthreads();

        // the steps, reading step records and matrices from the LDS copies
        // (LDS) or from global memory (false)
        auto sweeps = [&](auto lds_tag) __attribute__((always_inline)) {
          constexpr bool kLds = decltype(lds_tag)::value;
          for (int si = 0; si < ps.nsteps; ++si) {
            BStep sp;
            if constexpr (kLds)
                sp = scache[si];
            else
                sp = a.steps[ps.step0 + si];
            const C *M = kLds ? mcache + (sp.mat - ps.mat0) : mats + sp.mat;
            const int ta = sp.a, tb = sp.b;
            // Each sweep takes one group per thread per iteration (two or four
            // groups with all their LDS reads ahead were slower).
            if (sp.type <= 1) {
                const C m00 = M[0], m01 = M[1], m10 = M[2], m11 = M[3];
                const int lo = ta < tb ? ta : tb, hi = ta < tb ? tb : ta;
                const bool ctl = sp.type == 1;
                const uint32_t cnt = ctl ? TA / 4 : TA / 2;
                const uint32_t cbit = ctl ? 1u << tb : 0u;
                const uint32_t pt = swz(1u << ta) * uint32_t(sizeof(C));  // partner: byte offset XOR
                auto first = [&](uint32_t j) __attribute__((always_inline)) {
                    return swz((ctl ? ins2(j, lo, hi) : ins1(j, ta)) | cbit) * uint32_t(sizeof(C));
                };
                for (uint32_t j = tid; j < cnt; j += kBatchThreads) {
                    const uint32_t o = first(j);
                    const C v0 = lds_at<C>(tileb, o), v1 = lds_at<C>(tileb, o ^ pt);
                    lds_at<C>(tileb, o) = cfma(m01, v1, cmul(m00, v0));
                    lds_at<C>(tileb, o ^ pt) = cfma(m11, v1, cmul(m10, v0));
                }
            } else {
                C m[16];
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    m[e] = M[e];
                const int lo = ta < tb ? ta : tb, hi = ta < tb ? tb : ta;
                const uint32_t cnt = TA / 4;
                // byte-offset XORs of the group members (matrix index e:
                // bit 0 on tile bit ta, bit 1 on tile bit tb)
                uint32_t px[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    px[e] = swz(((e & 1) ? 1u << ta : 0u) | ((e & 2) ? 1u << tb : 0u)) * uint32_t(sizeof(C));
                for (uint32_t j = tid; j < cnt; j += kBatchThreads) {
                    const uint32_t o = swz(ins2(j, lo, hi)) * uint32_t(sizeof(C));
                    C v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e] = lds_at<C>(tileb, o ^ px[e]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        C acc = cmul(m[r * 4], v[0]);
#pragma unroll
                        for (int c = 1; c < 4; ++c)
                            acc = cfma(m[r * 4 + c], v[c], acc);
                        lds_at<C>(tileb, o ^ px[r]) = acc;
                    }
                }
            }
            __syncthreads();
          }
        };
        if (nruns > 0)
            with_nr([&](auto nr) {
                tile_runs<R, decltype(nr)::value>(tileb, a.runs + ps.run0, nruns, a.steps,
                                                  reinterpret_cast<const R *>(a.mats), tw);
            });
        else if (cached)
            sweeps(std::true_type{});
        else
            sweeps(std::false_type{});

        if (!ps.last) {
            if (wide) {
                with_nr([&](auto nr) { RunTile<R, decltype(nr)::value>(ps, tileb, tw).store(st + base); });
            } else if (nsteps_x >= kU) {
                for (uint32_t s0 = 0; s0 < nsteps_x; s0 += kU) {
                    VU v;
#pragma unroll
                    for (uint32_t u = 0; u < kU; ++u) {
                        const C x = tile[swz((s0 + u) * kBatchThreads + uint32_t(tid))];
                        v[2 * u] = x.x;
                        v[2 * u + 1] = x.y;
                    }
#pragma unroll
                    for (uint32_t u = 0; u < kU; ++u) {
                        C x;
                        x.x = v[2 * u];
                        x.y = v[2 * u + 1];
                        store_dev(&st[base + off_of(s0 + u)], x);
                    }
                }
            } else {
                for (uint32_t s = 0; s < nsteps_x; ++s) {
                    if (!active)
                        break;
                    store_dev(&st[base + off_of(s)], tile[swz(s * kBatchThreads + uint32_t(tid))]);
                }
            }
            // Every wave waits for its stores before the barrier; then one
            // thread raises the count.
            publish();
            __syncthreads();
            if (tid == 0)
                __hip_atomic_fetch_add(&done[tk.inst], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const uint64_t *zm = a.zmasks + in.term0;
            auto result = [&](int j, double v) __attribute__((always_inline)) {
                if (ps.ntiles == 1)
                    a.out[in.out0 + j] = v;
                else  // read by the workgroup that finishes the circuit
                    __hip_atomic_store(&a.partials[in.part0 + size_t(tk.tile) * in.nterms + j], v,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            if (runs_tile)
                with_nr([&](auto nr) {
                    tile_strings<R, decltype(nr)::value>(tileb, red, ps, base, zm, in.nterms, tw, result);
                });
            for (int c0 = runs_tile ? in.nterms : 0; c0 < in.nterms; c0 += 16) {
                double acc[16];
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    acc[j] = 0.0;
                for (uint32_t s = 0; s < nsteps_x; ++s) {
                    if (!active)
                        break;
                    const uint32_t x = s * kBatchThreads + uint32_t(tid);
                    const uint64_t gi = base + off_of(s);
                    const C v = tile[swz(x)];
                    const double p = double(v.x) * double(v.x) + double(v.y) * double(v.y);
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (c0 + j < in.nterms)
                            acc[j] += (__popcll(gi & zm[c0 + j]) & 1) ? -p : p;
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const double w = wave_sum(acc[j]);
                    if (lane == 0)
                        red[wave * 16 + j] = w;
                }
                __syncthreads();
                if (tid < 16 && c0 + tid < in.nterms) {
                    double v = red[tid];
#pragma unroll
                    for (int w = 1; w < kBatchThreads / 64; ++w)
                        v += red[16 * w + tid];
                    result(c0 + tid, v);
                }
                __syncthreads();
            }
            if (ps.ntiles > 1) {
                publish();
                __syncthreads();
                if (tid == 0)
                    s_flag = __hip_atomic_fetch_add(&fin[tk.inst], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                             ps.ntiles - 1;
                __syncthreads();
                if (s_flag) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    for (int j = tid; j < in.nterms; j += kBatchThreads) {
                        double sum = 0.0;
                        for (uint32_t tl = 0; tl < ps.ntiles; ++tl)
                            sum += __hip_atomic_load(&a.partials[in.part0 + size_t(tl) * in.nterms + j],
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        a.out[in.out0 + j] = sum;
                    }
                }
            }
        }
        __syncthreads();
    }
}

__global__ void k_batch_fill(uint32_t *ctr, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        ctr[i] = 0u;
}

}  // namespace

// The kernel for tiles of up to 2^tile_log amplitudes: one per widest run, so
// that small tiles keep their residency.
using BatchKernel = void (*)(BatchArgs);
static BatchKernel batch_kernel(int dtype, int tile_log)
{
    switch (batch_runs(tile_log) ? tile_log - kBatchThreadLog : 0) {
    case 3:
        return dtype == SV_C64 ? k_batch<float, 3> : k_batch<double, 3>;
    case 4:
        return dtype == SV_C64 ? k_batch<float, 4> : k_batch<double, 4>;
    case 5:
        return k_batch<float, 5>;  // complex128 tiles end at 2^12
    default:
        return dtype == SV_C64 ? k_batch<float, 0> : k_batch<double, 0>;
    }
}

hipError_t launch_batch(int dtype, const BatchArgs &a, uint32_t grid, size_t lds, hipStream_t s)
{
    if (dtype != SV_C64 && a.tile_log_max > 12)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_kernel(dtype, a.tile_log_max), dim3(grid), dim3(kBatchThreads), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_batch_fill(uint32_t *ctr, uint32_t n, hipStream_t s)
{
    const uint32_t grid = (n + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_batch_fill, dim3(grid < 1 ? 1 : grid), dim3(kThreads), 0, s, ctr, n);
    return hipGetLastError();
}

uint32_t batch_grid(int dtype, int tile_log, size_t lds)
{
    const void *k = reinterpret_cast<const void *>(batch_kernel(dtype, tile_log));
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kBatchThreads, lds) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    return uint32_t(cus * per_cu);
}

}  // namespace sv
