// LDS passes: a sequence of fused 4-qubit blocks applied to one tile per HBM
// round trip.
//
// A pass is a set Q of at most 8 qubits and the blocks of the circuit that act
// inside Q, in circuit order.  Its tile holds the amplitudes spanned by Q and
// the lowest free index bits (2^12 complex64 or 2^11 complex128 amplitudes on
// 256 threads, so that contiguous runs stay at least 128 bytes; twice that on
// 512 threads for passes of at most two (complex64) or three (complex128)
// blocks, which are bound by HBM).  Every block is applied to the tile in LDS
// before the tile goes back to HBM: the state moves once per pass instead of
// once per block, which is the same product of unitaries in the same order
// (paper Sec. 2.1: gate application as sweeps over the amplitudes; Sec. 2.2:
// gate fusion to cut the number of sweeps).
//
// Each block is a dense 16 x 16 unitary on four tile slots (smaller blocks
// are padded with identity on other tile slots by the host).  It runs as the
// complex GEMM Y = U V over the 2^(T-4) groups of the tile, with the three
// real products of the matrix-core sweep (Gauss):
//     P1 = Ur Vr, P2 = Ui Vi, P3 = (Ur + Ui)(Vr + Vi),  Yr = P1 - P2,
//     Yi = P3 - P1 - P2,
// on v_mfma_f32_16x16x4f32 / v_mfma_f64_16x16x4f64.  The block descriptors
// are read with scalar loads; the U fragment of the next block is fetched
// while the current one is multiplied.
//
// Gates may also reach qubits outside the tile: diagonal gates with any of
// their qubits, other gates with their controls.  Those index bits are
// constant within a tile, so on each tile such a gate is a diagonal phase on
// the block's slots, or the gate itself or the identity.  A block whose gates
// reach at most four outer qubits is stored as one fused matrix per value of
// those bits and the tile picks its variant; otherwise (phase gates only) the
// phases are folded into the block's matrix as a column phase (applied before
// the block) or a row phase (after it), from a list of monomials (outer-bit
// mask, slot mask, angle) per block evaluated once per tile into LDS.
#include <algorithm>
#include <cstring>

#include "sv_device.h"
#include "sv_internal.h"

namespace sv {
namespace {

using namespace dev;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename R>
struct PassAcc;
template <>
struct PassAcc<float> {
    using T = floatx4;
};
template <>
struct PassAcc<double> {
    using T = doublex4;
};

__device__ __forceinline__ floatx4 mma16(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mma16(double a, double b, doublex4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// sin and cos of 2 pi u / 2^32 (u: fixed-point turns).  The nearest quarter
// turn k comes from the top bits, the rest x lies in [-pi/4, pi/4) and goes
// through the Taylor series of sin and cos (truncation error below
// (pi/4)^11 / 11! = 2e-9 and (pi/4)^12 / 12! = 1e-10); then the quarter-turn
// rotation.
__device__ __forceinline__ void turn_sincos(uint32_t u, float &sn, float &cs)
{
    const uint32_t k = (u + (1u << 29)) >> 30;
    const float x = float(int32_t(u - (k << 30))) * float(2.0 * M_PI / 4294967296.0);
    const float x2 = x * x;
    const float s = x * (1.0f + x2 * (-1.0f / 6 + x2 * (1.0f / 120 + x2 * (-1.0f / 5040 + x2 * (1.0f / 362880)))));
    const float c = 1.0f + x2 * (-0.5f + x2 * (1.0f / 24 + x2 * (-1.0f / 720 + x2 * (1.0f / 40320 + x2 * (-1.0f / 3628800)))));
    sn = (k & 1) ? c : s;
    cs = (k & 1) ? s : c;
    if (k & 2)
        sn = -sn;
    if ((k + 1) & 2)
        cs = -cs;
}

// The same for 2 pi u / 2^64 in FP64: Taylor terms through x^17 (sin) and
// x^18 (cos), truncation error below (pi/4)^19 / 19! = 2e-19.  (Horner with
// rounded coefficients; a quotient per term took five times the instructions.)
__device__ __forceinline__ void turn_sincos(uint64_t u, double &sn, double &cs)
{
    const uint64_t k = (u + (uint64_t(1) << 61)) >> 62;
    const double x = double(int64_t(u - (k << 62))) * (2.0 * M_PI / 18446744073709551616.0);
    const double x2 = x * x;
    // signed reciprocal factorials
    double s = 1.0 / 355687428096000.0, c = -1.0 / 6402373705728000.0;
    s = fma(s, x2, -1.0 / 1307674368000.0);
    s = fma(s, x2, 1.0 / 6227020800.0);
    s = fma(s, x2, -1.0 / 39916800.0);
    s = fma(s, x2, 1.0 / 362880.0);
    s = fma(s, x2, -1.0 / 5040.0);
    s = fma(s, x2, 1.0 / 120.0);
    s = fma(s, x2, -1.0 / 6.0);
    s = fma(s * x2, x, x);
    c = fma(c, x2, 1.0 / 20922789888000.0);
    c = fma(c, x2, -1.0 / 87178291200.0);
    c = fma(c, x2, 1.0 / 479001600.0);
    c = fma(c, x2, -1.0 / 3628800.0);
    c = fma(c, x2, 1.0 / 40320.0);
    c = fma(c, x2, -1.0 / 720.0);
    c = fma(c, x2, 1.0 / 24.0);
    c = fma(c, x2, -0.5);
    c = fma(c, x2, 1.0);
    sn = (k & 1) ? c : s;
    cs = (k & 1) ? s : c;
    if (k & 2)
        sn = -sn;
    if ((k + 1) & 2)
        cs = -cs;
}

// XOR of x[b] over the set bits b < n of v.
__device__ __forceinline__ uint32_t lane_bits(int v, const uint32_t *x, int n)
{
    uint32_t r = 0;
#pragma unroll
    for (int b = 0; b < n; ++b)
        r ^= x[b] & uint32_t(-((v >> b) & 1));
    return r;
}

// Number of a block's matrix variant on the tile at tbase (scalar unit: read
// through byte loads its latency stood before every tile's and block's loads).
__device__ __forceinline__ uint32_t variant_of(uint64_t tbase, const PassSub &d)
{
    uint32_t var = 0;
    for (uint32_t j = 0; j < d.nvar; ++j)
        var |= uint32_t((tbase >> ((d.vpos >> (8 * j)) & 63)) & 1) << j;
    return var;
}

// Integer add to an LDS word (wrapping).
__device__ __forceinline__ void lds_add(uint32_t *p, uint32_t v)
{
    atomicAdd(p, v);
}
__device__ __forceinline__ void lds_add(uint64_t *p, uint64_t v)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(p), static_cast<unsigned long long>(v));
}

// Diagonal step of a complex64 tile: amplitude x times exp(2 pi i f(x)), f a
// constant, one coefficient per tile bit and one per pair of bits (row: fixed
// point turns at diag_entry()); their sums are exact, each term of the pass was
// rounded to 2^-32 turns (error at most 7e-10 rad).  The angles of a thread's
// amplitudes start from the sum over its thread bits and grow by one addition
// each over the bits its accesses differ in; then a sine and a cosine and one
// complex product per amplitude, on the vector unit.  About 1.4 split blocks or
// one FP32 block, whatever the number of gates (a QFT pass held up to ten
// blocks of nothing else).  In FP64 the kernel would spill (130 registers at
// the four workgroups per CU it needs) and whole QFTs ran 0.88 times as fast.
template <int TA_LOG, int NTH>
__device__ __forceinline__ void diag_step(float2 *tile, const uint32_t *row, int tid)
{
    constexpr int TB = NTH == 512 ? 9 : 8;
    constexpr int NB = TA_LOG - TB;  // bits of a thread's amplitudes: 0 and the highest
    auto reg = [](int b) { return b == 0 ? 0 : TB + b; };
    // x where thread bit k (tile bit k + 1) is set
    auto where = [&](uint32_t x, int k) { return x & uint32_t(-((tid >> k) & 1)); };
    uint32_t f[1 << NB];
    f[0] = row[0];
#pragma unroll
    for (int l = 0; l < TB; ++l) {
        uint32_t s = row[diag_entry(l + 1)];
#pragma unroll
        for (int k = 0; k < l; ++k)
            s += where(row[diag_entry(k + 1, l + 1)], k);
        f[0] += where(s, l);
        __builtin_amdgcn_sched_barrier(0);  // not every coefficient in registers at once
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        __builtin_amdgcn_sched_barrier(0);
        uint32_t s = row[diag_entry(reg(b))];
#pragma unroll
        for (int k = 0; k < TB; ++k)
            s += where(row[k + 1 < reg(b) ? diag_entry(k + 1, reg(b)) : diag_entry(reg(b), k + 1)], k);
        // over the amplitudes with lower register bits e
        uint32_t c[1 << NB];
        c[0] = s;
#pragma unroll
        for (int a = 0; a < b; ++a)
#pragma unroll
            for (int e = 0; e < (1 << a); ++e)
                c[e | 1 << a] = c[e] + row[diag_entry(reg(a), reg(b))];
#pragma unroll
        for (int e = 0; e < (1 << b); ++e)
            f[e | 1 << b] = f[e] + c[e];
    }
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t slot = swz_p<float>(uint32_t(tid) << 1) << 3;
#pragma unroll
    for (int s = 0; s < (1 << NB) / 2; ++s) {
        float4 *p = reinterpret_cast<float4 *>(reinterpret_cast<char *>(tile) +
                                               (slot ^ (swz_p<float>(uint32_t(s * NTH) << 1) << 3)));
        const float4 v = *p;
        float s0, c0, s1, c1;
        turn_sincos(f[2 * s], s0, c0);
        turn_sincos(f[2 * s + 1], s1, c1);
        *p = make_float4(v.x * c0 - v.y * s0, v.x * s0 + v.y * c0, v.z * c1 - v.w * s1, v.z * s1 + v.w * c1);
    }
}

// Residency target: five workgroups per CU fill the LDS with 32 KiB tiles,
// so the complex64 256-thread kernel without phase terms is held to 96
// registers (which also keeps the matrix products in VGPR form, without
// accumulator copies); the others stay at four.
template <typename R, int TA_LOG, bool PAIR, int NTH, bool PHASES>
__global__ __launch_bounds__(NTH)
__attribute__((amdgpu_waves_per_eu(NTH == kThreads && std::is_same<R, float>::value && PAIR && !PHASES ? 5 : 4)))
void k_pass(R *__restrict__ st, const TileArgs a, const PassSub *__restrict__ subs, int nsub,
            const char *__restrict__ mats)
{
    using C = typename CT<R>::C;
    using AccT = typename PassAcc<R>::T;
    constexpr int D = 16, NT = 16, KT = 4, NS = D / KT;
    constexpr int NGS = (1 << (TA_LOG - 4)) / NT;  // group sets (NMT = 1)
    constexpr int NW = NTH / 64;  // waves
    constexpr int PER_WAVE = NGS / NW;
    constexpr bool F64 = std::is_same<R, double>::value;
    constexpr int LG = TA_LOG - 8;  // group bits above the lanes'
    static_assert(NGS % NW == 0 && PER_WAVE >= 1 && LG <= 5, "tile shape");

    __shared__ __align__(16) C tile[1 << TA_LOG];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int ai = lane % 16, akk = lane / 16;  // A operand: U[ai][4 s + akk]
    const int bj = lane % 16, bkk = lane / 16;  // B operand: V[4 s + bkk][group bj]
    const int q = lane / 16;

    // this tile's index bits outside the tile (variant selection, phase terms)
    const uint64_t tbase = insert_zeros_n<TA_LOG>(uint64_t(blockIdx.y) * gridDim.x + blockIdx.x, a.outer);
    // this lane's fragment of block sb's matrix: U[ai][4 s + akk], s < NS;
    // a block with variants stores one matrix per value of its selecting
    // index bits, consecutively
    auto load_u = [&](int sb, R *xr, R *xi) {
        const PassSub &d = subs[sb];
        const uint32_t var = variant_of(tbase, d);
        const C *U = reinterpret_cast<const C *>(mats + d.u_off) + size_t(var) * (D * D) + ai * D + akk;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const C u = U[s * KT];
            xr[s] = u.x;
            xi[s] = u.y;
        }
    };
    // a diagonal step (complex64 passes with phases) has no matrix
    auto has_matrix = [&](int sb) { return !(PHASES && !F64 && subs[sb].diag); };
    R ur[NS], ui[NS];

    // Per-tile phase angles of the blocks carrying phase terms, in an LDS
    // table: row pslot holds the 16 column angles (front terms) and the 16
    // row angles (back terms) of that block on this tile, in fixed-point
    // turns (exact sums wrapping mod 2 pi: 32 bits for complex64, to which
    // the terms come rounded, 64 for complex128).  Wave w fills the rows of
    // term blocks w, w + NW, ...: its lanes take the block's monomials
    // e = lane, lane + 64, ... and each one
    // whose outer bits this tile has adds its turn to the row's (side, slot
    // mask) entry with an LDS atomic add (integer sums: the same in any
    // order); a subset sum over the four mask bits across lanes then gives
    // angle(c) = sum of the entries m within c.
    using TurnT = typename std::conditional<F64, uint64_t, uint32_t>::type;
    __shared__ TurnT angles[PHASES ? kMaxTermBlocks * 32 : 1];
    auto fill_angles = [&]() {
        for (int sb = 0; sb < nsub; ++sb) {
            const PassSub &d = subs[sb];
            // a diagonal step reads its rows also where no term is left
            if ((d.nterm == 0 && !d.diag) || int(d.pslot % NW) != wave)
                continue;
            const PassTerm *tm = reinterpret_cast<const PassTerm *>(mats + d.t_off);
            TurnT *row = angles + d.pslot * 32;
            for (int k = lane; k < (d.diag ? kDiagRows * 32 : 32); k += 64)
                row[k] = 0;
            for (uint32_t e = uint32_t(lane); e < d.nterm; e += 64) {
                const PassTerm t = tm[e];
                if ((tbase & t.omask) == t.omask)
                    lds_add(&row[t.back * 16 + t.smask], TurnT(F64 ? t.turn : (t.turn >> 32)));
            }
            if (d.diag)
                continue;  // coefficients, not sums
            // this wave's LDS operations complete in order: the entries are final
            TurnT acc = lane < 32 ? row[lane] : TurnT(0);
#pragma unroll
            for (int bit = 1; bit < 16; bit <<= 1) {
                const TurnT other = __shfl_xor(acc, bit);
                if (lane & bit)
                    acc += other;
            }
            if (lane < 32)
                row[lane] = acc;
        }
    };
    // U[r][c] * exp(i (front(c) + back(r))) for this lane's fragment of a
    // block carrying phase terms (table filled for this tile)
    auto apply_phases = [&](const PassSub &d) {
        if (PHASES && d.nterm > 0 && !d.diag) {
            const TurnT *row = angles + d.pslot * 32;
            const TurnT tb = row[16 + ai];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                R sn, cs;
                turn_sincos(TurnT(row[s * KT + akk] + tb), sn, cs);
                const R r0 = ur[s], i0 = ui[s];
                ur[s] = r0 * cs - i0 * sn;
                ui[s] = r0 * sn + i0 * cs;
            }
        }
    };

    // the first block's operands follow the tile's loads
    auto first = [&]() {
        if (has_matrix(0))
            load_u(0, ur, ui);
    };
    tile_sweep<R, TA_LOG, PAIR, NTH, true>(st, a, tile, [&](C *t) {
        if (PHASES) {
            fill_angles();
            __syncthreads();
        }
        // phases of block sb + 1 are folded in at the end of iteration sb,
        // where no accumulator is live
        apply_phases(subs[0]);
        for (int sb = 0; sb < nsub; ++sb) {
            R nr[NS], ni[NS];
            if (sb + 1 < nsub && has_matrix(sb + 1))
                load_u(sb + 1, nr, ni);
            const PassSub &d = subs[sb];
            if constexpr (PHASES && !F64)
                if (d.diag) {
                    diag_step<TA_LOG, NTH>(t, angles + d.pslot * 32, tid);
                    __syncthreads();
                    if (sb + 1 < nsub && has_matrix(sb + 1)) {
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            ur[s] = nr[s];
                            ui[s] = ni[s];
                        }
                        apply_phases(subs[sb + 1]);
                    }
                    continue;
                }
            // LDS addresses.  The byte offset of a (row, group) is linear over
            // XOR in its bits (d.rx, d.gx: swizzled), and the bits are the
            // lane's (row bits from bkk or the accumulator row, group bits
            // 0..3 from bj) or wave-uniform (row bits from the k-step or
            // register, group bits from wave + NW j): the lane parts are
            // computed once per block, the uniform parts on the scalar unit,
            // and each access costs one XOR.
            const uint32_t gl = lane_bits(bj, d.gx, 4);
            const uint32_t in_lane = gl ^ lane_bits(bkk, d.rx, 2);
            const uint32_t out_lane = F64 ? in_lane : gl ^ lane_bits(q, d.rx + 2, 2);
            uint32_t hj[PER_WAVE];
#pragma unroll
            for (int j = 0; j < PER_WAVE; ++j)
                hj[j] = lane_bits(wave + NW * j, d.gx + 4, LG);
            char *tb = reinterpret_cast<char *>(t);
            AccT p1[PER_WAVE], p2[PER_WAVE], p3[PER_WAVE];
#pragma unroll
            for (int j = 0; j < PER_WAVE; ++j) {
                p1[j] = AccT{};
                p2[j] = AccT{};
                p3[j] = AccT{};
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const uint32_t ss = lane_bits(s, d.rx + 2, 2);
                const R us = ur[s] + ui[s];
#pragma unroll
                for (int j = 0; j < PER_WAVE; ++j) {
                    const C x = *reinterpret_cast<const C *>(tb + (in_lane ^ (ss ^ hj[j])));
                    p1[j] = mma16(ur[s], x.x, p1[j]);
                    p2[j] = mma16(ui[s], x.y, p2[j]);
                    p3[j] = mma16(us, x.x + x.y, p3[j]);
                }
            }
            // Each item writes back exactly the 16 groups x 16 rows it read,
            // so no other wave touches these locations within this block:
            // only the next block (other slots) needs the barrier below.
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // accumulator row: 4 (lane / 16) + r (FP32), 4 r + lane / 16 (FP64)
                const uint32_t rr = lane_bits(r, d.rx + (F64 ? 2 : 0), 2);
#pragma unroll
                for (int j = 0; j < PER_WAVE; ++j) {
                    C y;
                    y.x = p1[j][r] - p2[j][r];
                    y.y = p3[j][r] - p1[j][r] - p2[j][r];
                    *reinterpret_cast<C *>(tb + (out_lane ^ (rr ^ hj[j]))) = y;
                }
            }
            __syncthreads();
            if (sb + 1 < nsub && has_matrix(sb + 1)) {
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    ur[s] = nr[s];
                    ui[s] = ni[s];
                }
                apply_phases(subs[sb + 1]);
            }
        }
    }, SameSlot(), first);
}

// ---------------------------------------------------------------------------
// Complex64 passes with FP32-accurate split BF16 products.
//
// Each FP32 value x is split exactly into three BF16 parts, x = h + m + l
// (h = bf16(x), m = bf16(x - h), l = x - h - m, rounding to nearest: x - h
// and x - h - m are exact FP32 differences and the last has at most 8
// significant bits, so l is exact as well; |m| <= 2^-8 |x|, |l| <= 2^-16 |x|).
// A real product X Y is then the six BF16 products Xh Yh + Xh Ym + Xm Yh +
// Xh Yl + Xm Ym + Xl Yh; the three dropped ones (Xm Yl, Xl Ym, Xl Yl) are
// below 2^-23 |X||Y| together, and the BF16 products are exact in the FP32
// accumulator.  The block runs as one real contraction of the complex
// product: [Yr; Yi] = [[Ur, -Ui], [Ui, Ur]] [Vr; Vi], K = 32 real terms, on
// v_mfma_f32_16x16x32_bf16 (BF16 matrix rate, 16x that of FP32): two 16-row
// output tiles (real and imaginary rows) x six products per group set.
//
// The K index is ordered so that lane l (q = l / 16, j = l % 16) supplies
// B[8 q + 2 r + c][j] = component c of amplitude row 4 q + r of group j, and
// receives D[4 q + i][j]: output tile t holds component i % 2 of row
// 4 q + 2 t + i / 2 there, so each lane reads and writes the same four
// amplitudes of a group (no barrier between group sets) and each amplitude's
// components come out in two adjacent registers, as the LDS write takes them.
// A[j][8 q + 2 r + c] of tile t holds U entries of row 4 (j / 4) + 2 t +
// j % 4 / 2, column 4 q + r.  Products are accumulated smallest first.
//
// What bounds it: the matrix products of a group set take 192 cycles of a SIMD,
// and each also takes issue slots from the 52 other vector instructions (44 of
// them the splits); both together run in 338 cycles with five waves per SIMD and
// nothing else in the loop.  On 28 qubits a pass of one block takes 0.69 ms (the
// copy rate), of two to five 0.80, 0.90, 1.02 and 1.17; with outputs moved into
// adjacent registers, operands copied between blocks, group bits in ascending
// order on the lanes and masks read one by one (69 instructions per group set,
// 268 instead of 105 for a wave's share of a tile's loads and stores, half the
// LDS cycles bank conflicts) 0.69, 0.81, 0.93, 1.17 and 1.41.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// (a, b) as two BF16 values in one register, a in the low half.  The empty
// asm keeps the compiler from re-deriving either half by a separate
// conversion.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const bf16x2_t p = {__bf16(a), __bf16(b)};
    uint32_t r = __builtin_bit_cast(uint32_t, p);
    asm("" : "+v"(r));
    return r;
}

// Exact three-part split of the pair (a, b): parts packed as by pack_bf16.
// (The residuals as BF16 dot products with (-1, 0) and (0, -1) take 7 instead
// of 11 instructions, but those do not run beside the matrix products: 12 of
// the products, 12 conversions and 41 plain instructions take 338 cycles at
// 2.4 GHz, with 16 dot products for 32 of the 41 448.)
__device__ __forceinline__ void split3(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = pack_bf16(a, b);
    const float ra = a - __builtin_bit_cast(float, h << 16);
    const float rb = b - __builtin_bit_cast(float, h & 0xffff0000u);
    m = pack_bf16(ra, rb);
    const float sa = ra - __builtin_bit_cast(float, m << 16);
    const float sb = rb - __builtin_bit_cast(float, m & 0xffff0000u);
    l = pack_bf16(sa, sb);
}

// x of another lane of the lane's four: SEL holds two bits per lane.
template <int SEL>
__device__ __forceinline__ float quad_move(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), SEL, 0xf, 0xf, true));
}

__device__ __forceinline__ bf16x8_t as_bf16x8(const uint32_t *w)
{
    const u32x4_t v = {w[0], w[1], w[2], w[3]};
    return __builtin_bit_cast(bf16x8_t, v);
}

// acc + (Ah + Am + Al)(Bh + Bm + Bl) without the three smallest products,
// smallest first
__device__ __forceinline__ floatx4 mma_split6(const uint32_t *ah, const uint32_t *am, const uint32_t *al,
                                              const bf16x8_t &bh, const bf16x8_t &bm, const bf16x8_t &bl)
{
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(al), bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(am), bm, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ah), bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(am), bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ah), bm, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ah), bh, acc, 0, 0, 0);
    return acc;
}

// PHASES: some block carries per-tile phase terms; the blocks' matrices are
// FP32 and every workgroup applies its tile's phases and splits them.
// Otherwise the matrices come split already (pass_presplit), and the kernel
// only loads each lane's A fragments.  NTH: 256 threads (five workgroups per
// CU, for passes of several blocks) or 512 (three, for one-block passes only,
// which are bound by HBM: 8 waves share a tile's loads and its one block).
template <bool PHASES, int NTH>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(PHASES ? 4 : (NTH == 256 ? 5 : 1))))
void k_pass_split(float *__restrict__ st, const TileArgs a, const PassSub *__restrict__ subs, int nsub,
                  const char *__restrict__ mats)
{
    using C = float2;
    constexpr int TA_LOG = 12;
    constexpr int D = 16, NT = 16;
    constexpr int NGS = (1 << (TA_LOG - 4)) / NT;  // group sets of 16 groups
    constexpr int NW = NTH / 64;
    constexpr int PER_WAVE = NGS / NW;
    static_assert(PER_WAVE >= 1 && NGS % NW == 0, "tile shape");

    __shared__ __align__(16) C tile[1 << TA_LOG];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int q = lane / 16, j16 = lane % 16;

    const uint64_t tbase = insert_zeros_n<TA_LOG>(uint64_t(blockIdx.y) * gridDim.x + blockIdx.x, a.outer);
    // PHASES: this lane's FP32 fragment of block sb, U[j16][4 q + r], r < 4
    auto load_u = [&](int sb, float *ur, float *ui) {
        const PassSub &d = subs[sb];
        const float4 *U = reinterpret_cast<const float4 *>(reinterpret_cast<const C *>(mats + d.u_off) +
                                                           size_t(variant_of(tbase, d)) * (D * D) + j16 * D + 4 * q);
        const float4 u0 = U[0], u1 = U[1];
        ur[0] = u0.x;
        ui[0] = u0.y;
        ur[1] = u0.z;
        ui[1] = u0.w;
        ur[2] = u1.x;
        ui[2] = u1.y;
        ur[3] = u1.z;
        ui[3] = u1.w;
    };
    // otherwise: this lane's split A fragments of block sb, in the order
    // (h, tile 0), (h, tile 1), (m, 0), (m, 1), (l, 0), (l, 1), four registers
    // each
    auto load_a = [&](int sb, uint32_t *A) {
        const PassSub &d = subs[sb];
        const uint4 *P = reinterpret_cast<const uint4 *>(mats + d.u_off + size_t(variant_of(tbase, d)) * kPresplitBytes) + lane;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const uint4 v = P[i * 64];
            A[4 * i] = v.x;
            A[4 * i + 1] = v.y;
            A[4 * i + 2] = v.z;
            A[4 * i + 3] = v.w;
        }
    };
    float ur[4], ui[4];
    uint32_t a0[24], a1[24];  // this block's and the next one's

    // per-tile phase angles, as in k_pass (fixed-point turns, 32 bits)
    __shared__ uint32_t angles[PHASES ? kMaxTermBlocks * 32 : 1];
    auto fill_angles = [&]() {
        for (int sb = 0; sb < nsub; ++sb) {
            const PassSub &d = subs[sb];
            // a diagonal step reads its rows also where no term is left
            if ((d.nterm == 0 && !d.diag) || int(d.pslot % NW) != wave)
                continue;
            const PassTerm *tm = reinterpret_cast<const PassTerm *>(mats + d.t_off);
            uint32_t *row = angles + d.pslot * 32;
            for (int k = lane; k < (d.diag ? kDiagRows * 32 : 32); k += 64)
                row[k] = 0;
            for (uint32_t e = uint32_t(lane); e < d.nterm; e += 64) {
                const PassTerm t = tm[e];
                if ((tbase & t.omask) == t.omask)
                    lds_add(&row[t.back * 16 + t.smask], uint32_t(t.turn >> 32));
            }
            if (d.diag)
                continue;  // coefficients, not sums
            uint32_t acc = lane < 32 ? row[lane] : 0u;
#pragma unroll
            for (int bit = 1; bit < 16; bit <<= 1) {
                const uint32_t other = __shfl_xor(acc, bit);
                if (lane & bit)
                    acc += other;
            }
            if (lane < 32)
                row[lane] = acc;
        }
    };

    // the first block's operands follow the tile's loads
    auto first = [&]() {
        if constexpr (PHASES) {
            if (!subs[0].diag)
                load_u(0, ur, ui);
        } else {
            load_a(0, a0);
        }
    };
    tile_sweep<float, TA_LOG, true, NTH, true>(st, a, tile, [&](C *t) {
        if (PHASES) {
            fill_angles();
            __syncthreads();
        }
        // A operands of block sb from its FP32 fragment, this tile's phases
        // applied
        auto split_u = [&](int sb, uint32_t *A) {
            const PassSub &d = subs[sb];
            if (d.nterm > 0) {
                // U[r][c] exp(i (front(c) + back(r))), r = j16, c = 4 q + k
                const uint32_t *row = angles + d.pslot * 32;
                const uint32_t tb = row[16 + j16];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float sn, cs;
                    turn_sincos(uint32_t(row[4 * q + k] + tb), sn, cs);
                    const float r0 = ur[k], i0 = ui[k];
                    ur[k] = r0 * cs - i0 * sn;
                    ui[k] = r0 * sn + i0 * cs;
                }
            }
            // output tile t takes row 2 t + j16 % 4 / 2 of the lane's four:
            // real rows [Ur, -Ui], imaginary rows [Ui, Ur]
            const bool im = (lane & 1) != 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float r0 = quad_move<0x50>(ur[k]), i0 = quad_move<0x50>(ui[k]);
                const float r1 = quad_move<0xfa>(ur[k]), i1 = quad_move<0xfa>(ui[k]);
                split3(im ? i0 : r0, im ? r0 : -i0, A[k], A[8 + k], A[16 + k]);
                split3(im ? i1 : r1, im ? r1 : -i1, A[4 + k], A[12 + k], A[20 + k]);
            }
        };
        // LDS byte offsets (XOR-linear parts, as in k_pass): lane part from
        // (q, j16), register part from the row r, wave-uniform part from the
        // group set
        char *tb = reinterpret_cast<char *>(t);
        auto block = [&](int sb, const uint32_t *A) {
            const PassSub &d = subs[sb];
            const uint32_t lane_off = lane_bits(j16, d.gx, 4) ^ lane_bits(q, d.rx + 2, 2);
            uint32_t uoff[PER_WAVE][4];
#pragma unroll
            for (int g = 0; g < PER_WAVE; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    uoff[g][r] = lane_bits(wave + NW * g, d.gx + 4, 4) ^ lane_bits(r, d.rx, 2);
            float v[8];
            auto read = [&](int g) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const C x = *reinterpret_cast<const C *>(tb + (lane_off ^ uoff[g][r]));
                    v[2 * r] = x.x;
                    v[2 * r + 1] = x.y;
                }
            };
            read(0);
#pragma unroll
            for (int g = 0; g < PER_WAVE; ++g) {
                uint32_t bh[4], bm[4], bl[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    split3(v[2 * r], v[2 * r + 1], bh[r], bm[r], bl[r]);
                if (g + 1 < PER_WAVE)
                    read(g + 1);  // other groups than the ones written below
                const bf16x8_t Bh = as_bf16x8(bh), Bm = as_bf16x8(bm), Bl = as_bf16x8(bl);
                const floatx4 y0 = mma_split6(A, A + 8, A + 16, Bh, Bm, Bl);
                const floatx4 y1 = mma_split6(A + 4, A + 12, A + 20, Bh, Bm, Bl);
                *reinterpret_cast<C *>(tb + (lane_off ^ uoff[g][0])) = make_float2(y0[0], y0[1]);
                *reinterpret_cast<C *>(tb + (lane_off ^ uoff[g][1])) = make_float2(y0[2], y0[3]);
                *reinterpret_cast<C *>(tb + (lane_off ^ uoff[g][2])) = make_float2(y1[0], y1[1]);
                *reinterpret_cast<C *>(tb + (lane_off ^ uoff[g][3])) = make_float2(y1[2], y1[3]);
            }
            __syncthreads();
        };
        if constexpr (PHASES) {
            for (int sb = 0; sb < nsub; ++sb) {
                const bool diag = subs[sb].diag != 0;
                if (!diag)
                    split_u(sb, a0);
                if (sb + 1 < nsub && !subs[sb + 1].diag)
                    load_u(sb + 1, ur, ui);
                if (diag) {
                    diag_step<TA_LOG, NTH>(t, angles + subs[sb].pslot * 32, tid);
                    __syncthreads();
                } else {
                    block(sb, a0);
                }
            }
        } else if constexpr (NTH == 512) {
            block(0, a0);  // one-block passes only: no second operand set
        } else {
            // two blocks per iteration, each loading the other's operands
            for (int sb = 0; sb < nsub; sb += 2) {
                if (sb + 1 < nsub)
                    load_a(sb + 1, a1);
                block(sb, a0);
                if (sb + 1 < nsub) {
                    if (sb + 2 < nsub)
                        load_a(sb + 2, a0);
                    block(sb + 1, a1);
                }
            }
        }
    }, SameSlot(), first);
}

template <typename R, int TA_LOG, int NTH>
hipError_t launch_pass_t(void *st, const TileArgs &a, const void *subs, int nsub, const void *mats, bool phases,
                         hipStream_t s)
{
    constexpr bool F32 = std::is_same<R, float>::value;
    // a pass tile always holds physical bit 0 (a pass qubit or the lowest
    // free bit), so complex64 moves 16-byte amplitude pairs
    if (F32 && a.dep[0] != 1)
        return hipErrorInvalidValue;
    const PassSub *ps = static_cast<const PassSub *>(subs);
    const char *m = static_cast<const char *>(mats);
    if (phases)
        hipLaunchKernelGGL((k_pass<R, TA_LOG, F32, NTH, true>), tile_grid(a.ntiles), dim3(NTH), 0, s, (R *)st, a, ps,
                           nsub, m);
    else
        hipLaunchKernelGGL((k_pass<R, TA_LOG, F32, NTH, false>), tile_grid(a.ntiles), dim3(NTH), 0, s, (R *)st, a, ps,
                           nsub, m);
    return hipGetLastError();
}

}  // namespace

// BF16 bits of x rounded to nearest even (x finite), as v_cvt_pk_bf16_f32.
static uint32_t bf16_rne_bits(float x)
{
    uint32_t u;
    std::memcpy(&u, &x, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// Host twin of split3: (a, b) -> packed parts h, m, l.
static void split3_host(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    auto part = [](float x, float &rest) {
        const uint32_t bits = bf16_rne_bits(x);
        const uint32_t w = bits << 16;
        float v;
        std::memcpy(&v, &w, 4);
        rest = x - v;  // exact
        return bits;
    };
    float ra, rb, sa, sb;
    const uint32_t ha = part(a, ra), hb = part(b, rb);
    const uint32_t ma = part(ra, sa), mb = part(rb, sb);
    h = ha | (hb << 16);
    m = ma | (mb << 16);
    l = bf16_rne_bits(sa) | (bf16_rne_bits(sb) << 16);
}

void pass_presplit(const std::complex<double> *U, void *dst)
{
    uint32_t *o = static_cast<uint32_t *>(dst);
    for (int lane = 0; lane < 64; ++lane) {
        const int q = lane / 16, j = lane % 16;
        for (int t = 0; t < 2; ++t)
            for (int k = 0; k < 4; ++k) {
                const std::complex<double> u = U[(4 * (j / 4) + 2 * t + j % 4 / 2) * 16 + 4 * q + k];
                const float re = float(u.real()), im = float(u.imag());
                uint32_t p[3];
                if (j % 2 == 0)
                    split3_host(re, -im, p[0], p[1], p[2]);
                else
                    split3_host(im, re, p[0], p[1], p[2]);
                for (int part = 0; part < 3; ++part)
                    o[((part * 2 + t) * 64 + lane) * 4 + k] = p[part];
            }
    }
}

// Bank bit that tile bit b reaches under swz_p, -1 for none: complex64 accesses
// are 8 bytes wide and half a wave's cover 32 slots (bits 0..4), complex128 ones
// 16 bytes and a quarter wave's cover 16 (bits 0..3).
static int bank_bit(int dtype, int b)
{
    const uint32_t y = dtype == SV_C64 ? swz_p<float>(1u << b) : swz_p<double>(1u << b);
    const uint32_t m = y & (dtype == SV_C64 ? 31u : 15u);
    return m ? __builtin_ctz(m) : -1;
}

// The lanes that one access serves together differ in the four group bits and,
// complex64, in the low lane row bit (row bit 2 of the split kernel, whose lanes
// take row bits 2 and 3, 0 of the others).  Each should reach a bank bit of its
// own: the row bit takes one that no group bit reaches, if there is one.
// (Group bits in ascending order and the swizzle x ^ (x >> 6): two thirds of
// the LDS cycles of a 29-qubit QFT's low passes were conflicts.)
void pass_layout(int dtype, bool split, int T, const int *slots, int *order, PassSub &d)
{
    const bool f32 = dtype == SV_C64;
    const int nbank = f32 ? 5 : 4;
    auto off = [&](int b) { return f32 ? swz_p<float>(1u << b) << 3 : swz_p<double>(1u << b) << 4; };
    uint32_t used = 0;
    for (int j = 0; j < 4; ++j)
        used |= 1u << slots[j];
    int by_bank[5] = {-1, -1, -1, -1, -1};  // lowest group bit reaching each bank bit
    for (int b = T - 1; b >= 0; --b)
        if (!((used >> b) & 1) && bank_bit(dtype, b) >= 0)
            by_bank[bank_bit(dtype, b)] = b;
    int row = 0, row_bank = -1;  // the slot of the lanes' low row bit
    if (f32)
        for (int j = 0; j < 4; ++j) {
            const int k = bank_bit(dtype, slots[j]);
            if (k >= 0 && (row_bank < 0 || (by_bank[k] < 0 && by_bank[row_bank] >= 0))) {
                row = j;
                row_bank = k;
            }
        }
    int g[9], n = 0;
    for (int k = 0; k < nbank && n < 4; ++k)
        if (k != row_bank && by_bank[k] >= 0) {
            g[n++] = by_bank[k];
            used |= 1u << by_bank[k];
        }
    for (int b = 0; b < T; ++b)
        if (!((used >> b) & 1))
            g[n++] = b;
    for (int b = 0; b < T - 4; ++b)
        d.gx[b] = off(g[b]);
    for (int b = 0; b < 4; ++b)
        order[b] = b;
    std::swap(order[split ? 2 : 0], order[row]);
    for (int b = 0; b < 4; ++b)
        d.rx[b] = off(slots[order[b]]);
}

int pass_tile_log(int dtype)
{
    return dtype == SV_C64 ? 12 : 11;
}

int pass_tile_log_for(int n, int dtype, int nsub)
{
    // Passes with few blocks are bound by HBM, and twice the tile (512
    // threads, 64 KiB of LDS) doubles the contiguous runs of a pass whose
    // qubits are all high; with more blocks the matrix cores bind and the
    // smaller tile, with more workgroups per CU, overlaps better.  Complex128
    // takes the larger tile up to three blocks.  Complex64 keeps the 2^12
    // tile throughout: its runs are already 128 bytes, and on MI355X the
    // 2^13 tile measured no faster for one or two blocks (whole circuits
    // 0.2-0.7 % slower with it).  Small states keep the small tile (enough
    // tiles to spread).
    const int T = pass_tile_log(dtype);
    const int few = dtype == SV_C64 ? 0 : 3;
    return (nsub <= few && n >= T + 1 + 6) ? T + 1 : T;
}

int pass_tile_bits(int n, int T, uint64_t phys_qmask, uint64_t phys_avoid, int *tile_bits)
{
    const int q = __builtin_popcountll(phys_qmask);
    if (T < 1 || T > 16 || n < T || n > 63 || q > T || (phys_qmask >> n) != 0 ||
        (phys_qmask & phys_avoid) != 0)
        return -1;
    int got = 0;
    for (int p = 0; p < n; ++p)
        if ((phys_qmask >> p) & 1)
            tile_bits[got++] = p;
    for (int p = 0; p < n && got < T; ++p)
        if (!(((phys_qmask | phys_avoid) >> p) & 1))
            tile_bits[got++] = p;
    if (got != T)
        return -1;
    std::sort(tile_bits, tile_bits + T);
    return T;
}

hipError_t launch_pass(void *st, int n, int dtype, int T, const int *tile_bits, const void *d_subs, int nsub,
                       const void *d_mats, bool phases, bool split, hipStream_t s)
{
    const int T0 = pass_tile_log(dtype);
    if (nsub < 1 || (T != T0 && T != T0 + 1) || n < T)
        return hipErrorInvalidValue;
    if (split && (dtype != SV_C64 || T != 12))
        return hipErrorInvalidValue;
    TileArgs a{};
    std::vector<int> bits(tile_bits, tile_bits + T);
    for (int b = 0; b < T; ++b)
        a.dep[b] = uint64_t(1) << bits[b];
    a.outer = make_insert_masks(bits);
    a.ntiles = uint64_t(1) << (n - T);
    if (split) {
        if (a.dep[0] != 1)
            return hipErrorInvalidValue;
        const PassSub *ps = static_cast<const PassSub *>(d_subs);
        const char *m = static_cast<const char *>(d_mats);
        // one-block passes on 512 threads: on 28-qubit tiles 0.67-0.77 ms
        // against 0.70-0.93 on 256 (most for high pass qubits), while from
        // two blocks on 256 threads are faster (2 blocks 0.775 against 0.823,
        // 4 blocks 1.11 against 1.27 ms)
        const dim3 g = tile_grid(a.ntiles);
        if (nsub == 1) {
            if (phases)
                hipLaunchKernelGGL((k_pass_split<true, 512>), g, dim3(512), 0, s, (float *)st, a, ps, nsub, m);
            else
                hipLaunchKernelGGL((k_pass_split<false, 512>), g, dim3(512), 0, s, (float *)st, a, ps, nsub, m);
        } else {
            if (phases)
                hipLaunchKernelGGL((k_pass_split<true, 256>), g, dim3(256), 0, s, (float *)st, a, ps, nsub, m);
            else
                hipLaunchKernelGGL((k_pass_split<false, 256>), g, dim3(256), 0, s, (float *)st, a, ps, nsub, m);
        }
        return hipGetLastError();
    }
    if (dtype == SV_C64)
        return T == 12 ? launch_pass_t<float, 12, kThreads>(st, a, d_subs, nsub, d_mats, phases, s)
                       : launch_pass_t<float, 13, 512>(st, a, d_subs, nsub, d_mats, phases, s);
    return T == 11 ? launch_pass_t<double, 11, kThreads>(st, a, d_subs, nsub, d_mats, phases, s)
                   : launch_pass_t<double, 12, 512>(st, a, d_subs, nsub, d_mats, phases, s);
}

}  // namespace sv
