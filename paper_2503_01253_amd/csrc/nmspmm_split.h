// Tiled kernel of the 16-wave tiles: fp32 products on the bf16 matrix
// instruction (device code, included by the per-shape instantiation units).
//
// v_mfma_f32_32x32x2_f32 does 128 flops per cycle and SIMD, 157 TFLOP/s on
// the chip; v_mfma_f32_32x32x16_bf16 does 1024.  Every fp32 operand is
// therefore split into three bf16 parts, x = h + m + l, each the bf16 nearest
// to what the parts before it leave: 3 x 8 significant bits and their signs
// hold all 24 bits of x, so the split is exact (for |x| >= 2^-110; below that
// the last part ends at bf16's smallest step and x is off by at most 2^-134).
// A product a*b is then the six part products of weight 2^-16 and above
//   hh + hm + mh + mm + hl + lh
// (the three left out are below 2^-25 of |a*b|), each exact in fp32, summed
// in the fp32 accumulators.  Against fp64 the sum is closer than the fp32
// instruction's, which rounds after every second term where this one rounds
// after every sixteenth: relative error on U[-1, 1] data at w = 32 / 512 /
// 2048 / 4096 terms 6.8e-8 / 3.3e-7 / 7.0e-7 / 9.8e-7, against 1.0e-7 /
// 4.1e-7 / 8.1e-7 / 1.1e-6 (three part products alone: 3.8e-6, so six it is).
// Six instructions of 32 cycles for 16 compressed rows of a 32 x 32 tile take
// the place of eight of 64 cycles.
//
// An operand that is infinite or NaN, or that rounds to an infinite bf16, has
// no such split (its further parts are NaN), and one below 2^-110 an inexact
// one.  A workgroup whose sums the split cannot vouch for forms its tile again
// on the fp32 instruction, so that such inputs give what that instruction
// gives (see the end of the kernel for the conditions).
//
// One workgroup of 16 waves owns a BM x BN tile of C (and, with split-k, one
// slice of the k range), each wave WM x 32 of it inside one column block.  It
// walks k in stages of KA columns of A (KA/M whole windows, RS = (KA/M)*N
// compressed rows, padded to 16*KS).
//   A_s : the BM x KA slab of A as three bf16 planes, k-major: plane row c
//         holds column c of A, BM rows.  Global -> registers -> split -> LDS.
//         Each thread splits a TR x TC block and writes, per column and
//         plane, TR consecutive rows.
//   gather: ds_read_b64_tr_b16 reads, for 16 lanes, four plane rows of 16
//         output rows each and hands every lane the four values of its own
//         output row.  The four plane rows are four consecutive compressed
//         rows, each at its own address: the N:M gather of Eq. 1 costs no
//         instruction beyond the read itself.
//   Bc  : straight from global memory into registers (8 rows of its column
//         per lane, one K step ahead), split there: no LDS traffic.
//   X_s : for each of the stage's compressed rows and the tile's column blocks
//         the place in A_s of the plane row it gathers, formed from the offset
//         byte by the thread that loads it (by the readers, 18 instructions a
//         K step and four registers more).
// LDS rows are 16-output-row granules of 32 bytes; granule g of plane row c
// lies at position g ^ swz(c), which spreads both the transposed reads (four
// plane rows at one granule) and the writes (one granule of many plane rows)
// over the banks.
#ifndef NMSPMM_SPLIT_H
#define NMSPMM_SPLIT_H

#include "nmspmm_tiled.h"

namespace nmspmm {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) unsigned char lds_u8;

// The three bf16 parts of two floats, packed in pairs (x0 in the low half).
// (Subtracting a part by v_dot2_f32_bf16 instead of unpacking it first saves
// two of eleven instructions and measured 0-4 % slower: the chip is at its
// power limit, and the dot product costs more than the unpack.)
__device__ __forceinline__ void split3(float x0, float x1, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0, x1}), bf16x2));
    const float r0 = x0 - __builtin_bit_cast(float, h << 16);
    const float r1 = x1 - __builtin_bit_cast(float, h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
    const float s0 = r0 - __builtin_bit_cast(float, m << 16);
    const float s1 = r1 - __builtin_bit_cast(float, m & 0xffff0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{s0, s1}), bf16x2));
}

template <int BM_, int BN_, int WM_>
struct SplitTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, NW = (BM / WM) * (BN / 32), NT = 64 * NW;
    static constexpr int NRT = WM / 32;          // 32-row MFMA tiles per wave
    static constexpr int NGRAN = BM / 16;        // granules per plane row
    static constexpr int STRIDE = 2 * BM;        // bytes of a plane row
    static constexpr int QBMAX = BN / 32;        // column blocks per tile, at most
    static_assert(NW == 16 && NGRAN % 8 == 0 && WM % 32 == 0, "tile shape");
};

// Per-instantiation constants: stages of KA columns of A and KS K steps of 16
// padded compressed rows.
template <class T, int KA, int KS>
struct SplitShape {
    static constexpr int RST = 16 * KS;
    static constexpr int PLANE = KA * T::STRIDE, A_BYTES = 3 * PLANE;
    static constexpr int X_ENTRIES = RST * T::QBMAX, X_BYTES = 4 * X_ENTRIES;
    // two A slots where they fit; otherwise one, overwritten after a second
    // barrier from the registers that hold the next stage's slab
    static constexpr bool TWO_A = 2 * (A_BYTES + X_BYTES) <= LDS_CAPACITY;
    static constexpr int A_SLOTS = TWO_A ? 2 : 1;
    static constexpr int LDS_BYTES = A_SLOTS * A_BYTES + 2 * X_BYTES;
    // a thread's TR x TC block of A, in its wave's chunk of CR rows x 32 columns
    static constexpr int E = T::BM * KA / T::NT;
    static constexpr int TR = E >= 8 ? 4 : 2, TC = E / TR, CR = 2 * TC * TR;
    static constexpr bool FITS = LDS_BYTES <= LDS_CAPACITY && X_ENTRIES <= T::NT &&
                                 (E == 4 || E == 8 || E == 16) && (T::BM / CR) * (KA / 32) == T::NW;
};

// Position, in granules, that granule g of plane row c is stored at: g ^ swz(c).
__device__ __forceinline__ int swz(int c) { return (2 * (c & 3) + (c >> 2)) & 7; }

// The bits of x without its sign, shifted up.  (A function: clang's
// __builtin_bit_cast of an element of a vector takes the first one.)
__device__ __forceinline__ uint32_t unsigned_bits(float x) { return __builtin_bit_cast(uint32_t, x) << 1; }

// An order (of unsigned values) that puts the operands that do not split last:
// from 2^-110 on by size, then infinities and NaN, then zero (SPLIT_ZERO),
// then the non-zero ones below 2^-110.
constexpr uint32_t SPLIT_MIN = 2 * 0x08800000u;   // unsigned_bits of 2^-110
constexpr uint32_t SPLIT_ZERO = 0u - SPLIT_MIN;
__device__ __forceinline__ uint32_t split_rank(float x) { return unsigned_bits(x) - SPLIT_MIN; }

// min(m, |a|, |b|), as one instruction (fminf would first quieten a and b)
__device__ __forceinline__ float min_abs(float m, float a, float b)
{
    asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a), "v"(b));
    return m;
}

// What follows the stages: whether the split can vouch for every sum of the
// workgroup's tile, and if not, the tile again on v_mfma_f32_32x32x2_f32, into
// the same accumulators.  `tiny`: this wave split a non-zero operand below
// 2^-110.
//
// Again, where a sum is infinite, NaN, or non-zero below 2^-96 (part products
// may be subnormal there).  An operand below 2^-110 is off by at most 2^-134
// in its three parts, a sum of R terms therefore by R * 2^-133 * top, top the
// largest operand: below 2^-26 of a sum that is at least R * 2^-107 * top.  So
// where an operand was tiny, A and Bc are searched for the largest, and the
// tile is formed again if a sum is below that.
// Measured on MI355X: the watch (12 instructions for 8 operands of A, 4 and a
// branch for 8 of Bc) and this cost 0-4 % (4096^3 at 16:32 337.6 -> 337.1 us,
// 8:32 194.4 -> 193.7, 4:32 123.2 -> 128.1, 600 x 4096 x 4096 at 16:32 90.5 ->
// 91.4; with the 12 for Bc, too, the last 94.8; with the 4 for A, too, 3 %
// more at 4:32 where half of A is zero; A's after its stores no difference).  4096^3 at 16:32 takes 435 with a few operands of 1e-39 in
// Bc, 1230 with a NaN in A, 1240 with every sum below 2^-96 (sums formed again
// one by one from memory: 1720 and 6080; the fp32 tiles: 550).
//
// Everything is formed anew from laundered copies of the kernel's arguments
// and ids, and the accumulators are gone through before it is, so that nothing
// of this takes a register of the kernel's loop.
template <class T, int KA, int KS>
__device__ __forceinline__ void split_check(f32x16 (&acc)[T::NRT], unsigned char *lds, uint32_t tiny)
{
    using S = SplitShape<T, KA, KS>;
    constexpr int BM = T::BM, BN = T::BN, WM = T::WM, NRT = T::NRT, QBMAX = T::QBMAX, NT = T::NT;
    typedef const __attribute__((address_space(4))) TiledArgs *args_ptr;
    args_ptr p = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    int pid = blockIdx.x, tid = threadIdx.x;
    asm volatile("" : "+s"(p), "+s"(pid), "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    uint32_t *word = reinterpret_cast<uint32_t *>(lds);
    auto any_wave = [&](uint32_t bits) {   // OR of a wave-uniform value over the workgroup
        if (lane == 0) word[wave] = bits;
        lds_sync();
        const uint32_t x = word[lane % T::NW];
        return (__any(x & 1) ? 1u : 0u) | (__any(x & 2) ? 2u : 0u);
    };
    // of this lane's sums the least non-zero one, without its sign, and the
    // largest ones of either sign: five instructions for two sums
    uint32_t lo = ~0u, minus = 0;
    int plus = 0;
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float x = acc[t][e];
            lo = min(lo, unsigned_bits(x) - 1u);
            plus = max(plus, __builtin_bit_cast(int, x));
            minus = max(minus, __builtin_bit_cast(uint32_t, x));
        }
    const bool unsure = lo < 2 * 0x0f800000u - 1u || plus >= 0x7f800000 || minus >= 0xff800000u;
    uint32_t again = any_wave((__any(unsure) ? 1u : 0u) | tiny << 1);
    if (again == 0 || NMSPMM_POISON_LDS) return;
    __builtin_amdgcn_sched_barrier(0);

    const int64_t m = p->m, n = p->n, k = p->k;
    const int N = p->N, M = p->M, V = p->V, RS = p->RS;
    int tm, tn, split;
    map_tile(pid, (int)gridDim.x, p->tiles_m, p->tiles_n, tm, tn, split);
    const int64_t row0 = (int64_t)tm * BM, col0 = p->col_begin + (int64_t)tn * BN;
    const int64_t w = (k / M) * N, q = n / V;
    const int sps = (p->stages + p->splits - 1) / p->splits;
    const int s_begin = split * sps, s_end = min(p->stages, s_begin + sps);
    const int wm = wave / QBMAX, wn = wave % QBMAX, r = lane & 31, half = lane >> 5;
    const int64_t col = col0 + wn * 32 + r;
    const float *A = p->A, *Bc = p->Bc;

    if (again == 2) {
        const int64_t u0 = (int64_t)s_begin * RS, u1 = min64((int64_t)s_end * RS, w);
        const int64_t k0 = (int64_t)s_begin * KA, k1 = min64((int64_t)s_end * KA, k);
        uint32_t least = ~0u;
#pragma unroll
        for (int t = 0; t < NRT; ++t) {
            asm volatile("" : "+v"(acc[t]));   // a new value: the bits formed above are not kept for this
#pragma unroll
            for (int e = 0; e < 16; ++e) least = min(least, unsigned_bits(acc[t][e]));
        }
        float top = 0.f;
        // 16-byte pieces of `rows` rows of `src`, several a thread at a time
        auto search = [&](const float *src, int64_t rows, int64_t cols, int64_t stride) {
            constexpr int BATCH = 8 / NRT;
            const uint32_t c4 = (uint32_t)(cols / 4);
            const int64_t pieces = rows * c4;
#pragma unroll 1
            for (int64_t f0 = tid; f0 < pieces; f0 += NT * BATCH) {
                f32x4 v[BATCH];   // (the last piece again in place of those past it)
#pragma unroll
                for (int y = 0; y < BATCH; ++y) {
                    const uint32_t f = (uint32_t)min64(f0 + NT * y, pieces - 1), row = f / c4;
                    v[y] = *reinterpret_cast<const f32x4 *>(src + row * stride + 4 * (f - row * c4));
                }
#pragma unroll
                for (int y = 0; y < BATCH; ++y)
#pragma unroll
                    for (int x = 0; x < 4; ++x) top = fmaxf(top, __builtin_fabsf(v[y][x]));
            }
        };
        search(A + row0 * k + k0, min64(BM, m - row0), k1 - k0, k);
        search(Bc + u0 * n + col0, u1 - u0, min64(BN, n - col0), n);
        lds_sync();
        if (tid == 0) word[0] = 0;
        lds_sync();
        atomicMax(word, __builtin_bit_cast(uint32_t, top));
        lds_sync();
        const float bound = (float)(u1 - u0) * 0x1p-107f * __builtin_bit_cast(float, word[0]);
        lds_sync();
        if (any_wave(__any(least < unsigned_bits(bound)) ? 1u : 0u) == 0) return;
    }

    // Stages of KA columns of A, as it is, k-major, in one LDS slot, and of the
    // offset bytes; a lane reads its rows of Bc from memory.
    float *A_s = reinterpret_cast<float *>(lds);
    int *X_s = reinterpret_cast<int *>(lds + S::A_BYTES);
    const int QB = BN >= V ? BN / V : 1, blk = (int)(min64(col, n - 1) / V - col0 / V);
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll 1
    for (int s = s_begin; s < s_end; ++s) {
        lds_sync();
#pragma unroll 1
        for (int i = tid; i < BM * KA / 4; i += NT) {
            const int row = i / (KA / 4), c = i % (KA / 4) * 4;
            const int64_t kc = (int64_t)s * KA + c;
            const f32x4 v = row0 + row < m && kc < k ? *reinterpret_cast<const f32x4 *>(A + (row0 + row) * k + kc)
                                                     : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < 4; ++x) A_s[(c + x) * BM + row] = v[x];
        }
        if (tid < S::X_ENTRIES) {
            const int64_t u = (int64_t)s * RS + tid / QBMAX, b = col0 / V + tid % QBMAX;
            X_s[tid] = tid / QBMAX < RS && u < w && tid % QBMAX < QB && b < q ? p->idx[u * q + b] : 0;
        }
        lds_sync();
        const int nu = (int)min64(RS, w - (int64_t)s * RS);
#pragma unroll 1
        for (int y = 0; y < nu; y += 2) {   // two compressed rows, one per half wave
            const int i = y + half, j = min(i, nu - 1);
            const int c = j / N * M + min(X_s[j * QBMAX + blk], M - 1);
            const float bv = i < nu && col < n ? Bc[((int64_t)s * RS + i) * n + col] : 0.f;
#pragma unroll
            for (int t = 0; t < NRT; ++t) {
                // (a row past the last one must not bring an infinity of A to a zero)
                const float av = i < nu ? A_s[c * BM + wm * WM + 32 * t + r] : 0.f;
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc[t], 0, 0, 0);
            }
        }
    }
}

template <class T, int KA, int KS>
__global__ __launch_bounds__(T::NT) void nm_tiled_split_kernel(TiledArgs p)
{
    using S = SplitShape<T, KA, KS>;
    constexpr int BM = T::BM, BN = T::BN, WM = T::WM, NRT = T::NRT, QBMAX = T::QBMAX, STRIDE = T::STRIDE;
    constexpr int TR = S::TR, TC = S::TC, CR = S::CR;
    typedef typename vec_of<TC>::type cvec;

    // (aligned to 256 bytes: the MFMA tiles of a wave are told apart by an XOR
    // of address bits 6 and 7)
    __shared__ __align__(256) unsigned char lds[S::LDS_BYTES];
    static_assert(STRIDE % 256 == 0 && NRT <= 4, "row pieces of 64 bytes");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn, split;
    map_tile(blockIdx.x, gridDim.x, p.tiles_m, p.tiles_n, tm, tn, split);
    const int64_t row0 = (int64_t)tm * BM, col0 = p.col_begin + (int64_t)tn * BN;
    const int64_t m = p.m, n = p.n, k = p.k;
    const int N = p.N, M = p.M, V = p.V, RS = p.RS;
    const int64_t w = (k / M) * N, q = n / V;
    const int64_t b_first = col0 / V;
    const int QB = BN >= V ? BN / V : 1;

    const int sps = (p.stages + p.splits - 1) / p.splits;
    const int s_begin = split * sps;
    const int s_end = min(p.stages, s_begin + sps);
    if (p.splits > 1 && s_begin >= s_end) return;  // uniform over the workgroup
    const int nst = max(s_end - s_begin, 0);

    const int wm = wave / QBMAX, wn = wave % QBMAX;
    const int blk = (int)((col0 + wn * 32) / V - b_first);
    const int r = lane & 31, half = lane >> 5;
    const bool col_ok = col0 + wn * 32 + r < n;

    // ---- A: global -> registers -> three bf16 planes in LDS, k-major ----
    const int chunk_r = (wave % (BM / CR)) * CR, chunk_c = wave / (BM / CR) * 32;
    const int ac = chunk_c + TC * (lane % (32 / TC)), ar = chunk_r + TR * (lane / (32 / TC));
    const int rows_valid = (int)min64(BM, m - row0);
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(p.A + row0 * k, (uint32_t)((int64_t)rows_valid * k * 4));
    const uint32_t a_off = (uint32_t)((ar * k + ac) * 4);
    cvec ra[TR];
    // `valid` false: the loads are still issued (so that every stage issues
    // the same memory instructions) but read zeros
    auto load_a = [&](int s, bool valid) {
        const uint32_t kc0 = (uint32_t)s * KA;   // k < 2^22: BM rows of A are under 2^31 bytes
        const uint32_t off = valid && kc0 + ac < (uint32_t)k ? a_off + kc0 * 4 : OOB;
#pragma unroll
        for (int t = 0; t < TR; ++t) {
            if constexpr (TC == 4)
                ra[t] = __builtin_bit_cast(cvec, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)off, (int)(t * k * 4), 0));
            else
                ra[t] = __builtin_bit_cast(cvec, __builtin_amdgcn_raw_buffer_load_b64(a_rsrc, (int)off, (int)(t * k * 4), 0));
        }
    };
    uint32_t tiny = 0;   // set once this wave has split a non-zero operand below 2^-110
    const int a_dst = ac * STRIDE + 2 * ar, a_swz = (2 * (ac & 3) + (ac >> 2)) << 5;
    auto store_a = [&](int slot) {
        unsigned char *As = lds + (S::TWO_A ? slot * S::A_BYTES : 0);
        // from copies the compiler takes for new values: the TC addresses are
        // then formed here and not kept in registers through the loop
        int d0 = a_dst, sw = a_swz;
        asm volatile("" : "+v"(d0), "+v"(sw));
        uint32_t rank = 0;
#pragma unroll
        for (int t = 0; t < TR; ++t)
#pragma unroll
            for (int c = 0; c < TC; ++c) rank = max(rank, split_rank(ra[t][c]));
        tiny |= __any(rank > SPLIT_ZERO) ? 1u : 0u;
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            // swz(ac + c): ac is a multiple of TC, so ac & 3 plus c stays below 4
            unsigned char *dst = As + c * STRIDE + (d0 ^ ((sw + 64 * c) & 0xe0));
            uint32_t part[3][TR / 2];
#pragma unroll
            for (int t = 0; t < TR; t += 2)
                split3(ra[t][c], ra[t + 1][c], part[0][t / 2], part[1][t / 2], part[2][t / 2]);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if constexpr (TR == 4)
                    *reinterpret_cast<u32x2 *>(dst + j * S::PLANE) = u32x2{part[j][0], part[j][1]};
                else
                    *reinterpret_cast<uint32_t *>(dst + j * S::PLANE) = part[j][0];
            }
        }
    };

    // (debug build) NaN in the places that this thread's next store_a will fill
    auto poison_a = [&](int slot) {
        cvec keep[TR];
        const float nan = __builtin_nanf("");
#pragma unroll
        for (int t = 0; t < TR; ++t) {
            keep[t] = ra[t];
#pragma unroll
            for (int c = 0; c < TC; ++c) ra[t][c] = nan;
        }
        store_a(slot);
#pragma unroll
        for (int t = 0; t < TR; ++t) ra[t] = keep[t];
        asm volatile("" ::: "memory");
    };

    // ---- D offsets: global -> register -> LDS, entry u * QBMAX + block: where
    // the plane row of the column of A that compressed row u gathers lies ----
    const int gps = KA / M;
    const int x_u = tid / QBMAX, x_b = tid % QBMAX;
    const bool x_ok = tid < S::X_ENTRIES && x_u < RS && x_b < QB && b_first + x_b < q;
    const uint32_t x_off = (uint32_t)(x_u * q + b_first + x_b);
    // padding rows (>= RS, zero in Bc) gather the last window's first column
    const int x_window = min(x_u / N, gps - 1) * M;
    int rx = 0;
    auto load_x = [&](int s, bool valid) {
        const int64_t u0 = (int64_t)s * RS;
        const int64_t rows_left = valid ? max64(0, min64(RS, w - u0)) : 0;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.idx + u0 * q, (uint32_t)(rows_left * q));
        rx = __builtin_amdgcn_raw_buffer_load_b8(rs, (int)(x_ok ? x_off : OOB), 0, 0);
    };
    auto x_area = [&](int slot) { return reinterpret_cast<int *>(lds + S::A_SLOTS * S::A_BYTES + slot * S::X_BYTES); };
    auto store_x = [&](int slot) {
        const int c = x_window + min(rx, M - 1);
        if (tid < S::X_ENTRIES) x_area(slot)[tid] = c * STRIDE + (swz(c) << 5);
    };

    // ---- Bc: 8 rows of this lane's column per K step, straight to registers ----
    float rb[8];
    const uint32_t b_off = col_ok ? (uint32_t)((8 * half * n + col0 + wn * 32 + r) * 4) : OOB;
    auto load_b = [&](int s, int ks, bool valid) {
        const int64_t u0 = (int64_t)s * RS;
        const int64_t rows_left = valid ? max64(0, min64(RS, w - u0)) : 0;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.Bc + u0 * n, (uint32_t)(rows_left * n * 4));
#pragma unroll
        for (int j = 0; j < 8; ++j)
            rb[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)b_off, (int)((16 * ks + j) * n * 4), 0));
    };

    // (1 in the places outside C, which split_check then takes for ordinary sums)
    f32x16 acc[NRT];
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            acc[t][e] = col_ok && wm * WM + 32 * t + 8 * (e / 4) + 4 * half + e % 4 < rows_valid ? 0.f : 1.f;

    // Lane l of a transposed read addresses piece l%4 (four output rows) of
    // granule l/16%2 of the plane row of compressed row 16*ks + 8*(l/32) +
    // l%16/4, the second read that of the row 4 further on.
    const int tu = 8 * half + ((lane >> 2) & 3);
    const int t_row = (wm * WM + 16 * ((lane >> 4) & 1)) * 2 + 8 * (lane & 3);

    if (nst > 0) {
        load_x(s_begin, true);
        load_a(s_begin, true);
        store_x(0);
        store_a(0);
        load_b(s_begin, 0, true);
        lds_sync();
    }
    for (int it = 0; it < nst; ++it) {
        const int cur = it & 1;
        const bool next = it + 1 < nst;
        if constexpr (NMSPMM_POISON_LDS) {
            // the other slots are free: in the places this thread's stores will
            // fill, NaN (A) and the place of the stage's last column (offsets)
            if (S::TWO_A) poison_a(cur ^ 1);
            if (tid < S::X_ENTRIES) x_area(cur ^ 1)[tid] = (KA - 1) * STRIDE + (swz(KA - 1) << 5);
        }
        const lds_u8 *As = (const lds_u8 *)(lds_void *)lds + (S::TWO_A ? cur * S::A_BYTES : 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const lds_u8 *at[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) at[x] = As + (x_area(cur)[(16 * ks + tu + 4 * x) * QBMAX + blk] ^ t_row);
            float least = 1.f;
#pragma unroll
            for (int j = 0; j < 8; j += 2) least = min_abs(least, rb[j], rb[j + 1]);
            if (__any(least < 0x1p-110f)) {   // zero (rare in weights) or tiny
                uint32_t rank = 0;
#pragma unroll
                for (int j = 0; j < 8; ++j) rank = max(rank, split_rank(rb[j]));
                tiny |= __any(rank > SPLIT_ZERO) ? 1u : 0u;
            }
            u32x4 bp[3];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t h, md, l;
                split3(rb[2 * j], rb[2 * j + 1], h, md, l);
                bp[0][j] = h;
                bp[1][j] = md;
                bp[2][j] = l;
            }
            if (ks == 0) {
                load_x(s_begin + it + 1, next);
                load_a(s_begin + it + 1, next);
            }
            if (ks + 1 < KS) load_b(s_begin + it, ks + 1, true);
            else load_b(s_begin + it + 1, 0, next);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NRT; ++t) {
                bf16x8 a[3];
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    s16x4 v[2];
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const lds_u8 *src = (const lds_u8 *)(uintptr_t)((uint32_t)(uintptr_t)at[x] ^ (uint32_t)(t << 6)) + j * S::PLANE;
                        v[x] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)src);
                    }
                    a[j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
                }
                // smallest products first
                const auto mma = [&](int i, int j) {
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], __builtin_bit_cast(bf16x8, bp[j]), acc[t], 0, 0, 0);
                };
                mma(1, 1);
                mma(0, 2);
                mma(2, 0);
                mma(0, 1);
                mma(1, 0);
                mma(0, 0);
            }
        }
        store_x(cur ^ 1);
        // one A slot: every wave must be done reading it
        if constexpr (!S::TWO_A) lds_sync();
        if constexpr (NMSPMM_POISON_LDS && !S::TWO_A) poison_a(0);
        store_a(cur ^ 1);
        lds_sync();
    }

    // ---- the sums the split cannot vouch for, then the epilogue ----
    // (the lds areas are free: the last stage ended with a barrier)
    split_check<T, KA, KS>(acc, lds, tiny);
    // element e of MFMA tile t is row 32*t + 8*(e/4) + 4*half + e%4 of the
    // wave's rows, column `col`.  The lane's place again, from a copy of the
    // lane id the compiler takes for another value: what follows is then not
    // kept in registers through the loop
    int elane = lane;
    asm volatile("" : "+v"(elane));
    const int64_t col = col0 + wn * 32 + (elane & 31);
    const int64_t wrow = row0 + wm * WM + 4 * (elane >> 5);
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t row = wrow + 32 * t + 8 * (e / 4) + e % 4;
            if (row >= m || col >= n) continue;
            float *dst = p.C + row * n + col;
            if (p.splits == 1) *dst = apply_epilogue(p.epi, acc[t][e], col);
            else unsafeAtomicAdd(dst, acc[t][e]);
        }
}

// Host-side launcher of one instantiation.
template <class T, int KA, int KS>
hipError_t launch_split(const TiledArgs &a, hipStream_t stream)
{
    if constexpr (!SplitShape<T, KA, KS>::FITS) {
        return hipErrorInvalidConfiguration;
    } else {
        const unsigned grid = (unsigned)a.tiles_m * (unsigned)a.tiles_n * (unsigned)a.splits;
        hipLaunchKernelGGL((nm_tiled_split_kernel<T, KA, KS>), dim3(grid), dim3(T::NT), 0, stream, a);
        return hipGetLastError();
    }
}

// The stage depths instantiated: (KA, KS); a stage of NQ quads takes
// ceil(NQ/4) K steps.
#define NMSPMM_SPLIT_STAGES(X) X(32, 1) X(32, 2) X(64, 1) X(64, 2) X(128, 1) X(128, 3)

template <class T>
hipError_t launch_split_any(int KA, int NQ, const TiledArgs &a, hipStream_t stream)
{
#define NMSPMM_CASE(ka, ks) \
    if (KA == ka && (NQ + 3) / 4 == ks) return launch_split<T, ka, ks>(a, stream);
    NMSPMM_SPLIT_STAGES(NMSPMM_CASE)
#undef NMSPMM_CASE
    return hipErrorInvalidValue;
}

template <class T>
constexpr bool split_fits(int BV, int KA, int NQ)
{
#define NMSPMM_CASE(ka, ks) || (KA == ka && (NQ + 3) / 4 == ks && SplitShape<T, ka, ks>::FITS)
    return BV == 1 && (false NMSPMM_SPLIT_STAGES(NMSPMM_CASE));
#undef NMSPMM_CASE
}

}  // namespace nmspmm

#endif
