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
// no such split (its further parts are NaN), and a sum below 2^-96 may come
// from operands too small for one: a wave whose sums are not all zero or of
// ordinary size forms those sums again in plain fp32 from A and Bc
// (resum_terms), so that such inputs give what fp32 arithmetic gives.
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
//   X_s : the stage's offset bytes, buffer->LDS DMA, a zero-extended dword
//         each.
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

// A sum the split cannot vouch for: infinite, NaN, or non-zero below 2^-96.
__device__ __forceinline__ bool split_unsure(float x)
{
    const float a = __builtin_fabsf(x);
    return !(a <= 3.4028234663852886e38f) || (a < 0x1p-96f && a != 0.f);
}

// The 16 sums of one 32 x 32 MFMA tile of this lane (rows row0 + 8*(e/4) + e%4,
// one column) over compressed rows [u0, u1), in plain fp32 in row order.
__device__ inline void resum_terms(float (&sum)[16], const TiledArgs &p, int64_t row0, int64_t col, int64_t u0,
                                   int64_t u1)
{
    const int64_t q = p.n / p.V, b = col / p.V;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum[e] = 0.f;
    for (int64_t u = u0; u < u1; ++u) {
        const int64_t c = u / p.N * p.M + min((int)p.idx[u * q + b], p.M - 1);
        const float bv = p.Bc[u * p.n + col];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t row = min64(row0 + 8 * (e / 4) + e % 4, p.m - 1);
            sum[e] = fmaf(p.A[row * p.k + c], bv, sum[e]);
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

    __shared__ __align__(16) unsigned char lds[S::LDS_BYTES];
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
    const int a_dst = ac * STRIDE + 2 * ar, a_swz = (2 * (ac & 3) + (ac >> 2)) << 5;
    auto store_a = [&](int slot) {
        unsigned char *As = lds + (S::TWO_A ? slot * S::A_BYTES : 0);
        // from copies the compiler takes for new values: the TC addresses are
        // then formed here and not kept in registers through the loop
        int d0 = a_dst, sw = a_swz;
        asm volatile("" : "+v"(d0), "+v"(sw));
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

    // ---- D offsets: global -> register -> LDS, entry u * QBMAX + block ----
    const int x_u = tid / QBMAX, x_b = tid % QBMAX;
    const bool x_ok = tid < S::X_ENTRIES && x_u < RS && x_b < QB && b_first + x_b < q;
    const uint32_t x_off = (uint32_t)(x_u * q + b_first + x_b);
    int rx = 0;
    auto load_x = [&](int s, bool valid) {
        const int64_t u0 = (int64_t)s * RS;
        const int64_t rows_left = valid ? max64(0, min64(RS, w - u0)) : 0;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.idx + u0 * q, (uint32_t)(rows_left * q));
        rx = __builtin_amdgcn_raw_buffer_load_b8(rs, (int)(x_ok ? x_off : OOB), 0, 0);
    };
    auto x_area = [&](int slot) { return reinterpret_cast<int *>(lds + S::A_SLOTS * S::A_BYTES + slot * S::X_BYTES); };
    auto store_x = [&](int slot) {
        if (tid < S::X_ENTRIES) x_area(slot)[tid] = rx;
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

    f32x16 acc[NRT];
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

    // Lane l of a transposed read addresses piece l%4 (four output rows) of
    // granule l/16%2 of the plane row of compressed row 16*ks + 8*(l/32) +
    // l%16/4, the second read that of the row 4 further on.
    const int gps = KA / M, tu = 8 * half + ((lane >> 2) & 3);
    const int t_row = (wm * WM + 16 * ((lane >> 4) & 1)) * 2 + 8 * (lane & 3);
    int window[KS][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        // padding rows (>= RS, zero in Bc) address the last window's columns
        for (int x = 0; x < 2; ++x) window[ks][x] = min((16 * ks + tu + 4 * x) / N, gps - 1) * M;

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
        if constexpr (NMSPMM_POISON_LDS && S::TWO_A) {
            // the other A slot is free: NaN in the places this thread's store
            // will fill
            const float nan = __builtin_nanf("");
#pragma unroll
            for (int t = 0; t < TR; ++t)
#pragma unroll
                for (int c = 0; c < TC; ++c) ra[t][c] = nan;
            store_a(cur ^ 1);
        }
        const lds_u8 *As = (const lds_u8 *)(lds_void *)lds + (S::TWO_A ? cur * S::A_BYTES : 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const lds_u8 *at[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int d = x_area(cur)[(16 * ks + tu + 4 * x) * QBMAX + blk];
                const int c = window[ks][x] + min(d, M - 1);
                at[x] = As + c * STRIDE + (t_row ^ (swz(c) << 5));
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
        // one A slot: every wave must be done reading it
        if constexpr (!S::TWO_A) lds_sync();
        store_x(cur ^ 1);
        store_a(cur ^ 1);
        lds_sync();
    }

    // ---- epilogue: element e of MFMA tile t is row 32*t + 8*(e/4) + 4*half +
    // e%4 of the wave's rows, column `col` ----
    // the lane's place again, from a copy of the lane id the compiler takes for
    // another value: what follows is then not kept in registers through the loop
    int elane = lane;
    asm volatile("" : "+v"(elane));
    const int64_t col = col0 + wn * 32 + (elane & 31);
    const int64_t wrow = row0 + wm * WM + 4 * (elane >> 5);
    auto put = [&](int64_t row, float v) {
        if (row >= m || col >= n) return;
        float *dst = p.C + row * n + col;
        if (p.splits == 1) *dst = apply_epilogue(p.epi, v, col);
        else unsafeAtomicAdd(dst, v);
    };
    uint32_t unsure[NRT];
#pragma unroll
    for (int t = 0; t < NRT; ++t) {
        unsure[t] = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (!NMSPMM_POISON_LDS && split_unsure(acc[t][e])) unsure[t] |= 1u << e;
            else put(wrow + 32 * t + 8 * (e / 4) + e % 4, acc[t][e]);
        }
    }
#pragma unroll
    for (int t = 0; t < NRT; ++t) {
        if (!__any(unsure[t] != 0 && col < n)) continue;
        float sum[16];
        const int64_t u0 = min64((int64_t)s_begin * RS, w), u1 = min64((int64_t)s_end * RS, w);
        resum_terms(sum, p, wrow + 32 * t, min64(col, n - 1), u0, u1);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (unsure[t] >> e & 1) put(wrow + 32 * t + 8 * (e / 4) + e % 4, sum[e]);
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
