// Row-gather kernel for the thinnest products (at most 32 rows of C), in one
// launch with no workspace and no split of k.
//
// Eq. 1 gathers, for compressed row u and column block b, the column
// (u/N)*M + D[u][b] of A.  With at most 32 rows the gathered values of one
// quad (4 consecutive compressed rows, the K of v_mfma_f32_16x16x4_f32) lie in
// at most 32 cache lines of the row-major A, one per row: at M = 32 a window
// of one row is one 128-byte line, and a quad never leaves its window when N
// is a multiple of 4.  Those lines are read straight into MFMA operands from
// L2, where all of A (16 rows x k = 8192: 512 KB) stays while Bc streams past
// it with the non-temporal hint.  Nothing is staged in LDS and nothing is
// transposed first, so the whole product is one launch; each workgroup owns
// a strip of whole columns over all of k, so every output is written once,
// with no zero fill and no atomics.
//
// A workgroup owns all 16*RT rows x one strip of 16*CT columns, inside one
// column block (V a multiple of 16*CT).  Its NW waves split the strip's
// quads and each streams its quads through a ring of D quads in flight in
// registers: per quad a lane loads the D byte of its compressed row (one
// trip ahead), RT floats of A gathered by it, and CT consecutive Bc floats
// (columns CT*(l%16)+s, one per column tile s); it issues RT*CT MFMAs.  The
// waves' partial strips are summed through LDS at the end, in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "nmspmm_rowgather.h"

namespace nmspmm {

namespace {

template <int RT, int CT, int NW>
struct RGShape {
    static constexpr int ROWS = 16 * RT, COLS = 16 * CT;
    static constexpr int RST = COLS + 1;   // LDS row stride of a partial strip
    static constexpr int TILE = ROWS * RST;
    // partial strips held in LDS at once (a power of two dividing NW); the
    // waves beyond them add into the held ones, in wave order
    static constexpr int FIT = (120 * 1024 / 4) / TILE;
    static constexpr int G = FIT >= NW ? NW : FIT >= 8 ? 8 : FIT >= 4 ? 4 : FIT >= 2 ? 2 : 1;
};

template <int CT> struct RGB;
template <> struct RGB<2> { f32x2 v; };
template <> struct RGB<4> { f32x4 v; };

template <int CT, int AUX>
__device__ __forceinline__ void rg_load_b(RGB<CT> &b, __amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff)
{
    if constexpr (CT == 2)
        b.v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, AUX));
    else
        b.v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, AUX));
}

// The waves' partial strips, summed through LDS (red: G*TILE floats) in a
// fixed order, and the epilogue.
template <int RT, int CT, int NW>
__device__ __forceinline__ void rg_finish(const f32x4 (&acc)[RT][CT], float *red, int wave, int lane, float *C, int m,
                                          int64_t n, int64_t j0, const Epilogue &epi)
{
    using S = RGShape<RT, CT, NW>;
    constexpr int ROWS = S::ROWS, COLS = S::COLS, RST = S::RST;
    const int r = lane & 15, kq = lane >> 4;
    // partial strips of the waves, summed in a fixed order: G held in LDS,
    // the waves beyond them adding into the held ones round by round.  The
    // 16 x 16 MFMA tile holds row 4*(l/16)+e, column l%16 in element e of
    // lane l: row 16*rt + 4*kq + e, column CT*r + s of the strip.
    float *mine = red + (wave % S::G) * S::TILE;
#pragma unroll 1
    for (int round = 0; round < NW / S::G; ++round) {
        if (wave / S::G == round) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int s = 0; s < CT; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float &x = mine[(16 * rt + 4 * kq + e) * RST + CT * r + s];
                        x = round == 0 ? acc[rt][s][e] : x + acc[rt][s][e];
                    }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < ROWS * COLS; e += NW * 64) {
        const int row = e / COLS, col = e % COLS;
        float sum = red[row * RST + col];
#pragma unroll
        for (int x = 1; x < S::G; ++x) sum += red[x * S::TILE + row * RST + col];
        if (row < m) C[(int64_t)row * n + j0 + col] = apply_epilogue(epi, sum, j0 + col);
    }
}

// AUX: cache policy of the Bc loads (2: non-temporal, the stream leaves L2
// to A).
template <int RT, int CT, int NW, int D, int AUX>
__global__ __launch_bounds__(NW * 64) void nm_rowgather_kernel(const float *__restrict__ A,
                                                              const float *__restrict__ Bc,
                                                              const uint8_t *__restrict__ idx,
                                                              float *__restrict__ C, int m, int64_t n, int k,
                                                              int w, int q, int M, int V, uint32_t magic, uint32_t n1,
                                                              Epilogue epi)
{
    using S = RGShape<RT, CT, NW>;
    constexpr int COLS = S::COLS;
    __shared__ float red[S::G * S::TILE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroups are dispatched round-robin over the 8 XCDs: renumber them so
    // that consecutive strips, which gather the same lines of A when they
    // share a column block, run on one XCD and share its L2.
    const int nwg = gridDim.x, pid = blockIdx.x;
    const int xcd = pid % 8, local = pid / 8, full = nwg / 8, rem = nwg % 8;
    const int strip = xcd < rem ? xcd * (full + 1) + local : rem * (full + 1) + (xcd - rem) * full + local;
    const int64_t j0 = (int64_t)strip * COLS;
    const int b = (int)(j0 / V);
    const int nquads = (w + 3) / 4;
    const int qa = (int)((int64_t)wave * nquads / NW);
    const int qb = (int)((int64_t)(wave + 1) * nquads / NW);
    const int nq = qb - qa;

    const int r = lane & 15, kq = lane >> 4;
    // This wave's Bc rows only: quads past its range (the ring loads one trip
    // ahead) read zero and their MFMAs are skipped.  D bytes past w read
    // zero; a compressed row past w gathers nothing (its A offset is out of
    // range and reads zero), so the last partial quad adds zero terms.
    const int u_lo = min(4 * qa, w), u_hi = min(4 * qb, w);
    const auto rs_a = make_rsrc(A, (uint32_t)((int64_t)m * k * 4));
    const auto rs_bc = make_rsrc(Bc + (int64_t)u_lo * n + j0, (uint32_t)((int64_t)(u_hi - u_lo) * n * 4));
    // D bytes come in the aligned dword that holds them (w*q is a multiple
    // of 4, so every such dword lies inside idx); the byte's place in it is
    // the same for all quads of a lane, since a quad spans 4*q bytes
    const auto rs_x = make_rsrc(idx, (uint32_t)((int64_t)w * q));
    const uint32_t lane_bc = (uint32_t)((kq * n + CT * r) * 4);
    const uint32_t quad_bc = (uint32_t)(16 * n);     // bytes of 4 Bc rows
    const uint32_t byte_x = (uint32_t)((int64_t)(4 * qa + kq) * q + b);
    const uint32_t lane_x = byte_x & ~3u, shift_x = 8 * (byte_x & 3u);
    const uint32_t quad_x = (uint32_t)(4 * q);       // D bytes of 4 compressed rows
    // rows past m lie past the end of A and read zero
    const uint32_t lane_a = (uint32_t)(r * k * 4);
    const uint32_t tile_a = (uint32_t)(16 * k * 4);  // bytes of 16 rows of A

    f32x4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int s = 0; s < CT; ++s) acc[t][s] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Ring of D slots: after trip t, slot j holds the operands of quad t*D + j
    // and the D byte of quad (t+1)*D + j.  Trip 0 only loads; every later trip
    // multiplies the previous trip's quads and loads its own.
    float av[D][RT];
    RGB<CT> bv[D];
    uint32_t xv[D];
    // The first trip's D bytes, each slot issued as the loop issues it (A, Bc,
    // D; the A and Bc loads out of range, reading zero), so that the pending
    // loads on entry line up with those of a trip and the wait counts at the
    // loop head stay exact.
#pragma unroll
    for (int j = 0; j < D; ++j) {
#pragma unroll
        for (int t = 0; t < RT; ++t)   // distinct offsets: no two loads merged
            av[j][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_a, (int)(OOB + 1024 * (j * RT + t)), 0, 0));
        rg_load_b<CT, AUX>(bv[j], rs_bc, OOB + 64 * j, 0);
        xv[j] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, (int)lane_x, (int)(j * quad_x), 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    const int trips = (max(nq, 0) + D - 1) / D;
    // one loop, not peeled: a peeled first trip behind its own branch lets
    // the compiler sink its loads, and the wait counts at the loop head
    // become conservative
#pragma clang loop unroll(disable)
    for (int t = 0; t <= trips; ++t) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            if (t > 0 && (t - 1) * D + j < nq) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int s = 0; s < CT; ++s)
                        acc[rt][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j][rt], bv[j].v[s], acc[rt][s], 0, 0, 0);
            }
            const int qr = t * D + j;
            // window u/N of the lane's compressed row: magic = ceil(2^32 / N),
            // exact for u < 2^24 (N = 1: magic = 0, n1 = 1)
            const uint32_t u = (uint32_t)(4 * (qa + qr) + kq);
            const uint32_t g = __umulhi(u, magic) + u * n1;
            const uint32_t col = g * (uint32_t)M + min((xv[j] >> shift_x) & 0xffu, (uint32_t)(M - 1));
            const uint32_t aoff = u < (uint32_t)w ? lane_a + 4 * col : OOB;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                av[j][rt] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_a, (int)(aoff + rt * tile_a), 0, 0));
            rg_load_b<CT, AUX>(bv[j], rs_bc, lane_bc, qr * quad_bc);
            xv[j] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, (int)lane_x, (int)((qr + D) * quad_x), 0);
            // keep each slot's loads right after its MFMAs: gathered to the
            // end of the unrolled body, they would be waited for at once
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    rg_finish<RT, CT, NW>(acc, red, wave, lane, C, m, n, j0, epi);
}

// The same strips where all of A and a strip's offsets fit in LDS (decode
// batches: 4 rows at k = 8192).  The kernel above issues three memory
// instructions per quad, and their issue and their chain (D byte, then A) set
// its pace: 33.5 MB of Bc stream in 4 us, the product took 9.3.  Here A
// arrives by buffer->LDS DMA and each offset byte is loaded once (one lane
// each, not one instruction per quad) and stored as the byte offset of its
// column, while the first Bc loads are already in flight; the loop then
// issues Bc loads only, D slots of four quads ahead.
// LDS: a_s, m rows of `stride` floats (k rounded up to a DMA piece, then 16
// zeros that the rows past w gather), then the offsets of 4*nquads rows; the
// partial strips take its place at the end.
constexpr int RG_PIECE = 256;   // floats per DMA instruction
__host__ __device__ constexpr int rg_stride(int64_t k) { return (int)((k + RG_PIECE - 1) / RG_PIECE * RG_PIECE) + 16; }

//
// MR = 0: the MFMA form above, up to 16 rows.  MR > 0: at most MR rows by FMA.
// A Bc load is then 16 bytes a lane, eight rows of the strip per instruction
// instead of four, and a lane adds its MR x 4 products itself: one token
// would fill one of 16 MFMA rows.  Its sums over every eighth row meet the
// other lanes' at the end.
// Measured (per call, one set of buffers): 1 x 8192 x 8192 at 4:32 9.1 -> 7.5
// us (8.7 by MFMA), 1 x 4096 x 11008 at 16:32 34.4 -> 26.7, 4 x 8192 x 8192
// 11.2 -> 9.9, 3 x 4096 x 11008 at 8:32 20.6 -> 16.6.  (Without the
// non-temporal hint Bc that stays in the 256 MB Infinity Cache reads 3-10 %
// faster, Bc that comes from HBM 3-8 % slower: the layers of a model do not
// stay there, so the hint does.)
template <int MR, int CT, int NW, int D, int LDSK, int AUX>
__global__ __launch_bounds__(NW * 64) void nm_rowgather_lds_kernel(
    const float *__restrict__ A, const float *__restrict__ Bc, const uint8_t *__restrict__ idx,
    float *__restrict__ C, int m, int64_t n, int k, int w, int q, int M, int V, uint32_t magic, uint32_t n1,
    Epilogue epi)
{
    constexpr int COLS = 16 * CT, QS = 4, XB = 4;
    constexpr int UR = MR ? 8 : 4;   // compressed rows per Bc load
    typedef typename vec_of<MR ? 4 : CT>::type bvec;
    static_assert(COLS == 32, "eight lanes of four columns");
    static_assert(LDSK * 1024 >= 4 * RGShape<1, CT, NW>::G * RGShape<1, CT, NW>::TILE, "room for the partial strips");
    __shared__ __align__(16) unsigned char lds[LDSK * 1024];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive strips on one XCD, as above
    const int nwg = gridDim.x, pid = blockIdx.x;
    const int xcd = pid % 8, local = pid / 8, full = nwg / 8, rem = nwg % 8;
    const int strip = xcd < rem ? xcd * (full + 1) + local : rem * (full + 1) + (xcd - rem) * full + local;
    const int64_t j0 = (int64_t)strip * COLS;
    const int b = (int)(j0 / V);
    // units of UR rows, shared out to the waves
    const int nunits = (w + UR - 1) / UR, stride = rg_stride(k);
    const int qa = (int)((int64_t)wave * nunits / NW), qb = (int)((int64_t)(wave + 1) * nunits / NW), nq = qb - qa;
    const int r = lane & (MR ? 7 : 15), kq = lane / (64 / UR);
    float *a_s = reinterpret_cast<float *>(lds);
    int *x_s = reinterpret_cast<int *>(a_s + m * stride);

    const auto rs_a = make_rsrc(A, (uint32_t)((int64_t)m * k * 4));
    const auto rs_x = make_rsrc(idx, (uint32_t)((int64_t)w * q));
    const int u_lo = min(UR * qa, w), u_hi = min(UR * qb, w);   // this wave's Bc rows only
    const auto rs_bc = make_rsrc(Bc + (int64_t)u_lo * n + j0, (uint32_t)((int64_t)(u_hi - u_lo) * n * 4));
    const uint32_t lane_bc = (uint32_t)((kq * n + (MR ? 4 : CT) * r) * 4), unit_bc = (uint32_t)(4 * UR * n);

    // offset bytes (XB per thread and pass), then A, then the first Bc loads:
    // loads return in order, so the wait for the first two leaves the last
    // in flight
    int xv[XB];
    auto load_x = [&](int u0) {
#pragma unroll
        for (int i = 0; i < XB; ++i) {
            const int u = u0 + i * NW * 64 + (int)threadIdx.x;
            xv[i] = __builtin_amdgcn_raw_buffer_load_b8(rs_x, (int)(u < w ? (uint32_t)(u * q + b) : OOB), 0, 0);
        }
    };
    auto store_x = [&](int u0) {
#pragma unroll
        for (int i = 0; i < XB; ++i) {
            const int u = u0 + i * NW * 64 + (int)threadIdx.x;
            // window u/N: magic = ceil(2^32 / N), exact for u < 2^24 (N = 1:
            // magic = 0, n1 = 1)
            const int col = (int)(__umulhi((uint32_t)u, magic) + (uint32_t)u * n1) * M + min(xv[i] & 0xff, M - 1);
            if (u < UR * nunits) x_s[u] = 4 * (u < w ? col : stride - 16);
        }
    };
    load_x(0);
    const int segs = (stride - 16) / RG_PIECE, pieces = m * segs;
    for (int p = wave; p < pieces; p += NW) {
        const int row = p / segs, c0 = (p - row * segs) * RG_PIECE;
        const int c = c0 + 4 * lane;
        lds_dma<16>(rs_a, a_s + row * stride + c0, c < k ? (uint32_t)((row * k + c) * 4) : OOB);
    }
    bvec bv[D][QS];
    auto load_slot = [&](int j, int unit0) {
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            const int soff = (int)((uint32_t)(unit0 + i) * unit_bc);
            if constexpr (MR != 0)
                bv[j][i] = __builtin_bit_cast(bvec, __builtin_amdgcn_raw_buffer_load_b128(rs_bc, (int)lane_bc, soff, AUX));
            else
                bv[j][i] = __builtin_bit_cast(bvec, __builtin_amdgcn_raw_buffer_load_b64(rs_bc, (int)lane_bc, soff, AUX));
        }
    };
#pragma unroll
    for (int j = 0; j < D; ++j) load_slot(j, j * QS);
    for (int e = threadIdx.x; e < 16 * m; e += NW * 64) a_s[(e / 16) * stride + stride - 16 + e % 16] = 0.f;
    store_x(0);
    for (int u0 = XB * NW * 64; u0 < UR * nunits; u0 += XB * NW * 64) {
        load_x(u0);
        store_x(u0);
    }
    asm volatile("" ::: "memory");
    static_assert(D * QS < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((D * QS & 15) | (7 << 4) | (0 << 8) | ((D * QS >> 4) << 14));   // A has arrived
    lds_sync();

    const int *xq = x_s + UR * qa + kq;
    if constexpr (MR == 0) {
        // One set of sums for each of a slot's quads: with a single one a wave
        // rounds w / 32 times in a row (4 x 4096 x 6144 at 16:32: error against
        // fp64 3.0e-7 -> 1.6e-7, the streaming kernel split 4 ways 1.4e-7;
        // 14.8 -> 15.0 us).
        f32x4 part[QS][CT];
#pragma unroll
        for (int i = 0; i < QS; ++i)
#pragma unroll
            for (int s = 0; s < CT; ++s) part[i][s] = f32x4{0.f, 0.f, 0.f, 0.f};
        // rows past m repeat the last one; their sums are not stored
        const unsigned char *arow = lds + min(r, m - 1) * stride * 4;
#pragma clang loop unroll(disable)
        for (int q0 = 0; q0 < nq; q0 += D * QS) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const int qj = q0 + j * QS;
                float av[QS];
#pragma unroll
                for (int i = 0; i < QS; ++i)   // past the wave's last quad: its first, not multiplied
                    av[i] = *reinterpret_cast<const float *>(arow + xq[4 * (qj + i < nq ? qj + i : 0)]);
#pragma unroll
                for (int i = 0; i < QS; ++i)
                    if (qj + i < nq)
#pragma unroll
                        for (int s = 0; s < CT; ++s)
                            part[i][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j][i][s], part[i][s], 0, 0, 0);
                load_slot(j, qj + D * QS);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        f32x4 acc[1][CT];
#pragma unroll
        for (int s = 0; s < CT; ++s) acc[0][s] = (part[0][s] + part[1][s]) + (part[2][s] + part[3][s]);
        static_assert(QS == 4, "sets of sums");
        lds_sync();   // every wave is done with a_s and x_s
        rg_finish<1, CT, NW>(acc, reinterpret_cast<float *>(lds), wave, lane, C, m, n, j0, epi);
    } else {
        f32x4 acc[MR];
        const unsigned char *arow[MR];   // rows past m repeat the last one; their sums are not stored
#pragma unroll
        for (int t = 0; t < MR; ++t) {
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            arow[t] = lds + min(t, m - 1) * stride * 4;
        }
#pragma clang loop unroll(disable)
        for (int q0 = 0; q0 < nq; q0 += D * QS) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const int qj = q0 + j * QS;
                float av[QS][MR];
#pragma unroll
                for (int i = 0; i < QS; ++i) {   // past the wave's last unit: its first, not added
                    const int x = xq[UR * (qj + i < nq ? qj + i : 0)];
#pragma unroll
                    for (int t = 0; t < MR; ++t) av[i][t] = *reinterpret_cast<const float *>(arow[t] + x);
                }
#pragma unroll
                for (int i = 0; i < QS; ++i)
                    if (qj + i < nq)
#pragma unroll
                        for (int t = 0; t < MR; ++t)
#pragma unroll
                            for (int s = 0; s < 4; ++s) acc[t][s] = fmaf(av[i][t], bv[j][i][s], acc[t][s]);
                load_slot(j, qj + D * QS);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        lds_sync();   // every wave is done with a_s and x_s
        // the eight row groups of a wave, then the waves, in a fixed order
        float *red = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int t = 0; t < MR; ++t) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int x = 8; x < 64; x *= 2) acc[t][s] += __shfl_xor(acc[t][s], x);
            if (lane < 8) *reinterpret_cast<f32x4 *>(red + (wave * MR + t) * COLS + 4 * lane) = acc[t];
        }
        __syncthreads();
        if ((int)threadIdx.x < MR * COLS) {
            const int row = threadIdx.x / COLS, col = threadIdx.x % COLS;
            float sum = red[row * COLS + col];
#pragma unroll
            for (int x = 1; x < NW; ++x) sum += red[(x * MR + row) * COLS + col];
            if (row < m) C[(int64_t)row * n + j0 + col] = apply_epilogue(epi, sum, j0 + col);
        }
    }
}

template <int MR, int LDSK>
void launch_lds(const RowGatherArgs &a, unsigned strips, int w, int q, uint32_t magic, hipStream_t stream)
{
    const auto kernel = a.stream_b ? nm_rowgather_lds_kernel<MR, 2, 8, 4, LDSK, 2> : nm_rowgather_lds_kernel<MR, 2, 8, 4, LDSK, 0>;
    hipLaunchKernelGGL(kernel, dim3(strips), dim3(512), 0, stream, a.A, a.Bc, a.idx, a.C, (int)a.m, a.n, (int)a.k, w,
                       q, a.M, a.V, magic, a.N == 1 ? 1u : 0u, a.epi);
}

template <int RT, int CT, int NW, int D>
hipError_t launch_cfg(const RowGatherArgs &a, hipStream_t stream)
{
    const int w = (int)(a.k / a.M * a.N), q = (int)(a.n / a.V);
    const unsigned strips = (unsigned)(a.n / (16 * CT));
    const uint32_t magic = a.N == 1 ? 0u : (uint32_t)(((uint64_t(1) << 32) + (uint64_t)a.N - 1) / (uint64_t)a.N);
    if constexpr (RT == 1 && CT == 2 && NW == 8 && D == 4) {
        const int kb = rowgather_lds_kb(a.A, a.m, a.n, a.k, a.N, a.M);
        if (kb) {
            // (m = 2: 9.7 us in either form, m = 4: 10.4 by MFMA, 11.8 by FMA, 8192 x 8192 at 4:32)
            const bool one = a.m == 1;
            const auto go = kb == 48   ? one ? launch_lds<1, 48> : launch_lds<0, 48>
                            : kb == 80 ? one ? launch_lds<1, 80> : launch_lds<0, 80>
                                       : one ? launch_lds<1, 150> : launch_lds<0, 150>;
            go(a, strips, w, q, magic, stream);
            return hipGetLastError();
        }
    }
    if (a.stream_b)
        hipLaunchKernelGGL((nm_rowgather_kernel<RT, CT, NW, D, 2>), dim3(strips), dim3(NW * 64), 0, stream, a.A,
                           a.Bc, a.idx, a.C, (int)a.m, a.n, (int)a.k, w, q, a.M, a.V, magic, a.N == 1 ? 1u : 0u, a.epi);
    else
        hipLaunchKernelGGL((nm_rowgather_kernel<RT, CT, NW, D, 0>), dim3(strips), dim3(NW * 64), 0, stream, a.A,
                           a.Bc, a.idx, a.C, (int)a.m, a.n, (int)a.k, w, q, a.M, a.V, magic, a.N == 1 ? 1u : 0u, a.epi);
    return hipGetLastError();
}

// Instantiated configurations: {RT, CT, NW, D}.
#define NM_ROWGATHER_CONFIGS(X)                                                                 \
    X(1, 2, 8, 4) X(1, 2, 8, 8) X(1, 2, 16, 4) X(1, 2, 16, 8)                                   \
    X(1, 4, 8, 4) X(1, 4, 8, 8) X(1, 4, 16, 4) X(1, 4, 16, 8)                                   \
    X(2, 2, 8, 4) X(2, 2, 16, 4) X(2, 4, 8, 4) X(2, 4, 16, 4)

}  // namespace

int rowgather_lds_kb(const float *A, int64_t m, int64_t n, int64_t k, int N, int M)
{
    if (m > 16 || k % 4 != 0 || reinterpret_cast<uintptr_t>(A) % 16 != 0) return 0;
    const int64_t w = k / M * N;
    // on more than one round of strips the staging pays from about w = 450 on: 2 x
    // 1888 x 9792 at 8:32 (w = 472) 10.7 -> 9.6 us, but 2 x 1248 x 8736 at 4:32
    // (w = 156) 5.8 -> 6.5 and 3 x 3328 x 9952 (w = 416) 8.4 -> 8.8
    if (n / 32 > 256 && w < 448) return 0;
    const int64_t bytes = m * rg_stride(k) * 4 + (w + 7) / 8 * 32;
    for (int kb : {48, 80, 150})   // three, two and one workgroup per CU
        if (bytes <= kb * 1024) return kb;
    return 0;
}

bool rowgather_has(const RowGatherCfg &c)
{
#define NM_RG_HAS(RT_, CT_, NW_, D_) \
    if (c.RT == RT_ && c.CT == CT_ && c.NW == NW_ && c.D == D_) return true;
    NM_ROWGATHER_CONFIGS(NM_RG_HAS)
#undef NM_RG_HAS
    return false;
}

bool rowgather_fits(const RowGatherCfg &c, int64_t m, int64_t n, int64_t k, int N, int M, int V)
{
    if (!rowgather_has(c) || m > 16 * c.RT || k == 0) return false;
    const int64_t cols = 16 * c.CT;
    if (V % cols != 0) return false;
    const int64_t w = k / M * N, q = n / V, nquads = (w + 3) / 4;
    // the window division (u < 2^24), D read in whole dwords, A offsets of
    // 16*RT rows, Bc and D offsets up to the quads the ring loads past the
    // last one, the grid
    if (w >= (int64_t(1) << 24) || (w * q) % 4 != 0) return false;
    if (16 * c.RT * k * 4 >= (int64_t(1) << 31)) return false;
    if ((4 * nquads + 32 * c.D + 64) * n * 4 >= (int64_t(1) << 31)) return false;
    if ((4 * nquads + 8 * c.D + 8) * q >= (int64_t(1) << 31)) return false;
    return n / cols <= INT32_MAX;
}

hipError_t launch_rowgather(const RowGatherCfg &c, const RowGatherArgs &a, hipStream_t stream)
{
#define NM_RG_LAUNCH(RT_, CT_, NW_, D_) \
    if (c.RT == RT_ && c.CT == CT_ && c.NW == NW_ && c.D == D_) return launch_cfg<RT_, CT_, NW_, D_>(a, stream);
    NM_ROWGATHER_CONFIGS(NM_RG_LAUNCH)
#undef NM_RG_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace nmspmm
