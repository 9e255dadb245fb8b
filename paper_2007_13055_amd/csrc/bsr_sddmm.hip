// The sampled sibling: D[p] = G[:, block-row of p]^T * X[:, block-column of p] for every stored
// block p -- the gradient of the block values when Y = X * W^T is a layer's forward pass (Y is
// linear in block_data[p][a][c] with coefficient X[i][col*bs_c + c] in Y[i][r*bs_r + a]).
//
// One workgroup (4 wavefronts) per stored block.  The reduction runs over the rows i of G and X, which is the slow
// axis of both, so the operands cannot be read in MFMA order from memory.  A wavefront takes every fourth chunk of 32
// rows: it copies the 32 x bs_r piece of G and the 32 x bs_c piece of X into its own LDS area with contiguous
// 16-byte reads (the next chunk's loads are in flight while this one is multiplied), and reads the
// operands back transposed -- 16-bit types with the LDS transpose read (ds_read_b64_tr_b16: each
// lane receives, for its row of the MFMA operand, 4 consecutive values of the reduction index),
// fp32 one value per lane and MFMA step.  Every wavefront accumulates the whole block over
// its chunks; the four partial blocks are added through LDS in fixed order and stored as one
// contiguous block.  Every block drags its own lines of G and X from L2, so a product that would move many of
// them goes through bsr_sddmm_slab.hip (takes_slabs()).
// Other block shapes: one thread per element of the block, a plain loop over i.
#include <algorithm>

#include "bsr_mfma_common.h"

using namespace bsr_dev;

namespace {

constexpr int kChunk = 32;                            // rows of G and X per step of a wavefront

typedef short s16x4 __attribute__((ext_vector_type(4)));

template <typename T, int BS_R, int BS_C>
struct sddmm_geom {
    static constexpr int S = (int)sizeof(T);
    static constexpr int MM = (BS_R >= 32 && BS_C >= 32) ? 32 : 16;   // MFMA tile edge
    static constexpr int NA = BS_R / MM, NC = BS_C / MM;
    static constexpr int RBG = BS_R * S, RBC = BS_C * S;               // bytes of a row of the G / X piece
    static constexpr int PG = RBG + 16, PC = RBC + 16;                 // padded LDS rows
    static constexpr int NLG = kChunk * RBG / 1024, NLX = kChunk * RBC / 1024;   // 1 KiB loads per chunk
    static constexpr int LDP = BS_C + 4;                               // padded row of the fp32 partial block
    static constexpr int STAGE = kChunk * (PG + PC);
    static constexpr int PART = BS_R * LDP * 4;
    static constexpr int REGION = ((STAGE > PART ? STAGE : PART) + 15) & ~15;
};

// The lane's 8 consecutive reduction-index values of operand row `row0 + lane's row`, 16-bit types.
//   tile   [kChunk][pitch] bytes, row-major pieces of G or X as they lie in memory
//   MM=32: lane l = 32*kappa + 16*beta + lambda feeds MFMA row 16*beta + lambda, values i0 + 8*kappa .. +7
//   MM=16: lane l = 16*g + lambda feeds MFMA row lambda, values i0 + 8*g .. +7
// ds_read_b64_tr_b16 works on groups of 16 lanes: lane mu supplies the address of 4 consecutive
// 16-bit values, and lane lambda receives value (lambda mod 4) of the lanes lambda/4 + 4j, j = 0..3.
// With lane mu pointing at row (mu div 4) and columns 4*(mu mod 4) .. +3 of a 4 x 16 piece, lane
// lambda therefore receives column lambda of its 4 rows: the transpose an MFMA operand needs.
template <typename T, int MM>
__device__ __forceinline__ u32x4 read_operand16(const unsigned char* tile, int pitch, int i0, int col0, int lane)
{
    const int lambda = lane & 15;
    int irow, ccol;
    if constexpr (MM == 32) {
        irow = i0 + 8 * (lane >> 5) + (lambda >> 2);
        ccol = col0 + 16 * ((lane >> 4) & 1) + 4 * (lambda & 3);
    } else {
        irow = i0 + 8 * (lane >> 4) + (lambda >> 2);
        ccol = col0 + 4 * (lambda & 3);
    }
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const unsigned char* p0 = tile + irow * pitch + ccol * 2;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p0 + 4 * pitch));
    const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
    return u32x4{a.x, a.y, b.x, b.y};
}

template <typename T, typename O, int BS_R, int BS_C>
__global__ __launch_bounds__(256) void bsr_sddmm_mfma(const T* __restrict__ G, const T* __restrict__ X,
                                                      const int32_t* __restrict__ block_row,
                                                      const int32_t* __restrict__ indices, O* __restrict__ D,
                                                      int m, int k, int n, int nnzb)
{
    typedef sddmm_geom<T, BS_R, BS_C> geo;
    constexpr int S = geo::S, MM = geo::MM, NA = geo::NA, NC = geo::NC;
    constexpr int RBG = geo::RBG, RBC = geo::RBC, PG = geo::PG, PC = geo::PC, NLG = geo::NLG, NLX = geo::NLX;
    constexpr int LDP = geo::LDP;
    static_assert(NLG >= 1 && NLX >= 1, "a chunk of either piece is at least one load per lane");
    typedef typename AccT<MM>::type acc_t;
    constexpr int NE = MM == 32 ? 16 : 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];   // [4 wavefronts][REGION]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroup b runs on XCD b mod 8: XCD x takes the x-th eighth of the blocks, so that the pieces of G
    // one XCD's L2 holds are those of consecutive block-rows
    const int per_xcd = (int)gridDim.x / 8;
    const int p = (int)(blockIdx.x % 8u) * per_xcd + (int)(blockIdx.x / 8u);
    if (p >= nnzb) return;                            // whole workgroup: the grid is rounded up to 8
    const int r = block_row[p];
    unsigned char* gt = lds + (size_t)wave * geo::REGION;     // G piece [kChunk][PG]
    unsigned char* xt = gt + kChunk * PG;                     // X piece [kChunk][PC]

    acc_t acc[NA][NC];
#pragma unroll
    for (int ua = 0; ua < NA; ++ua)
#pragma unroll
        for (int uc = 0; uc < NC; ++uc)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[ua][uc][e] = 0.f;

    // lane's pieces of a chunk: piece t*64 + lane is 16 bytes of row (piece div pieces-per-row)
    const unsigned char* gbase = reinterpret_cast<const unsigned char*>(G + (size_t)r * BS_R);
    const unsigned char* xbase = reinterpret_cast<const unsigned char*>(X + (size_t)indices[p] * BS_C);
    const size_t grow = (size_t)n * S, xrow = (size_t)k * S;
    int g_row[NLG], g_cb[NLG], x_row[NLX], x_cb[NLX];
#pragma unroll
    for (int t = 0; t < NLG; ++t) { const int q = t * 64 + lane; g_row[t] = q / (RBG / 16); g_cb[t] = (q % (RBG / 16)) * 16; }
#pragma unroll
    for (int t = 0; t < NLX; ++t) { const int q = t * 64 + lane; x_row[t] = q / (RBC / 16); x_cb[t] = (q % (RBC / 16)) * 16; }

    u32x4 gg[NLG], gx[NLX];
    auto fetch = [&](int i0) {                        // rows past m repeat row m-1 and are zeroed when staged
#pragma unroll
        for (int t = 0; t < NLG; ++t)
            gg[t] = *reinterpret_cast<const u32x4*>(gbase + (size_t)min(i0 + g_row[t], m - 1) * grow + g_cb[t]);
#pragma unroll
        for (int t = 0; t < NLX; ++t)
            gx[t] = *reinterpret_cast<const u32x4*>(xbase + (size_t)min(i0 + x_row[t], m - 1) * xrow + x_cb[t]);
    };
    auto stage = [&](int i0) {
        const bool tail = i0 + kChunk > m;            // uniform
        wave_lds_fence();                             // the other lanes have read the previous chunk
#pragma unroll
        for (int t = 0; t < NLG; ++t) {
            u32x4 v = gg[t];
            if (tail && i0 + g_row[t] >= m) v = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4*>(gt + g_row[t] * PG + g_cb[t]) = v;
        }
#pragma unroll
        for (int t = 0; t < NLX; ++t) {
            u32x4 v = gx[t];
            if (tail && i0 + x_row[t] >= m) v = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4*>(xt + x_row[t] * PC + x_cb[t]) = v;
        }
        wave_lds_fence();                             // what is read next is what the other lanes just wrote
    };
    auto compute = [&]() {
        if constexpr (std::is_same<T, float>::value) {
            constexpr int KS = MM == 32 ? 2 : 4;      // reduction steps per MFMA
            const int irow = lane / MM, col = lane % MM;
#pragma unroll
            for (int s = 0; s < kChunk / KS; ++s) {
                float av[NA], bv[NC];
#pragma unroll
                for (int ua = 0; ua < NA; ++ua) av[ua] = *reinterpret_cast<const float*>(gt + (s * KS + irow) * PG + (ua * MM + col) * 4);
#pragma unroll
                for (int uc = 0; uc < NC; ++uc) bv[uc] = *reinterpret_cast<const float*>(xt + (s * KS + irow) * PC + (uc * MM + col) * 4);
#pragma unroll
                for (int ua = 0; ua < NA; ++ua)
#pragma unroll
                    for (int uc = 0; uc < NC; ++uc) {
                        if constexpr (MM == 32) acc[ua][uc] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[ua], bv[uc], acc[ua][uc], 0, 0, 0);
                        else                    acc[ua][uc] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[ua], bv[uc], acc[ua][uc], 0, 0, 0);
                    }
            }
        } else {
            constexpr int KI = MM == 32 ? 16 : 32;    // rows of the chunk one MFMA reduces over
#pragma unroll
            for (int s = 0; s < kChunk / KI; ++s) {
                Frag<T, 8> af[NA], bf[NC];
#pragma unroll
                for (int ua = 0; ua < NA; ++ua) {
                    const u32x4 v = read_operand16<T, MM>(gt, PG, s * KI, ua * MM, lane);
                    af[ua].w[0] = v.x; af[ua].w[1] = v.y; af[ua].w[2] = v.z; af[ua].w[3] = v.w;
                }
#pragma unroll
                for (int uc = 0; uc < NC; ++uc) {
                    const u32x4 v = read_operand16<T, MM>(xt, PC, s * KI, uc * MM, lane);
                    bf[uc].w[0] = v.x; bf[uc].w[1] = v.y; bf[uc].w[2] = v.z; bf[uc].w[3] = v.w;
                }
#pragma unroll
                for (int ua = 0; ua < NA; ++ua)
#pragma unroll
                    for (int uc = 0; uc < NC; ++uc) mfma_frag<T, MM, 8>(acc[ua][uc], af[ua], bf[uc]);
            }
        }
    };

    // chunks wave, wave + 4, ...: the next chunk's loads are issued once this one's registers are in LDS
    const int n_chunks = (m + kChunk - 1) / kChunk;
    if (wave < n_chunks) fetch(wave * kChunk);
    for (int q = wave; q < n_chunks; q += 4) {
        stage(q * kChunk);
        if (q + 4 < n_chunks) fetch((q + 4) * kChunk);
        compute();
    }

    // The wavefront's partial block -> its LDS area as [bs_r][LDP] fp32 (the staged pieces are consumed: a wavefront's
    // own LDS operations complete in order), then the fixed-order sum of the four partial blocks, 4 consecutive
    // columns per thread, contiguous store.
    float* part = reinterpret_cast<float*>(gt);
    wave_lds_fence();
#pragma unroll
    for (int ua = 0; ua < NA; ++ua)
#pragma unroll
        for (int uc = 0; uc < NC; ++uc)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                int a, cc;
                if constexpr (MM == 32) { a = ua * 32 + 8 * (e / 4) + 4 * (lane / 32) + e % 4; cc = uc * 32 + lane % 32; }
                else                    { a = ua * 16 + 4 * (lane / 16) + e;                    cc = uc * 16 + lane % 16; }
                part[a * LDP + cc] = acc[ua][uc][e];
            }
    __syncthreads();
    O* dst = D + (size_t)p * (BS_R * BS_C);
    for (int e4 = threadIdx.x; e4 < BS_R * BS_C / 4; e4 += 256) {
        const int a = (e4 * 4) / BS_C, cc = (e4 * 4) % BS_C;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
            s += *reinterpret_cast<const f32x4*>(lds + (size_t)w * geo::REGION + ((size_t)a * LDP + cc) * 4);
        store4<O>(dst + e4 * 4, s.x, s.y, s.z, s.w);
    }
}

// Blocks below the MFMA tile with BS_R in {1, 2, 4, 8, 16} rows (any bs_c): a lane owns one column
// of one stored block and keeps its BS_R sums.
//   Workgroup (r, t): block-row r, lane slots 64t .. 64t+63 of its cnt*bs_c (block, column) pairs in
//   storage order.  Its four wavefronts take the same slots and a quarter of the rows i each: per row
//   a lane reads its one element of X (the slots of a block are adjacent elements), and the BS_R
//   elements of G -- the same for the whole wavefront -- come through scalar registers.  The four
//   partial sums are added through LDS in fixed order.
// The reads of X are what bounds it: a wavefront instruction gathers 64 different columns of one row.
template <typename T, typename O, int BS_R>
__global__ __launch_bounds__(256) void bsr_sddmm_lanes(const T* __restrict__ G, const T* __restrict__ X,
                                                       const int32_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ indices, O* __restrict__ D,
                                                       int m, int k, int n, int bs_c)
{
    constexpr int kUnroll = 8;
    __shared__ float part[4][BS_R][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = blockIdx.x;
    const int first = indptr[r], cnt = indptr[r + 1] - first;
    const int slot0 = (int)blockIdx.y * 64;
    if (slot0 >= cnt * bs_c) return;                  // whole workgroup
    const int slot = slot0 + lane;
    const bool live = slot < cnt * bs_c;
    const int j = live ? slot / bs_c : 0, cc = live ? slot - j * bs_c : 0;
    const int p = first + j;
    const T* __restrict__ xcol = X + (size_t)indices[p] * bs_c + cc;
    const T* __restrict__ gpiece = G + (size_t)r * BS_R;

    float acc[BS_R];
#pragma unroll
    for (int a = 0; a < BS_R; ++a) acc[a] = 0.f;

    const int per_wave = (m + 3) / 4;
    const int i_begin = min(wave * per_wave, m), i_end = min(i_begin + per_wave, m);
    int i = i_begin;
    for (; i + kUnroll <= i_end; i += kUnroll) {
        float xv[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) xv[u] = (float)xcol[(size_t)(i + u) * k];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const T* __restrict__ g = gpiece + (size_t)(i + u) * n;   // uniform address
#pragma unroll
            for (int a = 0; a < BS_R; ++a) acc[a] = fmaf((float)g[a], xv[u], acc[a]);
        }
    }
    for (; i < i_end; ++i) {
        const float x = (float)xcol[(size_t)i * k];
        const T* __restrict__ g = gpiece + (size_t)i * n;
#pragma unroll
        for (int a = 0; a < BS_R; ++a) acc[a] = fmaf((float)g[a], x, acc[a]);
    }
#pragma unroll
    for (int a = 0; a < BS_R; ++a) part[wave][a][lane] = acc[a];
    __syncthreads();
    if (!live) return;
    for (int a = wave; a < BS_R; a += 4) {
        const float sum = ((part[0][a][lane] + part[1][a][lane]) + part[2][a][lane]) + part[3][a][lane];
        D[((size_t)p * BS_R + a) * bs_c + cc] = (O)sum;
    }
}

// Thin blocks (16 x 1, fp32) with a transposed copy XT (k x m) of X in the caller's scratch: a column of X
// is then a contiguous row, and a block-row is a small dense product
//     D[p0 .. p1)[a] = sum_i G[i][16 r + a] * XT[block column of p][i]
// that the matrix cores take 16 stored blocks at a time: MFMA 16x16x4 with M = a, N = block, K = i.
//   Workgroup (r, t): block-row r, its stored blocks 64 t .. 64 t + 63; wavefront w the 16 blocks from
//   64 t + 16 w.  The rows i go by in pieces of 256: the workgroup copies that piece of G's 16 columns
//   into LDS (64 contiguous bytes per row), every wavefront reads its 64 A operands from there (pitch
//   20 words: the four row groups of a read fall on different banks), and then walks the piece 16 rows
//   at a time: one 16-byte read of XT per lane (4 consecutive i of its block's column) feeds 4 MFMAs.
//   MFMA u of a 16-row step reduces over i = I + 4 g + u for k-group g, on both operands.
// Rows past m: G is read from row m-1 and replaced by zero, XT is read as it lies (the scratch is padded)
// and replaced by zero; lanes past the block-row's last block repeat it and store nothing.
__global__ __launch_bounds__(256, 4) void bsr_sddmm_thin16(const float* __restrict__ G, const float* __restrict__ XT,
                                                        const int32_t* __restrict__ indptr,
                                                        const int32_t* __restrict__ indices, float* __restrict__ D,
                                                        int m, int n, int mp)
{
    constexpr int kPiece = 256, kPitch = 20;
    __shared__ float gs[kPiece * kPitch];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = blockIdx.x;
    const int first = indptr[r], cnt = indptr[r + 1] - first;
    const int j0 = ((int)blockIdx.y * 4 + wave) * 16;             // first block of this wavefront's 16
    if ((int)blockIdx.y * 64 >= cnt) return;                      // whole workgroup
    const bool active = j0 < cnt;                                 // uniform over the wavefront
    const int j = lane & 15, g = lane >> 4;
    const int p = first + min(j0 + j, cnt - 1);
    // XT is read with 4 consecutive lanes on the 64 contiguous bytes of one block's column (lane l: block
    // l / 4, k-group l mod 4) and moved to the MFMA's lane order (block l mod 16, k-group l / 16) by lane
    // permutes: four lanes of a quad on four different lines would quarter the load rate
    const int jl = lane >> 2, gl = lane & 3;
    const float* __restrict__ xrow = XT + (size_t)indices[first + min(j0 + jl, cnt - 1)] * mp + 4 * gl;
    const int from = (4 * j + g) * 4;                             // byte address of the source lane for ds_bpermute
    const float* __restrict__ gcols = G + (size_t)r * 16;

    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};   // two chains: even and odd steps
    for (int i0 = 0; i0 < m; i0 += kPiece) {
        if (i0 > 0) __syncthreads();                              // the piece before is read
        // rows i0 .. i0+255 of G's 16 columns -> LDS; thread t: rows t/4 + 64 q, 16 bytes at column 4 (t mod 4)
#pragma unroll
        for (int q = 0; q < kPiece / 64; ++q) {
            const int row = (tid >> 2) + 64 * q;
            const int i = i0 + row;
            f32x4 v = *reinterpret_cast<const f32x4*>(gcols + (size_t)min(i, m - 1) * n + 4 * (tid & 3));
            if (i >= m) v = f32x4{0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4*>(gs + row * kPitch + 4 * (tid & 3)) = v;
        }
        __syncthreads();
        if (!active) continue;
        float A[kPiece / 16][4];
#pragma unroll
        for (int b = 0; b < kPiece / 16; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) A[b][u] = gs[(16 * b + 4 * g + u) * kPitch + j];
        // the reads of XT of half a piece (8 steps) are issued before the first is used; a step past m
        // repeats the last step's address and is not multiplied
        const int last_step = ((m - 1) / 16) * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 xl[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) xl[b] = *reinterpret_cast<const u32x4*>(xrow + min(i0 + 16 * (8 * h + b), last_step));
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int I = i0 + 16 * (8 * h + b);
                if (I < m) {                                      // uniform
                    f32x4 x;
                    x.x = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, (int)xl[b].x));
                    x.y = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, (int)xl[b].y));
                    x.z = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, (int)xl[b].z));
                    x.w = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, (int)xl[b].w));
                    if (I + 16 > m) {                             // uniform: the last, partial step
                        if (I + 4 * g + 0 >= m) x.x = 0.f;
                        if (I + 4 * g + 1 >= m) x.y = 0.f;
                        if (I + 4 * g + 2 >= m) x.z = 0.f;
                        if (I + 4 * g + 3 >= m) x.w = 0.f;
                    }
                    f32x4& c = (b & 1) ? acc2 : acc;
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[8 * h + b][0], x.x, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[8 * h + b][1], x.y, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[8 * h + b][2], x.z, c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[8 * h + b][3], x.w, c, 0, 0, 0);
                }
            }
        }
    }
    // lane (block j, group g) holds D[p][4 g .. 4 g + 3]
    if (active && j0 + j < cnt) *reinterpret_cast<f32x4*>(D + (size_t)p * 16 + 4 * g) = acc + acc2;
}

// Any other block shape: thread e of the workgroup owns elements e, e + 256, ... of the block.
template <typename T, typename O>
__global__ __launch_bounds__(256) void bsr_sddmm_generic(const T* __restrict__ G, const T* __restrict__ X,
                                                         const int32_t* __restrict__ block_row,
                                                         const int32_t* __restrict__ indices, O* __restrict__ D,
                                                         int m, int k, int n, int bs_r, int bs_c)
{
    const int p = blockIdx.x;
    const int r = block_row[p], c = indices[p];
    for (int e = threadIdx.x; e < bs_r * bs_c; e += 256) {
        const int a = e / bs_c, cc = e - a * bs_c;
        const T* g = G + (size_t)r * bs_r + a;
        const T* x = X + (size_t)c * bs_c + cc;
        float acc = 0.f;
        for (int i = 0; i < m; ++i) acc = fmaf((float)g[(size_t)i * n], (float)x[(size_t)i * k], acc);
        D[(size_t)p * bs_r * bs_c + e] = (O)acc;
    }
}

template <typename T, typename O, int BS_R, int BS_C>
bsr_status launch_sddmm_shape(const bsr_matrix* W, int m, const void* G, const void* X, void* D, hipStream_t stream)
{
    typedef sddmm_geom<T, BS_R, BS_C> geo;
    const size_t lds = 4 * (size_t)geo::REGION;
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&bsr_sddmm_mfma<T, O, BS_R, BS_C>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return BSR_ERR_HIP;
    hipLaunchKernelGGL((bsr_sddmm_mfma<T, O, BS_R, BS_C>), dim3((unsigned)((W->nnzb + 7) / 8 * 8)), dim3(256), lds, stream,
                       (const T*)G, (const T*)X, W->block_row, W->indices, (O*)D, m, (int)W->k, (int)W->n, (int)W->nnzb);
    return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
}

// Whether the groups of bsr_sddmm_slab.hip take this product.  A block by itself drags two lines of G and X per row of
// the reduction, at 15-18 TB/s over the whole chip and 3 us to begin with; the groups move each slab once for many
// blocks, but their two launches cost 10 us.  Measured on bf16, m x (n, k): 16x16 4096 x (3072, 768) 1.9 GB of lines,
// 21 us against 37; 32x32 2048 x (2048, 2048) 107 MB, 14.6 against 11.3; fp32 16x16 2000 x (1024, 1024) 314 MB,
// 20.9 against 19.1.  Few blocks and many rows leave most CUs idle when a workgroup takes a block, 128 rows in 0.6 us
// (fp32: 0.6, 0.9 and 2.8 us for blocks of 256, 1024 and 4096 elements, the matrix cores' time), while the groups
// split the rows (29 fp16 64x64 blocks, 3903 rows: 14.8 us against 22).  8-wide blocks have no matrix-core kernel of their
// own: 16-bit ones take the groups from 256 rows on (530 x (576, 384): 8.1 us against 11.0); fp32 ones, three
// quarters of whose matrix-core tiles are padding, only when the lines are many.
//
// All that is for 16-bit blocks with room for the partial results.  Without, the groups are too few to fill the chip; and
// fp32 products are bound by the matrix cores, which a block per workgroup keeps as busy and spreads more evenly.  So
// these take the groups only if that is estimated to be quicker than the blocks by themselves as well.  Groups against
// blocks, us: without room 13 bf16 32x32 blocks, 5000 rows 73, 12.7; bf16 16x16 4096 x (3072, 768) 50, 77; fp32
// 32x32 1003 x (4096, 4096) 10 % 94, 44; fp32 with room 64x64 8192 x (4096, 4096) 10 % 926, 325, 32x32 716, 348,
// 16x16 798, 1170, 64x16 7778 x (3520, 6976) 15 % 1150, 712; 64x64 7596 x (7296, 3648) 4 % 234, 282, 41 blocks of
// 64x64, 1601 rows 19.5, 37.8, 75 of 64x16, 5869 rows 26, 60.  8-wide blocks stay with
// the groups (bf16 2178 x (512, 5632), 17 %: 29 against 118, fp32 5317 x (5376, 640), 12 %: 197 against 393).
bool takes_slabs(const bsr_matrix* W, int64_t m, size_t workspace_bytes)
{
    if (!sddmm_slab_supports(W, m)) return false;
    if (W->env_tune.sd) return W->env_tune.sd == 2 && sddmm_slab_ready(W);
    const int s = W->dtype == BSR_F32 ? 4 : 2;
    const double rows = (double)m, lines = (double)W->nnzb * rows * (std::max(128, W->bs_r * s) + std::max(128, W->bs_c * s));
    if (W->bs_r == 8 || W->bs_c == 8) return (W->dtype == BSR_F32 ? m >= 512 && lines > 2e9 : m >= 256) && sddmm_slab_ready(W);
    const int elems = W->bs_r * W->bs_c;
    const double alone = rows / 128 * (W->dtype != BSR_F32 || elems < 1024 ? 0.6 : elems < 4096 ? 0.9 : 2.8);
    if (!(lines > 350e6 || (W->nnzb <= 256 && 3.0 + alone > (W->nnzb <= 64 ? 13.0 : 17.0))) || !sddmm_slab_ready(W)) return false;
    const bool room = workspace_bytes >= sddmm_slab_workspace(W, m);
    if (room && W->dtype != BSR_F32) return true;
    double by_block = std::max(alone, lines / 16.5e6);
    if (W->dtype == BSR_F32) {                        // several blocks to a CU share its matrix cores
        // us for 128 rows of a block: 16-row or -column blocks of 256, 512 and 1024 elements, others of 1024, 2048, 4096;
        // half as much again (narrow), or a seventh, where a block has a CU to itself
        const bool narrow = std::min(W->bs_r, W->bs_c) == 16;
        const double block = narrow ? (elems < 512 ? 0.45 : elems < 1024 ? 0.52 : 0.85) : (elems < 2048 ? 0.78 : elems < 4096 ? 1.4 : 2.6);
        const int64_t per_cu = (W->nnzb + W->n_cu - 1) / W->n_cu;
        by_block = std::max(by_block, rows / 128 * block * (per_cu > 1 ? (double)per_cu : narrow ? 1.5 : 1.15));
    }
    return sddmm_slab_us(W, m, room) < 3.0 + by_block;
}

template <typename T, typename O>
bsr_status launch_sddmm_types(const bsr_matrix* W, int m, const void* G, const void* X, void* D, hipStream_t stream)
{
    const int br = W->bs_r, bc = W->bs_c;
    BSR_MFMA_SHAPES(launch_sddmm_shape, T, O, br, bc, W, m, G, X, D, stream);
    if constexpr (std::is_same<T, float>::value && std::is_same<O, float>::value) {
        // thin blocks with the caller's scratch lent: transposed copy of X, then the matrix-core kernel
        if (sddmm_transposes(W, m)) {
            float* XT = static_cast<float*>(W->scratch);
            const bsr_status st = launch_transpose_f32((const float*)X, XT, m, (int)W->k, stream);
            if (st != BSR_OK) return st;
            const int64_t groups = ((int64_t)W->max_row_blocks + 63) / 64;
            if (groups > 65535) return BSR_ERR_SHAPE;
            hipLaunchKernelGGL(bsr_sddmm_thin16, dim3((unsigned)W->R, (unsigned)groups), dim3(256), 0, stream,
                               (const float*)G, (const float*)XT, W->indptr, W->indices, (float*)D, m, (int)W->n,
                               (m + 3) & ~3);
            return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
        }
    }
    auto lanes = [&](auto rows_tag) -> bsr_status {
        constexpr int BS_R = decltype(rows_tag)::value;
        const int64_t tiles = ((int64_t)W->max_row_blocks * bc + 63) / 64;
        if (tiles > 65535 || W->R > 0x7fffffff) return BSR_ERR_SHAPE;
        hipLaunchKernelGGL((bsr_sddmm_lanes<T, O, BS_R>), dim3((unsigned)W->R, (unsigned)tiles), dim3(256), 0, stream,
                           (const T*)G, (const T*)X, W->indptr, W->indices, (O*)D, m, (int)W->k, (int)W->n, bc);
        return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
    };
    if (br == 16) return lanes(std::integral_constant<int, 16>{});
    if (br == 8) return lanes(std::integral_constant<int, 8>{});
    if (br == 4) return lanes(std::integral_constant<int, 4>{});
    if (br == 2) return lanes(std::integral_constant<int, 2>{});
    if (br == 1) return lanes(std::integral_constant<int, 1>{});
    hipLaunchKernelGGL((bsr_sddmm_generic<T, O>), dim3((unsigned)W->nnzb), dim3(256), 0, stream,
                       (const T*)G, (const T*)X, W->block_row, W->indices, (O*)D, m, (int)W->k, (int)W->n, br, bc);
    return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
}

}  // namespace

extern "C" bsr_status bsr_sddmm_workspace_size(const bsr_matrix* W, int64_t m, size_t* bytes)
{
    if (!W || !bytes) return BSR_ERR_NULL;
    *bytes = 0;
    if (m < 0) return BSR_ERR_SHAPE;
    const size_t b = takes_slabs(W, m, SIZE_MAX) ? sddmm_slab_workspace(W, m) : sddmm_thin_supports(W, m, SIZE_MAX) ? sddmm_thin_workspace(W, m) : 0;
    *bytes = (b + 255) & ~(size_t)255;
    return BSR_OK;
}

extern "C" bsr_status bsr_sddmm(const bsr_matrix* W, int64_t m, const void* G_dev, const void* X_dev, void* D_dev,
                                bsr_dtype d_dtype, void* hip_stream)
{
    return bsr_sddmm_ws(W, m, G_dev, X_dev, D_dev, d_dtype, nullptr, 0, hip_stream);
}

extern "C" bsr_status bsr_sddmm_ws(const bsr_matrix* W, int64_t m, const void* G_dev, const void* X_dev, void* D_dev,
                                   bsr_dtype d_dtype, void* workspace_dev, size_t workspace_bytes, void* hip_stream)
{
    if (!W) return BSR_ERR_NULL;
    if (m < 0) return BSR_ERR_SHAPE;
    if (d_dtype != W->dtype && d_dtype != BSR_F32) return BSR_ERR_DTYPE;
    if (W->nnzb == 0) return BSR_OK;
    if (!D_dev || (m > 0 && (!G_dev || !X_dev))) return BSR_ERR_NULL;
    if (m * std::max<int64_t>(W->k, W->n) >= ((int64_t)1 << 31)) return BSR_ERR_SHAPE;
    if (((uintptr_t)G_dev | (uintptr_t)X_dev | (uintptr_t)D_dev | (uintptr_t)workspace_dev) & 15u) return BSR_ERR_ALIGN;
    hipStream_t stream = (hipStream_t)hip_stream;
    order_after_upload(stream, W->plan_uploaded, W->plan_landed);
    if (W->debug) {
        const bsr_status dbg = debug_check_device_arrays(W, stream);
        if (dbg != BSR_OK) return dbg;
    }
    // m == 0 needs no special case: the kernels then read nothing and store zeros (an empty sum)
    const int mi = (int)m;
    if (takes_slabs(W, m, workspace_dev ? workspace_bytes : 0))
        return launch_sddmm_slab(W, mi, G_dev, X_dev, D_dev, d_dtype, workspace_dev, workspace_bytes, stream);
    if (sddmm_thin_supports(W, m, workspace_dev ? workspace_bytes : 0) && d_dtype == BSR_F32)
        return launch_sddmm_thin(W, mi, G_dev, X_dev, D_dev, workspace_dev, workspace_bytes, stream);
    if (W->dtype == BSR_F32) return launch_sddmm_types<float, float>(W, mi, G_dev, X_dev, D_dev, stream);
    if (W->dtype == BSR_F16) return d_dtype == BSR_F32 ? launch_sddmm_types<_Float16, float>(W, mi, G_dev, X_dev, D_dev, stream)
                                                       : launch_sddmm_types<_Float16, _Float16>(W, mi, G_dev, X_dev, D_dev, stream);
    return d_dtype == BSR_F32 ? launch_sddmm_types<__bf16, float>(W, mi, G_dev, X_dev, D_dev, stream)
                              : launch_sddmm_types<__bf16, __bf16>(W, mi, G_dev, X_dev, D_dev, stream);
}
