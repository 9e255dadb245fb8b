// The sampled product D[p] = G[:, block-row of p]^T * X[:, block-column of p] on the matrix cores, many rows of
// G and X: block shapes with bs_r and bs_c in {8, 16, 32, 64}.
//
// What bounds it.  A stored block needs an (m x bs_r) piece of G and an (m x bs_c) piece of X, and pieces narrower
// than a 128-byte line drag whole lines; taken block by block that is 5-20 times the two matrices.  So the unit of
// staging is a SLAB, 128 bytes of a row of G or X (64 16-bit or 32 fp32 columns) by 32 rows, and a workgroup takes
// a GROUP of stored blocks that share slabs: at most 12 slabs, of which the plan puts as many blocks as the
// accumulators hold.  The group's rows of G and X stream through LDS once, 32 rows at a time, and every wavefront
// keeps its blocks in registers over all rows.
//
//   tile   V x V outputs, the MFMA's own size: V = 32 when both block sides are at least 32, else 16.  A tile is a
//          part of a block, a block, or (8-wide blocks) up to four blocks, the missing ones computed and not stored.
//   chunk  the tiles a wavefront multiplies from one set of LDS reads: CC tiles of one row of tiles (CR = 1), or a
//          64x64 block (CR = CC = 2).  A chunk with fewer tiles repeats its last one and stores it once.
//   group  up to 8 * NCH chunks, chunk c on wavefront c mod 8; NG slabs of G, then those of X.
//
// The rows are split S ways when there are fewer groups than CUs; the S partial results (fp32, in the caller's
// workspace) are added in fixed order by a second kernel.  Workgroups are numbered split by split and cut into
// eight contiguous pieces, one per XCD, so that an XCD's L2 serves the groups that read the same rows and columns.
//
// Twelve wavefronts: eight multiply, four only move slabs (a wavefront that issues a load waits until the memory
// pipeline takes it; done by the multiplying ones the two times added up).  Loads write LDS directly
// (buffer_load_dwordx4 ... lds, 1 KiB = 8 rows of a slab) into a ring of three to eight buffers, one barrier per 32 rows.
// A slab's rows lie 128 bytes apart unpadded; the 16-byte pieces of row r are stored XOR sigma(r), which
// keeps the transpose reads (ds_read_b64_tr_b16; fp32: single values) off each other's banks.  Rows past m lie past
// the end of the buffer and arrive as zeros.  The loads are inline assembly: the compiler would wait for all of them
// before the first LDS read.
//
// Measured (MI355X, operands in the last-level cache or beyond): bf16 16x16, 4096 x (3072, 768), 1843 blocks: 21.1 us
// (15 + 6 for the sum of 6 splits) where a workgroup per 64 x 64 columns took 37.2; bf16 32x32, 4096 x (4096, 4096),
// 10 %: 42.8 against 99; fp16 64x64, 8192^3, 819 blocks by a power law: 103 (94 + 9) against 151.  A step of 32 rows takes
// 0.18 us plus 0.12 us per round of chunks.  Counters: on the bf16 product the matrix cores are busy 14 % and the LDS 18 % of
// the time and 3.3 TB/s come from beyond L2: a step's chain from barrier over LDS reads to the last product is what
// takes it, two multiplying wavefronts a SIMD deep.  The fp16 one waits for slabs, 456 MB from beyond L2 (62 us at the 7.4 TB/s
// that such loads reach at best).  fp32 products are bound by the matrix cores and mostly left to a workgroup per block
// (takes_slabs() in bsr_sddmm.hip).
#include <algorithm>
#include <numeric>
#include <cmath>

#include "bsr_mfma_common.h"

using namespace bsr_dev;
using namespace bsr_dev::lds_loads;

namespace {

constexpr int kRows = 32;                             // rows of G and X per step
constexpr int kWaves = 8;                             // wavefronts that multiply
constexpr int kLoaders = 4;                           // wavefronts that only move slabs
constexpr int kMaxSlabs = 12;                         // per group: 3 buffers of 12 slabs are 144 KiB of LDS
constexpr int kSlab = kRows * 128;                    // bytes of a slab in LDS
// Buffers of a group's slabs: as many as LDS holds, enough for 32 KiB a step to be a microsecond ahead.
constexpr int slab_buffers(int slabs) { return 40 / slabs < 8 ? 40 / slabs : 8; }
constexpr int kHdr = 16;                              // words of a group header: {slabs, of G, first chunk, chunks, first columns[12]}
constexpr int kHdrSlabsAt = 4;
constexpr int kXcds = 8;

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Chunk shape and chunks per wavefront by tile size and block shape.
struct slab_shape { int V, CR, CC, NCH; };
inline slab_shape slab_shape_of(int bs_r, int bs_c)
{
    if (bs_r == 64 && bs_c == 64) return {32, 2, 2, 1};
    if (bs_r >= 32 && bs_c >= 32) return {32, 1, 2, 3};
    return {16, 1, 4, 5};
}


template <typename T, int V>
__device__ __forceinline__ int sigma(int r)
{
    if constexpr (std::is_same<T, float>::value) return V == 16 ? ((r >> 1) & 1) << 2 : 0;
    else return V == 16 ? (((r >> 1) & 1) << 1) | (((r >> 3) & 1) << 2) : ((r >> 1) & 1) << 2;
}

// Byte offset, inside a slab, of what lane `lane` reads for the tile at columns 0.. of the slab; a tile at byte
// column b of slab q is at (q * kSlab + b) XOR this (b is a multiple of the tile's width, which sigma leaves whole).
template <typename T, int V>
__device__ __forceinline__ unsigned operand_lane_offset(int lane)
{
    int r, cb;
    if constexpr (std::is_same<T, float>::value) {
        r = lane / V;
        cb = (lane % V) * 4;
    } else {
        const int lambda = lane & 15;
        if constexpr (V == 32) { r = 8 * (lane >> 5) + (lambda >> 2); cb = 32 * ((lane >> 4) & 1) + 8 * (lambda & 3); }
        else                   { r = 8 * (lane >> 4) + (lambda >> 2); cb = 8 * (lambda & 3); }
    }
    return (unsigned)(r * 128 + ((((cb >> 4) ^ sigma<T, V>(r))) << 4) + (cb & 15));
}

// The lane's 8 values of the reduction index for operand step s (16-bit types).
template <int V>
__device__ __forceinline__ u32x4 read_tr(const unsigned char* p, int s)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const unsigned char* q = p + s * (V == 32 ? 16 : 32) * 128;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + 4 * 128));
    const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
    return u32x4{a.x, a.y, b.x, b.y};
}

// Where output (a, c .. c+3) of a tile goes (null: nowhere): the tile's quadrants (V/2 x V/2) each lie whole in one
// block; off[q] is the element of D at quadrant q's (0, 0), or -1 where no block is stored.
template <typename O, int V>
__device__ __forceinline__ O* tile4(O* __restrict__ D, const i32x4& off, int bs_c, int a, int c)
{
    constexpr int H = V / 2;
    const int top = c >= H ? off.y : off.x, bottom = c >= H ? off.w : off.z;
    const int o = a >= H ? bottom : top;
    return o >= 0 ? D + (size_t)(unsigned)o + (a % H) * bs_c + c % H : nullptr;
}

template <typename T, typename O, int V, int CR, int CC, int NCH, bool SPLIT>
__global__ __launch_bounds__(64 * (kWaves + kLoaders)) void bsr_sddmm_slab(const T* __restrict__ G, const T* __restrict__ X,
                                                             const int32_t* __restrict__ groups,
                                                             const i32x4* __restrict__ chunks,
                                                             const i32x4* __restrict__ tiles, O* __restrict__ D,
                                                             float* __restrict__ part, int m, int k, int n, int bs_c,
                                                             int n_groups, int splits, int n_tiles, int pieces)
{
    constexpr bool F32 = std::is_same<T, float>::value;
    constexpr int S = (int)sizeof(T);
    constexpr int NT = CR * CC;                       // tiles of a chunk
    constexpr int NQ = V == 32 ? 4 : 1;               // groups of 4 results per lane and tile
    constexpr int STEPS = F32 ? kRows / (V == 32 ? 2 : 4) : kRows / (V == 32 ? 16 : 32);   // MFMA steps over 32 rows
    typedef typename AccT<V>::type acc_t;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];   // [slab_buffers][slabs of the group][kSlab]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = (int)gridDim.x / kXcds;
    const int job = (int)(blockIdx.x % (unsigned)kXcds) * per_xcd + (int)(blockIdx.x / (unsigned)kXcds);
    if (job >= n_groups * splits) return;             // whole workgroup: the grid is rounded up to 8
    // SPLIT: workgroups share out the rows, split by split; else (where there is no place for partial results) `splits`
    // neighbouring ones share out a group's chunks
    const int split = SPLIT ? job / n_groups : 0, group = SPLIT ? job - split * n_groups : job / splits;
    const int32_t* __restrict__ hdr = groups + (size_t)group * kHdr;   // uniform: scalar reads
    const int n_slabs = hdr[0], n_g = hdr[1];
    int first_chunk = hdr[2], n_chunks = hdr[3];
    if constexpr (!SPLIT) {
        const int part = job - group * splits, c0 = n_chunks * part / splits, c1 = n_chunks * (part + 1) / splits;
        if (c0 == c1) return;                         // whole workgroup
        first_chunk += c0;
        n_chunks = c1 - c0;
    }

    const unsigned buf_bytes = (unsigned)n_slabs * kSlab, nb = (unsigned)slab_buffers(n_slabs);
    // steps [q0, q1) of 32 rows
    const unsigned n_steps = (unsigned)(m + kRows - 1) / kRows;
    const int row_splits = SPLIT ? splits : 1;
    const int q0 = (int)(n_steps * (unsigned)split / (unsigned)row_splits), q1 = (int)(n_steps * (unsigned)(split + 1) / (unsigned)row_splits);

    if (wave >= kWaves) {
        // ---- moving slabs: a wavefront that issues a load waits until the memory pipeline takes it, about as long as
        // a chunk takes to multiply, so the two are not done by the same wavefronts.  Loader w moves rows 8 w .. 8 w + 7
        // of every slab.
        const int r = 8 * (wave - kWaves) + (lane >> 3);
        const unsigned g_row = (unsigned)n * S, x_row = (unsigned)k * S;
        const unsigned piece = (unsigned)(((lane & 7) ^ sigma<T, V>(r)) << 4);
        const unsigned src_g = (unsigned)r * g_row + piece, src_x = (unsigned)r * x_row + piece;
        const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)lds + (unsigned)(wave - kWaves) * 1024u;
        // One loop per number of slabs: its loads and the count to wait for are fixed, so a step has no branch (one per
        // load cost as much as the loads).  Steps past the last read a buffer of no bytes (zeros, no traffic), which
        // keeps the count right to the end.
        auto move = [&](auto ns_tag) {
            constexpr int NS = decltype(ns_tag)::value, NB = slab_buffers(NS);
            unsigned src[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j) src[j] = (j < n_g ? src_g : src_x) + (unsigned)hdr[kHdrSlabsAt + j] * S;
            unsigned long long ga = reinterpret_cast<unsigned long long>(G) + (unsigned long long)q0 * kRows * g_row;
            unsigned long long xa = reinterpret_cast<unsigned long long>(X) + (unsigned long long)q0 * kRows * x_row;
            int left = q1 - q0;                       // steps still to issue
            long long rows_left = (long long)m - (long long)q0 * kRows;
            auto issue = [&](unsigned buf) {
                const long long g_left = rows_left * g_row, x_left = rows_left * x_row;
                i32x4 rg, rx;
                rg.x = (int)(unsigned)ga; rg.y = (int)((unsigned)(ga >> 32) & 0xFFFFu);
                rg.z = left <= 0 ? 0 : g_left > 0x7fffffffll ? 0x7fffffff : (int)g_left; rg.w = 0x00020000;
                rx.x = (int)(unsigned)xa; rx.y = (int)((unsigned)(xa >> 32) & 0xFFFFu);
                rx.z = left <= 0 ? 0 : x_left > 0x7fffffffll ? 0x7fffffff : (int)x_left; rx.w = 0x00020000;
                const unsigned base = lds0 + buf * (NS * kSlab);
#pragma unroll
                for (int j = 0; j < NS; ++j) {
                    i32x4 r;
                    r.x = j < n_g ? rg.x : rx.x; r.y = j < n_g ? rg.y : rx.y; r.z = j < n_g ? rg.z : rx.z; r.w = 0x00020000;
                    load_to_lds(r, src[j], base + j * kSlab);
                }
                ga += (unsigned long long)kRows * g_row;
                xa += (unsigned long long)kRows * x_row;
                rows_left -= kRows;
                --left;
            };
#pragma unroll
            for (int j = 0; j < NB - 1; ++j) issue((unsigned)j);
            unsigned buf = 0;
            for (int q = q0; q < q1; ++q) {
                wait_vm<(NB - 2) * NS>();             // this wavefront's share of step q has landed
                asm volatile("s_barrier" ::: "memory");   // everybody's has, and everybody has read step q - 1
                issue(buf == 0 ? NB - 1 : buf - 1);
                buf = buf == NB - 1 ? 0 : buf + 1;
            }
            wait_vm<0>();                             // nothing may land in LDS after the workgroup has gone
        };
        switch (n_slabs) {                            // 2 .. kMaxSlabs
            case 2: move(std::integral_constant<int, 2>{}); break;
            case 3: move(std::integral_constant<int, 3>{}); break;
            case 4: move(std::integral_constant<int, 4>{}); break;
            case 5: move(std::integral_constant<int, 5>{}); break;
            case 6: move(std::integral_constant<int, 6>{}); break;
            case 7: move(std::integral_constant<int, 7>{}); break;
            case 8: move(std::integral_constant<int, 8>{}); break;
            case 9: move(std::integral_constant<int, 9>{}); break;
            case 10: move(std::integral_constant<int, 10>{}); break;
            case 11: move(std::integral_constant<int, 11>{}); break;
            default: move(std::integral_constant<int, 12>{}); break;
        }
        return;
    }

    // ---- multiplying: this wavefront's chunks ----
    i32x4 rec[NCH];
#pragma unroll
    for (int j = 0; j < NCH; ++j)
        rec[j] = chunks[first_chunk + min(wave + kWaves * j, n_chunks - 1)];
    const int mine = max(0, (n_chunks - wave + kWaves - 1) / kWaves);

    acc_t acc[NCH][NT];

    const unsigned lane_off = operand_lane_offset<T, V>(lane);
    // byte offsets of chunk j's tiles in a buffer: G rows, X columns
    auto a_off = [&](int j, int u) -> unsigned { return ((unsigned)rec[j].x >> (16 * u)) & 0xFFFFu; };
    auto b_off = [&](int j, int u) -> unsigned { return ((unsigned)(u < 2 ? rec[j].y : rec[j].z) >> (16 * (u & 1))) & 0xFFFFu; };

    struct operands { u32x4 a[CR][F32 ? 1 : STEPS], b[CC][F32 ? 1 : STEPS]; };
    auto read = [&](operands& o, int j, unsigned buf) {
#pragma unroll
        for (int u = 0; u < CR; ++u)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) o.a[u][s] = read_tr<V>(lds + ((buf + a_off(j, u)) ^ lane_off), s);
#pragma unroll
        for (int u = 0; u < CC; ++u)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) o.b[u][s] = read_tr<V>(lds + ((buf + b_off(j, u)) ^ lane_off), s);
    };
    auto multiply = [&](const operands& o, int j) {
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int ur = 0; ur < CR; ++ur)
#pragma unroll
                for (int uc = 0; uc < CC; ++uc) {
                    Frag<T, 8> x, g;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { x.w[e] = o.b[uc][s][e]; g.w[e] = o.a[ur][s][e]; }
                    mfma_frag<T, V, 8>(acc[j][ur * CC + uc], x, g);
                }
    };

    // The rows in `pieces`, each summed by itself and added to what the pieces before it have left in D or among the
    // partial results: one chain over all rows is the less exact the longer it is.  A result of 16 bits does not show it,
    // and its kernel has no such loop (batched backward 44.1 us with one of a single piece, 41.7 without).
    const int n_pieces = std::is_same<O, float>::value ? pieces : 1;
    unsigned buf = 0;
    for (int piece = 0; piece < n_pieces; ++piece) {
        const int first_q = q0 + (q1 - q0) * piece / n_pieces, end_q = q0 + (q1 - q0) * (piece + 1) / n_pieces;
#pragma unroll
        for (int j = 0; j < NCH; ++j)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4 * NQ; ++e) acc[j][t][e] = 0.f;
        for (int q = first_q; q < end_q; ++q) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // step q has landed, step q - 1 is read
            const unsigned at = buf * buf_bytes;
            if constexpr (F32) {
#pragma unroll
                for (int j = 0; j < NCH; ++j)
                    if (j < mine) {                       // uniform
                        const float *ap[CR], *bp[CC];
#pragma unroll
                        for (int u = 0; u < CR; ++u) ap[u] = reinterpret_cast<const float*>(lds + ((at + a_off(j, u)) ^ lane_off));
#pragma unroll
                        for (int u = 0; u < CC; ++u) bp[u] = reinterpret_cast<const float*>(lds + ((at + b_off(j, u)) ^ lane_off));
#pragma unroll
                        for (int s = 0; s < STEPS; ++s) {
                            constexpr int KS = V == 32 ? 2 : 4;
                            float av[CR], bv[CC];
#pragma unroll
                            for (int u = 0; u < CR; ++u) av[u] = ap[u][s * KS * 32];
#pragma unroll
                            for (int u = 0; u < CC; ++u) bv[u] = bp[u][s * KS * 32];
#pragma unroll
                            for (int ur = 0; ur < CR; ++ur)
#pragma unroll
                                for (int uc = 0; uc < CC; ++uc) {
                                    if constexpr (V == 32) acc[j][ur * CC + uc] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[uc], av[ur], acc[j][ur * CC + uc], 0, 0, 0);
                                    else                   acc[j][ur * CC + uc] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[uc], av[ur], acc[j][ur * CC + uc], 0, 0, 0);
                                }
                        }
                    }
            } else {
                // the next chunk's operands are read while one is multiplied
                operands o[2];
                if (mine > 0) read(o[0], 0, at);
#pragma unroll
                for (int j = 0; j < NCH; ++j) {
                    if (j < mine) {                       // uniform
                        if (j + 1 < NCH && j + 1 < mine) read(o[(j + 1) & 1], j + 1 < NCH ? j + 1 : 0, at);
                        multiply(o[j & 1], j);
                    }
                }
            }
            buf = buf == nb - 1 ? 0 : buf + 1;
        }

        // lane holds, of every tile, row a = lane mod V and columns c .. c+3, c = 8 q + 4 (lane / V) (V = 16: 4 (lane / 16))
        const int a = lane % V, c0 = 4 * (lane / V);
#pragma unroll
        for (int j = 0; j < NCH; ++j)
            if (j < mine) {
                const int t0 = rec[j].w & 0x0fffffff, live = (int)((unsigned)rec[j].w >> 28);
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (t < live) {
#pragma unroll
                        for (int g = 0; g < NQ; ++g) {
                            f32x4 v = {acc[j][t][4 * g], acc[j][t][4 * g + 1], acc[j][t][4 * g + 2], acc[j][t][4 * g + 3]};
                            if constexpr (SPLIT) {
                                f32x4* dst = reinterpret_cast<f32x4*>(part + ((((size_t)split * n_tiles + t0 + t) * NQ + g) * 64 + lane) * 4);
                                if (n_pieces > 1 && piece > 0) v += *dst;
                                *dst = v;
                            } else if (O* dst = tile4<O, V>(D, tiles[t0 + t], bs_c, a, 8 * g + c0)) {
                                if constexpr (std::is_same<O, float>::value) {
                                    if (piece > 0) v += *reinterpret_cast<const f32x4*>(dst);
                                }
                                store4<O>(dst, v.x, v.y, v.z, v.w);
                            }
                        }
                    }
            }
    }
}

// Sum of the S partial results of every tile, in split order.
template <typename O, int V>
__global__ __launch_bounds__(256) void bsr_sddmm_slab_sum(const float* __restrict__ part, const i32x4* __restrict__ tiles,
                                                         O* __restrict__ D, int bs_c, int splits, int n_tiles)
{
    constexpr int NQ = V == 32 ? 4 : 1;
    const int lane = threadIdx.x & 63;
    const int unit = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (tile, group of 4 results)
    if (unit >= n_tiles * NQ) return;
    const int t = unit / NQ, g = unit - t * NQ;
    const f32x4* __restrict__ p = reinterpret_cast<const f32x4*>(part) + (size_t)unit * 64 + lane;
    const size_t step = (size_t)n_tiles * NQ * 64;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < splits; s += 8) {             // eight loads in flight; past the last split the last one again
        f32x4 x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = p[(size_t)min(s + j, splits - 1) * step];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s + j < splits) v += x[j];
    }
    if (O* dst = tile4<O, V>(D, tiles[t], bs_c, lane % V, 8 * g + 4 * (lane / V))) store4<O>(dst, v.x, v.y, v.z, v.w);
}

// Splits of the rows for m rows: as many as give every CU one workgroup, each at least 4 steps (128 rows) long; at
// most 16, beyond which adding up takes longer than is saved (32 where all blocks together are 256 KiB or less).
int sddmm_slab_splits(const bsr_matrix* W, int64_t m)
{
    const int64_t steps = (m + kRows - 1) / kRows;
    const int most = W->nnzb * W->bs_r * W->bs_c <= 65536 ? 32 : 16;
    return (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)W->n_cu / std::max(W->sl.groups, 1), steps / 4, (int64_t)most}));
}

// Workgroups a group's chunks are shared out over where the rows are not split: as many as there are CUs to spare (each
// reads all of the group's slabs; fp32 16x16, 6852 x (4800, 832), 10 %: 150 us, 242 with one for every 8 chunks).
int sddmm_slab_parts(const bsr_matrix* W)
{
    return std::max(1, std::min(W->sl.most_chunks, W->n_cu / std::max(W->sl.groups, 1)));
}

template <typename T, typename O, int V, int CR, int CC, int NCH>
bsr_status launch_shape(const bsr_matrix* W, int m, const void* G, const void* X, void* D, void* ws, size_t ws_bytes, hipStream_t stream)
{
    constexpr bsr_dtype d_dtype = std::is_same<O, float>::value ? BSR_F32 : BSR_F16;   // or BSR_BF16: 16 bits
    int splits = sddmm_slab_splits(W, m);
    const bool split = splits > 1 && ws && ws_bytes >= (size_t)splits * W->sl.n_tiles * V * V * sizeof(float);
    if (!split) splits = sddmm_slab_parts(W);
    // Four chains at least for a result in fp32, as a workgroup per block keeps (root mean square error of fp32
    // 8192 x (4096, 4096): 8.1e-7, 1.62e-6 with one); rounding to 16 bits hides the difference.
    const int chains = split ? splits : 1, steps = (m + kRows - 1) / kRows;
    const int pieces = d_dtype == BSR_F32 ? std::max(1, std::min((4 + chains - 1) / chains, steps / chains)) : 1;
    const int64_t jobs = (int64_t)W->sl.groups * splits;
    const int grid = (int)((jobs + kXcds - 1) / kXcds * kXcds);
    const size_t lds = (size_t)W->sl.lds;
    const i32x4* chunks = reinterpret_cast<const i32x4*>(W->sl_base + W->sl.chunks_at);
    const i32x4* tiles = reinterpret_cast<const i32x4*>(W->sl_base + W->sl.tiles_at);
    auto go = [&](auto split_tag) -> bsr_status {
        constexpr bool SPLIT = decltype(split_tag)::value;
        static const hipError_t attr =
            hipFuncSetAttribute(reinterpret_cast<const void*>(&bsr_sddmm_slab<T, O, V, CR, CC, NCH, SPLIT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (attr != hipSuccess) return BSR_ERR_HIP;
        hipLaunchKernelGGL((bsr_sddmm_slab<T, O, V, CR, CC, NCH, SPLIT>), dim3((unsigned)grid), dim3(64 * (kWaves + kLoaders)), lds, stream,
                           (const T*)G, (const T*)X, W->sl_base, chunks, tiles, (O*)D, (float*)ws, m, (int)W->k, (int)W->n,
                           W->bs_c, W->sl.groups, splits, W->sl.n_tiles, pieces);
        return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
    };
    if (!split) return go(std::false_type{});
    const bsr_status st = go(std::true_type{});
    if (st != BSR_OK) return st;
    constexpr int NQ = V == 32 ? 4 : 1;
    const int64_t units = (int64_t)W->sl.n_tiles * NQ;
    hipLaunchKernelGGL((bsr_sddmm_slab_sum<O, V>), dim3((unsigned)((units + 3) / 4)), dim3(256), 0, stream, (const float*)ws,
                       tiles, (O*)D, W->bs_c, splits, W->sl.n_tiles);
    return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
}

template <typename T, typename O>
bsr_status launch_types(const bsr_matrix* W, int m, const void* G, const void* X, void* D, void* ws, size_t ws_bytes, hipStream_t stream)
{
    const slab_shape sh = slab_shape_of(W->bs_r, W->bs_c);
    if (sh.CR == 2) return launch_shape<T, O, 32, 2, 2, 1>(W, m, G, X, D, ws, ws_bytes, stream);
    if (sh.V == 32) return launch_shape<T, O, 32, 1, 2, 3>(W, m, G, X, D, ws, ws_bytes, stream);
    return launch_shape<T, O, 16, 1, 4, 5>(W, m, G, X, D, ws, ws_bytes, stream);
}

bool slab_block_shape(int bs_r, int bs_c)
{
    auto ok = [](int b) { return b == 8 || b == 16 || b == 32 || b == 64; };
    return ok(bs_r) && ok(bs_c);
}

int slab_tiles_per_block(int bs_r, int bs_c)
{
    const slab_shape sh = slab_shape_of(bs_r, bs_c);
    return std::max(1, bs_r / sh.V) * std::max(1, bs_c / sh.V);
}

}  // namespace

size_t sddmm_slab_plan_words(int64_t k, int32_t bs_r, int32_t bs_c, int64_t nnzb)
{
    if (!slab_block_shape(bs_r, bs_c) || nnzb == 0) return 0;
    // per tile at most a chunk and its output record; per group a header: a group has at least two chunks, or is
    // the last of its range of columns (a range is at least one slab)
    const size_t tiles = (size_t)nnzb * slab_tiles_per_block(bs_r, bs_c);
    return (tiles * 8 + kHdr * (tiles / 2 + (size_t)k / 32 + 2) + 63) & ~(size_t)63;
}

bool sddmm_slab_supports(const bsr_matrix* W, int64_t m)
{
    // byte offsets of 32 rows are 32-bit, with room to spare
    return W->sl_words > 0 && std::max(W->n, W->k) < (1 << 23) && m > 0;
}

size_t sddmm_slab_workspace(const bsr_matrix* W, int64_t m)
{
    const int splits = sddmm_slab_splits(W, m);
    const int V = slab_shape_of(W->bs_r, W->bs_c).V;
    return splits > 1 ? (size_t)splits * W->sl.n_tiles * V * V * sizeof(float) : 0;
}

// Estimated time in microseconds (from 250 shapes, to 30 % where it matters): per 32 rows and workgroup 0.4 for the slabs,
// or what the matrix cores take for the chunks of a SIMD, fp32 0.43, 0.85 and 1.7 a chunk of four 16 x 16, two and four
// 32 x 32 tiles, 16-bit 0.03; the partial results written and read again at 6 TB/s in a second launch.
double sddmm_slab_us(const bsr_matrix* W, int64_t m, bool split)
{
    const slab_shape sh = slab_shape_of(W->bs_r, W->bs_c);
    const int splits = split ? sddmm_slab_splits(W, m) : 1, parts = splits > 1 ? 1 : sddmm_slab_parts(W);
    const double chunk = sh.V == 16 ? 0.43 : sh.CR == 2 ? 1.7 : 0.85;
    auto step = [&](double per_simd) { return W->dtype == BSR_F32 ? std::max(0.4, 0.1 + per_simd * chunk) : 0.4 + 0.03 * (per_simd - 1); };
    const int64_t jobs = (int64_t)W->sl.groups * splits * parts, turns = (jobs + W->n_cu - 1) / W->n_cu;
    const double most = std::ceil(std::ceil((double)W->sl.most_chunks / parts) / 4);
    const double mean = std::ceil((double)(W->sl.tiles_at - W->sl.chunks_at) / 4 / W->sl.groups / parts / 4);
    const int64_t steps = ((m + kRows - 1) / kRows + splits - 1) / splits;
    const double us = (double)steps * std::max(step(most), (double)turns * step(mean));   // the fullest group, or all in turn
    const double pass = (double)W->nnzb * W->bs_r * W->bs_c * 8 / 6e6;   // all results written and read again
    return 4.0 + us + (splits > 1 ? 4.0 + splits * pass : W->dtype == BSR_F32 ? 3 * pass : 0.0);   // whole rows: in four pieces
}

bsr_status launch_sddmm_slab(const bsr_matrix* W, int m, const void* G, const void* X, void* D, bsr_dtype d_dtype, void* ws,
                             size_t ws_bytes, hipStream_t stream)
{
    {
        std::lock_guard<std::mutex> lock(W->sl_mu);
        if (!W->sl.sent) {
            if (hipMemcpyAsync(W->sl_base, W->sl.host.data(), W->sl.host.size() * sizeof(int32_t), hipMemcpyHostToDevice, stream) != hipSuccess)
                return BSR_ERR_HIP;
            // A copy recorded into a graph runs when the graph does, perhaps never: it serves that graph's products only,
            // and the next product outside sends the plan itself.
            hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone) {
                if (hipEventCreateWithFlags(&W->sl.uploaded, hipEventDisableTiming) != hipSuccess) W->sl.uploaded = nullptr;
                if (W->sl.uploaded) (void)hipEventRecord(W->sl.uploaded, stream);
                W->sl.sent = true;
            }
            (void)hipGetLastError();
        } else {
            order_after_upload(stream, W->sl.uploaded, W->sl.landed);
        }
        const bsr_status dbg = debug_check_words(W, W->sl_base, W->sl.host, stream);   // its tile records are store offsets
        if (dbg != BSR_OK) return dbg;
    }
    if (W->dtype == BSR_F32) return launch_types<float, float>(W, m, G, X, D, ws, ws_bytes, stream);
    if (W->dtype == BSR_F16)
        return d_dtype == BSR_F32 ? launch_types<f16_t, float>(W, m, G, X, D, ws, ws_bytes, stream)
                                  : launch_types<f16_t, f16_t>(W, m, G, X, D, ws, ws_bytes, stream);
    return d_dtype == BSR_F32 ? launch_types<bf16_t, float>(W, m, G, X, D, ws, ws_bytes, stream)
                              : launch_types<bf16_t, bf16_t>(W, m, G, X, D, ws, ws_bytes, stream);
}

void build_sddmm_slab_plan(const bsr_matrix* W)
{
    if (W->sl.built) return;
    const int bs_r = W->bs_r, bs_c = W->bs_c;
    const int32_t *indptr = W->sl_indptr.data(), *indices = W->sl_indices.data();
    const slab_shape sh = slab_shape_of(bs_r, bs_c);
    const int V = sh.V, H = V / 2, line = 128 / (W->dtype == BSR_F32 ? 4 : 2), vpl = line / V, CC = sh.CC, CR = sh.CR;
    const int block = bs_r * bs_c;
    const int s_bytes = W->dtype == BSR_F32 ? 4 : 2;
    // rows and columns of "units": tiles, or (CR = 2) blocks of 2 x 2 tiles
    const int ur = CR * V, uc = CR == 2 ? CC * V : V;
    const int64_t UR = (W->n + ur - 1) / ur;

    // ---- columns in ranges of xs slabs: a group has G slabs x X slabs = the blocks it holds / their density, and
    // reads fewest bytes when the two are equal ----
    const int64_t GS = (W->n + line - 1) / line, XS = (W->k + line - 1) / line;
    const int per_unit = CR == 2 ? 1 : CC;            // tiles (CR = 2: blocks) a chunk can hold
    const double tiles_est = (double)W->nnzb * (CR == 2 ? 1 : slab_tiles_per_block(bs_r, bs_c)) *
                             (bs_r < V ? 0.7 : 1.0) * (bs_c < V ? 0.7 : 1.0);
    const double chunks_est = tiles_est / per_unit * 1.25;
    const double density = std::max(1e-9, chunks_est / ((double)GS * XS));   // chunks per pair of slabs
    // rounds of chunks per wavefront: enough that there are at most about 64 groups, so that a few splits of the rows
    // fill the chip
    const int rounds = std::max(1, std::min(sh.NCH, (int)std::ceil(chunks_est / (64.0 * kWaves))));
    const int cap = kWaves * rounds;
    // whole blocks of a slab's width: 10 slabs for 8 blocks (a fourth buffer, and less spread between the groups that
    // share rows in an XCD's L2: 110 against 123 us on the 8192^3 power-law workload)
    const int max_per_group = CR == 2 ? 10 : kMaxSlabs;
    int xs = (int)std::lround(std::sqrt(cap / density));
    xs = std::max(1, std::min({xs, kMaxSlabs / 2 + 2, (int)XS}));
    const int n_ranges = (int)((XS + xs - 1) / xs);
    xs = (int)((XS + n_ranges - 1) / n_ranges);

    struct unit { int32_t col; int32_t off[4]; };     // unit column; element offsets of its quadrants in D (CR = 2: off[0] of the block)
    std::vector<unit> row;                            // the units of one unit row
    struct chunk { int32_t range, urow, n, first; };  // n units from `first` in `units`
    std::vector<unit> units;
    units.reserve((size_t)W->nnzb);
    std::vector<chunk> list;
    list.reserve((size_t)W->nnzb / 2 + 16);
    const int sub_r = std::max(1, V / bs_r), sub_c = std::max(1, V / bs_c);   // blocks per tile side (8-wide blocks: 2)
    // rows whose slab of G is theirs alone may come in any order: longest first, as the plan's slots
    const bool free_order = vpl == 1 || CR == 2;
    const int blocks_per_urow_r = std::max(1, ur / bs_r), urows_per_block = std::max(1, bs_r / ur);
    for (int64_t o = 0; o < UR; ++o) {
        int64_t v = o;
        if (free_order && urows_per_block >= 1 && blocks_per_urow_r == 1)
            v = (int64_t)W->staging[(size_t)(o / urows_per_block)] * urows_per_block + o % urows_per_block;
        row.clear();
        bool sorted = true;
        for (int b = 0; b < blocks_per_urow_r; ++b) {
            const int64_t r = urows_per_block > 1 ? v / urows_per_block : v * blocks_per_urow_r + b;
            if (r >= W->R) break;
            const int a0 = urows_per_block > 1 ? (int)(v % urows_per_block) * ur : 0;   // unit's first row inside the block
            for (int32_t p = indptr[r]; p < indptr[r + 1]; ++p) {
                const int32_t e = p * block + a0 * bs_c;
                if (CR == 2) {
                    row.push_back(unit{indices[p], {p * block, 0, 0, 0}});
                } else if (sub_c > 1 || sub_r > 1) {
                    // 8-wide in at least one direction: the tile's quadrants are 8 x 8
                    for (int w = 0; w < std::max(1, bs_c / V); ++w) {
                        const int32_t col = sub_c > 1 ? indices[p] / sub_c : indices[p] * std::max(1, bs_c / V) + w;
                        unit u{col, {-1, -1, -1, -1}};
                        for (int qa = 0; qa < 2; ++qa)
                            for (int qc = 0; qc < 2; ++qc) {
                                const bool mine_r = sub_r > 1 ? qa == b : true, mine_c = sub_c > 1 ? qc == indices[p] % sub_c : true;
                                if (mine_r && mine_c)
                                    u.off[2 * qa + qc] = e + (sub_r > 1 ? 0 : qa * H) * bs_c + (sub_c > 1 ? 0 : w * V + qc * H);
                            }
                        row.push_back(u);
                    }
                } else {
                    for (int w = 0; w < bs_c / V; ++w) {
                        const int32_t b0 = e + w * V;
                        row.push_back(unit{indices[p] * (bs_c / V) + w, {b0, b0 + H, b0 + H * bs_c, b0 + H * bs_c + H}});
                    }
                }
                if (row.size() > 1 && row[row.size() - 1].col < row[row.size() - 2].col) sorted = false;
            }
            if (sub_r > 1) sorted = false;            // two block-rows interleave
        }
        if (!sorted) std::stable_sort(row.begin(), row.end(), [](const unit& x, const unit& y) { return x.col < y.col; });
        if (CR == 1 && (sub_c > 1 || sub_r > 1)) {    // merge the blocks of a tile; a position taken twice opens another
            size_t w = 0;
            for (size_t i = 0; i < row.size(); ++i) {
                bool merged = false;
                for (size_t z = w; z-- > 0 && row[z].col == row[i].col;) {
                    bool clash = false;
                    for (int q = 0; q < 4; ++q) clash |= row[z].off[q] >= 0 && row[i].off[q] >= 0;
                    if (clash) continue;
                    for (int q = 0; q < 4; ++q)
                        if (row[i].off[q] >= 0) row[z].off[q] = row[i].off[q];
                    merged = true;
                    break;
                }
                if (!merged) row[w++] = row[i];
            }
            row.resize(w);
        }
        // cut into ranges of columns, and those into chunks
        for (size_t i = 0; i < row.size();) {
            const int32_t range = (int32_t)((int64_t)row[i].col * uc / line / xs);
            size_t j = i;
            while (j < row.size() && (int32_t)((int64_t)row[j].col * uc / line / xs) == range) ++j;
            for (; i < j;) {
                const int32_t take = (int32_t)std::min<size_t>(j - i, CR == 2 ? 1 : CC);
                list.push_back(chunk{range, (int32_t)v, take, (int32_t)units.size()});
                for (int32_t z = 0; z < take; ++z) units.push_back(row[i++]);
            }
        }
    }
    // ---- chunks range by range (stable counting sort), then packed into groups ----
    std::vector<int32_t> at((size_t)n_ranges + 1, 0), order(list.size());
    for (const chunk& c : list) ++at[(size_t)c.range + 1];
    for (int i = 0; i < n_ranges; ++i) at[(size_t)i + 1] += at[(size_t)i];
    for (size_t i = 0; i < list.size(); ++i) order[(size_t)at[(size_t)list[i].range]++] = (int32_t)i;

    std::vector<int32_t> hdr, recs, tiles;
    hdr.reserve(list.size() / 4 * kHdr + kHdr);
    recs.reserve(list.size() * 4);
    tiles.reserve(units.size() * 4);
    std::vector<int32_t> g_at((size_t)GS, -1), x_at((size_t)XS, -1), g_stamp((size_t)GS, -1), x_stamp((size_t)XS, -1);
    std::vector<int32_t> gl, xl;
    size_t i = 0;
    int32_t group = 0, lds = 0, most_chunks = 0;
    while (i < order.size()) {
        gl.clear();
        xl.clear();
        const size_t first = i;
        const int32_t range = list[(size_t)order[i]].range;
        for (; i < order.size() && i - first < (size_t)cap; ++i) {
            const chunk& c = list[(size_t)order[i]];
            if (c.range != range) break;
            const size_t g0 = gl.size(), x0 = xl.size();
            auto want = [&](std::vector<int32_t>& l, std::vector<int32_t>& where, std::vector<int32_t>& stamp, int32_t slab) {
                if (stamp[(size_t)slab] == group) return;
                stamp[(size_t)slab] = group;
                where[(size_t)slab] = (int32_t)l.size();
                l.push_back(slab);
            };
            want(gl, g_at, g_stamp, (int32_t)((int64_t)c.urow * ur / line));
            if (ur > line) want(gl, g_at, g_stamp, (int32_t)((int64_t)c.urow * ur / line) + 1);
            for (int32_t z = 0; z < c.n; ++z) {
                want(xl, x_at, x_stamp, (int32_t)((int64_t)units[(size_t)(c.first + z)].col * uc / line));
                if (uc > line) want(xl, x_at, x_stamp, (int32_t)((int64_t)units[(size_t)(c.first + z)].col * uc / line) + 1);
            }
            if (gl.size() + xl.size() > (size_t)max_per_group) {          // does not fit: the next group starts with it
                while (gl.size() > g0) { g_stamp[(size_t)gl.back()] = -1; gl.pop_back(); }
                while (xl.size() > x0) { x_stamp[(size_t)xl.back()] = -1; xl.pop_back(); }
                break;
            }
        }
        const int32_t ng = (int32_t)gl.size(), ns = ng + (int32_t)xl.size();
        lds = std::max(lds, slab_buffers(ns) * ns * kSlab);
        most_chunks = std::max(most_chunks, (int32_t)(i - first));
        int32_t h[kHdr] = {ns, ng, (int32_t)(recs.size() / 4), (int32_t)(i - first)};
        for (int32_t z = 0; z < ns; ++z) h[kHdrSlabsAt + z] = (z < ng ? gl[(size_t)z] : xl[(size_t)(z - ng)]) * line;
        hdr.insert(hdr.end(), h, h + kHdr);
        for (size_t q = first; q < i; ++q) {
            const chunk& c = list[(size_t)order[q]];
            const int32_t t0 = (int32_t)(tiles.size() / 4);
            auto place = [&](const std::vector<int32_t>& where, int32_t base, int64_t col) -> uint32_t {   // column -> byte offset in a buffer
                return (uint32_t)(base + where[(size_t)(col / line)]) * kSlab + (uint32_t)(col % line) * s_bytes;
            };
            uint32_t a[2] = {0, 0}, b[4] = {0, 0, 0, 0};
            if (CR == 2) {
                const unit& u = units[(size_t)c.first];
                for (int z = 0; z < 2; ++z) {
                    a[z] = place(g_at, 0, (int64_t)c.urow * ur + z * V);
                    b[z] = place(x_at, ng, (int64_t)u.col * uc + z * V);
                }
                for (int z = 0; z < 4; ++z) {
                    const int32_t e = u.off[0] + (z / 2) * V * bs_c + (z % 2) * V;
                    const int32_t o4[4] = {e, e + H, e + H * bs_c, e + H * bs_c + H};
                    tiles.insert(tiles.end(), o4, o4 + 4);
                }
            } else {
                a[0] = place(g_at, 0, (int64_t)c.urow * ur);
                for (int z = 0; z < CC; ++z) {
                    const unit& u = units[(size_t)(c.first + std::min(z, c.n - 1))];
                    b[z] = place(x_at, ng, (int64_t)u.col * uc);
                    if (z < c.n) tiles.insert(tiles.end(), u.off, u.off + 4);
                }
            }
            const int32_t live = CR == 2 ? 4 : c.n;
            const uint32_t rec[4] = {a[0] | a[1] << 16, b[0] | b[1] << 16, b[2] | b[3] << 16, (uint32_t)t0 | (uint32_t)live << 28};
            for (uint32_t w : rec) recs.push_back((int32_t)w);
        }
        ++group;
    }
    bsr_matrix::slab_plan& plan = W->sl;
    plan.chunks_at = hdr.size();
    plan.tiles_at = plan.chunks_at + recs.size();
    plan.host = std::move(hdr);
    plan.host.reserve(plan.tiles_at + tiles.size());
    plan.host.insert(plan.host.end(), recs.begin(), recs.end());
    plan.host.insert(plan.host.end(), tiles.begin(), tiles.end());
    plan.groups = group;
    plan.most_chunks = most_chunks;
    plan.lds = lds;
    plan.n_tiles = (int32_t)(tiles.size() / 4);
    plan.built = true;                                // not before: whatever throws leaves it to be built again
}

bool sddmm_slab_ready(const bsr_matrix* W)
{
    std::lock_guard<std::mutex> lock(W->sl_mu);
    try {
        build_sddmm_slab_plan(W);
    } catch (const std::bad_alloc&) {                 // no memory for the plan: the caller takes a kernel that needs none
        return false;
    }
    return W->sl.host.size() <= W->sl_words;
}
