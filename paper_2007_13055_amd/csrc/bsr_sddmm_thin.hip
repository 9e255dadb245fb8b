// The sampled product for thin blocks (16 x 1, fp32) whose block-rows are stored in block-column order:
//     D[p][a] = sum over i of G[i][16 r + a] * X[i][column of p]
// without a transposed copy of X.
//
// A workgroup takes 16 slots (block-rows) x a range of 256 columns of X and walks the rows i, 32 at a time: it turns
// the 32 x 256 piece of X and the 32 x 16 pieces of G of its slots over on the way into LDS -- a thread loads a 4 x 4
// unit, 16 bytes of each of 4 rows, and writes it as 4 x 16 bytes of 4 columns -- so that a column is 128 contiguous
// bytes there and a matrix-core operand of either side is one 16-byte read: lane (index, k-group g) takes rows
// 16 s + 4 g .. + 3, the four v_mfma_f32_16x16x4_f32 of 16 rows reduce over row 16 s + 4 g + u.  Wavefront w multiplies
// slot w: its stored blocks of the range, 16 to a chunk (M = a, N = block), whose LDS addresses are the same for
// all rows and stay in registers, as do the results.  Two buffers, one barrier per 32 rows.
//
// What bounds it: per 32 rows and workgroup 64 KiB from L2 and the last-level cache (1 us at 2864 x (4672, 3840)), about
// as much matrix-core time (chunks that a run leaves partly empty included) and 0.6 us of LDS traffic; 1.4 us together.
// On 3394 x (544, 2880), 27 us, the matrix cores are busy 18 %, the LDS 29 % of the time (conflicts 12 of these) and the
// wavefronts wait for X and G for 45 %.  Times: other_us() below.
//
// LDS bank conflicts.  A column's line is at index col ^ (bit 2 of col) and its eight 16-byte pieces are XORed by bits
// 2-4 of col: 16 neighbouring lanes of a write (two pieces of 8 columns 4 apart) then fall on 16 different pieces of 256
// bytes, and 16 lanes of a read (one piece of 16 arbitrary columns) on pieces spread at random.  With the pieces XORed by one bit
// only, 256 x (4096, 4096) took 23.8 us instead of 17 and 2864 x (4672, 3840) 425 instead of 266.
//
// Few workgroups and many rows: the rows are split, the partial results go to the caller's workspace and are added
// in split order by a second kernel.
#include <algorithm>
#include <cmath>

#include "bsr_mfma_common.h"

using namespace bsr_dev;

namespace {

constexpr int kSlots = 16;                            // per workgroup: a wavefront each
constexpr int kThreads = 64 * kSlots;
constexpr int kTile = 32;                             // rows of G and X per step
constexpr int kXCols = kThinRange;                    // columns of X per workgroup
constexpr int kLine = kTile * 4;                      // bytes of a column of a step in LDS
constexpr int kXBuf = kXCols * kLine, kGBuf = kSlots * 16 * kLine;   // 32 KiB each
constexpr int kLds = 2 * (kXBuf + kGBuf);
constexpr int kXcds = 8;
static_assert(kXCols / 4 * (kTile / 4) + kSlots * 4 * (kTile / 4) == kThreads, "a unit of 4 x 4 per thread and step");

__device__ __forceinline__ unsigned line_of(unsigned col) { return (col ^ ((col >> 2) & 1u)) * kLine; }
__device__ __forceinline__ unsigned swz_of(unsigned col) { return ((col >> 2) & 7u) << 4; }   // XOR of the byte in the line

template <int NCH, bool SPLIT>
__global__ __launch_bounds__(kThreads) void bsr_sddmm_thin_rows(const float* __restrict__ G, const float* __restrict__ X,
                                                                const int32_t* __restrict__ indices,
                                                                const int32_t* __restrict__ row_desc,
                                                                const int32_t* __restrict__ pos, int pos_stride,
                                                                float* __restrict__ D, int m, int k, int n, int R,
                                                                int n_sets, int n_ranges, int group_sets, int splits,
                                                                int nnzb)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];   // [2][X columns | slots' columns of G]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // workgroup b runs on XCD b mod 8, and the 32 of an XCD at a time are about group_sets sets x as many ranges: its L2
    // then serves most of both sides (2864 x (4672, 3840): 258 us with all sets of a range after each other, 175)
    const int per_xcd = (int)gridDim.x / kXcds;
    const int job = (int)(blockIdx.x % (unsigned)kXcds) * per_xcd + (int)(blockIdx.x / (unsigned)kXcds);
    if (job >= n_sets * n_ranges * splits) return;    // whole workgroup: the grid is rounded up to 8
    const int split = job / (n_sets * n_ranges), j0 = job % (n_sets * n_ranges);
    const int group = j0 / (group_sets * n_ranges), j1 = j0 % (group_sets * n_ranges);
    const int width = min(group_sets, n_sets - group * group_sets);
    const int range = j1 / width, set = group * group_sets + j1 % width;

    // steps [t0, t1) of 32 rows
    const unsigned n_steps = (unsigned)(m + kTile - 1) / kTile;
    const int t0 = (int)(n_steps * (unsigned)split / (unsigned)splits), t1 = (int)(n_steps * (unsigned)(split + 1) / (unsigned)splits);

    // ---- this thread's unit: rows 4 u .. 4 u + 3 of a step, 4 columns ----
    // threads 0-511: X, 8 row groups x 8 column quads per wavefront (a row's 8 quads are one line of memory);
    // threads 512-1023: G, 8 row groups x 4 quads of 2 slots per wavefront
    const bool is_x = wave < kSlots / 2;
    const int u = (lane >> 3) & 7;
    const float* src;                                 // row 0 of the unit's columns
    unsigned row_floats, dst;
    int col;                                          // first column of the unit: of the range (X), 16 slot + a (G)
    if (is_x) {
        col = (wave * 8 + (lane & 7)) * 4;
        src = X + min(range * kXCols + col, k - 4);   // columns past k: no stored block names them
        row_floats = (unsigned)k;
        dst = 0;
    } else {
        const int s = (wave - kSlots / 2) * 2 + ((lane >> 2) & 1);
        const int slot = min(set * kSlots + s, R - 1);
        col = s * 16 + (lane & 3) * 4;
        src = G + (size_t)row_desc[(size_t)slot * kRowDescWords] * 16 + (lane & 3) * 4;
        row_floats = (unsigned)n;
        dst = kXBuf;
    }
    f32x4 in[4];
    auto fetch = [&](int t) {
        if (t * kTile + kTile <= m) {                 // uniform
            const float* p = src + (size_t)(unsigned)(t * kTile + 4 * u) * row_floats;
#pragma unroll
            for (int j = 0; j < 4; ++j) in[j] = *reinterpret_cast<const f32x4*>(p + (size_t)((unsigned)j * row_floats));
        } else {                                      // rows past m repeat row m - 1 and are zeroed when staged
#pragma unroll
            for (int j = 0; j < 4; ++j) in[j] = *reinterpret_cast<const f32x4*>(src + (size_t)min(t * kTile + 4 * u + j, m - 1) * row_floats);
        }
    };
    auto put = [&](int t, unsigned char* buf) {
        if (t * kTile + kTile > m) {                  // uniform: the last step
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (t * kTile + 4 * u + j >= m) in[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const f32x4 v = {in[0][e], in[1][e], in[2][e], in[3][e]};
            *reinterpret_cast<f32x4*>(buf + dst + line_of(col + e) + ((unsigned)(16 * u) ^ swz_of(col + e))) = v;
        }
    };
    if (t0 < t1) fetch(t0);

    // ---- this wavefront's blocks: the slot's run inside the range, 16 to a chunk ----
    const int lo = lane & 15, g = lane >> 4;
    const int slot = set * kSlots + wave;
    int first = 0, cnt = 0;
    if (slot < R) {                                   // uniform
        first = pos[(size_t)slot * pos_stride + range];
        cnt = pos[(size_t)slot * pos_stride + range + 1] - first;
    }
    unsigned at[NCH];                                 // LDS byte of the lane's first piece (rows 4 g ..) in an X buffer
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        at[c] = 0;
        if (16 * c < cnt) {                           // uniform
            const unsigned rel = (unsigned)(indices[first + min(16 * c + lo, cnt - 1)] - range * kXCols);   // past the run: its last block
            at[c] = line_of(rel) + ((unsigned)(16 * g) ^ swz_of(rel));
        }
    }
    const unsigned ga = kXBuf + line_of(wave * 16 + lo) + ((unsigned)(16 * g) ^ swz_of(wave * 16 + lo));

    // The rows' sums are kept in chains, as many as keep any kernel that this one replaces: four of a quarter of the rows,
    // or two where the rows are split and registers are few (32 chunk registers a chain).  Unsplit and few registers: four short
    // chains a step, added to what there is (16 vector instructions more for 8 of the matrix cores; everywhere that cost
    // 5-10 %: 1491 x (2800, 1712) 34 % 79 to 87 us).
    constexpr bool SHORT = NCH > 4 && !SPLIT;
    constexpr int CH = SHORT ? 1 : NCH > 4 ? 2 : 4;
    f32x4 acc[NCH][CH];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int e = 0; e < CH; ++e) acc[c][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Steps: t is multiplied, t + 1 goes from registers to LDS, t + 2 is fetched into them.  The loads of a step are taken
    // by the memory pipe over about as many clocks as its matrix instructions take, and a wavefront that issues them
    // waits meanwhile: the wavefronts of X do so before their products, those of G after them.
    auto advance = [&](int t) {
        if (t + 1 < t1) put(t + 1, lds + ((t + 1 - t0) & 1) * (kXBuf + kGBuf));
        if (t + 2 < t1) fetch(t + 2);
    };
    if (t0 < t1) {
        put(t0, lds);
        if (t0 + 1 < t1) fetch(t0 + 1);
    }
    for (int t = t0; t < t1; ++t) {
        // step t is in its buffer, step t - 1 is read; loads stay in flight (__syncthreads() waits for them)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (is_x) advance(t);
        const unsigned char* buf = lds + ((t - t0) & 1) * (kXBuf + kGBuf);
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(buf + ga), a1 = *reinterpret_cast<const f32x4*>(buf + (ga ^ 64u));
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            if (16 * c < cnt) {                       // uniform
                const f32x4 b0 = *reinterpret_cast<const f32x4*>(buf + at[c]), b1 = *reinterpret_cast<const f32x4*>(buf + (at[c] ^ 64u));
                if constexpr (SHORT) {
                    f32x4 s[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[e], b0[e], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[e], b1[e], s[e], 0, 0, 0);
                    acc[c][0] += (s[0] + s[1]) + (s[2] + s[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[c][e % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[e], b0[e], acc[c][e % CH], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[c][e % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[e], b1[e], acc[c][e % CH], 0, 0, 0);
                }
            }
        if (!is_x) advance(t);
    }
    // lane (block lo of the chunk, g) holds D[p][4 g .. 4 g + 3]
    float* out = SPLIT ? D + (size_t)split * nnzb * 16 : D;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (16 * c + lo < cnt) {
            f32x4 v = acc[c][0];
            if constexpr (CH == 2) v += acc[c][1];
            if constexpr (CH == 4) v = (v + acc[c][1]) + (acc[c][2] + acc[c][3]);
            *reinterpret_cast<f32x4*>(out + ((size_t)first + 16 * c + lo) * 16 + 4 * g) = v;
        }
}

__global__ __launch_bounds__(256) void bsr_sddmm_thin_sum(const f32x4* __restrict__ part, f32x4* __restrict__ D, int splits, int quads)
{
    const int q = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (q >= quads) return;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < splits; s += 8) {             // eight loads in flight; past the last split the last one again
        f32x4 x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = part[(size_t)min(s + j, splits - 1) * quads + q];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s + j < splits) v += x[j];
    }
    D[q] = v;
}

// Time of this kernel in microseconds, and the split of the rows at which it is least (to 10 % over the shapes of
// other_us(), 7 to 175 us): start and end 6; a step 0.7 and 0.5 for every chunk of blocks, a run's last one
// half full; the partial results written and read again at 6 TB/s in a second launch of 2.5.
struct thin_plan { double us; int splits; };
thin_plan plan_of(const bsr_matrix* W, int64_t m, int most_splits = 16)
{
    const int64_t ranges = W->thin_pos_stride - 1, jobs = (int64_t)((W->R + kSlots - 1) / kSlots) * ranges, steps = (m + kTile - 1) / kTile;
    const double step = 0.7 + 0.5 * ((double)W->nnzb / ((double)W->R * ranges) + 8) / 16, sum = (double)W->nnzb * 128 / 6e6;
    thin_plan best = {1e30, 1};
    for (int s = 1; s <= most_splits && (s == 1 || s <= steps); ++s) {
        const double t = 6 + (double)((jobs * s + W->n_cu - 1) / W->n_cu) * (1.0 + (double)((steps + s - 1) / s) * step) + (s > 1 ? 2.5 + s * sum : 0);
        if (t < best.us) best = {t, s};
    }
    return best;
}

// The kernels of bsr_sddmm.hip, one of which runs instead.
// With scratch lent and 32 rows or more: X^T into the scratch (4 TB/s) and a wavefront or two per slot over all rows,
// 0.0115 us each where there are few slots, 1.4 million blocks times rows a microsecond where there are many, 13000
// blocks where there are few rows.  Times of that way and of this, us:
//     256 x (4096, 4096) 5 %       14.1   16.9      2864 x (4672, 3840) 5.7 %   163   175     264 x (3968, 256)    9.7  12.7
//     3394 x (544, 2880) 4.3 %     65.2   27.3      4504 x (2560, 256)  8.2 %    62    23     1546 x (1632, 1152) 41.2  34.5
// Else a lane per block and column: a workgroup's start (200 a microsecond), and per row 0.035 or what the lines of X take
// that the block-rows touch, 160000 a microsecond while X is 8 MB or less, 90000 beyond.  That way, this and this unsplit:
//     6 x (4352, 3264) 10 %        10.5    6.8   6.8     8 x (8080, 2256) 2.3 %   5.0   8.4  8.6    31 x (2048, 4096) 10 %   9.2   6.3   6.3
//     3394 x (544, 2880) 4.3 %      149     29   139     7078 x (320, 304) 27 %   248    52  716    256 x (4096, 4096) 5 %  36.8  17.8  17.7
double other_us(const bsr_matrix* W, int64_t m)
{
    const double rows = (double)m, blocks = (double)W->nnzb;
    if (sddmm_transposes(W, m))
        return 5 + 8 * rows * (double)W->k / 4e6 + std::max({0.0115 * rows, rows * blocks / 1.4e6, blocks / 13000});
    const double lines = std::ceil((double)W->k / 32), touched = W->R * lines * (1 - std::exp(-blocks / ((double)W->R * lines)));
    const double rate = rows * (double)W->k * 4 <= 8e6 ? 160e3 : 90e3;
    return 3.5 + (blocks / 64 + 0.5 * W->R) / 200 + rows * std::max(0.035, touched / rate);
}

}  // namespace

bool sddmm_transposes(const bsr_matrix* W, int64_t m)
{
    return mfma_thin_supports(W) && m >= 32 && W->scratch && W->scratch_bytes >= mfma_thin_scratch_bytes(W, m) &&
           (m + 3) * W->k < ((int64_t)1 << 30);
}

// The longest run of a (block-row, range) has to fit the accumulators, 8 chunks of 16 blocks; and this kernel has to be
// the quicker one, as estimated, with the splits that the memory allows.
bool sddmm_thin_supports(const bsr_matrix* W, int64_t m, size_t workspace_bytes)
{
    if (W->thin_pos == nullptr || W->thin_max_range > 128 || m <= 0 || W->nnzb >= (1 << 26)) return false;
    if (W->env_tune.sd) return W->env_tune.sd == 2;
    const bool room = workspace_bytes >= sddmm_thin_workspace(W, m);
    return plan_of(W, m, room ? 16 : 1).us < 0.95 * other_us(W, m);
}

size_t sddmm_thin_workspace(const bsr_matrix* W, int64_t m)
{
    const int splits = plan_of(W, m).splits;
    return splits > 1 ? (size_t)splits * W->nnzb * 16 * sizeof(float) : 0;
}

bsr_status launch_sddmm_thin(const bsr_matrix* W, int m, const void* G, const void* X, void* D, void* ws, size_t ws_bytes, hipStream_t stream)
{
    int splits = plan_of(W, m).splits;
    if (splits > 1 && (!ws || ws_bytes < sddmm_thin_workspace(W, m))) splits = 1;
    const int n_sets = (W->R + kSlots - 1) / kSlots, n_ranges = W->thin_pos_stride - 1;
    const int groups = (n_sets + 5) / 6, group_sets = (n_sets + groups - 1) / groups;
    const int64_t jobs = (int64_t)n_sets * n_ranges * splits;
    if (jobs >= ((int64_t)1 << 30)) return BSR_ERR_SHAPE;
    auto go = [&](auto chunks_tag, auto split_tag) -> bsr_status {
        constexpr int NCH = decltype(chunks_tag)::value;
        constexpr bool SPLIT = decltype(split_tag)::value;
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bsr_sddmm_thin_rows<NCH, SPLIT>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (attr != hipSuccess) return BSR_ERR_HIP;
        hipLaunchKernelGGL((bsr_sddmm_thin_rows<NCH, SPLIT>), dim3((unsigned)((jobs + kXcds - 1) / kXcds * kXcds)), dim3(kThreads),
                           kLds, stream, (const float*)G, (const float*)X, W->indices, W->row_desc, W->thin_pos,
                           W->thin_pos_stride, SPLIT ? (float*)ws : (float*)D, m, (int)W->k, (int)W->n, W->R, n_sets, n_ranges,
                           group_sets, splits, (int)W->nnzb);
        return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
    };
    auto with = [&](auto split_tag) -> bsr_status {
        if (W->thin_max_range <= 32) return go(std::integral_constant<int, 2>{}, split_tag);
        if (W->thin_max_range <= 64) return go(std::integral_constant<int, 4>{}, split_tag);
        return go(std::integral_constant<int, 8>{}, split_tag);
    };
    if (splits == 1) return with(std::false_type{});
    const bsr_status st = with(std::true_type{});
    if (st != BSR_OK) return st;
    const int quads = (int)W->nnzb * 4;
    hipLaunchKernelGGL(bsr_sddmm_thin_sum, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, stream, (const f32x4*)ws, (f32x4*)D,
                       splits, quads);
    return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
}
