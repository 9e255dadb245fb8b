// Matrix-core kernel for blocks with sides 8 or 16 (both 16: 16-bit types only), swept over the columns of X.
//
// A stored 8x8 block touches 16 bytes of a row of X, so a kernel that fetches X block by block moves whole lines for a
// fraction of them, once per 16 outputs.  Here a workgroup takes TM = 16 * SUB rows of X and a few QUADS (64 outputs, four
// groups of 16 rows of W each).  It sweeps over the columns in WINDOWS of kSlabs * 128 bytes per row: the rows of X come in
// once, in whole lines, and stay in LDS while all of the workgroup's stored blocks of the window are multiplied; the sums
// stay in registers from the first window to the last.
//
//   granule  16 bytes of a row of X (8 16-bit or 4 fp32 columns), what a lane feeds to an MFMA step
//   entry    one group of 16 rows of W times four granules, anywhere in the window: one v_mfma_f32_16x16x32 (fp32: four
//            16x16x4) per 16 rows of X.  Blocks of 8 rows come two block-rows to an entry: of the 16 x 4 granules 55 % hold
//            stored values at 20 % density, where 16x16 tiles of W hold 34 %.
//   round    an entry for each of a quad's four groups.  Its record holds, for each granule and (blocks of 8 rows) half of
//            the 16 rows, {byte offset of the values in block_data, place of the granule in the window}; what is not stored
//            has an offset past the end of W (read as zeros), a granule that is not there the place of a granule of zeros.
//            A group that has fewer entries in a window than the others multiplies zeros (fp32: is left out).
//   list     a quad's rounds by window: one run of records from end to end, so that records are read two rounds and values
//            one round ahead whatever the windows hold.
//
// Twelve wavefronts: eight multiply, each a quad or every KS-th round of one (the shares are added in fixed order at the
// end), four only move X into a ring of two windows (loads that write LDS directly, one barrier per window).
//
// What bounds it: no unit by itself.  Counters, as shares of the kernel's clocks (bf16 8x8, 5889 x (1216, 5184), 21.8 %): LDS
// busy 42 (12 of them bank conflicts: an entry's four granules lie anywhere), matrix cores 26, and a wavefront issues in 20
// of 100 of its clocks; two multiplying wavefronts a SIMD do not cover the chain of a round (record, values, X, MFMAs) and the
// barrier of a window.  fp32 8x8: LDS 17, matrix cores 26.  bf16 16x16, 3540 x (5184, 1536): 23 and 21, and its 168 workgroups
// leave 88 CUs without one.  Windows of 512 columns take 0.86 of the time of windows of 256; values two rounds ahead, progress
// words polled in LDS in place of the barrier, and twelve multiplying wavefronts gain nothing.
// Measured (us in graph replays, with the kernel that ran before and now): that product 393, 61; fp16 8x8, 2662 x (832, 6528),
// 19.3 % 145, 31; fp16 8x8, 2285 x (6016, 1536), 15.6 %, power law 286, 49; fp32 8x8, 3607 x (320, 5056), 7.3 % 58, 52.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "bsr_mfma_common.h"

using namespace bsr_dev;
using namespace bsr_dev::lds_loads;

namespace {

constexpr int kSlabs = 8;                             // 128-byte slabs of a window
constexpr int kRing = 2;                              // windows in LDS
constexpr int kWaves = 8;                             // wavefronts that multiply
constexpr int kLoaders = 4;                           // wavefronts that move X
constexpr int kMine = kSlabs / kLoaders;              // slabs each of them moves
constexpr int kPitch = kSlabs * 2048 + 128;           // bytes of 16 rows of a window, and behind them the granule of zeros
constexpr int kZeroAt = kSlabs * 2048;
constexpr int kNone = 0xFFFF;                         // place of the granule of zeros
constexpr int kXcds = 8;
constexpr int kRowsOut = 32;                          // rows of Y per pass of the epilogue
constexpr int kLdOut = 64 + 4;                        // floats of a row there

// The 16-byte pieces of row r of a slab are stored XOR turn(r): sixteen rows' pieces of one column fill all banks once
// (measured: 6.4 clocks a read, as contiguous ones; 8.2 with r mod 8, 16 unturned).
__device__ __forceinline__ constexpr unsigned turn(unsigned r) { return (r >> 1) & 7; }
__device__ __forceinline__ void window_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// OWN: outputs that come out as NaN are summed again (below).
template <typename T, typename O, int SUB, bool OWN>
__global__ __launch_bounds__(64 * (kWaves + kLoaders), 3) void bsr_mfma_sweep(
    const T* __restrict__ X, const T* __restrict__ data, unsigned w_bytes, const i32x4* __restrict__ recs,
    const int32_t* __restrict__ win_ptr, const i32x4* __restrict__ quads, O* __restrict__ Y, int m, int k, int n,
    int n_tiles, int tiles_padded, int n_quads, int n_win, int q_log, int bs_r, int row_bytes,
    const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices)
{
    constexpr int S = (int)sizeof(T);
    constexpr int CH = 16 / S;                        // columns of a granule
    constexpr int BUF = SUB * kPitch;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];   // [kRing][SUB][kPitch], then the epilogue's tiles

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // group by group (the longest quads first), the tiles of a group side by side: where the tiles are padded to a
    // multiple of 8, all groups of a tile share an XCD and its L2 copy of the rows
    const int group = (int)(blockIdx.x / (unsigned)tiles_padded), tile = (int)(blockIdx.x % (unsigned)tiles_padded);
    if (tile >= n_tiles) return;                      // whole workgroup
    const int i_base = tile * 16 * SUB;
    const int Q = 1 << q_log, KS = kWaves / Q;

    __shared__ int column[kWaves];                    // first output of each of the workgroup's quads
    __shared__ int not_finite;                        // OWN: some sum may be a NaN
    const int li = lane & 15, h = lane >> 4;
    f32x4 acc[4][SUB];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int s = 0; s < SUB; ++s) acc[j][s] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (wave >= kWaves) {
        const int slab = (wave - kWaves) * kMine;
        const unsigned x_row = (unsigned)k * S;
        const unsigned r8 = (unsigned)lane >> 3;
        unsigned src[2 * SUB];
#pragma unroll
        for (int o = 0; o < 2 * SUB; ++o)
            src[o] = (o * 8 + r8) * x_row + slab * 128 + ((((unsigned)lane & 7) ^ turn(r8 + 8 * (o & 1))) << 4);
        const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)lds + slab * 2048;
        unsigned long long xa = reinterpret_cast<unsigned long long>(X) + (unsigned long long)i_base * x_row;
        long long left = (long long)(m - i_base) * x_row;   // bytes of X from here on
        int windows = n_win;                          // still to issue
        auto issue = [&](unsigned buf) {
            i32x4 r;
            r.x = (int)(unsigned)xa; r.y = (int)((unsigned)(xa >> 32) & 0xFFFFu);
            r.z = windows <= 0 || left <= 0 ? 0 : left > 0x7fffffffll ? 0x7fffffff : (int)left; r.w = 0x00020000;
#pragma unroll
            for (int o = 0; o < 2 * SUB; ++o)
#pragma unroll
                for (int u = 0; u < kMine; ++u)
                    load_to_lds(r, src[o] + u * 128, lds0 + buf * BUF + (o >> 1) * kPitch + (o & 1) * 1024 + u * 2048);
            xa += kSlabs * 128;
            left -= kSlabs * 128;
            --windows;
        };
#pragma unroll
        for (int b = 0; b < kRing - 1; ++b) issue((unsigned)b);
        unsigned buf = 0;
        for (int w = 0; w < n_win; ++w) {
            wait_vm<(kRing - 2) * 2 * SUB * kMine>();         // this wavefront's share of window w has landed
            asm volatile("s_barrier" ::: "memory");   // everybody's has, and everybody has read window w - 1
            issue(buf == 0 ? kRing - 1 : buf - 1);
            buf = buf == kRing - 1 ? 0 : buf + 1;
        }
        wait_vm<0>();                                 // nothing may land in the epilogue's tiles
    } else {
        if (tid < kRing * SUB) *reinterpret_cast<u32x4*>(lds + tid * kPitch + kZeroAt) = u32x4{0u, 0u, 0u, 0u};
        const int slot = (group << q_log) + wave / KS, ks = wave % KS;
        const i32x4 desc = quads[min(slot, n_quads - 1)];   // {quad, first round, end of the rounds, 0}
        const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(data), 0, (int)w_bytes, 0x00020000);
        const int32_t* __restrict__ wq = win_ptr + (size_t)min(slot, n_quads - 1) * (n_win + 1);
        int w = -1;
        const int e_first = desc.y, e_last = slot < n_quads ? desc.z : e_first;
        if (OWN && tid == 0) not_finite = 0;
        if (lane == 0 && ks == 0) column[wave / KS] = slot < n_quads ? desc.x * 64 : n;
        if (e_first + ks < e_last) {
            const unsigned lane_w = (unsigned)((li & (bs_r - 1)) * row_bytes + (h & (row_bytes / 16 - 1)) * 16);
            const unsigned lane_x = (unsigned)(li * 128 + turn(li) * 16);
            const int halves = bs_r == 8 ? 1 : 0;     // log2 of the parts of a granule's record
            const i32x4* __restrict__ rl = recs + ((h << halves) + (halves ? li >> 3 : 0)) * 2;
            const int e_max = e_first + ks + (e_last - 1 - e_first - ks) / KS * KS;   // this wavefront's last round
            struct record { i32x4 a, b; };            // {offset, place} of the round's four entries
            auto load_rec = [&](int e) {
                const i32x4* p = rl + ((size_t)min(e, e_max) << (3 + halves));
                return record{p[0], p[1]};
            };
            auto offset = [](const record& r, int j) { return j == 0 ? r.a.x : j == 1 ? r.a.z : j == 2 ? r.b.x : r.b.z; };
            auto place = [](const record& r, int j) { return (unsigned)(j == 0 ? r.a.y : j == 1 ? r.a.w : j == 2 ? r.b.y : r.b.w); };
            auto load_w = [&](int off) { return __builtin_amdgcn_raw_buffer_load_b128(wrsrc, off + (int)lane_w, 0, 0); };
            u32x4 wv[4];
            record now = load_rec(e_first + ks), next = load_rec(e_first + ks + KS), after = load_rec(e_first + ks + 2 * KS);
#pragma unroll
            for (int j = 0; j < 4; ++j) wv[j] = load_w(offset(now, j));

            int w_end = e_first, w_next = wq[min(1, n_win)];
            unsigned base = (unsigned)(kRing - 1) * BUF;   // of the window in LDS
            for (int e = e_first + ks; e <= e_max; e += KS) {
                while (e >= w_end) {                  // on to the next window
                    window_barrier();
                    ++w;
                    w_end = w_next;
                    w_next = wq[min(w + 2, n_win)];
                    base = base == (unsigned)(kRing - 1) * BUF ? 0u : base + BUF;
                }
                if constexpr (S == 2) {
                    Frag<T, CH> wf[4], xf[4][SUB];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const unsigned char* xp = lds + base + min(place(now, j) ^ lane_x, (unsigned)kZeroAt);
                        wf[j].w[0] = wv[j].x; wf[j].w[1] = wv[j].y; wf[j].w[2] = wv[j].z; wf[j].w[3] = wv[j].w;
#pragma unroll
                        for (int s = 0; s < SUB; ++s) xf[j][s].load(reinterpret_cast<const T*>(xp + s * kPitch));
                        if (j > 0) {
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int s = 0; s < SUB; ++s) mfma_frag<T, 16, CH>(acc[j - 1][s], wf[j - 1], xf[j - 1][s]);
                            wv[j - 1] = load_w(offset(next, j - 1));
                        }
                    }
#pragma unroll
                    for (int s = 0; s < SUB; ++s) mfma_frag<T, 16, CH>(acc[3][s], wf[3], xf[3][s]);
                    wv[3] = load_w(offset(next, 3));
                } else {                              // fp32: a multiplication saved is worth the branch
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned at = place(now, j);
                    if (__builtin_amdgcn_readfirstlane(at) != kNone) {   // uniform: this group of 16 rows has an entry left
                        const unsigned char* xp = lds + base + min(at ^ lane_x, (unsigned)kZeroAt);
                        Frag<T, CH> wf, xf[SUB];
                        wf.w[0] = wv[j].x; wf.w[1] = wv[j].y; wf.w[2] = wv[j].z; wf.w[3] = wv[j].w;
#pragma unroll
                        for (int s = 0; s < SUB; ++s) xf[s].load(reinterpret_cast<const T*>(xp + s * kPitch));
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int s = 0; s < SUB; ++s) mfma_frag<T, 16, CH>(acc[j][s], wf, xf[s]);
                    }
                    wv[j] = load_w(offset(next, j));
                }
                }
                now = next;
                next = after;
                after = load_rec(e + 3 * KS);
            }
        }
        for (; w < n_win - 1; ++w) window_barrier();
        if constexpr (OWN) {
            f32x4 all = acc[0][0];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int s = 0; s < SUB; ++s)
                    if (j + s > 0) all += acc[j][s];
            const float sum = all.x + all.y + all.z + all.w;
            if (sum != sum) not_finite = 1;           // behind the barriers of the windows
        }
    }

    // The wavefronts' sums through LDS: added over a quad's wavefronts in order, stored as whole lines of Y.
    constexpr int RP = SUB >= 2 ? kRowsOut : 16;      // rows per pass
    constexpr int EPT = 16 / (int)sizeof(O);          // outputs a thread stores
    constexpr int TPR = 64 / EPT;
    float* tiles = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int p = 0; p < 16 * SUB / RP; ++p) {
        __syncthreads();
        if (wave < kWaves) {
            float* mine = tiles + (size_t)wave * RP * kLdOut;
#pragma unroll
            for (int ss = 0; ss < RP / 16; ++ss)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<f32x4*>(mine + (ss * 16 + li) * kLdOut + j * 16 + 4 * h) = acc[j][p * (RP / 16) + ss];
        }
        __syncthreads();
        for (int t = tid; t < Q * RP * TPR; t += 64 * (kWaves + kLoaders)) {
            const int qi = t / (RP * TPR), row = t / TPR % RP, c = t % TPR * EPT;
            const int i = i_base + p * RP + row, col = column[qi] + c;
            if (col >= n || i >= m) continue;
            const float* src = tiles + ((size_t)(qi * KS) * RP + row) * kLdOut + c;
            float v[EPT];
#pragma unroll
            for (int e = 0; e < EPT; ++e) v[e] = src[e];
            for (int s = 1; s < KS; ++s) {
                src += RP * kLdOut;
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[e] += src[e];
            }
            O* dst = Y + (size_t)i * (size_t)n + col;
            if constexpr (EPT == 4) {
                *reinterpret_cast<f32x4*>(dst) = f32x4{v[0], v[1], v[2], v[3]};
            } else {
                typedef O o8 __attribute__((ext_vector_type(8)));
                o8 r;
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] = from_f32<O>(v[e]);
                *reinterpret_cast<o8*>(dst) = r;
            }
        }
    }
    // An entry of two block-rows multiplies the zeros of the one that does not store the column: an infinity or a NaN there
    // is no part of its outputs.  Outputs that came out as NaN are summed again, from their own blocks, by the thread that
    // has stored them.  (Looked for in the accumulators: in the loop above it takes 0.5 of 10 us.)
    if (OWN && not_finite) {
        asm volatile("" ::: "memory");
        const int bs_c = row_bytes / S;
        for (int p = 0; p < 16 * SUB / RP; ++p)
            for (int t = tid; t < Q * RP * TPR; t += 64 * (kWaves + kLoaders)) {
                const int i = i_base + p * RP + t / TPR % RP, col = column[t / (RP * TPR)] + t % TPR * EPT;
                if (col >= n || i >= m) continue;
                O* dst = Y + (size_t)i * (size_t)n + col;
                for (int e = 0; e < EPT; ++e) {
                    const float stored = (float)dst[e];
                    if (stored == stored) continue;
                    float own = 0.f;
                    for (int b = indptr[(col + e) >> 3]; b < indptr[((col + e) >> 3) + 1]; ++b) {
                        const T* x = X + (size_t)i * (size_t)k + (size_t)indices[b] * bs_c;
                        const T* w = data + ((size_t)b * 8 + ((col + e) & 7)) * bs_c;
                        for (int c = 0; c < bs_c; ++c) own += (float)x[c] * (float)w[c];
                    }
                    dst[e] = from_f32<O>(own);
                }
            }
    }
}

// Byte offsets into the rows of X of a workgroup are 32-bit, with the top bit left for what is not there.
bool reaches(const bsr_matrix* W, int sub) { return (int64_t)16 * sub * W->k * (W->dtype == BSR_F32 ? 4 : 2) < ((int64_t)1 << 31); }

// Rows of X and quads of a workgroup: the quickest by an estimate, fitted to bf16 and fp32 8x8 products of 17 to 2000
// rows by (512 .. 6016, 512 .. 4096), 5 to 25 % (within 3 % of the quickest of the twelve shapes, fp32 within 16 %).
// Microseconds: what a workgroup takes before its first and after its last round, a window, and a round.
struct sweep_shape_t { int sub, q_log; double us; };
sweep_shape_t choose(const bsr_matrix* W, int64_t m, int q_most, int64_t all_rounds, int64_t longest)
{
    const bool f32 = W->dtype == BSR_F32;
    sweep_shape_t best{1, 0, 1e30};
    for (int sub : {1, 2, 4}) {
        if (sub > 1 && !reaches(W, sub)) break;
        for (int q_log = 0; (1 << q_log) <= q_most; ++q_log) {
            const int Q = 1 << q_log, KS = kWaves / Q;
            if (q_log > 0 && (1 << (q_log - 1)) >= W->sw_quads) break;   // wavefronts without a quad
            const double wgs = (double)((m + 16 * sub - 1) / (16 * sub)) * ((W->sw_quads + Q - 1) / Q);
            const double start = sub == 4 ? 4.0 : sub == 2 ? 2.4 : 1.5;
            const double round = f32 ? 0.15 + 0.42 * sub : sub == 4 ? 0.40 : 0.32;
            auto us = [&](double rounds) { return start + W->sw_windows * 0.12 * sub + round * (rounds / KS + (KS > 1 ? 0.4 : 0.0) * W->sw_windows); };
            const double p = wgs / 256, passes = p <= 1 ? 1 : p <= 4 ? std::ceil(p) : p + 0.5;
            const double t = std::max(us((double)longest), passes * us((double)all_rounds / W->sw_quads));
            if (t < best.us) best = {sub, q_log, t};
        }
    }
    return best;
}

template <typename T, typename O, int SUB, bool OWN>
bsr_status launch_sub(const spmm_args& a, int q_log)
{
    const bsr_matrix* W = a.W;
    const int m = (int)a.m, TM = 16 * SUB;
    const int n_tiles = (m + TM - 1) / TM, Q = 1 << q_log;
    const int n_groups = (W->sw_quads + Q - 1) / Q;
    // tiles that would leave an XCD without are dealt out as they come: evenly over the XCDs comes first
    const int eight = (n_tiles + kXcds - 1) / kXcds * kXcds, padded = 5 * eight <= 6 * n_tiles ? eight : n_tiles;
    const int64_t blocks = (int64_t)padded * n_groups;
    if (blocks >= ((int64_t)1 << 31)) return BSR_ERR_SHAPE;
    constexpr size_t ring = (size_t)kRing * SUB * kPitch, out = (size_t)kWaves * (SUB >= 2 ? kRowsOut : 16) * kLdOut * sizeof(float);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bsr_mfma_sweep<T, O, SUB, OWN>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)std::max(ring, out));
    if (attr != hipSuccess) return BSR_ERR_HIP;
    hipLaunchKernelGGL((bsr_mfma_sweep<T, O, SUB, OWN>), dim3((unsigned)blocks), dim3(64 * (kWaves + kLoaders)), std::max(ring, out), a.stream,
                       (const T*)a.X, (const T*)W->data, (unsigned)(W->nnzb * W->bs_r * W->bs_c * sizeof(T)),
                       reinterpret_cast<const i32x4*>(W->sw_base + W->sw.recs_at), W->sw_base + W->sw.win_at,
                       reinterpret_cast<const i32x4*>(W->sw_base), (O*)a.Y, m, (int)W->k, (int)W->n,
                       n_tiles, padded, W->sw_quads, W->sw_windows, q_log, W->bs_r, W->bs_c * (int)sizeof(T),
                       W->indptr, W->indices);
    return hipGetLastError() == hipSuccess ? BSR_OK : BSR_ERR_HIP;
}

// A result in fp32 keeps as many chains of additions as the kernel of 16x16 tiles gives it: 8 where that starts few
// workgroups, at least 2 (root mean square error, fp32 8x8, m = 1000, (1024, 1024), 30 %: both 2.3e-7).
int most_quads(const bsr_matrix* W, int64_t m, bool f32_out)
{
    const int64_t items = ((m + 15) / 16) * ((W->n + 15) / 16);
    return !f32_out ? kWaves : items > 1024 ? kWaves / 2 : items > 256 ? kWaves / 4 : 1;
}

template <typename T, typename O>
bsr_status launch_types(const spmm_args& a, const tune_opts& tune)
{
    const int q_most = most_quads(a.W, a.m, std::is_same<O, float>::value);
    const sweep_shape_t c = choose(a.W, a.m, q_most, a.W->sw.rounds, a.W->sw.longest);
    int sub = c.sub, q_log = c.q_log;
    if ((tune.mt == 1 || tune.mt == 2 || tune.mt == 4) && reaches(a.W, tune.mt)) sub = tune.mt;
    if (tune.nw == 1 || tune.nw == 2 || tune.nw == 4 || tune.nw == 8)
        for (q_log = 0; (1 << q_log) < std::min(tune.nw, q_most);) ++q_log;
    auto launch = [&](auto own) {
        constexpr bool OWN = decltype(own)::value;
        return sub == 4 ? launch_sub<T, O, 4, OWN>(a, q_log) : sub == 2 ? launch_sub<T, O, 2, OWN>(a, q_log) : launch_sub<T, O, 1, OWN>(a, q_log);
    };
    // sizes without whole tiles: the wavefront kernels, which would run else, keep every output to its own blocks
    if (a.W->bs_r == 8 && !mfma_small_supports(a.W)) return launch(std::true_type{});
    return launch(std::false_type{});
}

}  // namespace

bool mfma_sweep_supports(const bsr_matrix* W) { return W->sw_base != nullptr; }

// Rounds of all quads and of the longest, without the plan (a window has as many as the longest of a quad's groups has
// entries), and the 16x16 tiles of W that hold a block, of all tile-rows and of the longest.  May throw.
struct sweep_counts { int64_t rounds, longest, tiles; int32_t longest_tiles; };
static sweep_counts count_plan(const bsr_matrix* W, const int32_t* indptr, const int32_t* indices)
{
    const int row_bytes = W->bs_c * (W->dtype == BSR_F32 ? 4 : 2), per_entry = 64 / row_bytes;
    const int per_window = kSlabs * 128 / row_bytes, per_tile = 16 / W->bs_c;      // block-columns
    std::vector<int32_t> most((size_t)W->sw_windows), mine((size_t)W->sw_windows), first(W->bs_r == 8 ? (size_t)W->C : 0);
    std::vector<int32_t> tile_of((size_t)(W->C / per_tile + 1), -1);
    sweep_counts c{0, 0, 0, 0};
    for (int32_t q = 0; q < W->sw_quads; ++q) {
        std::fill(most.begin(), most.end(), 0);
        for (int32_t g = 4 * q; g < 4 * q + 4; ++g) {
            std::fill(mine.begin(), mine.end(), 0);
            int32_t tiles = 0;
            const int32_t r = g * (16 / W->bs_r);
            auto row = [&](int32_t rr, auto visit) {
                if (rr >= W->R) return;
                for (int32_t p = indptr[rr]; p < indptr[rr + 1]; ++p) visit(indices[p]);
            };
            auto count = [&](int32_t col, bool opens) {
                mine[(size_t)(col / per_window)] += opens;
                int32_t& t = tile_of[(size_t)(col / per_tile)];
                tiles += t != g;
                t = g;
            };
            row(r, [&](int32_t col) { count(col, true); if (W->bs_r == 8) ++first[(size_t)col]; });
            if (W->bs_r == 8) {                       // the second block-row's block shares the first's slot of that column
                row(r + 1, [&](int32_t col) { int32_t& f = first[(size_t)col]; count(col, f == 0); f -= f > 0; });
                row(r, [&](int32_t col) { first[(size_t)col] = 0; });
            }
            for (size_t w = 0; w < mine.size(); ++w) most[w] = std::max(most[w], (mine[w] + per_entry - 1) / per_entry);
            c.tiles += tiles;
            c.longest_tiles = std::max(c.longest_tiles, tiles);
        }
        const int64_t rounds = std::accumulate(most.begin(), most.end(), (int64_t)0);
        c.rounds += rounds;
        c.longest = std::max(c.longest, rounds);
    }
    return c;
}

// The same for the choice of a product, once per handle; false if there is no memory for it.
static bool count_rounds(const bsr_matrix* W)
{
    if (W->sw.counted.load(std::memory_order_acquire)) return true;
    std::lock_guard<std::mutex> lock(W->sw_mu);
    if (W->sw.counted.load(std::memory_order_relaxed)) return true;
    try {
        const sweep_counts c = count_plan(W, W->sl_indptr.data(), W->sl_indices.data());
        W->sw.rounds = c.rounds;
        W->sw.longest = c.longest;
    } catch (const std::bad_alloc&) {
        return false;
    }
    W->sw.counted.store(true, std::memory_order_release);
    return true;
}

// Microseconds of the kernel that would run else.
// Stripes: X staged, Y stored, products, and a term for the rows' length.  k-split: stored blocks and block-rows of every tile
// of 16 rows (its X comes from L2 or beyond once per stored block), and the longest block-row.  16x16 tiles: workgroups,
// tiles of W (more where X is past L2: each fetches its own), and the longest tile-row's share of a wavefront.
static double rival_us(const bsr_matrix* W, int64_t m, sweep_rival than)
{
    const double mt = (double)((m + 15) / 16);
    if (than == sweep_rival::stripes)
        return 4.6 + 6.3e-7 * (double)(m * W->k) + 4.7e-7 * (double)(m * W->n) + 2.3e-5 * mt * (double)W->nnzb + 2.9e-3 * (double)W->k;
    if (than == sweep_rival::ksplit) return 4.1 + 0.84e-4 * mt * (double)W->nnzb + 3.7e-4 * mt * W->R + 2.7e-2 * W->max_row_blocks;
    const double items = mt * W->sb_rows, tiles = mt * (double)W->sb_tiles;
    const double chain = (double)W->sb_max_entries / std::max(1, std::min(items > 1024 ? 2 : items > 256 ? 4 : 8, (W->sb_max_entries + 1) / 2));
    const double x = (double)(m * W->k);
    if (W->dtype == BSR_F32) return 2.5 + 4e-4 * items + (7.4e-5 + 1.74e-4 * x / (x + 1.25e8)) * tiles + 0.257 * chain * (1 + 16.3 * x / (x + 1.25e8));
    return 2.5 + 4e-4 * items + (5.1e-5 + 5e-5 * std::min(1.0, x / 3.2e7)) * tiles + 0.244 * chain;
}

// The choice between this kernel and the one that would run else, from estimates in microseconds.
// 16x16 blocks, fitted to 225 bf16 products (16 .. 8192 rows, sides 128 .. 8192, 3 to 30 %, uniform and power law): half of
// the estimates are within 5 % (this kernel), 8 % (k-split) and 9 % (stripes) of the time and nine tenths within 16, 31 and
// 36 %, so this kernel is taken only where its own is lower by a quarter, against stripes by three tenths: of those and 268
// other products 65 are, up to 5 times quicker and none slower (a fifth lower: 96, five of them 4 to 28 % slower); of 809
// drawn afterwards 90 are more than a tenth quicker and four slower, by 8 to 36 % (2624 x (1440, 3008), 11 %: stripes 15.9 us).
// Blocks with a side of 8, fitted to half of 4000 products of the same ranges: half of the estimates within 4 % (this
// kernel), 5 % (tiles), fp32 8 and 6 %, nine tenths within 14, 15, 21 and 17 %.  On the other half, 16-bit: of 1011 products 14
// are more than 5 % slower than with the kernel of tiles and 7 than with this one (this one for all but long, thin rows of
// W: 240, up to 1.7 times as slow, 3.3 us where tiles take 2.5).  fp32 from 384 rows on: of 475 13 and 50 (this one for all: 151,
// up to 2.4 times as slow; 647 x (128, 960), 3.4 %, tiles 3.6, this one 5.5; 1073 x (832, 192), 4.1 % 4.4, 7.0).
static bool quicker(const bsr_matrix* W, int64_t m, bsr_dtype y_dtype, sweep_rival than, int64_t rounds, int64_t longest)
{
    const double us = choose(W, m, most_quads(W, m, y_dtype == BSR_F32), rounds, longest).us, out = (double)((m + 15) / 16) * (double)W->n;
    if (than == sweep_rival::tiles)
        return W->dtype == BSR_F32 ? 2.4 + 0.775 * us + 6.3e-6 * out < 0.95 * rival_us(W, m, than) : 1.64 + us + 2.9e-6 * out < rival_us(W, m, than);
    return 2.8 + 1.03 * us + 2.1e-6 * out < (than == sweep_rival::stripes ? 0.7 : 0.75) * rival_us(W, m, than);
}

bool sweep_is_quicker(const bsr_matrix* W, int64_t m, bsr_dtype y_dtype, sweep_rival than)
{
    if (!mfma_sweep_supports(W)) return false;
    // with as few rounds as that many blocks can have; only then are they counted
    const int slots = 64 / (W->bs_c * (W->dtype == BSR_F32 ? 4 : 2));   // block-columns of an entry
    if (!W->sw.counted.load(std::memory_order_acquire) &&
        (!quicker(W, m, y_dtype, than, W->nnzb / (4 * slots * (16 / W->bs_r)), W->max_row_blocks / slots) || !count_rounds(W)))
        return false;
    return quicker(W, m, y_dtype, than, W->sw.rounds, W->sw.longest);
}

bool sweep_leaves_tiles(bsr_matrix* W, const int32_t* indptr, const int32_t* indices)
{
    const sweep_counts c = count_plan(W, indptr, indices);
    W->sw.rounds = c.rounds;
    W->sw.longest = c.longest;
    W->sw.counted.store(true, std::memory_order_release);
    W->sb_tiles = c.tiles;
    W->sb_max_entries = c.longest_tiles;
    for (int64_t m : {16, 32, 64, 128, 256, 512, 1024})
        if (!quicker(W, m, W->dtype, sweep_rival::tiles, c.rounds, c.longest)) return true;
    return false;
}

bsr_status launch_mfma_sweep(const spmm_args& a, const tune_opts& t)
{
    const bsr_matrix* W = a.W;
    if (!mfma_sweep_supports(W) || !sweep_ready(W, a.stream)) return BSR_ERR_UNSUPPORTED;
    if (!W->sw_created) {
        const bsr_status dbg = debug_check_words(W, W->sw_base, W->sw.host, a.stream);
        if (dbg != BSR_OK) return dbg;
    }
    if (W->dtype == BSR_F32) return launch_types<float, float>(a, t);
    if (W->dtype == BSR_F16) return a.y_dtype == BSR_F32 ? launch_types<_Float16, float>(a, t) : launch_types<_Float16, _Float16>(a, t);
    return a.y_dtype == BSR_F32 ? launch_types<__bf16, float>(a, t) : launch_types<__bf16, __bf16>(a, t);
}

// Blocks of 8 rows or columns are smaller than an MFMA step takes, and 16x16 blocks of a 16-bit type touch 32 bytes of a row
// of X each.  Larger ones have kernels that stage them one by one and gain little here (bf16, kernels of staged tiles and
// this one, us: 32x32 3876 x (5824, 704), 17 %, power law 65, 52, but 4096 x (768, 3072), 20 % 17, 23; 64x64 4096 x
// (6016, 1536), 20 % 45, 63); 16x16 blocks of fp32 wait for the matrix cores wherever they are.
static bool sweep_shape(int32_t bs_r, int32_t bs_c) { return (bs_r == 8 || bs_r == 16) && (bs_c == 8 || bs_c == 16); }

// Words of a round's record: {offset, place} for four granules of four groups, blocks of 8 rows for two of them each.
static int round_words(int32_t bs_r) { return bs_r == 8 ? 64 : 32; }

// Words of the plan: {quad, rounds} and the windows' first rounds per quad, and the rounds' records.  A window has as many
// rounds as the longest of a quad's groups has entries: at worst all of its blocks are in that one.  fp32 makes the most of
// both: windows of 256 columns, entries of 16; 16x16 blocks are always of a 16-bit type, two to an entry.
size_t sweep_plan_words(int64_t n, int64_t k, int32_t bs_r, int32_t bs_c, int64_t nnzb)
{
    if (!sweep_shape(bs_r, bs_c) || nnzb == 0) return 0;
    const size_t quads = (size_t)(n + 63) / 64, windows = (size_t)(k + 255) / 256;
    // the table of first rounds must not outgrow the blocks (256 KiB are always fine); where most windows of a quad hold none,
    // moving all of X through LDS is no gain either
    if (quads * (windows + 1) > 4 * (size_t)nnzb + 65536) return 0;
    const size_t rounds = std::min((size_t)nnzb, (size_t)nnzb / (bs_r == 16 && bs_c == 16 ? 2 : 16 / bs_c) + quads * windows);
    return 4 * quads + quads * (windows + 1) + (size_t)round_words(bs_r) * rounds + 3 * 64;
}

int32_t sweep_windows(const bsr_matrix* W)
{
    const int cols = kSlabs * 128 / (W->dtype == BSR_F32 ? 4 : 2);
    return (int32_t)((W->k + cols - 1) / cols);
}

bool sweep_takes(const bsr_matrix* W)
{
    const int S = W->dtype == BSR_F32 ? 4 : 2;
    return sweep_plan_words(W->n, W->k, W->bs_r, W->bs_c, W->nnzb) > 0 && !(W->bs_r == 16 && W->bs_c == 16 && S == 4) &&
           W->nnzb * W->bs_r * W->bs_c * S < ((int64_t)1 << 31) && reaches(W, 1);
}

void build_sweep_plan(const bsr_matrix* W, const int32_t* indptr, const int32_t* indices, std::vector<int32_t>& plan)
{
    const int bs_r = W->bs_r, bs_c = W->bs_c, S = W->dtype == BSR_F32 ? 4 : 2;
    const int64_t row_bytes = (int64_t)bs_c * S, block = bs_r * row_bytes;
    const int gran = (int)(row_bytes / 16);           // granules of a block's row: 1, 2 or 4
    const int per_entry = 4 / gran;                   // block-columns of an entry
    const int win_cols = kSlabs * 128 / S, n_win = W->sw_windows;
    const int n_quads = W->sw_quads;
    struct slot { int32_t col; int32_t off[2]; };     // first column, byte offset of the values for rows 0-7 and 8-15
    std::vector<slot> rows[4];
    const size_t desc_at = plan.size(), win_at = desc_at + (4 * (size_t)n_quads + 63) / 64 * 64;
    const size_t recs_at = win_at + ((size_t)n_quads * (n_win + 1) + 63) / 64 * 64;
    plan.resize(recs_at, 0);
    const int rec = round_words(bs_r), part = rec / 4;   // words of a round, of a granule in it
    auto rounds_so_far = [&] { return (int32_t)((plan.size() - recs_at) / (size_t)rec); };
    std::vector<int32_t> ptr((size_t)n_quads * (n_win + 1));
    std::vector<int32_t> load((size_t)n_quads);
    struct stored { int32_t col, at; };               // block-column, number of the stored block
    std::vector<stored> sorted[2];
    auto sorted_row = [&](int64_t r, std::vector<stored>& v) {
        const int32_t first = r < W->R ? indptr[r] : 0, count = r < W->R ? indptr[r + 1] - first : 0;
        v.resize((size_t)count);
        bool in_order = true;
        for (int32_t i = 0; i < count; ++i) {
            v[(size_t)i] = {indices[first + i], first + i};
            in_order = in_order && (i == 0 || indices[first + i - 1] <= indices[first + i]);
        }
        if (!in_order) std::stable_sort(v.begin(), v.end(), [](const stored& a, const stored& b) { return a.col < b.col; });
    };
    for (int q = 0; q < n_quads; ++q) {
        for (int j = 0; j < 4; ++j) {
            auto& list = rows[j];
            list.clear();
            const int64_t g = (int64_t)q * 4 + j;
            sorted_row(bs_r == 8 ? 2 * g : g, sorted[0]);
            if (bs_r == 16) {
                for (const auto& b : sorted[0]) list.push_back({b.col * bs_c, {(int32_t)(b.at * block), (int32_t)(b.at * block)}});
                continue;
            }
            sorted_row(2 * g + 1, sorted[1]);         // two block-rows, by column; a block stored twice opens a second slot
            size_t a = 0, b = 0;
            while (a < sorted[0].size() || b < sorted[1].size()) {
                const int32_t ca = a < sorted[0].size() ? sorted[0][a].col : INT32_MAX;
                const int32_t cb = b < sorted[1].size() ? sorted[1][b].col : INT32_MAX;
                const int32_t c = std::min(ca, cb);
                slot s{c * bs_c, {INT32_MIN, INT32_MIN}};
                if (ca == c) s.off[0] = (int32_t)(sorted[0][a++].at * block);
                if (cb == c) s.off[1] = (int32_t)(sorted[1][b++].at * block);
                list.push_back(s);
            }
        }
        size_t at[4] = {0, 0, 0, 0}, end[4];
        const int32_t first = rounds_so_far();
        for (int w = 0; w < n_win; ++w) {
            ptr[(size_t)q * (n_win + 1) + w] = rounds_so_far();
            size_t rounds = 0;
            for (int j = 0; j < 4; ++j) {
                const auto& list = rows[j];
                end[j] = at[j];
                while (end[j] < list.size() && list[end[j]].col < (w + 1) * win_cols) ++end[j];
                rounds = std::max(rounds, (end[j] - at[j] + per_entry - 1) / per_entry);
            }
            const size_t here = plan.size();
            plan.resize(here + rounds * (size_t)rec);
            int32_t* r = plan.data() + here;
            for (size_t i = 0; i < rounds * (size_t)rec / 2; ++i) { r[2 * i] = INT32_MIN; r[2 * i + 1] = kNone; }
            for (int j = 0; j < 4; ++j) {
                for (size_t i = at[j]; i < end[j]; ++i) {
                    const slot& s = rows[j][i];
                    const size_t rd = (i - at[j]) / (size_t)per_entry, u = (i - at[j]) % (size_t)per_entry;
                    const int byte = (s.col - w * win_cols) * S, place = byte / 128 * 2048 + byte % 128;   // a block's granules share a slab
                    int32_t* e = r + rd * (size_t)rec + u * (size_t)(gran * part) + j * 2;
                    for (int v = 0; v < gran; ++v, e += part) {
                        e[0] = s.off[0];
                        e[1] = place + v * 16;
                        if (bs_r == 8) { e[8] = s.off[1]; e[9] = e[1]; }
                    }
                }
                at[j] = end[j];
            }
        }
        ptr[(size_t)q * (n_win + 1) + n_win] = rounds_so_far();
        load[(size_t)q] = rounds_so_far() - first;
    }
    std::vector<int32_t> order((size_t)n_quads);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return load[(size_t)a] > load[(size_t)b]; });
    for (int s = 0; s < n_quads; ++s) {
        const int32_t* p = ptr.data() + (size_t)order[(size_t)s] * (n_win + 1);
        int32_t* d = plan.data() + desc_at + 4 * (size_t)s;
        d[0] = order[(size_t)s];
        d[1] = p[0];
        d[2] = p[n_win];
        std::copy(p, p + n_win + 1, plan.begin() + (ptrdiff_t)(win_at + (size_t)s * (n_win + 1)));
    }
    const int32_t all_rounds = rounds_so_far();
    plan.resize((plan.size() + 63) & ~(size_t)63, 0);
    W->sw.win_at = win_at - desc_at;
    W->sw.recs_at = recs_at - desc_at;
    if (!W->sw.counted.load(std::memory_order_relaxed)) {
        W->sw.rounds = all_rounds;
        W->sw.longest = n_quads ? load[(size_t)order[0]] : 0;
        W->sw.counted.store(true, std::memory_order_release);
    }
    W->sw.built = true;                               // not before: whatever throws leaves it to be built again
}

bool sweep_ready(const bsr_matrix* W, hipStream_t stream)
{
    bsr_matrix::sweep_plan& p = W->sw;
    if (W->sw_created || p.landed.load(std::memory_order_acquire)) return true;
    std::lock_guard<std::mutex> lock(W->sw_mu);
    if (is_capturing(stream)) return p.sent && upload_landed(p.uploaded, p.landed);
    if (p.sent) {
        order_after_upload(stream, p.uploaded, p.landed);
        return true;
    }
    if (!p.built) {
        try {
            p.host.clear();
            build_sweep_plan(W, W->sl_indptr.data(), W->sl_indices.data(), p.host);
        } catch (const std::bad_alloc&) {             // no memory for the plan: the caller takes a kernel that needs none
            return false;
        }
    }
    p.sent = p.host.size() <= W->sw_words && upload_words(W->sw_base, p.host, stream, p.uploaded, p.landed);
    if (!p.sent) (void)hipGetLastError();             // nothing was launched, and another kernel will be
    return p.sent;
}
