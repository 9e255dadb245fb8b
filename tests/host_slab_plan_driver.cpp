// Host-side check of the sampled product's group plan (test infrastructure; no GPU).  For random patterns of every
// block shape the kernel takes, the plan is decoded as the kernel decodes it: every element of every stored block
// must be covered exactly once, by a tile whose staged columns of G and X are that element's row and column of W;
// every slab a chunk names is one of its group's, within the buffer; the plan fits the words promised for it.
// Build: hipcc --offload-arch=gfx950 -O1 -std=c++17 -I include -I paper_2007_13055_amd/csrc
//        tests/host_slab_plan_driver.cpp paper_2007_13055_amd/csrc/bsr_sddmm_slab.hip -o driver
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <numeric>
#include <vector>
#include "bsr_internal.h"

static long g_allocations_left = -1;                  // after so many, operator new throws (-1: never)
void* operator new(std::size_t bytes)
{
    if (g_allocations_left == 0) throw std::bad_alloc();
    if (g_allocations_left > 0) --g_allocations_left;
    if (void* p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

// the launcher's, not used here
void order_after_upload(hipStream_t, hipEvent_t, std::atomic<bool>&) {}
bsr_status debug_check_words(const bsr_matrix*, const int32_t*, const std::vector<int32_t>&, hipStream_t) { return BSR_OK; }

#define CHECK(c) do { if (!(c)) { std::printf("FAILED %s (line %d) trial %d: blocks %dx%d dtype %d R %d C %d\n", #c, __LINE__, trial, bs_r, bs_c, (int)W.dtype, R, C); return 1; } } while (0)

int main()
{
    std::srand(5);
    const int sides[4] = {8, 16, 32, 64};
    long groups = 0;
    for (int trial = 0; trial < 640; ++trial) {
        const int bs_r = sides[trial % 4], bs_c = sides[trial / 4 % 4];
        const int R = 1 + std::rand() % 60, C = 1 + std::rand() % 70, style = trial / 16 % 5;
        std::vector<int32_t> ptr(R + 1, 0), idx;
        for (int r = 0; r < R; ++r) {
            int c = std::rand() % (C + 1);
            if (style == 1) c = r == R / 2 ? C : std::rand() % 3;
            if (style == 2) c = (int)(C / (1.0 + r));
            if (style == 3) c = std::rand() % 4 ? 0 : 1;
            for (int j = 0; j < c; ++j) idx.push_back(style == 4 || trial % 7 == 0 ? std::rand() % C : (j * 5 + r) % C);   // any order, duplicates
            if (style == 0) std::sort(idx.begin() + ptr[r], idx.end());
            ptr[r + 1] = ptr[r] + c;
        }
        const int64_t nnzb = ptr[R];
        bsr_matrix W;
        W.n = (int64_t)R * bs_r; W.k = (int64_t)C * bs_c; W.nnzb = nnzb; W.bs_r = bs_r; W.bs_c = bs_c; W.R = R; W.C = C;
        W.dtype = trial / 16 % 2 ? BSR_F16 : BSR_F32;
        const int line = W.dtype == BSR_F32 ? 32 : 64, s = 128 / line, V = bs_r >= 32 && bs_c >= 32 ? 32 : 16, H = V / 2;
        const int CR = bs_r == 64 && bs_c == 64 ? 2 : 1, CC = V == 32 ? 2 : 4;
        const size_t order_words = (size_t)((R + 63) & ~63);
        W.staging.assign(order_words, 0);
        std::iota(W.staging.begin(), W.staging.begin() + R, 0);
        std::stable_sort(W.staging.begin(), W.staging.begin() + R, [&](int32_t a, int32_t b) { return ptr[a + 1] - ptr[a] > ptr[b + 1] - ptr[b]; });
        W.sl_words = sddmm_slab_plan_words(W.k, bs_r, bs_c, nnzb);
        CHECK((W.sl_words > 0) == (nnzb > 0));
        if (nnzb == 0) continue;
        W.sl_indptr = ptr;
        W.sl_indices = idx;
        // memory runs out part of the way, again and again, a little later each time: "not ready", and nothing lost
        bool ready = false;
        for (long some = trial % 3; !ready; some += 1 + some / 2) {
            g_allocations_left = some;
            ready = sddmm_slab_ready(&W);
            g_allocations_left = -1;
            CHECK(ready == W.sl.built && (ready || !W.sl.sent));
        }
        CHECK(W.sl.host.size() <= W.sl_words && W.sl.groups > 0 && W.sl.tiles_at + 4 * (size_t)W.sl.n_tiles == W.sl.host.size());
        CHECK(W.sl.chunks_at % 4 == 0 && W.sl.tiles_at % 4 == 0 && W.sl.lds <= 160 * 1024);
        const int32_t* hdr = W.sl.host.data();
        const int32_t* chunks = hdr + W.sl.chunks_at;
        const int32_t* tiles = hdr + W.sl.tiles_at;
        std::vector<int32_t> row_of((size_t)nnzb);
        for (int r = 0; r < R; ++r) for (int p = ptr[r]; p < ptr[r + 1]; ++p) row_of[(size_t)p] = r;
        std::vector<char> seen((size_t)nnzb * bs_r * bs_c, 0), tile_seen((size_t)W.sl.n_tiles, 0);
        int next = 0;
        for (int g = 0; g < W.sl.groups; ++g, ++groups) {
            const int32_t* h = hdr + 16 * g;
            CHECK(h[0] >= 2 && h[0] <= 12 && h[0] * 4096 <= W.sl.lds && h[1] >= 1 && h[1] < h[0] && h[2] == next && h[3] >= 1 && h[3] <= 8 * (V == 16 ? 5 : CR == 2 ? 1 : 3));
            next += h[3];
            for (int z = 0; z < h[0]; ++z) CHECK(h[4 + z] >= 0 && h[4 + z] % line == 0 && h[4 + z] < (z < h[1] ? W.n : W.k));
            for (int q = h[2]; q < h[2] + h[3]; ++q) {
                const uint32_t* c = reinterpret_cast<const uint32_t*>(chunks) + 4 * q;
                const int live = (int)(c[3] >> 28), t0 = (int)(c[3] & 0x0fffffffu);
                CHECK(live >= 1 && live <= CR * CC && t0 + live <= W.sl.n_tiles);
                for (int t = 0; t < CR * CC; ++t) {
                    const unsigned a = c[0] >> (16 * (t / CC)) & 0xffffu, b = c[1 + t % CC / 2] >> (16 * (t % CC % 2)) & 0xffffu;
                    const unsigned sa = a / 4096, sb = b / 4096;
                    CHECK(sa < (unsigned)h[1] && sb >= (unsigned)h[1] && sb < (unsigned)h[0]);
                    CHECK(a % 4096 + V * s <= 128 && b % 4096 + V * s <= 128 && a % (V * s) == 0 && b % (V * s) == 0);
                    if (t >= live) continue;
                    CHECK(!tile_seen[(size_t)(t0 + t)]++);
                    const int col_g = h[4 + sa] + (int)(a % 4096) / s, col_x = h[4 + sb] + (int)(b % 4096) / s;
                    for (int i = 0; i < V; ++i)
                        for (int j = 0; j < V; ++j) {
                            const int32_t off = tiles[4 * (t0 + t) + 2 * (i / H) + j / H];
                            if (off < 0) continue;
                            const int64_t e = (int64_t)off + (i % H) * bs_c + j % H;
                            CHECK(e < nnzb * bs_r * bs_c);
                            const int p = (int)(e / (bs_r * bs_c)), in = (int)(e % (bs_r * bs_c));
                            CHECK(row_of[(size_t)p] * bs_r + in / bs_c == col_g + i && idx[(size_t)p] * bs_c + in % bs_c == col_x + j);
                            CHECK(!seen[(size_t)e]++);
                        }
                }
            }
        }
        for (char v : seen) CHECK(v);
        for (char v : tile_seen) CHECK(v);
    }
    std::printf("%ld groups: all consistent\n", groups);
    return groups > 1000 ? 0 : 1;
}
