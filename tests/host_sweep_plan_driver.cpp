// Host-side check of the sweep kernel's plan (test infrastructure; no GPU).  For random patterns of every block shape and
// type the kernel takes, the plan is decoded as the kernel decodes it: every 16-byte granule of every stored block must be
// multiplied exactly once, by the lane of its row of W, with the columns of X it belongs to, in their window; whatever else
// a record names reads zeros on both sides; the plan fits the words promised for it; and the rounds that the choice of
// kernel counts without a plan are the plan's.
// Build: hipcc --offload-arch=gfx950 -O1 -std=c++17 -I include -I paper_2007_13055_amd/csrc
//        tests/host_sweep_plan_driver.cpp paper_2007_13055_amd/csrc/bsr_mfma_sweep.hip -o driver
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <new>
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

// the host's, not used here: nothing is captured, and every upload is over at once
void order_after_upload(hipStream_t, hipEvent_t, std::atomic<bool>&) {}
bool is_capturing(hipStream_t) { return false; }
bool upload_landed(hipEvent_t, std::atomic<bool>&) { return true; }
bool upload_words(int32_t*, const std::vector<int32_t>&, hipStream_t, hipEvent_t&, std::atomic<bool>&) { return true; }
bsr_status debug_check_words(const bsr_matrix*, const int32_t*, const std::vector<int32_t>&, hipStream_t) { return BSR_OK; }
bool mfma_small_supports(const bsr_matrix*) { return true; }

#define CHECK(c) do { if (!(c)) { std::printf("FAILED %s (line %d) trial %d: blocks %dx%d dtype %d R %d C %d\n", #c, __LINE__, trial, bs_r, bs_c, (int)dtype, R, C); return 1; } } while (0)

static void prepare(bsr_matrix& W, int bs_r, int bs_c, bsr_dtype dtype, const std::vector<int32_t>& ptr, const std::vector<int32_t>& idx, int R, int C, int32_t* base)
{
    W.n = (int64_t)R * bs_r; W.k = (int64_t)C * bs_c; W.nnzb = ptr[(size_t)R]; W.bs_r = bs_r; W.bs_c = bs_c; W.R = R; W.C = C; W.dtype = dtype;
    for (int r = 0; r < R; ++r) W.max_row_blocks = std::max(W.max_row_blocks, ptr[(size_t)r + 1] - ptr[(size_t)r]);
    W.sl_indptr = ptr;
    W.sl_indices = idx;
    W.sw_words = sweep_plan_words(W.n, W.k, bs_r, bs_c, W.nnzb);
    W.sw_quads = (int32_t)((W.n + 63) / 64);
    W.sw_windows = sweep_windows(&W);
    W.sw_base = base;
}

int main()
{
    std::srand(9);
    const int sides[4][2] = {{8, 8}, {8, 16}, {16, 8}, {16, 16}};
    long all = 0, compared = 0;
    int32_t base[4];
    for (int trial = 0; trial < 600; ++trial) {
        const int bs_r = sides[trial % 4][0], bs_c = sides[trial % 4][1], style = trial / 16 % 6;
        const bsr_dtype dtype = trial / 4 % 2 ? BSR_F16 : BSR_F32;
        const int S = dtype == BSR_F32 ? 4 : 2, R = 1 + std::rand() % 70, C = 1 + std::rand() % (trial % 3 ? 300 : 40);
        std::vector<int32_t> ptr((size_t)R + 1, 0), idx;
        for (int r = 0; r < R; ++r) {
            int c = std::rand() % (C + 1);
            if (style == 1) c = r == R / 2 ? C : std::rand() % 3;
            if (style == 2) c = (int)(C / (1.0 + r));
            if (style == 3) c = std::rand() % 4 ? 0 : 1;
            if (style == 5) c = r % 4 == 0 ? C : 0;   // one of four groups has everything: the most rounds
            for (int j = 0; j < c; ++j) idx.push_back(style == 4 ? std::rand() % C : style == 5 ? j : (int)(((int64_t)j * 7 + r) % C));   // any order, duplicates
            if (style == 0) std::sort(idx.begin() + ptr[(size_t)r], idx.end());
            ptr[(size_t)r + 1] = ptr[(size_t)r] + c;
        }
        const int64_t nnzb = ptr[(size_t)R];
        bsr_matrix W;
        prepare(W, bs_r, bs_c, dtype, ptr, idx, R, C, base);
        CHECK(sweep_takes(&W) == (nnzb > 0 && !(bs_r == 16 && bs_c == 16 && S == 4)));
        if (!sweep_takes(&W)) continue;
        // memory runs out part of the way, again and again, a little later each time: "not ready", and nothing lost
        bool ready = false;
        for (long some = trial % 3; !ready; some += 1 + some / 2) {
            g_allocations_left = some;
            ready = sweep_ready(&W, nullptr);
            g_allocations_left = -1;
            CHECK(ready == W.sw.built && ready == W.sw.sent);
        }
        const std::vector<int32_t>& plan = W.sw.host;
        CHECK(plan.size() <= W.sw_words && plan.size() % 64 == 0 && W.sw.win_at % 4 == 0 && W.sw.recs_at % 4 == 0);
        const int row_bytes = bs_c * S, gran = row_bytes / 16, block = bs_r * row_bytes, halves = bs_r == 8 ? 1 : 0;
        const int rec = bs_r == 8 ? 64 : 32, n_win = W.sw_windows, cols = 1024 / S;
        std::vector<int32_t> row_of((size_t)nnzb);
        for (int r = 0; r < R; ++r) for (int p = ptr[(size_t)r]; p < ptr[(size_t)r + 1]; ++p) row_of[(size_t)p] = r;
        std::vector<char> seen((size_t)nnzb * bs_r * gran, 0), quad_seen((size_t)W.sw_quads, 0);
        int64_t rounds = 0, longest = 0, before = INT64_MAX;
        for (int s = 0; s < W.sw_quads; ++s) {
            const int32_t* d = plan.data() + 4 * s;
            const int32_t* wq = plan.data() + W.sw.win_at + (size_t)s * (n_win + 1);
            CHECK(d[0] >= 0 && d[0] < W.sw_quads && !quad_seen[(size_t)d[0]]++ && d[1] >= 0 && d[2] >= d[1]);
            CHECK(wq[0] == d[1] && wq[n_win] == d[2] && W.sw.recs_at + (size_t)d[2] * rec <= plan.size());
            CHECK(d[2] - d[1] <= before);             // the longest first
            before = d[2] - d[1];
            rounds += before;
            longest = std::max(longest, before);
            for (int w = 0; w < n_win; ++w) {
                CHECK(wq[w] <= wq[w + 1]);
                for (int e = wq[w]; e < wq[w + 1]; ++e, ++all)
                    for (int h = 0; h < 4; ++h)
                        for (int j = 0; j < 4; ++j) {
                            const int32_t* r = plan.data() + W.sw.recs_at + (size_t)e * rec;
                            auto at = [&](int half) { return r + ((h << halves) + half) * 8 + j * 2; };
                            CHECK(at(0)[1] == at(halves)[1]);   // X is read by the lanes of both halves
                            const int place = at(0)[1];
                            CHECK(place == 0xFFFF || (place >= 0 && place < 8 * 2048 && place % 2048 < 128 && place % 16 == 0));
                            for (int li = 0; li < 16; ++li) {
                                const int64_t off = at(halves ? li >> 3 : 0)[0];
                                if (off == INT32_MIN) continue;
                                CHECK(place != 0xFFFF && off >= 0 && off % block == 0);
                                const int64_t a = off + (li & (bs_r - 1)) * row_bytes + (h & (gran - 1)) * 16;
                                CHECK(a + 16 <= nnzb * block);
                                const int p = (int)(a / block), row = (int)(a % block / row_bytes), g = (int)(a % row_bytes / 16);
                                CHECK((int64_t)row_of[(size_t)p] * bs_r + row == (int64_t)d[0] * 64 + j * 16 + li);
                                CHECK(idx[(size_t)p] * bs_c + g * (16 / S) == w * cols + place / 2048 * (128 / S) + place % 128 / S);
                                CHECK(!seen[((size_t)p * bs_r + row) * gran + g]++);
                            }
                        }
            }
        }
        for (char v : seen) CHECK(v);
        CHECK(rounds == W.sw.rounds && longest == W.sw.longest);
        bsr_matrix V;                                 // counted without the plan
        prepare(V, bs_r, bs_c, dtype, ptr, idx, R, C, base);
        if (bs_r == 16 && bs_c == 16) {
            for (int64_t m : {64, 1000, 8000}) (void)sweep_is_quicker(&V, m, dtype, sweep_rival::ksplit);
        } else {
            (void)sweep_leaves_tiles(&V, ptr.data(), idx.data());
            std::vector<int64_t> tiles;
            for (int64_t p = 0; p < nnzb; ++p) tiles.push_back((int64_t)(row_of[(size_t)p] * bs_r / 16) * 10000 + idx[(size_t)p] * bs_c / 16);
            std::sort(tiles.begin(), tiles.end());
            CHECK(V.sb_tiles == std::unique(tiles.begin(), tiles.end()) - tiles.begin() && V.sb_max_entries > 0);
        }
        if (V.sw.counted) { CHECK(V.sw.rounds == rounds && V.sw.longest == longest && !V.sw.built); ++compared; }
    }
    // a table of windows that outgrows the blocks: no plan
    if (sweep_plan_words(1 << 20, 1 << 20, 8, 8, 10000) != 0 || sweep_plan_words(8192, 8192, 8, 8, 1) == 0) return 1;
    std::printf("%ld rounds, %ld counts: all consistent\n", all, compared);
    return all > 50000 && compared > 200 ? 0 : 1;
}
