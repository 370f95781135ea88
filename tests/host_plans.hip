// Host-only check of the index arithmetic the kernels share with the host: workspace carving and
// the LDS plans of every kernel, over the extreme shapes the library accepts (B = 256, S = 4096,
// V = 2^24, d not a multiple of 4).  Built by tests/test_host_plans.py with hipcc
// and run on the CPU; no GPU call is made (the kernels in the headers are compiled but never launched).  Every region must start aligned, lie behind its
// predecessor and end inside what the size function reports.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1806_00588_amd/csrc/candidates.h"
#include "../paper_1806_00588_amd/csrc/fused.h"
#include "../paper_1806_00588_amd/csrc/logits.h"
#include "../paper_1806_00588_amd/csrc/report.h"
#include "../paper_1806_00588_amd/csrc/select.h"
#include "../paper_1806_00588_amd/csrc/workspace.h"

using namespace lshbeam;

static int failures = 0;
#define CHECK(cond, ...)                                                  \
    do {                                                                  \
        if (!(cond)) {                                                    \
            ++failures;                                                   \
            std::printf("FAILED %s:%d  %s  ", __FILE__, __LINE__, #cond); \
            std::printf(__VA_ARGS__);                                     \
            std::printf("\n");                                            \
        }                                                                 \
    } while (0)

constexpr size_t kLdsLimit = kMaxDynLds;   // what the host allows a kernel to ask for

static void check_workspace(int S, int B, int V, bool full) {
    char* base = reinterpret_cast<char*>((uintptr_t)1 << 40);   // never dereferenced
    const Workspace w = carve_workspace(S, B, V, full, base);
    const size_t R = (size_t)S * B;
    struct Region { const char* name; const void* p; size_t bytes; };
    const Region regs[] = {
        {"cand", w.cand, full ? 0 : (size_t)S * V * 4},
        {"count", w.count, (size_t)S * 4},
        {"logits", w.logits, R * (size_t)w.cpitch * 4},
        {"partials", w.partials, R * (size_t)w.ppitch * sizeof(TileRecord)},
        {"ids2", w.ids2, R * (size_t)w.ppitch * 4},
        {"lse", w.lse, R * 4},
        {"row_bitmaps", w.row_bitmaps, full ? 0 : R * (((size_t)V + 31) / 32) * 4},
    };
    const char* prev_end = base;
    for (const Region& r : regs) {
        const char* p = (const char*)r.p;
        CHECK(((uintptr_t)p % kAlign) == 0, "%s misaligned (S=%d B=%d V=%d)", r.name, S, B, V);
        CHECK(p >= prev_end, "%s overlaps its predecessor (S=%d B=%d V=%d)", r.name, S, B, V);
        CHECK(p + r.bytes <= base + w.bytes, "%s ends outside the workspace (S=%d B=%d V=%d)", r.name, S, B, V);
        CHECK(r.bytes / 4 <= w.bytes, "size overflow in %s", r.name);
        prev_end = p + r.bytes;
    }
    CHECK(w.cpitch >= V && w.cpitch % 64 == 0 && w.ppitch * kTileN >= w.cpitch && w.ppitch >= kMaxFusedGrid,
          "pitches V=%d", V);
    // forced narrow tiles of the fused plans: never more tiles than records fit in a row
    for (int C : {0, 1, 5, 100, 2224, 4095, 4096, V / 2, V})
        for (int forced : {0, 1, 3, 9, 16, 40}) {
            if (C > V) continue;
            const int tn = select_tile_width(C, forced, w.ppitch);
            CHECK(tn >= 1 && tn <= 16, "tile width %d", tn);
            CHECK(((int64_t)C + tn - 1) / tn <= w.ppitch, "tiles beyond the record pitch (C=%d forced=%d V=%d)", C, forced, V);
        }
    // the largest index any kernel forms: row R-1, last column / last tile
    CHECK((R - 1) * (size_t)w.cpitch + (size_t)V - 1 < R * (size_t)w.cpitch, "logit index");
    CHECK((size_t)(((size_t)V + 15) / 16) <= (size_t)w.ppitch, "tile count exceeds the record pitch V=%d", V);
}

// the LDS regions of build_presence_bitmap / k_candidates / k_cand_logits, as the kernels lay them out
static void check_candidate_lds(int V, int d, int P, int K, int W, int B) {
    const int mn = candidates_min_stage(d);
    CHECK(mn >= d && mn % 4 == 0, "min stage d=%d", d);
    for (int stage : {mn, mn + 4 * 1000, (int)((kLdsLimit / 4 - (bitmap_words_padded(V) + (size_t)P * K + 3 * kCandThreads + 64)) & ~(size_t)3)}) {
        if (stage < mn) continue;
        const size_t total = candidates_lds_words(V, P, K, stage);
        if (total * 4 > kLdsLimit) continue;   // the host refuses such a plan
        const size_t bmw = bitmap_words_padded(V);
        CHECK(bmw * 32 >= (size_t)V && bmw % 4 == 0, "bitmap words V=%d", V);
        const size_t stage_at = bmw, perms_at = stage_at + stage, start_at = perms_at + (size_t)P * K;
        const size_t band_at = start_at + kCandThreads, pref_at = band_at + kCandThreads, wsum_at = pref_at + kCandThreads;
        CHECK(wsum_at + 64 == total, "candidate regions do not add up (V=%d P=%d K=%d)", V, P, K);
        CHECK(stage_at % 4 == 0, "stage not 16-byte aligned");
        const int rows = candidates_rows_per_chunk(B, d, W, stage);
        CHECK(rows >= 1 && rows <= B, "rows per chunk %d (B=%d)", rows, B);
        CHECK((size_t)rows * d <= (size_t)stage, "chunk of %d rows x %d does not fit a stage of %d", rows, d, stage);
        CHECK(rows * W <= kCandThreads, "pairs of a chunk exceed the workgroup (rows=%d W=%d)", rows, W);
        CHECK(rows * P <= kCandThreads || true, "-");
        // fused kernel: prefix array and reduction buffer behind the candidate regions; the
        // selection's shared state from the start
        const size_t fused = fused_lds_words(V, P, K, stage);
        CHECK(total + kFusedTileIdWords + (size_t)kFusedWaves * 4 * kWave <= fused, "fused regions (V=%d)", V);
        CHECK(total % 4 == 0 || true, "-");
        CHECK(fused >= kSelSharedWords, "fused LDS smaller than the selection's state");
        // k_candidates reuses the stage for the dense-word list: stage / 2 entries of 8 bytes
        CHECK((size_t)(stage / 2) * 2 <= (size_t)stage, "dense list");
    }
    const size_t un = union_logits_lds_words(V);
    CHECK(bitmap_words_padded(V) + 64 + kFusedTileIdWords + (size_t)kFusedWaves * 4 * kWave <= un, "union regions V=%d", V);
    CHECK(un >= kSelSharedWords, "union LDS smaller than the selection's state");
    CHECK(union_compact_lds_words(V) == (size_t)bitmap_words_padded(V) + 64 + 2 * (size_t)kUnionDenseCap, "union compact V=%d", V);
}

static void check_hit_rows(int V, int d, int P) {
    const int vq = hit_slice_words(V);
    CHECK(vq % 128 == 0 && (size_t)vq * kHitSlices >= (size_t)V, "slices do not cover V=%d", V);
    CHECK((size_t)vq * (kHitSlices - 1) < (size_t)V + 128 * kHitSlices, "slices far beyond V=%d", V);
    const size_t fixed = hit_rows_fixed_lds_words(V, d, P);
    const size_t counters = (size_t)vq / 2, row = (size_t)((d + 3) & ~3), codes = ((size_t)P + 1) / 2;
    CHECK(counters + row + codes + 32 + (kCandThreads + 64) + 2 * (size_t)kCandThreads <= fixed,
          "hit-row regions exceed their size (V=%d d=%d P=%d)", V, d, P);
}

static void check_hlds(int S, int rows, int d) {
    for (int waves : {8, 16})
        for (bool planes : {false, true}) {
            const size_t bytes = hlds_lds_bytes(S, rows, d, waves, planes);
            const size_t pref = (size_t)((S + 1 + 3) & ~3), red = (size_t)waves * 4 * kWave;
            const size_t hidden = planes ? (size_t)rows * hlds_pitch_planes(d) * 6 : (size_t)rows * hlds_pitch(d) * 4;
            CHECK((pref + red) * 4 + hidden == bytes, "hlds regions (S=%d rows=%d d=%d)", S, rows, d);
            CHECK(hlds_pitch(d) >= d && hlds_pitch(d) % 32 == 4, "hlds pitch d=%d", d);
            CHECK(hlds_pitch_planes(d) >= d && hlds_pitch_planes(d) % 64 == 8, "plane pitch d=%d", d);
            CHECK(((pref + red) * 4) % 16 == 0, "hidden rows not 16-byte aligned in LDS");
        }
}

// k_logits_stream: its regions in LDS, which the kernel takes from the same constants; and the tiles of a sentence dealt to
// the XCDs, each once.
template <int MT, int KSN> static void check_stream_regions() {
    using L = StreamLds<MT, KSN>;
    // partial tiles [wave][tile][row group][register][lane], rings [wave][place][load][64 lanes of 16 bytes], candidates
    CHECK(L::kRed == sizeof(float[4][L::GT][MT][4][kWave]) && L::kRings == sizeof(char[4][L::RING][L::NI][kWave][16]) &&
          L::kPref - L::kIds == sizeof(int32_t[2][kStreamTiles][kTileN]), "stream regions (MT=%d KSN=%d)", MT, KSN);
    CHECK(L::kRed % 16 == 0 && L::kIds % 16 == 0 && L::kPref % 16 == 0 && L::kIds == L::kRed + L::kRings, "stream regions (MT=%d KSN=%d)", MT, KSN);
    CHECK(L::kPref + sizeof(uint32_t[kWave]) == L::kBytes && kWave * kWave >= kMaxSentencesLogits, "sentences in front (MT=%d KSN=%d)", MT, KSN);
    CHECK(L::kBytes <= kLdsLimit / 2, "two workgroups do not share a CU (MT=%d KSN=%d)", MT, KSN);
}
static void check_stream() {
    check_stream_regions<1, 1>(); check_stream_regions<1, 2>(); check_stream_regions<1, 4>();
    check_stream_regions<2, 1>(); check_stream_regions<2, 2>(); check_stream_regions<2, 4>();
}
// Counts the tiles of a run.
static void take(const TileRun& r, std::vector<int>& seen) {
    for (uint32_t u = 0; u < r.n; ++u) {
        CHECK(r.tile(u) < seen.size() && (u == 0 || r.tile(u) > r.tile(u - 1)), "tile %u of %zu", r.tile(u), seen.size());
        if (r.tile(u) < seen.size()) ++seen[r.tile(u)];
    }
}
// Sentences dealt to workgroups: every workgroup has one sentence, every sentence a workgroup at least, and all its
// tiles are taken once.
static void check_dealt() {
    for (uint32_t G : {1u, 2u, 21u, 64u, 96u})
        for (uint32_t S = 1; S <= 8 * G; S += S < 40 ? 1 : S < 8 * G - 4 ? 13 : 1) {
            std::vector<uint32_t> all(S, 0);
            for (uint32_t x = 0; x < 8; ++x) {
                CHECK(dealt_from(0, x, S, G) == 0 && dealt_from(S, x, S, G) == G, "S=%u G=%u", S, G);
                for (uint32_t s = 0; s < S; ++s) {
                    const uint32_t b0 = dealt_from(s, x, S, G), b1 = dealt_from(s + 1, x, S, G);
                    all[s] += b1 - b0;
                    for (uint32_t b = b0; b < b1; ++b) CHECK(dealt_sentence(b, x, S, G) == s, "workgroup %u of XCD %u (S=%u G=%u)", b, x, S, G);
                }
            }
            for (uint32_t s = 0; s < S; ++s) CHECK(all[s] >= 8 * G / S && all[s] <= 8 * G / S + 1, "sentence %u has %u workgroups (S=%u G=%u)", s, all[s], S, G);
            for (uint32_t s : {0u, S / 2, S - 1})
                for (uint32_t n : {0u, 1u, 9u, 130u, 1003u})
                    for (uint32_t shared : {0u, 1u, 62u, 5000u}) {
                        std::vector<int> seen(n, 0);
                        uint32_t before = 0;
                        for (uint32_t x = 0; x < 8; ++x) {
                            const uint32_t mine = dealt_from(s + 1, x, S, G) - dealt_from(s, x, S, G);
                            for (uint32_t i = 0; i < mine; ++i) take(dealt_run(n, shared, i, mine, before, all[s]), seen);
                            before += mine;
                        }
                        for (uint32_t i = 0; i < n; ++i) CHECK(seen[i] == 1, "tile %u of %u dealt %d times (S=%u G=%u)", i, n, seen[i], S, G);
                    }
        }
}
// Sentences dealt to workgroups by their lists' lengths, where the kernel does so: every workgroup is of one sentence, every
// sentence has one at least, all its tiles are taken once, and none takes twice its share of the weights.
static void check_dealt_by_count() {
    int unequal = 0;
    uint64_t rnd = 0x9E3779B97F4A7C15ull;
    for (uint32_t G : {8u, 32u, 60u, 64u, 96u, 192u})
        for (uint32_t S : {2u, 3u, 8u, 33u, 64u, 65u, 100u, 384u, 768u})
            for (int kind = 0; kind < 6; ++kind) {
                std::vector<uint32_t> n(S), weight(S), front(S + 1, 0);
                uint32_t most = 0, sum = 0;
                for (uint32_t s = 0; s < S; ++s) {
                    rnd ^= rnd << 13; rnd ^= rnd >> 7; rnd ^= rnd << 17;
                    n[s] = kind == 0 ? 100 : kind == 1 ? (s == S / 2 ? 2000 : 150) : kind == 2 ? (s ? 0 : 777) : kind == 3 ? (s % 5 ? 1 : 5000)
                         : kind == 4 ? (uint32_t)(rnd >> 54) * (uint32_t)(rnd % 7 == 0) * 20 : (s + 1 == S ? 1u << 20 : 3);
                    most = std::max(most, n[s]);
                    sum += n[s];
                }
                if (!dealt_by_count(most, sum, S, G, 1000)) continue;
                CHECK(!dealt_by_count(most, sum, S, G, 4000) || (uint64_t)most * S > 2ull * sum, "a line for long rows (S=%u G=%u kind=%d)", S, G, kind);
                ++unequal;
                const uint32_t least = least_weight(sum, S, G);
                for (uint32_t s = 0; s < S; ++s) { weight[s] = std::max(n[s], least); front[s + 1] = front[s] + weight[s]; }
                const uint32_t W = front[S];
                CHECK((uint64_t)W * G + (7ull * W >> 3) < (1ull << 32), "overflow (S=%u G=%u kind=%d)", S, G, kind);
                for (uint32_t s = 0; s < S; ++s) {
                    uint32_t all = 0, before = 0;
                    for (uint32_t x = 0; x < 8; ++x) all += dealt_from(front[s + 1], x, W, G) - dealt_from(front[s], x, W, G);
                    CHECK(all > 0 && (double)n[s] * 8 * G <= 2.0 * all * W, "%u workgroups for %u tiles (S=%u G=%u kind=%d)", all, n[s], S, G, kind);
                    std::vector<int> seen(n[s], 0);
                    for (uint32_t x = 0; x < 8 && all; ++x) {
                        const uint32_t mine = dealt_from(front[s + 1], x, W, G) - dealt_from(front[s], x, W, G);
                        for (uint32_t i = 0; i < mine; ++i) take(dealt_run(n[s], 62, i, mine, before, all), seen);
                        before += mine;
                    }
                    CHECK(std::all_of(seen.begin(), seen.end(), [](int k) { return k == 1; }), "tiles of sentence %u (S=%u G=%u kind=%d)", s, S, G, kind);
                }
            }
    for (uint32_t before : {0u, 1u, 2047u, 4094u})   // the largest list and number of workgroups
        CHECK(dealt_run(1u << 20, 0, 0, 1, before, 4095).b0 == ((uint64_t)before << 20) / 4095, "share %u", before);
    CHECK(unequal > 40 && !dealt_by_count(100, 100, 1, 64, 1000) && !dealt_by_count(1 << 20, 1 << 20, 1, 64, 4000), "%d unequal ones", unequal);
}
// An XCD's tiles by turns, and in pieces.
static void check_xcd_runs() {
    for (uint32_t n : {0u, 1u, 9u, 130u, 1003u})
        for (uint32_t shared : {0u, 1u, 62u, 5000u})
            for (uint32_t every : {1u, 2u, 3u, 64u}) {
                std::vector<int> seen(n, 0), pieces(n, 0);
                for (uint32_t x = 0; x < 8; ++x) {
                    const XcdTiles t = xcd_tiles(n, shared, 0, x);
                    for (uint32_t f = 0; f < every; ++f) take(xcd_run(t, x, f, every, t.n > f ? (t.n - f + every - 1) / every : 0), seen);
                    for (uint32_t f = 0; f < t.n; f += every) take(xcd_run(t, x, f, 1, std::min(every, t.n - f)), pieces);
                }
                for (uint32_t i = 0; i < n; ++i) CHECK(seen[i] == 1 && pieces[i] == 1, "tile %u of %u (every %u)", i, n, every);
            }
}
static void check_xcd_tiles() {
    for (uint32_t n : {0u, 1u, 7u, 8u, 9u, 130u, 1003u})
        for (uint32_t shared : {0u, 1u, 8u, 62u, 125u, 5000u})
            for (uint32_t s : {0u, 3u, 13u}) {
                std::vector<int> seen(n, 0);
                for (uint32_t x = 0; x < 8; ++x) {
                    const XcdTiles t = xcd_tiles(n, shared, s, x);
                    uint32_t before = 0;
                    for (uint32_t i = 0; i < t.n; ++i) {
                        const uint32_t tile = xcd_tile(t, x, i);
                        CHECK(tile < n && (i == 0 || tile > before), "tile %u of %u (XCD %u)", tile, n, x);
                        if (tile < n) ++seen[tile];
                        before = tile;
                    }
                }
                for (uint32_t i = 0; i < n; ++i) CHECK(seen[i] == 1, "tile %u of %u dealt %d times", i, n, seen[i]);
            }
}

// small_div() of the kernels: (int)((x + 0.5f) * r) with r = the hardware's reciprocal of y, which may
// differ from the correctly rounded 1 / y by one unit in the last place; checked here with r two
// units off either way, for every x < 1024 and y <= 1024.
static void check_small_div_margin() {
    for (int y = 1; y <= 1024; ++y) {
        const float exact = 1.0f / (float)y;
        float lo = exact, hi = exact;
        for (int i = 0; i < 2; ++i) { lo = std::nextafterf(lo, 0.0f); hi = std::nextafterf(hi, 2.0f); }
        for (float r : {lo, exact, hi})
            for (int x = 0; x < 1024; ++x)
                CHECK((int)(((float)x + 0.5f) * r) == x / y, "small_div x=%d y=%d", x, y);
    }
}

// nth_set_bit() against a bit-by-bit walk: every rank of a few thousand words (all one-bit and
// two-bit words, dense and random ones).
static void check_nth_set_bit() {
    std::vector<uint32_t> words = {0xFFFFFFFFu, 0x80000000u, 0x00000001u, 0xAAAAAAAAu, 0x55555555u, 0xFFFF0000u, 0x0000FFFFu};
    for (int a = 0; a < 32; ++a)
        for (int b = a; b < 32; ++b) words.push_back((1u << a) | (1u << b));
    uint64_t x = 0x9E3779B97F4A7C15ull;
    for (int i = 0; i < 4000; ++i) { x ^= x << 13; x ^= x >> 7; x ^= x << 17; words.push_back((uint32_t)(x >> 16)); }
    for (uint32_t w : words) {
        uint32_t r = 0;
        for (uint32_t bit = 0; bit < 32; ++bit)
            if (w >> bit & 1u) { CHECK(nth_set_bit(w, r) == bit, "nth_set_bit(%08x, %u)", w, r); ++r; }
    }
}

// The places that builds report to: one that no kernel was given comes back (a build that runs out of memory has one and
// launches nothing), one that may still be written to does not.
static void check_reports() {
    static uint32_t page[Report::kPlaces * Report::kWords];
    Report::page = page;   // (there is no GPU to pin it for)
    for (int i = 0; i < 3 * Report::kPlaces; ++i) {
        Report r;
        CHECK(r.take() == hipSuccess && r.place == 0 && r.words == page, "place %d after %d builds", r.place, i);
    }
    {
        Report r, q;
        CHECK(r.take() == hipSuccess && q.take() == hipSuccess && r.place == 0 && q.place == 1, "places %d, %d", r.place, q.place);
        r.idle = false;
    }
    Report r;
    CHECK(r.take() == hipSuccess && r.place == 1, "place %d", r.place);
}

// "bytes of an element, hidden rows, beams, V, d, pitch" from stdin: waves and rounds of k_logits_pass, 0 0 where k_logits_few has the call.
static int print_pass_plans() {
    int size, R, B, V, d;
    long long ld;
    while (std::scanf("%d %d %d %d %d %lld", &size, &R, &B, &V, &d, &ld) == 6) {
        const PassPlan p = size == 2 ? pass_plan<uint16_t>(R, B, V, d, ld) : pass_plan<float>(R, B, V, d, ld);
        std::printf("%d %d\n", p.waves, p.rounds);
    }
    return 0;
}

// Every word has its wave and round, at most 256 workgroups, the operands in LDS and 32-bit offsets.
template <typename ET>
static void check_pass(int R, int V, int d, int64_t ld) {
    const PassPlan p = pass_plan<ET>(R, std::min(R, 12), V, d, ld);
    if (!p.waves) return;
    const int tiles = (V + kTileN - 1) / kTileN, groups = (R + kTileM - 1) / kTileM;
    const int64_t words = (int64_t)p.waves * p.rounds * kTileN;
    CHECK(p.waves >= 4 && p.waves <= kPassWaves && words * 256 >= V, "R=%d V=%d d=%d", R, V, d);
    CHECK((int64_t)p.waves * p.rounds <= (tiles + 255) / 256 + 4 * p.rounds, "R=%d V=%d d=%d", R, V, d);
    CHECK(groups <= pass_most_tiles<ET>() && pass_lds_bytes<ET>(groups, d) <= kLdsLimit && pass_pitch<ET>(d) >= d, "R=%d V=%d d=%d", R, V, d);
    CHECK((kTileN - 1) * ld * (int64_t)sizeof(ET) + d * (int64_t)sizeof(ET) < (int64_t)1 << 31, "R=%d V=%d d=%d", R, V, d);
}

int main(int argc, char**) {
    if (argc > 1) return print_pass_plans();
    check_reports();
    check_small_div_margin();
    check_nth_set_bit();
    // workspace: the largest accepted S, B, V and their neighbours, ragged V
    for (int V : {1, 15, 16, 17, 63, 64, 65, 1000, 40000, 100000, 200000, (1 << 24) - 1, 1 << 24})
        for (int S : {1, 2, 64, 4096})
            for (int B : {1, 12, 17, 50, 256})
                for (bool full : {false, true}) {
                    if ((size_t)S * B * V > ((size_t)1 << 45)) continue;   // (keeps sizes below 2^48 bytes)
                    check_workspace(S, B, V, full);
                }
    check_workspace(4096, 256, 1 << 20, false);
    check_workspace(1, 256, 1 << 24, false);
    check_workspace(4096, 1, 1 << 24, true);
    // LDS plans: vocabulary sizes up to what fits a bitmap in LDS, odd hidden sizes, many codes
    for (int V : {1, 31, 32, 33, 1000, 40000, 100000, 200000, 1000000})
        for (int d : {8, 50, 64, 77, 1000, 1024, 1026, 4099, 20000})
            for (int W : {1, 4, 8, 16, 500, 1024})
                for (int K : {2, 8, 16}) {
                    if (K > d) continue;
                    const int P = W * 3;
                    for (int B : {1, 12, 29, 32, 50, 256}) check_candidate_lds(V, d, P, K, W, B);
                    check_hit_rows(V, d, P);
                }
    for (int S : {1, 32, 64, 4096})
        for (int rows : {1, 10, 16, 32})
            for (int d : {8, 50, 1000, 1024, 1026, 4099}) check_hlds(S, rows, d);
    for (int R : {1, 16, 17, 32, 33, 48, 49})
        for (int V = 8200; V < 600000; V += V / 37)
            for (int d : {8, 16, 255, 256, 600, 1000, 1536, 4000})
                for (int64_t ld : {(int64_t)d, (int64_t)d + 3, (int64_t)1 << 24, (int64_t)1 << 26}) {
                    check_pass<float>(R, V, d, ld);
                    check_pass<uint16_t>(R, V, d, ld);
                }
    check_stream();
    check_xcd_tiles();
    check_xcd_runs();
    check_dealt();
    check_dealt_by_count();
    CHECK(2 * rows_lds_bytes(5) <= kLdsLimit && 2 * few_lds_bytes<float>(3) <= kLdsLimit && 2 * few_lds_bytes<uint16_t>(2) <= kLdsLimit,
          "full-vocabulary kernels: two workgroups do not share a CU");
    CHECK(estage_lds_bytes() <= kLdsLimit, "estage LDS");
    CHECK(sizeof(SelShared) + 1024 <= 64 * 1024, "static LDS of the selection kernel");
    CHECK(kSelSharedWords * 4 >= sizeof(SelShared), "selection state words");
    if (failures) {
        std::printf("%d check(s) failed\n", failures);
        return 1;
    }
    std::printf("host plans ok\n");
    return 0;
}
