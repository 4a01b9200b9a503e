// The host planner (csrc/plan.cpp) under AddressSanitizer and UndefinedBehaviorSanitizer: plans for ragged,
// rectangular, scattered, strided and long-row masks, every tile size, every kernel choice, with and without
// gathered tiles, every export, both work orders, the wave form's lists and orders.  The device side is stubbed out (plans stay host-only).  Built and run by
// tests/test_planner_sanitizers.py.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "smha.h"
#include "smha_internal.hpp"
using namespace smha;
namespace smha {
smha_status_t upload_plan(smha_plan *, int) { return SMHA_OK; }
void release_device(smha_plan *) {}
int current_device_or_negative() { return -1; }
smha_status_t pack_device_mask(const uint8_t *, int, int, int, uint64_t *) { return SMHA_ERR_HIP; }
smha_status_t classify_device_mask(const uint8_t *, int, int, int, std::vector<TileInfo> &, std::vector<std::vector<uint64_t>> &) { return SMHA_ERR_HIP; }
}
static uint64_t rng_state = 12345;
static uint32_t rnd() { rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(rng_state >> 33); }
static void expect(bool ok, const char *what) {
    if (ok) return;
    printf("failed: %s\n", what);
    exit(1);
}
// The wave form's lists: made for the first call that takes the form, not with the plan; each entry's keys are those that any
// of its 32 rows has; every order hands each wave at most 64 entries and covers each entry once.
static void wave_form(smha_plan_t *p, int B, int H) {
    expect(!p->wave.counted && !p->wave.made, "nothing of the wave form's lists is made with the plan");
    int alone = 0;
    for (int D : {64, 128, 256})
        for (int form : {1, 3})
            if (p->has_block && (form == 1 || D > 64)) wave_form_pays(p, 0, form, B, H, D, alone);
    expect(!p->wave.made, "nor for an estimate");
    if (!count_wave_lists(p)) return;
    const WaveLists &wl = p->wave;
    int64_t n_items = 0, n_ents = 0;
    for (int n = 0; n <= kWaveWhole; ++n) { n_items += wl.of_length[n]; n_ents += (int64_t)n * wl.of_length[n]; }
    expect(n_ents == wl.n_ents, "the lengths add up");
    make_wave_lists(p);
    expect((int64_t)wl.items.size() == n_items && (int64_t)wl.ents.size() == n_ents + 1 && wl.used.size() == wl.ents.size(), "as many as counted");
    const int n_masks = p->Bm * p->Hm;
    int slots = 0, splits = 0;
    int64_t part = 0;
    for (int mi = 0; mi < n_masks; ++mi) {
        int s = 0, top = 0;
        for (int i = 0; i < wl.item_cnt[mi]; ++i) {
            const WaveItem &it = wl.items[wl.item_off[mi] + i];
            s += it.slot >= 0;
            top = std::max(top, it.split + 1);
            for (int e = it.begin; e < it.begin + it.n; ++e) {
                uint32_t any = 0xFFFFFFFFu;
                if (wl.ents[e].code >= 0) {
                    any = 0;
                    ++part;
                    for (int r = 0; r < 32; ++r)
                        any |= (uint32_t)(p->h_kt_bitmap[(size_t)wl.ents[e].code * 64 + 32 * (it.rg & 1) + r] >> (wl.ents[e].key & 32));
                }
                expect(any != 0 && any == wl.used[e], "the keys that any row of an entry has");
            }
        }
        slots = std::max(slots, s);
        splits = std::max(splits, top);
    }
    expect(slots == wl.max_slots && splits == wl.max_splits && part == wl.part_ents, "slots, split groups and partly filled entries as counted");
    for (int limit : {1, 2, 12, 64}) {
        std::vector<int32_t> table;
        const int wgs = build_wave_order(p, limit, table);
        expect(table.size() == (size_t)wgs * n_masks * 32, "four records of eight words a workgroup");
        const WaveItem *rec = reinterpret_cast<const WaveItem *>(table.data());
        std::vector<int> seen(wl.ents.size(), 0);
        for (size_t i = 0; i < (size_t)wgs * n_masks * 4; ++i) {
            expect(rec[i].n >= 0 && rec[i].n <= 64 && rec[i].begin >= 0 && (size_t)rec[i].begin + rec[i].n < wl.ents.size() + 1, "a wave's entries");
            expect(rec[i].team == rec[i / 4 * 4].team && (rec[i].team == 0 || rec[i].rg >= 0), "a team is a whole workgroup");
            expect(rec[i].n == 0 || (rec[i].key0 == wl.ents[rec[i].begin].key && rec[i].code0 == wl.ents[rec[i].begin].code), "the first entry's words");
            for (int e = 0; e < rec[i].n; ++e) ++seen[rec[i].begin + e];
        }
        for (int64_t e = 0; e < n_ents; ++e) expect(seen[e] == 1, "each entry once");
    }
}
static void exports(smha_plan_t *p, int n_masks) {
    smha_plan_info_t shape;
    if (smha_plan_info(p, &shape) == SMHA_OK) wave_form(p, shape.Bm == 1 ? 3 : shape.Bm, shape.Hm == 1 ? 9 : shape.Hm);
    for (int which = 0; which <= 17; ++which)
        for (int mi = 0; mi < n_masks; ++mi) {
            size_t need = 0;
            if (smha_plan_export(p, mi, (smha_export_t)which, nullptr, 0, &need) != SMHA_OK) continue;
            std::vector<char> buf(need + 1);
            smha_plan_export(p, mi, (smha_export_t)which, buf.data(), need, &need);
        }
    // the work order, both grains, for a few batch and head counts the plan's masks allow
    smha_plan_info_t info;
    if (smha_plan_info(p, &info) != SMHA_OK) return;
    for (int d : {8, 64, 128, 256, 12}) {  // the row kernel's form (refused without the row format)
        int rows = 0, keys = 0;
        if (smha_plan_row_form(p, info.Bm, info.Hm == 1 ? 9 : info.Hm, d, &rows, &keys) == SMHA_OK && (rows < 1 || keys < 2)) abort();
    }
    for (int fine = 0; fine < 2; ++fine)
        for (int B : {info.Bm, info.Bm == 1 ? 3 : info.Bm})
            for (int H : {info.Hm, info.Hm == 1 ? 9 : info.Hm})
                for (int slots : {1, 7, 128}) {
                    size_t need = 0;
                    int per = 0;
                    if (smha_plan_work_order(p, B, H, slots, fine, nullptr, 0, &need, &per) != SMHA_OK) continue;
                    std::vector<int32_t> buf(need);
                    smha_plan_work_order(p, B, H, slots, fine, buf.data(), need, &need, &per);
                    if (smha_plan_call_order(p, B, H, slots, fine, nullptr, 0, &need, &per) != SMHA_OK) continue;
                    buf.assign(need, 0);
                    smha_plan_call_order(p, B, H, slots, fine, buf.data(), need, &need, &per);
                }
}
int main() {
    int n = 0;
    for (int Sq : {1, 65, 130, 700}) for (int Sk : {1, 100, 777, 3000}) for (int variant = 0; variant < 5; ++variant) {
        std::vector<uint8_t> m((size_t)2 * Sq * Sk);
        for (size_t i = 0; i < m.size(); ++i) {
            const int r = (int)((i / Sk) % Sq), c = (int)(i % Sk);
            switch (variant) {
                case 0: m[i] = rnd() % 100 < 30; break;
                case 1: m[i] = rnd() % 1000 < 3; break;                       // scattered
                case 2: m[i] = (c % 37 == 5) || (c <= r && r - c < 70); break; // strided + band
                case 3: m[i] = c % 5 == 2; break;                              // many gathered tiles
                default: m[i] = (r < 64) || (c < 8) || (rnd() % 1000 < 2); break;
            }
        }
        for (int block : {16, 32, 64}) for (int force : {0, 1, 2}) for (int ng : {0, 1}) {
            smha_plan_opts_t o{}; o.block = block; o.force = force; o.device_id = -2; o.no_gather = ng; o.build_both = (variant == 0 && force == 0);
            o.head_dim = (n & 1) ? 128 : 64;
            smha_plan_t *p = nullptr;
            if (smha_plan_from_dense_rect(m.data(), 0, 1, 2, Sq, Sk, &o, &p) != SMHA_OK) { printf("plan failed\n"); return 1; }
            smha_plan_info_t info; smha_plan_info(p, &info);
            exports(p, 2);
            smha_plan_destroy(p);
            ++n;
        }
    }
    // descriptions
    for (int S : {100, 1000, 4100}) {
        smha_mask_desc_t d{}; d.flags = SMHA_MASK_BIGBIRD | SMHA_MASK_PADDING; d.block = 64; d.n_window_blocks = 3; d.n_global_blocks = 2; d.n_random_blocks = 3; d.seed = 5;
        int32_t vl[2] = {S - 17, S / 2}; d.valid_len = vl; d.per_head = 1;
        smha_plan_opts_t o{}; o.device_id = -2; o.head_dim = 128;
        smha_plan_t *p = nullptr;
        if (smha_plan_from_desc(&d, 2, 3, S, &o, &p) != SMHA_OK) { printf("desc plan failed\n"); return 1; }
        exports(p, 6); smha_plan_destroy(p); ++n;
        smha_mask_desc_t e{}; e.flags = SMHA_MASK_CAUSAL | SMHA_MASK_STRIDED | SMHA_MASK_WINDOW; e.window_left = 127; e.stride = 64;
        if (smha_plan_from_desc(&e, 1, 1, S, &o, &p) != SMHA_OK) { printf("desc plan failed\n"); return 1; }
        exports(p, 1); smha_plan_destroy(p); ++n;
    }
    printf("%d plans built and exported under the sanitizers\n", n);
    return 0;
}
