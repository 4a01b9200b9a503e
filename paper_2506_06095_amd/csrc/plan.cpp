// Host-side mask analysis: dense mask or pattern description -> per-row format, two-level
// block format (Sec. 4.2.1 of the paper), kernel selection (Sec. 4.2.3) and the block
// kernel's work lists.  Integer work only; runs without a GPU.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <thread>
#include <utility>
#include <vector>

#include "smha_internal.hpp"

namespace smha {
namespace {

// ---------------------------------------------------------------------------------------
// Row sources: produce one mask row as a bit string (bit j of word j/64 = entry (i, j)).
// ---------------------------------------------------------------------------------------
struct RowSource {
    virtual ~RowSource() = default;
    virtual void row_bits(int i, uint64_t *words) const = 0;  // words[W], W = ceil(Sk/64)
};

inline void set_range(uint64_t *w, int lo, int hi) {  // bits [lo, hi)
    if (lo >= hi) return;
    int wl = lo >> 6, wh = (hi - 1) >> 6;
    uint64_t ml = ~0ull << (lo & 63);
    uint64_t mh = ~0ull >> (63 - ((hi - 1) & 63));
    if (wl == wh) {
        w[wl] |= ml & mh;
        return;
    }
    w[wl] |= ml;
    for (int t = wl + 1; t < wh; ++t) w[t] = ~0ull;
    w[wh] |= mh;
}

inline void keep_below(uint64_t *w, int W, int n) {  // clear bits >= n
    int full = n >> 6;
    if (full < W) {
        int rem = n & 63;
        if (rem) {
            w[full] &= ~0ull >> (64 - rem);
            ++full;
        }
        for (int t = full; t < W; ++t) w[t] = 0;
    }
}

struct DenseSource final : RowSource {
    const uint8_t *m;
    int S, W;
    DenseSource(const uint8_t *mask, int S_) : m(mask), S(S_), W((S_ + 63) / 64) {}
    void row_bits(int i, uint64_t *words) const override {
        const uint8_t *r = m + (size_t)i * S;
        int j = 0;
        for (int t = 0; t < W; ++t) {
            uint64_t out = 0;
            for (int byte = 0; byte < 8 && j < S; ++byte) {
                if (j + 8 <= S) {
                    uint64_t x;
                    std::memcpy(&x, r + j, 8);
                    // any nonzero byte -> its bit 0, then gather the eight bit-0s
                    x |= x >> 4;
                    x |= x >> 2;
                    x |= x >> 1;
                    x &= 0x0101010101010101ull;
                    out |= ((x * 0x0102040810204080ull) >> 56) << (8 * byte);
                    j += 8;
                } else {
                    for (int b = 0; j < S; ++b, ++j)
                        if (r[j]) out |= 1ull << (8 * byte + b);
                }
            }
            words[t] = out;
        }
    }
};

// bit rows that were packed elsewhere (on the GPU, for a device mask)
struct BitSource final : RowSource {
    const uint64_t *w;
    int W;
    BitSource(const uint64_t *words, int S_) : w(words), W((S_ + 63) / 64) {}
    void row_bits(int i, uint64_t *words) const override { std::memcpy(words, w + (size_t)i * W, sizeof(uint64_t) * W); }
};

inline uint64_t mix64(uint64_t x) {  // splitmix64 output function
    x += 0x9E3779B97F4A7C15ull;
    uint64_t z = x;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

inline uint64_t block_hash(uint64_t seed, uint64_t head, uint32_t br, uint32_t bc) {
    uint64_t key = mix64(seed ^ mix64(head));
    return mix64(key ^ (((uint64_t)br << 32) | bc));
}

struct DescSource final : RowSource {
    smha_mask_desc_t d;
    int S, W, valid;
    std::vector<std::vector<int32_t>> keep;  // per block row of d.block: kept block columns
    DescSource(const smha_mask_desc_t &desc, int S_, int head, int valid_)
        : d(desc), S(S_), W((S_ + 63) / 64), valid(valid_) {
        if (!(d.flags & (SMHA_MASK_BLOCK_RANDOM | SMHA_MASK_BIGBIRD))) return;
        const int bs = d.block, nb = (S + bs - 1) / bs;
        keep.resize(nb);
        std::vector<uint8_t> row(nb);
        std::vector<std::pair<uint64_t, int32_t>> cand;
        for (int br = 0; br < nb; ++br) {
            std::fill(row.begin(), row.end(), 0);
            if (d.flags & SMHA_MASK_BLOCK_RANDOM) {
                for (int bc = 0; bc < nb; ++bc) {
                    double u = (double)(block_hash(d.seed, head, br, bc) >> 11) *
                               (1.0 / 9007199254740992.0);
                    if (bc == br || u < d.keep_p) row[bc] = 1;
                }
            }
            if (d.flags & SMHA_MASK_BIGBIRD) {
                std::vector<uint8_t> bb(nb, 0);
                const int half = (d.n_window_blocks - 1) / 2;
                if (d.n_window_blocks > 0)
                    for (int bc = std::max(0, br - half); bc < std::min(nb, br + half + 1); ++bc)
                        bb[bc] = 1;
                for (int bc = 0; bc < std::min(nb, d.n_global_blocks); ++bc) bb[bc] = 1;
                if (br < d.n_global_blocks) std::fill(bb.begin(), bb.end(), 1);
                cand.clear();
                for (int bc = 0; bc < nb; ++bc)
                    if (!bb[bc]) cand.emplace_back(block_hash(d.seed, head, br, bc), bc);
                std::sort(cand.begin(), cand.end());
                for (int t = 0; t < (int)cand.size() && t < d.n_random_blocks; ++t)
                    bb[cand[t].second] = 1;
                for (int bc = 0; bc < nb; ++bc) row[bc] |= bb[bc];
            }
            for (int bc = 0; bc < nb; ++bc)
                if (row[bc]) keep[br].push_back(bc);
        }
    }
    void row_bits(int i, uint64_t *w) const override {
        std::memset(w, 0, sizeof(uint64_t) * W);
        const uint32_t f = d.flags;
        const uint32_t additive = f & (SMHA_MASK_WINDOW | SMHA_MASK_GLOBAL | SMHA_MASK_STRIDED |
                                       SMHA_MASK_BLOCK_RANDOM | SMHA_MASK_BIGBIRD);
        if (!additive) set_range(w, 0, S);
        if (f & SMHA_MASK_WINDOW) {
            int64_t lo = (int64_t)i - d.window_left, hi = (int64_t)i + d.window_right + 1;
            set_range(w, (int)std::max<int64_t>(0, lo), (int)std::min<int64_t>(S, hi));
        }
        if (f & SMHA_MASK_GLOBAL) set_range(w, 0, i < d.n_global ? S : std::min(S, d.n_global));
        if (f & SMHA_MASK_STRIDED)
            for (int j = d.stride_phase; j < S; j += d.stride) w[j >> 6] |= 1ull << (j & 63);
        if (!keep.empty()) {
            const int bs = d.block;
            for (int32_t bc : keep[i / bs])
                set_range(w, bc * bs, std::min<int64_t>(S, (int64_t)(bc + 1) * bs));
        }
        if (f & SMHA_MASK_CAUSAL) keep_below(w, W, i + 1);
        if (f & SMHA_MASK_PADDING) keep_below(w, W, i < valid ? valid : 0);
    }
};

// ---------------------------------------------------------------------------------------
// One stripe = 64 consecutive mask rows.  Everything downstream is derived from its bits.
// ---------------------------------------------------------------------------------------
struct Stripe {
    int32_t row_nnz[64];
    std::vector<int32_t> cols;                // per-row format, rows concatenated
    std::vector<int32_t> load_col[4];         // per block row inside the stripe (64/block of them)
    std::vector<uint8_t> flag[4];
    std::vector<uint64_t> bitmap[4];
    std::vector<int32_t> kt_col, kt_bmp_local;  // 64x64 tiles (only when block != 64)
    std::vector<uint64_t> kt_bitmap;
    int64_t valid16 = 0, nnz = 0;
};

inline uint64_t extract_bits(const uint64_t *row, int c0, int n) {  // n <= 64, c0 % n == 0
    uint64_t w = row[c0 >> 6] >> (c0 & 63);
    return n == 64 ? w : (w & ((1ull << n) - 1));
}

void analyse_stripe(const RowSource &src, int Sq, int Sk, int block, bool want_rows, int stripe,
                    uint64_t *bits /* 64*W */, Stripe &out) {
    const int W = (Sk + 63) / 64;
    const int r0 = stripe * 64;
    for (int r = 0; r < 64; ++r) {
        uint64_t *w = bits + (size_t)r * W;
        if (r0 + r < Sq)
            src.row_bits(r0 + r, w);
        else
            std::memset(w, 0, sizeof(uint64_t) * W);
        int c = 0;
        for (int t = 0; t < W; ++t) c += __builtin_popcountll(w[t]);
        out.row_nnz[r] = c;
        out.nnz += c;
    }
    if (want_rows) {
        out.cols.reserve(out.nnz);
        for (int r = 0; r < 64; ++r) {
            const uint64_t *w = bits + (size_t)r * W;
            for (int t = 0; t < W; ++t) {
                uint64_t x = w[t];
                while (x) {
                    out.cols.push_back(t * 64 + __builtin_ctzll(x));
                    x &= x - 1;
                }
            }
        }
    }
    // non-empty 16x16 tiles (input of the paper's Eq. 1)
    for (int g = 0; g < 4; ++g) {
        if (r0 + g * 16 >= Sq) break;
        for (int t = 0; t < W; ++t) {
            uint64_t any = 0;
            for (int r = 0; r < 16; ++r) any |= bits[(size_t)(g * 16 + r) * W + t];
            for (int q = 0; q < 4; ++q)
                if ((any >> (16 * q)) & 0xFFFF) ++out.valid16;
        }
    }
    // tiles of edge `block`
    const int nb = (Sk + block - 1) / block;
    const int per = 64 / block;
    for (int sub = 0; sub < per; ++sub) {
        if (r0 + sub * block >= Sq) break;
        for (int bc = 0; bc < nb; ++bc) {
            uint64_t words[64];
            int cnt = 0;
            for (int r = 0; r < block; ++r) {
                words[r] = extract_bits(bits + (size_t)(sub * block + r) * W, bc * block, block);
                cnt += __builtin_popcountll(words[r]);
            }
            if (!cnt) continue;
            out.load_col[sub].push_back(bc);
            const bool full = cnt == block * block;
            out.flag[sub].push_back(full ? 1 : 0);
            if (!full) out.bitmap[sub].insert(out.bitmap[sub].end(), words, words + block);
        }
    }
    if (block != 64) {
        for (int kt = 0; kt < W; ++kt) {
            uint64_t words[64];
            int cnt = 0;
            for (int r = 0; r < 64; ++r) {
                words[r] = bits[(size_t)r * W + kt];
                cnt += __builtin_popcountll(words[r]);
            }
            if (!cnt) continue;
            out.kt_col.push_back(kt);
            if (cnt == 64 * 64) {
                out.kt_bmp_local.push_back(-1);
            } else {
                out.kt_bmp_local.push_back((int32_t)(out.kt_bitmap.size() / 64));
                out.kt_bitmap.insert(out.kt_bitmap.end(), words, words + 64);
            }
        }
    }
}

smha_status_t analyse_mask(const RowSource &src, int Sq, int Sk, int block, bool want_rows,
                           MaskFormats &mf) {
    const int W = (Sk + 63) / 64;
    const int n_stripes = (Sq + 63) / 64;
    std::vector<Stripe> stripes(n_stripes);
    std::atomic<int> next{0};
    std::atomic<bool> failed{false};
    int n_threads = (int)std::min<unsigned>(std::max(1u, std::thread::hardware_concurrency()), 16u);
    n_threads = std::min(n_threads, n_stripes);
    if ((int64_t)Sq * Sk < (1 << 20)) n_threads = 1;
    auto work = [&]() {
        try {
            std::vector<uint64_t> bits((size_t)64 * W);
            for (;;) {
                int s = next.fetch_add(1);
                if (s >= n_stripes) break;
                analyse_stripe(src, Sq, Sk, block, want_rows, s, bits.data(), stripes[s]);
            }
        } catch (const std::bad_alloc &) {
            failed = true;
        }
    };
    if (n_threads <= 1) {
        work();
    } else {
        std::vector<std::thread> pool;
        for (int t = 0; t < n_threads; ++t) pool.emplace_back(work);
        for (auto &t : pool) t.join();
    }
    if (failed) return SMHA_ERR_ALLOC;

    const int nbr = (Sq + block - 1) / block;
    const int per = 64 / block;
    mf.load_row_ptr.assign(nbr + 1, 0);
    mf.full_row_ptr.assign(nbr + 1, 0);
    mf.part_row_ptr.assign(nbr + 1, 0);
    if (want_rows) {
        mf.row_ptr.assign(Sq + 1, 0);
        int64_t total = 0;
        for (auto &st : stripes) total += st.nnz;
        if (total > INT32_MAX) return SMHA_ERR_UNSUPPORTED;
        mf.col_idx.reserve(total);
    }
    mf.kt_row_ptr.assign(n_stripes + 1, 0);
    for (int s = 0; s < n_stripes; ++s) {
        Stripe &st = stripes[s];
        mf.nnz += st.nnz;
        mf.n_valid16 += st.valid16;
        if (want_rows) {
            for (int r = 0; r < 64 && s * 64 + r < Sq; ++r)
                mf.row_ptr[s * 64 + r + 1] = mf.row_ptr[s * 64 + r] + st.row_nnz[r];
            mf.col_idx.insert(mf.col_idx.end(), st.cols.begin(), st.cols.end());
        }
        for (int sub = 0; sub < per; ++sub) {
            const int br = s * per + sub;
            if (br >= nbr) break;
            for (size_t e = 0; e < st.load_col[sub].size(); ++e) {
                mf.load_col_idx.push_back(st.load_col[sub][e]);
                mf.flags.push_back(st.flag[sub][e]);
                (st.flag[sub][e] ? mf.full_col_idx : mf.part_col_idx).push_back(st.load_col[sub][e]);
            }
            mf.bitmap.insert(mf.bitmap.end(), st.bitmap[sub].begin(), st.bitmap[sub].end());
            mf.load_row_ptr[br + 1] = (int32_t)mf.load_col_idx.size();
            mf.full_row_ptr[br + 1] = (int32_t)mf.full_col_idx.size();
            mf.part_row_ptr[br + 1] = (int32_t)mf.part_col_idx.size();
        }
        if (block != 64) {
            const int32_t base = (int32_t)(mf.kt_bitmap.size() / 64);
            for (size_t e = 0; e < st.kt_col.size(); ++e) {
                mf.kt_col.push_back(st.kt_col[e]);
                mf.kt_bmp.push_back(st.kt_bmp_local[e] < 0 ? -1 : base + st.kt_bmp_local[e]);
            }
            mf.kt_bitmap.insert(mf.kt_bitmap.end(), st.kt_bitmap.begin(), st.kt_bitmap.end());
            mf.kt_row_ptr[s + 1] = (int32_t)mf.kt_col.size();
        }
        Stripe().cols.swap(st.cols);  // release early
    }
    mf.own_kt_bitmap = block != 64;
    if (block == 64) {  // the kernel's tiles ARE the exported tiles
        mf.kt_row_ptr = mf.load_row_ptr;
        mf.kt_col = mf.load_col_idx;
        mf.kt_bmp.resize(mf.flags.size());
        int32_t part = 0;
        for (size_t e = 0; e < mf.flags.size(); ++e) mf.kt_bmp[e] = mf.flags[e] ? -1 : part++;
    }
    return SMHA_OK;
}

smha_status_t check_opts(const smha_plan_opts_t *in, smha_plan_opts_t &o) {
    o = smha_plan_opts_t{};
    if (in) o = *in;
    if (o.block == 0) o.block = 64;
    if (o.block != 16 && o.block != 32 && o.block != 64) return SMHA_ERR_UNSUPPORTED;
    if (o.force < SMHA_KERNEL_AUTO || o.force > SMHA_KERNEL_BLOCK) return SMHA_ERR_INVALID_ARG;
    if (o.selector != SMHA_SELECTOR_CALIBRATED && o.selector != SMHA_SELECTOR_PAPER_EQ1)
        return SMHA_ERR_INVALID_ARG;
    if (o.device_id < -2) return SMHA_ERR_INVALID_ARG;
    if (o.block_form < 0 || o.block_form > 3) return SMHA_ERR_INVALID_ARG;
    if (o.head_dim == 0) o.head_dim = 64;
    if (o.head_dim < 8 || o.head_dim > 256 || o.head_dim % 8) return SMHA_ERR_UNSUPPORTED;
    return SMHA_OK;
}

// The per-row column list is the one large array (4 bytes per unmasked entry, written entry by
// entry): it is built in the first pass only when it will certainly be kept.
bool rows_wanted(const smha_plan_opts_t &o) { return o.build_both || o.force == SMHA_KERNEL_ROW; }

}  // namespace

// ---------------------------------------------------------------------------------------
// Kernel selection (Sec. 4.2.3).
//   paper:      threshold = valid16 / n^2 - tau / (log2 n)^2, n = ceil(S/16), tau = 1.2;
//               row-wise iff threshold < 0 (n == 1: row-wise).  The paper states it for as many
//               queries as keys; with Sq != Sk the ratio is taken over the nq * nk tiles of the
//               mask and n in the logarithm is the key side, nk = ceil(Sk/16).
//   calibrated: compare modelled times per (batch, head) pair:
//               block = steps * t_step(d) + t_fixed ; row = nnz * t_entry(d) + Sq * t_rowfix
// ---------------------------------------------------------------------------------------
static double eq1_threshold(double valid16, int Sq, int Sk) {
    const double nq = std::ceil(Sq / 16.0), nk = std::ceil(Sk / 16.0);
    if (nk <= 1.0) return -INFINITY;
    const double lg = std::log2(nk);
    return valid16 / (nq * nk) - 1.2 / (lg * lg);
}

// Cost-model constants in nanoseconds of whole-chip time per (batch, head) pair, fitted to MI355X
// timings of both kernels with 64 pairs in flight (sequence 512 / 2048 / 4096, scattered masks of 2 to
// 64 random keys per row, sliding windows of 8 to 128, causal; least squares by hand on the 4096 rows):
//   block kernel: time = steps * step_ns + fixed_ns, steps = staged K/V tiles of a pair (the union lists
//                 of its 128-row groups) with a gathered tile counted as 1.5 (it takes the bitmap path
//                 and gathers its rows).  d = 64: scattered 4096 4924 ns / 2048 steps = 2.4, causal 4096
//                 3136 / 1056 = 3.0, scattered 2048 1330 / 512 = 2.6 -> 2.8; d = 128: 8400 / 2048 = 4.1,
//                 4889 / 1056 = 4.6, BigBird 8192 (32 pairs) 125 us / 32 / 866 = 4.5 -> 4.5.  fixed_ns = 60:
//                 what a launch of the block kernel costs beyond one of the row kernel, per pair at 64 pairs
//                 (decides only the smallest masks: both kernels are launch-bound there);
//   row kernel:   time = entries * entry_ns + rows * row_ns.  Rows of at most 32 keys on average share a wave:
//                 the constants are those of four rows a wave (two at 256 columns) with four keys in flight, before
//                 row_form chose among forms; 9 keys a row at 64 columns are priced at 28 us for 131072 rows and take
//                 18.7, so masks near the line may go to the slower block kernel.  d = 64: entry 0.0096 (2 vs 16 keys per row: 568 ns / 57344 entries; 32 vs
//                 64: 1134 / 129434 = 0.0088; causal 0.0100), row 0.13 shared / 0.44 with a wave per row;
//                 d = 128: entry 0.0195 (0.0198, 0.0188, causal 0.0203), row 0.12 / 0.43.
// Of the 60 measured cases the model picked the slower kernel in 4, by at most 1.17x; with the row kernel as it is now it
// picks the faster one on the 13 masks (2 to 64 scattered keys per row, narrow windows) timed again.
struct CostModel {
    double step_ns, fixed_ns, entry_ns, row_ns;
};
static CostModel cost_model(int d, double mean_row_nnz) {  // (a head narrower than 64, 128 or 256 columns costs what that kernel costs)
    const bool shared = mean_row_nnz <= 32.0;
    if (d > 128) return CostModel{10.0, 60.0, 0.039, shared ? 0.12 : 0.43};  // (256 columns, one workgroup of eight waves per compute unit: 9.9-10.0 ns per step measured; the row constants are twice those of 128 columns, not measured)
    return d > 64 ? CostModel{4.5, 60.0, 0.0195, shared ? 0.12 : 0.43} : CostModel{2.8, 60.0, 0.0096, shared ? 0.13 : 0.44};
}

// Formats of one mask (64-wide tiles, no per-row lists) from what the GPU reported per tile.
static void formats_from_tiles(const TileInfo *info, const std::vector<uint64_t> &part_bits, int nqt, int nkt,
                               MaskFormats &mf) {
    mf = MaskFormats{};
    mf.load_row_ptr.assign(nqt + 1, 0);
    mf.full_row_ptr.assign(nqt + 1, 0);
    mf.part_row_ptr.assign(nqt + 1, 0);
    for (int tr = 0; tr < nqt; ++tr) {
        for (int tc = 0; tc < nkt; ++tc) {
            const TileInfo &t = info[(size_t)tr * nkt + tc];
            const uint32_t cnt = t.cnt_v16 & 0xFFFFu;
            mf.nnz += cnt;
            mf.n_valid16 += (t.cnt_v16 >> 16) & 0xFFu;
            if (!cnt) continue;
            const bool full = cnt == 64 * 64;
            mf.load_col_idx.push_back(tc);
            mf.flags.push_back(full ? 1 : 0);
            (full ? mf.full_col_idx : mf.part_col_idx).push_back(tc);
            if (!full)  // (the GPU stored part tiles in the order its waves reached them: put them in list order)
                mf.bitmap.insert(mf.bitmap.end(), part_bits.begin() + (size_t)t.slot * 64, part_bits.begin() + (size_t)t.slot * 64 + 64);
        }
        mf.load_row_ptr[tr + 1] = (int32_t)mf.load_col_idx.size();
        mf.full_row_ptr[tr + 1] = (int32_t)mf.full_col_idx.size();
        mf.part_row_ptr[tr + 1] = (int32_t)mf.part_col_idx.size();
    }
    mf.kt_row_ptr = mf.load_row_ptr;  // the kernel's tiles are the exported tiles
    mf.kt_col = mf.load_col_idx;
    mf.kt_bmp.resize(mf.flags.size());
    int32_t part = 0;
    for (size_t e = 0; e < mf.flags.size(); ++e) mf.kt_bmp[e] = mf.flags[e] ? -1 : part++;
}

// Rows of at most this many keys on average may share a wave of the row kernel.
constexpr double kSharedRowMean = 32.0;

// steps of a form's waves over eight rows, given the longest of each wave's (a template: the divisors are constants)
template <int W, int F>
static void add_row_steps(const int *longest, smha_plan *p) {
    constexpr int keys = row_step_keys(W, F);
    int n = 0;
    for (int k = 0; k < 8 / kRowForms[W][F].rows; ++k) n += (longest[k] + keys - 1) / keys;
    p->row_steps[W][F] += n;
}

static void count_row_steps(const std::vector<int32_t> &row_ptr, int S, smha_plan *p) {
    static_assert(kRowForms[0][0].rows == 8 && kRowForms[0][1].rows == 4 && kRowForms[1][0].rows == 4 &&
                  kRowForms[1][1].rows == 4 && kRowForms[2][0].rows == 2 && kRowForms[2][1].rows == 2, "as used below");
    for (int i0 = 0; i0 < S; i0 += 8) {
        int one[8], two[4], four[2];
        for (int r = 0; r < 8; ++r) one[r] = i0 + r < S ? row_ptr[i0 + r + 1] - row_ptr[i0 + r] : 0;
        for (int r = 0; r < 4; ++r) two[r] = std::max(one[2 * r], one[2 * r + 1]);
        for (int r = 0; r < 2; ++r) four[r] = std::max(two[2 * r], two[2 * r + 1]);
        const int eight = std::max(four[0], four[1]);
        p->row_longest = std::max(p->row_longest, eight);
        add_row_steps<0, 0>(&eight, p);
        add_row_steps<0, 1>(four, p);
        add_row_steps<0, 2>(one, p);
        add_row_steps<1, 0>(four, p);
        add_row_steps<1, 1>(four, p);
        add_row_steps<1, 2>(one, p);
        add_row_steps<2, 0>(two, p);
        add_row_steps<2, 1>(two, p);
        add_row_steps<2, 2>(one, p);
    }
}

// After a first pass without the per-row lists: could the selector take the row kernel?  (The
// block estimate here ignores gathered tiles, so it is an upper bound: if the row kernel does not
// beat it, it will not beat the final one either.)  If so the masks are analysed again with rows.
static bool row_may_be_chosen(const smha_plan *p) {
    if (p->opts.force != SMHA_KERNEL_AUTO) return false;
    const int n_masks = p->Bm * p->Hm;
    double v16 = 0, nnz = 0, tiles = 0;
    for (auto &m : p->masks) {
        v16 += (double)m.n_valid16;
        nnz += (double)m.nnz;
        tiles += (double)m.kt_col.size();
    }
    if (p->opts.selector == SMHA_SELECTOR_PAPER_EQ1) return eq1_threshold(v16 / n_masks, p->S, p->Sk) < 0;
    const CostModel cm = cost_model(p->opts.head_dim, nnz / n_masks / p->S);
    // (a pair's steps are at most its tiles: two tile rows share a staged tile, gathered tiles replace several)
    return nnz / n_masks * cm.entry_ns + p->S * cm.row_ns < tiles / n_masks * cm.step_ns + cm.fixed_ns;
}

// The wave form's lists (see WaveItem), in two steps: what the estimates need of them (their lengths), once a call shape is
// first asked for, and the lists, once a call takes the form.  (Made with every plan they cost those that never use them
// 5 to 7 %: BigBird blocks at 8192, per-head 64-blocks at 4096.)  Masks with more than kMaxWaveEntries 32-key tiles in all get
// none: their lists would be a burden, and calls on masks so large fill the chip through the other forms.
//
static WaveTile wave_tile(const uint64_t *rows) {
    WaveTile t{{0, 0}, 0};
    for (int side = 0; side < 2; ++side) {
        uint64_t any = 0, all = ~(uint64_t)0;
        for (int r = 32 * side; r < 32 * side + 32; ++r) { any |= rows[r]; all &= rows[r]; }
        t.any[side] = any;
        t.full |= (uint8_t)((((uint32_t)all == 0xFFFFFFFFu) | ((uint32_t)(all >> 32) == 0xFFFFFFFFu) << 1) << (2 * side));
    }
    return t;
}
static int wave_parts(int32_t n) { return n <= kWaveWhole ? 1 : (n + 63) / 64; }  // (a wave holds one entry per lane, and four may share a list)

bool count_wave_lists(const smha_plan *p) {
    WaveLists &wl = p->wave;
    std::lock_guard<std::mutex> lock(wl.mutex);
    if (wl.counted) return wl.possible;
    constexpr int64_t kMaxWaveEntries = 1 << 20;
    const int n_masks = p->Bm * p->Hm, n_groups = (p->S + 31) / 32, stride = 2 * ((n_groups + 1) / 2);
    int64_t at_most = 0;
    for (const MaskFormats &m : p->masks) at_most += 4 * (int64_t)m.kt_col.size();
    wl.at_most = at_most;
    if (!p->has_block || p->opts.block_form != 0 || at_most > kMaxWaveEntries || n_groups > 16384 /* (a grid's y holds a mask's workgroups) */ ||
        p->h_kt_bitmap.size() * sizeof(uint64_t) >= ((size_t)1 << 31)) {
        wl.counted = true;
        return false;
    }
    std::vector<int32_t> lengths((size_t)n_masks * stride, 0);
    std::vector<char> touched(2 * (size_t)((p->Sk + 63) / 64), 0);                // 32-key tiles
    std::vector<int32_t> of_length(kWaveWhole + 1, 0);
    std::vector<WaveTile> tiles;
    size_t n_part = 0;
    for (const MaskFormats &m : p->masks) n_part += m.kt_bits().size() / 64;
    tiles.reserve(n_part);
    int64_t ents = 0, part_ents = 0;
    int max_splits = 0, max_slots = 0;
    for (int mi = 0; mi < n_masks; ++mi) {
        const MaskFormats &m = p->masks[mi];
        int32_t *const of = lengths.data() + (size_t)mi * stride;
        for (int tr = 0; 2 * tr < n_groups; ++tr)
            for (int e = m.kt_row_ptr[tr]; e < m.kt_row_ptr[tr + 1]; ++e) {
                char *const keys = touched.data() + 2 * (size_t)m.kt_col[e];
                if (m.kt_bmp[e] < 0) {
                    of[2 * tr] += 2;
                    of[2 * tr + 1] += 2;
                    keys[0] = keys[1] = 1;
                    continue;
                }
                tiles.push_back(wave_tile(m.kt_bits().data() + (size_t)m.kt_bmp[e] * 64));
                const WaveTile &t = tiles.back();
                for (int side = 0; side < 2; ++side)
                    for (int half = 0; half < 2; ++half)
                        if ((uint32_t)(t.any[side] >> (32 * half))) {
                            ++of[2 * tr + side];
                            part_ents += !(t.full >> (2 * side + half) & 1);
                            keys[half] = 1;
                        }
            }
        int slots = 0, splits = 0;
        for (int g = 0; g < n_groups; ++g) {
            const int parts = wave_parts(of[g]);
            for (int c = 0; c < parts; ++c) ++of_length[(size_t)((int64_t)of[g] * (c + 1) / parts - (int64_t)of[g] * c / parts)];
            ents += of[g];
            slots += parts > 1 ? parts : 0;
            splits += parts > 1;
        }
        max_slots = std::max(max_slots, slots);
        max_splits = std::max(max_splits, splits);
    }
    std::copy(of_length.begin(), of_length.end(), wl.of_length);
    wl.tiles.swap(tiles);
    wl.lengths.swap(lengths);
    wl.n_ents = ents;
    wl.part_ents = part_ents;
    wl.keys = 32 * (int)std::count(touched.begin(), touched.end(), 1);
    wl.max_slots = max_slots;
    wl.max_splits = max_splits;
    wl.possible = wl.counted = true;
    return true;
}

// Nearly all tiles are partly filled, and one in four or more of their 32 x 32 sub-tiles has no keys.
bool empty_sub_tiles(const smha_plan *p) {
    if (!p->mostly_partial) return false;
    try {
        if (!count_wave_lists(p)) return false;
    } catch (const std::bad_alloc &) {
        return false;
    }
    return (double)p->wave.n_ents < 0.75 * (double)p->wave.at_most;
}

void make_wave_lists(const smha_plan *p) {  // (count_wave_lists has said that they are possible)
    WaveLists &wl = p->wave;
    std::lock_guard<std::mutex> lock(wl.mutex);
    if (wl.made) return;
    const int n_masks = p->Bm * p->Hm, n_groups = (p->S + 31) / 32, stride = 2 * ((n_groups + 1) / 2);
    std::vector<WaveItem> all_items, items;
    std::vector<WaveEntry> ents((size_t)wl.n_ents + 1, WaveEntry{0, -1});  // (the last: an empty item's entry)
    std::vector<uint32_t> all_used((size_t)wl.n_ents + 1, 0u);
    std::vector<int32_t> item_off, item_cnt, split_off, first((size_t)stride + 1), next, at;  // first: of each 32-row group its first entry
    std::vector<SplitRow> all_splits;
    const WaveTile *tile = wl.tiles.data();
    first[0] = 0;
    for (int mi = 0; mi < n_masks; ++mi) {
        const MaskFormats &m = p->masks[mi];
        for (int g = 0; g < stride; ++g) first[g + 1] = first[g] + wl.lengths[(size_t)mi * stride + g];
        next.assign(first.begin(), first.end());
        for (int tr = 0; 2 * tr < n_groups; ++tr)
            for (int e = m.kt_row_ptr[tr]; e < m.kt_row_ptr[tr + 1]; ++e) {
                const int32_t key = m.kt_col[e] * 64;
                const bool whole = m.kt_bmp[e] < 0;
                const WaveTile t = whole ? WaveTile{{~(uint64_t)0, ~(uint64_t)0}, 15} : *tile++;
                for (int side = 0; side < 2; ++side)
                    for (int half = 0; half < 2; ++half) {
                        const uint32_t any = (uint32_t)(t.any[side] >> (32 * half));
                        if (any == 0) continue;
                        const size_t to = (size_t)next[2 * tr + side]++;
                        all_used[to] = any;
                        ents[to] = WaveEntry{key + 32 * half, t.full >> (2 * side + half) & 1 ? -1 : m.kt_bmp[e] + wl.bmp_base[mi]};
                    }
            }
        // lists of more than kWaveWhole entries are cut, and the parts' results are merged in memory
        items.clear();
        int32_t slots = 0, n_splits = 0;
        split_off.push_back((int32_t)all_splits.size());
        for (int g = 0; g < n_groups; ++g) {
            const int32_t b = first[g], n = first[g + 1] - b;
            const int parts = wave_parts(n);
            if (parts > 1) all_splits.push_back({g, slots, parts, 0});
            for (int c = 0; c < parts; ++c) {
                const int32_t cb = b + (int32_t)((int64_t)n * c / parts), ce = b + (int32_t)((int64_t)n * (c + 1) / parts);
                const WaveEntry e0 = ce > cb ? ents[cb] : WaveEntry{0, -1};
                items.push_back({g, cb, ce - cb, parts > 1 ? slots++ : -1, parts > 1 ? n_splits : -1, e0.key, e0.code, 0});
            }
            n_splits += parts > 1;
        }
        // longest first, in row order where equal: a counting sort
        at.assign(kWaveWhole + 2, 0);
        for (const WaveItem &i : items) ++at[kWaveWhole - i.n + 1];
        for (int c = 0; c <= kWaveWhole; ++c) at[c + 1] += at[c];
        const size_t base = all_items.size();
        all_items.resize(base + items.size());
        for (const WaveItem &i : items) all_items[base + at[kWaveWhole - i.n]++] = i;
        item_off.push_back((int32_t)base);
        item_cnt.push_back((int32_t)items.size());
        first[0] = first[stride];
    }
    wl.items.swap(all_items);
    wl.ents.swap(ents);
    wl.used.swap(all_used);
    wl.item_off.swap(item_off);
    wl.item_cnt.swap(item_cnt);
    wl.split_off.swap(split_off);
    wl.splits.swap(all_splits);
    std::vector<WaveTile>().swap(wl.tiles);
    std::vector<int32_t>().swap(wl.lengths);
    wl.made = true;
}

smha_status_t finish_plan(smha_plan *p) {
    const int n_masks = p->Bm * p->Hm;
    const int S = p->S;  // queries
    double v16 = 0, nnz = 0, tiles = 0;
    for (auto &m : p->masks) {
        v16 += (double)m.n_valid16;
        nnz += (double)m.nnz;
        tiles += (double)m.kt_col.size();
    }
    v16 /= n_masks;
    nnz /= n_masks;
    tiles /= n_masks;
    p->eq1_threshold = eq1_threshold(v16, S, p->Sk);
    const CostModel cm = cost_model(p->opts.head_dim, nnz / S);
    p->model_row_us = 1e-3 * (nnz * cm.entry_ns + S * cm.row_ns);
    p->row_mean_nnz = nnz / S;

    try {
        // ---- block path first (its work lists say how many tiles the kernel will really visit,
        // which the selector needs): tiles, work items, split rows --------------------------
        if (p->opts.force != SMHA_KERNEL_ROW || p->opts.build_both) {
            const int nqt = (S + kTile - 1) / kTile;
            const int nsup = (S + kSuper - 1) / kSuper;
            for (int mi = 0; mi < n_masks; ++mi) {
                MaskFormats &m = p->masks[mi];
                const int32_t bmp_base = (int32_t)(p->h_kt_bitmap.size() / 64);
                p->wave.bmp_base.push_back(bmp_base);
                p->h_kt_bitmap.insert(p->h_kt_bitmap.end(), m.kt_bits().begin(), m.kt_bits().end());
                // union of the two tile rows of every supertile (both lists ascending: merge); tiles
                // that use few key columns are repacked into gathered tiles (see UEntry), which go
                // to the end of the supertile's list
                std::vector<int32_t> sup_ptr(nsup + 1, 0);
                const int32_t ent_base = (int32_t)p->h_uent.size();
                const int64_t pad_key = (int64_t)p->Sk + 64;  // (past the sequence: loads as zeros)
                struct Sparse { int32_t col, ea, eb; uint64_t used; };
                std::vector<Sparse> sparse;
                std::vector<int32_t> keys;
                for (int sp = 0; sp < nsup; ++sp) {
                    const int r0 = 2 * sp, r1 = 2 * sp + 1;
                    int a = m.kt_row_ptr[r0], ae = m.kt_row_ptr[r0 + 1];
                    int b = r1 < nqt ? m.kt_row_ptr[r1] : 0, be = r1 < nqt ? m.kt_row_ptr[r1 + 1] : 0;
                    auto code = [&](int e) { return m.kt_bmp[e] < 0 ? -1 : m.kt_bmp[e] + bmp_base; };
                    auto used_cols = [&](int e) {  // which of the tile's 64 key columns any query uses
                        if (e < 0) return (uint64_t)0;
                        if (m.kt_bmp[e] < 0) return ~(uint64_t)0;
                        uint64_t u = 0;
                        const uint64_t *w = m.kt_bits().data() + (size_t)m.kt_bmp[e] * 64;
                        for (int r = 0; r < 64; ++r) u |= w[r];
                        return u;
                    };
                    sparse.clear();
                    int n_sparse_cols = 0;
                    while (a < ae || b < be) {
                        UEntry u{0, {-2, -2}, 0};
                        const int ca = a < ae ? m.kt_col[a] : INT32_MAX;
                        const int cb = b < be ? m.kt_col[b] : INT32_MAX;
                        u.col = std::min(ca, cb);
                        const int ea = ca == u.col ? a++ : -1, eb = cb == u.col ? b++ : -1;
                        const uint64_t used = used_cols(ea) | used_cols(eb);
                        if (!p->opts.no_gather && __builtin_popcountll(used) <= kGatherMaxCols) {
                            sparse.push_back({u.col, ea, eb, used});
                            n_sparse_cols += __builtin_popcountll(used);
                            continue;
                        }
                        if (ea >= 0) u.code[0] = code(ea);
                        if (eb >= 0) u.code[1] = code(eb);
                        p->h_uent.push_back(u);
                    }
                    // repacking pays only if it saves steps
                    if ((n_sparse_cols + 63) / 64 >= (int)sparse.size()) {
                        for (const Sparse &t : sparse) {
                            UEntry u{t.col, {-2, -2}, 0};
                            if (t.ea >= 0) u.code[0] = code(t.ea);
                            if (t.eb >= 0) u.code[1] = code(t.eb);
                            p->h_uent.push_back(u);
                        }
                        // (the list is no longer ascending in col; nothing depends on that)
                    } else {
                        keys.clear();
                        for (const Sparse &t : sparse) {
                            for (uint64_t x = t.used; x; x &= x - 1) keys.push_back(t.col * 64 + __builtin_ctzll(x));
                        }
                        // keys ascend (tiles ascend, bits ascend); 64 per gathered tile
                        size_t ti = 0;  // sparse tile that holds keys[k]
                        for (size_t k0 = 0; k0 < keys.size(); k0 += 64) {
                            const int nk = (int)std::min<size_t>(64, keys.size() - k0);
                            const int32_t gt = (int32_t)(p->h_gidx.size() / 64);
                            uint64_t wa[64] = {0}, wb[64] = {0};
                            for (int k = 0; k < 64; ++k) {
                                if (k >= nk) {
                                    p->h_gidx.push_back((int32_t)std::min<int64_t>(pad_key, INT32_MAX));
                                    continue;
                                }
                                const int32_t key = keys[k0 + k];
                                p->h_gidx.push_back(key);
                                while (sparse[ti].col != key / 64) ++ti;
                                const Sparse &t = sparse[ti];
                                const int bit = key & 63;
                                for (int side = 0; side < 2; ++side) {
                                    const int e = side ? t.eb : t.ea;
                                    if (e < 0) continue;
                                    uint64_t *dst = side ? wb : wa;
                                    if (m.kt_bmp[e] < 0) {
                                        for (int r = 0; r < 64; ++r) dst[r] |= 1ull << k;
                                    } else {
                                        const uint64_t *w = m.kt_bits().data() + (size_t)m.kt_bmp[e] * 64;
                                        for (int r = 0; r < 64; ++r) dst[r] |= ((w[r] >> bit) & 1ull) << k;
                                    }
                                }
                            }
                            UEntry u{0, {-2, -2}, gt + 1};
                            for (int side = 0; side < 2; ++side) {
                                const uint64_t *w = side ? wb : wa;
                                uint64_t any = 0;
                                for (int r = 0; r < 64; ++r) any |= w[r];
                                if (!any) continue;
                                u.code[side] = (int32_t)(p->h_kt_bitmap.size() / 64);
                                p->h_kt_bitmap.insert(p->h_kt_bitmap.end(), w, w + 64);
                            }
                            p->h_uent.push_back(u);
                            ++p->n_gathered;
                        }
                    }
                    sup_ptr[sp + 1] = (int32_t)p->h_uent.size() - ent_base;
                }
                // split supertiles whose list is much longer than the typical one, so that a
                // few heavy rows (global tokens) do not serialise on one workgroup
                int64_t n_nonempty = 0;
                for (int sp = 0; sp < nsup; ++sp) n_nonempty += sup_ptr[sp + 1] > sup_ptr[sp];
                const double avg = n_nonempty ? (double)sup_ptr[nsup] / n_nonempty : 0.0;
                for (int lvl = 0; lvl < 2; ++lvl) {
                // Grain 0: parts of at most `chunk` steps (the kernel holds one entry per lane: 64 at
                // most), and lists up to twice that stay whole: merging costs a second launch (4-6 us),
                // more than a workgroup that runs a few steps longer than the others.  Grain 1: at most
                // 16 steps per item, for calls with so few heads that one long list would be the launch.
                const int chunk = lvl == 0 ? std::min(64, std::max(16, (int)std::ceil(1.5 * avg))) : 16;
                const int whole = lvl == 0 ? std::min(64, 2 * chunk) : 16;
                WorkLists &wl = p->lists[lvl];
                std::vector<Item> items;
                std::vector<SplitRow> splits;
                int32_t slots = 0;
                auto make_item = [&](int sp, int32_t b, int32_t e, int32_t slot, int32_t split = -1) {
                    Item it{sp, b, e, slot, 0, 0, split, 0};
                    for (int32_t x = b; x < e; ++x)
                        if (p->h_uent[x].gather > 0) {
                            if (!it.gcount) it.gbegin = p->h_uent[x].gather - 1;
                            ++it.gcount;
                        }
                    return it;
                };
                std::vector<int32_t> cuts;
                for (int sp = 0; sp < nsup; ++sp) {
                    const int32_t b = ent_base + sup_ptr[sp], e = ent_base + sup_ptr[sp + 1];
                    const int n = e - b;
                    int n_gath = 0;
                    for (int32_t x = b; x < e; ++x) n_gath += p->h_uent[x].gather > 0;
                    if (n <= whole && n_gath <= kMaxGatherPerItem) {
                        items.push_back(make_item(sp, b, e, -1));
                        continue;
                    }
                    // equal parts of at most `chunk` entries, cut again where a part would hold more
                    // gathered tiles than the kernel keeps key numbers for
                    const int parts = (n + chunk - 1) / chunk;
                    cuts.clear();
                    cuts.push_back(b);
                    for (int c = 1; c <= parts; ++c) {
                        const int32_t ce = b + (int32_t)((int64_t)n * c / parts);
                        int g = 0;
                        for (int32_t x = cuts.back(); x < ce; ++x) {
                            if (p->h_uent[x].gather > 0 && ++g > kMaxGatherPerItem) {
                                cuts.push_back(x);
                                g = 1;
                            }
                        }
                        if (ce > cuts.back()) cuts.push_back(ce);
                    }
                    const int n_parts = (int)cuts.size() - 1;
                    if (n_parts == 1) {
                        items.push_back(make_item(sp, b, e, -1));
                        continue;
                    }
                    splits.push_back({sp, slots, n_parts, 0});
                    for (int c = 0; c < n_parts; ++c)
                        items.push_back(make_item(sp, cuts[c], cuts[c + 1], slots++, (int32_t)splits.size() - 1));
                }
                std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) {
                    return (a.end - a.begin) > (b.end - b.begin);
                });
                wl.item_off.push_back((int32_t)wl.items.size());
                wl.item_cnt.push_back((int32_t)items.size());
                wl.items.insert(wl.items.end(), items.begin(), items.end());
                wl.split_off.push_back((int32_t)wl.split_rows.size());
                wl.split_cnt.push_back((int32_t)splits.size());
                wl.split_rows.insert(wl.split_rows.end(), splits.begin(), splits.end());
                wl.max_items = std::max(wl.max_items, (int)items.size());
                wl.max_split_rows = std::max(wl.max_split_rows, (int)splits.size());
                wl.max_slots = std::max(wl.max_slots, (int)slots);
                }
            }
        }
        // (no block lists were built: the forced row kernel; the estimate then falls back to one step per tile)
        const double steps = p->h_uent.empty() ? tiles : ((double)p->h_uent.size() + 0.5 * (double)p->n_gathered) / n_masks;
        p->model_block_us = 1e-3 * (steps * cm.step_ns + cm.fixed_ns);
        int choice;
        if (p->opts.force != SMHA_KERNEL_AUTO)
            choice = p->opts.force;
        else if (p->opts.selector == SMHA_SELECTOR_PAPER_EQ1)
            choice = p->eq1_threshold < 0 ? SMHA_KERNEL_ROW : SMHA_KERNEL_BLOCK;
        else
            choice = p->model_row_us < p->model_block_us ? SMHA_KERNEL_ROW : SMHA_KERNEL_BLOCK;
        p->kernel = choice;
        p->has_row = p->opts.build_both || choice == SMHA_KERNEL_ROW;
        p->has_block = p->opts.build_both || choice == SMHA_KERNEL_BLOCK;
        p->fine_differs = p->lists[1].items.size() != p->lists[0].items.size();
        if (!p->fine_differs) p->lists[1] = WorkLists{};  // (same cuts: one copy serves both)
        {   // (measured at 128 columns: the third form loses 3-5 % on dense causal lists of 16 steps and more,
            // and wins up to 20 % wherever tiles are partially filled or lists are short)
            int64_t tiles_in_lists = 0, part_in_lists = 0;
            for (const UEntry &u : p->h_uent)
                for (int side = 0; side < 2; ++side) {
                    tiles_in_lists += u.code[side] != -2;
                    part_in_lists += u.code[side] >= 0;
                }
            const double groups = (double)n_masks * ((p->S + 127) / 128);
            p->mostly_partial = (double)part_in_lists > 0.9 * (double)tiles_in_lists;
            p->dense_long_lists = (double)part_in_lists < 0.15 * (double)tiles_in_lists && (double)p->h_uent.size() > 16.0 * groups;
        }
        if (p->has_block) {
            p->h_kt_bitmap.insert(p->h_kt_bitmap.end(), 64, 0ull);  // spare all-zero block
            p->h_uent.push_back(UEntry{0, {-2, -2}, 0});             // spare entry: an empty item may read one past its list
        } else {  // the row kernel was chosen: the block kernel's lists are not kept
            std::vector<UEntry>().swap(p->h_uent);
            std::vector<int32_t>().swap(p->h_gidx);
            std::vector<uint64_t>().swap(p->h_kt_bitmap);
            p->lists[0] = WorkLists{};
            p->lists[1] = WorkLists{};
            p->n_gathered = 0;
            p->fine_differs = false;
        }
        // ---- row path: concatenate -------------------------------------------------
        if (p->has_row) {
            p->h_row_ptr.reserve((size_t)n_masks * (S + 1));
            int64_t off = 0;
            for (auto &m : p->masks) {
                p->h_col_off.push_back(off);
                p->h_row_ptr.insert(p->h_row_ptr.end(), m.row_ptr.begin(), m.row_ptr.end());
                off += (int64_t)m.col_idx.size();
            }
            p->h_col_idx.reserve(off);
            for (auto &m : p->masks)
                p->h_col_idx.insert(p->h_col_idx.end(), m.col_idx.begin(), m.col_idx.end());
            if (p->row_mean_nnz <= kSharedRowMean)
                for (auto &m : p->masks) count_row_steps(m.row_ptr, S, p);
        }
        // the per-row column list is large; drop it when no kernel will read it
        if (!p->has_row)
            for (auto &m : p->masks) {
                // keep row_ptr/col_idx for export only when explicitly requested (build_both)
                std::vector<int32_t>().swap(m.col_idx);
                std::vector<int32_t>().swap(m.row_ptr);
            }
    } catch (const std::bad_alloc &) {
        return SMHA_ERR_ALLOC;
    }

    int dev = p->opts.device_id;
    if (dev == -2) return SMHA_OK;
    if (dev == -1) {
        dev = current_device_or_negative();
        if (dev < 0) return SMHA_OK;  // host-only plan; forward will report SMHA_ERR_HIP
    }
    return upload_plan(p, dev);
}

// The form of the row kernel with the least estimated time, for plans whose rows may share waves at all.  Two things
// bound a launch, and their root sum of squares is the estimate:
//   work   waves * fixed + steps * keys in flight * 0.067 ns: what the chip's waves take together; each lasts as long
//          as its longest row, and a step costs by the 1 KiB loads in it;
//   chain  steps of the longest row * trip: key numbers, then K and V, a serial chain that no other wave shortens; 0.42 us
//          a step while the call's K and V fit the L2s (up to 16 MB of them), 1.1 us beyond, 1.2 times that with four
//          keys in flight and 0.85 times with two.
// Fitted to rows of 1 to 32 keys, and of 9 keys with 1 to 64 rows of 16 to 2048 among them, 256 to 131072 rows: on these
// 360 the choice is within 1 % of the fastest form in the mean, and nowhere more than 2 % behind the forms that short rows
// of any length had first (four rows a wave, two at 256 columns, four keys in flight).  Where each wins, us:
//   64 columns, 64 x 2048 rows, eight / four rows a wave: 9 keys 19.2 / 29.2, 16 keys 29.3 / 30.4, 32 keys 50.8 / 47.3; one
//   row of 64 keys among the 9s 31.4 / 31.8, of 128 55.9 / 37.1, of 1024 411 / 140, and with a wave per row 84;
//   8 x 2048 rows, one of 24 keys 6.9 / 6.8; 4 x 1024 rows, 9 keys 4.4 / 4.9, 16 keys 5.6 / 4.9;
//   128 columns, 64 x 2048 rows, three / four keys in flight: 3 keys 22.7 / 24.0, 4 keys 26.8 / 24.3, 8 keys 32.6 / 30.5,
//   9 keys 33.8 / 38.0, 16 keys 55.0 / 49.0, 32 keys 92.5 / 87.5; 256 columns 4 keys 53.4 / 45.3, 9 keys 66.1 / 75.4.
// A wave per row starts so many waves that it is given another 1 us, and has to win by a tenth.
int row_form(const smha_plan *plan, int B, int H, int D) {
    constexpr int kWavePerRow = 2;
    if (plan->row_mean_nnz > kSharedRowMean) return kWavePerRow;
    const int w = row_width(D);
    const double heads = (double)B * H, masks = (double)plan->Bm * plan->Hm;
    const double trip_us = heads * plan->Sk * D * 4 <= 16e6 ? 0.42 : 1.1;
    int best = 0;
    double best_us = 0;
    for (int f = 0; f < 3; ++f) {
        const RowForm form = kRowForms[w][f];
        const double fixed_ns = form.rows == 8 ? 0.57 : form.rows == 1 ? 0.30 : 0.43;  // (per wave: start, queries, merge, store)
        const double waves = heads * ((plan->S + form.rows - 1) / form.rows), steps = heads / masks * (double)plan->row_steps[w][f];
        const int chain = (plan->row_longest + row_step_keys(w, f) - 1) / row_step_keys(w, f);
        const double work_us = 1e-3 * (waves * fixed_ns + steps * form.batch * 0.067);
        const double chain_us = chain * trip_us * (form.batch == 4 ? 1.2 : form.batch == 2 ? 0.85 : 1.0);
        double us = std::hypot(work_us, chain_us);
        if (f == kWavePerRow) us = 1.1 * (us + 1.0);
        if (f == 0 || us < best_us) {
            best = f;
            best_us = us;
        }
    }
    return best;
}

// One workspace of the block kernel for a call shape: per (batch*head) max_slots partial results of
// 128 rows (O, then reference and sum per row, each written per wave, with room for eight waves: 128 d + 1024 floats), then
// eight arrival counters (one per wave of the form with most) per (batch*head, split group).
size_t workspace_bytes(const smha_plan *plan, int lvl, int form, int B, int H, int d, size_t *counters_at) {
    if (form == 4) {  // 32 rows per partial result, one counter per split group
        const size_t at = ((size_t)B * H * plan->wave.max_slots * (size_t)(32 * d + 128) * sizeof(float) + 255) / 256 * 256;
        if (counters_at) *counters_at = at;
        return at + (size_t)B * H * plan->wave.max_splits * sizeof(uint32_t);
    }
    const WorkLists &wl = plan->lists[plan->fine_differs ? lvl : 0];
    const size_t partials = (size_t)B * H * wl.max_slots * (size_t)(128 * d + 1024) * sizeof(float);
    const size_t at = (partials + 255) / 256 * 256;
    if (counters_at) *counters_at = at;
    return at + (size_t)B * H * wl.max_split_rows * 8 * sizeof(uint32_t);
}

// The wave form's work for one call shape: four waves make a workgroup, and each mask gets as many workgroups (records
// past a mask's own have rg = -1).  An item of more than `alone` entries is shared by the four waves of a workgroup.
// Workgroups start in the order in which they are listed: those that last longest first, whichever kind (shared items
// first instead, however short their quarters: window 4 x 8 x 1089 x 128 with `alone` = 12 33.5 us, 27 so).
int build_wave_order(const smha_plan *plan, int alone, std::vector<int32_t> &table) {
    const WaveLists &wl = plan->wave;
    const int n_masks = plan->Bm * plan->Hm;
    std::vector<int32_t> shared(n_masks, 0);
    size_t most = 0;
    for (int mi = 0; mi < n_masks; ++mi) {
        const WaveItem *items = wl.items.data() + wl.item_off[mi];
        while (shared[mi] < wl.item_cnt[mi] && items[shared[mi]].n > alone) ++shared[mi];
        most = std::max(most, (size_t)shared[mi] + (wl.item_cnt[mi] - shared[mi] + 3) / 4);
    }
    static_assert(sizeof(WaveItem) == 32, "eight words a record");
    table.resize(most * n_masks * 32);
    for (int mi = 0; mi < n_masks; ++mi) {
        const WaveItem *items = wl.items.data() + wl.item_off[mi];
        WaveItem *to = reinterpret_cast<WaveItem *>(table.data()) + most * 4 * mi, *const end = to + most * 4;
        int32_t team = 0, solo = shared[mi];  // next of each kind; both kinds come longest first
        while (team < shared[mi] || solo < wl.item_cnt[mi]) {
            if (team < shared[mi] && (solo == wl.item_cnt[mi] || (items[team].n + 3) / 4 >= items[solo].n)) {
                const WaveItem &it = items[team++];
                for (int w = 0; w < 4; ++w) {
                    const int at = it.n * w / 4;
                    const WaveEntry &e = wl.ents[it.begin + at];
                    *to++ = WaveItem{it.rg, it.begin + at, it.n * (w + 1) / 4 - at, it.slot, it.split, e.key, e.code, 1};
                }
            } else {
                for (int w = 0; w < 4; ++w) *to++ = solo < wl.item_cnt[mi] ? items[solo++] : WaveItem{-1, 0, 0, -1, -1, 0, -1, 0};
            }
        }
        for (; to < end; ++to) *to = WaveItem{-1, 0, 0, -1, -1, 0, -1, 0};
    }
    return (int)most;
}

// Estimated times of a call, for the choice between the wave form and the other two (and for its `alone`).  Several things
// bound a launch: what the chip's compute units take together, the longest chain of steps in one wave or workgroup, and
// the bytes of Q, K, V and O; the estimate is the root of the sum of their p-th powers.  Constants are in us (per wave and
// step of the wave form: ns, `memory`: us per MB), fitted by least squares of the logarithms to 1207 calls of
// profiles/block_forms.csv (all kinds of masks, 64 to 8192 queries, 1 to 400 heads, 8 to 256 columns; clocks settled by 10 ms of the
// same work and three sets of inputs in turn: measured from idle clocks the first form took 15 % longer, the wave form 3 %,
// and the choice went wrong by that).  Mean error over 600 other calls of the table: 5 to 7 % (wave form), 5 % (the others).  At 96,
// 160 and 256 columns: the wave form's constants of 128, 128 and 256 columns at first with three of their own (`start`, `memory`, and one
// factor for `wave`, `step` and the chain's), the forms that the library takes there refitted (160 with gathered tiles: likewise scaled);
// mean error 5 to 8 %.  At 32 columns the wave form's constants were fitted to what the choice (and that of `alone`) gives away on 1257 calls, those of
// profiles/block_forms_partial.csv and the like, drawn ones and the table's: 0.8 % instead of 2.2 with the constants of 64 columns, scaled, which had made lists of 16 to
// 32 steps on one or two workgroups a compute unit 20 to 30 % too short (random 3 x 20 x 1000 x 32 29.0 us, 26.3 at 64 columns, now 23).  Over 340 calls that were not
// used: 0.990 of the time before in the mean, 45 more than 2 % faster, 11 slower (1.10 at most), none slower than at 64 columns.
// At 256 columns `start`, `join` and `memory` were fitted again with 920 more calls, to what the choice gives away: 1.04 % instead of 1.56 (over either half,
// fitted to the other, 1.0 and 1.1 instead of 1.4 and 1.7); `memory` had been so high that windows took the third form (1 x 20 x 676 x 192 13.7 us, wave form 11.6).
struct WaveCost {
    double start, wave, step, held, part, bf16, chain, chain_full, power, uneven, part_all, join, memory;
};
static const WaveCost kWaveCost[6] = {
    {2.487, 0.3727, 0.2368, 0.218, 0.030, 1.20, 0.3972, 0.065, 3.515, 0.237, 0.1279, 1.292, 0.0678},  // 32 columns
    {3.07, 0.7028, 0.4019, 0.22, 0.076, 1.20, 0.4933, 0.2096, 3.4, 0.0, -0.003, 1.946, 0.0461},     // 64
    {3.99, 1.246, 0.595, 0.05, 0.191, 1.17, 0.567, 0.1278, 4.0, 0.09, -0.076, 1.877, 0.0683},       // 96
    {3.80, 1.5978, 0.7627, 0.05, 0.191, 1.17, 0.7266, 0.1638, 4.0, 0.09, -0.076, 1.877, 0.0700},    // 128
    {4.594, 2.067, 0.987, 0.05, 0.191, 1.17, 0.940, 0.2120, 4.0, 0.09, -0.076, 1.877, 0.1045},      // 160
    {5.188, 4.5016, 1.4624, 0.63, 0.156, 1.17, 1.3585, 0.0, 4.0, 0.23, -0.041, 4.449, 0.1824}};     // 256
struct BlockCost {
    double start, unit, unit_act, unit_part, unit_sub, unit_lone, group, group_act, group_part, unit_bf16, group_bf16, gather, power, merge, memory;
};
static constexpr BlockCost kBlockCost[6][2] = {  // first form, third form (that the library takes at 96 to 256 columns)
    {{2.033, -1.240, 0.499, 0.061, 0.006, 0.075, -0.611, -0.179, 0.148, 1.224, 1.137, 1.136, 1.813, 3.040, 0.149}, {}},
    {{1.743, -0.920, 0.640, -0.040, -0.009, 0.049, -0.526, -0.291, 0.165, 1.304, 1.172, 1.136, 1.781, 5.390, 0.131}, {}},
    {{2.053, -0.572, 0.020, -0.040, 0.014, -0.150, -0.278, -0.053, 0.118, 1.219, 1.108, 1.073, 1.844, 5.286, 0.162},
     {2.371, -0.577, -0.168, -0.103, 0.100, -0.247, -0.402, 0.069, 0.160, 1.203, 1.045, 1.100, 1.580, 5.086, 0.142}},
    {{2.095, -0.519, -0.107, -0.089, 0.007, -0.154, -0.253, 0.255, 0.004, 1.254, 1.043, 1.073, 1.200, 11.641, 0.098},
     {1.686, -0.455, -0.179, -0.008, 0.097, -0.216, -0.378, 0.057, 0.132, 1.229, 1.057, 1.100, 1.570, 6.935, 0.145}},
    {{1.558, 0.565, 0.001, 0.086, 0.001, -0.329, -0.827, -0.182, -0.400, 1.158, 1.004, 0.900, 1.200, 10.146, 0.126},
     {2.347, -0.300, -0.098, 0.200, 0.107, -0.921, 0.091, 0.023, -0.223, 1.106, 1.142, 1.100, 1.718, 8.993, 0.141}},
    {{2.039, 0.773, 0.001, 0.086, 0.001, -0.329, 0.186, -0.182, -0.400, 1.158, 1.004, 0.900, 1.200, 10.146, 0.090},
     {1.576, -0.137, -0.049, 0.247, 0.065, -0.856, 0.186, 0.050, -0.400, 1.128, 1.147, 1.100, 1.384, 10.481, 0.128}}};

static_assert([] {  // every form that the library may take has constants
    for (int D = 32; D <= 256; D += 32)
        if (block_head_size(D) == D)
            for (int is = 0; is < 4; ++is)
                if (!(kBlockCost[block_width(D)][library_form(D, is & 1, is & 2) == 3].power > 0) || !(kBlockCost[block_width(D)][0].power > 0)) return false;
    return true;
}());

struct TypeTimes { double f16, bf16; };  // us with float16 and with bfloat16 inputs

// MB that a call on masks which touch `keys` keys reads and writes (the kernel's width in place of the head size)
static double call_mb(const smha_plan *plan, int B, int H, int D, int keys) {
    return 4e-6 * B * H * D * ((double)plan->S + std::min(keys, plan->Sk));
}

// The wave form.  Every wave has its start and end, every step its share of the chip; a workgroup's places are partly
// `held` until its longest wave ends, and steps of partly filled tiles and bfloat16 cost more.  A list shared by four
// waves is a chain of a quarter, but four starts and a merge: `alone` is the longest list that one wave walks, chosen
// for the least time (within 2 % of the best of the 12 in the mean).  us with the longest lists alone / shared:
// Longformer 8 x 12 x 512 x 64 14.1 / 8.8, window 1 x 2 x 1772 x 32 7.2 / 4.4.
static TypeTimes wave_time_us(const smha_plan *plan, int B, int H, int D, int &alone) {
    const WaveLists &wl = plan->wave;
    const double per_mask = 1.0 / (plan->Bm * plan->Hm), heads = (double)B * H;
    const WaveCost &c = kWaveCost[block_width(D)];
    const double slots = 4.0 * wave_groups(D) * plan->n_cu;
    const double part = (double)wl.part_ents / std::max<double>(1.0, (double)wl.n_ents);
    const double step_ns = c.step * (1 + c.part * part);
    int lengths[kWaveWhole + 1], n_lengths = 0;  // those that any item has, longest first
    for (int n = kWaveWhole; n >= 0; --n)
        if (wl.of_length[n] > 0) lengths[n_lengths++] = n;
    TypeTimes best{0, 0};
    alone = 0;
    for (int limit : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64}) {
        double teams = 0, solos = 0, steps = 0, held = 0, left = 0;  // of a mask; left: places in a workgroup already opened
        int chain = 0;
        for (int i = 0; i < n_lengths; ++i) {
            const int n = lengths[i];
            double k = per_mask * wl.of_length[n];
            steps += k * n;
            const int walked = n > limit ? (n + 3) / 4 : n;
            chain = std::max(chain, walked);
            if (n > limit) {
                teams += k;
                held += 4 * k * walked;
                continue;
            }
            solos += k;
            const double filled = std::min(k, left);
            left -= filled;
            k -= filled;
            const double opened = std::ceil(k / 4 - 1e-9);
            held += 4 * opened * n;
            left += 4 * opened - k;
        }
        const double waves = heads * (4 * teams + solos), groups = heads * (teams + std::ceil(solos / 4));
        const double uneven = groups > plan->n_cu ? std::ceil(groups / plan->n_cu) * plan->n_cu / groups - 1 : 0;
        const double walked = heads * (steps + c.held * (held - steps)) * step_ns;
        const double longest = chain * (c.chain + c.chain_full * std::min(1.0, waves / slots));
        auto us = [&](double type) {
            return std::pow(std::pow(1e-3 * (waves * c.wave + walked * type) * (1 + c.uneven * uneven), c.power) + std::pow(longest * type, c.power), 1 / c.power);
        };
        const double at = us(1.0);  // (the same limit for both types: one order serves them)
        if (alone == 0 || at < best.f16) {
            best = {at, us(c.bf16)};
            alone = limit;
        }
    }
    const double part_all = std::exp(c.part_all * part), memory = std::pow(c.memory * call_mb(plan, B, H, D, wl.keys), c.join);
    auto joined = [&](double us) { return c.start + std::pow(std::pow(us * part_all, c.join) + memory, 1 / c.join); };
    return {joined(best.f16), joined(best.bf16)};
}

// The first (four waves of 32 rows) and third form (eight of 16): the busiest compute unit's work and the longest
// workgroup's chain, in steps plus 2 per item (see build_work_order).  A step's cost follows the tile rows that have work
// in it (`act`: tiles per step), how many of the tiles are partly filled, how many 32 x 32 sub-tiles have keys (`subs`) and
// whether most steps are full tiles that one tile row has to itself (`lone`: the other's waves only wait); merging parts of
// a cut list costs extra.
static TypeTimes block_time_us(const smha_plan *plan, int lvl, int form, int B, int H, int D) {
    const WorkLists &wl = plan->lists[plan->fine_differs ? lvl : 0];
    const double per_xcd = (double)B * H / (plan->Bm * plan->Hm) / 8;
    double cost = 0, longest = 0;
    for (const Item &i : wl.items) {
        cost += 2 + i.end - i.begin;
        longest = std::max(longest, 2.0 + i.end - i.begin);
    }
    const double total = cost * per_xcd, items = (double)wl.items.size() * per_xcd;
    const double units = std::max(plan->n_cu / 8, 1), slots = units * (form == 3 ? block16_groups(D) : block_groups(D, plan->n_gathered > 0));
    const double unit = items > units ? std::max(longest, total / units + 0.35 * total / items) : longest;
    const double group = std::max(longest, total / std::max(1.0, std::min(slots, items)));
    int64_t tiles = 0, part = 0;
    for (const MaskFormats &m : plan->masks) {
        tiles += (int64_t)m.kt_col.size();
        part += (int64_t)(m.kt_bits().size() / 64);
    }
    const BlockCost &c = kBlockCost[block_width(D)][form == 3];
    const double steps = std::max<double>(1.0, (double)plan->h_uent.size() - 1);
    const double parts = tiles ? (double)part / (double)tiles : 0.0, act = std::min(2.0, (double)tiles / steps);
    const double subs = (double)plan->wave.n_ents / steps;
    const double lone = (1 - parts) * std::min(1.0, std::max(0.0, (1.35 - act) / 0.3));
    const double gather = plan->n_gathered > 0 ? c.gather : 1.0;
    const double unit_us = unit * std::exp(c.unit + c.unit_act * (act - 1.5) + c.unit_part * act * parts + c.unit_sub * (subs - 5) + c.unit_lone * lone);
    const double group_us = group * std::exp(c.group + c.group_act * (act - 1.5) + c.group_part * act * parts);
    const double memory = std::pow(c.memory * call_mb(plan, B, H, D, plan->wave.keys), c.power);
    auto us = [&](double unit_type, double group_type) {
        return c.start + (wl.max_slots > 0 ? c.merge : 0.0) +
               std::pow(std::pow(gather * unit_us * unit_type, c.power) + std::pow(gather * group_us * group_type, c.power) + memory, 1 / c.power);
    };
    return {us(1.0, 1.0), us(c.unit_bf16, c.group_bf16)};
}

// The wave form wins where tiles are filled poorly (BigBird with random 32-blocks 16 x 12 x 2048 x 64: 126 us, 77 with
// the wave form) and where a call has too few 128-row groups to fill the chip (causal 1 x 12 x 1024 x 64 15.2 / 8.5, per-head
// 64-blocks 1 x 2 x 2816 x 256 20.6 / 12.8); it loses where tiles are full and rows many (causal 16 x 12 x 4096 x 128:
// 870 / 1176), because every K and V tile is loaded once per 32 rows.  It has to win by 4 %: of 1600
// calls of the table that were drawn at random 15 then run the slower form by more than 2 % with one of the input types, and the mean
// against the other forms is 0.639, 0.675, 0.687, 0.722, 0.659, 0.725 at 32, 64, 96, 128, 160 and 256 columns, where the better form for
// each call would give 0.639, 0.672, 0.684, 0.718, 0.653, 0.722.
// The two input types are decided together (by the product of their ratios): one order and one set of workspaces serves both.
bool wave_form_pays(const smha_plan *plan, int lvl, int form, int B, int H, int D, int &alone) {
    if (H > 65535 || (int64_t)B * H > (1 << 18) /* (a grid's z holds an eighth of them) */) return false;
    if (!count_wave_lists(plan)) return false;
    if (workspace_bytes(plan, 0, 4, B, H, D, nullptr) > kStaticScratchBytes) return false;  // (smha_forward_static takes what it took)
    const TypeTimes wave = wave_time_us(plan, B, H, D, alone), block = block_time_us(plan, lvl, form, B, H, D);
    return wave.f16 * wave.bf16 < 0.96 * 0.96 * block.f16 * block.bf16;
}

// The block kernel's work order for B x H heads on `slots` resident workgroups per XCD.  Items
// differ in length (tile rows under global tokens, random blocks, padding), and with equal item
// counts per workgroup the slowest one ends well after the average one; so the items of each head
// go, longest first, to the compute unit with the least work so far and there to the workgroup with the
// least (cost: tiles plus a fixed part per item), head after head so that an XCD's workgroups stay on
// one head's K/V at a time.  The last heads, at most 2.25 items per workgroup of them (or one head), are dealt together,
// longest first over all of them, so that the last item dealt is a short one.  Their K and V are then in use at once,
// and an XCD's L2 holds 4 MB: with three items per workgroup at 128 and 256 columns BigBird blocks 2 x 20 x 3200 x 160 took
// 125.8 us instead of 108.4 with one head at a time (padded; three heads of 2 MB; with 2.25 items 107.4), per-head 32-blocks
// 3 x 32 x 2624 x 112 bf16 126 instead of 103 (110), and the mean over 113 masks was the same; two items: the same in
// the mean, BigBird blocks 1 x 32 x 8192 x 128 132.9 us instead of 130.9.  At 64 columns heads are half as large: three
// items, never more than 1 % slower than one head at a time on 37 masks (BigBird 16 x 12 x 2048 112.7 us, with two or
// 2.25 items 114.4).  Fine lists at 64 columns (few heads, every list cut into parts of about one length) with more than
// one item per workgroup and fewer than two are dealt head after head: together, the groups of all heads have their
// last parts in the second turn and are merged at the end (causal 1 x 20 x 3000 x 64 55.7 us instead of 47.0, BigBird
// 1 x 12 x 4096 x 64 58.5 instead of 54.6; with two items and more together is faster again, BigBird 1 x 10 x 5000 x 64
// 71.5 against 82.2, and so it is at 128 columns, causal 1 x 10 x 2500 x 128 50.9 against 53.3).
// The workgroups of ranks r, r + n_cu / 8, ... of an XCD share a compute unit (measured, all 1024 of them), and
// what a launch waits for is the unit with the most work.  Where four share one, the older ones are faster: the
// hardware issues the oldest wave first (equal work ended at 0.92 : 0.97 : 1.04 : 1.09 of the mean, the same on
// four masks), so work is dealt in that proportion (BigBird blocks 4 x 16 x 4000 x 64 66.8 -> 63.7 us, BigBird 16 x 12 x 2048
// 111.9 -> 113.4, most masks the same).
// spread: heads that are left over when their number is no multiple of 8 (all of them, if there are fewer) are not given
// to one XCD each but dealt over all: the eight XCDs stand in a row, each left-over head takes the same stretch of them
// (one or a few, so that its K and V come to few L2s), and its items go, longest first, to the XCD in that stretch with
// the least of them so far.  Without it 12 heads are two for four XCDs and one for the others: causal
// 5 x 12 x 3313 x 80 bf16 228.6 us, spread 214.9, BigBird blocks 3 x 12 x 4928 x 160 179.7 and 161.2, per-head 64-blocks
// 3 x 12 x 3712 x 96 61.3 and 55.9; 60 such calls 0.98 in the mean, none more than 2 % slower.
// table = {start of each XCD's list (8), its length (8), then (batch*head, item index) pairs};
// list position = turn * per_xcd + workgroup rank; a workgroup's unused turns hold batch*head = -1.
void build_work_order(const smha_plan *plan, int lvl, int B, int H, int slots, bool spread, std::vector<int32_t> &table, int &per_xcd) {
    const WorkLists &wl = plan->lists[plan->fine_differs ? lvl : 0];
    const int BH = B * H;
    auto mask_of = [&](int bh) { return (plan->Bm > 1 ? bh / H : 0) * plan->Hm + (plan->Hm > 1 ? bh % H : 0); };
    constexpr int kItemCost = 2;  // an item's start and end, in tiles
    // what each XCD gets: all items of every eighth head, then those items of left-over heads that are listed in `some`
    struct Share { int32_t bh; std::vector<int32_t> some; };
    std::vector<Share> parts[8];
    const int left_over = spread ? BH % 8 : 0, whole = BH - left_over;
    auto whole_heads = [&](int x) { return (whole - x + 7) / 8; };
    int64_t dealt[8] = {0};
    for (int l = 0; l < left_over; ++l) {
        const int mask = mask_of(whole + l), first = 8 * l / left_over, last = (8 * (l + 1) - 1) / left_over;
        for (int x = first; x <= last; ++x) parts[x].push_back({whole + l, {}});
        for (int32_t it = 0; it < wl.item_cnt[mask]; ++it) {
            const Item &item = wl.items[wl.item_off[mask] + it];
            int to = first;
            for (int x = first + 1; x <= last; ++x)
                if (dealt[x] < dealt[to]) to = x;
            dealt[to] += kItemCost + (item.end - item.begin);
            parts[to].back().some.push_back(it);
        }
        for (int x = first; x <= last; ++x)
            if (parts[x].back().some.empty()) parts[x].pop_back();
    }
    // of XCD x's i-th head: which it is, how many items, and which (null: all of them)
    auto head = [&](int x, int i) { return i < whole_heads(x) ? x + 8 * i : parts[x][i - whole_heads(x)].bh; };
    auto listed = [&](int x, int i) { return i < whole_heads(x) ? nullptr : parts[x][i - whole_heads(x)].some.data(); };
    auto count = [&](int x, int i) {
        return i < whole_heads(x) ? (int64_t)wl.item_cnt[mask_of(x + 8 * i)] : (int64_t)parts[x][i - whole_heads(x)].some.size();
    };
    auto heads = [&](int x) { return whole_heads(x) + (int)parts[x].size(); };
    int64_t items_of[8], most = 0;  // of the busiest XCD
    for (int x = 0; x < 8; ++x) {
        items_of[x] = 0;
        for (int i = 0; i < heads(x); ++i) items_of[x] += count(x, i);
        most = std::max(most, items_of[x]);
    }
    // (as many workgroups on every compute unit: an odd one would be a unit that takes its second item late)
    const int n_units = (int)std::min<int64_t>({(int64_t)std::max(plan->n_cu / 8, 1), (int64_t)slots, most});
    table.assign(16, 0);
    per_xcd = 0;
    if (most == 0) return;
    per_xcd = (int)std::min<int64_t>(slots, (most + n_units - 1) / n_units * n_units);
    const bool aged = slots == 4 * n_units, fine = lvl == 1 && plan->fine_differs;
    static const double kPace[4] = {1.09, 1.03, 0.96, 0.92};
    struct Pick { int32_t bh, index, cost; };
    std::vector<Pick> deal, sorted;
    std::vector<int32_t> start;
    // units by work so far, least on top: work << 20 | unit
    std::vector<int64_t> heap(n_units);
    std::vector<double> done(per_xcd);    // a workgroup's work so far, in terms of its pace
    std::vector<int32_t> turns(per_xcd);  // items it has
    for (int x = 0; x < 8; ++x) {
        if (x > 0 && left_over == 0 && plan->Bm * plan->Hm == 1 && (BH - 1 - x + 8) / 8 == (BH - x + 8) / 8) {
            // one mask for all heads, and as many heads as the XCD before: its deal, one head on
            const size_t from = 16 + 2 * (size_t)table[x - 1], n = 2 * (size_t)table[8 + x - 1];
            table[x] = (int32_t)((table.size() - 16) / 2);
            table[8 + x] = table[8 + x - 1];
            table.reserve(table.size() + (8 - x) * n);
            for (size_t i = from; i < from + n; i += 2) {
                const int32_t bh = table[i], index = table[i + 1];
                table.push_back(bh < 0 ? bh : bh + 1);
                table.push_back(index);
            }
            continue;
        }
        const size_t base = table.size();
        table[x] = (int32_t)((base - 16) / 2);
        int n_turns = 0;
        for (int u = 0; u < n_units; ++u) heap[u] = u;
        std::fill(done.begin(), done.end(), 0.0);
        std::fill(turns.begin(), turns.end(), 0);
        const int last = heads(x) - 1;  // this XCD's last head
        int joint = last;               // first head of the joint deal
        const int64_t here = items_of[x];
        const bool apart = aged && fine && here > per_xcd && here < 2 * (int64_t)per_xcd;
        for (int64_t n = 0; joint >= 0; --joint) {
            n += count(x, joint);
            if (apart && joint != last) break;
            if (4 * n > (aged ? 12 : 9) * (int64_t)per_xcd && joint != last) break;
        }
        ++joint;
        for (int i = 0; i <= last; ++i) {
            const int32_t bh = head(x, i);
            const int32_t *const some = listed(x, i);
            const int32_t off = wl.item_off[mask_of(bh)];
            if (i <= joint) deal.clear();
            const int64_t n = count(x, i);
            for (int64_t k = 0; k < n; ++k) {  // (sorted by length, longest first)
                const int32_t it = some ? some[k] : (int32_t)k;
                const Item &item = wl.items[off + it];
                deal.push_back({bh, off + it, kItemCost + (item.end - item.begin)});
            }
            if (i >= joint && i != last) continue;
            const bool mixed = joint < last && i == last;
            if (mixed) {  // longest first over all of them, head after head where equal: a counting sort
                int32_t top = 0;
                for (const Pick &p : deal) top = std::max(top, p.cost);
                start.assign((size_t)top + 2, 0);
                for (const Pick &p : deal) ++start[top - p.cost + 1];
                for (int32_t c = 0; c <= top; ++c) start[c + 1] += start[c];
                sorted.resize(deal.size());
                for (const Pick &p : deal) sorted[start[top - p.cost]++] = p;
                deal.swap(sorted);
            }
            for (const Pick &p : deal) {
                const int unit = (int)(heap[0] & 0xFFFFF);
                const int64_t load = heap[0] + ((int64_t)p.cost << 20);
                for (int at = 0;;) {  // (the top's new place)
                    int child = 2 * at + 1;
                    if (child >= n_units) { heap[at] = load; break; }
                    if (child + 1 < n_units) child += heap[child + 1] < heap[child];
                    if (heap[child] >= load) { heap[at] = load; break; }
                    heap[at] = heap[child];
                    at = child;
                }
                int best = unit;
                for (int r = unit + n_units; r < per_xcd; r += n_units)
                    if (done[r] < done[best]) best = r;
                done[best] += aged ? p.cost / kPace[best / n_units & 3] : (double)p.cost;
                if (turns[best] == n_turns) {
                    ++n_turns;
                    const size_t row = table.size();
                    table.resize(row + 2 * (size_t)per_xcd, 0);
                    for (int r = 0; r < per_xcd; ++r) table[row + 2 * (size_t)r] = -1;
                }
                // (its place among the workgroup's items: head after head)
                const size_t pitch = 2 * (size_t)per_xcd;
                int32_t *to = table.data() + base + pitch * turns[best]++ + 2 * (size_t)best;
                for (; mixed && to >= table.data() + base + pitch && to[-(ptrdiff_t)pitch] > p.bh; to -= pitch) {
                    to[0] = to[-(ptrdiff_t)pitch];
                    to[1] = to[1 - (ptrdiff_t)pitch];
                }
                to[0] = p.bh;
                to[1] = p.index;
            }
        }
        table[8 + x] = (int32_t)(n_turns * per_xcd);
    }
}

}  // namespace smha

using namespace smha;

extern "C" smha_status_t smha_plan_from_dense(const uint8_t *mask, int mask_on_device, int Bm,
                                              int Hm, int S, const smha_plan_opts_t *opts,
                                              smha_plan_t **out) {
    return smha_plan_from_dense_rect(mask, mask_on_device, Bm, Hm, S, S, opts, out);
}

extern "C" smha_status_t smha_plan_from_dense_rect(const uint8_t *mask, int mask_on_device, int Bm,
                                                   int Hm, int Sq, int Sk, const smha_plan_opts_t *opts,
                                                   smha_plan_t **out) {
    if (!mask || !out || Bm < 1 || Hm < 1 || Sq < 1 || Sk < 1) return SMHA_ERR_INVALID_ARG;
    smha_plan_opts_t o;
    smha_status_t st = check_opts(opts, o);
    if (st != SMHA_OK) return st;
    try {
        std::unique_ptr<smha_plan> p(new smha_plan);
        p->S = Sq; p->Sk = Sk; p->Bm = Bm; p->Hm = Hm; p->block = o.block; p->opts = o;
        const size_t per_mask = (size_t)Sq * Sk;
        const size_t words_per_mask = (size_t)Sq * ((Sk + 63) / 64);
        // A device mask whose plan needs neither per-row lists nor tiles narrower than 64 is analysed
        // by the GPU itself: 16 bytes per tile and the bitmaps of partially filled tiles cross over.
        bool analysed = false;
        if (mask_on_device && o.block == 64 && !rows_wanted(o)) {
            std::vector<TileInfo> info;
            std::vector<std::vector<uint64_t>> part_bits;
            st = classify_device_mask(mask, Bm * Hm, Sq, Sk, info, part_bits);
            if (st != SMHA_OK) return st;
            const int nqt = (Sq + 63) / 64, nkt = (Sk + 63) / 64;
            p->masks.assign((size_t)Bm * Hm, MaskFormats{});
            for (int mi = 0; mi < Bm * Hm; ++mi)
                formats_from_tiles(info.data() + (size_t)mi * nqt * nkt, part_bits[mi], nqt, nkt, p->masks[mi]);
            analysed = !row_may_be_chosen(p.get());  // (else: the row kernel may win, which needs the per-row lists)
        }
        std::vector<uint64_t> packed;  // otherwise a device mask is packed to bits on the GPU: 1/8 of the bytes cross over
        if (mask_on_device && !analysed) {
            packed.resize(words_per_mask * Bm * Hm);
            st = pack_device_mask(mask, Bm * Hm, Sq, Sk, packed.data());
            if (st != SMHA_OK) return st;
        }
        auto analyse_all = [&](bool rows) {
            p->masks.assign((size_t)Bm * Hm, MaskFormats{});
            for (int mi = 0; mi < Bm * Hm; ++mi) {
                smha_status_t s1;
                if (mask_on_device) {
                    BitSource src(packed.data() + words_per_mask * mi, Sk);
                    s1 = analyse_mask(src, Sq, Sk, o.block, rows, p->masks[mi]);
                } else {
                    DenseSource src(mask + per_mask * mi, Sk);
                    s1 = analyse_mask(src, Sq, Sk, o.block, rows, p->masks[mi]);
                }
                if (s1 != SMHA_OK) return s1;
            }
            return SMHA_OK;
        };
        if (!analysed) {
            st = analyse_all(rows_wanted(o));
            if (st == SMHA_OK && !rows_wanted(o) && row_may_be_chosen(p.get())) st = analyse_all(true);
            if (st != SMHA_OK) return st;
        }
        st = finish_plan(p.get());
        if (st != SMHA_OK) { release_device(p.get()); return st; }
        *out = p.release();
        return SMHA_OK;
    } catch (const std::bad_alloc &) {
        return SMHA_ERR_ALLOC;
    }
}

extern "C" smha_status_t smha_plan_from_desc(const smha_mask_desc_t *desc, int B, int H, int S,
                                             const smha_plan_opts_t *opts, smha_plan_t **out) {
    if (!desc || !out || B < 1 || H < 1 || S < 1) return SMHA_ERR_INVALID_ARG;
    const smha_mask_desc_t &d = *desc;
    const uint32_t known = SMHA_MASK_CAUSAL | SMHA_MASK_WINDOW | SMHA_MASK_GLOBAL | SMHA_MASK_STRIDED |
                           SMHA_MASK_BLOCK_RANDOM | SMHA_MASK_BIGBIRD | SMHA_MASK_PADDING;
    if (d.flags & ~known) return SMHA_ERR_INVALID_ARG;
    if ((d.flags & SMHA_MASK_WINDOW) && (d.window_left < 0 || d.window_right < 0)) return SMHA_ERR_INVALID_ARG;
    if ((d.flags & SMHA_MASK_GLOBAL) && d.n_global < 0) return SMHA_ERR_INVALID_ARG;
    if ((d.flags & SMHA_MASK_STRIDED) && (d.stride < 1 || d.stride_phase < 0 || d.stride_phase >= d.stride))
        return SMHA_ERR_INVALID_ARG;
    if (d.flags & (SMHA_MASK_BLOCK_RANDOM | SMHA_MASK_BIGBIRD)) {
        if (d.block < 1) return SMHA_ERR_INVALID_ARG;
        if ((d.flags & SMHA_MASK_BLOCK_RANDOM) && !(d.keep_p >= 0.0 && d.keep_p <= 1.0)) return SMHA_ERR_INVALID_ARG;
        if ((d.flags & SMHA_MASK_BIGBIRD) &&
            (d.n_window_blocks < 0 || d.n_global_blocks < 0 || d.n_random_blocks < 0))
            return SMHA_ERR_INVALID_ARG;
    }
    if (d.flags & SMHA_MASK_PADDING) {
        if (!d.valid_len) return SMHA_ERR_INVALID_ARG;
        for (int b = 0; b < B; ++b)
            if (d.valid_len[b] < 0 || d.valid_len[b] > S) return SMHA_ERR_INVALID_ARG;
    }
    smha_plan_opts_t o;
    smha_status_t st = check_opts(opts, o);
    if (st != SMHA_OK) return st;
    try {
        std::unique_ptr<smha_plan> p(new smha_plan);
        const int Bm = (d.flags & SMHA_MASK_PADDING) ? B : 1;
        const int Hm = (d.per_head && (d.flags & (SMHA_MASK_BLOCK_RANDOM | SMHA_MASK_BIGBIRD))) ? H : 1;
        p->S = S; p->Sk = S; p->Bm = Bm; p->Hm = Hm; p->block = o.block; p->opts = o;
        auto analyse_all = [&](bool rows) {
            p->masks.assign((size_t)Bm * Hm, MaskFormats{});
            for (int b = 0; b < Bm; ++b)
                for (int h = 0; h < Hm; ++h) {
                    const int valid = (d.flags & SMHA_MASK_PADDING) ? d.valid_len[b] : S;
                    DescSource src(d, S, h, valid);
                    const smha_status_t s1 = analyse_mask(src, S, S, o.block, rows, p->masks[(size_t)b * Hm + h]);
                    if (s1 != SMHA_OK) return s1;
                }
            return SMHA_OK;
        };
        st = analyse_all(rows_wanted(o));
        if (st == SMHA_OK && !rows_wanted(o) && row_may_be_chosen(p.get())) st = analyse_all(true);
        if (st != SMHA_OK) return st;
        st = finish_plan(p.get());
        if (st != SMHA_OK) { release_device(p.get()); return st; }
        *out = p.release();
        return SMHA_OK;
    } catch (const std::bad_alloc &) {
        return SMHA_ERR_ALLOC;
    }
}

static smha_status_t export_order(const smha_plan_t *p, int B, int H, int workgroups_per_xcd, int fine, bool spread,
                                  int32_t *host_dst, size_t cap, size_t *need, int *per_xcd) {
    if (!p || !need || B < 1 || H < 1 || workgroups_per_xcd < 1 || fine < 0 || fine > 1) return SMHA_ERR_INVALID_ARG;
    if (cap > 0 && !host_dst) return SMHA_ERR_INVALID_ARG;
    if ((p->Bm != 1 && p->Bm != B) || (p->Hm != 1 && p->Hm != H)) return SMHA_ERR_SHAPE;
    if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
    if ((int64_t)B * H > (1 << 24)) return SMHA_ERR_UNSUPPORTED;
    std::vector<int32_t> table;
    int n = 0;
    try { build_work_order(p, fine, B, H, workgroups_per_xcd, spread, table, n); } catch (const std::bad_alloc &) { return SMHA_ERR_ALLOC; }
    *need = table.size();
    if (per_xcd) *per_xcd = n;
    if (cap >= table.size()) std::memcpy(host_dst, table.data(), table.size() * sizeof(int32_t));
    return SMHA_OK;
}

extern "C" smha_status_t smha_plan_work_order(const smha_plan_t *p, int B, int H, int workgroups_per_xcd, int fine,
                                              int32_t *host_dst, size_t cap, size_t *need, int *per_xcd) {
    return export_order(p, B, H, workgroups_per_xcd, fine, false, host_dst, cap, need, per_xcd);
}

extern "C" smha_status_t smha_plan_call_order(const smha_plan_t *p, int B, int H, int workgroups_per_xcd, int fine,
                                              int32_t *host_dst, size_t cap, size_t *need, int *per_xcd) {
    return export_order(p, B, H, workgroups_per_xcd, fine, true, host_dst, cap, need, per_xcd);
}

extern "C" smha_status_t smha_plan_row_form(const smha_plan_t *p, int B, int H, int d, int *rows_per_wave, int *keys_in_flight) {
    if (!p || B < 1 || H < 1 || !rows_per_wave || !keys_in_flight) return SMHA_ERR_INVALID_ARG;
    if (d < 8 || d > 256 || d % 8 || !p->has_row) return SMHA_ERR_UNSUPPORTED;
    if ((p->Bm != 1 && p->Bm != B) || (p->Hm != 1 && p->Hm != H)) return SMHA_ERR_SHAPE;
    const int D = d <= 64 ? 64 : d <= 128 ? 128 : 256;
    const RowForm form = kRowForms[row_width(D)][row_form(p, B, H, D)];
    *rows_per_wave = form.rows;
    *keys_in_flight = form.batch;
    return SMHA_OK;
}

extern "C" smha_status_t smha_plan_info(const smha_plan_t *p, smha_plan_info_t *out) {
    if (!p || !out) return SMHA_ERR_INVALID_ARG;
    smha_plan_info_t i{};
    i.n_gathered = p->n_gathered;
    i.S = p->S; i.Sk = p->Sk; i.Bm = p->Bm; i.Hm = p->Hm; i.block = p->block; i.kernel = p->kernel;
    i.has_row_format = p->has_row; i.has_block_kernel_lists = p->has_block; i.on_device = p->device >= 0;
    for (auto &m : p->masks) {
        i.nnz += m.nnz;
        i.n_valid += (int64_t)m.load_col_idx.size();
        i.n_full += (int64_t)m.full_col_idx.size();
        i.n_part += (int64_t)m.part_col_idx.size();
        i.n_valid16 += m.n_valid16;
        i.n_tiles64 += (int64_t)m.kt_col.size();
    }
    i.n_union = p->h_uent.empty() ? 0 : (int64_t)p->h_uent.size() - 1;  // (without the spare entry)
    i.n_items = (int64_t)p->lists[0].items.size();
    i.n_split_rows = (int64_t)p->lists[0].split_rows.size();
    i.eq1_threshold = p->eq1_threshold;
    i.model_row_us = p->model_row_us;
    i.model_block_us = p->model_block_us;
    *out = i;
    return SMHA_OK;
}

extern "C" smha_status_t smha_plan_export(const smha_plan_t *p, int mask_index, smha_export_t which,
                                          void *host_dst, size_t cap, size_t *need) {
    if (!p || !need || mask_index < 0 || mask_index >= p->Bm * p->Hm) return SMHA_ERR_INVALID_ARG;
    if (cap > 0 && !host_dst) return SMHA_ERR_INVALID_ARG;
    const MaskFormats &m = p->masks[mask_index];
    const void *src = nullptr;
    size_t bytes = 0;
    std::vector<uint64_t> it8;
    auto vec = [&](const auto &v) { src = v.data(); bytes = v.size() * sizeof(v[0]); };
    switch (which) {
        case SMHA_EXPORT_ROW_PTR:
            if (m.row_ptr.empty()) return SMHA_ERR_UNSUPPORTED;
            vec(m.row_ptr); break;
        case SMHA_EXPORT_COL_IDX:
            if (m.row_ptr.empty()) return SMHA_ERR_UNSUPPORTED;
            vec(m.col_idx); break;
        case SMHA_EXPORT_LOAD_ROW_PTR: vec(m.load_row_ptr); break;
        case SMHA_EXPORT_LOAD_COL_IDX: vec(m.load_col_idx); break;
        case SMHA_EXPORT_BLOCK_FLAGS: vec(m.flags); break;
        case SMHA_EXPORT_BITMAP: vec(m.bitmap); break;
        case SMHA_EXPORT_FULL_ROW_PTR: vec(m.full_row_ptr); break;
        case SMHA_EXPORT_FULL_COL_IDX: vec(m.full_col_idx); break;
        case SMHA_EXPORT_PART_ROW_PTR: vec(m.part_row_ptr); break;
        case SMHA_EXPORT_PART_COL_IDX: vec(m.part_col_idx); break;
        case SMHA_EXPORT_BITMAP_IT8: {
            if (p->block != 64) return SMHA_ERR_UNSUPPORTED;
            const size_t np = m.bitmap.size() / 64;
            try { it8.assign(np * 64, 0); } catch (const std::bad_alloc &) { return SMHA_ERR_ALLOC; }
            for (size_t t = 0; t < np; ++t)
                for (int ir = 0; ir < 8; ++ir)
                    for (int ic = 0; ic < 8; ++ic) {
                        uint64_t w = 0;
                        for (int r = 0; r < 8; ++r)
                            w |= ((m.bitmap[t * 64 + ir * 8 + r] >> (8 * ic)) & 0xFFull) << (8 * r);
                        it8[t * 64 + ic * 8 + ir] = w;
                    }
            vec(it8);
            break;
        }
        case SMHA_EXPORT_KERNEL_ENTRIES:
            if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
            src = p->h_uent.data(); bytes = (p->h_uent.size() - 1) * sizeof(UEntry); break;  // (without the spare entry)
        case SMHA_EXPORT_KERNEL_GATHER_KEYS:
            if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
            vec(p->h_gidx); break;
        case SMHA_EXPORT_KERNEL_BITMAPS:
            if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
            src = p->h_kt_bitmap.data(); bytes = (p->h_kt_bitmap.size() - 64) * sizeof(uint64_t); break;  // (without the spare block)
        case SMHA_EXPORT_KERNEL_ITEMS:
            if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
            src = p->lists[0].items.data() + p->lists[0].item_off[mask_index];
            bytes = (size_t)p->lists[0].item_cnt[mask_index] * sizeof(Item); break;
        case SMHA_EXPORT_KERNEL_ITEMS_FINE: {
            if (!p->has_block) return SMHA_ERR_UNSUPPORTED;
            const WorkLists &wl = p->lists[p->fine_differs ? 1 : 0];
            src = wl.items.data() + wl.item_off[mask_index];
            bytes = (size_t)wl.item_cnt[mask_index] * sizeof(Item); break;
        }
        case SMHA_EXPORT_WAVE_ITEMS:
        case SMHA_EXPORT_WAVE_ENTRIES:
            try {
                if (!count_wave_lists(p)) return SMHA_ERR_UNSUPPORTED;
                make_wave_lists(p);
            } catch (const std::bad_alloc &) {
                return SMHA_ERR_ALLOC;
            }
            if (which == SMHA_EXPORT_WAVE_ENTRIES) {
                src = p->wave.ents.data(); bytes = (p->wave.ents.size() - 1) * sizeof(WaveEntry); break;  // (without the spare entry)
            }
            src = p->wave.items.data() + p->wave.item_off[mask_index];
            bytes = (size_t)p->wave.item_cnt[mask_index] * sizeof(WaveItem); break;
        default: return SMHA_ERR_INVALID_ARG;
    }
    *need = bytes;
    if (cap >= bytes && bytes) std::memcpy(host_dst, src, bytes);
    return SMHA_OK;
}

extern "C" void smha_plan_destroy(smha_plan_t *p) {
    if (!p) return;
    release_device(p);
    delete p;
}

extern "C" const char *smha_status_string(smha_status_t s) {
    switch (s) {
        case SMHA_OK: return "ok";
        case SMHA_ERR_INVALID_ARG: return "invalid argument";
        case SMHA_ERR_UNSUPPORTED: return "unsupported configuration";
        case SMHA_ERR_SHAPE: return "shape mismatch";
        case SMHA_ERR_ALLOC: return "allocation failed";
        case SMHA_ERR_HIP: return "HIP error or no usable GPU";
    }
    return "unknown status";
}
