// vp_api.cpp -- host side of the C ABI declared in include/vp.h.
//
// Host work per call: validate the items, derive grid_thw / cu_seqlens,
// choose each item's kernel from its axes' windows, pack the plan into one blob
// in pinned host memory, and launch the kernel that copies it into the
// caller's workspace and computes the streaming kernels' filter tables there
// (double precision, rounded once to float), then the kernels themselves.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <list>
#include <array>
#include <map>
#include <memory>
#include <tuple>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "vp.h"
#include "vp_plan.h"

namespace {

thread_local std::string g_last_error;
thread_local hipEvent_t g_timing_start = nullptr;   // vp_set_kernel_events, one call
thread_local hipEvent_t g_timing_stop = nullptr;

int32_t fail(int32_t status, const std::string& msg) {
    g_last_error = msg;
    return status;
}

// ---------------------------------------------------------------------------
// smart_resize and frame-index sampling
// ---------------------------------------------------------------------------

// Nearest integer of a double, ties to the even neighbour.
double nearest_even(double v) {
    const double lower = std::floor(v);
    const double frac = v - lower;  // exact for |v| < 2^52
    if (frac != 0.5) return frac < 0.5 ? lower : lower + 1.0;
    return std::fmod(lower, 2.0) == 0.0 ? lower : lower + 1.0;
}

// Index i of n spread evenly over [0, last], rounded half to even on the
// exact rational i * last / (n - 1).
int32_t spread_index(int64_t i, int64_t last, int64_t n) {
    if (n == 1) return 0;
    const int64_t num = i * last, den = n - 1;
    int64_t whole = num / den;
    const int64_t twice_rem = 2 * (num - whole * den);
    if (twice_rem > den || (twice_rem == den && (whole & 1))) ++whole;
    return static_cast<int32_t>(whole);
}

// ---------------------------------------------------------------------------
// Antialiased bicubic filter tables
// ---------------------------------------------------------------------------

struct AxisFilter {
    int32_t n_in = 0, n_out = 0, taps = 0;
    std::vector<int32_t> start, count;
    std::vector<float> weight;   // [n_out][taps]
    std::vector<int32_t> fixed;  // [n_out][taps]: the double weights times 2^22, rounded
};

// Keys (1981) kernel, a = -1/2, evaluated as the polynomial is written
// (left to right, no reassociation): the fixed-point weights of the uint8
// writer are rounded from these doubles, so every machine must get the same
// bits.
double cubic_a_half(double x) {
    const double t = std::fabs(x);
    if (t < 1.0) return 1.5 * t * t * t - 2.5 * t * t + 1.0;
    if (t < 2.0) return -0.5 * t * t * t + 2.5 * t * t - 4.0 * t + 2.0;
    return 0.0;
}

// Window [lo, hi) of output i; the same double expressions as the documented
// definition, in the same order, so that window bounds are reproducible.
void window(int32_t n_in, int32_t n_out, int32_t i, double* centre, double* sigma, int32_t* lo,
            int32_t* hi) {
    const double scale = static_cast<double>(n_in) / static_cast<double>(n_out);
    const double s = scale > 1.0 ? scale : 1.0;
    const double support = 2.0 * s;
    const double c = (static_cast<double>(i) + 0.5) * scale;
    double a = std::floor(c - support + 0.5);
    double b = std::floor(c + support + 0.5);
    if (a < 0.0) a = 0.0;
    if (b > n_in) b = n_in;
    *centre = c;
    *sigma = s;
    *lo = static_cast<int32_t>(a);
    *hi = static_cast<int32_t>(b);
}

int32_t axis_taps(int32_t n_in, int32_t n_out) {
    int32_t best = 0;
    for (int32_t i = 0; i < n_out; ++i) {
        double c, s;
        int32_t lo, hi;
        window(n_in, n_out, i, &c, &s, &lo, &hi);
        if (hi - lo > best) best = hi - lo;
    }
    return best;
}

void build_axis(int32_t n_in, int32_t n_out, int32_t taps, AxisFilter* f) {
    f->n_in = n_in;
    f->n_out = n_out;
    f->taps = taps;
    f->start.assign(n_out, 0);
    f->count.assign(n_out, 0);
    f->weight.assign(static_cast<size_t>(n_out) * taps, 0.0f);
    f->fixed.assign(static_cast<size_t>(n_out) * taps, 0);
    std::vector<double> raw(taps);
    for (int32_t i = 0; i < n_out; ++i) {
        double c, s;
        int32_t lo, hi;
        window(n_in, n_out, i, &c, &s, &lo, &hi);
        double sum = 0.0;
        for (int32_t j = lo; j < hi; ++j) {
            raw[j - lo] = cubic_a_half((static_cast<double>(j) + 0.5 - c) / s);
            sum += raw[j - lo];
        }
        f->start[i] = lo;
        f->count[i] = hi - lo;
        for (int32_t j = lo; j < hi; ++j) {
            const double w = raw[j - lo] / sum;
            f->weight[static_cast<size_t>(i) * taps + (j - lo)] = static_cast<float>(w);
            const double x = w * 4194304.0;   // 2^22
            f->fixed[static_cast<size_t>(i) * taps + (j - lo)] =
                static_cast<int32_t>(x < 0.0 ? x - 0.5 : x + 0.5);   // half away from zero
        }
    }
}

// ---------------------------------------------------------------------------
// Plan
// ---------------------------------------------------------------------------

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Plan {
    std::vector<vp::DevItem> items;
    std::vector<int32_t> prefix;
    std::vector<int32_t> indices;
    // the tables section: cached table words, each placed at its word offset
    std::vector<std::pair<int32_t, std::shared_ptr<const std::vector<int32_t>>>> tables;
    size_t table_words = 0;
    std::vector<vp::StreamUnit> units;
    std::vector<uint32_t> wgs;   // streaming workgroups: unit | band << 20, grouped per launch
    std::vector<vp::StreamLaunch> launches;
    std::vector<int32_t> grid;  // [n][3]
    std::vector<int32_t> cu;    // [n + 1]
    int64_t total_rows = 0;
    int64_t long_unit_rows = 0;   // most source rows of a float streaming unit where none is cut short (INT64_MAX: over 8 slots)
    std::vector<int64_t> byte_off;   // uint8 writer: [n + 1] output byte offsets of the items
    int64_t generic_cost = 0;   // source pixels the general kernel reads, roughly
    int64_t generic_chain = 0;  // most steps of one of its workgroups, each waiting for a load (INT64_MAX: the tile kernel)
    // tables computed on the device: their pieces, their words, and where they
    // begin (the blob up to there is copied)
    std::vector<vp::TableJob> jobs;
    size_t gen_words = 0;
    size_t off_items = 0, off_prefix = 0, off_indices = 0, off_tables = 0, off_units = 0, off_wgs = 0, off_jobs = 0,
           off_gen = 0, bytes = 0;
    // no tables of the device's: the whole blob is copied
    void all_copied() { off_jobs = off_gen = bytes; }
};

int32_t item_patch(const vp_item& it) { return it.patch == 0 ? vp::kPatch : it.patch; }

// Every item of one call must share one patch size (the rows of one output
// buffer have one width).
int32_t batch_patch(const vp_item* items, int32_t n, int32_t* patch) {
    *patch = vp::kPatch;
    if (items == nullptr || n < 1) return VP_OK;   // reported by the caller's own checks
    *patch = item_patch(items[0]);
    for (int32_t b = 1; b < n; ++b)
        if (item_patch(items[b]) != *patch)
            return fail(VP_ERR_ARG, "items of one call must share one patch size (item " +
                                        std::to_string(b) + ")");
    return VP_OK;
}

int32_t validate_item(const vp_item& it, int32_t b) {
    const std::string at = "item " + std::to_string(b) + ": ";
    if (it.frames == nullptr) return fail(VP_ERR_NULL, at + "frames is NULL");
    if (it.indices == nullptr) return fail(VP_ERR_NULL, at + "indices is NULL");
    if (it.n_src < 1) return fail(VP_ERR_FRAMES, at + "n_src < 1");
    if (it.src_h < 1 || it.src_w < 1) return fail(VP_ERR_DIMS, at + "source size < 1");
    if (it.n_idx < 1) return fail(VP_ERR_FRAMES, at + "n_idx < 1");
    if (it.patch != 0 && it.patch != 14 && it.patch != 16)
        return fail(VP_ERR_ARG, at + "patch must be 14 or 16 (0 for 16)");
    const int32_t win = 2 * item_patch(it);
    if (it.dst_h < win || it.dst_w < win || it.dst_h % win || it.dst_w % win)
        return fail(VP_ERR_DIMS, at + "target size not a positive multiple of " + std::to_string(win));
    for (int32_t k = 0; k < it.n_idx; ++k)
        if (it.indices[k] < 0 || it.indices[k] >= it.n_src)
            return fail(VP_ERR_INDEX, at + "index " + std::to_string(it.indices[k]) +
                                          " outside [0, " + std::to_string(it.n_src) + ")");
    const int64_t fb = int64_t(it.src_h) * it.src_w * 3;
    if (fb >= (int64_t(1) << 32)) return fail(VP_ERR_CAPACITY, at + "a source frame of 4 GiB or more");
    return VP_OK;
}

// Largest generic sub-tile (rh x cw output pixels) whose y-resampled column
// tile fits the kernel's LDS buffer for every merge window of the item.
bool generic_subtile(const AxisFilter& fx, int32_t win, int32_t* rh, int32_t* cw) {
    std::vector<int32_t> sizes;   // the divisors of the window edge, largest first
    for (int32_t d = win; d >= 1; --d)
        if (win % d == 0) sizes.push_back(d);
    for (int32_t r : sizes) {
        for (int32_t c : sizes) {
            int32_t worst = 0;
            for (int32_t j0 = 0; j0 < fx.n_out; j0 += c) {
                const int32_t span = fx.start[j0 + c - 1] + fx.count[j0 + c - 1] - fx.start[j0];
                if (span > worst) worst = span;
            }
            if (int64_t(r) * worst * 3 <= vp::kGenericTCap) {
                *rh = r;
                *cw = c;
                return true;
            }
        }
    }
    return false;
}

// ---------------------------------------------------------------------------
// Streaming-kernel routing and tables
// ---------------------------------------------------------------------------

// Slots of a y axis for a streaming kernel.  Output row i lives in accumulator
// slot i mod M while it is open: from the first row of its window to its close
// row, the last row of its window (close rows never decrease; several output
// rows close on the same source row when the axis is upscaled, and at the
// bottom border).  M is the most output rows open at once (at least 4), so two
// open rows never share a slot.  Returns M, or -1 if the axis needs more than
// kSlotWords slots (which kernel shapes take that many is up to the caller);
// *close_rows (may be null) receives the close row of every output row.
int32_t count_slots(const AxisFilter& f, std::vector<int32_t>* close_rows) {
    const int32_t n_out = f.n_out, rows = f.n_in + vp::kSlotMax;
    std::vector<int32_t> close(n_out, 0);
    for (int32_t i = 0; i < n_out; ++i) {
        close[i] = f.start[i] + f.count[i] - 1;
        if (i > 0 && (f.start[i] < f.start[i - 1] || close[i] < close[i - 1])) return -1;
    }
    // most rows open at once: a row is open on [start, close]
    std::vector<int32_t> delta(rows + 1, 0);
    for (int32_t i = 0; i < n_out; ++i) {
        ++delta[f.start[i]];
        --delta[close[i] + 1];
    }
    int32_t open = 0, most = 0;
    for (int32_t y = 0; y < rows; ++y) {
        open += delta[y];
        most = open > most ? open : most;
    }
    if (most > vp::kSlotWords) return -1;
    if (close_rows != nullptr) *close_rows = std::move(close);
    return most < 4 ? 4 : most;
}

// Slot table of a y axis for the uint8 writer's dot-product form: for every
// source row y and slot s < M the fixed-point weight of y in the output row
// that has slot s at y (zero if that row does not read y), then the close row
// of every output row, and two that no row reaches (the kernel reads one close
// row ahead).  (The float kernels' slot tables, laid out alike, and their
// column tables are computed on the device.)  Returns M or -1 as count_slots.
int32_t build_slots(const AxisFilter& f, std::vector<int32_t>* words) {
    std::vector<int32_t> close;
    const int32_t m = count_slots(f, &close);
    if (m < 0) return -1;
    const int32_t rows = f.n_in + vp::kSlotMax;
    words->assign(size_t(rows) * m + f.n_out + 2, 0);
    for (int32_t i = 0; i < f.n_out; ++i)
        for (int32_t k = 0; k < f.count[i]; ++k)
            (*words)[size_t(f.start[i] + k) * m + i % m] = f.fixed[size_t(i) * f.taps + k];
    std::memcpy(words->data() + size_t(rows) * m, close.data(), sizeof(int32_t) * f.n_out);
    (*words)[size_t(rows) * m + f.n_out] = INT32_MAX;
    (*words)[size_t(rows) * m + f.n_out + 1] = INT32_MAX;
    return m;
}

// Column table of an x axis for the uint8 streaming writer.  The kernel
// keeps each channel of a band's source row as signed bytes (value - 128),
// and column j reads kx of them from a dword-aligned start s_j (its window
// start relative to the band's x0, rounded down to a multiple of 4, lowered
// so that s_j + kx <= row_px), with the window's weights shifted to match.
// Each weight q splits into balanced base-256 digits, q = d2 2^16 + d1 2^8
// + d0 with every digit in [-128, 127], so that byte dot products (dot4 of
// four digits with four values) form the sums.  Per column: s_j / 4, then
// 128 * (sum of q) + 2^21 (the offset of the values and the rounding term),
// then for digits d0, d1, d2 the kx / 4 dwords of four taps' digits.
// Returns false if a weight does not fit three digits.
bool build_columns_dot(const AxisFilter& f, int32_t kx, int32_t band, int32_t row_px,
                       std::vector<int32_t>* words) {
    const int32_t g = kx / 4;
    const int32_t n = f.n_out;
    words->assign(size_t(n) * (2 + 3 * g), 0);
    int32_t* start = words->data();
    int32_t* cterm = start + n;
    int32_t* dig = cterm + n;
    for (int32_t j = 0; j < n; ++j) {
        const int32_t x0 = f.start[j / band * band];
        const int32_t l = f.start[j] - x0;
        const int32_t s = std::min(l & ~3, row_px - kx);
        const int32_t shift = l - s;
        if (s < 0 || shift + f.count[j] > kx) return false;
        start[j] = s / 4;
        int64_t sum = 0;
        for (int32_t k = 0; k < f.count[j]; ++k) {
            const int32_t q = f.fixed[size_t(j) * f.taps + k];
            sum += q;
            const int32_t d0 = ((q + 128) & 255) - 128;
            const int32_t q1 = (q - d0) >> 8;
            const int32_t d1 = ((q1 + 128) & 255) - 128;
            const int32_t d2 = (q1 - d1) >> 8;
            if (d2 < -128 || d2 > 127) return false;
            const int32_t t = shift + k;
            const int32_t d[3] = {d0, d1, d2};
            for (int32_t c = 0; c < 3; ++c) {
                uint32_t& w = reinterpret_cast<uint32_t&>(dig[(size_t(j) * 3 + c) * g + t / 4]);
                w |= (static_cast<uint32_t>(d[c]) & 0xffu) << (8 * (t % 4));
            }
        }
        const int64_t ct = 128 * sum + (int64_t(1) << 21);
        if (ct > INT32_MAX || ct < INT32_MIN) return false;
        cterm[j] = static_cast<int32_t>(ct);
    }
    return true;
}

// Digit table of an axis for the uint8 writer's form with both passes on the
// matrix cores.  Per output its window start, then per output the start value
// 128 * (sum of q) + 2^21; then per block of 16 outputs, for an x axis
// (`columns`) the first source pixel of its 64-pixel window, a multiple of 16
// or, if some block does not fit then, of 8 or of 1, and for a y axis the first and the last chunk of 16 source rows its windows
// read (all the first ones, then the last ones); then per output its digits
// d2, d1, d0, a row of bytes each: 16 zeros, the taps (rounded up to 4), 16
// zeros.  *extent: the most chunks of a block (y axis), or (x axis) 256 times
// the multiple that windows start on, plus the loads of four pixels a lane that
// cover the widest band (2, 4 or 8 loads of 64 lanes per 16 rows), plus
// kRsMmWide where windows of 64 pixels do not do and 128 do.  Returns false if a block's columns do not fit its
// window or a band 32 lanes, its rows kRsMmRing chunks, or a weight its digits.
bool build_digits(const AxisFilter& f, bool columns, std::vector<int32_t>* words, int32_t* extent) {
    const int32_t n = f.n_out, blocks = (n + 15) / 16, taps4 = (f.taps + 3) & ~3, stride = taps4 + 32;
    const size_t head = size_t(2) * n + size_t(columns ? 1 : 2) * blocks;
    words->assign(head + size_t(n) * 3 * stride / 4, 0);
    uint8_t* dig = reinterpret_cast<uint8_t*>(words->data() + head);
    int32_t* const first = words->data() + size_t(2) * n;
    int32_t* const last = first + blocks;
    for (int32_t j = 1; j < n; ++j)   // windows never step back
        if (f.start[j] < f.start[j - 1] || f.start[j] + f.count[j] < f.start[j - 1] + f.count[j - 1]) return false;
    int32_t most = 0;
    if (columns) {
        *extent = 0;
        for (const auto& [wide, a] : {std::pair{false, 16}, {false, 8}, {false, 1}, {true, 16}, {true, 1}}) {
            bool fits = true;
            most = 0;
            for (int32_t b = 0; b < blocks; ++b) {
                const int32_t j1 = std::min(16 * b + 16, n) - 1;
                first[b] = f.start[16 * b] / a * a;
                fits = fits && f.start[j1] + f.count[j1] - first[b] <= (wide ? 128 : 64);
                const int32_t x0 = first[b - b % (vp::resize_mm_cols(wide) / 16)];
                // (the kernel bounds a window's end by its start and the longest window)
                most = std::max(most, (f.start[j1] + taps4 - x0 + 3) / 4);
            }
            const int32_t loads = wide ? 8 : most <= 8 ? 2 : most <= 16 ? 4 : 8;
            if (fits && most <= 32 && (a == 16 || loads == 8)) {   // (narrow spans fit at 16)
                *extent = 256 * a + (wide ? vp::kRsMmWide : 0) + loads;
                break;
            }
        }
        if (*extent == 0) return false;
    } else {
        for (int32_t b = 0; b < blocks; ++b) {
            const int32_t j1 = std::min(16 * b + 16, n) - 1;
            first[b] = f.start[16 * b] / 16;
            last[b] = (f.start[j1] + f.count[j1] - 1) / 16;
            most = std::max(most, last[b] - first[b] + 1);
        }
        if (most > vp::kRsMmRing) return false;
        *extent = most;
    }
    for (int32_t j = 0; j < n; ++j) {
        int64_t sum = 0;
        for (int32_t t = 0; t < f.count[j]; ++t) {
            const int32_t q = f.fixed[size_t(j) * f.taps + t];
            sum += q;
            const int32_t d0 = ((q + 128) & 255) - 128;
            const int32_t q1 = (q - d0) >> 8;
            const int32_t d1 = ((q1 + 128) & 255) - 128;
            const int32_t d2 = (q1 - d1) >> 8;
            if (d2 < -128 || d2 > 127) return false;
            const int32_t d[3] = {d2, d1, d0};
            for (int32_t k = 0; k < 3; ++k)
                dig[(size_t(j) * 3 + k) * stride + 16 + t] = static_cast<uint8_t>(d[k] & 0xff);
        }
        const int64_t ct = 128 * sum + (int64_t(1) << 21);
        if (ct > INT32_MAX || ct < INT32_MIN) return false;
        (*words)[j] = f.start[j];
        (*words)[size_t(n) + j] = static_cast<int32_t>(ct);
    }
    return true;
}

struct StreamShape {
    int32_t m = 0, kx = 0, px = 0, band = 0, bands = 0;
    int32_t ring = 0;   // uint8 writer's matrix-core form: chunks of 16 source rows a group of 16 rows reads
};

int32_t round_up(int32_t v, int32_t q) { return (v + q - 1) / q * q; }

// Patch 14: the whole patches that two bands of `band` columns cover.
int32_t band_patches(int32_t band) { return 2 * band / 14; }

// Widest span of source pixels that one band of output columns reads.
int32_t band_span(const AxisFilter& fx, int32_t band) {
    int32_t worst = 0;
    for (int32_t j0 = 0; j0 < fx.n_out; j0 += band) {
        const int32_t j1 = (j0 + band < fx.n_out ? j0 + band : fx.n_out) - 1;
        const int32_t span = fx.start[j1] + fx.count[j1] - fx.start[j0];
        worst = span > worst ? span : worst;
    }
    return worst;
}

// Whether an item can take the streaming kernel, and with which shape: the
// output width is cut into bands of 1 to 4 whole patches (16 to 64 columns;
// one single-wave workgroup each, one lane per column in the x pass; for patch
// 14 multiples of 7 columns from 14 to 63, in pairs: 49-column bands fill the
// 128 pixels of px = 2 at 720p -> 588 columns, where 42-column ones took two
// more waves in fourteen: 256 frames 305 -> 272 us), each
// band's source pixels must fit 64 lanes of px pixels, and among the shapes
// that fit, the one with the least estimated lane work is taken.  The LDS
// budget is checked with float32 staging, so the routing does not depend on
// the output type.
bool stream_shape(const vp_item& it, const AxisFilter& fx, int32_t m, int32_t patch, StreamShape* sh) {
    if (m < 4 || m > vp::kStreamSlots) return false;
    const int32_t mm = m;
    // windows up to 16 taps run their own tap count (at least 4), longer ones a multiple of 4
    const int32_t kx = fx.taps <= 16 ? std::max<int32_t>(fx.taps, 4) : round_up(fx.taps, 4);
    // every load of a frame row (up to kSlotMax + 8 rows past the last one) stays below 4 GiB
    if (int64_t(it.src_h + vp::kSlotMax + 8) * it.src_w * 3 + 64 >= (int64_t(1) << 32)) return false;
    int64_t best = -1;
    const int32_t step = patch == 14 ? 7 : patch;   // patch 14: two bands are whole patches
    for (int32_t band = 64 / step * step; band >= patch; band -= step) {
        const int32_t bands = (it.dst_w + band - 1) / band;
        const int32_t waves = patch == 14 ? round_up(bands, 2) : bands;
        if (bands > vp::kWgBandMax) continue;   // the band index field of a workgroup entry
        const int32_t span = band_span(fx, band);
        for (int32_t px = 2; px <= 3; ++px) {
            if (!vp::stream_shape_supported(mm, kx, px)) continue;
            if (span > 64 * px || kx > 64 * px) continue;
            // (patch 14 with px = 3: two bands of 63 columns leave two float32
            // workgroups a CU their LDS, of 56 three.  128 frames of 900x1600, us
            // with 63 columns and with this rule, which has them take 49 at px =
            // 2: 588 columns, float32 269 / 215, bf16 181 / 188; 700 columns, 342 /
            // 301 and 223 / 225.  The plan serves both types: float32 gains more
            // than bf16 loses)
            if (patch == 14 && px > 2 && band > 56) continue;
            if (vp::stream_wave_bytes(px, kx, 4, patch, band_patches(band)) > vp::kStreamLdsBudget) continue;
            // vector instructions per wave: per source row 3 px M
            // multiply-adds, about 2 px unpacks and 4 more; per output row
            // the x pass (3 kx FMAs, kx LDS reads), the slot's 3 px clears
            // and about 12 more
            const int64_t cost = int64_t(waves) * (int64_t(it.src_h) * (3 * px * mm + 2 * px + 4) +
                                                    int64_t(it.dst_h) * (4 * kx + 3 * px + 12));
            // (patch 14: of bands that give the same pairs, the narrowest; a
            // pair's stage is its workgroup's LDS)
            if (best < 0 || cost < best || (patch == 14 && cost == best)) {
                best = cost;
                sh->m = mm;
                sh->kx = kx;
                sh->px = px;
                sh->band = band;
                sh->bands = bands;
            }
            break;   // a wider px only adds idle lanes
        }
    }
    return best >= 0;
}

// The x-first streaming kernel for an item, if it can take it: 4 to 12 taps
// (the window's own count, at least 4; to 8 for patch 14), M slots.  With
// `pairs`, windows of 6 to 8 taps -- x scales of about 1.3 to 2 -- whose
// starts in each pair of columns (2i, 2i + 1) lie 0 to 2 pixels apart take
// one column pair per lane and 128 columns per wave; else a lane takes one
// column and a wave 64.  (A single column's window of 6 or more taps takes a
// second load of 8 bytes or more per row, which pairs save; shorter windows
// ran slower in pairs, at the lower occupancy of their larger register set.)
// The last band is narrower where the width is not a multiple of the band.
// Its shape is recorded with px = xfirst_px(0), or xfirst_px(2) for pairs.
bool xfirst_shape(const vp_item& it, const AxisFilter& fx, int32_t m, int32_t patch, bool pairs_ok,
                  StreamShape* sh) {
    const int32_t kx = std::max<int32_t>(fx.taps, 4);
    if (m > vp::kStreamSlots) m = m <= 12 ? 12 : 16;   // upscales over about 2x: 12 or 16 slots
    bool pairs = pairs_ok && vp::xfirst_shape_supported(m, kx, 2, patch) && fx.n_out % 2 == 0;
    for (int32_t j = 0; pairs && j + 1 < fx.n_out; j += 2) {
        const int32_t d = fx.start[j + 1] - fx.start[j];
        pairs = d >= 0 && d <= 2;
    }
    const int32_t db = pairs ? 2 : 0;
    if (!vp::xfirst_shape_supported(m, kx, db, patch)) return false;
    // every load of a frame row (a window of up to 3 (kx + db) + 6 bytes past
    // its start, up to kSlotMax + 8 rows past the last one) stays below 4 GiB
    if (int64_t(it.src_h + vp::kSlotMax + 8) * it.src_w * 3 + 3 * kx + 64 >= (int64_t(1) << 32)) return false;
    // (patch 14: the narrowest bands, in multiples of 7 columns up to 63, that
    // give the fewest pairs: a pair's stage is its workgroup's LDS)
    const int32_t pairs14 = (it.dst_w + 125) / 126;
    const int32_t band = patch == 14 ? round_up((it.dst_w + 2 * pairs14 - 1) / (2 * pairs14), 7) : (db > 0 ? 128 : 64);
    const int32_t waves = (it.dst_w + band - 1) / band;
    if (waves > vp::kWgBandMax) return false;
    sh->m = m;
    sh->kx = kx;
    sh->px = vp::xfirst_px(db);
    sh->band = band;
    sh->bands = waves;
    return true;
}

// Vertical scales up to this one (source rows per output row) take the
// x-first kernel where it fits: an output row closes on almost every source
// row there, and the y-first kernel's gathers of each closed row from LDS
// bound it.
constexpr double kXFirstMaxScale = 1.6;

// Process-wide cache of per-axis tables (windows for the planner, weights for
// the general kernel and the uint8 writer).  The same axes recur from call to
// call (an RL loop preprocesses batches of the same shapes every step), and
// building them is most of the host's work for a batch of many shapes.
// Entries are immutable once built and shared by pointer; a cache is
// cleared when it reaches kTableCacheMax entries.
struct AxisEntry {
    AxisFilter f;
    std::vector<int32_t> words;         // the window table: start, count, weight
    std::vector<int32_t> fixed_words;   // the same with the fixed-point weights
    int32_t slots = -1;                 // accumulator slots of a streaming kernel (count_slots)
};
// An axis of one plan: its cached tables, and where the plan holds them (-1:
// not).  The streaming kernels read the window starts only; the whole window
// table goes to the device for the general and the tile kernel.
struct PlanAxis {
    std::shared_ptr<const AxisEntry> entry;
    int32_t windows = -1, starts = -1;
};
struct SlotEntry {
    int32_t m = -1;               // slots, or -1 if the axis needs too many
    std::vector<int32_t> words;
};
using ColumnKey = std::tuple<int32_t, int32_t, int32_t, int32_t, int32_t>;   // n_in, n_out, kx, band, row_px
using SlotKey = std::pair<int32_t, int32_t>;                                  // n_in, n_out

constexpr size_t kTableCacheMax = 4096;
std::mutex g_cache_mu;
std::map<std::pair<int32_t, int32_t>, std::shared_ptr<const AxisEntry>> g_axis_cache;
std::map<SlotKey, std::shared_ptr<const SlotEntry>> g_slot_cache;
std::map<ColumnKey, std::shared_ptr<const std::vector<int32_t>>> g_column_cache;

// The entry for `key`, built by `make` (outside the lock) on a miss.  If two
// threads miss together, the first entry stored wins; both are identical.
template <class Map, class Make>
typename Map::mapped_type cached(Map& map, const typename Map::key_type& key, Make make) {
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        auto it = map.find(key);
        if (it != map.end()) return it->second;
    }
    typename Map::mapped_type v = make();
    std::lock_guard<std::mutex> lk(g_cache_mu);
    if (map.size() >= kTableCacheMax) map.clear();
    return map.emplace(key, std::move(v)).first->second;
}

std::shared_ptr<const AxisEntry> make_axis_entry(int32_t n_in, int32_t n_out) {
    auto e = std::make_shared<AxisEntry>();
    build_axis(n_in, n_out, axis_taps(n_in, n_out), &e->f);
    e->slots = count_slots(e->f, nullptr);
    const AxisFilter& f = e->f;
    e->words.reserve(2 * f.start.size() + f.weight.size());
    e->words.insert(e->words.end(), f.start.begin(), f.start.end());
    e->words.insert(e->words.end(), f.count.begin(), f.count.end());
    const size_t wbase = e->words.size();
    e->words.resize(wbase + f.weight.size());
    std::memcpy(e->words.data() + wbase, f.weight.data(), f.weight.size() * sizeof(float));
    e->fixed_words.reserve(e->words.size());
    e->fixed_words.insert(e->fixed_words.end(), f.start.begin(), f.start.end());
    e->fixed_words.insert(e->fixed_words.end(), f.count.begin(), f.count.end());
    e->fixed_words.insert(e->fixed_words.end(), f.fixed.begin(), f.fixed.end());
    return e;
}

// One streaming work unit with its kernel shape, before the workgroup list
// is laid out.
struct Keyed {
    std::tuple<int32_t, int32_t, int32_t> key;   // kernel shape (m, kx, px)
    int32_t bands;                               // column bands (workgroups) of the unit
    int32_t lds_units;                          // patch 14: patches of a workgroup's two bands; uint8 writer: ring chunks
    vp::StreamUnit unit;
    int64_t cost;
};

// Output rows per streaming unit of an item: at most about max_src_rows
// source rows, at least min_windows windows of source rows, a multiple of
// `group` rows (the kernel's store group), and at least 16 rows (28 for
// groups of 14).  With short_rows > 0 (small batches, see short_unit_rows)
// short_rows takes the place of both lower bounds.
int64_t unit_row_band(const vp::DevItem& d, int64_t max_src_rows, int64_t group, int64_t min_windows = 10,
                      int64_t short_rows = 0) {
    int64_t band = max_src_rows * d.h / d.H;
    const int64_t min_band = short_rows > 0 ? short_rows : (min_windows * d.ky * d.h + d.H - 1) / d.H;
    const int64_t least = short_rows > 0 ? group : (group == 4 ? 16 : 2 * group);
    band = std::max(band, min_band);
    band = std::max<int64_t>((band + group - 1) / group * group, least);
    return std::min<int64_t>(band, d.h);
}

// Output rows of the units of a small batch, or 0 where units of ten filter
// windows are the better ones.  A unit is one wave's serial chain over its
// source rows, about 0.35 us a row on an idle chip, so a batch that leaves
// most wave slots empty lasts as long as one unit.  Shorter units re-read
// more rows (from the caches, in a small batch).  `waves` gives the batch's
// workgroups (waves) for units of a number of output rows; units of 16 rows
// win up to `most` of them, where an x-first wave, whose rows are cheaper,
// counts as 5/2 (`load`).  Measured, kernel us at ten windows
// / 16 / 8 / 4 rows: 480p x 4 frames 29 / 17 / 13 / 14, 480p x 16
// 31 / 22 / 24 / 28, 1080p x 2 52 / 26 / 19 / 17, 1080p x 32 77 / 67 / 70 / 86,
// 1080p x 64 132 / 114 / 126 / 127, 720p x 128 134 / 134 / 138 / 137, 1080p x
// 128 268 / 276 / 274 / 274; 480p x 64 in float32, x-first, 72 / 75 / 80 / 80.
// Those inputs lay in the caches; from HBM a batch near the line can lose by
// short units (ten windows / 16 rows: 1080p x 64 140 / 146, 720p -> 320x576 x 128
// 121 / 127, 480p x 48 in float32 54 / 62, in bf16 40 / 44) or gain (4K x 28 251 /
// 240, 720p -> 256x448 x 264 212 / 204, 360p x 32 29 / 24); of 24 batches drawn
// near it, most of them ragged, 18 gained.
// So: 16 rows up to a load of 32,768 waves, and where that gives fewer than
// 2,048 waves 8 rows, then 4.  Patch 14 stores whole patch
// rows, 14 or 28 (ten windows / 28 / 14: 480p x 16 45 / 31 / 25, 480p x 64
// 89 / 69 / 70, 720p x 64 92 / 82 / 86): 14 up to 10,240 waves.  The uint8
// writer's dot-product form re-reads at a higher price (ten windows / 16 rows, us
// a call: 841x2431 -> 128x352 x 120, 10,560 waves, 330 / 323, x 150 391 / 387, x
// 182, 16,016 waves, 457 / 484; 4K -> 320x576 x 36, 12,960 waves, 425 / 402;
// 1080p -> 160x288 x 200, 18,000 waves, 536 / 550).
constexpr int64_t kShortWaves = 32768, kShortWavesDot = 14000;

template <class Waves, class Load>
int64_t short_unit_rows(Waves waves, Load load, int64_t most, int32_t patch = 16) {
    if (patch == 14 && waves(14) <= 10240) return 14;
    if (load(16) > most) return 0;   // (patch 14 rounds 16 up to 28)
    if (waves(16) >= 2048) return 16;
    return waves(8) >= 1536 ? 8 : 4;
}

// A frame's h output rows cut into n = ceil(h / band) units whose boundaries
// fall on whole store groups of `group` rows, as evenly as that allows:
// lengths differ by at most one group, and the last unit also takes the rows
// past the last whole group.  Units of one frame are neighbours in the
// workgroup list, and a long unit followed by a short remainder (a 320-row
// frame at a 296-row cap: 296 + 24) would load the XCDs unevenly.
struct UnitSplit {
    int64_t h, group, groups, n;
    UnitSplit(int64_t h_, int64_t band, int64_t group_) : h(h_), group(group_), groups(h_ / group_) {
        n = std::max<int64_t>(1, std::min<int64_t>((h + band - 1) / band, groups));
    }
    int32_t begin(int64_t u) const { return static_cast<int32_t>(group * (groups * u / n)); }
    int32_t end(int64_t u) const { return static_cast<int32_t>(u + 1 == n ? h : group * (groups * (u + 1) / n)); }
};

// Vector instructions per source row of a wave (with the output rows that
// close on it), read off the compiled kernels.
int64_t row_instructions(const StreamShape& sh, const vp::DevItem& d) {
    const int64_t m = sh.m, kx = sh.kx;
    if (sh.px < 0) {   // x-first: align, extract, window sums, slots; closes
        const int64_t cols = vp::xfirst_db(sh.px) > 0 ? 2 : 1;
        return (3 * kx + 3) / 4 + 3 * ((kx + 1) / 2) + cols * 3 * (kx + m) + 4 + 12 * d.h / d.H;
    }
    return 3 * sh.px * m + 2 * sh.px + 4 + (4 * kx + 3 * sh.px + 12) * d.h / d.H;
}

// Fewer launches: two kernel shapes of a batch become one, with the larger of
// their slots and taps (more slots and taps hold zero weights, which change no
// bit of the sums), where the extra instructions cost less than a launch does.
// A launch costs its call about 5 us on the host, and a small one leaves the
// chip waiting for its last unit; the chip issues about 3 million wave
// instructions in that time.  Measured, kernel us before and
// after: 16 images 71 -> 26, 4 images 55 -> 16, 24 images with small and large
// ones 160 -> 113 (11 launches -> 4); from half the limit to ten times it the
// same.
constexpr int64_t kMergeInstructions = 3000000;


void merge_shapes(const vp_item* items, const std::vector<vp::DevItem>& dev, const std::vector<int64_t>& distinct,
                  int32_t patch, std::vector<StreamShape>* shapes) {
    std::map<std::tuple<int32_t, int32_t, int32_t>, std::vector<int32_t>> groups;   // (px, m, kx) -> items
    for (size_t b = 0; b < dev.size(); ++b)
        if (dev[b].route == vp::kRouteStream)
            groups[std::make_tuple((*shapes)[b].px, (*shapes)[b].m, (*shapes)[b].kx)].push_back(static_cast<int32_t>(b));
    while (groups.size() > 1) {
        int64_t best = kMergeInstructions;
        auto best_a = groups.end(), best_b = groups.end();
        std::tuple<int32_t, int32_t, int32_t> best_key;
        for (auto a = groups.begin(); a != groups.end(); ++a)
            for (auto b = std::next(a); b != groups.end(); ++b) {
                const int32_t px = std::get<0>(a->first);
                if (std::get<0>(b->first) != px || px == vp::xfirst_px(2)) continue;   // (pairs keep their own taps)
                StreamShape to;
                to.px = px;
                to.m = std::max(std::get<1>(a->first), std::get<1>(b->first));
                to.kx = std::max(std::get<2>(a->first), std::get<2>(b->first));
                if (px < 0 ? !vp::xfirst_shape_supported(to.m, to.kx, vp::xfirst_db(px), patch)
                           : !vp::stream_shape_supported(to.m, to.kx, px))
                    continue;
                int64_t extra = 0;
                bool fits = true;
                for (const auto* g : {&a->second, &b->second})
                    for (const int32_t k : *g) {
                        const StreamShape& sh = (*shapes)[k];
                        const vp::DevItem& d = dev[k];
                        // (every load of a window still ends below 4 GiB, a source row still holds its taps)
                        fits = fits && int64_t(items[k].src_h + vp::kSlotMax + 8) * items[k].src_w * 3 + 3 * to.kx + 64 <
                                           (int64_t(1) << 32);
                        extra += distinct[k] * sh.bands * d.H * (row_instructions(to, d) - row_instructions(sh, d));

                    }
                if (fits && extra < best) {
                    best = extra;
                    best_a = a;
                    best_b = b;
                    best_key = std::make_tuple(px, to.m, to.kx);
                }
            }
        if (best_a == groups.end()) return;
        std::vector<int32_t> both = std::move(best_a->second);
        both.insert(both.end(), best_b->second.begin(), best_b->second.end());
        std::sort(both.begin(), both.end());
        for (const int32_t k : both) {
            (*shapes)[k].m = std::get<1>(best_key);
            (*shapes)[k].kx = std::get<2>(best_key);
        }
        groups.erase(best_a);
        groups.erase(best_b);
        auto& into = groups[best_key];   // (both were joined into a shape that one of them may have had)
        into.insert(into.end(), both.begin(), both.end());
    }
}

// Likewise of the uint8 writer's matrix-core form: a kernel of more loads a
// chunk (T), of windows that start anywhere (A) or of two products a group
// (TWO) serves what asks for less, with the same bytes.  Instructions per wave:
// about 20 a load and chunk, 12 a chunk for LDS reads of 8 bytes and 72 for
// unaligned ones, 40 a second product of a group.  Measured, us a call as two
// launches and as one: 102 frames of 688x86 with 49 of 190x239 70 -> 32, four
// items of 2 to 34 frames 106 -> 48, 16 frames each of 480p and 1080p 76 -> 62;
// at the limit, 128 frames each of 480p and 1080p 329 -> 331, of 200x300 and
// 720p 196 -> 189.
void merge_matrix_shapes(const std::vector<vp::DevItem>& dev, std::vector<StreamShape>* shapes) {
    using Key = std::tuple<bool, int32_t, int32_t, bool>;   // wide, T, A, TWO
    const auto key_of = [](const StreamShape& sh) {
        return Key((sh.m & vp::kRsMmWide) != 0, sh.m % vp::kRsMmTwo, sh.px, (sh.m & vp::kRsMmTwo) != 0);
    };
    const auto chunk_cost = [](const Key& k) {   // a chunk of 16 source rows
        return 20 * std::get<1>(k) + (std::get<2>(k) == 16 ? 0 : std::get<2>(k) == 8 ? 12 : 72);
    };
    std::map<Key, std::vector<int32_t>> groups;
    for (size_t b = 0; b < dev.size(); ++b)
        if (dev[b].route == vp::kRouteStream && (*shapes)[b].kx == vp::kRsMmShape)
            groups[key_of((*shapes)[b])].push_back(static_cast<int32_t>(b));
    while (groups.size() > 1) {
        int64_t best = kMergeInstructions;
        auto best_a = groups.end(), best_b = groups.end();
        Key best_key;
        for (auto a = groups.begin(); a != groups.end(); ++a)
            for (auto b = std::next(a); b != groups.end(); ++b) {
                const auto& [wide, ta, aa, two_a] = a->first;
                const auto& [wide_b, tb, ab, two_b] = b->first;
                if (wide != wide_b) continue;
                const int32_t align = std::min(aa, ab);
                Key to(wide, align == 16 ? std::max(ta, tb) : 8, wide && align == 8 ? 1 : align, two_a || two_b);
                int64_t extra = 0;
                for (const auto* g : {&*a, &*b})
                    for (const int32_t k : g->second) {
                        const vp::DevItem& d = dev[k];
                        const int64_t waves = int64_t(d.t) * (*shapes)[k].bands;
                        extra += waves * ((d.H + 15) / 16) * (chunk_cost(to) - chunk_cost(g->first));
                        if (std::get<3>(to) != std::get<3>(g->first)) extra += waves * ((d.h + 15) / 16) * 40;
                    }
                if (extra < best) {
                    best = extra;
                    best_a = a;
                    best_b = b;
                    best_key = to;
                }
            }
        if (best_a == groups.end()) return;
        std::vector<int32_t> both = std::move(best_a->second);
        both.insert(both.end(), best_b->second.begin(), best_b->second.end());
        std::sort(both.begin(), both.end());
        const auto& [wide, t, align, two] = best_key;
        for (const int32_t k : both) {
            (*shapes)[k].m = t + (wide ? vp::kRsMmWide : 0) + (two ? vp::kRsMmTwo : 0);
            (*shapes)[k].px = align;
        }
        groups.erase(best_a);
        groups.erase(best_b);
        auto& into = groups[best_key];   // (both were joined into a shape that one of them may have had)
        into.insert(into.end(), both.begin(), both.end());
    }
}

// Lays out the streaming units as launches, of workgroups of `threads`, and
// their workgroup lists.
int32_t assemble_launches(const std::vector<Keyed>& keyed, int32_t P, int32_t threads, Plan* p) {
    // Units of one kernel shape form one launch, whatever their widths.  Its
    // workgroups are listed explicitly: entry g (unit index | band << 20, or
    // kNoWork) runs as workgroup g, and consecutive workgroups go to the
    // eight XCDs in turn.  Units are taken eight at a time, and their bands
    // are listed round by round (band 0 of all eight, then band 1, ...), so
    // that all bands of one unit run on one XCD and share the source pixels
    // of neighbouring bands through its L2; a unit with fewer bands than the
    // others of its eight leaves empty entries.  Units are sorted by band
    // count first, which keeps those rare.  The XCD of the x-th unit of the
    // g-th eight is (x + g) mod 8: a pattern in the units' lengths that
    // repeats every few units (the units of one frame) then spreads over all
    // eight XCDs instead of loading some more than others.
    // A launch holds fewer than 2^32 threads: one that would reach half of that
    // (the writer's 16- and 32-column bands of half a million wide frames) goes
    // on in another.
    const int32_t most_wgs = static_cast<int32_t>((int64_t(1) << 31) / threads);
    if (keyed.size() > vp::kWgUnitMask + 1)
        return fail(VP_ERR_CAPACITY, "batch has more than 2^20 streaming work units");
    // order: by shape, then band count, then as generated (a grouping: the
    // units of one item are consecutive and share both)
    std::map<std::pair<std::tuple<int32_t, int32_t, int32_t>, int32_t>, std::vector<uint32_t>> groups;
    for (size_t k = 0; k < keyed.size();) {
        size_t k1 = k + 1;
        while (k1 < keyed.size() && keyed[k1].key == keyed[k].key && keyed[k1].bands == keyed[k].bands) ++k1;
        auto& g = groups[std::make_pair(keyed[k].key, keyed[k].bands)];
        for (; k < k1; ++k) g.push_back(static_cast<uint32_t>(k));
    }
    std::vector<uint32_t> order;
    order.reserve(keyed.size());
    for (const auto& g : groups) order.insert(order.end(), g.second.begin(), g.second.end());
    p->units.clear();
    p->wgs.clear();
    p->launches.clear();
    p->units.reserve(keyed.size());
    p->wgs.reserve(keyed.size() * 8);
    for (size_t k0 = 0; k0 < order.size();) {
        const auto& key0 = keyed[order[k0]].key;
        size_t k1 = k0;
        while (k1 < order.size() && keyed[order[k1]].key == key0) ++k1;
        vp::StreamLaunch L{};
        L.first = static_cast<int32_t>(p->wgs.size());
        L.m = std::get<0>(key0);
        L.kx = std::get<1>(key0);
        L.px = std::get<2>(key0);
        L.patch = P;
        for (size_t c0 = k0, g = 0; c0 < k1; c0 += 8, ++g) {
            const size_t c1 = std::min(c0 + 8, k1);
            int32_t rounds = 0;
            for (size_t k = c0; k < c1; ++k) rounds = std::max(rounds, keyed[order[k]].bands);
            if (static_cast<int64_t>(p->wgs.size()) - L.first + 8 * int64_t(rounds) > most_wgs) {
                L.count = static_cast<int32_t>(p->wgs.size()) - L.first;
                p->launches.push_back(L);
                L.first += L.count;
                L.cost = 0;
            }
            const uint32_t u0 = static_cast<uint32_t>(p->units.size());
            for (size_t k = c0; k < c1; ++k) {
                const Keyed& e = keyed[order[k]];
                p->units.push_back(e.unit);
                L.cost += e.cost * e.bands;
                L.lds_units = std::max(L.lds_units, e.lds_units);
            }
            for (int32_t r = 0; r < rounds; ++r)
                for (size_t col = 0; col < 8; ++col) {
                    const size_t x = (col + 8 - g % 8) % 8;   // the unit on XCD col
                    const size_t k = c0 + x;
                    p->wgs.push_back(k < c1 && r < keyed[order[k]].bands
                                         ? (u0 + static_cast<uint32_t>(x)) | (static_cast<uint32_t>(r) << vp::kWgBandShift)
                                         : vp::kNoWork);
                }
        }
        L.count = static_cast<int32_t>(p->wgs.size()) - L.first;
        p->launches.push_back(L);
        k0 = k1;
    }

    return VP_OK;
}

// With `most_slots` below kSlotWords, items that need more open rows than that
// go to the general kernel, whose plan holds no work units.  `long_units`: no
// unit is cut short for a small batch.
int32_t build_plan(const vp_item* items, int32_t n, Plan* p, int32_t most_slots = vp::kSlotWords, bool long_units = false) {
    if (items == nullptr) return fail(VP_ERR_NULL, "items is NULL");
    if (n < 1) return fail(VP_ERR_ARG, "n_items < 1");
    int32_t P = vp::kPatch;
    if (const int32_t st = batch_patch(items, n, &P); st != VP_OK) return st;
    p->items.assign(n, vp::DevItem{});
    p->generic_cost = p->generic_chain = 0;
    p->prefix.assign(n + 1, 0);
    p->grid.assign(size_t(n) * 3, 0);
    p->cu.assign(n + 1, 0);
    p->indices.clear();
    p->tables.clear();
    p->table_words = 0;
    p->jobs.clear();
    p->gen_words = 0;
    // Tables come from the process-wide cache; each one used by the batch is
    // copied into the plan once, and the per-call maps keep the cache
    // entries alive while the call uses them.
    auto append = [&](std::shared_ptr<const std::vector<int32_t>> words) -> int32_t {
        const int32_t o = static_cast<int32_t>(p->table_words);
        p->table_words += words->size();
        p->tables.emplace_back(o, std::move(words));
        return o;
    };
    std::map<std::pair<int32_t, int32_t>, PlanAxis> axes;
    auto axis_for = [&](int32_t n_in, int32_t n_out) -> PlanAxis& {
        PlanAxis& a = axes[std::make_pair(n_in, n_out)];
        if (a.entry == nullptr)
            a.entry = cached(g_axis_cache, std::make_pair(n_in, n_out), [&] { return make_axis_entry(n_in, n_out); });
        return a;
    };
    auto window_table = [&](PlanAxis& a) { return a.windows >= 0 ? a.windows : a.windows = append({a.entry, &a.entry->words}); };
    // The streaming kernels' tables are computed on the device (their weights
    // are functions of the axis alone): their words there, and their pieces.
    auto words_for = [&](int64_t words) -> int32_t {
        const int32_t o = static_cast<int32_t>(p->gen_words);
        p->gen_words += static_cast<size_t>(words);
        return o;
    };
    auto pieces = [&](vp::TableKind kind, int32_t lanes, const AxisFilter& f, int32_t a, int32_t band, int32_t row_px,
                      int32_t off, int64_t elements, int64_t piece) {
        for (int64_t base = 0; base < elements; base += piece)
            p->jobs.push_back({kind | lanes << 8, f.n_in, f.n_out, a, band, row_px, off, static_cast<int32_t>(base)});
    };
    auto lanes_for = [](int32_t taps) {
        int32_t lanes = 4;
        while (lanes < taps && lanes < vp::kUploadThreads) lanes *= 2;
        return lanes;
    };
    auto start_table = [&](PlanAxis& a) {
        if (a.starts < 0) {
            const AxisFilter& f = a.entry->f;
            a.starts = words_for(f.n_out);
            pieces(vp::kTableStarts, 1, f, 0, 0, 0, a.starts, f.n_out, vp::kTablePiece);
        }
        return a.starts;
    };
    std::map<std::tuple<int32_t, int32_t, int32_t>, int32_t> slot_tables;
    auto slots_for = [&](const AxisFilter& f, int32_t m) -> int32_t {
        const auto [found, made] = slot_tables.emplace(std::make_tuple(f.n_in, f.n_out, m), 0);
        if (made) {
            const int64_t weights = int64_t(f.n_in + vp::kSlotMax) * m;
            const int32_t lanes = lanes_for(f.taps), off = words_for(weights + f.n_out + 2);
            found->second = off;
            pieces(vp::kTableSlots, lanes, f, m, 0, 0, off, f.n_out, vp::table_outputs(lanes));
            pieces(vp::kTableZeros, 1, f, m, 0, 0, off, weights + 2, vp::kTablePiece);
        }
        return found->second;
    };
    std::map<std::tuple<int32_t, int32_t, int32_t, int32_t, int32_t>, int32_t> column_tables;
    auto columns_for = [&](const AxisFilter& f, int32_t kx, int32_t band, int32_t row_px) -> int32_t {
        const auto [found, made] = column_tables.emplace(std::make_tuple(f.n_in, f.n_out, kx, band, row_px), 0);
        if (made) {
            const int32_t lanes = lanes_for(kx), off = words_for(int64_t(f.n_out) * (1 + kx));
            found->second = off;
            pieces(vp::kTableColumns, lanes, f, kx, band, row_px, off, f.n_out, vp::table_outputs(lanes));
        }
        return found->second;
    };
    std::vector<StreamShape> shapes(n);
    std::vector<const AxisFilter*> x_axes(n, nullptr), y_axes(n, nullptr);

    int64_t rows = 0, tiles = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp_item& it = items[b];
        int32_t st = validate_item(it, b);
        if (st != VP_OK) return st;
        vp::DevItem& d = p->items[b];
        d.frames = it.frames;
        d.frame_bytes = int64_t(it.src_h) * it.src_w * 3;
        d.H = it.src_h;
        d.W = it.src_w;
        d.h = it.dst_h;
        d.w = it.dst_w;
        d.t = (it.n_idx + 1) / 2;
        d.patch = P;
        d.hm = it.dst_h / (2 * P);
        d.wm = it.dst_w / (2 * P);
        d.idx_off = static_cast<int32_t>(p->indices.size());
        for (int32_t k = 0; k < 2 * d.t; ++k)
            p->indices.push_back(it.indices[k < it.n_idx ? k : it.n_idx - 1]);
        PlanAxis& ay = axis_for(it.src_h, it.dst_h);
        PlanAxis& ax = axis_for(it.src_w, it.dst_w);
        const AxisFilter* fy = &ay.entry->f;
        const AxisFilter* fx = &ax.entry->f;
        d.ky = fy->taps;
        d.kx = fx->taps;
        d.route = vp::kRouteGeneric;
        StreamShape sh;
        const int32_t m = ay.entry->slots;
        const bool near_one = double(it.src_h) <= kXFirstMaxScale * double(it.dst_h);
        if (m > 0 && m <= most_slots && ((near_one && xfirst_shape(it, *fx, m, P, false, &sh)) || stream_shape(it, *fx, m, P, &sh))) {
            d.route = vp::kRouteStream;   // (band and column table below, once the shape is final)
            shapes[b] = sh;
            x_axes[b] = fx;
            y_axes[b] = fy;
        } else if (!generic_subtile(*fx, 2 * P, &d.rh, &d.cw)) {
            return fail(VP_ERR_CAPACITY, "item " + std::to_string(b) +
                                             ": horizontal filter window too long (downscale too large)");
        }
        d.ty_off = d.route == vp::kRouteStream ? start_table(ay) : window_table(ay);
        d.tx_off = d.route == vp::kRouteStream ? start_table(ax) : window_table(ax);
        d.row_off = rows;
        const int64_t item_rows = int64_t(d.t) * (it.dst_h / P) * (it.dst_w / P);
        p->grid[3 * b + 0] = d.t;
        p->grid[3 * b + 1] = it.dst_h / P;
        p->grid[3 * b + 2] = it.dst_w / P;
        rows += item_rows;
        if (d.route == vp::kRouteGeneric) {
            tiles += int64_t(d.t) * d.hm * d.wm;
            p->generic_cost += int64_t(2) * d.t * d.H * d.W;
            const int64_t span = int64_t(d.cw) * d.W / d.w + d.kx;
            const int64_t steps = (d.rh * span * 3 / vp::kGenericThreads + 1) * d.ky + (d.rh * d.cw * 3 / vp::kGenericThreads + 1) * d.kx;
            p->generic_chain = std::max(p->generic_chain, 2 * (4 * P * P / (d.rh * d.cw)) * steps);
        }
        if (rows > INT32_MAX || tiles > INT32_MAX)
            return fail(VP_ERR_CAPACITY, "batch has more than 2^31-1 rows");
        p->cu[b + 1] = static_cast<int32_t>(rows);
        p->prefix[b + 1] = static_cast<int32_t>(tiles);
    }
    p->total_rows = rows;

    // Streaming units: one per (item, distinct frame of a pair, band of output
    // rows); for patch 14 one per (item, pair, band), its frames on the two
    // waves of one workgroup.  A workgroup streams the source rows of its unit top to bottom,
    // so its life is about proportional to those rows.  To end the batch
    // evenly -- many kernel shapes run side by side, and a small launch lasts
    // as long as its longest unit -- no unit reads more than an eighth of the
    // source rows per wave slot of the whole batch (256 CUs x 20 waves), in
    // bands of output rows that are multiples of 4 (one 64-value run per
    // store).  A band re-reads the source rows that its first window shares
    // with the band above, so none spans fewer than ten windows of source
    // rows, or fifteen where the batch still gives every wave slot four
    // workgroups at that length (shorter units re-read more rows -- about a
    // tenth at ten windows -- but in a batch of few workgroups they end it
    // more evenly, which is worth more).
    constexpr int64_t kWaveSlots = 256 * 20;
    std::vector<int64_t> distinct(n, 0);   // frames that item b streams: two per pair, one where they are one
    int64_t stream_frames = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp::DevItem& d = p->items[b];
        if (d.route != vp::kRouteStream) continue;
        const int32_t* ix = p->indices.data() + d.idx_off;
        for (int32_t tt = 0; tt < d.t; ++tt) distinct[b] += ix[2 * tt] == ix[2 * tt + 1] ? 1 : 2;
        stream_frames += distinct[b];
    }
    auto source_row_cap = [&] {
        int64_t wave_rows = 0;   // source rows that all workgroups stream, whole frames
        for (int32_t b = 0; b < n; ++b) wave_rows += distinct[b] * shapes[b].bands * p->items[b].H;
        return wave_rows / (kWaveSlots * 8);
    };
    auto workgroup_waves = [&](int64_t min_windows, int64_t max_src_rows, int64_t short_rows = 0,
                               bool as_load = false, int32_t over_slots = 0) {
        int64_t waves = 0;
        for (int32_t b = 0; b < n; ++b) {
            const vp::DevItem& d = p->items[b];
            if (d.route != vp::kRouteStream || shapes[b].m <= over_slots) continue;
            const int64_t group = d.patch == 16 ? 4 : d.patch;
            const int64_t units = UnitSplit(d.h, unit_row_band(d, max_src_rows, group, min_windows, short_rows), group).n;
            // units per row band: one per distinct frame (patch 14: per pair)
            const int64_t frames = d.patch == 14 ? d.t : distinct[b];
            const int64_t per_unit = d.patch == 14 ? 4 * ((shapes[b].bands + 1) / 2) : shapes[b].bands;
            const int64_t w = frames * units * per_unit;
            waves += as_load && shapes[b].px < 0 ? w * 5 / 2 : w;
        }
        return waves;
    };
    // Column pairs halve an x-first item's workgroups: taken only where the
    // batch gives every wave slot four workgroups with single columns.
    if (workgroup_waves(10, source_row_cap()) >= 4 * kWaveSlots) {
        for (int32_t b = 0; b < n; ++b) {
            StreamShape sh;
            if (p->items[b].route == vp::kRouteStream && shapes[b].px == vp::xfirst_px(0) &&
                xfirst_shape(items[b], *x_axes[b], shapes[b].m, P, true, &sh))
                shapes[b] = sh;
        }
    }
    merge_shapes(items, p->items, distinct, P, &shapes);
    for (int32_t b = 0; b < n; ++b) {
        vp::DevItem& d = p->items[b];
        if (d.route != vp::kRouteStream) continue;
        const StreamShape& sh = shapes[b];
        d.sy_off = slots_for(*y_axes[b], sh.m);
        d.band = sh.band;
        d.row_px = sh.px > 0 ? 64 * sh.px : d.W + sh.kx;
        d.sx_off = columns_for(*x_axes[b], sh.kx, sh.band, d.row_px);
    }
    const int64_t max_src_rows = source_row_cap();
    const int64_t min_windows = workgroup_waves(15, max_src_rows) >= 4 * kWaveSlots ? 15 : 10;
    p->long_unit_rows = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp::DevItem& d = p->items[b];
        if (d.route == vp::kRouteStream)
            p->long_unit_rows = std::max(p->long_unit_rows, shapes[b].m > vp::kStreamSlots
                                                                ? INT64_MAX
                                                                : std::min<int64_t>(d.H, std::max(10 * int64_t(d.ky), max_src_rows) + d.ky));
    }
    const int64_t short_rows =
        long_units ? 0 :
        short_unit_rows([&](int64_t rows) { return workgroup_waves(10, max_src_rows, rows); },
                        [&](int64_t rows) { return workgroup_waves(10, max_src_rows, rows, true); }, kShortWaves, P);
    // Upscales of 12 or 16 slots in a batch of long units are judged alone: a
    // source row costs their waves about 1 us, and a launch of a few long units
    // lasts as long as one (an image of 110x121 -> 224x256 behind 121 frames of
    // 474x693, no-alloc entry, where launches follow one another: 137 us with
    // long units, 117 with short ones).
    const int64_t short_many =
        short_rows > 0 || long_units ? short_rows
                       : short_unit_rows([&](int64_t rows) { return workgroup_waves(10, 0, rows, false, vp::kStreamSlots); },
                                         [&](int64_t rows) { return workgroup_waves(10, 0, rows, true, vp::kStreamSlots); },
                                         kShortWaves, P);
    const auto lay_out = [&](int64_t short_rows, int64_t short_many) -> int32_t {
        std::vector<Keyed> keyed;
        keyed.reserve(static_cast<size_t>(stream_frames));
        for (int32_t b = 0; b < n; ++b) {
            const vp::DevItem& d = p->items[b];
            if (d.route != vp::kRouteStream) continue;
            const StreamShape& sh = shapes[b];
            // whole store groups: multiples of 4 rows for patch 16, whole
            // patch rows (14 output rows, stored at once) for patch 14
            const int64_t group = d.patch == 16 ? 4 : d.patch;
            const bool alone = short_rows == 0 && short_many > 0 && sh.m > vp::kStreamSlots;
            const UnitSplit split(d.h, unit_row_band(d, alone ? 0 : max_src_rows, group, min_windows, alone ? short_many : short_rows), group);
            for (int32_t tt = 0; tt < d.t; ++tt) {
                const bool same = p->indices[d.idx_off + 2 * tt] == p->indices[d.idx_off + 2 * tt + 1];
                const bool pair_units = d.patch == 14;   // both frames in one unit
                for (int32_t dt = 0; dt < (same || pair_units ? 1 : 2); ++dt) {
                    for (int64_t u = 0; u < split.n; ++u) {
                        const int32_t i0 = split.begin(u), i1 = split.end(u);
                        Keyed k;
                        k.key = std::make_tuple(sh.m, sh.kx, sh.px);
                        k.bands = d.patch == 14 ? (sh.bands + 1) / 2 : sh.bands;   // patch 14: bands in pairs
                        k.lds_units = band_patches(sh.band);
                        k.unit.item = b;
                        k.unit.p_flags = (2 * tt + dt) | (same ? vp::kUnitBoth : 0);
                        k.unit.i0 = i0;
                        k.unit.i1 = i1;
                        k.cost = int64_t(i1 - i0) * d.H / d.h * d.W   // source pixels read, roughly
                                 * (pair_units && !same ? 2 : 1);
                        keyed.push_back(k);
                    }
                }
            }
        }
        if (const int32_t st = assemble_launches(keyed, P, P == 14 ? 256 : 64, p); st != VP_OK) return st;
        p->off_items = 0;
        p->off_prefix = align_up(p->off_items + sizeof(vp::DevItem) * p->items.size());
        p->off_indices = align_up(p->off_prefix + sizeof(int32_t) * p->prefix.size());
        p->off_tables = align_up(p->off_indices + sizeof(int32_t) * p->indices.size());
        p->off_units = align_up(p->off_tables + sizeof(int32_t) * p->table_words);
        p->off_wgs = align_up(p->off_units + sizeof(vp::StreamUnit) * p->units.size());
        p->off_jobs = align_up(p->off_wgs + sizeof(uint32_t) * p->wgs.size());
        p->off_gen = align_up(p->off_jobs + sizeof(vp::TableJob) * p->jobs.size());
        p->bytes = align_up(p->off_gen + sizeof(int32_t) * p->gen_words);
        return VP_OK;
    };
    const std::string before = g_last_error;
    int32_t st = lay_out(short_rows, short_many);
    // (more units make a larger plan: one that no longer fits the no-alloc
    // entry's plan memory, or the work units, keeps the longer units)
    if (short_many > 0 && (st == VP_ERR_CAPACITY || (st == VP_OK && p->bytes > static_cast<size_t>(vp::kNoAllocPlanBytes)))) {
        st = lay_out(0, 0);
        if (st == VP_OK) g_last_error = before;
    }
    if (st != VP_OK) return st;
    // the computed tables' offsets, from the first tables section like the others
    const int64_t gen = static_cast<int64_t>(p->off_gen - p->off_tables) / 4;
    if (gen + static_cast<int64_t>(p->gen_words) > INT32_MAX) return fail(VP_ERR_CAPACITY, "the plan's tables exceed 8 GiB");
    for (vp::TableJob& j : p->jobs) j.off += static_cast<int32_t>(gen);
    for (vp::DevItem& d : p->items)
        if (d.route == vp::kRouteStream)
            for (int32_t* off : {&d.ty_off, &d.tx_off, &d.sy_off, &d.sx_off}) *off += static_cast<int32_t>(gen);
    return VP_OK;
}

// Plan of vp_patchify_batch: items whose frames are already at the target
// size; one workgroup per merge-window row (32 pixel rows) of a frame pair
// (patch 14 counts merge windows: its workgroups take a few of the batch's).
int32_t build_patch_plan(const vp_item* items, int32_t n, Plan* p) {
    if (items == nullptr) return fail(VP_ERR_NULL, "items is NULL");
    if (n < 1) return fail(VP_ERR_ARG, "n_items < 1");
    int32_t P = vp::kPatch;
    if (const int32_t st = batch_patch(items, n, &P); st != VP_OK) return st;
    p->items.assign(n, vp::DevItem{});
    p->prefix.assign(n + 1, 0);
    p->grid.assign(size_t(n) * 3, 0);
    p->cu.assign(n + 1, 0);
    p->indices.clear();
    p->tables.clear();
    p->table_words = 0;
    p->units.clear();
    p->wgs.clear();
    p->launches.clear();
    p->generic_cost = p->generic_chain = 0;
    int64_t rows = 0, tiles = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp_item& it = items[b];
        int32_t st = validate_item(it, b);
        if (st != VP_OK) return st;
        const std::string at = "item " + std::to_string(b) + ": ";
        if (it.dst_h != it.src_h || it.dst_w != it.src_w)
            return fail(VP_ERR_DIMS, at + "vp_patchify_batch needs frames already at the target size");
        if (reinterpret_cast<uintptr_t>(it.frames) % 4 != 0)
            return fail(VP_ERR_ARG, at + "frames must be 4-byte aligned");
        vp::DevItem& d = p->items[b];
        d.frames = it.frames;
        d.frame_bytes = int64_t(it.src_h) * it.src_w * 3;
        d.H = d.h = it.dst_h;
        d.W = d.w = it.dst_w;
        d.t = (it.n_idx + 1) / 2;
        d.patch = P;
        d.hm = it.dst_h / (2 * P);
        d.wm = it.dst_w / (2 * P);
        d.idx_off = static_cast<int32_t>(p->indices.size());
        for (int32_t k = 0; k < 2 * d.t; ++k)
            p->indices.push_back(it.indices[k < it.n_idx ? k : it.n_idx - 1]);
        d.route = vp::kRoutePatch;
        d.row_off = rows;
        p->grid[3 * b + 0] = d.t;
        p->grid[3 * b + 1] = it.dst_h / P;
        p->grid[3 * b + 2] = it.dst_w / P;
        rows += int64_t(d.t) * (it.dst_h / P) * (it.dst_w / P);
        tiles += int64_t(d.t) * d.hm * (P == 14 ? d.wm : 1);   // patch 14: merge windows
        if (rows > INT32_MAX || tiles > INT32_MAX)
            return fail(VP_ERR_CAPACITY, "batch has more than 2^31-1 rows");
        p->cu[b + 1] = static_cast<int32_t>(rows);
        p->prefix[b + 1] = static_cast<int32_t>(tiles);
    }
    p->total_rows = rows;
    p->off_items = 0;
    p->off_prefix = align_up(p->off_items + sizeof(vp::DevItem) * p->items.size());
    p->off_indices = align_up(p->off_prefix + sizeof(int32_t) * p->prefix.size());
    p->off_tables = align_up(p->off_indices + sizeof(int32_t) * p->indices.size());
    p->off_units = p->off_tables;
    p->off_wgs = p->off_tables;
    p->bytes = p->off_tables;
    p->all_copied();
    return VP_OK;
}

// Plan of the row tables (vp_position_ids): per item its grid, with the
// items' row offsets (cu) as the prefix the kernel searches.
int32_t build_rows_plan(const vp_item* items, int32_t n, Plan* p) {
    if (items == nullptr) return fail(VP_ERR_NULL, "items is NULL");
    if (n < 1) return fail(VP_ERR_ARG, "n_items < 1");
    int32_t P = vp::kPatch;
    if (const int32_t st = batch_patch(items, n, &P); st != VP_OK) return st;
    p->items.assign(n, vp::DevItem{});
    p->grid.assign(size_t(n) * 3, 0);
    p->cu.assign(n + 1, 0);
    p->indices.clear();
    p->tables.clear();
    p->table_words = 0;
    p->units.clear();
    p->wgs.clear();
    p->launches.clear();
    p->generic_cost = p->generic_chain = 0;
    int64_t rows = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp_item& it = items[b];
        const int32_t st = validate_item(it, b);
        if (st != VP_OK) return st;
        vp::DevItem& d = p->items[b];
        d.h = it.dst_h;
        d.w = it.dst_w;
        d.t = (it.n_idx + 1) / 2;
        d.patch = P;
        d.hm = it.dst_h / (2 * P);
        d.wm = it.dst_w / (2 * P);
        d.row_off = rows;
        p->grid[3 * b + 0] = d.t;
        p->grid[3 * b + 1] = it.dst_h / P;
        p->grid[3 * b + 2] = it.dst_w / P;
        rows += int64_t(d.t) * (it.dst_h / P) * (it.dst_w / P);
        if (rows > INT32_MAX) return fail(VP_ERR_CAPACITY, "batch has more than 2^31-1 rows");
        p->cu[b + 1] = static_cast<int32_t>(rows);
    }
    p->prefix = p->cu;
    p->total_rows = rows;
    p->off_items = 0;
    p->off_prefix = align_up(p->off_items + sizeof(vp::DevItem) * p->items.size());
    p->off_indices = align_up(p->off_prefix + sizeof(int32_t) * p->prefix.size());
    p->off_tables = p->off_indices;
    p->off_units = p->off_indices;
    p->off_wgs = p->off_indices;
    p->bytes = p->off_indices;
    p->all_copied();
    return VP_OK;
}

// Output tile of the uint8 writer for an item: the largest rows x columns
// (rows from 32 down, then columns from 64 down) whose horizontal-pass rows,
// staged source span and weights fit the kernel's LDS budgets.
bool resize_tiles(const AxisFilter& fy, const AxisFilter& fx, int32_t* rb, int32_t* cb) {
    static const int32_t kRows[] = {32, 16, 8, 4, 2, 1};
    static const int32_t kCols[] = {64, 32, 16, 8};
    for (int32_t r : kRows) {
        if (int64_t(r) * fy.taps > vp::kRsQ) continue;
        int64_t rows = 0;   // source rows the tile's horizontal pass produces
        for (int32_t i0 = 0; i0 < fy.n_out; i0 += r) {
            const int32_t i1 = std::min(i0 + r, fy.n_out) - 1;
            rows = std::max<int64_t>(rows, fy.start[i1] + fy.count[i1] - fy.start[i0]);
        }
        for (int32_t c : kCols) {
            if (int64_t(c) * fx.taps > vp::kRsQ) continue;
            int64_t span = 0;   // source pixels the tile's columns read
            for (int32_t j0 = 0; j0 < fx.n_out; j0 += c) {
                const int32_t j1 = std::min(j0 + c, fx.n_out) - 1;
                span = std::max<int64_t>(span, fx.start[j1] + fx.count[j1] - fx.start[j0]);
            }
            if (rows * c * 3 <= vp::kRsMid && span * 3 + 6 <= vp::kRsSrcRow) {
                *rb = r;
                *cb = c;
                return true;
            }
        }
    }
    return false;
}

// Shape of the uint8 streaming writer for an item, if it can take it: the
// output width in bands of 64 columns (down to 16), each band's source span
// within 64 lanes of px pixels, the column taps rounded up to 4, M slots.
// The widest band that fits is taken: the horizontal pass costs the same per
// output column whatever the band, and fewer bands unpack fewer pixels.
bool resize_stream_shape(const vp_item& it, const AxisFilter& fx, int32_t m, StreamShape* sh) {
    if (m < 4 || m > vp::kStreamSlots) return false;
    const int32_t kx = round_up(fx.taps + 3, 4);   // any window start, rounded down to a dword
    if (!vp::resize_stream_supported(m, kx, vp::kRsPx)) return false;
    if (int64_t(it.src_h + vp::kSlotMax + 8) * it.src_w * 3 + 64 >= (int64_t(1) << 32)) return false;
    for (int32_t band = 64; band >= 16; band -= 16) {
        if (band_span(fx, band) > 64 * vp::kRsPx) continue;
        if ((it.dst_w + band - 1) / band > vp::kWgBandMax) continue;
        sh->m = m;
        sh->kx = kx;
        sh->px = vp::kRsPx;
        sh->band = band;
        sh->bands = (it.dst_w + band - 1) / band;
        return true;
    }
    return false;
}

// Plan of vp_resize_batch: per item its frames in index order (no padding),
// fixed-point tables, the route (streaming, or the tile kernel where an axis
// does not fit the streaming shapes) and its output byte offset.
// `few_units`: no more work units than whole frames and the dot-product form's
// long units need: the matrix-core form on whole frames, and only in place of
// the dot-product form, not of the general kernel, which needs none.
int32_t build_resize_plan(const vp_item* items, int32_t n, Plan* p, bool few_units = false) {
    if (items == nullptr) return fail(VP_ERR_NULL, "items is NULL");
    if (n < 1) return fail(VP_ERR_ARG, "n_items < 1");
    int32_t P = vp::kPatch;
    if (const int32_t st = batch_patch(items, n, &P); st != VP_OK) return st;
    p->items.assign(n, vp::DevItem{});
    p->prefix.assign(n + 1, 0);
    p->byte_off.assign(n + 1, 0);
    p->grid.clear();
    p->cu.clear();
    p->indices.clear();
    p->tables.clear();
    p->table_words = 0;
    p->units.clear();
    p->wgs.clear();
    p->launches.clear();
    p->generic_cost = p->generic_chain = 0;
    auto append = [&](std::shared_ptr<const std::vector<int32_t>> words) -> int32_t {
        const int32_t o = static_cast<int32_t>(p->table_words);
        p->table_words += words->size();
        p->tables.emplace_back(o, std::move(words));
        return o;
    };
    std::map<std::pair<int32_t, int32_t>, PlanAxis> axes;
    auto axis_for = [&](int32_t n_in, int32_t n_out) -> PlanAxis& {
        PlanAxis& a = axes[std::make_pair(n_in, n_out)];
        if (a.entry == nullptr)
            a.entry = cached(g_axis_cache, std::make_pair(n_in, n_out), [&] { return make_axis_entry(n_in, n_out); });
        return a;
    };
    auto window_table = [&](PlanAxis& a) { return a.windows >= 0 ? a.windows : a.windows = append({a.entry, &a.entry->fixed_words}); };
    auto start_table = [&](PlanAxis& a) { return a.starts >= 0 ? a.starts : a.starts = append({a.entry, &a.entry->f.start}); };
    std::map<SlotKey, std::pair<int32_t, std::shared_ptr<const SlotEntry>>> slot_tables;
    auto slots_for = [&](const AxisFilter& f, int32_t* off, int32_t* m) -> bool {
        const SlotKey key = std::make_pair(f.n_in, f.n_out);
        auto found = slot_tables.find(key);
        if (found == slot_tables.end()) {
            auto e = cached(g_slot_cache, key, [&] {
                auto v = std::make_shared<SlotEntry>();
                v->m = build_slots(f, &v->words);
                return std::shared_ptr<const SlotEntry>(std::move(v));
            });
            const int32_t o = e->m > 0 ? append(std::shared_ptr<const std::vector<int32_t>>(e, &e->words)) : -1;
            found = slot_tables.emplace(key, std::make_pair(o, e)).first;
        }
        *off = found->second.first;
        *m = found->second.second->m;
        return found->second.first >= 0;
    };
    std::map<ColumnKey, int32_t> column_tables;
    // the dot-product column table, or -1 if a weight does not fit its digits
    auto columns_for = [&](const AxisFilter& f, int32_t kx, int32_t band, int32_t row_px) -> int32_t {
        const ColumnKey key = std::make_tuple(f.n_in, f.n_out, kx, band, row_px);
        auto found = column_tables.find(key);
        if (found == column_tables.end()) {
            auto e = cached(g_column_cache, key, [&] {
                auto v = std::make_shared<std::vector<int32_t>>();
                if (!build_columns_dot(f, kx, band, row_px, v.get())) v->clear();
                return std::shared_ptr<const std::vector<int32_t>>(std::move(v));
            });
            found = column_tables.emplace(key, e->empty() ? -1 : append(e)).first;
        }
        return found->second;
    };
    std::map<std::tuple<int32_t, int32_t, bool>, std::pair<int32_t, int32_t>> digit_tables;
    // the digit table of an axis (offset, extent), or offset -1 if the axis does not fit
    auto digits_for = [&](const AxisFilter& f, bool columns) -> std::pair<int32_t, int32_t> {
        const auto at = std::make_tuple(f.n_in, f.n_out, columns);
        auto found = digit_tables.find(at);
        if (found == digit_tables.end()) {
            // (the extent rides behind the words)
            auto e = cached(g_column_cache, std::make_tuple(f.n_in, f.n_out, vp::kRsMmShape, columns ? 1 : 0, 0), [&] {
                auto v = std::make_shared<std::vector<int32_t>>();
                int32_t extent = 0;
                if (build_digits(f, columns, v.get(), &extent)) v->push_back(extent);
                else v->clear();
                return std::shared_ptr<const std::vector<int32_t>>(std::move(v));
            });
            const int32_t extent = e->empty() ? 0 : e->back();
            found = digit_tables.emplace(at, std::make_pair(e->empty() ? -1 : append(e), extent)).first;
        }
        return found->second;
    };
    std::vector<StreamShape> shapes(n);
    int64_t bytes = 0, tiles = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp_item& it = items[b];
        int32_t st = validate_item(it, b);
        if (st != VP_OK) return st;
        vp::DevItem& d = p->items[b];
        d.frames = it.frames;
        d.frame_bytes = int64_t(it.src_h) * it.src_w * 3;
        d.H = it.src_h;
        d.W = it.src_w;
        d.h = it.dst_h;
        d.w = it.dst_w;
        d.t = it.n_idx;
        d.idx_off = static_cast<int32_t>(p->indices.size());
        p->indices.insert(p->indices.end(), it.indices, it.indices + it.n_idx);
        PlanAxis& ay = axis_for(it.src_h, it.dst_h);
        PlanAxis& ax = axis_for(it.src_w, it.dst_w);
        const AxisFilter* fy = &ay.entry->f;
        const AxisFilter* fx = &ax.entry->f;
        d.ky = fy->taps;
        d.kx = fx->taps;
        d.patch = P;
        d.row_off = bytes;   // output byte offset of the item
        bytes += int64_t(it.n_idx) * it.dst_h * it.dst_w * 3;
        int32_t m = 0;
        StreamShape sh;
        std::pair<int32_t, int32_t> dx(-1, 0), dy(-1, 0);
        if ((it.dst_w + 15) / 16 <= vp::kWgBandMax && int64_t(it.src_h + 64) * it.src_w * 3 + 256 < (int64_t(1) << 32) &&
            (dx = digits_for(*fx, true)).first >= 0)
            dy = digits_for(*fy, false);
        const bool mm = dx.first >= 0 && dy.first >= 0 &&
                        !(few_units && ((dx.second & vp::kRsMmWide) != 0 || ay.entry->slots < 0 ||
                                        ay.entry->slots > vp::kStreamSlots));
        const bool slots = !mm && slots_for(*fy, &d.sy_off, &m);
        if (mm) {
            d.route = vp::kRouteStream;
            const int32_t cols = vp::resize_mm_cols((dx.second & vp::kRsMmWide) != 0);
            d.band = cols;
            d.row_px = 0;
            d.sx_off = dx.first;
            d.sy_off = dy.first;
            sh.m = dx.second % 256 + (dy.second > 4 ? vp::kRsMmTwo : 0);
            sh.px = dx.second / 256;
            sh.kx = vp::kRsMmShape;
            sh.band = cols;
            sh.bands = (it.dst_w + cols - 1) / cols;
            sh.ring = dy.second;
            shapes[b] = sh;
        } else if (slots && resize_stream_shape(it, *fx, m, &sh) &&
            (d.sx_off = columns_for(*fx, sh.kx, sh.band, 64 * sh.px)) >= 0) {
            d.route = vp::kRouteStream;
            d.band = sh.band;
            d.row_px = 64 * sh.px;
            shapes[b] = sh;
        } else {
            if (!resize_tiles(*fy, *fx, &d.rh, &d.cw))
                return fail(VP_ERR_CAPACITY, "item " + std::to_string(b) +
                                                 ": filter window too long for the uint8 writer's tiles");
            d.hm = (it.dst_h + d.rh - 1) / d.rh;
            d.wm = (it.dst_w + d.cw - 1) / d.cw;
            d.route = vp::kRouteResize;
            tiles += int64_t(it.n_idx) * d.hm * d.wm;
            p->generic_cost += int64_t(8) * it.n_idx * it.src_h * it.src_w;   // about 8x the streaming cost per pixel
            p->generic_chain = INT64_MAX;
        }
        if (!mm) {   // (the matrix-core form reads its digit tables only)
            d.ty_off = d.route == vp::kRouteStream ? start_table(ay) : window_table(ay);
            d.tx_off = d.route == vp::kRouteStream ? start_table(ax) : window_table(ax);
        }
        if (tiles > INT32_MAX) return fail(VP_ERR_CAPACITY, "batch has more than 2^31-1 tiles");
        p->byte_off[b + 1] = bytes;
        p->prefix[b + 1] = static_cast<int32_t>(tiles);
    }
    p->total_rows = 0;
    merge_matrix_shapes(p->items, &shapes);

    // Streaming units: one per (item, frame, band of output rows), the
    // bands sized as for the float path (multiples of the kernel's store
    // group of 4 rows).
    constexpr int64_t kWaveSlots = 256 * 20;
    int64_t wave_rows = 0;
    for (int32_t b = 0; b < n; ++b) {
        const vp::DevItem& d = p->items[b];
        if (d.route == vp::kRouteStream) wave_rows += int64_t(d.t) * shapes[b].bands * d.H;
    }
    const int64_t max_src_rows = wave_rows / (kWaveSlots * 8);
    // Units of the matrix-core form, by the batch's waves at 16-row units.
    // Setting one up costs about four chunks of source rows, so they are as
    // long as the chip stays full with: measured, kernel us at 16 / 32 / 64 /
    // 128 / 192 rows: 1080p x 2 frames 15 / 17 / 25 / 41 / 58, x 8
    // 30 / 23 / 27 / 42 / 59, x 16 49 / 42 / 35 / 47 / 61, x 64 160 / 131 / 124 /
    // 124 / 154, x 256 605 / 480 / 425 / 428 / 446; 480p x 8 15 / 15 / 19 / 27 /
    // 34, x 32 35 / 30 / 27 / 31 / 38, x 256 248 / 194 / 177 / 164 / 160.
    int64_t mm_waves = 0;
    for (int32_t b = 0; b < n; ++b)
        if (p->items[b].route == vp::kRouteStream && shapes[b].kx == vp::kRsMmShape)
            mm_waves += int64_t(p->items[b].t) * shapes[b].bands * ((p->items[b].h + 15) / 16);
    int64_t mm_rows = mm_waves < 3000 ? 16 : mm_waves < 6000 ? 32 : mm_waves < 60000 ? 64 : 128;
    int64_t mm_units = 0;
    for (int32_t b = 0; b < n; ++b)
        if (p->items[b].route == vp::kRouteStream && shapes[b].kx == vp::kRsMmShape)
            mm_units += int64_t(p->items[b].t) * ((p->items[b].h + mm_rows - 1) / mm_rows);
    // (whole frames: units are numbered below 2^20)
    if (few_units || mm_units > vp::kWgUnitMask / 2) mm_rows = INT32_MAX;
    const auto unit_waves = [&](int64_t rows) {   // of the dot-product form
        int64_t waves = 0;
        for (int32_t b = 0; b < n; ++b) {
            const vp::DevItem& d = p->items[b];
            if (d.route != vp::kRouteStream || shapes[b].kx == vp::kRsMmShape) continue;
            waves += int64_t(d.t) * shapes[b].bands *
                     UnitSplit(d.h, unit_row_band(d, max_src_rows, 4, 10, rows), 4).n;
        }
        return waves;
    };
    const int64_t short_rows = few_units ? 0 : short_unit_rows(unit_waves, unit_waves, kShortWavesDot);
    std::vector<Keyed> keyed;
    for (int32_t b = 0; b < n; ++b) {
        const vp::DevItem& d = p->items[b];
        if (d.route != vp::kRouteStream) continue;
        const StreamShape& sh = shapes[b];
        // whole store groups: 4 rows, or 16 of the matrix-core form
        const bool mm = sh.kx == vp::kRsMmShape;
        const UnitSplit split(d.h, mm ? mm_rows : unit_row_band(d, max_src_rows, 4, 10, short_rows), mm ? 16 : 4);
        for (int32_t k = 0; k < d.t; ++k) {
            for (int64_t u = 0; u < split.n; ++u) {
                const int32_t i0 = split.begin(u), i1 = split.end(u);
                Keyed e;
                e.key = std::make_tuple(sh.m, sh.kx, sh.px);
                e.bands = sh.bands;
                e.lds_units = sh.ring;
                e.unit.item = b;
                e.unit.p_flags = k;
                e.unit.i0 = i0;
                e.unit.i1 = i1;
                // (times the bands: those of the matrix-core form are a half or a quarter of 64 columns)
                e.cost = int64_t(i1 - i0) * d.H / d.h * d.W * sh.band / 64;
                keyed.push_back(e);
            }
        }
    }
    if (const int32_t st = assemble_launches(keyed, P, 64, p); st != VP_OK) return st;

    p->off_items = 0;
    p->off_prefix = align_up(p->off_items + sizeof(vp::DevItem) * p->items.size());
    p->off_indices = align_up(p->off_prefix + sizeof(int32_t) * p->prefix.size());
    p->off_tables = align_up(p->off_indices + sizeof(int32_t) * p->indices.size());
    p->off_units = align_up(p->off_tables + sizeof(int32_t) * p->table_words);
    p->off_wgs = align_up(p->off_units + sizeof(vp::StreamUnit) * p->units.size());
    p->bytes = align_up(p->off_wgs + sizeof(uint32_t) * p->wgs.size());
    p->all_copied();
    return VP_OK;
}

// ---------------------------------------------------------------------------
// Plan cache.  An RL loop or a serving loop hands the library the same batch
// (the same frame buffers, sizes and index lists) call after call; its plan
// is a pure function of those, so the last few plans are kept and reused
// when every field and every index matches.  Entries are immutable and
// shared by pointer; a cache holds kPlanCacheMax plans, the most recently
// used first.
// ---------------------------------------------------------------------------

// (kBatchSmall: kBatch in less memory, upscales of many slots on the general kernel)
// (kBatchLong: kBatch without short units)
enum class PlanKind : int64_t { kBatch = 1, kPatch = 2, kResize = 3, kRows = 4, kBatchSmall = 5, kBatchLong = 6 };

constexpr size_t kPlanCacheMax = 8;
std::mutex g_plan_mu;
std::list<std::pair<std::vector<int64_t>, std::shared_ptr<const Plan>>> g_plans;

// A first plan that needs more work units than a launch can index gives way to
// one with as many items as may be on kernels that need none, or fewer; the
// caller sees the error of a plan only where the call fails with it.
int32_t build_kind(PlanKind kind, const vp_item* items, int32_t n, Plan* p) {
    const std::string before = g_last_error;
    const auto or_else = [&](int32_t st, auto second) {
        if (st != VP_ERR_CAPACITY) return st;
        st = second();
        if (st == VP_OK) g_last_error = before;
        return st;
    };
    switch (kind) {
        case PlanKind::kBatch:
            return or_else(build_plan(items, n, p), [&] { return build_plan(items, n, p, vp::kStreamSlots); });
        case PlanKind::kBatchSmall: return build_plan(items, n, p, vp::kStreamSlots);
        case PlanKind::kBatchLong: return build_plan(items, n, p, vp::kSlotWords, true);
        case PlanKind::kPatch: return build_patch_plan(items, n, p);
        case PlanKind::kResize:
            return or_else(build_resize_plan(items, n, p), [&] { return build_resize_plan(items, n, p, true); });
        case PlanKind::kRows: return build_rows_plan(items, n, p);
    }
    return fail(VP_ERR_ARG, "unknown plan kind");
}

// The plan of `items` for `kind`: from the cache if an identical batch was
// planned recently, else built (and cached if valid).  Errors are those of
// the builder; nothing invalid is cached.
int32_t get_plan(PlanKind kind, const vp_item* items, int32_t n, std::shared_ptr<const Plan>* out) {
    bool cacheable = items != nullptr && n >= 1;
    for (int32_t b = 0; cacheable && b < n; ++b)
        cacheable = items[b].indices != nullptr && items[b].n_idx >= 1;
    if (!cacheable) {   // the builder reports the error
        Plan p;
        const int32_t st = build_kind(kind, items, n, &p);
        if (st == VP_OK) *out = std::make_shared<const Plan>(std::move(p));
        return st;
    }
    std::vector<int64_t> key;
    key.reserve(2 + size_t(n) * 8);
    key.push_back(static_cast<int64_t>(kind));
    key.push_back(n);
    for (int32_t b = 0; b < n; ++b) {
        const vp_item& it = items[b];
        key.insert(key.end(), {static_cast<int64_t>(reinterpret_cast<uintptr_t>(it.frames)), it.n_src,
                               it.src_h, it.src_w, it.n_idx, it.dst_h, it.dst_w, it.patch});
        key.insert(key.end(), it.indices, it.indices + it.n_idx);
    }
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        for (auto e = g_plans.begin(); e != g_plans.end(); ++e)
            if (e->first == key) {
                g_plans.splice(g_plans.begin(), g_plans, e);   // most recent first
                *out = e->second;
                return VP_OK;
            }
    }
    Plan p;
    const int32_t st = build_kind(kind, items, n, &p);
    if (st != VP_OK) return st;
    auto plan = std::make_shared<const Plan>(std::move(p));
    std::lock_guard<std::mutex> lk(g_plan_mu);
    g_plans.emplace_front(std::move(key), plan);
    if (g_plans.size() > kPlanCacheMax) g_plans.pop_back();
    *out = std::move(plan);
    return VP_OK;
}

// ---------------------------------------------------------------------------
// Pinned staging ring: the plan blob is written into pinned host memory,
// from where a kernel on the call's stream copies it; a slot is reused only
// after the kernel that read it has completed.  (Coherent memory: the kernel
// must see what the host wrote since the slot's last use.)
// ---------------------------------------------------------------------------

struct Slot {
    void* host = nullptr;
    size_t cap = 0;
    hipEvent_t done = nullptr;
    bool pending = false;
};

struct Ring {
    std::mutex mu;
    Slot slots[4];
    int next = 0;
};

std::mutex g_rings_mu;
std::map<int, Ring*> g_rings;

Ring* ring_for_device(int dev) {
    std::lock_guard<std::mutex> lk(g_rings_mu);
    Ring*& r = g_rings[dev];
    if (r == nullptr) r = new Ring();  // lives until process exit
    return r;
}

int32_t hip_fail(hipError_t e, const char* what) {
    return fail(VP_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Writes the copied part of the plan blob (p.off_gen bytes, the layout of
// vp_plan.h) to `base`:
// each section, then zeros up to the next one (the gaps are never read;
// zeroing them keeps the blob deterministic).
void pack_plan(const Plan& p, uint8_t* base) {
    auto put = [&](size_t off, const void* src, size_t n, size_t next) {
        if (n != 0) std::memcpy(base + off, src, n);
        std::memset(base + off + n, 0, next - off - n);
    };
    put(p.off_items, p.items.data(), sizeof(vp::DevItem) * p.items.size(), p.off_prefix);
    put(p.off_prefix, p.prefix.data(), sizeof(int32_t) * p.prefix.size(), p.off_indices);
    put(p.off_indices, p.indices.data(), sizeof(int32_t) * p.indices.size(), p.off_tables);
    for (const auto& part : p.tables)
        std::memcpy(base + p.off_tables + sizeof(int32_t) * part.first, part.second->data(),
                    sizeof(int32_t) * part.second->size());
    put(p.off_tables + sizeof(int32_t) * p.table_words, nullptr, 0, p.off_units);
    put(p.off_units, p.units.data(), sizeof(vp::StreamUnit) * p.units.size(), p.off_wgs);
    put(p.off_wgs, p.wgs.data(), sizeof(uint32_t) * p.wgs.size(), p.off_jobs);
    put(p.off_jobs, p.jobs.data(), sizeof(vp::TableJob) * p.jobs.size(), p.off_gen);
}

// The plan's copy of vp_preprocess_batch_noalloc comes from pageable memory.
// The runtime sends up to 16 KiB of that with the stream's commands: 4.4 us of
// the host and 2.5 us of the GPU a piece, measured; a larger copy is staged and
// costs 22 us of the host and 17 us of the GPU, up to 64 KB (131 KB 24 us).  So
// plans of up to four pieces go in pieces: 64 frames of 480p in float32 90 ->
// 78 us a call back to back, 8 frames 36 -> 32.
constexpr size_t kCopyPiece = 16384;
constexpr size_t kCopyPieces = 4;
constexpr int64_t kCopyRows = 32768;     // (upload_plan)
constexpr int64_t kCopyLongRows = 72;    // (run_batch)

// Whether that entry fills the computed tables on the host and copies them with
// the rest: a kernel that computes them between the copy and the batch costs a
// call 5 us of the GPU, the host about 1 ns a word, which a batch with work
// enough hides.  In a plan that goes in one copy the tables' share of it costs
// less than their kernel (64 frames of 1080p 155 -> 150 us, 32 of 4K 295 ->
// 291), in one that goes in pieces no less.  Many tables stay on the device (20
// ragged images 78 us, 338 with the host's), and so do those of small batches:
// at 256 source pixels a word a batch streams for four times the host's work.
// Tables that fit into the pieces that their plan takes anyway ride along too,
// and save the launch (13 frames of 18x19 -> 32x32 21.1 -> 18.4 us a call); at
// the price of one more piece they do not (an image of 110x121 -> 224x256 20.7
// with the kernel, 21.5 with the piece).
constexpr size_t kHostTableWords = 32768;
constexpr int64_t kHostTablePixels = 256;

size_t copy_pieces(size_t bytes) { return (bytes + kCopyPiece - 1) / kCopyPiece; }

bool tables_on_host(const Plan& p) {
    if (p.bytes <= kCopyPieces * kCopyPiece && copy_pieces(p.bytes) == copy_pieces(p.off_gen)) return true;
    if (p.off_gen <= kCopyPieces * kCopyPiece || p.gen_words > kHostTableWords) return false;
    int64_t pixels = 0;
    for (const vp::DevItem& d : p.items)
        if (d.route == vp::kRouteStream) pixels += int64_t(2) * d.t * d.H * d.W;
    return pixels >= kHostTablePixels * static_cast<int64_t>(p.gen_words);
}

// The plan's computed tables on the host, into `tables` (the first tables
// section's place in the blob; the computed words zeroed): the same words that
// the upload kernel computes from the same pieces.
void fill_tables(const Plan& p, int32_t* tables) {
    std::shared_ptr<const AxisEntry> axis;
    for (const vp::TableJob& t : p.jobs) {
        if (axis == nullptr || axis->f.n_in != t.n_in || axis->f.n_out != t.n_out)
            axis = cached(g_axis_cache, std::make_pair(t.n_in, t.n_out), [&] { return make_axis_entry(t.n_in, t.n_out); });
        const AxisFilter& f = axis->f;
        const int32_t kind = t.kind_lanes & 255, lanes = t.kind_lanes >> 8;
        int32_t* const out = tables + t.off;
        float* const weights = reinterpret_cast<float*>(out);
        const int64_t rows = f.n_in + vp::kSlotMax;
        const int32_t end = std::min(f.n_out, t.base + vp::table_outputs(lanes));   // (starts, zeros: one lane)
        if (kind == vp::kTableStarts) {
            std::copy(f.start.begin() + t.base, f.start.begin() + end, out + t.base);
        } else if (kind == vp::kTableZeros) {   // the two close rows that are never reached
            const int64_t words = rows * t.a;
            for (int64_t e = std::max<int64_t>(words, t.base); e < std::min<int64_t>(words + 2, t.base + vp::kTablePiece); ++e)
                out[e + f.n_out] = INT32_MAX;
        } else if (kind == vp::kTableSlots) {
            for (int32_t i = t.base; i < end; ++i) {
                const int32_t slot = i % t.a;
                for (int32_t k = 0; k < f.count[i]; ++k)
                    weights[int64_t(f.start[i] + k) * t.a + slot] = f.weight[size_t(i) * f.taps + k] * 16777216.0f;   // times 2^24
                out[rows * t.a + i] = f.start[i] + f.count[i] - 1;
            }
        } else {
            for (int32_t j = t.base; j < end; ++j) {
                const int32_t l = f.start[j] - f.start[j / t.band * t.band];
                const int32_t s = std::min(l, t.row_px - t.a);
                std::copy_n(f.weight.begin() + int64_t(j) * f.taps, f.count[j], weights + f.n_out + int64_t(j) * t.a + l - s);
                out[j] = s;
            }
        }
    }
}

int32_t upload_plan(const Plan& p, void* workspace, hipStream_t stream) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    Ring* ring = ring_for_device(dev);
    std::lock_guard<std::mutex> lk(ring->mu);
    Slot& s = ring->slots[ring->next];
    ring->next = (ring->next + 1) % 4;
    if (s.pending) {
        e = hipEventSynchronize(s.done);
        if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
        s.pending = false;
    }
    if (s.done == nullptr) {
        e = hipEventCreateWithFlags(&s.done, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    }
    if (s.cap < p.off_gen) {
        if (s.host != nullptr) (void)hipHostFree(s.host);
        s.host = nullptr;
        s.cap = 0;
        size_t cap = align_up(p.off_gen * 2);
        e = hipHostMalloc(&s.host, cap, hipHostMallocCoherent);
        if (e != hipSuccess) return hip_fail(e, "hipHostMalloc");
        s.cap = cap;
    }
    pack_plan(p, static_cast<uint8_t*>(s.host));
    void* src = nullptr;
    e = hipHostGetDevicePointer(&src, s.host, 0);
    if (e != hipSuccess) return hip_fail(e, "hipHostGetDevicePointer");
    // A small plan without computed tables: the runtime sends its copy with the
    // stream's commands, sooner than a kernel reads it, but takes the host 1 us
    // more, which calls of little GPU work wait for (position tables 16.3 ->
    // 17.7 us a call).  So: for the general (or the writer's tile) kernel alone
    // (59 frames of 42x67 -> 28x140 in float32 55.0 -> 51.7), and for patchify
    // of 100 MB of rows and more (64 frames of 512x704 in bf16 38.5 -> 37.2).
    const bool long_call = (p.generic_cost > 0 && p.launches.empty()) ||
                           (p.items[0].route == vp::kRoutePatch && p.total_rows >= kCopyRows);
    if (long_call && p.off_gen <= kCopyPiece)
        e = hipMemcpyAsync(workspace, s.host, p.off_gen, hipMemcpyHostToDevice, stream);
    else
        e = static_cast<hipError_t>(vp::launch_upload(
            workspace, src, static_cast<int64_t>(p.off_gen),
            reinterpret_cast<const vp::TableJob*>(static_cast<const uint8_t*>(src) + p.off_jobs),
            static_cast<int>(p.jobs.size()), reinterpret_cast<int32_t*>(static_cast<uint8_t*>(workspace) + p.off_tables),
            stream));
    if (e != hipSuccess) return hip_fail(e, "plan upload");
    e = hipEventRecord(s.done, stream);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
    s.pending = true;
    return VP_OK;
}

// ---------------------------------------------------------------------------
// Side streams.  The launches of one call (one per streaming-kernel shape,
// plus the general kernel) are independent of each other; on the caller's
// stream alone they would run one after another, and a small launch leaves
// most of the chip idle for the whole life of its longest workgroup.  Calls
// with several launches therefore fork to up to kSideStreams more streams of
// the device and join back with events, so the call stays one ordered step
// of the caller's stream.  The streams (default priority) and events are
// created on first use and kept until the process ends.
// ---------------------------------------------------------------------------

constexpr int kSideStreams = 3;

struct Side {
    std::mutex mu;   // held from fork to join: the events are shared by all calls
    bool ready = false;
    hipStream_t s[kSideStreams] = {};
    hipEvent_t fork = nullptr;
    hipEvent_t join[kSideStreams] = {};
};

std::mutex g_side_mu;
std::map<int, Side*> g_side;

int32_t side_for_device(int dev, Side** out) {
    Side* side = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_side_mu);
        Side*& r = g_side[dev];
        if (r == nullptr) r = new Side();   // lives until process exit
        side = r;
    }
    std::lock_guard<std::mutex> lk(side->mu);
    if (!side->ready) {
        hipError_t e = hipEventCreateWithFlags(&side->fork, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate (fork)");
        for (int i = 0; i < kSideStreams; ++i) {
            e = hipStreamCreateWithFlags(&side->s[i], hipStreamNonBlocking);
            if (e != hipSuccess) return hip_fail(e, "hipStreamCreate (side stream)");
            e = hipEventCreateWithFlags(&side->join[i], hipEventDisableTiming);
            if (e != hipSuccess) return hip_fail(e, "hipEventCreate (join)");
        }
        side->ready = true;
    }
    *out = side;
    return VP_OK;
}

// The plan's launches (the tile kernel, if it has tiles, and one per
// streaming shape), spread over the caller's stream and the side streams by
// estimated cost.  `resize`: the uint8 writer's kernels instead of the float
// path's (out_dtype and norm unused).
// With `one_stream` every launch goes to the caller's stream, one after
// another (no side streams, nothing created).
int32_t run_launches(const Plan& p, const vp::PlanView& view, void* out_rows, int32_t out_dtype,
                     const vp::Norm& norm, hipStream_t stream, bool resize = false,
                     bool one_stream = false) {
    struct Job {
        int32_t launch;   // index into p.launches, or -1 for the general kernel
        int64_t cost;
        int32_t rank;     // launched before those of a lower one
    };
    // A general or tile kernel whose workgroups run long goes first: of 57 KB
    // of LDS each, they find no room on CUs that small workgroups have filled
    // (132 frames of 350x915 with 12 of 408x5886 on the writer's tile kernel
    // 504 -> 279 us a call; 284 frames of 1037x236 and 1165x347 with 3 of
    // 335x2602 on the general one 2,128 -> 1,651).  Up to about 200 steps, 25
    // us, it follows by its cost (64 frames of 720p with 8 of 60x60 -> 320x320:
    // first 123, by cost 113).  The writer's dot products, a row at a time, go
    // before its matrix-core form (201 frames of 161x369 with 207 of 434x538 on
    // dot products 228 -> 139).
    std::vector<Job> jobs;
    if (view.n_tiles > 0) jobs.push_back(Job{-1, p.generic_cost, p.generic_chain > 200 ? 2 : 0});
    for (size_t k = 0; k < p.launches.size(); ++k)
        jobs.push_back(Job{static_cast<int32_t>(k), p.launches[k].cost, resize && p.launches[k].kx != vp::kRsMmShape ? 1 : 0});
    auto launch = [&](const Job& j, hipStream_t st) -> int32_t {
        if (resize) {
            const int err = j.launch < 0 ? vp::launch_resize(view, out_rows, st)
                                         : vp::launch_resize_stream(view, p.launches[j.launch], out_rows, st);
            if (err != 0) return hip_fail(static_cast<hipError_t>(err), "uint8 writer launch");
        } else if (j.launch < 0) {
            const int err = vp::launch_generic(view, out_rows, out_dtype, norm, st);
            if (err != 0) return hip_fail(static_cast<hipError_t>(err), "general kernel launch");
        } else {
            const int err = vp::launch_stream(view, p.launches[j.launch], out_rows, out_dtype, norm, st);
            if (err != 0) return hip_fail(static_cast<hipError_t>(err), "streaming kernel launch");
        }
        return VP_OK;
    };
    if (jobs.size() <= 1) return jobs.empty() ? VP_OK : launch(jobs[0], stream);
    if (one_stream) {
        for (const Job& j : jobs)
            if (const int32_t st = launch(j, stream); st != VP_OK) return st;
        return VP_OK;
    }

    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    Side* side = nullptr;
    int32_t st = side_for_device(dev, &side);
    if (st != VP_OK) return st;
    std::stable_sort(jobs.begin(), jobs.end(), [](const Job& a, const Job& b) { return std::make_pair(a.rank, a.cost) > std::make_pair(b.rank, b.cost); });
    const int lanes = std::min<int>(static_cast<int>(jobs.size()), kSideStreams + 1);
    std::vector<int> lane_of(jobs.size(), 0);
    std::vector<int64_t> load(lanes, 0);
    for (size_t k = 0; k < jobs.size(); ++k) {
        int best = 0;
        for (int l = 1; l < lanes; ++l)
            if (load[l] < load[best]) best = l;
        lane_of[k] = best;
        load[best] += jobs[k].cost;
    }
    std::lock_guard<std::mutex> lk(side->mu);
    e = hipEventRecord(side->fork, stream);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord (fork)");
    for (int l = 1; l < lanes; ++l) {
        e = hipStreamWaitEvent(side->s[l - 1], side->fork, 0);
        if (e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent (fork)");
    }
    st = VP_OK;
    for (size_t k = 0; k < jobs.size() && st == VP_OK; ++k)
        st = launch(jobs[k], lane_of[k] == 0 ? stream : side->s[lane_of[k] - 1]);
    // join even after a failed launch, so that the caller's stream still
    // orders after whatever was enqueued
    for (int l = 1; l < lanes; ++l) {
        e = hipEventRecord(side->join[l - 1], side->s[l - 1]);
        if (e == hipSuccess) e = hipStreamWaitEvent(stream, side->join[l - 1], 0);
        if (e != hipSuccess && st == VP_OK) st = hip_fail(e, "join of a side stream");
    }
    return st;
}

// Shared body of vp_preprocess_batch (resample + normalise + patchify),
// vp_patchify_batch (frames already at the target size) and
// vp_preprocess_batch_noalloc (no_alloc: the plan goes to the library's
// fixed device array instead of a workspace, copied from pageable host
// memory, and every launch runs on the caller's stream).
int32_t run_batch(bool patch_only, const vp_item* items, int32_t n_items, const float* mean,
                  const float* std, int32_t out_dtype, void* out_rows, int64_t out_rows_capacity,
                  int32_t* grid_thw, int32_t* cu_seqlens, void* workspace, int64_t workspace_bytes,
                  hipStream_t stream, bool no_alloc = false) {
    if (mean == nullptr || std == nullptr || out_rows == nullptr || (!no_alloc && workspace == nullptr))
        return fail(VP_ERR_NULL, no_alloc ? "mean, std and out_rows must be non-NULL"
                                          : "mean, std, out_rows and workspace must be non-NULL");
    if (out_dtype != VP_OUT_F32 && out_dtype != VP_OUT_BF16)
        return fail(VP_ERR_ARG, "out_dtype must be VP_OUT_F32 or VP_OUT_BF16");
    if (reinterpret_cast<uintptr_t>(out_rows) % 16 != 0)
        return fail(VP_ERR_ARG, "out_rows must be 16-byte aligned");
    if (!no_alloc && reinterpret_cast<uintptr_t>(workspace) % kAlign != 0)
        return fail(VP_ERR_ARG, "workspace must be 256-byte aligned");
    vp::Norm norm;
    for (int c = 0; c < 3; ++c) {
        if (!(std[c] > 0.0f) || !std::isfinite(std[c]) || !std::isfinite(mean[c]))
            return fail(VP_ERR_ARG, "std must be positive and finite, mean finite");
        norm.a[c] = static_cast<float>(1.0 / (255.0 * static_cast<double>(std[c])));
        norm.b[c] = static_cast<float>(-static_cast<double>(mean[c]) / static_cast<double>(std[c]));
        norm.z[c] = static_cast<float>(-255.0 * static_cast<double>(mean[c]));
    }
    std::shared_ptr<const Plan> plan;
    int32_t st = get_plan(patch_only ? PlanKind::kPatch : PlanKind::kBatch, items, n_items, &plan);
    if (st != VP_OK) return st;
    // Upscales of 2x to 4x: the x-first kernel's units (28 bytes a frame) are
    // most of such a plan, and the general kernel needs none, so a batch whose
    // plan is too large for the fixed memory may still fit on that kernel.
    if (no_alloc && plan->bytes > static_cast<size_t>(vp::kNoAllocPlanBytes)) {
        std::shared_ptr<const Plan> small;
        if (get_plan(PlanKind::kBatchSmall, items, n_items, &small) == VP_OK &&
            small->bytes <= static_cast<size_t>(vp::kNoAllocPlanBytes))
            plan = std::move(small);
    }
    // Frames of few rows: short units save up to 8 us of the GPU, which such a
    // call does not wait for, and make more pieces of the copy, which it does
    // (77 frames of 61x100 -> 64x96 24.6 -> 19.1 us a call, 500 28.7 -> 23.1, 200
    // of 111x121 -> 96x96, units of 55 rows, 24.9 -> 26.1; patch 14, whose units
    // take longer, 500 of 60x70 -> 56x56 22.5 -> 29.5).
    const auto submissions = [](const Plan& q) {
        return tables_on_host(q) ? copy_pieces(q.bytes) : copy_pieces(q.off_gen) + 1;
    };
    if (no_alloc && plan->items[0].patch == 16 && plan->long_unit_rows <= kCopyLongRows && submissions(*plan) > 1 &&
        plan->off_gen <= kCopyPieces * kCopyPiece) {
        std::shared_ptr<const Plan> longer;
        if (get_plan(PlanKind::kBatchLong, items, n_items, &longer) == VP_OK && submissions(*longer) < submissions(*plan))
            plan = std::move(longer);
    }
    const Plan& p = *plan;
    if (out_rows_capacity < p.total_rows)
        return fail(VP_ERR_CAPACITY, "out_rows holds " + std::to_string(out_rows_capacity) +
                                         " rows, batch needs " + std::to_string(p.total_rows));
    if (no_alloc) {
        if (p.bytes > static_cast<size_t>(vp::kNoAllocPlanBytes))
            return fail(VP_ERR_CAPACITY, "the plan needs " + std::to_string(p.bytes) +
                                             " bytes; the library's fixed plan memory holds " +
                                             std::to_string(vp::kNoAllocPlanBytes));
        const int err = vp::noalloc_plan_memory(&workspace);
        if (err != 0) return hip_fail(static_cast<hipError_t>(err), "hipGetSymbolAddress (plan memory)");
        // (pageable host memory: a copy has read it when hipMemcpyAsync returns)
        const bool host_tables = tables_on_host(p);
        const size_t copied = host_tables ? p.bytes : p.off_gen;
        thread_local std::vector<uint8_t> blob;
        if (blob.size() < copied) blob.resize(copied);
        pack_plan(p, blob.data());
        if (host_tables) {
            std::memset(blob.data() + p.off_gen, 0, p.bytes - p.off_gen);
            fill_tables(p, reinterpret_cast<int32_t*>(blob.data() + p.off_tables));
        }
        auto* const base = static_cast<uint8_t*>(workspace);
        const size_t piece = copied <= kCopyPieces * kCopyPiece ? kCopyPiece : copied;
        for (size_t at = 0; at < copied; at += piece) {
            const hipError_t e = hipMemcpyAsync(base + at, blob.data() + at, std::min(piece, copied - at),
                                                hipMemcpyHostToDevice, stream);
            if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync (plan)");
        }
        if (!host_tables) {
            const int te = vp::launch_upload(nullptr, nullptr, 0, reinterpret_cast<const vp::TableJob*>(base + p.off_jobs),
                                             static_cast<int>(p.jobs.size()),
                                             reinterpret_cast<int32_t*>(base + p.off_tables), stream);
            if (te != 0) return hip_fail(static_cast<hipError_t>(te), "plan tables launch");
        }
    } else {
        if (workspace_bytes < static_cast<int64_t>(p.bytes))
            return fail(VP_ERR_CAPACITY, "workspace holds " + std::to_string(workspace_bytes) +
                                             " bytes, plan needs " + std::to_string(p.bytes));
        st = upload_plan(p, workspace, stream);
        if (st != VP_OK) return st;
    }
    hipEvent_t t_start = g_timing_start, t_stop = g_timing_stop;
    g_timing_start = g_timing_stop = nullptr;
    if (t_start != nullptr) {
        const hipError_t e = hipEventRecord(t_start, stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing start)");
    }
    auto* ws = static_cast<uint8_t*>(workspace);
    vp::PlanView view;
    view.items = reinterpret_cast<const vp::DevItem*>(ws + p.off_items);
    view.tile_prefix = reinterpret_cast<const int32_t*>(ws + p.off_prefix);
    view.indices = reinterpret_cast<const int32_t*>(ws + p.off_indices);
    view.tables = reinterpret_cast<const int32_t*>(ws + p.off_tables);
    view.units = reinterpret_cast<const vp::StreamUnit*>(ws + p.off_units);
    view.wgs = reinterpret_cast<const uint32_t*>(ws + p.off_wgs);
    view.n_items = n_items;
    view.n_tiles = p.prefix[n_items];
    if (patch_only) {
        const int err = vp::launch_patchify(view, out_rows, out_dtype, norm, p.items[0].patch, stream);
        if (err != 0) return hip_fail(static_cast<hipError_t>(err), "patchify kernel launch");
    } else {
        st = run_launches(p, view, out_rows, out_dtype, norm, stream, false, no_alloc);
        if (st != VP_OK) return st;
    }
    if (t_stop != nullptr) {
        const hipError_t e = hipEventRecord(t_stop, stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing stop)");
    }
    if (grid_thw) std::memcpy(grid_thw, p.grid.data(), sizeof(int32_t) * p.grid.size());
    if (cu_seqlens) std::memcpy(cu_seqlens, p.cu.data(), sizeof(int32_t) * p.cu.size());
    g_last_error.clear();
    return VP_OK;
}

// vp_batch_kernels and vp_resize_kernels: a row of six words per launch.
int32_t describe_launches(PlanKind kind, const vp_item* items, int32_t n_items, int32_t* launches,
                          int32_t capacity, int32_t* n_launches) {
    if (n_launches == nullptr) return fail(VP_ERR_NULL, "n_launches is NULL");
    if (capacity < 0 || (launches == nullptr && capacity > 0))
        return fail(VP_ERR_ARG, "launches must hold capacity rows of 6 int32");
    std::shared_ptr<const Plan> plan;
    const int32_t st = get_plan(kind, items, n_items, &plan);
    if (st != VP_OK) return st;
    const Plan& p = *plan;
    std::vector<std::array<int32_t, 6>> rows;
    static_assert(VP_KERNEL_GENERIC == VP_WRITER_TILES);
    if (p.prefix[n_items] > 0) rows.push_back({VP_KERNEL_GENERIC, 0, 0, 0, 0, p.prefix[n_items]});
    for (const vp::StreamLaunch& L : p.launches) {
        if (kind == PlanKind::kResize && L.kx == vp::kRsMmShape)
            rows.push_back({VP_WRITER_MATRIX, 0, 0, 16 * (L.m % vp::kRsMmTwo),
                            vp::resize_mm_cols((L.m & vp::kRsMmWide) != 0), L.count});
        else if (kind == PlanKind::kResize)
            rows.push_back({VP_WRITER_DOT, L.m, L.kx, 0, 0, L.count});
        else if (L.px < 0)
            rows.push_back({VP_KERNEL_XFIRST, L.m, L.kx, 0, vp::xfirst_db(L.px) > 0 ? 2 : 1, L.count});
        else
            rows.push_back({VP_KERNEL_YFIRST, L.m, L.kx, L.px, 0, L.count});
    }
    for (size_t i = 0; i < rows.size() && i < size_t(capacity); ++i)
        std::memcpy(launches + 6 * i, rows[i].data(), sizeof(int32_t) * 6);
    *n_launches = static_cast<int32_t>(rows.size());
    return VP_OK;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================

extern "C" {

int32_t vp_smart_resize_dims(int32_t height, int32_t width, int32_t factor, int64_t min_pixels,
                             int64_t max_pixels, int32_t* out_h, int32_t* out_w) {
    if (out_h == nullptr || out_w == nullptr) return fail(VP_ERR_NULL, "output pointer is NULL");
    if (height <= 0 || width <= 0 || factor <= 0 || max_pixels <= 0 || min_pixels < 0 ||
        min_pixels > max_pixels)
        return fail(VP_ERR_ARG, "smart_resize: sizes, factor and max_pixels must be positive, "
                                "0 <= min_pixels <= max_pixels");
    const double H = height, W = width, F = factor;
    const double ratio = height > width ? H / W : W / H;
    if (ratio > 200.0) return fail(VP_ERR_ASPECT, "smart_resize: aspect ratio above 200");
    int64_t h = static_cast<int64_t>(nearest_even(H / F)) * factor;
    int64_t w = static_cast<int64_t>(nearest_even(W / F)) * factor;
    if (h < factor) h = factor;
    if (w < factor) w = factor;
    if (h * w > max_pixels) {
        const double beta = std::sqrt(static_cast<double>(int64_t(height) * width) /
                                      static_cast<double>(max_pixels));
        h = static_cast<int64_t>(std::floor(H / beta / F)) * factor;
        w = static_cast<int64_t>(std::floor(W / beta / F)) * factor;
        if (h < factor) h = factor;
        if (w < factor) w = factor;
    } else if (h * w < min_pixels) {
        const double beta = std::sqrt(static_cast<double>(min_pixels) /
                                      static_cast<double>(int64_t(height) * width));
        h = static_cast<int64_t>(std::ceil(H * beta / F)) * factor;
        w = static_cast<int64_t>(std::ceil(W * beta / F)) * factor;
    }
    if (h > INT32_MAX || w > INT32_MAX) return fail(VP_ERR_DIMS, "smart_resize: result too large");
    *out_h = static_cast<int32_t>(h);
    *out_w = static_cast<int32_t>(w);
    return VP_OK;
}

int32_t vp_sample_indices(int32_t total_frames, int32_t mode, int32_t nframes, double video_fps,
                          double fps, int32_t min_frames, int32_t max_frames, int32_t* out_idx,
                          int32_t capacity, int32_t* out_count) {
    if (out_count == nullptr) return fail(VP_ERR_NULL, "out_count is NULL");
    if (total_frames < 1) return fail(VP_ERR_FRAMES, "total_frames < 1");
    int64_t n = 0;
    if (mode == VP_SAMPLE_UNIFORM) {
        if (nframes < 1 || nframes > total_frames)
            return fail(VP_ERR_FRAMES, "uniform sampling needs 1 <= nframes <= total_frames");
        n = nframes;
    } else if (mode == VP_SAMPLE_FPS) {
        if (!(video_fps > 0.0) || !(fps > 0.0) || min_frames < 1 || max_frames < min_frames)
            return fail(VP_ERR_ARG, "fps sampling needs video_fps, fps > 0 and "
                                    "1 <= min_frames <= max_frames");
        const double lo = static_cast<double>((int64_t(min_frames) + 1) / 2 * 2);
        const double hi = static_cast<double>(int64_t(max_frames) / 2 * 2);
        double want = static_cast<double>(total_frames) / video_fps * fps;
        want = want < lo ? lo : want;
        want = want > hi ? hi : want;
        want = want > total_frames ? static_cast<double>(total_frames) : want;
        n = static_cast<int64_t>(std::floor(want / 2.0)) * 2;
        if (n < 2) return fail(VP_ERR_FRAMES, "fps sampling yields fewer than 2 frames");
    } else {
        return fail(VP_ERR_ARG, "unknown sampling mode");
    }
    *out_count = static_cast<int32_t>(n);
    if (out_idx == nullptr || capacity < n)
        return fail(VP_ERR_CAPACITY, "index buffer holds " + std::to_string(capacity) + " of " +
                                         std::to_string(n) + " indices");
    for (int64_t i = 0; i < n; ++i) out_idx[i] = spread_index(i, total_frames - 1, n);
    return VP_OK;
}

int32_t vp_filter_taps(int32_t n_in, int32_t n_out, int32_t* max_taps) {
    if (max_taps == nullptr) return fail(VP_ERR_NULL, "max_taps is NULL");
    if (n_in < 1 || n_out < 1) return fail(VP_ERR_ARG, "n_in and n_out must be >= 1");
    *max_taps = axis_taps(n_in, n_out);
    return VP_OK;
}

int32_t vp_filter_table(int32_t n_in, int32_t n_out, int32_t taps, int32_t* start, int32_t* count,
                        float* weights) {
    if (start == nullptr || count == nullptr || weights == nullptr)
        return fail(VP_ERR_NULL, "output pointer is NULL");
    if (n_in < 1 || n_out < 1) return fail(VP_ERR_ARG, "n_in and n_out must be >= 1");
    const int32_t need = axis_taps(n_in, n_out);
    if (taps < need) return fail(VP_ERR_CAPACITY, "taps below the longest window");
    AxisFilter f;
    build_axis(n_in, n_out, taps, &f);
    std::memcpy(start, f.start.data(), sizeof(int32_t) * n_out);
    std::memcpy(count, f.count.data(), sizeof(int32_t) * n_out);
    std::memcpy(weights, f.weight.data(), sizeof(float) * f.weight.size());
    return VP_OK;
}

int32_t vp_filter_table_fixed(int32_t n_in, int32_t n_out, int32_t taps, int32_t* start,
                              int32_t* count, int32_t* q) {
    if (start == nullptr || count == nullptr || q == nullptr)
        return fail(VP_ERR_NULL, "output pointer is NULL");
    if (n_in < 1 || n_out < 1) return fail(VP_ERR_ARG, "n_in and n_out must be >= 1");
    const int32_t need = axis_taps(n_in, n_out);
    if (taps < need) return fail(VP_ERR_CAPACITY, "taps below the longest window");
    AxisFilter f;
    build_axis(n_in, n_out, taps, &f);
    std::memcpy(start, f.start.data(), sizeof(int32_t) * n_out);
    std::memcpy(count, f.count.data(), sizeof(int32_t) * n_out);
    std::memcpy(q, f.fixed.data(), sizeof(int32_t) * f.fixed.size());
    return VP_OK;
}

int32_t vp_batch_layout(const vp_item* items, int32_t n_items, int32_t* grid_thw,
                        int32_t* cu_seqlens, int64_t* total_rows, int64_t* workspace_bytes) {
    std::shared_ptr<const Plan> plan;
    const int32_t st = get_plan(PlanKind::kBatch, items, n_items, &plan);
    if (st != VP_OK) return st;
    const Plan& p = *plan;
    if (grid_thw) std::memcpy(grid_thw, p.grid.data(), sizeof(int32_t) * p.grid.size());
    if (cu_seqlens) std::memcpy(cu_seqlens, p.cu.data(), sizeof(int32_t) * p.cu.size());
    if (total_rows) *total_rows = p.total_rows;
    if (workspace_bytes) *workspace_bytes = static_cast<int64_t>(p.bytes);
    return VP_OK;
}

int32_t vp_patchify_layout(const vp_item* items, int32_t n_items, int64_t* total_rows,
                           int64_t* workspace_bytes) {
    std::shared_ptr<const Plan> plan;
    const int32_t st = get_plan(PlanKind::kPatch, items, n_items, &plan);
    if (st != VP_OK) return st;
    if (total_rows) *total_rows = plan->total_rows;
    if (workspace_bytes) *workspace_bytes = static_cast<int64_t>(plan->bytes);
    return VP_OK;
}

int32_t vp_batch_kernels(const vp_item* items, int32_t n_items, int32_t* launches,
                         int32_t capacity, int32_t* n_launches) {
    return describe_launches(PlanKind::kBatch, items, n_items, launches, capacity, n_launches);
}

int32_t vp_resize_kernels(const vp_item* items, int32_t n_items, int32_t* launches,
                          int32_t capacity, int32_t* n_launches) {
    return describe_launches(PlanKind::kResize, items, n_items, launches, capacity, n_launches);
}

int32_t vp_preprocess_batch(const vp_item* items, int32_t n_items, const float* mean,
                            const float* std, int32_t out_dtype, void* out_rows,
                            int64_t out_rows_capacity, int32_t* grid_thw, int32_t* cu_seqlens,
                            void* workspace, int64_t workspace_bytes, hipStream_t stream) {
    return run_batch(false, items, n_items, mean, std, out_dtype, out_rows, out_rows_capacity,
                     grid_thw, cu_seqlens, workspace, workspace_bytes, stream);
}

int32_t vp_preprocess_batch_noalloc(const vp_item* items, int32_t n_items, const float* mean,
                                    const float* std, int32_t out_dtype, void* out_rows,
                                    int64_t out_rows_capacity, int32_t* grid_thw,
                                    int32_t* cu_seqlens, hipStream_t stream) {
    return run_batch(false, items, n_items, mean, std, out_dtype, out_rows, out_rows_capacity,
                     grid_thw, cu_seqlens, nullptr, 0, stream, true);
}

int32_t vp_patchify_batch(const vp_item* items, int32_t n_items, const float* mean,
                          const float* std, int32_t out_dtype, void* out_rows,
                          int64_t out_rows_capacity, int32_t* grid_thw, int32_t* cu_seqlens,
                          void* workspace, int64_t workspace_bytes, hipStream_t stream) {
    return run_batch(true, items, n_items, mean, std, out_dtype, out_rows, out_rows_capacity,
                     grid_thw, cu_seqlens, workspace, workspace_bytes, stream);
}
int32_t vp_resize_layout(const vp_item* items, int32_t n_items, int64_t* frame_off,
                         int64_t* workspace_bytes) {
    std::shared_ptr<const Plan> plan;
    const int32_t st = get_plan(PlanKind::kResize, items, n_items, &plan);
    if (st != VP_OK) return st;
    const Plan& p = *plan;
    if (frame_off) std::memcpy(frame_off, p.byte_off.data(), sizeof(int64_t) * p.byte_off.size());
    if (workspace_bytes) *workspace_bytes = static_cast<int64_t>(p.bytes);
    g_last_error.clear();
    return VP_OK;
}

int32_t vp_resize_batch(const vp_item* items, int32_t n_items, void* out_frames,
                        int64_t out_capacity, int64_t* frame_off, void* workspace,
                        int64_t workspace_bytes, hipStream_t stream) {
    if (out_frames == nullptr || workspace == nullptr)
        return fail(VP_ERR_NULL, "out_frames and workspace must be non-NULL");
    if (reinterpret_cast<uintptr_t>(out_frames) % 4 != 0)
        return fail(VP_ERR_ARG, "out_frames must be 4-byte aligned");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0)
        return fail(VP_ERR_ARG, "workspace must be 256-byte aligned");
    std::shared_ptr<const Plan> plan;
    int32_t st = get_plan(PlanKind::kResize, items, n_items, &plan);
    if (st != VP_OK) return st;
    const Plan& p = *plan;
    if (out_capacity < p.byte_off[n_items])
        return fail(VP_ERR_CAPACITY, "out_frames holds " + std::to_string(out_capacity) +
                                         " bytes, batch needs " + std::to_string(p.byte_off[n_items]));
    if (workspace_bytes < static_cast<int64_t>(p.bytes))
        return fail(VP_ERR_CAPACITY, "workspace holds " + std::to_string(workspace_bytes) +
                                         " bytes, plan needs " + std::to_string(p.bytes));
    st = upload_plan(p, workspace, stream);
    if (st != VP_OK) return st;
    hipEvent_t t_start = g_timing_start, t_stop = g_timing_stop;
    g_timing_start = g_timing_stop = nullptr;
    if (t_start != nullptr) {
        const hipError_t e = hipEventRecord(t_start, stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing start)");
    }
    auto* ws = static_cast<uint8_t*>(workspace);
    vp::PlanView view{};
    view.items = reinterpret_cast<const vp::DevItem*>(ws + p.off_items);
    view.tile_prefix = reinterpret_cast<const int32_t*>(ws + p.off_prefix);
    view.indices = reinterpret_cast<const int32_t*>(ws + p.off_indices);
    view.tables = reinterpret_cast<const int32_t*>(ws + p.off_tables);
    view.units = reinterpret_cast<const vp::StreamUnit*>(ws + p.off_units);
    view.wgs = reinterpret_cast<const uint32_t*>(ws + p.off_wgs);
    view.n_items = n_items;
    view.n_tiles = p.prefix[n_items];
    st = run_launches(p, view, out_frames, 0, vp::Norm{}, stream, true);
    if (st != VP_OK) return st;
    if (t_stop != nullptr) {
        const hipError_t e = hipEventRecord(t_stop, stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing stop)");
    }
    if (frame_off) std::memcpy(frame_off, p.byte_off.data(), sizeof(int64_t) * p.byte_off.size());
    g_last_error.clear();
    return VP_OK;
}

int32_t vp_position_ids(const vp_item* items, int32_t n_items, int32_t* vit_pos,
                        int32_t* llm_pos, int64_t rows_capacity, int32_t* vit_cu,
                        int32_t vit_cu_capacity, int32_t* n_slices, void* workspace,
                        int64_t workspace_bytes, hipStream_t stream) {
    if (workspace == nullptr) return fail(VP_ERR_NULL, "workspace must be non-NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0)
        return fail(VP_ERR_ARG, "workspace must be 256-byte aligned");
    if (reinterpret_cast<uintptr_t>(vit_pos) % 4 != 0 || reinterpret_cast<uintptr_t>(llm_pos) % 4 != 0)
        return fail(VP_ERR_ARG, "vit_pos and llm_pos must be 4-byte aligned");
    std::shared_ptr<const Plan> plan;
    int32_t st = get_plan(PlanKind::kRows, items, n_items, &plan);
    if (st != VP_OK) return st;
    const Plan& p = *plan;
    if ((vit_pos != nullptr || llm_pos != nullptr) && rows_capacity < p.total_rows)
        return fail(VP_ERR_CAPACITY, "position tables hold " + std::to_string(rows_capacity) +
                                         " rows, batch needs " + std::to_string(p.total_rows));
    int64_t slices = 0;
    for (int32_t b = 0; b < n_items; ++b) slices += p.items[b].t;
    if (vit_cu != nullptr && vit_cu_capacity < slices + 1)
        return fail(VP_ERR_CAPACITY, "vit_cu holds " + std::to_string(vit_cu_capacity) +
                                         " entries, batch needs " + std::to_string(slices + 1));
    if (workspace_bytes < static_cast<int64_t>(p.bytes))
        return fail(VP_ERR_CAPACITY, "workspace holds " + std::to_string(workspace_bytes) +
                                         " bytes, plan needs " + std::to_string(p.bytes));
    hipEvent_t t_start = g_timing_start, t_stop = g_timing_stop;
    g_timing_start = g_timing_stop = nullptr;
    if (vit_pos != nullptr || llm_pos != nullptr) {
        st = upload_plan(p, workspace, stream);
        if (st != VP_OK) return st;
        if (t_start != nullptr) {
            const hipError_t e = hipEventRecord(t_start, stream);
            if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing start)");
        }
        auto* ws = static_cast<uint8_t*>(workspace);
        vp::PlanView view{};
        view.items = reinterpret_cast<const vp::DevItem*>(ws + p.off_items);
        view.tile_prefix = reinterpret_cast<const int32_t*>(ws + p.off_prefix);
        view.indices = reinterpret_cast<const int32_t*>(ws + p.off_indices);
        view.n_items = n_items;
        view.n_tiles = 0;
        const int err = vp::launch_positions(view, vit_pos, llm_pos, p.total_rows, stream);
        if (err != 0) return hip_fail(static_cast<hipError_t>(err), "position kernel launch");
        if (t_stop != nullptr) {
            const hipError_t e = hipEventRecord(t_stop, stream);
            if (e != hipSuccess) return hip_fail(e, "hipEventRecord (timing stop)");
        }
    }
    if (vit_cu != nullptr) {
        int64_t s = 0;
        vit_cu[0] = 0;
        for (int32_t b = 0; b < n_items; ++b)
            for (int32_t k = 0; k < p.items[b].t; ++k, ++s)
                vit_cu[s + 1] = vit_cu[s] + p.grid[3 * b + 1] * p.grid[3 * b + 2];
    }
    if (n_slices) *n_slices = static_cast<int32_t>(slices);
    g_last_error.clear();
    return VP_OK;
}

const char* vp_status_string(int32_t status) {
    switch (status) {
        case VP_OK: return "VP_OK";
        case VP_ERR_NULL: return "VP_ERR_NULL";
        case VP_ERR_ARG: return "VP_ERR_ARG";
        case VP_ERR_ASPECT: return "VP_ERR_ASPECT";
        case VP_ERR_DIMS: return "VP_ERR_DIMS";
        case VP_ERR_INDEX: return "VP_ERR_INDEX";
        case VP_ERR_FRAMES: return "VP_ERR_FRAMES";
        case VP_ERR_CAPACITY: return "VP_ERR_CAPACITY";
        case VP_ERR_HIP: return "VP_ERR_HIP";
        default: return "VP_ERR_UNKNOWN";
    }
}

int32_t vp_set_kernel_events(hipEvent_t start, hipEvent_t stop) {
    if ((start == nullptr) != (stop == nullptr))
        return fail(VP_ERR_NULL, "vp_set_kernel_events needs both events or neither");
    g_timing_start = start;
    g_timing_stop = stop;
    g_last_error.clear();
    return VP_OK;
}

const char* vp_last_error_message(void) { return g_last_error.c_str(); }

}  // extern "C"
