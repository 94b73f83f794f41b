// zf_plan: per-chunk work units with device-specific tile shapes (Sec. 4),
// batches no larger than a staging slot, Johnson's order over the batches'
// (transfer, decode) estimates (Sec. 3.3), and the device workspace.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "plan.hpp"
#include "tune.hpp"

namespace zf {

// Output-balanced Group-Parallel units over n elements whose ng groups start
// at gof(g): about `unit` outputs each, cut at a group boundary when one is
// near, so a unit rarely rescans a group.  Tile {chunk, first group, first
// element, end element}.
template <class GroupOffset>
static void gp_tiles(std::vector<Tile> &T, uint32_t idx, uint32_t ng, uint32_t n, uint32_t unit,
                     GroupOffset gof) {
    uint32_t e = 0, g = 0;
    while (e < n) {
        while (g + 1 < ng && gof(g + 1) <= e) g++;
        const uint64_t target = uint64_t(e) + unit;
        uint32_t e_end;
        if (target >= n) {
            e_end = n;
        } else {
            uint32_t gb = g + 1;
            while (gb < ng && gof(gb) < target) gb++;
            e_end = (gb < ng && gof(gb) <= target + unit) ? gof(gb) : uint32_t(target);
        }
        T.push_back({idx, g, e, e_end});
        e = e_end;
    }
}

// The 16-byte entry records of a column token dictionary (host validated:
// every entry of 1..64 bytes lies inside the entry bytes): an entry's first
// 15 bytes, zero past its length, then its length, so that one aligned
// 16-byte read gives a token of up to 15 bytes and its length.
static void fat_records(const zf_column &col, std::vector<uint8_t> &out) {
    const uint8_t *d = col.buf.p + col.view.dict_off;
    const uint32_t ne = col.view.dict_count;
    const uint8_t *bytes = d + 16 + 4ull * ne;
    const size_t at = out.size();
    out.resize(at + uint64_t(kFatBytes) * ne, 0);
    for (uint32_t k = 0; k < ne; k++) {
        const uint32_t e = rd32(d + 16 + 4ull * k), len = e >> 24, off = e & 0xFFFFFFu;
        uint8_t *r = out.data() + at + uint64_t(kFatBytes) * k;
        std::memcpy(r, bytes + off, std::min(len, kFatInline));
        r[kFatInline] = uint8_t(len);
    }
}

static void add_chunk(WorkTables &w, const zf_column &col, uint32_t ci, uint32_t col_idx,
                      uint64_t comp_off, uint64_t dict_off, const TileShape &ts, uint64_t fat_off = 0) {
    const ChunkInfo &c = col.view.chunks[ci];
    ChunkDesc d{};
    d.comp_off = comp_off;
    d.out_off = c.plain_off;
    d.dict_off = dict_off;
    d.comp_len = c.comp_len;
    d.n_elems = c.n_elems;
    d.dict_count = col.view.dict_count;
    d.dict_bytes = col.view.dict_bytes;
    d.col = uint16_t(col_idx);
    d.codec = c.codec;
    d.dtype = uint8_t(col.view.dtype);
    const bool col_dict = c.codec == C_SDICT_COL || c.codec == C_SDICT_COL_ANS;
    d.fat_off = col_dict ? fat_off : 0;
    if (c.codec == C_SDICT_ANS || c.codec == C_SDICT_COL_ANS) {
        // first stage: ANS-decode the packed entry indices into the scratch
        // area; the String-dictionary stage reads them from there
        const uint8_t *s = col.buf.p + c.comp_off;
        const uint32_t nt = rd32(s), wd = rd32(s + (col_dict ? 4 : 8)), co = rd32(s + (col_dict ? 12 : 24));
        const uint64_t ncb = 4 * ((uint64_t(nt) * wd + 31) / 32);
        d.aux_off = w.scratch_bytes;
        if (ncb) {
            // one ANS unit per piece (the host checked the piece table)
            const uint32_t np = rd32(s + co);
            const uint64_t base = co + 4 + 4ull * np;
            uint64_t prev = 0;
            for (uint32_t k = 0; k < np; k++) {
                const uint64_t end = rd32(s + co + 4 + 4ull * k);
                ChunkDesc a = d;
                a.comp_off = comp_off + base + prev;
                a.comp_len = uint32_t(kAnsHdr + 2ull * rd32(s + base + prev + 4));  // without padding
                a.n_elems = uint32_t(std::min<uint64_t>(kSdAnsPiece, ncb - uint64_t(k) * kSdAnsPiece));
                a.out_off = d.aux_off + uint64_t(k) * kSdAnsPiece;
                a.col = uint16_t(kScratchCol);
                a.codec = C_ANS;
                a.dtype = D_BYTES;
                a.aux_off = 0;
                w.tiles[K_ANS].push_back({uint32_t(w.chunks.size()), 0, 0, 0});
                w.chunks.push_back(a);
                prev = end;
            }
            w.scratch_bytes = align_up(d.aux_off + ncb, 256);
        }
    }
    if (c.codec == C_DSTREE) {
        // first stage: the run starts S (R values) into the scratch area, as
        // units of the RLE kind of the column's width; the second stage
        // (kind TREE, launched after the RLE kinds) reads them there
        const uint8_t *s = col.buf.p + c.comp_off;
        const uint32_t R = rd32(s), ngA = rd32(s + 12);
        const uint32_t es = col.view.dtype == D_I32 ? 4 : 8;
        const Kind ks = col.view.dtype == D_I32 ? K_RLE32 : K_RLE64;
        d.aux_off = w.scratch_bytes;
        ChunkDesc a = d;
        a.out_off = d.aux_off;
        a.n_elems = R;
        a.col = uint16_t(kScratchCol);
        a.codec = C_DSTREE_STARTS;
        const uint32_t aidx = uint32_t(w.chunks.size());
        w.chunks.push_back(a);
        gp_tiles(w.tiles[ks], aidx, ngA, R, ts.unit[ks], [&](uint32_t g) { return rd32(s + 32 + 32ull * g); });
        w.scratch_bytes = align_up(d.aux_off + uint64_t(R) * es, 256);
    }
    const uint32_t idx = uint32_t(w.chunks.size());
    w.chunks.push_back(d);
    const Kind k = kind_of(c.codec, col.view.dtype);
    std::vector<Tile> &T = w.tiles[k];
    const uint32_t unit = scheduled_unit(k, c.sched, ts.unit[k]);
    switch (k) {
    case K_PLAIN:
        for (uint64_t a = 0; a < c.plain_len; a += unit)
            T.push_back({idx, uint32_t(a), uint32_t(std::min<uint64_t>(c.plain_len, a + unit)), 0});
        break;
    case K_FOR32:
    case K_FOR64:
    case K_DICT32:
    case K_DICT64:
    case K_DICT128:
    case K_F2I: {
        const uint32_t nb = (c.n_elems + kForBlock - 1) / kForBlock;
        for (uint32_t b = 0; b < nb; b += unit) T.push_back({idx, b, std::min(unit, nb - b), 0});
        break;
    }
    case K_RLE32:
    case K_RLE64: {
        const uint8_t *s = col.buf.p + c.comp_off;
        gp_tiles(T, idx, rd32(s + 4), c.n_elems, unit, [&](uint32_t g) { return rd32(s + 16 + 32ull * g); });
        break;
    }
    case K_TREE: {
        const uint8_t *s = col.buf.p + c.comp_off;
        const uint32_t b_off = rd32(s + 24);
        gp_tiles(T, idx, rd32(s + 4), c.n_elems, unit, [&](uint32_t g) { return rd32(s + b_off + 16ull * g); });
        break;
    }
    case K_SDICT: {
        // whole groups of 64 tokens, about `unit` output bytes per unit
        const uint8_t *s = col.buf.p + c.comp_off;
        const uint32_t ng = rd32(s + (col_dict ? 8 : 12)), n = c.plain_len, go = col_dict ? 16 : 32;
        auto gof = [&](uint32_t g) { return g < ng ? rd32(s + go + 4ull * g) : n; };
        for (uint32_t g = 0; g < ng;) {
            uint32_t gb = g + 1;
            while (gb < ng && gof(gb) - gof(g) < unit && gb - g < 63) gb++;  // at most 63 groups per unit
            T.push_back({idx, g, gb, 0});
            g = gb;
        }
        break;
    }
    case K_LZ:
    case K_ANS: T.push_back({idx, 0, 0, 0}); break;
    default: break;
    }
    w.plain_bytes += c.plain_len;
    w.comp_bytes += c.comp_len;
    w.t_dec += double(c.plain_len) / (ts.rate_gbps[k] * 1e9);
}

// What a launch holds of each kind, in the measure of the kind's unit: blocks
// of 2048 values (FP), elements (GP), bytes (PLAIN, SDICT), chunks (NP).
struct KindLoad {
    uint64_t n[K_COUNT] = {};
    uint64_t sd_col = 0, sd_col_ans = 0;  // bytes of SDICT_COL and SDICT_COL_ANS chunks
    void add(const zf_column &col, uint32_t ci) {
        const ChunkInfo &c = col.view.chunks[ci];
        const Kind k = kind_of(c.codec, col.view.dtype);
        switch (k) {
        case K_PLAIN:
        case K_SDICT:
            n[k] += c.plain_len;
            if (c.codec == C_SDICT_COL) sd_col += c.plain_len;
            if (c.codec == C_SDICT_COL_ANS) sd_col_ans += c.plain_len;
            break;
        case K_RLE32:
        case K_RLE64: n[k] += c.n_elems; break;
        case K_TREE:
            n[k] += c.n_elems;
            n[col.view.dtype == D_I32 ? K_RLE32 : K_RLE64] += rd32(col.buf.p + c.comp_off);  // the run starts
            break;
        case K_LZ:
        case K_ANS: n[k] += 1; break;
        default: n[k] += (c.n_elems + kForBlock - 1) / kForBlock;
        }
    }
};

// The tile shape of one launch.  The tune cache holds the shapes that were
// fastest on gigabytes; what a launch of less takes is the time of one unit as
// long as its units do not fill the GPU, so a kind's unit shrinks until the
// launch has 8,192 of them or more (32 waves on each of 256 compute units; 4,096
// for the group-parallel kinds, whose units begin with a longer prologue), and
// a workgroup holds no more waves than leaves two workgroups per compute unit (one,
// where a wave takes a whole chunk).
// Shapes the caller set stay.  Units of 256 elements, 1,024 bytes of tokens,
// one block and 8 KiB of plain copy are the smallest: smaller ones were no
// faster.  The DSTREE output, which the cache does not hold, takes units of at
// most 512 (30 M int64 keys 47 us, 51 with 1,024 and 56 with 4,096; 33.6 M int32
// 35, 36 and 44 us).  Measured,
// with the cache's shape and this rule's:
//   String-dictionary, 1.5 MB 81 -> 10.5 us, 16 MiB 83 -> 20, 64 MiB 86 -> 46
//   DSTREE output, 3 M keys 25 -> 10 us; RLE32, 300,000 dates 10.2 -> 7.0
//   Float2Int, 300,000 doubles 36 -> 12.4 us; DICT128, 300,000 16.4 -> 13.6
// The String-dictionary workgroups of 14 and 16 waves, which first fill an
// LDS copy of a column dictionary's hottest records, pay for many bytes over
// column dictionaries: those of 4 waves read faster while the entry indices
// come from the last-level cache (256 MB), slower from memory.  Behind ANS, which
// has just written them, the line is 832 MiB: whole decodes with 4 and 16 waves,
// two texts, 640 MiB 477 and 534, 443 and 477 us; 768 MiB 595 and 592, 532 and 564;
// 896 MiB 714 and 698, 642 and 628; 1 GiB 815 and 771, 747 and 712.  Without ANS
// it is 512 MiB, where first passes gain what repeated ones lose: first passes of
// 128 MiB 92 and 133 us, 256 172 and 165, 512 327 and 299, 768 482 and 440, 1,024
// 635 and 577; the same decoded again 74 and 132, 134 and 158, 266 and 291, 382
// and 428, 634 and 579.  Chunks with their own dictionary have a launch of their
// own beside those and do not count (1 GiB of them 1,113 us when they did, 1,059).
constexpr uint64_t kSdHotCol = 512ull << 20, kSdHotColAns = 832ull << 20;
static uint64_t pow2_floor(uint64_t x) { return x ? uint64_t(1) << (63 - __builtin_clzll(x)) : 0; }
static TileShape fit_tiles(TileShape t, const zf_plan_opts &o, const KindLoad &L, uint32_t cus) {
    for (uint32_t k = 0; k < K_COUNT; k++) {
        if (k == K_LZ || k == K_ANS) {  // (a unit is a whole chunk; LZ77's `unit` is its copy step's block)
            // (one wave a workgroup rather than some part of the cache's: 1,024 LZ77 chunks of
            // 10,000 bytes 47.6 us with one, 50.7 with two, 47.4 with four; 2,560 of 64
            // KiB 473, 472 and 477)
            if (!o.tiles[k].waves_per_block && L.n[k] < 2ull * cus * t.wpb[k]) t.wpb[k] = 1;
            continue;
        }
        const bool sd = k == K_SDICT, gp = k == K_RLE32 || k == K_RLE64 || k == K_TREE;
        const bool hot = sd && t.wpb[k] >= 14;
        if (hot && !o.tiles[k].waves_per_block &&
            double(L.sd_col) / kSdHotCol + double(L.sd_col_ans) / kSdHotColAns < 1.0) {
            t.wpb[k] = 4;
            if (!o.tiles[k].unit) t.unit[k] = std::min(t.unit[k], 16384u);
        }
        if (!o.tiles[k].unit) {
            if (k == K_TREE) t.unit[k] = std::min(t.unit[k], 512u);
            const uint32_t least = k == K_PLAIN ? 8192u : sd ? 1024u : gp ? 256u : 1u;
            uint64_t u = L.n[k] / ((sd || gp ? 16u : 32u) * cus);
            u = pow2_floor(u);  // (as the cache's)
            if (u < t.unit[k]) t.unit[k] = uint32_t(std::clamp<uint64_t>(u, std::min(least, t.unit[k]), t.unit[k]));
        }
        if (!o.tiles[k].waves_per_block && !(sd && t.wpb[k] >= 14))
            t.wpb[k] = uint32_t(std::clamp<uint64_t>(pow2_floor(L.n[k] / t.unit[k] / (2 * cus)), 1, t.wpb[k]));
    }
    return t;
}

// Johnson's rule (Sec. 3.3): batches whose copy is shorter than their decode
// first, by increasing copy time; the rest by decreasing decode time; equal
// keys keep the lower batch index first (stable sorts of ascending indices).
std::vector<uint32_t> johnson(const std::vector<double> &a, const std::vector<double> &b) {
    std::vector<uint32_t> first, rest;
    for (uint32_t i = 0; i < a.size(); i++) (a[i] < b[i] ? first : rest).push_back(i);
    std::stable_sort(first.begin(), first.end(), [&](uint32_t x, uint32_t y) { return a[x] < a[y]; });
    std::stable_sort(rest.begin(), rest.end(), [&](uint32_t x, uint32_t y) { return b[x] > b[y]; });
    first.insert(first.end(), rest.begin(), rest.end());
    return first;
}

std::vector<zf_unit> chunk_units(const zf_column &col, uint32_t ci, const zf_plan_opts &o) {
    ZF_REQUIRE(ci < col.view.n_chunks, ZF_E_INVALID, "chunk %u of %u", ci, col.view.n_chunks);
    WorkTables w;
    add_chunk(w, col, ci, 0, 0, 0, resolve_tiles(o));
    std::vector<zf_unit> u;
    for (uint32_t k = 0; k < K_COUNT; k++)
        for (const Tile &t : w.tiles[k]) u.push_back({k, t.a, t.b, t.c});
    return u;
}

// Size in bytes of a launch's flattened tables.
static uint64_t table_bytes(const WorkTables &w) {
    uint64_t n = align_up(w.chunks.size() * sizeof(ChunkDesc), 256);
    for (int k = 0; k < K_COUNT; k++) n += w.tiles[k].size() * sizeof(Tile);
    return align_up(n, 256);
}

// Output bytes of a whole-chunk unit.
static uint64_t unit_bytes(const ChunkDesc &c) { return uint64_t(c.n_elems) * elem_size(c.dtype); }

// A wave decodes a whole ANS or LZ77 chunk, so a long one taken up last would
// run on alone: the longest first (in chunk order where they are equal).
static void longest_first(WorkTables &w) {
    for (Kind k : {K_LZ, K_ANS}) {
        auto longer = [&](const Tile &a, const Tile &b) {
            return unit_bytes(w.chunks[a.chunk]) > unit_bytes(w.chunks[b.chunk]);
        };
        std::vector<Tile> &T = w.tiles[k];
        if (!std::is_sorted(T.begin(), T.end(), longer)) std::stable_sort(T.begin(), T.end(), longer);
    }
}

// Copy a launch's tables into host staging at `off`; fill its LaunchArgs.
static void flatten(WorkTables &w, std::vector<uint8_t> &host, uint64_t off, uint8_t *d_base,
                    LaunchArgs &A) {
    longest_first(w);
    uint8_t *h = host.data() + off;
    std::memcpy(h, w.chunks.data(), w.chunks.size() * sizeof(ChunkDesc));
    A.chunks = reinterpret_cast<const ChunkDesc *>(d_base + off);
    uint64_t t = align_up(w.chunks.size() * sizeof(ChunkDesc), 256);
    A.tiles = reinterpret_cast<const Tile *>(d_base + off + t);
    uint32_t u = 0;
    for (int k = 0; k < K_COUNT; k++) {
        A.kind_begin[k] = u;
        std::memcpy(h + t + uint64_t(u) * sizeof(Tile), w.tiles[k].data(), w.tiles[k].size() * sizeof(Tile));
        u += uint32_t(w.tiles[k].size());
    }
    A.kind_begin[K_COUNT] = u;
    A.two_stage = w.scratch_bytes > 0;
    A.sdict_codecs = 0;
    for (const Tile &t : w.tiles[K_SDICT]) {
        const uint32_t c = w.chunks[t.chunk].codec;
        A.sdict_codecs |= c == C_SDICT_COL || c == C_SDICT_COL_ANS ? 1u : 2u;
    }
    // (longest first: tile 0 is the largest)
    auto load = [&](Kind k, uint32_t &most) {
        uint64_t sum = 0;
        for (const Tile &t : w.tiles[k]) sum += unit_bytes(w.chunks[t.chunk]);
        most = w.tiles[k].empty() ? 0 : uint32_t(unit_bytes(w.chunks[w.tiles[k][0].chunk]));
        return uint32_t(sum / std::max(1u, most));
    };
    A.lz_load = load(K_LZ, A.lz_bytes);
    A.ans_load = load(K_ANS, A.ans_bytes);
}

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        ZF_HIP(hipGetDevice(&prev));
        if (prev != dev) ZF_HIP(hipSetDevice(dev));
    }
    ~DeviceGuard() {
        int cur = -1;
        if (hipGetDevice(&cur) == hipSuccess && cur != prev && prev >= 0) (void)hipSetDevice(prev);
    }
};

void build_plan(zf_plan_t *P, const zf_column *const *cols, uint32_t n_cols, int device,
                const zf_plan_opts &o) {
    ZF_REQUIRE(cols && n_cols >= 1 && n_cols <= kScratchCol, ZF_E_INVALID,
               "a plan needs 1..%u columns", kScratchCol);
    for (uint32_t c = 0; c < n_cols; c++) ZF_REQUIRE(cols[c], ZF_E_INVALID, "column %u is null", c);
    ZF_REQUIRE(o.n_slots >= 1, ZF_E_INVALID, "n_slots must be >= 1");
    P->device = device;
    P->opts = o;
    P->cols.assign(cols, cols + n_cols);

    const TileShape ts = resolve_tiles(o);

    DeviceGuard dg(device);
    hipDeviceProp_t prop;
    ZF_HIP(hipGetDeviceProperties(&prop, device));
    P->cu_count = uint32_t(prop.multiProcessorCount);
    P->lz_blk = ts.unit[K_LZ];
    P->persistent_waves = o.persistent ? P->cu_count * ts.wpcu : 0;

    // ---- the entry records of every column token dictionary
    std::vector<uint8_t> fat;
    std::vector<uint64_t> fat_at(n_cols, 0);
    for (uint32_t c = 0; c < n_cols; c++)
        if (cols[c]->view.dtype == D_BYTES && cols[c]->view.dict_count) {
            fat_at[c] = fat.size();
            fat_records(*cols[c], fat);
        }

    // ---- image layout and its tables
    WorkTables image;
    P->image_off.resize(n_cols);
    uint64_t at = 0;
    for (uint32_t c = 0; c < n_cols; c++) {
        P->image_off[c] = at;
        at = align_up(at + cols[c]->buf.n, 256);
    }
    P->image_bytes = at;
    KindLoad load;
    for (uint32_t c = 0; c < n_cols; c++)
        for (uint32_t i = 0; i < cols[c]->view.n_chunks; i++) load.add(*cols[c], i);
    const TileShape its = fit_tiles(ts, o, load, P->cu_count);
    std::copy(its.wpb, its.wpb + K_COUNT, image.wpb);
    for (uint32_t c = 0; c < n_cols; c++) {
        const zf_column &col = *cols[c];
        for (uint32_t i = 0; i < col.view.n_chunks; i++)
            add_chunk(image, col, i, c, P->image_off[c] + col.view.chunks[i].comp_off,
                      P->image_off[c] + col.view.dict_off, its, fat_at[c]);
    }
    std::copy(image.wpb, image.wpb + K_COUNT, P->image_wpb);

    // ---- staged mode: dictionaries, then batches of whole chunks
    std::vector<uint64_t> dict_at(n_cols, 0);
    uint64_t dict_total = 0;
    for (uint32_t c = 0; c < n_cols; c++) {
        const zf_column &col = *cols[c];
        if (!col.view.dict_count) continue;
        const uint64_t len = col.view.dict_bytes;
        dict_at[c] = dict_total;
        P->dict_copies.push_back({col.buf.p + col.view.dict_off, dict_total, len});
        dict_total = align_up(dict_total + len, 256);
    }
    P->dict_bytes = dict_total;

    uint64_t slot = o.slot_bytes ? o.slot_bytes : (256ull << 20);
    for (uint32_t c = 0; c < n_cols; c++)
        for (auto &ch : cols[c]->view.chunks) slot = std::max<uint64_t>(slot, align_up(ch.comp_len, 256));
    P->slot_bytes = slot;

    std::vector<Batch> batches;
    Batch cur;
    int64_t range_col = -1;
    uint64_t range_src = 0, range_dst = 0;  // current contiguous copy
    uint32_t range_next_chunk = 0;
    struct Placed {
        uint32_t col, chunk;
        uint64_t dst;
    };
    std::vector<Placed> placed;  // the current batch's chunks
    auto close = [&]() {
        if (!placed.empty()) {
            KindLoad load;
            for (const Placed &p : placed) load.add(*cols[p.col], p.chunk);
            const TileShape bts = fit_tiles(ts, o, load, P->cu_count);
            std::copy(bts.wpb, bts.wpb + K_COUNT, cur.w.wpb);
            for (const Placed &p : placed)
                add_chunk(cur.w, *cols[p.col], p.chunk, p.col, p.dst, dict_at[p.col], bts, fat_at[p.col]);
            batches.push_back(std::move(cur));
        }
        placed.clear();
        cur = Batch{};
        range_col = -1;
    };
    for (uint32_t c = 0; c < n_cols; c++) {
        const zf_column &col = *cols[c];
        for (uint32_t i = 0; i < col.view.n_chunks; i++) {
            const ChunkInfo &ch = col.view.chunks[i];
            const bool extends = range_col == int64_t(c) && range_next_chunk == i;
            uint64_t need = extends ? range_dst + (ch.comp_off + ch.comp_len - range_src)
                                    : align_up(cur.slot_used, 256) + ch.comp_len;
            if (need > slot) {
                close();
                need = ch.comp_len;
            }
            if (!(range_col == int64_t(c) && range_next_chunk == i)) {
                range_col = c;
                range_src = ch.comp_off;
                range_dst = align_up(cur.slot_used, 256);
                cur.copies.push_back({col.buf.p + range_src, range_dst, 0});
            }
            const uint64_t dst = range_dst + (ch.comp_off - range_src);
            cur.copies.back().len = ch.comp_off + ch.comp_len - range_src;
            cur.slot_used = dst + ch.comp_len;
            range_next_chunk = i + 1;
            placed.push_back({c, i, dst});
        }
    }
    close();
    const double pcie = (o.pcie_gbps > 0 ? o.pcie_gbps : 55.0) * 1e9;
    std::vector<double> ta, tb;
    for (uint32_t i = 0; i < batches.size(); i++) {
        Batch &b = batches[i];
        uint64_t bytes = 0;
        for (auto &cp : b.copies) bytes += cp.len;
        b.index = i;
        b.t_h2d = double(bytes) / pcie;
        ta.push_back(b.t_h2d);
        tb.push_back(b.w.t_dec);
    }
    std::vector<uint32_t> order(batches.size());
    std::iota(order.begin(), order.end(), 0u);
    if (o.order == 0) order = johnson(ta, tb);
    for (uint32_t k = 0; k < order.size(); k++) P->batches.push_back(std::move(batches[order[k]]));

    // ---- device memory
    uint64_t tb_total = table_bytes(image);
    for (auto &b : P->batches) tb_total += table_bytes(b.w);
    std::vector<uint8_t> host(tb_total, 0);
    ZF_HIP(hipMalloc(&P->d_tables, std::max<uint64_t>(tb_total, 256)));
    ZF_HIP(hipMalloc(&P->d_out_tab, sizeof(uint8_t *) * kMaxCols));
    // error word, then the persistent queue heads from byte 256 (2 x 8 of
    // them, 128 bytes apart)
    ZF_HIP(hipMalloc(&P->d_err, 256 + 16 * 128));
    ZF_HIP(hipMemset(P->d_err, 0, 256 + 16 * 128));
    uint64_t off = 0;
    flatten(image, host, off, P->d_tables, P->image_args);
    off += table_bytes(image);
    for (auto &b : P->batches) {
        flatten(b.w, host, off, P->d_tables, b.args);
        off += table_bytes(b.w);
    }
    ZF_HIP(hipMemcpy(P->d_tables, host.data(), tb_total, hipMemcpyHostToDevice));

    const int ns = o.n_slots;
    if (!P->batches.empty()) {
        P->d_slots.assign(std::min<size_t>(ns, P->batches.size()), nullptr);
        for (auto &sp : P->d_slots) ZF_HIP(hipMalloc(&sp, align_up(slot, 256)));  // (whole dwords at its end)
    }
    if (dict_total) ZF_HIP(hipMalloc(&P->d_dict, dict_total));
    if (!fat.empty()) {
        ZF_HIP(hipMalloc(&P->d_fat, fat.size()));
        ZF_HIP(hipMemcpy(P->d_fat, fat.data(), fat.size(), hipMemcpyHostToDevice));
    }
    P->scratch_bytes = image.scratch_bytes;
    for (auto &b : P->batches) P->scratch_bytes = std::max(P->scratch_bytes, b.w.scratch_bytes);
    if (P->scratch_bytes) ZF_HIP(hipMalloc(&P->d_scratch, P->scratch_bytes));

    auto fill = [&](LaunchArgs &A) {
        A.out_tab = P->d_out_tab;
        A.scratch = P->d_scratch;
        A.err = P->d_err;
        A.counter = P->d_err + 64;
        A.fat = P->d_fat;
        A.lz_whole = !o.tiles[K_LZ].unit && !o.tiles[K_LZ].waves_per_block;
        A.ans_alone = !o.tiles[K_ANS].waves_per_block;
    };
    fill(P->image_args);
    for (uint32_t k = 0; k < P->batches.size(); k++) {
        Batch &b = P->batches[k];
        b.slot = int(k % P->d_slots.size());
        fill(b.args);
        b.args.comp = P->d_slots[b.slot];
        b.args.dict = P->d_dict;
    }

    // ---- transfers by the copy kernel: the first batch's with the dictionaries
    // (Not in a plan with the persistent kernel, whose workgroups keep every
    // compute unit's LDS until a batch's queues are empty: the next batch's copy,
    // which asks for the whole of one's, would begin as the decode ends.  512 MiB
    // of LZ77 in slots of 128 MiB 6.32 ms by the kernel, 6.12 by commands.)
    std::vector<CopyPiece> pieces;
    bool readable = !P->batches.empty() && !P->persistent_waves;
    std::vector<const uint8_t *> dev_of(n_cols, nullptr);  // a column's bytes as the device reads them
    for (uint32_t c = 0; c < n_cols && readable; c++) {
        hipPointerAttribute_t at{};
        readable = cols[c]->buf.pinned && hipPointerGetAttributes(&at, cols[c]->buf.p) == hipSuccess &&
                   at.type == hipMemoryTypeHost && at.device == device && at.devicePointer;
        dev_of[c] = static_cast<const uint8_t *>(at.devicePointer);
    }
    if (readable) {
        auto device_view = [&](const uint8_t *src) {
            for (uint32_t c = 0; c < n_cols; c++)
                if (src >= cols[c]->buf.p && src < cols[c]->buf.p + cols[c]->buf.n)
                    return dev_of[c] + (src - cols[c]->buf.p);
            fail(ZF_E_INVALID, "a copy outside the plan's columns");
        };
        for (uint32_t k = 0; k < P->batches.size(); k++) {
            Batch &b = P->batches[k];
            uint64_t total = 0, ranges = b.copies.size() + (k ? 0 : P->dict_copies.size());
            for (auto &cp : b.copies) total += cp.len;
            if (!k)
                for (auto &cp : P->dict_copies) total += cp.len;
            // Ranges this long are left to copy commands: their cost no longer
            // counts, and a copy engine waits for no compute unit.  The table,
            // from short ranges to long, kernel and commands: 500,009 rows 491
            // and 666 us; 4,000,000 3.31 and 3.53 ms; 12,000,000 (ranges of
            // about 20 MiB) 9.25 and 9.35 ms; 30,000,000 (50 MiB) 22.67 and
            // 22.69 ms; 45,450,000 (75 MiB) 34.58 and 34.43 ms.  (Where decodes
            // keep LDS busy the kernel waits for some: one LZ77 column of 256
            // MiB in slots of 32 MiB 2.82 and 2.75 ms.)
            if (total >= ranges * kCopyRange) continue;
            // 64 pieces or more, of 16 to 256 KiB
            const uint64_t len = std::clamp<uint64_t>(align_up(total / 64, 16384), 16384, 262144);
            b.piece0 = uint32_t(pieces.size());
            auto cut = [&](const CopyOp &cp, uint8_t *base) {
                const uint8_t *src = cp.len ? device_view(cp.src) : nullptr;
                for (uint64_t a = 0; a < cp.len; a += len)
                    pieces.push_back({src + a, base + cp.dst_off + a, std::min(len, cp.len - a)});
            };
            if (!k)
                for (auto &cp : P->dict_copies) cut(cp, P->d_dict);
            for (auto &cp : b.copies) cut(cp, P->d_slots[b.slot]);
            b.n_pieces = uint32_t(pieces.size()) - b.piece0;
        }
        if (!pieces.empty()) {
            ZF_HIP(hipMalloc(&P->d_pieces, pieces.size() * sizeof(CopyPiece)));
            ZF_HIP(hipMemcpy(P->d_pieces, pieces.data(), pieces.size() * sizeof(CopyPiece), hipMemcpyHostToDevice));
        }
    }

    // ---- streams, events, graphs
    ZF_HIP(hipStreamCreateWithFlags(&P->copy_stream, hipStreamNonBlocking));
    const size_t nsl = P->d_slots.size();
    P->slot_full.resize(nsl);
    P->slot_free.resize(nsl);
    for (size_t s = 0; s < nsl; s++) {
        ZF_HIP(hipEventCreateWithFlags(&P->slot_full[s], hipEventDisableTiming));
        ZF_HIP(hipEventCreateWithFlags(&P->slot_free[s], hipEventDisableTiming));
    }
    auto mk = [&](std::vector<hipEvent_t> &v) {
        v.resize(P->batches.size());
        for (auto &e : v) ZF_HIP(hipEventCreate(&e));
    };
    mk(P->ev_h2d0);
    mk(P->ev_h2d1);
    mk(P->ev_dec0);
    mk(P->ev_dec1);
    ZF_HIP(hipEventCreate(&P->ev_start));
    ZF_HIP(hipEventCreate(&P->ev_end));
    ZF_HIP(hipEventCreateWithFlags(&P->ev_dict, hipEventDisableTiming));
    ZF_HIP(hipEventCreateWithFlags(&P->ev_fork, hipEventDisableTiming));
    ZF_HIP(hipEventCreateWithFlags(&P->ev_join, hipEventDisableTiming));

    // A batch of few launches goes without a graph, whose start costs the host
    // 10 us and the device more than the launches' gaps.  One staged call, one
    // batch of small columns, graph and launches: 1 kind 78 and 60 us, 3 kinds 80
    // and 64 us, 6 kinds 83 and 77 us (but 61 and 77 us a call queued back to
    // back), 13 kinds 131 and 134 us.  A batch whose kinds run beside each other
    // (6 kinds of a 16-column table of 20,011 rows 175 and 158 us) always does.
    auto as_graph = [&](const Batch &b) {
        uint32_t kinds = 0;
        for (uint32_t k = 0; k < K_COUNT; k++) kinds += b.args.kind_begin[k + 1] > b.args.kind_begin[k];
        return o.use_graphs && (P->persistent_waves || (kinds > 5 && !decode_forks(b.args)));
    };
    bool any_graph = false, any_fork = false;
    for (auto &b : P->batches) {
        any_graph |= as_graph(b);
        any_fork |= !as_graph(b) && !P->persistent_waves && decode_forks(b.args);
    }
    if (any_fork) ZF_HIP(hipStreamCreateWithFlags(&P->side_stream, hipStreamNonBlocking));
    if (any_graph) {
        hipStream_t cap;
        ZF_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
        try {
            for (auto &b : P->batches) {
                if (!as_graph(b)) continue;
                ZF_HIP(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal));
                hipError_t le = launch_decode(b.args, P->persistent_waves, b.w.wpb, P->lz_blk, cap);
                hipError_t ce = hipStreamEndCapture(cap, &b.graph);
                ZF_HIP(le);
                ZF_HIP(ce);
                ZF_HIP(hipGraphInstantiate(&b.exec, b.graph, nullptr, nullptr, 0));
            }
        } catch (...) {
            (void)hipStreamDestroy(cap);
            throw;
        }
        ZF_HIP(hipStreamDestroy(cap));
    }
}

void release_plan(zf_plan_t *P) {
    zf_plan_t &p = *P;
    int device = p.device;
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != device) (void)hipSetDevice(device);
    if (p.copy_stream) (void)hipStreamSynchronize(p.copy_stream);
    for (auto &b : p.batches) {
        if (b.exec) (void)hipGraphExecDestroy(b.exec);
        if (b.graph) (void)hipGraphDestroy(b.graph);
    }
    auto kill = [](std::vector<hipEvent_t> &v) {
        for (auto e : v)
            if (e) (void)hipEventDestroy(e);
    };
    kill(p.slot_full);
    kill(p.slot_free);
    kill(p.ev_h2d0);
    kill(p.ev_h2d1);
    kill(p.ev_dec0);
    kill(p.ev_dec1);
    for (auto e : {p.ev_start, p.ev_end, p.ev_dict, p.ev_fork, p.ev_join})
        if (e) (void)hipEventDestroy(e);
    for (uint32_t k = 0; k <= K_COUNT; k++)
        for (auto e : {p.kind_ev.e0[k], p.kind_ev.e1[k]})
            if (e) (void)hipEventDestroy(e);
    if (p.copy_stream) (void)hipStreamDestroy(p.copy_stream);
    if (p.side_stream) (void)hipStreamDestroy(p.side_stream);
    for (auto sp : p.d_slots)
        if (sp) (void)hipFree(sp);
    if (p.d_dict) (void)hipFree(p.d_dict);
    if (p.d_tables) (void)hipFree(p.d_tables);
    if (p.d_out_tab) (void)hipFree(p.d_out_tab);
    if (p.d_scratch) (void)hipFree(p.d_scratch);
    if (p.d_fat) (void)hipFree(p.d_fat);
    if (p.d_pieces) (void)hipFree(p.d_pieces);
    if (p.d_err) (void)hipFree(p.d_err);
    if (prev >= 0 && prev != device) (void)hipSetDevice(prev);
}

}  // namespace zf
