// Builders of the contraction work lists (host bookkeeping).
#include "plans.hpp"

namespace pdmrg {

int GemmList::add_item(int c_slot, int64_t c_off, int M, int N, int ldc) {
    GemmItem it{};
    it.c_off = c_off;
    it.c_slot = c_slot;
    it.M = M;
    it.N = N;
    it.ldc = ldc;
    it.seg0 = (int32_t)segs.size();
    it.nseg = 0;
    it.rmap = -1;
    items.push_back(it);
    blk0.push_back(-1);
    return (int)items.size() - 1;
}

int GemmList::add_stacked_item(int c_slot, int N, const std::vector<RowBlock> &blks) {
    PD_REQUIRE(!blks.empty(), PDMRG_EINVAL, "gemm list: stacked item without blocks");
    GemmItem it{};
    it.c_off = 0;
    it.c_slot = c_slot;
    it.N = N;
    it.ldc = N;
    it.seg0 = (int32_t)segs.size();
    it.nseg = 0;
    it.rmap = (int32_t)rowoff.size();
    blk0.push_back((int32_t)blocks.size());
    int M = 0;
    for (RowBlock b : blks) {
        PD_REQUIRE(b.rows > 0 && b.ldc >= N, PDMRG_EINVAL, "gemm list: bad stacked block");
        b.r0 = M;
        for (int r = 0; r < b.rows; ++r) rowoff.push_back(b.c_off + (int64_t)r * b.ldc);
        blocks.push_back(b);
        M += b.rows;
    }
    blocks.push_back(RowBlock{0, M, 0, 0});   // terminator: r0 = M
    it.M = M;
    items.push_back(it);
    return (int)items.size() - 1;
}

void GemmList::add_seg(int a_slot, int64_t a_off, int lda, int b_slot, int64_t b_off, int ldb, int K) {
    PD_REQUIRE(!items.empty(), PDMRG_EINVAL, "gemm list: segment without item");
    GemmSeg sg{};
    sg.a_off = a_off;
    sg.b_off = b_off;
    sg.a_slot = a_slot;
    sg.b_slot = b_slot;
    sg.K = K;
    sg.lda = lda;
    sg.ldb = ldb;
    segs.push_back(sg);
    GemmItem &it = items.back();
    it.nseg += 1;
    flops += 2.0 * it.M * (double)it.N * K;
}

static int64_t item_k(const GemmList &g, const GemmItem &it) {
    int64_t k = 0;
    for (int j = 0; j < it.nseg; ++j) k += g.segs[it.seg0 + j].K;
    return k;
}

int GemmList::split_parts(int64_t k, double krange) const {
    const int64_t most = elem_bytes == 8 ? kMaxParts64 : 8;
    return (int)std::max<int64_t>(1, std::min<int64_t>({most, std::llround(k / krange), k / 64}));
}

int GemmList::ntiles_for(TileShape t) const {
    const int bm = tile_bm(t), bn = tile_bn(t);
    int n = 0;
    for (const GemmItem &it : items) n += ((it.M + bm - 1) / bm) * ((it.N + bn - 1) / bn);
    return n;
}

double GemmList::operand_bytes() const {
    double b = 0.0;
    for (const GemmItem &it : items) b += (double)elem_bytes * (double)item_k(*this, it) * ((double)it.M + it.N);
    return b;
}

// The quad shapes to compare: as long as the 64 x 64 tiles leave a CU each, those,
// for a larger one only makes the launch longer (BF16x3, 8 x 4 cylinder, m = 33,
// stage 3: 6.4 us with 128 x 64, 4.1 with 64 x 64).
unsigned GemmList::quad_shapes(int parts) const {
    int64_t kmax = 0, n = 0;
    for (const GemmItem &it : items) kmax = std::max(kmax, item_k(*this, it));
    const double krange = std::max(1.0, (double)kmax / std::max(parts, 1));
    for (const GemmItem &it : items)
        n += (int64_t)((it.M + 63) / 64) * ((it.N + 63) / 64) * (parts > 1 ? split_parts(item_k(*this, it), krange) : 1);
    return n <= 256 ? 1u << (int)TileShape::T64x64_Q | 1u << (int)TileShape::T64x64_Q32 : kQuadShapes;
}

// Estimated time of a list under a register-direct (FP64) or quad (FP32, BF16x3)
// shape, in flops of one CU at full rate: the work (dimensions rounded up to the
// tile, register-direct ones to the 32 that a wave's edge tile keeps) spread
// over the chip at the shape's rate, plus the longest tile, which the last CU to
// finish may have started last.
double GemmList::cost(TileShape ts, int parts) const {
    // Relative rates.  Register-direct, 64 x 64, 128 x 64, 64 x 128, 128 x 128: H_eff
    // at m = 4000 with 98 channels, stage 1 6.9, 5.9, 5.5, 5.1 ms, stage 3 9.6, 8.2,
    // 6.6, 5.9.  Quads, 64 x 64, 128 x 64 and the same with K steps of 32: tri 12 x
    // 6, m = 3000, BF16x3 stage 1 (K = 330) 0.415, 0.349, 0.366, 0.359 ms, stage 3 (K =
    // 1100 a part) 0.382, 0.344, 0.335, 0.331, FP32 0.500, 0.488, 0.510, 0.512 and
    // 0.510, 0.514, 0.505, 0.519; the LDS-DMA kernel's best are 0.409, 0.388, 0.527,
    // 0.540.
    static const double kReg[4] = {0.66, 0.77, 0.91, 1.0}, kSplit[4] = {0.86, 0.98, 0.99, 1.02},
                        kF32[4] = {0.97, 1.0, 1.0, 0.98};
    const bool reg = (kR64Shapes >> (int)ts) & 1u, split = !(shapes_allowed & kStagedShapes);
    const double rate = reg ? kReg[(int)ts - (int)TileShape::T64x64_R]
                            : (split ? kSplit : kF32)[(int)ts - (int)TileShape::T64x64_Q];
    // start and end of a tile, in K units (deep steps: half a step of K wasted more)
    const double kTileK = ts == TileShape::T64x64_Q32 || ts == TileShape::T128x64_Q32 ? 80.0 : 48.0;
    const double partial = reg ? 240.0 : split ? 230.0 : 150.0;   // flops in the time of writing and reading a partial sum
    const int bm = tile_bm(ts), bn = tile_bn(ts), rm = reg ? 32 : bm, rn = reg ? 32 : bn;
    int64_t kmax = 0;
    for (const GemmItem &it : items) kmax = std::max(kmax, item_k(*this, it));
    const double krange = std::max(1.0, (double)kmax / std::max(parts, 1));
    double work = 0.0, longest = 0.0;
    for (const GemmItem &it : items) {
        const int64_t k = item_k(*this, it);
        const double ip = split_parts(k, krange);
        work += 2.0 * ((it.M + rm - 1) / rm * rm) * (double)((it.N + rn - 1) / rn * rn) * (k + ip * kTileK);
        if (ip > 1.0) work += partial * it.M * (double)it.N * ip;
        // four times a wave's tile: its SIMD has a quarter of the CU's rate
        longest = std::max(longest, 8.0 * std::min(bm / 2, it.M) * (double)std::min(bn / 2, it.N) * (k / ip + kTileK));
    }
    return (work / 256.0 + longest) / rate;
}

// Past 2 GB of operands (each item's counted once) FP64 lists stream from memory
// and run the register-direct kernel: H_eff at m = 4000, 98 channels, 7.8 GB,
// stage 1 5.9 -> 5.3 ms, stage 3 10.0 -> 6.0.  Below, the staged kernel is kept for
// its order of sums (over ascending k, with the splits it has always had), not for
// speed: an eigensolver stopped early can amplify a change of rounding.  What that
// costs, against the plans that the autotuner takes (which follow their own order
// of sums), us a product: 16-site chain, m = 64, 19.5 / 15.5; 8 x 4 cylinder, m =
// 1024, 168 / 151; 24 x 8, m = 2000, 422 / 410; tri 12 x 6, m = 3000, 2268 / 2001; 98
// channels, m = 500, 131 / 92.
//
// FP32 and BF16x3 take the quad shape of least cost() among quad_shapes().
void GemmList::pick_tile(double bytes) {
    double best = 0.0;
    bool have = false;
    streams = (shapes_allowed & kR64Shapes) && bytes > 2e9;
    const unsigned modelled = streams ? kR64Shapes : elem_bytes == 4 ? shapes_allowed & quad_shapes(1) : 0u;
    if (modelled) {
        for (int t = 0; t < kNumShapes; ++t) {
            if (!((modelled >> t) & 1u)) continue;
            const double c = cost((TileShape)t, 1);
            if (!have || c < best * 0.999) {
                best = c;
                shape = (TileShape)t;
                have = true;
            }
        }
        return;
    }
    // The staged kernel (in FP64 it measured faster than the LDS-DMA one; the
    // autotuner still times both): relative throughput per padded flop of each
    // shape, from timings of the H_eff GEMMs of the 8 x 4 cylinder (m = 1024) on
    // MI355X: shorter K steps (more resident workgroups) win on these short,
    // ragged K loops.
    static const double kRate[] = {1.0, 1.0, 0.8, 0.75, 1.1, 1.15, 1.05, 1.2};
    const unsigned shapes = shapes_allowed & kStagedShapes;
    std::vector<int64_t> kof(items.size());
    for (size_t i = 0; i < items.size(); ++i) kof[i] = item_k(*this, items[i]);
    double caps[4] = {-1.0, -1.0, -1.0, -1.0}, pads[4] = {};
    for (int t = 0; t < (int)TileShape::T128x32_D; ++t) {
        if (!(shapes & (1u << t))) continue;
        const TileShape ts = (TileShape)t;
        const int bm = tile_bm(ts), bn = tile_bn(ts);
        // tiles after the split-K the long items allow, and MFMA work: the same for
        // the depth variants (4, 6 and 5, 7) of 64 x 64 and 128 x 32
        double &cap = caps[t < 4 ? t : t & 1], &padded = pads[t < 4 ? t : t & 1];
        if (cap < 0.0) {
            const int lm = __builtin_ctz(bm), ln = __builtin_ctz(bn);
            cap = padded = 0.0;
            for (size_t i = 0; i < items.size(); ++i) {
                const int tm = (items[i].M + bm - 1) >> lm, tn = (items[i].N + bn - 1) >> ln;
                cap += tm * (double)tn * std::max<int64_t>(1, std::min<int64_t>(8, kof[i] / 256));
                padded += 2.0 * (tm * bm) * (double)(tn * bn) * (double)kof[i];
            }
        }
        const double fill = std::min(1.0, cap / 1024.0);
        const double cost = padded / (kRate[t] * std::max(fill, 1e-3));
        if (!have || cost < best * 0.999) {
            best = cost;
            shape = ts;
            have = true;
        }
    }
}

GemmList GemmList::host_copy() const {
    GemmList g;
    g.ta = ta;
    g.tb = tb;
    g.elem_bytes = elem_bytes;
    g.shape = shape;
    g.shapes_allowed = shapes_allowed;
    g.items = items;
    g.segs = segs;
    g.rowoff = rowoff;
    g.blk0 = blk0;
    g.blocks = blocks;
    g.flops = flops;
    return g;
}

// Launch order of the tiles.  Workgroup b of a launch runs on XCD b % 8 (the
// dispatcher deals workgroups to the 8 XCDs in turn) and tiles[b].  The tiles
// of an item are cut into chunks of consecutive rows, each about 1/128 of
// the launch's work (work = K + a fixed prologue/epilogue cost per tile), so an
// item, or a large item's row range, stays on one XCD and its L2 (the tiles
// of a row share the A panel, the rows of an item the B panel).  Chunks are
// dealt to XCDs largest first, each to the XCD of least work so far, then
// every XCD's list runs largest chunk first and the lists are interleaved;
// shorter lists are padded with idle tiles (item = -1).
static std::vector<GemmTile> place_tiles(const std::vector<GemmItem> &items, const std::vector<int64_t> &kof,
                                         int bm, int bn) {
    constexpr int kXcd = 8, kChunksPerXcd = 16;
    constexpr double kTileCost = 64.0;   // prologue + epilogue, in K units
    double total = 0.0;
    for (size_t i = 0; i < items.size(); ++i)
        if (items[i].M > 0 && items[i].N > 0)
            total += ((items[i].M + bm - 1) / bm) * (double)((items[i].N + bn - 1) / bn) * ((double)kof[i] + kTileCost);
    const double target = total / (kXcd * kChunksPerXcd);
    struct Chunk { int item, m_begin, m_end; double cost; };
    std::vector<Chunk> chunks;
    for (size_t i = 0; i < items.size(); ++i) {
        const GemmItem &it = items[i];
        if (it.M <= 0 || it.N <= 0) continue;
        const double row_cost = ((it.N + bn - 1) / bn) * ((double)kof[i] + kTileCost);
        Chunk c{(int)i, 0, 0, 0.0};
        for (int m0 = 0; m0 < it.M; m0 += bm) {
            c.m_end = std::min(m0 + bm, it.M);
            c.cost += row_cost;
            if (c.cost >= target) {
                chunks.push_back(c);
                c = Chunk{(int)i, c.m_end, c.m_end, 0.0};
            }
        }
        if (c.m_end > c.m_begin) chunks.push_back(c);
    }
    std::stable_sort(chunks.begin(), chunks.end(), [](const Chunk &a, const Chunk &b) { return a.cost > b.cost; });
    std::vector<std::vector<GemmTile>> lists(kXcd);
    double load[kXcd] = {};
    for (const Chunk &c : chunks) {
        const int x = (int)(std::min_element(load, load + kXcd) - load);
        load[x] += c.cost;
        for (int m0 = c.m_begin; m0 < c.m_end; m0 += bm)
            for (int n0 = 0; n0 < items[c.item].N; n0 += bn) lists[x].push_back(GemmTile{c.item, m0, n0, 0});
    }
    size_t len = 0;
    for (const auto &l : lists) len = std::max(len, l.size());
    std::vector<GemmTile> out(len * kXcd, GemmTile{-1, 0, 0, 0});
    for (int x = 0; x < kXcd; ++x)
        for (size_t j = 0; j < lists[x].size(); ++j) out[j * kXcd + x] = lists[x][j];
    return out;
}

void GemmList::finish(hipStream_t s) {
    build_tiles();
    ListStage st;
    stage(st);
    st.flush(d_lists, s);
}

void GemmList::stage(ListStage &st) {
    if (ftiles.empty()) {
        st.add(dev.items, items);
        st.add(dev.segs, segs);
        st.add(dev.tiles, tiles);
    } else {
        st.add(dev.ftiles, ftiles);
    }
    st.add(dev.rowoff, rowoff);
    if (epi_items.empty()) return;
    st.add(dev.epi.items, epi_items);
    st.add(dev.epi.row, epi_row);
    st.add(dev.epi.col, epi_col);
    st.add(dev.epi.dst, epi_dst);
}

void GemmList::build_tiles() {
    if (!(shapes_allowed & (1u << (int)shape)))
        shape = (shapes_allowed & (1u << (int)TileShape::T64x64)) ? TileShape::T64x64 : TileShape::T64x64_D;
    const int bm = tile_bm(shape), bn = tile_bn(shape);
    std::vector<int64_t> kof(items.size());
    ntiles_real = 0;
    for (size_t i = 0; i < items.size(); ++i) {
        kof[i] = item_k(*this, items[i]);
        if (items[i].M > 0 && items[i].N > 0)
            ntiles_real += ((items[i].M + bm - 1) / bm) * ((items[i].N + bn - 1) / bn);
    }
    tiles = place_tiles(items, kof, bm, bn);
    check_grid((int64_t)tiles.size(), 256, "gemm");
    PD_REQUIRE(std::count_if(tiles.begin(), tiles.end(), [](const GemmTile &t) { return t.item >= 0; }) ==
                   ntiles_real, PDMRG_ESHAPE, "gemm: tile placement lost tiles");
    if (!epi_items.empty())
        for (GemmTile &t : tiles) {
            if (t.item < 0) continue;
            const int32_t *r = epi_row.data() + epi_items[t.item].row0;
            while (r[t.chan + 1] <= t.m0) ++t.chan;
        }
    ftiles.clear();
    bool single = !ta && !tb;
    for (const GemmItem &it : items) single = single && it.nseg <= 1;
    if (!single || !(((kDmaShapes | kR64Shapes | kQuadShapes) >> (int)shape) & 1u)) return;
    ftiles.reserve(tiles.size());
    for (const GemmTile &t : tiles) {
        FlatTile f{};
        if (t.item >= 0) {
            const GemmItem &it = items[t.item];
            f.c_off = it.c_off;
            f.c_slot = f.a_slot = f.b_slot = it.c_slot;
            f.rmap = it.rmap;
            f.M = it.M;
            f.N = it.N;
            f.ldc = it.ldc;
            f.m0 = t.m0;
            f.n0 = t.n0;
            if (it.nseg == 1) {
                const GemmSeg &sg = segs[it.seg0];
                f.a_off = sg.a_off;
                f.b_off = sg.b_off;
                f.a_slot = sg.a_slot;
                f.b_slot = sg.b_slot;
                f.K = std::max(sg.K, 0);
                f.lda = sg.lda;
                f.ldb = sg.ldb;
            }
            if (!epi_items.empty()) {
                const EpiItem &ei = epi_items[t.item];
                f.erow = ei.row0 + t.chan;
                f.ecol = ei.col0;
                f.edst = ei.dst0 + t.chan * ei.nseg;
                f.eseg = ei.nseg;
            }
        }
        ftiles.push_back(f);
    }
}

static void check_span(const std::vector<int64_t> &slot_elems, int slot, int64_t off, int rows, int cols,
                       int64_t ld, const char *what) {
    if (rows <= 0 || cols <= 0) return;
    PD_REQUIRE(slot >= 0 && slot < (int)slot_elems.size(), PDMRG_ESHAPE, std::string(what) + ": bad slot");
    PD_REQUIRE(ld >= cols, PDMRG_ESHAPE, std::string(what) + ": leading dimension below width");
    const int64_t last = off + (int64_t)(rows - 1) * ld + (cols - 1);
    PD_REQUIRE(off >= 0 && last < slot_elems[slot], PDMRG_ESHAPE,
               std::string(what) + ": work list reaches outside its buffer");
}

void GemmList::validate(const std::vector<int64_t> &slot_elems) const {
    for (const GemmItem &it : items) {
        if (it.rmap >= 0) {
            PD_REQUIRE(it.rmap + (int64_t)it.M <= (int64_t)rowoff.size(), PDMRG_ESHAPE, "gemm C: row map too short");
            for (int r = 0; r < it.M; ++r)
                check_span(slot_elems, it.c_slot, it.c_off + rowoff[it.rmap + r], 1, it.N, it.N, "gemm C row");
        } else {
            check_span(slot_elems, it.c_slot, it.c_off, it.M, it.N, it.ldc, "gemm C");
        }
        // buffer-load descriptors address one segment operand with 32-bit byte offsets
        for (int k = 0; k < it.nseg; ++k) {
            const GemmSeg &sg = segs[it.seg0 + k];
            const int64_t span_a = ta ? (int64_t)sg.K * sg.lda : (int64_t)it.M * sg.lda;
            const int64_t span_b = tb ? (int64_t)it.N * sg.ldb : (int64_t)sg.K * sg.ldb;
            PD_REQUIRE(span_a * elem_bytes < ((int64_t)1 << 31) && span_b * elem_bytes < ((int64_t)1 << 31),
                       PDMRG_ESHAPE,
                       "gemm: operand block exceeds 2 GiB");
        }
        for (int k = 0; k < it.nseg; ++k) {
            const GemmSeg &sg = segs[it.seg0 + k];
            if (ta) check_span(slot_elems, sg.a_slot, sg.a_off, sg.K, it.M, sg.lda, "gemm A^T");
            else check_span(slot_elems, sg.a_slot, sg.a_off, it.M, sg.K, sg.lda, "gemm A");
            if (tb) check_span(slot_elems, sg.b_slot, sg.b_off, it.N, sg.K, sg.ldb, "gemm B^T");
            else check_span(slot_elems, sg.b_slot, sg.b_off, sg.K, it.N, sg.ldb, "gemm B");
        }
    }
}

void LcList::validate(const std::vector<int64_t> &slot_elems) const {
    for (const LcTask &t : tasks) {
        PD_REQUIRE((int64_t)t.rows * t.cols < ((int64_t)1 << 31), PDMRG_ESHAPE, "W stage: block too large");
        // the kernel forms row * ld + col in 32 bits
        PD_REQUIRE(t.rows == 0 || (int64_t)(t.rows - 1) * t.ld + t.cols < ((int64_t)1 << 32), PDMRG_ESHAPE,
                   "W stage: block span too large");
        for (int j = 0; j < t.nsrc; ++j)
            PD_REQUIRE(t.rows == 0 || (int64_t)(t.rows - 1) * srcs[t.src0 + j].ld + t.cols < ((int64_t)1 << 32),
                       PDMRG_ESHAPE, "W stage: source span too large");
        check_span(slot_elems, t.dst_slot, t.dst_off, t.rows, t.cols, t.ld, "W stage dst");
        for (int j = 0; j < t.nsrc; ++j) {
            const LcSrc &sj = srcs[t.src0 + j];
            check_span(slot_elems, sj.slot, sj.off, t.rows, t.cols, sj.ld, "W stage src");
        }
    }
}

int64_t GemmList::split_k(int parts, int pslot, LcList &reduce, bool all) {
    if (parts <= 1 && !all) return 0;
    std::vector<GemmItem> nitems;
    std::vector<GemmSeg> nsegs;
    std::vector<int32_t> nblk0;
    std::vector<RowBlock> nblocks;
    int64_t pel = 0;
    // K range length of the longest item's parts; every item is cut into
    // ranges of about that length, so no tile's K loop is much longer than
    // another's (the longest tile bounds the launch), each range >= 64
    int64_t kmax = 0;
    for (const GemmItem &it : items) kmax = std::max(kmax, item_k(*this, it));
    const double krange = std::max(1.0, (double)kmax / std::max(parts, 1));
    for (size_t ii = 0; ii < items.size(); ++ii) {
        const GemmItem &it = items[ii];
        const int64_t ktot = item_k(*this, it);
        const int ip = split_parts(ktot, krange);
        if (it.M == 0 || it.N == 0 || (ip == 1 && !all)) {
            GemmItem c = it;
            c.seg0 = (int32_t)nsegs.size();
            for (int k = 0; k < it.nseg; ++k) nsegs.push_back(segs[it.seg0 + k]);
            if (blk0[ii] >= 0) {
                nblk0.push_back((int32_t)nblocks.size());
                for (int b = blk0[ii];; ++b) {
                    nblocks.push_back(blocks[b]);
                    if (blocks[b].r0 == it.M && blocks[b].rows == 0) break;
                }
            } else {
                nblk0.push_back(-1);
            }
            nitems.push_back(c);
            continue;
        }
        // the output blocks this item writes: one plain block, or its stacked blocks
        std::vector<RowBlock> outb;
        if (blk0[ii] >= 0) {
            for (int b = blk0[ii]; blocks[b].rows > 0; ++b) outb.push_back(blocks[b]);
        } else {
            outb.push_back(RowBlock{it.c_off, 0, it.M, it.ldc});
        }
        const int64_t pbase = pel;
        for (int p = 0; p < ip; ++p) {
            // K range [kb, ke), boundaries rounded to multiples of 32
            const int64_t kb = (ktot * p / ip) / 32 * 32;
            const int64_t ke = p + 1 == ip ? ktot : (ktot * (p + 1) / ip) / 32 * 32;
            GemmItem c{};
            c.c_slot = pslot;
            c.c_off = pel;
            c.M = it.M;
            c.N = it.N;
            c.ldc = it.N;
            c.rmap = -1;
            c.seg0 = (int32_t)nsegs.size();
            c.nseg = 0;
            int64_t g0 = 0;   // global K index of the current segment's start
            for (int k = 0; k < it.nseg; ++k) {
                GemmSeg sg = segs[it.seg0 + k];
                const int64_t s0 = std::max<int64_t>(kb, g0), s1 = std::min<int64_t>(ke, g0 + sg.K);
                if (s1 > s0) {
                    const int64_t d = s0 - g0;
                    GemmSeg sub = sg;
                    sub.K = (int32_t)(s1 - s0);
                    sub.a_off += ta ? d * sg.lda : d;
                    sub.b_off += tb ? d : d * sg.ldb;
                    nsegs.push_back(sub);
                    c.nseg += 1;
                }
                g0 += sg.K;
            }
            nitems.push_back(c);
            nblk0.push_back(-1);
            pel += (int64_t)it.M * it.N;
        }
        // fixed-order reduction of the parts into each output block
        for (const RowBlock &ob : outb) {
            reduce.add_task(it.c_slot, ob.c_off, ob.rows, it.N, ob.ldc);
            for (int p = 0; p < ip; ++p)
                reduce.add_src(pslot, pbase + (int64_t)p * it.M * it.N + (int64_t)ob.r0 * it.N, it.N, 1.0);
        }
    }
    items.swap(nitems);
    segs.swap(nsegs);
    blk0.swap(nblk0);
    blocks.swap(nblocks);
    return pel;
}

void GemmList::launch(GemmPrec prec, bool c_is_f64, const Slots &sl, hipStream_t s) const {
    launch(prec, c_is_f64, sl, dev, s);
}

void GemmList::launch(GemmPrec prec, bool c_is_f64, const Slots &sl, const GemmDev &dv, hipStream_t s) const {
    PD_REQUIRE(prec != GemmPrec::BF16X3 || !ftiles.empty() || tiles.empty(), PDMRG_EINVAL,
               "gemm: BF16x3 needs an LDS-DMA or quad plan (split operands)");
    if ((1u << (int)shape) & kQuadShapes) {
        PD_REQUIRE(prec != GemmPrec::F64 && !c_is_f64 && (!ftiles.empty() || tiles.empty()), PDMRG_EINVAL,
                   "gemm: the quad kernel is for FP32 and BF16x3 and one segment per item");
        launch_gemm_quad(prec == GemmPrec::BF16X3, shape, sl, dv.ftiles, dv.rowoff, dv.epi, (int)ftiles.size(), s);
        return;
    }
    if ((1u << (int)shape) & kR64Shapes) {
        PD_REQUIRE(prec == GemmPrec::F64 && (!ftiles.empty() || tiles.empty()), PDMRG_EINVAL,
                   "gemm: the register-direct kernel is for FP64 and one segment per item");
        launch_gemm_r64(shape, sl, dv.ftiles, dv.rowoff, dv.epi, (int)ftiles.size(), s);
        return;
    }
    if (!ftiles.empty()) {
        launch_gemm_flat(prec, shape, c_is_f64, sl, dv.ftiles, dv.rowoff, dv.epi, (int)ftiles.size(), s);
        return;
    }
    launch_gemm(prec, shape, ta, tb, c_is_f64, sl, dv.items, dv.segs, dv.tiles, dv.rowoff, dv.epi,
                (int)tiles.size(), s);
}

int LcList::add_task(int dst_slot, int64_t dst_off, int rows, int cols, int ld) {
    LcTask t{};
    t.dst_off = dst_off;
    t.dst_slot = dst_slot;
    t.rows = rows;
    t.cols = cols;
    t.ld = ld;
    t.src0 = (int32_t)srcs.size();
    t.nsrc = 0;
    tasks.push_back(t);
    elems_out += (int64_t)rows * cols;
    return (int)tasks.size() - 1;
}

void LcList::add_src(int slot, int64_t off, int ld, double coef) {
    LcSrc sj{};
    sj.off = off;
    sj.slot = slot;
    sj.ld = ld;
    sj.coef = coef;
    srcs.push_back(sj);
    LcTask &t = tasks.back();
    t.nsrc += 1;
    flops += 2.0 * t.rows * (double)t.cols;
    elems_in += (int64_t)t.rows * t.cols;
}

void LcList::build_tiles() {
    tiles.clear();
    for (size_t i = 0; i < tasks.size(); ++i) {
        const LcTask &t = tasks[i];
        const int64_t n = (int64_t)t.rows * t.cols;
        for (int64_t c = 0; c * chunk < n; ++c) tiles.push_back(LcTile{(int32_t)i, (int32_t)c, chunk, 0});
    }
}

void LcList::finish(hipStream_t s) {
    build_tiles();
    ListStage st;
    stage(st);
    st.flush(d_lists, s);
}

void LcList::stage(ListStage &st) {
    st.add(dev.tasks, tasks);
    st.add(dev.srcs, srcs);
    st.add(dev.tiles, tiles);
}

void LcList::launch_f32_to_f64(const Slots &sl, hipStream_t s) const {
    launch_lincomb_f32_f64(chunk, sl, dev.tasks, dev.srcs, dev.tiles, (int)tiles.size(), s);
}

void LcList::launch_split(const Slots &sl, hipStream_t s) const {
    launch_lincomb_split(chunk, sl, dev.tasks, dev.srcs, dev.tiles, (int)tiles.size(), s);
}

void LcList::launch(bool f64, const Slots &sl, hipStream_t s) const {
    launch(f64, sl, dev, s);
}

void LcList::launch(bool f64, const Slots &sl, const LcDev &dv, hipStream_t s) const {
    launch_lincomb(f64, chunk, sl, dv.tasks, dv.srcs, dv.tiles, (int)tiles.size(), s);
}

std::vector<double> two_site_mpo(const MpoSite &W1, const MpoSite &W2) {
    // W12[w][s1][t1][s2][t2][w2] = sum_c W1[w][s1][t1][c] W2[c][s2][t2][w2]
    PD_REQUIRE(W1.Dr == W2.Dl && W1.d == W2.d, PDMRG_ESHAPE, "two-site MPO: inner channel mismatch");
    const int d = W1.d, Dl = W1.Dl, Dm = W1.Dr, Dr = W2.Dr;
    std::vector<double> W12((size_t)Dl * d * d * d * d * Dr, 0.0);
    for (int w = 0; w < Dl; ++w)
        for (int s1 = 0; s1 < d; ++s1)
            for (int t1 = 0; t1 < d; ++t1)
                for (int c = 0; c < Dm; ++c) {
                    const double a = W1.at(w, s1, t1, c);
                    if (a == 0.0) continue;
                    for (int s2 = 0; s2 < d; ++s2)
                        for (int t2 = 0; t2 < d; ++t2)
                            for (int w2 = 0; w2 < Dr; ++w2) {
                                const double b = W2.at(c, s2, t2, w2);
                                if (b == 0.0) continue;
                                W12[((((((size_t)w * d + s1) * d + t1) * d + s2) * d + t2) * Dr) + w2] += a * b;
                            }
                }
    return W12;
}

// A nonzero MPO entry: its two indices that a sum runs over, in the sum's order.
struct Entry {
    int x, y;
    double c;
};

// ---------------------------------------------------------------- H_eff
void HeffPlan::build(const Bond &bl_, const Bond &br_, const Phys &p_, const MpoSite &W1, const MpoSite &W2,
                     int prec, hipStream_t s) {
    bl = bl_;
    br = br_;
    p = p_;
    const int d = p.d(), d2 = d * d;
    PD_REQUIRE(W1.d == d && W2.d == d, PDMRG_ESHAPE, "heff: MPO local dimension mismatch");
    PD_REQUIRE(W1.Dr == W2.Dl, PDMRG_ESHAPE, "heff: W1/W2 channel mismatch");
    const int Dl = W1.Dl, Dr = W2.Dr;
    X = two_site_layout(bl, br, p);
    Lt = env_l_layout(bl, W1.dl);
    Rt = env_r_layout(br, W2.dr);
    const std::vector<double> W12 = two_site_mpo(W1, W2);
    auto w12 = [&](int w, int s1, int t1, int s2, int t2, int w2) {
        return W12[((((((size_t)w * d + s1) * d + t1) * d + s2) * d + t2) * Dr) + w2];
    };
    const int nl = bl.nsec();

    // stage 1: T1[j] = Lket[j] (rows (w, a)) x X[j] (rows a', cols (t1 t2 b'))
    std::vector<int64_t> t1base(nl, -1);
    std::vector<int> chan((size_t)nl * Dl, -1), seg((size_t)nl * d2, -1), item_of(nl, -1);   // EpiItem indices
    nT1 = 0;
    g1 = GemmList();
    g1.elem_bytes = prec == PDMRG_F64 ? 8 : 4;
    for (int j = 0; j < nl; ++j) {
        const int M = Lt.rows[j], N = X.cols[j], K = bl.dim[j];
        if (M == 0 || N == 0) continue;
        t1base[j] = nT1;
        g1.add_item(4, nT1, M, N, N);
        g1.add_seg(2, Lt.base[j], K, 0, X.base[j], N, K);
        nT1 += (int64_t)M * N;
        EpiItem ei{(int32_t)g1.epi_row.size(), (int32_t)g1.epi_col.size(), (int32_t)g1.epi_dst.size(), 0};
        int nc = 0;
        for (int ww = 0; ww < Dl; ++ww) {
            const int r0 = Lt.rowo[(size_t)j * Dl + ww];
            if (r0 < 0) continue;
            chan[(size_t)j * Dl + ww] = nc++;
            g1.epi_row.push_back(r0);
        }
        g1.epi_row.push_back(M);
        for (int tg = 0; tg < d2; ++tg) {
            const int c0 = X.colo[(size_t)j * d2 + tg];
            if (c0 < 0) continue;
            seg[(size_t)j * d2 + tg] = ei.nseg++;
            g1.epi_col.push_back(c0);
        }
        g1.epi_col.push_back(N);
        g1.epi_dst.resize(g1.epi_dst.size() + (size_t)nc * ei.nseg, EpiDst{-1, 0.0, 0, 0});
        item_of[j] = (int)g1.epi_items.size();
        g1.epi_items.push_back(ei);
    }
    auto epi_at = [&](int j, int ww, int tg) -> EpiDst & {
        const EpiItem &ei = g1.epi_items[item_of[j]];
        return g1.epi_dst[ei.dst0 + (size_t)chan[(size_t)j * Dl + ww] * ei.nseg + seg[(size_t)j * d2 + tg]];
    };

    // T2 blocks: one per output block (i, s1 s2) -> [dim(q_i) x Rt.rows[k]],
    // grouped by the bra sector k they multiply, so that the blocks sharing
    // R[k] form one contiguous (sum of dims) x Rt.rows[k] matrix.
    std::vector<int64_t> t2base((size_t)nl * d2, -1);
    std::vector<std::vector<std::pair<int, int>>> by_k(br.nsec());
    for (int i = 0; i < nl; ++i)
        for (int sg = 0; sg < d2; ++sg) {
            if (X.colo[(size_t)i * d2 + sg] < 0) continue;
            by_k[br.find(bl.q[i] + p.q[sg / d] + p.q[sg % d])].push_back({i, sg});
        }
    nT2 = 0;
    for (int k = 0; k < br.nsec(); ++k)
        for (auto [i, sg] : by_k[k]) {
            t2base[(size_t)i * d2 + sg] = nT2;
            nT2 += (int64_t)bl.dim[i] * Rt.rows[k];
        }

    // stage 2: W stage
    w = LcList();
    const std::vector<int64_t> sz = {X.size, X.size, Lt.size, Rt.size, nT1, nT2, 0};
    struct Term {
        int j, ww, tg;
        int64_t off;
        double c;
    };
    std::vector<Term> terms;
    // below this the W stage is latency, and looking blocks up costs stage 1 more
    // than it saves (16-site chain, m = 64, 0.1 MB: 19.0 -> 21.6 us; 8 x 4 cylinder,
    // m = 1024, 63 MB: 187 -> 181)
    const bool direct = nT1 * g1.elem_bytes >= (int64_t(32) << 20);
    std::vector<std::vector<Entry>> nz((size_t)d2 * Dr);   // of (s1 s2, w2): (w, t1 t2) in order
    for (int ww = 0; ww < Dl; ++ww)
        for (int sg = 0; sg < d2; ++sg)
            for (int tg = 0; tg < d2; ++tg)
                for (int w2 = 0; w2 < Dr; ++w2) {
                    const double c = w12(ww, sg / d, tg / d, sg % d, tg % d, w2);
                    if (c != 0.0) nz[(size_t)sg * Dr + w2].push_back(Entry{ww, tg, c});
                }
    for (int i = 0; i < nl; ++i)
        for (int sg = 0; sg < d2; ++sg) {
            const int64_t tb = t2base[(size_t)i * d2 + sg];
            if (tb < 0) continue;
            const int s1 = sg / d, s2 = sg % d;
            const int qb = bl.q[i] + p.q[s1] + p.q[s2];
            const int k = br.find(qb);
            for (int w2 = 0; w2 < Dr; ++w2) {
                const int ro = Rt.rowo[(size_t)k * Dr + w2];
                if (ro < 0) continue;
                const int cols = br.dim_of(qb - W2.dr[w2]);
                terms.clear();
                for (const Entry &e : nz[(size_t)sg * Dr + w2]) {
                    const int ww = e.x, tg = e.y;
                    const int j = bl.find(bl.q[i] - W1.dl[ww]);
                    if (j < 0 || t1base[j] < 0) continue;
                    const int lro = Lt.rowo[(size_t)j * Dl + ww];
                    if (lro < 0) continue;
                    const int co = X.colo[(size_t)j * d2 + tg];
                    if (co < 0) continue;
                    PD_REQUIRE(X.width[(size_t)j * d2 + tg] == cols, PDMRG_ESHAPE,
                               "heff: MPO entry violates charge conservation");
                    terms.push_back(Term{j, ww, tg, t1base[j] + (int64_t)lro * X.cols[j] + co, e.c});
                }
                // a sum of one term is left to stage 1 (a block goes to one place besides T1)
                EpiDst *one = direct && terms.size() == 1 ? &epi_at(terms[0].j, terms[0].ww, terms[0].tg) : nullptr;
                if (one && one->off < 0) {
                    one->off = tb + ro;
                    one->coef = terms[0].c;
                    one->ld = Rt.rows[k];
                    check_span(sz, 5, one->off, bl.dim[i], cols, one->ld, "W stage dst");
                    w.flops += 2.0 * bl.dim[i] * (double)cols;
                    continue;
                }
                w.add_task(5, tb + ro, bl.dim[i], cols, Rt.rows[k]);
                for (const Term &t : terms) {
                    w.add_src(4, t.off, X.cols[t.j], t.c);
                    epi_at(t.j, t.ww, t.tg).keep = 1;
                }
            }
        }

    // stage 3: y[i, s1 s2] = T2[i, s1 s2] x Rbra[k], one stacked item per k
    // (cut into several where the stacked T2 operand would span 2 GiB or
    // more, the reach of the kernels' 32-bit buffer offsets)
    g3 = GemmList();
    const int64_t es3 = prec == PDMRG_F64 ? 8 : 4;
    g3.elem_bytes = (int)es3;
    for (int k = 0; k < br.nsec(); ++k) {
        if (by_k[k].empty()) continue;
        const int64_t ld = std::max(Rt.rows[k], 1);
        size_t b0 = 0;
        while (b0 < by_k[k].size()) {
            std::vector<RowBlock> blks;
            int64_t rows = 0;
            size_t b1 = b0;
            for (; b1 < by_k[k].size(); ++b1) {
                const auto [i, sg] = by_k[k][b1];
                if (!blks.empty() && (rows + bl.dim[i]) * ld * es3 >= (int64_t(1) << 31)) break;
                blks.push_back(RowBlock{X.base[i] + X.colo[(size_t)i * d2 + sg], 0, bl.dim[i], X.cols[i]});
                rows += bl.dim[i];
            }
            g3.add_stacked_item(1, br.dim[k], blks);
            const auto [i0, sg0] = by_k[k][b0];
            if (Rt.rows[k] > 0)
                g3.add_seg(5, t2base[(size_t)i0 * d2 + sg0], Rt.rows[k], 3, Rt.base[k], br.dim[k], Rt.rows[k]);
            b0 = b1;
        }
    }

    // diag(H_eff): sum over channels with delta = 0 of L[a,w,a] W12 R[b,w2,b]
    diag_terms.clear();
    diag_groups.assign(1, 0);
    diag_max_rows = 0;
    for (int i = 0; i < nl; ++i)
        for (int sg = 0; sg < d2; ++sg) {
            if (X.colo[(size_t)i * d2 + sg] < 0) continue;
            const int s1 = sg / d, s2 = sg % d;
            const int k = br.find(bl.q[i] + p.q[s1] + p.q[s2]);
            DiagTerm base{};
            base.out_off = X.base[i] + X.colo[(size_t)i * d2 + sg];
            base.rows = bl.dim[i];
            base.cols = br.dim[k];
            base.ld = X.cols[i];
            diag_max_rows = std::max(diag_max_rows, base.rows);
            bool any = false;
            for (int ww = 0; ww < Dl; ++ww) {
                if (W1.dl[ww] != 0) continue;
                const int lro = Lt.rowo[(size_t)i * Dl + ww];
                if (lro < 0) continue;
                for (int w2 = 0; w2 < Dr; ++w2) {
                    if (W2.dr[w2] != 0) continue;
                    const double c = w12(ww, s1, s1, s2, s2, w2);
                    if (c == 0.0) continue;
                    const int rro = Rt.rowo[(size_t)k * Dr + w2];
                    if (rro < 0) continue;
                    DiagTerm t = base;
                    t.coef = c;
                    t.l_off = Lt.base[i] + (int64_t)lro * Lt.cols[i];
                    t.lstride = Lt.cols[i] + 1;
                    t.r_off = Rt.base[k] + (int64_t)rro * Rt.cols[k];
                    t.rstride = Rt.cols[k] + 1;
                    diag_terms.push_back(t);
                    any = true;
                }
            }
            if (!any) {   // still write zeros
                DiagTerm t = base;
                t.coef = 0.0;
                t.l_off = 0;
                t.r_off = 0;
                t.lstride = 0;
                t.rstride = 0;
                diag_terms.push_back(t);
            }
            diag_groups.push_back((int32_t)diag_terms.size());
        }

    // tile shapes: both lists are non-transposed with one segment per item,
    // so the LDS-DMA, register-direct and quad shapes apply; BF16x3 (split
    // operands) runs only the first and the last
    g1.shapes_allowed = g3.shapes_allowed = prec == PDMRG_BF16X3 ? kDmaShapes | kQuadShapes
                                            : prec == PDMRG_F32  ? kStagedShapes | kDmaShapes | kQuadShapes
                                                                 : kStagedShapes | kDmaShapes | kR64Shapes;
    const double bytes = g1.operand_bytes() + g3.operand_bytes();
    g1.pick_tile(bytes);
    g3.pick_tile(bytes);
    g1.dev.epi.slot = 5;
    if (!direct) g1.epi_items.clear();
    g1.validate(sz);
    w.validate(sz);
    g1.finish(s);
    w.finish(s);
    g3_base = g3.host_copy();
    lowp = prec != PDMRG_F64;
    TileShape shape = g3.shape;
    int parts = default_parts(shape);
    if (lowp || g3.streams) {
        // The split and the shape together.  FP32 and BF16x3 split as far as K
        // allows: stage 3 with its reduction at 2, 4, 8 parts takes 0.365, 0.356,
        // 0.335 ms (BF16x3, tri 12 x 6, m = 3000), 0.108, 0.093, 0.090 (FP32, 24 x 8
        // cylinder, m = 2000), 0.037, 0.030, 0.032 (BF16x3, 8 x 4, m = 1024).
        const unsigned shapes = lowp ? g3_base.quad_shapes(8) : kR64Shapes;
        double best = 0.0;
        for (int p = lowp ? 8 : 1; p <= (lowp ? 8 : kMaxParts64); ++p)
            for (int t = 0; t < kNumShapes; ++t) {
                if (!((shapes >> t) & 1u)) continue;
                const double c = g3_base.cost((TileShape)t, p);
                if (best == 0.0 || c < best * 0.999) best = c, parts = p, shape = (TileShape)t;
            }
    }
    set_g3_shape(shape, s, parts);
}

void HeffPlan::set_g1_shape(TileShape t, hipStream_t s) {
    g1.shape = t;
    g1.finish(s);
}

int HeffPlan::default_parts(TileShape t) const {
    // split-K for stage 3: aim at >= 1024 output tiles (4 per CU)
    const int tiles3 = std::max(1, g3_base.ntiles_for(t));
    return std::max(1, std::min(8, (1024 + tiles3 - 1) / tiles3));
}

void HeffPlan::set_g3_shape(TileShape t, hipStream_t s, int parts) {
    g3 = g3_base.host_copy();
    g3.shape = t;
    if (parts <= 0) parts = default_parts(t);
    r3 = LcList();
    r3.chunk = kLcChunkSmall;
    // low precision: every item goes through the FP32 partial buffer and the
    // reduction writes the FP64 output
    nP = g3.split_k(parts, 6, r3, lowp);
    parts3 = parts;
    const std::vector<int64_t> sz = {X.size, X.size, Lt.size, Rt.size, nT1, nT2, nP};
    g3.validate(sz);
    r3.validate(sz);
    g3.finish(s);
    r3.finish(s);
}

// ---------------------------------------------------------------- environments
void EnvPlan::begin(int dir_, const Bond &bl_, const Bond &br_, const Phys &p_, const MpoSite &W) {
    dir = dir_;
    bl = bl_;
    br = br_;
    p = p_;
    const int d = p.d();
    PD_REQUIRE(W.d == d, PDMRG_ESHAPE, "env: MPO local dimension mismatch");
    S = site_layout(bl, br, p);
    const int nl = bl.nsec(), nr = br.nsec();
    g1 = GemmList();
    nU1 = nU2 = 0;
    if (dir > 0) {
        Ein = env_l_layout(bl, W.dl);
        Eout = env_l_layout(br, W.dr);
        Aux = env_r_layout(br, W.dr);     // column structure of U2 blocks
        // E1: U1[j] = Lket[j] x A[j]
        u1base.assign(nl, -1);
        for (int j = 0; j < nl; ++j) {
            const int M = Ein.rows[j], N = S.cols[j], K = bl.dim[j];
            if (M == 0 || N == 0) continue;
            u1base[j] = nU1;
            g1.add_item(3, nU1, M, N, N);
            g1.add_seg(0, Ein.base[j], K, 1, S.base[j], N, K);
            nU1 += (int64_t)M * N;
        }
        // U2 blocks (i, s): [dim(q_i) x Aux.rows[k]]
        u2base.assign((size_t)nl * d, -1);
        for (int i = 0; i < nl; ++i)
            for (int sp = 0; sp < d; ++sp) {
                if (S.colo[(size_t)i * d + sp] < 0) continue;
                const int k = br.find(bl.q[i] + p.q[sp]);
                u2base[(size_t)i * d + sp] = nU2;
                nU2 += (int64_t)bl.dim[i] * Aux.rows[k];
            }
    } else {
        Ein = env_r_layout(br, W.dr);
        Eout = env_r_layout(bl, W.dl);
        // F1: Z1[(k,s)] = Rbra[k] x B[(i,s)]^T, i = q_k - q_s
        u1base.assign((size_t)nr * d, -1);
        g1.tb = true;
        for (int k = 0; k < nr; ++k)
            for (int sp = 0; sp < d; ++sp) {
                const int i = bl.find(br.q[k] - p.q[sp]);
                if (i < 0 || Ein.rows[k] == 0) continue;
                u1base[(size_t)k * d + sp] = nU1;
                g1.add_item(3, nU1, Ein.rows[k], bl.dim[i], bl.dim[i]);
                g1.add_seg(0, Ein.base[k], br.dim[k], 1, S.base[i] + S.colo[(size_t)i * d + sp], S.cols[i],
                           br.dim[k]);
                nU1 += (int64_t)Ein.rows[k] * bl.dim[i];
            }
        // Z2 blocks (i, w): [S.cols[i'] x dim(q_i)], i' = q_i - dl_w
        u2base.assign((size_t)nl * W.Dl, -1);
        for (int i = 0; i < nl; ++i)
            for (int ww = 0; ww < W.Dl; ++ww) {
                const int ip = bl.find(bl.q[i] - W.dl[ww]);
                if (ip < 0 || S.cols[ip] == 0) continue;
                u2base[(size_t)i * W.Dl + ww] = nU2;
                nU2 += (int64_t)S.cols[ip] * bl.dim[i];
            }
    }
    g1.validate({Ein.size, S.size, Eout.size, nU1});
    g1.pick_tile();
}

void EnvPlan::finish(const MpoSite &W) {
    const int d = p.d(), Dl = W.Dl, Dr = W.Dr;
    const int nl = bl.nsec(), nr = br.nsec();
    g3 = GemmList();
    w = LcList();
    if (dir > 0) {
        // E2: U2[(i,s)][a, (w', b')] = sum W[w,s,t,w'] U1[q_i - dl_w][(w,a), (t,b')]
        std::vector<std::vector<Entry>> nz((size_t)d * Dr);   // of (s, w'): (w, t) in order
        for (int ww = 0; ww < Dl; ++ww)
            for (int sp = 0; sp < d; ++sp)
                for (int t = 0; t < d; ++t)
                    for (int w2 = 0; w2 < Dr; ++w2) {
                        const double c = W.at(ww, sp, t, w2);
                        if (c != 0.0) nz[(size_t)sp * Dr + w2].push_back(Entry{ww, t, c});
                    }
        for (int i = 0; i < nl; ++i)
            for (int sp = 0; sp < d; ++sp) {
                const int64_t ub = u2base[(size_t)i * d + sp];
                if (ub < 0) continue;
                const int qb = bl.q[i] + p.q[sp];
                const int k = br.find(qb);
                for (int w2 = 0; w2 < Dr; ++w2) {
                    const int ro = Aux.rowo[(size_t)k * Dr + w2];
                    if (ro < 0) continue;
                    const int cols = br.dim_of(qb - W.dr[w2]);
                    w.add_task(4, ub + ro, bl.dim[i], cols, Aux.rows[k]);
                    for (const Entry &e : nz[(size_t)sp * Dr + w2]) {
                        const int ww = e.x, t = e.y;
                        const int j = bl.find(bl.q[i] - W.dl[ww]);
                        if (j < 0 || u1base[j] < 0) continue;
                        const int lro = Ein.rowo[(size_t)j * Dl + ww];
                        if (lro < 0) continue;
                        const int co = S.colo[(size_t)j * d + t];
                        if (co < 0) continue;
                        PD_REQUIRE(S.width[(size_t)j * d + t] == cols, PDMRG_ESHAPE,
                                   "env: MPO entry violates charge conservation");
                        w.add_src(3, u1base[j] + (int64_t)lro * S.cols[j] + co, S.cols[j], e.c);
                    }
                }
            }
        // E3: Lout[j'] rows (w', b) = sum_s A[(i,s)]^T U2[(i,s)][:, w' segment]
        g3.ta = true;
        for (int jp = 0; jp < nr; ++jp)
            for (int w2 = 0; w2 < Dr; ++w2) {
                const int ro = Eout.rowo[(size_t)jp * Dr + w2];
                if (ro < 0) continue;
                const int k = br.find(br.q[jp] + W.dr[w2]);
                g3.add_item(2, Eout.base[jp] + (int64_t)ro * br.dim[jp], br.dim[k], br.dim[jp], br.dim[jp]);
                for (int sp = 0; sp < d; ++sp) {
                    const int i = bl.find(br.q[k] - p.q[sp]);
                    if (i < 0) continue;
                    const int64_t ub = u2base[(size_t)i * d + sp];
                    if (ub < 0) continue;
                    const int aro = Aux.rowo[(size_t)k * Dr + w2];
                    g3.add_seg(1, S.base[i] + S.colo[(size_t)i * d + sp], S.cols[i], 4, ub + aro, Aux.rows[k],
                               bl.dim[i]);
                }
            }
    } else {
        // F2: Z2[(i,w)][(s', b'), a] = sum W[w,s,s',w2] Z1[(k,s)][(w2,b'), a]
        std::vector<std::vector<Entry>> nz((size_t)Dl * d);   // of (w, s'): (s, w2) in order
        for (int ww = 0; ww < Dl; ++ww)
            for (int sp = 0; sp < d; ++sp)
                for (int spp = 0; spp < d; ++spp)
                    for (int w2 = 0; w2 < Dr; ++w2) {
                        const double c = W.at(ww, sp, spp, w2);
                        if (c != 0.0) nz[(size_t)ww * d + spp].push_back(Entry{sp, w2, c});
                    }
        for (int i = 0; i < nl; ++i)
            for (int ww = 0; ww < Dl; ++ww) {
                const int64_t zb = u2base[(size_t)i * Dl + ww];
                if (zb < 0) continue;
                const int ip = bl.find(bl.q[i] - W.dl[ww]);
                for (int spp = 0; spp < d; ++spp) {
                    const int co = S.colo[(size_t)ip * d + spp];
                    if (co < 0) continue;
                    const int rows = S.width[(size_t)ip * d + spp];
                    w.add_task(4, zb + (int64_t)co * bl.dim[i], rows, bl.dim[i], bl.dim[i]);
                    for (const Entry &e : nz[(size_t)ww * d + spp]) {
                        const int sp = e.x, w2 = e.y;
                        const int k = br.find(bl.q[i] + p.q[sp]);
                        if (k < 0) continue;
                        const int64_t z1 = u1base[(size_t)k * d + sp];
                        if (z1 < 0) continue;
                        const int ro = Ein.rowo[(size_t)k * Dr + w2];
                        if (ro < 0) continue;
                        PD_REQUIRE(br.dim_of(br.q[k] - W.dr[w2]) == rows, PDMRG_ESHAPE,
                                   "env: MPO entry violates charge conservation");
                        w.add_src(3, z1 + (int64_t)ro * bl.dim[i], bl.dim[i], e.c);
                    }
                }
            }
        // F3: Rout[i] rows (w, a') = B[i'] x Z2[(i,w)]
        for (int i = 0; i < nl; ++i)
            for (int ww = 0; ww < Dl; ++ww) {
                const int ro = Eout.rowo[(size_t)i * Dl + ww];
                if (ro < 0) continue;
                const int ip = bl.find(bl.q[i] - W.dl[ww]);
                g3.add_item(2, Eout.base[i] + (int64_t)ro * bl.dim[i], bl.dim[ip], bl.dim[i], bl.dim[i]);
                const int64_t zb = u2base[(size_t)i * Dl + ww];
                if (zb >= 0) g3.add_seg(1, S.base[ip], S.cols[ip], 4, zb, bl.dim[i], S.cols[ip]);
            }
    }
    const std::vector<int64_t> sz = {Ein.size, S.size, Eout.size, nU1, nU2};
    w.validate(sz);
    g3.validate(sz);
    g3.pick_tile();
}

void EnvPlan::run(const MpoSite &W, const void *env_in, const void *site, void *env_out, DevBuf &ws, hipStream_t s) {
    Slots sl{};
    sl.p[0] = env_in;
    sl.p[1] = site;
    sl.p[2] = env_out;
    const size_t n1 = (size_t)std::max<int64_t>(nU1, 1);
    ws.ensure((n1 + (size_t)std::max<int64_t>(nU2, 1)) * sizeof(double));
    sl.p[3] = ws.as<double>();
    sl.p[4] = ws.as<double>() + n1;
    ListStage st;
    g1.build_tiles();
    g1.stage(st);
    st.flush(d_lists1, s);
    g1.launch(GemmPrec::F64, true, sl, s);
    try {
        finish(W);
        w.build_tiles();
        g3.build_tiles();
        w.stage(st);
        g3.stage(st);
        st.flush(d_lists, s);
    } catch (...) {
        (void)hipStreamSynchronize(s);   // nothing left running on the caller's buffers
        throw;
    }
    w.launch(true, sl, s);
    g3.launch(GemmPrec::F64, true, sl, s);
}

void EnvPlan::run(GemmPrec prec, const void *env_in, const void *site, void *env_out, void *U1, void *U2,
                  const GemmDev &d1, const LcDev &dw, const GemmDev &d3, hipStream_t s) const {
    Slots sl{};
    sl.p[0] = env_in;
    sl.p[1] = site;
    sl.p[2] = env_out;
    sl.p[3] = U1;
    sl.p[4] = U2;
    const bool f64 = prec == GemmPrec::F64;
    g1.launch(prec, f64, sl, d1, s);
    w.launch(f64, sl, dw, s);
    g3.launch(prec, f64, sl, d3, s);
}

// ---------------------------------------------------------------- gradient
void GradPlan::run(const Bond &bl_, const Bond &br_, const Phys &p_, const MpoSite &W, const double *L,
                   const double *psi, const double *R, DevBuf &ws, DevBuf &ws2, double *G, hipStream_t s) {
    bl = bl_;
    br = br_;
    p = p_;
    const int d = p.d();
    PD_REQUIRE(W.d == d, PDMRG_ESHAPE, "grad: MPO local dimension mismatch");
    Dl = W.Dl;
    Dr = W.Dr;
    S = site_layout(bl, br, p);
    Lt = env_l_layout(bl, W.dl);
    Rt = env_r_layout(br, W.dr);
    const int nl = bl.nsec();
    // stage 1: U1[j] = Lket[j] x psi[j]
    g1 = GemmList();
    std::vector<int64_t> u1base(nl, -1);
    nU1 = 0;
    for (int j = 0; j < nl; ++j) {
        const int M = Lt.rows[j], N = S.cols[j], K = bl.dim[j];
        if (M == 0 || N == 0) continue;
        u1base[j] = nU1;
        g1.add_item(3, nU1, M, N, N);
        g1.add_seg(0, Lt.base[j], K, 1, S.base[j], N, K);
        nU1 += (int64_t)M * N;
    }
    g1.validate({Lt.size, S.size, Rt.size, nU1});
    g1.pick_tile();
    Slots sl{};
    sl.p[0] = L;
    sl.p[1] = psi;
    sl.p[2] = R;
    ws.ensure((size_t)std::max<int64_t>(nU1, 1) * sizeof(double));
    sl.p[3] = ws.ptr;
    ListStage st;
    g1.build_tiles();
    g1.stage(st);
    st.flush(d_lists1, s);
    launch_fill(G, 0.0, (int64_t)Dl * d * d * Dr, s);
    g1.launch(GemmPrec::F64, true, sl, s);
    try {
        rest(W, u1base);
        gz.build_tiles();
        gz.stage(st);
        st.add(d_dots, dots);
        st.add(d_dtiles, dtiles);
        st.add(d_roff, r_off);
        st.add(d_pos, pos);
        st.add(d_order, order);
        st.add(d_sums, sums);
        st.flush(d_lists, s);
        ws2.ensure((std::max<size_t>(nZ, 1) + std::max<size_t>(npartial, 1)) * sizeof(double));
    } catch (...) {
        (void)hipStreamSynchronize(s);   // nothing left running on the caller's buffers
        throw;
    }
    double *partial = ws2.as<double>() + std::max<int64_t>(nZ, 1);
    sl.p[4] = ws2.ptr;
    gz.launch(GemmPrec::F64, true, sl, s);
    int max_ch = 0;
    for (const GradDot &t : dots) max_ch = std::max(max_ch, t.nch);
    launch_grad_dots(ws2.as<double>(), R, d_dots, d_dtiles, (int)dtiles.size(), max_ch, d_roff, partial, s);
    launch_grad_sums(partial, d_dots, d_order, d_sums, (int)sums.size(), d_pos, Dr, G, s);
}

// stage 2: Z blocks [b'][b] = U1^T psi, then stage-3 dot tasks
void GradPlan::rest(const MpoSite &W, const std::vector<int64_t> &u1base) {
    const int d = p.d(), nl = bl.nsec();
    gz = GemmList();
    gz.ta = true;
    dots.clear();
    dtiles.clear();
    r_off.clear();
    pos.clear();
    sums.clear();
    nZ = npartial = 0;
    std::vector<int> charge;                  // of the channels of R, each once
    std::vector<std::vector<int>> channels;   // with that charge, ascending
    for (int w2 = 0; w2 < Dr; ++w2) {
        const size_t c = std::find(charge.begin(), charge.end(), W.dr[w2]) - charge.begin();
        if (c == charge.size()) {
            charge.push_back(W.dr[w2]);
            channels.emplace_back();
        }
        channels[c].push_back(w2);
    }
    struct List {
        int list0 = -1, nch = 0, pos = 0;
    };
    std::vector<List> lists((size_t)br.nsec() * charge.size());   // by sector of R and charge
    std::vector<int> group;                                       // (w, s, t) of each dot
    dots.reserve((size_t)nl * Dl * d * d);
    group.reserve(dots.capacity());
    for (int i = 0; i < nl; ++i)
        for (int w = 0; w < Dl; ++w) {
            const int j = bl.find(bl.q[i] - W.dl[w]);
            if (j < 0 || u1base[j] < 0) continue;
            const int lro = Lt.rowo[(size_t)j * Dl + w];
            if (lro < 0) continue;
            for (int sp = 0; sp < d; ++sp) {
                const int cs = S.colo[(size_t)i * d + sp];
                if (cs < 0) continue;
                const int qb = bl.q[i] + p.q[sp];
                const int kb = br.find(qb);
                for (int t = 0; t < d; ++t) {
                    const int ct = S.colo[(size_t)j * d + t];
                    if (ct < 0) continue;
                    const int qbk = bl.q[j] + p.q[t];
                    // channels w' of R with delta = qb - qbk
                    const size_t ch = std::find(charge.begin(), charge.end(), qb - qbk) - charge.begin();
                    if (ch == charge.size()) continue;
                    const int M = br.dim_of(qbk), N = br.dim[kb], K = bl.dim[i];
                    List &ls = lists[kb * charge.size() + ch];
                    if (ls.list0 < 0) {
                        ls.list0 = (int)r_off.size();
                        ls.pos = (int)pos.size();
                        pos.resize(pos.size() + Dr, -1);
                        for (int w2 : channels[ch]) {
                            const int ro = Rt.rowo[(size_t)kb * Dr + w2];
                            if (ro < 0) continue;
                            pos[ls.pos + w2] = (int)r_off.size() - ls.list0;
                            r_off.push_back(Rt.base[kb] + (int64_t)ro * N);
                            PD_REQUIRE(r_off.back() >= 0 && r_off.back() + (int64_t)M * N <= Rt.size, PDMRG_ESHAPE,
                                       "grad: channel outside its buffer");
                        }
                        ls.nch = (int)r_off.size() - ls.list0;
                    }
                    if (ls.nch == 0) continue;
                    gz.add_item(4, nZ, M, N, N);
                    gz.add_seg(3, u1base[j] + (int64_t)lro * S.cols[j] + ct, S.cols[j], 1, S.base[i] + cs, S.cols[i],
                               K);
                    PD_REQUIRE(M > 0 && N > 0, PDMRG_ESHAPE, "grad: empty block");
                    const int nx = (M * N + kDotChunk - 1) / kDotChunk;
                    for (int x = 0; x < nx; ++x) dtiles.push_back(DotTile{(int)dots.size(), x});
                    dots.push_back(GradDot{nZ, npartial, M * N, ls.list0, ls.nch, ls.pos});
                    group.push_back((w * d + sp) * d + t);
                    flops += 2.0 * M * N * ls.nch;
                    npartial += (int64_t)nx * ls.nch;
                    nZ += (int64_t)M * N;
                }
            }
        }
    // dots by output entry, those of one entry in build order (a counting sort)
    order.resize(dots.size());
    std::vector<int> first((size_t)Dl * d * d + 1, 0);
    for (int g : group) ++first[(size_t)g + 1];
    for (size_t g = 0; g + 1 < first.size(); ++g) {
        if (first[g + 1] > 0) sums.push_back(GradSum{first[g], first[g] + first[g + 1], (int)g * Dr, 0});
        first[g + 1] += first[g];
    }
    for (size_t k = 0; k < dots.size(); ++k) order[first[group[k]]++] = (int)k;
    flops += g1.flops + gz.flops;
    gz.validate({Lt.size, S.size, Rt.size, nU1, nZ});
    gz.pick_tile();
}

// ---------------------------------------------------------------- merge
void MergePlan::build(const Bond &bl_, const Bond &bm_, const Bond &br_, const Phys &p_, hipStream_t s) {
    bl = bl_;
    bm = bm_;
    br = br_;
    p = p_;
    const int d = p.d(), d2 = d * d;
    SL = site_layout(bl, bm, p);
    SR = site_layout(bm, br, p);
    X = two_site_layout(bl, br, p);
    rs_base.clear();
    rs_vbase.clear();
    rs_rows.clear();
    rs_cols.clear();
    rs_max = 0;
    for (int k = 0; k < bm.nsec(); ++k) {
        if (SR.cols[k] == 0) continue;
        rs_base.push_back(SR.base[k]);
        rs_vbase.push_back(bm.off[k]);
        rs_rows.push_back(bm.dim[k]);
        rs_cols.push_back(SR.cols[k]);
        rs_max = std::max<int64_t>(rs_max, (int64_t)bm.dim[k] * SR.cols[k]);
    }
    g = GemmList();
    for (int i = 0; i < bl.nsec(); ++i)
        for (int s3 = 0; s3 < d; ++s3) {
            const int lco = SL.colo[(size_t)i * d + s3];
            if (lco < 0) continue;
            const int k = bm.find(bl.q[i] + p.q[s3]);
            if (SR.cols[k] == 0) continue;
            int col0 = -1;
            for (int s4 = 0; s4 < d; ++s4) {
                const int xc = X.colo[(size_t)i * d2 + s3 * d + s4];
                const int rc = SR.colo[(size_t)k * d + s4];
                PD_REQUIRE((xc < 0) == (rc < 0), PDMRG_ESHAPE, "merge: sector mismatch");
                if (xc < 0) continue;
                if (col0 < 0) col0 = xc - rc;
                PD_REQUIRE(xc - rc == col0, PDMRG_ESHAPE, "merge: column layout mismatch");
            }
            g.add_item(2, X.base[i] + col0, bl.dim[i], SR.cols[k], X.cols[i]);
            g.add_seg(0, SL.base[i] + lco, SL.cols[i], 1, SR.base[k], SR.cols[k], bm.dim[k]);
        }
    g.validate({SL.size, SR.size, X.size});
    g.pick_tile();
    ListStage st;
    g.build_tiles();
    g.stage(st);
    st.add(d_rs_base, rs_base);
    st.add(d_rs_vbase, rs_vbase);
    st.add(d_rs_rows, rs_rows);
    st.add(d_rs_cols, rs_cols);
    st.flush(d_lists, s);
}

void MergePlan::run(const double *psiL, const double *V, const double *psiR, double *out, double *scaled,
                    hipStream_t s) const {
    launch_row_scale(psiR, scaled, d_rs_base, d_rs_rows, d_rs_cols, d_rs_vbase, (int)rs_base.size(), rs_max, V, s);
    launch_fill(out, 0.0, X.size, s);
    Slots sl{};
    sl.p[0] = psiL;
    sl.p[1] = scaled;
    sl.p[2] = out;
    g.launch(GemmPrec::F64, true, sl, s);
}

}  // namespace pdmrg
