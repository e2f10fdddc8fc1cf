// Quad section of the device image (host only): the layout the batched products read (QuadPlan).
//
// Role in the method: Sec. 4.3.1 gives a kernel matrix to a PE group in passes of P x Q and Sec. 5.2 asks for equal
// shares of that uneven work.  Here a pass is at most 8 columns by the (at most 32) kernel rows of one block that
// land in one row tile, and the passes of a tile are dealt to 16 lists, each pass to the list with the least work so
// far, in column order: the wavefronts of all workgroups then walk the input at about the same pace,
// which keeps the rows they gather in the caches.  Work is that of four-row steps; the panels of 16-bit operands take any pass for the
// same time, four lists side by side, and so have 1.07 times the panels of an even deal (8192 x 8192 at 12x, counted).
#include <algorithm>
#include <cstring>
#include <new>

#include "csb_internal.hpp"

namespace csb {
namespace {

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct QPass {
    uint32_t b;            // CSB block
    uint16_t a0, q0;       // first kernel row and column
    uint8_t nrows, ncols;
    uint8_t shifted;       // 1: summed into row + shift (GRU split)
};

// Work of a pass, in units of about one instruction of a wavefront: what it costs whatever it multiplies, its input
// rows, its products and its row sums.
uint32_t pass_cost(const QPass &p) { return 90u + p.ncols * ((p.nrows + 3u) / 4u) * 4u + 3u * p.nrows; }

size_t pass_value_bytes(uint32_t nrows, uint32_t ncols, bool bits16) {
    return bits16 ? (size_t)nrows * kQuadCols * 2u : (size_t)((ncols + 3u) / 4u) * ((nrows + 3u) / 4u) * 64u;
}
uint32_t pass_stride(uint32_t quads, bool bits16) { return bits16 ? 0u : quads * 16u; }
uint32_t value_unit(bool bits16) { return bits16 ? 16u : 1u; }
// Position of the value at (row q, column j) among a pass's values.
size_t value_at(uint32_t quads, uint32_t q, uint32_t j, bool bits16) {
    return bits16 ? (size_t)q * kQuadCols + j : (j * 4u + (q & 3u)) * (size_t)quads + (q >> 2);
}

// The parts of block b's columns [q0, q1) that are summed together (GRU split) and come from one source.
struct ColPart { int q0, q1; bool lower, upper, shifted, second; };

template <typename F>
void for_column_parts(const csb_matrix *m, size_t b, int32_t bj, F f) {
    const int nc = m->ncols[b];
    const SplitSpec &sp = m->plan.split;
    const uint16_t *ci = m->colidx.data() + m->col_off[b];
    auto pos = [&](int64_t col) {
        int q = 0;
        while (q < nc && (int64_t)bj * m->bc + ci[q] < col) ++q;
        return q;
    };
    const int qs = sp.active() ? pos(sp.split_col) : nc, qx = m->quad_split > 0 ? pos(m->quad_split) : nc;
    auto cut = [&](int q0, int q1, bool lower, bool upper, bool shifted) {   // at the border between the sources
        const int c = std::min(std::max(qx, q0), q1);
        if (q0 < c) f(ColPart{q0, c, lower, upper, shifted, false});
        if (c < q1) f(ColPart{c, q1, lower, upper, shifted, true});
    };
    if (!sp.active()) { cut(0, nc, true, true, false); return; }
    cut(0, nc, true, false, false);
    cut(0, qs, false, true, false);
    cut(qs, nc, false, true, true);
}

// All passes of the matrix: f(tile, pass, second source, slots of the rows).
template <typename F>
void for_passes(const csb_matrix *m, const QuadPlan &qp, F f) {
    const SplitSpec &sp = m->plan.split;
    uint8_t slot[kQuadRows];
    for (int32_t bi = 0; bi < m->nbr; ++bi)
        for (int32_t bj = 0; bj < m->nbc; ++bj) {
            const size_t b = (size_t)bi * m->nbc + bj;
            const int nr = m->nrows[b], nc = m->ncols[b];
            if (nr == 0 || nc == 0) continue;
            const uint16_t *ri = m->rowidx.data() + m->row_off[b];
            for_column_parts(m, b, bj, [&](const ColPart &part) {
                int a = 0;
                while (a < nr) {
                    const int64_t gr = (int64_t)bi * m->br + ri[a];
                    const bool lower = !sp.active() || gr < sp.split_row;
                    if (lower ? !part.lower : !part.upper) { ++a; continue; }
                    const int64_t shift = part.shifted ? sp.shift : 0;
                    const uint32_t tile = (uint32_t)((gr + shift) / qp.tile_rows);
                    const int64_t row0 = (int64_t)tile * qp.tile_rows, end = row0 + qp.tile_rows;
                    int e = a;                           // the kernel rows of this tile
                    while (e < nr) {
                        const int64_t orow = (int64_t)bi * m->br + ri[e];
                        if ((!sp.active() || orow < sp.split_row) != lower || orow + shift >= end) break;
                        slot[e - a] = (uint8_t)(orow + shift - row0);
                        ++e;
                    }
                    for (int q = part.q0; q < part.q1; q += kQuadCols) {
                        const QPass p{(uint32_t)b, (uint16_t)a, (uint16_t)q, (uint8_t)(e - a), (uint8_t)std::min(kQuadCols, part.q1 - q),
                                      (uint8_t)part.shifted};
                        f(tile, p, part.second, slot);
                    }
                    a = e;
                }
            });
        }
}

}  // namespace

// Builds a section of tiles of `tile_rows` rows and appends it to the plan's image; leaves out->valid false where the
// matrix does not fit it, or the section the host's memory.
static void build_section(csb_matrix *m, uint32_t tile_rows, QuadPlan *out) {
    Plan &pl = m->plan;
    const size_t image_before = pl.image.size();
    *out = QuadPlan{};
    const int64_t rows = m->rows + (pl.split.active() ? pl.split.shift : 0);
    if (m->cols > kMaxStageCols || rows > 0x7fffffff || rows == 0) return;
    try {
        QuadPlan qp{};
        qp.rows = (uint32_t)rows;
        qp.tile_rows = tile_rows;
        qp.n_tiles = (qp.rows + qp.tile_rows - 1) / qp.tile_rows;
        qp.split_col = m->quad_split > 0 ? (uint32_t)m->quad_split : 0u;
        qp.val_fmt = (uint32_t)m->val_fmt;
        const bool bits16 = m->val_fmt != CSB_VAL_F32;

        // ---- the passes, dealt to the lists of their tiles as they come ------------------------
        struct Entry { QPass p; uint32_t list, pos, val; uint8_t second; uint8_t slot[kQuadRows]; };   // (val: from the list's first value)
        struct List { uint64_t work; uint32_t passes, bytes; };
        std::vector<Entry> entries;
        std::vector<List> lists((size_t)qp.n_tiles * kQuadLists, List{});
        uint64_t bytes = 0;
        uint32_t longest = 0;
        for_passes(m, qp, [&](uint32_t tile, const QPass &p, bool second, const uint8_t *slot) {
            List *best = &lists[(size_t)tile * kQuadLists];
            for (List *l = best + 1, *end = best + kQuadLists; l < end; ++l) if (l->work < best->work) best = l;
            entries.emplace_back();
            Entry &e = entries.back();
            e.p = p; e.second = second;
            e.list = (uint32_t)(best - lists.data()); e.pos = best->passes; e.val = best->bytes;
            std::memset(e.slot, kQuadRows, sizeof(e.slot));
            std::memcpy(e.slot, slot, p.nrows);
            const size_t n = pass_value_bytes(p.nrows, p.ncols, bits16);
            best->work += pass_cost(p);
            const uint32_t quads = (p.nrows + 3u) / 4u;
            qp.work.steps += quads * p.ncols; qp.work.rows += p.nrows;
            best->bytes += (uint32_t)n;
            longest = std::max(longest, ++best->passes);
            bytes += n;
        });
        qp.n_passes = entries.size();
        qp.work.passes = (double)qp.n_passes;
        double all = 0, most = 0;
        for (const List &l : lists) { all += (double)l.work; most = std::max(most, (double)l.work); }
        if (all > 0) qp.work.uneven = most * (double)lists.size() / all;
        qp.vals_bytes = bytes + kQuadPad;
        if (qp.vals_bytes >= 0x7fffff00ull || qp.n_passes >= 0x7fffffffull / sizeof(QuadRec)) return;
        // (the gaps are never read but for a count: half as many records again, or 4 MB, are worth the trip)
        if ((uint64_t)longest * lists.size() <= qp.n_passes + std::max<uint64_t>(qp.n_passes / 2, 65536)) qp.list_stride = std::max(longest, 1u);
        std::vector<uint32_t> table(lists.size() + 1, 0);
        for (size_t l = 0; l < lists.size(); ++l) table[l + 1] = table[l] + (uint32_t)(qp.list_stride ? qp.list_stride : lists[l].passes);
        qp.n_recs = table.back() + kQuadSpareRecs;

        // ---- image ------------------------------------------------------------------------------
        qp.off_table = align_up(pl.image.size(), 256);
        qp.off_recs = align_up(qp.off_table + table.size() * 4, 256);
        qp.off_vals = align_up(qp.off_recs + qp.n_recs * sizeof(QuadRec), 256);
        pl.image.resize(align_up(qp.off_vals + qp.vals_bytes, 256));
        uint8_t *im = pl.image.data();
        std::memcpy(im + qp.off_table, table.data(), table.size() * 4);
        auto *recs = (QuadRec *)(im + qp.off_recs);
        std::vector<uint32_t> val0(lists.size());            // values lie list after list
        uint32_t at = 0;
        for (size_t l = 0; l < lists.size(); ++l) {
            val0[l] = at;
            at += lists[l].bytes;
            if (lists[l].passes) recs[table[l]].list_len = lists[l].passes;
        }
        for (const Entry &e : entries) {
            const QPass &p = e.p;
            const uint32_t quads = (p.nrows + 3u) / 4u;
            QuadRec &r = recs[table[e.list] + e.pos];
            r.val = (val0[e.list] + e.val) / value_unit(bits16);
            r.stride = (uint16_t)pass_stride(quads, bits16);
            r.quads = (uint8_t)quads;
            r.flags = (uint8_t)((p.ncols > 4 ? kQuadWide : 0) | (e.second ? kQuadSecond : 0));
            const uint16_t *ci = m->colidx.data() + m->col_off[p.b];
            const uint32_t col0 = (uint32_t)(p.b % (uint32_t)m->nbc) * (uint32_t)m->bc - (e.second ? qp.split_col : 0u);
            for (int j = 0; j < kQuadCols; ++j) r.col[j] = j < p.ncols ? (uint16_t)(col0 + ci[p.q0 + j]) : kQuadNoCol;
            std::memcpy(r.slot, e.slot, sizeof(r.slot));
            for (uint32_t q = 0; q < p.nrows; ++q) r.rows |= 1u << e.slot[q];
            const int nc = m->ncols[p.b];
            const float *src = m->val.data() + m->val_off[p.b] + p.q0;
            uint8_t *dst = im + qp.off_vals + (size_t)r.val * value_unit(bits16);
            for (uint32_t q = 0; q < p.nrows; ++q) {
                const float *row = src + (size_t)(p.a0 + q) * nc;
                if (!bits16)
                    for (uint32_t j = 0; j < p.ncols; ++j) ((float *)dst)[value_at(quads, q, j, false)] = row[j];
                else
                    for (uint32_t j = 0; j < p.ncols; ++j)
                        ((uint16_t *)dst)[value_at(quads, q, j, true)] = m->val_fmt == CSB_VAL_F16 ? f32_to_f16_bits(row[j]) : f32_to_bf16_bits(row[j]);
            }
        }
        qp.valid = true;
        *out = qp;
    } catch (const std::bad_alloc &) {               // the section is for speed alone: products read the tile-based ones
        *out = QuadPlan{};
        pl.image.resize(image_before);               // (shrinks)
        return;
    }
}

// The section, or the two, that the batched products of a matrix read; none where it does not fit (they then read the
// tile-based sections).  Tiles of 16 rows alone where the blocks are no taller and tiles of 32 would not give each of 256
// workgroups one: a wavefront then has half the passes.  Taller blocks are cut by tiles of 16 rows, so that all tiles together
// have about twice the passes, of half the rows: better as long as they still find idle CUs (quad_us), which they never
// do beyond 256 tiles.
// None for the 16-bit values of a recurrent handle's gate matrix: its steps multiply float32 right-hand sides, and the
// products of 16-bit ones take passes from one source alone (LSTM 1024 -> 1024 at 12x in binary16: 15.8 MB of image, without
// them 8.5).
void plan_quad(csb_matrix *m) {
    Plan &pl = m->plan;
    pl.before_quad = pl.image.size();
    if (m->val_fmt != CSB_VAL_F32 && m->quad_split > 0) return;
    const int64_t rows = m->rows + (pl.split.active() ? pl.split.shift : 0);
    pl.quad_low = QuadPlan{};
    build_section(m, m->br <= 16 && rows < 256 * 32 ? 16u : 32u, &pl.quad);
    if (pl.quad.valid && m->br > 16 && rows <= 256 * 16) build_section(m, 16u, &pl.quad_low);
}

void drop_quad(csb_matrix *m) {
    m->plan.quad = m->plan.quad_low = QuadPlan{};
    m->plan.image.resize(m->plan.before_quad);           // (shrinks)
}

// The matrix belongs to a handle whose steps bring its columns from `split_col` on from a second source.  A plan that the
// caller made before knows nothing of that border: its sections are cut anew, as long as they are on the host alone (an image
// that is uploaded stays as it is, and its batched steps read the tile-based sections).
void cut_quad(csb_matrix *m, int64_t split_col) {
    m->quad_split = (int32_t)split_col;
    Plan &pl = m->plan;
    if (!pl.valid || m->uploaded || pl.quad.split_col == (uint32_t)split_col) return;
    const uint64_t told = std::max<uint64_t>(pl.bytes_told, pl.image.size());
    drop_quad(m);
    plan_quad(m);
    pl.bytes_told = told;
}

// Walks the section the way the kernels do, with bounds checks, and compares what it adds up with the matrix: every
// (output row, input column) must be multiplied once, by its value.
static int validate_section(const csb_matrix *m, const QuadPlan &qp) {
    const Plan &pl = m->plan;
    auto fail = [&](const char *what) { set_error(std::string("csb_plan_validate: quad section: ") + what); return CSB_EINVAL; };
    if (qp.off_vals + qp.vals_bytes > pl.image.size() || qp.off_recs + qp.n_recs * sizeof(QuadRec) > qp.off_vals) return fail("section size");
    const auto *table = (const uint32_t *)(pl.image.data() + qp.off_table);
    const auto *recs = (const QuadRec *)(pl.image.data() + qp.off_recs);
    const uint8_t *vals = pl.image.data() + qp.off_vals;
    const bool bits16 = qp.val_fmt != CSB_VAL_F32;
    const int64_t rows = m->rows + (pl.split.active() ? pl.split.shift : 0);
    if (qp.rows != (uint64_t)rows || qp.n_tiles != (rows + qp.tile_rows - 1) / qp.tile_rows) return fail("tiles");
    // what is expected: (output row, column) -> value, and how often it was seen
    const size_t cells = (size_t)rows * (size_t)m->cols;
    std::vector<float> expect(cells, 0.0f), got(cells, 0.0f);
    std::vector<uint8_t> in(cells, 0);
    size_t n_expect = 0, n_got = 0;
    for (int32_t bi = 0; bi < m->nbr; ++bi)
        for (int32_t bj = 0; bj < m->nbc; ++bj) {
            const size_t b = (size_t)bi * m->nbc + bj;
            for (int a = 0; a < m->nrows[b]; ++a)
                for (int q = 0; q < m->ncols[b]; ++q) {
                    int64_t row = (int64_t)bi * m->br + m->rowidx[m->row_off[b] + a];
                    const int64_t col = (int64_t)bj * m->bc + m->colidx[m->col_off[b] + q];
                    if (pl.split.active() && row >= pl.split.split_row && col >= pl.split.split_col) row += pl.split.shift;
                    const size_t cell = (size_t)row * (size_t)m->cols + (size_t)col;
                    expect[cell] = m->val[m->val_off[b] + (int64_t)a * m->ncols[b] + q];
                    in[cell] = 1;
                    ++n_expect;
                }
        }
    for (uint32_t t = 0; t < qp.n_tiles; ++t) {
        const int64_t row0 = (int64_t)t * qp.tile_rows, end = std::min<int64_t>(row0 + qp.tile_rows, rows);
        for (int l = 0; l < kQuadLists; ++l) {
            const size_t list = (size_t)t * kQuadLists + l;
            const uint64_t i0 = table[list];
            if (i0 + kQuadSpareRecs > qp.n_recs || table[list + 1] < i0 || table[list + 1] + kQuadSpareRecs > qp.n_recs) return fail("list");
            if (qp.list_stride && i0 != list * qp.list_stride) return fail("list stride");
            const uint64_t i1 = i0 + (qp.list_stride ? recs[i0].list_len : table[list + 1] - i0);
            if (i1 > table[list + 1] || (i1 > i0 && recs[i0].list_len != i1 - i0)) return fail("list length");
            if ((i1 - table[(size_t)t * kQuadLists]) * sizeof(QuadRec) > 0x7fffffffull) return fail("a tile's records");      // (byte offsets of 31 bits)
            for (uint64_t i = i0; i < i1; ++i) {
                const QuadRec &r = recs[i];
                uint32_t ncols = 0, nrows = 0;
                while (ncols < (uint32_t)kQuadCols && r.col[ncols] != kQuadNoCol) ++ncols;
                while (nrows < (uint32_t)kQuadRows && r.slot[nrows] != kQuadRows) ++nrows;
                const bool second = (r.flags & kQuadSecond) != 0;
                if (!ncols || !nrows || r.quads != (nrows + 3u) / 4u || r.stride != pass_stride(r.quads, bits16) ||
                    ((r.flags & kQuadWide) != 0) != (ncols > 4) || (second && !qp.split_col)) return fail("pass size");
                const size_t bytes = pass_value_bytes(nrows, ncols, bits16);
                const uint64_t val = (uint64_t)r.val * value_unit(bits16);
                if (val + bytes + kQuadPad > qp.vals_bytes) return fail("values");
                for (uint32_t j = ncols; j < (uint32_t)kQuadCols; ++j) if (r.col[j] != kQuadNoCol) return fail("gap in the columns");
                uint32_t places = 0;
                for (uint32_t q = 0; q < (uint32_t)kQuadRows; ++q) {
                    if (q >= nrows ? r.slot[q] != kQuadRows : q > 0 && r.slot[q] <= r.slot[q - 1]) return fail("gap in the rows, or their order");
                    if (q < nrows) places |= 1u << r.slot[q];
                }
                if (r.rows != places) return fail("row mask");
                for (uint32_t q = 0; q < (bits16 ? nrows : r.quads * 4u); ++q)
                    for (uint32_t j = 0; j < (bits16 ? (uint32_t)kQuadCols : (ncols + 3u) / 4u * 4u); ++j) {
                        float v;
                        if (!bits16) v = ((const float *)(vals + val))[value_at(r.quads, q, j, false)];
                        else {
                            const uint16_t bits = ((const uint16_t *)(vals + val))[value_at(r.quads, q, j, true)];
                            v = qp.val_fmt == CSB_VAL_F16 ? f16_bits_to_f32(bits) : bf16_bits_to_f32(bits);
                        }
                        if (q >= nrows || j >= ncols) {
                            if (v != 0.0f) return fail("value without an entry");
                            continue;
                        }
                        const int64_t row = row0 + r.slot[q], col = (int64_t)r.col[j] + (second ? qp.split_col : 0);
                        if (row >= end) return fail("row outside of its tile");
                        if (col >= m->cols || (qp.split_col && (col >= (int64_t)qp.split_col) != second)) return fail("column");
                        const size_t cell = (size_t)row * (size_t)m->cols + (size_t)col;
                        if (in[cell] != 1) return fail(in[cell] ? "entry multiplied twice" : "entry that the matrix does not have");
                        in[cell] = 2;
                        ++n_got;
                        got[cell] = v;
                    }
            }
        }
    }
    if (n_got != n_expect) return fail("entry missing");
    if (std::memcmp(expect.data(), got.data(), cells * sizeof(float)) != 0) return fail("values do not decode to the matrix");
    return CSB_OK;
}

int validate_quad(const csb_matrix *m) {
    const int rc = validate_section(m, m->plan.quad);
    return rc == CSB_OK && m->plan.quad_low.valid ? validate_section(m, m->plan.quad_low) : rc;
}

}  // namespace csb
