// Work maps of the launches: which tile (and which piece of the token axis) a workgroup owns, how a Gram call is cut
// into pieces, how wide the sweep's super-blocks are.  Plain integer logic shared by the kernels (device) and the
// launchers (host); it compiles as ordinary C++ too, so that a host program can enumerate the maps and check that
// every tile is owned exactly once (tests/planner_check.cpp).  No arithmetic of the method lives here.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define ONECOMP_HD __host__ __device__ inline
#else
#define ONECOMP_HD inline
#endif

namespace onecomp {
namespace plan {

ONECOMP_HD int imin(int a, int b) { return a < b ? a : b; }
ONECOMP_HD int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- symmetric Gram, square tiles: rank v in the banded order -> (ti, tk), ti <= tk < n_t.  Bands of GRAM_BAND tile
// rows; inside a band first the triangle on the diagonal (column by column), then the rectangle right of it column
// by column, rows fastest.
constexpr int GRAM_BAND = 4;
template <int BAND>
ONECOMP_HD void tile_from_rank_band(int v, int n_t, int& ti, int& tk) {
    int a = 0;
    while (true) {
        int rows = imin(BAND, n_t - a * BAND);
        int cols = n_t - a * BAND;
        int cnt = rows * cols - rows * (rows - 1) / 2;
        if (v < cnt) {
            int tri = rows * (rows + 1) / 2;
            if (v < tri) {
                int c = 0;
                while ((c + 1) * (c + 2) / 2 <= v) ++c;
                tk = a * BAND + c;
                ti = a * BAND + (v - c * (c + 1) / 2);
            } else {
                int w = v - tri;
                tk = a * BAND + rows + w / rows;
                ti = a * BAND + w % rows;
            }
            return;
        }
        v -= cnt;
        ++a;
    }
}
ONECOMP_HD void tile_from_rank(int v, int n_t, int& ti, int& tk) { tile_from_rank_band<GRAM_BAND>(v, n_t, ti, tk); }
// ---- factor: the tiles of a trailing update.  The trailing matrix has n_t block columns; a launch updates column 0 (its
// first tile is the next diagonal block) and the columns 1, 1 + stride, 1 + 2 stride, ...: tiles (tm, tn), tn <= tm < n_t.
// Workgroup 0 owns tile (0, 0) (and factors it: it has been brought up to date before the launch), the next ones the
// strided columns, dealt to the XCDs in runs of consecutive ranks (bands of SYRK_BAND of these columns walked row by row:
// two workgroups per CU, 64 tiles of an XCD in flight, an 8 x 8 patch of them shares 16 operand panels), the last ones the
// rest of column 0.
constexpr int SYRK_BAND = 8;
struct SyrkGrid {
    int n_t, stride, n_c, n_s, chunk, total;   // strided columns and their tiles, ranks per XCD, workgroups
};
ONECOMP_HD SyrkGrid syrk_grid(int n_t, int stride) {
    SyrkGrid q;
    q.n_t = n_t;
    q.stride = stride;
    q.n_c = n_t > 1 ? (n_t - 2) / stride + 1 : 0;
    q.n_s = q.n_c * (n_t - 1) - stride * (q.n_c * (q.n_c - 1) / 2);
    q.chunk = (q.n_s + 7) >> 3;
    q.total = 1 + 8 * q.chunk + (n_t - 1);
    return q;
}
// Returns false for a workgroup with nothing to do.
ONECOMP_HD bool syrk_tile(int bid, const SyrkGrid& q, int& tm, int& tn) {
    tn = 0;
    tm = 0;
    if (bid == 0) return true;
    const int u = bid - 1;
    if (u >= 8 * q.chunk) {
        tm = u - 8 * q.chunk + 1;
        return tm < q.n_t;
    }
    int v = (u & 7) * q.chunk + (u >> 3);
    if (v >= q.n_s) return false;
    for (int c0 = 0;; c0 += SYRK_BAND) {
        const int cols = imin(SYRK_BAND, q.n_c - c0), first = 1 + q.stride * c0, rows = q.n_t - first;
        const int steps = (cols - 1) * q.stride;   // rows that do not reach every column of the band
        const int head = q.stride * (cols * (cols - 1) / 2), cnt = head + (rows - steps) * cols;
        if (v >= cnt) {
            v -= cnt;
            continue;
        }
        int r, c;
        if (v < head) {
            int i = 1;   // columns that the row reaches
            while (v >= q.stride * i) v -= q.stride * i++;
            r = (i - 1) * q.stride + v / i;
            c = v % i;
        } else {
            r = steps + (v - head) / cols;
            c = (v - head) % cols;
        }
        tm = first + r;
        tn = first + q.stride * c;
        return true;
    }
}
// Every column but the next one is brought up to date in every lag-th launch only, by all panels solved since: column
// tn of the trailing matrix behind block `step` still lacks the panels [syrk_first_panel, step] (`base`: the first
// panel after the last launch that updated every column).
ONECOMP_HD int syrk_first_panel(int tn, int step, int lag, int base) {
    const int k = step - (lag - tn % lag) % lag;
    return k > base ? k : base;
}
// Lag while n_t block columns trail: 4 halves the bytes once more, but a launch has half as many tiles, twice as long, and
// its last round of them costs more the fewer there are.  Per step, us, with lag 1 / 2 / 4 (d_in 28672, mean over 24
// steps): 223 - 200 trailing: 1906 / 1618 / 1470; 151 - 128: 810 / 725 / 700; 103 - 80: 367 / 334 / 334; 79 - 56: 211 / 197 /
// 207; 31 - 8: 48 / 46 / 50.  Lag 8: 1341, 725, 375 and 242.
constexpr int SYRK_LAG4_MIN = 80;
// With few columns a launch is as long as its longest workgroup: a 128 x 128 tile of k = 256 is 40 us on its CU, the next
// diagonal block 14, so every column is updated in every step and the tiles are half as wide (syrk_narrow_tile).
// Cholesky alone, us, narrow below 2 / 32 / 48 / 56 / 64 / 80 columns (with a diagonal block of 18): d_in 2048: 820 / 545 /
// 544 / - ..; 4096: 1798 / 1357 / 1357 / - ..; 8192: 6027 / 5598 / 5387 / 5386 / 5528 / 5600; 14336: 21957 / - / 21270 /
// 21226 / 21346 / 21822.  Narrow tiles with lag 2 are slower up to d_in 4096 (3 %) and not faster at 6144.
constexpr int SYRK_LAG2_MIN = 56;
ONECOMP_HD int syrk_lag(int n_t) { return n_t >= SYRK_LAG4_MIN ? 4 : n_t >= SYRK_LAG2_MIN ? 2 : 1; }
// Launches with lag 1: tiles of 128 rows x 64 columns, tile (tm, tc) with tc < 2 (tm + 1), 1 <= tm < n_t (block (0, 0) has
// been brought up to date before), row by row; then, in a factor whose inverse goes along, its update: tiles (tm, tc) of
// n_t block rows by inv_cols columns, row by row.  A run of consecutive ranks per XCD; workgroup 0 has the diagonal block.
ONECOMP_HD int syrk_narrow_tiles(int n_t, int inv_cols) { return n_t * (n_t + 1) - 2 + n_t * inv_cols; }
ONECOMP_HD int syrk_narrow_grid(int n_t, int inv_cols) { return 1 + ((syrk_narrow_tiles(n_t, inv_cols) + 7) & ~7); }
ONECOMP_HD bool syrk_narrow_tile(int bid, int n_t, int inv_cols, int& tm, int& tc, bool& inverse) {
    const int n = syrk_narrow_tiles(n_t, inv_cols), n_syrk = syrk_narrow_tiles(n_t, 0), chunk = (n + 7) >> 3, u = bid - 1;
    const int v = (u & 7) * chunk + (u >> 3);
    if (v >= n) return false;
    inverse = v >= n_syrk;
    if (inverse) {
        tm = (v - n_syrk) / inv_cols;
        tc = (v - n_syrk) % inv_cols;
        return true;
    }
    // row tm begins at rank tm (tm + 1) - 2 (a walk over the rows: half a microsecond per workgroup)
    tm = int(0.5f * __builtin_sqrtf(4.0f * float(v + 2) + 1.0f) - 0.5f);
    if (tm * (tm + 1) > v + 2) --tm;
    if ((tm + 1) * (tm + 2) <= v + 2) ++tm;
    tc = v + 2 - tm * (tm + 1);
    return true;
}
// Launches inside a slab of a left-looking factorization (factor_slabs), which has `cols` >= 1 block columns left: the tiles
// above of the first 2 cols columns only.
ONECOMP_HD int syrk_slab_tiles(int n_t, int cols) {
    const int c = imin(cols, n_t);
    return c * (c + 1) - 2 + 2 * c * (n_t - c);
}
ONECOMP_HD int syrk_slab_grid(int n_t, int cols) { return 1 + ((syrk_slab_tiles(n_t, cols) + 7) & ~7); }
ONECOMP_HD bool syrk_slab_tile(int bid, int n_t, int cols, int& tm, int& tc) {
    const int c = imin(cols, n_t), n = syrk_slab_tiles(n_t, cols), chunk = (n + 7) >> 3, u = bid - 1;
    const int v = (u & 7) * chunk + (u >> 3) + 2;   // the two tiles of row 0 are not there
    if (v >= n + 2) return false;
    const int head = c * (c + 1);   // rows 0 .. c - 1
    if (v >= head) {
        tm = c + (v - head) / (2 * c);
        tc = (v - head) % (2 * c);
        return true;
    }
    tm = 0;
    while ((tm + 1) * (tm + 2) <= v) ++tm;
    tc = v - tm * (tm + 1);
    return true;
}
// Factors of up to this many blocks take their inverse along (factor_run), wider ones have it by recursive doubling
// afterwards, in products with longer inner ranges.  Afterwards : along, us: d_in 512 186 : 144 and 2048 729 : 594 (with a
// diagonal block of 18 us), 4096 1659 : 1533, 5120 2572 : 2495, 6144 3727 : 3765, 6784 4727 : 4751.
constexpr int INVERSE_ALONG_MAX = 40;
ONECOMP_HD int n_upper_tiles(int n_t) { return n_t * (n_t + 1) / 2; }

// ---- symmetric Gram, 128 x 256 tiles: tile (i, k) = rows [128 i, +128) x columns [256 k, +256) is computed when it
// reaches above the diagonal (k >= i / 2).  Bands of GRAM_RBAND tile rows, inside a band column by column, rows fastest.
constexpr int GRAM_RBAND = 8;
ONECOMP_HD void tile128_from_rank(int v, int n_rt, int n_ct, int& ti, int& tk) {
    for (int a = 0;; ++a) {
        const int r0 = a * GRAM_RBAND, rows = imin(GRAM_RBAND, n_rt - r0);
        for (int k = r0 / 2; k < n_ct; ++k) {
            const int valid = imin(rows, 2 * k + 2 - r0);   // rows r0 .. r0+valid-1 satisfy i / 2 <= k
            if (v < valid) { ti = r0 + v; tk = k; return; }
            v -= valid;
        }
    }
}
ONECOMP_HD int n_tiles128(int n_rt, int n_ct) {
    int n = 0;
    for (int i = 0; i < n_rt; ++i) n += n_ct - i / 2;
    return n;
}

// ---- symmetric Gram, 384 x 256 tiles: tile (i, k) = rows [384 i, +384) x columns [256 k, +256) is computed when it
// reaches above the diagonal (256 (k + 1) > 384 i, i.e. k >= floor(3 i / 2)).  Bands of GRAM_BAND tile rows, inside a
// band column by column, rows fastest.
ONECOMP_HD void tile_wide_from_rank(int v, int n_rt, int n_ct, int& ti, int& tk) {
    for (int a = 0;; ++a) {
        const int r0 = a * GRAM_BAND, rows = imin(GRAM_BAND, n_rt - r0);
        for (int k = 3 * r0 / 2; k < n_ct; ++k) {
            const int valid = imin(rows, (2 * k + 1) / 3 - r0 + 1);   // rows r0 .. r0+valid-1 satisfy 3 i / 2 <= k
            if (v < valid) { ti = r0 + v; tk = k; return; }
            v -= valid;
        }
    }
}
ONECOMP_HD int n_tiles_wide(int n_rt, int n_ct) {
    int n = 0;
    for (int i = 0; i < n_rt; ++i) n += n_ct - 3 * i / 2;
    return n;
}

// ---- cross-Gram (every tile): bands of GRAM_BAND tile rows, column by column inside a band
ONECOMP_HD void cross_tile_from_rank(int v, int n_rt, int n_ct, int& ti, int& tk) {
    const int band = imin(v / (GRAM_BAND * n_ct), (n_rt - 1) / GRAM_BAND);
    const int w = v - band * GRAM_BAND * n_ct, rows = imin(GRAM_BAND, n_rt - band * GRAM_BAND);
    tk = w / rows;
    ti = band * GRAM_BAND + w % rows;
}

// ---- ring kernel: workgroup `bid` of the whole schedule -> tile rank and piece.
// Workgroups 0 .. 8 chunk - 1 take whole tiles: the ranks outside [split0, split0 + n_split), `chunk` of them per
// XCD (hardware deals consecutive workgroups round-robin to the 8 XCDs, so workgroup b takes position
// (b % 8) * chunk + b / 8: each XCD owns a contiguous run of the order).  The workgroups after them take the n_split
// tiles of that range in n_piece pieces of the token axis each, an eighth of all pieces per XCD; on an XCD the pieces run tile
// after tile for one range of tokens, then for the next.  Returns false for a workgroup with nothing to do.
// (With an eighth of the tiles and all their pieces instead, 36 tiles in 7 pieces are 35 workgroups on seven XCDs of 32 CUs and 7 on
// the last: a second round.  us of a call, so : pieces dealt: d_in 1408, 32768 tokens 148 : 98; 2048, 32768
// 236 : 153; 3072, 32768 411 : 376; 3584, 16384 307 : 264; 8192, 98304 5960 : 5540.)
struct RingWork {
    int v;         // tile rank in the order of the tile map
    int piece;     // -1: the whole token axis; else the piece number
    int m_split;   // index of the tile among the split ones
};
ONECOMP_HD bool ring_work(int bid, int chunk, int n_tiles, int split0, int n_split, int n_piece, RingWork& w) {
    w.piece = -1;
    w.m_split = 0;
    if (bid < 8 * chunk) {
        w.v = (bid & 7) * chunk + (bid >> 3);
        if (w.v >= n_tiles - n_split) return false;
        if (w.v >= split0) w.v += n_split;
        return true;
    }
    // an XCD's run of (tile, piece): the first tile from piece s0 on, the last one up to piece l1; taken piece by piece
    const int b = bid - 8 * chunk, total = n_split * n_piece, per_xcd = (total + 7) >> 3, j = b >> 3;
    const int first = (b & 7) * per_xcd, end = imin(first + per_xcd, total);
    if (first + j >= end) return false;
    const int t0 = first / n_piece, t1 = (end - 1) / n_piece, s0 = first - t0 * n_piece, l1 = end - t1 * n_piece;
    int p = 0, before = 0;   // pieces of the run with numbers below p
    for (;; ++p) {
        const int here = t1 - t0 + 1 - (p < s0) - (p >= l1);
        if (j < before + here) break;
        before += here;
    }
    w.piece = p;
    w.m_split = t0 + (p < s0) + j - before;
    w.v = split0 + w.m_split;
    return true;
}
// total workgroups of the schedule
ONECOMP_HD int ring_total_blocks(int chunk, int n_split, int n_piece) { return chunk * 8 + 8 * int(cdiv(n_split * n_piece, 8)); }
// tokens [t_begin, t_begin + count) of a piece: whole steps of kt tokens; count <= 0: nothing left for this piece
ONECOMP_HD void piece_tokens(int64_t n_tokens, int n_piece, int piece, int kt, int64_t& t_begin, int64_t& count) {
    const int64_t n_st_all = (n_tokens + kt - 1) / kt;
    const int64_t t_piece = (n_st_all + n_piece - 1) / n_piece * kt;
    t_begin = piece * t_piece;
    count = n_tokens - t_begin < t_piece ? n_tokens - t_begin : t_piece;
}

// ---- which 256 x 256 tiles of the symmetric Gram are computed in pieces of the token axis, and the estimated
// duration of the launch in units of one whole tile on one CU.
// Without a workspace only two pieces per tile are possible (the second partial sum is parked in the tile's mirror
// position), for tiles strictly above the diagonal and inside the matrix: the short last round is taken from the
// rectangular part of the first band.  With a workspace any tile can be cut into 2 .. 16 pieces: either the tiles
// left over after whole rounds, or all of them when there are fewer than two rounds.  A piece costs its share of
// the tile plus about half a percent of a tile for filling the pipeline and storing the partial sum, and it must
// keep at least 2048 tokens.
// ws_slots: how many 256 x 256 partial sums the workspace holds (0: none).
struct SplitPlan {
    int split0 = 0, n_split = 0, n_piece = 1;
    bool use_ws = false;
    double rounds = 0.0;
};
// mirror_ok: the tiles are 256 x 256, so the workspace-free form exists (other tile shapes split only with a workspace,
// whose slots are then partial sums of that shape).
inline SplitPlan plan_split(int64_t n_tiles, int64_t n_ct, int64_t d_in, int64_t n_tokens, int n_cus, int64_t ws_slots,
                            bool mirror_ok = true) {
    SplitPlan best;
    best.rounds = double(cdiv(n_tiles, n_cus));
    const int64_t r = n_tiles % n_cus;
    if (mirror_ok && r > 0 && r <= n_cus / 2 && n_tokens >= 1024 && n_ct >= GRAM_BAND + cdiv(r, GRAM_BAND) &&
        (GRAM_BAND + cdiv(r, GRAM_BAND)) * 256 <= d_in) {
        best.split0 = GRAM_BAND * (GRAM_BAND + 1) / 2;
        best.n_split = int(r);
        best.n_piece = 2;
        best.rounds = double(n_tiles / n_cus) + 0.5 * 1.06;
    }
    const int max_pc = mirror_ok ? 16 : 8;   // the larger slots of the other shapes: fewer of them
    for (int pc = 2; pc <= max_pc; ++pc) {
        // Pieces of 512 tokens and more where all pieces together leave a third of the CUs idle (short_pieces_bf16): what is written and
        // read back grows with their number, and beyond some 150 of 256 KB faster than it.
        const bool long_pieces = n_tokens / pc >= 2048;
        if (!long_pieces && !(mirror_ok && n_tokens / pc >= 512 && 3 * n_tiles * pc <= 2 * n_cus)) break;
        const double piece_cost = 1.0 / pc + 0.005;
        if (long_pieces && r > 0 && n_tiles > n_cus && r * pc <= ws_slots) {   // the leftover tiles, from the end of the rank order
            const double rounds = double(n_tiles / n_cus) + double(cdiv(r * pc, n_cus)) * piece_cost;
            if (rounds < best.rounds) best = SplitPlan{int(n_tiles - r), int(r), pc, true, rounds};
        }
        if (n_tiles < 2 * n_cus && n_tiles * pc <= ws_slots) {   // every tile
            const double rounds = double(cdiv(n_tiles * pc, n_cus)) * piece_cost;
            if (rounds < best.rounds) best = SplitPlan{0, int(n_tiles), pc, true, rounds};
        }
    }
    return best;
}

// ---- sweep: far-update tiles.  Workgroup bid -> tile (mt, nt) of n_mt x n_nt; each XCD (bid % 8) owns a contiguous
// run of `chunk` positions, m fastest inside bands of TRAIL_BAND row tiles.  Returns false for an idle workgroup.
constexpr int TRAIL_BAND = 8;
ONECOMP_HD bool trail_tile(int bid, int chunk, int n_mt, int n_nt, int& mt, int& nt) {
    const int v = (bid & 7) * chunk + (bid >> 3);
    if (v >= n_mt * n_nt) return false;
    const int band = imin(v / (TRAIL_BAND * n_nt), (n_mt - 1) / TRAIL_BAND);
    const int rem = v - band * TRAIL_BAND * n_nt;
    const int mb = imin(TRAIL_BAND, n_mt - TRAIL_BAND * band);
    mt = band * TRAIL_BAND + rem % mb;
    nt = rem / mb;
    return true;
}

// Products with a triangular right operand: workgroup bid -> tile (mt, nt), the columns with the longest inner ranges first
// (lower: the left ones), so that the short ones fill up the last round; behind the first `fold` tiles the shortest first.
ONECOMP_HD bool triangular_tile(int bid, int n_mt, int n_nt, bool lower, int fold, int& mt, int& nt) {
    const int total = n_mt * n_nt;
    if (bid >= total) return false;
    const int v = bid < fold ? bid : fold + total - 1 - bid, rank = v / n_mt;
    mt = v % n_mt;
    nt = lower ? rank : n_nt - 1 - rank;
    return true;
}

// ---- sweep: the feedback sums of a panel workgroup's `rows` rows, read from the working copy into MFMA accumulators:
// lane `lane`, register r of row tile mt, column col; byte offsets from the first of the rows.  A buffer load's scalar
// offset is no part of its bounds check, so only whole workgroups (rows == PANEL_ROWS) may step through the rows with it;
// in a short one the row is part of the lane's offset, and rows past the end read the last one again.
constexpr int PANEL_ROWS = 64;
struct FeedbackOffset {
    uint32_t lane, scalar;
};
template <bool WHOLE>
ONECOMP_HD FeedbackOffset panel_feedback_offset(int rows, int d_in, int lane, int mt, int r, int col) {
    const int lane_row = (lane >> 5) * 4, row = mt * 32 + (r / 4) * 8 + (r % 4);
    if (WHOLE) return {uint32_t(lane_row * d_in + col) * 4, uint32_t(row) * uint32_t(d_in) * 4};
    return {uint32_t(imin(lane_row + row, rows - 1) * d_in + col) * 4, 0u};
}

// ---- sweep: width of a super-block.  512 columns; for groups wider than a 128-column block that are not the whole
// row, the largest of 512 / 384 / 256 / 128 that divides the group, so that a group is a run of whole super-blocks.
inline int sweep_superblock_width(int group_size, int64_t d_in) {
    if (group_size > 128 && group_size != d_in)
        for (int c = 512; c >= 128; c -= 128)
            if (group_size % c == 0) return c;
    return 512;
}

}  // namespace plan
}  // namespace onecomp
