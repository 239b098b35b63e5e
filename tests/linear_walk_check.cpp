// Follows the loads of every work-group of a linear layer through the library's own walk (csrc/linear_walk.h), on the CPU.
#include "linear_walk.h"

#include <stddef.h>

#include <vector>

using namespace ragged;

namespace {

enum { kOk = 0, kTileTwice = 1, kTileMissed = 2, kWrongPlace = 3, kLiveOutOfRange = 4, kReadsPastTheEnd = 5, kWorkWithoutRows = 6 };

// One step's loads of an operand of `end` rows; want: the (first, step) that the arithmetic needs there, or first < 0.
int check_loads(const LinearCursor& c, int tile_rows, int64_t end, uint32_t row_bytes, int want_first, uint32_t want_soff) {
    if (want_first >= 0 && (c.first != want_first || c.soff != want_soff)) return kWrongPlace;
    const int64_t live = end - c.first < tile_rows ? end - c.first : tile_rows;
    const int64_t rows[] = {0, 1, live - 1, live, live + 1, tile_rows - 1};
    for (const int64_t r : rows) {
        if (r < 0 || r >= tile_rows) continue;
        for (uint32_t chunk = 0; chunk < 128; chunk += 112) {
            const uint32_t voff = (uint32_t)r * row_bytes + chunk;
            const bool in_range[2] = {voff < c.bytes, voff < c.bytes - c.soff};       // the two readings of the range check
            const bool inside = c.first * (int64_t)row_bytes + voff + c.soff + 16 <= end * (int64_t)row_bytes;
            for (const bool reads : in_range) {
                if (reads && !inside) return kReadsPastTheEnd;
                if (want_first >= 0 && r < live && !reads) return kLiveOutOfRange;
            }
        }
    }
    return kOk;
}

template <int NJ, int MT, int PER_CU>
int check(int rows_cap, int rows, int N, int K) {
    typedef LinearShape<NJ, MT, PER_CU> S;
    const LinearGrid grid(NJ, MT, PER_CU, rows_cap, N);
    const uint32_t row_bytes = (uint32_t)K * 2u;
    const int ksteps = K / kTK;
    const int64_t valid = rows < 0 ? 0 : rows;
    const int m_tiles = (int)((valid + S::TM - 1) / S::TM);
    std::vector<int> seen((size_t)m_tiles * grid.n_tiles, 0);
    for (int block = 0; block < grid.groups; ++block) {
        const LinearWalk walk(rows, S::TM, grid.n_tiles, grid.panel, 0xFFFFFFFFu / grid.panel, 0xFFFFFFFFu / grid.last, block, grid.groups);
        if (walk.t_first >= walk.t_end) continue;
        if (valid == 0) return kWorkWithoutRows;
        std::vector<int> m0s, n0s;
        for (int t = walk.t_first; t < walk.t_end; t += walk.stride) {
            int m0, n0;
            walk.tile_of(t, S::TM, S::TN, m0, n0);
            if (m0 < 0 || m0 >= rows || n0 < 0 || n0 + S::TN > N) return kWrongPlace;
            if (seen[(size_t)(m0 / S::TM) * grid.n_tiles + n0 / S::TN]++) return kTileTwice;
            m0s.push_back(m0);
            n0s.push_back(n0);
        }
        const int steps = (int)m0s.size() * ksteps;
        LinearCursor x, w;
        x.tile = w.tile = walk.t_first;
        x.set<S::TM, S::TN, true>(walk, row_bytes);
        w.set<S::TM, S::TN, false>(walk, row_bytes);
        for (int i = 0; i < steps + S::kAheadX; ++i) {         // what is loaded in front of the loop, then one step's per step
            const int err = check_loads(x, S::TM, valid, row_bytes, i < steps ? m0s[i / ksteps] : -1, i % ksteps * kTK * 2u);
            if (err) return err;
            x.next<S::TM, S::TN, true>(walk, row_bytes);
        }
        for (int i = 0; i < steps + S::kAheadW; ++i) {
            const int err = check_loads(w, S::TN, N, row_bytes, i < steps ? n0s[i / ksteps] : -1, i % ksteps * kTK * 2u);
            if (err) return err;
            w.next<S::TM, S::TN, false>(walk, row_bytes);
        }
    }
    for (const int n : seen)
        if (n != 1) return kTileMissed;
    return kOk;
}

}  // namespace

extern "C" {

int linear_walk_check(int nj, int mt, int per_cu, int rows_cap, int rows, int N, int K) {
#define CASE(NJ, MT, PER_CU) if (nj == NJ && mt == MT && per_cu == PER_CU) return check<NJ, MT, PER_CU>(rows_cap, rows, N, K);
    LINEAR_SHAPES(CASE)
#undef CASE
    return -1;
}

int linear_shape_count(void) {
    int n = 0;
#define CASE(NJ, MT, PER_CU) ++n;
    LINEAR_SHAPES(CASE)
#undef CASE
    return n;
}

// {nj, mt, per_cu, LDS stages} of shape i
void linear_shape(int i, int* out) {
#define CASE(NJ, MT, PER_CU) if (i-- == 0) { out[0] = NJ; out[1] = MT; out[2] = PER_CU; out[3] = LinearShape<NJ, MT, PER_CU>::kStages; }
    LINEAR_SHAPES(CASE)
#undef CASE
}

// The table that the rule chooses from
int linear_table_size(void) { return (int)(sizeof(kTileShapes) / sizeof(kTileShapes[0])); }
void linear_table_shape(int i, int* out) {
    out[0] = kTileShapes[i].nj;
    out[1] = kTileShapes[i].mt;
    out[2] = kTileShapes[i].per_cu;
}

// {nj, mt, per_cu, tiles of a call over `rows` rows} of the shape that the rule picks
void linear_pick(int rows_hint, int rows, int N, int K, int act, int* out) {
    const TileShape c = pick_linear_shape(rows_hint, N, K, act);
    out[0] = c.nj;
    out[1] = c.mt;
    out[2] = c.per_cu;
    out[3] = (rows + 32 * c.mt - 1) / (32 * c.mt) * (N / (32 * c.nj));
}

}  // extern "C"
