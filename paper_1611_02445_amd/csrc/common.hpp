// Shared definitions of the tiled LBM library: error reporting, the D3Q19
// velocity set as compile-time tables, and the device-side table layout.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>

#include "lbm.h"

namespace tlbm {

// ---------------------------------------------------------------------------
// errors: a thread-local message behind lbm_last_error()
// ---------------------------------------------------------------------------
int fail(int code, const char *fmt, ...);
void clear_error();

// ---------------------------------------------------------------------------
// D3Q19 (Section 2.2, Fig. 1 caption; weights listed after Eq. 4).
// 0 rest; 1..6 E N W S T B; 7..18 NE NW SW SE ET EB WT WB NT NB ST SB.
// ---------------------------------------------------------------------------
constexpr int Q = 19;
constexpr int CX[Q] = {0, 1, 0, -1, 0, 0, 0, 1, -1, -1, 1, 1, 1, -1, -1, 0, 0, 0, 0};
constexpr int CY[Q] = {0, 0, 1, 0, -1, 0, 0, 1, 1, -1, -1, 0, 0, 0, 0, 1, 1, -1, -1};
constexpr int CZ[Q] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1};

constexpr int opposite(int i) {
    for (int j = 0; j < Q; ++j)
        if (CX[j] == -CX[i] && CY[j] == -CY[i] && CZ[j] == -CZ[i]) return j;
    return -1;
}
constexpr double weight(int i) { return i == 0 ? 1.0 / 3.0 : (i <= 6 ? 1.0 / 18.0 : 1.0 / 36.0); }

// multiple relaxation times: moment k of direction i, the D3Q19 basis of
// d'Humieres, Ginzburg, Krafczyk, Lallemand and Luo (2002) written as
// polynomials of c (rho, e, eps, j_x, q_x, j_y, q_y, j_z, q_z, 3p_xx, 3pi_xx,
// p_ww, pi_ww, p_xy, p_yz, p_xz, m_x, m_y, m_z); the rows are orthogonal
constexpr int mrt_coef(int k, int i) {
    const int cx = CX[i], cy = CY[i], cz = CZ[i];
    const int c2 = cx * cx + cy * cy + cz * cz;
    switch (k) {
    case 0: return 1;
    case 1: return 19 * c2 - 30;
    case 2: return (21 * c2 * c2 - 53 * c2 + 24) / 2;
    case 3: return cx;
    case 4: return (5 * c2 - 9) * cx;
    case 5: return cy;
    case 6: return (5 * c2 - 9) * cy;
    case 7: return cz;
    case 8: return (5 * c2 - 9) * cz;
    case 9: return 3 * cx * cx - c2;
    case 10: return (3 * cx * cx - c2) * (3 * c2 - 5);
    case 11: return cy * cy - cz * cz;
    case 12: return (cy * cy - cz * cz) * (3 * c2 - 5);
    case 13: return cx * cy;
    case 14: return cy * cz;
    case 15: return cx * cz;
    case 16: return (cy * cy - cz * cz) * cx;
    case 17: return (cz * cz - cx * cx) * cy;
    default: return (cx * cx - cy * cy) * cz;
    }
}
constexpr int mrt_norm(int k) {
    int n = 0;
    for (int i = 0; i < Q; ++i) n += mrt_coef(k, i) * mrt_coef(k, i);
    return n;
}
// the same as a table, evaluated by the compiler
struct MrtTable {
    int c[Q][Q];
    int n[Q];
};
constexpr MrtTable make_mrt_table() {
    MrtTable t{};
    for (int k = 0; k < Q; ++k) {
        for (int i = 0; i < Q; ++i) t.c[k][i] = mrt_coef(k, i);
        t.n[k] = mrt_norm(k);
    }
    return t;
}
constexpr MrtTable MRT = make_mrt_table();
// relaxation rate of moment k; 0 marks the conserved moments (rho, j), whose
// non-equilibrium part vanishes; -1 marks the viscous moments (rate 1/tau)
constexpr double mrt_rate(int k) {
    switch (k) {
    case 0: case 3: case 5: case 7: return 0.0;
    case 1: return 1.19;
    case 2: case 10: case 12: return 1.4;
    case 4: case 6: case 8: return 1.2;
    case 16: case 17: case 18: return 1.98;
    default: return -1.0;
    }
}

// Opposite directions pair up (9 pairs, the lower index first); every moment
// row is either even or odd under c -> -c (the scalar and tensor moments even,
// the vector ones odd)
constexpr int pair_first(int p) {
    int n = 0;
    for (int i = 1; i < Q; ++i) {
        if (opposite(i) < i) continue;
        if (n == p) return i;
        ++n;
    }
    return -1;
}
constexpr int NPAIR = 9;
constexpr bool mrt_row_odd(int k) {
    for (int i = 1; i < Q; ++i)
        if (mrt_coef(k, i) != -mrt_coef(k, opposite(i))) return false;
    return true;
}

// lane n = x + 4y + 16z inside a tile (the XYZ map of Eq. 11)
constexpr int TILE = 64;

// ---------------------------------------------------------------------------
// lattice layout
//   runs  (FP64, FP32): tile t with k fluid nodes owns one contiguous run of
//         19*k values, direction i at base[t] + i*k + slot, slot = number of
//         fluid nodes of the tile below the node; the run is padded to whole
//         128-byte lines
//   plain (FP16): tile t owns 19 blocks of 64 values at t*19*64 + i*64 + n;
//         a block is exactly one 128-byte line
// ---------------------------------------------------------------------------
inline size_t storage_size(int storage) { return storage == LBM_F64 ? 8 : (storage == LBM_F32 ? 4 : 2); }
// Per-node fields with three components (the force density and its
// gradient) are kept per fluid slot as well: tile t owns 3*k entries at
// fbase[t] + c*k + slot (c = x, y, z), padded to a multiple of FIELD_PAD
// entries (128 bytes of FP64, 64 of FP32).
constexpr uint64_t FIELD_PAD = 16;
inline uint64_t field_elems(uint64_t mask) {
    const uint64_t k = (uint64_t)__builtin_popcountll(mask);
    return (3 * k + FIELD_PAD - 1) / FIELD_PAD * FIELD_PAD;
}
inline bool runs_layout(int storage) { return storage != LBM_F16S; }
inline uint64_t run_elems(uint64_t mask, int storage) {
    const uint64_t L = 128 / storage_size(storage);
    const uint64_t k = (uint64_t)__builtin_popcountll(mask);
    return (Q * k + L - 1) / L * L;
}

// ---------------------------------------------------------------------------
// device table layout inside the caller's `tables` buffer
//   [rec_off]    TileRec per tile: fluid mask, element offset of its data
//   [row_off]    NbRow per tile, 256 bytes on a 256-byte boundary: the fluid
//                masks and 32-bit data offsets of the 19 tiles a D3Q19 step
//                reads from (the tile itself, 6 face and 12 edge neighbours;
//                corners are never needed; mask 0 for a missing tile), the
//                offsets in elements for the kernels with 32-bit
//                lattice offsets and in lines of 128 bytes, where every
//                tile's data begins, for the others; the entry offset of the tile's per-node field run and its corner
//   [xyz_off]    int32  [n_tiles][4]: corner x, y, z, 0
//   [fld_off]    uint64 [n_tiles]: entry offset of the tile's per-node field run
//   [map_off]    int32  [tz][ty][tx]: device tile number of each tile of the
//                box, -1 for a dropped one (kernels that walk a dense array;
//                absent where they do not)
// The neighbourhood is gathered once on the host, so a wave reads it with a
// few wide scalar loads instead of chasing 19 tile numbers.  Everything a step
// needs to know about a tile is in its row: one round trip to memory, where a
// record read before the row and a field offset read after it cost a wave two
// more.
// ---------------------------------------------------------------------------
struct TileRec {
    uint64_t mask;
    uint64_t base;
};
// slot of neighbour k = (dx+1) + 3(dy+1) + 9(dz+1) in a neighbourhood row,
// -1 for the 8 corners
constexpr int nb_slot(int k) {
    int slot = 0;
    for (int j = 0; j < 27; ++j) {
        const int nz = (j % 3 != 1) + ((j / 3) % 3 != 1) + (j / 9 != 1);
        if (nz == 3) {
            if (j == k) return -1;
            continue;
        }
        if (j == k) return slot;
        ++slot;
    }
    return -1;
}
struct NbRow {
    uint64_t mask[19];
    uint32_t base32[19];
    uint32_t pad0;
    uint64_t fbase;
    int32_t xyz[3];
    int32_t pad1;
};
static_assert(sizeof(NbRow) == 256, "a row is the size of two 128-byte lines");
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
// Groups of 4 tiles along x (along y in a box of one tile along x) in which a
// dense array is walked, -1 if there are too many to number.
inline int64_t dense_groups(int32_t nx, int32_t ny, int32_t nz) {
    const int64_t tx = ((int64_t)nx + 3) / 4, ty = ((int64_t)ny + 3) / 4, tz = ((int64_t)nz + 3) / 4;
    const int64_t row = tx == 1 ? (ty + 3) / 4 : (tx + 3) / 4, rows = tx == 1 ? tz : ty * tz;
    return row > 0 && rows > (int64_t)(INT32_MAX / 2) / row ? -1 : row * rows;
}
// Whether a pass over a dense array walks the box, or takes its kept tiles one
// by one after the array has been cleared: it walks up to two groups of four
// tiles per kept tile.  A 384^3 box, FP64, us walked and tile by tile:
//   kept tiles (groups per kept tile)  all fields  sums alone   lattice    per-node field
//   one 170 x 170 duct (1.2)            755   864   313   290  2271  2415   390   378
//   15% scattered (1.7)                 668   983   251   226  2780  3338   475   560
//   10% scattered (2.5)                 582   787   178   157  2635  2790   446   473
//   one 120 x 120 duct (2.6)            582   601   179   154  2040  1975   355   309
//   6% scattered (4.2)                  516   624   138   102  2305  2327   413   401
//   one 64 x 64 duct (9)                456   421   119    53  1907  1663   341   259
inline bool walks_box(int64_t n_tiles, int32_t nx, int32_t ny, int32_t nz) {
    const int64_t groups = dense_groups(nx, ny, nz);
    return n_tiles > 0 && groups >= 0 && groups <= 2 * n_tiles;
}
struct TableLayout {
    size_t rec_off, row_off, xyz_off, fld_off, map_off, map_size, used, total;
    // the map is there if the box is walked
    TableLayout(int64_t n_tiles, int32_t nx, int32_t ny, int32_t nz) {
        const size_t n = (size_t)n_tiles;
        rec_off = 0;
        row_off = align_up(rec_off + n * sizeof(TileRec), 256);
        xyz_off = align_up(row_off + n * sizeof(NbRow), 256);
        fld_off = align_up(xyz_off + n * 16, 256);
        map_off = align_up(fld_off + n * 8, 256);
        map_size = walks_box(n_tiles, nx, ny, nz) ? ((size_t)nx + 3) / 4 * (((size_t)ny + 3) / 4) * (((size_t)nz + 3) / 4) : 0;
        used = n ? align_up(map_off + map_size * 4, 256) : 0;
        // at least 432 bytes a tile are asked for, of which the tables take about
        // 300: tests/test_abi.py holds the size that is reported to that bound
        total = used < n * 432 ? align_up(n * 432, 256) : used;
    }
};

struct DevTables {
    const TileRec *rec;
    const NbRow *row;
    const int32_t *xyz;
    const uint64_t *fbase;
    const int32_t *map;
};
// reduction scratch: rows of 8 doubles, at most one row per tile + the final 8
constexpr int NSUM = 8;

}  // namespace tlbm
