// Loader addressing of the bf16 contraction kernel (k2_contract_ws): the
// tile order, and for every direct-to-LDS load the buffer descriptor (base
// and range) and the byte offset within it.  The kernel computes its loads
// with these functions, and so does the host-side checker
// (k2_check_loads in contract.hip), which walks every load of a launch and
// verifies that each descriptor lies inside its operand's allocation and that
// every element a tile needs arrives from the address the operand's layout
// gives it.
//
// Every offset travels in the lane offset (voffset); the scalar offset of the
// loads is always 0.  A load whose part of the tile lies outside the operand
// (rows past the panel, a transposed operand's column blocks past its last
// one) gets a range that excludes it, or the empty descriptor, so it reads
// zeros without touching memory.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace trimul {

constexpr int kK2Tile = 256;   // output tile side (rows of A and of B per tile)
constexpr int kK2BK = 32;      // k per step
constexpr int kK2Row = kK2BK * 2;          // bytes of one operand row of a step in LDS
constexpr int kK2Loaders = 4;              // loader waves
constexpr int kK2LoadsPerOperand = 4;      // loads per loader wave, operand and step
// The blocked layout holds one 256-row x 32-k block per panel block: a tile's
// k-step is one block only when the tile side and the step equal the block's.
static_assert(kK2Tile == kBlkRows && kK2BK == kBlkK, "a K2 tile step must be exactly one panel block");
static_assert(kK2Loaders * kK2LoadsPerOperand * 16 == kK2Tile, "loader waves cover the tile's rows");

// Operand layouts.
enum { kK2Blocked = 0, kK2RowMajor = 1, kK2Transposed = 2 };

struct K2Operand {
    int mode;        // kK2Blocked, kK2RowMajor or kK2Transposed
    int rows;        // logical rows (M for A, N for B)
    int K;           // contraction length
    int ld;          // kK2RowMajor: elements between rows
    int64_t stride;  // kK2RowMajor: elements between channels
};

struct K2Desc {
    int64_t base;    // element offset of the descriptor's base from the operand start
    uint32_t range;  // bytes covered (0: the empty descriptor)
};

// ------------------------------------------------------------- tile order
//
// Persistent grid of G work-groups.  Work-group wg runs on XCD wg % 8 (the
// dispatcher deals work-groups round-robin over the 8 XCDs); perm renumbers
// them so that the 32 work-groups of one XCD hold consecutive numbers.  In
// round it, work-group perm takes logical tile it * G + perm.  Logical tiles
// run channel by channel; within a channel in groups of 4 tile rows, and
// within a group column-major, so 32 consecutive tiles form a 4 x 8 block
// whose A row panels and B column panels the XCD's L2 shares.
__host__ __device__ __forceinline__ int k2_perm(int wg, int G) {
    return (G & 7) == 0 ? (wg & 7) * (G >> 3) + (wg >> 3) : wg;
}
__host__ __device__ __forceinline__ int k2_my_tiles(int perm, int G, int total) {
    return perm < total ? (total - 1 - perm) / G + 1 : 0;
}
//
// Tile sides.  A side of `rows` rows is ceil(rows / 64) units of 64 rows over
// ceil(rows / 256) tiles of one to four units; the matrix-core waves skip the
// units a tile does not have, so a ragged size is padded to 64 and not to 256
// (N = 300: 320^2 against 512^2).  The units are spread evenly over the tiles
// (1300 rows: 4 4 4 3 3 3, not 4 4 4 4 4 1, whose narrow tile would pay the
// loads and barriers of a wide one); a plain blocked operand keeps the
// 256-row grid of its panel blocks, only its last tile is short.  Row-major
// operands (panels too long for the padding to matter) always get whole tiles.
constexpr int kK2Unit = 64;
struct K2Side {
    int units, tiles, even;
};
__host__ __device__ __forceinline__ K2Side k2_side(int mode, int rows) {
    const int tiles = (rows + kK2Tile - 1) / kK2Tile;
    if (mode == kK2RowMajor) return K2Side{tiles * (kK2Tile / kK2Unit), tiles, 0};
    return K2Side{(rows + kK2Unit - 1) / kK2Unit, tiles, mode == kK2Transposed};
}
struct K2Tile {
    int ch, m0, n0;   // channel, first row of A and of B
    int mu, nu;       // units of A and of B
};
__host__ __device__ __forceinline__ void k2_span(const K2Side& s, int i, int& t0, int& units) {
    constexpr int kPer = kK2Tile / kK2Unit;
    if (s.even) {
        const int q = s.units / s.tiles, r = s.units - q * s.tiles;
        t0 = (i * q + (i < r ? i : r)) * kK2Unit;
        units = q + (i < r ? 1 : 0);
    } else {
        t0 = i * kK2Tile;
        units = s.units - i * kPer < kPer ? s.units - i * kPer : kPer;
    }
}
__host__ __device__ __forceinline__ K2Tile k2_tile(const K2Side& sm, const K2Side& sn, int ch, int ti, int tj) {
    K2Tile t;
    t.ch = ch;
    k2_span(sm, ti, t.m0, t.mu);
    k2_span(sn, tj, t.n0, t.nu);
    return t;
}
__host__ __device__ __forceinline__ void k2_index(const K2Side& sm, const K2Side& sn, int L, int& ch, int& ti, int& tj) {
    constexpr int GR = 4;
    const int tiles = sm.tiles * sn.tiles;
    ch = L / tiles;
    const int rem = L - ch * tiles;
    const int gid = rem / (GR * sn.tiles);
    const int first_m = gid * GR;
    const int gsz = sm.tiles - first_m < GR ? sm.tiles - first_m : GR;
    const int in_g = rem - gid * GR * sn.tiles;
    ti = first_m + in_g % gsz;
    tj = in_g / gsz;
}
__host__ __device__ __forceinline__ K2Tile k2_decode(const K2Side& sm, const K2Side& sn, int L) {
    int ch, ti, tj;
    k2_index(sm, sn, L, ch, ti, tj);
    return k2_tile(sm, sn, ch, ti, tj);
}
// The 32-row blocks of a tile that MFMA wave w (0..7) owns: `rows` blocks of A
// from block rb, `cols` blocks of B from block cb.  Waves w and w + 4 share a
// SIMD, i.e. row pairs w / 2 and w / 2 + 2: the split gives every SIMD the
// same work for any number of units (three units: 2 2 1 1 blocks).
struct K2Wave {
    int rb, rows, cb, cols;
};
__host__ __device__ __forceinline__ K2Wave k2_wave(const K2Tile& t, int wave) {
    const int wm = wave >> 1, wn = wave & 1;
    K2Wave w;
    w.rows = t.mu == 4 ? 2 : t.mu == 3 ? (wm < 2 ? 2 : 1) : t.mu == 2 ? 1 : (wm < 2 ? 1 : 0);
    w.rb = t.mu == 4 ? 2 * wm : t.mu == 3 ? (wm < 2 ? 2 * wm : 2 + wm) : wm;
    w.cols = t.nu;
    w.cb = wn * t.nu;
    return w;
}

// ------------------------------------------------------------- loads
//
// Loader wave lw (0..3) issues, per operand and step, loads jj = 0..3, each
// 64 lanes x 16 bytes into LDS rows 64 lw + 16 jj .. + 15 of the operand's
// half of the stage (lane i writes bytes 16 i .. + 15 of that 1 KB piece).
//
// Blocked / row-major: LDS row r holds operand row t0 + r of the step, its
// 16-byte chunk q (k = 32 kt + 8 q .. + 7) at slot q ^ ((r >> 2) & 3); lane i
// fills row r = 64 lw + 16 jj + i / 4, slot i % 4.
// Transposed (the operand is given as X with X[k][row] = operand[row][k]):
// the 1 KB piece (2 lw + jj / 2, jj % 2) is rows 16 (jj % 2) .. + 15 of
// the step (k = 32 kt + those) of the tile's 32-column block 2 lw + jj / 2, 64
// bytes per k row, no swizzle.

// Byte offset of lane `lane` of loader wave lw within the step's first piece
// (the part of the lane offset that does not change from load to load).
__host__ __device__ __forceinline__ uint32_t k2_lane_off(const K2Operand& op, int lw, int lane) {
    if (op.mode == kK2Transposed) return (uint32_t)(lane * 16);
    const int row = lw * 64 + (lane >> 2);
    const int chunk = (lane & 3) ^ ((lane >> 4) & 3);   // the k chunk that lands in slot lane % 4
    const int rs = op.mode == kK2Blocked ? kK2BK : op.ld;
    return (uint32_t)((row * rs + chunk * 8) * 2);
}

// Number of 256-row tiles of the X panel (transposed operand: X has K rows)
// and its 32-column blocks.
__host__ __device__ __forceinline__ int k2_tr_blocks(const K2Operand& op) { return (op.rows + 31) / 32; }

// Descriptor of the operand part that tile rows t0 .. t0 + 255 read in step
// kt: for the blocked and row-major layouts the same for every step of a
// tile, for a transposed operand the 256-row tile of X that holds the step.
__host__ __device__ __forceinline__ K2Desc k2_desc(const K2Operand& op, int ch, int t0, int kt) {
    const int nk = (op.K + kK2BK - 1) / kK2BK;
    const int tiles = (op.rows + kK2Tile - 1) / kK2Tile;
    K2Desc d;
    if (op.mode == kK2Blocked) {
        d.base = ((int64_t)ch * tiles + t0 / kK2Tile) * nk * (kK2Tile * kK2BK);
        d.range = (uint32_t)nk * (uint32_t)(kK2Tile * kK2BK * 2);
    } else if (op.mode == kK2RowMajor) {   // rows past the operand fall outside the range
        d.base = (int64_t)ch * op.stride + (int64_t)t0 * op.ld;
        const int live = op.rows - t0 < kK2Tile ? op.rows - t0 : kK2Tile;
        d.range = (uint32_t)live * (uint32_t)op.ld * 2u;
    } else {
        const int xs = k2_tr_blocks(op), xt = (op.K + kK2Tile - 1) / kK2Tile;
        d.base = ((int64_t)ch * xt + (kt >> 3)) * xs * (kK2Tile * kK2BK);
        d.range = (uint32_t)xs * (uint32_t)(kK2Tile * kK2BK * 2);
    }
    return d;
}

// Wave-uniform byte offset of load jj of loader wave lw in step kt (added to
// k2_lane_off).  Returns false when the tile does not have the loader wave's
// unit of rows, or the whole load lies outside the operand (a transposed
// operand's column block past its last one): the load then goes to the empty
// descriptor.
__host__ __device__ __forceinline__ bool k2_load_off(const K2Operand& op, int t0, int units, int kt, int lw, int jj,
                                                      uint32_t& off) {
    if (op.mode == kK2Transposed) {
        const int cb = (t0 >> 5) + 2 * lw + (jj >> 1);
        off = (uint32_t)cb * (uint32_t)(kK2Tile * kK2BK * 2) + (uint32_t)((kt & 7) * 32 + 16 * (jj & 1)) * kK2Row;
        return lw < units && cb < k2_tr_blocks(op);
    }
    if (op.mode == kK2Blocked) {
        off = (uint32_t)(jj * 16 * kK2BK * 2) + (uint32_t)kt * (uint32_t)(kK2Tile * kK2BK * 2);
    } else {
        off = (uint32_t)jj * (uint32_t)(16 * op.ld * 2) + (uint32_t)kt * kK2Row;
    }
    return lw < units;
}

// LDS byte offset (within the operand's half of a stage) of load jj of
// loader wave lw: the same for every layout.
__host__ __device__ __forceinline__ uint32_t k2_lds_off(int lw, int jj) {
    return (uint32_t)(lw * 64 + 16 * jj) * kK2Row;
}

// ------------------------------------------------------------- pair-blocked C
//
// The result C of nch channels in the pair-blocked layout (result_off):
// element (ch, i, j) at ((i * J + j / 32) * nch + ch) * 32 + j % 32 floats,
// J = ceil(N / 32); a row is crs = J * nch * 32 floats long.  MFMA wave w
// (0..7) of a tile owns its blocks k2_wave, up to eight 32 x 32 blocks x =
// 4 (row block) + column block; in the accumulator layout lane l holds column
// l % 32 and, in register r, row 8 (r / 4) + 4 (l / 32) + r % 4 of a block.
// Each of the wave's column blocks goes through one descriptor from the block's
// first element whose range covers the rows < M, so that rows past M fall
// outside it; a column block past C's last gets the empty descriptor (its
// memory belongs to the next row).  Columns past N inside C's last block
// are the layout's padding and are accessed like the rest.  The byte offset
// is the lane part (k2_c_lane_off) plus the wave-uniform part of block x,
// register r (k2_c_reg_off); both travel in the lane offset.
__host__ __device__ __forceinline__ uint32_t k2_c_row_floats(int N, int nch) {
    return (uint32_t)((N + kResJ - 1) / kResJ) * (uint32_t)nch * kResJ;
}
__host__ __device__ __forceinline__ K2Desc k2_c_desc(int M, int N, int nch, const K2Tile& t, const K2Wave& w, int j) {
    const int jblocks = (N + kResJ - 1) / kResJ;
    const int wrow0 = t.m0 + 32 * w.rb, wcol0 = t.n0 + 32 * w.cb;
    const int nrows = M - wrow0 < 32 * w.rows ? M - wrow0 : 32 * w.rows;
    const bool live = nrows > 0 && j < w.cols && wcol0 / kResJ + j < jblocks;
    K2Desc d;
    d.base = live ? result_off(jblocks, nch, t.ch, wrow0, wcol0 + kResJ * j) : 0;
    d.range = live ? ((uint32_t)(nrows - 1) * k2_c_row_floats(N, nch) + kResJ) * 4u : 0u;
    return d;
}
__host__ __device__ __forceinline__ uint32_t k2_c_lane_off(uint32_t crs, int lane) {
    return (4u * (uint32_t)(lane >> 5) * crs + (uint32_t)(lane & 31)) * 4u;
}
__host__ __device__ __forceinline__ uint32_t k2_c_reg_off(uint32_t crs, int x, int r) {
    return (uint32_t)((x >> 2) * 32 + 8 * (r >> 2) + (r & 3)) * crs * 4u;
}
// The logical row and column of that element (for the host check).
__host__ __device__ __forceinline__ void k2_c_elem(const K2Tile& t, int wave, int lane, int x, int r, int& row, int& col) {
    const K2Wave w = k2_wave(t, wave);
    row = t.m0 + (w.rb + (x >> 2)) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    col = t.n0 + (w.cb + (x & 3)) * 32 + (lane & 31);
}

}  // namespace trimul
