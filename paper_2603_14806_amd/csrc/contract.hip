// K2: the per-channel contraction of Eq. 2 / Eq. 3 (Section 3.3), which the
// paper describes as a batched matrix multiplication.  After K1's layout
// change both directions are the same "NT" product per hidden channel c:
//
//     C[c][i][j] (+)= sum_k A[c][i][k] * m_k * B[c][j][k]
//
// m_k is an optional token mask over k (used by the block path, where the
// panels arrive unmasked).  The bf16 path runs on gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation), and so does the fp32 path
// (v_mfma_f32_32x32x2_f32).
#include <type_traits>
#include <vector>

#include "common.h"
#include "k2_addr.h"
#include "kernels.h"

namespace trimul {
namespace {

// ---------------------------------------------------------------- bf16 MFMA
//
// Persistent kernel, one work-group per CU, looping over 256 x 256 output
// tiles.  The k loop runs in steps of 32 through an LDS ring of 32 KB stages
// filled by direct-to-LDS buffer loads (no VGPR staging) several steps ahead
// of the step being multiplied; the ring flows straight from one output
// tile into the next.
//
// Tile order: in round r the work-groups on XCD x take 32 consecutive
// logical tiles, i.e. a 4 x 8 block of one channel, so the A row panels and B
// column panels of a block are fetched once into that XCD's L2 and served to
// the 32 CUs that share it.
//
// LDS layout of a stage: 256 A rows then 256 B rows of 32 bf16 (64 bytes =
// 4 chunks of 16 bytes); chunk q of row r sits at slot q ^ ((r >> 2) & 3).
// gfx950's LDS has 64 banks and serves a 16-byte-per-lane read 16 lanes per
// cycle; the 16 rows those lanes read then cover all 64 banks.
constexpr int BN = 256, BK = 32;
constexpr int ROWB = BK * 2;                    // 64 bytes per row per stage
constexpr int B_ST = BN * ROWB;                 // 16 KB
constexpr int kLdsBytes = 160 * 1024;           // gfx950 LDS per work-group

// Eight bf16 of an MFMA operand from a row-major [k][32] LDS block through
// two ds_read_b64_tr_b16 (k values 0-3, then 4-7 from four rows further on).
typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef short v8i16_t __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8_t lds_read_tr8(const char* p) {
    typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;
    const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(p));
    const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(p + 4 * ROWB));
    const v8i16_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
}

// ------------------------------------------- bf16 MFMA, 8 + 4 specialised waves
//
// The contraction with the loads taken off the MFMA waves: 12 waves per
// work-group (three per SIMD); waves 0-7 each own a 64 x 128 sub-tile (2 x 4
// MFMA blocks, 128 accumulator registers) and issue only LDS reads and
// MFMAs, waves 8-11 issue all 32 direct-to-LDS loads of a k-step (64 A rows
// and 64 B rows each) and wait for them, so a load that stalls in a busy L2
// never stops a matrix-core stream.  The one barrier per k-step hands
// filled stages from the loaders to the MFMA waves and a consumed one back;
// at barrier s steps s and s + 1 are complete, and the MFMA waves read step
// s + 1's first operands behind step s's last MFMAs.
//
// Operands either blocked (one tile's k-step is a contiguous 16 KB block:
// the full update, the outer product mean, and a device tile's panels
// repacked by k_panel_block) or row-major (a device tile's caller panels
// [ch][rows][ld]); C either in the pair-blocked result layout (the full
// update) or row-major [ch][rows][ldc] (a device tile's accumulator).  k values that must not reach the sums -- masked by the
// optional k-mask, or past K in the last step (row-major padding columns
// hold arbitrary data) -- are zeroed in LDS by the loader waves, in the rows
// each loaded, before the barrier that publishes the stage: only steps that
// hold such k pay, and the MFMA waves never mask.
// LDS ring of 5 stages, swizzle and tile order as described above.
//
// Transposed operands (TA / TB, blocked only, no k-mask): the operand is
// given as its transpose X in the panel layout, A[c][i][k] = X[c][k][i], so
// the products of the backward, dC B and dC^T A, run without transposing
// panels in memory.  A k-step of a 256-wide tile is then the 32 rows k of
// eight 32-column blocks of X: eight contiguous 2 KB pieces, copied to LDS
// as they are (block b of the tile at 2 KB b, 64 bytes per row k, no
// swizzle).  The MFMA waves read such an operand with ds_read_b64_tr_b16:
// lanes 16 g + 4 i + a (g < 4, i < 4, a < 4) address row 8 (g >> 1) + i,
// columns 16 (g & 1) + 4 a .. + 3 of a block, and lane 16 g + 4 a + b receives
// element b of the four chunks lanes 16 g + a, + 4, + 8, + 12 address, i.e.
// column 16 (g & 1) + 4 a + b of rows 8 (g >> 1) .. + 3 -- the MFMA operand
// layout, 4 of its 8 k values; a second read 4 rows further gives the rest.
// A half-wave reads 256 contiguous bytes: no bank conflicts.
// Round pacing.  The work-groups of one XCD share their round's A row
// panels and B column panels through that XCD's L2 only while they stream
// the same k range; left alone they drift apart (measured: up to ~100 us,
// about 100 k-steps, within a few rounds, far beyond the ~20 k-steps of
// operand traffic the L2 holds), and every lagging tile then refetches its
// panels from memory.  So at the start of every full round each work-group
// counts in on its XCD's counter and waits until all G / 8 of them have (a
// bounded wait: 20 us, after which it goes on anyway -- pacing changes only
// where the data comes from, never the results).  One 128-byte line per XCD;
// reset by k_pace_reset before every paced launch.  Concurrent contraction
// launches on one device share the counters and then mostly wait the bound.
constexpr int kPaceLine = 32;   // counters per 128-byte line
__device__ unsigned int g_k2_pace[8 * kPaceLine];
__global__ void k_pace_reset() {
    if (threadIdx.x < 8 * kPaceLine) g_k2_pace[threadIdx.x] = 0u;
}

// RAGGED: tiles of one to four units a side (k2_addr.h); without it every tile
// is whole.  (One more instance of the tile loop per shape costs whole tiles
// about 1%, so launches that have only those run without it.)  Ragged tiles
// took the contraction from 34.0 to 32.0 us at N = 384 (3 + 3 units), from
// 28.2 to 25.3 at N = 300 and from 676 to 646 at N = 1300.
template <bool BLOCKED, bool KMASK, bool CBLOCKED, bool TA, bool TB, bool RAGGED>
__global__ __attribute__((amdgpu_flat_work_group_size(768, 768), amdgpu_waves_per_eu(3, 3)))
void k2_contract_ws(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, float* __restrict__ C, int M,
                    int N, int K, int lda, int ldb, int64_t ldc, int64_t sA, int64_t sB, int64_t sC, int total,
                    int accumulate, const uint8_t* __restrict__ kmask, int pace) {
    constexpr int BM = kK2Tile;
    constexpr int A_ST = BM * ROWB, ST_BYTES = A_ST + B_ST;
    constexpr int STAGES = kLdsBytes / ST_BYTES;  // 5
    constexpr int LOADS = 2 * kK2LoadsPerOperand;  // direct-to-LDS loads per loader wave per step
    static_assert(!(TA || TB) || (BLOCKED && !KMASK), "transposed operands are blocked and unmasked");
    // a blocked operand's k-step must be exactly one panel block (256 rows x 32 k)
    static_assert(!BLOCKED || (BM == kBlkRows && BN == kBlkRows && BK == kBlkK), "blocked tiles are panel blocks");
    static_assert(BN == kK2Tile && BK == kK2BK && ROWB == kK2Row, "loader addressing assumes this tile");
    __shared__ __attribute__((aligned(16))) char smem[STAGES * ST_BYTES];

    const int G = gridDim.x, wg = blockIdx.x;
    const int perm = k2_perm(wg, G);
    const int my_tiles = k2_my_tiles(perm, G, total);
    const int nk = (K + BK - 1) / BK;
    const int steps = my_tiles * nk;
    const K2Side sm = k2_side(TA ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, M);
    const K2Side sn = k2_side(TB ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, N);
    const int nchan = total / (sm.tiles * sn.tiles);
    auto decode = [&](int L) -> K2Tile {
        if constexpr (RAGGED) return k2_decode(sm, sn, L);
        int ch, ti, tj;
        k2_index(sm, sn, L, ch, ti, tj);
        return K2Tile{ch, ti * kK2Tile, tj * kK2Tile, 4, 4};
    };

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);   // 0 .. 11
    const uint32_t lds_base = lds_addr(smem);

    if (wave >= 8) {
        // Loader wave lw: rows 64 lw .. 64 lw + 63 of the A and B halves of a
        // stage as four 16-row loads each (k2_addr.h).  Every offset is in the
        // lane offset; the scalar offset is 0.
        const int lw = wave - 8;
        const K2Operand opa{TA ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, M, K, lda, sA};
        const K2Operand opb{TB ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, N, K, ldb, sB};
        const uint32_t la = k2_lane_off(opa, lw, lane), lb = k2_lane_off(opb, lw, lane);
        int l_it = 0, l_kt = 0, l_stage = 0, l_ch = 0, l_m0 = 0, l_n0 = 0, l_mu = 4, l_nu = 4;
        const v4i_t rnone = buffer_desc(A, 0u);
        v4i_t ra = rnone, rb = rnone;
        auto desc = [&](const bf16_t* X, const K2Operand& op, int t0, int kt) {
            const K2Desc d = k2_desc(op, l_ch, t0, kt);
            return buffer_desc(X + d.base, d.range);
        };
        auto load_tile = [&]() {
            if (pace && lw == 0 && l_it > 0 && (l_it + 1) * G <= total) {   // every full round but the first
                unsigned int* cnt = &g_k2_pace[(wg & 7) * kPaceLine];
                const unsigned int target = (unsigned int)l_it * (unsigned int)(G >> 3);
                if (lane == 0) atomicAdd(cnt, 1u);
                const uint64_t t0 = __builtin_amdgcn_s_memrealtime();   // 100 MHz
                while (true) {
                    const unsigned int v = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    if (v >= target || __builtin_amdgcn_s_memrealtime() - t0 > 2000u) break;
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            const K2Tile tl = decode(l_it * G + perm);
            l_ch = tl.ch;
            l_m0 = tl.m0;
            l_n0 = tl.n0;
            if (RAGGED) l_mu = tl.mu, l_nu = tl.nu;
            if (!TA) ra = desc(A, opa, l_m0, 0);
            if (!TB) rb = desc(B, opb, l_n0, 0);
        };
        auto issue_step = [&](bool live) {
            const uint32_t st = lds_base + (uint32_t)(l_stage * ST_BYTES);
            const v4i_t rta = TA ? desc(A, opa, l_m0, l_kt) : ra, rtb = TB ? desc(B, opb, l_n0, l_kt) : rb;
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {   // j < 4: A loads, j >= 4: B loads
                const bool isb = j >= kK2LoadsPerOperand;
                const int jj = j % kK2LoadsPerOperand;
                uint32_t off;
                const bool in = k2_load_off(isb ? opb : opa, isb ? l_n0 : l_m0, RAGGED ? (isb ? l_nu : l_mu) : 4, l_kt, lw, jj, off);
                const uint32_t dst = st + (isb ? A_ST : 0) + k2_lds_off(lw, jj);
                lds_load16((live && in) ? (isb ? rtb : rta) : rnone, (isb ? lb : la) + off, 0u, dst);
            }
        };
        auto advance = [&]() {
            l_stage = l_stage == STAGES - 1 ? 0 : l_stage + 1;
            if (++l_kt == nk) {
                l_kt = 0;
                if (++l_it < my_tiles) load_tile();
            }
        };
        // Dead-k bitmaps of the k-mask (bit k of step kt set if k-mask byte
        // kt * 32 + k is 0), computed once before any load is in flight:
        // lane l holds steps l + 64 j in mwords[j] (K <= 65536 -> j < 32).
        uint32_t mwords[KMASK ? 32 : 1];
        if (KMASK) {
            const uint32_t* km4 = reinterpret_cast<const uint32_t*>(kmask);   // staged: 0/1 bytes, padded to 32
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                const int kt = lane + 64 * j;
                uint32_t wbits = 0;
                if (kt < nk) {
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        const uint32_t m4 = km4[kt * 8 + d];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (((m4 >> (8 * e)) & 0xffu) == 0) wbits |= 1u << (4 * d + e);
                    }
                }
                mwords[j] = wbits;
            }
        }
        // Zero, in this wave's 64 A and 64 B rows of step u's stage, the k
        // values of the step that are masked out or past K.
        auto zero_dead = [&](int u) {
            const int kt = u % nk;
            const int kv = K - kt * BK;                   // valid k of the step
            uint32_t bits = kv >= BK ? 0u : ~((1u << kv) - 1u);
            if (KMASK) {
                uint32_t wsel = 0;
#pragma unroll
                for (int j = 0; j < 32; ++j) wsel = (j == (kt >> 6)) ? mwords[j] : wsel;
                bits |= (uint32_t)__builtin_amdgcn_readlane((int)wsel, kt & 63);
            }
            bits = __builtin_amdgcn_readfirstlane(bits);
            if (bits == 0) return;
            char* st = smem + (u % STAGES) * ST_BYTES;
            const int r = lw * 64 + lane;                 // this lane's row of the A and of the B block
            if (TA || TB) {   // in a transposed operand the row is k = lane % 32 of a column block
                if ((bits >> (lane & 31)) & 1u) {
                    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (TA) *reinterpret_cast<uint4*>(st + r * ROWB + 16 * q) = zero;
                        if (TB) *reinterpret_cast<uint4*>(st + A_ST + r * ROWB + 16 * q) = zero;
                    }
                }
                if (TA && TB) return;
            }
            const int sw = (r >> 2) & 3;
            while (bits) {
                const int k = __builtin_ctz(bits);
                bits &= bits - 1;
                const uint32_t o = (uint32_t)(r * ROWB + ((((k >> 3) ^ sw)) << 4) + (k & 7) * 2);
                if (!TA) *reinterpret_cast<bf16_t*>(st + o) = 0;
                if (!TB) *reinterpret_cast<bf16_t*>(st + A_ST + o) = 0;
            }
        };
        if (my_tiles > 0) load_tile();
        const int pro = min(STAGES - 1, steps);
        for (int s0 = 0; s0 < pro; ++s0) {
            issue_step(true);
            advance();
        }
        for (int s = 0; s < steps; ++s) {
            // steps s and s + 1 complete at barrier s; later ones in flight.
            // (Waits with a memory clobber: the LDS zeroing below must not
            // be moved above them.)
            const int ahead = min(STAGES - 3, steps - 2 - s);
            if (ahead >= 2) wait_vmcnt_pinned<2 * LOADS>();
            else if (ahead == 1) wait_vmcnt_pinned<LOADS>();
            else wait_vmcnt_pinned<0>();
            if (s == 0) zero_dead(0);
            if (s + 1 < steps) zero_dead(s + 1);
            __syncthreads();
            const bool fetch = s + STAGES - 1 < steps;
            issue_step(fetch);
            if (fetch) advance();
        }
        wait_vmcnt_pinned<0>();
        return;
    }

    // The matrix-core waves issue ahead of the loader wave that shares their
    // SIMD (instruction-issue priority inside the work-group; 1% faster than
    // equal priority, the reverse 0.5% slower).
    __builtin_amdgcn_s_setprio(1);
    const int rl = lane & 31, hi = lane >> 5;
    const int q = (rl >> 2) & 3;
    uint32_t rd[2];   // plain operand: this lane's row of a 32-row block, sub-step 0 and 1
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) rd[sub] = (uint32_t)(rl * ROWB + (((2 * sub + hi) ^ q) << 4));
    // transposed operands: this lane's address in a column block
    const int tg = lane >> 4;
    const uint32_t trb = (uint32_t)((8 * (tg >> 1) + ((lane >> 2) & 3)) * ROWB + (16 * (tg & 1) + 4 * (lane & 3)) * 2);
    // Pair-blocked C (CBLOCKED): descriptors and offsets from k2_addr.h
    // (rows past M fall outside a block's descriptor: loads read 0, stores
    // are dropped).
    const uint32_t crs = k2_c_row_floats(N, nchan);
    const uint32_t cvo = k2_c_lane_off(crs, lane);
    // byte offset of register r of 32 x 32 block x from the lane's base vo.
    // Each use site passes a fresh copy of the base (opaque to the
    // compiler), so that the 32 row offsets are formed where they are used
    // instead of being hoisted out of the tile loop and kept in registers
    // the accumulators need.
    auto coff = [&](uint32_t vo, int x, int r) -> uint32_t { return vo + k2_c_reg_off(crs, x, r); };
    auto fresh = [](uint32_t v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    int c_stage = 0;
    // One tile of NI x NJ blocks for this wave (NI = 0: it only keeps the
    // barriers).
    auto tile = [&](const K2Tile& tl, auto ni, auto nj) {
        constexpr int NI = decltype(ni)::value, NJ = decltype(nj)::value;
        if constexpr (NI == 0) {
            for (int kt = 0; kt < nk; ++kt) {
                __syncthreads();
                c_stage = c_stage == STAGES - 1 ? 0 : c_stage + 1;
            }
        } else {
        const K2Wave wv = RAGGED ? k2_wave(tl, wave) : K2Wave{2 * (wave >> 1), 2, 4 * (wave & 1), 4};
        // this lane's address of operand block i (A) / j (B) of the wave in the
        // stage at st, sub-step sub (2 KB per 32-row block in either layout)
        const uint32_t oa[2] = {(TA ? trb : rd[0]) + wv.rb * 2048, (TA ? trb + 16 * ROWB : rd[1]) + wv.rb * 2048};
        const uint32_t ob[2] = {(TB ? trb : rd[0]) + A_ST + wv.cb * 2048, (TB ? trb + 16 * ROWB : rd[1]) + A_ST + wv.cb * 2048};
        auto opA = [&](const char* st, int sub, int i) -> bf16x8_t {
            if constexpr (TA) return lds_read_tr8(st + oa[0] + i * 2048 + sub * 16 * ROWB);
            else return *reinterpret_cast<const bf16x8_t*>(st + oa[sub] + i * 2048);
        };
        auto opB = [&](const char* st, int sub, int j) -> bf16x8_t {
            if constexpr (TB) return lds_read_tr8(st + ob[0] + j * 2048 + sub * 16 * ROWB);
            else return *reinterpret_cast<const bf16x8_t*>(st + ob[sub] + j * 2048);
        };
        auto cdesc = [&](__amdgpu_buffer_rsrc_t* rc) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const K2Desc d = k2_c_desc(M, N, nchan, tl, wv, j);
                rc[j] = make_rsrc(C + d.base, d.range);
            }
        };
        bf16x8_t a0[NI], b0[NJ];  // sub-step 0 operands, read one step ahead within a tile
        f32x16_t acc[NI][NJ];
        if (CBLOCKED && accumulate) {
            // accumulating: the accumulators start from C, all loads issued
            // together and waited for once (one HBM round trip per tile
            // instead of one per 32 x 32 block at the end)
            __amdgpu_buffer_rsrc_t rc[NJ];
            cdesc(rc);
            const uint32_t vo = fresh(cvo);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[i][j][r] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(rc[j], coff(vo, 4 * i + j, r), 0, 0));
            wait_vmcnt_pinned<0>();
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        }

        // a tile's first step: barrier, then its sub-step 0 operands (nothing
        // is read ahead across the C stores)
        __syncthreads();
        {
            const char* st = smem + c_stage * ST_BYTES;
#pragma unroll
            for (int j = 0; j < NJ; ++j) b0[j] = opB(st, 0, j);
#pragma unroll
            for (int i = 0; i < NI; ++i) a0[i] = opA(st, 0, i);
        }
        for (int kt = 0; kt < nk; ++kt) {
            if (kt > 0) __syncthreads();
            const char* st = smem + c_stage * ST_BYTES;
            c_stage = c_stage == STAGES - 1 ? 0 : c_stage + 1;
            const char* stn = smem + c_stage * ST_BYTES;             // the next step
            bf16x8_t a1[NI], b1[NJ];
            // sub-step 0; the operand reads of sub-step 1 start after its
            // first two MFMAs (what is left of them comes after the last)
#pragma unroll
            for (int x = 0; x < NI * NJ + NI + NJ; ++x) {
                const int i = x / NJ, j = x % NJ, y = x - 2;
                if (x < NI * NJ) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[i], b0[j], acc[i][j], 0, 0, 0);
                if (y >= 0 && y < NJ) b1[y] = opB(st, 1, y);
                else if (y >= NJ && y < NJ + NI) a1[y - NJ] = opA(st, 1, y - NJ);
            }
            if (NI * NJ + NI + NJ < 2 + NI + NJ) a1[NI - 1] = opA(st, 1, NI - 1);
            // sub-step 1; after MFMA x, the operand read x - 2 of the next
            // step's sub-step 0 (its stage is complete since this step's
            // barrier; after a tile's last step the values go unused)
#pragma unroll
            for (int x = 0; x < NI * NJ + NI + NJ; ++x) {
                const int i = x / NJ, j = x % NJ, y = x - 2;
                if (x < NI * NJ) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], b1[j], acc[i][j], 0, 0, 0);
                if (y >= 0 && y < NJ) b0[y] = opB(stn, 0, y);
                else if (y >= NJ && y < NJ + NI) a0[y - NJ] = opA(stn, 0, y - NJ);
            }
            if (NI * NJ + NI + NJ < 2 + NI + NJ) a0[NI - 1] = opA(stn, 0, NI - 1);
        }

        // 32x32 accumulator layout: lane holds column (lane & 31) and, in
        // register r, row 8 (r / 4) + 4 (lane / 32) + r % 4.
        if constexpr (CBLOCKED) {   // the sums (C included when accumulating) go straight out
            __amdgpu_buffer_rsrc_t rc[NJ];
            cdesc(rc);
            const uint32_t vo = fresh(cvo);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r]), rc[j],
                                                              coff(vo, 4 * i + j, r), 0, 0);
        } else {
            const int row0 = tl.m0 + 32 * wv.rb + 4 * hi, col0 = tl.n0 + 32 * wv.cb + rl;
            const bool full = tl.m0 + 32 * (wv.rb + NI) <= M && tl.n0 + 32 * (wv.cb + NJ) <= N;
            float* Cb = C + tl.ch * sC + (int64_t)row0 * ldc + col0;
            const int64_t row_step = ldc;   // elements between rows
            // One 32 x 32 block at a time.  Accumulating, the block's 16 loads
            // go out together (a lane outside C reads C[0] instead) and are
            // waited for once, before its 16 guarded stores; element by element
            // the compiler would wait for every load.
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float* pb = Cb + j * 32;   // column block j
                    const bool colok = full || col0 + j * 32 < N;
                    float v[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = acc[i][j][r];
                    if (accumulate) {
                        float old[16];
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int dr = i * 32 + 8 * (r >> 2) + (r & 3);
                            const bool ok = colok && (full || row0 + dr < M);
                            old[r] = *(ok ? pb + (int64_t)dr * row_step : C);
                        }
#pragma unroll
                        for (int r = 0; r < 16; ++r) v[r] += old[r];
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int dr = i * 32 + 8 * (r >> 2) + (r & 3);
                        if (colok && (full || row0 + dr < M)) pb[(int64_t)dr * row_step] = v[r];
                    }
                }
        }
        }
    };
    for (int it = 0; it < my_tiles; ++it) {
        const K2Tile tl = decode(it * G + perm);
        using std::integral_constant;
        typedef integral_constant<int, 0> c0;
        typedef integral_constant<int, 1> c1;
        typedef integral_constant<int, 2> c2;
        typedef integral_constant<int, 3> c3;
        typedef integral_constant<int, 4> c4;
        if constexpr (!RAGGED) {
            tile(tl, c2{}, c4{});
            continue;
        }
        const int rows = k2_wave(tl, wave).rows;
        if (rows == 2) {
            if (tl.nu == 4) tile(tl, c2{}, c4{});
            else if (tl.nu == 3) tile(tl, c2{}, c3{});
            else if (tl.nu == 2) tile(tl, c2{}, c2{});
            else tile(tl, c2{}, c1{});
        } else if (rows == 1) {
            if (tl.nu == 4) tile(tl, c1{}, c4{});
            else if (tl.nu == 3) tile(tl, c1{}, c3{});
            else if (tl.nu == 2) tile(tl, c1{}, c2{});
            else tile(tl, c1{}, c1{});
        } else {
            tile(tl, c0{}, c1{});
        }
    }
}

// ---------------------------------------------------------------- fp32 MFMA
//
// The fp32 storage path on v_mfma_f32_32x32x2_f32.  One work-group of 4
// waves (2 x 2) per T x T output tile, steps of 32 k through LDS (rows
// padded to 36 floats: the 16 rows a 16-byte read serves per cycle start in
// distinct banks), the next step's global loads in registers while the
// current one is multiplied.  Lane l takes k = 8 q + 4 (l / 32) + e of its
// row for element e of the 16-byte read q, on both operands, so one read
// feeds four products.  Bound by the matrix cores; several work-groups per
// compute unit cover each other's barriers and loads.  k past K and masked k
// are zeroed in both operands (either may hold a NaN there).  N = 384: 309 us
// with scalar FMAs, now 128 (113 TFLOP/s); N = 64: 13 and 7.5.
constexpr int kFr = 36;   // row stride (floats) of an operand in LDS

template <int T, bool BLOCKED>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2)))
void k2_contract_f32(const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int M, int N, int K,
                     int64_t lda, int64_t ldb, int64_t ldc, int64_t sA, int64_t sB, int64_t sC, int tm, int tn,
                     int batch, int accumulate, const uint8_t* __restrict__ kmask) {
    constexpr int WB = T / 64;    // 32 x 32 blocks per wave and side
    constexpr int RL = T / 32;    // 16-byte loads per thread, operand and step
    __shared__ __attribute__((aligned(16))) float As[T * kFr], Bs[T * kFr];
    // Work-groups go to the XCDs round-robin by index: give each XCD a
    // contiguous run of tiles, so that a channel's panels stay in one L2.
    const unsigned nu = gridDim.x, per = nu >> 3, extra = nu & 7, xcd = blockIdx.x & 7;
    const unsigned u = xcd * per + min(xcd, extra) + (blockIdx.x >> 3);   // a bijection of [0, nu)
    const int ch = (int)(u / (unsigned)(tm * tn)), rem = (int)(u - (unsigned)ch * (unsigned)(tm * tn));
    const int m0 = (rem / tn) * T, n0 = (rem % tn) * T;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int rl = lane & 31, hi = lane >> 5;
    const int wm = (wave >> 1) * (T / 2), wn = (wave & 1) * (T / 2);

    // This thread's loads: rows t / 8 + 32 s of the tile, k = 4 (t % 8) .. + 3
    // of the step, straight-line range-checked buffer loads that stay in
    // flight behind the products (rows past a row-major operand read zeros).
    // What must not reach the sums -- k past K, masked k -- is zeroed when a
    // step that holds any is staged.
    const int kk = 4 * (t & 7);
    auto desc = [&](const float* X, int rows, int64_t ld, int64_t stride, int r0, int live, uint32_t& off, uint32_t& rs, uint32_t& ks) {
        const PanelGeom g = panel_geom(rows, K);
        const int64_t base = BLOCKED ? ((int64_t)ch * g.tiles_r + r0 / kBlkRows) * g.ksteps * (kBlkRows * kBlkK)
                                     : ch * stride + (int64_t)r0 * ld;
        const uint32_t bytes = BLOCKED ? (uint32_t)g.ksteps * (kBlkRows * kBlkK * 4) : (uint32_t)live * (uint32_t)ld * 4u;
        rs = BLOCKED ? kBlkK * 4 : (uint32_t)ld * 4u;                    // bytes between rows
        ks = BLOCKED ? kBlkRows * kBlkK * 4 : kBlkK * 4;                 // bytes between steps
        off = (uint32_t)((BLOCKED ? r0 % kBlkRows : 0) + (t >> 3)) * rs + 4 * kk;
        return make_rsrc(X + base, bytes);
    };
    uint32_t oa, ob, rsa, rsb, ksa, ksb;
    const __amdgpu_buffer_rsrc_t ra = desc(A, M, lda, sA, m0, min(T, M - m0), oa, rsa, ksa);
    const __amdgpu_buffer_rsrc_t rb = desc(B, N, ldb, sB, n0, min(T, N - n0), ob, rsb, ksb);
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(kmask, kmask ? (uint32_t)K : 0u);
    float4 va[RL], vb[RL];
    uint32_t km[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int s = 0; s < RL; ++s) {
            va[s] = __builtin_bit_cast(float4, buf_load16(ra, oa + 32u * s * rsa));
            vb[s] = __builtin_bit_cast(float4, buf_load16(rb, ob + 32u * s * rsb));
        }
        oa += ksa;
        ob += ksb;
        if (!BLOCKED) {
#pragma unroll
            for (int e = 0; e < 4; ++e) km[e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rk, k0 + kk + e, 0, 0);
        }
    };
    auto zero_dead = [&](int k0) {
        uint32_t on[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            on[e] = k0 + kk + e < K && (BLOCKED || !kmask || km[e] != 0) ? 0xffffffffu : 0u;
        auto clear = [&](float4& v) {
            const uint4 u = __builtin_bit_cast(uint4, v);
            v = __builtin_bit_cast(float4, make_uint4(u.x & on[0], u.y & on[1], u.z & on[2], u.w & on[3]));
        };
#pragma unroll
        for (int s = 0; s < RL; ++s) {
            clear(va[s]);
            clear(vb[s]);
        }
    };
    f32x16_t acc[WB][WB];
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < WB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    load(0);
    for (int k0 = 0; k0 < K; k0 += 32) {
        if (k0 + 32 > K || (!BLOCKED && kmask)) zero_dead(k0);
        __syncthreads();   // every wave has read the previous step
#pragma unroll
        for (int s = 0; s < RL; ++s) {
            *reinterpret_cast<float4*>(&As[((t >> 3) + 32 * s) * kFr + kk]) = va[s];
            *reinterpret_cast<float4*>(&Bs[((t >> 3) + 32 * s) * kFr + kk]) = vb[s];
        }
        __syncthreads();
        load(k0 + 32);   // past the last step: read and never staged (in range of the operand, or zeros)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 a[WB], b[WB];
#pragma unroll
            for (int i = 0; i < WB; ++i) {
                a[i] = *reinterpret_cast<const float4*>(&As[(wm + 32 * i + rl) * kFr + 8 * q + 4 * hi]);
                b[i] = *reinterpret_cast<const float4*>(&Bs[(wn + 32 * i + rl) * kFr + 8 * q + 4 * hi]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < WB; ++i)
#pragma unroll
                    for (int j = 0; j < WB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f4_get(a[i], e), f4_get(b[j], e), acc[i][j], 0, 0, 0);
        }
    }
    // lane holds column lane % 32; register r holds row 8 (r / 4) + 4 (lane / 32) + r % 4
    const int64_t jblocks = (N + kResJ - 1) / kResJ;
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < WB; ++j) {
            const int col = n0 + wn + 32 * j + rl, row0 = m0 + wm + 32 * i + 4 * hi;
            if (col >= N) continue;
            float* p = BLOCKED ? C + result_off(jblocks, batch, ch, row0, col) : C + ch * sC + (int64_t)row0 * ldc + col;
            const int64_t rs = BLOCKED ? jblocks * batch * kResJ : ldc;
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = acc[i][j][r];
            if (accumulate) {   // all 16 loads together; a row past M reads the block's first one
                if (row0 >= M) continue;
                float old[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 8 * (r >> 2) + (r & 3);
                    old[r] = p[(row0 + dr < M ? dr : 0) * rs];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] += old[r];
            }
            const bool full = m0 + T <= M;   // uniform: no per-row guards
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                if (full || row0 + dr < M) p[dr * rs] = v[r];
            }
        }
}

__global__ void k_stage_kmask(const uint8_t* __restrict__ mask, int klen, int padded, uint8_t* __restrict__ dst) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < padded) dst[k] = (k < klen && (!mask || mask[k] != 0)) ? 1 : 0;
}

// Repack a device tile's row-major panel [ch][rows][ld] (bf16) into the
// blocked operand layout of the contraction, [ch][tiles][nk][256][32], with
// the staged k-mask applied and zeros for rows >= rows and k >= klen (the
// staged mask is 0 there).  One work-group per (two k-steps, 256-row tile,
// channel).  Thread t moves 16-byte piece e = t % 8 of the 128 bytes (two
// k-steps) of rows t / 8 + 32 j, j < 8: a load instruction reads eight whole
// 128-byte row segments, a store writes two runs of eight consecutive
// 64-byte block rows (one per k-step).
__global__ __launch_bounds__(256) void k_panel_block(const bf16_t* __restrict__ P, int rows, int ld, int64_t sP,
                                                     int tiles, int nk, const uint8_t* __restrict__ kst,
                                                     bf16_t* __restrict__ dst) {
    // Work-groups are dealt to the 8 XCDs round-robin by linear index; give
    // each XCD a contiguous run of (k-step pair, tile, channel) units, k-step
    // pairs fastest, so that the two 128-byte lines a row segment straddles
    // (rows are ld * 2 bytes apart, rarely a multiple of 128) are fetched
    // into one XCD's L2 and serve both neighbouring units.
    const unsigned gx = gridDim.x, gy = gridDim.y;
    const unsigned nu = gx * gy * gridDim.z, lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
    const unsigned per = nu >> 3, extra = nu & 7, xcd = lin & 7;
    const unsigned u = xcd * per + min(xcd, extra) + (lin >> 3);   // a bijection of [0, nu)
    const int kp = (int)(u % gx), tile = (int)((u / gx) % gy), c = (int)(u / (gx * gy)), t = threadIdx.x;
    const int r0 = tile * 256;
    const int nrow = min(256, rows - r0);
    const int e = t & 7, h = e >> 2, q = e & 3;   // k-step 2 kp + h, k = 8 q .. + 7 within it
    const int kt = 2 * kp + h;
    // rows past the panel fall outside the descriptor and read as zero
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(P + c * sP + (int64_t)r0 * ld, (uint32_t)nrow * (uint32_t)ld * 2u);
    uint4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = buf_load16(rp, (uint32_t)(((t >> 3) + 32 * j) * ld + kp * 64 + 8 * e) * 2u);
    if (kt >= nk) return;   // the odd last k-step of the panel has no second half
    // staged 0/1 bytes of k = 32 kt + 8 q .. + 7 (fresh for every k < 32 nk)
    const uint2 m8 = *reinterpret_cast<const uint2*>(kst + kt * 32 + 8 * q);
    const uint32_t mw[2] = {m8.x, m8.y};
    uint32_t keep[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b2 = mw[i >> 1] >> (16 * (i & 1));
        keep[i] = ((b2 & 0xffu) ? 0xffffu : 0u) | ((b2 & 0xff00u) ? 0xffff0000u : 0u);
    }
    bf16_t* out = dst + (((int64_t)c * tiles + tile) * nk + kt) * (256 * 32) + 8 * q;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        *reinterpret_cast<uint4*>(out + ((t >> 3) + 32 * j) * 32) =
            make_uint4(v[j].x & keep[0], v[j].y & keep[1], v[j].z & keep[2], v[j].w & keep[3]);
}

}  // namespace

hipError_t launch_panel_block(const void* P, int64_t rows, int64_t ld, int64_t klen, int nch, const uint8_t* kst,
                              void* dst, hipStream_t s) {
    const int tiles = (int)((rows + 255) / 256), nk = (int)((klen + 31) / 32);
    hipLaunchKernelGGL(k_panel_block, dim3((unsigned)((nk + 1) / 2), (unsigned)tiles, (unsigned)nch), dim3(256), 0, s,
                       (const bf16_t*)P, (int)rows, (int)ld, rows * ld, tiles, nk, kst, (bf16_t*)dst);
    return hipGetLastError();
}

// The pair-blocked result is addressed per 64 rows of a column block with
// 32-bit byte offsets: 64 rows of jblocks * batch * 32 floats must stay
// below 4 GiB (N = 65536 with 128 channels uses half of it).
bool cblocked_fits(int64_t N, int batch) {
    const int64_t rs = (N + kResJ - 1) / kResJ * batch * kResJ;
    return 64 * rs * 4 < ((int64_t)1 << 32);
}

// Pacing needs whole XCD groups (G a multiple of 8, all resident) and at
// least two full rounds; it resets the counters first (a kernel, not a
// memset, so that the sequence can be captured in a graph).  It pays only for
// long tiles: shorter ones drift apart less than the wait and the reset cost
// (N = 4096 13.67 ms paced, 13.96 not; N = 2048 1954 against 1910 us, N = 1300
// 695 against 649, N = 512 55 against 51).  The line itself was put between the
// two.  Measured around it since: square products lose up to about 3900 (N =
// 3072 6.03 ms paced, 5.87 not; 3584 9.48 and 9.18; 3840 11.56 and 11.28) and gain
// above (5120 26.9 and 27.3; 6144 46.0 and 47.9); an accumulating ring step of
// 3000 tokens gains (6.49 against 6.73), one of 2560 loses (4.18 against 3.93).
constexpr int64_t kPaceMinK = 3072;
namespace {
int pace_launch(int grid, int total, int64_t K, hipStream_t s) {
    if ((grid & 7) != 0 || total < 2 * grid || K < kPaceMinK) return 0;
    hipLaunchKernelGGL(k_pace_reset, dim3(1), dim3(8 * kPaceLine), 0, s);
    return 1;
}
}  // namespace

namespace {
// One launch of the bf16 contraction (arguments as launch_contract's).
template <bool BLOCKED, bool KMASK, bool CBLOCKED, bool TA = false, bool TB = false>
hipError_t launch_ws(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                     int64_t ldc, int64_t sA, int64_t sB, int64_t sC, int batch, int accumulate, const uint8_t* kmask,
                     int cus, hipStream_t s) {
    if (CBLOCKED && !cblocked_fits(N, batch)) return hipErrorInvalidValue;
    const K2Side sm = k2_side(TA ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, (int)M);
    const K2Side sn = k2_side(TB ? kK2Transposed : BLOCKED ? kK2Blocked : kK2RowMajor, (int)N);
    const int total = sm.tiles * sn.tiles * batch;
    const int grid = total < cus ? total : cus;
    const int pace = pace_launch(grid, total, K, s);
    const bool ragged = sm.units != 4 * sm.tiles || sn.units != 4 * sn.tiles;
#define K2_WS(R_)                                                                                                  \
    hipLaunchKernelGGL((k2_contract_ws<BLOCKED, KMASK, CBLOCKED, TA, TB, R_>), dim3(grid), dim3(768), 0, s,        \
                       (const bf16_t*)A, (const bf16_t*)B, C, (int)M, (int)N, (int)K, (int)lda, (int)ldb, ldc, sA, \
                       sB, sC, total, accumulate, kmask, pace)
    if constexpr (BLOCKED) {   // row-major operands have whole tiles only
        if (ragged) K2_WS(true);
        else K2_WS(false);
    } else {
        K2_WS(false);
    }
#undef K2_WS
    return hipGetLastError();
}
}  // namespace

hipError_t launch_contract_blocked_rowc(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K,
                                        int batch, int accumulate, int cus, hipStream_t s) {
    return launch_ws<true, false, false>(A, B, C, M, N, K, 0, 0, N, 0, 0, M * N, batch, accumulate, nullptr, cus, s);
}

hipError_t launch_contract_blocked_packed(const void* A, const void* B, float* C, int64_t M, int64_t N, int64_t K,
                                          int batch, int accumulate, int cus, hipStream_t s) {
    return launch_ws<true, false, true>(A, B, C, M, N, K, 0, 0, 0, 0, 0, 0, batch, accumulate, nullptr, cus, s);
}

hipError_t launch_contract_transposed(int ta, int tb, const void* A, const void* B, float* C, int64_t M, int64_t N,
                                      int64_t K, int batch, int cus, hipStream_t s, int accumulate) {
    if (!ta && !tb) return hipErrorInvalidValue;
    if (!ta) return launch_ws<true, false, true, false, true>(A, B, C, M, N, K, 0, 0, 0, 0, 0, 0, batch, accumulate, nullptr, cus, s);
    if (tb) return launch_ws<true, false, true, true, true>(A, B, C, M, N, K, 0, 0, 0, 0, 0, 0, batch, accumulate, nullptr, cus, s);
    return launch_ws<true, false, true, true, false>(A, B, C, M, N, K, 0, 0, 0, 0, 0, 0, batch, accumulate, nullptr, cus, s);
}

hipError_t launch_stage_kmask(const uint8_t* mask, int64_t klen, uint8_t* dst, hipStream_t s) {
    const int padded = (int)((klen + 31) / 32 * 32);
    hipLaunchKernelGGL(k_stage_kmask, dim3((padded + 255) / 256), dim3(256), 0, s, mask, (int)klen, padded, dst);
    return hipGetLastError();
}

// Tiles of 128 halve the L2 traffic of a product, tiles of 64 give four times
// the work-groups and pad less.  128 from 16 tiles per compute unit on where
// its padding costs at most 5% (N = 1024: 2.01 against 2.18 ms; equal at N =
// 512; at N = 384 148 against 128 us, at N = 700 792 against 719, at N = 64 8.9
// against 7.5).
int contract_f32_tile(int64_t M, int64_t N, int batch, int cus) {
    const int64_t t1 = (M + 127) / 128 * ((N + 127) / 128), t2 = (M + 63) / 64 * ((N + 63) / 64);
    return t1 * batch >= 16 * (int64_t)cus && 80 * t1 <= 21 * t2 ? 128 : 64;
}

hipError_t launch_contract(int dtype, int blocked, const void* A, const void* B, float* C, int64_t M,
                           int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc, int64_t sA,
                           int64_t sB, int64_t sC, int batch, int accumulate, const uint8_t* kmask, int cus,
                           hipStream_t s) {
    if (dtype == 0) {
        const int T = contract_f32_tile(M, N, batch, cus);
        const bool wide = T == 128;
        const int tm = (int)((M + T - 1) / T), tn = (int)((N + T - 1) / T);
#define K2_F32(T_, BL_)                                                                                             \
    hipLaunchKernelGGL((k2_contract_f32<T_, BL_>), dim3((unsigned)(tm * tn * batch)), dim3(256), 0, s,              \
                       (const float*)A, (const float*)B, C, (int)M, (int)N, (int)K, lda, ldb, ldc, sA, sB, sC, tm, \
                       tn, batch, accumulate, kmask)
        if (wide && blocked) K2_F32(128, true);
        else if (wide) K2_F32(128, false);
        else if (blocked) K2_F32(64, true);
        else K2_F32(64, false);
#undef K2_F32
        return hipGetLastError();
    }
    if (blocked) {   // the k-mask of a blocked operand was applied when it was written
        if (kmask) return hipErrorInvalidValue;
        return launch_ws<true, false, true>(A, B, C, M, N, K, 0, 0, 0, 0, 0, 0, batch, accumulate, nullptr, cus, s);
    }
    if (kmask) return launch_ws<false, true, false>(A, B, C, M, N, K, lda, ldb, ldc, sA, sB, sC, batch, accumulate, kmask, cus, s);
    return launch_ws<false, false, false>(A, B, C, M, N, K, lda, ldb, ldc, sA, sB, sC, batch, accumulate, nullptr, cus, s);
}

// Host-side walk over the direct-to-LDS loads of one k2_contract_ws launch,
// computed with the kernel's own addressing functions (k2_addr.h).
//
// Tile order: every (channel, row tile, column tile) must be taken by exactly
// one (work-group, round) of the persistent grid.  Loads: for the channels in
// `chans` (the kernel's addressing is the same in every channel apart from
// the channel offset, so the first and last channel bound it), every row tile
// of A and every column tile of B, every step, loader wave, load, lane and
// element: the descriptor must lie inside the operand's allocation (base >= 0,
// base + range <= bytes, range a multiple of 16), and every element the tile
// needs (row < rows, k < K) must be inside the range at the byte address the
// operand's layout gives it.  Elements the tile does not need (rows past the
// operand, k past K) may read anything inside the range, or zeros.
namespace {
int64_t k2_layout_off(const K2Operand& op, int ch, int64_t row, int64_t k) {
    if (op.mode == kK2Blocked) return panel_off(panel_geom(op.rows, op.K), ch, row, k);
    if (op.mode == kK2RowMajor) return (int64_t)ch * op.stride + row * op.ld + k;
    return panel_off(panel_geom(op.K, op.rows), ch, k, row);   // X[k][row] in the panel layout of X
}

void k2_check_operand(const K2Operand& op, uint64_t bytes, int ch, K2CheckCounts& n) {
    const int nk = (op.K + kK2BK - 1) / kK2BK;
    const K2Side side = k2_side(op.mode, op.rows);
    for (int tt = 0; tt < side.tiles; ++tt) {
        int t0, units;
        k2_span(side, tt, t0, units);
        for (int kt = 0; kt < nk; ++kt) {
            const K2Desc d = k2_desc(op, ch, t0, kt);
            const bool desc_ok = d.base >= 0 && (d.range % 16) == 0 && (uint64_t)d.base * 2 + d.range <= bytes;
            for (int lw = 0; lw < kK2Loaders; ++lw)
                for (int jj = 0; jj < kK2LoadsPerOperand; ++jj) {
                    uint32_t off = 0;
                    const bool in = k2_load_off(op, t0, units, kt, lw, jj, off);
                    ++n.loads;
                    if (in && !desc_ok) ++n.bad_desc;
                    const uint32_t lds = k2_lds_off(lw, jj);
                    for (int lane = 0; lane < 64; ++lane) {
                        const uint64_t voff = (uint64_t)k2_lane_off(op, lw, lane) + off;
                        if (voff + 16 > 0xffffffffull) ++n.bad_elem;   // the lane offset is 32-bit
                        const uint32_t lb = lds + 16u * (uint32_t)lane;   // LDS byte the lane's 16 bytes go to
                        for (int e = 0; e < 8; ++e) {
                            int64_t row, k;
                            if (op.mode == kK2Transposed) {   // 2 KB per 32-column block, 64 bytes per k row
                                const int blk = (int)(lb / 2048), kr = (int)(lb % 2048) / kK2Row;
                                row = t0 + 32 * blk + ((lb % kK2Row) / 2 + e);
                                k = (int64_t)kt * kK2BK + kr;
                            } else {   // row r, slot s holds chunk s ^ ((r >> 2) & 3)
                                const int r = (int)(lb / kK2Row), slot = (int)(lb % kK2Row) / 16;
                                row = t0 + r;
                                k = (int64_t)kt * kK2BK + 8 * (slot ^ ((r >> 2) & 3)) + e;
                            }
                            if (row >= op.rows || row >= t0 + units * kK2Unit || k >= op.K) continue;   // not needed by the tile
                            ++n.elems;
                            const uint64_t byte = voff + 2u * (uint32_t)e;
                            const bool hit = in && byte + 2 <= d.range &&
                                             d.base * 2 + (int64_t)byte == 2 * k2_layout_off(op, ch, row, k);
                            if (!hit) ++n.bad_elem;
                        }
                    }
                }
        }
    }
}
}  // namespace

namespace {
void k2_check_c_sides(const K2Side& sm, const K2Side& sn, int64_t M, int64_t N, int batch, uint64_t c_bytes,
                      int all_channels, K2CheckCounts& n) {
    const int J = (int)((N + kResJ - 1) / kResJ);
    const uint32_t crs = k2_c_row_floats((int)N, batch);
    n.tiles = (int64_t)sm.tiles * sn.tiles * batch;
    for (int ch = 0; ch < batch; ++ch) {
        if (!all_channels && ch != 0 && ch != batch - 1) continue;
        std::vector<uint8_t> hit((size_t)M * (size_t)N, 0);
        for (int ti = 0; ti < sm.tiles; ++ti)
            for (int tj = 0; tj < sn.tiles; ++tj) {
                const K2Tile t = k2_tile(sm, sn, ch, ti, tj);
                for (int wave = 0; wave < 8; ++wave) {
                    const K2Wave w = k2_wave(t, wave);
                    for (int j = 0; j < w.cols; ++j) {
                        const K2Desc d = k2_c_desc((int)M, (int)N, batch, t, w, j);
                        if (d.range && (d.base < 0 || (uint64_t)d.base * 4 + d.range > c_bytes)) ++n.bad_desc;
                        for (int i = 0; i < w.rows; ++i) {
                            const int x = 4 * i + j;
                            ++n.loads;
                            for (int r = 0; r < 16; ++r)
                                for (int lane = 0; lane < 64; ++lane) {
                                    int row, col;
                                    k2_c_elem(t, wave, lane, x, r, row, col);
                                    const uint64_t off = (uint64_t)k2_c_lane_off(crs, lane) + k2_c_reg_off(crs, x, r);
                                    const bool in = off < d.range;
                                    if (!in) {   // must be a row past M or a column block past C's last
                                        if (row < M && col / kResJ < J) ++n.bad_elem;
                                        continue;
                                    }
                                    // accessed: the element the layout puts there, inside C
                                    const int64_t want = result_off(J, batch, ch, row, col);
                                    if (off % 4 || d.base + (int64_t)(off / 4) != want || row >= M || col / kResJ >= J)
                                        ++n.bad_elem;
                                    if (row < M && col < N) {
                                        ++n.elems;
                                        uint8_t& h = hit[(size_t)row * N + col];
                                        if (h) ++n.bad_elem;
                                        h = 1;
                                    }
                                }
                        }
                    }
                }
            }
        for (uint8_t h : hit) n.bad_elem += h ? 0 : 1;
    }
}
}  // namespace

void k2_check_c(int64_t M, int64_t N, int batch, uint64_t c_bytes, int all_channels, K2CheckCounts& n) {
    n = K2CheckCounts{};
    // the tile sides of two blocked operands, then every other pairing of
    // blocked and transposed sides that differs from those before it
    const K2Side sm[2] = {k2_side(kK2Blocked, (int)M), k2_side(kK2Transposed, (int)M)};
    const K2Side sn[2] = {k2_side(kK2Blocked, (int)N), k2_side(kK2Transposed, (int)N)};
    k2_check_c_sides(sm[0], sn[0], M, N, batch, c_bytes, all_channels, n);
    const bool dm = sm[0].units % 4 != 0 && sm[0].tiles > 1, dn = sn[0].units % 4 != 0 && sn[0].tiles > 1;
    for (int ta = 0; ta < 2; ++ta)
        for (int tb = 0; tb < 2; ++tb) {
            if ((!ta && !tb) || (ta && !dm) || (tb && !dn)) continue;
            K2CheckCounts e;
            k2_check_c_sides(sm[ta], sn[tb], M, N, batch, c_bytes, all_channels, e);
            if (e.elems != n.elems) ++n.bad_elem;
            n.bad_desc += e.bad_desc;
            n.bad_elem += e.bad_elem;
        }
}

void k2_check_loads(int a_mode, int b_mode, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t sA,
                    int64_t sB, int batch, uint64_t a_bytes, uint64_t b_bytes, int grid, int all_channels,
                    K2CheckCounts& n) {
    n = K2CheckCounts{};
    const K2Side sm = k2_side(a_mode, (int)M), sn = k2_side(b_mode, (int)N);
    const int64_t total = (int64_t)sm.tiles * sn.tiles * batch;
    std::vector<uint8_t> seen((size_t)total, 0);
    for (int wg = 0; wg < grid; ++wg) {
        const int perm = k2_perm(wg, grid), mine = k2_my_tiles(perm, grid, (int)total);
        for (int it = 0; it < mine; ++it) {
            int ch, ti, tj;
            k2_index(sm, sn, it * grid + perm, ch, ti, tj);
            const K2Tile t = k2_tile(sm, sn, ch, ti, tj);
            const bool ok = ch >= 0 && ch < batch && ti >= 0 && ti < sm.tiles && tj >= 0 && tj < sn.tiles && t.m0 < M &&
                            t.n0 < N && t.mu >= 1 && t.mu <= 4 && t.nu >= 1 && t.nu <= 4;
            if (!ok) {
                ++n.bad_tiles;
                continue;
            }
            uint8_t& v = seen[((size_t)ch * sm.tiles + ti) * sn.tiles + tj];
            if (v) ++n.bad_tiles;
            v = 1;
        }
    }
    for (uint8_t v : seen) n.bad_tiles += v ? 0 : 1;
    n.tiles = total;
    for (const K2Side* s : {&sm, &sn}) {   // the spans follow each other and cover the side
        int next = 0;
        for (int i = 0; i < s->tiles; ++i) {
            int t0, units;
            k2_span(*s, i, t0, units);
            if (t0 != next) ++n.bad_tiles;
            next = t0 + units * kK2Unit;
        }
        if (next != s->units * kK2Unit) ++n.bad_tiles;
    }
    const K2Operand opa{a_mode, (int)M, (int)K, (int)lda, sA}, opb{b_mode, (int)N, (int)K, (int)ldb, sB};
    for (int ch = 0; ch < batch; ++ch) {
        if (!all_channels && ch != 0 && ch != batch - 1) continue;
        k2_check_operand(opa, a_bytes, ch, n);
        k2_check_operand(opb, b_bytes, ch, n);
    }
}

}  // namespace trimul
