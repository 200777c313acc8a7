// Backward of the per-channel contraction (training; the paper gives every
// distributed module an explicit backward that runs the same schedule as its
// forward, Section 3.1).  With the channel-major operands of the forward,
// C[c] = A[c] B[c]^T, the gradients are two more products of the same size:
//
//     dA[c] = dC[c] B[c]        dB[c] = dC[c]^T A[c]
//
// and both are again "NT" products once the right operands are transposed:
// dA = NT(dC, B^T), dB = NT(dC^T, A^T).  This file holds the two layout
// kernels that prepare those operands in the blocked panel layout; the
// products run on the contraction kernels.
#include "common.h"
#include "kernels.h"

namespace trimul {
namespace {

// dC in the pair-blocked result layout (fp32) -> the panel layout, element
// (c, i, j) -> X_c[i][k = j], converted to T.  One unit = two rows i, i + 1
// (i even) and one 32-column block: 2 x 128 channels x 32 floats, contiguous
// per channel in the result layout; in the panel the two rows of a channel
// are adjacent (one 128-byte line in bf16), so no store writes a partial
// line.  Thread t moves channel t / 2, columns 16 (t % 2) .. + 15 of both
// rows.  Columns past N carry whatever the result layout holds there into
// the k padding of the panel, which the contraction never uses.
template <typename T>
__global__ __launch_bounds__(256) void k_result_to_panel(const float* __restrict__ R, T* __restrict__ P, int N,
                                                        int64_t units) {
    const int t = threadIdx.x, ch = t >> 1, h = t & 1;
    const int J = (N + kResJ - 1) / kResJ;
    const PanelGeom pg = panel_geom(N, N);
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int64_t ip = u / J, jb = u - (u / J) * J;
        const int64_t i0 = 2 * ip;
        const int nr = i0 + 1 < N ? 2 : 1;                 // an odd N's last unit holds one row
        float4 v[2][4];
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
            if (rr < nr) {
                const float4* src = reinterpret_cast<const float4*>(R + result_off(J, kCh, ch, i0 + rr, jb * kResJ) + 16 * h);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[rr][q] = src[q];
            }
        }
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
            if (rr >= nr) break;
            T* dst = P + panel_off(pg, ch, i0 + rr, jb * kResJ + 16 * h);
            if constexpr (sizeof(T) == 2) {
                uint4 o[2];
                o[0] = make_uint4(pack_bf16x2(v[rr][0].x, v[rr][0].y), pack_bf16x2(v[rr][0].z, v[rr][0].w),
                                  pack_bf16x2(v[rr][1].x, v[rr][1].y), pack_bf16x2(v[rr][1].z, v[rr][1].w));
                o[1] = make_uint4(pack_bf16x2(v[rr][2].x, v[rr][2].y), pack_bf16x2(v[rr][2].z, v[rr][2].w),
                                  pack_bf16x2(v[rr][3].x, v[rr][3].y), pack_bf16x2(v[rr][3].z, v[rr][3].w));
                reinterpret_cast<uint4*>(dst)[0] = o[0];
                reinterpret_cast<uint4*>(dst)[1] = o[1];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) reinterpret_cast<float4*>(dst)[q] = v[rr][q];
            }
        }
    }
}

// Per-channel transpose in the panel layout: Y_c[k][i] = X_c[i][k].  One wave
// moves one 32 x 32 block (rows 32 ib.., columns 32 kb..) through LDS: lane l
// reads 16 consecutive elements of row l / 2 (half l % 2) and writes 16
// consecutive elements of output row l / 2.  Blocks cover [0, 32 S)^2 with
// S = ceil(N / 32), which lies inside the panel allocation; padding elements
// move along with the rest.
template <typename T>
__global__ __launch_bounds__(256) void k_panel_transpose(const T* __restrict__ X, T* __restrict__ Y, int N,
                                                        int64_t blocks) {
    constexpr int kPad = 34;   // row stride (elements) of the wave's tile
    __shared__ T tile[4][32 * kPad];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int S = (N + 31) / 32;
    const PanelGeom pg = panel_geom(N, N);
    const int rr = lane >> 1, hh = lane & 1;
    T* tl = tile[w];
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t b = (int64_t)blockIdx.x * 4 + w; b < blocks; b += waves) {
        const int64_t ch = b / ((int64_t)S * S);
        const int64_t rem = b - ch * S * S;
        const int ib = (int)(rem / S), kb = (int)(rem - (int64_t)(rem / S) * S);
        const T* src = X + panel_off(pg, ch, 32 * ib + rr, 32 * kb + 16 * hh);   // 16 elements, 32 B aligned
        T* dst = Y + panel_off(pg, ch, 32 * kb + rr, 32 * ib + 16 * hh);
        T* trow = tl + rr * kPad + 16 * hh;
        if constexpr (sizeof(T) == 2) {
            const uint4 a0 = reinterpret_cast<const uint4*>(src)[0], a1 = reinterpret_cast<const uint4*>(src)[1];
            const uint32_t w8[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<uint32_t*>(trow)[q] = w8[q];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 f = reinterpret_cast<const float4*>(src)[q];
                reinterpret_cast<float*>(trow)[4 * q] = f.x;
                reinterpret_cast<float*>(trow)[4 * q + 1] = f.y;
                reinterpret_cast<float*>(trow)[4 * q + 2] = f.z;
                reinterpret_cast<float*>(trow)[4 * q + 3] = f.w;
            }
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        T v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = tl[(16 * hh + q) * kPad + rr];
        if constexpr (sizeof(T) == 2) {
            uint32_t w8[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                w8[q] = (uint32_t)__builtin_bit_cast(uint16_t, v[2 * q]) |
                        ((uint32_t)__builtin_bit_cast(uint16_t, v[2 * q + 1]) << 16);
            reinterpret_cast<uint4*>(dst)[0] = make_uint4(w8[0], w8[1], w8[2], w8[3]);
            reinterpret_cast<uint4*>(dst)[1] = make_uint4(w8[4], w8[5], w8[6], w8[7]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                reinterpret_cast<float4*>(dst)[q] = make_float4(__builtin_bit_cast(float, v[4 * q]),
                                                                __builtin_bit_cast(float, v[4 * q + 1]),
                                                                __builtin_bit_cast(float, v[4 * q + 2]),
                                                                __builtin_bit_cast(float, v[4 * q + 3]));
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// ---------------------------------------------------------------- layer backward
//
// Work unit = 32 pairs (one row r, columns k = 32 kb .. 32 kb + 31), the
// unit of the result layout.  The per-pair intermediates that feed the
// gradients of the projection weights are written as "unit blocks": for unit
// u = r * J + kb, a bf16 block [128 channels][32 slots] at u * 4096 elements.
// Each of those gradients is then a sum over units of U_block * V_block^T
// (k_wgrad4; the epilogue's two weights are summed in place); slots of pairs
// past N or masked out carry a zero in at least one of the two blocks.
//
// The per-pair stages are 128-wide products per unit, run on matrix cores
// (v_mfma_f32_16x16x32_bf16): 8 waves, wave w owns the 16 output columns
// 16 w .. 16 w + 15 of every product and keeps its slice of the weights in
// VGPRs as the B operand.  Activations are the A operand, split into
// bf16 hi + lo (two products), so the products carry about 16 mantissa bits
// of the fp32 activations; the weights are bf16 already.  Operand layout of
// the 16 x 16 x 32 product: lane l supplies row (or column) l % 16 and the
// eight k values 8 (l / 16) .. + 7; the result gives lane l column l % 16 and
// rows 4 (l / 16) + 0 .. 3.
constexpr int kQ = 32;        // pairs per unit
constexpr int kBT = 512;      // threads of the per-pair backward kernels
constexpr int kCs = 36;       // row stride (floats) of [channel][pair] tiles
constexpr int kPq = 148;      // row stride (floats) of [pair][channel] tiles (the fewest bank conflicts
                              // over their four access patterns)
constexpr int kArow = 256;    // bytes of one bf16 activation row [128]

// Byte offset of 16-byte chunk ch of row p in a bf16 [q][128] tile.  Chunks
// are XOR-swizzled by a bijection of the row's low four bits, so the A-operand
// reads (16 rows, one chunk each) hit distinct banks; row bits 0 and 1 move
// chunk bits 2 and 3, so the transposing reads (4 consecutive rows, 4
// consecutive chunks) do too, and row bits 2 and 3 move chunk bits 1 and 2,
// so the 2-byte stores of 16 columns in rows 4 apart do as well.
__device__ __forceinline__ uint32_t arow(int p, int ch) {
    return (uint32_t)(p * kArow + ((ch ^ ((p & 3) << 2) ^ ((p >> 1) & 2) ^ (((p >> 3) & 1) * 5)) << 4));
}

// A weight-gradient operand from such a tile, transposed: lane l gets column
// 32 blk + l % 32 of rows 16 ks + 8 (l / 32) .. + 7, i.e. eight pairs of one
// channel, through two ds_read_b64_tr_b16 (rows + 0 .. 3, then + 4 .. 7; row
// bit 2 moves chunk bit 1).  Lane 16 g + 4 i + a addresses row 8 (g >> 1) + i
// and columns 16 (g & 1) + 4 a .. + 3.
typedef short v4i16_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8_t ld_frag_tr(const char* tile, int lane, int ks, int blk) {
    typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;
    const int g = lane >> 4, a = lane & 3, q = 16 * ks + 8 * (g >> 1) + ((lane >> 2) & 3);
    const uint32_t o = arow(q, 4 * blk + 2 * (g & 1) + (a >> 1)) + 8 * (a & 1);
    const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(tile + o));
    const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(tile + ((o + 4 * kArow) ^ 32)));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The value itself, hidden from the optimiser: lane indices passed through
// this inside a loop make the LDS addresses derived from them loop-variant,
// so they are recomputed where used instead of being hoisted out of the loop
// and held in (or spilled from) registers for the whole kernel.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ float sum_lanes16(float v) {
    v = sum_lanes8(v);
    v += dpp_mov<0x140>(v);   // row_mirror: lane i meets lane 15 - i (the other group of 8)
    return v;
}

__device__ __forceinline__ void st_hilo(char* hi, char* lo, uint32_t off, float v) {
    const bf16_t h = f2bf(v);
    *reinterpret_cast<bf16_t*>(hi + off) = h;
    *reinterpret_cast<bf16_t*>(lo + off) = f2bf(v - bf2f(h));
}

__device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8_t ld_frag(const char* base, uint32_t off) {
    return *reinterpret_cast<const bf16x8_t*>(base + off);
}

// Range-checked buffer access (make_rsrc): loads past the resource's size
// read zero and stores past it are dropped, so tails need no branches and
// every pass of a unit loop issues the same memory instructions (which keeps
// the compiler's wait counts exact).
__device__ __forceinline__ float4 bld_f4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(float4, buf_load16(r, off));
}
__device__ __forceinline__ uint32_t bld_u8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b8(r, (int)off, 0, 0);
}
__device__ __forceinline__ void bst_f32(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)off, 0, 0);
}
__device__ __forceinline__ void bst_u4(__amdgpu_buffer_rsrc_t r, uint32_t off, uint4 v) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, 0);
}

// Four bf16 (rows 4 kq .. + 3 of one 16 x 16 result tile) as one 8-byte word.
__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
    return make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}

template <typename TO> struct DoutRegs;
template <> struct DoutRegs<float> { float4 a, b; };
template <> struct DoutRegs<bf16_t> { uint4 a; };

// Epilogue backward.  For the unit's pairs (r, k): recompute x = LN_in(z),
// y = LN_out(C), u = W_o y, g = sigmoid(W_g x); then
//   du = dout m g,  dgg = dout m u g (1 - g),  dy = du W_o,  dx_g = dgg W_g,
//   dC = LN_out backward of dy.
// Writes dC into the panel (row r, columns k), dx_g [pair][c_z] fp32, and
// per-work-group sums of dgamma_out, dbeta_out at partial[(2 wg + {0, 1}) * 128
// + c] and of the weight gradients
//   dW_o = sum du y^T,  dW_g = sum dgg x^T   (operands rounded to bf16)
// at wpart[wg] and wpart[grid + wg], [128][128] each.  Those sums run here,
// from the activation tiles in LDS (transposing reads) into 64 accumulator
// registers per lane: the four unit blocks they used to travel in were a third
// of the kernel's memory traffic, and two passes of their own read them back.
// N = 1024: 717 us and 2 x 120 us for those passes before, 767 now (about half
// of it LDS traffic: every wave reads all of the activations).
// All 256 registers are in use, and the fp32 instance keeps two values in
// scratch across the unit loop: stored before it, loaded after it.  Seven forms
// without that (an address recomputed in one phase or another) made the whole
// backward 0.3 to 1.6% slower at N = 1500 and none faster.
template <typename TO>
__global__ __launch_bounds__(kBT) void k_epilogue_backward(
    const float* __restrict__ C, const bf16_t* __restrict__ z, const uint8_t* __restrict__ mask,
    const TO* __restrict__ dout, int N, int64_t units, const bf16_t* __restrict__ wfwd,
    const bf16_t* __restrict__ wbwd, const float* __restrict__ lniw, const float* __restrict__ lnib,
    const float* __restrict__ lnow, const float* __restrict__ lnob, float eps, bf16_t* __restrict__ dCp,
    float* __restrict__ dxg, float* __restrict__ wpart, float* __restrict__ partial) {
    __shared__ __align__(16) float cs[kCh * kCs];        // C [c][q]
    __shared__ __align__(16) float dq[kQ * kPq];         // dout [q][d], then dy [q][c]
    __shared__ __align__(16) float dct[kCh * kCs];       // dC [c][q]
    __shared__ __align__(16) char act[4][kQ * kArow];    // y hi, y lo, x hi, x lo  [q][128]
    __shared__ __align__(16) char act2[4][kQ * kArow];   // du hi, du lo, dgg hi, dgg lo  [q][128]
    // gamma_out, beta_out, gamma_in, beta_in; rows 2 and 3 put channel d at
    // d + 4 (d / 64), so that the 16 addresses 8 l + 2 i of a LayerNorm-input
    // read fall in distinct banks
    __shared__ float prm[4][136];
    __shared__ float mq[kQ];                             // pair mask of the unit
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int lp = t >> 4, lq = t & 15;                  // LayerNorms: pair lp, 16 lanes per pair
    const int col = lane & 15, kq = lane >> 4;           // MFMA operand / result lanes
    const int sc = t >> 2, sq = t & 3;                   // channel-major stores: channel sc, pairs 8 sq .. + 7
    const int J = (N + kQ - 1) / kQ;
    const PanelGeom pg = panel_geom(N, N);

    // Global loads of one unit, issued one unit ahead into the registers the
    // current unit has just released; nothing here reads the loaded
    // registers, so the loads stay in flight until the unit starts.
    struct Pre {
        float4 c0, c1;        // C block floats 4 t .. and 2048 + 4 t ..
        uint4 zv;             // z of pair lp, channels 8 lq .. + 7
        DoutRegs<TO> o;       // dout of pair lp, channels 8 lq .. + 7
        uint32_t mr, mk;      // mask bytes of row r and of column k0 + t % 32 (zero past N)
    };
    auto load = [&](int64_t u, Pre& p) {
        const bool valid = u < units;                     // past the end: zero-size resources
        const int64_t uu = valid ? u : 0;
        const int r = (int)(uu / J), k0 = (int)(uu - (int64_t)r * J) * kQ;
        const int np = min(kQ, N - k0);
        const int64_t pr0 = (int64_t)r * N + k0;          // the unit's first pair
        const auto rc = make_rsrc(C + uu * (kCh * kQ), valid ? kCh * kQ * 4 : 0);
        p.c0 = bld_f4(rc, 16 * t);
        p.c1 = bld_f4(rc, 16 * (t + kBT));
        const auto rzr = make_rsrc(z + pr0 * kCz, valid ? np * kCz * 2 : 0);
        p.zv = buf_load16(rzr, lp * kCz * 2 + 16 * lq);
        if constexpr (sizeof(TO) == 4) {
            const auto ro = make_rsrc(dout + pr0 * kCz, valid ? np * kCz * 4 : 0);
            p.o.a = bld_f4(ro, lp * kCz * 4 + 32 * lq);
            p.o.b = bld_f4(ro, lp * kCz * 4 + 32 * lq + 16);
        } else {
            const auto ro = make_rsrc(dout + pr0 * kCz, valid ? np * kCz * 2 : 0);
            p.o.a = buf_load16(ro, lp * kCz * 2 + 16 * lq);
        }
        const auto rm = make_rsrc(mask, (valid && mask) ? (uint32_t)N : 0u);
        p.mr = bld_u8(rm, opaque(r));                    // per lane: a uniform load would be waited for at once
        p.mk = bld_u8(rm, k0 + (t & (kQ - 1)));
    };

    float accg[8], accb[8];                              // dgamma_out, dbeta_out of c = lq + 16 i
#pragma unroll
    for (int i = 0; i < 8; ++i) accg[i] = accb[i] = 0.f;
    f32x16_t gwo[2], gwg[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) gwo[j][i] = gwg[j][i] = 0.f;
    Pre cur;
    load(blockIdx.x, cur);
    bf16x8_t wo[4], wg[4], wot[4], wgt[4];               // B operands: W_o, W_g rows n; W_o^T, W_g^T rows n
    {
        const int n = 16 * w + col;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int k = 32 * ks + 8 * kq;
            wo[ks] = *reinterpret_cast<const bf16x8_t*>(wfwd + n * 128 + k);
            wg[ks] = *reinterpret_cast<const bf16x8_t*>(wfwd + (128 + n) * 128 + k);
            wot[ks] = *reinterpret_cast<const bf16x8_t*>(wbwd + n * 128 + k);
            wgt[ks] = *reinterpret_cast<const bf16x8_t*>(wbwd + (128 + n) * 128 + k);
        }
    }
    if (t < 128) {
        prm[0][t] = lnow[t];
        prm[1][t] = lnob[t];
        prm[2][t + 4 * (t >> 6)] = lniw[t];
        prm[3][t + 4 * (t >> 6)] = lnib[t];
    }

    // Everything issued so far completes here, in a wait the compiler sees
    // (otherwise its waits for the weights land inside the unit loop).
    wait_vmcnt<0>();
    __syncthreads();

    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int r = (int)(u / J), k0 = (int)(u - (int64_t)r * J) * kQ;
        const int np = min(kQ, N - k0);
        {   // stage C (columns past N read as zero) and the pair mask
            const int c = t >> 3, q = 4 * (t & 7);
            float4 a = cur.c0, b = cur.c1;
            if (q + 4 > np) {
                if (q + 0 >= np) a.x = b.x = 0.f;
                if (q + 1 >= np) a.y = b.y = 0.f;
                if (q + 2 >= np) a.z = b.z = 0.f;
                if (q + 3 >= np) a.w = b.w = 0.f;
            }
            *reinterpret_cast<float4*>(&cs[c * kCs + q]) = a;
            *reinterpret_cast<float4*>(&cs[(c + 64) * kCs + q]) = b;
            if (t < kQ) mq[t] = (t < np && (!mask || (cur.mr != 0 && cur.mk != 0))) ? 1.f : 0.f;
        }
        {   // LN_in of pair lp over d = 8 lq + i -> x hi / lo rows; dout -> dq
            const uint32_t zw[4] = {cur.zv.x, cur.zv.y, cur.zv.z, cur.zv.w};
            float x[8], s1 = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = __uint_as_float(zw[i] << 16);
                x[2 * i + 1] = __uint_as_float(zw[i] & 0xffff0000u);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) s1 += x[i];
            const float mz = sum_lanes16(s1) * (1.f / kCz);
            float q2 = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) { x[i] -= mz; q2 += x[i] * x[i]; }
            const float rz = rsqrtf(sum_lanes16(q2) * (1.f / kCz) + eps);
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int d = 8 * lq + 2 * i;
                const int dp = d + 4 * (d >> 6);             // padded position of d, d + 1
                const float x0 = x[2 * i] * rz * prm[2][dp] + prm[3][dp];
                const float x1 = x[2 * i + 1] * rz * prm[2][dp + 1] + prm[3][dp + 1];
                hw[i] = pack_bf16x2(x0, x1);
                lw[i] = pack_bf16x2(x0 - __uint_as_float(hw[i] << 16), x1 - __uint_as_float(hw[i] & 0xffff0000u));
            }
            *reinterpret_cast<uint4*>(act[2] + arow(lp, lq)) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            *reinterpret_cast<uint4*>(act[3] + arow(lp, lq)) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
            float4 o0, o1;
            if constexpr (sizeof(TO) == 4) {
                o0 = cur.o.a;
                o1 = cur.o.b;
            } else {
                const uint4 v = cur.o.a;
                o0 = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                                 __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
                o1 = make_float4(__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xffff0000u),
                                 __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xffff0000u));
            }
            *reinterpret_cast<float4*>(&dq[lp * kPq + 8 * lq]) = o0;
            *reinterpret_cast<float4*>(&dq[lp * kPq + 8 * lq + 4]) = o1;
        }
        load(u + gridDim.x, cur);                        // the next unit, into the released registers
        __syncthreads();
        float yh[8], rs;                                 // LN_out(C) normalised, c = lq + 16 i; 1 / std
        {   // LN_out of pair lp over c = lq + 16 i -> y hi / lo rows
            float s1 = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) { yh[i] = cs[(lq + 16 * i) * kCs + lp]; s1 += yh[i]; }
            const float mu = sum_lanes16(s1) * (1.f / kCh);
            float q2 = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) { yh[i] -= mu; q2 += yh[i] * yh[i]; }
            rs = rsqrtf(sum_lanes16(q2) * (1.f / kCh) + eps);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = lq + 16 * i;
                yh[i] *= rs;
                st_hilo(act[0], act[1], arow(lp, c >> 3) + 2 * (c & 7), yh[i] * prm[0][c] + prm[1][c]);
            }
        }
        __syncthreads();
        {   // u = y W_o^T, gg = x W_g^T (columns d = 16 w + col); du, dgg
            f32x4_t au[2], ag[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) au[mb] = ag[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    const uint32_t o = arow(16 * mb + col, 4 * ks + kq);
                    au[mb] = mfma16(ld_frag(act[0], o), wo[ks], au[mb]);
                    ag[mb] = mfma16(ld_frag(act[2], o), wg[ks], ag[mb]);
                    au[mb] = mfma16(ld_frag(act[1], o), wo[ks], au[mb]);
                    ag[mb] = mfma16(ld_frag(act[3], o), wg[ks], ag[mb]);
                }
            const int d = 16 * w + col;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = 16 * mb + 4 * kq + i;
                    const float o = dq[q * kPq + d] * mq[q];
                    const float g = sigmoidf_(ag[mb][i]);
                    const uint32_t off = arow(q, d >> 3) + 2 * (d & 7);
                    st_hilo(act2[0], act2[1], off, o * g);
                    st_hilo(act2[2], act2[3], off, o * au[mb][i] * g * (1.f - g));
                }
            }
        }
        __syncthreads();
        {   // dy = du W_o -> dq; dx_g = dgg W_g -> HBM (columns n = 16 w + col)
            f32x4_t ay[2], ax[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) ay[mb] = ax[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    const uint32_t o = arow(16 * mb + col, 4 * ks + kq);
                    ay[mb] = mfma16(ld_frag(act2[0], o), wot[ks], ay[mb]);
                    ax[mb] = mfma16(ld_frag(act2[2], o), wgt[ks], ax[mb]);
                    ay[mb] = mfma16(ld_frag(act2[1], o), wot[ks], ay[mb]);
                    ax[mb] = mfma16(ld_frag(act2[3], o), wgt[ks], ax[mb]);
                }
            const int n = 16 * w + col;
            const auto rx = make_rsrc(dxg + ((int64_t)r * N + k0) * kCz, np * kCz * 4);   // pairs past N: dropped
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = 16 * mb + 4 * kq + i;
                    dq[q * kPq + n] = ay[mb][i];
                    bst_f32(rx, (q * kCz + n) * 4, ax[mb][i]);
                }
            // dW_o, dW_g: rows d = 32 (w / 2) .., columns 64 (w % 2) ..
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int lo = opaque(lane);
                const bf16x8_t fu = ld_frag_tr(act2[0], lo, ks, w >> 1), fg = ld_frag_tr(act2[2], lo, ks, w >> 1);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    gwo[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fu, ld_frag_tr(act[0], lo, ks, 2 * (w & 1) + j), gwo[j], 0, 0, 0);
                    gwg[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fg, ld_frag_tr(act[2], lo, ks, 2 * (w & 1) + j), gwg[j], 0, 0, 0);
                }
            }
        }
        __syncthreads();
        {   // LN_out backward of pair lp: dC = rs (dy gamma - mean(dy gamma) - yh mean(dy gamma yh))
            float dy[8], s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = lq + 16 * i;
                dy[i] = dq[lp * kPq + c];
                const float dh = dy[i] * prm[0][c];
                s1 += dh;
                s2 += dh * yh[i];
            }
            s1 = sum_lanes16(s1) * (1.f / kCh);
            s2 = sum_lanes16(s2) * (1.f / kCh);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = lq + 16 * i;
                dct[c * kCs + lp] = rs * (dy[i] * prm[0][c] - s1 - yh[i] * s2);
                accg[i] += dy[i] * yh[i];
                accb[i] += dy[i];
            }
        }
        __syncthreads();
        {   // dC row r, columns k0 + 8 sq .. + 7 of channel sc into the panel
            const float4 a = *reinterpret_cast<const float4*>(&dct[sc * kCs + 8 * sq]);
            const float4 b = *reinterpret_cast<const float4*>(&dct[sc * kCs + 8 * sq + 4]);
            *reinterpret_cast<uint4*>(dCp + panel_off(pg, sc, r, k0 + 8 * sq)) =
                make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
        }
    }
    {   // lane holds column lane % 32; register i holds row 8 (i / 4) + 4 (lane / 32) + i % 4
        float* pw = wpart + (int64_t)blockIdx.x * (kCh * kCh) + (32 * (w >> 1) + 4 * (lane >> 5)) * kCh + 64 * (w & 1) + (lane & 31);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int o = (8 * (i >> 2) + (i & 3)) * kCh + 32 * j;
                pw[o] = gwo[j][i];
                pw[(int64_t)gridDim.x * (kCh * kCh) + o] = gwg[j][i];
            }
    }
    // per-work-group sums over the pairs lanes (lp) through LDS
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        cs[lp * kCh + lq + 16 * i] = accg[i];
        dct[lp * kCh + lq + 16 * i] = accb[i];
    }
    __syncthreads();
    if (t < 2 * kCh) {
        const float* src = t < kCh ? cs : dct;
        const int c = t & (kCh - 1);
        float s = 0.f;
        for (int q = 0; q < kQ; ++q) s += src[q * kCh + c];
        partial[((int64_t)blockIdx.x * 2 + (t >> 7)) * kCh + c] = s;
    }
}

// Projection backward.  Unit (r, kb) of dA / dB; its pairs are P(q) = (r, k)
// (outgoing) or (k, r) (incoming).  Recompute x = LN_in(z) and the four
// projections p_a, g_a, p_b, g_b (pre-sigmoid gates); then
//   dpa = da m s_a,  dga = da m p_a s_a (1 - s_a)  (the same for b),
//   dx = dx_g + [dpa dga dpb dgb] [W_a; W_ga; W_b; W_gb],  dz = LN_in backward of dx
// (the four gradients enter that product rounded to bf16; x enters the
// projections as bf16 hi + lo).
// Writes dz, unit blocks dpa, dga, dpb, dgb, x, and per-work-group sums of
// dgamma_in, dbeta_in at partial[(2 wg + {0, 1}) * 128 + d].
//
// 8 waves, wave w owning the 16 output columns 16 w .. of every product, as in
// the epilogue backward, with both weight slices in registers: rows 16 w + col
// of W_a, W_ga, W_b, W_gb for the projections and row d = 16 w + col of
// [W_a^T | W_ga^T | W_b^T | W_gb^T] (512 long) for dx, 128 registers.  (Four
// waves of 32 columns read the gradients from LDS half as often, but fill the
// register file with one wave per SIMD, whose every wait stood alone: N =
// 1024 961 us, now 793; N = 384 166, now 144.)
constexpr int kPq4 = 136;     // [pair][channel] row stride: rows 4 apart land 32 banks apart
// Padded bf16 row tiles: a row of 128 (x) or 512 (the four gradients)
// values plus one 16-byte chunk, so the 16 rows an operand read touches
// start 4 banks apart (conflict-free) and every access is the lane's base
// address plus an immediate offset.
constexpr int kXrow = 256 + 16;
constexpr int kGrow = 1024 + 16;

// 8 bf16 of column `col` of a padded [q][128] bf16 tile, rows q0 .. q0 + 7, packed.
__device__ __forceinline__ uint4 gather_col8p(const char* tile, int q0, int col) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = *reinterpret_cast<const bf16_t*>(tile + (q0 + 2 * i) * kXrow + 2 * col);
        const uint32_t b = *reinterpret_cast<const bf16_t*>(tile + (q0 + 2 * i + 1) * kXrow + 2 * col);
        w[i] = a | (b << 16);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

template <bool INCOMING>
__global__ __launch_bounds__(kBT) void k_projection_backward(
    const bf16_t* __restrict__ z, const uint8_t* __restrict__ mask, int N, int64_t units, const float* __restrict__ dA,
    const float* __restrict__ dB, const float* __restrict__ dxg, const bf16_t* __restrict__ wproj,
    const bf16_t* __restrict__ wprojt, const float* __restrict__ lniw, const float* __restrict__ lnib, float eps,
    bf16_t* __restrict__ dz, bf16_t* __restrict__ b_dpa, bf16_t* __restrict__ b_dga, bf16_t* __restrict__ b_dpb,
    bf16_t* __restrict__ b_dgb, bf16_t* __restrict__ b_x, float* __restrict__ partial) {
    __shared__ __align__(16) float das[kCh * kCs];       // da [c][q]
    __shared__ __align__(16) float dbs[kCh * kCs];       // db [c][q]
    __shared__ __align__(16) char xa[2][kQ * kXrow];     // x hi, x lo  [q][128]
    __shared__ __align__(16) char d4[kQ * kGrow];        // bf16 [q][dpa | dga | dpb | dgb]
    __shared__ __align__(16) float dxs[kQ * kPq4];       // dx from the projections [q][d]
    __shared__ __align__(16) float xhs[kQ * kPq4];       // LN_in(z) normalised [q][d]
    __shared__ float rzs[kQ];                            // 1 / std of LN_in per pair
    __shared__ __align__(16) float prm[2][128];          // gamma_in, beta_in
    __shared__ float mq[kQ];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int lp = t >> 4, lq = t & 15;                  // LayerNorm: pair lp, d = 8 lq .. + 7
    const int J = (N + kQ - 1) / kQ;
    auto pair_of = [&](int r, int k) -> int64_t { return INCOMING ? (int64_t)k * N + r : (int64_t)r * N + k; };

    // One unit's loads, issued one unit ahead; dx_g is fetched separately
    // (it is used last).  Nothing here reads the loaded registers.
    struct Pre {
        float4 a[2], b[2];       // dA, dB block floats 4 (t + 512 s) ..
        uint4 z0;                // z of pair lp, channels 8 lq .. + 7
        uint32_t mr, mk;
    };
    // Byte distance between consecutive pairs of a unit in [pair][c_z]
    // tensors: adjacent columns (outgoing) or adjacent rows (incoming).
    const uint32_t step2 = INCOMING ? (uint32_t)N * kCz * 2 : kCz * 2;   // bf16
    const uint32_t step4 = 2 * step2;                                    // fp32
    auto load = [&](int64_t u, Pre& p) {
        const bool valid = u < units;                     // past the end: zero-size resources
        const int64_t uu = valid ? u : 0;
        const int r = (int)(uu / J), k0 = (int)(uu - (int64_t)r * J) * kQ;
        const int np = min(kQ, N - k0);
        const auto ra = make_rsrc(dA + uu * (kCh * kQ), valid ? kCh * kQ * 4 : 0);
        const auto rb = make_rsrc(dB + uu * (kCh * kQ), valid ? kCh * kQ * 4 : 0);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            p.a[s] = bld_f4(ra, 16 * (t + kBT * s));
            p.b[s] = bld_f4(rb, 16 * (t + kBT * s));
        }
        const auto rzr = make_rsrc(z + pair_of(r, k0) * kCz, valid ? (np - 1) * step2 + kCz * 2 : 0);
        p.z0 = buf_load16(rzr, lp * step2 + 16 * lq);
        const auto rm = make_rsrc(mask, (valid && mask) ? (uint32_t)N : 0u);
        p.mr = bld_u8(rm, opaque(r));                    // per lane: a uniform load would be waited for at once
        p.mk = bld_u8(rm, k0 + (t & (kQ - 1)));
    };
    auto load_dxg = [&](int64_t u, float4 (&g)[2]) {
        const bool valid = u < units;
        const int64_t uu = valid ? u : 0;
        const int r = (int)(uu / J), k0 = (int)(uu - (int64_t)r * J) * kQ;
        const int np = min(kQ, N - k0);
        const auto rg = make_rsrc(dxg + pair_of(r, k0) * kCz, valid ? (np - 1) * step4 + kCz * 4 : 0);
#pragma unroll
        for (int s = 0; s < 2; ++s) g[s] = bld_f4(rg, lp * step4 + 32 * lq + 16 * s);
    };

    float accg[8], accb[8];                              // dgamma_in, dbeta_in of d = 8 lq + i
#pragma unroll
    for (int i = 0; i < 8; ++i) accg[i] = accb[i] = 0.f;
    Pre cur;
    float4 xg[2];
    load(blockIdx.x, cur);
    load_dxg(blockIdx.x, xg);
    bf16x8_t wp[4][4], wt[16];   // wp[m][ks]: map m, k = 32 ks + 8 kq;  wt[ks]: k = 32 ks + 8 kq
    {
        const int c = 16 * w + (lane & 15), kq = lane >> 4;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                wp[m][ks] = *reinterpret_cast<const bf16x8_t*>(
                    wproj + ((int64_t)(c >> 5) * 128 + m * 32 + (c & 31)) * 128 + 32 * ks + 8 * kq);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            wt[ks] = *reinterpret_cast<const bf16x8_t*>(wprojt + (int64_t)c * 512 + 32 * ks + 8 * kq);
    }
    if (t < 128) {
        prm[0][t] = lniw[t];
        prm[1][t] = lnib[t];
    }
    // Everything issued so far completes here, in a wait the compiler sees:
    // otherwise it places the waits for the weights inside the unit loop,
    // where on later passes they stall on the next unit's prefetch.
    wait_vmcnt<0>();
    __syncthreads();   // the first unit's LN_in reads prm before the loop's first barrier

    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int r = (int)(u / J), k0 = (int)(u - (int64_t)r * J) * kQ;
        const int np = min(kQ, N - k0);
        float xh[8], rz;   // LN_in(z) normalised, d = 8 lq + i, and 1 / std: to LDS after the barrier
        {   // stage da, db and the mask; LN_in of pair lp -> x hi / lo rows
            const int t = opaque(threadIdx.x), lp = t >> 4, lq = t & 15;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int c = (t >> 3) + 64 * s, q = 4 * (t & 7);
                *reinterpret_cast<float4*>(&das[c * kCs + q]) = cur.a[s];
                *reinterpret_cast<float4*>(&dbs[c * kCs + q]) = cur.b[s];
            }
            if (t < kQ) mq[t] = (t < np && (!mask || (cur.mr != 0 && cur.mk != 0))) ? 1.f : 0.f;
            const uint32_t zw[4] = {cur.z0.x, cur.z0.y, cur.z0.z, cur.z0.w};
            float s1 = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xh[2 * i] = __uint_as_float(zw[i] << 16);
                xh[2 * i + 1] = __uint_as_float(zw[i] & 0xffff0000u);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) s1 += xh[i];
            const float mz = sum_lanes16(s1) * (1.f / kCz);
            float q2 = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) { xh[i] -= mz; q2 += xh[i] * xh[i]; }
            rz = rsqrtf(sum_lanes16(q2) * (1.f / kCz) + eps);
            float gam[8], bet[8];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float4 g = *reinterpret_cast<const float4*>(&prm[0][8 * lq + 4 * s]);
                const float4 b = *reinterpret_cast<const float4*>(&prm[1][8 * lq + 4 * s]);
                gam[4 * s] = g.x; gam[4 * s + 1] = g.y; gam[4 * s + 2] = g.z; gam[4 * s + 3] = g.w;
                bet[4 * s] = b.x; bet[4 * s + 1] = b.y; bet[4 * s + 2] = b.z; bet[4 * s + 3] = b.w;
            }
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xh[2 * i] *= rz;
                xh[2 * i + 1] *= rz;
                const float x0 = xh[2 * i] * gam[2 * i] + bet[2 * i];
                const float x1 = xh[2 * i + 1] * gam[2 * i + 1] + bet[2 * i + 1];
                hw[i] = pack_bf16x2(x0, x1);
                lw[i] = pack_bf16x2(x0 - __uint_as_float(hw[i] << 16), x1 - __uint_as_float(hw[i] & 0xffff0000u));
            }
            *reinterpret_cast<uint4*>(xa[0] + lp * kXrow + 16 * lq) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            *reinterpret_cast<uint4*>(xa[1] + lp * kXrow + 16 * lq) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
        load(u + gridDim.x, cur);                        // next unit's dA, dB, z, mask
        __syncthreads();
        {   // xhs and rzs are read by the previous unit's last phase: written only past the barrier
            const int t = opaque(threadIdx.x), lp = t >> 4, lq = t & 15;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                *reinterpret_cast<float4*>(&xhs[lp * kPq4 + 8 * lq + 4 * s]) =
                    make_float4(xh[4 * s], xh[4 * s + 1], xh[4 * s + 2], xh[4 * s + 3]);
            if (lq == 0) rzs[lp] = rz;
        }
        {   // projections of channel c = 16 w + col; the four gradients
            const int lo = opaque(lane), col = lo & 15, kq = lo >> 4;
            const int c = 16 * w + col;
#pragma unroll
            for (int h = 0; h < 2; ++h) {                // h = 0: (p_a, g_a), h = 1: (p_b, g_b)
                f32x4_t ap[2], ag[2];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) ap[mb] = ag[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) {
                        const uint32_t o = (16 * mb + col) * kXrow + 64 * ks + 16 * kq;
                        const bf16x8_t xhi = ld_frag(xa[0], o), xlo = ld_frag(xa[1], o);
                        ap[mb] = mfma16(xhi, wp[2 * h][ks], ap[mb]);
                        ag[mb] = mfma16(xhi, wp[2 * h + 1][ks], ag[mb]);
                        ap[mb] = mfma16(xlo, wp[2 * h][ks], ap[mb]);
                        ag[mb] = mfma16(xlo, wp[2 * h + 1][ks], ag[mb]);
                    }
                const float* dsrc = h ? dbs : das;
                bf16_t* bp = h ? b_dpb : b_dpa;
                bf16_t* bg = h ? b_dgb : b_dga;
                const int kp = 256 * h + c, kg = 256 * h + 128 + c;
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    const int q0 = 16 * mb + 4 * kq;
                    const float4 dd4 = *reinterpret_cast<const float4*>(&dsrc[c * kCs + q0]);
                    const float dd[4] = {dd4.x, dd4.y, dd4.z, dd4.w};
                    float vp[4], vg[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int q = q0 + i;
                        const bool m = mq[q] != 0.f;
                        const float s = sigmoidf_(ag[mb][i]);
                        vp[i] = m ? dd[i] * s : 0.f;
                        vg[i] = m ? dd[i] * ap[mb][i] * s * (1.f - s) : 0.f;
                        *reinterpret_cast<bf16_t*>(d4 + q * kGrow + 2 * kp) = f2bf(vp[i]);
                        *reinterpret_cast<bf16_t*>(d4 + q * kGrow + 2 * kg) = f2bf(vg[i]);
                    }
                    const int64_t bo = u * (kCh * kQ) + c * kQ + q0;
                    *reinterpret_cast<uint2*>(bp + bo) = pack4(vp[0], vp[1], vp[2], vp[3]);
                    *reinterpret_cast<uint2*>(bg + bo) = pack4(vg[0], vg[1], vg[2], vg[3]);
                }
            }
        }
        __syncthreads();
        {   // dx (projection part) of column d = 16 w + col over K = 512; unit block of x
            const int lo = opaque(lane), col = lo & 15, kq = lo >> 4;
            f32x4_t ax[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) ax[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 16; ++ks)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
                    ax[mb] = mfma16(ld_frag(d4, (16 * mb + col) * kGrow + 64 * ks + 16 * kq), wt[ks], ax[mb]);
            const int to = opaque(threadIdx.x), sc = to >> 2, sq = to & 3;
            *reinterpret_cast<uint4*>(b_x + u * (kCh * kQ) + sc * kQ + 8 * sq) = gather_col8p(xa[0], 8 * sq, sc);
            const int d = 16 * w + col;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) dxs[(16 * mb + 4 * kq + i) * kPq4 + d] = ax[mb][i];
        }
        __syncthreads();
        {   // LN_in backward of pair lp: dz = rz (dx gamma - mean(dx gamma) - xh mean(dx gamma xh))
            const int t = opaque(threadIdx.x), lp = t >> 4, lq = t & 15;
            float dx[8], xh[8], gam[8], s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float4 p = *reinterpret_cast<const float4*>(&dxs[lp * kPq4 + 8 * lq + 4 * s]);
                const float4 hh = *reinterpret_cast<const float4*>(&xhs[lp * kPq4 + 8 * lq + 4 * s]);
                const float4 g = *reinterpret_cast<const float4*>(&prm[0][8 * lq + 4 * s]);
                dx[4 * s] = p.x + xg[s].x;
                dx[4 * s + 1] = p.y + xg[s].y;
                dx[4 * s + 2] = p.z + xg[s].z;
                dx[4 * s + 3] = p.w + xg[s].w;
                xh[4 * s] = hh.x; xh[4 * s + 1] = hh.y; xh[4 * s + 2] = hh.z; xh[4 * s + 3] = hh.w;
                gam[4 * s] = g.x; gam[4 * s + 1] = g.y; gam[4 * s + 2] = g.z; gam[4 * s + 3] = g.w;
            }
            const float rz = rzs[lp];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float dh = dx[i] * gam[i];
                s1 += dh;
                s2 += dh * xh[i];
                accg[i] += dx[i] * xh[i];
                accb[i] += dx[i];
            }
            s1 = sum_lanes16(s1) * (1.f / kCz);
            s2 = sum_lanes16(s2) * (1.f / kCz);
            uint32_t o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o[i] = pack_bf16x2(rz * (dx[2 * i] * gam[2 * i] - s1 - xh[2 * i] * s2),
                                   rz * (dx[2 * i + 1] * gam[2 * i + 1] - s1 - xh[2 * i + 1] * s2));
            const auto rd = make_rsrc(dz + pair_of(r, k0) * kCz, (np - 1) * step2 + kCz * 2);   // pairs past N: dropped
            bst_u4(rd, lp * step2 + 16 * lq, make_uint4(o[0], o[1], o[2], o[3]));
        }
        load_dxg(u + gridDim.x, xg);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        das[lp * kCz + 8 * lq + i] = accg[i];
        dbs[lp * kCz + 8 * lq + i] = accb[i];
    }
    __syncthreads();
    if (t < 2 * kCz) {
        const float* src = t < kCz ? das : dbs;
        const int d = t & (kCz - 1);
        float s = 0.f;
        for (int q = 0; q < kQ; ++q) s += src[q * kCz + d];
        partial[((int64_t)blockIdx.x * 2 + (t >> 7)) * kCz + d] = s;
    }
}

// Four weight gradients that share their second operand (W_a, W_ga, W_b,
// W_gb all multiply the x blocks): W_o[m][n] = sum over units of U_blk[m][.] .
// V_blk[n][.] (both [128][32] bf16 unit blocks, the dot product over the 32
// slots) for o = 0..3, reading each unit's V block once.  8 waves: wave w
// owns rows 32 (w % 4) .. + 31 of outputs 2 (w / 4) and 2 (w / 4) + 1
// (two 32 x 128 accumulators).  Partials: [o][grid][128][128].
//
// Bound by memory: 40 KB per unit.  A unit's five blocks come through a ring
// of three 40 KB stages in LDS, filled by direct loads two units ahead (80 KB
// in flight per compute unit), so that each byte is loaded once; with every
// wave loading its own operands into registers a unit ahead the x block came
// eight times, 96 KB of loads per unit (N = 1024 311 us under the profiler,
// now about 255; N = 384 57 and 47).  Rows of 64 bytes, chunk c at slot
// c ^ (row / 4) % 4: the 16 rows a read serves per cycle hit distinct banks.
struct Wgrad4Args {
    const bf16_t* u[4];
};

__global__ __launch_bounds__(512) void k_wgrad4(Wgrad4Args a, const bf16_t* __restrict__ V, int64_t units,
                                                float* __restrict__ partial) {
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int rl = lane & 31, hi = lane >> 5;
    const int rb = 32 * (w & 3), o0 = 2 * (w >> 2);
    f32x16_t acc[2][4];
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[o][j][r] = 0.f;
    // Fill of a stage: 40 loads of 1 KB (16 rows of a block), five per wave.
    constexpr int kBlk = kCh * kQ * 2, kStage = 5 * kBlk;
    __shared__ __align__(1024) char ring[3 * kStage];
    const uint32_t ring_base = lds_addr(ring);
    const bf16_t* src[5];
    uint32_t dst[5], voff[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int l = __builtin_amdgcn_readfirstlane(5 * w + i), m = l >> 3, p = l & 7;
        src[i] = m == 0 ? a.u[0] : m == 1 ? a.u[1] : m == 2 ? a.u[2] : m == 3 ? a.u[3] : V;
        dst[i] = (uint32_t)(m * kBlk + p * 1024);
        voff[i] = (uint32_t)(p * 1024 + (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
    }
    auto issue = [&](int64_t u, int stage) {   // a unit past the end loads nothing (empty descriptor)
        const bool valid = u < units;
        const int64_t base = valid ? u * (kCh * kQ) : 0;
#pragma unroll
        for (int i = 0; i < 5; ++i)
            lds_load16(buffer_desc(src[i] + base, valid ? kBlk : 0), voff[i], 0, ring_base + (uint32_t)(stage * kStage) + dst[i]);
    };
    issue(blockIdx.x, 0);
    issue((int64_t)blockIdx.x + gridDim.x, 1);
    const int x = (rl >> 2) & 3;
    const uint32_t rd[2] = {(uint32_t)(rl * 64 + ((hi ^ x) << 4)), (uint32_t)(rl * 64 + (((2 + hi) ^ x) << 4))};
    int stage = 0;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        wait_vmcnt_pinned<5>();   // this unit's loads; the next one's stay in flight
        __syncthreads();
        issue(u + 2 * (int64_t)gridDim.x, stage == 0 ? 2 : stage - 1);   // into the stage read one unit ago
        const char* st = ring + stage * kStage;
        stage = stage == 2 ? 0 : stage + 1;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8_t fa[2], fb[4];
#pragma unroll
            for (int o = 0; o < 2; ++o) fa[o] = *reinterpret_cast<const bf16x8_t*>(st + (o0 + o) * kBlk + rb * 64 + rd[ks]);
#pragma unroll
            for (int j = 0; j < 4; ++j) fb[j] = *reinterpret_cast<const bf16x8_t*>(st + 4 * kBlk + j * 2048 + rd[ks]);
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[o][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[o], fb[j], acc[o][j], 0, 0, 0);
        }
    }
    wait_vmcnt_pinned<0>();   // nothing may still write LDS when the work-group ends
    // lane holds column 32 j + rl; register r holds row rb + 8 (r / 4) + 4 hi + r % 4
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        float* pw = partial + ((int64_t)(o0 + o) * gridDim.x + blockIdx.x) * (kCh * kCh);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) pw[(rb + 8 * (r >> 2) + 4 * hi + (r & 3)) * kCh + 32 * j + rl] = acc[o][j][r];
    }
}

// Sums of the per-work-group partials: out[i] = sum over g < parts of
// in[g * stride + i], for several outputs in one launch.  A work-group takes
// 32 consecutive outputs of one sum (one 128-byte line of every partial): 32
// slices of 8 lanes each add every 32nd partial, then the slices are added in
// order, so the result is the same every time for one number of compute units
// (each partial is the sum of one work-group's units).  Bound by the latency of
// reading the partials (16 MB for one 128 x 128 gradient): one thread per
// output, which walked all of them alone, kept 64 work-groups on a serial chain
// of 256 to 512 loads, 96 us a sum and 870 us of a backward call; now a call's
// one launch for all ten sums takes 20 us (N = 384, 256 compute units).
__global__ __launch_bounds__(256) void k_sum_parts(SumTasks a) {
    __shared__ __align__(16) float4 red[32][8];
    int i = 0;
    while (i + 1 < a.count && (int)blockIdx.x >= a.task[i + 1].block0) ++i;
    const SumTask q = a.task[i];
    const int t = threadIdx.x, lane = t & 7, slice = t >> 3;
    const float* p = q.in + 32 * ((int)blockIdx.x - q.block0) + 4 * lane;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int g = slice; g < q.parts; g += 32) {
        const float4 v = *reinterpret_cast<const float4*>(p + (int64_t)g * q.stride);
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    }
    red[slice][lane] = s;
    __syncthreads();
    if (t < 32) {
        const float* r = reinterpret_cast<const float*>(red) + t;
        float o = 0.f;
#pragma unroll
        for (int g = 0; g < 32; ++g) o += r[32 * g];
        q.out[32 * ((int)blockIdx.x - q.block0) + t] = o;
    }
}

}  // namespace

hipError_t launch_result_to_panel(int dtype, const float* R, void* P, int64_t N, int cus, hipStream_t s) {
    const int64_t units = (N + 1) / 2 * ((N + kResJ - 1) / kResJ);   // row pairs x column blocks
    const unsigned g = (unsigned)(units < 8 * (int64_t)cus ? units : 8 * (int64_t)cus);
    if (dtype == 0)
        hipLaunchKernelGGL(k_result_to_panel<float>, dim3(g), dim3(256), 0, s, R, (float*)P, (int)N, units);
    else
        hipLaunchKernelGGL(k_result_to_panel<bf16_t>, dim3(g), dim3(256), 0, s, R, (bf16_t*)P, (int)N, units);
    return hipGetLastError();
}

hipError_t launch_panel_transpose(int dtype, const void* X, void* Y, int64_t N, int cus, hipStream_t s) {
    const int64_t S = (N + 31) / 32;
    const int64_t blocks = (int64_t)kCh * S * S;
    const int64_t wgs = (blocks + 3) / 4;
    const unsigned g = (unsigned)(wgs < 8 * (int64_t)cus ? wgs : 8 * (int64_t)cus);
    if (dtype == 0)
        hipLaunchKernelGGL(k_panel_transpose<float>, dim3(g), dim3(256), 0, s, (const float*)X, (float*)Y, (int)N,
                           blocks);
    else
        hipLaunchKernelGGL(k_panel_transpose<bf16_t>, dim3(g), dim3(256), 0, s, (const bf16_t*)X, (bf16_t*)Y,
                           (int)N, blocks);
    return hipGetLastError();
}

}  // namespace trimul

namespace trimul {

int backward_grid(int64_t units, int cus, int per_cu) {
    return (int)(units < (int64_t)per_cu * cus ? units : (int64_t)per_cu * cus);
}

hipError_t launch_epilogue_backward(int out_dtype, const DeviceWeights& w, const float* C, const void* z,
                                    const uint8_t* mask, const void* dout, int64_t N, void* dCp, float* dxg,
                                    float* wpart, float* partial, int grid, hipStream_t s) {
    const int64_t units = N * ((N + 31) / 32);
    if (out_dtype == 0)
        hipLaunchKernelGGL(k_epilogue_backward<float>, dim3(grid), dim3(kBT), 0, s, C, (const bf16_t*)z, mask,
                           (const float*)dout, (int)N, units, w.epi_bf, w.epit_bf, w.ln_in_w, w.ln_in_b, w.ln_out_w,
                           w.ln_out_b, w.eps, (bf16_t*)dCp, dxg, wpart, partial);
    else
        hipLaunchKernelGGL(k_epilogue_backward<bf16_t>, dim3(grid), dim3(kBT), 0, s, C, (const bf16_t*)z, mask,
                           (const bf16_t*)dout, (int)N, units, w.epi_bf, w.epit_bf, w.ln_in_w, w.ln_in_b,
                           w.ln_out_w, w.ln_out_b, w.eps, (bf16_t*)dCp, dxg, wpart, partial);
    return hipGetLastError();
}

hipError_t launch_projection_backward(const DeviceWeights& w, const void* z, const uint8_t* mask, int64_t N,
                                      int incoming, const float* dA, const float* dB, const float* dxg, void* dz,
                                      const BackwardBlocks& bb, float* partial, int grid, hipStream_t s) {
    const int64_t units = N * ((N + 31) / 32);
    if (incoming)
        hipLaunchKernelGGL(k_projection_backward<true>, dim3(grid), dim3(kBT), 0, s, (const bf16_t*)z, mask, (int)N,
                           units, dA, dB, dxg, w.proj_bf, w.projt_bf, w.ln_in_w, w.ln_in_b, w.eps, (bf16_t*)dz,
                           bb.dpa, bb.dga, bb.dpb, bb.dgb, bb.xp, partial);
    else
        hipLaunchKernelGGL(k_projection_backward<false>, dim3(grid), dim3(kBT), 0, s, (const bf16_t*)z, mask, (int)N,
                           units, dA, dB, dxg, w.proj_bf, w.projt_bf, w.ln_in_w, w.ln_in_b, w.eps, (bf16_t*)dz,
                           bb.dpa, bb.dga, bb.dpb, bb.dgb, bb.xp, partial);
    return hipGetLastError();
}

hipError_t launch_wgrad4(const bf16_t* const U[4], const bf16_t* V, int64_t N, float* partial, int grid,
                         hipStream_t s) {
    const int64_t units = N * ((N + 31) / 32);
    Wgrad4Args a{{U[0], U[1], U[2], U[3]}};
    hipLaunchKernelGGL(k_wgrad4, dim3(grid), dim3(512), 0, s, a, V, units, partial);
    return hipGetLastError();
}

hipError_t launch_sum_parts(const SumTask* tasks, int count, hipStream_t s) {
    SumTasks a;
    a.count = count;
    int blocks = 0;
    for (int i = 0; i < count; ++i) {
        a.task[i] = tasks[i];
        a.task[i].block0 = blocks;
        blocks += tasks[i].n / 32;
    }
    hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace trimul
