// K1: input LayerNorm + gated a/b projections + pair mask, writing the
// channel-major operands of the contraction (Section 3.3: a, b are gated
// projections of z; Eq. 2 / Eq. 3 pick which token index is contracted).
//
// Work unit: a "line" of 32 pairs that share one output row.  Outgoing line
// (r, k0): pairs (r, k0..k0+31), A[c][r][k0+p] = a(r, k0+p).  Incoming line
// (r, k0): pairs (k0..k0+31, r), A[c][r][k0+p] = a(k0+p, r).  Either way the 32
// results of one channel are contiguous in A and B.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace trimul {
namespace {

// ------------------------------------------------------------ fp32 MFMA
//
// The fp32 storage path, on v_mfma_f32_32x32x2_f32 (fp32 operands and sums,
// 157 TFLOP/s at 2.4 GHz).  A work-group of 4 waves takes a line of 32 pairs
// and four of the eight gated groups, one per wave: a gated group is 32
// hidden channels of a or of b, i.e. two 32-row weight blocks (value and
// gate) whose products land in the same lane and register, so the gating
// stays in registers.  x goes through LDS (rows padded to 132 floats: the 16
// rows a 16-byte read serves per cycle start 4 banks apart); the weights
// stream from L2 as 1 KB loads in operand order (DeviceWeights::proj_f), one
// k group ahead.  In group q lane l holds k = 8 q + 4 (l / 32) + e of its row
// in element e, so one 16-byte read feeds four products.  A pair's 128-byte
// channel runs go straight from the accumulators to the panels.
//
// Bound by the matrix cores (4 x 128 x 128 multiply-adds a pair); the scalar
// kernel it replaces took 595 us at N = 384 and 72 us at N = 64, this one 175
// and 8 (113 TFLOP/s).  Lines of 64 pairs and all eight groups per
// work-group (an eighth of the weight reads) gained 2% at N = 512 and took
// 20 us at N = 64.
constexpr int kXf = kCz + 4;   // row stride (floats) of x in LDS
constexpr int kPf = 32;        // pairs per line

template <bool INCOMING>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(4)))
void k1_project_f32(const float* __restrict__ z, const uint8_t* __restrict__ mask, int N, const float4* __restrict__ wf,
                    const float* __restrict__ lnw, const float* __restrict__ lnb, float eps, float* __restrict__ A,
                    float* __restrict__ B) {
    __shared__ __attribute__((aligned(16))) float xs[kPf * kXf];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // rows fastest: neighbouring work-groups write neighbouring rows of the
    // same panel blocks (and read neighbouring pairs when incoming)
    const int kc = (int)(blockIdx.x / (unsigned)N), r = (int)(blockIdx.x - (unsigned)kc * (unsigned)N);
    const int k0 = kc * kPf, np = min(kPf, N - k0);
    const int gg = (int)blockIdx.y * 4 + wave;           // gated group: a's four, then b's

    {   // LayerNorm of pair p, 8 lanes each
        const int p = t >> 3, q = t & 7;
        const int64_t pair = INCOMING ? (int64_t)(k0 + p) * N + r : (int64_t)r * N + k0 + p;
        float4 v[4];
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = p < np ? *reinterpret_cast<const float4*>(z + pair * kCz + 4 * (q + 8 * i))
                          : make_float4(0.f, 0.f, 0.f, 0.f);
            s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
        }
        s = sum_lanes8(s);
        const float mu = s * (1.0f / kCz);
        float q2 = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i].x -= mu; v[i].y -= mu; v[i].z -= mu; v[i].w -= mu;
            q2 += (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
        }
        q2 = sum_lanes8(q2);
        const float rs = rsqrtf(q2 * (1.0f / kCz) + eps);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = 4 * (q + 8 * i);
            const float4 g = *reinterpret_cast<const float4*>(lnw + c), b = *reinterpret_cast<const float4*>(lnb + c);
            *reinterpret_cast<float4*>(&xs[p * kXf + c]) = make_float4(v[i].x * rs * g.x + b.x, v[i].y * rs * g.y + b.y,
                                                                       v[i].z * rs * g.z + b.z, v[i].w * rs * g.w + b.w);
        }
    }
    const int rl = lane & 31, hi = lane >> 5;
    const PanelGeom pg = panel_geom(N, N);
    const int64_t chs = panel_elems(pg);
    const uint32_t keep = rl < np && (!mask || (mask[r] != 0 && mask[k0 + rl] != 0)) ? 0xffffffffu : 0u;
    __syncthreads();

    // [value, gate][k group q][lane]
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(wf + (int64_t)gg * 2 * 16 * 64, 2 * 16 * 1024);
    f32x16_t acc[2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[m][i] = 0.f;
    struct Ops { float4 w[2], x; };
    auto load = [&](int q, Ops& o) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
            o.w[m] = __builtin_bit_cast(float4, buf_load16(rw, (uint32_t)((m * 16 + q) * 1024 + 16 * lane)));
        o.x = *reinterpret_cast<const float4*>(&xs[rl * kXf + 8 * q + 4 * hi]);
        __builtin_amdgcn_sched_barrier(0);   // issued here, a group ahead of their products
    };
    auto products = [&](const Ops& o) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(f4_get(o.w[m], e), f4_get(o.x, e), acc[m], 0, 0, 0);
    };
    Ops o0, o1;
    load(0, o0);
#pragma unroll 1
    for (int q = 0; q < 16; q += 2) {
        load(q + 1, o1);
        products(o0);
        load(q < 14 ? q + 2 : 0, o0);   // the last one goes unused
        products(o1);
    }
    // Lane holds pair lane % 32; register i holds channel 8 (i / 4) +
    // 4 (lane / 32) + i % 4 of the group.
    float* X = ((gg >> 2) ? B : A) + (32 * (gg & 3) + 4 * hi) * chs + panel_off(pg, 0, r, k0) + rl;
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)   // a masked pair's are 0, whatever z holds
        v[i] = __uint_as_float(__float_as_uint(sigmoidf_(acc[1][i]) * acc[0][i]) & keep);
    if (rl < np) {
#pragma unroll
        for (int i = 0; i < 16; ++i) X[(8 * (i >> 2) + (i & 3)) * chs] = v[i];
    }
}


// ------------------------------------------------------------ bf16 MFMA
//
// Persistent kernel, 4 waves, work unit = line of 32 pairs.  Wave g owns
// hidden channels [32 g, 32 g + 32): its 128 weight rows (W_a, W_ga, W_b,
// W_gb of those channels) stay in VGPRs for the whole kernel as the MFMA A
// operand, so the 4 x 32 outputs of a channel land in the same lane and
// register and the gating is element-wise in registers.
//
// z and the token mask reach LDS through a 3-stage ring filled by
// direct-to-LDS buffer loads two lines ahead of the line being computed, so
// the HBM latency of z hides behind two lines of work.  Every wave issues
// the same number of vector-memory instructions per line (3 loads, 2 without a
// mask, and 4 stores, tails included), which makes the vmcnt waits exact
// constants.
//
// Precision: the matrix cores take fp16 operands, 11 significant bits
// against bf16's 8.  The weights (bf16 values) and the LayerNormed x
// (fp32) are scaled by powers of two chosen at initialisation so that the
// largest possible operand lies in [2^14, 2^15]: the weights convert
// exactly (down to 2^-17 of that largest entry) and x rounds once to
// 2^-11 relative, with no overflow and no subnormal x.  So values and gates
// carry ~11 bits, and the main error of a and b stays their bf16 store.
// The gating undoes the scales (DeviceWeights::K1Scales) inside the
// logistic at no extra instruction.
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
constexpr int kP1 = 32;                 // pairs per line
constexpr int kXRow = kCz * 2;          // bytes of one bf16 row of 128 channels (256)
constexpr int kZSt = kP1 * kXRow;       // z bytes of one line (8 KB)
constexpr int kMSt = 4 * 256;           // per-wave token-mask bytes of one line
constexpr int kSt = kZSt + kMSt;        // one ring stage
constexpr int kRing = 3;

// x rows [p][128] bf16: 16-byte chunk q of row p lives at slot q ^ (p & 15).
__device__ __forceinline__ uint32_t xoff(int p, int chunk) {
    return (uint32_t)(p * kXRow + ((chunk ^ (p & 15)) << 4));
}

// The operands are M x K: operand row i (M of them) and contraction index k
// (K).  Outgoing, pair (i, k) is z[i][k]; incoming, pair (k, i) is z[k][i];
// z rows are ldz pairs apart (the full update: M = K = ldz = N; a device
// tile: its rows and columns).  MASK: mask holds token bytes, the k-range's at
// koff, the operand rows' at roff; mrange bytes are readable.  Without one every
// token is real and no mask load is issued (loads through an empty descriptor in
// its place cost 0.2 to 0.5% at N = 4096).
template <bool INCOMING, bool MASK>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
void k1_project_mfma(const bf16_t* __restrict__ z, int ldz, const uint8_t* __restrict__ mask, uint32_t koff,
                     uint32_t roff, uint32_t mrange, int M, int K, int nlines, const uint16_t* __restrict__ wproj,
                     const float* __restrict__ lnw, const float* __restrict__ lnb, float eps,
                     DeviceWeights::K1Scales ks, bf16_t* __restrict__ A, bf16_t* __restrict__ B) {
    __shared__ __attribute__((aligned(16))) char ring[kRing * kSt];     // z rows [p][256 B], mask
    __shared__ __attribute__((aligned(16))) char xs[kP1 * kXRow];      // x (fp16, scaled)
    __shared__ __attribute__((aligned(16))) float os[2][kCh][kP1];      // a, b as [c][p]
    // LayerNorm gain, bias; channel c at (c / 16) * 20 + c % 16, so that the
    // 8 broadcast addresses of a read (c = 16 lq + 4 i) fall in distinct banks
    __shared__ __attribute__((aligned(16))) float gb[2][8 * 20];
    const int t = threadIdx.x, lane = t & 63;
    const int g = __builtin_amdgcn_readfirstlane(t >> 6);
    const int lp = t >> 3, lq = t & 7;     // LayerNorm: pair lp, channels 16 lq .. 16 lq + 15
    // Line order: rows fastest (line = kc * M + r covers pairs k0 = 32 kc ..
    // k0 + 31 of operand row r), and the work-groups of one XCD take consecutive
    // lines; the grid's lines of one round then fill whole 256-row blocks of
    // the operands and read long runs of z in either direction.
    const int G = gridDim.x;
    const int first = (G & 7) == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;

    // Ring fill.  Stage row p holds pair k0 + p of the line; its 16-byte
    // chunk q sits at slot q ^ (p & 1), so that the LayerNorm reads of two
    // neighbouring rows hit disjoint banks.  Wave g loads rows 8 g .. 8 g + 7
    // (two 1 KB loads: lane i -> row 8 g + 4 h + i / 16, slot i % 16) and its
    // own copy of the line's mask bytes, one per dword: pairs k0 .. k0 + 31,
    // then row r (straight from the caller's mask: staging it took a launch of
    // its own, 5 us).  Lines past the end load nothing (zero-size descriptor).
    const uint32_t zstep = INCOMING ? (uint32_t)ldz * kXRow : (uint32_t)kXRow;   // bytes between pairs
    const uint32_t ring_base = lds_addr(ring);
    const int drow = g * 8 + (lane >> 4);
    const uint32_t dchunk = (uint32_t)(((lane & 15) ^ (drow & 1)) << 4);
    const uint32_t dv0 = (uint32_t)drow * zstep + dchunk, dv1 = (uint32_t)(drow + 4) * zstep + dchunk;
    auto issue = [&](int line, int stage) {
        const bool valid = line < nlines;
        int r = 0, k0 = 0;
        if (valid) {
            const int kc = line / M;
            r = line - kc * M;
            k0 = kc * kP1;
        }
        const int np = valid ? min(kP1, K - k0) : 0;
        const int64_t pair0 = INCOMING ? (int64_t)k0 * ldz + r : (int64_t)r * ldz + k0;
        const v4i_t rz = buffer_desc(z + pair0 * kCz, np > 0 ? (uint32_t)(np - 1) * zstep + kXRow : 0u);
        const uint32_t st = ring_base + (uint32_t)(stage * kSt);
        lds_load16(rz, dv0, 0, st + g * 2048);
        lds_load16(rz, dv1, 0, st + g * 2048 + 1024);
        if constexpr (MASK) {
            const v4i_t rm = buffer_desc(mask, valid ? mrange : 0u);
            const uint32_t mo = lane < 32 ? koff + (uint32_t)(k0 + lane) : lane == 32 ? roff + (uint32_t)r : 0xfffffff0u;
            lds_load_u8(rm, mo, st + kZSt + g * 256);
        }
    };
    constexpr int kLd = MASK ? 3 : 2;   // loads per line and wave
    issue(first, 0);
    issue(first + G, 1);

    f16x8_t w[4][8];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int kq = 0; kq < 8; ++kq)
            w[ob][kq] = *reinterpret_cast<const f16x8_t*>(
                wproj + (size_t)(g * 128 + ob * 32 + (lane & 31)) * kCz + kq * 16 + 8 * (lane >> 5));
    if (t < kCz) {
        gb[0][(t >> 4) * 20 + (t & 15)] = lnw[t];
        gb[1][(t >> 4) * 20 + (t & 15)] = lnb[t];
    }
    const PanelGeom pg = panel_geom(M, K);
    // Store mapping: thread t writes pairs 8 (t & 3) .. 8 (t & 3) + 7 of
    // channel (t >> 2) + 64 (i & 1) of A (i < 2) or B (i >= 2).
    const int64_t ch_stride = panel_elems(pg);
    const int64_t st_lane = (t >> 2) * ch_stride + 8 * (t & 3);

    int stage = 0;
    for (int it = 0, line = first; line < nlines; ++it, line += G) {
        // Vector-memory instructions issued after this line's loads: the
        // next line's loads and, from the second line on, the 4 stores of
        // every line in between.
        if (it == 0) wait_vmcnt_pinned<kLd>();
        else if (it == 1) wait_vmcnt_pinned<kLd + 4>();
        else wait_vmcnt_pinned<kLd + 4 + 4>();
        __syncthreads();
        issue(line + 2 * G, stage == 0 ? 2 : stage - 1);   // into the stage read one line ago
        const char* zs = ring + stage * kSt;
        stage = stage == 2 ? 0 : stage + 1;

        // LayerNorm of pair lp over 128 channels (8 lanes x 16 channels).
        float v[16];
        {
            const uint4 z0 = *reinterpret_cast<const uint4*>(zs + lp * kXRow + (((2 * lq) ^ (lp & 1)) << 4));
            const uint4 z1 = *reinterpret_cast<const uint4*>(zs + lp * kXRow + (((2 * lq + 1) ^ (lp & 1)) << 4));
            const uint32_t u[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[2 * i] = __uint_as_float(u[i] << 16);
                v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
            }
        }
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) s += v[i];
        s = sum_lanes8(s);
        const float mu = s * (1.0f / kCz);
        float q2 = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            v[i] -= mu;
            q2 += v[i] * v[i];
        }
        q2 = sum_lanes8(q2);
        const float rs = rsqrtf(q2 * (1.0f / kCz) + eps);
        float gam[16], bet[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 a4 = *reinterpret_cast<const float4*>(&gb[0][20 * lq + 4 * i]);
            const float4 b4 = *reinterpret_cast<const float4*>(&gb[1][20 * lq + 4 * i]);
            gam[4 * i] = a4.x; gam[4 * i + 1] = a4.y; gam[4 * i + 2] = a4.z; gam[4 * i + 3] = a4.w;
            bet[4 * i] = b4.x; bet[4 * i + 1] = b4.y; bet[4 * i + 2] = b4.z; bet[4 * i + 3] = b4.w;
        }
        f16x8_t xh[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) xh[i >> 3][i & 7] = (_Float16)(v[i] * rs * gam[i] + bet[i]);
        // A masked pair (and a ragged line's tail past K) gets x = 0, so W x
        // and with it a and b are exactly 0; the AND also clears what a NaN in
        // z would have left.
        const int kc = line / M, r0 = line - kc * M, k0 = kc * kP1;
        const uint32_t* ms = reinterpret_cast<const uint32_t*>(zs + kZSt + g * 256);   // this wave's copy
        const uint32_t keep = k0 + lp < K && (!MASK || (ms[lp] != 0 && ms[32] != 0)) ? 0xffffffffu : 0u;
        uint4 x0 = __builtin_bit_cast(uint4, xh[0]), x1 = __builtin_bit_cast(uint4, xh[1]);
        x0 = make_uint4(x0.x & keep, x0.y & keep, x0.z & keep, x0.w & keep);
        x1 = make_uint4(x1.x & keep, x1.y & keep, x1.z & keep, x1.w & keep);
        *reinterpret_cast<uint4*>(xs + xoff(lp, 2 * lq)) = x0;
        *reinterpret_cast<uint4*>(xs + xoff(lp, 2 * lq + 1)) = x1;
        __syncthreads();

        // [W_a; W_ga; W_b; W_gb](32 channels each) x x (32 pairs), all scaled
        f32x16_t acc[4];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ob][r] = 0.f;
        const int bp = lane & 31;
#pragma unroll
        for (int kq = 0; kq < 8; ++kq) {
            const f16x8_t xk = *reinterpret_cast<const f16x8_t*>(xs + xoff(bp, 2 * kq + (lane >> 5)));
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
                acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[ob][kq], xk, acc[ob], 0, 0, 0);
        }

        // Gate and stage as [c][p] fp32.  Lane holds pair (lane & 31); in
        // register r, channel 32 g + 8 (r / 4) + 4 (lane / 32) + r % 4.
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int c = g * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            const float ga = __builtin_amdgcn_rcpf(ks.kv_a + __builtin_amdgcn_exp2f(fmaf(acc[1][r], ks.cg_a, ks.sv_a)));
            const float gb2 = __builtin_amdgcn_rcpf(ks.kv_b + __builtin_amdgcn_exp2f(fmaf(acc[3][r], ks.cg_b, ks.sv_b)));
            os[0][c][bp] = ga * acc[0][r];
            os[1][c][bp] = gb2 * acc[2][r];
        }
        __syncthreads();

        // Channel-major stores: 4 lanes write the 32 pairs (64 bytes) of one
        // panel row, one k-step of the blocked layout.  A ragged line's tail
        // writes zeros into the k padding of its step, so every wave issues
        // exactly 4 stores per line.
        const int64_t line_off = panel_off(pg, 0, r0, k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ab = i >> 1, c = (t >> 2) + 64 * (i & 1);
            const float4 f0 = *reinterpret_cast<const float4*>(&os[ab][c][8 * (t & 3)]);
            const float4 f1 = *reinterpret_cast<const float4*>(&os[ab][c][8 * (t & 3) + 4]);
            bf16_t* dst = (ab ? B : A) + (line_off + st_lane + 64 * (i & 1) * ch_stride);
            *reinterpret_cast<uint4*>(dst) = make_uint4(pack_bf16x2(f0.x, f0.y), pack_bf16x2(f0.z, f0.w),
                                                        pack_bf16x2(f1.x, f1.y), pack_bf16x2(f1.z, f1.w));
        }
    }
    wait_vmcnt_pinned<0>();   // the ring loads past the last line land before the work-group ends
}

}  // namespace

hipError_t launch_project_mfma(const DeviceWeights& w, const void* z, int64_t ldz, const uint8_t* mask, int64_t m0,
                               int64_t k0, int64_t M, int64_t K, int incoming, void* A, void* B, hipStream_t s) {
    const int nch = (int)((K + kP1 - 1) / kP1);
    const int nlines = (int)(M * nch);
    // Two work-groups per compute unit, but one up to four lines each: every
    // work-group reads the 128 KB of weights, which is what a small call waits
    // for (N = 100 12.0 -> 10.4 us, N = 130 15.4 -> 12.6, N = 160 15.6 -> 14.2;
    // N = 200 18.6 against 19.0, N = 512 59 against 68).
    const int cap = nlines <= 4 * w.cus ? w.cus : 2 * w.cus;
    const unsigned g = (unsigned)(nlines < cap ? nlines : cap);
    const int64_t lo = std::min(m0, k0);   // the mask bytes read start here
    const uint32_t koff = (uint32_t)(k0 - lo), roff = (uint32_t)(m0 - lo);
    const uint8_t* mk = mask ? mask + lo : nullptr;
    const uint32_t mrange = mask ? std::max(koff + (uint32_t)K, roff + (uint32_t)M) : 0u;
#define K1_BF16(IN_, MASK_)                                                                                        \
    hipLaunchKernelGGL((k1_project_mfma<IN_, MASK_>), dim3(g), dim3(256), 0, s, (const bf16_t*)z, (int)ldz, mk, koff, \
                       roff, mrange, (int)M, (int)K, nlines, w.proj_h, w.ln_in_w_h, w.ln_in_b_h, w.eps, w.k1s,      \
                       (bf16_t*)A, (bf16_t*)B)
    if (incoming && mask) K1_BF16(true, true);
    else if (incoming) K1_BF16(true, false);
    else if (mask) K1_BF16(false, true);
    else K1_BF16(false, false);
#undef K1_BF16
    return hipGetLastError();
}

hipError_t launch_project(int dtype, const DeviceWeights& w, const void* z, const uint8_t* mask,
                          int64_t N, int incoming, void* A, void* B, hipStream_t s) {
    if (dtype == 0) {
        const dim3 grid((unsigned)(N * ((N + kPf - 1) / kPf)), 2);
        const float4* wf = reinterpret_cast<const float4*>(w.proj_f);
        if (incoming)
            hipLaunchKernelGGL(k1_project_f32<true>, grid, dim3(256), 0, s, (const float*)z, mask, (int)N, wf,
                               w.ln_in_w, w.ln_in_b, w.eps, (float*)A, (float*)B);
        else
            hipLaunchKernelGGL(k1_project_f32<false>, grid, dim3(256), 0, s, (const float*)z, mask, (int)N, wf,
                               w.ln_in_w, w.ln_in_b, w.eps, (float*)A, (float*)B);
        return hipGetLastError();
    }
    return launch_project_mfma(w, z, N, mask, 0, 0, N, N, incoming, A, B, s);
}

}  // namespace trimul
