// gfx950 kernels of the streaming flow-decoder chunk step.
//
// One estimator evaluation is a chain of launches over the rows of the call
// (both guidance branches of every stream): an MFMA GEMM per Linear layer
// with its elementwise tail fused into the epilogue (bias, GELU, the gated
// residual add, the scatter of keys and values into the carry), a LayerNorm
// with the step's modulation, and an attention kernel that walks the carried
// keys and values in place.  Rows never interact outside the attention, and the
// order of every sum is fixed by the layer and by two switches on the call's
// size, at 512 rows (the few-row GEMM, which splits K, and the many-row one) and
// at 64 blocks of 64 queries (the two attention shapes).  Between calls on the
// same side of both, a stream's result does not depend on the batch or on which
// other streams share the call.
#include <type_traits>

#include "dc_philox.h"
#include "flow_internal.h"

namespace dcf {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// Two floats -> packed bfloat16 pair (round to nearest even).
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint16_t f2bf1(float v) { return (uint16_t)(pack2(v, 0.0f) & 0xffffu); }

// Store four consecutive values in the operand type.
template <bool BF16> __device__ __forceinline__ void store4(void* base, size_t idx, f32x4 v)
{
    if constexpr (BF16) {
        u32x2 w = {pack2(v[0], v[1]), pack2(v[2], v[3])};
        *(u32x2*)((uint16_t*)base + idx) = w;
    } else {
        *(f32x4*)((float*)base + idx) = v;
    }
}
template <bool BF16> __device__ __forceinline__ void store1(void* base, size_t idx, float v)
{
    if constexpr (BF16) ((uint16_t*)base)[idx] = f2bf1(v);
    else ((float*)base)[idx] = v;
}

// GELU in its tanh form, 0.5 v (1 + tanh(y)) with y = sqrt(2/pi) (v + 0.044715 v^3),
// as v / (1 + e^-2y): one exponential and one division instead of tanhf (whose
// branches took about half of the MLP-up GEMM at 14,336 rows), and no
// cancellation for negative v.
template <bool BF16> __device__ __forceinline__ float gelu_tanh(float v)
{
    const float k2 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;   // -2 sqrt(2 / pi) log2(e)
    const float d = 1.0f + __builtin_amdgcn_exp2f(v * (k2 + k2 * 0.044715f * (v * v)));
    if constexpr (BF16) return v * __builtin_amdgcn_rcpf(d);   // 1 ulp, rounded to bf16 next
    else return v / d;
}

// Sum over the 16 lanes of a DPP row, in every lane (rotations within the row:
// one fixed order, no LDS round trip).
template <int CTRL> __device__ __forceinline__ float row_ror(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float v)
{
    v += row_ror<0x128>(v);   // row_ror:8, 4, 2, 1
    v += row_ror<0x124>(v);
    v += row_ror<0x122>(v);
    v += row_ror<0x121>(v);
    return v;
}

// v plus the value of the lane 16 apart (within pairs of DPP rows).
__device__ __forceinline__ float sum_xor16(float v)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a0 = a[0], a1 = a[1];   // (scalars: a bit cast straight from element 1 reads element 0)
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
}

// Frame where the call's own frames start in stream b's carry regions.
__device__ __forceinline__ int own_base(const CarryRef& c, int prompt, int b)
{
    if (prompt) return 0;
    return c.Pr + c.slot[b] * c.Sl;
}

// ------------------------------------------------------------------- GEMM
//
// Both GEMM kernels take the weight as the MFMA's A operand (a lane's four
// results are four consecutive output columns of one row) and the activation
// row as the B operand, and hand every 4-column group of a row to the same
// epilogue.  With a LayerNorm operand (p.ln_h set) the activation is
// LN(h) * (1 + scale) + shift of the fp32 residual stream h, normalised while
// it is staged: mean and variance per row from sums shifted by the row's
// first value, eps 1e-6.

// The epilogue's operands of one 4-column group (bias; for E_RES also the
// gate and the residual row), loaded apart from their use so that a kernel
// can fetch them before its main loop.
struct EpiPre {
    f32x4 bias, gate, h;
};
template <int EPI>
__device__ __forceinline__ EpiPre epi_prefetch(const GemmParams& p, int row, int col)
{
    EpiPre e;
    e.bias = *(const f32x4*)(p.bias + col);
    if constexpr (EPI == E_RES) {
        e.gate = *(const f32x4*)(p.gate + col);
        e.h = *(const f32x4*)(p.h + (size_t)row * p.N + col);
    }
    return e;
}

template <bool BF16, int EPI>
__device__ __forceinline__ void epilogue4(const GemmParams& p, int row, int col, f32x4 acc, const EpiPre& e)
{
    const f32x4 y = acc + e.bias;
    if constexpr (EPI == E_H) {
        *(f32x4*)(p.h + (size_t)row * p.N + col) = y;
    } else if constexpr (EPI == E_RES) {
        f32x4 hv = e.h;
#pragma unroll
        for (int r = 0; r < 4; r++) hv[r] = hv[r] + e.gate[r] * y[r];
        *(f32x4*)(p.h + (size_t)row * p.N + col) = hv;
    } else if constexpr (EPI == E_GELU) {
        f32x4 z;
#pragma unroll
        for (int r = 0; r < 4; r++) z[r] = gelu_tanh<BF16>(y[r]);
        store4<BF16>(p.out, (size_t)row * p.N + col, z);
    } else if constexpr (EPI == E_VEL) {
        *(f32x4*)((float*)p.out + (size_t)row * p.N + col) = y;
    } else {   // E_QKV
        const int part = col / p.dim, hd = (col % p.dim) >> 6, d = col & 63;
        const int bp = row / (2 * p.n), c = (row / p.n) & 1, f = row % p.n;
        if (part == 0) {
            store4<BF16>(p.q, ((((size_t)bp * 2 + c) * p.heads + hd) * p.Fq + f) * 64 + d, y);
        } else {
            const int b = p.b0 + bp;
            const int frame = own_base(p.carry, p.prompt, b) + f;
            const size_t region = (size_t)b * p.carry.stream_stride +
                                  ((size_t)((c * 2 + (part - 1)) * p.heads + hd)) * p.carry.Fr * 64;
            if (part == 1) {
                store4<BF16>(p.carry.base, region + (size_t)frame * 64 + d, y);
            } else {
#pragma unroll
                for (int r = 0; r < 4; r++) store1<BF16>(p.carry.base, region + (size_t)(d + r) * p.carry.Fr + frame, y[r]);
            }
        }
    }
}

// GEMM of many rows (calls of more than kSkinnyRows).  A block computes 16 MB
// rows, each of its column waves all these rows of its own 16 NB columns (and,
// of a LayerNorm operand, of p.groups such column groups one after another).
// The activations sit in LDS, where every wave reads them; a weight fragment
// is used by one wave only, so it goes from L2 straight to registers, in
// fragment order, D steps ahead.
//   LayerNorm operand: the block's rows are normalised into LDS once, all K
//     (the launch of its own that this took wrote and read the operand again);
//   plain operand: K runs in chunks through two LDS buffers, the next chunk
//     loaded into registers while this one is multiplied.
// Every output element adds its K steps in ascending order, in one chain in
// every tile, and a row's LayerNorm sums have one order, so a row's result does
// not depend on the tile or, among calls of many rows, on the batch.
// What bounds it: at 14,336 rows the weight stream from L2 (64 rows per
// fragment, about 64 B/clk per CU at the full matrix rate) and the epilogue's
// vector work; at 1,792 rows load latency and the rows' LayerNorm, which every
// column block repeats.  Us per launch, bf16, against 32 MB x 32 NB tiles with
// both operands in LDS and a LayerNorm launch: 14,336 rows QKV 79.6 -> 44.3,
// MLP up 95.3 -> 51.7, MLP down 55.4 -> 45.8; 1,792 rows 22.8 -> 16.8,
// 22.7 -> 16.7, 20.7 -> 16.5.
//
// Waves of a block.  8 waves halve how often rows are normalised and weights
// read; 64 x 256-column tiles keep 4, since two such blocks per CU run in
// different phases (QKV and MLP up at 14,336 rows: 44.3 and 51.7 us with 4
// waves, 63.0 and 59.9 with 8).
template <int MB, int NB> constexpr int gemm_waves() { return MB == 4 && NB == 4 ? 4 : 8; }

// K values of an LDS row: the whole (padded) K of a LayerNorm operand, else a
// chunk of kStepPad steps.
template <bool BF16, bool LN> __host__ __device__ constexpr int panel_row(int KS)
{
    return (LN ? KS : kStepPad) * (BF16 ? 32 : 16) + (BF16 ? 8 : 4);   // padded: conflict-free 16-byte reads
}

template <int EPI> constexpr bool ln_operand() { return EPI == E_QKV || EPI == E_GELU || EPI == E_VEL; }

constexpr int kBigK = 1024;   // K from which a plain operand's GEMM takes more waves (few rows) or more rows a block

// Where a row of the call goes (E_QKV): its q row, its carry region, its frame there.
struct RowOut {
    int64_t q, kv;
    int frame, pad;
};

template <bool BF16, int EPI, int MB, int NB>
__global__ __launch_bounds__((64 * gemm_waves<MB, NB>()), 2) void gemm_kernel(const GemmParams p)
{
    constexpr int NW = gemm_waves<MB, NB>(), NT = 64 * NW;
    using T = typename std::conditional<BF16, uint16_t, float>::type;
    using Frag = typename std::conditional<BF16, bf16x8_t, f32x4>::type;
    constexpr bool LN = ln_operand<EPI>();
    constexpr int BM = 16 * MB;
    constexpr int KQ = BF16 ? 32 : 16, VE = BF16 ? 8 : 4;
    constexpr int D = NB >= 4 ? 4 : 8;                 // weight steps in flight
    extern __shared__ __align__(16) unsigned char smem[];
    const int LD = panel_row<BF16, LN>(p.KS);
    T* As = (T*)smem;                                  // [LN ? 1 : 2][BM][LD]
    float* ss = (float*)(As + (size_t)BM * LD);        // LN: scale, shift
    RowOut* ro = (RowOut*)(ss + 2 * p.K);              // E_QKV

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int cs = blockIdx.x % p.nsplit, m0 = (blockIdx.x / p.nsplit) * BM;
    const int N16 = (p.N + 15) >> 4;
    const int cb0 = (cs * p.groups * NW + wave) * NB;  // the wave's first column block; groups are NW NB apart

    const u32x4* Wl = (const u32x4*)p.W + lane;
    const u32x4* wn[NB];                               // fragments of the next steps to load
    auto aim = [&](int grp) {
#pragma unroll
        for (int j = 0; j < NB; j++) wn[j] = Wl + ((size_t)min(cb0 + grp * NW * NB + j, N16 - 1) * p.KS) * 64;
    };
    u32x4 w[D][NB];
    auto load_w = [&](int i) {
#pragma unroll
        for (int j = 0; j < NB; j++) w[i][j] = wn[j][i * 64];
    };
    aim(0);
#pragma unroll
    for (int i = 0; i < D; i++) load_w(i);

    constexpr int NVA = (BM * kStepPad * KQ / VE + NT - 1) / NT;   // a plain chunk's vectors per thread
    constexpr int VPR = kStepPad * KQ / VE;
    u32x4 ra[NVA];
    auto gload = [&](int c) {
#pragma unroll
        for (int v = 0; v < NVA; v++) {
            const int idx = tid + NT * v, r = min(idx / VPR, BM - 1), k = c * kStepPad * KQ + (idx % VPR) * VE;
            const u32x4 x = *(const u32x4*)((const T*)p.A + (size_t)min(m0 + r, p.M - 1) * p.K + min(k, p.K - VE));
#pragma unroll
            for (int e = 0; e < 4; e++) ra[v][e] = k < p.K ? x[e] : 0u;
        }
    };
    auto lstore = [&](int buf) {
#pragma unroll
        for (int v = 0; v < NVA; v++) {
            const int idx = tid + NT * v, r = idx / VPR, kv = (idx % VPR) * VE;
            if (BM * VPR % NT == 0 || r < BM) *(u32x4*)(As + (size_t)(buf * BM + r) * LD + kv) = ra[v];
        }
    };

    if constexpr (LN) {
        for (int k4 = tid; k4 < (p.K >> 2); k4 += NT) {   // 1 + scale, shift
            const f32x4 sc = ((const f32x4*)p.ln_scale)[k4];
            ((f32x4*)ss)[k4] = f32x4{1.0f + sc[0], 1.0f + sc[1], 1.0f + sc[2], 1.0f + sc[3]};
            ((f32x4*)(ss + p.K))[k4] = ((const f32x4*)p.ln_shift)[k4];
        }
        if constexpr (EPI == E_QKV) {
            if (tid < BM) {
                const int row = min(m0 + tid, p.M - 1), bp = row / (2 * p.n), f = row % p.n, c = row / p.n - 2 * bp;
                const int b = p.b0 + bp;
                ro[tid] = RowOut{((((int64_t)bp * 2 + c) * p.heads) * p.Fq + f) * 64,
                                 (int64_t)b * p.carry.stream_stride + (int64_t)(c * 2 * p.heads) * p.carry.Fr * 64,
                                 own_base(p.carry, p.prompt, b) + f, 0};
            }
        }
        // NT / 16 rows at a time, 16 threads (one DPP row) per row: thread q takes
        // the row's 4-column vectors q, q + 16, ...; the next rows load
        // meanwhile.  Not unrolled: the code runs once per block, and its
        // instruction fetches cost more than the loop.
        constexpr int NV = 8;                          // K <= 512
        constexpr int NP = (BM + NT / 16 - 1) / (NT / 16);   // passes
        const int q = tid & 15, nv = p.K >> 6;
        f32x4 x[NV], nx[NV];
        auto hload = [&](int mb, f32x4 (&v)[NV]) {
            const f32x4* hr = (const f32x4*)(p.ln_h + (size_t)min(m0 + mb * (NT / 16) + min(tid >> 4, BM - 1), p.M - 1) * p.K) + q;
#pragma unroll
            for (int i = 0; i < NV; i++) v[i] = hr[16 * min(i, nv - 1)];
        };
        hload(0, x);
        __syncthreads();                               // scale and shift are in place
#pragma unroll 1
        for (int mb = 0; mb < NP; mb++) {
            hload(min(mb + 1, NP - 1), nx);
            // the row's first value (lane 0 of the DPP row: row_newbcast:0).  The mean is
            // subtracted before the scaling, as in the few-row kernel: folded into
            // x rstd - mean rstd it is rounded twice (rows whose mean is 20 times their
            // deviation: error of a solve 1.78e-6, folded 2.17e-6, at the same time).
            const float x0 = row_ror<0x150>(x[0][0]);
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int i = 0; i < NV; i++)
                if (i < nv) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const float d = x[i][e] - x0;
                        s1 += d;
                        s2 = fmaf(d, d, s2);
                    }
                }
            s1 = row_sum(s1);
            s2 = row_sum(s2);
            const float md = s1 / (float)p.K;
            const float mean = x0 + md, rstd = 1.0f / sqrtf(fmaxf(s2 / (float)p.K - md * md, 0.f) + 1e-6f);
            const int r = mb * (NT / 16) + (tid >> 4);
            T* row = As + (size_t)r * LD;
            if (r < BM) {
#pragma unroll
            for (int i = 0; i < NV; i++)
                if (i < nv) {
                    const int k = 4 * (q + 16 * i);
                    const f32x4 sc = *(const f32x4*)(ss + k), sh = *(const f32x4*)(ss + p.K + k);
                    f32x4 a;
#pragma unroll
                    for (int e = 0; e < 4; e++) a[e] = fmaf((x[i][e] - mean) * rstd, sc[e], sh[e]);
                    store4<BF16>(row, k, a);
                }
            for (int k = p.K + 4 * q; k < p.KS * KQ; k += 64) store4<BF16>(row, k, f32x4{0.f, 0.f, 0.f, 0.f});
            }
#pragma unroll
            for (int i = 0; i < NV; i++) x[i] = nx[i];
        }
    } else {
        gload(0);
        lstore(0);
    }
    __syncthreads();

    f32x4 acc[MB][NB];
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < MB; i++)
#pragma unroll
            for (int j = 0; j < NB; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // D steps from LDS column `a` of this lane; the weights of the D steps
    // after them (wn) replace the ones that are done.  ROWS: the lane's four
    // results are four rows of one column instead of four columns of one row
    // (the operands change places).
    auto steps = [&](auto rows_tag, const T* a) {
        constexpr bool ROWS = decltype(rows_tag)::value;
        Frag x[2][MB];
#pragma unroll
        for (int i = 0; i < MB; i++) x[0][i] = *(const Frag*)(a + (size_t)16 * i * LD);
#pragma unroll
        for (int s = 0; s < D; s++) {
            if (s + 1 < D) {
#pragma unroll
                for (int i = 0; i < MB; i++) x[(s + 1) & 1][i] = *(const Frag*)(a + (size_t)16 * i * LD + (s + 1) * KQ);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < (BF16 ? 1 : 4); u++)
#pragma unroll
                for (int j = 0; j < NB; j++)
#pragma unroll
                    for (int i = 0; i < MB; i++) {
                        const Frag wf = __builtin_bit_cast(Frag, w[s][j]), xf = x[s & 1][i];
                        if constexpr (BF16)
                            acc[i][j] = ROWS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, wf, acc[i][j], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc[i][j], 0, 0, 0);
                        else
                            acc[i][j] = ROWS ? __builtin_amdgcn_mfma_f32_16x16x4f32(xf[u], wf[u], acc[i][j], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_16x16x4f32(wf[u], xf[u], acc[i][j], 0, 0, 0);
                    }
            load_w(s);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const T* a_lane = As + (size_t)l16 * LD + VE * g;
    auto ahead = [&](int ks) {   // aim at the D steps from ks of this group
#pragma unroll
        for (int j = 0; j < NB; j++) wn[j] += ks * 64;
    };

    if constexpr (LN) {
        for (int grp = 0; grp < p.groups; grp++) {
            const int cb = cb0 + grp * NW * NB;
            clear();
            auto run = [&](auto rows_tag) {
                for (int ks = 0; ks < p.KS; ks += D) {
                    if (ks + D < p.KS) ahead(D);
                    else aim(grp + 1 < p.groups ? grp + 1 : grp);   // the next group's first steps
                    steps(rows_tag, a_lane + ks * KQ);
                }
            };
            // values are stored transposed: their lanes take four frames of one dimension
            const bool vcols = EPI == E_QKV && cb * 16 >= 2 * p.dim;
            if (EPI == E_QKV && vcols) run(std::true_type{});
            else run(std::false_type{});
            if (cb >= N16) break;
            if constexpr (EPI == E_QKV) {
                // the group's columns lie in one head (dim and 16 NB divide by 64 and into it)
                const int col0 = cb * 16, part = col0 / p.dim, hd = (col0 - part * p.dim) >> 6, d0 = col0 & 63;
                const int64_t head_off = (int64_t)((part - 1) * p.heads + hd) * p.carry.Fr * 64;
                if (!vcols) {
                    f32x4 bias[NB];
#pragma unroll
                    for (int j = 0; j < NB; j++) bias[j] = *(const f32x4*)(p.bias + col0 + 16 * j + 4 * g);
#pragma unroll
                    for (int i = 0; i < MB; i++) {
                        if (m0 + 16 * i + l16 >= p.M) continue;
                        const RowOut r = ro[16 * i + l16];
                        T* dst = part == 0 ? (T*)p.q + r.q + (int64_t)hd * p.Fq * 64
                                           : (T*)p.carry.base + r.kv + head_off + (int64_t)r.frame * 64;
#pragma unroll
                        for (int j = 0; j < NB; j++) store4<BF16>(dst, d0 + 16 * j + 4 * g, acc[i][j] + bias[j]);
                    }
                } else {
                    float bias[NB];
#pragma unroll
                    for (int j = 0; j < NB; j++) bias[j] = p.bias[col0 + 16 * j + l16];
#pragma unroll
                    for (int i = 0; i < MB; i++) {
                        const int r0 = 16 * i + 4 * g;
                        // n a multiple of 4: the four rows are four frames of one stream
                        // and branch from a multiple of 4 (the regions start at one too)
                        if ((p.n & 3) == 0) {
                            if (m0 + r0 >= p.M) continue;
                            const RowOut r = ro[r0];
                            T* dst = (T*)p.carry.base + r.kv + head_off + (int64_t)(d0 + l16) * p.carry.Fr + r.frame;
#pragma unroll
                            for (int j = 0; j < NB; j++) {
                                const float bj = bias[j];
                                store4<BF16>(dst, (size_t)(16 * j) * p.carry.Fr, acc[i][j] + f32x4{bj, bj, bj, bj});
                            }
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                if (m0 + r0 + e >= p.M) continue;
                                const RowOut r = ro[r0 + e];
                                T* dst = (T*)p.carry.base + r.kv + head_off + (int64_t)(d0 + l16) * p.carry.Fr + r.frame;
#pragma unroll
                                for (int j = 0; j < NB; j++)
                                    store1<BF16>(dst, (size_t)(16 * j) * p.carry.Fr, acc[i][j][e] + bias[j]);
                            }
                        }
                    }
                }
            } else {
                // columns past N: clamped loads, nothing stored
                f32x4 bias[NB];
#pragma unroll
                for (int j = 0; j < NB; j++) bias[j] = *(const f32x4*)(p.bias + min((cb + j) * 16 + 4 * g, p.N - 4));
#pragma unroll
                for (int i = 0; i < MB; i++) {
                    if (m0 + 16 * i + l16 >= p.M) continue;
                    const size_t at = (size_t)(m0 + 16 * i + l16) * p.N + cb * 16 + 4 * g;
#pragma unroll
                    for (int j = 0; j < NB; j++) {
                        if ((cb + j) * 16 + 4 * g >= p.N) continue;
                        f32x4 y = acc[i][j] + bias[j];
                        if constexpr (EPI == E_GELU) {
#pragma unroll
                            for (int e = 0; e < 4; e++) y[e] = gelu_tanh<BF16>(y[e]);
                            store4<BF16>(p.out, at + 16 * j, y);
                        } else {
                            store4<false>(p.out, at + 16 * j, y);
                        }
                    }
                }
            }
        }
    } else {
        clear();
        const int nc = p.KS / kStepPad;
        for (int c = 0; c < nc; c++) {
            if (c + 1 < nc) gload(c + 1);
            const T* a = a_lane + (size_t)(c & 1) * BM * LD;
#pragma unroll
            for (int ks = 0; ks < kStepPad; ks += D) {
                if (ks + D < kStepPad || c + 1 < nc) ahead(D);
                steps(std::false_type{}, a + ks * KQ);
            }
            if (c + 1 < nc) lstore((c + 1) & 1);
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < NB; j++) {
            const int col = (cb0 + j) * 16 + 4 * g;
            if (col >= p.N) continue;
            EpiPre e[MB];
#pragma unroll
            for (int i = 0; i < MB; i++) e[i] = epi_prefetch<EPI>(p, min(m0 + 16 * i + l16, p.M - 1), col);
#pragma unroll
            for (int i = 0; i < MB; i++) {
                const int row = m0 + 16 * i + l16;
                if (row < p.M) epilogue4<BF16, EPI>(p, row, col, acc[i][j], e[i]);
            }
        }
    }
}

// A kernel launched with more than 64 KB of dynamic LDS needs its limit
// raised first, on each device it runs on: `set` caches, per device, the
// largest size already allowed for that kernel (a race between two threads
// only repeats the call).
constexpr int kMaxDevices = 64;
// Blocks that a LayerNorm GEMM keeps when it gives a block more column groups:
// about two per CU (QKV and MLP up at 14,336 rows: 44.3 and 51.7 us; 59.1 and
// 72.5 from 224 blocks, 56.9 and 64.9 from 900).
constexpr int kGroupBlocks = 448;
static hipError_t allow_lds(const void* kernel, size_t lds, size_t (&set)[kMaxDevices])
{
    if (lds <= 64 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool cached = dev >= 0 && dev < kMaxDevices;
    if (cached && lds <= set[dev]) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess && cached) set[dev] = lds;
    return e;
}

template <bool BF16, int EPI, int MB, int NB>
hipError_t launch_tiled(GemmParams p, hipStream_t st)
{
    constexpr bool LN = ln_operand<EPI>();
    const size_t rows = (size_t)16 * MB * panel_row<BF16, LN>(p.KS) * (BF16 ? 2 : 4);
    const size_t lds = LN ? rows + (size_t)8 * p.K + (EPI == E_QKV ? 16 * MB * sizeof(RowOut) : 0) : 2 * rows;
    constexpr int BN = 16 * NB * gemm_waves<MB, NB>();
    const int tiles_m = (p.M + 16 * MB - 1) / (16 * MB), tiles_n = (p.N + BN - 1) / BN;
    // a LayerNorm operand: one block per row tile normalises once for all its
    // column groups, as long as that leaves kGroupBlocks blocks
    p.nsplit = tiles_n;
    if (LN)
        while (p.nsplit > 1 && tiles_m * (p.nsplit - 1) >= kGroupBlocks) p.nsplit--;
    p.groups = (tiles_n + p.nsplit - 1) / p.nsplit;
    p.nsplit = (tiles_n + p.groups - 1) / p.groups;
    static size_t set[kMaxDevices] = {};
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(&gemm_kernel<BF16, EPI, MB, NB>), lds, set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_kernel<BF16, EPI, MB, NB>), dim3(tiles_m * p.nsplit), dim3(64 * gemm_waves<MB, NB>()), lds, st, p);
    return hipGetLastError();
}

// Tile size by the number of 64 x 64 tiles the call would have: at least
// DCF_TILE_BIG_BLOCKS -> 64 rows x 256 columns, at least DCF_TILE_MID_BLOCKS ->
// 64 x 256 by 8 waves, fewer -> 16 x 128 (more blocks for calls that would not
// fill the machine), or 32 x 128 for a plain operand of K >= 1024 (MLP down, us,
// bf16: 1,792 rows 16.4, 16 x 128 20.7, 32 x 256 23.6; 560 rows 14.0).
#ifndef DCF_TILE_BIG_BLOCKS
#define DCF_TILE_BIG_BLOCKS 1024
#endif
#ifndef DCF_TILE_MID_BLOCKS
#define DCF_TILE_MID_BLOCKS 256
#endif

template <bool BF16, int EPI>
hipError_t launch_tiled_any(const GemmParams& p, hipStream_t st)
{
    const long small_blocks = (long)((p.N + 63) / 64) * ((p.M + 63) / 64);
    if (small_blocks >= DCF_TILE_BIG_BLOCKS) return launch_tiled<BF16, EPI, 4, 4>(p, st);
    if (small_blocks >= DCF_TILE_MID_BLOCKS) return launch_tiled<BF16, EPI, 4, 2>(p, st);
    if constexpr (!ln_operand<EPI>())
        if (p.K >= kBigK) return launch_tiled<BF16, EPI, 2, 1>(p, st);
    return launch_tiled<BF16, EPI, 1, 1>(p, st);
}

// Skinny GEMM for few rows (a call of a handful of streams): block = 16 RB
// rows x 16 NBLK columns, NW waves that split K into contiguous ranges of whole
// MFMA steps; each wave loads its weight and activation fragments for 4
// steps at once, so a block costs few memory round trips.  The weight loads
// of the first batch and the epilogue's operands are issued before anything
// waits.  The partial tiles are summed through LDS in wave order.  With a
// LayerNorm operand the block first normalises its 16 RB rows into LDS
// (operand type, all K).
template <bool BF16, int EPI, bool LN, int NW, int NBLK, int RB>
__global__ __launch_bounds__(64 * NW) void skinny_kernel(const GemmParams p)
{
    using T = typename std::conditional<BF16, uint16_t, float>::type;
    constexpr int KQ = BF16 ? 32 : 16;               // K of one MFMA step group (one 16-byte load per lane)
    constexpr int BATCH = 4;
    constexpr int PAD = BF16 ? 8 : 4;
    constexpr int NPAIR = RB * NBLK;                 // (column block, row block) output tiles of 16 x 16
    constexpr int TPR = 4 * NW / RB;                 // LayerNorm: threads per row
    static_assert(TPR >= 1 && (TPR & (TPR - 1)) == 0 && TPR * 16 * RB == 64 * NW, "skinny shape");
    constexpr int PPW = (NPAIR + NW - 1) / NW;       // tiles each wave finalises
    extern __shared__ __align__(16) unsigned char smem[];
    T* As = (T*)smem;                                 // LN: [16 RB][K + PAD], then scale and shift
    f32x4* red = (f32x4*)smem;                        // after the main loop: [NW waves][NPAIR][64 lanes]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.y * 16 * RB, n0 = blockIdx.x * 16 * NBLK;
    const int LDA = p.K + PAD;
    const T* A = (const T*)p.A;

    const int ng = p.K / KQ;
    const int q0 = wave * ng / NW, q1 = (wave + 1) * ng / NW;
    const u32x4* W[NBLK];   // this lane's fragments of each column block (packed: one per K step)
#pragma unroll
    for (int j = 0; j < NBLK; j++) W[j] = (const u32x4*)p.W + (size_t)min(n0 / 16 + j, (p.N - 1) / 16) * p.KS * 64 + lane;
    // the first batch's weight fragments (they do not wait for the LayerNorm)
    u32x4 wf[BATCH][NBLK];
#pragma unroll
    for (int b = 0; b < BATCH; b++)
#pragma unroll
        for (int j = 0; j < NBLK; j++)
            wf[b][j] = W[j][min(q0 + b, max(q1 - 1, 0)) * 64];
    // the epilogue's operands of the tiles this wave finalises
    EpiPre pre[PPW];
#pragma unroll
    for (int u = 0; u < PPW; u++) {
        const int pp = min(wave + u * NW, NPAIR - 1), j = pp / RB, i = pp % RB;
        pre[u] = epi_prefetch<EPI>(p, min(m0 + 16 * i + l16, p.M - 1), min(n0 + 16 * j + 4 * g, p.N - 4));
    }

    if constexpr (LN) {
        // TPR threads per row, thread q taking the row's 4-column vectors
        // q, q + TPR, ... (whole lines of a row per load), their sums added
        // across DPP rows; each thread a contiguous run, added by shuffles, took
        // 9.0 and 8.8 us per QKV and MLP-up launch at 112 rows in bf16, now 8.2
        // and 8.1 (fp32 11.5 and 12.0, now 10.5 and 11.0).  Scale and shift go
        // through LDS: in registers they cost a block per CU.  Mean and variance
        // come from sums shifted by the row's first value.
        float* ss = (float*)(smem + (size_t)16 * RB * LDA * sizeof(T));   // 1 + scale, shift
        static_assert(TPR == 16 || TPR == 32, "one or two DPP rows per LayerNorm row");
        constexpr int NV = 128 / TPR;                 // K <= 512
        const int r = tid / TPR, q = tid % TPR, nv = p.K / (4 * TPR);
        const f32x4* hr = (const f32x4*)(p.ln_h + (size_t)min(m0 + r, p.M - 1) * p.K) + q;
        f32x4 v[NV];
#pragma unroll
        for (int i = 0; i < NV; i++) v[i] = hr[TPR * min(i, nv - 1)];
        for (int k4 = tid; k4 < (p.K >> 2); k4 += 64 * NW) {
            const f32x4 sc = ((const f32x4*)p.ln_scale)[k4];
            ((f32x4*)ss)[k4] = f32x4{1.0f + sc[0], 1.0f + sc[1], 1.0f + sc[2], 1.0f + sc[3]};
            ((f32x4*)(ss + p.K))[k4] = ((const f32x4*)p.ln_shift)[k4];
        }
        float x0, s1 = 0.f, s2 = 0.f;
        if constexpr (TPR == 16) {
            x0 = row_ror<0x150>(v[0][0]);             // lane 0 of the DPP row
        } else {
            const int u = __builtin_bit_cast(int, v[0][0]);
            const int lo = __builtin_amdgcn_readlane(u, 0), hi = __builtin_amdgcn_readlane(u, 32);
            x0 = __builtin_bit_cast(float, lane < 32 ? lo : hi);
        }
#pragma unroll
        for (int i = 0; i < NV; i++)
            if (i < nv) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float d = v[i][e] - x0;
                    s1 += d;
                    s2 = fmaf(d, d, s2);
                }
            }
        s1 = row_sum(s1);
        s2 = row_sum(s2);
        if constexpr (TPR == 32) {
            s1 = sum_xor16(s1);
            s2 = sum_xor16(s2);
        }
        const float md = s1 / (float)p.K;
        const float mean = x0 + md, rstd = 1.0f / sqrtf(fmaxf(s2 / (float)p.K - md * md, 0.f) + 1e-6f);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NV; i++)
            if (i < nv) {
                const int k = 4 * (q + TPR * i);
                const f32x4 sc = *(const f32x4*)(ss + k), sh = *(const f32x4*)(ss + p.K + k);
                f32x4 a;
#pragma unroll
                for (int e = 0; e < 4; e++) a[e] = fmaf((v[i][e] - mean) * rstd, sc[e], sh[e]);
                store4<BF16>(As, (size_t)r * LDA + k, a);
            }
        __syncthreads();
    }

    int xr[RB];
#pragma unroll
    for (int i = 0; i < RB; i++) xr[i] = min(m0 + 16 * i + l16, p.M - 1);
    f32x4 acc[NBLK][RB];
#pragma unroll
    for (int j = 0; j < NBLK; j++)
#pragma unroll
        for (int i = 0; i < RB; i++) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int q = q0; q < q1; q += BATCH) {
        // all loads of the batch first; a step past the wave's range reloads
        // its last one with a zero weight fragment, so the loop has no branch
        // (its products add exact zeros: the activations are finite)
        u32x4 xf[BATCH][RB];
        if (q != q0) {
#pragma unroll
            for (int b = 0; b < BATCH; b++)
#pragma unroll
                for (int j = 0; j < NBLK; j++)
                    wf[b][j] = W[j][min(q + b, q1 - 1) * 64];
        }
#pragma unroll
        for (int b = 0; b < BATCH; b++) {
            const int k = min(q + b, q1 - 1) * KQ + (BF16 ? 8 : 4) * g;
#pragma unroll
            for (int i = 0; i < RB; i++) {
                if constexpr (LN) xf[b][i] = *(const u32x4*)(As + (16 * i + l16) * LDA + k);
                else xf[b][i] = *(const u32x4*)(A + (size_t)xr[i] * p.K + k);
            }
        }
#pragma unroll
        for (int b = 0; b < BATCH; b++) {
            const bool live = q + b < q1;
#pragma unroll
            for (int j = 0; j < NBLK; j++) {
                u32x4 w = wf[b][j];
#pragma unroll
                for (int e = 0; e < 4; e++) w[e] = live ? w[e] : 0u;
#pragma unroll
                for (int i = 0; i < RB; i++) {
                    if constexpr (BF16) {
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w),
                                                                            __builtin_bit_cast(bf16x8_t, xf[b][i]),
                                                                            acc[j][i], 0, 0, 0);
                    } else {
                        const f32x4 wv = __builtin_bit_cast(f32x4, w), xv = __builtin_bit_cast(f32x4, xf[b][i]);
#pragma unroll
                        for (int u = 0; u < 4; u++)
                            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u], xv[u], acc[j][i], 0, 0, 0);
                    }
                }
            }
        }
    }
    if constexpr (LN) __syncthreads();   // the LDS tile becomes the reduction buffer
#pragma unroll
    for (int j = 0; j < NBLK; j++)
#pragma unroll
        for (int i = 0; i < RB; i++) red[(wave * NPAIR + RB * j + i) * 64 + lane] = acc[j][i];
    __syncthreads();
    // wave w sums its tiles over the waves, in wave order
#pragma unroll
    for (int u = 0; u < PPW; u++) {
        const int pp = wave + u * NW;
        if (pp >= NPAIR) break;
        f32x4 y = red[pp * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; w++) y += red[(w * NPAIR + pp) * 64 + lane];
        const int j = pp / RB, i = pp % RB;
        const int row = m0 + 16 * i + l16, c4 = n0 + 16 * j + 4 * g;
        if (row < p.M && c4 < p.N) epilogue4<BF16, EPI>(p, row, c4, y, pre[u]);
    }
}

// Skinny shapes: waves and 16-column blocks per block, by operand kind.
#ifndef DCF_SK_LN_NBLK
#define DCF_SK_LN_NBLK 2
#endif
#ifndef DCF_SK_PLAIN_NBLK
#define DCF_SK_PLAIN_NBLK 1
#endif
#ifndef DCF_SK_BIGK_WAVES
#define DCF_SK_BIGK_WAVES 8
#endif
#ifndef DCF_SK_PLAIN_WAVES
#define DCF_SK_PLAIN_WAVES 4
#endif
#ifndef DCF_SK_LN_WAVES
#define DCF_SK_LN_WAVES 8
#endif
// 16-row blocks per skinny block, by operand kind
#ifndef DCF_SK_LN_RB
#define DCF_SK_LN_RB 1
#endif
#ifndef DCF_SK_PLAIN_RB
#define DCF_SK_PLAIN_RB 1
#endif

size_t skinny_lds_bytes(const GemmParams& p, int bf16, int nw, int nblk, int rb)
{
    const size_t red = (size_t)nw * rb * nblk * 64 * 16;
    if (!p.ln_h) return red;
    // the normalised tile, then scale and shift
    const size_t a = (size_t)16 * rb * (p.K + (bf16 ? 8 : 4)) * (bf16 ? 2 : 4) + (size_t)2 * p.K * 4;
    return a > red ? a : red;
}

template <bool BF16, int EPI, bool LN, int NW, int NBLK, int RB>
hipError_t launch_skinny(const GemmParams& p, hipStream_t st)
{
    const size_t lds = skinny_lds_bytes(p, BF16, NW, NBLK, RB);
    static size_t set[kMaxDevices] = {};
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(&skinny_kernel<BF16, EPI, LN, NW, NBLK, RB>), lds, set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((skinny_kernel<BF16, EPI, LN, NW, NBLK, RB>),
                       dim3((p.N + 16 * NBLK - 1) / (16 * NBLK), (p.M + 16 * RB - 1) / (16 * RB)),
                       dim3(64 * NW), lds, st, p);
    return hipGetLastError();
}

template <bool BF16, int EPI, bool LN>
hipError_t launch_one(const GemmParams& p, hipStream_t st)
{
    if (p.M <= kSkinnyRows) {
        if constexpr (LN) {
            // the LayerNorm staging gives each of a row's 4 NW / RB threads a
            // whole number of 4-column vectors; 4 waves suffice for K = 64
            if (p.K % (16 * DCF_SK_LN_WAVES / DCF_SK_LN_RB) == 0)
                return launch_skinny<BF16, EPI, true, DCF_SK_LN_WAVES, DCF_SK_LN_NBLK, DCF_SK_LN_RB>(p, st);
            return launch_skinny<BF16, EPI, true, 4, DCF_SK_LN_NBLK, 1>(p, st);
        }
        else if (p.K >= kBigK)
            return launch_skinny<BF16, EPI, false, DCF_SK_BIGK_WAVES, DCF_SK_PLAIN_NBLK, DCF_SK_PLAIN_RB>(p, st);
        else
            return launch_skinny<BF16, EPI, false, DCF_SK_PLAIN_WAVES, DCF_SK_PLAIN_NBLK, DCF_SK_PLAIN_RB>(p, st);
    }
    return launch_tiled_any<BF16, EPI>(p, st);
}

hipError_t launch_gemm(const GemmParams& p, int epi, int bf16, hipStream_t st)
{
    const bool ln = p.ln_h != nullptr;
#define DCF_GEMM(B, E, L)                                     \
    if (bf16 == B && epi == E && ln == L) return launch_one<B, E, L>(p, st);
    // the LayerNorm operand exists for exactly the GEMMs that follow one
    DCF_GEMM(1, E_H, false) DCF_GEMM(1, E_QKV, true) DCF_GEMM(1, E_RES, false) DCF_GEMM(1, E_GELU, true)
    DCF_GEMM(1, E_VEL, true)
    DCF_GEMM(0, E_H, false) DCF_GEMM(0, E_QKV, true) DCF_GEMM(0, E_RES, false) DCF_GEMM(0, E_GELU, true)
    DCF_GEMM(0, E_VEL, true)
#undef DCF_GEMM
    return hipErrorInvalidValue;
}

// --------------------------------------------------------------- attention
//
// Two block shapes: 64 queries by 8 waves when the call has enough (stream,
// branch, head) blocks to fill the device (attn_wide), else 16 queries by 4
// waves, which gives a small call four times the blocks.  The shape fixes the
// order of the softmax merge, so results of the two shapes differ in rounding
// only.  The keys, in Eq. carry's logical order (the retained chunks newest
// first, the prompt, the call's own frames), are cut into tiles of 32 inside
// each segment; a wave takes every second or fourth tile with a running maximum
// per query (online softmax), and the waves' partial results are merged through
// LDS in wave order.  Per tile and group of 16 queries:
//   S^T (keys x queries) = K Q^T        : A = key rows, B = query rows
//   O^T (dims x queries) += V^T P^T     : A = value columns (stored [dim][frame]),
//                                         B = the lane's own probabilities
// In S^T a lane holds eight keys of the tile for query l16; those eight keys,
// in that order, are the lane's K slice of the second product, so P never
// leaves its registers, and the running maximum, sum and rescale of O^T stay
// per lane.
constexpr int kAttnLd = 68;   // padded row of the merge buffer (floats)
// Scores in base 2: q.k / sqrt(64) * log2(e), so the softmax's exponentials are
// plain exp2 (the maximum and the merge work in the same units).
constexpr float kScoreLog2 = 0.125f * 1.4426950408889634f;
constexpr int kAttnWideBlocks = 64;   // blocks of 64 queries below which the narrow shape is used


// Stream b's keys as segments of frames cut into tiles of 32: tile t of the
// call lies at frames [base + t0, base + len) of its carry region.
struct AttnKeys {
    int nh, cur, R, Pr, Sl, f_chunk, plen, own, n, tc, tp;
    __device__ __forceinline__ AttnKeys(const AttnParams& p, int b)
    {
        const CarryRef& cr = p.carry;
        const int64_t hist = p.prompt ? 0 : cr.hist[b];
        nh = hist < cr.R ? (int)hist : cr.R;
        cur = cr.slot[b];
        R = cr.R;
        Pr = cr.Pr;
        Sl = cr.Sl;
        f_chunk = p.f_chunk;
        plen = p.prompt ? 0 : cr.plen[b];
        own = own_base(cr, p.prompt, b);
        n = p.n;
        tc = (f_chunk + 31) >> 5;
        tp = (plen + 31) >> 5;
    }
    __device__ __forceinline__ int total() const { return nh * tc + tp + ((n + 31) >> 5); }
    __device__ __forceinline__ void locate(int t, int& base, int& len, int& t0) const
    {
        int r = 0;
        while (r < nh && t >= tc) {
            t -= tc;
            r++;
        }
        base = Pr + (cur > r ? cur - 1 - r : cur - r + R) * Sl;
        len = f_chunk;
        if (r == nh) {
            const bool prompt = t < tp;
            base = prompt ? 0 : own;
            len = prompt ? plen : n;
            t -= prompt ? 0 : tp;
        }
        t0 = 32 * t;
    }
};

// Mask of an operand word's keys (two in bf16, one in fp32) that are the
// segment's own, `left` of them from the word's first on.  The frames behind a
// segment hold what an earlier call or turn left there, and a probability of
// zero does not cancel an infinity or a NaN.
template <bool BF16> __device__ __forceinline__ uint32_t own_keys(int left)
{
    if constexpr (BF16) return left >= 2 ? ~0u : left == 1 ? 0xffffu : 0u;
    else return left >= 1 ? ~0u : 0u;
}

// Maximum over the lanes that differ in bits 4 and 5 (the four groups of 16).
// (The swaps' results go through scalars: a bit cast straight from a vector's
// element 1 reads element 0.)
__device__ __forceinline__ float max_xor16_32(float v)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a0 = a[0], a1 = a[1];
    const uint32_t w = __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
    const auto c = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const uint32_t c0 = c[0], c1 = c[1];
    return fmaxf(__builtin_bit_cast(float, c0), __builtin_bit_cast(float, c1));
}

// Calls with enough (stream, branch, head) blocks to fill the device: a block
// of 8 waves works on 64 queries.  Wave w owns 16 queries (group w % 4) and
// every second 32-key tile (half w / 4); the four waves of a half share its
// tiles through LDS, and the two halves are merged at the end.  A tile's keys
// and values are loaded by the half's own waves two to three steps ahead into
// registers and stored to the LDS slot that the previous step has left, in
// 16-byte units whose place within a row is XORed with bits of the row, so
// that the 16 rows of an operand read hit 16 different bank groups.
//   bf16: row 4 a + r of score block j is key 8 a + 4 j + r of the tile, so a
//     lane's eight probabilities are eight consecutive keys and its value
//     operand is one 16-byte read.
// What bounds it: HBM, the carried keys and values once: 269 MB per launch at
// 128 streams in 68 us with the launch (4.2 TB/s; 106 us when the eight waves
// split the keys for all 64 queries and merged eight partial results, one
// block of 140 KB LDS per CU; 67.2 without the mask over a segment's last
// values).  At 16 streams, one block per CU, its eight steps' latency: 15.0 us
// (17.9).
template <bool BF16>
__device__ __forceinline__ void attn_wide(const AttnParams& p)
{
    using T = typename std::conditional<BF16, uint16_t, float>::type;
    using Frag = typename std::conditional<BF16, bf16x8_t, f32x4>::type;
    constexpr int VE = BF16 ? 8 : 4;                   // elements of a 16-byte unit
    constexpr int UK = 64 / VE, UV = 32 / VE;          // units of a key row, of a value row (one dimension)
    constexpr int NLK = 8 * UK / 64, NLV = 16 * UV / 64;   // loads per wave and tile
    constexpr int TILE = 32 * UK + 64 * UV;            // units of a tile's keys and values
    constexpr int NSF = 64 / (BF16 ? 32 : 16);         // operand fragments of a 64-value row
    extern __shared__ __align__(16) unsigned char smem[];
    u32x4* ring = (u32x4*)smem;                        // [2 slots][2 halves][TILE]
    int2* tiles = (int2*)(ring + 4 * TILE);            // first frame, frames left in the segment

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int half = wave >> 2, part = wave & 3;       // part: query group, and which quarter of a tile to load
    const int bh = blockIdx.x;
    const int bp = bh / (2 * p.heads), c = (bh / p.heads) & 1, hd = bh % p.heads;
    const int b = p.b0 + bp;
    const int q0 = blockIdx.y * 64 + 16 * part;
    const CarryRef& cr = p.carry;
    const T* Kb = (const T*)cr.base + (size_t)b * cr.stream_stride + ((size_t)((c * 2 + 0) * p.heads + hd)) * cr.Fr * 64;
    const T* Vb = Kb + (size_t)p.heads * cr.Fr * 64;
    const AttnKeys keys(p, b);
    const int total = keys.total(), steps = (total + 1) >> 1;
    for (int t = threadIdx.x; t < total; t += 512) {
        int base, len, t0;
        keys.locate(t, base, len, t0);
        tiles[t] = int2{base + t0, len - t0};
    }

    Frag qf[NSF];                                      // B operand of S^T; rows past n are computed and dropped
    {
        const T* qr = (const T*)p.q + ((((size_t)bp * 2 + c) * p.heads + hd) * p.Fq + q0 + l16) * 64;
#pragma unroll
        for (int s = 0; s < NSF; s++) qf[s] = *(const Frag*)(qr + 4 * VE * s + VE * g);
    }

    // place of unit u of a key row, of a value row
    auto kplace = [](int r, int u) { return r * UK + (u ^ (BF16 ? ((r >> 3) & 3) * 2 + ((r >> 1) & 1) : r & 15)); };
    auto vplace = [](int d, int u) { return 32 * UK + d * UV + (u ^ (BF16 ? (d >> 2) & 3 : (d >> 1) & 7)); };
    struct Regs {
        u32x4 k[NLK], v[NLV];
        int left;
    };
    auto load = [&](int step, Regs& r) {
        const int2 tl = tiles[min(2 * step + half, total - 1)];
        const int first = __builtin_amdgcn_readfirstlane(tl.x), left = __builtin_amdgcn_readfirstlane(tl.y);
        const int last = (left - 1) & ~(VE - 1);
        r.left = left;
#pragma unroll
        for (int i = 0; i < NLK; i++) {
            const int idx = lane + 64 * i, row = 8 * part + idx / UK, u = idx % UK;
            r.k[i] = *(const u32x4*)(Kb + (size_t)(first + min(row, left - 1)) * 64 + VE * u);
        }
#pragma unroll
        for (int i = 0; i < NLV; i++) {   // units past the segment stay in its (padded) storage
            const int idx = lane + 64 * i, d = 16 * part + idx / UV, u = idx % UV;
            r.v[i] = *(const u32x4*)(Vb + (size_t)d * cr.Fr + first + min(VE * u, last));
        }
    };
    auto put = [&](int step, const Regs& r) {
        u32x4* slot = ring + (2 * (step & 1) + half) * TILE;
#pragma unroll
        for (int i = 0; i < NLK; i++) {
            const int idx = lane + 64 * i;
            slot[kplace(8 * part + idx / UK, idx % UK)] = r.k[i];
        }
#pragma unroll
        for (int i = 0; i < NLV; i++) {
            const int idx = lane + 64 * i, u = idx % UV;
            u32x4 v = r.v[i];
            if (r.left < 32) {
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] &= own_keys<BF16>(r.left - VE * u - e * (VE / 4));
            }
            slot[vplace(16 * part + idx / UV, u)] = v;
        }
    };

    float m = -INFINITY, lsum = 0.f;
    f32x4 O[4];
#pragma unroll
    for (int db = 0; db < 4; db++) O[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto work = [&](int step) {
        const int t = 2 * step + half;
        if (t >= total) return;
        const int left = __builtin_amdgcn_readfirstlane(tiles[t].y);
        const u32x4* slot = ring + (2 * (step & 1) + half) * TILE;
        f32x4 st[2];
#pragma unroll
        for (int j = 0; j < 2; j++) {
            st[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int row = BF16 ? 8 * (l16 >> 2) + 4 * j + (l16 & 3) : 16 * j + l16;
#pragma unroll
            for (int s = 0; s < NSF; s++) {
                const Frag kf = __builtin_bit_cast(Frag, slot[kplace(row, 4 * s + g)]);
                if constexpr (BF16) {
                    st[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[s], st[j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; u++)
                        st[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u], qf[s][u], st[j], 0, 0, 0);
                }
            }
        }
        if (left < 32) {   // keys past the segment
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if ((BF16 ? 8 * g + 4 * j : 16 * j + 4 * g) + r >= left) st[j][r] = -INFINITY;
        }
        float mt = fmaxf(fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3])),
                         fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
        mt = max_xor16_32(mt) * kScoreLog2;
        if (__any(mt > m)) {
            const float mn = fmaxf(m, mt), alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < 4; db++) O[db] *= alpha;
        }
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                st[j][r] = __builtin_amdgcn_exp2f(fmaf(st[j][r], kScoreLog2, -m));
                lsum += st[j][r];
            }
        if constexpr (BF16) {
            const u32x4 pw = {pack2(st[0][0], st[0][1]), pack2(st[0][2], st[0][3]), pack2(st[1][0], st[1][1]),
                              pack2(st[1][2], st[1][3])};
#pragma unroll
            for (int db = 0; db < 4; db++)
                O[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(Frag, slot[vplace(16 * db + l16, g)]),
                                                                __builtin_bit_cast(Frag, pw), O[db], 0, 0, 0);
        } else {
#pragma unroll
            for (int db = 0; db < 4; db++)
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    const Frag vf = __builtin_bit_cast(Frag, slot[vplace(16 * db + l16, 4 * j + g)]);
#pragma unroll
                    for (int u = 0; u < 4; u++) O[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[u], st[j][u], O[db], 0, 0, 0);
                }
        }
    };

    // step s: store step s + 1 (loaded two steps ago) to the slot that step
    // s - 1 has left, load step s + 3 in its place, work on step s
    Regs ra, rb;
    __syncthreads();                                   // the tile table is in place
    load(0, ra);
    load(1, rb);
    __builtin_amdgcn_sched_barrier(0);
    put(0, ra);
    load(2, ra);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {   // (a step past the last loads the last tile and does nothing)
        put(s + 1, rb);
        load(s + 3, rb);
        __builtin_amdgcn_sched_barrier(0);
        work(s);
        __syncthreads();
        put(s + 2, ra);
        load(s + 4, ra);
        __builtin_amdgcn_sched_barrier(0);
        work(s + 1);
        __syncthreads();
    }

    // the second half's partial results through LDS; the first half merges and stores
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    float* Os = (float*)smem + (size_t)part * 16 * (kAttnLd + 2);
    if (half) {
#pragma unroll
        for (int db = 0; db < 4; db++) *(f32x4*)(Os + l16 * kAttnLd + 16 * db + 4 * g) = O[db];
        if (g == 0) {
            Os[16 * kAttnLd + l16] = m;
            Os[16 * kAttnLd + 16 + l16] = lsum;
        }
    }
    __syncthreads();
    const int fq = q0 + l16;
    if (half || fq >= p.n) return;
    const float m1 = Os[16 * kAttnLd + l16], mx = fmaxf(m, m1);   // (half 0 has at least one key)
    const float a0 = __builtin_amdgcn_exp2f(m - mx), a1 = __builtin_amdgcn_exp2f(m1 - mx);
    const float inv = 1.0f / (lsum * a0 + Os[16 * kAttnLd + 16 + l16] * a1);
    const size_t row = ((size_t)bp * 2 + c) * p.n + fq;
#pragma unroll
    for (int db = 0; db < 4; db++)
        store4<BF16>(p.o, row * p.dim + hd * 64 + 16 * db + 4 * g,
                     (O[db] * a0 + *(const f32x4*)(Os + l16 * kAttnLd + 16 * db + 4 * g) * a1) * inv);
}

// LDS of a block: the wide shape's ring of tiles (and then the second half's
// partial results) and its table of tiles; of the narrow one, per wave: the partial O of its 16
// queries, their running maxima and sums.
template <bool BF16, int QG, int NW> constexpr size_t attn_lds_bytes()
{
    constexpr size_t ring = (size_t)4 * 32 * 64 * 2 * (BF16 ? 2 : 4), part = (size_t)NW * 16 * (kAttnLd + 2) * 4;
    return QG == 4 ? (ring > part / 2 ? ring : part / 2) : part;   // (without the table)
}

template <bool BF16, int QG, int NW>
__global__ __launch_bounds__(64 * NW, QG == 4 ? 4 : 1) void attn_kernel(const AttnParams p)
{
    static_assert((QG == 4 && NW == 8) || QG == 1, "attention shapes");
    if constexpr (QG == 4) {
        attn_wide<BF16>(p);
        return;
    }
    using T = typename std::conditional<BF16, uint16_t, float>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int QB = 16;                             // queries of the block
    float* Os = (float*)smem;                          // [NW waves][QB queries][kAttnLd]
    float* Ms = Os + NW * QB * kAttnLd;                // [NW][QB]
    float* Ls = Ms + NW * QB;                          // [NW][QB]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int bh = blockIdx.x;
    const int bp = bh / (2 * p.heads), c = (bh / p.heads) & 1, hd = bh % p.heads;
    const int b = p.b0 + bp;
    const int qb0 = blockIdx.y * 16;
    const CarryRef& cr = p.carry;
    const T* Kb = (const T*)cr.base + (size_t)b * cr.stream_stride + ((size_t)((c * 2 + 0) * p.heads + hd)) * cr.Fr * 64;
    const T* Vb = (const T*)cr.base + (size_t)b * cr.stream_stride + ((size_t)((c * 2 + 1) * p.heads + hd)) * cr.Fr * 64;
    const T* qp = (const T*)p.q + (((size_t)bp * 2 + c) * p.heads + hd) * p.Fq * 64;
    const AttnKeys keys(p, b);
    const int total = keys.total();

    // one tile's operands: keys (two blocks of 16) and the value groups
    struct Tile {
        u32x4 kf[2][4];
        u32x4 va[4], vb[4];
    };
    auto load = [&](int t, Tile& tl) {
        int base, len, t0;
        keys.locate(t, base, len, t0);
        const int last4 = (len - 1) & ~3;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const T* kr = Kb + (size_t)(base + min(t0 + 16 * j + l16, len - 1)) * 64;
            if constexpr (BF16) {
#pragma unroll
                for (int s2 = 0; s2 < 2; s2++) tl.kf[j][s2] = *(const u32x4*)(kr + 32 * s2 + 8 * g);
            } else {
#pragma unroll
                for (int s4 = 0; s4 < 4; s4++) tl.kf[j][s4] = *(const u32x4*)(kr + 16 * s4 + 4 * g);
            }
        }
        // value groups: keys t0 + 4 g (+16) .. +3, clamped into the segment's storage
        const int ga = min(t0 + 4 * g, last4), gb2 = min(t0 + 16 + 4 * g, last4);
#pragma unroll
        for (int db = 0; db < 4; db++) {
            const T* vr = Vb + (size_t)(16 * db + l16) * cr.Fr + base;
            if constexpr (BF16) {
                const u32x2 x = *(const u32x2*)(vr + ga), y = *(const u32x2*)(vr + gb2);
                tl.va[db] = u32x4{x[0], x[1], y[0], y[1]};
            } else {
                tl.va[db] = *(const u32x4*)(vr + ga);
                tl.vb[db] = *(const u32x4*)(vr + gb2);
            }
        }
    };

    // query fragments (B operand of S^T)
    struct QFrag {
        bf16x8_t b[2];
        f32x4 f[4];
    };
    auto load_q = [&](QFrag& qfr) {
        const T* qr = qp + (size_t)(qb0 + l16) * 64;   // rows past n are computed and dropped
        if constexpr (BF16) {
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) qfr.b[s2] = *(const bf16x8_t*)(qr + 32 * s2 + 8 * g);
        } else {
#pragma unroll
            for (int s4 = 0; s4 < 4; s4++) qfr.f[s4] = *(const f32x4*)(qr + 16 * s4 + 4 * g);
        }
    };
    // one tile: scores, running maximum and sum, O^T update
    auto step = [&](Tile& cur, int t0, int len, const QFrag& qfr, float& m, float& lsum, f32x4 (&O)[4]) {
        f32x4 st[2];
#pragma unroll
        for (int j = 0; j < 2; j++) {
            st[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (BF16) {
#pragma unroll
                for (int s2 = 0; s2 < 2; s2++)
                    st[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur.kf[j][s2]),
                                                                    qfr.b[s2], st[j], 0, 0, 0);
            } else {
#pragma unroll
                for (int s4 = 0; s4 < 4; s4++) {
                    const f32x4 kv = __builtin_bit_cast(f32x4, cur.kf[j][s4]);
#pragma unroll
                    for (int u = 0; u < 4; u++)
                        st[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[u], qfr.f[s4][u], st[j], 0, 0, 0);
                }
            }
        }
        float mt = -INFINITY;
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const bool live = t0 + 16 * j + 4 * g + r < len;
                st[j][r] = live ? st[j][r] * kScoreLog2 : -INFINITY;
                mt = fmaxf(mt, st[j][r]);
            }
        mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
        mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
        const float mn = fmaxf(m, mt);
        const float alpha = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
        float ps = 0.f;
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                st[j][r] = __builtin_amdgcn_exp2f(st[j][r] - mn);
                ps += st[j][r];
            }
        lsum = lsum * alpha + ps;
#pragma unroll
        for (int db = 0; db < 4; db++) O[db] *= alpha;
        if (len - t0 < 32) {   // values past the segment
            const int left = len - t0 - 4 * g;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t ma = own_keys<BF16>(left - (!BF16 ? e : e < 2 ? 2 * e : 12 + 2 * e));
                const uint32_t mb = own_keys<BF16>(left - 16 - e);
#pragma unroll
                for (int db = 0; db < 4; db++) {
                    cur.va[db][e] &= ma;
                    if constexpr (!BF16) cur.vb[db][e] &= mb;
                }
            }
        }
        if constexpr (BF16) {
            const u32x4 pw = {pack2(st[0][0], st[0][1]), pack2(st[0][2], st[0][3]), pack2(st[1][0], st[1][1]),
                              pack2(st[1][2], st[1][3])};
            const bf16x8_t pf = __builtin_bit_cast(bf16x8_t, pw);
#pragma unroll
            for (int db = 0; db < 4; db++)
                O[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur.va[db]), pf, O[db], 0, 0, 0);
        } else {
#pragma unroll
            for (int db = 0; db < 4; db++) {
                const f32x4 va = __builtin_bit_cast(f32x4, cur.va[db]), vb = __builtin_bit_cast(f32x4, cur.vb[db]);
#pragma unroll
                for (int u = 0; u < 4; u++) O[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u], st[0][u], O[db], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 4; u++) O[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vb[u], st[1][u], O[db], 0, 0, 0);
            }
        }
    };
    QFrag qfr;
    load_q(qfr);
    float m = -INFINITY, lsum = 0.f;
    f32x4 O[4];
#pragma unroll
    for (int db = 0; db < 4; db++) O[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto work = [&](int t, Tile& cur) {
        int base, len, t0;
        keys.locate(t, base, len, t0);
        step(cur, t0, len, qfr, m, lsum, O);
    };
    if constexpr (BF16) {
        // the next tile (or this one again) is in flight while one is worked on
        Tile cur;
        load(min(wave, total - 1), cur);
        for (int t = wave; t < total; t += NW) {
            Tile nxt;
            load(min(t + NW, total - 1), nxt);
            work(t, cur);
            cur = nxt;
        }
    } else {   // fp32 tiles are twice the registers: one at a time
        for (int t = wave; t < total; t += NW) {
            Tile cur;
            load(t, cur);
            work(t, cur);
        }
    }
    // this wave's partial result: O^T lane (l16, g) holds dims 16 db + 4 g + r of query l16
    {
        float l1 = lsum + __shfl_xor(lsum, 16, 64);
        l1 += __shfl_xor(l1, 32, 64);
#pragma unroll
        for (int db = 0; db < 4; db++) *(f32x4*)(Os + ((size_t)wave * QB + l16) * kAttnLd + 16 * db + 4 * g) = O[db];
        if (g == 0) {
            Ms[wave * QB + l16] = m;
            Ls[wave * QB + l16] = l1;
        }
    }
    __syncthreads();
    if (wave > 0) return;
    // merged over the waves, in wave order
    const int qq = l16;
    float mx = Ms[qq];
#pragma unroll
    for (int w = 1; w < NW; w++) mx = fmaxf(mx, Ms[w * QB + qq]);
    float L = 0.f;
    f32x4 acc[4];
#pragma unroll
    for (int db = 0; db < 4; db++) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; w++) {
        const float sc = __builtin_amdgcn_exp2f(Ms[w * QB + qq] - mx);
        L += sc * Ls[w * QB + qq];
#pragma unroll
        for (int db = 0; db < 4; db++) acc[db] += sc * *(const f32x4*)(Os + ((size_t)w * QB + qq) * kAttnLd + 16 * db + 4 * g);
    }
    const float inv = 1.0f / L;
    const int fq = qb0 + qq;
    if (fq < p.n) {
        const size_t row = ((size_t)bp * 2 + c) * p.n + fq;
#pragma unroll
        for (int db = 0; db < 4; db++) store4<BF16>(p.o, row * p.dim + hd * 64 + 16 * db + 4 * g, acc[db] * inv);
    }
}

template <bool BF16, int QG, int NW>
hipError_t launch_attn_shape(const AttnParams& p, int Bc, hipStream_t st)
{
    const dim3 grid(Bc * 2 * p.heads, (p.n + 16 * QG - 1) / (16 * QG));
    const size_t lds = attn_lds_bytes<BF16, QG, NW>() + (QG == 4 ? (size_t)8 * p.max_tiles : 0);
    static size_t set[kMaxDevices] = {};
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(&attn_kernel<BF16, QG, NW>), lds, set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_kernel<BF16, QG, NW>), grid, dim3(64 * NW), lds, st, p);
    return hipGetLastError();
}

// (8 waves in the narrow shape: 0.6 us slower in bf16, 0.3 us faster in fp32 at batch 1)
hipError_t launch_attn(const AttnParams& p, int Bc, int bf16, hipStream_t st)
{
    const bool wide = Bc * 2 * p.heads * ((p.n + 63) / 64) >= kAttnWideBlocks;
    if (bf16) return wide ? launch_attn_shape<true, 4, 8>(p, Bc, st) : launch_attn_shape<true, 1, 4>(p, Bc, st);
    return wide ? launch_attn_shape<false, 4, 8>(p, Bc, st) : launch_attn_shape<false, 1, 4>(p, Bc, st);
}

// ------------------------------------------------------ inputs and the solver

// Row (b', c, f) of the input projection's operand: x | mu | spk | cond, the
// last three zero on the unconditional branch.  x is the initial noise:
// frame tau = pos[b] + f, mel pair j draws Philox4x64-10 at (tau, j, 2, 0)
// under key (seed, keys[b]); Box-Muller of its first two words in fp64.
template <bool BF16>
__global__ __launch_bounds__(256) void assemble_kernel(const AssembleParams p)
{
    const int M4 = 4 * p.n_mel;
    const int64_t total = (int64_t)p.Bc * 2 * p.n * M4;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int col = (int)(e % M4);
    const int row = (int)(e / M4);
    const int bp = row / (2 * p.n), c = (row / p.n) & 1, f = row % p.n;
    const int b = p.b0 + bp;
    const int part = col / p.n_mel, mm = col % p.n_mel;
    float v = 0.f;
    if (part == 0) {
        const dc::Philox4 r = dc::philox4x64_10((uint64_t)(p.pos[b] + f), (uint64_t)(mm >> 1), 2, 0, p.seed, p.keys[b]);
        const double rad = sqrt(-2.0 * log(dc::to_u01(r.v[0])));
        const double ang = 2.0 * M_PI * dc::to_u01(r.v[1]);
        v = p.temperature * (float)((mm & 1) ? rad * sin(ang) : rad * cos(ang));
        if (c == 0) p.x[((size_t)bp * p.n + f) * p.n_mel + mm] = v;
    } else if (c == 0) {
        const size_t fi = ((size_t)bp * p.n + f) * p.n_mel + mm;
        v = part == 1 ? p.mu[fi] : part == 2 ? p.spk[(size_t)b * p.n_mel + mm] : (p.cond ? p.cond[fi] : 0.f);
    }
    store1<BF16>(p.xin, (size_t)row * M4 + col, v);
}

hipError_t launch_assemble(const AssembleParams& p, int bf16, hipStream_t st)
{
    const int64_t total = (int64_t)p.Bc * 2 * p.n * 4 * p.n_mel;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (bf16) hipLaunchKernelGGL((assemble_kernel<true>), grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL((assemble_kernel<false>), grid, dim3(256), 0, st, p);
    return hipGetLastError();
}

// x += dt * ((1 + w) v_cond - w v_uncond); the x columns of both branches'
// operand rows follow; the last step writes the mel output instead.
template <bool BF16>
__global__ __launch_bounds__(256) void euler_kernel(const EulerParams p)
{
    const int64_t total = (int64_t)p.Bc * p.n * p.n_mel;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int mm = (int)(e % p.n_mel);
    const int f = (int)((e / p.n_mel) % p.n);
    const int bp = (int)(e / ((int64_t)p.n_mel * p.n));
    const size_t rc = ((size_t)bp * 2 * p.n + f), ru = rc + p.n;
    const float vc = p.v[rc * p.n_mel + mm], vu = p.v[ru * p.n_mel + mm];
    const float x = p.x[e] + p.dt[0] * ((1.0f + p.w) * vc - p.w * vu);
    p.x[e] = x;
    if (p.mel) {
        p.mel[e] = x;
    } else {
        store1<BF16>(p.xin, rc * 4 * p.n_mel + mm, x);
        store1<BF16>(p.xin, ru * 4 * p.n_mel + mm, x);
    }
}

hipError_t launch_euler(const EulerParams& p, int bf16, hipStream_t st)
{
    const int64_t total = (int64_t)p.Bc * p.n * p.n_mel;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (bf16) hipLaunchKernelGGL((euler_kernel<true>), grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL((euler_kernel<false>), grid, dim3(256), 0, st, p);
    return hipGetLastError();
}

// -------------------------------------------------- per-step constants (init)
//
// The modulations depend only on the step's time t_i: one block per step
// computes the time grid, the sinusoidal embedding of 1000 t_i, the time MLP
// and SiLU of its output; a second launch maps that through every block's
// ada layer (one thread per output).
__global__ __launch_bounds__(256) void temb_kernel(const ConstParams p)
{
    __shared__ float e[1024];
    __shared__ float g[1024];
    const int i = blockIdx.x, tid = threadIdx.x;
    const double ti = 1.0 - cos(0.5 * M_PI * (double)i / (double)p.NS);
    if (tid == 0) {
        const double tn = 1.0 - cos(0.5 * M_PI * (double)(i + 1) / (double)p.NS);
        p.t[i] = (float)ti;
        p.dt[i] = (float)(tn - ti);
        if (i == p.NS - 1) p.t[p.NS] = (float)tn;
    }
    const int half = p.t_dim / 2;
    for (int j = tid; j < half; j += 256) {
        const double arg = 1000.0 * ti * exp(-log(10000.0) * (double)j / (double)half);
        e[j] = (float)cos(arg);
        e[half + j] = (float)sin(arg);
    }
    __syncthreads();
    for (int o = tid; o < p.dim; o += 256) {
        float s = p.b1[o];
        for (int k = 0; k < p.t_dim; k++) s += p.W1[(size_t)o * p.t_dim + k] * e[k];
        g[o] = s / (1.0f + expf(-s));
    }
    __syncthreads();
    for (int o = tid; o < p.dim; o += 256) {
        float s = p.b2[o];
        for (int k = 0; k < p.dim; k++) s += p.W2[(size_t)o * p.dim + k] * g[k];
        p.silu_temb[(size_t)i * p.dim + o] = s / (1.0f + expf(-s));
    }
}

__global__ __launch_bounds__(256) void mods_kernel(const ConstParams p)
{
    const int i = blockIdx.y, l = blockIdx.z;   // l == NL: the final layer
    const int outs = l < p.NL ? 6 * p.dim : 2 * p.dim;
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o >= outs) return;
    const float* W = l < p.NL ? p.ada + (size_t)l * p.ada_stride : p.fada;
    const float* bias = W + (size_t)outs * p.dim;
    const float* s = p.silu_temb + (size_t)i * p.dim;
    float acc = bias[o];
    for (int k = 0; k < p.dim; k++) acc += W[(size_t)o * p.dim + k] * s[k];
    if (l < p.NL) p.mods[((size_t)i * p.NL + l) * 6 * p.dim + o] = acc;
    else p.fmods[(size_t)i * 2 * p.dim + o] = acc;
}

hipError_t launch_consts(const ConstParams& p, hipStream_t st)
{
    hipLaunchKernelGGL(temb_kernel, dim3(p.NS), dim3(256), 0, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mods_kernel, dim3((6 * p.dim + 255) / 256, p.NS, p.NL + 1), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ------------------------------------------------------------ stream state

__global__ void advance_kernel(int64_t* hist, int64_t* pos, int* plen, int* slot, int mode, int b, int P, int B,
                               int f_chunk, int R)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (mode == 0) {
        if (t == 0) {
            hist[b] = 0;
            pos[b] = 0;
            plen[b] = 0;
            slot[b] = 0;
        }
    } else if (mode == 1) {
        if (t == 0) {
            pos[b] = P;
            plen[b] = P;
        }
    } else if (t < B) {
        hist[t] += 1;
        pos[t] += f_chunk;
        slot[t] = slot[t] == R ? 0 : slot[t] + 1;
    }
}

hipError_t launch_advance(int64_t* hist, int64_t* pos, int* plen, int* slot, int mode, int b, int P, int B,
                          int f_chunk, int R, hipStream_t st)
{
    hipLaunchKernelGGL(advance_kernel, dim3((B + 255) / 256), dim3(256), 0, st, hist, pos, plen, slot, mode, b, P, B,
                       f_chunk, R);
    return hipGetLastError();
}

// Carry of (stream b, branch c, kv) at the step and block of cr.base in
// logical order: frames [0, nh * f_chunk) the retained chunks newest first,
// then the prompt; out [frames][heads * 64] fp32.
template <bool BF16>
__global__ __launch_bounds__(256) void gather_kernel(const CarryRef cr, int b, int c, int kv, int heads, int f_chunk,
                                                     int frames, float* out)
{
    using T = typename std::conditional<BF16, uint16_t, float>::type;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int dim = heads * 64;
    if (e >= (int64_t)frames * dim) return;
    const int f = (int)(e / dim), col = (int)(e % dim), hd = col >> 6, d = col & 63;
    const int64_t hist = cr.hist[b];
    const int nh = hist < cr.R ? (int)hist : cr.R;
    int phys;
    if (f < nh * f_chunk) {
        const int r = f / f_chunk;
        phys = cr.Pr + (int)((hist - 1 - r) % (cr.R + 1)) * cr.Sl + f % f_chunk;
    } else {
        phys = f - nh * f_chunk;
    }
    const T* reg = (const T*)cr.base + (size_t)b * cr.stream_stride + ((size_t)((c * 2 + kv) * heads + hd)) * cr.Fr * 64;
    const T v = kv == 0 ? reg[(size_t)phys * 64 + d] : reg[(size_t)d * cr.Fr + phys];
    if constexpr (BF16) out[e] = bf2f(v);
    else out[e] = v;
}

hipError_t launch_carry_gather(const CarryRef& c, int b, int branch, int kv, int heads, int bf16, int frames,
                               int f_chunk, float* out, hipStream_t st)
{
    const int64_t total = (int64_t)frames * heads * 64;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (bf16) hipLaunchKernelGGL((gather_kernel<true>), grid, dim3(256), 0, st, c, b, branch, kv, heads, f_chunk, frames, out);
    else hipLaunchKernelGGL((gather_kernel<false>), grid, dim3(256), 0, st, c, b, branch, kv, heads, f_chunk, frames, out);
    return hipGetLastError();
}

}  // namespace dcf
