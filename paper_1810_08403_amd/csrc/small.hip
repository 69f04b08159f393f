// A small layer in one launch: propagation and ApplyVertex of a few thousand vertices (the fused propagation of Section 3.2 with the
// vertex stage behind it).
#include <type_traits>

#include "device_math.h"
#include "saga_internal.h"
#include "split_bf16.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr uint32_t kPastTheEnd = 0xffff0000u;  // an offset past every table this kernel takes, whatever is added for the lane

template <int AGG>
__device__ __forceinline__ float join(float a, float b)
{
    return AGG == SAGA_AGG_SUM ? a + b : __builtin_fmaxf(b, a);
}

// ---------------------------------------------------------------------------
// What bounds a layer of a few thousand vertices is its launches, each of which waits for the one before, and in a launch the chain
// of memory round trips (and of instruction fetches: the general product is 36 KB of code, read cold). Here a workgroup takes 32
// work items: LPR lanes a column (16, or 32 for rows of more than 64 values), so that its eight wavefronts hold them all at once or
// in two passes, 16 row reads in flight a lane; the sums go to LDS, where the product finds its rows. The weights are read before the
// first item and split behind the last one, by all wavefronts together; each then multiplies 32 columns.
// The results are those of the general kernels bit for bit: edge k goes to partial sum k mod (64 / lanes of a row), and these are
// added pairwise in the order of their numbers' bits; products are formed by the same instructions in the same order (see
// k_gemm_rows for the split, the rows' signs and the results formed again).
// GCN layer, 4,096 vertices of 8 edges, 64 -> 64: 4.2 us of propagation, 3.4 of packing the weights and 7.1 of product before, the call
// 15.0 to 16.4 us; now 9.9, which is the host's part of a call. Making the weights' parts inside the general product instead saved 1.6 us here and cost 1 to 9 us at
// 8,000 to 18,000 vertices.
// ---------------------------------------------------------------------------
template <int AGG, int LPR>
__global__ __launch_bounds__(512) void k_layer_small(const SmallLayerArgs a, const int p2_log2, const uint32_t x_bytes, const uint32_t id_bytes)
{
    constexpr int G = 64 / LPR;  // columns a wavefront works at once, and partial sums a lane holds
    extern __shared__ u32x4 lds[];
    __shared__ int row_v[kSmallRows];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = lane / LPR, sub = lane % LPR;
    const int F = a.F, n_ks = (F + 31) / 32 * 2, n_ct = (a.N + 31) / 32;
    u32x4* const units = lds;  // [32-column tile][16-wide K step][part][lane]
    float* const rows = reinterpret_cast<float*>(lds + n_ct * n_ks * 3 * 64);
    const int stride = n_ks * 16 + 4;
    const int p2 = 1 << p2_log2, part = sub >> p2_log2, ep_log2 = (LPR == 16 ? 4 : 5) - p2_log2;
    const int nvec = (F + 3) / 4;
    const int col = min((sub & (p2 - 1)) * 4, F - 4);  // a row's last fragment ends with the row
    const bool mine = (sub & (p2 - 1)) < nvec;
    const auto xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.X), 0, x_bytes, 0x00020000);
    const auto ids = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.row_idx), 0, id_bytes, 0x00020000);
    const auto ws = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.edge_w), 0, a.edge_w ? id_bytes : 0, 0x00020000);
    const uint32_t ldb = (uint32_t)(a.ldx * 4);
    const int m = lane & 31, h = lane >> 5;

    // this wavefront's units of the weights: column 32 ct + m, k = 16 ks + 8 h + 0..7
    float wt[kSmallUnits / 8][8];
#pragma unroll
    for (int i = 0; i < kSmallUnits / 8; ++i) {
        const int u = wave + 8 * i;
        if (u < n_ct * n_ks) {
            const float* const src = a.W + min(u / n_ks * 32 + m, a.N - 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) wt[i][e] = src[(int64_t)min(u % n_ks * 16 + 8 * h + e, F - 1) * a.ldw];
        }
    }

#pragma unroll 1
    for (int r0 = wave * 4; r0 < wave * 4 + 4; r0 += G) {
        const int r = r0 + grp;
        const int64_t id = (int64_t)blockIdx.x * kSmallRows + r;
        int4 it = make_int4(-1, 0, 0, 0);
        if (id < a.n_items) it = *reinterpret_cast<const int4*>(a.items + id);
        int longest = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) longest = max(longest, __builtin_amdgcn_readlane(it.z - it.y, g * LPR));
        float acc[G][4];
#pragma unroll
        for (int c = 0; c < G; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[c][j] = AGG == SAGA_AGG_SUM ? 0.f : -__builtin_huge_valf();
        int next_id;
        float next_w;
        auto ask = [&](const int e) __attribute__((always_inline)) {
            const uint32_t o = it.y + e + sub < it.z ? (uint32_t)(it.y + e + sub) * 4u : 0xfffffff0u;
            next_id = __builtin_amdgcn_raw_buffer_load_b32(ids, (int)o, 0, 0);
            next_w = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ws, (int)o, 0, 0));
        };
        ask(0);
#pragma unroll 1
        for (int e = 0; e < longest; e += LPR) {
            // an edge past the column's end reads past the table, which gives zeros and no traffic, and adds nothing
            const bool valid = it.y + e + sub < it.z;
            const uint32_t off = valid ? (uint32_t)next_id * ldb : kPastTheEnd;
            const float we = !valid ? (AGG == SAGA_AGG_SUM ? 0.f : __builtin_huge_valf()) : a.edge_w ? next_w : 1.0f;
            const int steps = (min(longest - e, LPR) + (1 << ep_log2) - 1) >> ep_log2;
#pragma unroll 1
            for (int j0 = 0; j0 < steps; j0 += 16) {
                u32x4 x[16];
                const int from = (grp * LPR + (j0 << ep_log2) + part) * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j0 + 4 * q < steps)
#pragma unroll
                        for (int k = 4 * q; k < 4 * q + 4; ++k)
                            x[k] = __builtin_amdgcn_raw_buffer_load_b128(
                                xs, (int)((uint32_t)__builtin_amdgcn_ds_bpermute(from + (k << (ep_log2 + 2)), (int)off) + (uint32_t)col * 4u), 0, 0);
                if (j0 + 16 >= steps && e + LPR < longest) ask(e + LPR);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j0 + 4 * q < steps)
#pragma unroll
                        for (int k = 4 * q; k < 4 * q + 4; ++k) {
                            const float w = __int_as_float(__builtin_amdgcn_ds_bpermute(from + (k << (ep_log2 + 2)), __float_as_int(we)));
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                float& s = acc[k % G][j];
                                const float v = __uint_as_float(x[k][j]);
                                s = AGG == SAGA_AGG_SUM ? fmaf(w, v, s) : __builtin_fmaxf(w * v, s);
                            }
                        }
            }
        }
        for (int o = p2; o < LPR; o <<= 1)
#pragma unroll
            for (int c = 0; c < G; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[c][j] = join<AGG>(acc[c][j], __shfl_xor(acc[c][j], o));
        f32x4_a4 sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float s = join<AGG>(acc[0][j], acc[1][j]);
            if constexpr (G == 4) s = join<AGG>(s, join<AGG>(acc[2][j], acc[3][j]));
            sum[j] = it.y == it.z ? 0.f : s;  // (a maximum over nothing is zero, and so is a row of no item)
        }
        if (part == 0 && mine) {
#pragma unroll
            for (int j = 0; j < 4; ++j) rows[r * stride + col + j] = sum[j];
            if (a.A && it.x >= 0) *reinterpret_cast<f32x4_a4*>(a.A + (int64_t)it.x * a.lda + col) = sum;
        }
        for (int k = F + sub; k < n_ks * 16; k += LPR) rows[r * stride + k] = 0.f;
        if (sub == 0) row_v[r] = it.x;
    }
#pragma unroll
    for (int i = 0; i < kSmallUnits / 8; ++i) {
        const int u = wave + 8 * i;
        if (u < n_ct * n_ks) {
            const int left = F - (u % n_ks * 16 + 8 * h);  // values of k the unit has
            u32x4 p[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t p0, p1, p2_;
                split_pair(2 * d < left ? wt[i][2 * d] * kScale : 0.f, 2 * d + 1 < left ? wt[i][2 * d + 1] * kScale : 0.f, p0, p1, p2_);
                p[0][d] = p0;
                p[1][d] = p1;
                p[2][d] = p2_;
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) units[(u * 3 + q) * 64 + lane] = p[q];
        }
    }
    __syncthreads();
    if (wave >= n_ct) return;

    auto mma = [](const u32x4& x, const u32x4& y, const floatx16& c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
    };
    floatx16 acc, low;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = low[r] = 0.f;
    uint32_t rows_odd = 0, rows_signed = 0;
    const float* const row = rows + m * stride + 8 * h;
#pragma unroll 1
    for (int ks = 0; ks < n_ks; ++ks) {
        const u32x4 x[2] = {*reinterpret_cast<const u32x4*>(row + ks * 16), *reinterpret_cast<const u32x4*>(row + ks * 16 + 4)};
        uint32_t any = 0, hash = (uint32_t)h;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t two = row_code(x[d >> 1][2 * (d & 1)]) + (row_code(x[d >> 1][2 * (d & 1) + 1]) << 1);
            any |= two;
            hash = (hash ^ two) * 0x85ebca6bu;
        }
        const uint64_t odd2 = __builtin_amdgcn_ballot_w64((int32_t)hash < 0), any2 = __builtin_amdgcn_ballot_w64(any != 0);
        const uint32_t now = ((uint32_t)any2 | (uint32_t)(any2 >> 32)) & ~rows_signed;
        rows_odd |= ((uint32_t)odd2 ^ (uint32_t)(odd2 >> 32)) & now;
        rows_signed |= now;
        const float sign = __uint_as_float(__float_as_uint(kScale) ^ ((rows_odd >> m) << 31));
        u32x4 op[3], w[3];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t p0, p1, p2_;
            split_pair(__uint_as_float(x[d >> 1][2 * (d & 1)]) * sign, __uint_as_float(x[d >> 1][2 * (d & 1) + 1]) * sign, p0, p1, p2_);
            op[0][d] = p0;
            op[1][d] = p1;
            op[2][d] = p2_;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) w[q] = units[((wave * n_ks + ks) * 3 + q) * 64 + lane];
        acc = mma(op[0], w[0], acc);
#pragma unroll
        for (int s = 2; s >= 1; --s)
#pragma unroll
            for (int i = 0; i <= s; ++i) low = mma(op[i], w[s - i], low);
    }
    const int n = wave * 32 + m;
    bool not_finite = false;
    {
#pragma clang fp contract(off)
        const uint32_t odd = rows_odd >> (4 * h);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float f = __uint_as_float(((odd << (31 - ((r >> 2) * 8 + (r & 3)))) & 0x80000000u) | __float_as_uint(1.f / (kScale * kScale)));
            acc[r] = (acc[r] + low[r]) * f;
            not_finite |= !(fabsf(acc[r]) < __builtin_huge_valf());
        }
    }
    if (__builtin_expect(__any(not_finite), 0)) {  // these again, with the fp32 instruction
        floatx16 f;
#pragma unroll
        for (int r = 0; r < 16; ++r) f[r] = 0.f;
#pragma unroll 1
        for (int k0 = 0; k0 < F; k0 += 16)
#pragma unroll 1
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + 8 * h + e;
                const float w = a.W[(int64_t)min(k, F - 1) * a.ldw + min(n, a.N - 1)];
                f = __builtin_amdgcn_mfma_f32_32x32x2f32(row[k0 + e], k < F ? w : 0.f, f, 0, 0, 0);
            }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = fabsf(acc[r]) < __builtin_huge_valf() ? acc[r] : f[r];
    }
    if (n >= a.N) return;
    const float bias = a.bias ? a.bias[n] : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int v = row_v[4 * h + (r >> 2) * 8 + (r & 3)];
        float y = acc[r] + bias;
        if (a.act == SAGA_ACT_SIGMOID) y = sigmoid_f32(y);
        if (a.act == SAGA_ACT_RELU && !(y > 0.f)) y = 0.f;
        if (v >= 0) a.Y[(int64_t)v * a.ldy + n] = y;
    }
}

}  // namespace

hipError_t launch_layer_small(const SmallLayerArgs& a, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const int nvec = (a.F + 3) / 4;
    const int64_t x_bytes = ((a.n_src - 1) * a.ldx + a.F) * 4;
    const int n_units = (a.F + 31) / 32 * 2 * ((a.N + 31) / 32);
    if (a.F < kSmallMinF || n_units > kSmallUnits || a.N > kSmallMaxN || a.F > kSmallMaxF || a.N < 1 || a.n_src < 1 || a.n_edges < 0 || a.n_edges >= (1LL << 30) - 64 || a.ldx < a.F ||
        x_bytes > (int64_t)kPastTheEnd)
        return hipErrorInvalidValue;
    int p2_log2 = 2;
    while ((1 << p2_log2) < nvec) ++p2_log2;
    const dim3 grid((unsigned)((a.n_items + kSmallRows - 1) / kSmallRows));
    const uint32_t xb = (uint32_t)x_bytes, ib = (uint32_t)(a.n_edges * 4);
    const size_t lds = (size_t)small_layer_lds(a.F, a.N);
    auto go = [&](auto agg_c, auto lpr_c) -> hipError_t {
        constexpr int AGG = decltype(agg_c)::value, LPR = decltype(lpr_c)::value;
        static PerDevice lds_raised;
        const hipError_t e = lds_raised.once(
            [] { return hipFuncSetAttribute(reinterpret_cast<const void*>(k_layer_small<AGG, LPR>), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024); });
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_layer_small<AGG, LPR>), grid, dim3(512), lds, s, a, p2_log2, xb, ib);
        return hipGetLastError();
    };
    using std::integral_constant;
    using L16 = integral_constant<int, 16>;
    using L32 = integral_constant<int, 32>;
    if (a.agg == SAGA_AGG_SUM) {
        using Sum = integral_constant<int, SAGA_AGG_SUM>;
        return p2_log2 <= 4 ? go(Sum{}, L16{}) : go(Sum{}, L32{});
    }
    using Max = integral_constant<int, SAGA_AGG_MAX>;
    return p2_log2 <= 4 ? go(Max{}, L16{}) : go(Max{}, L32{});
}
