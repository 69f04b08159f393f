// Parameter gradients of backward-ApplyVertex (Section 2.2): C[FP x FQ] = P^T Q, a contraction over all vertices of two
// row-major fp32 matrices (P = the Gather output or the vertices' own features, Q = the gradient of the pre-activation).
//
// The vertex range is divided over splits (the output is tiny, the contraction long); every split writes its own FP x FQ
// partial and a second kernel adds the partials in a fixed tree, so the result does not depend on scheduling. The same
// file holds the two small reductions beside it: the activation's derivative applied to the incoming gradient, and the
// column sums that give the bias gradient.
#include "saga_internal.h"
#include "device_math.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kKT = kTnStep;  // vertices per step

// N consecutive values of a row at the alignment of one: fp32, or bf16 as raw bits
template <typename T, int N>
struct Vals {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
    static __device__ __forceinline__ T get(type v, int j) { return v[j]; }
};
template <typename T>
struct Vals<T, 1> {
    typedef T type;
    static __device__ __forceinline__ T get(type v, int) { return v; }
};
template <typename T>
constexpr int kParts = sizeof(T) == 4 ? 3 : 1;  // bf16 parts of a value

__device__ __forceinline__ float widened(float x) { return x; }
__device__ __forceinline__ float widened(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }

// fp32 values are split times 2^16, so that the third part of any of them is a bf16 value (see gemm.hip)
constexpr float kScale = 65536.f;
template <typename T>
constexpr float kScaleOf = sizeof(T) == 4 ? kScale : 1.f;

// the operands of the matrix instruction for eight values: x kScale = part 0 + part 1 + part 2 exactly, three bf16 values of an
// fp32 one; a bf16 value is its only part. flip: the sign bit, to negate them, or 0.
__device__ __forceinline__ void operands(const float (&v)[8], uint32_t flip, u32x4 (&o)[3])
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const float scale = __uint_as_float(__float_as_uint(kScale) ^ flip);
        float lo = v[2 * d] * scale, hi = v[2 * d + 1] * scale;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t q = __builtin_bit_cast(uint32_t, (bf16x2){(__bf16)lo, (__bf16)hi});
            o[p][d] = q;
            lo -= __uint_as_float(q << 16);
            hi -= __uint_as_float(q & 0xffff0000u);
        }
    }
}
__device__ __forceinline__ void operands(const uint16_t (&v)[8], uint32_t flip, u32x4 (&o)[1])
{
#pragma unroll
    for (int d = 0; d < 4; ++d) o[0][d] = ((uint32_t)v[2 * d] | ((uint32_t)v[2 * d + 1] << 16)) ^ (flip | (flip >> 16));
}

// The product of one split and 32 MTF x 32 NTF block of C per wavefront, nothing shared between wavefronts. Lane l (f = l % 32,
// h = l / 32) reads, of each of the eight vertices 8 h .. 8 h + 7 of a step, MTF consecutive features of P and NTF of Q:
// wave-wide reads are whole row segments, and what a lane holds then is, feature by feature, eight consecutive k of one
// row of P^T (column of Q): the operand of the 32x32x16 bf16 instruction, without a transposition and without LDS. Operand
// row m of tile j is feature MTF m + j. fp32 values enter as three bf16 parts, six of the nine products, as in the products
// over rows (gemm.hip); the five small ones are summed on their own, so that the sum is rounded twice per 16 vertices. A bf16
// matrix (the gradient of a bf16 layer, its features) is read as it is: three products with an fp32 one, one with a bf16 one.
// Every second split takes P negated and brings its partial back with the scale: the instruction cuts addends towards minus infinity,
// a bias that would add up over the splits. A lane whose features end past the matrix takes the last ones again (the same
// values to the same place). A partial with a value that is not finite is formed again with the fp32 instruction.
// Bound: memory for one tile of C (262,144 x 128 x 128 reads 0.27 GB), the matrix instructions and the splitting beside them
// for several; the reads of the next step are in flight while one is multiplied, by eight to twelve wavefronts per compute
// unit. Two steps in flight cost wavefronts and are slower (88 instead of 77 us). MI355X, before (fp32 instruction, tiles
// through LDS) -> now, product + reduction of the partials: 262,144 x 64 x 64 56 + 8 -> 29 + 7 us; 131,072 x 602 x 41
// 158 + 11 -> 118 + 6; 500 x 16 58 + 9 -> 47 + 8; 1,048,576 x 128 x 128 315 -> 288; as backward calls without dX: 262,144 x 128 x
// 128 189 -> 133, 131,072 x 256 x 256 245 -> 190, 512 x 256 371 -> 314, but 65,536 x 640 x 300 348 -> 377, 640 x 640 542 ->
// 618: every tile of C splits its own operands again (now 488 for 131,072 x 640 x 300, 430 for 65,536 x 640 x 640: see gemm_tn_plan).
// The small products in accumulators of their own through all steps: the same times.
template <typename TP, typename TQ, int MTF, int NTF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_gemm_tn(const GemmTnArgs a, const int wm_count, const int tiles_m,
                                                                                             const int tiles_n)
{
    typedef typename Vals<TP, MTF>::type PV;
    typedef typename Vals<TQ, NTF>::type QV;
    typedef typename Vals<float, NTF>::type CV;
    constexpr int PP = kParts<TP>, QP = kParts<TQ>;
    const TP* const P = static_cast<const TP*>(a.P);
    const TQ* const Q = static_cast<const TQ*>(a.Q);
    // blocks b, b + 8, b + 16, ... run on one XCD: give them the tiles of one split, which read the same vertex rows
    const int T = tiles_m * tiles_n;
    const int64_t blk = blockIdx.x;
    const int64_t grp = blk / (8 * (int64_t)T);
    const int within = (int)(blk % (8 * (int64_t)T));
    const int64_t split = grp * 8 + (within & 7);
    const int tile = within >> 3;
    if (split >= a.n_split) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % wm_count, wn = wave / wm_count, wn_count = (int)(blockDim.x >> 6) / wm_count;
    const int i0 = ((tile / tiles_n) * wm_count + wm) * 32 * MTF, j0 = ((tile % tiles_n) * wn_count + wn) * 32 * NTF;
    if (i0 >= a.FP || j0 >= a.FQ) return;
    const int64_t v_begin = split * a.rows_per_split;
    const int64_t v_end = v_begin + a.rows_per_split < a.n ? v_begin + a.rows_per_split : a.n;

    const int f = lane & 31, h = lane >> 5;
    const int fp = min(i0 + MTF * f, a.FP - MTF), fq = min(j0 + NTF * f, a.FQ - NTF);
    const uint32_t flip = (split & 1) ? 0x80000000u : 0u;

    floatx16 acc[MTF][NTF];
#pragma unroll
    for (int i = 0; i < MTF; ++i)
#pragma unroll
        for (int j = 0; j < NTF; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    PV pr[8];
    QV qr[8];
    // addresses of a whole step: the (wave-uniform) row plus a 32-bit offset of the lane (the launcher checks the strides)
    const uint32_t ldpb = (uint32_t)(a.ldp * sizeof(TP)), ldqb = (uint32_t)(a.ldq * sizeof(TQ));
    const uint32_t offp = 8u * h * ldpb + (uint32_t)(fp * sizeof(TP)), offq = 8u * h * ldqb + (uint32_t)(fq * sizeof(TQ));
    auto load = [&](int64_t v0) __attribute__((always_inline)) {
        const char* const pb = reinterpret_cast<const char*>(P + v0 * a.ldp);
        const char* const qb = reinterpret_cast<const char*>(Q + v0 * a.ldq);
        if (v0 + kKT <= v_end) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                pr[k] = *reinterpret_cast<const PV*>(pb + (uint64_t)k * ldpb + offp);
                qr[k] = *reinterpret_cast<const QV*>(qb + (uint64_t)k * ldqb + offq);
            }
        } else {  // the last step of a split: rows past its end are zeros
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                pr[k] = PV{};
                qr[k] = QV{};
                if (v0 + 8 * h + k < v_end) {
                    pr[k] = *reinterpret_cast<const PV*>(pb + (uint64_t)k * ldpb + offp);
                    qr[k] = *reinterpret_cast<const QV*>(qb + (uint64_t)k * ldqb + offq);
                }
            }
        }
    };
    if (v_begin < v_end) load(v_begin);
    for (int64_t v0 = v_begin; v0 < v_end; v0 += kKT) {
        TP x[MTF][8];
        TQ y[NTF][8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
#pragma unroll
            for (int i = 0; i < MTF; ++i) x[i][k] = Vals<TP, MTF>::get(pr[k], i);
#pragma unroll
            for (int j = 0; j < NTF; ++j) y[j][k] = Vals<TQ, NTF>::get(qr[k], j);
        }
        if (v0 + kKT < v_end) load(v0 + kKT);
        __builtin_amdgcn_sched_barrier(0);
        u32x4 oq[NTF][QP];
#pragma unroll
        for (int j = 0; j < NTF; ++j) operands(y[j], 0, oq[j]);
#pragma unroll
        for (int i = 0; i < MTF; ++i) {
            u32x4 op[PP];
            operands(x[i], flip, op);
            auto mma = [](const u32x4& u, const u32x4& w, const floatx16& c) __attribute__((always_inline)) {
                return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u), __builtin_bit_cast(bf16x8, w), c, 0, 0, 0);
            };
            if constexpr (PP + QP > 2) {
                floatx16 low[NTF];
#pragma unroll
                for (int j = 0; j < NTF; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) low[j][r] = 0.f;
#pragma unroll
                for (int s = 2; s >= 1; --s)  // the smallest first
#pragma unroll
                    for (int p = 0; p <= s; ++p)
                        if (p < PP && s - p < QP)
#pragma unroll
                            for (int j = 0; j < NTF; ++j) low[j] = mma(op[p < PP ? p : 0], oq[j][s - p < QP ? s - p : 0], low[j]);
#pragma unroll
                for (int j = 0; j < NTF; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] += low[j][r];
            }
#pragma unroll
            for (int j = 0; j < NTF; ++j) acc[i][j] = mma(op[0], oq[j][0], acc[i][j]);
        }
    }

    const float unscale = __uint_as_float(__float_as_uint(1.f / (kScaleOf<TP> * kScaleOf<TQ>)) ^ flip);
    bool bad = false;
#pragma unroll
    for (int i = 0; i < MTF; ++i)
#pragma unroll
        for (int j = 0; j < NTF; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] *= unscale;
                bad |= !(fabsf(acc[i][j][r]) < __builtin_huge_valf());
            }
    // this split's partial: the lane holds, of every tile, column f and the 16 rows 8 (r / 4) + 4 h + r % 4
    float* const out = a.part + split * (int64_t)a.FP * a.FQ + fq;
    int hh = h;
    asm volatile("" : "+v"(hh));  // or the addresses of all rows are kept in registers through the whole kernel
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = min(i0 + MTF * ((r >> 2) * 8 + 4 * hh + (r & 3)), a.FP - MTF);
#pragma unroll
        for (int i = 0; i < MTF; ++i) {
            CV v;
            if constexpr (NTF == 1) {
                v = acc[i][0][r];
            } else {
#pragma unroll
                for (int j = 0; j < NTF; ++j) v[j] = acc[i][j][r];
            }
            *reinterpret_cast<CV*>(out + (int64_t)(row + i) * a.FQ) = v;
        }
    }

    if (__builtin_expect(__any(bad), 0)) {
        // the values that are not finite again, over what has just been written there (a lane's own stores; lanes that write
        // the same place write the same value). Bound by the latency of reads eight vertices at a time: 262,144 x 128 x 128 with
        // one infinite value, as a layer's backward call of 332 us: 513 us (two vertices at a time: 1273)
#pragma unroll 1
        for (int b = 0; b < MTF * NTF; ++b) {
            const int i = b / NTF, j = b % NTF;
            int h2 = h;
            asm volatile("" : "+v"(h2));
            bool here = false;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = min(i0 + MTF * ((r >> 2) * 8 + 4 * h2 + (r & 3)), a.FP - MTF);
                here |= !(fabsf(out[(int64_t)(row + i) * a.FQ + j]) < __builtin_huge_valf());
            }
            if (!__any(here)) continue;
            floatx16 g;
#pragma unroll
            for (int r = 0; r < 16; ++r) g[r] = 0.f;
            const TP* p = P + (v_begin + 8 * h) * a.ldp + fp + i;
            const TQ* q = Q + (v_begin + 8 * h) * a.ldq + fq + j;
#pragma unroll 1
            for (int64_t v0 = v_begin; v0 < v_end; v0 += kKT, p += kKT * a.ldp, q += kKT * a.ldq) {
                float x[8], y[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool in = v0 + 8 * h + k < v_end;
                    x[k] = in ? widened(p[k * a.ldp]) : 0.f;
                    y[k] = in ? widened(q[k * a.ldq]) : 0.f;
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) g = __builtin_amdgcn_mfma_f32_32x32x2f32(x[k], y[k], g, 0, 0, 0);
            }
            asm volatile("" : "+v"(h2));
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = min(i0 + MTF * ((r >> 2) * 8 + 4 * h2 + (r & 3)), a.FP - MTF);
                float* const o = out + (int64_t)(row + i) * a.FQ + j;
                if (!(fabsf(*o) < __builtin_huge_valf())) *o = g[r];
            }
        }
    }
}

// Rows so far apart that a step's offsets don't fit 32 bits (a stride of 64 M values: a few rows of a huge buffer): one
// thread per split and element of C
template <typename TP, typename TQ>
__global__ __launch_bounds__(256) void k_gemm_tn_far(const GemmTnArgs a)
{
    const int64_t count = (int64_t)a.FP * a.FQ, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count * a.n_split) return;
    const int64_t split = i / count, e = i % count, p = e / a.FQ, q = e % a.FQ;
    const int64_t v_begin = split * a.rows_per_split;
    const int64_t v_end = v_begin + a.rows_per_split < a.n ? v_begin + a.rows_per_split : a.n;
    float s = 0.f;
    for (int64_t v = v_begin; v < v_end; ++v)
        s = fmaf(widened(static_cast<const TP*>(a.P)[v * a.ldp + p]), widened(static_cast<const TQ*>(a.Q)[v * a.ldq + q]), s);
    a.part[i] = s;
}

// C[r][c] = sum over splits. A block of 1,024 threads owns EL consecutive elements; 1024 / EL lanes per element each add
// every (1024 / EL)-th split in order, eight loads in flight at a time, and the lanes' sums are added in a fixed tree: the
// grouping depends on n_split and EL alone, and EL on the number of elements.
// Bound by the latency of a load: the partials (n_split x count, up to some 60 MB) sit in the caches, but with four lanes
// per element that each waited for one load after the other a launch took 62 us for 16,384 elements x 1,024 splits and
// still 61 us for 128 elements; now 11 and 5 us. Few elements (a bias) get 64 lanes each so that the chain stays short,
// many get 64-element rows for whole 256-byte reads.
template <int EL>
__global__ __launch_bounds__(1024) void k_sum_splits(const float* __restrict__ part, int64_t count, int n_split, int FQ, float* __restrict__ C,
                                                     int64_t ldc, int accumulate)
{
    constexpr int LANES = 1024 / EL, U = 8;
    __shared__ float red[LANES][EL + 1];
    const int e = threadIdx.x % EL, q = threadIdx.x / EL;
    const int64_t i = (int64_t)blockIdx.x * EL + e;
    float s = 0.f;
    if (i < count) {
        const float* p = part + i;
        int k = q;
        for (; k + (U - 1) * LANES < n_split; k += U * LANES) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = p[(int64_t)(k + u * LANES) * count];
#pragma unroll
            for (int u = 0; u < U; ++u) s += x[u];
        }
        for (; k < n_split; k += LANES) s += p[(int64_t)k * count];
    }
    red[q][e] = s;
#pragma unroll
    for (int h = LANES / 2; h > 0; h /= 2) {
        __syncthreads();
        if (q < h) red[q][e] += red[q + h][e];
    }
    if (q == 0 && i < count) {
        float* c = C + (i / FQ) * ldc + (i % FQ);
        const float r = red[0][e];
        *c = accumulate ? *c + r : r;  // accumulate: a later tile of rows adds to what earlier tiles left (streamed calls)
    }
}

hipError_t sum_splits(const float* part, int64_t count, int n_split, int FQ, float* C, int64_t ldc, int accumulate, hipStream_t s)
{
    // 64-element rows from the count on that gives every compute unit a block of them: fewer blocks than compute units
    // would leave the others idle behind the same chain of loads
    if (count >= 256 * 64)
        hipLaunchKernelGGL((k_sum_splits<64>), dim3((unsigned)((count + 63) / 64)), dim3(1024), 0, s, part, count, n_split, FQ, C, ldc, accumulate);
    else
        hipLaunchKernelGGL((k_sum_splits<16>), dim3((unsigned)((count + 15) / 16)), dim3(1024), 0, s, part, count, n_split, FQ, C, ldc, accumulate);
    return hipGetLastError();
}

// backward-ApplyVertex's elementwise part over a slab of rows: the activation's derivative taken from the
// layer's output (MODE 1, ReLU: dZ = dY where Y > 0, else 0; MODE 2, sigmoid: dZ = dY * Y (1 - Y); MODE 0: dZ
// is dY itself and nothing is stored), and the slab's column sums of dZ for the bias gradient. A thread owns VEC consecutive columns
// and every RL-th row of the slab (RL row lanes when the matrix is narrower than the block); the
// row lanes' sums are added in lane order.
__device__ __forceinline__ float act_grad(int mode, float g, float y)
{
    if (mode == 1) return y > 0.f ? g : 0.f;
    return g * (y * (1.0f - y));
}

// bf16: the gradient stays bf16 (ReLU or no activation; without one it is copied, since the caller's rows may be where dX is
// written). 0 on NaN, as y > 0 is false for it. Bound by memory (two bf16 reads and a write: 131,072 x 256 at 5.9 TB/s): a pass
// that found row and column of every value by a 64-bit division and wrote dZ as bf16 and fp32 took 110 us, the column sums
// of the fp32 copy 28 more, the parameter-gradient product over it 131; now 34 together and 101.
__device__ __forceinline__ uint16_t act_grad(int, uint16_t g, uint16_t y)
{
    return widened(y) > 0.f ? g : (uint16_t)0;
}

template <typename T, int VEC, int MODE>
__global__ __launch_bounds__(256) void k_dz_colsum(const T* __restrict__ dY, int64_t lddy, const T* __restrict__ Y, int64_t ldy,
                                                   T* __restrict__ dZ, int64_t lddz, int64_t rows, int F, int64_t R,
                                                   float* __restrict__ part)
{
    // bf16 rows are read VEC values at a time at any alignment; four 16-byte values (fp32) only from aligned rows
    typedef typename std::conditional<sizeof(T) == 4 && VEC == 4, float4, typename Vals<T, VEC>::type>::type V;
    constexpr bool STORE = MODE != 0 || sizeof(T) == 2;
    __shared__ float red[256 * VEC];
    const int ncg = (F + VEC - 1) / VEC;                  // column groups
    const int RL = ncg >= 256 ? 1 : 256 / ncg;            // row lanes
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int64_t r1 = r0 + R < rows ? r0 + R : rows;
    for (int cg0 = 0; cg0 < ncg; cg0 += 256) {            // one pass unless the matrix is wider than 256 groups
        const int t = threadIdx.x;
        const int cg = cg0 + (RL == 1 ? t : t % ncg), rl = RL == 1 ? 0 : t / ncg;
        const bool live = cg < ncg && rl < RL;
        float sum[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) sum[j] = 0.f;
        if (live) {
            const int c = cg * VEC;
#pragma unroll 4
            for (int64_t r = r0 + rl; r < r1; r += RL) {
                const V gv = *reinterpret_cast<const V*>(dY + r * lddy + c);
                T g[VEC];
                __builtin_memcpy(g, &gv, sizeof(g));
                if constexpr (MODE != 0) {
                    const V yv = *reinterpret_cast<const V*>(Y + r * ldy + c);
                    T y[VEC];
                    __builtin_memcpy(y, &yv, sizeof(y));
#pragma unroll
                    for (int j = 0; j < VEC; ++j) g[j] = act_grad(MODE, g[j], y[j]);
                }
                if constexpr (STORE) {
                    V zv;
                    __builtin_memcpy(&zv, g, sizeof(g));
                    *reinterpret_cast<V*>(dZ + r * lddz + c) = zv;
                }
#pragma unroll
                for (int j = 0; j < VEC; ++j) sum[j] += widened(g[j]);
            }
        }
        if (part) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < VEC; ++j) red[t * VEC + j] = sum[j];
            __syncthreads();
            if (live && rl == 0) {
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    float s = 0.f;
                    for (int l = 0; l < RL; ++l) s += red[(RL == 1 ? t : l * ncg + (cg - cg0)) * VEC + j];
                    if (cg * VEC + j < F) part[(int64_t)blockIdx.x * F + cg * VEC + j] = s;
                }
            }
        }
    }
}

// out[i] = in[perm[i]]
__global__ __launch_bounds__(256) void k_permute_f32(const float* __restrict__ in, const int32_t* __restrict__ perm, float* __restrict__ out,
                                                     int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) out[i] = in[perm[i]];
}

// d[i] *= sigmoid'(z[i]). The slope is formed from the pre-activation, not from a stored sigmoid h as h (1 - h): an
// fp32 h close to 1 has lost 1 - h (z = 9: 1 - h = 1.2e-4 known to 2^-25, a relative error of 2.4e-4 in the slope).
__global__ __launch_bounds__(256) void k_sigmoid_grad(float* __restrict__ d, const float* __restrict__ z, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        float g, slope;
        sigmoid_and_slope_f32(z[i], g, slope);
        d[i] *= slope;
    }
}

template <typename TP, typename TQ, int MTF, int NTF>
hipError_t launch_tn_cfg(const GemmTnArgs& a, const TnShape& t, hipStream_t s)
{
    const int64_t tiles_m = t.tiles_m(a.FP), tiles_n = t.tiles_n(a.FQ);
    const int64_t blocks = (a.n_split + 7) / 8 * 8 * tiles_m * tiles_n;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_tn<TP, TQ, MTF, NTF>), dim3((unsigned)blocks), dim3((unsigned)(64 * t.wm * t.wn)), 0, s, a, t.wm, (int)tiles_m, (int)tiles_n);
    return hipGetLastError();
}

template <typename TP, typename TQ>
hipError_t launch_tn(const GemmTnArgs& a, hipStream_t s)
{
    const TnShape t = tn_shape(a.FP, a.FQ);
    constexpr int64_t kNear = 1LL << 26;  // 8 rows of fp32 at this stride are 2^31 bytes
    if (a.ldp >= kNear || a.ldq >= kNear || a.ldp < 0 || a.ldq < 0) {
        const int64_t blocks = ((int64_t)a.FP * a.FQ * a.n_split + 255) / 256;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_gemm_tn_far<TP, TQ>), dim3((unsigned)blocks), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    if (t.ntf == 2) return t.mtf == 2 ? launch_tn_cfg<TP, TQ, 2, 2>(a, t, s) : launch_tn_cfg<TP, TQ, 1, 2>(a, t, s);
    return t.mtf == 4 ? launch_tn_cfg<TP, TQ, 4, 1>(a, t, s) : launch_tn_cfg<TP, TQ, 1, 1>(a, t, s);
}

}  // namespace

hipError_t launch_gemm_tn(const GemmTnArgs& a, float* C, int64_t ldc, int accumulate, hipStream_t s)
{
    if (a.FP <= 0 || a.FQ <= 0) return hipSuccess;
    if (a.n_split < 1 || a.rows_per_split < 1 || a.rows_per_split % kKT != 0 || !a.part) return hipErrorInvalidValue;
    if ((int64_t)a.n_split * a.rows_per_split < a.n) return hipErrorInvalidValue;
    if (a.p_dtype == SAGA_BF16 && a.q_dtype != SAGA_BF16) return hipErrorInvalidValue;  // no caller has this pair
    const hipError_t e = a.q_dtype != SAGA_BF16   ? launch_tn<float, float>(a, s)
                         : a.p_dtype != SAGA_BF16 ? launch_tn<float, uint16_t>(a, s)
                                                  : launch_tn<uint16_t, uint16_t>(a, s);
    if (e != hipSuccess) return e;
    const int64_t count = (int64_t)a.FP * a.FQ;
    return sum_splits(a.part, count, a.n_split, a.FQ, C, ldc, accumulate, s);
}

int64_t colsum_slabs(int64_t rows) { return std::max<int64_t>(1, std::min<int64_t>(1024, (rows + 127) / 128)); }

hipError_t launch_dz_colsum(const float* dY, int64_t lddy, const float* Y, int64_t ldy, int32_t act, float* dZ, int64_t rows, int32_t F,
                            float* part, float* dbias, int accumulate, hipStream_t s, int64_t lddz)
{
    if (F <= 0) return hipSuccess;
    if (lddz <= 0) lddz = F;
    if (act == SAGA_ACT_NONE) Y = nullptr;
    if (act != SAGA_ACT_NONE && !Y) return hipErrorInvalidValue;
    if (!Y && !part) return hipSuccess;  // nothing to mask, nothing to sum
    const int64_t slabs = colsum_slabs(rows);
    const int64_t R = (std::max<int64_t>(rows, 1) + slabs - 1) / slabs;
    const bool mask = Y != nullptr;
    const bool sig = act == SAGA_ACT_SIGMOID;
    const bool vec4 = F % 4 == 0 && lddy % 4 == 0 && (!mask || (ldy % 4 == 0 && lddz % 4 == 0)) && (reinterpret_cast<uintptr_t>(dY) & 15u) == 0 &&
                      (!mask || ((reinterpret_cast<uintptr_t>(Y) & 15u) == 0 && (reinterpret_cast<uintptr_t>(dZ) & 15u) == 0));
    const dim3 grid((unsigned)slabs), block(256);
    if (vec4 && mask && sig)
        hipLaunchKernelGGL((k_dz_colsum<float, 4, 2>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    else if (vec4 && mask)
        hipLaunchKernelGGL((k_dz_colsum<float, 4, 1>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    else if (vec4)
        hipLaunchKernelGGL((k_dz_colsum<float, 4, 0>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    else if (mask && sig)
        hipLaunchKernelGGL((k_dz_colsum<float, 1, 2>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    else if (mask)
        hipLaunchKernelGGL((k_dz_colsum<float, 1, 1>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    else
        hipLaunchKernelGGL((k_dz_colsum<float, 1, 0>), grid, block, 0, s, dY, lddy, Y, ldy, dZ, lddz, rows, F, R, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !part) return e;
    return sum_splits(part, F, (int)slabs, F, dbias, F, accumulate, s);
}

hipError_t launch_permute_f32(const float* in, const int32_t* perm, float* out, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((count + 255) / 256, 1 << 20);
    hipLaunchKernelGGL(k_permute_f32, dim3(grid), dim3(256), 0, s, in, perm, out, count);
    return hipGetLastError();
}

hipError_t launch_sigmoid_grad(float* d, const float* z, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((count + 255) / 256, 1 << 20);
    hipLaunchKernelGGL(k_sigmoid_grad, dim3(grid), dim3(256), 0, s, d, z, count);
    return hipGetLastError();
}

hipError_t launch_dz_bf16(const uint16_t* dY, int64_t lddy, const uint16_t* Y, int64_t ldy, uint16_t* dZ, int64_t rows, int32_t F,
                          float* part, float* dbias, hipStream_t s)
{
    if (F <= 0) return hipSuccess;
    const int64_t slabs = colsum_slabs(rows);
    const int64_t R = (std::max<int64_t>(rows, 1) + slabs - 1) / slabs;
    auto go = [&](auto vec) {
        constexpr int VEC = decltype(vec)::value;
        if (Y)
            hipLaunchKernelGGL((k_dz_colsum<uint16_t, VEC, 1>), dim3((unsigned)slabs), dim3(256), 0, s, dY, lddy, Y, ldy, dZ, F, rows, F, R, part);
        else
            hipLaunchKernelGGL((k_dz_colsum<uint16_t, VEC, 0>), dim3((unsigned)slabs), dim3(256), 0, s, dY, lddy, Y, ldy, dZ, F, rows, F, R, part);
    };
    // the widest read that divides the row: a lane's values don't cross into the next one
    if (F % 8 == 0)
        go(std::integral_constant<int, 8>{});
    else if (F % 2 == 0)
        go(std::integral_constant<int, 2>{});
    else
        go(std::integral_constant<int, 1>{});
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    return part ? sum_splits(part, F, (int)slabs, F, dbias, F, 0, s) : hipSuccess;
}
