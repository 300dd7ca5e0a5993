// HIP kernels of the MDOT-PNCG hot path for gfx950 (MI355X).
//
// One solver step is three kernels on the context stream, with no synchronisation between
// workgroups inside them:
//   k_sweep : one fused pass over the cost for a line-search trial: every workgroup forms
//             X_ij = u_i + v_j - gamma C_ij for a BR x BC tile (FP64 argument), takes one exp
//             per element and accumulates BOTH the row sums and the column sums from that
//             single read of C (row sums reduced across the wave64 through an LDS transpose,
//             column sums across the four waves). It writes per-tile partials only.
//             The same kernel runs the two Round / certificate passes of a stage.
//   k_fin   : a group of lanes per entry of the (m + n)-vectors: stores the vector update decided
//             by the previous step (accept a line-search step, start a stage with smoothing
//             and warm start, prepare Round), combines the tile partials of its row or column
//             in FP64 in a fixed order and reduces the dot products of the line search and of
//             PNCG per workgroup.
//   k_decide: one wave: reduces those dots in a fixed order and runs the scalar logic of
//             the line search (App. B), PNCG (Alg. 2) and the annealing loop (Alg. 1), then
//             stores the next state. Kernel boundaries order the three; no atomics or fences.
// Problems of at most 1024 tiles run the steps between a stage's start and its end in one kernel,
// k_steps, whose workgroups exchange the same values through memory; mdot_lse2 up to 512 tiles is one
// kernel, k_lse. Both give the bits of the three kernels, which run everything else.
// The sweeps evaluate the pending vector update on the fly for their own rows and columns
// with the same function k_fin uses to store it (explicit fma, so both are bit-identical).
// The host never reads a value between steps; it replays a captured graph of steps and
// polls the done flag once per chunk.
//
// Exponent shifts: the row sum of row i is taken relative to a predicted log row sum s_i
// (the last accepted log r(P)_i moved by alpha p_i, or log r~_i at a stage start), so
// every exp argument of the entries that matter is O(1). Column sums reuse the same exp
// through per-row weights exp(s_i - S_I), S_I = max of s_i over the tile. A row or column
// whose shifted sum leaves [2^-64, 2^64] (FP32) is reported and the sweep is re-run with
// FP64 exp.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "mdot_internal.h"

namespace mdot {

#define LOG2E_D 1.4426950408889634074
#define LN2_D 0.6931471805599453094

static_assert(kBR == 64, "a sweep tile has one row per lane of a wave64");

// Members of the control block that starts at a Work struct in device memory. `w` must be a
// reference to that struct (not a copy): the addresses follow from &w without loading it.
__device__ __forceinline__ Control& ctl_of(const Work& w) { return *reinterpret_cast<Control*>(const_cast<Work*>(&w)); }
__device__ __forceinline__ State* state_slot(const Work& w, int s) { return ctl_of(w).st + s; }
__device__ __forceinline__ const DevParams& params_of(const Work& w) { return ctl_of(w).prm; }
__device__ __forceinline__ double* bdots_of(const Work& w) { return ctl_of(w).bdots; }

// ------------------------------------------------------------------ cross-lane reductions
// DPP moves of an FP64 value (two 32-bit halves): lane i receives v from the lane the control
// selects; lanes outside `ROW_MASK` or whose source lies outside the row receive `id`.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_d(double id, double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v), o = __builtin_bit_cast(uint64_t, id);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(b >> 32), CTRL,
                                                               ROW_MASK, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// The same with every row enabled and 0 for lanes whose source lies outside the row (bound
// control): a sum's identity without initialising the destination.
template <int CTRL>
__device__ __forceinline__ double dpp_d0(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double readlane_d(double v, int lane)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int OP>  // 0: sum, 1: min, 2: max
__device__ __forceinline__ double red_op(double a, double b)
{
    if constexpr (OP == 0) return a + b;
    else if constexpr (OP == 1) return fmin(a, b);
    else return fmax(a, b);
}

// Reduction over the 64 lanes of a wave in a fixed order: inclusive scans within each row of
// 16 lanes (row_shr 1, 2, 4, 8), then row 0 into row 1 and row 2 into row 3 (row_bcast:15),
// then rows 0-1 into rows 2-3 (row_bcast:31); lane 63 holds the result, returned to all lanes.
template <int OP>
__device__ __forceinline__ double wave_reduce(double v)
{
    const double id = (OP == 0) ? 0.0 : (OP == 1 ? INFINITY : -INFINITY);
    v = red_op<OP>(v, dpp_d<0x111>(id, v));
    v = red_op<OP>(v, dpp_d<0x112>(id, v));
    v = red_op<OP>(v, dpp_d<0x114>(id, v));
    v = red_op<OP>(v, dpp_d<0x118>(id, v));
    v = red_op<OP>(v, dpp_d<0x142, 0xa>(id, v));
    v = red_op<OP>(v, dpp_d<0x143, 0xc>(id, v));
    return readlane_d(v, 63);
}
// N sums at once, stage by stage: the same operations in the same order per value as
// wave_reduce<0>, with the independent chains interleaved (one after another they run at the
// latency of the DPP moves).
template <int N>
__device__ __forceinline__ void wave_sums(double v[N])
{
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d0<0x111>(v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d0<0x112>(v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d0<0x114>(v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d0<0x118>(v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d<0x142, 0xa>(0.0, v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] += dpp_d<0x143, 0xc>(0.0, v[d]);
#pragma unroll
    for (int d = 0; d < N; ++d) v[d] = readlane_d(v[d], 63);
}
__device__ __forceinline__ void wave_sum_dots(double v[kNDot]) { wave_sums<kNDot>(v); }
__device__ __forceinline__ double wave_min(double v) { return wave_reduce<1>(v); }
__device__ __forceinline__ double wave_max(double v) { return wave_reduce<2>(v); }

// ------------------------------------------------------------------ cost access
// Dense costs are read with buffer loads through a resource descriptor based at the first
// row of the tile (offsets stay far below 2^31 for any supported n). Each wave issues the
// loads of all of its rows before computing on any of them, so a workgroup keeps
// 4 x 16 rows x 1 KiB of the cost in flight.
constexpr int kBufDword3 = 0x00020000;  // gfx9 buffer descriptor word 3 (32-bit data format)

template <int DT>
struct DenseCost {
    // raw element bytes and per-lane raw type for 4 consecutive columns
    static constexpr int kBytes = (DT == MDOT_DT_F64) ? 8 : (DT == MDOT_DT_F32 ? 4 : 2);
    using Raw = typename std::conditional<DT == MDOT_DT_F64, double4,
                typename std::conditional<DT == MDOT_DT_F32, float4, uint2>::type>::type;
    __amdgpu_buffer_rsrc_t rs;
    int n;
    int odd;  // 16-bit types: 2 when the tile's first row starts in the upper half of a dword
    int end;  // 16-bit types: where the matrix ends, in bytes like at(), if that is inside a dword
    __device__ __forceinline__ DenseCost(const Work& w, int i0) : n(w.n), odd(0), end(0x7fffffff)
    {
        const char* base = (const char*)w.cost + (size_t)i0 * w.n * kBytes;
        size_t rem = ((size_t)w.m - i0) * w.n * kBytes;
        if constexpr (kBytes == 2) {
            // based at the dword that holds the first element and ending with the dword that
            // holds the last one, so that no valid element fails the per-dword range check. The
            // half of that dword behind the last element is not the matrix's: load() clears it.
            odd = (int)((uintptr_t)base & 2);
            base -= odd;
            rem += odd;
            if ((rem & 2) && rem < 0x7ffffff0u) end = (int)rem;
            rem = (rem + 3) & ~(size_t)3;
        }
        rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(rem > 0x7ffffffcu ? 0x7ffffffcu : rem),
                                               kBufDword3);
    }
    __device__ __forceinline__ void cols(int) {}
    // rows r .. r + B - 1 of the tile (global row i0 + r), columns j0..j0+3; columns >= n are masked
    // by the caller, their values are unspecified (or 0 past the end of the matrix), and so are rows
    // past the end. The loads need dword alignment only, which every FP32 and FP64 row and every
    // 16-bit row of even length in a matrix that starts on a dword has; the range check is per dword.
    // Other 16-bit rows read the three dwords around their 8 bytes and shift, all loads of the batch
    // before the first shift (one branch per row instead makes every row wait for its own load). Where
    // a lane's batch reaches past a matrix that ends inside a dword, the half behind the end is cleared
    // first: a padding column, or the row past the last one, would decode it.
    // n = 8191 BF16 sweep: 64.8 us with four 2-byte loads per lane and row, 36.6 us so and 37.7 us with
    // the clearing; 30 us at 8192.
    // FP32 and FP64 rows from `rows` on may be left out.
    template <int B>
    __device__ __forceinline__ void load(int r, int j0, Raw* v, int rows = B) const
    {
        auto at = [&](int u) { return ((r + u) * n + j0) * kBytes + odd; };
        if constexpr (DT == MDOT_DT_F64) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (u >= rows) continue;
                auto a = __builtin_amdgcn_raw_buffer_load_b128(rs, at(u), 0, 0);
                auto b = __builtin_amdgcn_raw_buffer_load_b128(rs, at(u) + 16, 0, 0);
                double2 da = *(double2*)&a, db = *(double2*)&b;
                v[u].x = da.x; v[u].y = da.y; v[u].z = db.x; v[u].w = db.y;
            }
        } else if constexpr (DT == MDOT_DT_F32) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (u >= rows) continue;
                auto a = __builtin_amdgcn_raw_buffer_load_b128(rs, at(u), 0, 0);
                v[u] = *(float4*)&a;
            }
        } else if (((n & 1) | odd) == 0) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                auto a = __builtin_amdgcn_raw_buffer_load_b64(rs, at(u), 0, 0);
                v[u] = *(uint2*)&a;
            }
        } else {
            uint32_t d[B][3];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                auto a = __builtin_amdgcn_raw_buffer_load_b96(rs, at(u) & ~3, 0, 0);
                d[u][0] = a[0]; d[u][1] = a[1]; d[u][2] = a[2];
            }
            if (at(B - 1) + 8 > end) {
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if ((at(u) & ~3) + 4 * k + 2 == end) d[u][k] &= 0xffffu;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const uint32_t sh = (uint32_t)(at(u) & 2) * 8;
                v[u].x = __builtin_amdgcn_alignbit(d[u][1], d[u][0], sh);
                v[u].y = __builtin_amdgcn_alignbit(d[u][2], d[u][1], sh);
            }
        }
    }
    // Direct-to-LDS load of row r (FP32, n % 4 == 0): lane l's 16 bytes land at lds + 16 l.
    __device__ __forceinline__ void stage(int r, int j0, void* lds) const
    {
        static_assert(DT == MDOT_DT_F32, "staging is for FP32 rows");
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16,
                                                 (r * n + j0) * kBytes, 0, 0, 0);
    }
    __device__ __forceinline__ void decode(const Raw& v, double c[4]) const
    {
        if constexpr (DT == MDOT_DT_F64) {
            c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
        } else if constexpr (DT == MDOT_DT_F32) {
            c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
        } else if constexpr (DT == MDOT_DT_F16) {
            c[0] = __half2float(__ushort_as_half((unsigned short)(v.x & 0xffffu)));
            c[1] = __half2float(__ushort_as_half((unsigned short)(v.x >> 16)));
            c[2] = __half2float(__ushort_as_half((unsigned short)(v.y & 0xffffu)));
            c[3] = __half2float(__ushort_as_half((unsigned short)(v.y >> 16)));
        } else {  // BF16: the high half of an FP32
            c[0] = __uint_as_float(v.x << 16); c[1] = __uint_as_float(v.x & 0xffff0000u);
            c[2] = __uint_as_float(v.y << 16); c[3] = __uint_as_float(v.y & 0xffff0000u);
        }
    }
    __device__ __forceinline__ void row(int r, int j0, double c[4]) const
    {
        Raw v;
        load<1>(r, j0, &v);
        decode(v, c);
    }
    // LSE exponent arguments (log2 units) of one row for this lane's 4 columns:
    // x_k = -g2 C_ik + V_k + A, with g2 = gamma * scale * log2(e).
    __device__ __forceinline__ void bind_rows(void*, void*) {}
    __device__ __forceinline__ void row_setup(int, int, double, double&) {}
    __device__ __forceinline__ void prepare(double, const double*) {}
    __device__ __forceinline__ double row_fixed(int, int) { return 0.0; }
    static __device__ __forceinline__ double row_term(double, double, double a) { return a; }
    __device__ __forceinline__ void cols_fixed(double) {}
    __device__ __forceinline__ void bind_cols(double, const double*) {}
    __device__ __forceinline__ void args(const Raw& raw, double g2, const double V[4], double A, double x[4]) const
    {
        double c[4];
        decode(raw, c);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = fma(-g2, c[k], V[k]) + A;
    }
};

// Point clouds: raw C_ij = sum_k (x_ik - y_jk)^2 (KIND 1) or sum_k |x_ik - y_jk| (KIND 2),
// evaluated in FP64 from FP32 coordinates (d <= 8). In the LSE tile the rows' coordinates are
// the same for every lane: row_setup() puts them in LDS once and "Raw" is just the tile row.
// D is the number of coordinates the arithmetic carries: D = 3 serves every d <= 3, D = 2
// (planar clouds, d <= 2) leaves out the third coordinate's operations, D = 8 serves 4 <= d <= 8.
// Coordinates past d are zero, so every term a smaller D leaves out is an exact zero and the
// instances give identical results on a cloud padded with zero coordinates.
template <int KIND, int D = 3>
struct PointCost {
    static_assert(D == 2 || D == 3 || D == 8, "point instances carry 2, 3 or 8 coordinates");
    static constexpr int kRowF = D <= 4 ? 4 : 8;  // coordinates per row held for the loop
    // Up to 3 coordinates the tile's rows are kept in LDS as FP64 (the FP32 values converted
    // once per row at set-up, exactly), so the loop reads them without a conversion per row and
    // lane; 8-coordinate rows stay FP32 (two float4), as FP64 they would not fit the LDS.
    static constexpr bool kRowF64 = D <= 3;
    using RowT = typename std::conditional<kRowF64, double, float>::type;
    using Raw = int;
    const float* X;
    const float* Y;
    int m, n, d, i0;
    double y[4][D];
    const void* sX;   // row coordinates 0..3 (float4), or 0..1 (double2) (LDS)
    const void* sX2;  // coordinates 4..7 (float4, D = 8), or 2 (double, D = 3)
    __device__ __forceinline__ PointCost(const Work& w, int i0_)
        : X((const float*)w.cost), Y((const float*)w.cost + (size_t)w.m * w.d), m(w.m), n(w.n), d(w.d), i0(i0_) {}
    __device__ __forceinline__ void cols(int j0)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < D; ++e) y[k][e] = (j0 + k < n && e < d) ? (double)Y[(size_t)(j0 + k) * d + e] : 0.0;
    }
    struct RowX {
        RowT v[kRowF];
    };
    __device__ __forceinline__ RowX xrow(int r) const
    {
        const int i = i0 + r;
        RowX x;
#pragma unroll
        for (int e = 0; e < kRowF; ++e) x.v[e] = (RowT)((e < D && i < m && e < d) ? X[(size_t)i * d + e] : 0.f);
        return x;
    }
    __device__ __forceinline__ void decode(const RowX& x, double c[4]) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < D; ++e) {
                double t = (double)x.v[e] - y[k][e];
                s = (KIND == 1) ? fma(t, t, s) : s + fabs(t);
            }
            c[k] = s;
        }
    }
    __device__ __forceinline__ void row(int r, int, double c[4]) const { decode(xrow(r), c); }
    template <int B>
    __device__ __forceinline__ void load(int r, int, Raw* v, int = B) const
    {
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = r + u;
    }
    // LSE tile set-up: sX (and sX2 for D = 8) = kBR float4 rows of LDS; thread r < kBR stores row
    // r's coordinates and, for squared distances, folds -g2 |x_r|^2 into the row term a.
    __device__ __forceinline__ void bind_rows(void* lds, void* lds_hi)
    {
        sX = lds;
        sX2 = lds_hi;
    }
    __device__ __forceinline__ void row_setup(int r, int i, double g2, double& a)
    {
        const RowX v = xrow(r);
        if constexpr (kRowF64) {
            ((double2*)sX)[r] = make_double2(v.v[0], v.v[1]);
            if constexpr (D == 3) ((double*)sX2)[r] = v.v[2];
        } else {
            ((float4*)sX)[r] = make_float4(v.v[0], v.v[1], v.v[2], v.v[3]);
            if constexpr (kRowF == 8) ((float4*)sX2)[r] = make_float4(v.v[4], v.v[5], v.v[6], v.v[7]);
        }
        if (KIND == 1 && i < m) {
            double ss;
            if constexpr (D > 2) {
                ss = (double)v.v[D - 1] * (double)v.v[D - 1];
#pragma unroll
                for (int e = D - 2; e >= 0; --e) ss = fma((double)v.v[e], (double)v.v[e], ss);
            } else {
                ss = 0.0;
#pragma unroll
                for (int e = D - 1; e >= 0; --e) ss = fma((double)v.v[e], (double)v.v[e], ss);
            }
            a = fma(-g2, ss, a);
        }
    }
    // LSE exponent arguments, as DenseCost::args. For squared distances the expansion
    // |x - y|^2 = |x|^2 + |y|^2 - 2 <x, y> moves |y_k|^2 into W_k = V_k - g2 |y_k|^2 and |x|^2 into
    // the row term, leaving D FMAs per element (prepare() turns y into 2 g2 y). The large
    // terms cancel in FP64 to an absolute error ~1e-16 g2 |x|^2, far below the FP32 exp error.
    double W[4];
    __device__ __forceinline__ void prepare(double g2, const double V[4])
    {
        if constexpr (KIND == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                double yy = D > 2 ? y[k][D - 1] * y[k][D - 1] : 0.0;
#pragma unroll
                for (int e = (D > 2 ? D - 2 : D - 1); e >= 0; --e) yy = fma(y[k][e], y[k][e], yy);
                W[k] = fma(-g2, yy, V[k]);
#pragma unroll
                for (int e = 0; e < D; ++e) y[k][e] *= 2.0 * g2;
            }
        }
    }
    // The same in parts, for a kernel that runs many sweeps at one g2: the row's coordinates and
    // |x_r|^2 (0 for L1), the scaled columns and |y_k|^2, and the step's own terms.
    double YY[4];
    __device__ __forceinline__ double row_fixed(int r, int i)
    {
        double a = 0.0;
        row_setup(r, i, -1.0, a);  // fma(1, |x|^2, 0)
        return a;
    }
    static __device__ __forceinline__ double row_term(double g2, double xx, double a) { return KIND == 1 ? fma(-g2, xx, a) : a; }
    __device__ __forceinline__ void cols_fixed(double g2)
    {
        const double zero[4] = {0.0, 0.0, 0.0, 0.0};
        if constexpr (KIND == 1) {
            prepare(-1.0, zero);  // W = |y|^2, y <- -2 y
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                YY[k] = W[k];
#pragma unroll
                for (int e = 0; e < D; ++e) y[k][e] *= -g2;  // exactly 2 g2 y: both factors of 2 are exact
            }
        }
    }
    __device__ __forceinline__ void bind_cols(double g2, const double V[4])
    {
        if constexpr (KIND == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) W[k] = fma(-g2, YY[k], V[k]);
        }
    }
    __device__ __forceinline__ RowX lds_row(int r) const
    {
        RowX x;  // one address for the whole wave: LDS broadcasts
        if constexpr (kRowF64) {
            const double2 a = ((const double2*)sX)[r];
            x.v[0] = a.x; x.v[1] = a.y; x.v[2] = D == 3 ? ((const double*)sX2)[r] : 0.0; x.v[3] = 0.0;
        } else {
            const float4 a = ((const float4*)sX)[r];
            x.v[0] = a.x; x.v[1] = a.y; x.v[2] = a.z; x.v[3] = a.w;
            if constexpr (kRowF == 8) {
                const float4 b = ((const float4*)sX2)[r];
                x.v[4] = b.x; x.v[5] = b.y; x.v[6] = b.z; x.v[7] = b.w;
            }
        }
        return x;
    }
    __device__ __forceinline__ void args(const Raw& r, double g2, const double V[4], double A, double x[4]) const
    {
        const RowX xr = lds_row(r);
        if constexpr (KIND == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                double acc = W[k] + A;
#pragma unroll
                for (int e = D - 1; e >= 0; --e) acc = fma((double)xr.v[e], y[k][e], acc);
                x[k] = acc;
            }
        } else {
            double c[4];
            decode(xr, c);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = fma(-g2, c[k], V[k]) + A;
        }
    }
};

// ------------------------------------------------------------------ tile bodies
struct TileCtx {
    int I, J, i0, j0lane, lane, wave, tid;
};

__device__ __forceinline__ TileCtx tile_ctx(const Work& w, int blk)
{
    TileCtx t;
    t.tid = threadIdx.x;
    t.lane = t.tid & 63;
    t.wave = t.tid >> 6;
    t.I = blk / w.nct;
    t.J = blk % w.nct;
    t.i0 = t.I * kBR;
    t.j0lane = t.J * kBC + t.lane * 4;
    return t;
}

// Scalars a kernel needs from the state: the trial and the pending vector update.
struct SweepArgs {
    double alpha, gamma, gamma_prev;
    double alpha_acc, beta, w, ws_ratio, ws_scale;
    int va, reset, stage;
};

__device__ __forceinline__ SweepArgs args_of(const State* S)
{
    SweepArgs a;
    const int mode = S->sweep_mode, ph = S->ls_phase;
    const double alpha = S->alpha;  // read unconditionally: no branch between the state reads
    a.alpha = ((mode == SM_LSE) & ((ph == LS_TRIAL) | (ph == LS_FORCE) | (ph == LS_SINK))) ? alpha : 0.0;
    a.gamma = S->gamma;
    a.gamma_prev = S->gamma_prev;
    a.alpha_acc = S->alpha_acc;
    a.beta = S->beta;
    a.w = S->w;
    a.ws_ratio = S->ws_ratio;
    a.ws_scale = S->ws_scale;
    a.va = S->vec_action;
    a.reset = S->reset;
    a.stage = S->stage;
    return a;
}

// Entry k of the (m + n)-vectors (rows then columns) after the pending vector update:
//   accept : (u, v) += alpha p, log r(P) <- trial log-sums, p <- d + beta p or d (Alg. 2), with
//            d the Sinkhorn direction s or (precond variant) the stored s~, restricted to the
//            rows or the columns for the Sinkhorn projector's half-steps (Alg. 4)
//   stage  : smoothed marginals (Alg. 1), rank-1 start (stage 1) or warm start
//            z' = scale z + ratio (z - z_prev): eq. (approx-znext) with scale = 1, the
//            epsilon-scaling start (Sec. 4.2.1) with ratio = 0; p = 0, shifts = log r~.
// zacc is z after the accept and before the stage start (the stage's solution).
struct Entry {
    double z, zacc, p, lz, logt, rt, zprev;
};

// The direction entry of an accepted step (see ResetBits).
__device__ __forceinline__ double next_dir(const SweepArgs& a, double p, double logt, double lz, double sdt, bool row)
{
    const double sdir = (a.reset & RS_TILDE) ? sdt : logt - lz;  // eq. (s-tilde) / eq. (sinkhorn-direction)
    double pn = (a.reset & RS_RESET) ? sdir : fma(a.beta, p, sdir);
    if (((a.reset & RS_ROWS) && !row) || ((a.reset & RS_COLS) && row)) pn = 0.0;
    return pn;
}

__device__ __forceinline__ Entry entry_after(const Work& w, const SweepArgs& a, int k)
{
    Entry e;
    e.z = w.z[k];
    e.p = w.p[k];
    e.lz = w.lz[k];
    e.logt = w.logt[k];
    e.rt = w.rt[k];
    e.zprev = w.zprev[k];
    if (a.va & VA_ACCEPT) {
        e.z = fma(a.alpha_acc, e.p, e.z);
        e.lz = w.lzt[k];
        const double sdt = (a.reset & RS_TILDE) ? w.sdt[k] : 0.0;
        e.p = next_dir(a, e.p, e.logt, e.lz, sdt, k < w.m);
    }
    e.zacc = e.z;
    if (a.va & VA_STAGE_INIT) {
        const bool row = k < w.m;
        const double mk = row ? w.r[k] : w.c[k - w.m];
        e.rt = fma(1.0 - a.w, mk, a.w / (row ? w.m : w.n));  // smoothed toward the uniform law of the side
        e.logt = log(e.rt);
        if (a.stage == 1) {
            e.z = e.logt;
            e.zprev = e.logt;  // z^0 at gamma^0 = 0
        } else {
            const double zp = e.zprev;
            e.zprev = e.z;
            e.z = fma(a.ws_ratio, e.z - zp, a.ws_scale * e.z);
        }
        e.p = 0.0;
        e.lz = e.logt;
    }
    return e;
}

// Round row factor x_i = r_i / r(P)_i ^ 1 (Alg. 3), with r(P)_i = 0 giving 1.
__device__ __forceinline__ double round_x(double ri, double lz)
{
    const double rp = exp(lz);
    return (rp > 0.0) ? fmin(ri / rp, 1.0) : 1.0;
}

// One Horner step a * x + c with the coefficient c in an SGPR pair: left to itself the
// compiler holds every polynomial coefficient of exp2_f64 in a VGPR pair across the sweep loops.
__device__ __forceinline__ double fma_sc(double a, double x, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(x), "s"(c));
    return r;
}

// 2^x in FP64 for the sweeps' exponent arguments. x is clamped to [-1022, 1000], split as
// x = k + f with k = round-to-nearest(x) by the 1.5 * 2^52 shift (its low word is k) and
// |f| <= 1/2; 2^f = 1 + f q(f) with q of degree 9, a weighted least-squares fit driven to equal
// ripple (relative error below 4e-16 in exact arithmetic, a few ulp after Horner rounding).
// 2^f lies in [0.707, 1.414], so 2^k is applied by adding k to its exponent field: exact for
// normal results, and at the clamp -1022 (which x = -inf meets) the result is a positive
// subnormal or 2^-1022, below any sum the sweeps accept. No range branches: 16 VALU
// operations. c9 is q's leading coefficient (kExp2C9), which the caller keeps in a VGPR.
constexpr double kExp2C9 = 0x1.e3a9131404cdep-28;
__device__ __forceinline__ double exp2_f64(double x, double c9)
{
    constexpr double kShift = 0x1.8p52;
    x = fmin(fmax(x, -1022.0), 1000.0);
    const double y = x + kShift;
    const double f = x - (y - kShift);
    const uint32_t k = (uint32_t)__builtin_bit_cast(uint64_t, y);
    double q = fma_sc(f, c9, 0x1.b671b6a900f80p-24);
    q = fma_sc(q, f, 0x1.62c147a08947dp-20);
    q = fma_sc(q, f, 0x1.ffcb58c5cff22p-17);
    q = fma_sc(q, f, 0x1.4309126bff6b0p-13);
    q = fma_sc(q, f, 0x1.5d87fe9b90bb4p-10);
    q = fma_sc(q, f, 0x1.3b2ab6fbd6d27p-7);
    q = fma_sc(q, f, 0x1.c6b08d703e16ap-5);
    q = fma_sc(q, f, 0x1.ebfbdff82c431p-3);
    q = fma_sc(q, f, 0x1.62e42fefa3a12p-1);
    const double p = fma(q, f, 1.0);
    return __hiloint2double(__double2hiint(p) + (int)(k << 20), __double2loint(p));
}

// Four Horner steps q_k = q_k f_k + c of independent exponentials in one block (one SGPR
// coefficient): the steps of the four chains stay interleaved, so no step waits on the one
// before it.
__device__ __forceinline__ void fma4_sc(double q[4], const double f[4], double c)
{
    double r0, r1, r2, r3;
    asm("v_fma_f64 %0, %4, %8, %12\n\t"
        "v_fma_f64 %1, %5, %9, %12\n\t"
        "v_fma_f64 %2, %6, %10, %12\n\t"
        "v_fma_f64 %3, %7, %11, %12"
        : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
        : "v"(q[0]), "v"(q[1]), "v"(q[2]), "v"(q[3]), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "s"(c));
    q[0] = r0; q[1] = r1; q[2] = r2; q[3] = r3;
}

// exp2_f64 of four arguments at once (the same operations in the same order per value; exp2_f64 itself
// is what the CPU test of the coefficients reads).
__device__ __forceinline__ void exp2_f64x4(const double x[4], double e[4], double c9)
{
    constexpr double kShift = 0x1.8p52;
    double f[4], q[4];
    uint32_t k[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double xc = fmin(fmax(x[i], -1022.0), 1000.0);
        const double y = xc + kShift;
        f[i] = xc - (y - kShift);
        k[i] = (uint32_t)__builtin_bit_cast(uint64_t, y);
        q[i] = c9;
    }
    fma4_sc(q, f, 0x1.b671b6a900f80p-24);
    fma4_sc(q, f, 0x1.62c147a08947dp-20);
    fma4_sc(q, f, 0x1.ffcb58c5cff22p-17);
    fma4_sc(q, f, 0x1.4309126bff6b0p-13);
    fma4_sc(q, f, 0x1.5d87fe9b90bb4p-10);
    fma4_sc(q, f, 0x1.3b2ab6fbd6d27p-7);
    fma4_sc(q, f, 0x1.c6b08d703e16ap-5);
    fma4_sc(q, f, 0x1.ebfbdff82c431p-3);
    fma4_sc(q, f, 0x1.62e42fefa3a12p-1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double p = fma(q[i], f[i], 1.0);
        e[i] = __hiloint2double(__double2hiint(p) + (int)(k[i] << 20), __double2loint(p));
    }
}

// Column combine: per-wave column values (4 per lane) -> one value per column of the tile.
__device__ __forceinline__ void col_combine_store(double* sbuf, const double v[4], const TileCtx& t, int op,
                                                  double* dst, int n, int jt0)
{
    // sbuf: [4 waves][kBC]
#pragma unroll
    for (int k = 0; k < 4; ++k) sbuf[t.wave * kBC + t.lane * 4 + k] = v[k];
    __syncthreads();
    {
        const int col = t.tid;  // kWG == kBC
        double a = sbuf[col], b = sbuf[kBC + col], c = sbuf[2 * kBC + col], d = sbuf[3 * kBC + col];
        double r = (op == 0) ? ((a + b) + (c + d)) : (op == 1 ? fmin(fmin(a, b), fmin(c, d)) : fmax(fmax(a, b), fmax(c, d)));
        if (jt0 + col < n) dst[jt0 + col] = r;
    }
    __syncthreads();
}

// As col_combine_store, with wave w's values at sbuf + w * stride.
__device__ __forceinline__ void col_combine_store_strided(double* sbuf, int stride, const double v[4], const TileCtx& t,
                                                          double* dst, int n, int jt0)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) sbuf[t.wave * stride + t.lane * 4 + k] = v[k];
    __syncthreads();
    const int col = t.tid;  // kWG == kBC
    const double a = sbuf[col], b = sbuf[stride + col], c = sbuf[2 * stride + col], d = sbuf[3 * stride + col];
    if (jt0 + col < n) dst[jt0 + col] = (a + b) + (c + d);
    __syncthreads();
}

// LDS of one sweep workgroup: five per-row arrays, the per-wave column buffer, and the
// per-wave row-partial transpose buffer (kRPW rows x 64 lanes, padded to 65, FP32).
constexpr int kRowPad = 65;
// The LSE tile lays its LDS out as: five per-row arrays (5 kBR doubles), the column values
// (kBC doubles), then one region per wave (kWaveRegion doubles) that first receives the wave's
// second batch of cost rows by direct-to-LDS loads and then, once the wave has read them, holds
// its row-partial transpose buffer and its slice of the column combine. The other tile kinds
// use the first 5 kBR + 4 kBC doubles.
constexpr int kWaveRegion = 1024;                        // 8 KiB: 8 rows x 64 lanes x 16 B
constexpr int kRowBufD = (kRPW * kRowPad + 1) / 2;      // transpose buffer, in doubles
static_assert(kRowBufD + kBC <= kWaveRegion, "wave region too small");
constexpr int kSmem = 5 * kBR + kBC + 4 * kWaveRegion;
constexpr int kSmemAll = kSmem + 2 * kBR;  // plus the upper coordinates of 8-D point rows
static_assert(kSmem >= 5 * kBR + 4 * kBC, "LDS for the Round tiles");

// Sum the per-lane FP32 row partials rp[r] of the wave's kRPW rows across the 64 lanes:
// a transpose through LDS, then 4 lanes per row each sum 16 values in FP64 and combine.
// Returns the row total in the lane with (lane & 3) == 0 of row lane >> 2.
__device__ __forceinline__ double rows_reduce_f32(const float rp[kRPW], float* rb, int lane)
{
#pragma unroll
    for (int r = 0; r < kRPW; ++r) rb[r * kRowPad + lane] = rp[r];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int rr = lane >> 2, q = lane & 3;
    const float* src = rb + rr * kRowPad + q * 16;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += (double)src[k];
    s += dpp_d<0xb1>(0.0, s);  // quad_perm [1,0,3,2]
    s += dpp_d<0x4e>(0.0, s);  // quad_perm [2,3,0,1]
    return s;
}

// The same for FP64 row partials, which the caller has stored as rb[r * 64 + lane] (the wave's
// kRPW x 64 values fill its region); lane (rr, q) walks its 16 entries in the order k ^ rr, so
// that the lanes of each read hit distinct banks.
__device__ __forceinline__ double rows_reduce_f64(const double* rb, int lane)
{
    static_assert(kRPW * 64 <= kWaveRegion, "FP64 row transpose fits the wave region");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int rr = lane >> 2, q = lane & 3;
    const double* src = rb + rr * 64 + q * 16;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += src[k ^ rr];
    s += dpp_d<0xb1>(0.0, s);  // quad_perm [1,0,3,2]
    s += dpp_d<0x4e>(0.0, s);  // quad_perm [2,3,0,1]
    return s;
}

// Smallest and largest raw entry seen, in the type T the entries are exact in, and whether a
// non-finite one was.
template <class T>
struct RawRange {
    T lo = INFINITY, hi = -INFINITY;
    bool bad = false;
    __device__ __forceinline__ void add(T c)
    {
        bad |= !isfinite(c);
        lo = lo < c ? lo : c;
        hi = hi > c ? hi : c;
    }
    // the first `cols` of a lane's four consecutive columns
    __device__ __forceinline__ void add4(const double c[4], int cols)
    {
        if (cols >= 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) add((T)c[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < cols) add((T)c[k]);
        }
    }
};
// FP32 holds every FP32, FP16 and BF16 entry exactly
template <class Cost>
using RangeOf = RawRange<typename std::conditional<sizeof(typename Cost::Raw) <= 16 && !std::is_same<typename Cost::Raw, int>::value,
                                                   float, double>::type>;

// The first `rows` rows of a batch, kept apart from the exponentials that follow: interleaved with
// them it takes more registers than there are.
template <class Cost, int RB>
__device__ __forceinline__ void range_rows(RangeOf<Cost>& range, const Cost& cost, const typename Cost::Raw* raw, int rows,
                                           int cols)
{
#pragma unroll
    for (int r = 0; r < RB; ++r)
        if (r < rows) {
            double c[4];
            cost.decode(raw[r], c);
            range.add4(c, cols);
        }
    __builtin_amdgcn_sched_barrier(0);
}

// The fused LSE tile (the hot loop of every line-search trial):
//   e_ij = exp(X_ij - s_i),  row partial sum_j e_ij,  column partial sum_i w_i e_ij,
// with w_i = exp(s_i - S_I). Exponent argument in FP64 (log2 units), exp2 in FP32 (E64 =
// false) or FP64 (E64 = true). RANGE (dense costs) adds the tile's raw entries to `range`.
template <class Cost, bool E64, bool RANGE = false>
__device__ void tile_lse(const Work& w, const SweepArgs& S, const TileCtx& t, double* sm, RangeOf<Cost>* range = nullptr)
{
    double* sA = sm;
    double* sWt = sm + kBR;
    double* sS = sm + 2 * kBR;
    double* sColV = sm + 5 * kBR;
    double* region = sm + 5 * kBR + kBC;                   // the kWaveRegion per-wave regions
    double* myRegion = region + t.wave * kWaveRegion;
    float* sRow = (float*)myRegion;                         // after the staged rows are read
    double* sColSlices = region + kRowBufD;                 // wave w's slice at + w kWaveRegion
    const int m = w.m, n = w.n;
    const double alpha = S.alpha;
    const double g2 = S.gamma * w.scale * LOG2E_D;
    const int j0 = t.j0lane;
    Cost cost(w, t.i0);
    cost.cols(j0);
    const int rbase = t.wave * kRPW;
    const int nrows = min(kRPW, m - (t.i0 + rbase));  // rows of this wave (may be <= 0)
    // loads of a batch of rows are issued before any compute on them (all 16 rows of the wave
    // for <= 8 B per lane-row, 8 rows for 16 B, 4 for 32 B); the first batch does not depend on the
    // solver state and is issued before the per-row and per-column set-up, which it overlaps
    constexpr int RB = sizeof(typename Cost::Raw) <= 8 ? kRPW : (sizeof(typename Cost::Raw) <= 16 ? kRPW / 2 : kRPW / 4);
    // FP32 exponentials with rows of at most 16 B: rows past the end of the matrix are loaded
    // too (the buffer range check returns 0 for them) and computed without a branch. Their row
    // term is -inf, so every exponential of theirs is exactly 0, and one straight-line loop
    // over the batch lets the compiler overlap one row's exponentials with the next row's
    // arguments. Elsewhere (FP64 exponentials, 32 B rows) that overlap costs more registers
    // than there are, and each row stays behind its own branch.
    constexpr bool kRowGuard = E64 || sizeof(typename Cost::Raw) > 16;
    typename Cost::Raw raw[RB];
    cost.template load<RB>(rbase, j0, raw, kRowGuard ? nrows : RB);
    // FP32 rows with n % 4 == 0 and more tiles than stay resident at once: the second batch
    // goes straight to the wave's LDS region, so all 16 rows of the wave are in flight from the
    // start without holding registers. With a single round of workgroups (n <= ~5800) the
    // extra requests only delay the first batch, so it is not used there.
    constexpr bool kCanStage = std::is_same<Cost, DenseCost<MDOT_DT_F32>>::value && RB < kRPW;
    bool staged = false;
    if constexpr (kCanStage) {
        staged = (n & 3) == 0 && w.nrt * w.nct > w.stage_min_tiles;
        if (staged) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (RB + r < nrows) cost.stage(rbase + RB + r, j0, myRegion + r * (kWaveRegion / RB));
        }
    }
    // per-row values: shift s_i (predicted log row sum) and A_i = (u_i - lz_i) log2 e;
    // per-column V_j = (v_j + alpha p_j) log2 e, one column per thread, through LDS
    cost.bind_rows(sm + 3 * kBR, sm + kSmem);  // 2 kBR doubles, free in this tile, and 2 kBR past the rest
    if (t.tid < kBR) {
        const int i = t.i0 + t.tid;
        double sh = -INFINITY, aa = -INFINITY;
        if (i < m) {
            const Entry e = entry_after(w, S, i);
            sh = fma(alpha, e.p, e.lz);
            aa = (e.z - e.lz) * LOG2E_D;
        }
        cost.row_setup(t.tid, i, g2, aa);
        sS[t.tid] = sh;
        sA[t.tid] = aa;
    }
    {
        const int j = t.J * kBC + t.tid;
        double vv = 0.0;
        if (j < n) {
            const Entry e = entry_after(w, S, m + j);
            vv = fma(alpha, e.p, e.z) * LOG2E_D;
        }
        sColV[t.tid] = vv;
    }
    __syncthreads();
    const double SI = wave_max(sS[t.lane]);  // S_I = max_i s_i over the kBR (= 64) rows
    if (t.tid < kBR) sWt[t.tid] = exp(sS[t.tid] - SI);
    // padding columns (j >= n) get V = -inf: their arguments are -inf and their exponentials 0
    double V[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) V[k] = (j0 + k < n) ? sColV[t.lane * 4 + k] : -INFINITY;
    __syncthreads();
    cost.prepare(g2, V);

    double col64[4] = {0, 0, 0, 0};
    if constexpr (!E64) {
        float col32[4] = {0, 0, 0, 0};
        float rp[kRPW];
#pragma unroll
        for (int b = 0; b < kRPW; b += RB) {
            if (b > 0) {
                if constexpr (kCanStage) {
                    if (staged) {
                        __builtin_amdgcn_s_waitcnt(0);  // the wave's direct-to-LDS loads have landed
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int r = 0; r < RB; ++r)
                            raw[r] = (b + r < nrows)
                                ? reinterpret_cast<const typename Cost::Raw*>(myRegion + r * (kWaveRegion / RB))[t.lane]
                                : typename Cost::Raw{};
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                if (!staged) cost.template load<RB>(rbase + b, j0, raw, kRowGuard ? nrows - b : RB);
            }
            if constexpr (RANGE) range_rows<Cost, RB>(*range, cost, raw, nrows - b, n - j0);
#pragma unroll
            for (int r0 = 0; r0 < RB; ++r0) {
                const int r = b + r0;
                rp[r] = 0.f;
                if (!kRowGuard || r < nrows) {
                    double xa[4];
                    cost.args(raw[r0], g2, V, sA[rbase + r], xa);
                    const float wt = (float)sWt[rbase + r];
                    float e[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) e[k] = __builtin_amdgcn_exp2f((float)xa[k]);
                    rp[r] = (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) col32[k] = fmaf(wt, e[k], col32[k]);
                }
                if ((r & 7) == 7) {  // FP32 column sums over at most 8 rows, then FP64
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        col64[k] += (double)col32[k];
                        col32[k] = 0.f;
                    }
                }
            }
        }
        const double rs = rows_reduce_f32(rp, sRow, t.lane);
        const int rr = t.lane >> 2;
        if ((t.lane & 3) == 0 && rr < nrows) w.rowpart[(size_t)t.J * m + t.i0 + rbase + rr] = rs;
    } else {
        double rp[kRPW];
        double c9 = kExp2C9;
        asm volatile("" : "+v"(c9));  // one VGPR pair for the whole tile instead of a move per exp
#pragma unroll
        for (int b = 0; b < kRPW; b += RB) {
            if (b > 0) {
                if constexpr (kCanStage) {
                    if (staged) {
                        __builtin_amdgcn_s_waitcnt(0);  // the wave's direct-to-LDS loads have landed
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int r = 0; r < RB; ++r)
                            raw[r] = (b + r < nrows)
                                ? reinterpret_cast<const typename Cost::Raw*>(myRegion + r * (kWaveRegion / RB))[t.lane]
                                : typename Cost::Raw{};
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                if (!staged) cost.template load<RB>(rbase + b, j0, raw, kRowGuard ? nrows - b : RB);
                // the region no longer holds staged rows: park the previous batch's partials
                // (the compiler barrier keeps these FP64 stores after the float4 reads above)
                asm volatile("" ::: "memory");
#pragma unroll
                for (int r = b - RB; r < b; ++r) myRegion[r * 64 + t.lane] = rp[r];
            }
            if constexpr (RANGE) range_rows<Cost, RB>(*range, cost, raw, nrows - b, n - j0);
#pragma unroll
            for (int r0 = 0; r0 < RB; ++r0) {
                const int r = b + r0;
                rp[r] = 0.0;
                if (r < nrows) {  // kRowGuard holds on this path
                    double xa[4];
                    cost.args(raw[r0], g2, V, sA[rbase + r], xa);
                    const double wt = sWt[rbase + r];
                    double e[4];
                    exp2_f64x4(xa, e, c9);
                    rp[r] = (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) col64[k] = fma(wt, e[k], col64[k]);
                }
            }
        }
#pragma unroll
        for (int r = kRPW - RB; r < kRPW; ++r) myRegion[r * 64 + t.lane] = rp[r];
        const double rs = rows_reduce_f64(myRegion, t.lane);
        const int rr = t.lane >> 2;
        if ((t.lane & 3) == 0 && rr < nrows) w.rowpart[(size_t)t.J * m + t.i0 + rbase + rr] = rs;
    }
    col_combine_store_strided(sColSlices, kWaveRegion, col64, t, w.colpart + (size_t)t.I * n, n, t.J * kBC);
    // every tile of row block I writes the same S_I, so the finalizer of any column block
    // reads it from one of the tiles it waited for
    if (t.tid == 0) w.tshift[t.I] = SI;
}

// Row reductions of the Round tiles. A wave leaves B rows of NS sums, then NM minima, per lane in
// its LDS region (slot (quantity * B + row) at kRoundPad apart) and reduces them all at once, four
// lanes per slot: one write and about three operations per row and quantity, where a reduction
// across the lanes of each by itself takes 18. The sums are added in the same balanced tree over
// the lanes as wave_reduce<0>. Returns slot (lane >> 2)'s value in all four of its lanes. With the rows'
// loads issued four rows ahead as well, n = 4096 FP32: R1 41 -> 32 us, R2 47 -> 42.5 us. (With the
// column values in registers, at 166 VGPRs and three waves per SIMD, R1 33.5 and R2 38 us, but the LSE
// path shares the kernel and needs four.)
constexpr int kRoundPad = 65;       // doubles: the four lanes' reads of 16 slots hit distinct banks
constexpr int kRoundSlots = 10;     // per wave
constexpr int kRoundRegion = kRoundSlots * kRoundPad;
// The Round tiles lay their LDS out as five per-row arrays, five per-column arrays (a lane reads its
// four columns' values of a row when it needs them: in registers, with those of the other arrays, they
// do not fit the cap) and the waves' regions.
constexpr int kRoundAt = 5 * kBR + 5 * kBC;
static_assert(kRoundAt + 4 * kRoundRegion <= kSmemAll, "LDS for the Round tiles");
template <int NS, int NM, int B>
__device__ __forceinline__ double round_reduce(const double* region, int lane)
{
    static_assert((NS + NM) * B <= kRoundSlots, "one slot per row and quantity");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int slot = min(lane >> 2, (NS + NM) * B - 1);
    const double* src = region + slot * kRoundPad + (lane & 3) * 16;
    const bool sum = slot < NS * B;
    double v[16], r;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = src[k];
    // lanes of sums and of minima in turn: both for every lane and a choice between them is 96 more
    // instructions
    if (NS > 0 && sum) {
#pragma unroll
        for (int w = 1; w < 16; w *= 2)
#pragma unroll
            for (int k = 0; k < 16; k += 2 * w) v[k] += v[k + w];
        r = v[0];
        r += dpp_d<0xb1>(0.0, r);  // quad_perm [1,0,3,2]
        r += dpp_d<0x4e>(0.0, r);  // quad_perm [2,3,0,1]
    } else {
#pragma unroll
        for (int w = 1; w < 16; w *= 2)
#pragma unroll
            for (int k = 0; k < 16; k += 2 * w) v[k] = fmin(v[k], v[k + w]);
        r = v[0];
        r = fmin(r, dpp_d<0xb1>(0.0, r));
        r = fmin(r, dpp_d<0x4e>(0.0, r));
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return r;
}

// The exponentials of one row's four entries (log2 arguments).
template <bool E64>
__device__ __forceinline__ void exp2x4(const double x[4], double e[4])
{
    if constexpr (E64) {
        exp2_f64x4(x, e, kExp2C9);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = (double)__builtin_amdgcn_exp2f((float)x[k]);
    }
}

// The four consecutive per-column values of a lane.
__device__ __forceinline__ void cols4(const double* col, int lane, double v[4])
{
    const double2 a = ((const double2*)col)[2 * lane], b = ((const double2*)col)[2 * lane + 1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}

// Rows of a Round tile, B at a time, the next B being loaded meanwhile (points: read when needed).
template <class Cost, int B>
struct RoundRows {
    typename Cost::Raw raw[B], next[B];
    static constexpr bool kPoints = std::is_same<typename Cost::Raw, int>::value;
    __device__ __forceinline__ void ask(const Cost& cost, int r, int j0)
    {
        if constexpr (!kPoints) {
            cost.template load<B>(r, j0, next);
        }
    }
    __device__ __forceinline__ void take(const Cost& cost, int r, int j0)
    {
        if constexpr (!kPoints) {
#pragma unroll
            for (int u = 0; u < B; ++u) raw[u] = next[u];
            ask(cost, r + B, j0);
        }
    }
    __device__ __forceinline__ void get(const Cost& cost, int r, int j0, int u, double c[4]) const
    {
        if constexpr (kPoints) cost.row(r + u, j0, c);
        else cost.decode(raw[u], c);
    }
};

// Round pass 1 (Alg. 3, first half): column sums of F = D(x) P and the column c-transform
// g'_j = min_i (C_ij - f_i); also the row c-transform f''_i = min_j (C_ij - g_j), for the
// two potential sets (u, v)/gamma and their finite differences along the annealing path.
template <class Cost, bool E64>
__device__ void tile_r1(const Work& w, const SweepArgs& S, const TileCtx& t, double* sm)
{
    double* sA = sm;
    double* sWt = sm + kBR;
    double* sS = sm + 2 * kBR;
    double* sF1 = sm + 3 * kBR;
    double* sF2 = sm + 4 * kBR;
    double* sCol = sm + 5 * kBR;
    const int m = w.m, n = w.n;
    const double g2 = S.gamma * w.scale * LOG2E_D;
    const double inv_g = 1.0 / S.gamma;
    const double dg = S.gamma - S.gamma_prev;
    const bool ext = dg > 0.0;
    const double inv_dg = ext ? 1.0 / dg : 0.0;
    double* sX = sWt;  // Round row factors, then weights
    if (t.tid < kBR) {
        int i = t.i0 + t.tid;
        double sh = -INFINITY, aa = 0.0, f1 = INFINITY, f2 = INFINITY, x = 0.0;
        if (i < m) {
            const Entry e = entry_after(w, S, i);
            sh = e.lz;
            aa = (e.z - e.lz) * LOG2E_D;
            f1 = e.z * inv_g;
            f2 = ext ? (e.z - e.zprev) * inv_dg : f1;
            x = round_x(w.r[i], e.lz);
        }
        sS[t.tid] = sh; sA[t.tid] = aa; sF1[t.tid] = f1; sF2[t.tid] = f2; sX[t.tid] = x;
    }
    {
        const int j = t.J * kBC + t.tid;
        // padding columns: v = -inf makes their exponentials 0, g = -inf their differences +inf
        double vv = -INFINITY, g1 = -INFINITY, g2v = -INFINITY;
        if (j < n) {
            const Entry e = entry_after(w, S, m + j);
            vv = e.z * LOG2E_D;
            g1 = e.z * inv_g;
            g2v = ext ? (e.z - e.zprev) * inv_dg : g1;
        }
        sCol[t.tid] = vv;
        sCol[kBC + t.tid] = g1;
        sCol[2 * kBC + t.tid] = g2v;
    }
    __syncthreads();
    const double SI = wave_max(sS[t.lane]);  // S_I = max_i s_i over the kBR (= 64) rows
    const int j0 = t.j0lane;
    if (t.tid < kBR) sWt[t.tid] = exp(sS[t.tid] - SI) * sX[t.tid];
    __syncthreads();
    Cost cost(w, t.i0);
    cost.cols(j0);
    double col64[4] = {0, 0, 0, 0};
    double cm1[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, cm2[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
    const double sc = w.scale;
    const int rbase = t.wave * kRPW;
    const int nrows = min(kRPW, m - (t.i0 + rbase));
    constexpr int B = sizeof(typename Cost::Raw) > 16 ? 2 : 4;
    double* region = sm + kRoundAt + t.wave * kRoundRegion;
    RoundRows<Cost, B> rows;
    rows.ask(cost, rbase, j0);
#pragma unroll 1
    for (int b = 0; b < nrows; b += B) {
        rows.take(cost, rbase + b, j0);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (b + u >= nrows) break;
            const int ir = rbase + b + u;
            double c[4], x[4], e[4], V[4];
            rows.get(cost, rbase + b, j0, u, c);
            cols4(sCol, t.lane, V);
            const double A = sA[ir], wt = sWt[ir];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = fma(-g2, c[k], V[k]) + A;
            exp2x4<E64>(x, e);
#pragma unroll
            for (int k = 0; k < 4; ++k) col64[k] = fma(wt, e[k], col64[k]);
            __builtin_amdgcn_sched_barrier(0);  // rows (and their halves) mixed with each other spill
            const double f1 = sF1[ir], f2 = sF2[ir];
            double G1[4], G2[4], rm1 = INFINITY, rm2 = INFINITY;
            cols4(sCol + kBC, t.lane, G1);
            cols4(sCol + 2 * kBC, t.lane, G2);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double cv = sc * c[k];
                cm1[k] = fmin(cm1[k], cv - f1);
                cm2[k] = fmin(cm2[k], cv - f2);
                rm1 = fmin(rm1, cv - G1[k]);
                rm2 = fmin(rm2, cv - G2[k]);
            }
            region[u * kRoundPad + t.lane] = rm1;
            region[(B + u) * kRoundPad + t.lane] = rm2;
            __builtin_amdgcn_sched_barrier(0);
        }
        const double v = round_reduce<0, 2, B>(region, t.lane);
        const int slot = t.lane >> 2, u = slot % B;
        if ((t.lane & 3) == 0 && slot < 2 * B && b + u < nrows)
            w.rowmin[(size_t)(slot < B ? t.J : w.nct + t.J) * m + t.i0 + rbase + b + u] = v;
    }
    __syncthreads();
    col_combine_store(sCol, col64, t, 0, w.colpart + (size_t)t.I * n, n, t.J * kBC);
    col_combine_store(sCol, cm1, t, 1, w.colmin + (size_t)t.I * n, n, t.J * kBC);
    col_combine_store(sCol, cm2, t, 1, w.colmin + (size_t)(w.nrt + t.I) * n, n, t.J * kBC);
    // every tile of row block I writes the same S_I, so the finalizer of any column block
    // reads it from one of the tiles it waited for
    if (t.tid == 0) w.tshift[t.I] = SI;
}

// Round pass 2: row sums of F' = D(x) P D(y): r(F')_i and sum_j F'_ij C_ij; (C err_c)_i;
// the row c-transform f'_i = min_j (C_ij - g'_j) and the column c-transform
// g''_j = min_i (C_ij - f''_i) (both potential sets).
template <class Cost, bool E64>
__device__ void tile_r2(const Work& w, const SweepArgs& S, const TileCtx& t, double* sm)
{
    double* sA = sm;
    double* sF1 = sm + 3 * kBR;
    double* sF2 = sm + 4 * kBR;
    double* sCol = sm + 5 * kBR;
    const int m = w.m, n = w.n;
    const double g2 = S.gamma * w.scale * LOG2E_D;
    if (t.tid < kBR) {
        int i = t.i0 + t.tid;
        double aa = 0.0, f1 = INFINITY, f2 = INFINITY;
        if (i < m) {
            const Entry e = entry_after(w, S, i);
            aa = (e.z - e.lz) * LOG2E_D;
            f1 = w.fpp[i];
            f2 = w.fpp[m + i];
        }
        sA[t.tid] = aa; sF1[t.tid] = f1; sF2[t.tid] = f2;
    }
    {
        // Padding columns add exact zeros to the sums and +inf to the minima.
        const int j = t.J * kBC + t.tid;
        const bool ok = j < n;
        sCol[t.tid] = ok ? entry_after(w, S, m + j).z * LOG2E_D : -INFINITY;
        sCol[kBC + t.tid] = ok ? w.yc[j] : 0.0;
        sCol[2 * kBC + t.tid] = ok ? w.errc[j] : 0.0;
        sCol[3 * kBC + t.tid] = ok ? w.gp[j] : -INFINITY;
        sCol[4 * kBC + t.tid] = ok ? w.gp[n + j] : -INFINITY;
    }
    __syncthreads();
    // V is the same as in pass 1, so every exp below is bit-identical to pass 1's and the
    // implicit plan F' = D(x) P D(y) is one matrix across both passes; y is applied in FP64.
    const int j0 = t.j0lane;
    Cost cost(w, t.i0);
    cost.cols(j0);
    double cm1[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, cm2[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
    const double sc = w.scale;
    const int rbase = t.wave * kRPW;
    const int nrows = min(kRPW, m - (t.i0 + rbase));
    constexpr int B = sizeof(typename Cost::Raw) > 16 ? 2 : 4, H = 2;  // rows loaded, and reduced, at a time
    double* region = sm + kRoundAt + t.wave * kRoundRegion;
    RoundRows<Cost, B> rows;
    rows.ask(cost, rbase, j0);
#pragma unroll 1
    for (int b = 0; b < nrows; b += B) {
        rows.take(cost, rbase + b, j0);
#pragma unroll
        for (int h = 0; h < B; h += H) {
            if (b + h >= nrows) break;
#pragma unroll
            for (int u = 0; u < H; ++u) {
                if (b + h + u >= nrows) break;
                const int ir = rbase + b + h + u;
                double c[4], x[4], e[4], V[4], Y[4], EC[4];
                rows.get(cost, rbase + b, j0, h + u, c);
                cols4(sCol, t.lane, V);
                const double A = sA[ir];
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = fma(-g2, c[k], V[k]) + A;
                exp2x4<E64>(x, e);
                cols4(sCol + kBC, t.lane, Y);
                cols4(sCol + 2 * kBC, t.lane, EC);
                double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double cv = sc * c[k];
                    const double ey = e[k] * Y[k];
                    s0 += ey;
                    s1 = fma(ey, cv, s1);
                    s2 = fma(cv, EC[k], s2);
                }
                region[u * kRoundPad + t.lane] = s0;
                region[(H + u) * kRoundPad + t.lane] = s1;
                region[(2 * H + u) * kRoundPad + t.lane] = s2;
                __builtin_amdgcn_sched_barrier(0);
                const double f1 = sF1[ir], f2 = sF2[ir];
                double GP1[4], GP2[4], rm1 = INFINITY, rm2 = INFINITY;
                cols4(sCol + 3 * kBC, t.lane, GP1);
                cols4(sCol + 4 * kBC, t.lane, GP2);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double cv = sc * c[k];
                    rm1 = fmin(rm1, cv - GP1[k]);
                    rm2 = fmin(rm2, cv - GP2[k]);
                    cm1[k] = fmin(cm1[k], cv - f1);
                    cm2[k] = fmin(cm2[k], cv - f2);
                }
                region[(3 * H + u) * kRoundPad + t.lane] = rm1;
                region[(4 * H + u) * kRoundPad + t.lane] = rm2;
                __builtin_amdgcn_sched_barrier(0);
            }
            const double v = round_reduce<3, 2, H>(region, t.lane);
            const int slot = t.lane >> 2, d = slot / H, r = b + h + slot % H;
            if ((t.lane & 3) == 0 && d < 5 && r < nrows) {
                double* dst = d == 0 ? w.rowpart : (d == 1 ? w.rowpart2 : (d == 2 ? w.rowpart3 : w.rowmin));
                dst[(size_t)(d == 4 ? w.nct + t.J : t.J) * m + t.i0 + rbase + r] = v;
            }
        }
    }
    __syncthreads();
    col_combine_store(sCol, cm1, t, 1, w.colmin + (size_t)t.I * n, n, t.J * kBC);
    col_combine_store(sCol, cm2, t, 1, w.colmin + (size_t)(w.nrt + t.I) * n, n, t.J * kBC);
}

// ------------------------------------------------------------------ finalizers
// Block reduction of kNDot values (fixed tree). sred: LDS of kNDot * 4 doubles.
__device__ void block_dots(double v[kNDot], double* dst, int tid, double* sred)
{
    wave_sum_dots(v);
    if ((tid & 63) == 0) {
#pragma unroll
        for (int d = 0; d < kNDot; ++d) sred[d * 4 + (tid >> 6)] = v[d];
    }
    __syncthreads();
    if (tid < kNDot) dst[tid] = (sred[tid * 4 + 0] + sred[tid * 4 + 1]) + (sred[tid * 4 + 2] + sred[tid * 4 + 3]);
    __syncthreads();
}

__device__ __forceinline__ bool in_range(double s, bool e64)  // shifted sum representable
{
    const double lo = e64 ? 0x1p-900 : 0x1p-64, hi = e64 ? 0x1p900 : 0x1p64;
    return s >= lo && s <= hi;  // false for NaN
}

// Tile partials of one entry, combined (the fields a sweep mode uses):
//   a: sum of the LSE partials (columns: each scaled by exp(S_I - M))
//   b: min of the first minima array (R1, R2)
//   c: min of the second minima array (finite-difference variant)
//   d, e: sums of the second and third row partials (R2)
struct Comb {
    double a, b, c, d, e;
};

template <int OP>  // 0: fma(x, f, acc), 1: min (red_op follows the same codes)
__device__ __forceinline__ double fold_op(double acc, double x, double f)
{
    if constexpr (OP == 0) return fma(x, f, acc);
    else return fmin(acc, x);
}

// Lane l of an entry's L-lane group folds partials l, l + L, l + 2L, ... of the m partials at
// base[I * stride], in that order, B loads in flight at a time. With `fac` (column LSE
// partials) partial I is scaled by fac[I] = exp(S_I - M), a table the workgroup forms once.
template <int OP, int B = 8>
__device__ __forceinline__ double lane_fold(const double* __restrict__ base, size_t stride, int l, int L, int m,
                                            const double* __restrict__ fac, bool use)
{
    double acc = (OP == 0) ? 0.0 : INFINITY;
    if (!use) return acc;
    for (int q0 = l; q0 < m; q0 += B * L) {
        double x[B], f[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int I = q0 + u * L;
            x[u] = (I < m) ? base[(size_t)I * stride] : 0.0;
            f[u] = (fac && I < m) ? fac[I] : 1.0;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int I = q0 + u * L;
            if (I < m) acc = fold_op<OP>(acc, x[u], f[u]);
        }
    }
    return acc;
}

// Fold over the L lanes of a group (L a power of two, groups aligned to L): scans towards
// lower lanes (row_shl 1, 2, 4, 8 within a row of 16, then lanes 16 and 32 further on), so
// lane 0 of each group ends with the group's value; the order depends only on L. Called by
// whole waves; the other lanes end with partial values.
template <int OP>
__device__ __forceinline__ double group_fold(double v, int L)
{
    const double id = (OP == 0) ? 0.0 : INFINITY;
    if (L >= 2) v = red_op<OP>(v, dpp_d<0x101>(id, v));
    if (L >= 4) v = red_op<OP>(v, dpp_d<0x102>(id, v));
    if (L >= 8) v = red_op<OP>(v, dpp_d<0x104>(id, v));
    if (L >= 16) v = red_op<OP>(v, dpp_d<0x108>(id, v));
    if (L >= 32) v = red_op<OP>(v, __shfl_down(v, 16, 64));
    if (L >= 64) v = red_op<OP>(v, __shfl_down(v, 32, 64));
    return v;
}

// Combine the tile partials of entry k (row k < n, column k - n otherwise) for `mode`. The LSE
// fold keeps BL loads in flight per lane (the other modes 8). Called by every lane of the wave;
// `valid` is false past the end of the (m + n)-vector.
template <int BL = 8>
__device__ __forceinline__ Comb combine(const Work& w, int mode, int k, bool valid, int l, int L, const double* fac)
{
    // row entries (k < m) combine the nct column-tile partials at stride m, column entries the nrt
    // row-tile partials at stride n
    const int m = w.m;
    const bool row = k < m;
    const int np = row ? w.nct : w.nrt;
    const size_t st = row ? (size_t)m : (size_t)w.n;
    const size_t ix = row ? (size_t)k : (size_t)(k - m);
    Comb cb{0.0, INFINITY, INFINITY, 0.0, 0.0};
    if (mode == SM_LSE) {
        cb.a = group_fold<0>(lane_fold<0, BL>((row ? w.rowpart : w.colpart) + ix, st, l, L, np, row ? nullptr : fac, valid), L);
    } else {
        const double* mn = (row ? w.rowmin : w.colmin) + ix;
        cb.b = group_fold<1>(lane_fold<1>(mn, st, l, L, np, nullptr, valid), L);
        cb.c = group_fold<1>(lane_fold<1>(mn + (size_t)np * st, st, l, L, np, nullptr, valid), L);
        if (mode == SM_R1) {
            cb.a = group_fold<0>(lane_fold<0>(w.colpart + ix, st, l, L, np, fac, valid && !row), L);
        } else {
            cb.a = group_fold<0>(lane_fold<0>(w.rowpart + ix, st, l, L, np, nullptr, valid && row), L);
            cb.d = group_fold<0>(lane_fold<0>(w.rowpart2 + ix, st, l, L, np, nullptr, valid && row), L);
            cb.e = group_fold<0>(lane_fold<0>(w.rowpart3 + ix, st, l, L, np, nullptr, valid && row), L);
        }
    }
    return cb;
}

// The line search and PNCG terms of one entry: gradient entry gnew at the trial, y its change.
__device__ __forceinline__ void lse_dots(const Entry& e, double gnew, double y, double l, double sum, bool e64,
                                         double v[kNDot])
{
    const double snew = e.logt - l;
    v[D_PHI] += e.p * gnew;
    v[D_NUM] += -y * snew;
    v[D_DEN] += y * e.p;
    v[D_SG] += snew * gnew;
    v[D_GN] += fabs(gnew);
    v[D_BAD] += in_range(sum, e64) ? 0.0 : 1.0;
}

// Terms of the LSE sweep's dots for entry k with trial log-sum l (row or column): the line
// search and PNCG dots, the row-only gradient norm (Sinkhorn projector) or, with `pre`, the
// diagonal-Hessian direction s~ = r~/r(P) - 1 (stored for the accept) and its dots.
__device__ __forceinline__ void lse_terms(const Work& w, const Entry& e, double g_cur, int k, double l, double sum,
                                          bool e64, bool pre, bool row, double v[kNDot])
{
    w.lzt[k] = l;
    const double rp = exp(l);
    const double gnew = rp - e.rt;
    const double y = gnew - g_cur;
    lse_dots(e, gnew, y, l, sum, e64, v);
    if (pre) {  // eq. (s-tilde) and the [0.01, 100] switch (Sec. 4.3)
        const double ratio = e.rt / rp;
        const double st = ratio - 1.0;
        w.sdt[k] = st;
        v[D_NUMT] += -y * st;
        v[D_SGT] += st * gnew;
        v[D_BAD] += (ratio >= 0.01 && ratio <= 100.0) ? 0.0 : kOutrUnit;
    } else if (row) {
        v[D_GNR] += fabs(gnew);
    }
}

// Finalize entry k of the (m + n)-vector after a sweep from its combined partials and add this
// entry's terms to the dots. M = max_I S_I (column entries of LSE and R1 sweeps).
__device__ __forceinline__ void finalize_entry(const Work& w, const SweepArgs& a, const Entry& e, double g_cur, int k,
                                               int mode, bool e64, bool pre, const Comb& cb, double M,
                                               double v[kNDot])
{
    const int m = w.m, n = w.n;
    if (k < m) {  // row i = k
        const int i = k;
        if (mode == SM_LSE) {
            const double sum = cb.a;
            const double l = fma(a.alpha, e.p, e.lz) + log(sum);  // shift used by the sweep
            lse_terms(w, e, g_cur, k, l, sum, e64, pre, true, v);
        } else if (mode == SM_R1) {
            w.fpp[i] = cb.b;
            w.fpp[m + i] = cb.c;
            v[D_RF1] += w.r[i] * cb.b;
            v[D_RF2] += w.r[i] * cb.c;
        } else {  // SM_R2
            const double ex = w.xr[i] * exp(e.lz);
            const double er = w.r[i] - ex * cb.a;  // err_r = r - r(F')
            v[D_A] += ex * cb.d;
            v[D_ERRR] += er;
            v[D_EC] += er * cb.e;
            v[D_RFP1] += w.r[i] * cb.b;
            v[D_RFP2] += w.r[i] * cb.c;
        }
        return;
    }
    const int j = k - m;  // column
    if (mode == SM_LSE) {
        const double sum = cb.a;
        const double l = M + log(sum);
        lse_terms(w, e, g_cur, k, l, sum, e64, pre, false, v);
    } else if (mode == SM_R1) {  // c(F)_j, y_j = c_j / c(F)_j ^ 1, err_c, g'_j (Alg. 3)
        const double cF = exp(M) * cb.a;
        const double cj = w.c[j];
        const double y = (cF > 0.0) ? fmin(cj / cF, 1.0) : 1.0;
        const double ec = cj - y * cF;
        w.yc[j] = y;
        w.errc[j] = ec;
        w.gp[j] = cb.b;
        w.gp[n + j] = cb.c;
        v[D_CG1] += cj * cb.b;
        v[D_CG2] += cj * cb.c;
        v[D_ERRC] += ec;
    } else {  // R2: g''_j
        v[D_CGP1] += w.c[j] * cb.b;
        v[D_CGP2] += w.c[j] * cb.c;
    }
}

// ------------------------------------------------------------------ scalar state machine
__device__ __forceinline__ void next_stage(State& S, const DevParams& P)
{
    const double gnew = fmin(S.gamma + (P.q - 1.0) * S.gamma, P.gamma_f);  // Alg. 1
    const double dg = gnew - S.gamma, dgp = S.gamma - S.gamma_prev;
    // warm start: eq. (approx-znext) (1), epsilon-scaling z' = (gamma' / gamma) z (2, Sec. 4.2.1),
    // or the previous solution unchanged (0)
    S.ws_ratio = P.warm_start == 1 ? dg / dgp : 0.0;
    S.ws_scale = P.warm_start == 2 ? gnew / S.gamma : 1.0;
    S.gamma_prev = S.gamma;
    S.gamma = gnew;
    S.stage += 1;
    S.eps_d = P.hterm / pow(gnew, P.p);  // entropy-aware tolerance (H_min, or log n: App. C)
    S.w = P.smooth_fixed ? P.w_fixed : fmin(S.eps_d / 4.0, 0.5);  // variable smoothing weight (fixed: App. D)
    S.tol = fmax(S.eps_d / 2.0, P.tol_floor);
    // precision ladder: FP32 exp while the tolerance is far above FP32 resolution
    S.exp64_stage = P.exp64_default || S.tol < S.f32_floor;
    S.exp64 = S.exp64_stage;
    S.alpha_prev = 1.0;
    S.vec_action |= VA_STAGE_INIT;
    S.sweep_mode = SM_LSE;
    S.ls_phase = LS_INIT;
    // MIXED: the first stage past the switch point runs on the exact cost; the host swaps the
    // cost and resumes (done = 2 pauses the solve with this stage's start already stored)
    if (S.on_proxy && S.gamma > P.mix_gamma) {
        S.on_proxy = 0;
        S.done = 2;
    }
}

__device__ __forceinline__ void end_stage(State& S, const DevParams& P, bool converged)
{
    if (!converged) S.inner_warn = 1;
    if (S.on_proxy) {  // MIXED: stages on the FP16 copy only provide warm starts
        S.proxy_stages++;
        if (S.gamma < P.gamma_f && !S.budget_stop) {
            next_stage(S, P);
            return;
        }
        S.on_proxy = 0;  // certify on the exact cost: pause for the swap first
        S.done = 2;
    }
    if (P.adaptive || S.gamma >= P.gamma_f || S.budget_stop) {
        S.vec_action |= VA_ROUND_PREP;
        S.sweep_mode = SM_R1;
    } else {
        next_stage(S, P);
    }
}

__device__ __forceinline__ void finish(State& S, int status)
{
    S.done = 1;
    S.status = status;
    S.sweep_mode = SM_NONE;
}

template <class T>
__device__ __forceinline__ void start_line_search(T& S)
{
    S.alpha = S.alpha_prev;
    S.alo = 0.0;
    S.dlo = S.dphi0;
    S.ahi = INFINITY;
    S.dhi = 0.0;
    S.ls_trials_cur = 0;
}

template <class Q>
__device__ __forceinline__ bool wolfe(const Q& P, double dphi0, double d)  // eq. (approximate-wolfe)
{
    return ((2.0 * P.c1 - 1.0) * dphi0 >= d) && (d >= P.c2 * dphi0);
}

// An accepted step's next direction: beta with the numerator of the direction this iterate takes
// (s, or s~ under the switch), and the restart. Returns the new slope <p, g>.
template <class T>
__device__ __forceinline__ double next_direction(T& S, double num, double den, double sg, double phi, int reset_bits)
{
    const double beta = (den != 0.0) ? num / den : 0.0;  // eq. (beta_PPR_OT)
    double pg = sg + beta * phi;                         // <s + beta p, g_new>
    const int reset = !(pg < 0.0);
    if (reset) {  // not a descent direction: restart with s (Alg. 2)
        pg = sg;
        S.cg_resets++;
    }
    S.alpha_acc = S.alpha;
    S.alpha_prev = S.alpha;
    S.beta = beta;
    S.reset = (reset ? RS_RESET : 0) | reset_bits;
    S.dphi0 = pg;
    return pg;
}

// A trial that was not accepted: shrink the bracket [alpha_lo, alpha_hi] with phi'(lo) < 0 < phi'(hi),
// then the next trial in it.
template <class T>
__device__ __forceinline__ void shrink_bracket(T& S, double d)
{
    if (d < 0.0) {
        S.alo = S.alpha;
        S.dlo = d;
    } else {  // NaN (range failure in FP64 too) also lands here: step too long
        S.ahi = S.alpha;
        S.dhi = d;
    }
}
template <class T>
__device__ __forceinline__ void next_trial(T& S)
{
    if (isinf(S.ahi)) {
        S.alpha = 2.0 * S.alpha;
    } else {  // hybrid step: mean of the secant point and the bisection point
        double asec = (S.alo * S.dhi - S.ahi * S.dlo) / (S.dhi - S.dlo);
        const double amid = 0.5 * (S.alo + S.ahi);
        if (!(asec > S.alo && asec < S.ahi)) asec = amid;
        S.alpha = 0.5 * asec + 0.5 * amid;
    }
}

// Scalar logic after a sweep: line search (App. B), PNCG bookkeeping (Alg. 2), stage
// control (Alg. 1) and the certified-gap termination. `sum` holds the global dots.
constexpr int kStallF32 = 256, kStallF64 = 4096;

// Precision ladder and stall guard after an accepted iteration with gradient norm gn: a stage
// whose gradient norm has not halved in kStallF32 iterations with FP32 exp continues with FP64
// exp (and so do the later stages, whose tolerances are smaller); after kStallF64 more
// iterations without halving it ends unconverged (returns true).
__device__ __forceinline__ bool stall_guard(State& S, double gn)
{
    if (gn <= 0.5 * S.stall_best) {
        S.stall_best = gn;
        S.stall_k = S.k;
    } else if (!S.exp64_stage && S.k - S.stall_k >= kStallF32) {
        S.exp64_stage = 1;
        S.exp64 = 1;
        S.f32_floor = fmax(S.f32_floor, 2.0 * S.tol);
        S.prec_switches++;
        S.stall_best = gn;
        S.stall_k = S.k;
    } else if (S.k - S.stall_k >= kStallF64) {
        return true;
    }
    return false;
}

// The Sinkhorn projector (Alg. 4) after a sweep: every half-step is taken whole (alpha = 1).
// The stage start's sweep gives log r(P), so the first half-step updates the rows; the sweep
// after a row update gives log c(P) for the column update; the sweep after a column update
// gives log r(P) again, ends the iteration and is where the stop test and the caps apply.
// gn is ||r(P) - r~||_1 (the column residual is zero up to rounding after a column update).
__device__ __forceinline__ void decide_sinkhorn(State& S, const DevParams& P, double gn, bool bad)
{
    S.alpha_acc = 0.0;
    S.beta = 0.0;
    S.vec_action = VA_ACCEPT;
    if (S.ls_phase == LS_INIT) {
        S.reset = RS_RESET | RS_ROWS;
        S.gnorm = gn;
        S.k = 1;
        S.stall_best = gn;
        S.stall_k = 1;
        S.sk_half = 0;
        if (gn <= S.tol) end_stage(S, P, true);
        else if (S.budget_stop || P.max_pncg_iters < 1 || bad) end_stage(S, P, false);
        else {
            S.ls_phase = LS_SINK;
            S.alpha = 1.0;
        }
        return;
    }
    S.alpha_acc = 1.0;
    if (S.sk_half == 0) {  // after the row update: the column update comes next
        S.reset = RS_RESET | RS_COLS;
        S.sk_half = 1;
        return;
    }
    S.reset = RS_RESET | RS_ROWS;
    S.sk_half = 0;
    S.pncg_iters++;
    S.k++;
    S.gnorm = gn;
    const bool stalled = stall_guard(S, gn);
    if (gn <= S.tol && !bad) end_stage(S, P, true);
    else if (S.k - 1 >= P.max_pncg_iters || S.budget_stop || stalled || bad) end_stage(S, P, false);
}

__device__ __forceinline__ void decide(State& S, const DevParams& P, const double* sum)
{
    const int mode = S.sweep_mode;
    S.vec_action = 0;
    if (mode == SM_LSE) {
        // D_BAD counts range failures plus kOutrUnit per ratio outside [0.01, 100] (precond)
        const double outr = floor(sum[D_BAD] * (1.0 / kOutrUnit));
        const bool bad = sum[D_BAD] - outr * kOutrUnit > 0.0;
        const bool tilde = P.precond && outr == 0.0;  // diagonal-Hessian direction this time
        if (bad && !S.exp64) {  // re-run this sweep with FP64 exp
            S.exp64 = 1;
            S.fallbacks++;
            return;
        }
        S.exp64 = S.exp64_stage;
        if (S.standalone) {
            if (bad) S.status = MDOT_W_RANGE;
            if (S.standalone == 2) {  // round-and-certify: lzt -> lz, then Round
                S.alpha_acc = 0.0;
                S.beta = 0.0;
                S.reset = 1;
                S.vec_action = VA_ACCEPT | VA_ROUND_PREP;
                S.sweep_mode = SM_R1;
            } else {
                finish(S, S.status);
            }
            return;
        }
        S.sweeps++;
        if (P.max_sweeps > 0 && S.sweeps >= P.max_sweeps) S.budget_stop = 1;
        if (P.projector == 1) {
            decide_sinkhorn(S, P, sum[D_GNR], bad);
            return;
        }
        const double gn = sum[D_GN], sg = tilde ? sum[D_SGT] : sum[D_SG];
        const double d = bad ? NAN : sum[D_PHI];
        if (S.ls_phase == LS_INIT) {  // first sweep of a stage: p = s (or s~), beta = 0
            S.alpha_acc = 0.0;
            S.beta = 0.0;
            S.reset = RS_RESET | (tilde ? RS_TILDE : 0);
            S.vec_action = VA_ACCEPT;
            S.gnorm = gn;
            S.k = 1;
            S.stall_best = gn;
            S.stall_k = 1;
            S.dphi0 = sg;
            if (gn <= S.tol) end_stage(S, P, true);
            else if (!(sg < 0.0) || S.budget_stop) end_stage(S, P, false);
            else {
                S.tilde_iters += tilde;
                S.ls_phase = LS_TRIAL;
                start_line_search(S);
            }
            return;
        }
        bool accept;
        if (S.ls_phase == LS_FORCE) {
            accept = true;
        } else {
            S.ls_trials++;
            S.ls_trials_cur++;
            accept = wolfe(P, S.dphi0, d);
        }
        if (accept) {
            // numerator of beta with the direction this iterate takes (s, or s~ under the switch)
            const double num = tilde ? sum[D_NUMT] : sum[D_NUM], den = sum[D_DEN];
            const double pg = next_direction(S, num, den, sg, sum[D_PHI], tilde ? RS_TILDE : 0);
            S.vec_action = VA_ACCEPT;
            S.pncg_iters++;
            S.k++;
            S.gnorm = gn;
            const bool stalled = stall_guard(S, gn);
            if (gn <= S.tol) end_stage(S, P, true);
            else if (S.k > P.max_pncg_iters || S.budget_stop || !(pg < 0.0) || stalled) end_stage(S, P, false);
            else {
                S.tilde_iters += tilde;
                S.ls_phase = LS_TRIAL;
                start_line_search(S);
            }
            return;
        }
        shrink_bracket(S, d);
        if (S.budget_stop) {  // stop at the last accepted iterate
            end_stage(S, P, false);
            return;
        }
        next_trial(S);
        if (S.ls_trials_cur >= P.max_ls_trials) {
            S.ls_failures++;
            if (S.alo > 0.0) {
                S.alpha = S.alo;
                S.ls_phase = LS_FORCE;
            } else {
                end_stage(S, P, false);
            }
        }
        return;
    }
    if (mode == SM_R1) {
        S.cert_sweeps++;
        S.r1[0] = sum[D_CG1];
        S.r1[1] = sum[D_CG2];
        S.r1[2] = sum[D_RF1];
        S.r1[3] = sum[D_RF2];
        S.errc_sum = sum[D_ERRC];
        S.sweep_mode = SM_R2;
        return;
    }
    // SM_R2: UB = <G, C> with G = F' + err_r err_c^T / ||err_r||_1 (Alg. 3), LB, termination
    S.cert_sweeps++;
    const double L = sum[D_ERRR];
    const double ub = sum[D_A] + (L > 0.0 ? sum[D_EC] / L : 0.0);
    const double lb = fmax(fmax(S.r1[0] + sum[D_RFP1], S.r1[1] + sum[D_RFP2]),
                           fmax(S.r1[2] + sum[D_CGP1], S.r1[3] + sum[D_CGP2]));
    const double me = fabs(S.errc_sum - L);
    S.last_ub = ub;
    S.last_lb = lb;
    if (S.standalone) {
        S.best_ub = ub;
        S.best_lb = lb;
        S.best_me = me;
        finish(S, S.status);
        return;
    }
    if (ub < S.best_ub) {
        S.best_ub = ub;
        S.best_gamma = S.gamma;
        S.best_me = me;
        S.vec_action |= VA_SAVE_BEST;
    }
    if (lb > S.best_lb) S.best_lb = lb;
    if (P.adaptive && S.best_ub - S.best_lb <= P.target) finish(S, MDOT_OK);
    else if (S.budget_stop) finish(S, MDOT_W_NOT_CONVERGED);
    else if (S.gamma >= P.gamma_f) finish(S, (P.adaptive || S.inner_warn) ? MDOT_W_NOT_CONVERGED : MDOT_OK);
    else next_stage(S, P);
}

// ------------------------------------------------------------------ the sweep kernel
// Cost types of a kernel instance (one per stored dtype / point metric).
// CC_PTS_SQ2 / CC_PTS_L12 are the planar (d <= 2) point instances: single-problem launches of
// planar clouds take them, and so does the engine when every problem in flight is planar. Their
// results are identical to the general instances'.
enum CostCode { CC_F64 = 0, CC_F32 = 1, CC_F16 = 2, CC_BF16 = 3, CC_PTS_SQ = 4, CC_PTS_L1 = 5, CC_PTS_SQ2 = 6,
                CC_PTS_L12 = 7, CC_PTS_SQ8 = 8, CC_PTS_L18 = 9 };
static_assert(CC_PTS_L18 + 1 == kCostCodes, "one kernel instance per cost code");
template <int CC> struct CostOf;
// The cost type of a kernel instance code (kOccHi marks the 2-waves-per-SIMD variant).
constexpr int base_code(int cc) { return cc >= kOccHi ? cc - kOccHi : cc; }
template <> struct CostOf<CC_F64> { using T = DenseCost<MDOT_DT_F64>; };
template <> struct CostOf<CC_F32> { using T = DenseCost<MDOT_DT_F32>; };
template <> struct CostOf<CC_F16> { using T = DenseCost<MDOT_DT_F16>; };
template <> struct CostOf<CC_BF16> { using T = DenseCost<MDOT_DT_BF16>; };
template <> struct CostOf<CC_PTS_SQ> { using T = PointCost<1>; };
template <> struct CostOf<CC_PTS_L1> { using T = PointCost<2>; };
template <> struct CostOf<CC_PTS_SQ2> { using T = PointCost<1, 2>; };
template <> struct CostOf<CC_PTS_L12> { using T = PointCost<2, 2>; };
template <> struct CostOf<CC_PTS_SQ8> { using T = PointCost<1, 8>; };
template <> struct CostOf<CC_PTS_L18> { using T = PointCost<2, 8>; };

template <int CC, bool E64, bool ROUND>
__device__ __forceinline__ void sweep_tiles(const Work& w, const SweepArgs& a, const TileCtx& t, int mode, double* smem)
{
    using Cost = typename CostOf<base_code(CC)>::T;
    if constexpr (!ROUND) {
        tile_lse<Cost, E64>(w, a, t, smem);
    } else {
        if (mode == SM_R1) tile_r1<Cost, E64>(w, a, t, smem);
        else tile_r2<Cost, E64>(w, a, t, smem);
    }
}

// Body of the sweep kernel for one tile. ROUND = false: LSE sweeps (the hot path);
// ROUND = true: the two Round/certificate sweeps (twice per stage).
template <int CC, bool ROUND>
__device__ __forceinline__ void sweep_kernel_body(const Work& w, const SweepArgs& a, int mode, bool e64, int blk,
                                                  double* smem)
{
    const TileCtx t = tile_ctx(w, blk);
    if (e64) sweep_tiles<CC, true, ROUND>(w, a, t, mode, smem);
    else sweep_tiles<CC, false, ROUND>(w, a, t, mode, smem);
}

// One kernel for every sweep mode, so a step is a fixed sequence of launches. The register
// cap keeps four workgroups per CU (the LDS limit is five). Every instance but the 8-coordinate ones
// fits it without spills (114 to 128 VGPRs), so their kOccHi codes launch the same kernel; the
// 8-coordinate clouds spill some 190 values under it and have an instance capped at two waves per SIMD
// (162 and 165 VGPRs, no spills), which they take unless the tuning table says otherwise.
template <int CC>
__device__ __forceinline__ void sweep_any(const Work& w, int parity, int blk, double* smem)
{
    // The state and the Work fields that locate the tile's cost rows are read in one group:
    // the compiler barrier keeps every one of these loads ahead of the first branch.
    const State* Sp = state_slot(w, parity);
    const int mode = Sp->sweep_mode, done = Sp->done, exp64 = Sp->exp64;
    const SweepArgs a = args_of(Sp);
    const int n = w.n, nct = w.nct;
    const void* cost = w.cost;
    asm volatile("" ::"s"(mode), "s"(done), "s"(exp64), "s"(n), "s"(nct), "s"(cost), "s"(a.alpha), "s"(a.gamma),
                 "s"(a.va)
                 : "memory");
    if ((mode == SM_NONE) | (done != 0)) return;
    if ((mode == SM_R1) | (mode == SM_R2)) sweep_kernel_body<CC, true>(w, a, mode, exp64 != 0, blk, smem);
    else sweep_kernel_body<CC, false>(w, a, mode, exp64 != 0, blk, smem);
}

template <int CC>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(CC >= kOccHi ? 2 : 4)))
k_sweep(const Work* __restrict__ wp, int parity)
{
    __shared__ double smem[kSmemAll];
    sweep_any<CC>(*wp, parity, blockIdx.x, smem);
}

// ------------------------------------------------------------------ the finalize kernel
// Reads state slot `parity` (the one this step's sweep used): stores the pending vector
// update, combines the tile partials of every entry of the (m + n)-vectors and writes per-workgroup
// dot products. The decide kernel that follows reduces them and writes the other slot.
constexpr int kFacMax = (MDOT_MAX_N + kBR - 1) / kBR;  // row tiles at the largest n
struct FinShared {
    double red[kNDot * 4];
    double fac[kFacMax];  // exp(S_I - M) of the column partials of row tile I
};

// Raw inputs of entry k for entry_after and the finalizer, loaded without data-dependent
// branches (k is clamped into range by the caller) so that every load of an entry is in
// flight at once. The marginal is read only when the update starts a stage: only solves do
// that, and only solves bind r and c.
struct EntryIn {
    double z, p, lz, logt, rt, zprev, lzt, m, g, sdt;
};
__device__ __forceinline__ EntryIn entry_load(const Work& w, const SweepArgs& a, int k)
{
    const int m = w.m;
    EntryIn in;
    in.z = w.z[k];
    in.p = w.p[k];
    in.lz = w.lz[k];
    in.logt = w.logt[k];
    in.rt = w.rt[k];
    in.zprev = w.zprev[k];
    in.lzt = w.lzt[k];
    in.m = (a.va & VA_STAGE_INIT) ? *((k < m) ? w.r + k : w.c + (k - m)) : 0.0;
    in.g = w.g[k];
    in.sdt = ((a.va & VA_ACCEPT) && (a.reset & RS_TILDE)) ? w.sdt[k] : 0.0;
    return in;
}
// entry_after from loaded inputs (same arithmetic, so bit-identical to the sweeps' copy)
__device__ __forceinline__ Entry entry_from(const EntryIn& in, const SweepArgs& a, int m, int n, int k)
{
    Entry e;
    e.z = in.z;
    e.p = in.p;
    e.lz = in.lz;
    e.logt = in.logt;
    e.rt = in.rt;
    e.zprev = in.zprev;
    if (a.va & VA_ACCEPT) {
        e.z = fma(a.alpha_acc, e.p, e.z);
        e.lz = in.lzt;
        e.p = next_dir(a, e.p, e.logt, e.lz, in.sdt, k < m);
    }
    e.zacc = e.z;
    if (a.va & VA_STAGE_INIT) {
        e.rt = fma(1.0 - a.w, in.m, a.w / (k < m ? m : n));
        e.logt = log(e.rt);
        if (a.stage == 1) {
            e.z = e.logt;
            e.zprev = e.logt;
        } else {
            const double zp = e.zprev;
            e.zprev = e.z;
            e.z = fma(a.ws_ratio, e.z - zp, a.ws_scale * e.z);
        }
        e.p = 0.0;
        e.lz = e.logt;
    }
    return e;
}

// Store the pending vector update of entry k and return the gradient entry at z.
__device__ __forceinline__ double store_update(const Work& w, const SweepArgs& a, const Entry& e, double g_old, int k)
{
    const int va = a.va;
    if (va & (VA_ACCEPT | VA_STAGE_INIT)) {
        w.z[k] = e.z;
        w.p[k] = e.p;
        w.lz[k] = e.lz;
    }
    double g_cur = g_old;
    if (va & VA_STAGE_INIT) {
        w.rt[k] = e.rt;
        w.logt[k] = e.logt;
        w.zprev[k] = e.zprev;
        g_cur = 0.0;
        w.g[k] = g_cur;
    } else if (va & VA_ACCEPT) {
        g_cur = exp(e.lz) - e.rt;
        w.g[k] = g_cur;
    }
    if (va & VA_SAVE_BEST) w.zbest[k] = e.zacc;
    if ((va & VA_ROUND_PREP) && k < w.m) w.xr[k] = round_x(w.r[k], e.lz);
    return g_cur;
}

// LSE finalize of one entry group when every partial fits one load per slot (at most PER per
// lane) and nrt <= 256: all loads of the group (tile shifts, partials, and unless LATE the entry
// inputs) are issued before any arithmetic. LATE loads the entry inputs after the fold, in the
// group's lane 0 only, which keeps them out of the registers the partials occupy.
template <int PER, bool LATE = false>
__device__ __forceinline__ void fin_lse_entry(const Work& w, const SweepArgs& a, int k, bool valid, int l, int L,
                                              bool e64, bool pre, double v[kNDot], double* sfac, bool first)
{
    const int m = w.m, n = w.n, nrt = w.nrt;
    const int kc = valid ? k : 0;
    const bool row = kc < m;
    const int np = row ? w.nct : nrt;               // partials of this entry
    const size_t st = row ? (size_t)m : (size_t)n;  // their stride
    const int lane = threadIdx.x & 63;
    const double* base = row ? w.rowpart + kc : w.colpart + (kc - m);
    double ts[4], x[PER];
#pragma unroll
    for (int q = 0; q < 4; ++q) ts[q] = w.tshift[min(lane + 64 * q, nrt - 1)];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int I = min(l + u * L, np - 1);
        x[u] = base[(size_t)I * st];
    }
    EntryIn in{};
    if constexpr (!LATE) in = entry_load(w, a, kc);
    // M = max_I S_I, the same value in every lane
    const double M = wave_max(fmax(fmax(ts[0], ts[1]), fmax(ts[2], ts[3])));
    // the column partials' factors exp(S_I - M) depend on I alone: thread I of the workgroup
    // forms factor I once (its wave holds S_I in ts[wave]), the entries read them from LDS
    if (first) {
        const int tid = threadIdx.x, wv = tid >> 6;
        const double sI = wv == 0 ? ts[0] : (wv == 1 ? ts[1] : (wv == 2 ? ts[2] : ts[3]));
        if (tid < nrt) sfac[tid] = exp(sI - M);
        __syncthreads();
    }
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (l + u * L < np) acc = fma(x[u], row ? 1.0 : sfac[min(l + u * L, 255)], acc);
    Comb cb{};
    cb.a = group_fold<0>(acc, L);
    if (!valid || l != 0) return;
    if constexpr (LATE) in = entry_load(w, a, kc);
    const Entry e = entry_from(in, a, m, n, k);
    const double g_cur = store_update(w, a, e, in.g, k);
    finalize_entry(w, a, e, g_cur, k, SM_LSE, e64, pre, cb, M, v);
}

// Finalize workgroup `blk` of the problem's `nblk` (= fin_grid(m, n)) workgroups. A row entry is
// handled by a group of fin_Lr lanes, a column entry by one of fin_L lanes; the row groups fill
// virtual blocks [0, fin_nvbr) of kVecWG / fin_Lr rows each, the column groups the rest, and the
// workgroups take the virtual blocks in a grid-stride loop.
// Instances (V, fin_instance):
//   kFinSmall: at most 8192 rows and columns (8 partials per lane in the fast path);
//   kFinMid:   more, with at most 256 row tiles (32 partials per lane in the fast path, the entry
//              inputs loaded after the fold); capped at 256 VGPRs, two waves per SIMD;
//   kFinAll:   any size (past 256 row tiles the general path folds in batches of 32 loads).
template <int V>
__device__ __forceinline__ void fin_body(const Work& w, int parity, int blk, int nblk, FinShared& sh)
{
    // Every control read (the Work fields and the state) is issued before the first branch,
    // through a pointer held in a vector register (as scalar data these reads overflow the
    // SGPRs and are issued in dependent groups), so the latency of the first access after
    // the kernel boundary is paid once.
    uint64_t cb = reinterpret_cast<uint64_t>(&ctl_of(w));
    asm volatile("" : "+v"(cb));
    const Control* C = reinterpret_cast<const Control*>(cb);
    const Work wl = C->w;
    const State* Sp = C->st + parity;
    const int done = Sp->done, mode = Sp->sweep_mode, exp64 = Sp->exp64;
    const SweepArgs a = args_of(Sp);
    const bool pre = C->prm.precond != 0;
    asm volatile("" ::: "memory");
    const int tid = threadIdx.x;
    const int m = wl.m, n = wl.n;
    const bool active = (done == 0) & (mode != SM_NONE);
    const bool e64 = exp64 != 0;
    const int per = wl.fin_per;
    // the fast path: LSE entries whose partials take one load per slot, with the factor table
    // of at most 256 row tiles
    const bool lse = active & (mode == SM_LSE) & (wl.nrt <= 256);
    const bool fast_r = lse & (wl.nct <= per * wl.fin_Lr), fast_c = lse & (wl.nrt <= per * wl.fin_L);
    double v[kNDot];
#pragma unroll
    for (int d = 0; d < kNDot; ++d) v[d] = 0.0;
    // M = max_I S_I (every wave forms the same maximum) for the general path, and the factors
    // exp(S_I - M) of the column partials, formed once per workgroup (instead of once per entry
    // and partial: 2 x 10^8 FP64 exps per sweep at n = 10^5)
    double M = 0.0;
    if (!(fast_r && fast_c) && active && (mode == SM_LSE || mode == SM_R1)) {
        double mx = -INFINITY;
        for (int I = tid & 63; I < wl.nrt; I += 64) mx = fmax(mx, wl.tshift[I]);
        M = wave_max(mx);
        for (int I = tid; I < wl.nrt; I += kVecWG) sh.fac[I] = exp(wl.tshift[I] - M);
        __syncthreads();
    }
    const int nvb = wl.fin_nvb, nvbr = wl.fin_nvbr;
    for (int vb = blk; vb < nvb; vb += nblk) {
        // virtual workgroups [0, nvbr) hold the row groups, the rest the column groups
        const bool rseg = vb < nvbr;
        const int L = rseg ? wl.fin_Lr : wl.fin_L;
        const int l = tid & (L - 1);
        const int k = rseg ? (vb * kVecWG + tid) >> wl.fin_lgLr : m + (((vb - nvbr) * kVecWG + tid) >> wl.fin_lgL);
        const bool valid = k < (rseg ? m : m + n);
        if (rseg ? fast_r : fast_c) {
            if (V == kFinSmall || per == 8) fin_lse_entry<8>(wl, a, k, valid, l, L, e64, pre, v, sh.fac, vb == blk);
            else fin_lse_entry<32, V == kFinMid>(wl, a, k, valid, l, L, e64, pre, v, sh.fac, vb == blk);
            continue;
        }
        const int kc = valid ? k : 0;
        const EntryIn in = entry_load(wl, a, kc);
        Comb cb{};
        // past 256 row tiles (the kFinAll instance only) an LSE entry folds its partials in
        // batches of 32 loads: 8 lanes share some hundreds of partials there
        if (active) cb = combine<V == kFinAll ? 32 : 8>(wl, mode, k, valid, l, L, sh.fac);
        if (!valid || l != 0) continue;
        const Entry e = entry_from(in, a, m, n, k);
        const double g_cur = store_update(wl, a, e, in.g, k);
        if (active) finalize_entry(wl, a, e, g_cur, k, mode, e64, pre, cb, M, v);
    }
    if (active) block_dots(v, bdots_of(w) + (size_t)blk * kNDot, tid, sh.red);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2. With `xcd`,
// physical workgroup b takes the place of workgroup (b % 8) (G / 8) + b / 8 (8 divides the grid
// G): runs of consecutive virtual workgroups then run on one XCD at about the same time. With 16
// or more lanes per column entry, a virtual workgroup holds 16 or fewer columns, and the partials
// of consecutive columns share cache lines, which each XCD then fetches once instead of once per
// workgroup. Everything a workgroup computes and stores depends on its virtual index alone.
template <int V>
__global__ void __launch_bounds__(kVecWG, V == kFinMid ? 2 : 1) k_fin(const Work* __restrict__ wp, int parity, int xcd)
{
    __shared__ FinShared sh;
    const int G = gridDim.x, b = blockIdx.x;
    fin_body<V>(*wp, parity, xcd ? (b & 7) * (G >> 3) + (b >> 3) : b, G, sh);
}

// ------------------------------------------------------------------ the decide kernel
// One wave per problem: reduce the finalize kernel's per-workgroup dots in a fixed order, run
// the scalar state machine on slot `parity` (every lane holds the same values; lane 0 stores)
// and write the next state into the other slot (a finished or idle state is carried over with
// its vector update cleared).
constexpr int kDecideWG = 64;

__device__ __forceinline__ void decide_body(const Work& w, int parity, int to)
{
    const int lane = threadIdx.x;
    // Every read of this kernel is issued together: the state, the parameters, the finalize
    // workgroup count and the first 4 x 64 workgroups' dots (the dots array has kFinMaxGrid
    // entries, so these loads are in bounds for any size; entries past fin_grid are masked). The control block is read through
    // a pointer held in a vector register, so the state is loaded into VGPRs (as scalar data it
    // would overflow the SGPRs and be reloaded piecemeal).
    uint64_t cb = reinterpret_cast<uint64_t>(&ctl_of(w));
    asm volatile("" : "+v"(cb));
    const Control* C = reinterpret_cast<const Control*>(cb);
    State S = C->st[parity];
    const DevParams P = C->prm;
    const int nblk = C->w.fin_nblk;
    double x[4][kNDot];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < kNDot; ++d) x[q][d] = C->bdots[(lane + 64 * q) * kNDot + d];
    double v[kNDot];
#pragma unroll
    for (int d = 0; d < kNDot; ++d) v[d] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < kNDot; ++d) v[d] += (lane + 64 * q < nblk) ? x[q][d] : 0.0;
    const bool active = !S.done && S.sweep_mode != SM_NONE;
    if (active) {
        // the workgroups past the first 256, in the same order, four rounds' loads at a time
        int b = lane + 256;
        for (; b + 192 < nblk; b += 256) {
            double y[4][kNDot];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int d = 0; d < kNDot; ++d) y[u][d] = C->bdots[(b + 64 * u) * kNDot + d];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int d = 0; d < kNDot; ++d) v[d] += y[u][d];
        }
        for (; b < nblk; b += 64)
#pragma unroll
            for (int d = 0; d < kNDot; ++d) v[d] += C->bdots[b * kNDot + d];
        wave_sum_dots(v);
        decide(S, P, v);
    } else {
        S.vec_action = 0;
    }
    S.undecided = 0;
    if (lane == 0) *state_slot(w, to) = S;
}

__global__ void __launch_bounds__(kDecideWG) k_decide(const Work* __restrict__ wp, int parity)
{
    decide_body(*wp, parity, parity ^ 1);
}

// The decision a resident-steps kernel left to this one, in state slot 0.
__global__ void __launch_bounds__(kDecideWG) k_settle(const Work* __restrict__ wp)
{
    if (state_slot(*wp, 0)->undecided) decide_body(*wp, 0, 0);
}

// ------------------------------------------------------------------ resident steps
// k_steps runs the LSE steps of a problem of at most 1024 tiles (n = 4096 square) inside one
// kernel: sweep, finalize and decision of a trial, then the next trial, until the state machine
// asks for something else (Round, the stage's end, a cap), which k_settle and the one-step kernels
// do. What bounds a step of three kernels at these sizes is not its work but the three boundaries;
// inside one kernel a step has two exchanges between workgroups instead, of 1 to 1.5 us each, and
// the cost stays in registers. Per step, in solves with FP32 cost and exponentials: n = 256 14.5 ->
// 8.2 us, n = 1024 14.8 -> 8.7, n = 4096 24.7 -> 15.5. Of the 8.2 us the sweep takes 1.5 (one wave
// per SIMD), its set-up and partials 1.2, the first exchange 1.3, folding, log and exp of the
// finalize block and its dots 1.7, the second exchange 1.4, the decision 1.0.
//
// Every workgroup holds up to four tiles (a quad of four waves takes one or two: n = 4096 is 256
// workgroups, one per compute unit, of two quads, or of four for a point cloud) with their rows' and
// columns' vector entries in LDS, and does the work of the finalize block of its own number if there is
// one. Arithmetic and orders are those of k_sweep, k_fin and k_decide, so the results are the same bits.
// Per step:
//   1. sweep: tile partials and row-tile shifts are stored for the finalize blocks;
//   2. the finalize blocks fold them and store log-sums and dots;
//   3. every workgroup reads all dots, takes the decision (the same in each; anything but the
//      next trial is left to k_settle) and reads the log-sums of its own rows and columns.
// Values travel through memory with agent-scope loads and stores, which meet where every XCD
// sees them. An empty slot holds kEmpty, a NaN no arithmetic produces, and a reader waits until
// its value is there: data and flag arrive in one trip. Slots are used in turns of three. A writer
// empties a slot, waits for that store, and then fills a slot of an earlier turn, so whoever has
// seen that one filled finds the emptied slot empty or filled again:
//   - a tile's partials of step s + 1 are emptied in step s - 1, after its partials of s - 1 are
//     stored and its dots read (so the slot's last readers, in step s - 2, are through);
//   - log-sums and dots of step s + 1 are emptied at the start of step s. Their last readers are
//     those of step s - 2, and all dots of step s - 1 having been read, everybody is past it.
//
// All workgroups have to run at the same time. They meet once at the start, with a limit of
// kStartTicks: if the GPU is shared and some cannot start, all of them leave with nothing
// changed and the one-step kernels that follow carry on. Later waits cannot starve; they have a
// limit all the same (kWaitLooks), after which the solve ends with an error.
constexpr uint64_t kEmpty = 0x7ff8dead0000beefull;
constexpr uint32_t kStepsAbort = 0x80000000u;
constexpr uint64_t kStartTicks = 5000;  // 50 us of the 100 MHz wall clock

template <class T>
__device__ __forceinline__ T xload(const T* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void xstore(T* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double empty_slot() { return __builtin_bit_cast(double, kEmpty); }
__device__ __forceinline__ bool is_empty(double v) { return __builtin_bit_cast(uint64_t, v) == kEmpty; }
// every memory operation of this wave before it has completed
__device__ __forceinline__ void wave_drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A bounded wait: again() after an unsuccessful look.
struct Wait {
    StepsX* x;
    uint32_t n = 0;
    bool dead = false;
    __device__ __forceinline__ explicit Wait(StepsX* x_) : x(x_) {}
    __device__ __forceinline__ bool again()
    {
        if (++n % kWaitFlag == 0) {
            if (n >= kWaitLooks) xstore(&x->abort, 1u);
            dead = xload(&x->abort) != 0;
        }
        return !dead;
    }
};

// The steps this kernel takes: a stage's first sweep and its line-search trials.
__device__ __forceinline__ bool steps_go(const State& S)
{
    return S.done == 0 && S.sweep_mode == SM_LSE && (S.ls_phase == LS_INIT || S.ls_phase == LS_TRIAL) && !S.standalone &&
           !S.undecided && !S.budget_stop && !(S.reset & RS_TILDE);
}

// The part of State that these steps change (beside it, vec_action: the pending update is taken
// when the kernel starts).
struct Trial {
    double alpha, alpha_acc, alpha_prev, beta, dphi0, alo, dlo, ahi, dhi, gnorm, stall_best;
    int64_t k, sweeps, pncg_iters, ls_trials, cg_resets, stall_k;
    int32_t vec_action, reset, ls_trials_cur, ls_phase, exp64;
    template <class A, class B>
    static __device__ __forceinline__ void copy(A& a, const B& b)
    {
        a.alpha = b.alpha; a.alpha_acc = b.alpha_acc; a.alpha_prev = b.alpha_prev; a.beta = b.beta;
        a.dphi0 = b.dphi0; a.alo = b.alo; a.dlo = b.dlo; a.ahi = b.ahi; a.dhi = b.dhi;
        a.gnorm = b.gnorm; a.stall_best = b.stall_best;
        a.k = b.k; a.sweeps = b.sweeps; a.pncg_iters = b.pncg_iters; a.ls_trials = b.ls_trials;
        a.cg_resets = b.cg_resets; a.stall_k = b.stall_k;
        a.vec_action = b.vec_action; a.reset = b.reset; a.ls_trials_cur = b.ls_trials_cur;
        a.ls_phase = b.ls_phase; a.exp64 = b.exp64;
    }
};

// What a decision inside a stage needs besides.
struct TrialParams {
    double c1, c2, tol;
    int64_t max_sweeps, max_pncg_iters, stall;
    int32_t max_ls_trials, exp64_stage;
    __device__ __forceinline__ void set(const DevParams& P, const State& S)
    {
        c1 = P.c1;
        c2 = P.c2;
        tol = S.tol;
        max_sweeps = P.max_sweeps;
        max_pncg_iters = P.max_pncg_iters;
        max_ls_trials = P.max_ls_trials;
        exp64_stage = S.exp64_stage;
        stall = S.exp64_stage ? kStallF64 : kStallF32;
    }
};

constexpr int kStepDots = D_GN + 1;  // the dots these steps need: D_PHI .. D_GN, and whether any D_BAD

// decide() for a step that stays inside its stage: false, with T unchanged, where anything else
// follows (range, budget, caps, the stage's end, a stall), which is left to it.
__device__ __forceinline__ bool decide_trial(Trial& T, const TrialParams& P, const double* sum, bool bad)
{
    if (bad || (P.max_sweeps > 0 && T.sweeps + 1 >= P.max_sweeps)) return false;
    const double gn = sum[D_GN], d = sum[D_PHI], sg = sum[D_SG];
    if (T.ls_phase == LS_INIT) {
        if (gn <= P.tol || !(sg < 0.0)) return false;
        T.alpha_acc = 0.0;
        T.beta = 0.0;
        T.reset = RS_RESET;
        T.vec_action = VA_ACCEPT;
        T.k = 1;
        T.stall_best = gn;
        T.stall_k = 1;
        T.dphi0 = sg;
        T.gnorm = gn;
        T.ls_phase = LS_TRIAL;
        start_line_search(T);
    } else if (wolfe(P, T.dphi0, d)) {
        Trial t = T;
        const double pg = next_direction(t, sum[D_NUM], sum[D_DEN], sg, d, 0);
        t.k++;
        if (gn <= 0.5 * t.stall_best) {
            t.stall_best = gn;
            t.stall_k = t.k;
        } else if (t.k - t.stall_k >= P.stall) {
            return false;
        }
        if (gn <= P.tol || t.k > P.max_pncg_iters || !(pg < 0.0)) return false;
        t.vec_action = VA_ACCEPT;
        t.pncg_iters++;
        t.ls_trials++;
        t.gnorm = gn;
        start_line_search(t);
        T = t;
    } else {
        if (T.ls_trials_cur + 1 >= P.max_ls_trials) return false;
        shrink_bracket(T, d);
        next_trial(T);
        T.vec_action = 0;
        T.ls_trials++;
        T.ls_trials_cur++;
    }
    T.sweeps++;
    T.exp64 = P.exp64_stage;
    return true;
}

template <int NT>
struct StepsShared {  // NT: tiles of the workgroup
    double region[NT][4][kRowBufD];  // per tile and wave: row transpose, then its columns' values
    double A[NT][kBR], wt[NT][kBR], s[NT][kBR], x[NT][3 * kBR], colv[NT][kBC];
    double cz[NT][kBC], cp[NT][kBC], clt[NT][kBC];                                   // column entries
    double rz[NT][kBR], rp[NT][kBR], rlz[NT][kBR], rlt[NT][kBR], rxx[NT][kBR];       // row entries
    double fz[kVecWG], fp[kVecWG], flz[kVecWG], flt[kVecWG], frt[kVecWG], fg[kVecWG], fl[kVecWG];  // finalize entries
    double fac[kStepsMaxRowTiles];
    double red[(kStepDots + 1) * 4];
    double y[kStepDots + 1][kStepsMaxGrid];  // the dots of all finalize blocks, and D_BAD
    double *rowp[3], *colp[3], *logr[3], *logc[3];  // the three turns of the slots
    Trial T;
    TrialParams P;
    int go, dead;
};
static_assert(8 * 64 <= kRowBufD, "eight rows of FP64 partials fit a wave region");
static_assert(sizeof(StepsShared<4>) <= 160 * 1024, "LDS of one compute unit");

// Where a thread stands. Its index is made opaque to the compiler wherever it is read, so that
// nothing derived from it stays in registers from one part of a step to the next: hoisted out of
// the step loop, addresses and masks take more registers than a tile's cost. What is the same in a wave is kept in scalar registers.
struct Lane {
    int t, lane, wave, q;  // thread of the quad, lane and wave of it, quad
    __device__ __forceinline__ Lane()
    {
        int i = threadIdx.x;
        asm volatile("" : "+v"(i));
        const int wv = __builtin_amdgcn_readfirstlane(i >> 6);
        t = i & 255;
        lane = i & 63;
        wave = wv & 3;
        q = wv >> 2;
    }
};

// One tile of a quad (all scalar): the workgroup's tile `at`.
struct StepTile {
    int m, n, at, I, J, i0, rbase, nrows;
    bool has;
    __device__ __forceinline__ void set(const Work& w, int blk, int nt, int at_)
    {
        const Lane me;
        m = w.m;
        n = w.n;
        at = at_;
        const int tile = blk * nt + at;
        has = tile < w.nrt * w.nct;
        I = has ? tile / w.nct : 0;
        J = has ? tile % w.nct : 0;
        i0 = I * kBR;
        rbase = me.wave * kRPW;
        nrows = has ? min(kRPW, m - (i0 + rbase)) : 0;
    }
    __device__ __forceinline__ bool has_col(const Lane& me) const { return has && J * kBC + me.t < n; }
    __device__ __forceinline__ bool has_row(const Lane& me) const { return has && me.t < kBR && i0 + me.t < m; }
    // the row whose partial a lane stores (as rows_reduce_* leave them), and whether there is one
    __device__ __forceinline__ bool has_prow(const Lane& me) const { return (me.lane & 3) == 0 && (me.lane >> 2) < nrows; }
    __device__ __forceinline__ bool has_shift(const Lane& me) const { return has && J == 0 && me.t == 0; }
};

// The sizes the steps need, in scalar registers throughout, and which of the problem's workgroups
// this is.
struct StepSize {
    int blk, nblk, m, n, nrt, nct, nvb, nvbr, Lr, L, lgLr, lgL;
    __device__ __forceinline__ StepSize(const Work& w, int blk_, int nblk_)
        : blk(blk_), nblk(nblk_), m(w.m), n(w.n), nrt(w.nrt), nct(w.nct), nvb(w.fin_nvb), nvbr(w.fin_nvbr), Lr(w.fin_Lr), L(w.fin_L), lgLr(w.fin_lgLr),
          lgL(w.fin_lgL) {}
};

// The three slots of every exchanged value, in buffers that LSE steps leave unused. The log-sums'
// third is the trial vector itself, which holds the pending step's log-sums at the start. Their
// addresses are kept in LDS: read from the Work struct in every part of a step they cost 2 us.
template <int NT>
__device__ __forceinline__ void steps_slots(const Work& w, StepsShared<NT>& sh)
{
    sh.rowp[0] = w.rowpart; sh.rowp[1] = w.rowpart2; sh.rowp[2] = w.rowpart3;
    sh.colp[0] = w.colpart; sh.colp[1] = w.colmin;   sh.colp[2] = w.colmin + (size_t)w.nrt * w.n;
    sh.logr[0] = w.sdt;     sh.logr[1] = w.fpp;      sh.logr[2] = w.lzt;
    sh.logc[0] = w.sdt + w.m; sh.logc[1] = w.gp;     sh.logc[2] = w.lzt + w.m;
}
template <int NT>
__device__ __forceinline__ double* row_slot(const StepsShared<NT>& sh, const StepTile& t, const Lane& me, int b)
{
    return sh.rowp[b] + (size_t)t.J * t.m + (t.i0 + t.rbase) + (me.lane >> 2);
}
template <int NT>
__device__ __forceinline__ double* col_slot(const StepsShared<NT>& sh, const StepTile& t, const Lane& me, int b)
{
    return sh.colp[b] + (size_t)t.I * t.n + t.J * kBC + me.t;
}

// A thread's entry of its workgroup's finalize block (the first quad of the first fin_nvb workgroups),
// as in fin_body.
struct FinEntry {
    bool row, valid, own;
    int L, l, k, np;       // lanes and lane of the group, row or column, its partials
    __device__ __forceinline__ FinEntry(const StepSize& z, const Lane& me)
    {
        const int vb = z.blk;
        row = vb < z.nvbr;
        L = row ? z.Lr : z.L;
        l = me.t & (L - 1);
        k = row ? (vb * kVecWG + me.t) >> z.lgLr : ((vb - z.nvbr) * kVecWG + me.t) >> z.lgL;
        np = row ? z.nct : z.nrt;
        valid = vb < z.nvb && me.q == 0 && k < (row ? z.m : z.n);
        own = valid && l == 0;
    }
    __device__ __forceinline__ int entry(const StepSize& z) const { return row ? k : z.m + k; }
};

// Empty the slots of turn b: a tile's partials, and a finalize block's results.
template <int NT>
__device__ __forceinline__ void clear_tile(const StepsShared<NT>& sh, StepsX* x, const StepTile& t, int b)
{
    const Lane me;
    if (t.has_prow(me)) xstore(row_slot(sh, t, me, b), empty_slot());
    if (t.has_col(me)) xstore(col_slot(sh, t, me, b), empty_slot());
    if (t.has_shift(me)) xstore(&x->shift[b][t.I], empty_slot());
}
template <int NT>
__device__ __forceinline__ void clear_fin(const StepsShared<NT>& sh, const StepSize& z, StepsX* x, int b)
{
    const Lane me;
    const FinEntry f(z, me);
    if (f.own) xstore((f.row ? sh.logr[b] : sh.logc[b]) + f.k, empty_slot());
    if (me.q == 0 && me.t <= kStepDots) xstore(&x->dots[b][z.blk][me.t], empty_slot());
}

// Entry k with the pending update of the last step (or stage) taken. The trial log-sums are read as
// the steps will read them, since their buffer is one of the slots.
__device__ __forceinline__ EntryIn steps_entry_in(const Work& w, const SweepArgs& a, int k)
{
    EntryIn in;
    in.z = w.z[k];
    in.p = w.p[k];
    in.lz = w.lz[k];
    in.logt = w.logt[k];
    in.rt = w.rt[k];
    in.zprev = w.zprev[k];
    in.lzt = xload(w.lzt + k);
    in.m = (a.va & VA_STAGE_INIT) ? *((k < w.m) ? w.r + k : w.c + (k - w.m)) : 0.0;
    in.g = w.g[k];
    in.sdt = 0.0;
    return in;
}

// The vector entries of a tile.
template <int NT>
__device__ __forceinline__ void steps_load(const Work& w, const SweepArgs& a, StepsShared<NT>& sh, const StepTile& t)
{
    const Lane me;
    if (t.has_col(me)) {
        const int k = t.m + t.J * kBC + me.t;
        const Entry e = entry_from(steps_entry_in(w, a, k), a, t.m, t.n, k);
        sh.cz[t.at][me.t] = e.z;
        sh.cp[t.at][me.t] = e.p;
        sh.clt[t.at][me.t] = e.logt;
    }
    if (t.has_row(me)) {
        const int k = t.i0 + me.t;
        const Entry e = entry_from(steps_entry_in(w, a, k), a, t.m, t.n, k);
        sh.rz[t.at][me.t] = e.z;
        sh.rp[t.at][me.t] = e.p;
        sh.rlz[t.at][me.t] = e.lz;
        sh.rlt[t.at][me.t] = e.logt;
    }
}

// The finalize block's entries, with the update stored as the finalize kernel does. Only when every
// workgroup has loaded its own: they read the same vectors.
template <int NT>
__device__ __forceinline__ void steps_load_fin(const Work& w, const StepSize& z, const SweepArgs& a, StepsShared<NT>& sh)
{
    const Lane me;
    const FinEntry f(z, me);
    if (!f.own) return;
    const int k = f.entry(z);
    const EntryIn in = steps_entry_in(w, a, k);
    const Entry e = entry_from(in, a, w.m, w.n, k);
    sh.fg[me.t] = store_update(w, a, e, in.g, k);
    sh.fz[me.t] = e.z;
    sh.fp[me.t] = e.p;
    sh.flz[me.t] = e.lz;
    sh.flt[me.t] = e.logt;
    sh.frt[me.t] = e.rt;
    sh.fl[me.t] = in.lzt;
}

// Wait until every workgroup has announced itself; false if one of them does not get to run.
__device__ __forceinline__ bool steps_wait_all(const StepSize& z, StepsX* x)
{
    uint32_t seen = xload(&x->arrive);
    const uint64_t t0 = wall_clock64();
    while (!(seen & kStepsAbort) && seen != (uint32_t)z.nblk) {
        if (wall_clock64() - t0 > kStartTicks)  // give up, unless the last one has just come
            __hip_atomic_compare_exchange_strong(&x->arrive, &seen, seen | kStepsAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        seen = xload(&x->arrive);
    }
    return !(seen & kStepsAbort);
}
__device__ __forceinline__ bool steps_meet(const StepSize& z, StepsX* x)
{
    __hip_atomic_fetch_add(&x->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return steps_wait_all(z, x);
}
// The last workgroup to end clears both counts for the next kernel, and notes a meeting that failed (not
// before: a workgroup that starts late must not find the note and leave without being counted).
__device__ __forceinline__ void steps_leave(const StepSize& z, StepsX* x, bool missed = false)
{
    if (threadIdx.x == 0 &&
        __hip_atomic_fetch_add(&x->leave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == (uint32_t)z.nblk) {
        xstore(&x->leave, 0u);
        xstore(&x->arrive, 0u);
        if (missed) xstore(&x->skip, 1u);
    }
}

// What the next step does with the vectors.
template <int NT>
__device__ __forceinline__ SweepArgs steps_args(const StepsShared<NT>& sh)
{
    SweepArgs a{};
    a.alpha = sh.T.ls_phase == LS_TRIAL ? sh.T.alpha : 0.0;
    a.alpha_acc = sh.T.alpha_acc;
    a.beta = sh.T.beta;
    a.reset = sh.T.reset;
    a.va = sh.T.vec_action;
    return a;
}

// The pending update of a tile's entries, and its set-up: row shifts and terms, column terms (see
// tile_lse).
template <class Cost, int NT>
__device__ __forceinline__ void steps_update(StepsShared<NT>& sh, const StepTile& t, double g2, double lzt_r, double lzt_c)
{
    const Lane me;
    const SweepArgs a = steps_args(sh);
    const bool acc = (a.va & VA_ACCEPT) != 0;
    if (me.t < kBR) {
        double s = -INFINITY, aa = -INFINITY;
        if (t.has_row(me)) {
            double z = sh.rz[t.at][me.t], p = sh.rp[t.at][me.t], lz = sh.rlz[t.at][me.t];
            if (acc) {
                z = fma(a.alpha_acc, p, z);
                lz = lzt_r;
                p = next_dir(a, p, sh.rlt[t.at][me.t], lz, 0.0, true);
                sh.rz[t.at][me.t] = z;
                sh.rp[t.at][me.t] = p;
                sh.rlz[t.at][me.t] = lz;
            }
            s = fma(a.alpha, p, lz);
            aa = Cost::row_term(g2, sh.rxx[t.at][me.t], (z - lz) * LOG2E_D);
        }
        sh.s[t.at][me.t] = s;
        sh.A[t.at][me.t] = aa;
    }
    double vv = -INFINITY;
    if (t.has_col(me)) {
        double z = sh.cz[t.at][me.t], p = sh.cp[t.at][me.t];
        if (acc) {
            z = fma(a.alpha_acc, p, z);
            p = next_dir(a, p, sh.clt[t.at][me.t], lzt_c, 0.0, false);
            sh.cz[t.at][me.t] = z;
            sh.cp[t.at][me.t] = p;
        }
        vv = fma(a.alpha, p, z) * LOG2E_D;
    }
    sh.colv[t.at][me.t] = vv;
}

// One finalize block (fin_lse_entry<8>): the pending update of its entries while the partials are
// on their way, then fold them and store log-sums and dots. kGuard: after a wait that ran out the dots are
// not stored, so that nobody takes results made of a value that never came (k_steps looks at the abort
// flag behind its last step instead; the flag in LDS costs it 1.5 % of a step).
template <bool kGuard, int NT>
__device__ __forceinline__ void steps_finalize(const StepSize& z, StepsX* x, StepsShared<NT>& sh, int b, bool e64, Wait& wait)
{
    double M = 0.0, xs[8];
    {
        const Lane me;
        if (me.q == 0) {
            const FinEntry f(z, me);
            const int nrt = z.nrt;
            const size_t st = f.row ? (size_t)z.m : (size_t)z.n;
            const double* base = (f.row ? sh.rowp[b] : sh.colp[b]) + f.k;
            double ts[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) ts[u] = (!f.row && me.lane + 64 * u < nrt) ? xload(&x->shift[b][me.lane + 64 * u]) : -INFINITY;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                xs[u] = (f.valid && f.l + u * f.L < f.np) ? xload(base + (size_t)(f.l + u * f.L) * st) : 0.0;
            clear_fin(sh, z, x, b == 2 ? 0 : b + 1);
            const SweepArgs a = steps_args(sh);
            if (f.own && (a.va & VA_ACCEPT)) {
                const double p = sh.fp[me.t], lz = sh.fl[me.t];
                sh.fz[me.t] = fma(a.alpha_acc, p, sh.fz[me.t]);
                sh.flz[me.t] = lz;
                sh.fp[me.t] = next_dir(a, p, sh.flt[me.t], lz, 0.0, f.row);
                sh.fg[me.t] = exp(lz) - sh.frt[me.t];
            }
            for (;;) {
                bool miss = false;
#pragma unroll
                for (int u = 0; u < 2; ++u) miss |= is_empty(ts[u]);
#pragma unroll
                for (int u = 0; u < 8; ++u) miss |= is_empty(xs[u]);
                if (!miss || !wait.again()) break;
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (is_empty(ts[u])) ts[u] = xload(&x->shift[b][me.lane + 64 * u]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (is_empty(xs[u])) xs[u] = xload(base + (size_t)(f.l + u * f.L) * st);
            }
            wave_drain();  // the emptied slots of the next turn
            if (kGuard && wait.dead) sh.dead = 1;
            if (!f.row) {
                M = wave_max(fmax(ts[0], ts[1]));
                if (me.t < nrt) sh.fac[me.t] = exp((me.t < 64 ? ts[0] : ts[1]) - M);
            }
        }
    }
    __syncthreads();
    {
        const Lane me;
        if (me.q == 0) {
            const FinEntry f(z, me);
            double v[kNDot];
#pragma unroll
            for (int d = 0; d < kNDot; ++d) v[d] = 0.0;
            double acc = 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (f.l + u * f.L < f.np)
                    acc = fma(xs[u], f.row ? 1.0 : sh.fac[min(f.l + u * f.L, kStepsMaxRowTiles - 1)], acc);
            const double sum = group_fold<0>(acc, f.L);
            if (f.own) {
                Entry e;
                e.p = sh.fp[me.t];
                e.lz = sh.flz[me.t];
                e.logt = sh.flt[me.t];
                e.rt = sh.frt[me.t];
                const double lg = f.row ? fma(steps_args(sh).alpha, e.p, e.lz) + log(sum) : M + log(sum);
                sh.fl[me.t] = lg;
                xstore((f.row ? sh.logr[b] : sh.logc[b]) + f.k, lg);
                const double gnew = exp(lg) - e.rt;
                lse_dots(e, gnew, gnew - sh.fg[me.t], lg, sum, e64, v);
            }
            // D_BAD counts, exactly: the number of lanes with a 1
            const double bad = (double)__popcll(__ballot(v[D_BAD] != 0.0));
            wave_sums<kStepDots>(v);
            if (me.lane == 0) {
#pragma unroll
                for (int d = 0; d < kStepDots; ++d) sh.red[d * 4 + me.wave] = v[d];
                sh.red[kStepDots * 4 + me.wave] = bad;
            }
        }
    }
    static_assert(D_BAD == kStepDots, "the dots of a step are the first ones");
    __syncthreads();
    const Lane me;
    if (me.q == 0 && me.t <= kStepDots && !(kGuard && sh.dead))
        xstore(&x->dots[b][z.blk][me.t], (sh.red[me.t * 4 + 0] + sh.red[me.t * 4 + 1]) + (sh.red[me.t * 4 + 2] + sh.red[me.t * 4 + 3]));
}

// All dots, 64 blocks per wave of the first quad: ask() starts the loads, take() waits and leaves
// them in LDS. One 128-byte line per block, read 16 bytes at a time with the agent-scope cache
// policy (each 8-byte half is one value, looked at by itself).
constexpr int kAgentScope = 16 | (int)0x80000000u;  // sc1 of a buffer load, and volatile
struct StepDots {
    static_assert((kStepDots + 1) % 2 == 0, "whole 16-byte loads");
    static constexpr int N = (kStepDots + 1) / 2;
    double2 y[N];
    bool mine;
    __device__ __forceinline__ void load(StepsX* x, int b, int vb)
    {
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(x->dots[b], (short)0, (int)sizeof x->dots[b], kBufDword3);
#pragma unroll
        for (int d = 0; d < N; ++d) {
            auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, vb * (int)sizeof x->dots[b][0] + d * 16, 0, kAgentScope);
            y[d] = *(double2*)&v;
        }
    }
    __device__ __forceinline__ bool missing() const
    {
        bool miss = false;
#pragma unroll
        for (int d = 0; d < N; ++d) miss |= is_empty(y[d].x) || is_empty(y[d].y);
        return miss;
    }
    __device__ __forceinline__ void ask(const StepSize& z, StepsX* x, int b)
    {
        const Lane me;
#pragma unroll
        for (int d = 0; d < N; ++d) y[d] = make_double2(0.0, 0.0);
        mine = me.q == 0 && me.wave * 64 < z.nvb;
        if (mine && me.t < z.nvb) load(x, b, me.t);
    }
    template <int NT>
    __device__ __forceinline__ void take(const StepSize& z, StepsX* x, StepsShared<NT>& sh, int b, Wait& wait)
    {
        if (!mine) return;
        const Lane me;
        while (missing() && wait.again()) load(x, b, me.t);
#pragma unroll
        for (int d = 0; d < N; ++d) {
            sh.y[2 * d][me.t] = y[d].x;
            sh.y[2 * d + 1][me.t] = y[d].y;
        }
    }
};

// The decision, in the first wave.
template <int NT>
__device__ __forceinline__ void steps_decide(const StepSize& z, StepsShared<NT>& sh, bool more)
{
    const int nvb = z.nvb;
    const Lane me;
    if ((me.q | me.wave) != 0) return;
    double v[kStepDots];
    bool bad = false;
#pragma unroll
    for (int d = 0; d < kStepDots; ++d) v[d] = 0.0;
    for (int u = 0; u * 64 < nvb; ++u) {
#pragma unroll
        for (int d = 0; d < kStepDots; ++d) v[d] += sh.y[d][u * 64 + me.lane];
        bad |= sh.y[kStepDots][u * 64 + me.lane] != 0.0;
    }
    wave_sums<kStepDots>(v);
    Trial t = sh.T;
    const bool decided = decide_trial(t, sh.P, v, __any(bad));
    if (me.lane == 0) {
        sh.T = t;
        sh.go = decided ? more : -1;
    }
}

// Make a register value opaque to the compiler, word by word.
template <class T>
__device__ __forceinline__ void opaque(T& v)
{
    uint32_t d[sizeof(T) / 4];
    __builtin_memcpy(d, &v, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) asm volatile("" : "+v"(d[i]));
    __builtin_memcpy(&v, d, sizeof(T));
}

template <class Cost, int TP>
struct TileCosts {
    Cost c[TP];
};
template <class Cost, int TP>
__device__ __forceinline__ TileCosts<Cost, TP> tile_costs(const Work& w, const StepTile* t)
{
    if constexpr (TP == 1) return {{Cost(w, t[0].i0)}};
    else return {{Cost(w, t[0].i0), Cost(w, t[1].i0)}};
}

// How the tiles' cost is held: in registers where it takes at most 128 of the 256 a thread has, else
// the rows are read again in every sweep, RB at a time.
template <class Cost, int TP>
struct StepKind {
    using Raw = typename Cost::Raw;
    static constexpr bool kPoints = std::is_same<Raw, int>::value;
    static constexpr bool kHold = !kPoints && sizeof(Raw) * TP <= 32;
    static constexpr int RB = kHold ? kRPW : (sizeof(Raw) <= 16 ? kRPW / 2 : kRPW / 4);
    static constexpr int kTiles = kHold ? TP : 1;  // tiles' worth of rows in registers
};

// The sweep of the workgroup's tiles (tile_lse, with the tiles' own state) from the set-up in LDS:
// weights, exponentials, and the partials stored in turn b's slots, which were emptied before.
template <class Cost, int NQ, int TP, class K = StepKind<Cost, TP>>
__device__ __forceinline__ void steps_sweep(StepsShared<NQ * TP>& sh, StepsX* x, const StepTile (&t)[TP], Cost* cost,
                                            typename Cost::Raw (&raw)[K::kTiles][K::RB], double g2, bool e64, int b)
{
    double SI[TP];
    {
        const Lane me;
#pragma unroll
        for (int u = 0; u < TP; ++u) SI[u] = wave_max(sh.s[t[u].at][me.lane]);
        // the weights of this wave's rows, kRPW lanes per tile
        const int u = TP > 1 ? (me.lane / kRPW) % TP : 0, r = me.wave * kRPW + me.lane % kRPW, at = me.q * TP + u;
        if (me.lane < TP * kRPW) sh.wt[at][r] = exp(sh.s[at][r] - (u == 0 ? SI[0] : SI[TP - 1]));
    }
#pragma unroll
    for (int u = 0; u < TP; ++u) {
        // ---- sweep (tile_lse, with the tile's own state)
        double rs = 0.0, col64[4] = {0, 0, 0, 0};
        const Lane me;
        Cost& c = cost[u];
        const double* A = sh.A[t[u].at] + t[u].rbase;
        const double* wts = sh.wt[t[u].at] + t[u].rbase;
        double* region = sh.region[t[u].at][me.wave];
        double V[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) V[k] = sh.colv[t[u].at][me.lane * 4 + k];
        c.bind_cols(g2, V);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if constexpr (K::kHold && TP > 1) {
            // or the entries' conversions to FP64 move out of the step loop, at two registers
            // each (with one tile that is welcome: there are registers for it)
#pragma unroll
            for (int r = 0; r < K::RB; ++r) opaque(raw[u][r]);
        }
        if (t[u].has) {
            if (!e64) {
                float col32[4] = {0, 0, 0, 0};
                float rp[kRPW];
#pragma unroll
                for (int b0 = 0; b0 < kRPW; b0 += K::RB) {
                    if constexpr (!K::kHold) {
                        c.template load<K::RB>(t[u].rbase + b0, t[u].J * kBC + me.lane * 4, raw[0]);
                    }
#pragma unroll
                    for (int r0 = 0; r0 < K::RB; ++r0) {
                        const int r = b0 + r0;
                        double xa[4];
                        if constexpr (K::kPoints) c.args(t[u].rbase + r, g2, V, A[r], xa);
                        else c.args(raw[K::kHold ? u : 0][r0], g2, V, A[r], xa);
                        const float wt = (float)wts[r];
                        float e[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) e[k] = __builtin_amdgcn_exp2f((float)xa[k]);
                        rp[r] = (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) col32[k] = fmaf(wt, e[k], col32[k]);
                        if ((r & 7) == 7) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                col64[k] += (double)col32[k];
                                col32[k] = 0.f;
                            }
                        }
                    }
                }
                rs = rows_reduce_f32(rp, (float*)region, me.lane);
            } else {
                double c9 = kExp2C9;
                asm volatile("" : "+v"(c9));
#pragma unroll
                for (int b0 = 0; b0 < kRPW; b0 += K::RB) {
                    if constexpr (!K::kHold) {
                        c.template load<K::RB>(t[u].rbase + b0, t[u].J * kBC + me.lane * 4, raw[0]);
                    }
#pragma unroll
                    for (int r0 = 0; r0 < K::RB; ++r0) {
                        const int r = b0 + r0;
                        if (r < t[u].nrows) {
                            double xa[4], e[4];
                            if constexpr (K::kPoints) c.args(t[u].rbase + r, g2, V, A[r], xa);
                            else c.args(raw[K::kHold ? u : 0][r0], g2, V, A[r], xa);
                            const double wt = wts[r];
                            exp2_f64x4(xa, e, c9);
                            region[(r & 7) * 64 + me.lane] = (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
                            for (int k = 0; k < 4; ++k) col64[k] = fma(wt, e[k], col64[k]);
                        }
                        if ((r & 7) == 7) {  // eight rows' partials are there: lanes of these rows sum them
                            __builtin_amdgcn_wave_barrier();
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                            const int rr = me.lane >> 2, hq = me.lane & 3;
                            if ((rr >> 3) == (r >> 3)) {
                                const double* src = region + (rr & 7) * 64 + hq * 16;
#pragma unroll
                                for (int k = 0; k < 16; ++k) rs += src[k ^ rr];
                            }
                            __builtin_amdgcn_wave_barrier();
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        }
                    }
                }
                rs += dpp_d<0xb1>(0.0, rs);  // quad_perm [1,0,3,2]
                rs += dpp_d<0x4e>(0.0, rs);  // quad_perm [2,3,0,1]
            }
        }
        // ---- publish the row partials; the slots of this turn were emptied before
        if (u == 0) wave_drain();
        if (t[u].has_prow(me)) xstore(row_slot(sh, t[u], me, b), rs);
        if (t[u].has_shift(me)) xstore(&x->shift[b][t[u].I], SI[u]);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int k = 0; k < 4; ++k) region[me.lane * 4 + k] = col64[k];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < TP; ++u) {  // and the column partials
        const Lane me;
        if (t[u].has_col(me)) {
            const double* r0 = sh.region[t[u].at][0] + me.t;
            const double c0 = r0[0], c1 = r0[kRowBufD], c2 = r0[2 * kRowBufD], c3 = r0[3 * kRowBufD];
            xstore(col_slot(sh, t[u], me, b), (c0 + c1) + (c2 + c3));
        }
    }
}

// The item a workgroup of a batched launch belongs to: the largest b with prefix[b] <= g.
__device__ __forceinline__ int batch_item(const int32_t* prefix, int nitems, int g)
{
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// NQ quads of TP tiles each, for one problem (wp), or for the problems in flight (bd): each has its
// own workgroups and its own exchange memory, and they go on independently of each other.
template <int CC, int NQ, int TP>
__global__ void __launch_bounds__(256 * NQ) k_steps(const Work* __restrict__ wp, const BatchDesc* __restrict__ bd,
                                                    StepsX* __restrict__ x, int max_steps)
{
    using Cost = typename CostOf<CC>::T;
    using K = StepKind<Cost, TP>;
    __shared__ StepsShared<NQ * TP> sh;

    int blk = blockIdx.x, nblk = gridDim.x;
    if (bd) {
        const int item = batch_item(bd->steps_prefix, bd->nitems, blk), first = bd->steps_prefix[item];
        nblk = bd->steps_prefix[item + 1] - first;
        blk -= first;
        wp = bd->items[item];
        x += item;
    }
    State* const S0 = state_slot(*wp, 0);
    if (!steps_go(*S0) || x->skip) return;  // the same in every workgroup

    // Work never changes while a kernel runs. Said so, its fields are read as scalars, which the
    // compiler otherwise gives up for a pointer that comes out of memory (+40 registers).
    uint64_t wa = reinterpret_cast<uint64_t>(wp);
    asm volatile("" : "+s"(wa));
    const Work& w = *(const Work*)(const __attribute__((address_space(4))) Work*)wa;
    const StepSize z(w, blk, nblk);
    const SweepArgs a0 = args_of(S0);  // the pending update
    const bool fin_wg = z.blk < z.nvb;
    const double g2 = S0->gamma * w.scale * LOG2E_D;
    if (threadIdx.x == 0) {
        Trial::copy(sh.T, *S0);
        sh.T.vec_action = 0;
        sh.P.set(params_of(*wp), *S0);
        sh.dead = 0;
        steps_slots(w, sh);
    }
    __syncthreads();
    StepTile t[TP];
    {
        const Lane me;
#pragma unroll
        for (int u = 0; u < TP; ++u) t[u].set(w, z.blk, NQ * TP, me.q * TP + u);
    }
    TileCosts<Cost, TP> cost = tile_costs<Cost, TP>(w, t);
    typename Cost::Raw raw[K::kTiles][K::RB];
    double lzt_r[TP], lzt_c[TP];  // trial log-sums of this thread's rows and columns
#pragma unroll
    for (int u = 0; u < TP; ++u) {
        const Lane me;
        Cost& c = cost.c[u];
        const int j0 = t[u].J * kBC + me.lane * 4;
        c.cols(j0);
        c.bind_rows(sh.x[t[u].at], sh.x[t[u].at] + 2 * kBR);
        if (me.t < kBR) sh.rxx[t[u].at][me.t] = c.row_fixed(me.t, t[u].i0 + me.t);
        c.cols_fixed(g2);
        if constexpr (K::kHold) {
            c.template load<K::RB>(t[u].rbase, j0, raw[u]);
        }
        lzt_r[u] = lzt_c[u] = 0.0;
        steps_load(w, a0, sh, t[u]);
        clear_tile(sh, x, t[u], 0);
        clear_tile(sh, x, t[u], 1);
    }
    if (fin_wg) clear_fin(sh, z, x, 0);

    wave_drain();
    __syncthreads();
    if (threadIdx.x == 0) sh.go = steps_meet(z, x);
    __syncthreads();
    const bool started = sh.go != 0;
    if (started && fin_wg) steps_load_fin(w, z, a0, sh);

    int last = 0;  // turn of the step that ended last
    for (int step = 0, b = 0; started; ++step, b = b == 2 ? 0 : b + 1) {
        // ---- pending update and tile set-up
#pragma unroll
        for (int u = 0; u < TP; ++u) steps_update<Cost>(sh, t[u], g2, lzt_r[u], lzt_c[u]);
        __syncthreads();
        const bool e64 = __builtin_amdgcn_readfirstlane(sh.T.exp64) != 0;
        steps_sweep<Cost, NQ, TP>(sh, x, t, cost.c, raw, g2, e64, b);
        // ---- finalize, decide
        Wait wait(x);
        if (fin_wg) steps_finalize<false>(z, x, sh, b, e64, wait);
        // the dots and this thread's log-sums are asked for first and looked at after the work that
        // need not wait for them
        StepDots dots;
        dots.ask(z, x, b);
#pragma unroll
        for (int u = 0; u < TP; ++u) {
            const Lane me;
            lzt_r[u] = t[u].has_row(me) ? xload(sh.logr[b] + t[u].i0 + me.t) : 0.0;
            lzt_c[u] = t[u].has_col(me) ? xload(sh.logc[b] + t[u].J * kBC + me.t) : 0.0;
        }
#pragma unroll
        for (int u = 0; u < TP; ++u) clear_tile(sh, x, t[u], b == 0 ? 2 : b - 1);  // the turn of the step after the next
        dots.take(z, x, sh, b, wait);
        if (z.nvb > 64) __syncthreads();  // uniform in the grid
        steps_decide(z, sh, step + 1 < max_steps);
        for (;;) {
            bool miss = false;
#pragma unroll
            for (int u = 0; u < TP; ++u) miss |= is_empty(lzt_c[u]) || is_empty(lzt_r[u]);
            if (!miss || !wait.again()) break;
#pragma unroll
            for (int u = 0; u < TP; ++u) {
                const Lane me;
                if (is_empty(lzt_c[u])) lzt_c[u] = xload(sh.logc[b] + t[u].J * kBC + me.t);
                if (is_empty(lzt_r[u])) lzt_r[u] = xload(sh.logr[b] + t[u].i0 + me.t);
            }
        }
        if (wait.dead) sh.dead = 1;
        __syncthreads();
        last = b;
        if (sh.go <= 0 || sh.dead) break;
    }

    // ---- what the one-step kernels go on from
    const Lane me;
    if (started) {
        if (fin_wg && !sh.dead) {
            const FinEntry f(z, me);
            if (f.own) {
                const int k = f.entry(z);
                w.z[k] = sh.fz[me.t];
                w.p[k] = sh.fp[me.t];
                w.lz[k] = sh.flz[me.t];
                w.g[k] = sh.fg[me.t];
                if (last != 2) xstore(w.lzt + k, sh.fl[me.t]);
            }
        }
        if (z.blk == 0 && me.q == 0 && sh.go < 0 && me.t < z.nvb) {  // the dots of the decision left open
            double* bd = bdots_of(*wp) + (size_t)me.t * kNDot;
#pragma unroll
            for (int d = 0; d < kNDot; ++d) bd[d] = d <= kStepDots ? sh.y[d][me.t] : 0.0;
        }
        if (z.blk == 0 && threadIdx.x == 0) {
            Trial::copy(*S0, sh.T);
            S0->undecided = sh.go < 0;
            if (sh.dead) {
                S0->done = 1;
                S0->status = MDOT_E_DEVICE;
            }
        }
    }
    steps_leave(z, x, !started);
}

// ------------------------------------------------------------------ resident standalone LSE
// mdot_lse2 of a problem of one or two tiles per workgroup, as one kernel: load the vectors
// and the cost, row maxima (where no shifts are given) with the cost range, sweep, finalize, again
// with FP64 exponentials where FP32 rows or columns left the range, outputs. As six kernels (n = 256)
// it is bound by their boundaries, and the cost is read twice; here the tiles are loaded once and the
// workgroups exchange row maxima, partials and dots as in k_steps. Same arithmetic, same bits.
// out->done stays 0 if the workgroups could not meet, and out->retry is set by any workgroup whose wait
// ran out (it leaves at once, so that no step is completed with what it did not get); the caller then
// takes the kernels.

// A caller's u, v or shift entry. Arithmetic hands the payload of a NaN on, and kEmpty is one: every
// NaN that comes in is replaced by the one arithmetic makes, or a reader would wait for a value that is
// there. So is the smallest entry of a tile of nothing but NaNs. (Other values made of a cost with NaNs
// lose them in minima, maxima and exponentials; a solve's vectors are made by the library.)
__device__ __forceinline__ double plain_nan(double v) { return v == v ? v : NAN; }

// Raw entries of row r of the tile (columns j0 ..): held, or recomputed from points.
template <class Cost, class K>
__device__ __forceinline__ void lse_row(const Cost& c, const StepTile& t, typename Cost::Raw (&raw)[K::kTiles][K::RB], int u,
                                        int r, int j0, double e[4])
{
    static_assert(K::kPoints || K::kHold, "the cost is read once");
    if constexpr (K::kPoints) c.row(t.rbase + r, j0, e);
    else c.decode(raw[u][r], e);
}

// Row i's shift: the largest of its tiles' maxima, as they arrive.
__device__ __forceinline__ double lse_shift(const Work& w, const StepSize& z, int i, Wait& wait)
{
    double mx = -INFINITY;
    for (int J0 = 0; J0 < z.nct; J0 += 8) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = J0 + k < z.nct ? xload(w.rowmin + (size_t)(J0 + k) * z.m + i) : -INFINITY;
        for (;;) {
            bool miss = false;
#pragma unroll
            for (int k = 0; k < 8; ++k) miss |= is_empty(v[k]);
            if (!miss || !wait.again()) break;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (is_empty(v[k])) v[k] = xload(w.rowmin + (size_t)(J0 + k) * z.m + i);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) mx = fmax(mx, v[k]);
    }
    return mx;
}

// Cost range over all tiles, as they arrive, with the whole workgroup.
template <int NT>
__device__ __forceinline__ void lse_range(StepsX* x, StepsShared<NT>& sh, int ntiles, int nq, Wait& wait, double* lo, double* hi)
{
    double a = INFINITY, b = -INFINITY;
    bool bad = false;
    for (int i = threadIdx.x; i < ntiles; i += 256 * nq) {
        double p = xload(&x->range[i][0]), q = xload(&x->range[i][1]);
        while ((is_empty(p) || is_empty(q)) && wait.again()) {
            p = xload(&x->range[i][0]);
            q = xload(&x->range[i][1]);
        }
        a = fmin(a, p);
        bad |= q != q;
        b = fmax(b, q);
    }
    a = wave_min(a);
    b = wave_max(b);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh.y[0][wv] = a;
        sh.y[1][wv] = b;
    }
    bad = __syncthreads_or(bad);
    a = sh.y[0][0];
    b = sh.y[1][0];
    for (int q = 1; q < 4 * nq; ++q) {
        a = fmin(a, sh.y[0][q]);
        b = fmax(b, sh.y[1][q]);
    }
    __syncthreads();
    *lo = a;
    *hi = bad ? NAN : b;
}

template <int CC, int NQ, int TP>
__global__ void __launch_bounds__(256 * NQ) k_lse(LseArgs A, StepsX* __restrict__ x)
{
    using Cost = typename CostOf<CC>::T;
    using K = StepKind<Cost, TP>;
    __shared__ StepsShared<NQ * TP> sh;

    const Work& w = A.w;
    const StepSize z(w, blockIdx.x, gridDim.x);
    const bool fin_wg = z.blk < z.nvb;
    if (threadIdx.x == 0) {
        sh.T = Trial{};
        sh.T.ls_phase = LS_STANDALONE;
        sh.dead = 0;
        steps_slots(w, sh);
    }
    __syncthreads();
    StepTile t[TP];
    {
        const Lane me;
#pragma unroll
        for (int u = 0; u < TP; ++u) t[u].set(w, z.blk, NQ * TP, me.q * TP + u);
    }
    // ---- empty the slots, announce this workgroup, load
    const int ntiles = z.nrt * z.nct;
#pragma unroll
    for (int u = 0; u < TP; ++u) {
        const Lane me;
        clear_tile(sh, x, t[u], 0);
        clear_tile(sh, x, t[u], 1);
        if (t[u].has_prow(me))
            xstore(w.rowmin + (size_t)t[u].J * z.m + (t[u].i0 + t[u].rbase) + (me.lane >> 2), empty_slot());
        if (t[u].has && me.t < 2) xstore(&x->range[t[u].I * z.nct + t[u].J][me.t], empty_slot());
    }
    if (fin_wg) clear_fin(sh, z, x, 0);
    wave_drain();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(&x->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    TileCosts<Cost, TP> cost = tile_costs<Cost, TP>(w, t);
    typename Cost::Raw raw[K::kTiles][K::RB];
#pragma unroll
    for (int u = 0; u < TP; ++u) {
        const Lane me;
        Cost& c = cost.c[u];
        const int j0 = t[u].J * kBC + me.lane * 4;
        c.cols(j0);
        c.bind_rows(sh.x[t[u].at], sh.x[t[u].at] + 2 * kBR);
        if (me.t < kBR) sh.rxx[t[u].at][me.t] = c.row_fixed(me.t, t[u].i0 + me.t);
        if constexpr (K::kHold) {
            c.template load<K::RB>(t[u].rbase, j0, raw[u]);
        }
        if (t[u].has_col(me)) sh.cz[t[u].at][me.t] = plain_nan(A.in.v[t[u].J * kBC + me.t]);
        if (t[u].has_row(me)) sh.rz[t[u].at][me.t] = plain_nan(A.in.u[t[u].i0 + me.t]);
    }
    if (fin_wg) {
        const Lane me;
        const FinEntry f(z, me);
        if (f.own) sh.fp[me.t] = sh.flz[me.t] = sh.flt[me.t] = sh.frt[me.t] = sh.fg[me.t] = 0.0;
    }
    if (threadIdx.x == 0) sh.go = steps_wait_all(z, x);
    __syncthreads();
    const bool started = sh.go != 0;
    Wait wait(x);
    if (started) {
        double scale = w.scale;
        // ---- cost range of the tiles; the scale first, where it follows from the range
#pragma unroll
        for (int u = 0; u < TP; ++u) {
            const Lane me;
            const int j0 = t[u].J * kBC + me.lane * 4;
            RangeOf<Cost> rg;
#pragma unroll
            for (int r = 0; r < kRPW; ++r)
                if (r < t[u].nrows) {
                    double e[4];
                    lse_row<Cost, K>(cost.c[u], t[u], raw, u, r, j0, e);
                    rg.add4(e, t[u].n - j0);
                }
            const double lo = wave_min((double)rg.lo), hi = wave_max((double)rg.hi);
            const bool bad = __any(rg.bad);
            if (me.lane == 0) {
                sh.y[0][t[u].at * 4 + me.wave] = lo;
                sh.y[1][t[u].at * 4 + me.wave] = bad ? NAN : hi;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < TP; ++u) {
            const Lane me;
            if (t[u].has && me.t == 0) {
                const double *lo = sh.y[0] + t[u].at * 4, *hi = sh.y[1] + t[u].at * 4;
                double a = lo[0], c = hi[0];
#pragma unroll
                for (int q = 1; q < 4; ++q) {
                    a = fmin(a, lo[q]);
                    c = (c != c || hi[q] != hi[q]) ? NAN : fmax(c, hi[q]);
                }
                double* dst = x->range[t[u].I * z.nct + t[u].J];
                xstore(dst, plain_nan(a));
                xstore(dst + 1, c);
            }
        }
        __syncthreads();
        if (A.choose) {
            double lo, hi;
            lse_range(x, sh, ntiles, NQ, wait, &lo, &hi);
            scale = hi > 0.0 ? 1.0 / hi : 1.0;
        }
        const double g2 = A.gamma * scale * LOG2E_D;
        // ---- row shifts: given, or the maxima of X_ij over the columns (k_row_max, k_fold_max)
        if (A.in.shift) {
#pragma unroll
            for (int u = 0; u < TP; ++u) {
                const Lane me;
                if (t[u].has_row(me)) sh.rlz[t[u].at][me.t] = plain_nan(A.in.shift[t[u].i0 + me.t]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < TP; ++u) {
                const Lane me;
                double* region = sh.region[t[u].at][me.wave];
                const int j0 = t[u].J * kBC + me.lane * 4;
                double V[4], mx = -INFINITY;
#pragma unroll
                for (int k = 0; k < 4; ++k) V[k] = j0 + k < t[u].n ? sh.cz[t[u].at][me.lane * 4 + k] * LOG2E_D : -INFINITY;
#pragma unroll
                for (int r = 0; r < kRPW; ++r) {
                    if (r < t[u].nrows) {
                        double e[4], m = -INFINITY;
                        lse_row<Cost, K>(cost.c[u], t[u], raw, u, r, j0, e);
#pragma unroll
                        for (int k = 0; k < 4; ++k) m = fmax(m, fma(-g2, e[k], V[k]));
                        region[(r & 7) * 64 + me.lane] = m;
                    }
                    if ((r & 7) == 7) {
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        const int rr = me.lane >> 2, hq = me.lane & 3;
                        if ((rr >> 3) == (r >> 3)) {
                            const double* src = region + (rr & 7) * 64 + hq * 16;
#pragma unroll
                            for (int k = 0; k < 16; ++k) mx = fmax(mx, src[k ^ rr]);
                        }
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    }
                }
                mx = fmax(mx, dpp_d<0xb1>(-INFINITY, mx));
                mx = fmax(mx, dpp_d<0x4e>(-INFINITY, mx));
                if (t[u].has_prow(me)) {
                    const int i = t[u].rbase + (me.lane >> 2);
                    xstore(w.rowmin + (size_t)t[u].J * z.m + t[u].i0 + i, fma(sh.rz[t[u].at][i], LOG2E_D, mx) * LN2_D);
                }
            }
#pragma unroll
            for (int u = 0; u < TP; ++u) {
                const Lane me;
                if (t[u].has_row(me)) sh.rlz[t[u].at][me.t] = lse_shift(w, z, t[u].i0 + me.t, wait);
            }
        }
        if (fin_wg) {
            const Lane me;
            const FinEntry f(z, me);
            if (f.own && f.row) sh.flz[me.t] = A.in.shift ? plain_nan(A.in.shift[f.k]) : lse_shift(w, z, f.k, wait);
        }
        // ---- tile set-up (steps_update with z = (u, v), p = 0)
        // a wait that ran out ends the workgroup's part: it publishes nothing from here on (the flag is set
        // again only behind the barriers of a sweep)
        if (wait.dead) sh.dead = 1;
        __syncthreads();
        bool e64 = A.e64 != 0, any = false, more = !sh.dead;
#pragma unroll
        for (int u = 0; u < TP; ++u) {
            const Lane me;
            cost.c[u].cols_fixed(g2);
            if (me.t < kBR) {
                const bool hr = t[u].has_row(me);
                const double lz = hr ? sh.rlz[t[u].at][me.t] : 0.0, zz = hr ? sh.rz[t[u].at][me.t] : 0.0;
                sh.s[t[u].at][me.t] = hr ? lz : -INFINITY;
                sh.A[t[u].at][me.t] = hr ? Cost::row_term(g2, sh.rxx[t[u].at][me.t], (zz - lz) * LOG2E_D) : -INFINITY;
            }
            sh.colv[t[u].at][me.t] = t[u].has_col(me) ? sh.cz[t[u].at][me.t] * LOG2E_D : -INFINITY;
        }
        __syncthreads();
        // ---- sweep, at most twice
        for (int b = 0; more; ++b) {
            steps_sweep<Cost, NQ, TP>(sh, x, t, cost.c, raw, g2, e64, b);
            if (fin_wg) steps_finalize<true>(z, x, sh, b, e64, wait);
            StepDots dots;
            dots.ask(z, x, b);
            dots.take(z, x, sh, b, wait);
            if (wait.dead) sh.dead = 1;
            __syncthreads();
            any = false;
            for (int i = threadIdx.x; i < z.nvb; i += blockDim.x) any |= sh.y[kStepDots][i] != 0.0;
            any = __syncthreads_or(any);
            more = any && !e64 && !sh.dead;
            e64 = true;
        }
        // ---- outputs, if every entry of the scaled cost lies in [0, 1]
        if ((fin_wg || z.blk == 0) && !sh.dead) {
            double lo, hi;
            lse_range(x, sh, ntiles, NQ, wait, &lo, &hi);
            if (wait.dead) sh.dead = 1;
            __syncthreads();
            const bool dead = sh.dead != 0, valid = range_valid(scale, lo, hi);
            if (fin_wg && valid && !dead) {
                const Lane me;
                const FinEntry f(z, me);
                if (f.own) (f.row ? A.lr_out : A.lc_out)[f.k] = sh.fl[me.t];
            }
            if (z.blk == 0 && threadIdx.x == 0 && !dead) {
                A.out->valid = valid;
                A.out->status = any ? MDOT_W_RANGE : MDOT_OK;
                A.out->scale = scale;
                A.out->done = 1;
            }
        }
        if (threadIdx.x == 0 && sh.dead) A.out->retry = 1;
    }
    steps_leave(z, x);
}

// ------------------------------------------------------------------ batched kernels
// Batched sweep: one workgroup per tile of the problems in flight that need this kernel
// instance (the descriptor's tiles [tile_begin, tile_end), launched exactly), tiles of problems
// that share a cost interleaved so that they meet in one XCD's L2 (ranges start at multiples of
// 8). Same register cap as the single-problem sweep; a grid-stride loop here would keep the
// loop-invariant values of the tile code live across tiles and spill.
template <int CC>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(CC >= kOccHi ? 2 : 4)))
k_sweep_batch(const BatchDesc* __restrict__ bd, int parity, int tile_begin, int tile_end)
{
    __shared__ double smem[kSmemAll];
    const int g = tile_begin + (int)blockIdx.x;
    if (g >= tile_end) return;
    const int q = batch_item(bd->grp_prefix, bd->ngroups, g);
    const int l = g - bd->grp_prefix[q];
    const int K = bd->grp_size[q], T = bd->grp_tiles[q];
    const int run = l >> 3, k = run % K;
    const int t = (run / K) * 8 + (l & 7);
    if (t >= T) return;
    sweep_any<CC>(*bd->items[bd->grp_items[bd->grp_first[q] + k]], parity, t, smem);
}

// Batched finalize: one workgroup per finalize block of every problem in flight.
template <int V>
__global__ void __launch_bounds__(kVecWG, V == kFinMid ? 2 : 1) k_fin_batch(const BatchDesc* __restrict__ bd, int parity)
{
    __shared__ FinShared sh;
    const int g = blockIdx.x;
    if (g >= bd->total_fin) return;
    const int b = batch_item(bd->fin_prefix, bd->nitems, g);
    fin_body<V>(*bd->items[b], parity, g - bd->fin_prefix[b], bd->fin_prefix[b + 1] - bd->fin_prefix[b], sh);
}

__global__ void __launch_bounds__(kDecideWG) k_decide_batch(const BatchDesc* __restrict__ bd, int parity)
{
    for (int b = blockIdx.x; b < bd->nitems; b += gridDim.x) decide_body(*bd->items[b], parity, parity ^ 1);
}

// k_settle of every item. A wait that ran out (StepsX::abort) ends its solve with an error.
__global__ void __launch_bounds__(kDecideWG) k_settle_batch(const BatchDesc* __restrict__ bd, StepsX* __restrict__ x)
{
    const int b = blockIdx.x;
    if (b >= bd->nitems) return;
    State* S = state_slot(*bd->items[b], 0);
    const bool dead = x[b].abort != 0;
    if (!dead && S->undecided) decide_body(*bd->items[b], 0, 0);
    if (dead && threadIdx.x == 0) {
        x[b].abort = 0;
        S->done = 1;
        S->status = MDOT_E_DEVICE;
    }
}

// kChunkMissed if a meeting failed in this chunk; the next one may try again.
__device__ __forceinline__ int chunk_missed(StepsX* x)
{
    if (!x || !x->skip) return 0;
    x->skip = 0;
    return kChunkMissed;
}

// End-of-chunk done flags and step counts, written straight into pinned host memory (a stream-ordered copy
// between chunks would stall the stream for tens of microseconds). The chunk counter *seq,
// kept on the device, picks the host buffer: chunk s writes buffer s & 1, so the chunk queued
// behind it never overwrites flags the host has not read yet.
__global__ void k_gather_done(const BatchDesc* __restrict__ bd, StepsX* x, int* out, int* seq)
{
    const int b = threadIdx.x;  // one wave: every lane reads the counter before lane 0 advances it
    const int s = *seq;
    if (b < bd->nitems) {
        const State& S = bd->items[b]->st[0];
        out[(s & 1) * kMaxBatch + b] = S.done + chunk_missed(x ? x + b : nullptr);
        out[(2 + (s & 1)) * kMaxBatch + b] = (int)(S.sweeps + S.fallbacks + S.cert_sweeps);
    }
    if (b == 0) *seq = s + 1;
}

__global__ void k_chunk_done(const Work* __restrict__ wp, StepsX* x, int* out, int* seq)
{
    const int s = *seq;
    out[s & 1] = ctl_of(*wp).st[0].done + chunk_missed(x);
    *seq = s + 1;
}

// ------------------------------------------------------------------ standalone sweeps
// mdot_lse2 and mdot_round_certify on given potentials, with no host round trip between their
// kernels:
//   k_alone_setup  control block, z = (u, v), shifts, zeros (and bounds of a point cloud)
//   k_row_max      without given shifts: row maxima of X_ij per tile, and the raw cost range
//   k_fold_max     row maxima -> shifts; its last workgroup reduces the range
//   sweep, k_fin   the solver's kernels (k_sweep_range where the range is still unknown)
//   k_alone_out    range verdict, out-of-range rows, outputs, summary in host memory
// The cost has to lie in [0, 1] after scaling, which takes every entry; its smallest and largest
// raw value come out of a pass that reads it anyway, and outputs are written only if they do.
// A point cloud whose bounding boxes already bound scale * distance by 1 needs no such pass.

// Range of one tile over the workgroup -> part[0..1] ({lo, hi}; hi NaN with a non-finite entry).
template <class R>
__device__ __forceinline__ void block_range(const R& rg, double* part, int tid, double* sred)
{
    const double lo = wave_min((double)rg.lo), hi = wave_max((double)rg.hi);
    const bool bad = __any(rg.bad);
    __syncthreads();
    if ((tid & 63) == 0) {
        sred[tid >> 6] = lo;
        sred[4 + (tid >> 6)] = bad ? NAN : hi;
    }
    __syncthreads();
    if (tid == 0) {
        double a = sred[0], b = sred[4];
        for (int q = 1; q < 4; ++q) {
            a = fmin(a, sred[q]);
            b = (b != b || sred[4 + q] != sred[4 + q]) ? NAN : fmax(b, sred[4 + q]);
        }
        part[0] = a;
        part[1] = b;
    }
}

// Reduce the tiles' ranges with the whole workgroup; every thread returns the result.
__device__ __forceinline__ void reduce_range(const double* part, int ntiles, double* lo, double* hi, double* sred)
{
    const int tid = threadIdx.x, nw = blockDim.x >> 6;
    double a = INFINITY, b = -INFINITY;
    bool bad = false;
#pragma unroll 8
    for (int t = tid; t < ntiles; t += blockDim.x) {
        const double2 p = ((const double2*)part)[t];
        a = fmin(a, p.x);
        bad |= p.y != p.y;
        b = fmax(b, p.y);
    }
    a = wave_min(a);
    b = wave_max(b);
    bad = __any(bad);
    if ((tid & 63) == 0) {
        sred[tid >> 6] = a;
        sred[16 + (tid >> 6)] = bad ? NAN : b;
    }
    __syncthreads();
    a = sred[0];
    b = sred[16];
    for (int q = 1; q < nw; ++q) {
        a = fmin(a, sred[q]);
        b = (b != b || sred[16 + q] != sred[16 + q]) ? NAN : fmax(b, sred[16 + q]);
    }
    __syncthreads();
    *lo = a;
    *hi = b;
}

// Bounding boxes of the two point sets, from the kBoxBlocks partial boxes k_alone_setup left at
// `box` ([block][set][lo, hi][8 coordinates]): true if they bound scale * distance by 1, with
// every coordinate finite. |x - y| and the sums below round monotonically and in the order of
// PointCost::decode, so no entry can exceed the bound.
__device__ __forceinline__ bool box_settles(const double* box, int d, int kind, double scale)
{
    const int lane = threadIdx.x & 63;
    static_assert(kBoxBlocks <= 64, "one lane per partial box");
    double s = 0.0;
    for (int e = 0; e < d; ++e) {
        const bool in = lane < kBoxBlocks;
        const double* b = box + (size_t)lane * 32;
        const double xlo = wave_min(in ? b[e] : INFINITY), xhi = wave_max(in ? b[8 + e] : -INFINITY);
        const double ylo = wave_min(in ? b[16 + e] : INFINITY), yhi = wave_max(in ? b[24 + e] : -INFINITY);
        const double t = fmax(fabs(xhi - ylo), fabs(yhi - xlo));
        s = kind == MDOT_COST_POINTS_SQEUCLID ? fma(t, t, s) : s + t;
    }
    return scale * s <= 1.0;  // false for infinity (a non-finite coordinate makes its box infinite) and NaN
}

__global__ void __launch_bounds__(256) k_alone_setup(Control* __restrict__ ctl, Work w, State s, DevParams prm, AloneIn in,
                                                     int fill_blocks)
{
    const int tid = threadIdx.x, m = w.m, n = w.n;
    if ((int)blockIdx.x >= fill_blocks) {  // bounding boxes of a slice of the points
        const float* X = (const float*)w.cost;
        const int b = blockIdx.x - fill_blocks, d = w.d;
        __shared__ double sred[4][2];
        double* box = ctl->bdots + (size_t)b * 32;
        for (int set = 0; set < 2; ++set) {
            const int cnt = set ? n : m;
            const float* P = X + (set ? (size_t)m * d : 0);
            for (int e = 0; e < d; ++e) {
                float lo = INFINITY, hi = -INFINITY;
                bool bad = false;
                for (int i = b * 256 + tid; i < cnt; i += kBoxBlocks * 256) {
                    const float v = P[(size_t)i * d + e];
                    bad |= !isfinite(v);
                    lo = fminf(lo, v);
                    hi = fmaxf(hi, v);
                }
                const double l = wave_min((double)lo), h = wave_max((double)hi);
                bad = __any(bad);
                if ((tid & 63) == 0) {
                    sred[tid >> 6][0] = l;
                    sred[tid >> 6][1] = bad ? NAN : h;
                }
                __syncthreads();
                if (tid == 0) {
                    double a = sred[0][0], c = sred[0][1];
                    bool nan = c != c;
                    for (int q = 1; q < 4; ++q) {
                        a = fmin(a, sred[q][0]);
                        nan |= sred[q][1] != sred[q][1];
                        c = fmax(c, sred[q][1]);
                    }
                    // a non-finite coordinate: an infinite box settles nothing
                    box[set * 16 + e] = nan ? -INFINITY : a;
                    box[set * 16 + 8 + e] = nan ? INFINITY : c;
                }
                __syncthreads();
            }
        }
        return;
    }
    if (blockIdx.x == 0) {
        if (tid == 0) ctl->w = w;
        if (tid == 64) ctl->st[0] = s;
        if (tid == 128) ctl->prm = prm;
    }
    const int k = blockIdx.x * 256 + tid;
    if (k >= m + n) return;
    const bool row = k < m;
    const int j = k - m;
    w.rt[k] = 0.0;
    w.logt[k] = 0.0;
    w.z[k] = row ? in.u[k] : in.v[j];
    w.zprev[k] = in.u_prev ? (row ? in.u_prev[k] : in.v_prev[j]) : 0.0;
    w.zbest[k] = 0.0;
    w.p[k] = 0.0;
    w.g[k] = 0.0;
    w.lz[k] = (row && in.shift) ? in.shift[k] : 0.0;
    w.lzt[k] = 0.0;
    if (row) w.xr[k] = 0.0;
    else {
        w.yc[j] = 0.0;
        w.errc[j] = 0.0;
    }
}

// Row maxima of X_ij = u_i + v_j - gamma C_ij over one tile, and the tile's raw cost range. The
// row term is added to the maximum over the columns: rounding is monotone, so it is the maximum
// of the rounded sums (any shift near the maximum serves). Bound by the read of the cost: every row of a wave is in flight before the
// first is used (32-byte rows eight at a time), and the lanes' maxima meet once per 16 rows, in LDS.
// n = 16384 FP32: 191 us (5.6 TB/s); with a row per load, a wave reduction per row and the range in
// a pass of its own it was 318 + 194 us.
template <int CC>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(4)))
k_row_max(const Work* __restrict__ wp, double* __restrict__ part)
{
    using Cost = typename CostOf<CC>::T;
    __shared__ double smem[4 * kRPW * 64];
    const Work& w = *wp;
    const double gamma = ctl_of(w).st[0].gamma;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int I = blockIdx.x / w.nct, J = blockIdx.x % w.nct, i0 = I * kBR, j0 = J * kBC + lane * 4;
    const int m = w.m, n = w.n, rbase = wave * kRPW, nrows = min(kRPW, m - (i0 + rbase));
    const double g2 = gamma * w.scale * LOG2E_D;
    Cost cost(w, i0);
    cost.cols(j0);
    constexpr bool kPoints = std::is_same<typename Cost::Raw, int>::value;
    constexpr int RB = kPoints ? 1 : (sizeof(typename Cost::Raw) <= 16 ? kRPW : kRPW / 2);
    double V[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) V[k] = (j0 + k < n) ? w.z[m + j0 + k] * LOG2E_D : -INFINITY;
    RangeOf<Cost> rg;
    double* mine = smem + wave * kRPW * 64;
    auto take = [&](int r, const double c[4]) {
        rg.add4(c, n - j0);
        double mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) mx = fmax(mx, fma(-g2, c[k], V[k]));
        mine[r * 64 + lane] = mx;
    };
    if constexpr (kPoints) {
        for (int r = 0; r < nrows; ++r) {
            double c[4];
            cost.row(rbase + r, j0, c);
            take(r, c);
        }
    } else {
#pragma unroll
        for (int b = 0; b < kRPW; b += RB) {
            typename Cost::Raw raw[RB];
            cost.template load<RB>(rbase + b, j0, raw);
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (b + r < nrows) {
                    double c[4];
                    cost.decode(raw[r], c);
                    take(b + r, c);
                }
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // four lanes per row, each in the order k ^ row, so that the reads hit distinct banks
    const int rr = lane >> 2, q = lane & 3;
    double mx = -INFINITY;
    if (rr < nrows) {
#pragma unroll
        for (int k = 0; k < 16; ++k) mx = fmax(mx, mine[rr * 64 + q * 16 + (k ^ rr)]);
    }
    mx = fmax(mx, dpp_d<0xb1>(-INFINITY, mx));  // quad_perm [1,0,3,2]
    mx = fmax(mx, dpp_d<0x4e>(-INFINITY, mx));  // quad_perm [2,3,0,1]
    if (q == 0 && rr < nrows) {
        const int i = i0 + rbase + rr;
        w.rowmin[(size_t)J * m + i] = fma(w.z[i], LOG2E_D, mx) * LN2_D;
    }
    block_range(rg, part + 2 * blockIdx.x, tid, smem);
}

// Row shifts = maxima over the column tiles, four threads per row; the last workgroup reduces the
// cost range. A chain of loads per thread is what takes the time: with one thread per row (and 256
// threads for the range) n = 16384 took 27 us, 12 us now.
__global__ void __launch_bounds__(1024) k_fold_max(const Work* __restrict__ wp, const double* __restrict__ part)
{
    __shared__ double sred[1024];
    const Work& w = *wp;
    const int m = w.m, nct = w.nct, tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        double lo, hi;
        reduce_range(part, w.nrt * nct, &lo, &hi, sred);
        if (tid == 0) {
            ctl_of(w).range[0] = lo;
            ctl_of(w).range[1] = hi;
        }
        return;
    }
    const int i = blockIdx.x * 256 + (tid & 255);
    double mx = -INFINITY;
    if (i < m) {
#pragma unroll 8
        for (int J = tid >> 8; J < nct; J += 4) mx = fmax(mx, w.rowmin[(size_t)J * m + i]);
    }
    sred[tid] = mx;
    __syncthreads();
    if (tid < 256 && i < m) w.lz[i] = fmax(fmax(mx, sred[tid + 256]), fmax(sred[tid + 512], sred[tid + 768]));
}

// Range of a point cloud whose scale the library chooses (1 / the largest raw value).
__global__ void __launch_bounds__(1024) k_pick_scale(Work* __restrict__ wp, const double* __restrict__ part)
{
    __shared__ double sred[32];
    double lo, hi;
    reduce_range(part, wp->nrt * wp->nct, &lo, &hi, sred);
    if (threadIdx.x == 0) wp->scale = hi > 0.0 ? 1.0 / hi : 1.0;
}

// The LSE sweep of a dense cost whose range is still unknown (shifts given by the caller).
template <int CC>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(4)))
k_sweep_range(const Work* __restrict__ wp, double* __restrict__ part)
{
    using Cost = typename CostOf<CC>::T;
    __shared__ double smem[kSmemAll];
    const Work& w = *wp;
    const State* Sp = state_slot(w, 0);
    const SweepArgs a = args_of(Sp);
    const TileCtx t = tile_ctx(w, blockIdx.x);
    RangeOf<Cost> rg;
    if (Sp->exp64 != 0) tile_lse<Cost, true, true>(w, a, t, smem, &rg);
    else tile_lse<Cost, false, true>(w, a, t, smem, &rg);
    block_range(rg, part + 2 * blockIdx.x, t.tid, smem);
}

// End of a standalone call: check the scaled cost range (`where` it is found), then for an LSE
// (run with FP64 exponentials if e64) look for rows and columns out of range and copy the log-sums
// out, or ask for the FP64 re-run, which reads state slot 0; for a certificate report the final
// state in slot `slot`. Every workgroup forms the verdict and copies its share; the first reports.
__global__ void __launch_bounds__(1024) k_alone_out(Work* __restrict__ wp, int slot, const double* __restrict__ part,
                                                    int where, int lse, int e64, double* __restrict__ lr_out,
                                                    double* __restrict__ lc_out, AloneOut* __restrict__ out)
{
    __shared__ double sred[32];
    const Work& w = *wp;
    Control& C = ctl_of(w);
    const int tid = threadIdx.x, m = w.m, n = w.n;
    double lo = C.range[0], hi = C.range[1];
    const double scale = w.scale;
    if (where == kRangeBox && C.range[2] != 0.0) lo = hi = 0.0;  // settled by the boxes
    else if (where != kRangeDone) reduce_range(part, w.nrt * w.nct, &lo, &hi, sred);
    const bool valid = range_valid(scale, lo, hi);
    const State& S = C.st[slot];
    int status = S.status, retry = 0;
    if (lse) {
        const bool any = __syncthreads_or(tid < w.fin_nblk && C.bdots[(size_t)tid * kNDot + D_BAD] != 0.0);
        static_assert(kFinMaxGrid <= 1024, "one thread per finalize workgroup");
        retry = any && !e64;
        status = any ? MDOT_W_RANGE : MDOT_OK;
        if (valid && !retry && lr_out) {
            const int step = gridDim.x * 1024;
            for (int k = blockIdx.x * 1024 + tid; k < m + n; k += step) *(k < m ? lr_out + k : lc_out + (k - m)) = w.lzt[k];
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
        out->valid = valid;
        out->retry = retry;
        out->status = status;
        out->scale = scale;
        out->ub = S.best_ub;
        out->lb = S.best_lb;
        out->me = S.best_me;
        out->done = S.done;
        if (retry) C.st[0].exp64 = 1;
    }
}

// ------------------------------------------------------------------ set-up kernels
__global__ void k_init(const Work* __restrict__ wp)
{
    const Work w = *wp;
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const DevParams P = *w.prm;
    State S;
    memset(&S, 0, sizeof(S));
    S.stage = 1;
    S.gamma = fmin(P.gamma_i, P.gamma_f);
    S.gamma_prev = 0.0;
    S.eps_d = P.hterm / pow(S.gamma, P.p);
    S.w = P.smooth_fixed ? P.w_fixed : fmin(S.eps_d / 4.0, 0.5);
    S.tol = fmax(S.eps_d / 2.0, P.tol_floor);
    S.ws_scale = 1.0;
    S.f32_floor = P.f32_min_tol;
    S.on_proxy = P.mix_gamma > 0.0 && S.gamma <= P.mix_gamma;
    S.exp64_stage = P.exp64_default || S.tol < S.f32_floor;
    S.exp64 = S.exp64_stage;
    S.alpha_prev = 1.0;
    S.vec_action = VA_STAGE_INIT;
    S.sweep_mode = SM_LSE;
    S.ls_phase = LS_INIT;
    S.best_ub = INFINITY;
    S.best_lb = -INFINITY;
    S.best_gamma = S.gamma;
    w.st[0] = S;
    w.st[1] = S;
}

// Intake statistics: out8 = {sum r, sum c, min r, min c, H(r), H(c), nonfinite count, 0}
__global__ void k_intake(const Work* __restrict__ wp, double* out8)
{
    const Work w = *wp;
    __shared__ double sred[8][kWG];
    const int m = w.m, n = w.n, t = threadIdx.x;
    double sr = 0, sc = 0, mr = INFINITY, mc = INFINITY, hr = 0, hc = 0, bad = 0;
    for (int i = t; i < m; i += kWG) {
        const double a = w.r[i];
        if (!isfinite(a)) bad += 1;
        sr += a;
        mr = fmin(mr, a);
        if (a > 0) hr -= a * log(a);
    }
    for (int j = t; j < n; j += kWG) {
        const double b = w.c[j];
        if (!isfinite(b)) bad += 1;
        sc += b;
        mc = fmin(mc, b);
        if (b > 0) hc -= b * log(b);
    }
    sred[0][t] = sr; sred[1][t] = sc; sred[2][t] = mr; sred[3][t] = mc;
    sred[4][t] = hr; sred[5][t] = hc; sred[6][t] = bad; sred[7][t] = 0;
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if (t < h) {
            for (int d = 0; d < 8; ++d) {
                if (d == 2 || d == 3) sred[d][t] = fmin(sred[d][t], sred[d][t + h]);
                else sred[d][t] += sred[d][t + h];
            }
        }
        __syncthreads();
    }
    if (t < 8) out8[t] = sred[t][0];
}

// Cost range over a dense matrix or the maximum raw point distance: out2 = {min, max} of raw
// values (non-finite entries make max NaN).
template <class Cost>
__device__ void cost_range_body(const Work& w, int tile, double* mn, double* mx)
{
    const int m = w.m, n = w.n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int I = tile / w.nct, J = tile % w.nct;
    const int j0 = J * kBC + lane * 4;
    Cost cost(w, I * kBR);
    cost.cols(j0);
    double lo = INFINITY, hi = -INFINITY;
    for (int rr = 0; rr < kRPW; ++rr) {
        const int i = I * kBR + wave * kRPW + rr;
        if (i >= m) break;
        double c[4];
        cost.row(wave * kRPW + rr, j0, c);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j0 + k < n) {
                if (!isfinite(c[k])) hi = NAN;
                lo = fmin(lo, c[k]);
                hi = (hi != hi) ? hi : fmax(hi, c[k]);
            }
    }
    *mn = lo;
    *mx = hi;
}

// `box`: the workgroups first look at the point cloud's bounding boxes, and return if these
// settle that the cost is in range (workgroup 0 notes it for k_alone_out).
template <int CC>
__global__ void __launch_bounds__(kWG) k_cost_range(const Work* __restrict__ wp, double* part, int box)
{
    const Work w = *wp;
    if (box) {
        const bool settled = box_settles(ctl_of(*wp).bdots, w.d, w.cost_kind, w.scale);
        if (blockIdx.x == 0 && threadIdx.x == 0) ctl_of(*wp).range[2] = settled ? 1.0 : 0.0;
        if (settled) return;
    }
    __shared__ double s0[kWG], s1[kWG];
    const int t = threadIdx.x;
    for (int tile = blockIdx.x; tile < w.nrt * w.nct; tile += gridDim.x) {
        double lo, hi;
        cost_range_body<typename CostOf<base_code(CC)>::T>(w, tile, &lo, &hi);
        s0[t] = lo;
        s1[t] = hi;
        __syncthreads();
        for (int h = kWG / 2; h > 0; h >>= 1) {
            if (t < h) {
                s0[t] = fmin(s0[t], s0[t + h]);
                double a = s1[t], b = s1[t + h];
                s1[t] = (a != a || b != b) ? NAN : fmax(a, b);
            }
            __syncthreads();
        }
        if (t == 0) {
            part[2 * tile] = s0[0];
            part[2 * tile + 1] = s1[0];
        }
        __syncthreads();
    }
}

// Copy the reported potentials out, gauge-fixed so that sum(u) = sum(v) (the dual is
// invariant under (u + delta, v - delta), paper Sec. 4.1 footnote). Reads the newest state
// (slot 0 after an even number of steps): when the save of the best potentials is still
// pending there, they are the accepted iterate of that state.
__device__ __forceinline__ double best_entry(const Work& w, const SweepArgs& a, int k)
{
    return (a.va & VA_SAVE_BEST) ? entry_after(w, a, k).zacc : w.zbest[k];
}

__global__ void k_finish(const Work* __restrict__ wp, double* u_out, double* v_out)
{
    __shared__ double sred[kWG];
    __shared__ double sdelta;
    const Work& w = *wp;
    const SweepArgs a = args_of(w.st);
    const int m = w.m, n = w.n, t = threadIdx.x;
    const int mx = m > n ? m : n;
    double s = 0.0;
    for (int i = t; i < mx; i += kWG) s += (i < n ? best_entry(w, a, m + i) : 0.0) - (i < m ? best_entry(w, a, i) : 0.0);
    sred[t] = s;
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if (t < h) sred[t] += sred[t + h];
        __syncthreads();
    }
    if (t == 0) sdelta = sred[0] / (double)(m + n);
    __syncthreads();
    const double dl = sdelta;
    for (int i = t; i < m; i += kWG)
        if (u_out) u_out[i] = best_entry(w, a, i) + dl;
    for (int j = t; j < n; j += kWG)
        if (v_out) v_out[j] = best_entry(w, a, m + j) - dl;
}

// ------------------------------------------------------------------ launchers
int cost_code_of(int cost_kind, int dtype)
{
    if (cost_kind == MDOT_COST_POINTS_SQEUCLID) return CC_PTS_SQ;
    if (cost_kind == MDOT_COST_POINTS_L1) return CC_PTS_L1;
    switch (dtype) {
        case MDOT_DT_F64: return CC_F64;
        case MDOT_DT_F16: return CC_F16;
        case MDOT_DT_BF16: return CC_BF16;
        default: return CC_F32;
    }
}

int cost_code_dim(int cc, int d)
{
    if (cc == CC_PTS_SQ) return d <= 2 ? CC_PTS_SQ2 : (d <= 3 ? CC_PTS_SQ : CC_PTS_SQ8);
    if (cc == CC_PTS_L1) return d <= 2 ? CC_PTS_L12 : (d <= 3 ? CC_PTS_L1 : CC_PTS_L18);
    return cc;
}

// Kernel instance of a launch: point clouds take the instance for their dimension, and the
// tuning table's 2-waves-per-SIMD variant adds kOccHi (of the 8-coordinate instances the one without
// spills; elsewhere the same kernel).
int cost_code(const Work& w)
{
    return cost_code_dim(cost_code_of(w.cost_kind, w.dtype), w.d) + (w.occ2 ? kOccHi : 0);
}

#define MDOT_CC_SWITCH_BASE(cc, F)                                     \
    switch (cc) {                                                      \
        case CC_F64: F(CC_F64); break;                                 \
        case CC_F32: F(CC_F32); break;                                 \
        case CC_F16: F(CC_F16); break;                                 \
        case CC_BF16: F(CC_BF16); break;                               \
        case CC_PTS_SQ: F(CC_PTS_SQ); break;                           \
        case CC_PTS_SQ2: F(CC_PTS_SQ2); break;                         \
        case CC_PTS_L12: F(CC_PTS_L12); break;                         \
        case CC_PTS_L1: F(CC_PTS_L1); break;                           \
        case CC_PTS_SQ8: F(CC_PTS_SQ8); break;                         \
        default: F(CC_PTS_L18); break;                                 \
    }

#define MDOT_CC_SWITCH(cc, F)                                          \
    switch (cc) {                                                      \
        case CC_F64: F(CC_F64); break;                                 \
        case CC_F32: F(CC_F32); break;                                 \
        case CC_F16: F(CC_F16); break;                                 \
        case CC_BF16: F(CC_BF16); break;                               \
        case CC_PTS_SQ: F(CC_PTS_SQ); break;                           \
        case CC_PTS_SQ2: F(CC_PTS_SQ2); break;                         \
        case CC_PTS_L12: F(CC_PTS_L12); break;                         \
        case CC_PTS_L1: F(CC_PTS_L1); break;                           \
        case CC_PTS_SQ8: F(CC_PTS_SQ8); break;                         \
        case CC_PTS_L18: F(CC_PTS_L18); break;                         \
        case kOccHi + CC_F64: F(CC_F64); break;                        \
        case kOccHi + CC_F32: F(CC_F32); break;                        \
        case kOccHi + CC_F16: F(CC_F16); break;                        \
        case kOccHi + CC_BF16: F(CC_BF16); break;                      \
        case kOccHi + CC_PTS_SQ: F(CC_PTS_SQ); break;                  \
        case kOccHi + CC_PTS_SQ2: F(CC_PTS_SQ2); break;                \
        case kOccHi + CC_PTS_L12: F(CC_PTS_L12); break;                \
        case kOccHi + CC_PTS_L1: F(CC_PTS_L1); break;                  \
        case kOccHi + CC_PTS_SQ8: F(kOccHi + CC_PTS_SQ8); break;       \
        default: F(kOccHi + CC_PTS_L18); break;                        \
    }

int launch_finalize(const Work& hw, const Work* wd, int parity, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const int xcd = hw.fin_L >= 16 && hw.fin_nblk % 8 == 0;
    const int fv = fin_instance(hw.fin_per, hw.nrt);
    if (fv == kFinSmall) hipLaunchKernelGGL(k_fin<kFinSmall>, dim3(hw.fin_nblk), dim3(kVecWG), 0, s, wd, parity, xcd);
    else if (fv == kFinMid) hipLaunchKernelGGL(k_fin<kFinMid>, dim3(hw.fin_nblk), dim3(kVecWG), 0, s, wd, parity, xcd);
    else hipLaunchKernelGGL(k_fin<kFinAll>, dim3(hw.fin_nblk), dim3(kVecWG), 0, s, wd, parity, xcd);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_decide(const Work* wd, int parity, void* stream)
{
    hipLaunchKernelGGL(k_decide, dim3(1), dim3(kDecideWG), 0, (hipStream_t)stream, wd, parity);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_step(const Work& hw, const Work* wd, int parity, void* stream)
{
    int rc = launch_sweep(hw, wd, parity, stream);
    if (!rc) rc = launch_finalize(hw, wd, parity, stream);
    return rc ? rc : launch_decide(wd, parity, stream);
}

int launch_sweep(const Work& hw, const Work* wd, int parity, void* stream)
{
    const int tiles = hw.nrt * hw.nct;
#define L_(CC) hipLaunchKernelGGL(k_sweep<CC>, dim3(tiles), dim3(kWG), 0, (hipStream_t)stream, wd, parity)
    MDOT_CC_SWITCH(cost_code(hw), L_)
#undef L_
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Tiles per workgroup of the resident-steps kernel for these problems, all in one launch, on a GPU of
// `cus` compute units, 0 if it does not apply: one cost type, at most one workgroup per unit in all, one
// finalize block each. Up to one tile per unit the workgroup is one quad; two tiles take two quads.
// Four take two quads of two tiles where the cost is held, which does not fit the 128 registers a
// thread of four quads has, and four quads for a point cloud, whose sweep is bound by its FP64
// arithmetic and wants four waves per SIMD in flight (n = 4096 in the plane 20.99 -> 19.22 us per step
// of a schedule with FP32 exponentials, 30.2 -> 27.1 with FP64; six 3-D clouds in the engine 27.0 ->
// 23.9 ms). Sizes past 8192 have a finalize layout of their own, clouds of more than 3 coordinates
// more registers per column.
int steps_tiles(const Work* const* hw, int count, int cus)
{
    const int most = std::min(cus, kStepsMaxGrid);
    for (int k = 0; k < count; ++k) {
        const Work& w = *hw[k];
        if (w.fin_per != 8 || w.nrt > kStepsMaxRowTiles) return 0;
        if (w.cost_kind != MDOT_COST_DENSE && w.d > 3) return 0;
        if (base_code_of(w) != base_code_of(*hw[0])) return 0;
    }
    for (int nt : {1, 2, 4}) {
        int blocks = 0;
        for (int k = 0; k < count; ++k) blocks += steps_blocks(*hw[k], nt);
        if (blocks <= most) return nt;
    }
    return 0;
}

template <int CC>
static void launch_steps_as(int nt, int grid, const Work* wd, const BatchDesc* bd, StepsX* x, int max_steps, hipStream_t s)
{
    if (nt == 1) hipLaunchKernelGGL((k_steps<CC, 1, 1>), dim3(grid), dim3(256), 0, s, wd, bd, x, max_steps);
    else if (nt == 2) hipLaunchKernelGGL((k_steps<CC, 2, 1>), dim3(grid), dim3(512), 0, s, wd, bd, x, max_steps);
    else if constexpr (StepKind<typename CostOf<CC>::T, 1>::kPoints)
        hipLaunchKernelGGL((k_steps<CC, 4, 1>), dim3(grid), dim3(1024), 0, s, wd, bd, x, max_steps);
    else
        hipLaunchKernelGGL((k_steps<CC, 2, 2>), dim3(grid), dim3(512), 0, s, wd, bd, x, max_steps);
}

int base_code_of(const Work& hw) { return base_code(cost_code(hw)); }

int steps_blocks(const Work& hw, int nt) { return std::max((hw.nrt * hw.nct + nt - 1) / nt, hw.fin_nvb); }

static int launch_steps_of(int code, int nt, int grid, const Work* wd, const BatchDesc* bd, StepsX* x, int max_steps, hipStream_t s)
{
#define L_(CC) launch_steps_as<CC>(nt, grid, wd, bd, x, max_steps, s)
    switch (code) {
        case CC_F64: L_(CC_F64); break;
        case CC_F32: L_(CC_F32); break;
        case CC_F16: L_(CC_F16); break;
        case CC_BF16: L_(CC_BF16); break;
        case CC_PTS_SQ: L_(CC_PTS_SQ); break;
        case CC_PTS_L1: L_(CC_PTS_L1); break;
        case CC_PTS_SQ2: L_(CC_PTS_SQ2); break;
        case CC_PTS_L12: L_(CC_PTS_L12); break;
        default: return -1;
    }
#undef L_
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int CC>
static void launch_lse_as(int nt, int grid, const LseArgs& a, StepsX* x, hipStream_t s)
{
    if (nt == 1) hipLaunchKernelGGL((k_lse<CC, 1, 1>), dim3(grid), dim3(256), 0, s, a, x);
    else hipLaunchKernelGGL((k_lse<CC, 2, 1>), dim3(grid), dim3(512), 0, s, a, x);
}

// Up to two tiles per workgroup (n about 2900) one kernel is faster: 17 to 27 us, where the six
// kernels take 27 us at n = 256 and the host queues each. With four the compute units hold one
// workgroup of two waves per SIMD and nothing overlaps its exchanges: n = 4096 with shifts 42 us,
// 34 us as kernels.
bool lse_resident(int nt) { return nt == 1 || nt == 2; }

int launch_lse(const LseArgs& a, StepsX* x, int nt, void* stream)
{
    const Work& hw = a.w;
    const int tiles = hw.nrt * hw.nct, grid = std::max((tiles + nt - 1) / nt, hw.fin_nvb);
    hipStream_t s = (hipStream_t)stream;
#define L_(CC) launch_lse_as<CC>(nt, grid, a, x, s)
    switch (base_code(cost_code(hw))) {
        case CC_F64: L_(CC_F64); break;
        case CC_F32: L_(CC_F32); break;
        case CC_F16: L_(CC_F16); break;
        case CC_BF16: L_(CC_BF16); break;
        case CC_PTS_SQ: L_(CC_PTS_SQ); break;
        case CC_PTS_L1: L_(CC_PTS_L1); break;
        case CC_PTS_SQ2: L_(CC_PTS_SQ2); break;
        case CC_PTS_L12: L_(CC_PTS_L12); break;
        default: return -1;
    }
#undef L_
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_steps(const Work& hw, const Work* wd, StepsX* x, int nt, int max_steps, void* stream)
{
    return launch_steps_of(base_code(cost_code(hw)), nt, steps_blocks(hw, nt), wd, nullptr, x, max_steps, (hipStream_t)stream);
}

int launch_steps_batch(const BatchDesc& hb, const BatchDesc* bd, StepsX* x, int max_steps, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const int rc = launch_steps_of(hb.steps_code, hb.steps_nt, hb.steps_prefix[hb.nitems], nullptr, bd, x, max_steps, s);
    hipLaunchKernelGGL(k_settle_batch, dim3(kMaxBatch), dim3(kDecideWG), 0, s, bd, x);
    return rc || hipGetLastError() != hipSuccess ? -1 : 0;
}

int launch_settle(const Work* wd, void* stream)
{
    hipLaunchKernelGGL(k_settle, dim3(1), dim3(kDecideWG), 0, (hipStream_t)stream, wd);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_alone_setup(const Work& w, const State& s, const DevParams& prm, const AloneIn& in, Work* wd, int boxes,
                       void* stream)
{
    const int fill = (w.m + w.n + 255) / 256;
    hipLaunchKernelGGL(k_alone_setup, dim3(fill + (boxes ? kBoxBlocks : 0)), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<Control*>(wd), w, s, prm, in, fill);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_row_max(const Work& hw, const Work* wd, double* part, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const int tiles = hw.nrt * hw.nct;
#define L_(CC) hipLaunchKernelGGL(k_row_max<CC>, dim3(tiles), dim3(kWG), 0, s, wd, part)
    MDOT_CC_SWITCH_BASE(base_code(cost_code(hw)), L_)
#undef L_
    hipLaunchKernelGGL(k_fold_max, dim3((hw.m + 255) / 256 + 1), dim3(1024), 0, s, wd, (const double*)part);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_sweep_range(const Work& hw, const Work* wd, double* part, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const dim3 tiles(hw.nrt * hw.nct);
    switch (base_code(cost_code(hw))) {
        case CC_F64: hipLaunchKernelGGL(k_sweep_range<CC_F64>, tiles, dim3(kWG), 0, s, wd, part); break;
        case CC_F32: hipLaunchKernelGGL(k_sweep_range<CC_F32>, tiles, dim3(kWG), 0, s, wd, part); break;
        case CC_F16: hipLaunchKernelGGL(k_sweep_range<CC_F16>, tiles, dim3(kWG), 0, s, wd, part); break;
        case CC_BF16: hipLaunchKernelGGL(k_sweep_range<CC_BF16>, tiles, dim3(kWG), 0, s, wd, part); break;
        default: return -1;  // point costs take their bounding boxes
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_pick_scale(Work* wd, const double* part, void* stream)
{
    hipLaunchKernelGGL(k_pick_scale, dim3(1), dim3(1024), 0, (hipStream_t)stream, wd, part);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_alone_out(const Work& hw, Work* wd, int slot, const double* part, int where, int lse, int e64, double* lr_out,
                     double* lc_out, AloneOut* out, void* stream)
{
    const int grid = lse ? std::min(16, (hw.m + hw.n + 4095) / 4096) : 1;
    hipLaunchKernelGGL(k_alone_out, dim3(grid), dim3(1024), 0, (hipStream_t)stream, wd, slot, part, where, lse, e64,
                       lr_out, lc_out, out);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_step_batch(const BatchDesc& hb, const BatchDesc* bd, int parity, int fin_grid, int fin_v, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    for (int c = 0; c < hb.ncodes; ++c) {
        const int b = hb.code_begin[c], e = hb.code_begin[c + 1];
        if (e <= b) continue;
#define L_(CC) hipLaunchKernelGGL(k_sweep_batch<CC>, dim3(e - b), dim3(kWG), 0, s, bd, parity, b, e)
        MDOT_CC_SWITCH(hb.code[c], L_)
#undef L_
    }
    if (fin_v == kFinSmall) hipLaunchKernelGGL(k_fin_batch<kFinSmall>, dim3(fin_grid), dim3(kVecWG), 0, s, bd, parity);
    else if (fin_v == kFinMid) hipLaunchKernelGGL(k_fin_batch<kFinMid>, dim3(fin_grid), dim3(kVecWG), 0, s, bd, parity);
    else hipLaunchKernelGGL(k_fin_batch<kFinAll>, dim3(fin_grid), dim3(kVecWG), 0, s, bd, parity);
    hipLaunchKernelGGL(k_decide_batch, dim3(kMaxBatch), dim3(kDecideWG), 0, s, bd, parity);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_gather_done(const BatchDesc* bd, StepsX* x, int* out, int* seq, void* stream)
{
    hipLaunchKernelGGL(k_gather_done, dim3(1), dim3(kMaxBatch), 0, (hipStream_t)stream, bd, x, out, seq);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_chunk_done(const Work* wd, StepsX* x, int* out, int* seq, void* stream)
{
    hipLaunchKernelGGL(k_chunk_done, dim3(1), dim3(1), 0, (hipStream_t)stream, wd, x, out, seq);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_init(const Work* wd, void* stream)
{
    hipLaunchKernelGGL(k_init, dim3(1), dim3(64), 0, (hipStream_t)stream, wd);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_intake(const Work* wd, double* out8, void* stream)
{
    hipLaunchKernelGGL(k_intake, dim3(1), dim3(kWG), 0, (hipStream_t)stream, wd, out8);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_cost_range(const Work& hw, const Work* wd, double* part, int box, void* stream)
{
    const int tiles = hw.nrt * hw.nct;
    // with boxes most calls end at the look at them: no more workgroups than are resident at once
    const int grid = box ? std::min(tiles, 2048) : tiles;
#define L_(CC) hipLaunchKernelGGL(k_cost_range<CC>, dim3(grid), dim3(kWG), 0, (hipStream_t)stream, wd, part, box)
    MDOT_CC_SWITCH_BASE(base_code(cost_code(hw)), L_)
#undef L_
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// FP16 copy of a dense cost (round to nearest) and the largest rounding error per block.
template <class T>
__global__ void __launch_bounds__(256) k_to_f16(const T* __restrict__ src, __half* __restrict__ dst, size_t count,
                                                double* part)
{
    __shared__ double sm[4];
    double mx = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) {
        const double c = (double)src[i];
        const _Float16 h = static_cast<_Float16>(c);  // the error is measured, so the rounding path does not matter
        dst[i] = __half_raw{h};
        mx = fmax(mx, fabs((double)h - c));
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
}

int launch_to_f16(const void* src, int src_dtype, void* dst, size_t count, double* part, int nblocks, void* stream)
{
    if (src_dtype == MDOT_DT_F32)
        hipLaunchKernelGGL(k_to_f16<float>, dim3(nblocks), dim3(256), 0, (hipStream_t)stream, (const float*)src,
                           (__half*)dst, count, part);
    else
        hipLaunchKernelGGL(k_to_f16<double>, dim3(nblocks), dim3(256), 0, (hipStream_t)stream, (const double*)src,
                           (__half*)dst, count, part);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_finish(const Work* wd, double* u_out, double* v_out, void* stream)
{
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kWG), 0, (hipStream_t)stream, wd, u_out, v_out);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------------------ allocation-free entry point
// Control block and workspace of mdot_lse2_noalloc: one array per device, loaded with the code
// object and held until the process ends. In host code `scratch` names a host-side stand-in,
// not the device array: host code only ever uses the address noalloc_scratch() returns.
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

int noalloc_scratch(int device, void** out)
{
    if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return (int)e;
        if (cur != device) return (int)hipErrorInvalidDevice;  // the caller makes `device` current
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!ptr) return (int)hipErrorInvalidSymbol;
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return 0;
}

// Read `count` doubles (used to evict a matrix from the L2 and last-level caches between timed
// sweeps by filling them with other, clean lines); the sum is stored only if it equals `never`,
// which keeps the loads without writing anything in practice.
__global__ void __launch_bounds__(256) k_touch(const double* __restrict__ src, size_t count, double never,
                                               double* sink)
{
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) acc += src[i];
    if (acc == never) sink[0] = acc;
}

int launch_touch(const double* src, size_t count, double* sink, void* stream)
{
    if (count == 0) return 0;
    hipLaunchKernelGGL(k_touch, dim3(4096), dim3(256), 0, (hipStream_t)stream, src, count, -1.2345e300, sink);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace mdot
