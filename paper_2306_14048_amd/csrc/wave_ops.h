// Wave-level building blocks of the generation-step kernels: streaming loads,
// DPP reductions over 4..64 lanes, wave-uniform broadcasts, the eviction rank.
// Everything lives in an unnamed namespace: each translation unit gets its own copy.
#pragma once
#include "h2o_internal.h"

namespace {

// Workgroup barrier that waits for this wave's LDS traffic only, so global
// loads issued earlier (prefetched rows) stay in flight across it.
__device__ inline void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// All of a step's arguments are read here, in one go: left to itself the compiler reads some of
// them where they are first used, a memory latency in the middle of the step.
__device__ inline void args_here(const StepArgs &a)
{
    asm volatile("" ::"s"(a.scale), "s"(a.k), "s"(a.n_occ), "s"(a.t), "s"(a.recent), "s"(a.rank), "s"(a.protect));
}

// 128-bit load of a cache row piece with the non-temporal hint: the cache is
// streamed once per step, and hinting that lifts the achieved read bandwidth by
// 12-14 % on this part (measured with a plain streaming-read kernel).
__device__ inline uint4 load_stream(const char *p)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

// Behind every second of `count` first requests of a wave, in kernels with two waves per SIMD: the workgroup's
// waves issue them in step.  Left alone the first wave of every SIMD issues all of its own before the second, whose first
// row then arrives after the first's last; their arithmetic takes turns instead of sharing the SIMD.
// Register-resident steps of eight waves, with / without, in a graph: caches in turn 1 to 2048 heads 0.93 .. 1.02; one cache over and
// over, which the last-level caches hold, 32 to 128 heads 0.92 .. 1.01, 1 and 12 heads 0.95 .. 1.04, 256 and 320 x 410 (256-byte rows)
// 1.04 .. 1.07, 512 and more 0.88 .. 1.06.
__device__ inline void in_step(int u, int count)
{
    if ((u & 1) && u + 1 < count) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Marks the point from which a loaded row may be unpacked: inside a loop the
// compiler otherwise moves the unpacking of 16-bit pairs to the end of the
// previous iteration, right behind the loads, and with it the wait for them.
__device__ inline void pin(uint4 &v)
{
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

// The elements of a loaded 16-byte piece as floats, taken from its four 32-bit
// words with integer operations (a 16-bit element view of the registers makes the
// compiler carry every half in a register of its own across loop iterations).
template <int DT>
__device__ inline void piece_to_float(const uint4 &v, float (&f)[Elem<DT>::EPL])
{
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    if constexpr (DT == H2O_F32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(w[i]);
    } else if constexpr (DT == H2O_F16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(w[i] & 0xffffu));
            f[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (unsigned short)(w[i] >> 16));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
}

// ---- DPP helpers (row = 16 lanes) ---------------------------------------------
constexpr int DPP_XOR1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int DPP_XOR2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141; // lane i <-> 7-i inside each 8 lanes
constexpr int DPP_MIRROR = 0x140;      // lane i <-> 15-i inside each 16 lanes
constexpr int DPP_ROR8 = 0x128;        // lane i <-> i^8 inside each 16 lanes (a rotation by 8)

template <int CTRL> __device__ inline int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ inline double dpp(double v)
{
    return __hiloint2double(dpp<CTRL>(__double2hiint(v)), dpp<CTRL>(__double2loint(v)));
}
template <int CTRL> __device__ inline unsigned long long dpp(unsigned long long v)
{
    const unsigned hi = (unsigned)dpp<CTRL>((int)(v >> 32)), lo = (unsigned)dpp<CTRL>((int)v);
    return ((unsigned long long)hi << 32) | lo;
}

// Sums of a and of b over the lanes l and l ^ M, M = 16 or 32: lanes with bit M clear get a's, the
// others b's.  The swap hands each half what it adds up, so a sum costs half a swap and half an addition.
template <int M> __device__ inline float pair_sums(float a, float b)
{
    const unsigned u = __float_as_uint(a), v = __float_as_uint(b);
    if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, v, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        static_assert(M == 32, "");
        const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
}
// After the xor-1 and xor-2 steps all four lanes of a quad agree, so the two
// mirror steps act as xor-4 and xor-8: every lane ends with its group's total.
template <int LANES> __device__ inline double group_sum(double a)
{
    a += dpp<DPP_XOR1>(a);
    a += dpp<DPP_XOR2>(a);
    if (LANES >= 8) a += dpp<DPP_HALF_MIRROR>(a);
    if (LANES >= 16) a += dpp<DPP_MIRROR>(a);
    if (LANES >= 32) a += __shfl_xor(a, 16, 64);
    if (LANES >= 64) a += __shfl_xor(a, 32, 64);
    return a;
}
__device__ inline double row_max(double a)
{
    a = fmax(a, dpp<DPP_XOR1>(a));
    a = fmax(a, dpp<DPP_XOR2>(a));
    a = fmax(a, dpp<DPP_HALF_MIRROR>(a));
    return fmax(a, dpp<DPP_MIRROR>(a));
}
// value of lane L of the wave, as a wave-uniform scalar
__device__ inline double lane_value(double v, int L)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), L),
                            __builtin_amdgcn_readlane(__double2loint(v), L));
}
__device__ inline unsigned long long lane_value(unsigned long long v, int L)
{
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), L);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, L);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ inline double wave_max(double v)
{
    v = row_max(v);
    return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}
__device__ inline double wave_min_f64(double v)   // NaN entries are ignored
{
    v = fmin(v, dpp<DPP_XOR1>(v));
    v = fmin(v, dpp<DPP_XOR2>(v));
    v = fmin(v, dpp<DPP_HALF_MIRROR>(v));
    v = fmin(v, dpp<DPP_MIRROR>(v));
    return fmin(fmin(lane_value(v, 0), lane_value(v, 16)), fmin(lane_value(v, 32), lane_value(v, 48)));
}
__device__ inline double wave_sum(double v)
{
    v = group_sum<16>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
// Adds this lane's fp32 partial output (EPL columns of row group `sub`) into the
// workgroup's output row, multiplies nothing: o_l[wave][column] gets the wave's sum.
//
// Each step halves the columns a lane is left with (up to 8 lanes per row: the first keeps them
// all), and at the end every lane stores its own one or two.  In registers, because a shuffle through LDS takes
// some 130 cycles and these stand in the tail of a step, where nothing else is left to do: 300 to
// 400 cycles of a step's 4600 on 8 heads x 64 slots.  (All columns in all lanes, a register swapped with itself, takes
// three times the instructions: with fourteen workgroups per CU those count, 3584 heads x 1 slot 12.1 us
// against 11.3.)
template <int EPL, int LPR, int D>
__device__ inline void wave_output_to_lds(float (&o)[EPL], float *o_l, int wave, int sub, int li)
{
    static_assert(LPR == 8 || LPR == 16 || LPR == 32, "");
    constexpr int H = LPR <= 16 ? EPL / 2 : EPL, Q = H / 2;
    const int lane = sub * LPR + li;
    int col = li * EPL;
    if constexpr (LPR == 8) {
#pragma unroll
        for (int i = 0; i < EPL; ++i) o[i] += __int_as_float(dpp<DPP_ROR8>(__float_as_int(o[i])));
    }
    if constexpr (LPR <= 16) {
#pragma unroll
        for (int i = 0; i < H; ++i) o[i] = pair_sums<16>(o[i], o[i + H]);
        col += lane & 16 ? H : 0;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) o[i] = pair_sums<32>(o[i], o[i + Q]);
    col += lane & 32 ? Q : 0;
    if (LPR > 8 || !(lane & 8)) {
#pragma unroll
        for (int i = 0; i < Q; ++i) o_l[wave * D + col + i] = o[i];
    }
}

constexpr unsigned long long NO_CANDIDATE = ~0ull;

// What ranks a slot for eviction after the query at position t: its accumulated
// score, or (averaged ranking) that score over the number of queries that have
// scored the token, t - pos + 1, as a correctly rounded binary32 quotient.  The
// new token itself has been scored once, so its value is its first score either way.
__device__ inline float rank_value(float acc, int pos, int t, int rank)
{
    return rank == H2O_RANK_AVERAGED ? __fdiv_rn(acc, (float)(t - pos + 1)) : acc;
}

// What an eviction may not touch when the query sits at position t.  protect 0:
// the last `recent` positions (the method's recent window).  Otherwise the
// positions a sparse-attention pattern lets that query attend to (Sec. 5.2,
// the strided and fixed patterns combined with heavy hitters): strided = a band
// of `recent` positions and every stride-th position counted back from t;
// fixed = the block of `stride` positions holding t and the last `recent`
// positions of every block.
__device__ inline bool is_protected(int p, int t, int recent, int protect, int stride)
{
    if (protect == H2O_PROTECT_STRIDED) return t - p < recent || (t - p) % stride == 0;
    if (protect == H2O_PROTECT_FIXED) return p / stride == t / stride || p % stride >= stride - recent;
    return p > t - recent;
}

// ---- 4-bit group-wise storage ------------------------------------------------------
//
// A lane holds 64 / LANES consecutive elements of a row (exact binary32 images); the LANES
// lanes of an aligned group together hold one quantisation group of 64.
// Returns the lane's codes packed into one word (element i in bits 4i..4i+3)
// and the group's (scale, min).  Every operation is a single correctly rounded
// binary32 operation, in the order the storage format is defined in.
template <int LANES>
__device__ inline unsigned q4_quantise(const float (&x)[64 / LANES], float &scale, float &mn)
{
    static_assert(LANES == 8 || LANES == 16, "");
    float lo = x[0], hi = x[0];
#pragma unroll
    for (int i = 1; i < 64 / LANES; ++i) { lo = fminf(lo, x[i]); hi = fmaxf(hi, x[i]); }
    lo = fminf(lo, __int_as_float(dpp<DPP_XOR1>(__float_as_int(lo))));
    hi = fmaxf(hi, __int_as_float(dpp<DPP_XOR1>(__float_as_int(hi))));
    lo = fminf(lo, __int_as_float(dpp<DPP_XOR2>(__float_as_int(lo))));
    hi = fmaxf(hi, __int_as_float(dpp<DPP_XOR2>(__float_as_int(hi))));
    lo = fminf(lo, __int_as_float(dpp<DPP_HALF_MIRROR>(__float_as_int(lo))));
    hi = fmaxf(hi, __int_as_float(dpp<DPP_HALF_MIRROR>(__float_as_int(hi))));
    if constexpr (LANES == 16) {
        lo = fminf(lo, __int_as_float(dpp<DPP_MIRROR>(__float_as_int(lo))));
        hi = fmaxf(hi, __int_as_float(dpp<DPP_MIRROR>(__float_as_int(hi))));
    }
    mn = lo;
    scale = __fdiv_rn(__fsub_rn(hi, lo), 15.0f);
    unsigned word = 0;
    if (scale > 0.0f) {
#pragma unroll
        for (int i = 0; i < 64 / LANES; ++i) {
            float c = rintf(__fdiv_rn(__fsub_rn(x[i], lo), scale));   // half to even
            c = fminf(fmaxf(c, 0.0f), 15.0f);
            word |= (unsigned)c << (4 * i);
        }
    }
    return word;
}

// 8 consecutive elements starting at p (16-byte aligned for 16-bit types, 32 for binary32)
template <int DT>
__device__ inline void load8(const typename Elem<DT>::T *p, float (&f)[8])
{
    if constexpr (DT == H2O_F32) {
        const float4 a = *reinterpret_cast<const float4 *>(p);
        const float4 b = *reinterpret_cast<const float4 *>(p + 4);
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
        f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    } else {
        const uint4 v = *reinterpret_cast<const uint4 *>(p);
        piece_to_float<DT>(v, f);
    }
}

}  // namespace
