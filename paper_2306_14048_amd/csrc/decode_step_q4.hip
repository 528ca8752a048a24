// Fused H2O generation step over a cache that stores 4-bit codes (group-wise
// min-max quantisation along the head dimension, Sec. 5.4 and the appendix on
// combining H2O with quantisation): one workgroup per (batch, head).
//
// The step is the one of the unquantised kernel (Definition 2.2 softmax over the
// cached tokens and the token itself, Algorithm 2 accumulate, evict the smallest
// score outside the recent window, overwrite in place) on the stored values
// x = min + code * scale; the new token attends to itself with its key and value
// as given and is quantised when it is written into its slot.
//
// Both contractions run on the integer matrix cores, exactly.  With the row's
// (scale s_g, min m_g) per group g of 64 elements,
//     <q, x>  = sum_g  s_g * sum_{e in g} q_e c_e  +  m_g * sum_{e in g} q_e
//     out_e   = sum_j (p_j s_gj) c_je  +  sum_j p_j m_gj .
// The codes c (0..15) are one operand as bytes; the other is q, respectively
// w_j = p_j s_gj, as a fixed-point number cut into signed 8-bit digits (base 256, digits
// -128..127): q_e * 2^(54-E) with the group's max|q| < 2^E in eight digits, w_j * 2^(30-E') with
// the group's largest w of 64 slots < 2^E' in four (binary32 elements: w_j * 2^(62-E') in
// eight).  v_mfma_i32_16x16x64_i8 then forms the digit sums without rounding and they are
// put together in float64: an element of q is off by at most half a unit, 2^-54 of its group's
// max|q| (which may be as small as 2^(E-1)), a logit by at most 64 * 15 of those times the
// scale; a weight by half a unit, at most 2^-30 (binary32: 2^-53, its own rounding) of the
// largest in its group.  The kernel before this one had binary32 products and sums for 16-bit
// elements and float64 for binary32 ones; p itself is a binary32 number in both.
//   logits   A = digits of q (row = digit; rows 0-7 group 0, rows 8-15 group 1, zero where a
//            row's group is not the lane's piece of the head dimension), B = 16 cached rows
//   output   A = digits of w (rows 0-3 group 0, 4-7 group 1; rows 8-15 the lower four of the
//            eight), B = 64 rows x 16 elements, read from the row-major codes with the
//            4-bit transposing LDS read
// Turning codes into bytes takes three vector instructions per eight codes.  The kernel
// before this one formed both sums on the vector ALU (an AND-OR and an fp64 or mixed fma
// per code, 6.3 k vector instructions per head of 410 slots; now 4.7 k, most of them the
// softmax and bookkeeping of each wave).  Measured, before -> this, f16, d = 128, one cache
// stepped repeatedly: 512 heads x 410 slots 11.9 -> 10.1 us (36.7 MB), x 2048 45.2 -> 32.6; 3584 x
// 205 34.9 -> 30.2 (4.3 TB/s), x 64 25.4 -> 14.7; 4096 x 410 70.8 -> 57.1 (5.1 TB/s); 32 x 2000
// 17.7 -> 12.1; binary32 elements 512 x 410 13.8 -> 10.0.
//
// What a step of few slots waits for is one chain: arguments, q, its digits, logits, normaliser, output, the sums over
// the waves (32 heads x 410: 4.8 us between the first and the last stamp, every wave nearly alone on its SIMD).
// Taken out of that chain: a division by the number of waves (0.3 us), the quantiser's second
// four elements per lane (0.2), the reads of the final sums one after the other (0.45), the scores behind the
// output.  Steps in a graph, before -> this, us, one cache / caches in turn: 512 heads x 410 9.6 -> 8.4 / 12.0 ->
// 10.6, 32 x 410 6.15 -> 5.5 / 6.9 -> 5.9, 3584 x 205 29.3 -> 27.4 / 30.2 -> 28.7, 512 x 2000 32.5 -> 31.6 / 35.7 -> 34.9.
//
// Memory plan.  A wave owns blocks of 64 consecutive slots, one slot per lane.  A
// block's stored rows are one contiguous image of 64 * 80 (or 48) bytes; the K images of a
// wave's blocks followed by the V images are copied straight into a ring of LDS buffers of
// its own (no registers, no barriers).  Requested are, at the start, the K images that the ring
// holds and behind them the slots' bookkeeping, once q's digits are cut the V images that it
// holds besides, and every other image when the buffer it goes to has been read.
// Every global read of the kernel is such a copy, so that each wait names exactly the
// copies it needs (a load that the compiler waits for would wait for all of them).
#include "wave_ops.h"
#include "lds_copy.h"
#include <type_traits>

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// streaming form of dma16: the cache is read once per step
__device__ inline void dma16_stream(i32x4 rsrc, unsigned voff, unsigned lds_base)
{
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen nt lds"
                 :
                 : "v"(voff), "s"(rsrc), "{m0}"(lds_base)
                 : "memory");
}

// 16 codes (two words) as 16 bytes: codes 0,2,4,6 | 1,3,5,7 of each word
__device__ inline i32x4 codes_to_bytes(unsigned w0, unsigned w1)
{
    constexpr unsigned M = 0x0F0F0F0Fu;
    return i32x4{(int)(w0 & M), (int)((w0 >> 4) & M), (int)(w1 & M), (int)((w1 >> 4) & M)};
}

// sum of a over the lanes l, l ^ 32 (result: a's in lanes 0..31, b's in lanes 32..63)
__device__ inline double fold32(double a, double b)
{
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// sum over the lanes l, l ^ 16 (result: a's in the even rows of 16 lanes, b's in the odd ones)
__device__ inline double fold16(double a, double b)
{
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// smallest E with |x| < 2^E for a finite x (at least -126)
__device__ inline int exponent_above(float x) { return (int)((__float_as_uint(x) >> 23) & 255u) - 126; }
// for two non-negative values per lane, the exponents above the largest of each in the wave
// (a's in lanes 0..31, b's in lanes 32..63 after the swap: one reduction for both)
__device__ inline void exponents_above(float a, float b, int &ea, int &eb)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    int v = max((int)r[0], (int)r[1]);          // (non-negative floats order like their bits)
    v = max(v, dpp<DPP_XOR1>(v));
    v = max(v, dpp<DPP_XOR2>(v));
    v = max(v, dpp<DPP_HALF_MIRROR>(v));
    v = max(v, dpp<DPP_MIRROR>(v));
    ea = exponent_above(__int_as_float(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16))));
    eb = exponent_above(__int_as_float(max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48))));
}
// the same for one value per lane
__device__ inline int exponent_above_wave(float a)
{
    int v = __float_as_int(a);
    v = max(v, dpp<DPP_XOR1>(v));
    v = max(v, dpp<DPP_XOR2>(v));
    v = max(v, dpp<DPP_HALF_MIRROR>(v));
    v = max(v, dpp<DPP_MIRROR>(v));
    return exponent_above(__int_as_float(max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                                             max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)))));
}
// exact power of two, |n| <= 1022
__device__ inline double pow2(int n) { return __hiloint2double((1023 + n) << 20, 0); }

// Four digit sums: sum_i v[i] 256^i = lo + 65536 hi.  (One MFMA's or two MFMAs' sums are below
// 2 * 64 * 128 * 15 < 2^18, so neighbours fit one 32-bit integer.)
__device__ inline i32x2 digit_pairs(const i32x4 &v) { return i32x2{v[0] + (v[1] << 8), v[2] + (v[3] << 8)}; }
__device__ inline double joined(const i32x2 &v) { return fma((double)v.y, 65536.0, (double)v.x); }

constexpr int MAX_WAVES = 8;

// LDS of a workgroup: the shared part, then one part per wave
template <int D> struct Shared {
    unsigned char raw[3][512];                 // q, the new key, the new value as given
    signed char digit[8][D];                   // q's digits; elements in the byte order of codes_to_bytes
    double red_sum[MAX_WAVES], red_max[MAX_WAVES], red_key[MAX_WAVES];
    double min_sum[2][MAX_WAVES];              // sum p m_g over a wave's slots
    double s_self, qsum[2];                    // the token's own logit; scale * sum q per group
    int q_exp[2];                              // |q| < 2^q_exp in each group
    unsigned new_row[96];                      // the new token as stored: words, scales, mins
};
template <int DT, int D, int SPL> struct Ring {
    static constexpr int IMG = 64 * H2O_Q4_ROW_BYTES(D);       // one block's rows
    static constexpr int NB = SPL == 1 ? 2 : 3;                // buffers
    static constexpr int RECB = DT == H2O_F32 ? 16 : 8;        // bytes of digits per slot: 4 or 8 digits, 2 groups
    // images | positions and scores of the wave's slots | digits of the weights of one
    // block (one block per wave: in the K image, which is done with by then)
    static constexpr int META = NB * IMG, REC = SPL == 1 ? 0 : META + SPL * 512;
    static constexpr int BYTES = META + SPL * 512 + (SPL == 1 ? 0 : 64 * RECB);
};

// SPL: blocks of 64 slots per wave (block s of wave w: s * waves + w).  PAT: built for
// a sparse-attention pattern as the protected set (the plain recent window's build
// carries none of that code).
template <int DT, int D, int SPL, bool PAT>
__global__ __launch_bounds__(MAX_WAVES * 64, 4) void decode_q4_kernel(const StepArgs args)
{
    char *__restrict__ Kc = args.K;
    char *__restrict__ Vc = args.V;
    float *__restrict__ acc_g = args.acc;
    int32_t *__restrict__ pos_g = args.pos;
    const char *__restrict__ q_g = args.q, *__restrict__ kn_g = args.kn, *__restrict__ vn_g = args.vn;
    char *__restrict__ out_g = args.out;
    const int k = args.k, n_occ = args.n_occ, t = args.t, recent = args.recent, rank = args.rank, protect = args.protect,
              stride = args.stride;
    const double scale = args.scale;
    args_here(args);
    using E = Elem<DT>;
    using T = typename E::T;
    using L = Ring<DT, D, SPL>;
    constexpr int CODEB = D / 2;                // bytes of codes per row
    constexpr unsigned ROWB = H2O_Q4_ROW_BYTES(D);
    constexpr int NG = D / 64;                  // groups per row = MFMAs per 16 rows
    constexpr int IPB = L::IMG / 1024;          // copy instructions per image
    constexpr int NB = L::NB;
    constexpr int QL = D / 8;                   // lanes holding the new key, 8 elements each
    constexpr int META_COPIES = 2 * SPL;
    constexpr bool WIDE = DT == H2O_F32;        // output weights of eight digits instead of four
    static_assert(L::IMG % 1024 == 0 && (D == 64 || D == 128), "whole copies");

    const int head = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x, nw = nthr >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quarter = lane >> 4;

    extern __shared__ __align__(16) unsigned char smem[];
    Shared<D> &sh = *reinterpret_cast<Shared<D> *>(smem);
    unsigned char *mine_l = smem + ((sizeof(Shared<D>) + 15) & ~(size_t)15) + (size_t)wave * L::BYTES;
    const unsigned raw_b = (unsigned)reinterpret_cast<size_t>(smem);
    const unsigned mine_b = __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<size_t>(mine_l));

    const size_t hoff = (size_t)head * k;
    char *Kb = Kc + hoff * ROWB;
    char *Vb = Vc + hoff * ROWB;

    // ---- requests: q and the new token (wave 0), then the wave's first K images, then the
    // bookkeeping (value images: behind q's digits).  Pieces past the occupied slots repeat the last
    // occupied piece (in bounds; what they hold is masked).
    if (wave == 0) {
        constexpr unsigned RB = D * sizeof(T);
        const i32x4 rq = make_rsrc(q_g + (size_t)head * RB, RB);
        const i32x4 rk = make_rsrc(kn_g + (size_t)head * RB, RB);
        const i32x4 rv = make_rsrc(vn_g + (size_t)head * RB, RB);
        if (lane < (int)RB / 16) {
            dma16(rq, lane * 16u, 0u, raw_b);
            dma16(rk, lane * 16u, 0u, raw_b + 512);
            dma16(rv, lane * 16u, 0u, raw_b + 1024);
        }
    }
    const unsigned occ_bytes = (unsigned)max(n_occ, 1) * ROWB;
    const i32x4 rsrc_k = make_rsrc(Kb, (unsigned)k * ROWB);
    const i32x4 rsrc_v = make_rsrc(Vb, (unsigned)k * ROWB);
    auto fetch = [&](int item) {                // item: K of blocks 0..SPL-1, then V of them
        const int s = item % SPL;
        const unsigned first = (unsigned)(s * nw + wave) * L::IMG + lane * 16u;
#pragma unroll
        for (int i = 0; i < IPB; ++i)
            dma16_stream(item < SPL ? rsrc_k : rsrc_v, min(first + i * 1024u, occ_bytes - 16u),
                         mine_b + (item % NB) * L::IMG + i * 1024);
    };
    constexpr int KFIRST = SPL < NB ? SPL : NB;     // K images among the first NB
#pragma unroll
    for (int i = 0; i < KFIRST; ++i) fetch(i);
    int my_slot[SPL];
    bool owner[SPL];
    {
        const i32x4 rsrc_p = make_rsrc(pos_g + hoff, (unsigned)k * 4u);
        const i32x4 rsrc_a = make_rsrc(acc_g + hoff, (unsigned)k * 4u);
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            my_slot[s] = (s * nw + wave) * 64 + lane;
            owner[s] = my_slot[s] < n_occ;
            const unsigned off = (unsigned)min(my_slot[s], max(n_occ, 1) - 1) * 4u;
            dma4(rsrc_p, off, 0u, mine_b + L::META + s * 512);
            dma4(rsrc_a, off, 0u, mine_b + L::META + s * 512 + 256);
        }
    }

    // ---- q: the token's own logit, group sums, digits --------------------------------
    dma_wait_upto<KFIRST * IPB + META_COPIES>();    // (wave 0: its three copies have landed)
    lds_barrier();
    const T *q_l = reinterpret_cast<const T *>(sh.raw[0]), *kn_l = reinterpret_cast<const T *>(sh.raw[1]),
            *vn_l = reinterpret_cast<const T *>(sh.raw[2]);
    // Sums over the head dimension and the new token as it will be stored are each worked
    // out by one wave (in the wait for the first image), the digits by the first D threads.
    if (tid < MAX_WAVES) {                      // entries of waves that do not exist
        sh.red_sum[tid] = 0.0;
        sh.red_max[tid] = -INFINITY;
        sh.red_key[tid] = __longlong_as_double((long long)NO_CANDIDATE);
        sh.min_sum[0][tid] = sh.min_sum[1][tid] = 0.0;
    }
    // (waves 0 and 1 cut the digits; job j goes to wave (j + 2) mod waves, from a table: a division by a
    // number of waves that is only known here takes 300 ns)
    const unsigned jobs = (unsigned)(nw <= 4 ? 0x1032210210100000ull >> (16 * (nw - 1)) : 0x5432543254320432ull >> (16 * (nw - 5)));
    auto job = [&](int j) { return wave == (int)((jobs >> (4 * j)) & 15u); };
    if (job(0)) {
        double a = 0.0;
#pragma unroll
        for (int g = 0; g < NG; ++g)
            a = fma((double)E::to_f(q_l[64 * g + lane]), (double)E::to_f(kn_l[64 * g + lane]), a);
        a = wave_sum(a);
        if (lane == 0) sh.s_self = a * scale;
    }
    if (job(1)) {
        const double a = wave_sum((double)E::to_f(q_l[lane]));
        if (lane == 0) sh.qsum[0] = a * scale;
    }
    if (job(2)) {
        const double a = NG == 2 ? wave_sum((double)E::to_f(q_l[D - 64 + lane])) : 0.0;
        if (lane == 0) sh.qsum[1] = a * scale;
    }
    if (job(3)) {                               // four elements per lane: the longest of the jobs
        const T *x = ((lane / (2 * QL)) == 1 ? vn_l : kn_l) + (lane % (2 * QL)) * 4;
        const float n4[4] = {E::to_f(x[0]), E::to_f(x[1]), E::to_f(x[2]), E::to_f(x[3])};
        float new_scale, new_min;
        const unsigned new_half = q4_quantise<16>(n4, new_scale, new_min);
        if (lane < 4 * QL) {
            reinterpret_cast<unsigned short *>(sh.new_row)[lane] = (unsigned short)new_half;
            if (!(lane & 1)) {
                sh.new_row[32 + lane / 2] = __float_as_uint(new_scale);
                sh.new_row[64 + lane / 2] = __float_as_uint(new_min);
            }
        }
    }
    for (int e = tid; e < D; e += nthr) {       // (a wave has the 64 elements of one group)
        const float q_e = E::to_f(q_l[e]);
        const int qe = exponent_above_wave(fabsf(q_e));
        if (lane == 0) sh.q_exp[e >> 6] = qe;
        // rounded first: the low word of what is left is then exactly one in [0, 2^32)
        const double x = rint((double)q_e * pow2(54 - qe));
        const double hi = floor(x * 0x1p-32);
        const unsigned lo = (unsigned)fma(hi, -0x1p32, x);
        const unsigned long long bias = 0x0080808080808080ull;
        const unsigned long long d =
            ((((unsigned long long)(unsigned)(int)hi << 32) | lo) + bias) ^ bias;
        const int at = (e & ~7) | ((e & 1) << 2) | ((e & 7) >> 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) sh.digit[i][at] = (signed char)(d >> (8 * i));
    }
    lds_barrier();
    // The first value images are only requested here: a copy is issued no faster than the CU's share of the
    // stream comes in, and a wave that issues them all at the start gets to q 1 to 2 us later (512 heads x 410
    // slots, 24 caches in turn: all at the start 12.0 us per step, here 11.1, behind the logits 10.4; but 1024
    // heads 19.2 / 18.1 / 18.3, 3584 x 205 30.2 / 30.0 / 31.2).
#pragma unroll
    for (int i = KFIRST; i < NB; ++i) fetch(i);
    i32x4 aq[NG];
#pragma unroll
    for (int m = 0; m < NG; ++m) {
        const bool in_group = (l16 >> 3) == (NG == 2 ? quarter >> 1 : 0);
        const i32x4 v = *reinterpret_cast<const i32x4 *>(&sh.digit[l16 & 7][quarter * 16 * NG + 16 * m]);
#pragma unroll
        for (int i = 0; i < 4; ++i) aq[m][i] = in_group ? v[i] : 0;
    }
    // a lane's digit sums: quarter 0 / 1 = digits 0-3 / 4-7 of group 0, quarters 2 / 3 of group 1
    const int my_group = NG == 2 ? quarter >> 1 : 0;
    const bool used = NG == 2 || quarter < 2;
    const double s_self = sh.s_self, qsum[2] = {sh.qsum[0], sh.qsum[1]};
    // (digits cannot hold an infinity or a NaN in q: the logits are then not numbers)
    const bool q_finite = fabs(qsum[0] + qsum[1]) <= 1.79769313486231570815e+308;
    const double digit_unit = !q_finite ? (double)NAN : used ? pow2(sh.q_exp[my_group] - 54 + ((quarter & 1) ? 32 : 0)) * scale : 0.0;
    const double min_unit = used && !(quarter & 1) ? qsum[my_group] : 0.0;

    // ---- logits ------------------------------------------------------------------------
    double s_j[SPL];
    auto refill = [&](int item) {               // after item's buffer has been read
        if (item + NB < 2 * SPL) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch(item + NB);
        }
    };
    auto for_blocks = [&](auto f) {
        f(std::integral_constant<int, 0>{});
        if constexpr (SPL > 1) f(std::integral_constant<int, 1>{});
        if constexpr (SPL > 2) {
            f(std::integral_constant<int, 2>{});
            f(std::integral_constant<int, 3>{});
        }
    };
    // copies issued behind item i by the time it is waited for
    constexpr auto behind = [](int i) {
        const int last = i + NB - 1 < 2 * SPL - 1 ? i + NB - 1 : 2 * SPL - 1;
        return (last - i) * IPB + (i < KFIRST ? META_COPIES : 0);
    };
    for_blocks([&](auto tag) {
        constexpr int s = decltype(tag)::value;
        dma_wait_upto<behind(s)>();
        const unsigned char *img = mine_l + (s % NB) * L::IMG;
        double part[4];
#pragma unroll
        for (int tl = 0; tl < 4; ++tl) {
            part[tl] = 0.0;
            if ((s * nw + wave) * 64 + tl * 16 < n_occ) {      // wave-uniform
                const unsigned char *row = img + (tl * 16 + l16) * ROWB;
                i32x4 sums = {0, 0, 0, 0};
                if constexpr (NG == 2) {
                    const uint4 w = *reinterpret_cast<const uint4 *>(row + quarter * 16);
                    sums = __builtin_amdgcn_mfma_i32_16x16x64_i8(aq[0], codes_to_bytes(w.x, w.y), sums, 0, 0, 0);
                    sums = __builtin_amdgcn_mfma_i32_16x16x64_i8(aq[1], codes_to_bytes(w.z, w.w), sums, 0, 0, 0);
                } else {
                    const uint2 w = *reinterpret_cast<const uint2 *>(row + quarter * 8);
                    sums = __builtin_amdgcn_mfma_i32_16x16x64_i8(aq[0], codes_to_bytes(w.x, w.y), sums, 0, 0, 0);
                }
                const f32x2 sm = *reinterpret_cast<const f32x2 *>(row + CODEB + 8 * my_group);
                part[tl] = fma(joined(digit_pairs(sums)) * digit_unit, (double)sm.x, (double)sm.y * min_unit);
            }
        }
        // the four quarters' parts of a row added up; lane l gets row l of the block
        s_j[s] = fold16(fold32(part[0], part[2]), fold32(part[1], part[3]));
        refill(s);
    });

    // ---- exact softmax over the occupied slots + the token itself -------------------
    double e_j[SPL];
    double e_sum = 0.0;
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
        e_j[s] = owner[s] ? exp(s_j[s] - s_self) : 0.0;
        e_sum += e_j[s];
    }
    double e_self = 1.0;
    {
        const double dw = wave_sum(e_sum);
        if (lane == 0) sh.red_sum[wave] = dw;
    }
    lds_barrier();
    double den = e_self;
#pragma unroll
    for (int w = 0; w < MAX_WAVES; ++w) den += sh.red_sum[w];
    if (!(den <= 1.79769313486231570815e+308)) {
        // some logit is > ~709 above the token's own: redo with the true maximum
        double m = -INFINITY;
#pragma unroll
        for (int s = 0; s < SPL; ++s) m = fmax(m, owner[s] ? s_j[s] : -INFINITY);
        const double mw = wave_max(m);
        if (lane == 0) sh.red_max[wave] = mw;
        lds_barrier();
        double mx = s_self;
#pragma unroll
        for (int w = 0; w < MAX_WAVES; ++w) mx = fmax(mx, sh.red_max[w]);
        e_sum = 0.0;
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            e_j[s] = owner[s] ? exp(s_j[s] - mx) : 0.0;
            e_sum += e_j[s];
        }
        e_self = exp(s_self - mx);
        const double dw = wave_sum(e_sum);
        if (lane == 0) sh.red_sum[wave] = dw;
        lds_barrier();
        den = e_self;
#pragma unroll
        for (int w = 0; w < MAX_WAVES; ++w) den += sh.red_sum[w];
    }
    const float p_self = (float)(e_self / den);
    float p_j[SPL];
#pragma unroll
    for (int s = 0; s < SPL; ++s) p_j[s] = (float)(e_j[s] / den);          // 0 for unoccupied rows

    // ---- score update (Algorithm 2, accumulate line: binary32 add of the binary32
    // probability) and the eviction candidate: smallest (rank value, position) outside
    // the window
    // (with a sparse-attention pattern as the protected set the candidates are the slots
    // it does not cover; the minimum over all slots is reduced alongside for the case
    // that it covers them all, in the LDS words of the overflow path, idle by now)
    dma_wait_upto<(SPL < NB ? SPL : NB) * IPB>();           // (behind the bookkeeping: value images)
    unsigned long long key = NO_CANDIDATE, key_all = NO_CANDIDATE;
    int key_slot = -1, key_all_slot = -1;
    float acc_j[SPL];
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
        const int pos_j = *reinterpret_cast<const int *>(mine_l + L::META + s * 512 + lane * 4);
        acc_j[s] = *reinterpret_cast<const float *>(mine_l + L::META + s * 512 + 256 + lane * 4);
        acc_j[s] += p_j[s];
        if (owner[s]) {
            const unsigned long long c =
                ((unsigned long long)__float_as_uint(rank_value(acc_j[s], pos_j, t, rank)) << 32) |
                (unsigned)pos_j;
            if (PAT ? !is_protected(pos_j, t, recent, protect, stride) : pos_j <= t - recent) {
                if (c < key) { key = c; key_slot = my_slot[s]; }
            }
            if (PAT && c < key_all) { key_all = c; key_all_slot = my_slot[s]; }
        }
    }
    {
        const double kw = wave_min_f64(__longlong_as_double((long long)key));
        if (lane == 0) sh.red_key[wave] = kw;
    }
    if constexpr (PAT) {
        const double ka = wave_min_f64(__longlong_as_double((long long)key_all));
        if (lane == 0) sh.red_max[wave] = ka;
    }

    // ---- output ------------------------------------------------------------------------
    // (the weights of a block have exponents of their own, one per group: the scales of later
    // blocks may not have arrived yet, and those of the groups need not be alike)
    constexpr int NDT = D / 16;                 // 16-element tiles of the output
    double o[NDT / NG];                         // lanes of quarter g (and 2 + g): group g's elements 16 dt + l16
#pragma unroll
    for (int i = 0; i < NDT / NG; ++i) o[i] = 0.0;
    double msum[2] = {0.0, 0.0};
    for_blocks([&](auto tag) {
        constexpr int s = decltype(tag)::value;
        dma_wait_upto<behind(SPL + s)>();
        const unsigned char *img = mine_l + ((SPL + s) % NB) * L::IMG;
        if ((s * nw + wave) * 64 < n_occ) {                    // wave-uniform
            // this lane's weights, one per group, as fixed-point digits (p is 0 for a slot that
            // is not occupied; it takes the last occupied row's scales)
            const unsigned char *meta = img + min(lane, n_occ - 1 - (s * nw + wave) * 64) * ROWB + CODEB;
            double w[2] = {0.0, 0.0};
            bool fine[2] = {true, true};
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const f32x2 sm = *reinterpret_cast<const f32x2 *>(meta + 8 * g);
                w[g] = (double)p_j[s] * (double)sm.x;
                msum[g] = fma((double)p_j[s], (double)sm.y, msum[g]);
                // infinite or not a number: so is the group's output, and the group's alone
                fine[g] = __ballot(!(w[g] <= 1.79769313486231570815e+308)) == 0;
                if (!fine[g]) w[g] = 0.0;
            }
            int we[2];
            exponents_above((float)w[0], (float)w[NG - 1], we[0], we[1]);
            const int mg = quarter & (NG - 1);
            const double down = (quarter & 1 ? fine[NG - 1] : fine[0])
                                    ? pow2((mg ? we[1] : we[0]) - (quarter < 2 ? 30 : 62))
                                    : (double)NAN;
            unsigned char *rec = mine_l + L::REC;
            if constexpr (WIDE) {
                const unsigned long long bias = 0x0080808080808080ull;
                unsigned hi[2] = {0u, 0u}, lo[2] = {0u, 0u};
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const double x = rint(w[g] * pow2(62 - we[g])), h = floor(x * 0x1p-32);
                    const unsigned long long d =
                        ((((unsigned long long)(unsigned)h << 32) | (unsigned)fma(h, -0x1p32, x)) + bias) ^ bias;
                    hi[g] = (unsigned)(d >> 32);
                    lo[g] = (unsigned)d;
                }
                *reinterpret_cast<uint4 *>(rec + lane * 16) = make_uint4(hi[0], hi[1], lo[0], lo[1]);
            } else {
                const unsigned bias = 0x00808080u;
                uint2 d;
                d.x = ((unsigned)rint(w[0] * pow2(30 - we[0])) + bias) ^ bias;
                d.y = NG == 2 ? ((unsigned)rint(w[1] * pow2(30 - we[1])) + bias) ^ bias : 0u;
                *reinterpret_cast<uint2 *>(rec + lane * 8) = d;
            }
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            // A operand: digit l16 (0-3 group 0, 4-7 group 1, binary32: 8-11 and 12-15 the lower
            // digits of each) of the quarter's 16 rows, in the byte order of codes_to_bytes.
            // (8-bit transposing read: lane i < 8 of 16 receives byte i of the 8-byte pieces that
            // the even lanes point at, lane 8 + i byte i of those of the odd lanes.)
            i32x4 aw;
            {
                typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
                const int i = l16 >> 1, r = ((i & 3) << 1) | (i >> 2);       // 0 2 4 6 1 3 5 7
                const unsigned char *at = rec + (quarter * 16 + r) * L::RECB + (WIDE ? (l16 & 1) * 8 : 0);
                const i32x2 a = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)at);
                const i32x2 b = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)(at + 8 * L::RECB));
                aw = i32x4{a.x, a.y, b.x, b.y};
            }
            // B operand: lane = element 16 dt + l16 of the quarter's 16 rows (4-bit transposing read)
            const unsigned char *row = img + lane * ROWB;
#pragma unroll
            for (int i = 0; i < NDT / NG; ++i) {
                i32x4 sums[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
                    const int dt = g * (NDT / NG) + i;
                    const i32x2 c = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_i32x2 *)(row + 8 * dt));
                    sums[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        aw, codes_to_bytes((unsigned)c.x, (unsigned)c.y), i32x4{0, 0, 0, 0}, 0, 0, 0);
                }
                // rows 4g..4g+3 of a group's tile are its digits: quarter g of the lanes has them
                // (and quarter 2 + g the lower ones)
                i32x2 v = digit_pairs(sums[0]);
                if constexpr (NG == 2) {
                    const i32x2 v1 = digit_pairs(sums[1]);
                    if (quarter & 1) v = v1;
                }
                o[i] = fma(joined(v), down, o[i]);
            }
        }
        refill(SPL + s);
    });
    {
        // the wave's columns, in its first buffer (every image has been read)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        double *o_w = reinterpret_cast<double *>(mine_l);
        if ((quarter & 1) < NG && (WIDE || quarter < 2)) {
#pragma unroll
            for (int i = 0; i < NDT / NG; ++i)
                o_w[(quarter >> 1) * D + ((quarter & 1) * (NDT / NG) + i) * 16 + l16] = o[i];
        }
        // lanes 0..31 add up group 0, lanes 32..63 group 1 (d = 64: a second copy)
        double mg = fold32(msum[0], msum[NG - 1]);
        mg = group_sum<16>(mg);
        mg = fold16(mg, mg);
        if ((lane & 31) == 0 && (lane >> 5) < NG) sh.min_sum[lane >> 5][wave] = mg;
    }

    lds_barrier();

    // ---- write-back ---------------------------------------------------------------------
    // All reads first, over every wave there can be: these sums end the step.  binary32 elements, which have two sums
    // per wave, read those of two waves where there are no more (in a graph, one cache, eight / two: d = 128, 3584 heads x
    // 33 slots 13.8 / 12.6 us, 1024 x 64 6.45 / 6.15, 32 x 100 5.2 / 5.05; 16-bit elements gain 1 to 2 % there and lose 1 %
    // with more waves to the second way).
    auto column = [&](int e, auto count) {
        constexpr int W = decltype(count)::value;
        const unsigned char *w0 = smem + ((sizeof(Shared<D>) + 15) & ~(size_t)15) + (size_t)e * 8;
        double mins[W], parts[WIDE ? 2 : 1][W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            mins[w] = sh.min_sum[e / 64][w];
            const unsigned char *at = w0 + (size_t)min(w, nw - 1) * L::BYTES;
            parts[0][w] = *reinterpret_cast<const double *>(at);
            if constexpr (WIDE) parts[1][w] = *reinterpret_cast<const double *>(at + D * 8);
        }
        double r = (double)p_self * (double)E::to_f(vn_l[e]);
#pragma unroll
        for (int w = 0; w < W; ++w) r += mins[w];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            r += w < nw ? parts[0][w] : 0.0;
            if constexpr (WIDE) r += w < nw ? parts[1][w] : 0.0;
        }
        return r;
    };
    for (int e = tid; e < D; e += nthr) {
        const double r = !WIDE || __builtin_expect(nw > 2, 1) ? column(e, std::integral_constant<int, MAX_WAVES>{})
                                                              : column(e, std::integral_constant<int, 2>{});
        reinterpret_cast<T *>(out_g)[(size_t)head * D + e] = E::from_f((float)r);
    }
    int tslot = -1;          // wave-uniform: the slot this wave has to fill, if any
    int lost_slot = -1;      // per lane: its slot that has just been evicted
    if (n_occ < k) {
        if (wave == 0) tslot = n_occ;
    } else {
        double wd = sh.red_key[0];
#pragma unroll
        for (int w = 1; w < MAX_WAVES; ++w) wd = fmin(wd, sh.red_key[w]);
        if (PAT && wd != wd) {                               // the pattern covers every slot
            wd = sh.red_max[0];
            for (int w = 1; w < nw; ++w) wd = fmin(wd, sh.red_max[w]);
            key = key_all;
            key_slot = key_all_slot;
        }
        const unsigned long long win = (unsigned long long)__double_as_longlong(wd);
        const unsigned long long self_key =
            ((unsigned long long)__float_as_uint(p_self) << 32) | (unsigned)t;
        const bool evict = wd == wd && (PAT || recent != 0 || win < self_key);
        const bool mine = evict && key == win && key != NO_CANDIDATE;   // keys are unique (positions are)
        if (mine) lost_slot = key_slot;
        const unsigned long long b = __ballot(mine);
        if (b != 0) tslot = __builtin_amdgcn_readlane(key_slot, __ffsll((long long)b) - 1);
    }
#pragma unroll
    for (int s = 0; s < SPL; ++s)
        if (owner[s] && my_slot[s] != lost_slot) acc_g[hoff + my_slot[s]] = acc_j[s];
    if (tslot >= 0) {
        if (lane == 0) { pos_g[hoff + tslot] = t; acc_g[hoff + tslot] = p_self; }
        // lanes [0, QL) hold the new key's codes, lanes [QL, 2 QL) the new value's
        if (lane < 2 * QL) {
            char *row = (lane < QL ? Kb : Vb) + (size_t)tslot * ROWB;
            const int l = lane % QL;
            *reinterpret_cast<unsigned *>(row + l * 4) = sh.new_row[lane];
            if ((l & 7) == 0)
                *reinterpret_cast<f32x2 *>(row + CODEB + (l / 8) * 8) =
                    f32x2{__uint_as_float(sh.new_row[32 + lane]), __uint_as_float(sh.new_row[64 + lane])};
        }
    }
}

template <int DT, int D, int SPL> constexpr size_t lds_of(int waves)
{
    return ((sizeof(Shared<D>) + 15) & ~(size_t)15) + (size_t)waves * Ring<DT, D, SPL>::BYTES;
}

template <int DT, int D, int SPL>
hipError_t launch_q4(const h2o_cache &c, int waves, const void *q, const void *kn, const void *vn,
                     void *out, hipStream_t st)
{
    const size_t smem = lds_of<DT, D, SPL>(waves);
    auto launch = [&](auto kern, std::atomic<uint64_t> &raised) -> hipError_t {
        if (smem > 48 * 1024) {
            const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), 150 * 1024, raised);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(c.cfg.batch * c.cfg.heads), dim3(waves * 64), smem, st, step_args(c, q, kn, vn, out));
        return hipGetLastError();
    };
    static std::atomic<uint64_t> raised_window{0}, raised_pattern{0};
    if (c.cfg.protect == H2O_PROTECT_RECENT) return launch(decode_q4_kernel<DT, D, SPL, false>, raised_window);
    return launch(decode_q4_kernel<DT, D, SPL, true>, raised_pattern);
}

// Blocks per wave: as few as leave room for two workgroups in a CU's LDS (512 heads, d =
// 128, us: 480 slots 1 / 2 blocks per wave 12.8 / 9.8; 600 2 / 4 blocks 16.1 / 12.3; 1000
// 19.8 / 15.3; below that line more waves win: 205 slots 1 / 2 blocks 7.1 / 8.4).
template <int DT, int D>
hipError_t pick_q4(const h2o_cache &c, const void *q, const void *kn, const void *vn, void *out,
                   hipStream_t st)
{
    constexpr size_t HALF = 80 * 1024;
    const int occ = c.t < c.k ? c.t : c.k;
    const int blocks = occ > 64 ? (occ + 63) / 64 : 1;
    // (a second wave shares the work on q and the new token where all heads run at once:
    // 8 heads x 64 slots 5.6 -> 5.2 us; with more heads it only takes a place: 3584 x 64 14.7 / 18.1)
    const int least = c.cfg.batch * c.cfg.heads <= 512 ? 2 : 1;
    if (blocks <= MAX_WAVES && lds_of<DT, D, 1>(blocks) <= HALF)
        return launch_q4<DT, D, 1>(c, blocks < least ? least : blocks, q, kn, vn, out, st);
    if (const int w = (blocks + 1) / 2; w <= MAX_WAVES && lds_of<DT, D, 2>(w) <= HALF)
        return launch_q4<DT, D, 2>(c, w, q, kn, vn, out, st);
    if (blocks <= 4 * MAX_WAVES) return launch_q4<DT, D, 4>(c, (blocks + 3) / 4, q, kn, vn, out, st);
    return hipErrorInvalidValue;               // beyond H2O_Q4_MAX_BUDGET: refused at configuration time
}

}  // namespace

hipError_t h2o_launch_decode_q4(const h2o_cache &c, const void *q, const void *k_new,
                                const void *v_new, void *out, hipStream_t st)
{
    const int d = c.cfg.head_dim;
    switch (c.cfg.dtype) {
    case H2O_F32:
        return d == 64 ? pick_q4<H2O_F32, 64>(c, q, k_new, v_new, out, st)
                       : pick_q4<H2O_F32, 128>(c, q, k_new, v_new, out, st);
    case H2O_F16:
        return d == 64 ? pick_q4<H2O_F16, 64>(c, q, k_new, v_new, out, st)
                       : pick_q4<H2O_F16, 128>(c, q, k_new, v_new, out, st);
    default:
        return d == 64 ? pick_q4<H2O_BF16, 64>(c, q, k_new, v_new, out, st)
                       : pick_q4<H2O_BF16, 128>(c, q, k_new, v_new, out, st);
    }
}
