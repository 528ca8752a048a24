// The generation step for few heads with long budgets: several workgroups per head.
//
// One workgroup per head leaves most of the chip idle when there are fewer heads
// than CUs, and a head's cache then streams at the rate of one CU (about 130 GB/s):
// 64 heads x 3277 slots (bf16, d = 128, 110 MB) took 41.5 us, 2.6 TB/s; split it takes
// 24.3 us: 15-18 us for the parts (6.0-7.1 TB/s), 1.8 between the launches and 3-4 for joining them.  Here `parts`
// workgroups share a head, each with a run of its slots, and a second, short launch
// puts the parts together.  What one part needs of the others (the softmax normaliser)
// is only needed for the scores and for the final scale of the output, so nothing in
// the first launch waits for anything:
//
//   decode_part_kernel    logits of the part's slots, e_j = exp(s_j - shift) and their
//                         sum (all fp64), output of the part normalised by the part's
//                         own sum (fp32 like the one-workgroup kernels)
//   decode_finish_kernel  one workgroup per head: the common normaliser, every slot's
//                         probability (rounded once to binary32), scores, eviction,
//                         overwrite, weighted sum of the parts' outputs (fp64)
//
// The shift is the token's own logit in every part, as in the one-workgroup kernels, so
// e_j, the normaliser and with them the probabilities and scores are the same numbers, to
// the order of the fp64 sum.  A part whose sum passes SHIFT_LIMIT takes its own maximum
// instead.  The limit is far below the range of a double, so that what the other parts are
// then scaled by, exp(token's logit - maximum), is either a normal number or belongs to
// probabilities that are zero in binary32: a part still on the token's logit has e_j <= e^345,
// and the factor is no longer normal only from a maximum 708 above it on (p < e^-363).  With the
// limit at the end of the range, tokens e^-40 to e^-100 below a part's maximum got wrong
// probabilities, or zero.
#include "wave_ops.h"

namespace {

constexpr int SPLIT_MAX_PARTS = 32;
constexpr int PNW = 8;                 // waves per workgroup (parts)
constexpr int FNT = 1024;              // threads per workgroup (finish)
constexpr int FSPT = H2O_MAX_BUDGET / FNT;
constexpr double SHIFT_LIMIT = 1e150;  // (e^345)

struct PartStat { double shift, sum, s_self, unused; };

// Scratch of one cache: e[heads][k], stat[heads][32], o[heads][32][d]
struct Scratch { double *e; PartStat *stat; float *o; };

// How a step is split: `parts` workgroups per head, `per` slots each (parts <= 1: it is not).
struct Plan { int parts, per; };

// The one-workgroup kernel's body without the bookkeeping: see decode_resident_kernel
// for the plan of the loads (all requests first, straight-line, none conditional) and
// for slot ownership.  Requires per <= U * RPI and 1 <= slots of every part.
template <int DT, int D, int U>
__global__ __launch_bounds__(PNW * 64, 4) void decode_part_kernel(const StepArgs args, const Scratch scratch, const Plan plan)
{
    const char *__restrict__ Kc = args.K, *__restrict__ Vc = args.V;
    const char *__restrict__ q_g = args.q, *__restrict__ kn_g = args.kn;
    double *__restrict__ e_g = scratch.e;
    PartStat *__restrict__ stat_g = scratch.stat;
    float *__restrict__ o_g = scratch.o;
    const int k = args.k, n_occ = args.n_occ, per = plan.per, parts = plan.parts;
    const double scale = args.scale;
    args_here(args);
    using E = Elem<DT>;
    using T = typename E::T;
    constexpr int EPL = E::EPL;
    constexpr int LPR = D / EPL;
    constexpr int RPW = 64 / LPR;
    constexpr int RPI = PNW * RPW;
    constexpr int OWN = U * RPW;
    constexpr int PITCH = LPR + 1;
    constexpr unsigned ROWB = D * sizeof(T);
    static_assert(OWN <= 64, "one slot per lane");

    const int head = blockIdx.x / parts, part = blockIdx.x % parts;
    const int first = part * per, n_loc = min(per, n_occ - first);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane / LPR, li = lane % LPR;

    __shared__ double part_l[PNW * OWN * PITCH];
    __shared__ double red_sum[PNW], red_max[PNW];
    __shared__ float p_l[PNW * OWN];
    __shared__ __align__(16) float o_l[PNW * D];
    double *part_w = part_l + wave * OWN * PITCH;
    float *p_w = p_l + wave * OWN;

    const size_t hoff = (size_t)head * k + first;
    const char *Kb = Kc + hoff * ROWB;
    const char *Vb = Vc + hoff * ROWB;
    const T *qh = reinterpret_cast<const T *>(q_g) + (size_t)head * D;
    const T *knh = reinterpret_cast<const T *>(kn_g) + (size_t)head * D;

    const int row0 = wave * RPW + sub, last = n_loc - 1;
    const int my_slot = (lane / RPW) * RPI + wave * RPW + (lane % RPW);
    const bool owner = lane < OWN && my_slot < n_loc;

    const uint4 qraw = *reinterpret_cast<const uint4 *>(qh + li * EPL);
    const uint4 kraw = *reinterpret_cast<const uint4 *>(knh + li * EPL);
    unsigned off[U];
    uint4 buf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        off[u] = (unsigned)min(u * RPI + row0, last) * ROWB + (unsigned)li * 16u;
        buf[u] = load_stream(Kb + off[u]);
        in_step(u, U);
    }
    __builtin_amdgcn_sched_barrier(0);

    double qd[EPL];
    double s_self;
    {
        const T *qe = reinterpret_cast<const T *>(&qraw);
        const T *ke = reinterpret_cast<const T *>(&kraw);
        double a = 0.0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            qd[i] = (double)E::to_f(qe[i]);
            a = fma((double)E::to_f(ke[i]), qd[i], a);
        }
        s_self = group_sum<LPR>(a) * scale;
    }

    // ---- logits
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const T *x = reinterpret_cast<const T *>(&buf[u]);
        double a0 = 0.0, a1 = 0.0;
#pragma unroll
        for (int i = 0; i < EPL; i += 2) {
            a0 = fma((double)E::to_f(x[i]), qd[i], a0);
            a1 = fma((double)E::to_f(x[i + 1]), qd[i + 1], a1);
        }
        buf[u] = load_stream(Vb + off[u]);
        part_w[(u * RPW + sub) * PITCH + li] = a0 + a1;
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();

    // ---- exponentials and the part's sum
    double s_j = 0.0;
    if (lane < OWN) {
        const double *pr = part_w + lane * PITCH;
        double a = pr[0], b = pr[1];
#pragma unroll
        for (int c = 2; c < LPR; c += 2) { a += pr[c]; b += pr[c + 1]; }
        s_j = (a + b) * scale;
    }
    double shift = s_self;
    double e_j = owner ? exp(s_j - shift) : 0.0;
    {
        const double dw = wave_sum(e_j);
        if (lane == 0) red_sum[wave] = dw;
    }
    lds_barrier();
    double den = 0.0;
#pragma unroll
    for (int w = 0; w < PNW; ++w) den += red_sum[w];
    if (!(den <= SHIFT_LIMIT)) {
        // some logit is > ~345 above the token's own: this part takes its maximum
        const double mw = wave_max(owner ? s_j : -INFINITY);
        if (lane == 0) red_max[wave] = mw;
        lds_barrier();
#pragma unroll
        for (int w = 0; w < PNW; ++w) shift = fmax(shift, red_max[w]);
        // (a logit of -inf has weight zero also where the whole part and the token's own have it)
        e_j = owner && s_j != -INFINITY ? exp(s_j - shift) : 0.0;
        const double dw = wave_sum(e_j);
        if (lane == 0) red_sum[wave] = dw;
        lds_barrier();
        den = 0.0;
#pragma unroll
        for (int w = 0; w < PNW; ++w) den += red_sum[w];
    }
    if (owner) e_g[hoff + my_slot] = e_j;
    // (a part whose logits all lie > ~745 below the token's own has weight zero)
    const float p_j = den == 0.0 ? 0.f : (float)(e_j / den);
    if (lane < OWN) p_w[lane] = p_j;
    __builtin_amdgcn_wave_barrier();

    // ---- output of the part
    float o[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) o[i] = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float p = p_w[u * RPW + sub];
        const T *x = reinterpret_cast<const T *>(&buf[u]);
#pragma unroll
        for (int i = 0; i < EPL; ++i) o[i] = fmaf(p, E::to_f(x[i]), o[i]);
        __builtin_amdgcn_sched_barrier(0);
    }
    wave_output_to_lds<EPL, LPR, D>(o, o_l, wave, sub, li);
    lds_barrier();
    const size_t po = (size_t)head * SPLIT_MAX_PARTS + part;
    if (tid < D) {
        float r = 0.f;
#pragma unroll
        for (int w = 0; w < PNW; ++w) r += o_l[w * D + tid];
        o_g[po * D + tid] = r;
    }
    if (tid == 0) {
        stat_g[po].shift = shift;
        stat_g[po].sum = den;
        stat_g[po].s_self = s_self;
    }
}

// One workgroup per head; a thread has the slots tid, tid + 1024, ...  Latency-bound
// (20 bytes per slot): every load is requested before the first use, a part's output is loaded
// by one group of D threads, and every wave works out the normaliser for itself, so that only one barrier is met.
// 64 heads x 3277 slots, first to last stamp: with all outputs in every thread, the factors in LDS behind a
// barrier of their own and their exponentials also where no part has left the token's logit 4.2 us, now 3.1.
template <int DT, int D, bool PAT>
__global__ __launch_bounds__(FNT) void decode_finish_kernel(const StepArgs args, const Scratch scratch, const Plan plan)
{
    char *__restrict__ Kc = args.K;
    char *__restrict__ Vc = args.V;
    float *__restrict__ acc_g = args.acc;
    int32_t *__restrict__ pos_g = args.pos;
    const char *__restrict__ kn_g = args.kn, *__restrict__ vn_g = args.vn;
    char *__restrict__ out_g = args.out;
    const double *__restrict__ e_g = scratch.e;
    const PartStat *__restrict__ stat_g = scratch.stat;
    const float *__restrict__ o_g = scratch.o;
    const int k = args.k, n_occ = args.n_occ, t = args.t, recent = args.recent, rank = args.rank, protect = args.protect,
              stride = args.stride, per = plan.per, parts = plan.parts;
    args_here(args);
    using E = Elem<DT>;
    using T = typename E::T;
    constexpr int EPL = E::EPL, LPR = D / EPL;
    constexpr unsigned ROWB = D * sizeof(T);
    constexpr int FNW = FNT / 64;
    constexpr int OG = FNT / D;                  // groups of D threads; group g adds up the parts g, g + OG, ...
    constexpr int OPG = SPLIT_MAX_PARTS / OG;

    const int head = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / (D / 64);
    const size_t hoff = (size_t)head * k, po = (size_t)head * SPLIT_MAX_PARTS;
    __shared__ double w_l[SPLIT_MAX_PARTS];      // factor of a part's exponentials
    __shared__ double red_key[FNW], red_all[FNW];
    __shared__ double o_l[OG][D];
    static_assert(SPLIT_MAX_PARTS <= 64 && D % 64 == 0, "one lane per part, whole waves per group");

    const PartStat st = stat_g[po + min(lane, parts - 1)];
    double e_j[FSPT];
    float acc_j[FSPT];
    int pos_j[FSPT];
#pragma unroll
    for (int i = 0; i < FSPT; ++i) {
        if (i * FNT >= n_occ) break;
        const int s = min(tid + i * FNT, n_occ - 1);
        e_j[i] = e_g[hoff + s];
        acc_j[i] = acc_g[hoff + s];
        pos_j[i] = pos_g[hoff + s];
    }
    // the outputs of this group's parts (column tid % D)
    float o_p[OPG];
#pragma unroll
    for (int i = 0; i < OPG; ++i) {
        if (i * OG >= parts) break;
        o_p[i] = o_g[(po + min(group + i * OG, parts - 1)) * D + tid % D];
    }
    const T v_self = reinterpret_cast<const T *>(vn_g)[(size_t)head * D + tid % D];
    const int li = lane % LPR;
    uint4 row = *reinterpret_cast<const uint4 *>(((lane / LPR) & 1 ? vn_g : kn_g) + (size_t)head * ROWB + li * 16);

    // the common normaliser: sums of the parts (lane p of every wave has part p), brought to
    // one shift by factors that are exactly one unless a part left the token's logit
    const bool has = lane < parts;
    const double s_self = lane_value(st.s_self, 0);
    // (every wave finds the same; a difference, so that an infinite logit does not pass)
    const bool plain = __ballot(!(st.shift - s_self == 0.0)) == 0;
    double f = 1.0, e_self = 1.0;
    if (!plain) {
        const double ref = fmax(s_self, wave_max(st.shift));
        f = exp(st.shift - ref);
        e_self = exp(s_self - ref);
        if (wave == 0 && has) w_l[lane] = f;
        __syncthreads();
    }
    const double sum = has ? st.sum * f : 0.0;
    const double den = e_self + wave_sum(sum);                 // (at most 32 x SHIFT_LIMIT)
    const float p_self = (float)(e_self / den);

    // ---- scores and the eviction candidates (as in the one-workgroup kernels)
    unsigned long long key = NO_CANDIDATE, key_all = NO_CANDIDATE;
    int key_slot = -1, key_all_slot = -1;
#pragma unroll
    for (int i = 0; i < FSPT; ++i) {
        if (i * FNT >= n_occ) break;
        const int s = tid + i * FNT;
        if (s < n_occ) {
            const float p_j = (float)((plain ? e_j[i] : e_j[i] * w_l[s / per]) / den);
            acc_j[i] += p_j;                                         // binary32 accumulate
            acc_g[hoff + s] = acc_j[i];
            const unsigned long long c =
                ((unsigned long long)__float_as_uint(rank_value(acc_j[i], pos_j[i], t, rank)) << 32) |
                (unsigned)pos_j[i];
            if (PAT ? !is_protected(pos_j[i], t, recent, protect, stride) : pos_j[i] <= t - recent) {
                if (c < key) { key = c; key_slot = s; }
            }
            if (PAT && c < key_all) { key_all = c; key_all_slot = s; }
        }
    }
    {
        const double kw = wave_min_f64(__longlong_as_double((long long)key));
        if (lane == 0) red_key[wave] = kw;
        if constexpr (PAT) {
            const double ka = wave_min_f64(__longlong_as_double((long long)key_all));
            if (lane == 0) red_all[wave] = ka;
        }
    }
    // ---- output: this group's parts, then the groups
    {
        const float w = (float)(sum / den);                          // (lane p: the weight of part p's output)
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < OPG; ++i) {
            const int p = group + i * OG;
            if (p >= parts) break;
            r = fma((double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), p)), (double)o_p[i], r);
        }
        o_l[group][tid % D] = r;
    }
    pin(row);                                        // the new token has arrived before any wave writes `out` (over it, perhaps)
    __syncthreads();
    if (tid < D) {
        double r = (double)p_self * (double)E::to_f(v_self);
#pragma unroll
        for (int g = 0; g < OG; ++g) r += o_l[g][tid];
        reinterpret_cast<T *>(out_g)[(size_t)head * D + tid] = E::from_f((float)r);
    }

    int tslot = -1;
    if (n_occ < k) {
        if (wave == 0) tslot = n_occ;
    } else {
        double wd = red_key[0];
#pragma unroll
        for (int w = 1; w < FNW; ++w) wd = fmin(wd, red_key[w]);
        if constexpr (PAT) {
            if (wd != wd) {                                          // the pattern covers every slot
                wd = red_all[0];
#pragma unroll
                for (int w = 1; w < FNW; ++w) wd = fmin(wd, red_all[w]);
                key = key_all;
                key_slot = key_all_slot;
            }
        }
        const unsigned long long win = (unsigned long long)__double_as_longlong(wd);
        const unsigned long long self_key =
            ((unsigned long long)__float_as_uint(p_self) << 32) | (unsigned)t;
        const bool evict = wd == wd && (PAT || recent != 0 || win < self_key);
        const unsigned long long b = __ballot(evict && key == win && key != NO_CANDIDATE);
        if (b != 0) tslot = __builtin_amdgcn_readlane(key_slot, __ffsll((long long)b) - 1);
    }
    if (tslot >= 0) {
        // (the lane that holds the winner also wrote that slot's old score above: the new
        // one goes out from the same lane, behind it)
        if (n_occ < k ? lane == 0 : key_slot == tslot) {
            pos_g[hoff + tslot] = t;
            acc_g[hoff + tslot] = p_self;
        }
        if (lane < 2 * LPR)
            *reinterpret_cast<uint4 *>((lane < LPR ? Kc : Vc) + (hoff + tslot) * ROWB + li * 16) = row;
    }
}

// How a step over n_occ slots is split (parts <= 1: it is not).  Rows of `rpw` per
// wave and load; a part holds at most `umax` rounds.
Plan plan_of(int heads, int n_occ, int rpw, bool f32)
{
    const int rpi = PNW * rpw, umax = rpw * 13 <= 64 ? 13 : 8;
    // Where the line lies.  A budget that the one-workgroup kernel holds in registers is
    // bound by the latency of one pass over it, which a second launch (1.8 us between the two and
    // 3 in the second) only adds to.  Beyond it, split / one workgroup (time of a step in a graph, one cache over and
    // over / 12 to 24 caches in turn, whose rows all come from HBM):
    //   16-bit, d = 128     33 to 64 heads: 481 0.85 .. 0.95 / 0.83 .. 0.94, 520 to 571 0.85 .. 0.95 / 0.79 .. 1.01, 700 0.82 / 0.91; 72 to 96: 481
    //                       to 520 0.94 .. 0.96 / 1.02 .. 1.09, 571 0.92 / 0.99 .. 1.03, from 600 on 0.74 .. 0.92 / 0.80 .. 0.98; 97 to 128:
    //                       545 1.01 (one), 571 0.92 .. 1.04 / 1.03 .. 1.10, from 600 on 0.75 .. 0.97 / 0.86 .. 1.05; 160: 0.97 .. 1.07; 200: 0.96 ..
    //                       1.22
    //   binary32, d = 64    33 to 88 heads: 577 0.83 .. 0.91 / 0.78 .. 1.00, 700 0.79 .. 0.97 / 0.81 .. 1.00; 96: 577 to 700 0.87 .. 0.95 / 0.93 ..
    //                       1.04; 128: 700 and 811 1.00 (one), 900 0.95 / 0.95; 160: 0.97 .. 1.14; 200: 1.01 .. 1.29
    //   binary32, d = 128   33 to 88 heads: 257 0.91 .. 1.07 (one), 300 0.82 .. 0.90 / 0.77 .. 0.99; 96: 300 to 345 0.86 .. 0.97 / 0.96 .. 1.05;
    //                       104 to 128: 300 to 416 0.85 .. 0.97 / 0.91 .. 1.12, 440 0.81 .. 0.94 / 0.91 .. 1.02; 160: 0.96 .. 1.11; 200: 1.03 .. 1.31
    //   16-bit, d = 64      to 160 heads: 513 to 640 0.75 .. 0.90 / 0.69 .. 0.98, 700 and 768 1.01 .. 1.12, 783 and 855 0.60 .. 0.93 / 0.63 ..
    //                       0.93; 200 and 255: 513 to 600 0.95 .. 1.03 / 0.99 .. 1.04, 640 0.96 / 0.97 .. 1.00, 783 on 0.82 .. 0.95 / 0.87 .. 0.96
    // Where the two disagree (72 to 128 heads next to a line) the line follows the first: with two or three caches in turn it is
    // still 0.79 .. 1.04, and what many lose, a tenth at most, is less than what few gain.
    // Up to 32 heads the first three lines are older and lie higher than what measures now (one cache: 0.76 .. 0.97 from
    // 481, 600 and 300 slots on).
    // With 128-byte rows the one-workgroup kernel's time depends on its ring: 8 and 2 rounds
    // are slow, 6 and 4 fast (255 heads: 1000 slots, ring 8, 20.2 us / split 16.0; 2048 40 / 27; 1061, ring 6, 13.0 /
    // 17.1; 1793 20.8 / 25.3; 1183, ring 4, 16.0 / 18.4;  160 heads: ring 6 1793 17.5 / 18.7, ring 4 1183 14.6 /
    // 14.0, 2708 29.5 / 24.4, 200 heads 1183 15.1 / 16.9;  128 heads: ring 6 1061 11.3 / 12.6, 1793 17.0 / 15.2).
    const int resident = rpi * (umax > 8 ? 15 : 8), rounds = (n_occ + rpi - 1) / rpi;
    int most_heads = 128;
    const int least_slots = rpw == 8 ? 0
                            : rpw == 2 ? (heads > 32 ? 300 : 417)
                            : f32      ? (heads <= 32 ? 865 : heads <= 96 ? 577 : 900)
                                       : (heads <= 32 ? 577 : heads <= 96 ? 0 : 571);
    if (rpw == 8) {
        const int ring = chunk_ring(rounds, umax);
        most_heads = ring == 6 ? (rounds > 18 ? 128 : 0) : ring == 4 ? 160 : 255;
    }
    if (heads > most_heads || n_occ <= resident || n_occ < least_slots) return {1, n_occ};
    int parts = 512 / heads;                                     // two workgroups per CU
    const int least = (n_occ + rpi * umax - 1) / (rpi * umax), most = (n_occ + rpi * 4 - 1) / (rpi * 4);
    if (parts > most) parts = most;
    if (parts < least) parts = least;
    if (parts > SPLIT_MAX_PARTS) parts = SPLIT_MAX_PARTS;
    if (parts < least) return {1, n_occ};
    const int per = ((n_occ + parts - 1) / parts + rpi - 1) / rpi * rpi;    // whole rounds
    return {(n_occ + per - 1) / per, per};
}

Scratch carve(const h2o_cache &c)
{
    const size_t heads = (size_t)c.cfg.batch * c.cfg.heads;
    Scratch s;
    s.e = static_cast<double *>(c.step_scratch);
    s.stat = reinterpret_cast<PartStat *>(s.e + heads * c.k);
    s.o = reinterpret_cast<float *>(s.stat + heads * SPLIT_MAX_PARTS);
    return s;
}

template <int DT, int D>
hipError_t launch(const h2o_cache &c, const void *q, const void *kn, const void *vn, void *out,
                  Plan p, hipStream_t st)
{
    constexpr int RPW = 64 / (D / Elem<DT>::EPL);
    constexpr int RPI = PNW * RPW;
    const int heads = c.cfg.batch * c.cfg.heads;
    const Scratch s = carve(c);
    const StepArgs args = step_args(c, q, kn, vn, out);
    auto part = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)heads * p.parts), dim3(PNW * 64), 0, st, args, s, p);
    };
    const int rounds = p.per / RPI;
    if (rounds <= 4) part(decode_part_kernel<DT, D, 4>);
    else if (rounds <= 6) part(decode_part_kernel<DT, D, 6>);
    else if (rounds <= 8) part(decode_part_kernel<DT, D, 8>);
    else if constexpr (RPW * 13 <= 64) {
        if (rounds <= 10) part(decode_part_kernel<DT, D, 10>);
        else part(decode_part_kernel<DT, D, 13>);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto finish = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(heads), dim3(FNT), 0, st, args, s, p);
    };
    if (c.cfg.protect == H2O_PROTECT_RECENT) finish(decode_finish_kernel<DT, D, false>);
    else finish(decode_finish_kernel<DT, D, true>);
    return hipGetLastError();
}

inline Plan plan_of(const h2o_config &c, int n_occ)
{
    return plan_of(c.batch * c.heads, n_occ, 1024 / (c.head_dim * h2o_esize(c.dtype)), c.dtype == H2O_F32);
}

}  // namespace

size_t h2o_split_scratch_bytes(const h2o_config &c)
{
    const size_t heads = (size_t)c.batch * c.heads, k = (size_t)c.heavy + c.recent;
    if (c.kv_bits != 0 || heads > 255 || plan_of(c, (int)k).parts <= 1) return 0;
    return heads * (k * sizeof(double) + SPLIT_MAX_PARTS * (sizeof(PartStat) + c.head_dim * sizeof(float)));
}

bool h2o_split_wanted(const h2o_cache &c)
{
    return c.step_scratch && plan_of(c.cfg, c.t < c.k ? c.t : c.k).parts > 1;
}

hipError_t h2o_launch_decode_split(const h2o_cache &c, const void *q, const void *k_new,
                                   const void *v_new, void *out, hipStream_t st)
{
    const int d = c.cfg.head_dim;
    const Plan p = plan_of(c.cfg, c.t < c.k ? c.t : c.k);
    switch (c.cfg.dtype) {
    case H2O_F32:
        return d == 64 ? launch<H2O_F32, 64>(c, q, k_new, v_new, out, p, st)
                       : launch<H2O_F32, 128>(c, q, k_new, v_new, out, p, st);
    case H2O_F16:
        return d == 64 ? launch<H2O_F16, 64>(c, q, k_new, v_new, out, p, st)
                       : launch<H2O_F16, 128>(c, q, k_new, v_new, out, p, st);
    default:
        return d == 64 ? launch<H2O_BF16, 64>(c, q, k_new, v_new, out, p, st)
                       : launch<H2O_BF16, 128>(c, q, k_new, v_new, out, p, st);
    }
}
