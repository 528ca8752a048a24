// Causal attention over the prompt on gfx950 (MFMA), with the row statistics
// that the column-sum pass needs as a by-product.  The nq queries are the last
// nq of nk key positions (nq = nk: the whole prompt; nq < nk: a chunk of the
// prompt attending to cached tokens in front of it): query i sees keys
// j <= nk - nq + i.
//
// The prompt phase of H2O is ordinary full attention over the prompt (App. A,
// generation commentary: the prompt is processed with the full cache and only
// then compressed); the accumulated scores are the column sums of the same
// softmax matrix (Algorithm 2's accumulate line over the prompt rows).  A layer
// therefore needs  O = softmax(scale * Q K^T) V  anyway, and the log-sum-exp of
// every row falls out of it: with this kernel the scoring costs one extra
// matrix pass (the column sums) instead of two.
//
// Shape of the computation.  A workgroup of 4 waves owns 128 queries (32 per
// wave, kept in registers as MFMA B-operand fragments) and streams 64-key
// tiles.  Per tile and wave:
//     S^T (keys x queries)  = K_tile . Q^T          16 MFMAs 32x32x16
//     online softmax over the keys seen so far (per query = per lane)
//     O^T (dims x queries) += V^T_tile . P^T        16 MFMAs 32x32x16 (d = 128)
// In the 32x32 result layout a lane holds ONE query's products with 16 keys
// (S^T) or 16 output dims (O^T): row maximum, normaliser and the rescaling of
// the output accumulator are per-lane scalars; the only cross-lane traffic is
// one exchange of the tile maximum between the two lane halves that share a
// query.  V is needed with the key index innermost (A operand of the second
// product): its tiles are copied into LDS row by row, exactly like key tiles, and
// read with the transposing LDS read, in which 16 lanes fetch 4 keys x 16 dims and
// each lane receives the 4 keys of one dim.  (A first version transposed V in global
// memory once per call: 49-52 us of the 650 + 50 us that 128 heads x 4096 tokens x 128
// take, and 20 of 160 us on a 1024-token chunk.)  The key rows of a tile are visited
// in an order that makes the 8 probabilities a lane holds for one MFMA step belong to
// 8 consecutive keys, so P^T goes from the accumulator registers into the second
// product without any shuffle and the V^T fragment is two 64-bit LDS reads.
//
// Schedule.  The copy of tile u+1 into the other stage runs while tile u is worked on.  Three forms:
//   one group of 4 waves: one barrier per tile.  Two workgroups share a CU (64 KB of LDS and 2 x 4
//     waves at ~200 registers each), and drift apart by themselves: while one multiplies the other
//     is in its softmax.
//   two groups together: for grids that leave CUs idle the keys of a tile are shared out to two groups
//     of 4 waves (two_groups); one barrier per tile still, and nothing keeps the groups of a
//     workgroup, mostly alone on its CU, out of each other's phase.
//   two groups one phase apart (groups_apart, SKEW below): two barriers per tile, and the second group
//     enters the loop one barrier late, so that one group multiplies while the other is in its softmax.
// An early version kept the halves of 8 waves with 256 queries one phase apart; one group of 4 measured
// against it (us, attention only, d = 128, f16): 8 heads x 300 tokens 14.8 -> 10.5, 32 x
// 1531 46 -> 41, 32 x 4096 153 -> 148, 128 x 4096 574 -> 563 (976 TFLOP/s), 3584 x 256 242 -> 191:
// short and few prompts gain most (half the work on the longest block), long ones lose
// nothing.
#include "h2o_internal.h"
#include "lds_copy.h"
#include <type_traits>

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int DT>
__device__ inline f32x16 mma16(const uint4 &a, const uint4 &b, f32x16 acc)
{
    if constexpr (DT == H2O_BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *reinterpret_cast<const bf16x8 *>(&a), *reinterpret_cast<const bf16x8 *>(&b), acc, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(
            *reinterpret_cast<const f16x8 *>(&a), *reinterpret_cast<const f16x8 *>(&b), acc, 0, 0, 0);
    }
}

// two floats -> one register of two 16-bit values (round to nearest even)
template <int DT> __device__ inline unsigned pack2(float a, float b)
{
    const f32x2 v = {a, b};
    if constexpr (DT == H2O_BF16) {
        const bf16x2 h = __builtin_convertvector(v, bf16x2);
        return *reinterpret_cast<const unsigned *>(&h);
    } else {
        const f16x2 h = __builtin_convertvector(v, f16x2);
        return *reinterpret_cast<const unsigned *>(&h);
    }
}

// value of the lane that shares this lane's query (lane ^ 32), combined with op
__device__ inline float other_half(float x)
{
    const unsigned own = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(own, own, false, false);
    // one of the two results is this lane's own value, the other the partner's
    return __uint_as_float(r[0] == own ? r[1] : r[0]);
}

constexpr int ARW = 4;       // waves over a workgroup's rows
constexpr int ANS = 2;       // stages (key tile + value tile each); copies run one tile ahead
constexpr int ABN = 64;      // keys per tile

// the 4 consecutive keys of one dim out of a row-major tile in LDS (transposing read: see above)
__device__ inline uint2 read_keys4(const unsigned char *lds)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)lds);
    return __builtin_bit_cast(uint2, r);
}

// ---- attention -------------------------------------------------------------------
// TWO: the first kf.rows keys and values of a head sit elsewhere (FrontRows): a tile is
// copied from one place or the other, and row by row in the one tile that has rows of both.
//
// G: groups of four waves over the same 128 queries.  With two, a tile is 128 keys and each
// group takes 64 of them; the two partial results are joined at the end.  For grids that
// leave CUs idle: the longest block has half the steps.
// SKEW: the groups run one phase apart, with a barrier between a step's MFMAs and its softmax.  Group
// g copies its own half of a tile at the start of its step u - 1 into rows that it has read
// last in step u - 2, and waits for them in front of the barrier that ends the step.
template <int DT, int D, bool TWO, int G, bool SKEW>
__global__ __launch_bounds__(ARW * G * 64, 2) void prefill_attn_kernel(
    const char *__restrict__ Qg, const char *__restrict__ Kg, const char *__restrict__ Vg,
    FrontRows kf, FrontRows vf, int nq, int nk, int heads, float c2, float *__restrict__ lse2,
    float *__restrict__ lse_nat, char *__restrict__ Og)
{
    const int off = nk - nq;               // key position of query 0
    constexpr int ROWB = D * 2;            // bytes per Q/K row
    constexpr int NF = ROWB / 32;          // 16-byte fragments per row per lane half
    constexpr int MB = ABN / 32;           // 32-key blocks per tile
    constexpr int NDB = D / 32;            // 32-dim blocks of the output
    constexpr int KS = ABN / 16;           // MFMA steps of the second product per tile
    constexpr int ANW = ARW * G;           // waves per workgroup
    constexpr int SBN = ABN * G;           // keys per tile, all groups
    constexpr int TILEK = SBN * ROWB;      // key tile bytes
    constexpr int STAGE = 2 * TILEK;       // key tile + value tile
    // XOR swizzle of 16-byte chunks inside a row (see the scoring passes)
    constexpr int CPRK = ROWB / 16, RSHK = ROWB >= 256 ? 0 : 1, KMASKK = (CPRK < 16 ? CPRK : 16) - 1;
    // Value rows are swizzled by 64-byte groups: a transposing read touches 4 consecutive
    // rows x 64 bytes per 32 lanes, which have to fall into four different bank groups.
    constexpr int VSH = ROWB >= 256 ? 0 : 1, VMASK = ROWB >= 256 ? 3 : 1;
    constexpr int NT = ANW * 64;
    constexpr int SROWS = ARW * 32;
    constexpr int CPTK = SBN * CPRK / NT;
    static_assert(SBN * CPRK % NT == 0 && CPTK >= 1, "copy split");

    extern __shared__ __align__(16) unsigned char smem[];   // [ANS][STAGE]

    const int tid = threadIdx.x, lane = tid & 63;
    // (the wave index as a scalar: branches on it are then uniform for the compiler
    // too, which otherwise keeps a second copy of the accumulators around them)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % ARW, grp = G > 1 ? wave / ARW : 0;
    const int half = lane >> 5, l32 = lane & 31;
    const int nblk = (nq + SROWS - 1) / SROWS;
    // a head lives on one XCD (one L2); heaviest (last) row blocks first
    const int hg = head_group(heads);
    const int xcd = blockIdx.x & 7, turn = blockIdx.x >> 3;
    const int group = turn / (hg * nblk), idx = turn % (hg * nblk);
    const int head = (group * hg + idx % hg) * 8 + xcd;
    if (head >= heads) return;
    const int blk = nblk - 1 - idx / hg;
    const int s0 = blk * SROWS;
    const char *Qh = Qg + (size_t)head * nq * ROWB;
    const int nf = TWO ? kf.rows : 0;
    const char *Kh = Kg + (size_t)head * (nk - nf) * ROWB;
    const char *Vh = Vg + (size_t)head * (nk - nf) * ROWB;

    const int srow = s0 + rw * 32 + l32;             // this lane's query

    // key tiles of this block (>= 1): up to the one that holds the last query's own key
    const int T = min((nk + SBN - 1) / SBN, (off + s0 + SROWS + SBN - 1) / SBN);

    // Copy plan: instruction c of a wave fills 64 chunks of LDS, the waves side by side; groups that
    // run one phase apart copy the rows that they read themselves, so that only their own waves
    // wait for them.
    const int first_copy = SKEW ? grp * CPTK * ARW + rw : wave;
    constexpr int copy_step = SKEW ? ARW : ANW;
    unsigned koff[CPTK], kchunk[CPTK], vchunk[CPTK];
#pragma unroll
    for (int c = 0; c < CPTK; ++c) {
        const unsigned q = (unsigned)(first_copy + c * copy_step) * 64u + lane;
        const unsigned r = q / CPRK, pos = q % CPRK;
        koff[c] = r * ROWB;
        kchunk[c] = (pos ^ ((r >> RSHK) & KMASKK)) * 16u;
        vchunk[c] = (pos ^ (((r >> VSH) & VMASK) << 2)) * 16u;
    }
    const i32x4 rsrc_k = make_rsrc(Kh, (unsigned)(nk - nf) * ROWB);
    const i32x4 rsrc_v = make_rsrc(Vh, (unsigned)(nk - nf) * ROWB);
    const i32x4 rsrc_kf = TWO ? make_rsrc(kf.front + (size_t)head * kf.stride * ROWB, (unsigned)nf * ROWB) : rsrc_k;
    const i32x4 rsrc_vf = TWO ? make_rsrc(vf.front + (size_t)head * vf.stride * ROWB, (unsigned)nf * ROWB) : rsrc_v;
    const unsigned edge = (unsigned)nf * ROWB;
    const unsigned lds_w = __builtin_amdgcn_readfirstlane(
        (unsigned)reinterpret_cast<size_t>(smem) + first_copy * 1024);
    const unsigned last_row_off = (unsigned)(nk - 1) * ROWB;
    // stage u holds what matrix phase u reads: key tile u (u < T) and value tile u-1 (u > 0)
    auto fetch = [&](int u, int stg) {
        const unsigned base = lds_w + stg * STAGE;
        // (rows past the end, only in a ragged last tile, repeat row nk-1: masked)
        auto tile = [&](const i32x4 &rsrc, const i32x4 &rsrc_f, int t, const unsigned *chunk, unsigned lds) {
            const unsigned t0 = (unsigned)t * (SBN * ROWB);
            if (TWO && t0 < edge) {
                if (t0 + SBN * ROWB <= edge) {                 // whole tile in front
#pragma unroll
                    for (int c = 0; c < CPTK; ++c) dma16(rsrc_f, koff[c] + chunk[c], t0, lds + c * copy_step * 1024);
                } else {                                       // rows of both
#pragma unroll
                    for (int c = 0; c < CPTK; ++c) {
                        const unsigned off = min(t0 + koff[c], last_row_off);
                        if (off < edge) dma16(rsrc_f, off + chunk[c], 0u, lds + c * copy_step * 1024);
                        else dma16(rsrc, off - edge + chunk[c], 0u, lds + c * copy_step * 1024);
                    }
                }
            } else if (t0 + SBN * ROWB <= (unsigned)nk * ROWB) {
#pragma unroll
                for (int c = 0; c < CPTK; ++c) dma16(rsrc, koff[c] + chunk[c], t0 - edge, lds + c * copy_step * 1024);
            } else {
#pragma unroll
                for (int c = 0; c < CPTK; ++c)
                    dma16(rsrc, min(t0 + koff[c], last_row_off) - edge + chunk[c], 0u, lds + c * copy_step * 1024);
            }
        };
        if (u < T) tile(rsrc_k, rsrc_kf, u, kchunk, base);
        if (u > 0) tile(rsrc_v, rsrc_vf, u - 1, vchunk, base + TILEK);
    };
    // The block's queries, through LDS as well (a fragment load straight from memory has 64 lanes on 32 rows: four
    // times the address work of whole rows, and two groups would load them twice), in stage 1, swizzled like key rows.
    static_assert(SROWS * ROWB <= STAGE, "a block's queries fit a stage");
    {
        const i32x4 rsrc_q = make_rsrc(Qh, (unsigned)nq * ROWB);
        const unsigned to = __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<size_t>(smem) + STAGE + wave * 1024);
#pragma unroll
        for (int c = 0; c < SROWS * CPRK / NT; ++c) {
            const unsigned q = (unsigned)(c * ANW + wave) * 64u + lane, r = q / CPRK, pos = q % CPRK;
            dma16(rsrc_q, (unsigned)min(s0 + (int)r, nq - 1) * ROWB + (pos ^ ((r >> RSHK) & KMASKK)) * 16u, 0u,
                  to + c * ANW * 1024);
        }
    }
    fetch(0, 0);

    // LDS read offsets.  Key rows are visited so that MFMA row 16a + 8b + 4c + e
    // of a 32-row block is key 16a + 8c + 4b + e (bits 2 and 3 exchanged): the
    // accumulator registers 8s..8s+7 of lane half h then hold keys
    // 16s + 8h + (0..7) of the block, which is exactly what the second
    // product's B operand needs.
    const int krow = (l32 & ~12) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    unsigned ka[NF][MB], va[NDB];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int row = mb * 32 + krow;
            ka[f][mb] = row * ROWB + (((2 * f + half) ^ ((row >> RSHK) & KMASKK)) * 16);
        }
    // Value fragments: lane 4q + i of a group of 16 fetches dims 4i..4i+3 of key q (and,
    // second read, of key 4 + q); lane halves take keys 0..7 / 8..15 of an MFMA step, the
    // two groups of a half dims 0..15 / 16..31 of a 32-dim block.
    {
        const int q = (lane & 15) >> 2, i = lane & 3;
        const int row = 8 * half + q;                    // (steps of 4 and 16 rows leave the swizzle alone)
#pragma unroll
        for (int db = 0; db < NDB; ++db)
            va[db] = TILEK + row * ROWB +
                     (((4 * db) ^ (((row >> VSH) & VMASK) << 2)) + 2 * ((lane >> 4) & 1) + (i >> 1)) * 16 + 8 * (i & 1);
    }
    auto value_fragment = [&](const unsigned char *sb, int db, int ks) {
        const uint2 lo = read_keys4(sb + va[db] + ks * 16 * ROWB);
        const uint2 hi = read_keys4(sb + va[db] + ks * 16 * ROWB + 4 * ROWB);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };

    float m_run = -INFINITY, l_run = 0.f;   // running maximum of the raw products / normaliser part
    f32x16 oacc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
    uint4 pfrag[KS];                        // probabilities of the previous tile, packed 16-bit
    bool live_prev = false;

    dma_wait_upto<0>();
    wg_barrier();
    uint4 st[NF];
    {
        const int row = rw * 32 + l32;
        const unsigned char *q = smem + STAGE + row * ROWB;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            st[f] = *reinterpret_cast<const uint4 *>(q + (((2 * f + half) ^ ((row >> RSHK) & KMASKK)) * 16));
    }
    if (srow >= nq) {
#pragma unroll
        for (int f = 0; f < NF; ++f) st[f] = make_uint4(0, 0, 0, 0);
    }
    wg_barrier();                           // every wave has its queries: stage 1 may be filled
    if (SKEW && grp == 1) wg_barrier();     // the second group runs one phase behind

    int stg = 0;
    // Iteration u: matrix phase = P.V of tile u-1 and Q.K of tile u, vector phase
    // = softmax of tile u.  MASKED: tile u touches the diagonal of this block's
    // rows; LAST: u == T (only the trailing P.V).
    auto step = [&](int u, auto masked_tag, auto last_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        constexpr bool LAST = decltype(last_tag)::value;
        if constexpr (!LAST) fetch(u + 1, stg ^ 1);          // into the stage of iteration u-1
        const unsigned char *sb = smem + stg * STAGE + grp * (ABN * ROWB);     // this group's rows of the tiles
        const int r0 = u * SBN + grp * ABN;
        const int w0 = s0 + rw * 32;
        // keys r0.. are visible to this wave only if r0 <= its last query
        const bool live = !LAST && (!MASKED || r0 <= off + w0 + 31);
        f32x16 sacc[MB];
        __builtin_amdgcn_s_setprio(2);
        // The waves that share a SIMD are in no fixed phase relation (they may all be in
        // their softmax; with SKEW one of them is), so a wave hides the LDS latency of its operand
        // reads itself: they run PF fragments ahead of the MFMAs that use them (a ring of PF
        // register quadruples).
        constexpr int PF = 4;
        if (live_prev) {
            constexpr int N = KS * NDB;
            uint4 ring[PF];
#pragma unroll
            for (int i = 0; i < PF; ++i)
                ring[i] = value_fragment(sb, i % NDB, i / NDB);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int ks = i / NDB, db = i % NDB;
                __builtin_amdgcn_sched_barrier(0);      // keep the reads PF ahead (the scheduler would pull them back)
                oacc[db] = mma16<DT>(ring[i % PF], pfrag[ks], oacc[db]);
                if (i + PF < N)
                    ring[i % PF] = value_fragment(sb, (i + PF) % NDB, (i + PF) / NDB);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (live) {
            constexpr int N = NF * MB;
            uint4 ring[PF];
#pragma unroll
            for (int i = 0; i < PF; ++i)
                ring[i] = *reinterpret_cast<const uint4 *>(sb + ka[i / MB][i % MB]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) sacc[mb][v] = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int f = i / MB, mb = i % MB;
                __builtin_amdgcn_sched_barrier(0);
                sacc[mb] = mma16<DT>(ring[i % PF], st[f], sacc[mb]);
                if (i + PF < N)
                    ring[i % PF] = *reinterpret_cast<const uint4 *>(sb + ka[(i + PF) / MB][(i + PF) % MB]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        // (m_run as an operand: the softmax, which starts from it, stays behind the barrier)
        if constexpr (SKEW) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : "+v"(m_run) : : "memory");

        if (live) {
            if constexpr (MASKED) {
                // a wave whose 32 queries all see the whole tile needs no mask (wave-uniform)
                if (r0 + ABN - 1 > off + w0) {
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int j = r0 + mb * 32 + 16 * (v >> 3) + 8 * half + (v & 7);
                            if (j > off + srow) sacc[mb][v] = -INFINITY;
                        }
                }
            }
            float mx = m_run;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; v += 2) mx = fmaxf(fmaxf(mx, sacc[mb][v]), sacc[mb][v + 1]);
            mx = fmaxf(mx, other_half(mx));              // both halves of a query use one reference
            // mx is finite from the first group's first tile on: key 0 is visible to every query
            if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {      // rescale only when a maximum moved
                float alpha = __builtin_amdgcn_exp2f((m_run - mx) * c2);         // 0 on the first tile
                if (G > 1 && m_run == mx) alpha = 1.f;     // (a query of the second group may have seen no key yet)
                l_run *= alpha;
                // in place (written as an instruction so that the branch leaves the
                // accumulator in the registers it already occupies).  The compiler does
                // not see what an asm statement reads, so the wait states a consumer of
                // a transcendental result needs are spelled out here.
                asm volatile("s_nop 4" : "+v"(alpha));
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        asm volatile("v_mul_f32 %0, %0, %1" : "+v"(oacc[db][v]) : "v"(alpha));
                m_run = mx;
            }
            const float nms = G > 1 && m_run == -INFINITY ? 0.f : -m_run * c2;
            float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    float p[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[mb][8 * s + e], c2, nms));
                    sum0 += (p[0] + p[2]) + (p[4] + p[6]);
                    sum1 += (p[1] + p[3]) + (p[5] + p[7]);
                    pfrag[2 * mb + s] = make_uint4(pack2<DT>(p[0], p[1]), pack2<DT>(p[2], p[3]),
                                                   pack2<DT>(p[4], p[5]), pack2<DT>(p[6], p[7]));
                }
            l_run += sum0 + sum1;
        }
        live_prev = live;
        stg ^= 1;
        dma_wait_upto<0>();                    // the next iteration's stage has landed
        if constexpr (SKEW)
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : "+v"(m_run), "+v"(l_run) : : "memory");
        else
            wg_barrier();
    };
    {
        const int t_diag0 = min(T, (off + s0 + 1) / SBN);   // tiles every query of the block sees in full
        for (int u = 0; u < t_diag0; ++u) step(u, std::false_type{}, std::false_type{});
        for (int u = t_diag0; u < T; ++u) step(u, std::true_type{}, std::false_type{});
        step(T, std::false_type{}, std::true_type{});
    }
    if (SKEW && grp == 0) wg_barrier();     // the barrier the second group spent at the start

    // ---- the groups' parts of a query, brought to the larger reference ----------------
    // Each group hands the other half of the output dims and finishes the rest.
    constexpr int FDB = NDB / G;            // 32-dim blocks that a wave finishes
    if constexpr (G > 1) {
        constexpr int PART = (FDB * 16 + 2) * 64;
        static_assert(ARW * 2 * PART * (int)sizeof(float) <= ANS * STAGE && NDB % G == 0, "the stages hold what both groups hand over");
        float *parts = reinterpret_cast<float *>(smem) + (size_t)rw * 2 * PART + lane;    // (stages are done with)
        float *mine = parts + grp * PART;
        const float *other = parts + (1 - grp) * PART;
        auto hand_over = [&](auto first) {
            mine[0] = m_run;
            mine[64] = l_run;
#pragma unroll
            for (int db = 0; db < FDB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(2 + db * 16 + v) * 64] = oacc[decltype(first)::value + db][v];
        };
        if (grp == 0) hand_over(std::integral_constant<int, FDB>{});
        else hand_over(std::integral_constant<int, 0>{});
        wg_barrier();
        // (group 0 has key 0: its reference is finite; group 1 may have seen nothing: weight 0)
        const float m1 = other[0], mx = fmaxf(m_run, m1);
        const float f0 = __builtin_amdgcn_exp2f((m_run - mx) * c2), f1 = __builtin_amdgcn_exp2f((m1 - mx) * c2);
        l_run = l_run * f0 + other[64] * f1;
        auto take_over = [&](auto first) {
#pragma unroll
            for (int db = 0; db < FDB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    constexpr int F = decltype(first)::value;
                    oacc[F + db][v] = oacc[F + db][v] * f0 + other[(2 + db * 16 + v) * 64] * f1;
                }
        };
        if (grp == 0) take_over(std::integral_constant<int, 0>{});
        else take_over(std::integral_constant<int, FDB>{});
        m_run = mx;
    }

    // ---- normalise and store ------------------------------------------------------
    const float l_tot = l_run + other_half(l_run);
    const float inv = 1.0f / l_tot;
    using E = Elem<DT>;
    typename E::T *orow = reinterpret_cast<typename E::T *>(Og) + ((size_t)head * nq + srow) * D;
    // The lane halves hold 4 dims each of every 8: they exchange so that one has all 8 of one group of
    // dims and the other those of the next, and 16 bytes go out at a time.  (A pair per conversion: element by
    // element, bf16 took a branch for NaNs on every one.)
    auto finish = [&](auto first) {
#pragma unroll
        for (int db = decltype(first)::value; db < decltype(first)::value + FDB; ++db)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                auto pair = [&](int v) { return pack2<DT>(oacc[db][v] * inv, oacc[db][v + 1] * inv); };
                const auto x = __builtin_amdgcn_permlane32_swap(pair(4 * g), pair(4 * g + 4), false, false);
                const auto y = __builtin_amdgcn_permlane32_swap(pair(4 * g + 2), pair(4 * g + 6), false, false);
                if (srow < nq)
                    *reinterpret_cast<uint4 *>(orow + 32 * db + 8 * (g + half)) = make_uint4(x[0], y[0], x[1], y[1]);
            }
    };
    if (G == 1 || grp == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, (G > 1 ? FDB : 0)>{});
    if (srow < nq && half == 0 && grp == 0) {
        const float l2 = m_run * c2 + __builtin_amdgcn_logf(l_tot);      // log2 of the row's normaliser
        lse2[(size_t)head * nq + srow] = l2;
        if (lse_nat) lse_nat[(size_t)head * nq + srow] = l2 * 0.69314718055994531f;
    }
}

template <int DT, int D, int G, bool SKEW>
hipError_t launch_attn(const h2o_config &cfg, double scale, const void *Q, const void *K,
                       const void *V, const FrontRows &kf, const FrontRows &vf, int nq, int nk, void *vcopy,
                       float *lse2, float *lse_nat, void *out, hipStream_t st)
{
    const int heads = cfg.batch * cfg.heads;
    hipError_t e = hipSuccess;
    // V is read until the last workgroup ends: an output written over it (in place) needs a copy
    const char *v0 = static_cast<const char *>(V), *o0 = static_cast<const char *>(out);
    const size_t vbytes = (size_t)heads * (nk - vf.rows) * D * 2, obytes = (size_t)heads * nq * D * 2;
    if (v0 < o0 + obytes && o0 < v0 + vbytes) {
        e = hipMemcpyAsync(vcopy, V, vbytes, hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) return e;
        V = vcopy;
    }
    constexpr int ANW = ARW * G;
    constexpr size_t smem = (size_t)ANS * 2 * ABN * G * D * 2;
    auto kern = kf.rows ? prefill_attn_kernel<DT, D, true, G, SKEW> : prefill_attn_kernel<DT, D, false, G, SKEW>;
    static std::atomic<uint64_t> raised[2] = {};
    if (smem > 48 * 1024) {
        e = allow_lds(reinterpret_cast<const void *>(kern), (int)smem, raised[kf.rows != 0]);
        if (e != hipSuccess) return e;
    }
    const int nblk = (nq + ARW * 32 - 1) / (ARW * 32);
    const float c2 = (float)(scale * 1.4426950408889634);
    hipLaunchKernelGGL(kern, dim3((unsigned)head_slots(heads) * nblk), dim3(ANW * 64), smem, st,
                       static_cast<const char *>(Q), static_cast<const char *>(K),
                       static_cast<const char *>(V), kf, vf, nq, nk, heads, c2, lse2, lse_nat,
                       static_cast<char *>(out));
    return hipGetLastError();
}

}  // namespace

size_t h2o_attn_vcopy_bytes(const h2o_config &cfg, int n)
{
    const size_t npad = ((size_t)n + ABN - 1) / ABN * ABN;      // (whole tiles: part of the ABI's scratch sizes)
    return (size_t)cfg.batch * cfg.heads * cfg.head_dim * npad * 2;
}

hipError_t h2o_launch_prefill_attention(const h2o_config &cfg, double scale, const void *Q,
                                        const void *K, const void *V, const FrontRows &Kf, const FrontRows &Vf,
                                        int nq, int nk, void *vcopy, float *lse2, float *lse_nat, void *out,
                                        hipStream_t st)
{
    const int d = cfg.head_dim;
    if (nq < 1 || nq > nk) return hipErrorInvalidValue;
    const bool few = two_groups(cfg.batch * cfg.heads, nq, nk, false, d);
    const bool apart = few && groups_apart(cfg.batch * cfg.heads, nq, nk, d);
#define H2O_ATTN(DT, D)                                                                                         \
    (apart ? launch_attn<DT, D, 2, true>(cfg, scale, Q, K, V, Kf, Vf, nq, nk, vcopy, lse2, lse_nat, out, st)    \
     : few ? launch_attn<DT, D, 2, false>(cfg, scale, Q, K, V, Kf, Vf, nq, nk, vcopy, lse2, lse_nat, out, st)   \
           : launch_attn<DT, D, 1, false>(cfg, scale, Q, K, V, Kf, Vf, nq, nk, vcopy, lse2, lse_nat, out, st))
    if (cfg.dtype == H2O_F16) return d == 64 ? H2O_ATTN(H2O_F16, 64) : H2O_ATTN(H2O_F16, 128);
    return d == 64 ? H2O_ATTN(H2O_BF16, 64) : H2O_ATTN(H2O_BF16, 128);
#undef H2O_ATTN
}
