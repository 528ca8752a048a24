// Prompt scoring for H2O on gfx950 (MFMA): the column sums of the prompt's
// causal softmax matrix, which seed the accumulated attention scores
// (exact generative process of App. D "Eviction policy"; Algorithm 2's
// accumulate line applied to every prompt row).
//
//   pass 1 (row statistics) : LSE_i = log sum_{j<=i} exp(scale * <Q_i, K_j>)
//   pass 2 (column sums)    : c_j   = sum_{i>=j} exp(scale * <Q_i, K_j> - LSE_i)
//
// Both passes are the same dense contraction QK^T and run on the matrix cores;
// they differ in which operand stays in registers.  A workgroup's waves own 32
// "stationary" rows each (queries in pass 1, keys in pass 2; kept in registers as
// MFMA B-operand fragments) and stream tiles of the other operand through LDS
// as A-operand fragments.  Eight waves (four in the shape for smaller grids, two in
// binary32's for the smallest; either may have a second group of waves for half of a
// tile's rows) share one streamed tile: the copy into LDS and its address arithmetic are paid
// once per 256 stationary rows, which matters because the matrix pipe, the
// vector ALU (one exponential per product) and the vector memory path are all
// close to saturated by this loop.  With the 32x32 MFMA
// result layout a lane then holds one stationary row's products with 16 streamed
// rows per tile, so the reduction each pass needs (over keys for the row
// statistics, over queries for the column sums) runs inside a lane across the
// whole stream and needs no cross-lane traffic and no atomics; the two lane
// halves are merged once at the end.
//
// Everything is computed in base 2: x = (scale*log2 e) * <q,k>, the stored row
// statistic is log2 of the row's normaliser.
#include "h2o_internal.h"
#include "lds_copy.h"
#include <type_traits>

namespace {

#define CPR_OF(rowb) ((rowb) / 16)

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;


template <int DT>
__device__ inline f32x16 mma(const uint4 &a, const uint4 &b, f32x16 acc)
{
    if constexpr (DT == H2O_BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *reinterpret_cast<const bf16x8 *>(&a), *reinterpret_cast<const bf16x8 *>(&b), acc, 0, 0, 0);
    } else if constexpr (DT == H2O_F16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(
            *reinterpret_cast<const f16x8 *>(&a), *reinterpret_cast<const f16x8 *>(&b), acc, 0, 0, 0);
    } else {
        const float *af = reinterpret_cast<const float *>(&a);
        const float *bf = reinterpret_cast<const float *>(&b);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[e], bf[e], acc, 0, 0, 0);
        return acc;
    }
}

constexpr int NTB = 3;         // streamed-tile buffers (copies run two tiles ahead)
constexpr int NLB = 4;         // row-statistic buffers (pass 2; read one phase later than the tile)

// DT: element type; D: head_dim; MB: 32-row blocks per streamed tile;
// COLSUM: false = pass 1 (row statistics), true = pass 2 (column sums).
//
// Schedule.  Per streamed tile a wave has a matrix phase (16 MFMAs fed from LDS)
// and a vector phase (scale, exponential and sum of its 32x64 products), about
// equally long.  A SIMD runs both pipes at once only if its waves are in
// different phases, and waves that start together and meet at a barrier per
// tile stay in the same phase.  The eight waves therefore form two groups of
// four (wave w and w+4 sit on the same SIMD) that are kept one phase apart by
// the barriers themselves: the second group enters the loop one barrier late,
// so whenever one group is in its matrix phase the other is in its vector
// phase ("ping-pong").  s_setprio lets the matrix phase win the issue slot.
//
// RWV: waves over a workgroup's rows.  Eight (256 stationary rows, two workgroups per CU) is
// the shape for a full chip.  Four (128 rows) is for grids that do not fill it: the longest
// block then has half the work per tile.  Without SKEW its waves meet at one barrier per tile and
// the overlap is left to the workgroups that share a CU.  Two (64 rows, with two groups) is binary32's shape for the
// smallest grids (small_blocks): half the work again.
//
// The first kf.rows keys of a head may sit elsewhere (FrontRows).  Stationary rows are
// simply loaded from where they are; streamed ones (pass 1, TWO) are copied tile by tile
// from one or the other, and row by row in the one tile that has rows of both.
//
// G (shapes of four and of two waves): groups of waves over the same 128 or 64 stationary rows.  With two, a
// tile has twice the rows and each group takes half of them; the parts are joined at the
// end.  For grids that leave CUs idle: the longest block has half the steps.
// SKEW: the two halves of eight waves, of one shape or of two groups of four, run one phase apart: two
// barriers per tile, the second half one barrier behind.  (Two groups have a CU to themselves, no other
// workgroup overlaps with them.)
template <int DT, int D, int MB, int RWV, int G, bool TWO, bool COLSUM, bool SKEW>
__device__ __forceinline__ void prefill_pass(
    const char *__restrict__ Qg, const char *__restrict__ Kg, const FrontRows &kf, int nq, int nk, int heads,
    float c2, float *__restrict__ lse2, float *__restrict__ colsum, unsigned *zero)
{
    constexpr int ES = DT == H2O_F32 ? 4 : 2;
    constexpr int ROWB = D * ES;          // bytes per row
    constexpr int NF = ROWB / 32;         // 16-byte fragments per row per lane half
    constexpr int NWV = RWV * G;          // waves per workgroup
    constexpr int GN = 32 * MB;           // streamed rows per tile and group
    constexpr int BN = GN * G;            // streamed rows per tile
    constexpr int LROW = ROWB;            // LDS row pitch (chunks are XOR-swizzled instead of padded)
    constexpr int TILEB = BN * LROW;
    // Swizzle: 16-byte chunk c of tile row r is stored at chunk position
    // c ^ key(r), key = low bits of the row (of the row pair for 128-byte rows,
    // two of which span the banks once), so the 16 or 32 lanes that read the same
    // chunk of consecutive rows hit different banks.
    constexpr int RSH = ROWB >= 256 ? 0 : 1;
    constexpr int KMASK = (CPR_OF(ROWB) < 16 ? CPR_OF(ROWB) : 16) - 1;
    constexpr int CPR = ROWB / 16;        // 16-byte chunks per row
    constexpr int CHUNKS = BN * CPR;      // 16-byte chunks per tile
    constexpr int NT = NWV * 64;          // threads per workgroup
    constexpr int SROWS = RWV * 32;       // stationary rows per workgroup
    constexpr int CPT = CHUNKS / NT;      // tile-copy instructions per wave per tile
    constexpr int CPF = CPT + (COLSUM ? 1 : 0);   // copy instructions per wave per fetch
    constexpr int LPW = BN / NWV;         // row statistics each wave copies per tile
    // Pieces in which a wave's stationary rows fit its share of two tile buffers.  Loaded directly: where these are more
    // than two, or two halves of a 128-byte row (512 heads x 2048, d = 64, 410 us, copied 415), and binary32 rows without
    // a second group (a block is its matrix instructions there: 256 x 300, d = 128, 93.7 / 94.9, 8 x 256, d = 64, 25.8 / 25.1).
    // Prompts of up to 32 tokens pay 0.1 to 0.5 us for it (a barrier and an LDS read in front of their one tile; both passes, direct /
    // staged: f16, d = 128, 32 x 1 7.6 / 7.9, 32 x 17 7.7 / 7.75, d = 64 1024 x 17 9.8 / 10.4); leaving out that tile's second copy
    // there gains 2 to 4 % and costs 65 to 300 tokens 0.5 to 1.
    constexpr int SROUNDS = NWV * 16 / BN;
    constexpr bool STAGED = (SROUNDS == 1 || (SROUNDS == 2 && ROWB >= 256)) && (DT != H2O_F32 || G > 1);
    static_assert(CHUNKS % NT == 0 && CPT >= 1, "every thread moves the same number of chunks");
    static_assert(SROWS % BN == 0 && BN % NWV == 0 && LPW <= 64, "tiles divide the workgroup's rows");

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *tile_l = smem;                                        // [NTB][TILEB]
    float *lse_l = reinterpret_cast<float *>(smem + NTB * TILEB);        // [NLB][BN] (pass 2)

    const int tid = threadIdx.x, lane = tid & 63;
    // (the wave index as a scalar: branches on it are then uniform for the compiler too)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    static_assert(!SKEW || NWV == 8, "two groups of four waves");
    const int grp = SKEW ? wave >> 2 : 0; // ping-pong group
    const int rw = wave % RWV, part = G > 1 ? wave / RWV : 0;   // its 32 stationary rows, its part of a tile
    // The nq queries are the LAST nq positions of the nk keys (nq == nk for a whole
    // prompt; nq < nk when a chunk of new tokens attends to nk - nq cached tokens in
    // front of it): query row i sits at key position off + i and sees keys <= off + i.
    const int off = nk - nq;
    const int ns = COLSUM ? nk : nq;      // stationary rows
    const int nt = COLSUM ? nq : nk;      // streamed rows
    const int nblk = (ns + SROWS - 1) / SROWS;
    // Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD
    // has its own L2.  All blocks of a head share the streamed operand, so a head
    // lives on ONE XCD (ids that agree modulo 8) and its blocks run close together
    // in time: the operand is then fetched from HBM about once instead of once
    // per block.  On an XCD, heads are taken in groups of hg (about as many
    // workgroups as the XCD holds at once); inside a group the order is by block
    // weight, heaviest first over all its heads, so that the kernel does not end
    // on a few long blocks.
    const int hg = head_group(heads);
    const int xcd = blockIdx.x & 7, turn = blockIdx.x >> 3;
    const int group = turn / (hg * nblk), idx = turn % (hg * nblk);
    const int head = (group * hg + idx % hg) * 8 + xcd;
    if (head >= heads) return;                       // padding of the last head group
    const int ord = idx / hg;
    // heaviest blocks first: pass 1's last row block sees every key tile,
    // pass 2's first key block sees every query tile
    const int blk = COLSUM ? ord : nblk - 1 - ord;
    const int s0 = blk * SROWS;
    const int nf = kf.rows;                          // keys that sit in front
    const char *Kh = Kg + (size_t)head * (nk - nf) * ROWB;
    const char *Kfh = kf.front + (size_t)head * kf.stride * ROWB;
    const char *Sg = COLSUM ? Kh : Qg + (size_t)head * nq * ROWB;       // stationary operand
    const char *Tg = COLSUM ? Qg + (size_t)head * nq * ROWB : Kh;       // streamed operand

    const int srow = s0 + rw * 32 + l32;             // this lane's stationary row
    uint4 st[NF];
    // Rows past the end are clamped to the last row (in bounds) and zeroed after arrival.
    if constexpr (!STAGED) {
        const int r = min(srow, ns - 1);
        const char *row = !COLSUM ? Sg + (size_t)r * ROWB
                          : r < nf ? Kfh + (size_t)r * ROWB : Kh + (size_t)(r - nf) * ROWB;
#pragma unroll
        for (int f = 0; f < NF; ++f) st[f] = *reinterpret_cast<const uint4 *>(row + (2 * f + half) * 16);
        if (srow >= ns) {
#pragma unroll
            for (int f = 0; f < NF; ++f) st[f] = make_uint4(0, 0, 0, 0);
        }
    }

    const int ntile_all = (nt + BN - 1) / BN;
    // pass 1 streams the keys its last query can see; pass 2 streams the queries
    // from the first one that sees this block's first key
    const int t_begin = COLSUM ? max(0, s0 - off) / BN : 0;
    const int t_end = COLSUM ? ntile_all : min(ntile_all, (off + s0 + SROWS + BN - 1) / BN);

    // Staging of a streamed tile: copy instruction c of wave w fills LDS chunks
    // [(c*NWV + w)*64, +64) of the buffer; lane l's chunk q = that base + l sits in
    // tile row q / CPR at position q % CPR and comes from global chunk
    // (q % CPR) ^ key(row).  A head's operand is < 4 GiB: a 32-bit per-lane offset
    // inside the tile plus the tile's wave-uniform offset.  Rows past the end (only in a
    // ragged last tile) are clamped to the last row; what they hold is never used
    // (both passes mask them).  Pass 2 also copies the tile's BN row statistics,
    // LPW lanes of every wave taking LPW of them, so that every wave issues the
    // same number of copy instructions per tile and one wait count fits all.
    unsigned goff[CPT], gchunk[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const unsigned q = (unsigned)(c * NWV + wave) * 64u + lane;
        const unsigned r = q / CPR, pos = q % CPR;
        goff[c] = r * ROWB;
        gchunk[c] = ((pos ^ ((r >> RSH) & KMASK)) * 16u);
    }
    const i32x4 rsrc = make_rsrc(Tg, (unsigned)(COLSUM ? nt : nt - nf) * ROWB);
    const i32x4 rsrc_f = make_rsrc(TWO ? Kfh : Tg, TWO ? (unsigned)nf * ROWB : 0u);
    const i32x4 rsrc_lse = make_rsrc(lse2 + (size_t)head * nq, (unsigned)nq * 4u);
    // the low 32 bits of a generic pointer into LDS are the LDS byte offset
    const unsigned lds_w = __builtin_amdgcn_readfirstlane(
        (unsigned)reinterpret_cast<size_t>(tile_l) + wave * 1024);
    const unsigned lds_lse = (unsigned)reinterpret_cast<size_t>(lse_l);
    const unsigned last_row_off = (unsigned)(nt - 1) * ROWB;
    // i = index of the tile in this block's sequence (selects the buffers)
    auto fetch = [&](int tile, int tb, int lb) {
        const unsigned t0 = (unsigned)tile * (BN * ROWB);
        if (TWO && tile * BN < nf) {
            if (tile * BN + BN <= nf) {                        // whole tile in front
#pragma unroll
                for (int c = 0; c < CPT; ++c)
                    dma16(rsrc_f, goff[c] + gchunk[c], t0, lds_w + tb * TILEB + c * NWV * 1024);
            } else {                                           // rows of both
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const unsigned off = min(t0 + goff[c], last_row_off), edge = (unsigned)nf * ROWB;
                    const unsigned to = lds_w + tb * TILEB + c * NWV * 1024;
                    if (off < edge) dma16(rsrc_f, off + gchunk[c], 0u, to);
                    else dma16(rsrc, off - edge + gchunk[c], 0u, to);
                }
            }
        } else if (t0 + BN * ROWB <= (unsigned)nt * ROWB) {    // whole tile inside the operand
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                dma16(rsrc, goff[c] + gchunk[c], TWO ? t0 - (unsigned)nf * ROWB : t0,
                      lds_w + tb * TILEB + c * NWV * 1024);
        } else {
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                dma16(rsrc, min(t0 + goff[c], last_row_off) - (TWO ? (unsigned)nf * ROWB : 0u) + gchunk[c], 0u,
                      lds_w + tb * TILEB + c * NWV * 1024);
        }
        if constexpr (COLSUM) {
            // wave w copies the words [w * LPW, (w + 1) * LPW) of the buffer; statistics past
            // nq read as 0 (end of the descriptor) and are masked later
            // (two groups: clamped to the last one, a tile reaches twice as far)
            const unsigned to = lds_lse + lb * (BN * 4) + wave * (LPW * 4);
            if (lane < LPW) {
                if constexpr (G > 1)
                    dma4(rsrc_lse, (unsigned)min(tile * BN + wave * LPW + lane, nq - 1) * 4u, 0u, to);
                else
                    dma4(rsrc_lse, (unsigned)(wave * LPW + lane) * 4u, (unsigned)tile * (BN * 4u), to);
            }
        }
    };

    float m_run = -INFINITY, l_run = 0.f;   // pass 1: running max / sum (base 2)
    float c_run = 0.f;                      // pass 2: running column sum

    // Every block has at least one tile.  The first two are requested
    // here.  Requests past the block's last tile repeat
    // that tile (harmless, keeps the request count per iteration constant).
    if constexpr (STAGED) {
        // A wave's stationary rows go through its share of the tile buffers 1 and 2, SROUNDS pieces of each row in
        // turn: copied row by row they take a quarter of the address work of fragment loads, where
        // 64 lanes are on 32 rows (both passes, d = 128, us: 512 heads x 2048 654 -> 636, 3584 x 256 183 -> 166, 200 x 300 20.9
        // -> 18.3, 32 x 1531 37.7 -> 34.7, 32 x 512 17.3 -> 15.1, 8 x 4096 70.9 -> 68.3).
        constexpr int SEG = ROWB / SROUNDS, SCH = SEG / 16;        // bytes and chunks of a row per round
        constexpr int SSH = SEG >= 256 ? 0 : SEG >= 128 ? 1 : 2, SMASK = SCH - 1;
        constexpr int SCPT = 32 * SEG / 1024;                      // copies per wave and round
        const i32x4 rsrc_s = make_rsrc(Sg, (unsigned)(COLSUM ? nk - nf : nq) * ROWB);
        const i32x4 rsrc_sf = make_rsrc(COLSUM && nf ? Kfh : Sg, COLSUM ? (unsigned)nf * ROWB : 0u);
        unsigned char *area = tile_l + TILEB + wave * (32 * SEG);
        const unsigned area_lds = __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<size_t>(area));
        auto copy_rows = [&](int round) {
#pragma unroll
            for (int c = 0; c < SCPT; ++c) {
                const unsigned q = (unsigned)c * 64u + lane, r = q / SCH, pos = q % SCH;
                const int row = min(s0 + rw * 32 + (int)r, ns - 1);
                const unsigned at = (unsigned)round * SEG + (pos ^ ((r >> SSH) & SMASK)) * 16u;
                if (COLSUM && row < nf) dma16(rsrc_sf, (unsigned)row * ROWB + at, 0u, area_lds + c * 1024);
                else dma16(rsrc_s, (unsigned)(COLSUM ? row - nf : row) * ROWB + at, 0u, area_lds + c * 1024);
            }
        };
        copy_rows(0);
        fetch(t_begin, 0, 0);
#pragma unroll
        for (int round = 0; round < SROUNDS; ++round) {
            if (round == 0) dma_wait_upto<CPF>();
            else dma_wait_upto<0>();
#pragma unroll
            for (int i = 0; i < NF / SROUNDS; ++i)
                st[round * (NF / SROUNDS) + i] = *reinterpret_cast<const uint4 *>(
                    area + l32 * SEG + (((2 * i + half) ^ ((l32 >> SSH) & SMASK)) * 16));
            if (round + 1 < SROUNDS) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                copy_rows(round + 1);
            }
        }
        if (srow >= ns) {
#pragma unroll
            for (int f = 0; f < NF; ++f) st[f] = make_uint4(0, 0, 0, 0);
        }
        wg_barrier();                      // every wave has its rows: the buffers may be filled
        fetch(min(t_begin + 1, t_end - 1), 1, 1);
        dma_wait_upto<CPF>();
    } else {
        // (waiting for the first tile also completes the stationary loads above: vector loads finish in order)
        fetch(t_begin, 0, 0);
        fetch(min(t_begin + 1, t_end - 1), 1, 1);
        dma_wait_upto<CPF>();
        // tell the compiler that the stationary fragments have arrived (it cannot see
        // the wait above), or it would re-wait for them, and with them for the tile
        // copies in flight, in front of the MFMAs of every iteration
#pragma unroll
        for (int f = 0; f < NF; ++f)
            asm volatile("" ::"v"(st[f].x), "v"(st[f].y), "v"(st[f].z), "v"(st[f].w));
    }
    wg_barrier();
    if (grp == 1) wg_barrier();            // second group runs one phase behind

    int tb = 0, lb = 0;                    // buffers of the current tile
    // One streamed tile.  MASKED = the tile touches the causal diagonal of this
    // workgroup's rows or runs past the prompt's end; those tiles run in loops of
    // their own so that the others (most) carry no masking arithmetic at all.
    // In a diagonal tile a wave whose 32 rows see none of the tile's rows skips
    // the arithmetic (it still copies its share of a later tile and meets the
    // barriers).
    //
    // Buffer life times: the tile two ahead is requested at the start of the
    // matrix phase into the buffer of the previous tile, which both groups have
    // finished reading (the later group's matrix phase of that tile ended at the
    // barrier this group has just passed; without SKEW everybody's did).  Row statistics are read in the
    // vector phase, one barrier later, hence one buffer more.  Before either barrier a
    // wave waits until only its newest request is outstanding, so that by the
    // barrier in front of any matrix phase every wave's share of that tile has
    // landed.
    auto tile_step = [&](int tile, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        const int tb2 = tb == 0 ? NTB - 1 : tb - 1;               // (tb + 2) % 3
        fetch(min(tile + 2, t_end - 1), tb2, (lb + 2) & (NLB - 1));
        const int r0 = tile * BN + part * GN;     // first row of this wave's part of the tile
        const int w0 = s0 + rw * 32;              // first stationary row of this wave
        // pass 1: keys r0.. are visible to the queries at positions >= r0; pass 2:
        // the queries up to position off+r0+BN-1 see the keys up to there
        const bool live = !MASKED || (COLSUM ? off + r0 + GN - 1 >= w0 : r0 <= off + w0 + 31);
        // Of the tiles that touch the block's diagonal, a wave's own 32 rows straddle
        // only one; those in front of it are fully visible to the wave and need no
        // mask arithmetic (wave-uniform test).
        const bool clear = !COLSUM && r0 + GN - 1 <= off + w0;
        f32x16 acc[MB];
        if (live) {
            __builtin_amdgcn_s_setprio(2);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;
            const unsigned char *tbp = tile_l + tb * TILEB + part * (GN * LROW);
            auto fragment = [&](int f, int mb) {
                const int row = mb * 32 + l32;
                return *reinterpret_cast<const uint4 *>(
                    tbp + row * LROW + (((2 * f + half) ^ ((row >> RSH) & KMASK)) * 16));
            };
            if constexpr (ROWB >= 256) {
                // the fragments of k-step f + 1 are requested before the MFMAs of k-step f
                // are issued (the scheduling fences keep it that way; left alone the compiler
                // requests a k-step's fragments and waits for them on the spot): an LDS read
                // then has two MFMAs' time to come back
                uint4 a_cur[MB], a_nxt[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) a_cur[mb] = fragment(0, mb);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    if (f + 1 < NF) {
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) a_nxt[mb] = fragment(f + 1, mb);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[mb] = mma<DT>(a_cur[mb], st[f], acc[mb]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) a_cur[mb] = a_nxt[mb];
                }
            } else {
                // (128-byte rows: four k-steps per tile; the read-ahead's eight registers
                // would cost pass 2 its third workgroup per CU, which is worth more)
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[mb] = mma<DT>(fragment(f, mb), st[f], acc[mb]);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        if constexpr (SKEW) {
            dma_wait_upto<CPF>();
            wg_barrier();
        }

        if (live) {
            if constexpr (!COLSUM) {
                // streamed rows are keys j, this lane's row is the query at position
                // off + srow: need j <= off + srow.
                // m_run tracks the maximum of the raw products (c2 > 0 keeps the order);
                // the scale is folded into the exponent's fma
                if constexpr (MASKED) {
                    if (!clear) {
                        const int last = off + srow - r0 - 4 * half;     // last visible row of this lane's
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                if (mb * 32 + 8 * (v >> 2) + (v & 3) > last) acc[mb][v] = -INFINITY;
                    }
                }
                float mx = m_run;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int v = 0; v < 16; v += 2) mx = fmaxf(fmaxf(mx, acc[mb][v]), acc[mb][v + 1]);
                const float ms = mx == -INFINITY ? 0.f : mx;
                const float nms = -ms * c2;
                float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        sum0 += __builtin_amdgcn_exp2f(fmaf(acc[mb][v], c2, nms));
                        sum1 += __builtin_amdgcn_exp2f(fmaf(acc[mb][v + 1], c2, nms));
                    }
                l_run = l_run * __builtin_amdgcn_exp2f((m_run - ms) * c2) + (sum0 + sum1);
                m_run = mx;
            } else {
                // streamed rows are queries i (at position off + i), this lane's row is
                // key j = srow: need j <= off + i, i < nq
                const float *ll = lse_l + lb * BN + part * GN;
                float sum0 = 0.f, sum1 = 0.f;
                // `count` of this lane's rows of the stream count, from row `first` of the tile on
                const int first = srow - off - r0 - 4 * half;
                const unsigned count = max(0, nq + off - srow);
                auto add_up = [&](auto first_tag, auto end_tag) {
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int gq = 0; gq < 4; ++gq) {
                            const float4 l4 = *reinterpret_cast<const float4 *>(ll + mb * 32 + 8 * gq + 4 * half);
                            const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
                            float x[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                x[e] = fmaf(acc[mb][4 * gq + e], c2, -lv[e]);
                                const int row = mb * 32 + 8 * gq + e;
                                if constexpr (decltype(end_tag)::value)
                                    x[e] = (unsigned)(row - first) >= count ? -INFINITY : x[e];
                                else if constexpr (decltype(first_tag)::value)
                                    x[e] = row < first ? -INFINITY : x[e];
                            }
                            sum0 += __builtin_amdgcn_exp2f(x[0]) + __builtin_amdgcn_exp2f(x[2]);
                            sum1 += __builtin_amdgcn_exp2f(x[1]) + __builtin_amdgcn_exp2f(x[3]);
                        }
                };
                // (what a tile needs is the same for the whole wave; tested per element, a masked
                // tile took three times the instructions: both passes 1 to 6 % slower, 256
                // heads x 300 24.3 us against 22.8, 32 x 1531 40.8 / 39.0, 128 x 4096 555 / 549.  binary32,
                // d = 128, has no registers for three ways and takes both ends as one range: two comparisons
                // per element had made it 2 % slower where several workgroups share a CU, 256 heads x 300
                // 96.1 us, now 93.6, tested per element 93.8; 128 x 300 79.1 / 78.2 / 81.0)
                if constexpr (!MASKED) {
                    add_up(std::false_type{}, std::false_type{});
                } else if constexpr (ROWB >= 512) {
                    add_up(std::true_type{}, std::true_type{});
                } else if (r0 + GN > nq) {
                    add_up(std::true_type{}, std::true_type{});
                } else if (off + r0 < w0 + 31) {
                    add_up(std::true_type{}, std::false_type{});
                } else {
                    add_up(std::false_type{}, std::false_type{});
                }
                c_run += sum0 + sum1;
            }
        }
        tb = tb == NTB - 1 ? 0 : tb + 1;
        lb = (lb + 1) & (NLB - 1);
        dma_wait_upto<CPF>();
        // The step's closing barrier takes the running sums as operands: pass 1's vector
        // phase touches no memory, so only this data dependence keeps its arithmetic in
        // front of the barrier.  (Left free, a build has put the whole vector phase behind
        // it; the two wave groups then take turns instead of overlapping.)
        if constexpr (COLSUM)
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : "+v"(c_run) : : "memory");
        else
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : "+v"(m_run), "+v"(l_run) : : "memory");
    };
    // Tiles that need the mask: in pass 1 from the first key tile that reaches past
    // the position of this block's first query; in pass 2 up to the last query tile
    // that does not yet see this block's last key.
    if constexpr (!COLSUM) {
        const int t_diag0 = min(t_end, (off + s0 + 1) / BN);
        for (int tile = t_begin; tile < t_diag0; ++tile) tile_step(tile, std::false_type{});
        for (int tile = t_diag0; tile < t_end; ++tile) tile_step(tile, std::true_type{});
    } else {
        const int x = s0 + SROWS - 1 - off;      // first query (local) that sees the whole block
        const int t_diag1 = min(t_end, max(t_begin, x > 0 ? (x + BN - 1) / BN : 0));
        // a ragged last tile holds rows past nq: it takes the masking path as well
        const int t_rag = (nq % BN) ? max(t_diag1, t_end - 1) : t_end;
        for (int tile = t_begin; tile < t_diag1; ++tile) tile_step(tile, std::true_type{});
        for (int tile = t_diag1; tile < t_rag; ++tile) tile_step(tile, std::false_type{});
        for (int tile = t_rag; tile < t_end; ++tile) tile_step(tile, std::true_type{});
    }
    if (SKEW && grp == 0) wg_barrier();    // the barrier the second group spent at the start
    dma_wait_upto<0>();                    // trailing repeat requests land before the LDS is released

    if constexpr (G > 1) {
        // the second group's part of every row (the tiles are done with)
        float2 *join = reinterpret_cast<float2 *>(smem) + rw * 64 + lane;
        wg_barrier();
        if (part == 1) *join = COLSUM ? make_float2(c_run, 0.f) : make_float2(m_run, l_run);
        wg_barrier();
        if (part == 1) return;
        const float2 o = *join;
        if constexpr (COLSUM) {
            c_run += o.x;
        } else {
            const float M = fmaxf(m_run, o.x), ms = M == -INFINITY ? 0.f : M;     // (a lane half may have seen no key)
            l_run = l_run * __builtin_amdgcn_exp2f((m_run - ms) * c2) + o.y * __builtin_amdgcn_exp2f((o.x - ms) * c2);
            m_run = M;
        }
    }
    if constexpr (!COLSUM) {
        const float m2 = __shfl_xor(m_run, 32, 64), l2 = __shfl_xor(l_run, 32, 64);
        const float M = fmaxf(m_run, m2);            // finite: key 0 is visible to every query
        const float L = l_run * __builtin_amdgcn_exp2f((m_run - M) * c2) +
                        l2 * __builtin_amdgcn_exp2f((m2 - M) * c2);
        if (half == 0 && srow < nq) lse2[(size_t)head * nq + srow] = M * c2 + __builtin_amdgcn_logf(L);
    } else {
        const float c = c_run + __shfl_xor(c_run, 32, 64);
        if (half == 0 && srow < nk) colsum[(size_t)head * nk + srow] = c;
        if (zero && srow == 0) zero[head] = 0u;
    }
}

template <int DT, int D, int MB, bool COLSUM>
__global__ __launch_bounds__(8 * 64, 4) void prefill_pass_kernel(
    const char *__restrict__ Qg, const char *__restrict__ Kg, FrontRows kf, int nq, int nk, int heads, float c2,
    float *__restrict__ lse2, float *__restrict__ colsum, unsigned *zero)
{
    prefill_pass<DT, D, MB, 8, 1, false, COLSUM, true>(Qg, Kg, kf, nq, nk, heads, c2, lse2, colsum, zero);
}

template <int DT, int D, int MB, int G, bool TWO, bool COLSUM, bool SKEW>
__global__ __launch_bounds__(4 * G * 64, G == 1 ? 4 : 2) void prefill_pass4_kernel(
    const char *__restrict__ Qg, const char *__restrict__ Kg, FrontRows kf, int nq, int nk, int heads, float c2,
    float *__restrict__ lse2, float *__restrict__ colsum, unsigned *zero)
{
    prefill_pass<DT, D, MB, 4, G, TWO, COLSUM, SKEW>(Qg, Kg, kf, nq, nk, heads, c2, lse2, colsum, zero);
}

// Two groups of two waves: 64 stationary rows
template <int DT, int D, bool TWO, bool COLSUM>
__global__ __launch_bounds__(4 * 64, 2) void prefill_pass2_kernel(
    const char *__restrict__ Qg, const char *__restrict__ Kg, FrontRows kf, int nq, int nk, int heads, float c2,
    float *__restrict__ lse2, float *__restrict__ colsum, unsigned *zero)
{
    prefill_pass<DT, D, 1, 2, 2, TWO, COLSUM, false>(Qg, Kg, kf, nq, nk, heads, c2, lse2, colsum, zero);
}

// TWO: streamed rows in two places (pass 1 with keys in front, four waves)
template <int DT, int D, int RWV, int G, bool TWO, bool COLSUM, bool SKEW = false>
hipError_t launch_pass(const h2o_config &cfg, double scale, const void *Q, const void *K, const FrontRows &kf,
                       int nq, int nk, float *lse2, float *colsum, unsigned *zero, hipStream_t st)
{
    constexpr int SROWS = RWV * 32, NWV = RWV * G;
    constexpr int ES = DT == H2O_F32 ? 4 : 2;
    constexpr int MB = (D * ES >= 512 || RWV == 2) ? 1 : 2;      // keep a group's tile buffers at 48 KiB
    constexpr int BN = 32 * MB * G;
    constexpr size_t smem = NTB * (size_t)BN * (D * ES) + NLB * BN * sizeof(float);
    const int heads = cfg.batch * cfg.heads;
    const int nblk = ((COLSUM ? nk : nq) + SROWS - 1) / SROWS;
    const float c2 = (float)(scale * 1.4426950408889634);
    auto kern = [] {
        if constexpr (RWV == 8) return prefill_pass_kernel<DT, D, MB, COLSUM>;
        else if constexpr (RWV == 2) return prefill_pass2_kernel<DT, D, TWO, COLSUM>;
        else return prefill_pass4_kernel<DT, D, MB, G, TWO, COLSUM, SKEW>;
    }();
    if (smem > 48 * 1024) {
        static std::atomic<uint64_t> raised{0};
        const hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), (int)smem, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern,
                       dim3((unsigned)head_slots(heads) * nblk),
                       dim3(NWV * 64), smem, st, static_cast<const char *>(Q),
                       static_cast<const char *>(K), kf, nq, nk, heads, c2, lse2, colsum, zero);
    return hipGetLastError();
}

// Whether a grid below the line of pick_waves takes eight waves all the same: where their
// blocks fill the CUs evenly.  binary32 (a pass is bound by its matrix instructions) loses
// 10-18 % to four waves on equal numbers of rows, which their finer blocks make up for elsewhere.
// Measured, both passes, four waves / eight:
//   one block per head (129..256 rows)
//     binary32, d = 128     heads 128: 0.72, 130-256: 1.16, 264-448: 0.95, 456-512: 1.10-1.18, 528-640:
//                           0.92-0.97, 768: 1.10-1.13, 896: 1.00, 1024: 1.10, 1280-3584: 0.99-1.08
//     16-bit, d = 128       heads 136-448: 0.85-0.95, 456-512: 1.10, 528-1024: 0.83-1.00; d = 64: 0.79-1.01
//   two blocks, binary32    385..512 rows: heads 288: 0.96, 296-320: 1.04-1.11, 328: 0.86; 128 and below: two
//                           groups (pick_waves)
//   a chunk of 512 tokens on 410..2048 cached ones, binary32, d = 128 (all blocks about equally
//   heavy), the whole call: 256 heads 1.06-1.10, 192: 0.92-0.98, 384: 0.91-0.98
template <int DT, int D> bool eight_fill_the_chip(long long blocks8, int rows, int streamed)
{
    if ((rows - 1) % 256 < 128 || rows > 512) return false;     // the last block half empty / many blocks
    const bool last_round = blocks8 > 448 && blocks8 <= 512;     // two workgroups on (nearly) every CU
    if (DT != H2O_F32) return D == 128 && rows <= 256 && last_round;
    if (rows <= 256) {
        const long long rounds = (blocks8 + 255) / 256;
        return rounds == 1 ? blocks8 > 128 : 8 * blocks8 > 7 * 256 * rounds;
    }
    return 2LL * streamed >= 3LL * rows ? last_round : streamed == rows && blocks8 > 576 && blocks8 <= 640;
}

template <int DT, int D, bool COLSUM>
hipError_t pick_waves(const h2o_config &cfg, double scale, const void *Q, const void *K, const FrontRows &kf,
                      int nq, int nk, float *lse2, float *colsum, unsigned *zero, hipStream_t st)
{
    const int rows = COLSUM ? nk : nq, streamed = COLSUM ? nq : nk;
    const bool few = two_groups(cfg.batch * cfg.heads, rows, streamed, DT == H2O_F32, D);
    // The two groups one phase apart, as the halves of eight waves are: one barrier more per tile, which
    // short streams and binary32 (a pass is its MFMAs there) do not pay back.  Apart / together, time of
    // both passes, whole prompts, both 16-bit types, d = 128, 1 to 256 heads:
    //   to 256 blocks  2500 rows on 0.89 .. 0.95, 1100 on 0.91 .. 0.97, 800 on 0.96 .. 1.03, below 1.00 .. 1.04
    //   to 512         2500 rows on 0.91 .. 0.98, 1100 on 0.93 .. 1.06 by how the last round of blocks fills (mean
    //                  0.99: 16 heads x 2300 0.93, 32 x 1531 1.04; left together), below 1.03 .. 1.08
    // d = 64 8 heads x 4096 61.6 us together / 60.3 apart, 16 x 4000 70.8 / 71.4, 32 x 700 17.3 / 17.8; binary32 16 x 1500 209 / 213.
    constexpr bool CAN = DT != H2O_F32 && D == 128;
    const bool apart = CAN && few &&
                       (streamed >= 2500 || (streamed >= 800 && (long long)cfg.batch * cfg.heads * ((rows + 127) / 128) <= 256));
    if constexpr (DT == H2O_F32)
        if (small_blocks(cfg.batch * cfg.heads, rows, streamed, D)) {
            if constexpr (!COLSUM)
                if (kf.rows) return launch_pass<DT, D, 2, 2, true, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
            return launch_pass<DT, D, 2, 2, false, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
        }
    if constexpr (!COLSUM)
        if (kf.rows)
            return apart ? launch_pass<DT, D, 4, 2, true, COLSUM, CAN>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
                   : few ? launch_pass<DT, D, 4, 2, true, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
                       : launch_pass<DT, D, 4, 1, true, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
    // Eight waves pay off when the grid fills the chip several times over with long streams:
    // the line is drawn on blocks x streamed rows.  Both passes, us, eight / four waves:
    //   16-bit, d = 128   32 heads x 512: 26.5 / 19.7, 32 x 1531: 59 / 51, 32 x 4096 (2.1 M):
    //                     198 / 186, 128 x 2048 (2.1 M): 181 / 178, 64 x 4096 (4.2 M): 286 / 302,
    //                     512 x 2048 (8.4 M): 655 / 670, 128 x 4096 (8.4 M): 566 / 586
    //                     (1 to 3 M: four waves at 0.88 to 1.04 of eight, by how the last round fills)
    //   16-bit, d = 64    128 x 2048: 127 / 120, 128 x 4096 (8.4 M): 396 / 394, 128 x 8192 (34 M): 1420 / 1448
    //   binary32          d = 64, 64 x 2048: 382 / 304, 128 x 4096 (8.4 M): 2197 / 2172;
    //                     d = 128, 128 x 1024: 489 / 336, 128 x 4096: 4187 / 4173
    const long long blocks8 = (long long)cfg.batch * cfg.heads * ((rows + 255) / 256);
    constexpr long long LINE = DT != H2O_F32 && D == 128 ? 3000000 : 16000000;
    if (blocks8 * streamed > LINE || (!few && eight_fill_the_chip<DT, D>(blocks8, rows, streamed)))
        return launch_pass<DT, D, 8, 1, false, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
    return apart ? launch_pass<DT, D, 4, 2, false, COLSUM, CAN>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
           : few ? launch_pass<DT, D, 4, 2, false, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
               : launch_pass<DT, D, 4, 1, false, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
}

template <bool COLSUM>
hipError_t dispatch(const h2o_config &cfg, double scale, const void *Q, const void *K, const FrontRows &kf,
                    int nq, int nk, float *lse2, float *colsum, unsigned *zero, hipStream_t st)
{
    const int d = cfg.head_dim;
    switch (cfg.dtype) {
    case H2O_F32:
        return d == 64 ? pick_waves<H2O_F32, 64, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
                       : pick_waves<H2O_F32, 128, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
    case H2O_F16:
        return d == 64 ? pick_waves<H2O_F16, 64, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
                       : pick_waves<H2O_F16, 128, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
    default:
        return d == 64 ? pick_waves<H2O_BF16, 64, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st)
                       : pick_waves<H2O_BF16, 128, COLSUM>(cfg, scale, Q, K, kf, nq, nk, lse2, colsum, zero, st);
    }
}

}  // namespace

hipError_t h2o_launch_prefill_lse(const h2o_config &cfg, double scale, const void *Q,
                                  const void *K, const FrontRows &Kf, int nq, int nk, float *lse, hipStream_t st)
{
    return dispatch<false>(cfg, scale, Q, K, Kf, nq, nk, lse, nullptr, nullptr, st);
}

hipError_t h2o_launch_prefill_colsum(const h2o_config &cfg, double scale, const void *Q,
                                     const void *K, const FrontRows &Kf, int nq, int nk, const float *lse,
                                     float *colsum, hipStream_t st, unsigned *zero)
{
    return dispatch<true>(cfg, scale, Q, K, Kf, nq, nk, const_cast<float *>(lse), colsum, zero, st);
}
