// Internal declarations shared by the translation units of the HIP library.
// Not part of the public ABI (see include/h2o.h for that).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include "h2o.h"

struct h2o_cache {
    h2o_config cfg;
    double scale;      // logit scale actually used (cfg.scale, or 1/sqrt(d) in double)
    int k;             // heavy + recent
    int esize;         // bytes per element of Q/K/V/q/k/v/out
    int rowb;          // bytes of one cached K (or V) row as stored
    int t;             // tokens seen so far
    bool sorted;       // occupied slots hold ascending positions (true until a step evicts)
    char *K;           // [B*Hh][k][d]
    char *V;           // [B*Hh][k][d]
    float *acc;        // [B*Hh][k]
    int32_t *pos;      // [B*Hh][k]
    size_t kv_bytes;   // bytes of the K (= V) region
    void *step_scratch;   // the caller's scratch for split steps, or nullptr (h2o_cache_set_step_scratch)
};

static inline int h2o_esize(int dtype) { return dtype == H2O_F32 ? 4 : 2; }
static inline int h2o_row_bytes(const h2o_config &c)
{
    return c.kv_bits == 4 ? H2O_Q4_ROW_BYTES(c.head_dim) : c.head_dim * h2o_esize(c.dtype);
}
static inline double h2o_scale_of(const h2o_config &c)
{
    return c.scale != 0.0f ? (double)c.scale : 1.0 / sqrt((double)c.head_dim);
}

// What a generation-step kernel gets.  One structure instead of sixteen arguments: the runtime
// spends about 80 ns of host time on every argument of a launch, and a small step is as long as
// its launch (a kernel with these fields as arguments 4.1 us per launch, as one structure 2.8).
struct StepArgs {
    char *K, *V;
    float *acc;
    int32_t *pos;
    const char *q, *kn, *vn;
    char *out;
    double scale;
    int k, n_occ, t, recent, rank, protect, stride;
};
static inline StepArgs step_args(const h2o_cache &c, const void *q, const void *kn, const void *vn, void *out)
{
    return {c.K, c.V, c.acc, c.pos, static_cast<const char *>(q), static_cast<const char *>(kn),
            static_cast<const char *>(vn), static_cast<char *>(out), c.scale, c.k, c.t < c.k ? c.t : c.k, c.t,
            c.cfg.recent, c.cfg.rank, c.cfg.protect, c.cfg.stride};
}

// ---- kernel launchers (each enqueues on `st` and returns hipGetLastError()) ----
hipError_t h2o_launch_mark_free(const h2o_cache &c, hipStream_t st);
hipError_t h2o_launch_decode(const h2o_cache &c, const void *q, const void *k_new,
                             const void *v_new, void *out, hipStream_t st);
// the same step with several workgroups per head (few heads, long budgets), on the
// cache's step scratch; h2o_split_scratch_bytes: 0 for a configuration it is not used for
size_t h2o_split_scratch_bytes(const h2o_config &c);
bool h2o_split_wanted(const h2o_cache &c);
hipError_t h2o_launch_decode_split(const h2o_cache &c, const void *q, const void *k_new,
                                   const void *v_new, void *out, hipStream_t st);
// the same step over a cache that stores 4-bit codes
hipError_t h2o_launch_decode_q4(const h2o_cache &c, const void *q, const void *k_new,
                                const void *v_new, void *out, hipStream_t st);
// Keys (or values) in front of the ones a caller passes: the first `rows` of a head's nk
// rows sit at front + head * stride * row bytes (the cache), the rest in the caller's
// array [heads][nk - rows].  {} = none.
struct FrontRows {
    const char *front = nullptr;
    int rows = 0, stride = 0;
};
// prompt scoring: the nq queries (rows of Q) are the last nq positions of the nk
// keys; lse [B*Hh][nq] = log2 of the row normalisers, colsum [B*Hh][nk]; zero (nullable): one word
// per head that the column sums' launch clears for the one behind it
hipError_t h2o_launch_prefill_lse(const h2o_config &cfg, double scale, const void *Q,
                                  const void *K, const FrontRows &Kf, int nq, int nk, float *lse, hipStream_t st);
hipError_t h2o_launch_prefill_colsum(const h2o_config &cfg, double scale, const void *Q,
                                     const void *K, const FrontRows &Kf, int nq, int nk, const float *lse,
                                     float *colsum, hipStream_t st, unsigned *zero = nullptr);
// causal attention of nq queries (the last nq of nk key positions) over nk keys: V
// ([nk][d] per head) is copied to `vcopy` (h2o_attn_vcopy_bytes(cfg, nk) bytes) first if
// `out` overlaps it,
// `lse2` receives log2 of every row's normaliser of exp2(scale*log2(e)*<q,k>),
// `lse_nat` (nullable) the natural-log row log-sum-exp; 16-bit element types only
size_t h2o_attn_vcopy_bytes(const h2o_config &cfg, int nk);
hipError_t h2o_launch_prefill_attention(const h2o_config &cfg, double scale, const void *Q,
                                        const void *K, const void *V, const FrontRows &Kf, const FrontRows &Vf,
                                        int nq, int nk, void *vcopy, float *lse2, float *lse_nat, void *out,
                                        hipStream_t st);
// compression of n candidates per head (entry j: position pos_in[j] or j, score
// base[j] + score[j] or score[j]) into the cache; t_new = tokens seen afterwards
hipError_t h2o_launch_select_gather(const h2o_cache &c, const void *K, const void *V,
                                    const float *score, const float *base, const int32_t *pos_in,
                                    int n, int t_new, hipStream_t st);
// compression in place: the n_occ cached tokens (slots in position order) followed by the
// m tokens Kn, Vn at positions t.. are the candidates, with column sums score[heads][n_occ + m];
// arrived: one word per head, zero
hipError_t h2o_launch_compact(const h2o_cache &c, const void *Kn, const void *Vn, const float *score,
                              int m, int n_occ, unsigned *arrived, hipStream_t st);
// the n_occ cached tokens in position order followed by the m chunk tokens as one
// candidate list; `order` (heads * k ints of scratch) is needed when the slots are
// not in position order, nullptr when they are
hipError_t h2o_launch_concat(const h2o_cache &c, const void *Kn, const void *Vn, int m, int n_occ,
                             int32_t *order, void *Kcat, void *Vcat, float *base, int32_t *pos_cat,
                             hipStream_t st);

// rolled[B*Hh][k]: rank of every occupied slot's token among the cached tokens by position
hipError_t h2o_launch_rolled_positions(const h2o_cache &c, int32_t *rolled, hipStream_t st);

// flags[B*Hh]: 0 for a head whose bookkeeping is consistent, else a bit mask (h2o.h)
hipError_t h2o_launch_validate(const h2o_cache &c, int32_t *flags, hipStream_t st);

// The prompt kernels hand out workgroups as (head, block) with a head on one XCD: 8 XCDs take
// head groups of 8 * hg heads, hg at most 8 and no larger than the heads need (a grid padded to
// whole groups of 64 heads made 8 heads wait behind seven times as many empty workgroups).
static __host__ __device__ inline int head_group(int heads) { return heads >= 64 ? 8 : (heads + 7) / 8; }
static inline long long head_slots(int heads)
{
    const int step = 8 * head_group(heads);
    return (long long)(heads + step - 1) / step * step;
}

// Whether two groups of four waves share a block of 128 rows and halve its streamed rows (one
// workgroup per CU then, instead of two or three): while blocks leave CUs idle, and the
// stream is long enough to be worth joining two parts.  Up to 256 blocks every one has a CU;
// beyond, the light blocks of a causal triangle fit in behind the heavy ones (not those of a
// chunk behind many cached tokens, which are all about equally heavy).  Both scoring passes / attention,
// f16, d = 128, us, one -> two groups:
//   to 256 blocks       8 heads x 1024 31 -> 26 / 25 -> 21, 8 x 4096 101 -> 80 / 83 -> 67
//   257 to 384          48 x 768 27 -> 23 / 22.6 -> 20.4, 40 x 900 32.3 -> 29.3 / 25.1 -> 23.9, 64 x 640 24.3 -> 22.9 /
//                       20.7 -> 20.6, 32 x 1531 47 -> 40 / 40 -> 34; past the line: 48 x 900 32.9 -> 33.8, 80 x 512
//                       24.5 -> 26.6 / 21.2 -> 23.3, 128 x 300 19 -> 23 / 16 -> 20; chunks: 192 heads x 256 tokens on
//                       410 cached 96.4 -> 101.5, 96 x 512 on 820 148.8 -> 153.1 (the whole call)
//   385 to 512          32 x 1800 58 -> 53 / 48 -> 44, 32 x 2048 63 -> 57 / 56 -> 50, 40 x 1531 50.4 -> 48.7 / 43 -> 41;
//                       past the line: 48 x 1280 42.9 -> 42.0 / 37.5 -> 37.1, 64 x 1024 37.6 -> 38.0
//   more                24 x 3000 92.8 -> 97.3, 32 x 3000 (768) 110 -> 123 / 95 -> 106
// binary32, d = 128 (four waves cost it more, see the scoring passes): 64 x 900 193 -> 164, 112 x 450 133 -> 107,
// 128 x 512 140 -> 106, 32 x 2048 412 -> 304, a chunk of 512 tokens on 410 cached
// ones, 96 heads, 286 -> 275 (the whole call); past the line: 160 x 384 (480) 102 -> 121, 80 x 1024 (640)
// 329 -> 310, 160 x 768 (960) 272 -> 307, heads of one block (192 x 256) 77 -> 72 with eight waves at 66.
static inline bool two_groups(int heads, int rows, int streamed, bool f32, int d)
{
    const long long blocks = (long long)heads * ((rows + 127) / 128);
    if (blocks <= 256) return streamed >= 480;
    if (f32) return rows > 256 && streamed > 384 && blocks <= 512;
    if (d == 128 && 2LL * streamed >= 3LL * rows) return false;             // (all blocks about equally heavy)
    return streamed >= (d == 128 ? 600 : 480) && blocks <= (streamed >= 1500 ? 512 : 384);
}

// Whether a binary32 scoring pass takes blocks of 64 rows, two groups of two waves each, instead of 128 rows: on
// grids that leave CUs idle the longest block then has half the work (a binary32 pass is its matrix
// instructions).  Reset, both passes and selection, us, 128 rows / 64: d = 64, 8 heads x 256 32.8 / 23.1, 8 x 1500 117 / 76, 56 x
// 512 (448 slots) 48.7 / 41.2, 128 x 256 (512) 33.9 / 31.9; d = 128, 8 x 256 52.4 / 33.0, 32 x 1000 (512) 147 / 101, 128 x 300 (640)
// 87.5 / 65.3.  At d = 64 no grid up to 512 slots loses (0.58 .. 0.99).  At d = 128 a workgroup has its CU to itself (97 KiB of
// LDS), and a block of 64 rows counts as half a round of the CUs (both passes alone, 64 rows / 128):
//   to 32 streamed rows the second group has nothing to do: 8 to 256 heads x 1 .. 32 1.09 .. 1.17, 512 1.29 .. 1.44
//   fewer rounds        264 to 320 heads x 100 and 128 0.83 .. 0.85, 136 to 192 x 129 .. 192 0.81 .. 0.96, one block per head to
//                       640 heads 0.73 .. 0.97; but 264 to 320 x 65 (a second block of one row) 1.05 .. 1.07
//   as many             blocks of a causal triangle are uneven, the light ones fill in: 128 heads x 129 .. 256 0.76 .. 0.91, 64 x
//                       512 0.71; one or two blocks per head are not: 136 to 192 x 65 .. 128 0.98 .. 1.25, 200 to 256 1.10 .. 1.46.
//                       Chunks behind cached tokens are the less so the more there are (the whole call, one pass on either side).
//                       Statistics, to 352 slots 0.85 .. 0.92, then by streamed / rows: 1.6 .. 2.4 0.92 .. 0.98, 3 0.97 .. 1.03, 3.7
//                       and more 1.05.  Column sums, by rows / streamed, at 280 to 320 slots 1.5 .. 2.7 0.83 .. 0.97, 2.9 and
//                       more 1.06, at 352 1.6 0.88, 2.3 .. 2.6 1.02, at 416 to 512 1.7 .. 2 1.06 .. 1.10, 8 and more 1.06 .. 1.12
// Beyond 512 and 640 slots nothing was measured.
static inline bool small_blocks(int heads, int rows, int streamed, int d)
{
    const long long slots = head_slots(heads) * ((rows + 63) / 64), slots128 = head_slots(heads) * ((rows + 127) / 128);
    if (d == 64) return slots <= 512;
    if (streamed <= 32 || slots > 640) return false;
    if (slots <= 256 || rows <= 64) return true;
    const long long rounds = (slots + 255) / 256, rounds128 = 2 * ((slots128 + 255) / 256);
    if (rounds < rounds128) return rows > 96;
    if (rounds > rounds128 || rows <= 128) return false;
    return streamed > rows ? slots <= 352 || 2LL * streamed < 5LL * rows : slots * rows < 820LL * streamed;
}

// Whether the attention's two groups (two_groups) run one phase apart: while one is in its MFMAs the
// other is in its softmax.  That takes a second barrier per tile and, at d = 64, 143 registers
// instead of 127, with which a second workgroup does not fit on the CU any more; blocks beyond the CUs then wait
// for a whole round where the groups in step would have run beside them.  What counts is the grid with its
// empty workgroups (slots: heads go to XCDs eight at a time, one head's blocks all to one XCD), for causal
// streams of some tiles up to two rounds of it.  Apart / together (time of the attention alone, 1 to 400
// heads; d = 128: both 16-bit types):
//   d = 128  to 256 slots from 1100 keys on 0.90 .. 0.98, below 0.95 .. 1.01; more slots from 1100 on 0.90 .. 1.01
//            (mean 0.97; 1 head x 65 536 0.91), below 1.00 .. 1.04
//   d = 64   to 256 slots 0.88 .. 1.02.  More, whole prompts: 33 heads x 860 tokens (231 blocks, 280 slots) 0.93, 36 x 800 0.99, 50 x
//            560 1.06; to 352 slots x 1100 to 1500 0.91 .. 0.97, 33 x 1150 (297 blocks) 0.95, 36 x 1100 (324) 1.02, 36 x 1200 1.03; from
//            1500 on to 512 slots 0.88 .. 0.98, from 4000 on to 576 0.89 .. 0.98; more slots 36 x 1650 (520) 1.11, 20 x
//            3000 (576) 1.04, 12 x 5000 (640) 1.04, 1 x 16 000 (1000) 1.17, 1 x 65 536 (4096) 1.23;
//            chunks behind many cached tokens (all blocks equally heavy): to 256 0.95 .. 1.01, more 0.99 .. 1.14
static inline bool groups_apart(int heads, int nq, int nk, int d)
{
    const long long row_blocks = (nq + 127) / 128, blocks = heads * row_blocks, slots = head_slots(heads) * row_blocks;
    if (slots <= 256) return true;
    if (d == 128) return nk >= 1100;
    if (2LL * nk >= 3LL * nq) return false;
    if (nk < 1100) return nk >= 800 && blocks <= 256;
    if (nk < 1500) return slots <= 352 || blocks <= 320;
    return slots <= (nk < 4000 ? 512 : 576);
}

// How a compression of n candidates per head into k slots is laid out: workgroups per head, slots
// of each, and whether they have sixteen waves instead of eight.
constexpr int SG_LDS_KEYS = 28672;     // ranking keys kept in LDS up to this many candidates (112 KiB)
struct SelectPlan { int parts, part_slots; bool wide; };
static inline SelectPlan select_plan(int heads, int k, int n, bool in_place)
{
    // Workgroups per head: enough to give every CU one, but at least 32 slots each (one round of
    // the row copy); in place one, which alone knows what it has read.
    int parts = in_place ? 1 : (256 + heads - 1) / heads;
    // Beyond SG_LDS_KEYS candidates every sweep reads the scores again.  Those that an XCD's workgroups read have to
    // stay in its 4 MB L2: an eighth of the heads where heads come in eights (all workgroups of a head on one
    // XCD), else parts / 8 of them, all from 8 parts on.  us, eights, halved by the other count / not: 32 heads,
    // 2048 of 40 000 68.5 / 66.3, 64 heads, 2048 of 30 000 77.3 / 66.2, 16 heads, 4000 of 60 000 92.9 / 87.5.  Not
    // in eights, parts halved / not (measured on such counts before eights were put on one XCD, eight waves): 32 heads, 2048 of 40 000
    // (2.6 / 5.1 MB) 123 / 180 (one workgroup per head 138), 64 heads 131 / 185, 64 heads, 200 of 28 673
    // (1.8 / 3.7 MB) 76 / 114; 16 heads, 2048 of 40 000 (2.6 MB as it is) 119 / 117.
    if (n > SG_LDS_KEYS)
        while (parts > 1 && (long long)heads * (heads % 8 == 0 ? 1 : parts < 8 ? parts : 8) * n * 4 > 8 * (3LL << 20))
            parts /= 2;
    // Every workgroup makes the whole selection.  Beyond 4096 candidates that is most of the time, and
    // rounding up, which puts a second one on some CUs, costs more than the CUs that rounding down leaves
    // idle.  f16, d = 128, us, reset included, up with eight waves / down with sixteen: 12 heads, 840 of 4200 14.2 /
    // 11.5, 1600 of 8000 17.4 / 13.2, 3276 of 16 384 23.8 / 19.4, 4000 of 20 000 73 / 31, 4096 of 60 000 152 / 87; 24 heads 15.6 / 12.8,
    // 19.1 / 16.5, 30.5 / 27.0, 82 / 39; 56 heads 18.6 / 17.0, 27.9 / 24.7, 57.7 / 47.1, 113 / 62; 112 heads 25.9 / 24.5, 49.6 /
    // 41.6, 102 / 86, 180 / 123; 192 heads 42.2 / 41.7, 74.8 / 70.9, 145 / 138, 234 / 178.  Up to 4096 the row copy weighs as
    // much, and two workgroups of eight waves on a CU copy faster than one (144 heads, 4-bit rows, 1500
    // of 2048, rounded up / down, eight waves: 80 / 90; 32 heads, 306 of 1531 10.1 with one per CU, 11.5 with two).
    if (n > 4096 && (long long)heads * parts > 256) parts = heads < 256 ? 256 / heads : 1;
    if (const int most = (k + 31) / 32; parts > most) parts = most;
    const int part_slots = (k + parts - 1) / parts;
    parts = (k + part_slots - 1) / part_slots;
    // Sixteen waves where the selection is long and a workgroup has its CU to itself: one for every CU, or
    // more than 64 KiB of keys in LDS.  Sixteen over eight waves at the same workgroups (time, 1 to 256
    // heads, 64 to 4096 slots): to 8192 candidates 0.87 .. 1.01 (d = 64, binary32 and averaged ranking too; 4-bit
    // rows 0.87 .. 1.07, mean 0.96; a pattern 0.80 .. 0.99), to 16 384 0.86 .. 1.01 (4-bit 0.86 .. 1.04; pattern 0.72 .. 0.95), to
    // 28 672 0.68 .. 0.94, beyond 0.56 .. 0.84; in place 0.5 to 12 us less per call.  257 to 1024 heads: to 8192 0.86 .. 1.09,
    // to 16 384 1.00 .. 1.36 (pattern 0.70 .. 0.93), to 28 672 0.66 .. 0.87, beyond 0.61 .. 0.86 (pattern 0.92 .. 1.04).  Up to
    // 4096: 128 heads, 819 of 4096 30.5 us against 31.3, 8 heads, 800 of 4096 11.3 / 11.9, in place 0.3 to 1.7 us more.
    const bool wide = n > 4096 && ((long long)heads * parts <= 256 || n > 16384);
    return {parts, part_slots, wide};
}

// Workgroups per head of the compression in place: each moves its own columns of the rows, 128 bytes of them (K and
// V taken as one row) and 64 KiB of K's and V's together at least.  A head's rows go through one CU otherwise.  Whole chunked calls, us,
// one workgroup / several: 32 heads x 819 slots of 256 bytes, chunks of 512, 370.6 / 349.0; 8 x 1000, 2048, 220.0 / 211.7;
// 8 x 600, 256, averaged 414.5 / 400.0; 128 x 819, 1024, 676 / 672.  Below 128 KiB of K the rows are a round or two either
// way: 56 x 300 158 / 161, 16 x 819 of 128 bytes 207.6 / 209.6.  (Every workgroup selects for itself; the scores that they all read
// again beyond SG_LDS_KEYS candidates do not show: 127 heads x 1000, 29 000 tokens 29.76 / 29.86 ms, 20 x 1000, 31 000, a pattern 6.21 / 6.19.)
static inline int compact_parts(int heads, int k, int rowb)
{
    int parts = 1;
    if ((size_t)k * rowb >= 131072)
        while (parts < 2 * rowb / 128 && heads * parts * 2 <= 256 && (size_t)k * rowb / parts >= 65536) parts *= 2;
    return parts;
}

// Rounds per chunk of the one-workgroup step beyond its registers: of umax, umax - 2, umax - 4
// and umax - 6 the one that wastes the fewest rounds on the last chunk (rounds past the
// occupied slots re-read the last row), the deepest of equals.
static inline int chunk_ring(int rounds, int umax)
{
    auto waste = [&](int u) { return (rounds + u - 1) / u * u - rounds; };
    int best = umax;
    for (int u = umax - 2; u >= umax - 6 && u >= 2; u -= 2)
        if (waste(u) < waste(best)) best = u;
    return best;
}

// Lets a kernel have up to `bytes` of dynamic LDS on the current device (the attribute belongs
// to a device's copy of the kernel); `done` remembers the devices, one per kernel.
static inline hipError_t allow_lds(const void *kern, int bytes, std::atomic<uint64_t> &done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

// ---- element types ----------------------------------------------------------
// Raw storage views: f32 -> float, f16 -> _Float16, bf16 -> uint16_t bit pattern.
template <int DT> struct Elem;
template <> struct Elem<H2O_F32> {
    using T = float;
    static constexpr int EPL = 4;   // elements per 16-byte lane load
    __device__ static inline float to_f(T v) { return v; }
    __device__ static inline T from_f(float v) { return v; }
};
template <> struct Elem<H2O_F16> {
    using T = _Float16;
    static constexpr int EPL = 8;
    __device__ static inline float to_f(T v) { return (float)v; }
    __device__ static inline T from_f(float v) { return (T)v; }   // round-to-nearest-even
};
template <> struct Elem<H2O_BF16> {
    using T = uint16_t;
    static constexpr int EPL = 8;
    __device__ static inline float to_f(T v) { return __uint_as_float(((uint32_t)v) << 16); }
    __device__ static inline T from_f(float v)
    {
        uint32_t u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) return (T)((u >> 16) | 0x40u);   // NaN stays NaN
        u += 0x7fffu + ((u >> 16) & 1u);                                      // nearest-even
        return (T)(u >> 16);
    }
};
