// Prompt compression for H2O on gfx950: given one score per prompt token, keep
// the `recent` last tokens plus the `heavy` best-scoring older ones (or all n
// tokens when n fits in the budget) and copy their key/value rows into the
// cache slots in ascending position order (App. A: the prompt phase returns the
// heavy hitters and the recent tokens, or everything for a short prompt).
//
// Selecting the `heavy` largest under the order (score, then position) is the
// same as repeatedly evicting the smallest (score, position) pair, the rule the
// generation steps use.  An exact radix select on the order-preserving integer
// image of the scores finds the threshold, the positions of equal-score tokens
// break the tie at the threshold, ballots and a scan over the waves assign slots,
// then all threads copy rows with 128-bit accesses.
#include "wave_ops.h"

namespace {

constexpr int SG_BITS = 11;                 // radix digit: 11 + 11 + 10 bits
constexpr int SG_BINS = 1 << SG_BITS;
// where the ranking keys live during the selection
// the compression inside the cache: one workgroup per head, or several with some columns each
constexpr int IN_PLACE = 1, IN_PLACE_COLUMNS = 2;
constexpr int SG_KEYS_NONE = 0, SG_KEYS_LDS = 1;   // (any larger value: that many registers per thread)

__device__ inline unsigned order_key(float x)
{
    const unsigned u = __float_as_uint(x);
    return u ^ ((unsigned)((int)u >> 31) | 0x80000000u);   // monotone in x
}

// Inclusive prefix sum over the lanes of a wave: DPP moves (six shuffles through LDS, each
// waiting for the one before, took 800 cycles, twice per digit).
__device__ inline unsigned wave_inclusive_scan(unsigned v)
{
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);    // row_shr:1
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);    // row_shr:2
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);    // row_shr:4
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);    // row_shr:8
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

// The bin of a digit's histogram in which the count from the top reaches `need`, the count above that bin and its own.
// Every wave adds up its share of the bins (highest first), a barrier, then every wave finds the share and
// in it the bin: all counters are read once by the workgroup instead of once by each wave (1700 -> 900 cycles).
// `sums` holds NW words that nothing else uses.
struct BinAt { int bin; unsigned above, count; };
template <int NW> __device__ inline BinAt find_bin(const unsigned *hist, unsigned need, unsigned *sums)
{
    constexpr int SHARE = SG_BINS / NW, PER = SHARE / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    struct __align__(4 * PER) Bins { unsigned c[PER]; };          // ascending
    auto bins_of = [&](int w) {
        return *reinterpret_cast<const Bins *>(hist + SG_BINS - SHARE * w - PER * (lane + 1));
    };
    auto total = [](const Bins &b) {
        unsigned t = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) t += b.c[i];
        return t;
    };
    const unsigned share = wave_inclusive_scan(total(bins_of(wave)));
    if (lane == 63) sums[wave] = share;
    __syncthreads();
    unsigned mine = lane < NW ? sums[lane] : 0;
    unsigned upto = wave_inclusive_scan(mine);
    const int w = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(upto >= need)) - 1);
    unsigned above = __builtin_amdgcn_readlane((int)(upto - mine), w);
    const Bins b = bins_of(w);
    mine = total(b);
    upto = above + wave_inclusive_scan(mine);
    const int at = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(upto >= need)) - 1);
    above = __builtin_amdgcn_readlane((int)(upto - mine), at);
    int i = PER - 1;
    unsigned count = __builtin_amdgcn_readlane((int)b.c[PER - 1], at);
#pragma unroll
    for (int next = PER - 2; next >= 0; --next) {
        if (above + count < need) {                   // (all of it is wave-uniform)
            above += count;
            count = __builtin_amdgcn_readlane((int)b.c[next], at);
            i = next;
        }
    }
    return {SG_BINS - SHARE * w - PER * (at + 1) + i, above, count};
}

// Sum over the workgroup of one non-negative int per thread (every thread gets it).  `scratch`
// holds NW ints (waves of the workgroup).
template <int NW> __device__ inline int block_sum(int v, int *scratch)
{
    const unsigned w = wave_inclusive_scan((unsigned)v);
    __syncthreads();                       // scratch may still be read from a previous use
    if ((threadIdx.x & 63) == 63) scratch[threadIdx.x >> 6] = (int)w;
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) tot += scratch[i];
    return tot;
}

// Entry j of a head's n candidates is the token at position pos_in[j] (ascending;
// pos_in == nullptr: position j) with score base[j] + score[j] (base == nullptr:
// score[j]); t_new = number of tokens seen once these are stored.
// QDT < 0: the cache stores rows as they are (ROWB bytes each).  QDT = an element
// type: the cache stores 4-bit codes and the kept rows (ROWB bytes of QDT
// elements) are quantised on their way in.  PAT: built for a sparse-attention
// pattern as the protected set (the recent-window build carries none of that code).
//
// `parts` workgroups share a head: each makes the whole selection for itself and
// fills its own share of the slots (positions, scores, rows), so they need nothing
// from each other.  What bounds the kernel is the row copy; one workgroup per head
// left most of the chip idle at few heads, and a head's copy then runs at the rate
// of one CU.  The selection is a few microseconds of latency: a wave works on a
// contiguous run of entries, 64 at a time, so that reads are coalesced and ranks come
// from ballots; the ranking keys are formed once and kept in KEYS registers per
// thread (all reads in flight at once, no LDS latency in the sweeps), in LDS for
// longer prompts, and beyond SG_LDS_KEYS candidates formed again for every sweep.
// The selection is issue-bound (every workgroup makes all of it), hence the keys that carry
// their kind, a histogram that the workgroup reads once per digit, no digit behind one whose bin is kept
// whole (nearly always the third) and one compare per key for the count; what a wave does after the sweeps is
// latency, hence scans in registers, no slots for entries that other workgroups copy, and
// bookkeeping that is requested in front of the row copy and stored behind it.  Cycles of 32 heads,
// 3277 of 16 384: 29 000 for the selection with all three digits, every wave reading the whole histogram, two ballots
// per key and the scores fetched by every XCD (8600 until they had come), 20 100 now (5500 until the scores have come, 4900
// first sweep, 4400 second, 1100 to find each bin, 4500 count and slots), then 32 000 for the rows (110 MB, 8 TB/s of read + write).
// This kernel alone (three prompts in turn, so that rows come from HBM; us, before that / now): 32 heads, 3277 of 16 384
// tokens, f16 d = 128: 32.7 / 29.1; 306 of 1531 7.2 / 6.55; 128 heads, 819 of 4096 25.3 / 24.1; 512 heads, 410 of 2048 40.5 /
// 39.6; 12 heads, 1600 of 8000 11.9 / 10.1.
// (Tried: four counters per bin of the first digit, no gain, so the atomics' queue is not what
// that sweep waits for.)
//
// COMPACT: the cache itself is the front of the candidate list: entries j < n_occ are its
// slots (in position order, with their scores), the others the tokens Kp, Vp at positions
// t_new - m + (j - n_occ).  A workgroup then moves rows, or its columns of them, inside the cache: the
// entry kept in slot s is never in front of it (j >= s), so filling the slots in ascending
// rounds, every round's reads before its writes, never overwrites what is still to be read.
// (The list used to be copied together first, rows and all, and gathered back from there:
// 34 + 26 us per 1024-token chunk at 128 heads x 819 slots.)  Rounds overlap: the next one's reads are
// in flight while one is written (a whole call, us: 8 heads x 2048 tokens on 4000 slots 186 -> 172, 32 x 1024 on
// 819 77.1 -> 74.8, 256 x 512 on 410, d = 64, 84.3 -> 82.3).
template <int ROWB, int QDT, bool PAT, int KEYS, int COMPACT, int SG_NT>
__global__ __launch_bounds__(SG_NT, 4) void select_gather_kernel(
    const char *__restrict__ Kp, const char *__restrict__ Vp, const float *__restrict__ score,
    const float *__restrict__ base, const int32_t *__restrict__ pos_in, int n, int t_new,
    char *Kc, char *Vc, float *acc_g, int32_t *pos_g, int k, int heavy, int recent, int rank, int protect,
    int stride, int parts, int part_slots, int n_occ, unsigned *arrived)
{
    constexpr int SG_NW = SG_NT / 64;
    extern __shared__ __align__(16) unsigned char smem[];
    int *sel_l = reinterpret_cast<int *>(smem);        // [part_slots] slot -> candidate
    unsigned *key_l = reinterpret_cast<unsigned *>(sel_l + part_slots);   // [n] (SG_KEYS_LDS)
    __shared__ __align__(16) unsigned hist[3][SG_BINS];      // one per digit
    __shared__ int scan_l[2 * SG_NW];
    __shared__ unsigned sums_l[3][SG_NW];

    const int tid = threadIdx.x;
    // Consecutive workgroups go to the 8 XCDs in turn.  All workgroups of a head read all of its scores: on one XCD
    // (heads in eights) these come from memory once and from its L2 then, instead of once for each XCD.
    const bool eights = parts > 1 && gridDim.x % (8 * parts) == 0;
    const int turn = eights ? blockIdx.x >> 3 : blockIdx.x;
    const int head = eights ? turn / parts * 8 + (blockIdx.x & 7) : turn / parts;
    const int sb = COMPACT ? 0 : turn % parts * part_slots;     // this workgroup's slots [sb, se)
    const int se = min(k, sb + part_slots);
    const float *sc_in = score + (size_t)head * n;
    const float *bs = base ? base + (size_t)head * n : nullptr;
    const int32_t *pos_src = pos_in ? pos_in + (size_t)head * n : nullptr;
    const size_t hoff = (size_t)head * k;
    // the score of entry j as it will be stored, and its position
    auto sc_of = [&](int j) {
        if constexpr (COMPACT) return (j < n_occ ? acc_g[hoff + j] : 0.f) + sc_in[j];
        else return bs ? bs[j] + sc_in[j] : sc_in[j];
    };
    auto pos_of = [&](int j) {
        if constexpr (COMPACT) return j < n_occ ? pos_g[hoff + j] : t_new - (n - j);
        else return pos_src ? pos_src[j] : j;
    };

    // what ranks an older token: its score, or (averaged ranking) its score over
    // the n - j prompt queries that scored it
    auto ranked = [&](float v, int j) {
        return rank == H2O_RANK_AVERAGED ? __fdiv_rn(v, (float)(t_new - pos_of(j))) : v;
    };
    // this wave's run of entries
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int run = ((n + SG_NW - 1) / SG_NW + 63) & ~63;
    const int j0 = min(n, wave * run), j1 = min(n, j0 + run);
    constexpr bool IN_REGS = KEYS > SG_KEYS_LDS;
    unsigned key_r[IN_REGS ? KEYS : 1];
    // what an entry is (set once the candidates are known): see below
    struct { int older; bool overflow; } kinds = {0, false};
    auto kind_of = [&](int j, unsigned key) -> unsigned {
        if constexpr (PAT) {
            const bool cov = j < n && is_protected(pos_of(j), t_new - 1, recent, protect, stride);
            return cov == kinds.overflow ? key : cov ? ~0u : 0u;
        } else {
            return j < kinds.older ? key : ~0u;
        }
    };
    // f(entry, its key) for every entry of the wave's run, one per lane, ascending.  A key
    // also says what the entry is: KEY_OUT = none (past the run's end, or not to be kept),
    // KEY_SURE = kept outright, any other value = a candidate, so that the sweeps test
    // nothing but the key.
    constexpr unsigned KEY_OUT = 0u, KEY_SURE = ~0u;
    auto candidate_key = [&](float v, int j) {
        return min(max(order_key(ranked(v, j)), 1u), KEY_SURE - 1u);   // (the ends are NaNs)
    };
    auto sweep = [&](auto f) {
        if constexpr (IN_REGS) {
#pragma unroll
            for (int i = 0; i < KEYS; ++i) {
                if (j0 + i * 64 >= j1) break;          // wave-uniform
                f(j0 + i * 64 + lane, key_r[i]);
            }
        } else {
            for (int b = j0; b < j1; b += 64) {
                const int j = b + lane;
                unsigned key = KEY_OUT;
                if (j < j1) {
                    if constexpr (KEYS == SG_KEYS_LDS) key = key_l[j];
                    else key = kind_of(j, candidate_key(sc_of(j), j));
                }
                f(j, key);
            }
        }
    };

    for (int s = sb + tid; s < se; s += SG_NT) sel_l[s - sb] = n <= k && s < n ? s : -1;
    for (int b = tid; b < 3 * SG_BINS / 4; b += SG_NT)
        reinterpret_cast<uint4 *>(hist[0])[b] = make_uint4(0, 0, 0, 0);

    if (n > k) {
        // Which entries compete.  With the recent window (protect 0) the candidates are
        // the entries in front of the last `recent` positions; positions ascend, so they
        // are a prefix [0, older) and `heavy` of them are kept.  With a sparse-attention
        // pattern as the protected set, the entries the pattern covers for the last
        // query (position t_new - 1) are kept and the best of the others fill the budget;
        // should it cover more than the budget, the covered entries compete for all
        // k slots and the others are dropped (the rule "evict one at a time, protection
        // void once everything left is covered", in one shot).
        int older = n - recent;
        bool overflow = false;
        int want = heavy;                              // candidates to keep
        auto covered = [&](int j) { return is_protected(pos_of(j), t_new - 1, recent, protect, stride); };
        if constexpr (PAT) {
            int cnt = 0;
            for (int j = tid; j < n; j += SG_NT) cnt += covered(j);
            const int total = block_sum<SG_NW>(cnt, scan_l);
            overflow = total > k;
            want = overflow ? k : k - total;
        } else if (COMPACT ? recent > n - n_occ : pos_src != nullptr) {
            // (COMPACT with a window inside the chunk: the chunk's positions are consecutive)
            int cnt = 0;
            for (int j = tid; j < n; j += SG_NT) cnt += pos_of(j) < t_new - recent;
            older = block_sum<SG_NW>(cnt, scan_l);
        }
        kinds.older = older;
        kinds.overflow = overflow;
        if constexpr (IN_REGS) {
            // every score requested before the first is looked at
            float v[KEYS];
#pragma unroll
            for (int i = 0; i < KEYS; ++i) v[i] = sc_in[min(j0 + i * 64 + lane, n - 1)];
            if constexpr (COMPACT) {
#pragma unroll
                for (int i = 0; i < KEYS; ++i) {
                    const int j = min(j0 + i * 64 + lane, n - 1);
                    const float a = acc_g[hoff + min(j, max(n_occ, 1) - 1)];
                    v[i] = (j < n_occ ? a : 0.f) + v[i];
                }
            } else if (bs) {
#pragma unroll
                for (int i = 0; i < KEYS; ++i) v[i] = bs[min(j0 + i * 64 + lane, n - 1)] + v[i];
            }
            if (rank == H2O_RANK_AVERAGED) {
#pragma unroll
                for (int i = 0; i < KEYS; ++i) v[i] = ranked(v[i], min(j0 + i * 64 + lane, n - 1));
            }
#pragma unroll
            for (int i = 0; i < KEYS; ++i) {
                const int j = j0 + i * 64 + lane;
                key_r[i] = min(max(order_key(v[i]), 1u), KEY_SURE - 1u);
                if (PAT || j0 + i * 64 + 64 > min(older, j1)) {       // wave-uniform: not candidates throughout
                    const unsigned key = kind_of(j, key_r[i]);
                    key_r[i] = j < j1 ? key : KEY_OUT;
                }
            }
        } else if constexpr (KEYS == SG_KEYS_LDS) {
            // (written and read by the same wave)
#pragma unroll 8
            for (int j = j0 + lane; j < j1; j += 64) key_l[j] = kind_of(j, candidate_key(sc_of(j), j));
        }
        unsigned thr = KEY_SURE - 1u, need = 0;        // keep keys > thr, and `need` of those == thr
        bool whole = false;                            // ... or simply all keys >= thr
        if (want > 0) {
            // radix select: the want-th largest key among the candidates (there are more
            // than `want` of them: n exceeds the budget).  Three digits of 11, 11 and 10
            // bits: the first one (sign, exponent, two mantissa bits) already spreads
            // scores over dozens of bins, where 8 bits had put nearly all of them, and the
            // LDS atomics with them, into a handful.
            // A digit whose bin is kept whole is the last one: every key from its lowest on is kept.
            unsigned prefix = 0, mask = 0;
            need = (unsigned)want;
            __syncthreads();                           // the counters are zero (and keys in LDS written)
            sweep([&](int, unsigned key) {
                if (key - 1u < KEY_SURE - 1u) atomicAdd(&hist[0][key >> 21], 1u);
            });
#pragma unroll 1
            for (int d = 0; d < 3; ++d) {
                const int shift = d == 0 ? 21 : d == 1 ? 10 : 0;
                const unsigned dmask = d == 2 ? 1023u : 2047u;
                // (a key that agrees with the digits found so far is a candidate, unless those are
                // all zeros or all ones, which the two marks agree with as well)
                if (d > 0 && prefix != 0 && prefix != mask) {
                    const unsigned known = prefix >> (shift + (d == 1 ? 11 : 10));
                    sweep([&](int, unsigned key) {
                        if (key >> (shift + (d == 1 ? 11 : 10)) == known) atomicAdd(&hist[d][(key >> shift) & dmask], 1u);
                    });
                } else if (d > 0) {
                    sweep([&](int, unsigned key) {
                        if (((key ^ prefix) & mask) == 0 && key - 1u < KEY_SURE - 1u)
                            atomicAdd(&hist[d][(key >> shift) & dmask], 1u);
                    });
                }
                __syncthreads();
                const BinAt at = find_bin<SG_NW>(hist[d], need, sums_l[d]);
                need -= at.above;                      // still needed inside that bin
                prefix |= (unsigned)at.bin << shift;
                mask |= dmask << shift;
                whole = at.count == need;
                if (whole) break;
            }
            thr = whole ? max(prefix, 1u) : prefix;
        }
        // Ranks in position order.  A wave first counts, in its run, the entries that are kept
        // outright and those at the threshold, then (knowing how many of both the waves in
        // front have) it assigns slots.
        int sure_cnt = 0, eq_cnt = 0;
        if (whole) {
            unsigned kept = 0;
            sweep([&](int, unsigned key) { kept += key >= thr; });
            sure_cnt = __builtin_amdgcn_readlane((int)wave_inclusive_scan(kept), 63);
            need = 0;
        } else {
            sweep([&](int, unsigned key) {
                sure_cnt += __popcll(__ballot(key > thr));
                eq_cnt += __popcll(__ballot(key == thr));
            });
        }
        __syncthreads();
        if (lane == 0) { scan_l[wave] = sure_cnt; scan_l[SG_NW + wave] = eq_cnt; }
        __syncthreads();
        // (entries of the waves in front, by a scan over the waves in the lanes)
        auto in_front = [&](const int *counts, int &total) {
            const unsigned mine = lane < SG_NW ? (unsigned)counts[lane] : 0u, upto = wave_inclusive_scan(mine);
            total = __builtin_amdgcn_readlane((int)upto, SG_NW - 1);
            return __builtin_amdgcn_readlane((int)(upto - mine), wave);
        };
        int eq_total = 0, sure_total;
        int slot = in_front(scan_l, sure_total);
        const int e = whole ? 0 : in_front(scan_l + SG_NW, eq_total);
        // among equal scores the higher positions are kept: the last `need` of them
        const int eq_first = eq_total - (int)need;
        slot += max(0, e - eq_first);
        // Waves whose slots belong to other workgroups are done.
        const int mine_end = slot + sure_cnt + max(0, min(eq_cnt, e + eq_cnt - eq_first));
        if (slot < se && mine_end > sb) {
            if (eq_first == 0) {
                // every entry at the threshold is kept (nearly always: scores are distinct)
                sweep([&](int j, unsigned key) {
                    const bool keep = key >= thr;
                    const unsigned long long kept = __ballot(keep);
                    const int mine = (int)__builtin_amdgcn_mbcnt_hi(
                        (unsigned)(kept >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)kept, (unsigned)slot));
                    if (keep && mine >= sb && mine < se) sel_l[mine - sb] = j;
                    slot += __popcll(kept);
                });
            } else {
                const unsigned long long below = (1ull << lane) - 1ull;
                int eq = e;
                sweep([&](int j, unsigned key) {
                    const unsigned long long eqs = __ballot(key == thr);
                    bool keep = key > thr;
                    if (eqs) {                         // wave-uniform, rare
                        keep = keep || (key == thr && eq + __popcll(eqs & below) >= eq_first);
                        eq += __popcll(eqs);
                    }
                    const unsigned long long kept = __ballot(keep);
                    const int mine = slot + __popcll(kept & below);
                    if (keep && mine >= sb && mine < se) sel_l[mine - sb] = j;
                    slot += __popcll(kept);
                });
            }
        }
    }
    __syncthreads();

    if constexpr (COMPACT) {
        // In rounds of slots: reads (waited for), a barrier, writes.  No wave's write can then pass
        // another's read: round r writes slots that only rounds up to r read.  The next round's
        // reads lie behind what this round writes, so they are requested first and are in flight
        // while this round is written.
        constexpr int LPR = ROWB / 16, OWN = H2O_MAX_BUDGET / SG_NT;
        int p[OWN];
        float a[OWN];
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            if (i * SG_NT >= k) break;
            const int s = i * SG_NT + tid, j = s < k ? max(sel_l[s], 0) : 0;
            p[i] = pos_of(j);
            a[i] = sc_of(j);
        }
        auto bookkeeping_read = [&] {          // ... by every wave
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                if (i * SG_NT >= k) break;
                asm volatile("" ::"v"(p[i]), "v"(a[i]));
            }
            lds_barrier();
        };
        auto store_bookkeeping = [&] {
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                if (i * SG_NT >= k) break;
                const int s = i * SG_NT + tid;
                if (s < k) {
                    const bool any = sel_l[s] >= 0;
                    pos_g[hoff + s] = any ? p[i] : -1;
                    acc_g[hoff + s] = any ? a[i] : 0.f;
                }
            }
        };
        if constexpr (COMPACT == IN_PLACE_COLUMNS) {
            // Several workgroups share a head, each moves its own columns (pieces of 16 bytes) of the row that K and V
            // are together; a thread has one piece of every rpr-th slot.  All of them read the positions and
            // scores; the last to have read them stores the new ones.
            constexpr int UNR = 8;
            const int cols = 2 * LPR / parts, rpr = SG_NT / cols, round = UNR * rpr;     // (powers of two)
            const int piece = turn % parts * cols + (tid & (cols - 1)), rsub = tid >> (__ffs(cols) - 1);
            const bool value = piece >= LPR;
            const char *New = (value ? Vp : Kp) + (size_t)head * (n - n_occ) * ROWB + piece % LPR * 16;
            char *Row = (value ? Vc : Kc) + hoff * ROWB + piece % LPR * 16;
            struct Rows { int j[UNR]; uint4 x[UNR]; };
            auto request = [&](Rows &r, int s0) {
#pragma unroll
                for (int u = 0; u < UNR; ++u) {
                    const int s = s0 + u * rpr + rsub;
                    int j = s < k ? sel_l[s] : -1;
                    if (j == s && s < n_occ) j = -1;               // stays where it is
                    r.j[u] = j;
                    r.x[u] = *reinterpret_cast<const uint4 *>((j < n_occ ? Row : New) +
                                                              (size_t)(j < n_occ ? max(j, 0) : j - n_occ) * ROWB);
                }
            };
            auto write = [&](Rows &r, int s0) {
#pragma unroll
                for (int u = 0; u < UNR; ++u) pin(r.x[u]);         // (they have arrived)
                lds_barrier();
#pragma unroll
                for (int u = 0; u < UNR; ++u)
                    if (r.j[u] >= 0) *reinterpret_cast<uint4 *>(Row + (size_t)(s0 + u * rpr + rsub) * ROWB) = r.x[u];
            };
            __shared__ unsigned before;
            Rows even, odd;
            bookkeeping_read();
            if (tid == 0) before = atomicAdd(arrived + head, 1u);
            request(even, 0);
            // The first round in front of the loop: positions and scores are in registers no longer than to here (kept
            // through the loop they spilled 23 registers, waited for with the rows in flight).
            request(odd, round);                 // (past the end: row 0, not written)
            write(even, 0);
            if (before == (unsigned)parts - 1) store_bookkeeping();     // (behind write's barrier)
            for (int s0 = round; s0 < k; s0 += 2 * round) {
                request(even, s0 + round);
                write(odd, s0);
                request(odd, s0 + 2 * round);
                write(even, s0 + round);
            }
            return;
        }
        constexpr int RPR = SG_NT / LPR, UNR = 4, ROUND = UNR * RPR;
        const int li = tid % LPR, rsub = tid / LPR;
        const char *Kn = Kp + (size_t)head * (n - n_occ) * ROWB, *Vn = Vp + (size_t)head * (n - n_occ) * ROWB;
        char *Kh = Kc + hoff * ROWB, *Vh = Vc + hoff * ROWB;
        struct Rows { int j[UNR]; uint4 k[UNR], v[UNR]; };
        auto request = [&](Rows &r, int s0) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int s = s0 + u * RPR + rsub;
                int j = s < k ? sel_l[s] : -1;
                if (j == s && s < n_occ) j = -1;               // stays where it is
                const size_t off = (size_t)(j < n_occ ? max(j, 0) : j - n_occ) * ROWB + li * 16;
                r.j[u] = j;
                r.k[u] = *reinterpret_cast<const uint4 *>((j < n_occ ? Kh : Kn) + off);
                r.v[u] = *reinterpret_cast<const uint4 *>((j < n_occ ? Vh : Vn) + off);
            }
        };
        auto write = [&](Rows &r, int s0) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) { pin(r.k[u]); pin(r.v[u]); }      // (they have arrived)
            lds_barrier();
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int s = s0 + u * RPR + rsub;
                if (r.j[u] >= 0) {
                    *reinterpret_cast<uint4 *>(Kh + (size_t)s * ROWB + li * 16) = r.k[u];
                    *reinterpret_cast<uint4 *>(Vh + (size_t)s * ROWB + li * 16) = r.v[u];
                }
            }
        };
        Rows even, odd;
        request(even, 0);
        bookkeeping_read();
        store_bookkeeping();
        for (int s0 = 0; s0 < k; s0 += 2 * ROUND) {
            request(odd, s0 + ROUND);        // (past the end: row 0, not written)
            write(even, s0);
            request(even, s0 + 2 * ROUND);
            write(odd, s0 + ROUND);
        }
        return;
    }
    // bookkeeping of this workgroup's slots: requested here, stored behind the row copy (beyond the
    // first SG_NT slots: all of it there)
    const int own = sb + tid < se ? sel_l[tid] : -1;
    const int own_pos = pos_of(max(own, 0));
    const float own_score = sc_of(max(own, 0));
    auto store_bookkeeping = [&] {
        if (sb + tid < se) {
            pos_g[hoff + sb + tid] = own >= 0 ? own_pos : -1;
            acc_g[hoff + sb + tid] = own >= 0 ? own_score : 0.f;
        }
        for (int s = sb + tid + SG_NT; s < se; s += SG_NT) {
            const int j = sel_l[s - sb];
            pos_g[hoff + s] = j >= 0 ? pos_of(j) : -1;
            acc_g[hoff + s] = j >= 0 ? sc_of(j) : 0.f;
        }
    };
    if constexpr (QDT >= 0) {
        // quantising gather: D/8 lanes per row, 8 elements each; an aligned group of 8
        // lanes is one group of 64 elements
        using T = typename Elem<QDT>::T;
        constexpr int D = ROWB / (int)sizeof(T);
        constexpr int QL = D / 8;
        constexpr int CODEB = D / 2;
        constexpr unsigned QROWB = H2O_Q4_ROW_BYTES(D);
        constexpr int RPR = SG_NT / QL;              // rows per round
        const int l = tid % QL, rsub = tid / QL;
        const size_t pbase = (size_t)head * n * ROWB;
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        // every lane runs every round (the reductions inside the quantiser span lanes)
        for (int s0 = sb; s0 < se; s0 += RPR) {
            const int s = s0 + rsub;
            const int j = s < se ? sel_l[s - sb] : -1;
            const size_t off = pbase + (size_t)max(j, 0) * ROWB;
            float kx[8], vx[8];
            load8<QDT>(reinterpret_cast<const T *>(Kp + off) + l * 8, kx);
            load8<QDT>(reinterpret_cast<const T *>(Vp + off) + l * 8, vx);
            float ks, km, vs, vm;
            const unsigned kw = q4_quantise<8>(kx, ks, km);
            const unsigned vw = q4_quantise<8>(vx, vs, vm);
            if (j >= 0) {
                char *kr = Kc + (hoff + s) * QROWB, *vr = Vc + (hoff + s) * QROWB;
                *reinterpret_cast<unsigned *>(kr + l * 4) = kw;
                *reinterpret_cast<unsigned *>(vr + l * 4) = vw;
                if ((l & 7) == 0) {
                    *reinterpret_cast<f32x2 *>(kr + CODEB + (l / 8) * 8) = f32x2{ks, km};
                    *reinterpret_cast<f32x2 *>(vr + CODEB + (l / 8) * 8) = f32x2{vs, vm};
                }
            }
        }
        store_bookkeeping();
        return;
    }
    // gather rows: LPR lanes copy one row of ROWB bytes
    constexpr int LPR = ROWB / 16;
    constexpr int ROWS_PER_ROUND = SG_NT / LPR;
    const int li = tid % LPR, rsub = tid / LPR;
    const size_t pbase = (size_t)head * n * ROWB;
    // four rows per thread in flight (unconditional loads of a clamped row, so that
    // the requests of a batch leave back to back)
    constexpr int UNR = 4;
    for (int s0 = sb + rsub; s0 < se; s0 += UNR * ROWS_PER_ROUND) {
        int j[UNR];
        uint4 kv[UNR], vv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int s = s0 + u * ROWS_PER_ROUND;
            j[u] = s < se ? sel_l[s - sb] : -1;
            const size_t off = pbase + (size_t)max(j[u], 0) * ROWB + li * 16;
            kv[u] = *reinterpret_cast<const uint4 *>(Kp + off);
            vv[u] = *reinterpret_cast<const uint4 *>(Vp + off);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int s = s0 + u * ROWS_PER_ROUND;
            if (j[u] >= 0) {
                *reinterpret_cast<uint4 *>(Kc + (hoff + s) * ROWB + li * 16) = kv[u];
                *reinterpret_cast<uint4 *>(Vc + (hoff + s) * ROWB + li * 16) = vv[u];
            }
        }
    }
    store_bookkeeping();
}

// Marks every slot free (acc = 0, pos = -1).  Slot 0 of every head is what a step on an
// empty cache reads in place of the rows that do not exist yet (with weight zero): it
// must hold finite numbers, so its K and V rows (`pieces` 16-byte pieces each) are zeroed.
// One launch for both: two dependent launches of this size cost 4.5 us each.
__global__ __launch_bounds__(256) void mark_free_kernel(
    float *__restrict__ acc, int32_t *__restrict__ pos, size_t count, char *__restrict__ K,
    char *__restrict__ V, size_t row_pieces, int pieces, size_t head_bytes)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) { acc[i] = 0.f; pos[i] = -1; }
    if (i < row_pieces) {
        const size_t off = i / pieces * head_bytes + i % pieces * 16;
        *reinterpret_cast<uint4 *>(K + off) = make_uint4(0, 0, 0, 0);
        *reinterpret_cast<uint4 *>(V + off) = make_uint4(0, 0, 0, 0);
    }
}

}  // namespace

hipError_t h2o_launch_mark_free(const h2o_cache &c, hipStream_t st)
{
    const size_t heads = (size_t)c.cfg.batch * c.cfg.heads, count = heads * c.k;
    const int pieces = c.rowb / 16;                    // (stored rows are whole 16-byte pieces)
    const size_t row_pieces = heads * pieces, most = count > row_pieces ? count : row_pieces;
    hipLaunchKernelGGL(mark_free_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, st, c.acc, c.pos,
                       count, c.K, c.V, row_pieces, pieces, (size_t)c.k * c.rowb);
    return hipGetLastError();
}

namespace {

// Launches the compression of n candidates per head.  COMPACT: see the kernel (16-bit and
// binary32 storage only: a chunked prompt is refused on a 4-bit cache).
template <int COMPACT>
hipError_t launch_select(const h2o_cache &c, const void *K, const void *V, const float *score, const float *base,
                         const int32_t *pos_in, int n, int t_new, int n_occ, unsigned *arrived, hipStream_t st)
{
    const int heads = c.cfg.batch * c.cfg.heads;
    const int rowb = c.cfg.head_dim * c.esize;
    const char *Kp = static_cast<const char *>(K), *Vp = static_cast<const char *>(V);
    const SelectPlan plan = select_plan(heads, c.k, n, COMPACT);
    const int parts = COMPACT == IN_PLACE_COLUMNS ? compact_parts(heads, c.k, rowb) : plan.parts, part_slots = plan.part_slots;
    const bool window = c.cfg.protect == H2O_PROTECT_RECENT, wide = plan.wide;
    // Keys in registers: 8 per thread up to 4096 (sixteen waves: 8192) candidates, 32 (16) up to
    // 16 384 (window mode; the pattern modes, whose sweeps also test the pattern, keep them in LDS).
    const int keys = window && n <= (wide ? 8192 : 4096) ? 8
                     : window && n <= 16384              ? 32
                     : n <= SG_LDS_KEYS                  ? SG_KEYS_LDS
                                                         : SG_KEYS_NONE;
    const size_t smem = (size_t)part_slots * sizeof(int) + (keys == SG_KEYS_LDS && n > c.k ? (size_t)n * 4 : 0);
    auto launch = [&](auto kern, std::atomic<uint64_t> &raised) -> hipError_t {
        if (smem > 32 * 1024) {
            const hipError_t e =
                allow_lds(reinterpret_cast<const void *>(kern), (SG_LDS_KEYS + H2O_MAX_BUDGET) * 4, raised);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)heads * parts), dim3(wide ? 1024 : 512), smem, st, Kp, Vp, score, base,
                           pos_in, n, t_new, c.K, c.V, c.acc, c.pos, c.k, c.cfg.heavy, c.cfg.recent,
                           c.cfg.rank, c.cfg.protect, c.cfg.stride, parts, part_slots, n_occ, arrived);
        return hipGetLastError();
    };
    // (eight waves never see more than 16 384 candidates)
#define H2O_SG1(RB, QDT, PAT, KEYS, NT)                                                         \
    do {                                                                                        \
        static std::atomic<uint64_t> raised{0};                                                 \
        return launch(select_gather_kernel<RB, QDT, PAT, KEYS, COMPACT, NT>, raised);           \
    } while (0)
#define H2O_SG(RB, QDT)                                                                         \
    do {                                                                                        \
        if (!wide) {                                                                            \
            if (window && keys == 8) H2O_SG1(RB, QDT, false, 8, 512);                           \
            if (window) H2O_SG1(RB, QDT, false, 32, 512);                                       \
            H2O_SG1(RB, QDT, true, SG_KEYS_LDS, 512);                                           \
        }                                                                                       \
        if (window && keys == 8) H2O_SG1(RB, QDT, false, 8, 1024);                              \
        if (window && keys == 32) H2O_SG1(RB, QDT, false, 16, 1024);                            \
        if (window && keys == SG_KEYS_LDS) H2O_SG1(RB, QDT, false, SG_KEYS_LDS, 1024);          \
        if (window) H2O_SG1(RB, QDT, false, SG_KEYS_NONE, 1024);                                \
        if (keys == SG_KEYS_LDS) H2O_SG1(RB, QDT, true, SG_KEYS_LDS, 1024);                     \
        H2O_SG1(RB, QDT, true, SG_KEYS_NONE, 1024);                                             \
    } while (0)
    if constexpr (!COMPACT) {
        if (c.cfg.kv_bits == 4) {
            const int d = c.cfg.head_dim;
            switch (c.cfg.dtype) {
            case H2O_F32: if (d == 64) H2O_SG(256, H2O_F32); else H2O_SG(512, H2O_F32); break;
            case H2O_F16: if (d == 64) H2O_SG(128, H2O_F16); else H2O_SG(256, H2O_F16); break;
            default: if (d == 64) H2O_SG(128, H2O_BF16); else H2O_SG(256, H2O_BF16); break;
            }
        }
    }
    switch (rowb) {
    case 128: H2O_SG(128, -1); break;
    case 256: H2O_SG(256, -1); break;
    case 512: H2O_SG(512, -1); break;
    default: return hipErrorInvalidValue;
    }
#undef H2O_SG
#undef H2O_SG1
}

}  // namespace

hipError_t h2o_launch_select_gather(const h2o_cache &c, const void *K, const void *V,
                                    const float *score, const float *base, const int32_t *pos_in,
                                    int n, int t_new, hipStream_t st)
{
    return launch_select<0>(c, K, V, score, base, pos_in, n, t_new, 0, nullptr, st);
}

hipError_t h2o_launch_compact(const h2o_cache &c, const void *Kn, const void *Vn, const float *score, int m,
                              int n_occ, unsigned *arrived, hipStream_t st)
{
    return (arrived ? launch_select<IN_PLACE_COLUMNS> : launch_select<IN_PLACE>)(
        c, Kn, Vn, score, nullptr, nullptr, n_occ + m, c.t + m, n_occ, arrived, st);
}

// ---- cache + chunk -> one candidate list per head ---------------------------------
//
// Chunked prompt processing treats the n_occ cached tokens (slots in ascending
// position order) followed by the m tokens of the chunk as one sequence of
// ncat = n_occ + m candidates: their K/V rows, the scores they already have
// (zero for the chunk) and their positions are laid out contiguously per head.
// `order` (nullable): order[head][r] = the slot that holds the r-th cached token in
// position order; nullptr = the slots already are in that order.
template <int ROWB>
__global__ __launch_bounds__(256) void concat_kernel(
    const char *__restrict__ Kc, const char *__restrict__ Vc, const float *__restrict__ acc_g,
    const int32_t *__restrict__ pos_g, const int32_t *__restrict__ order, const char *__restrict__ Kn,
    const char *__restrict__ Vn, int k, int n_occ, int m, int t, int blocks_per_head,
    char *__restrict__ Kcat, char *__restrict__ Vcat, float *__restrict__ base,
    int32_t *__restrict__ pos_cat)
{
    constexpr int LPR = ROWB / 16;
    const int head = blockIdx.x / blocks_per_head, ncat = n_occ + m;
    const int row = (blockIdx.x % blocks_per_head) * (256 / LPR) + threadIdx.x / LPR, li = threadIdx.x % LPR;
    if (row >= ncat) return;
    const bool cached = row < n_occ;
    const int slot = cached ? (order ? order[(size_t)head * k + row] : row) : 0;
    const char *ks = cached ? Kc + ((size_t)head * k + slot) * ROWB : Kn + ((size_t)head * m + (row - n_occ)) * ROWB;
    const char *vs = cached ? Vc + ((size_t)head * k + slot) * ROWB : Vn + ((size_t)head * m + (row - n_occ)) * ROWB;
    const size_t o = ((size_t)head * ncat + row) * ROWB + li * 16;
    *reinterpret_cast<uint4 *>(Kcat + o) = *reinterpret_cast<const uint4 *>(ks + li * 16);
    *reinterpret_cast<uint4 *>(Vcat + o) = *reinterpret_cast<const uint4 *>(vs + li * 16);
    if (li == 0) {
        base[(size_t)head * ncat + row] = cached ? acc_g[(size_t)head * k + slot] : 0.f;
        pos_cat[(size_t)head * ncat + row] = cached ? pos_g[(size_t)head * k + slot] : t + (row - n_occ);
    }
}

// Generation steps overwrite evicted slots in place, so slot order stops following
// position order.  order[head][r] = slot of the r-th smallest position among the
// n_occ occupied slots (the first n_occ), by counting: positions are distinct.
__global__ __launch_bounds__(256) void order_slots_kernel(const int32_t *__restrict__ pos_g, int k,
                                                          int n_occ, int32_t *__restrict__ order)
{
    extern __shared__ int32_t pos_l[];
    const size_t hoff = (size_t)blockIdx.x * k;
    for (int s = threadIdx.x; s < n_occ; s += 256) pos_l[s] = pos_g[hoff + s];
    __syncthreads();
    for (int s = threadIdx.x; s < n_occ; s += 256) {
        const int p = pos_l[s];
        int rank = 0;
        for (int j = 0; j < n_occ; ++j) rank += pos_l[j] < p;
        order[hoff + rank] = s;
    }
}

// rolled[head][slot] = how many cached tokens have a smaller position (-1 for a free slot)
__global__ __launch_bounds__(256) void rolled_positions_kernel(const int32_t *__restrict__ pos_g, int k,
                                                               int n_occ, int32_t *__restrict__ rolled)
{
    extern __shared__ int32_t pos_l[];
    const size_t hoff = (size_t)blockIdx.x * k;
    for (int s = threadIdx.x; s < n_occ; s += 256) pos_l[s] = pos_g[hoff + s];
    __syncthreads();
    for (int s = threadIdx.x; s < k; s += 256) {
        int rank = -1;
        if (s < n_occ) {
            const int p = pos_l[s];
            rank = 0;
            for (int j = 0; j < n_occ; ++j) rank += pos_l[j] < p;
        }
        rolled[hoff + s] = rank;
    }
}

hipError_t h2o_launch_rolled_positions(const h2o_cache &c, int32_t *rolled, hipStream_t st)
{
    const int n_occ = c.t < c.k ? c.t : c.k;
    hipLaunchKernelGGL(rolled_positions_kernel, dim3(c.cfg.batch * c.cfg.heads), dim3(256),
                       (size_t)(n_occ > 0 ? n_occ : 1) * sizeof(int32_t), st, c.pos, c.k, n_occ, rolled);
    return hipGetLastError();
}

// flags[head] = bit mask of what is wrong with the head's bookkeeping (0 = consistent):
//   1  a slot below n_occ is free (the occupied slots are not the prefix [0, n_occ))
//   2  a slot from n_occ on is occupied
//   4  a position outside [0, t)
//   8  two slots hold the same position
//  16  a score that is negative (sign bit set), infinite or NaN
__global__ __launch_bounds__(256) void validate_kernel(const int32_t *__restrict__ pos_g,
                                                       const float *__restrict__ acc_g, int k, int n_occ,
                                                       int t, int32_t *__restrict__ flags)
{
    extern __shared__ int32_t pos_l[];
    __shared__ int bad;
    const size_t hoff = (size_t)blockIdx.x * k;
    if (threadIdx.x == 0) bad = 0;
    for (int s = threadIdx.x; s < k; s += 256) pos_l[s] = pos_g[hoff + s];
    __syncthreads();
    int mine = 0;
    for (int s = threadIdx.x; s < k; s += 256) {
        const int p = pos_l[s];
        if (s < n_occ) {
            if (p < 0) mine |= 1;
            else if (p >= t) mine |= 4;
            const unsigned a = __float_as_uint(acc_g[hoff + s]);
            if (a >= 0x7f800000u) mine |= 16;          // sign bit, infinity or NaN
            if (p >= 0)
                for (int j = 0; j < s; ++j) mine |= (pos_l[j] == p) ? 8 : 0;
        } else if (p != -1) {
            mine |= 2;
        }
    }
    if (mine) atomicOr(&bad, mine);                    // LDS atomic
    __syncthreads();
    if (threadIdx.x == 0) flags[blockIdx.x] = bad;
}

hipError_t h2o_launch_validate(const h2o_cache &c, int32_t *flags, hipStream_t st)
{
    const int n_occ = c.t < c.k ? c.t : c.k;
    hipLaunchKernelGGL(validate_kernel, dim3(c.cfg.batch * c.cfg.heads), dim3(256),
                       (size_t)c.k * sizeof(int32_t), st, c.pos, c.acc, c.k, n_occ, c.t, flags);
    return hipGetLastError();
}

hipError_t h2o_launch_concat(const h2o_cache &c, const void *Kn, const void *Vn, int m, int n_occ,
                             int32_t *order, void *Kcat, void *Vcat, float *base, int32_t *pos_cat,
                             hipStream_t st)
{
    const int heads = c.cfg.batch * c.cfg.heads;
    const int rowb = c.cfg.head_dim * c.esize;
    const int ncat = n_occ + m;
    if (order && n_occ > 0) {
        hipLaunchKernelGGL(order_slots_kernel, dim3(heads), dim3(256), (size_t)n_occ * sizeof(int32_t), st,
                           c.pos, c.k, n_occ, order);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // one-dimensional grid: heads x blocks per head (at most 2^24 x 4352 / 8 < 2^34 is refused below)
#define H2O_CC(RB)                                                                               \
    do {                                                                                         \
        const int bph = (ncat + 256 / (RB / 16) - 1) / (256 / (RB / 16));                        \
        if ((long long)heads * bph > 0x7fffffffLL) return hipErrorInvalidValue;                  \
        hipLaunchKernelGGL((concat_kernel<RB>), dim3((unsigned)(heads * bph)), dim3(256), 0, st, \
                           c.K, c.V, c.acc, c.pos, order, static_cast<const char *>(Kn),         \
                           static_cast<const char *>(Vn), c.k, n_occ, m, c.t, bph,               \
                           static_cast<char *>(Kcat), static_cast<char *>(Vcat), base, pos_cat); \
    } while (0)
    switch (rowb) {
    case 128: H2O_CC(128); break;
    case 256: H2O_CC(256); break;
    case 512: H2O_CC(512); break;
    default: return hipErrorInvalidValue;
    }
#undef H2O_CC
    return hipGetLastError();
}
