// ffs_lane.h -- lane-per-chromosome mapping of the decode and of the
// generation step, for populations large enough to fill the chip with it.
//
// The decode (the list-scheduling rule of include/ffs.h over the Section 3
// problem) runs one chromosome per lane.  A lane walks every stage itself,
// so the stage that runs is the same on all 64 lanes of a wave: the
// insertion network of a stage has exactly m_k entries (a branch on the
// wave-uniform m_k), and nothing moves between lanes.
//
// Slots.  Stage k dispatches its n jobs at slots off_k .. off_k + n - 1
// (off_k = m_0 + ... + m_{k-1}); the key it removes at a dispatch (the
// machine's previous job: completion, in the three-field format the dispatch
// index within the window, job) is written back to the slot it read, so the
// slot sequence of stage k's writes is its release order.  The first m_k of
// them are the machines' initial empty entries; after its last dispatch the
// stage writes its remaining entries, in order, to slots off_k + n .. off_k + n
// + m_k - 1.  Stage k + 1 therefore reads exactly its input order at slots
// off_{k+1} .. off_{k+1} + n - 1.
// Entries of one stage leave in (completion, dispatch order) order -- the
// first-in-first-out rule at the next stage -- because a newly dispatched
// job is inserted after every entry whose completion is not later than its
// own.
//
// Windows.  The slots are processed in windows of kLaneD held in registers:
// for each window, stage 0, 1, ..., S-1 in turn transform the window in
// place.  A stage's m_k sorted keys stay in LDS between windows.  Windows
// that lie inside a stage's dispatch range run unguarded; the first and
// last windows of a stage run with per-slot (wave-uniform) guards.
//
// The generation kernel of this mapping builds each wave's 64 children one
// after the other with the operators of ffs_kernels.h on all 64 lanes,
// writes them to the next generation's rows, decodes them one per lane from
// there, then writes back the parent's row of every cellular cell whose
// child is not strictly better.
#pragma once
#include <algorithm>
#include <type_traits>

#include "ffs_kernels.h"

namespace flowshop {

constexpr int kLaneD = 16;           // slots per window
constexpr int kLaneMaxMsum = 160;    // machine entries per lane (sum over stages) kept in LDS

// LDS of one wave of the lane generation kernel: the operators' row, later reused for the decode state (64 lanes x msum keys).
__host__ __device__ inline size_t lane_gen_wave_lds(int n_pad, int msum)
{
    const size_t ops = (size_t)wave_row(n_pad) * 2;
    const size_t st = (size_t)64 * msum * 4;
    return align16(ops > st ? ops : st);
}

// LDS of one wave of the lane decode of caller-supplied rows: the decode
// state, then the per-lane bit sets of the validity check (2^jb bits).
__host__ __device__ inline int lane_seen_words(int jb) { return jb <= 5 ? 1 : 1 << (jb - 5); }

__host__ __device__ inline size_t lane_eval_wave_lds(int jb, int msum)
{
    return (size_t)64 * (msum + lane_seen_words(jb)) * 4;
}

// How the lane decode of caller-supplied rows fills a CU: waves per workgroup
// (0: not even one fits), waves resident, and the time of a round of them.
struct LaneEval {
    int waves, resident;
    double round;
};

// Time of a SIMD's share of a round, in units that one wave alone takes 5 of.
inline double lane_round(int share) { return std::max(5.0, 3.0 * share); }

// The split with the most waves per unit of time (`table` bytes of LDS per
// workgroup, `wave` bytes per wave; at most sixteen waves per CU, the register
// limit).  A workgroup's waves are dealt to the four SIMDs from the first one
// on, so that several workgroups of three, five, six or seven leave the SIMDs
// unequal shares, and the fullest one's counts.  131072 rows of 500 x 10: two
// workgroups of five waves 430 us, of four 348; of 500 x 20 with 30 machines:
// two of six 834, two of four 546; a million rows of 20 x 10 with 41 machines:
// three of five 321, seven of two 249; 262144 rows of 20 x 20 with 80
// machines: one of seven 266, three of two 272.  Of equals the nearest to four:
// eight are up to 5 % slower for short rows, one up to 14 % for long ones,
// whose table every workgroup copies.
inline LaneEval lane_eval_split(size_t table, size_t wave, size_t max_lds)
{
    static const int order[] = {4, 2, 1, 8, 7, 6, 5, 3};
    LaneEval best{0, 0, 0.0};
    for (int w : order) {
        const size_t lds = table + w * wave;
        if (lds > max_lds) continue;
        const int groups = std::max(1, std::min((int)(max_lds / lds), 16 / w));
        const int share = (w & (w - 1)) ? groups * ((w + 3) / 4) : (groups * w + 3) / 4;
        const LaneEval e{w, groups * w, lane_round(share)};
        if (best.waves == 0 || e.resident * best.round > best.resident * e.round) best = e;
    }
    return best;
}

// Index field of the lane decode's keys (see KeyFormat): a stage's list takes
// the indices below kLaneFirst at the start of a window, the window's slot i
// the index kLaneFirst + i.
constexpr int kLaneFirst = 8;       // >= machines per stage
constexpr int kLaneIndexBits = 5;   // kLaneFirst + kLaneD <= 32
// kKeyIdx is the lane decode's format for up to 512 jobs whose completions fit
// beside nine job bits (18 bits: 262143); others take the checked one with
// the instance's own job bits.
constexpr int kLaneJB = 9;

// (x & m) | o in one VALU operation (opaque, so that the compiler does not
// take the and apart from the or where the masked value would serve too).
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t m, uint32_t o)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(m), "s"(o));
    return r;
}

// The LDS address n entries below p, which may lie before the LDS: formed as a
// number, mod 2^32, as the hardware adds what brings it back.
template <typename T>
__device__ __forceinline__ lds_ptr<T> lds_below(lds_ptr<T> p, uint32_t n)
{
    return (lds_ptr<T>)(uintptr_t)((uint32_t)(uintptr_t)p - n * (uint32_t)sizeof(T));
}

// sorted list key[0 .. M-1] without key[0] and with nk
template <int M>
__device__ __forceinline__ void lane_insert(uint32_t (&key)[M], uint32_t nk)
{
    if (M == 1) {
        key[0] = nk;
        return;
    }
    uint32_t nkey[M];
    nkey[0] = key[1 < M ? 1 : 0] < nk ? key[1 < M ? 1 : 0] : nk;
#pragma unroll
    for (int q = 1; q + 1 < M; ++q) nkey[q] = umed3(key[q], nk, key[q + 1]);
    nkey[M - 1] = key[M - 1] > nk ? key[M - 1] : nk;
#pragma unroll
    for (int q = 0; q < M; ++q) key[q] = nkey[q];
}

// One stage over one window.  r[i] holds slot lo + i: a key from the previous
// stage, or a gene at stage 0 (completion 0).  Key formats: see KeyFormat;
// kKeyTwo places a new key after every entry with the same completion by a
// threshold compare per entry.
// With GUARD, slot i dispatches only if bit i of `act` is set, and if bit i
// of `fl` is set it receives the list's first entry, which leaves the list
// (the flush after the last dispatch); job indices are clamped to n - 1 for
// the table read.
//
// The indexed unguarded step is M + 5 VALU operations: the slot's job with
// its index (which also addresses the table: the row's address less that
// index), start = max(machine free, job ready) -- the larger key has the
// larger (or equal) time in its high bits --, the new key from the start's
// time and that word, plus the shifted processing time, and M for the list.
// `over` collects the carries out of the completion field (kKeyIdxChecked).
//
// With two or three waves per SIMD a wave issues one instruction per four
// cycles, so scalar instructions cost what vector ones do: JB > 0 (at most
// 2^JB jobs, the job field that wide) makes the table addresses' index part
// an immediate offset instead of a scalar subtraction per slot.
template <int M, bool GUARD, int KEY, int JB, typename PT>
__device__ __forceinline__ void lane_stage(uint32_t (&r)[kLaneD], uint32_t (&key)[M], lds_ptr<PT> prow, uint32_t jb,
                                           uint32_t jmask, uint32_t act, uint32_t fl, uint32_t nmax, bool& over)
{
    const uint32_t sh = KEY == kKeyTwo ? jb : jb + kLaneIndexBits;
    const uint32_t himask = ~((1u << sh) - 1u);
    uint32_t low[kLaneD], pj[kLaneD];
    if (GUARD || KEY == kKeyTwo) {
#pragma unroll
        for (int i = 0; i < kLaneD; ++i) {
            const uint32_t j = r[i] & jmask;
            low[i] = GUARD ? (j < nmax ? j : nmax) : j;
        }
#pragma unroll
        for (int i = 0; i < kLaneD; ++i) pj[i] = (uint32_t)prow[low[i]];
    } else {
#pragma unroll
        for (int i = 0; i < kLaneD; ++i) low[i] = and_or(r[i], jmask, (uint32_t)(kLaneFirst + i) << jb);
        if (JB > 0) {
            // prow - index of slot i = (prow - the last slot's) + an offset
            const lds_ptr<PT> at = lds_below(prow, (uint32_t)(kLaneFirst + kLaneD - 1) << JB);
#pragma unroll
            for (int i = 0; i < kLaneD; ++i) pj[i] = (uint32_t)(at + low[i])[(kLaneD - 1 - i) << JB];
        } else {
#pragma unroll
            for (int i = 0; i < kLaneD; ++i) {
                const lds_ptr<PT> at = lds_below(prow, (uint32_t)(kLaneFirst + i) << jb);   // uniform
                pj[i] = (uint32_t)at[low[i]];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kLaneD; ++i) {
        if (!GUARD || ((act >> i) & 1u)) {
            const uint32_t o = key[0];
            const uint32_t mx = o > r[i] ? o : r[i];
            if (KEY != kKeyTwo) {
                const uint32_t y = (mx & himask) | (GUARD ? low[i] | ((uint32_t)(kLaneFirst + i) << jb) : low[i]);
                const uint32_t nk = (pj[i] << sh) + y;
                if (KEY == kKeyIdxChecked) over |= nk < y;
                lane_insert<M>(key, nk);
            } else {
                const uint32_t c = (mx >> jb) + pj[i];
                const uint32_t nk = (c << jb) | low[i];
                if (M == 1) {
                    key[0] = nk;
                } else {
                    // drop entry 0, insert nk after every entry with completion <= c
                    const uint32_t thr = (c + 1u) << jb;
                    uint32_t nkey[M];
                    bool prev = true;
#pragma unroll
                    for (int q = 0; q + 1 < M; ++q) {
                        const bool lt = key[q + 1] < thr;
                        nkey[q] = lt ? key[q + 1] : (prev ? nk : key[q]);
                        prev = lt;
                    }
                    nkey[M - 1] = prev ? nk : key[M - 1];
#pragma unroll
                    for (int q = 0; q < M; ++q) key[q] = nkey[q];
                }
            }
            r[i] = o;
        } else if (GUARD && ((fl >> i) & 1u)) {
            r[i] = key[0];
#pragma unroll
            for (int q = 0; q + 1 < M; ++q) key[q] = key[q + 1];
        }
    }
}

// Per-lane decode state in LDS.
typedef __attribute__((address_space(3))) uint32_t* lane_state;

// Stage k (m_k = M) over window [lo, lo + kLaneD): its dispatch slots are
// [d0, d0 + n), its flush slots [d0 + n, d0 + n + M) unless it is the last
// stage.  Keys live at st[q * 64] (q < M) between windows (during a flush
// that spans two windows, the entries not yet written, first at q = 0), and
// take their places' indices when a window begins.  Returns the makespan on
// the last window of the last stage, else 0.
template <int M, int KEY, int JB, typename PT>
__device__ __forceinline__ uint32_t lane_stage_window(uint32_t (&r)[kLaneD], lane_state st, lds_ptr<PT> prow, int lo,
                                                      int d0, int n, bool last, bool full, uint32_t jb,
                                                      uint32_t jmask, bool& over)
{
    const uint32_t field = ((1u << kLaneIndexBits) - 1u) << jb;
    uint32_t key[M];
    if (full) {   // every stage dispatches in every slot, and none ends
#pragma unroll
        for (int q = 0; q < M; ++q) {
            key[q] = st[q * 64];
            if (KEY != kKeyTwo && M > 1) key[q] = (key[q] & ~field) | ((uint32_t)q << jb);
        }
        lane_stage<M, false, KEY, JB, PT>(r, key, prow, jb, jmask, 0u, 0u, 0u, over);
#pragma unroll
        for (int q = 0; q < M; ++q) st[q * 64] = key[q];
        return 0u;
    }
    const int d1 = d0 + n, end = last ? d1 : d1 + M;
    if (d0 >= lo) {
#pragma unroll
        for (int q = 0; q < M; ++q) key[q] = 0u;
    } else {
#pragma unroll
        for (int q = 0; q < M; ++q) {
            key[q] = st[q * 64];
            if (KEY != kKeyTwo && M > 1) key[q] = (key[q] & ~field) | ((uint32_t)q << jb);
        }
    }
    if (d0 <= lo && lo + kLaneD <= d1) {
        lane_stage<M, false, KEY, JB, PT>(r, key, prow, jb, jmask, 0u, 0u, 0u, over);
    } else {
        const int a0 = d0 > lo ? d0 - lo : 0, a1 = (d1 < lo + kLaneD ? d1 : lo + kLaneD) - lo;
        const uint32_t act = (a1 > a0) ? ((0xFFFFFFFFu >> (32 - (a1 - a0))) << a0) : 0u;
        uint32_t fl = 0u;
        if (!last) {
            const int f0 = (d1 > lo ? d1 : lo) - lo, f1 = (end < lo + kLaneD ? end : lo + kLaneD) - lo;
            fl = (f1 > f0) ? ((0xFFFFFFFFu >> (32 - (f1 - f0))) << f0) : 0u;
        }
        lane_stage<M, true, KEY, JB, PT>(r, key, prow, jb, jmask, act, fl, (uint32_t)(n - 1), over);
    }
    if (end <= lo + kLaneD) return last ? (key[M - 1] >> (KEY == kKeyTwo ? jb : jb + kLaneIndexBits)) : 0u;
#pragma unroll
    for (int q = 0; q < M; ++q) st[q * 64] = key[q];
    return 0u;
}

// Genes of slots [lo, lo + kLaneD) of a row (positions past the row's end
// read the row's padding; the guards never dispatch them).
struct GenesU16 {
    const uint16_t* row;   // n_pad entries, 64-byte aligned
    __device__ __forceinline__ void load(int lo, uint32_t (&g)[kLaneD]) const
    {
        const auto* v = as_global(reinterpret_cast<const u32x4*>(row + lo));
        const u32x4 a = v[0], b = v[1];
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            g[2 * i] = w[i] & 0xFFFFu;
            g[2 * i + 1] = w[i] >> 16;
        }
    }
    __device__ __forceinline__ void mark(int, const uint32_t (&)[kLaneD]) {}
};

// Caller-supplied int32 rows of exactly n entries, read as 16-byte vectors of
// a window.  mark() sets the bits of a window's genes in the lane's bit set
// (word q at seen[q * 64]) and collects all bits of the values: a row is a
// permutation if no value has a bit from jb on and exactly the bits below n
// are set.  Values beyond 2^jb cannot leave the table: every look-up masks.
struct GenesI32 {
    const int* row;
    int n, jb;
    lane_state seen;
    uint32_t bits;
    __device__ __forceinline__ void load(int lo, uint32_t (&g)[kLaneD]) const
    {
        if (lo + kLaneD <= n) {
            const row_vec_ptr v = (row_vec_ptr)(row + lo);
#pragma unroll
            for (int q = 0; q < kLaneD / 4; ++q) {
                const row_vec x = v[q];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[4 * q + e] = (uint32_t)x[e];
            }
        } else {
            const auto* p = as_global(row);
#pragma unroll
            for (int i = 0; i < kLaneD; ++i) g[i] = (uint32_t)p[lo + i < n ? lo + i : n - 1];
        }
    }
    __device__ __forceinline__ void mark(int lo, const uint32_t (&g)[kLaneD])
    {
        if (lo >= n) return;
        const int wbits = jb > 5 ? jb - 5 : 0;
#pragma unroll
        for (int i = 0; i < kLaneD; ++i) {
            bits |= g[i];
            // (past the row's end: its last value again)
            const uint32_t q = __builtin_amdgcn_ubfe(g[i], 5, wbits);
            __hip_atomic_fetch_or(seen + q * 64, 1u << (g[i] & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
};

// Makespan of one chromosome per lane with one key format.  pT is the LDS
// table (row stride pts), mach the stage machine counts, st this lane's LDS
// state (msum keys per lane, lane-interleaved).
template <int MMAX, int KEY, int JB, typename PT, typename Src>
__device__ __forceinline__ uint32_t lane_decode_keys(Src& src, lds_ptr<PT> pT, int pts, const int* mach, int S,
                                                     int n, int jb, lane_state st, bool& over)
{
    // the job field is JB wide, its mask the instance's own width: whatever a
    // row holds, a look-up stays below 2^jb
    const uint32_t ujb = (uint32_t)(JB > 0 ? JB : jb), jmask = (1u << jb) - 1u;
    int off_last = 0;
    for (int k = 0; k + 1 < S; ++k) off_last += mach[k];
    const int nwin = (off_last + n + kLaneD - 1) / kLaneD;
    // a full window ends no stage: of one stage alone the last window, whose
    // list gives the makespan, may hold nothing but dispatches
    const int nfull = off_last > 0 ? n : n - 1;
    uint32_t cmax = 0u;
    uint32_t gnext[kLaneD];
    src.load(0, gnext);
    for (int w = 0; w < nwin; ++w) {
        const int lo = w * kLaneD;
        uint32_t r[kLaneD];
#pragma unroll
        for (int i = 0; i < kLaneD; ++i) r[i] = gnext[i];
        if (lo + kLaneD < n) src.load(lo + kLaneD, gnext);
        src.mark(lo, r);
        const bool full = lo > off_last && lo + kLaneD <= nfull;
        int off = 0;
        for (int k = 0; k < S; ++k) {
            const int M = mach[k];
            const bool last = (k == S - 1);
            if (!full && off >= lo + kLaneD) break;   // this and later stages start after the window
            if (full || off + n + (last ? 0 : M) > lo) {
                const lds_ptr<PT> prow = pT + k * pts;
                const lane_state sk = st + off * 64;
                uint32_t cm = 0u;
                switch (M) {
#define FFS_LANE_CASE(MM)                                                                       \
    case MM:                                                                                    \
        if (MM <= MMAX)                                                                         \
            cm = lane_stage_window<(MM <= MMAX ? MM : 1), KEY, JB, PT>(r, sk, prow, lo, off, n, last, full, ujb,     \
                                                                       jmask, over);                            \
        break;
                    FFS_LANE_CASE(1) FFS_LANE_CASE(2) FFS_LANE_CASE(3) FFS_LANE_CASE(4)
                    FFS_LANE_CASE(5) FFS_LANE_CASE(6) FFS_LANE_CASE(7) FFS_LANE_CASE(8)
#undef FFS_LANE_CASE
                    default: break;
                }
                cmax = last ? (cm > cmax ? cm : cmax) : cmax;
            }
            off += M;
        }
    }
    return cmax;
}

// The two-field decode as a function of its own, so that its code stays out
// of the kernels' main path.
template <typename Src>
struct LaneResult {
    uint32_t cm;
    Src src;
};

template <int MMAX, typename PT, typename Src>
__device__ __attribute__((noinline)) LaneResult<Src> lane_decode_two(Src src, lds_ptr<PT> pT, int pts, const int* mach,
                                                                     int S, int n, int jb, lane_state st)
{
    bool over = false;
    const uint32_t cm = lane_decode_keys<MMAX, kKeyTwo, 0, PT>(src, pT, pts, mach, S, n, jb, st, over);
    return LaneResult<Src>{cm, src};
}

// Makespan of one chromosome per lane with the instance's key format; wst is
// the wave's LDS state.  If completions outgrow the checked format on any
// lane, the wave decodes again with the two-field key and those lanes take
// that result.
template <int MMAX, typename PT, typename Src>
__device__ __forceinline__ uint32_t lane_decode(Src& src, const PT* table, int pts, const InstDesc* I, uint32_t* wst,
                                                int lane)
{
    const int *mach = I->mach, S = I->S, n = I->n, jb = I->jb, fmt = I->lkey;
    const lds_ptr<PT> pT = as_lds(table);
    const lane_state st = (lane_state)wst + lane;
    bool over = false;
    if (fmt == kKeyIdx) return lane_decode_keys<MMAX, kKeyIdx, kLaneJB, PT>(src, pT, pts, mach, S, n, jb, st, over);
    uint32_t cm = 0u;
    if (fmt == kKeyIdxChecked) {
        cm = lane_decode_keys<MMAX, kKeyIdxChecked, 0, PT>(src, pT, pts, mach, S, n, jb, st, over);
        if (__ballot(over) == 0ull) return cm;
    }
    const LaneResult<Src> two = lane_decode_two<MMAX, PT>(src, pT, pts, mach, S, n, jb, st);
    src = two.src;
    return fmt == kKeyTwo || over ? two.cm : cm;
}

// ---- one generation (mode 0) or generation 0 (mode 1), lane mapping --------
// Work item = up to 64 * waves chromosomes of one island; wave w takes 64 of
// them.  Same generation bookkeeping, best-ever workgroup and XCD placement
// as k_generation.  Mode 0 leaves line-sweep islands alone; mode 2 runs the
// cells of anti-diagonal `cnt_off` of line-sweep island work[blockIdx.y]
// for the generation the last mode-0 launch counted (one launch per
// anti-diagonal, in order, after that launch).
template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) k_generation_lane(const InstDesc* __restrict__ insts,
                                                         const IslandDesc* __restrict__ isls,
                                                         const WorkItem* __restrict__ work, Control* ctl, int n_inst,
                                                         int mode, int cnt_off, int has_extra)
{
    __shared__ int s_gen;
    const bool sweep = mode == 2;
    if (threadIdx.x == 0) {
        int gg = 0;
        if (mode == 0) {
            int* cnt = ctl->counts + cnt_off + blockIdx.x;
            const int t = *cnt;
            *cnt = t + 1;
            gg = ctl->base + 1 + t;
        } else if (sweep) {
            gg = completed_gen(ctl);
        }
        s_gen = gg;
    }
    // has_extra = 1 + group: the last workgroup folds that fold group's
    // previous generation
    if (has_extra && blockIdx.x == gridDim.x - 1) {
        __syncthreads();
        const int prev = s_gen - 1, group = has_extra - 1;
        if (ctl->best_gen[group] < prev)
            fold_best(insts, isls, n_inst, prev, ctl, reinterpret_cast<int*>(ffs_smem), group);
        return;
    }
    const int nw = (int)gridDim.x - (has_extra ? 1 : 0);
    int widx = sweep ? (int)blockIdx.y : (int)blockIdx.x;
    if (!sweep && nw <= 256) {
        const int per = (nw + 7) / 8, full = nw - 8 * (per - 1);
        const int xcd = widx & 7, rnk = widx >> 3;
        widx = (xcd < full) ? xcd * per + rnk : full * per + (xcd - full) * (per - 1) + rnk;
    }
    const WorkItem wi = work[widx];
    const InstDesc* I = insts + wi.inst;
    const IslandDesc* L = isls + wi.island;
    if (mode == 0 && L->sweep) return;   // line-sweep islands have launches of their own
    // line sweep: the cells of anti-diagonal diag, rows rlo .. rlo + dcount - 1
    const int diag = sweep ? cnt_off : -1;
    int rlo = 0, dcount = 0;
    if (sweep) {
        rlo = diag - (L->cols - 1) > 0 ? diag - (L->cols - 1) : 0;
        const int rhi = diag < L->rows - 1 ? diag : L->rows - 1;
        dcount = rhi - rlo + 1;
        if (dcount <= 0) return;
    }
    const int n = I->n, S = I->S, n_pad = I->n_pad;

    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int gen = s_gen;
    const int cur = (gen + 1) & 1, nxt = gen & 1;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    unsigned char* wbase = ffs_smem + pt_lds_bytes<PT>(S, n_pad) + (size_t)wave * I->lane_wlds;
    // chromosome i of this wave sits in slot slot_of(sbase + i)
    const int w0 = wave * kWave + (sweep ? (int)blockIdx.x * (int)blockDim.x : 0);
    const int total = sweep ? dcount : wi.count;
    const int wcount = total - w0 < 0 ? 0 : (total - w0 > kWave ? kWave : total - w0);
    const int sbase = sweep ? w0 : wi.slot0 + w0;
    const int lcols = L->cols;
    auto slot_of = [&](int i) { return sweep ? (rlo + i) * lcols + (diag - rlo - i) : i; };

    // children, one at a time on all 64 lanes, into the next generation's
    // rows.  Lane c first takes the parents and draws of child c (one Philox
    // block per cell, two per pair); while a child is built, the parents'
    // rows of the next one are already on their way into registers.
    {
        uint16_t* A = reinterpret_cast<uint16_t*>(wbase);
        // the row's padding is zero (readers of a row look up its genes unmasked)
        for (int t = n + lane; t < n_pad; t += kWave) A[t] = 0;
        if (mode == 1) {
            for (int c = 0; c < wcount; ++c) {
                const int slot = slot_of(sbase + c);
                initial_row(I, L, slot, A, L->genes[cur] + (size_t)slot * n_pad, lane, kWave, true);
                row_l2g(L->genes[nxt] + (size_t)slot * n_pad, A, n_pad, lane, kWave);
                wave_sync();
            }
        } else if (wcount > 0) {
            const bool cell = L->kind == 0;
            const int pslot = slot_of(sbase + (lane < wcount ? lane : 0));
            uint32_t w_src, w_cut, w_mut;
            if (cell) {
                // slots < 2^14; bits 15 and 31: that parent's row is the new generation's
                const CellPlan pl = cell_plan(I, L, pslot, 0u, gen, cur, diag);
                w_src = (uint32_t)pl.p1 | ((uint32_t)pl.p2 << 16) | (pl.n1 ? 1u << 15 : 0u) | (pl.n2 ? 1u << 31 : 0u);
                w_cut = (uint32_t)pl.meta.a | ((uint32_t)pl.meta.b << 12) | (pl.meta.cx ? 1u << 24 : 0u) |
                        (pl.meta.mx ? 1u << 25 : 0u);
                w_mut = (uint32_t)pl.meta.mi | ((uint32_t)pl.meta.mj << 12);
            } else {
                // both parents are X's row; bit 15: the odd slot of the pair
                const PairPlan pl = pair_plan(I, L, pslot, gen, cur);
                w_src = (uint32_t)pl.xs | ((uint32_t)pl.xs << 16) | (pl.odd ? 1u << 15 : 0u);
                w_cut = (uint32_t)pl.a | ((uint32_t)pl.b << 12) | (pl.cx ? 1u << 24 : 0u) | (pl.mx ? 1u << 25 : 0u);
                w_mut = (uint32_t)pl.mi | ((uint32_t)pl.mj << 12);
            }
            auto parent1 = [&](uint32_t src) {
                return L->genes[cell && (src & 0x8000u) ? nxt : cur] + (size_t)(src & 0x7FFFu) * n_pad;
            };
            auto parent2 = [&](uint32_t src) {
                return L->genes[cell && (src >> 31) ? nxt : cur] + (size_t)((src >> 16) & 0x7FFFu) * n_pad;
            };
            auto cut_of = [&](uint32_t src, uint32_t cut) {
                const bool odd = !cell && (src & 0x8000u);
                return ox_cut(n, ((cut >> 24) & 1u) != 0u, (int)(cut & 0xFFFu), (int)((cut >> 12) & 0xFFFu), odd,
                              !cell && !odd);
            };
            auto finish = [&](int c) {
                const uint32_t cut = (uint32_t)__builtin_amdgcn_readlane((int)w_cut, c);
                const uint32_t mut = (uint32_t)__builtin_amdgcn_readlane((int)w_mut, c);
                swap_genes(A, ((cut >> 25) & 1u) != 0u && lane == 0, (int)(mut & 0xFFFu), (int)(mut >> 12));
                row_l2g(L->genes[nxt] + (size_t)slot_of(sbase + c) * n_pad, A, n_pad, lane, kWave);
                wave_sync();
            };
            // Building a child is a chain of LDS round trips, the decode is bound
            // by vector issue: the waves that build go first on their SIMD, so
            // that their round trips pass under the others' decodes (a large
            // generation 660 -> 586 us; the decode first instead: no gain).
            __builtin_amdgcn_s_setprio(3);
            auto build = [&](auto cc) {
                constexpr int C = decltype(cc)::value;   // genes per lane
                LaneGenes<C> ra, rb;
                auto fetch = [&](int c) {
                    const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)w_src, c);
                    lane_genes_load<C>(ra, parent1(src), lane, n_pad);
                    if (cell) lane_genes_load<C>(rb, parent2(src), lane, n_pad);
                };
                fetch(0);
                for (int c = 0; c < wcount; ++c) {
                    const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)w_src, c);
                    const uint32_t cut = (uint32_t)__builtin_amdgcn_readlane((int)w_cut, c);
                    const LaneGenes<C> x1 = ra;
                    LaneGenes<C> x2 = ra;
                    if (cell) x2 = rb;
                    if (c + 1 < wcount) fetch(c + 1);
                    ox_wave<C>(A, x1, x2, cut_of(src, cut), lane);
                    finish(c);
                }
            };
            // up to 1024 jobs the next child's parents are read while this one
            // is built; longer rows are read when they are needed
            if (n <= 64) {
                build(std::integral_constant<int, 1>{});
            } else if (n <= 128) {
                build(std::integral_constant<int, 2>{});
            } else if (n <= 256) {
                build(std::integral_constant<int, 4>{});
            } else if (n <= 512) {
                build(std::integral_constant<int, 8>{});
            } else if (n <= 1024) {
                build(std::integral_constant<int, 16>{});
            } else {
                for (int c = 0; c < wcount; ++c) {
                    const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)w_src, c);
                    const uint32_t cut = (uint32_t)__builtin_amdgcn_readlane((int)w_cut, c);
                    ox_wave_long(A, n_pad, parent1(src), parent2(src), cut_of(src, cut), lane);
                    finish(c);
                }
            }
        }
    }
    // the rows just written are read back by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    const bool active = lane < wcount;
    const int slot = slot_of(sbase + (active ? lane : 0));
    unsigned long long wkey = ~0ull;
    if (wcount > 0) {
        GenesU16 src{L->genes[nxt] + (size_t)slot * n_pad};
        __builtin_amdgcn_s_setprio(0);
        const uint32_t cm = lane_decode<MMAX, PT>(src, pT, pt_stride<PT>(n_pad), I, reinterpret_cast<uint32_t*>(wbase),
                                                  lane);
        bool keep_old = false;
        if (active) {
            int mk_new = (int)cm;
            if (mode != 1 && L->kind == 0) {
                const int mk_old = as_global(L->mk[cur])[slot];
                keep_old = !((int)cm < mk_old);
                mk_new = keep_old ? mk_old : (int)cm;
            }
            L->mk[nxt][slot] = mk_new;
            wkey = ((unsigned long long)(unsigned)mk_new << 32) | (unsigned)slot;
        }
        // cells that keep their individual get the parent's row back, four
        // rows at a time by the whole wave
        unsigned long long km = __ballot(keep_old);
        const int nv = n_pad >> 3;
        const u32x4* s4 = reinterpret_cast<const u32x4*>(L->genes[cur]);
        u32x4* d4 = reinterpret_cast<u32x4*>(L->genes[nxt]);
        while (km) {
            int rows[4];
            int cnt = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                rows[t] = -1;
                if (km) {
                    rows[t] = slot_of(sbase + (int)__builtin_ctzll(km));
                    km &= km - 1ull;
                    ++cnt;
                }
            }
            for (int v0 = lane; v0 < nv; v0 += kWave) {
                u32x4 x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (rows[t] >= 0) x[t] = as_global(s4)[(size_t)rows[t] * nv + v0];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (rows[t] >= 0) as_global(d4)[(size_t)rows[t] * nv + v0] = x[t];
            }
            (void)cnt;
        }
    }
#pragma unroll
    for (int offx = 32; offx > 0; offx >>= 1) {
        const unsigned long long o = __shfl_xor(wkey, offx, 64);
        wkey = o < wkey ? o : wkey;
    }
    __shared__ unsigned long long s_wmin[8];
    if (lane == 0) s_wmin[wave] = wkey;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long mn = ~0ull;
        for (int x = 0; x < (int)(blockDim.x >> 6); ++x) mn = s_wmin[x] < mn ? s_wmin[x] : mn;
        if (mn != ~0ull) atomicMin(L->genkey + (gen & 1), mn);
    }
}

// ---- decode of caller-supplied permutations, lane mapping ------------------
// One row per lane.  Each window of a row is read once, as four 16-byte
// vectors, decoded, and marked in the lane's bit set (LDS atomics without
// return, which nothing waits for); an invalid row gets makespan -1 and
// sets the control block's error word.  Bound by vector issue (M + 5
// operations per job and stage, four more per job for the check), by latency
// where its LDS holds few waves.  A million rows of 100 x 5 take 238 us (371
// pipelined), 262144 rows of 500 x 10 593 us (731 pipelined; about 1380 with
// every row read twice, value by value, and an atomic that returns per value).
template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) k_evaluate_lane(const InstDesc* __restrict__ I, const int* __restrict__ perms,
                                                       int count, int* __restrict__ out, Control* ctl)
{
    const int n = I->n, S = I->S, n_pad = I->n_pad, jb = I->jb;
    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int wpb = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t* wbase = reinterpret_cast<uint32_t*>(ffs_smem + pt_lds_bytes<PT>(S, n_pad) +
                                                  (size_t)wave * I->lane_wlds_eval);
    const long long base = ((long long)blockIdx.x * wpb + wave) * kWave;
    if (base >= count) return;
    const long long idx = base + lane;
    const bool active = idx < count;
    uint32_t* seen = wbase + I->msum * 64 + lane;
    const int nwords = lane_seen_words(jb);
    for (int q = 0; q < nwords; ++q) seen[q * 64] = 0u;
    GenesI32 src{perms + (active ? idx : base) * (long long)n, n, jb, (lane_state)seen, 0u};
    const uint32_t cm = lane_decode<MMAX, PT>(src, pT, pt_stride<PT>(n_pad), I, wbase, lane);
    bool bad = (src.bits >> jb) != 0u;
    for (int q = 0; q < nwords; ++q) {
        const int left = n - 32 * q;
        bad |= seen[q * 64] != (left >= 32 ? 0xFFFFFFFFu : (left > 0 ? (1u << left) - 1u : 0u));
    }
    if (active) out[idx] = bad ? -1 : (int)cm;
    if (active && bad) flag_invalid(ctl);
}

}  // namespace flowshop

namespace flowshop {

// ---- candidates of the learned pre-screen, one wave per cell ----------------
// Features of the chromosome in A (n genes) as features_group computes them,
// from the job-major table pJ (row of job j at pJ + j * rsb bytes, the
// stages' processing times, zero past S): lane l sums the positions
// [l C, l C + C) (C = ceil(n / 64)) stage by stage in registers and adds each
// bucket's partial sums into acc[b * S + k] in LDS (integer sums: the order
// does not matter), then the 256 entries are written to out.
template <int SM, typename PT>
__device__ __forceinline__ void cand_features(const uint16_t* A, const unsigned char* pJ, int rsb, const InstDesc* I,
                                              const CellMeta& cm, uint32_t* acc, int lane, uint16_t* out)
{
    const int n = I->n, S = I->S, B = 240 / S;
    for (int e = lane; e < B * S; e += kWave) acc[e] = 0u;
    wave_sync();
    const int C = (n + kWave - 1) / kWave;
    const int t0 = lane * C < n ? lane * C : n, t1 = t0 + C < n ? t0 + C : n;
    // per-lane sums over at most 64 positions; with one-byte processing
    // times (<= 255) they fit in 16 bits, so stages 4d + {0, 2} and
    // 4d + {1, 3} share a register and are added pairwise (integer packed adds)
    constexpr bool PK = sizeof(PT) == 1;
    constexpr int NR = PK ? (SM + 1) / 2 : SM;   // accumulator registers
    uint32_t s[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) s[k] = 0u;
    int cb = (int)(((long long)t0 * B) / n);
    int next = (int)(((long long)(cb + 1) * n + B - 1) / B);   // first position of bucket cb + 1
    auto add_row = [&](uint32_t* x, int t) {
        const PT* row = reinterpret_cast<const PT*>(pJ + (size_t)A[t] * rsb);
        constexpr int PV = 16 / (int)sizeof(PT);   // processing times per 16-byte read
        constexpr int NB = (SM + PV - 1) / PV;     // 16-byte reads per row
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const uint4 w = reinterpret_cast<const uint4*>(row)[v];
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
            if (PK) {
                typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int r = 2 * (v * 4 + d);   // registers of stages 4 (4v + d) + {0, 2} and + {1, 3}
                    if (r < NR) {
                        const u16x2 lo = __builtin_bit_cast(u16x2, ww[d] & 0x00FF00FFu);
                        const u16x2 hi = __builtin_bit_cast(u16x2, (ww[d] >> 8) & 0x00FF00FFu);
                        x[r] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, x[r]) + lo);
                        x[r + 1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, x[r + 1]) + hi);
                    }
                }
            } else {
#pragma unroll
                for (int q = 0; q < PV; ++q)
                    if (v * PV + q < SM) x[v * PV + q] += (ww[q >> 1] >> (16 * (q & 1))) & 0xFFFFu;
            }
        }
    };
    auto flush = [&]() {
#pragma unroll
        for (int k = 0; k < SM; ++k)
            if (k < S) {
                // stage k sits in register 2 (k / 4) + (k & 1), half (k >> 1) & 1
                const uint32_t v = PK ? (s[2 * (k >> 2) + (k & 1)] >> (16 * ((k >> 1) & 1))) & 0xFFFFu : s[k];
                if (v) atomicAdd(&acc[cb * S + k], v);
            }
#pragma unroll
        for (int k = 0; k < NR; ++k) s[k] = 0u;
    };
    if (n / B >= C) {
        // every bucket holds at least C positions, so [t0, t1) meets at most
        // one boundary, tb: the sums are snapshotted there (a select per
        // register, no divergent flush inside the loop) and split after it
        const int tb = next < t1 ? next : t1;
        uint32_t snap[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) snap[k] = 0u;
#pragma unroll 2
        for (int t = t0; t < t1; ++t) {
            const bool at = t == tb;
#pragma unroll
            for (int k = 0; k < NR; ++k) snap[k] = at ? s[k] : snap[k];
            add_row(s, t);
        }
        if (tb >= t1) {
#pragma unroll
            for (int k = 0; k < NR; ++k) snap[k] = s[k];
        }
        // s - snap per 16-bit half (each half only grows, so no borrow crosses)
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            if (PK) {
                typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
                s[k] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, s[k]) - __builtin_bit_cast(u16x2, snap[k]));
            } else {
                s[k] -= snap[k];
            }
        }
#pragma unroll
        for (int k = 0; k < SM; ++k)
            if (k < S && t0 < t1) {
                const uint32_t v0 = PK ? (snap[2 * (k >> 2) + (k & 1)] >> (16 * ((k >> 1) & 1))) & 0xFFFFu : snap[k];
                const uint32_t v1 = PK ? (s[2 * (k >> 2) + (k & 1)] >> (16 * ((k >> 1) & 1))) & 0xFFFFu : s[k];
                if (v0) atomicAdd(&acc[cb * S + k], v0);
                if (v1) atomicAdd(&acc[(cb + 1) * S + k], v1);
            }
    } else {
        for (int t = t0; t < t1; ++t) {
            if (t >= next) {
                flush();
                cb += 1;
                next = (int)(((long long)(cb + 1) * n + B - 1) / B);
            }
            add_row(s, t);
        }
        if (t0 < t1) flush();
    }
    wave_sync();
    const float fn = (float)n, fLB = (float)I->LB;
    for (int e = lane; e < kFeat; e += kWave) {
        float v = 0.f;
        if (e < B * S) {
            const int k = e - (e / S) * S;
            v = __fdiv_rn((float)((uint64_t)acc[e] * (uint64_t)B), (float)I->Pk[k]);
        } else {
            switch (e - 240) {
                case 0: v = __fdiv_rn((float)cm.mk1, fLB); break;
                case 1: v = __fdiv_rn((float)cm.mk2, fLB); break;
                case 2: v = __fdiv_rn((float)cm.a, fn); break;
                case 3: v = __fdiv_rn((float)cm.b, fn); break;
                case 4: v = cm.cx ? 1.f : 0.f; break;
                case 5: v = cm.mx ? 1.f : 0.f; break;
                case 6: v = __fdiv_rn((float)cm.mi, fn); break;
                case 7: v = __fdiv_rn((float)cm.mj, fn); break;
                case 8: v = __fdiv_rn(fLB, (float)I->E); break;
                case 9: v = __fdiv_rn(fn, 1000.f); break;
                case 10: v = __fdiv_rn((float)S, 20.f); break;
                case 11: v = __fdiv_rn((float)I->msum, (float)(6 * S)); break;
                default: break;
            }
        }
        out[e] = f32_to_bf16(v);
    }
}

// One wave per cell of the pre-screened instance's cellular islands: lane c
// (< K) takes the parents and draws of candidate c (candidate stream c of
// the CELL purpose, generation completed + 1); the wave then builds each
// candidate on all 64 lanes (order crossover, swap mutation) and writes its
// features to Xout[(cell * K + c) * 256].  LDS: the job-major table (rows of
// rsb bytes), then per wave wave_row(n_pad) entries and 240 words of bucket
// sums.
template <int SM, typename PT>
__global__ void __launch_bounds__(1024) k_cand_features(const InstDesc* __restrict__ insts,
                                                       const IslandDesc* __restrict__ isls, int inst,
                                                       const Control* ctl, int cells, uint16_t* __restrict__ Xout)
{
    const InstDesc* I = insts + inst;
    const int n = I->n, S = I->S, n_pad = I->n_pad, K = I->surr_k;
    const int rsb = I->pj_row_bytes;
    const int done = completed_gen(ctl);
    const int gen = done + 1, cur = done & 1;
    unsigned char* pJ = ffs_smem;
    {
        const size_t words = (size_t)n * rsb / 16;
        const auto* s4 = as_global(reinterpret_cast<const u32x4*>(I->pJ));
        u32x4* d4 = reinterpret_cast<u32x4*>(pJ);
        for (size_t v = threadIdx.x; v < words; v += blockDim.x) d4[v] = s4[v];
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cell = blockIdx.x * (blockDim.x >> 6) + wave;
    if (cell >= cells) return;
    uint16_t* A = reinterpret_cast<uint16_t*>(pJ + align16((size_t)n * rsb) +
                                              (size_t)wave * (wave_row(n_pad) * 2 + 240 * 4));
    uint32_t* acc = reinterpret_cast<uint32_t*>(A + wave_row(n_pad));
    // the cellular island holding this cell
    const IslandDesc* L = isls + I->island0;
    int slot = 0;
    for (int x = 0; x < I->n_islands; ++x) {
        const IslandDesc* X = isls + I->island0 + x;
        if (X->kind == 0 && cell >= X->cell_base && cell < X->cell_base + X->size) {
            L = X;
            slot = cell - X->cell_base;
        }
    }
    const CellPlan pl = cell_plan(I, L, slot, (uint32_t)(lane < K ? lane : 0), gen, cur);
    const uint32_t w_src = (uint32_t)pl.p1 | ((uint32_t)pl.p2 << 16);
    const uint32_t w_cut = (uint32_t)pl.meta.a | ((uint32_t)pl.meta.b << 12) | (pl.meta.cx ? 1u << 24 : 0u) |
                           (pl.meta.mx ? 1u << 25 : 0u);
    const uint32_t w_mut = (uint32_t)pl.meta.mi | ((uint32_t)pl.meta.mj << 12);
    const uint16_t* gp = L->genes[cur];
    for (int t = n + lane; t < n_pad; t += kWave) A[t] = 0;   // the row's padding
    auto parents = [&](int c, const uint16_t*& p1, const uint16_t*& p2) {
        const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)w_src, c);
        p1 = gp + (size_t)(src & 0xFFFFu) * n_pad;
        p2 = gp + (size_t)(src >> 16) * n_pad;
    };
    auto meta = [&](int c) {
        const uint32_t cut = (uint32_t)__builtin_amdgcn_readlane((int)w_cut, c);
        const uint32_t mut = (uint32_t)__builtin_amdgcn_readlane((int)w_mut, c);
        CellMeta cm;
        cm.mk1 = __builtin_amdgcn_readlane(pl.meta.mk1, c);
        cm.mk2 = __builtin_amdgcn_readlane(pl.meta.mk2, c);
        cm.a = (int)(cut & 0xFFFu);
        cm.b = (int)((cut >> 12) & 0xFFFu);
        cm.cx = ((cut >> 24) & 1u) != 0u;
        cm.mx = ((cut >> 25) & 1u) != 0u;
        cm.mi = (int)(mut & 0xFFFu);
        cm.mj = (int)(mut >> 12);
        return cm;
    };
    auto finish = [&](int c, const CellMeta& cm) {
        swap_genes(A, cm.mx && lane == 0, cm.mi, cm.mj);
        cand_features<SM, PT>(A, pJ, rsb, I, cm, acc, lane, Xout + ((size_t)cell * K + c) * kFeat);
        wave_sync();
    };
    auto build = [&](auto cc) {
        constexpr int C = decltype(cc)::value;   // genes per lane
        LaneGenes<C> ra, rb;
        auto fetch = [&](int c) {
            const uint16_t *p1, *p2;
            parents(c, p1, p2);
            lane_genes_load<C>(ra, p1, lane, n_pad);
            lane_genes_load<C>(rb, p2, lane, n_pad);
        };
        fetch(0);
        for (int c = 0; c < K; ++c) {
            const CellMeta cm = meta(c);
            const LaneGenes<C> x1 = ra, x2 = rb;
            if (c + 1 < K) fetch(c + 1);
            ox_wave<C>(A, x1, x2, ox_cut(n, cm.cx, cm.a, cm.b, false, false), lane);
            finish(c, cm);
        }
    };
    // up to 512 and 1024 jobs the next candidate's parents are read while this
    // one is built; longer rows are read when they are needed
    if (n <= 512) {
        build(std::integral_constant<int, 8>{});
    } else if (n <= 1024) {
        build(std::integral_constant<int, 16>{});
    } else {
        for (int c = 0; c < K; ++c) {
            const CellMeta cm = meta(c);
            const uint16_t *p1, *p2;
            parents(c, p1, p2);
            ox_wave_long(A, n_pad, p1, p2, ox_cut(n, cm.cx, cm.a, cm.b, false, false), lane);
            finish(c, cm);
        }
    }
}

// LDS bytes of a k_cand_features workgroup of `waves` waves.
__host__ __device__ inline size_t cand_lds_bytes(int n, int n_pad, int rsb, int waves)
{
    return align16((size_t)n * rsb) + (size_t)waves * ((size_t)wave_row(n_pad) * 2 + 240 * 4);
}

}  // namespace flowshop
