// ffs_kernels.h -- gfx950 kernels of the island GA hot path.
//
// Mapping (one wave = 64 lanes):
//   * a wave holds G = floor(64 / S) chromosomes; lane g*S + k works on
//     stage k of chromosome g ("group" g).  Lanes beyond G*S idle.
//   * decode (paper Section 3 problem; list-scheduling rule documented in
//     include/ffs.h) runs as a systolic pipeline along the group: the lane of
//     stage k keeps the m_k machine-free times of its stage, sorted, in
//     registers, dispatches one job per step and hands the job it takes off
//     the list, in (completion, dispatch order), to the lane of stage k+1.
//   * the genetic operators (Section 4.1-4.2: neighbourhood choice, order
//     crossover, swap mutation, complementary pairs) run on the same group of
//     lanes, the parents in registers and the child in LDS.
//   * populations live in HBM as rows of n_pad uint16 genes (slot-major,
//     64-byte aligned rows), double buffered by generation parity.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ffs_mlp.h"
#include "philox.h"

namespace flowshop {

constexpr int kWave = 64;
constexpr int kMaxStages = 64;
constexpr int kMaxMachines = 16;

// The islands of a context form fold groups: the islands whose generations
// one launch sequence runs (a launch chain of a large instance's islands, or
// a launch class's instances), whose best individuals the extra workgroup of
// that sequence's launches folds into the best-ever records.  Between
// migration epochs the groups' sequences are independent.  An instance split
// over two chains keeps a record per chain (record slot); its record is the
// better of the two by (makespan, generation, island, slot).
constexpr int kChains = 2;      // record slots per instance
constexpr int kMaxGroups = 16;  // fold groups per context

struct InstDesc {
    const void* pT;          // [S][n_pad] processing times, uint8 or uint16
    uint16_t* best_perm;     // [kChains][n_pad]
    int* best_rec;           // [kChains][4]: makespan, generation, island (local), slot
    long long* counters;     // migration epochs with moves, migrants
    unsigned long long seed;
    unsigned long long theta_T;  // floor(theta * 2^32)
    long long E;                 // sum of all processing times
    int inst_id;
    int n, S, n_pad, jb, G;
    int lkey, pkey;              // KeyFormat of the lane decode and of the pipelined decode
    int island0, n_islands;
    int interval, topology;
    // learned pre-screen (surr_k > 1): candidate streams per cell, replay ring
    int surr_k, surr_warmup, n_cells, ring_size;
    int* surr_choice;            // [n_cells] candidate chosen for the next generation
    const uint16_t* surr_X;      // [n_cells * surr_k][256] features of the scored candidates
    uint16_t* ring_X;            // [ring_size][256] features of decoded children
    float* ring_T;               // [ring_size] (C - LB) / LB
    int LB, msum;
    int lane_wlds, lane_wlds_eval;   // lane mapping: LDS bytes per wave (generation, ffs_evaluate)
    const void* pJ;              // pre-screen: job-major processing times, rows of pj_row_bytes
    int pj_row_bytes;
    int mach[kMaxStages];
    int Pk[kMaxStages];          // sum over jobs of p[j][k]
};

struct IslandDesc {
    uint16_t* genes[2];          // [size][n_pad] per generation parity
    int* mk[2];                  // [size]
    unsigned long long* genkey;  // [2]: min of (makespan << 32 | slot), by generation parity
    unsigned long long* minmax;  // [2] min / max keys (ring migration)
    int* sorted;                 // [size] slots by (makespan, slot) (migration)
    int* sortbest;               // [1] island minimum makespan when `sorted` was built
    unsigned long long tc, tm;   // crossover / mutation thresholds (< tc, < tm)
    int kind, rows, cols, size;
    int inst;
    int local;                   // island index inside its instance
    int cell_base;               // index of slot 0 among the instance's cellular cells
    int sel;                     // cellular parent selection variant (0, 1, 2)
    int sweep;                   // cellular update: 0 synchronous, 1 line sweep
    int chain;                   // fold group of the island's generations
    int rec;                     // its instance's record slot for that group
    uint16_t* ep_perm;           // resident epochs: the epoch's best row [n_pad] and its record
    int* ep_rec;                 // [3]: makespan, generation, slot
};

struct WorkItem {
    int island, slot0, count, inst;
};

struct PairDesc {
    int a, b, inst, pad;
};

// Generation bookkeeping without a last-workgroup handshake or a shared
// counter: workgroup b of every generation launch keeps its own count of the
// launches it has run, counts[b], so launch number counts[b] after `base`
// runs generation base + 1 + counts[b]; the counts of all workgroups agree
// between launches, and kernels that run between launches read counts[0].
struct Control {
    int* counts;                 // [workgroups per generation launch]
    int base;                    // completed generation when the counts were zero
    int best_gen[kMaxGroups];    // per fold group: last generation folded into the records
    int* err;                    // set to 1 by a decode of an invalid row (host memory, or noalloc scratch)
};

__device__ __forceinline__ void flag_invalid(const Control* c)
{
    __hip_atomic_store(c->err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ int completed_gen(const Control* c)
{
    return c->base + c->counts[0];
}

extern __shared__ __align__(16) unsigned char ffs_smem[];

// Four values of a caller's row, which is aligned as an int is.  (Pointers to
// it are formed with this type: as a template's argument it would lose the
// alignment, and the reads would claim 16 bytes.)
typedef int row_vec __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(1))) row_vec* row_vec_ptr;

// Global-memory views of generic pointers: accesses through them compile to
// global (not flat) instructions, which the compiler may keep in flight
// across LDS accesses.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* as_global(const T* p)
{
    return (const __attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p)
{
    return (__attribute__((address_space(1))) T*)p;
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// Vectors of eight genes that a lane owns when S lanes share a row, and the
// most that the register path of the crossover holds.
__host__ __device__ inline int ox_vectors(int n, int S) { return ((n + 7) / 8 + S - 1) / S; }
constexpr int kOxVec = 13;
constexpr int kOxSmall = 3;   // its smallest tier

// LDS of one group: the child's row of n_pad uint16 and 16 bytes of padding,
// so that the groups of a wave start 4 banks apart and same-offset accesses of
// different groups do not collide.  The crossover marks parent 1's positions
// in the row itself before it writes the child there; rows of more than
// kOxVec vectors per lane have the marks in a second row.
__host__ __device__ inline int group_stride(int n, int n_pad, int S)
{
    return ox_vectors(n, S) <= kOxVec ? n_pad + 8 : 2 * n_pad + 8;
}

__host__ __device__ inline size_t wave_lds_bytes(int G, int n, int n_pad, int S)
{
    return (size_t)G * group_stride(n, n_pad, S) * 2;
}

// LDS entries of a wave that builds whole rows, one at a time.
// Above 2048 jobs the crossover's marks have a row of their own.
__host__ __device__ inline int wave_row(int n_pad) { return n_pad <= 2048 ? n_pad + 8 : 2 * n_pad + 8; }

// The processing-time table is staged into LDS stage-major with each row
// padded by 4 bytes, so that the S rows start on different LDS banks (the S
// lanes of a group read the same job in S different rows).
template <typename PT>
__host__ __device__ inline int pt_stride(int n_pad) { return n_pad + 4 / (int)sizeof(PT); }

template <typename PT>
__host__ __device__ inline size_t pt_lds_bytes(int S, int n_pad)
{
    return align16((size_t)S * pt_stride<PT>(n_pad) * sizeof(PT));
}

// HBM rows of n_pad elements -> LDS rows of pt_stride elements (32-bit words).
template <typename PT>
__device__ __forceinline__ void stage_pt(PT* dst, const void* src, int S, int n_pad)
{
    constexpr int U = 4;
    const int wpr = (int)(n_pad * sizeof(PT) / 4), ld = wpr + 1, nw = S * wpr;
    const auto* s = as_global(reinterpret_cast<const uint32_t*>(src));
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
    for (int w0 = threadIdx.x; w0 < nw; w0 += U * blockDim.x) {
        uint32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int w = w0 + u * blockDim.x;
            x[u] = s[w < nw ? w : nw - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // past the end: the last word again, with the same value
            const int w = w0 + u * blockDim.x < nw ? w0 + u * blockDim.x : nw - 1;
            const int r = w / wpr, c = w - r * wpr;
            d[r * ld + c] = x[u];
        }
    }
}

// ---- row copies by the S lanes of a group (16-byte vectors) ---------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void row_g2g(uint16_t* dst, const uint16_t* src, int n_pad, int k, int S)
{
    constexpr int U = 4;
    const auto* s4 = as_global(reinterpret_cast<const u32x4*>(src));
    auto* d4 = as_global(reinterpret_cast<u32x4*>(dst));
    const int nv = n_pad >> 3;
    for (int v0 = k; v0 < nv; v0 += U * S) {
        u32x4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = s4[v0 + u * S < nv ? v0 + u * S : nv - 1];
#pragma unroll
        for (int u = 0; u < U; ++u) d4[v0 + u * S < nv ? v0 + u * S : nv - 1] = x[u];
    }
}

__device__ __forceinline__ void row_l2g(uint16_t* dst, const uint16_t* src, int n_pad, int k, int S)
{
    const u32x4* s4 = reinterpret_cast<const u32x4*>(src);
    auto* d4 = as_global(reinterpret_cast<u32x4*>(dst));
    const int nv = n_pad >> 3;
#pragma unroll 4
    for (int v = k; v < nv; v += S) d4[v] = s4[v];
}

// ---- pipelined decode -----------------------------------------------------
// Value of `x` held by lane - 1 (whole-wave rotation by one lane, DPP; lane 0
// reads lane 63).
__device__ __forceinline__ uint32_t from_prev_lane(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x13C /* wave_ror:1 */, 0xF, 0xF, true);
}

// Median of three unsigned words (one VALU operation, v_med3_u32).
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c)
{
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    const uint32_t m = hi < c ? hi : c;
    return lo > m ? lo : m;
}

// Key formats of the decodes (InstDesc::pkey, lkey), both with the completion
// time in the high bits:
//   kKeyTwo: completion << jb | job; a new key enters after the entries of
//     equal completion by a threshold compare per entry (3 M operations for a
//     list of M);
//   kKeyIdx: completion << (jb + IB) | index << jb | job; the keys of one list
//     are distinct and their numeric order is (completion, dispatch order), so
//     a new key enters by one min, max or median per entry (M operations).
//     The index only has to order the entries of one list, so it is local to a
//     block of consecutive dispatches: at a block's start the list's entries
//     are renumbered by their place (0, 1, ...), and the block's dispatches
//     take the indices after them.  IB bits hold both, whatever the number of
//     jobs (a dispatch index of the whole stage would take jb bits and leave
//     12 for the completion at 1000 jobs; this leaves 18);
//   kKeyIdxChecked: the same, and the largest completion is kept, since the
//     instance's completions may outgrow the field: the wave then decodes
//     again with kKeyTwo.
enum KeyFormat { kKeyTwo = 0, kKeyIdx = 1, kKeyIdxChecked = 2 };

// The pipelined decode's blocks are eight steps: the list takes the indices
// below 8 (16 with up to 16 machines), the block's dispatches the next eight.
constexpr int kPipeBlock = 8;
constexpr int pipe_first(int mmax) { return mmax <= 8 ? 8 : 16; }
constexpr int pipe_index_bits(int mmax) { return mmax <= 8 ? 4 : 5; }

// LDS views of generic pointers, for code behind a call: accesses through
// them compile to LDS (not flat) instructions.
template <typename T>
using lds_ptr = const __attribute__((address_space(3))) T*;
template <typename T>
__device__ __forceinline__ lds_ptr<T> as_lds(const T* p)
{
    return (lds_ptr<T>)p;
}

// What one lane of the pipelined decode is given.
template <typename PT>
struct PipeLane {
    lds_ptr<uint16_t> feed_row;  // the permutation that this lane feeds (in bounds on every lane)
    lds_ptr<PT> prow;            // processing times it looks up: the next stage's, the first stage's if it feeds
    bool feed;                   // this lane feeds the next group
    int k;                       // its stage
};

// One step of stage k (see decode_pipe).  With PRED the lane inserts
// nothing while rel >= n_act (the key it removed goes back in: the list stays
// as it is), padding while rel >= n, and a job below that; without PRED the
// caller guarantees that every lane that matters takes a job.
template <int MMAX, bool PRED, int KEY, typename PT>
__device__ __forceinline__ void pipe_step(uint32_t (&key)[MMAX], uint32_t& o_key, uint32_t& o_p, uint32_t& nx_key,
                                          uint32_t& pn, uint32_t feed_gene, uint32_t rel, uint32_t n_act,
                                          uint32_t un, bool feed, uint32_t sh, uint32_t jmask, lds_ptr<PT> prow,
                                          uint32_t idx, uint32_t& cmx)
{
    constexpr uint32_t PAD = 0xFFFFFFFFu;
    const uint32_t in_key = from_prev_lane(o_key);
    const uint32_t in_p = from_prev_lane(o_p);
    const bool have = !PRED || rel < un;
    const bool act = !PRED || rel < n_act;
    const uint32_t o = key[0];
    // start = max(machine free, job ready): the larger key has the larger (or
    // equal) time in its high bits
    const uint32_t mx = o > in_key ? o : in_key;
    const uint32_t c = (mx >> sh) + in_p;
    if (KEY == kKeyTwo) {
        uint32_t nk = (c << sh) | (in_key & jmask), ithr = (c + 1u) << sh;
        if (PRED) {
            nk = have ? nk : PAD;
            nk = act ? nk : o;
            ithr = have ? ithr : PAD;
            ithr = act ? ithr : 0u;
        }
        uint32_t nkey[MMAX];
        bool prev = true;
#pragma unroll
        for (int i = 0; i < MMAX; ++i) {
            const bool lt = (i + 1 < MMAX) ? (key[(i + 1 < MMAX) ? i + 1 : i] < ithr) : false;
            nkey[i] = lt ? key[(i + 1 < MMAX) ? i + 1 : i] : (prev ? nk : key[i]);
            prev = lt;
        }
#pragma unroll
        for (int i = 0; i < MMAX; ++i) key[i] = nkey[i];
    } else {
        uint32_t nk = (c << sh) | ((in_key & jmask) | idx);
        if (KEY == kKeyIdxChecked) {
            const uint32_t cc = (PRED && !have) ? 0u : c;
            cmx = cc > cmx ? cc : cmx;
        }
        if (PRED) {
            nk = have ? nk : PAD;
            nk = act ? nk : o;
        }
        if (MMAX == 1) {
            key[0] = nk;
        } else {
            uint32_t nkey[MMAX];
            nkey[0] = key[1 < MMAX ? 1 : 0] < nk ? key[1 < MMAX ? 1 : 0] : nk;
#pragma unroll
            for (int i = 1; i + 1 < MMAX; ++i) nkey[i] = umed3(key[i], nk, key[i + 1]);
            nkey[MMAX - 1] = key[MMAX - 1] > nk ? key[MMAX - 1] : nk;
#pragma unroll
            for (int i = 0; i < MMAX; ++i) key[i] = nkey[i];
        }
    }
    // handed on in the next step: the key removed next and its job's time at
    // the next stage, whose read has a whole step to arrive; a feeding lane
    // hands on the next gene but one and its time at the first stage
    o_key = nx_key;
    o_p = pn;
    nx_key = feed ? feed_gene : key[0];
    pn = (uint32_t)prow[nx_key & jmask];
}

// One group of S lanes decodes one permutation; lane k runs stage k.
//
// Stage k keeps its m_k machine-free times as a sorted list of keys (see
// KeyFormat) in registers; a machine that has not run a job yet holds
// completion 0, a padding entry (fewer than MMAX machines) all ones.  Each
// step dispatches the next job: it takes the machine of entry 0 (free first;
// ties on time only relabel machines), starts at max(free, ready) and inserts
// its completion.  The removed entry 0 is handed to stage k+1: entries leave
// the list in (completion, dispatch order) order, which is the order in which
// stage k+1 must dispatch them.  After its last job a stage hands on its
// remaining entries, one per step.
//
// The timing of this pipeline does not depend on the data: stage k acts in
// steps [a_k, a_k + n) (dispatch) and, unless it is the last stage, in
// [a_k + n, a_k + n + m_k) (hand-on of the rest); the first m_k entries it
// removes are the never-used machines, so its real jobs leave in steps
// [a_k + m_k, a_k + m_k + n) and stage k+1 starts at a_{k+1} = a_k + m_k + 1.
// The decode therefore runs exactly n + sum_{k<S-1} (m_k + 1) steps, and a
// job handed on in one step is taken by the next lane in the next step, so
// one register pair per lane carries it: (key, processing time at k+1).
//
// Stage 0 takes its jobs the same way: the lane before it, whose own stage is
// the last one and hands nothing on (lane 63 for group 0), feeds it the
// permutation's genes, each with completion 0 and its time at the first
// stage.  So every lane runs the same instructions, without selects for the
// first stage and without a table of (time, job) words built beforehand, and
// the permutation's 16-bit row is all a group keeps in LDS: 13.5 VALU
// operations a step for lists of M = 4 (four insert the key, half of one
// renumbers a block's indices), from about 31, and a third of the LDS.
// What bounds it: the chain of a step, about 15 dependent VALU operations and
// the table read that the next step waits for, when a SIMD holds one or two
// waves; VALU issue beyond that.  ffs_evaluate, from the version with table
// words and two-field keys: a million rows of 100 jobs and 5 stages 562 ->
// 376 us, 4099 rows of 1000 jobs and 20 stages 275 -> 147 us (one round of
// workgroups instead of two).
//
// Steps run in blocks of eight.  A block in which every stage dispatches in
// every step runs without predication; lanes of unused groups then compute
// values nobody reads (a job index never exceeds jmask, so their reads stay
// inside the workgroup's LDS: prow reaches at most 2 n entries into a table
// that the groups' rows follow).
//
// Returns the makespan on the lane of the last stage; cmx receives the
// largest completion (kKeyIdxChecked).
template <int MMAX, int KEY, typename PT>
__device__ __forceinline__ uint32_t decode_pipe(const PipeLane<PT>& pl, const int* mach, int S, int n, int n_pad,
                                                int jb, uint32_t& cmx)
{
    constexpr uint32_t PAD = 0xFFFFFFFFu;
    constexpr int IB = pipe_index_bits(MMAX), NB0 = pipe_first(MMAX);
    const int k = pl.k;
    int a_k = 0, total = n;
    for (int i = 0; i + 1 < S; ++i) {
        const int step = mach[i] + 1;
        if (i < k) a_k += step;
        total += step;
    }
    const int a_last = total - n;
    const int mstage = mach[k];
    const bool feed = pl.feed;
    const uint32_t jmask = (1u << jb) - 1u;
    const uint32_t sh = (uint32_t)(KEY == kKeyTwo ? jb : jb + IB);
    const uint32_t keep = ~(((1u << IB) - 1u) << jb);
    const uint32_t un = (uint32_t)n;
    const uint32_t n_act = (k == S - 1) ? un : un + (uint32_t)mstage;
    uint32_t key[MMAX];
#pragma unroll
    for (int i = 0; i < MMAX; ++i) key[i] = (i < mstage) ? 0u : PAD;
    // the genes, eight per 16-byte read (rows hold n_pad + 8 entries)
    typedef const __attribute__((address_space(3))) u32x4* row_vec;
    const row_vec row = (row_vec)pl.feed_row;
    const int vmax = n_pad >> 3;
    u32x4 cur = row[0], nxt = row[vmax < 1 ? vmax : 1];
    auto gene = [&](const u32x4& v, int e) -> uint32_t {
        return __builtin_amdgcn_ubfe(v[e >> 1], 16 * (e & 1), jb);
    };
    uint32_t o_key = gene(cur, 0), nx_key = gene(cur, 1);
    uint32_t o_p = (uint32_t)pl.prow[o_key], pn = (uint32_t)pl.prow[nx_key];
    for (int t = 0; t < total; t += kPipeBlock) {
        const int vn = (t >> 3) + 2;
        const u32x4 nn = row[vn < vmax ? vn : vmax];   // for the next block
        if (KEY != kKeyTwo) {
#pragma unroll
            for (int i = 0; i < MMAX; ++i) key[i] = (key[i] & keep) | ((uint32_t)i << jb);
        }
        if (t >= a_last && t + kPipeBlock <= n) {
#pragma unroll
            for (int i = 0; i < kPipeBlock; ++i) {
                const uint32_t fg = i < 6 ? gene(cur, i + 2) : gene(nxt, i - 6);
                pipe_step<MMAX, false, KEY, PT>(key, o_key, o_p, nx_key, pn, fg, 0u, 0u, un, feed, sh, jmask, pl.prow,
                                                (uint32_t)(NB0 + i) << jb, cmx);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kPipeBlock; ++i) {
                const uint32_t fg = i < 6 ? gene(cur, i + 2) : gene(nxt, i - 6);
                pipe_step<MMAX, true, KEY, PT>(key, o_key, o_p, nx_key, pn, fg, (uint32_t)(t + i - a_k), n_act, un,
                                               feed, sh, jmask, pl.prow, (uint32_t)(NB0 + i) << jb, cmx);
            }
        }
        cur = nxt;
        nxt = nn;
    }
    // the last stage's list now holds every machine's final completion time
    uint32_t cmax = 0;
#pragma unroll
    for (int i = 0; i < MMAX; ++i) {
        const uint32_t c = (key[i] >> sh) == (PAD >> sh) ? 0u : (key[i] >> sh);
        cmax = c > cmax ? c : cmax;
    }
    return cmax;
}

// The two-field decode as a function of its own: the fallback of the checked
// one, and the decode of instances whose completions do not fit beside an
// index.
template <int MMAX, typename PT>
__device__ __attribute__((noinline)) uint32_t decode_pipe_two(PipeLane<PT> pl, const int* mach, int S, int n,
                                                              int n_pad, int jb)
{
    uint32_t cmx = 0u;
    return decode_pipe<MMAX, kKeyTwo, PT>(pl, mach, S, n, n_pad, jb, cmx);
}

// The pipelined decode with the instance's key format.
template <int MMAX, typename PT>
__device__ __forceinline__ uint32_t decode_pipelined(const PipeLane<PT>& pl, const InstDesc* I, bool active)
{
    const int *mach = I->mach, S = I->S, n = I->n, n_pad = I->n_pad, jb = I->jb, fmt = I->pkey;
    uint32_t cmx = 0u;
    if (fmt == kKeyIdx) return decode_pipe<MMAX, kKeyIdx, PT>(pl, mach, S, n, n_pad, jb, cmx);
    if (fmt == kKeyTwo) return decode_pipe_two<MMAX, PT>(pl, mach, S, n, n_pad, jb);
    const uint32_t cm = decode_pipe<MMAX, kKeyIdxChecked, PT>(pl, mach, S, n, n_pad, jb, cmx);
    // a completion that reaches the field's largest value (padding's) or
    // outgrows it, on any lane of any group: every group takes the two-field
    // result, which is the same wherever both are right
    const uint32_t cap = 0xFFFFFFFFu >> (jb + pipe_index_bits(MMAX));
    if (__ballot(active && cmx >= cap) == 0ull) return cm;
    return decode_pipe_two<MMAX, PT>(pl, mach, S, n, n_pad, jb);
}

// The lane's part in the pipeline: group g of a wave of G groups, stage k,
// of which the first `groups` hold a chromosome (one at least); rows at
// gbase, `stride` entries apart.
template <typename PT>
__device__ __forceinline__ PipeLane<PT> pipe_lane(const uint16_t* gbase, int stride, const PT* pT, int n_pad, int lane,
                                                  int g, int k, int S, int G, int groups)
{
    PipeLane<PT> pl;
    pl.k = k;
    pl.feed = k == S - 1 || lane == kWave - 1;
    int fg = lane == kWave - 1 ? 0 : g + 1;
    fg = (fg < G && fg < groups) ? fg : 0;
    pl.feed_row = as_lds(gbase + (size_t)fg * stride);
    pl.prow = as_lds(pT + (size_t)(pl.feed ? 0 : k + 1) * pt_stride<PT>(n_pad));
    return pl;
}

// ---- order crossover on rows read as vectors --------------------------------
// child[a..b] = P1[a..b]; P2 read cyclically from b+1 fills b+1, ..., n-1, 0,
// ..., a-1 with the genes not in the segment (a = 0, b = n - 1: the child is
// P1).  A parent may be given as its reversal (rev: position p of the parent
// is entry n-1-p of the row), so a pseudo pair needs no reversed copy.
//
// Lane k of the S lanes that share a row owns 16-byte vectors [v0, v0 + vpl)
// of both rows, in registers.  P1's genes mark the row, indexed by gene, with
// their position - a (unsigned: the segment's are <= b - a); each P2 gene
// reads its mark, and the genes to keep become one bit each; a scan over the
// lanes gives every kept gene its place: with K kept genes before it in P2's
// order, Ta kept genes after position b and T = n - 1 - (b - a) in all, its
// rank from b+1 is (K + Ta) mod T, and the free positions in ascending order
// start at rank T - a.  Then the child is written over the marks.  Three LDS
// round trips and one scan; the rows themselves go from HBM to registers.
// One LDS row per chromosome instead of three is what it gains where a
// workgroup's LDS decides how many waves are resident: a generation of fifty
// seeds of 300 jobs and 4 stages (400 workgroups of 124 KB, two rounds; now
// 42 KB, one round) 92 -> 48 us, of 8192 chromosomes of 1000 jobs and 20
// stages with the pre-screen 541 -> 463 us, of the medium size 20.7 -> 19.9 us.
struct OxCut {
    int n, a, len;       // segment [a, a + len]
    bool rev1, rev2;     // parents 1 / 2 reversed
};

__device__ __forceinline__ uint32_t ox_gene(const u32x4& v, int e)
{
    return (e & 1) ? v[e >> 1] >> 16 : v[e >> 1] & 0xFFFFu;
}

// Vectors [v0, v0 + vpl) of a row of nv (past the row's end: its last one).
template <int VC>
__device__ __forceinline__ void ox_load(u32x4 (&x)[VC], const uint16_t* row, int v0, int vpl, int nv)
{
    const auto* r4 = as_global(reinterpret_cast<const u32x4*>(row));
#pragma unroll
    for (int v = 0; v < VC; ++v)
        if (v < vpl) x[v] = r4[v0 + v < nv ? v0 + v : nv - 1];
}

// Marks of parent 1's genes; the lane holds `lim` genes from position 8 v0 on.
template <int VC>
__device__ __forceinline__ void ox_mark(uint16_t* M, const u32x4 (&x)[VC], const OxCut& o, int v0, int vpl, int lim)
{
    const int st = o.rev1 ? -1 : 1;
    int t = (o.rev1 ? o.n - 1 - 8 * v0 : 8 * v0) - o.a;
#pragma unroll
    for (int v = 0; v < VC; ++v)
        if (v < vpl) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (8 * v + e < lim) M[ox_gene(x[v], e)] = (uint16_t)t;
                t += st;
            }
        }
}

// Bits of parent 2's genes to keep (gene e of a vector at bit 7 - e) and
// their count, in the high half those after position b in P2's order.
template <int VC>
__device__ __forceinline__ int ox_keep(const uint16_t* M, const u32x4 (&x)[VC], uint32_t (&keep)[VC], const OxCut& o,
                                       int v0, int vpl, int lim)
{
    const int b = o.a + o.len;
    const int split = (o.rev2 ? o.n - 1 - b : b + 1) - 8 * v0;   // genes below it: after b if reversed, else up to b
    const uint32_t flip = o.rev2 ? 0u : 0xFFu;
    int cnt = 0;
#pragma unroll
    for (int v = 0; v < VC; ++v)
        if (v < vpl) {
            uint32_t m[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) m[e] = M[ox_gene(x[v], e)];
            uint32_t kb = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e)   // outside the segment: len - mark < 0
                kb = __builtin_amdgcn_alignbit(kb, (uint32_t)o.len - m[e], 31);
            const int nval = lim - 8 * v, ns = split - 8 * v;
            kb &= 0xFF00u >> (nval < 0 ? 0 : (nval > 8 ? 8 : nval));
            const uint32_t below_split = (0xFF00u >> (ns < 0 ? 0 : (ns > 8 ? 8 : ns))) & 0xFFu;
            keep[v] = kb & 0xFFu;
            cnt += __popc(keep[v]) + (__popc(keep[v] & (below_split ^ flip)) << 16);
        }
    return cnt;
}

// Parent 1's genes at their positions in the child.  Those outside the
// segment are overwritten by the kept genes, so a parent that is not reversed
// goes in as whole vectors.
template <int VC>
__device__ __forceinline__ void ox_place1(uint16_t* A, const u32x4 (&x)[VC], const OxCut& o, int v0, int vpl, int lim)
{
    if (!o.rev1) {
        u32x4* a4 = reinterpret_cast<u32x4*>(A) + v0;
#pragma unroll
        for (int v = 0; v < VC; ++v)
            if (v < vpl && 8 * v < lim) a4[v] = x[v];
    } else {
#pragma unroll
        for (int v = 0; v < VC; ++v)
            if (v < vpl) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (8 * v + e < lim) A[o.n - 1 - 8 * (v0 + v) - e] = (uint16_t)ox_gene(x[v], e);
            }
    }
}

// The free positions in P2's order: from one, the next is beside it, with the
// segment and the row's end skipped.
struct OxStep {
    int st, seg, seg_to, end, end_to;
};

__device__ __forceinline__ OxStep ox_step(const OxCut& o)
{
    const int b1 = o.a + o.len + 1;
    OxStep s;
    s.st = o.rev2 ? -1 : 1;
    s.seg = o.rev2 ? b1 - 1 : o.a;
    s.seg_to = o.rev2 ? o.a - 1 : b1;
    s.end = o.rev2 ? -1 : o.n;
    s.end_to = o.rev2 ? (b1 == o.n ? o.a - 1 : o.n - 1) : (o.a == 0 ? b1 : 0);
    return s;
}

__device__ __forceinline__ int ox_next(const OxStep& s, int pos)
{
    pos += s.st;
    pos = pos == s.seg ? s.seg_to : pos;
    return pos == s.end ? s.end_to : pos;
}

// Writes the kept genes from position `pos` of the first one on; returns the
// next position.
template <int VC>
__device__ __forceinline__ int ox_place2(uint16_t* A, const u32x4 (&x)[VC], const uint32_t (&keep)[VC], const OxCut& o,
                                         int vpl, int pos)
{
    const OxStep s = ox_step(o);
#pragma unroll
    for (int v = 0; v < VC; ++v)
        if (v < vpl) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (keep[v] & (0x80u >> e)) {
                    A[pos] = (uint16_t)ox_gene(x[v], e);
                    pos = ox_next(s, pos);
                }
        }
    return pos;
}

// Inclusive sum over the wave's lanes (DPP: 1, 2, 4, 8 inside 16-lane rows,
// then the rows' last lanes).
template <int CTRL, int ROWS>
__device__ __forceinline__ int scan_step(int x)
{
    return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}

__device__ __forceinline__ int wave_scan(int x)
{
    x = scan_step<0x111, 0xF>(x);
    x = scan_step<0x112, 0xF>(x);
    x = scan_step<0x114, 0xF>(x);
    x = scan_step<0x118, 0xF>(x);
    x = scan_step<0x142, 0xA>(x);
    x = scan_step<0x143, 0xC>(x);
    return x;
}

// Position of the first kept gene of this lane from the scanned counts:
// `excl` kept genes on the lanes before it, `after` kept genes after b in all.
__device__ __forceinline__ int ox_first(const OxCut& o, int excl, int after)
{
    const int T = o.n - 1 - o.len;
    if (T <= 0) return 0;
    int z = after + o.a;                    // <= 2 T
    z -= z >= 2 * T ? 2 * T : (z >= T ? T : 0);
    int idx = (o.rev2 ? T - 1 - excl : excl) + z;   // excl <= T
    idx = idx < 0 ? idx + T : idx;
    idx = idx >= T ? (idx >= 2 * T ? idx - 2 * T : idx - T) : idx;
    return idx + (idx >= o.a ? o.len + 1 : 0);
}

// Counts of the lanes below in this group and after-b total of the group.
__device__ __forceinline__ int ox_group_first(const OxCut& o, int cnt, int g, int S)
{
    const int incl = wave_scan(cnt);
    const int lo = __shfl(incl - cnt, g * S, 64), hi = __shfl(incl, g * S + S - 1, 64);
    return ox_first(o, (incl - cnt - lo) & 0xFFFF, (hi >> 16) - (lo >> 16));
}

// The group's crossover with every vector in registers: row A (marks, then
// the child) is in LDS, the parents' rows in HBM.  Above seven vectors a lane
// reads parent 1 again, half at a time, for its place in the child: held
// through the crossover, both parents took k_generation to 179 registers, two
// waves per SIMD instead of three, whatever the length of its rows (8192
// individuals of 20 jobs, 20 stages and 80 machines 31.9 -> 35.4 us a
// generation, of 1000 x 20 133 -> 149; now 28.8 and 133, and rows of eight to
// thirteen vectors within 1 % of before).
template <int VC>
__device__ __forceinline__ void ox_group_regs(uint16_t* A, const uint16_t* P1, const uint16_t* P2, const OxCut& o,
                                              int vpl, int g, int k, int S, bool active)
{
    constexpr bool kAgain = VC > 7;
    constexpr int H = kAgain ? (VC + 1) / 2 : VC;
    const int nv = (o.n + 7) >> 3, v0 = k * vpl;
    const int lim = active ? o.n - 8 * v0 : 0;   // genes past vector vpl - 1 are not looked at
    u32x4 x1[VC], x2[VC];
    uint32_t keep[VC];
    ox_load<VC>(x1, P1, v0, vpl, nv);
    ox_load<VC>(x2, P2, v0, vpl, nv);
    ox_mark<VC>(A, x1, o, v0, vpl, lim);
    wave_sync();
    const int cnt = ox_keep<VC>(A, x2, keep, o, v0, vpl, lim);
    const int pos = ox_group_first(o, cnt, g, S);
    wave_sync();
    if (kAgain) {
#pragma unroll
        for (int h = 0; h < VC; h += H) {
            u32x4 y[H];
            const int c = vpl - h < H ? vpl - h : H;
            ox_load<H>(y, P1, v0 + h, c, nv);
            ox_place1<H>(A, y, o, v0 + h, c, lim - 8 * h);
        }
    } else {
        ox_place1<VC>(A, x1, o, v0, vpl, lim);
    }
    wave_sync();
    ox_place2<VC>(A, x2, keep, o, vpl, pos);
    wave_sync();
}

// A row shared by a whole wave: lane l holds genes [C l, C l + C), as many as
// the row needs (C = 1, 2, 4, 8, 16).
template <int C>
struct LaneGenes {
    uint32_t w[C > 1 ? C / 2 : 1];
    __device__ __forceinline__ uint32_t gene(int e) const
    {
        return C == 1 ? w[0] : ((e & 1) ? w[e >> 1] >> 16 : w[e >> 1] & 0xFFFFu);
    }
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The lane's genes of a row of n_pad entries (past its end: its last ones).
template <int C>
__device__ __forceinline__ void lane_genes_load(LaneGenes<C>& x, const uint16_t* row, int lane, int n_pad)
{
    const uint16_t* p = row + (C * lane < n_pad ? C * lane : n_pad - C);
    if constexpr (C == 1) {
        x.w[0] = as_global(p)[0];
    } else if constexpr (C == 2) {
        x.w[0] = as_global(reinterpret_cast<const uint32_t*>(p))[0];
    } else if constexpr (C == 4) {
        const u32x2 v = as_global(reinterpret_cast<const u32x2*>(p))[0];
        x.w[0] = v.x;
        x.w[1] = v.y;
    } else {
#pragma unroll
        for (int q = 0; q < C / 8; ++q) {
            const u32x4 v = as_global(reinterpret_cast<const u32x4*>(p))[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) x.w[4 * q + e] = v[e];
        }
    }
}

// The lane's genes at their positions of an LDS row.
template <int C>
__device__ __forceinline__ void lane_genes_store(uint16_t* A, const LaneGenes<C>& x, int lane)
{
    uint16_t* p = A + C * lane;
    if constexpr (C == 1) {
        p[0] = (uint16_t)x.w[0];
    } else if constexpr (C == 2) {
        *reinterpret_cast<uint32_t*>(p) = x.w[0];
    } else if constexpr (C == 4) {
        *reinterpret_cast<u32x2*>(p) = u32x2{x.w[0], x.w[1]};
    } else {
#pragma unroll
        for (int q = 0; q < C / 8; ++q)
            reinterpret_cast<u32x4*>(p)[q] = u32x4{x.w[4 * q], x.w[4 * q + 1], x.w[4 * q + 2], x.w[4 * q + 3]};
    }
}

// The crossover of a whole wave on one row of up to 64 C genes, both parents
// already in registers.  The kept genes of each entry are one wave mask, so
// the counts below a lane come from mask bit counts instead of a scan over the
// lanes.  About 170 VALU and 26 to 33 LDS instructions a child at 500 jobs (C =
// 8; from 240 and 50 to 80, with a reversed copy for pseudo pairs): a large
// generation 724 -> 690 us, the pre-screen's candidates of 1000 jobs 145 -> 125
// us.  The cost goes with C, not with the row: eight genes a lane for every row
// took generations of 20 and 60 jobs 10 % longer than a scan over single genes
// had (147456 individuals, one lane per chromosome: 20 jobs x 3 stages 142 ->
// 155 us, 86 with C = 1; 60 x 3 150 -> 165, 97; 100 x 5 189 -> 197, 136 with
// C = 2; the uneven batch of 256 instances 157.6 -> 136.4 ms).
template <int C>
__device__ __forceinline__ void ox_wave(uint16_t* A, const LaneGenes<C>& x1, const LaneGenes<C>& x2, const OxCut& o,
                                        int lane)
{
    const int lim = o.n - C * lane;
    {
        const int st = o.rev1 ? -1 : 1;
        int t = (o.rev1 ? o.n - 1 - C * lane : C * lane) - o.a;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (i < lim) A[x1.gene(i)] = (uint16_t)t;
            t += st;
        }
    }
    wave_sync();
    uint32_t m[C];
#pragma unroll
    for (int i = 0; i < C; ++i) m[i] = A[x2.gene(i)];
    // entries of lane l lie after position b in P2's order from lane
    // (q - i + C) / C on (below it if reversed)
    const int b = o.a + o.len, q = o.rev2 ? o.n - 2 - b : b;
    bool kp[C];
    uint32_t excl = 0;
    int after = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        kp[i] = i < lim && m[i] > (uint32_t)o.len;
        const uint64_t bal = __ballot(kp[i]);
        excl = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, excl));
        const int s = (q - i + C) / C;   // q - i + C >= 0
        const uint64_t up = s < 64 ? ~0ull << s : 0ull;
        after += __popcll(bal & (o.rev2 ? ~up : up));
    }
    wave_sync();
    // parent 1's genes at their positions in the child (those outside the
    // segment are overwritten by the kept genes)
    if (!o.rev1) {
        if (lim > 0) lane_genes_store<C>(A, x1, lane);
    } else {
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i < lim) A[o.n - 1 - C * lane - i] = (uint16_t)x1.gene(i);
    }
    wave_sync();
    int pos = ox_first(o, (int)excl, after);
    const OxStep st = ox_step(o);
#pragma unroll
    for (int i = 0; i < C; ++i)
        if (kp[i]) {
            A[pos] = (uint16_t)x2.gene(i);
            pos = ox_next(st, pos);
        }
    wave_sync();
}

// Longer rows: the same passes over chunks of VC vectors, read from HBM
// (L2) once per pass, with the marks in a row of their own.
template <int VC>
__device__ __forceinline__ void ox_group_long(uint16_t* A, uint16_t* M, const uint16_t* P1, const uint16_t* P2,
                                              const OxCut& o, int vpl, int g, int k, int S, bool active)
{
    const int nv = (o.n + 7) >> 3, v0 = k * vpl, v1 = v0 + vpl;
    u32x4 x[VC];
    uint32_t keep[VC];
    auto lim = [&](int v) { return active ? o.n - 8 * v : 0; };
    for (int v = v0; v < v1; v += VC) {
        const int c = v1 - v < VC ? v1 - v : VC;
        ox_load<VC>(x, P1, v, c, nv);
        ox_mark<VC>(M, x, o, v, c, lim(v));
    }
    wave_sync();
    int cnt = 0;
    for (int v = v0; v < v1; v += VC) {
        const int c = v1 - v < VC ? v1 - v : VC;
        ox_load<VC>(x, P2, v, c, nv);
        cnt += ox_keep<VC>(M, x, keep, o, v, c, lim(v));
    }
    int pos = ox_group_first(o, cnt, g, S);
    for (int v = v0; v < v1; v += VC) {
        const int c = v1 - v < VC ? v1 - v : VC;
        ox_load<VC>(x, P1, v, c, nv);
        ox_place1<VC>(A, x, o, v, c, lim(v));
    }
    wave_sync();
    for (int v = v0; v < v1; v += VC) {
        const int c = v1 - v < VC ? v1 - v : VC;
        ox_load<VC>(x, P2, v, c, nv);
        ox_keep<VC>(M, x, keep, o, v, c, lim(v));
        pos = ox_place2<VC>(A, x, keep, o, c, pos);
    }
    wave_sync();
}

// The whole wave on a row of more than 1024 genes: up to 2048 in registers,
// above that in passes with the marks in a row of their own (A + n_pad).  Not
// as a function of its own: each call saved its registers to scratch memory,
// which was most of it (147456 individuals, one lane per chromosome: 1500 jobs
// of one stage 737 us with three LDS rows, 854 in passes behind a call, 631
// now; 2000 jobs of three stages 1706, 1183, 973).
__device__ __forceinline__ void ox_wave_long(uint16_t* A, int n_pad, const uint16_t* P1, const uint16_t* P2,
                                             const OxCut& o, int lane)
{
    const int vpl = ox_vectors(o.n, kWave);
    if (n_pad <= 2048) ox_group_regs<4>(A, P1, P2, o, vpl, 0, lane, kWave, true);
    else ox_group_long<2>(A, A + n_pad, P1, P2, o, vpl, 0, lane, kWave, true);
}

template <bool SMALL>   // at most kOxSmall vectors per lane
__device__ __forceinline__ void ox_group_rows(uint16_t* A, int n_pad, const uint16_t* P1, const uint16_t* P2,
                                              const OxCut& o, int g, int k, int S, bool active)
{
    const int vpl = ox_vectors(o.n, S);
    if (SMALL) {
        ox_group_regs<kOxSmall>(A, P1, P2, o, vpl, g, k, S, active);
        return;
    }
    if (vpl <= 3) ox_group_regs<3>(A, P1, P2, o, vpl, g, k, S, active);
    else if (vpl <= 7) ox_group_regs<7>(A, P1, P2, o, vpl, g, k, S, active);
    else if (vpl <= kOxVec) ox_group_regs<kOxVec>(A, P1, P2, o, vpl, g, k, S, active);
    else ox_group_long<4>(A, A + n_pad, P1, P2, o, vpl, g, k, S, active);
}

__device__ __forceinline__ void swap_genes(uint16_t* A, bool doit, int i, int j)
{
    if (doit) {
        const uint16_t x = A[i], y = A[j];
        A[i] = y;
        A[j] = x;
    }
    wave_sync();
}

// ---- cellular offspring ----------------------------------------------------
struct CellMeta {
    int mk1, mk2, a, b, mi, mj;
    bool cx, mx;
};

// Parents and draws of the child of cell `slot` at generation `gen` from
// candidate stream `sub` (sub 0 is the plain GA's stream): P1, P2 = the two
// best of (self, N, E, S, W) by (makespan, that order) in generation gen-1
// (or the selection variant of the island), then the crossover flag and
// cuts and the swap mutation's flag and positions.
struct CellPlan {
    int p1, p2;
    bool n1, n2;      // line sweep: the parent's row is already the new generation's
    CellMeta meta;
};

// Parents and draws of cell `slot` at generation `gen` (Section 4.2).  With
// sdiag >= 0 (the cell's anti-diagonal r + c in a line sweep) a neighbour on
// a lower anti-diagonal precedes the cell in row-major order, the torus's
// wrapped neighbours included, so its makespan and row are read from the
// generation being built (buffer cur ^ 1); the others and the cell itself
// from generation gen - 1.
__device__ __forceinline__ CellPlan cell_plan(const InstDesc* I, const IslandDesc* L, int slot, uint32_t sub, int gen,
                                              int cur, int sdiag = -1)
{
    const int n = I->n;
    const auto* mkp = as_global(L->mk[cur]);
    const auto* mkn = as_global(L->mk[cur ^ 1]);
    const int rows = L->rows, cols = L->cols;
    const int r = slot / cols, c = slot - r * cols;
    const int nb0 = slot;
    const int nb1 = ((r == 0) ? rows - 1 : r - 1) * cols + c;
    const int nb2 = r * cols + ((c == cols - 1) ? 0 : c + 1);
    const int nb3 = ((r == rows - 1) ? 0 : r + 1) * cols + c;
    const int nb4 = r * cols + ((c == 0) ? cols - 1 : c - 1);
    const bool sw = sdiag >= 0;
    const bool u1 = sw && r > 0, u2 = sw && c == cols - 1, u3 = sw && r == rows - 1, u4 = sw && c > 0;
    const int v0 = mkp[nb0];
    const int v1 = (u1 ? mkn : mkp)[nb1], v2 = (u2 ? mkn : mkp)[nb2];
    const int v3 = (u3 ? mkn : mkp)[nb3], v4 = (u4 ? mkn : mkp)[nb4];
    const Block4 bk = stream_block(I->seed, (uint64_t)I->inst_id, (uint32_t)L->local, (uint32_t)slot, sub,
                                   (uint32_t)gen, kCell, 0);
    int bv, bs, sv, ss;
    const int sel = L->sel;
    if (sel == 1) {
        // self + the best of (N, E, S, W) by (makespan, order)
        bv = v0;
        bs = nb0;
        sv = v1;
        ss = nb1;
        if (v2 < sv) { sv = v2; ss = nb2; }
        if (v3 < sv) { sv = v3; ss = nb3; }
        if (v4 < sv) { sv = v4; ss = nb4; }
    } else if (sel == 2) {
        // binary tournaments: draws 6 and 7 each pick two positions of the
        // neighbourhood (x / 5, x % 5 with x uniform in [0, 25)); the better
        // by (makespan, position) wins
        const int vv[5] = {v0, v1, v2, v3, v4}, nn[5] = {nb0, nb1, nb2, nb3, nb4};
        int win[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int x = (int)below(draw32(bk, 6 + t), 25u);
            const int i = x / 5, j = x - 5 * (x / 5);
            int vi = vv[0], vj = vv[0];
#pragma unroll
            for (int q = 1; q < 5; ++q) {
                vi = (i == q) ? vv[q] : vi;
                vj = (j == q) ? vv[q] : vj;
            }
            win[t] = (vj < vi || (vj == vi && j < i)) ? j : i;
        }
        bv = vv[0]; bs = nn[0]; sv = vv[0]; ss = nn[0];
#pragma unroll
        for (int q = 1; q < 5; ++q) {
            if (win[0] == q) { bv = vv[q]; bs = nn[q]; }
            if (win[1] == q) { sv = vv[q]; ss = nn[q]; }
        }
    } else {
        // the two best of (self, N, E, S, W) by (makespan, order)
        int bo = 0;
        bv = v0;
        bs = nb0;
        if (v1 < bv) { bv = v1; bs = nb1; bo = 1; }
        if (v2 < bv) { bv = v2; bs = nb2; bo = 2; }
        if (v3 < bv) { bv = v3; bs = nb3; bo = 3; }
        if (v4 < bv) { bv = v4; bs = nb4; bo = 4; }
        sv = 0x7FFFFFFF;
        ss = -1;
        if (bo != 0 && v0 < sv) { sv = v0; ss = nb0; }
        if (bo != 1 && v1 < sv) { sv = v1; ss = nb1; }
        if (bo != 2 && v2 < sv) { sv = v2; ss = nb2; }
        if (bo != 3 && v3 < sv) { sv = v3; ss = nb3; }
        if (bo != 4 && v4 < sv) { sv = v4; ss = nb4; }
        if (ss < 0) ss = nb1;   // only when every makespan is INT_MAX (never)
    }
    CellPlan pl;
    pl.p1 = bs;
    pl.p2 = ss;
    pl.n1 = (bs == nb1 && u1) || (bs == nb2 && u2) || (bs == nb3 && u3) || (bs == nb4 && u4);
    pl.n2 = (ss == nb1 && u1) || (ss == nb2 && u2) || (ss == nb3 && u3) || (ss == nb4 && u4);
    pl.meta.mk1 = bv;
    pl.meta.mk2 = sv;
    pl.meta.cx = (uint64_t)draw32(bk, 0) < L->tc;
    const int u = (int)below(draw32(bk, 1), (uint32_t)n), w = (int)below(draw32(bk, 2), (uint32_t)n);
    pl.meta.a = u < w ? u : w;
    pl.meta.b = u < w ? w : u;
    pl.meta.mx = (uint64_t)draw32(bk, 3) < L->tm;
    pl.meta.mi = (int)below(draw32(bk, 4), (uint32_t)n);
    int mj = pl.meta.mi + 1 + (int)below(draw32(bk, 5), (uint32_t)(n - 1));
    if (mj >= n) mj -= n;
    pl.meta.mj = mj;
    return pl;
}

// The segment of a crossover with cuts a <= b; without one the child is
// parent 1: the whole row.
__device__ __forceinline__ OxCut ox_cut(int n, bool cx, int a, int b, bool rev1, bool rev2)
{
    OxCut o;
    o.n = n;
    o.a = cx ? a : 0;
    o.len = cx ? b - a : n - 1;
    o.rev1 = rev1;
    o.rev2 = rev2;
    return o;
}

// The child of cell `slot` (cell_plan) built in the group's LDS row A: order
// crossover of P1 and P2, then the swap mutation.
__device__ __forceinline__ CellMeta cellular_offspring(const InstDesc* I, const IslandDesc* L, int slot, uint32_t sub,
                                                   int gen, int cur, uint16_t* A, int g, int k, int S, bool active)
{
    const int n = I->n, n_pad = I->n_pad;
    const CellPlan pl = cell_plan(I, L, slot, sub, gen, cur);
    const uint16_t* gp = L->genes[cur];
    ox_group_rows<false>(A, n_pad, gp + (size_t)pl.p1 * n_pad, gp + (size_t)pl.p2 * n_pad,
                  ox_cut(n, pl.meta.cx, pl.meta.a, pl.meta.b, false, false), g, k, S, active);
    swap_genes(A, pl.meta.mx && active && k == 0, pl.meta.mi, pl.meta.mj);
    return pl.meta;
}

// Draws of the pseudo island's slot `slot` at generation `gen` (Section
// 4.1, complementary parents): X = the better of its pair (2q, 2q + 1) by
// (makespan, slot) in generation gen-1; the even slot gets OX(X, Y), the odd
// one OX(Y, X) with Y = reverse(X), both with the pair's cuts; each child has
// its own mutation draws.
struct PairPlan {
    int xs;
    bool odd, cx, mx;
    int a, b, mi, mj;
};

__device__ __forceinline__ PairPlan pair_plan(const InstDesc* I, const IslandDesc* L, int slot, int gen, int cur)
{
    const int n = I->n;
    const auto* mkp = as_global(L->mk[cur]);
    const int q = slot >> 1;
    PairPlan pl;
    pl.odd = slot & 1;
    pl.xs = (mkp[2 * q] <= mkp[2 * q + 1]) ? 2 * q : 2 * q + 1;
    const uint64_t seed = I->seed, iid = (uint64_t)I->inst_id;
    const uint32_t isl_local = (uint32_t)L->local;
    const Block4 b0 = stream_block(seed, iid, isl_local, (uint32_t)q, 0, (uint32_t)gen, kPair, 0);
    const Block4 b1 = stream_block(seed, iid, isl_local, (uint32_t)q, 0, (uint32_t)gen, kPair, 1);
    pl.cx = (uint64_t)draw32(b0, 0) < L->tc;
    const int u = (int)below(draw32(b0, 1), (uint32_t)n), w = (int)below(draw32(b0, 2), (uint32_t)n);
    pl.a = u < w ? u : w;
    pl.b = u < w ? w : u;
    const uint32_t dm = pl.odd ? draw32(b0, 6) : draw32(b0, 3);
    const uint32_t di = pl.odd ? draw32(b0, 7) : draw32(b0, 4);
    const uint32_t dj = pl.odd ? draw32(b1, 0) : draw32(b0, 5);
    pl.mx = (uint64_t)dm < L->tm;
    pl.mi = (int)below(di, (uint32_t)n);
    int mj = pl.mi + 1 + (int)below(dj, (uint32_t)(n - 1));
    if (mj >= n) mj -= n;
    pl.mj = mj;
    return pl;
}

// Pre-screen input of the chromosome in A (the group's S lanes): lane k sums
// stage k's processing times over each of B = floor(240 / S) position
// buckets (position t is in bucket floor(t B / n)) and writes
// bf16(fp32(load * B) / fp32(P_k)) at index b * S + k; indices B*S .. 239 and
// 252 .. 255 are 0; 240 .. 251 hold the scalars (parents' makespans / LB,
// cut points / n, crossover flag, mutation flag, swap positions / n, LB / E,
// n / 1000, S / 20, sum m / (6 S)).  Every ratio is one correctly rounded
// FP32 division.
template <typename PT>
__device__ __forceinline__ void features_group(const uint16_t* A, const PT* pT, const InstDesc* I, int k, bool active,
                                               const CellMeta& cm, uint16_t* out)
{
    if (!active) return;
    const int n = I->n, S = I->S, n_pad = I->n_pad;
    const int B = 240 / S;
    const PT* prow = pT + (size_t)k * pt_stride<PT>(n_pad);
    const float Pk = (float)I->Pk[k];
    int t = 0;
    for (int bb = 0; bb < B; ++bb) {
        const int tend = ((bb + 1) * n + B - 1) / B;
        uint32_t load = 0;
#pragma unroll 8
        for (; t < tend; ++t) load += prow[A[t]];
        out[bb * S + k] = f32_to_bf16(__fdiv_rn((float)((uint64_t)load * (uint64_t)B), Pk));
    }
    const float fn = (float)n, fLB = (float)I->LB;
    for (int e = B * S + k; e < kFeat; e += S) {
        float v = 0.f;
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
        out[e] = f32_to_bf16(v);
    }
}

// Generation 0's chromosome of `slot` in row A of a group of S lanes (lane
// k): Fisher-Yates from the INIT stream; a pseudo pair is a permutation (even
// slot) and its reversal (odd slot).  The swap partners pass through
// `scratch`, a row of n_pad entries in HBM (the slot's row of the other
// generation parity).
__device__ __forceinline__ void initial_row(const InstDesc* I, const IslandDesc* L, int slot, uint16_t* A,
                                            uint16_t* scratch, int k, int S, bool active)
{
    const int n = I->n;
    const int fy_slot = (L->kind == 0) ? slot : (slot >> 1);
    const bool rev = (L->kind == 1) && (slot & 1);
    const int nblk = (n - 1 + 7) / 8;
    u32x4* s4 = reinterpret_cast<u32x4*>(scratch);
    if (active) {
        for (int blk = k; blk < nblk; blk += S) {
            const Block4 bb = stream_block(I->seed, (uint64_t)I->inst_id, (uint32_t)L->local, (uint32_t)fy_slot, 0, 0,
                                           kInit, (uint32_t)blk);
            uint32_t j[8];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const int idx = blk * 8 + d;
                j[d] = idx < n - 1 ? below(draw32(bb, d), (uint32_t)(n - idx)) : 0u;
            }
            as_global(s4)[blk] = u32x4{j[0] | (j[1] << 16), j[2] | (j[3] << 16), j[4] | (j[5] << 16), j[6] | (j[7] << 16)};
        }
        for (int t = k; t < n; t += S) A[t] = (uint16_t)t;
    }
    // the partners are read back by another lane of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (active && k == 0 && nblk > 0) {
        u32x4 nx = as_global((const u32x4*)s4)[0];
        for (int blk = 0; blk < nblk; ++blk) {
            const u32x4 w = nx;
            if (blk + 1 < nblk) nx = as_global((const u32x4*)s4)[blk + 1];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const int i = n - 1 - (blk * 8 + d);
                if (i >= 1) {
                    const uint32_t j = ox_gene(w, d);
                    const uint16_t x = A[i], y = A[j];
                    A[i] = y;
                    A[j] = x;
                }
            }
        }
    }
    wave_sync();
    if (active && rev) {
        for (int t = k; t < n / 2; t += S) {
            const uint16_t x = A[t], y = A[n - 1 - t];
            A[t] = y;
            A[n - 1 - t] = x;
        }
    }
    wave_sync();
}

// The chromosome of `slot` at generation `gen`, built in row A of a group of
// S lanes (lane k): generation 0 (mode 1) draws it; a cellular cell gets the
// child of its neighbourhood's two best from candidate stream `sub`; a pseudo
// slot gets its pair's complementary child.
template <bool SMALL>
__device__ __forceinline__ CellMeta make_child(const InstDesc* I, const IslandDesc* L, int slot, uint32_t sub,
                                               int gen, int cur, int mode, uint16_t* A, int g, int k, int S,
                                               bool active)
{
    const int n = I->n, n_pad = I->n_pad;
    CellMeta meta{};
    if (mode == 1) {
        initial_row(I, L, slot, A, L->genes[cur] + (size_t)slot * n_pad, k, S, active);
        return meta;
    }
    int p1, p2, mi, mj;
    bool mx;
    OxCut o;
    if (L->kind == 0) {
        const CellPlan pl = cell_plan(I, L, slot, sub, gen, cur);
        meta = pl.meta;
        p1 = pl.p1;
        p2 = pl.p2;
        o = ox_cut(n, meta.cx, meta.a, meta.b, false, false);
        mx = meta.mx;
        mi = meta.mi;
        mj = meta.mj;
    } else {
        // pseudo: X = better of the pair, Y = reverse(X); even slot gets
        // OX(X, Y), odd slot OX(Y, X), with shared cut points.
        const PairPlan pl = pair_plan(I, L, slot, gen, cur);
        p1 = p2 = pl.xs;
        o = ox_cut(n, pl.cx, pl.a, pl.b, pl.odd, !pl.odd);
        mx = pl.mx;
        mi = pl.mi;
        mj = pl.mj;
    }
    const uint16_t* gp = L->genes[cur];
    ox_group_rows<SMALL>(A, n_pad, gp + (size_t)p1 * n_pad, gp + (size_t)p2 * n_pad, o, g, k, S, active);
    swap_genes(A, mx && active && k == 0, mi, mj);
    return meta;
}

// ---- best-ever records ------------------------------------------------------
// Folds generation g into the best-ever records of every instance: the
// minimum (makespan, slot) key of each island, ties on makespan to the lowest
// island; a strictly better makespan replaces the record and copies the
// permutation from generation g's population.  Resets the islands' keys of
// g's parity for generation g + 2.  Run by one workgroup; s_tmp holds
// 3 * blockDim.x ints (fold_lds_bytes).
__host__ __device__ inline size_t fold_lds_bytes(int threads) { return (size_t)3 * sizeof(int) * threads; }

__device__ void fold_best(const InstDesc* __restrict__ insts, const IslandDesc* __restrict__ isls, int n_inst,
                          int g, Control* ctl, int* s_tmp, int group)
{
    const int par = g & 1;
    int* s_imp = s_tmp;
    int* s_isl = s_imp + blockDim.x;
    int* s_slot = s_isl + blockDim.x;
    for (int base = 0; base < n_inst; base += blockDim.x) {
        const int ii = base + threadIdx.x;
        int imp = 0, bisl = -1, bslot = -1;
        if (ii < n_inst) {
            const InstDesc* J = insts + ii;
            unsigned long long bkey = ~0ull;
            for (int x = 0; x < J->n_islands; ++x) {
                if (isls[J->island0 + x].chain != group) continue;
                unsigned long long* gk = isls[J->island0 + x].genkey + par;
                const unsigned long long v = __hip_atomic_load(gk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (bisl < 0 || (v >> 32) < (bkey >> 32)) {
                    bkey = v;
                    bisl = x;
                }
                __hip_atomic_store(gk, ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (bisl >= 0) {
                const int slot = isls[J->island0 + bisl].rec;
                int* rec = J->best_rec + 4 * slot;
                bslot = (int)(bkey & 0xFFFFFFFFu);
                const int bmk = (int)(bkey >> 32);
                if (bmk < rec[0]) {
                    rec[0] = bmk;
                    rec[1] = g;
                    rec[2] = bisl;
                    rec[3] = bslot;
                    imp = 1;
                }
            }
        }
        s_imp[threadIdx.x] = imp;
        s_isl[threadIdx.x] = bisl;
        s_slot[threadIdx.x] = bslot;
        __syncthreads();
        const int lim = (n_inst - base) < (int)blockDim.x ? (n_inst - base) : (int)blockDim.x;
        for (int t = 0; t < lim; ++t) {
            if (!s_imp[t]) continue;
            const InstDesc* J = insts + base + t;
            const IslandDesc* X = isls + J->island0 + s_isl[t];
            const uint4* s4 = reinterpret_cast<const uint4*>(X->genes[par] + (size_t)s_slot[t] * J->n_pad);
            uint4* d4 = reinterpret_cast<uint4*>(J->best_perm + (size_t)X->rec * J->n_pad);
            for (int v = threadIdx.x; v < (J->n_pad >> 3); v += blockDim.x) d4[v] = s4[v];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) ctl->best_gen[group] = g;
}

// Folds the completed generation into the best-ever records of every fold
// group that has not done so yet (one workgroup).
static __global__ void __launch_bounds__(256) k_best_flush(const InstDesc* __restrict__ insts,
                                                    const IslandDesc* __restrict__ isls, Control* ctl, int n_inst,
                                                    int groups)
{
    __shared__ int s_tmp[3 * 256];
    const int g = completed_gen(ctl);
    for (int group = 0; group < groups; ++group)
        if (ctl->best_gen[group] < g) fold_best(insts, isls, n_inst, g, ctl, s_tmp, group);
}

// ---- one generation (mode 0) or generation 0 (mode 1) of every island -----
template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3))) k_generation(const InstDesc* __restrict__ insts,
                                                    const IslandDesc* __restrict__ isls,
                                                    const WorkItem* __restrict__ work, Control* ctl, int n_inst,
                                                    int mode, int cnt_off, int has_extra)
{
    // generation number from this workgroup's launch count (generation 0 has none)
    __shared__ int s_gen;
    if (threadIdx.x == 0) {
        int gg = 0;
        if (mode == 0) {
            int* cnt = ctl->counts + cnt_off + blockIdx.x;
            const int t = *cnt;
            *cnt = t + 1;
            gg = ctl->base + 1 + t;
        }
        s_gen = gg;
    }
    // the workgroup after the work items folds the previous generation into
    // the best-ever records while the others run this one
    // has_extra = 1 + group: the last workgroup folds that fold group's
    // previous generation
    if (has_extra && blockIdx.x == gridDim.x - 1) {
        __syncthreads();
        const int prev = s_gen - 1, group = has_extra - 1;
        if (ctl->best_gen[group] < prev)
            fold_best(insts, isls, n_inst, prev, ctl, reinterpret_cast<int*>(ffs_smem), group);
        return;
    }
    // When every workgroup is resident at once, give each XCD (the hardware
    // places workgroup b on XCD b % 8) a contiguous run of work items, so
    // that neighbouring cells share an L2; larger grids keep the
    // largest-first order.
    const int nw = (int)gridDim.x - (has_extra ? 1 : 0);
    int widx = (int)blockIdx.x;
    if (nw <= 256) {
        const int per = (nw + 7) / 8, full = nw - 8 * (per - 1);
        const int xcd = widx & 7, rnk = widx >> 3;
        widx = (xcd < full) ? xcd * per + rnk : full * per + (xcd - full) * (per - 1) + rnk;
    }
    const WorkItem wi = work[widx];
    const InstDesc* I = insts + wi.inst;
    const IslandDesc* L = isls + wi.island;
    if (mode == 0 && L->sweep) return;   // line-sweep islands have launches of their own
    const int S = I->S, n_pad = I->n_pad, G = I->G;

    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int gen = s_gen;
    const int cur = (gen + 1) & 1, nxt = gen & 1;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int stride = group_stride(I->n, n_pad, S);
    uint16_t* gbase = reinterpret_cast<uint16_t*>(ffs_smem + pt_lds_bytes<PT>(S, n_pad)) + (size_t)wave * G * stride;
    const int g = lane / S, k = lane - g * S;
    const int local = wave * G + g;
    const bool active = (g < G) && (local < wi.count);
    uint16_t* A = gbase + (size_t)(active ? g : 0) * stride;
    // the row's padding is zero (readers of a row look up its genes unmasked)
    if (active)
        for (int t = I->n + k; t < n_pad; t += S) A[t] = 0;
    const int slot = wi.slot0 + (active ? local : 0);

    const bool screened = mode == 0 && L->kind == 0 && I->surr_k > 1 && gen > I->surr_warmup;
    const uint32_t sub = screened ? (uint32_t)I->surr_choice[L->cell_base + slot] : 0u;
    const CellMeta meta = make_child<false>(I, L, slot, sub, gen, cur, mode, A, g, k, S, active);

    // waves past the work item's chromosomes have nothing to decode
    const int groups = wi.count - wave * G;
    uint32_t cm = 0u;
    if (groups > 0)
        cm = decode_pipelined<MMAX, PT>(
            pipe_lane<PT>(gbase, stride, pT, n_pad, lane, g, k, S, G, groups), I, active);
    const int src = active ? (g * S + S - 1) : lane;
    const int cmg = __shfl((int)cm, src, 64);

    unsigned long long wkey = ~0ull;
    if (active) {
        uint16_t* dstrow = L->genes[nxt] + (size_t)slot * n_pad;
        int mk_new;
        if (mode == 1 || L->kind == 1) {
            mk_new = cmg;
            row_l2g(dstrow, A, n_pad, k, S);
        } else {
            const int mk_old = as_global(L->mk[cur])[slot];
            const bool rep = cmg < mk_old;
            mk_new = rep ? cmg : mk_old;
            if (rep) {
                row_l2g(dstrow, A, n_pad, k, S);
            } else {
                row_g2g(dstrow, L->genes[cur] + (size_t)slot * n_pad, n_pad, k, S);
            }
        }
        if (k == 0) L->mk[nxt][slot] = mk_new;
        wkey = (k == 0) ? (((unsigned long long)(unsigned)mk_new << 32) | (unsigned)slot) : ~0ull;
    }
    if (mode == 0 && L->kind == 0 && I->surr_k > 1) {
        // training data of the pre-screen: the decoded child and its exact
        // makespan; a screened child's features were computed when it was scored
        const int cell = L->cell_base + slot;
        const long long ri = ((long long)(gen - 1) * I->n_cells + cell) % I->ring_size;
        uint16_t* dst = I->ring_X + ri * kFeat;
        if (gen > I->surr_warmup) {
            if (active) {
                const uint4* s4 = reinterpret_cast<const uint4*>(
                    I->surr_X + ((size_t)cell * I->surr_k + (size_t)I->surr_choice[cell]) * kFeat);
                uint4* d4 = reinterpret_cast<uint4*>(dst);
                for (int v = k; v < kFeat / 8; v += S) d4[v] = s4[v];
            }
        } else {
            features_group<PT>(A, pT, I, k, active, meta, dst);
        }
        if (active && k == 0) I->ring_T[ri] = __fdiv_rn((float)(cmg - I->LB), (float)I->LB);
    }
    // island minimum of (makespan, slot): wave reduction, then one atomic per workgroup
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(wkey, off, 64);
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

// ---- a migration epoch of small islands in one launch ------------------------
// `gens` generations of islands that are one workgroup's work each (rows of at
// most kOxSmall vectors per lane, kKeyIdx).  Islands are independent between
// migration epochs, so a workgroup needs nothing but its own barrier between
// generations; it keeps its epoch's best row and record, which k_epoch_fold
// folds afterwards.  A generation of the tiny workload (two islands of 64, 20
// jobs) is a chain of latencies: 6.1 us in here, 9.4 us with a launch of its
// own, of which the rest is the launch, the time table's way to LDS and the
// records' fold; the workload's 100 generations 1264 -> 826 us.  Longer rows
// would put the crossover's larger register tiers inside the loop (256
// registers and spills), and there a launch is a small part of a generation.
template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) k_epoch(const InstDesc* __restrict__ insts, const IslandDesc* __restrict__ isls,
                                               const WorkItem* __restrict__ work, Control* ctl, int gens)
{
    __shared__ int s_gen;
    __shared__ unsigned long long s_wmin[8];
    __shared__ int s_best[4];   // makespan, generation, slot; improved in this generation
    if (threadIdx.x == 0) {
        int* cnt = ctl->counts + blockIdx.x;
        const int t = *cnt;
        *cnt = t + gens;
        s_gen = ctl->base + 1 + t;
        s_best[0] = 0x7FFFFFFF;
    }
    const WorkItem wi = work[blockIdx.x];
    const InstDesc* I = insts + wi.inst;
    const IslandDesc* L = isls + wi.island;
    const int n = I->n, S = I->S, n_pad = I->n_pad, G = I->G, kind = L->kind;
    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int gen0 = s_gen;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int stride = group_stride(n, n_pad, S);
    uint16_t* gbase = reinterpret_cast<uint16_t*>(ffs_smem + pt_lds_bytes<PT>(S, n_pad)) + (size_t)wave * G * stride;
    const int g = lane / S, k = lane - g * S;
    const int local = wave * G + g;
    const bool active = (g < G) && (local < wi.count);
    uint16_t* A = gbase + (size_t)(active ? g : 0) * stride;
    if (active)
        for (int t = n + k; t < n_pad; t += S) A[t] = 0;   // the row's padding
    const int slot = wi.slot0 + (active ? local : 0);
    const int groups = wi.count - wave * G;
    const PipeLane<PT> pl = pipe_lane<PT>(gbase, stride, pT, n_pad, lane, g, k, S, G, groups);
    const int src = active ? (g * S + S - 1) : lane;
#pragma clang loop unroll(disable)
    for (int gen = gen0; gen < gen0 + gens; ++gen) {
        const int cur = (gen + 1) & 1, nxt = gen & 1;
        make_child<true>(I, L, slot, 0u, gen, cur, 0, A, g, k, S, active);
        uint32_t cm = 0u, cmx = 0u;
        if (groups > 0) cm = decode_pipe<MMAX, kKeyIdx, PT>(pl, I->mach, S, n, n_pad, I->jb, cmx);
        const int cmg = __shfl((int)cm, src, 64);
        unsigned long long wkey = ~0ull;
        if (active) {
            uint16_t* dstrow = L->genes[nxt] + (size_t)slot * n_pad;
            int mk_new = cmg;
            bool rep = true;
            if (kind == 0) {
                const int mk_old = as_global(L->mk[cur])[slot];
                rep = cmg < mk_old;
                mk_new = rep ? cmg : mk_old;
            }
            if (rep) row_l2g(dstrow, A, n_pad, k, S);
            else row_g2g(dstrow, L->genes[cur] + (size_t)slot * n_pad, n_pad, k, S);
            if (k == 0) {
                L->mk[nxt][slot] = mk_new;
                wkey = ((unsigned long long)(unsigned)mk_new << 32) | (unsigned)slot;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(wkey, off, 64);
            wkey = o < wkey ? o : wkey;
        }
        if (lane == 0) s_wmin[wave] = wkey;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long mn = ~0ull;
            for (int x = 0; x < (int)(blockDim.x >> 6); ++x) mn = s_wmin[x] < mn ? s_wmin[x] : mn;
            const int mk = (int)(mn >> 32);
            s_best[3] = mk < s_best[0] ? 1 : 0;
            if (s_best[3]) {
                s_best[0] = mk;
                s_best[1] = gen;
                s_best[2] = (int)(mn & 0xFFFFFFFFu);
            }
        }
        // the generation's rows, makespans and best: visible to the whole
        // workgroup from here on
        __syncthreads();
        if (s_best[3]) {
            const auto* s4 = as_global(reinterpret_cast<const u32x4*>(L->genes[nxt] + (size_t)s_best[2] * n_pad));
            auto* d4 = as_global(reinterpret_cast<u32x4*>(L->ep_perm));
            for (int v = threadIdx.x; v < (n_pad >> 3); v += blockDim.x) d4[v] = s4[v];
        }
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) L->ep_rec[q] = s_best[q];
}

// Folds an epoch's island records (k_epoch) into the best-ever records, one
// wave per instance: the least (makespan, generation, island, slot) of the
// epoch, which is the record that folding generation by generation ends with,
// if its makespan is strictly lower than the record's.  Workgroup `block` of
// those that fold; the migration's first launch carries them (k_mig_sort), and
// k_epoch_fold where nothing migrates.  Instances one after the other in a
// single workgroup took 0.8 us each, per epoch: 256 instances of 2 x 64
// individuals and 20 jobs 277 us a generation with a migration after each,
// 27 now.
__device__ __forceinline__ void epoch_fold(const InstDesc* __restrict__ insts, const IslandDesc* __restrict__ isls,
                                           Control* ctl, int n_inst, int n_work, int block)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (block == 0 && threadIdx.x == 0) {
        ctl->counts[n_work] = ctl->counts[0];   // the launch count of k_generation's folding workgroup
        ctl->best_gen[0] = completed_gen(ctl);
    }
    const int ii = block * (int)(blockDim.x >> 6) + wave;
    if (ii >= n_inst) return;
    const InstDesc* J = insts + ii;
    unsigned long long key = ~0ull;
    int isl = 0x7FFFFFFF;
    for (int x = lane; x < J->n_islands; x += 64) {
        const int* r = isls[J->island0 + x].ep_rec;
        const unsigned long long v = ((unsigned long long)(unsigned)r[0] << 32) | (unsigned)r[1];
        if (v < key) {
            key = v;
            isl = x;
        }
    }
    unsigned long long best = key;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long v = __shfl_xor(best, o, 64);
        best = v < best ? v : best;
    }
    isl = key == best ? isl : 0x7FFFFFFF;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int v = __shfl_xor(isl, o, 64);
        isl = v < isl ? v : isl;
    }
    int* rec = J->best_rec;
    if ((int)(best >> 32) >= rec[0]) return;
    const IslandDesc* L = isls + J->island0 + isl;
    const uint4* s4 = reinterpret_cast<const uint4*>(L->ep_perm);
    uint4* d4 = reinterpret_cast<uint4*>(J->best_perm);
    for (int v = lane; v < (J->n_pad >> 3); v += 64) d4[v] = s4[v];
    if (lane == 0) {
        rec[0] = (int)(best >> 32);
        rec[1] = (int)(best & 0xFFFFFFFFu);
        rec[2] = isl;
        rec[3] = L->ep_rec[2];
    }
}

static __global__ void __launch_bounds__(256) k_epoch_fold(const InstDesc* __restrict__ insts,
                                                           const IslandDesc* __restrict__ isls, Control* ctl,
                                                           int n_inst, int n_work)
{
    epoch_fold(insts, isls, ctl, n_inst, n_work, (int)blockIdx.x);
}

// ---- decode of caller-supplied permutations -------------------------------
// A group of S lanes per row.  The row's genes go to LDS as 16-bit values and
// set their bits in a bit set beside it; a row is a permutation if every
// value is in range and all n bits are set.
// LDS of one group: the row with 16 bytes of padding, then the bit set.
__host__ __device__ inline int eval_stride(int n_pad) { return n_pad + 8 + ((2 * (n_pad / 32) + 7) & ~7); }

template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) k_evaluate(const InstDesc* __restrict__ I, const int* __restrict__ perms,
                                                  int count, int* __restrict__ out, Control* ctl)
{
    const int n = I->n, S = I->S, n_pad = I->n_pad, G = I->G;
    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int wpb = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int stride = eval_stride(n_pad);
    uint16_t* gbase = reinterpret_cast<uint16_t*>(ffs_smem + pt_lds_bytes<PT>(S, n_pad)) + (size_t)wave * G * stride;
    const int g = lane / S, k = lane - g * S;
    const long long first = ((long long)blockIdx.x * wpb + wave) * G;
    if (first >= count) return;
    const long long idx = first + g;
    const bool active = (g < G) && (idx < count);
    uint16_t* A = gbase + (size_t)(active ? g : 0) * stride;
    uint32_t* W = reinterpret_cast<uint32_t*>(A + n_pad + 8);
    const int nw = (n + 31) >> 5;
    if (active)
        for (int q = k; q < nw; q += S) W[q] = 0u;
    wave_sync();
    bool bad = false;
    if (active) {
        // four values per read, sixteen in flight per lane
        constexpr int U = 4;
        const int* row = perms + idx * (long long)n;
        const row_vec_ptr r4 = (row_vec_ptr)row;
        typedef uint16_t gene_vec __attribute__((ext_vector_type(4)));
        gene_vec* a4 = reinterpret_cast<gene_vec*>(A);
        auto take = [&](int x) {
            const bool ob = (unsigned)x >= (unsigned)n;
            bad |= ob;
            if (!ob) atomicOr(&W[x >> 5], 1u << (x & 31));
            return ob ? (uint16_t)0 : (uint16_t)x;
        };
        const int n4 = n >> 2;
        for (int q0 = k; q0 < n4; q0 += U * S) {
            row_vec x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = r4[q0 + u * S < n4 ? q0 + u * S : n4 - 1];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (q0 + u * S < n4) {
                    gene_vec g;
#pragma unroll
                    for (int e = 0; e < 4; ++e) g[e] = take(x[u][e]);
                    a4[q0 + u * S] = g;
                }
        }
        for (int t = 4 * n4 + k; t < n; t += S) A[t] = take(as_global(row)[t]);
    }
    wave_sync();
    if (active)
        for (int q = k; q < nw; q += S) {
            const int left = n - 32 * q;
            bad |= W[q] != (left >= 32 ? 0xFFFFFFFFu : (1u << left) - 1u);
        }
    const uint64_t gmask = (S >= 64) ? ~0ull : ((1ull << S) - 1ull);
    const uint64_t bb = __ballot(bad && active);
    const int shift = g * S;
    const bool gbad = ((shift < 64 ? (bb >> shift) : 0ull) & gmask) != 0ull;
    const int groups = count - first < G ? (int)(count - first) : G;
    const uint32_t cm = decode_pipelined<MMAX, PT>(
        pipe_lane<PT>(gbase, stride, pT, n_pad, lane, g, k, S, G, groups), I, active);
    if (active && k == S - 1) out[idx] = gbad ? -1 : (int)cm;
    if (active && k == 0 && gbad) flag_invalid(ctl);
}

// ---- candidates of the learned pre-screen ----------------------------------
// Row q = cell * K + c: the child cell `cell` would get at the next
// generation from candidate stream c, as features (Xout[q]) and, when Tout
// is given, its exact (C - LB) / LB (the judge of the pre-screen's ranking).
template <int MMAX, typename PT>
__global__ void __launch_bounds__(512) k_candidates(const InstDesc* __restrict__ insts,
                                                    const IslandDesc* __restrict__ isls, int inst,
                                                    const Control* ctl, int Nc, uint16_t* __restrict__ Xout,
                                                    float* __restrict__ Tout)
{
    const InstDesc* I = insts + inst;
    const int S = I->S, n_pad = I->n_pad, G = I->G, K = I->surr_k;
    const int done = completed_gen(ctl);
    const int gen = done + 1, cur = done & 1;
    PT* pT = reinterpret_cast<PT*>(ffs_smem);
    stage_pt<PT>(pT, I->pT, S, n_pad);
    __syncthreads();
    const int wpb = blockDim.x >> 6;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int stride = group_stride(I->n, n_pad, S);
    uint16_t* gbase = reinterpret_cast<uint16_t*>(ffs_smem + pt_lds_bytes<PT>(S, n_pad)) + (size_t)wave * G * stride;
    const int g = lane / S, k = lane - g * S;
    const int q = (blockIdx.x * wpb + wave) * G + g;
    const bool active = (g < G) && (q < Nc);
    const int qq = active ? q : 0;
    const int cell = qq / K, c = qq - cell * K;
    const IslandDesc* L = isls + I->island0;
    int slot = 0;
    for (int x = 0; x < I->n_islands; ++x) {
        const IslandDesc* X = isls + I->island0 + x;
        if (X->kind == 0 && cell >= X->cell_base && cell < X->cell_base + X->size) {
            L = X;
            slot = cell - X->cell_base;
        }
    }
    uint16_t* A = gbase + (size_t)(active ? g : 0) * stride;
    const CellMeta meta = cellular_offspring(I, L, slot, (uint32_t)c, gen, cur, A, g, k, S, active);
    features_group<PT>(A, pT, I, k, active, meta, Xout + (size_t)qq * kFeat);
    if (Tout) {
        const int groups = Nc - (blockIdx.x * wpb + wave) * G;
        uint32_t cm = 0u;
        if (groups > 0)
            cm = decode_pipelined<MMAX, PT>(
                pipe_lane<PT>(gbase, stride, pT, n_pad, lane, g, k, S, G, groups), I, active);
        const int cmg = __shfl((int)cm, active ? (g * S + S - 1) : lane, 64);
        if (active && k == 0) Tout[q] = __fdiv_rn((float)(cmg - I->LB), (float)I->LB);
    }
}

// Parameters of the 256-512-512-1 network, one FP32 vector: W1 [512][256],
// b1 [512], W2 [512][512], b2 [512], w3 [512], b3.  Weights uniform in
// +-sqrt(6 / fan_in) from the MLP_INIT stream (slot = tensor index, draw =
// element index), biases 0; Adam moments 0.
constexpr int kP_W1 = 0, kP_b1 = 131072, kP_W2 = 131584, kP_b2 = 393728, kP_w3 = 394240, kP_b3 = 394752;
constexpr int kParams = 394753;

static __global__ void __launch_bounds__(256) k_mlp_init(uint64_t seed, uint64_t inst, float* __restrict__ w,
                                                  uint16_t* __restrict__ wb, float* __restrict__ m,
                                                  float* __restrict__ v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kParams) return;
    int tensor, elem, fan_in;
    if (i < kP_b1) { tensor = 0; elem = i; fan_in = 256; }
    else if (i < kP_W2) { tensor = 1; elem = i - kP_b1; fan_in = 0; }
    else if (i < kP_b2) { tensor = 2; elem = i - kP_W2; fan_in = 512; }
    else if (i < kP_w3) { tensor = 3; elem = i - kP_b2; fan_in = 0; }
    else if (i < kP_b3) { tensor = 4; elem = i - kP_w3; fan_in = 512; }
    else { tensor = 5; elem = 0; fan_in = 0; }
    float x = 0.f;
    if (fan_in > 0) {
        const Block4 b = stream_block(seed, inst, 0, (uint32_t)tensor, 0, 0, kMlpInit, (uint32_t)(elem >> 3));
        const uint64_t word = b.w[(elem & 7) >> 1];
        const uint32_t u = (elem & 1) ? (uint32_t)(word >> 32) : (uint32_t)word;
        const float f = ((float)(u >> 8) + 0.5f) * 5.9604644775390625e-08f;   // (0, 1), 2^-24 steps
        x = (2.f * f - 1.f) * sqrtf(6.f / (float)fan_in);
    }
    w[i] = x;
    wb[i] = f32_to_bf16(x);
    m[i] = 0.f;
    v[i] = 0.f;
}

// Minibatch rows of the training step after the last completed generation
// g: uniform over the filled part of the replay ring (min(g * cells, ring)
// rows), from the MLP_BATCH stream of step g (draw r -> row r).  The
// generation comes from the control block, so a captured graph replays it.
static __global__ void __launch_bounds__(256) k_batch_idx(uint64_t seed, uint64_t inst, const Control* __restrict__ ctl,
                                                   int cells, int ring, int rows, int* __restrict__ idx)
{
    const int blk = blockIdx.x * blockDim.x + threadIdx.x;
    if (blk * 8 >= rows) return;
    const int gen = completed_gen(ctl);
    const long long f = (long long)gen * cells;
    const uint32_t filled = (uint32_t)(f < ring ? f : ring);
    const Block4 b = stream_block(seed, inst, 0, 0, 0, (uint32_t)gen, kMlpBatch, (uint32_t)blk);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int r = blk * 8 + d;
        if (r < rows) idx[r] = (int)below(draw32(b, d), filled);
    }
}

static __global__ void __launch_bounds__(256) k_zero_u32(uint32_t* __restrict__ p, size_t count)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// ---- migration (paper Section 4.3) -----------------------------------------
__device__ __forceinline__ bool migrating_now(const InstDesc* I, int inst, int gen, int force_inst)
{
    if (force_inst >= 0) return inst == force_inst;
    return I->interval > 0 && gen > 0 && (gen % I->interval) == 0;
}

static __global__ void __launch_bounds__(256) k_mig_minmax(const InstDesc* __restrict__ insts,
                                                    const IslandDesc* __restrict__ isls, const Control* ctl,
                                                    int force_inst)
{
    const IslandDesc* L = isls + blockIdx.x;
    const InstDesc* I = insts + L->inst;
    const int gen = completed_gen(ctl);
    if (!migrating_now(I, L->inst, gen, force_inst) || I->topology != 1) return;
    const int* mk = L->mk[gen & 1];
    unsigned long long mn = ~0ull, mx = 0ull;
    for (int s = threadIdx.x; s < L->size; s += blockDim.x) {
        const unsigned long long v = ((unsigned long long)(unsigned)mk[s] << 32) | (unsigned)s;
        mn = v < mn ? v : mn;
        mx = v > mx ? v : mx;
    }
    __shared__ unsigned long long smn[256], smx[256];
    smn[threadIdx.x] = mn;
    smx[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            smn[threadIdx.x] = smn[threadIdx.x + w] < smn[threadIdx.x] ? smn[threadIdx.x + w] : smn[threadIdx.x];
            smx[threadIdx.x] = smx[threadIdx.x + w] > smx[threadIdx.x] ? smx[threadIdx.x + w] : smx[threadIdx.x];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        L->minmax[0] = smn[0];
        L->minmax[1] = smx[0];
    }
}

// ring c0, p0, c1, p1, ...: island x receives its predecessor's best into its worst slot
static __global__ void __launch_bounds__(256) k_mig_ring(const InstDesc* __restrict__ insts,
                                                  const IslandDesc* __restrict__ isls, const Control* ctl,
                                                  int force_inst)
{
    const IslandDesc* L = isls + blockIdx.x;
    const InstDesc* I = insts + L->inst;
    const int gen = completed_gen(ctl);
    if (!migrating_now(I, L->inst, gen, force_inst) || I->topology != 1) return;
    const int H = I->n_islands / 2;
    if (H == 0) return;
    const int l = L->local;
    const int pos = (l < H) ? 2 * l : 2 * (l - H) + 1;
    const int pp = (pos == 0) ? 2 * H - 1 : pos - 1;
    const int pl = (pp & 1) ? H + (pp >> 1) : (pp >> 1);
    const IslandDesc* P = isls + I->island0 + pl;
    const int par = gen & 1;
    const int ss = (int)(P->minmax[0] & 0xFFFFFFFFu);
    const int ds = (int)(L->minmax[1] & 0xFFFFFFFFu);
    const int n_pad = I->n_pad;
    const uint4* s4 = reinterpret_cast<const uint4*>(P->genes[par] + (size_t)ss * n_pad);
    uint4* d4 = reinterpret_cast<uint4*>(L->genes[par] + (size_t)ds * n_pad);
    for (int v = threadIdx.x; v < (n_pad >> 3); v += blockDim.x) d4[v] = s4[v];
    if (threadIdx.x == 0) L->mk[par][ds] = P->mk[par][ss];
}

// Stable sort of one island's slots by makespan (ties keep slot order): a
// least-significant-digit-first radix sort over the bits of (makespan -
// island minimum), two bits per pass.  1024 threads hold R = max(1, P/1024)
// items each in striped order (item i = r * 1024 + thread); per pass, a wave
// ballot per digit value and the per-(digit, r, wave) counts, prefixed in
// that order, give every item its place; a pass is three block barriers, and
// an island whose makespans span 2^b values needs ceil(b / 2) passes.
// Padding items (i >= size) carry all ones and stay at the end.
// Islands of at most kRankMax slots need no passes: every item's place is the
// count of the items before it, taken by the threads / size lanes that share
// the item.  For 64 slots the sort took 11.6 us by passes and takes 4.6 us
// by counting.  At 256 a lane compares 64 items, which is still below one pass;
// the compares grow with the square of the size.
// Where the islands are few, larger ones are counted too, over gridDim.y
// workgroups of kRankItems slots each that would otherwise idle: two islands
// of 4096 slots take 8.0 us instead of 21 by passes on a workgroup each.
constexpr int kRankMax = 256;
constexpr int kRankItems = 32;
constexpr int kRankSplitMax = 4096;   // their keys are 32 KB of LDS
constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortRMax = 16;
constexpr int kSortDigits = 4;   // two bits per pass
constexpr int kSortEnt = kSortDigits * kSortRMax * kSortWaves;   // counts per pass, at most

__host__ __device__ inline size_t sort_lds_bytes(int R)
{
    return (size_t)R * kSortThreads * (sizeof(uint32_t) + sizeof(uint16_t)) +
           (size_t)2 * kSortEnt * sizeof(uint32_t) + (size_t)2 * kSortWaves * sizeof(uint32_t);
}
// the counted islands' keys fit into it
static_assert(kRankSplitMax / kSortThreads * kSortThreads * 2 <= 2 * kSortEnt * 4 + 2 * kSortWaves * 4, "8 bytes a slot");

static __global__ void __launch_bounds__(kSortThreads) k_mig_sort(const InstDesc* __restrict__ insts,
                                                           const IslandDesc* __restrict__ isls, Control* ctl,
                                                           int force_inst, int only_inst, int fold_inst, int n_work)
{
    // after a launch of k_epoch: the workgroups past the islands fold its records
    if (fold_inst > 0) {
        const int sorts = (int)gridDim.x - (fold_inst + kSortWaves - 1) / kSortWaves;
        if ((int)blockIdx.x >= sorts) {
            if (blockIdx.y == 0) epoch_fold(insts, isls, ctl, fold_inst, n_work, (int)blockIdx.x - sorts);
            return;
        }
    }
    const IslandDesc* L = isls + blockIdx.x;
    const InstDesc* I = insts + L->inst;
    const int gen = completed_gen(ctl);
    if (only_inst >= 0 && L->inst != only_inst) return;
    if (!migrating_now(I, L->inst, gen, force_inst)) return;
    const int N = L->size;
    int R = 1;
    while (R * kSortThreads < N) R <<= 1;
    const int P = R * kSortThreads;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    uint32_t* dbuf = reinterpret_cast<uint32_t*>(ffs_smem);
    uint16_t* sbuf = reinterpret_cast<uint16_t*>(dbuf + P);
    uint32_t* zcnt = reinterpret_cast<uint32_t*>(sbuf + P);      // [digit][r][wave] counts
    uint32_t* zpre = zcnt + kSortEnt;                            // their exclusive prefix, same order
    uint32_t* misc = zpre + kSortEnt;                            // [0..15] wave minima, [16..31] maxima
    const int* mk = L->mk[gen & 1];
    if (gridDim.y > 1 || N <= kRankMax) {
        int sh = 2, i0 = 0;   // 2^sh lanes per item, the workgroup's first item
        if (gridDim.y > 1) {
            static_assert(kSortThreads >> 5 == kRankItems, "32 lanes per item");
            sh = 5;
            i0 = (int)blockIdx.y * kRankItems;
            if (i0 >= N) return;
        } else {
            while (sh < 6 && (N << (sh + 1)) <= kSortThreads) ++sh;
        }
        unsigned long long* key = reinterpret_cast<unsigned long long*>(ffs_smem);
        for (int j = t; j < N; j += kSortThreads) key[j] = ((unsigned long long)(unsigned)mk[j] << 32) | (unsigned)j;
        __syncthreads();
        const int i = i0 + (t >> sh), part = t & ((1 << sh) - 1);
        const unsigned long long mine = key[i < N ? i : 0];
        int rank = 0;
#pragma unroll 8
        for (int j = part; j < N; j += 1 << sh) rank += key[j] < mine ? 1 : 0;
        for (int o = 1; o < (1 << sh); o <<= 1) rank += __shfl_xor(rank, o, 64);
        if (i < N && part == 0) {
            L->sorted[rank] = i;
            if (rank == 0) L->sortbest[0] = (int)(mine >> 32);
        }
        return;
    }

    uint32_t d[kSortRMax], sl[kSortRMax];
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
    for (int r = 0; r < kSortRMax; ++r) {
        const int i = r * kSortThreads + t;
        d[r] = 0xFFFFFFFFu;
        sl[r] = (uint32_t)i;
        if (r < R && i < N) {
            d[r] = (uint32_t)mk[i];
            mn = d[r] < mn ? d[r] : mn;
            mx = d[r] > mx ? d[r] : mx;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t a = (uint32_t)__shfl_xor((int)mn, o, 64), b = (uint32_t)__shfl_xor((int)mx, o, 64);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
    }
    if (lane == 0) {
        misc[wave] = mn;
        misc[kSortWaves + wave] = mx;
    }
    __syncthreads();
    mn = 0xFFFFFFFFu;
    mx = 0u;
    for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t a = misc[w], b = misc[kSortWaves + w];
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
    }
    // the island's best makespan, read by the migration decision (the rows
    // that the migration rewrites cannot change it afterwards)
    if (t == 0) L->sortbest[0] = (int)mn;
    const uint32_t span = mx - mn;   // N >= 1, so mn <= mx
    const int bits = span == 0u ? 0 : 32 - __clz((int)span);
#pragma unroll
    for (int r = 0; r < kSortRMax; ++r)
        if (r < R && r * kSortThreads + t < N) d[r] -= mn;

    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int nent = kSortDigits * R * kSortWaves;
    for (int bit = 0; bit < bits; bit += 2) {
        // items of each digit value per (r, wave)
#pragma unroll
        for (int r = 0; r < kSortRMax; ++r)
            if (r < R) {
                const uint32_t dg = (d[r] >> bit) & 3u;
#pragma unroll
                for (int v = 0; v < kSortDigits; ++v) {
                    const uint64_t bm = __ballot(dg == (uint32_t)v);
                    if (lane == 0) zcnt[(v * R + r) * kSortWaves + wave] = (uint32_t)__popcll(bm);
                }
            }
        __syncthreads();
        // exclusive prefix over (digit, r, wave) order, by wave 0: up to 16
        // consecutive entries per lane
        if (wave == 0) {
            const int per = (nent + 63) >> 6;
            uint32_t v[kSortEnt / 64], run = 0;
#pragma unroll
            for (int e = 0; e < kSortEnt / 64; ++e) {
                const int idx = lane * per + e;
                v[e] = (e < per && idx < nent) ? zcnt[idx] : 0u;
                run += v[e];
            }
            uint32_t incl = run;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t up = (uint32_t)__shfl_up((int)incl, o, 64);
                if (lane >= o) incl += up;
            }
            uint32_t ex = incl - run;
#pragma unroll
            for (int e = 0; e < kSortEnt / 64; ++e) {
                const int idx = lane * per + e;
                if (e < per && idx < nent) zpre[idx] = ex;
                ex += v[e];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRMax; ++r)
            if (r < R) {
                const uint32_t dg = (d[r] >> bit) & 3u;
                // the lanes of this wave whose item has the same digit
                uint64_t m = 0;
#pragma unroll
                for (int v = 0; v < kSortDigits; ++v) {
                    const uint64_t bm = __ballot(dg == (uint32_t)v);
                    m = (dg == (uint32_t)v) ? bm : m;
                }
                const uint32_t pos = zpre[(dg * R + r) * kSortWaves + wave] + (uint32_t)__popcll(m & below);
                dbuf[pos] = d[r];
                sbuf[pos] = (uint16_t)sl[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRMax; ++r)
            if (r < R) {
                d[r] = dbuf[r * kSortThreads + t];
                sl[r] = sbuf[r * kSortThreads + t];
            }
    }
    int* out = L->sorted;
#pragma unroll
    for (int r = 0; r < kSortRMax; ++r) {
        const int i = r * kSortThreads + t;
        if (r < R && i < N) out[i] = (int)sl[r];
    }
}

// adaptive penetration rule of equations (1)-(2) on one island pair, and the
// copy of the r-th best emigrant over the r-th worst immigrant.  Every block
// of the pair takes the decision from the bests that k_mig_sort recorded
// before any row moved, so all blocks agree whatever their order (when every
// immigrant slot is replaced, the immigrant's best row itself is rewritten).
constexpr int kMigRows = 32;

static __global__ void __launch_bounds__(256) k_mig_adapt(const InstDesc* __restrict__ insts,
                                                   const IslandDesc* __restrict__ isls,
                                                   const PairDesc* __restrict__ pairs, const Control* ctl,
                                                   int force_inst)
{
    const PairDesc pd = pairs[blockIdx.x];
    const InstDesc* I = insts + pd.inst;
    const int gen = completed_gen(ctl);
    if (!migrating_now(I, pd.inst, gen, force_inst)) return;
    const IslandDesc* A = isls + pd.a;
    const IslandDesc* B = isls + pd.b;
    const int par = gen & 1;
    const long long ba = A->sortbest[0], bb = B->sortbest[0];
    long long fa = I->E - ba, fb = I->E - bb;
    if (fa < 0) fa = 0;
    if (fb < 0) fb = 0;
    if (fa == fb) return;
    const unsigned long long hi = (unsigned long long)(fa > fb ? fa : fb);
    const unsigned long long lo = (unsigned long long)(fa > fb ? fb : fa);
    if (hi == 0) return;
    if (!(((hi - lo) << 32) < I->theta_T * hi)) return;
    const unsigned long long N = (unsigned long long)(A->size < B->size ? A->size : B->size);
    unsigned long long count = (N * (hi - lo) + hi - 1) / hi;
    if (count > N) count = N;
    const IslandDesc* Em = (fa > fb) ? A : B;
    const IslandDesc* Im = (fa > fb) ? B : A;
    if (blockIdx.y == 0 && threadIdx.x == 0) {
        atomicAdd((unsigned long long*)&I->counters[0], 1ull);
        atomicAdd((unsigned long long*)&I->counters[1], count);
    }
    const int r0 = blockIdx.y * kMigRows;
    const int r1 = (int)((unsigned long long)(r0 + kMigRows) < count ? (unsigned long long)(r0 + kMigRows) : count);
    if (r0 >= r1) return;
    const int n_pad = I->n_pad, nv = n_pad >> 3;
    const int rows = r1 - r0;
    for (int e = threadIdx.x; e < rows * nv; e += blockDim.x) {
        const int r = r0 + e / nv, v = e - (e / nv) * nv;
        const int ss = Em->sorted[r];
        const int ds = Im->sorted[Im->size - 1 - r];
        const uint4* s4 = reinterpret_cast<const uint4*>(Em->genes[par] + (size_t)ss * n_pad);
        uint4* d4 = reinterpret_cast<uint4*>(Im->genes[par] + (size_t)ds * n_pad);
        d4[v] = s4[v];
    }
    for (int r = r0 + threadIdx.x; r < r1; r += blockDim.x) {
        const int ss = Em->sorted[r];
        const int ds = Im->sorted[Im->size - 1 - r];
        Im->mk[par][ds] = Em->mk[par][ss];
    }
}

}  // namespace flowshop
