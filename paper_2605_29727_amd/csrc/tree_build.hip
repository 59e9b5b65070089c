// Best-first draft-tree construction on the GPU (gfx950).
//
// Sec. 3.3 / Prop. 3.3 / Algorithm 1's frontier rule at a fixed budget N: repeatedly emit the
// frontier prefix with the largest path score rho (Eq. 1), then push its best child and its next
// sibling.  Two kernels:
//   1. tb_thread_max   per slot of up to 32 marginals (one thread's share of a chunk): the largest, its place in
//                      the slot, and the second largest (one pass over [B, V], all CUs; not for small vocabularies);
//   2. tb_rank_expand  workgroup k derives from the maxima of position k a bound below which no token can be
//                      among its K best (K = min(V, N): a rank-j token is preceded by its j earlier siblings, so
//                      ranks >= N can never be emitted); a slot whose maximum reaches the bound and whose second
//                      largest does not gives its maximum as a candidate, the few other slots that reach the
//                      bound are read again; the candidates are ranked (order: probability desc, token id asc);
//                      the workgroup that finishes last runs the expansion.
// Keys are 64-bit  prob_bits << 32 | ~id  (probabilities are non-negative, so the bit pattern orders like
// the value; keys are distinct).
// rho(child) = rho(parent) * q is one fp32 multiply (never fused), the root has rho = 1.
// Frontier order: rho desc, depth asc, rank path lexicographic asc.
#include "btv_common.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef unsigned long long u64;

constexpr int MAXB = BTV_MAX_DEPTH;

// A row is seen as slots of 2^lge marginals, one per thread and chunk of 256 << lge of them: the smallest lge that leaves at
// most 16 chunks (the ranking workgroup keeps 4 slot records per thread in registers), 5 at most.  lge = 0, up to 4096
// marginals, needs no pass ahead of the ranking: every slot is one marginal, read where it is needed.  Slots of 32 for
// every vocabulary left too few of them where it is small: 5000 marginals were 256 slots, and the best 256 tokens of a
// row, which the slots' maxima are to bound, were looked for in the whole row (110 .. 217 us instead of 30).
constexpr int LGE_MAX = 5;
__device__ __forceinline__ int slot_first(int lge, int chunk, int t) { return (chunk << (8 + lge)) + t * (lge ? 4 : 1); }      // + 1024 per piece of four

__device__ __forceinline__ u64 make_key(float prob, uint32_t id)
{
    uint32_t b = __float_as_uint(prob);
    if (b == 0x80000000u) b = 0u;                  // -0.0 sorts as 0
    return ((u64)b << 32) | (u64)(0xFFFFFFFFu - id);
}

__device__ __forceinline__ uint32_t prob_bits(float p) { return __float_as_uint(p) & 0x7FFFFFFFu; }   // -0.0 counts as 0

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// Wave-wide maximum as a wave-uniform value: quad swaps, row mirrors, then the row maxima travel down the rows
// (row_bcast), so that lane 63 ends up with the maximum.  The DPP operand sits on the max instruction itself;
// lanes whose source is masked out keep their value.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    uint32_t out;
    asm volatile("s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n s_nop 1\n"
                 "v_max_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n s_nop 1\n"
                 "v_readlane_b32 %1, %0, 63"
                 : "+v"(v), "=s"(out));
    return out;
}

// Inclusive prefix sum over the wavefront on the vector ALU: shifts within the rows of 16 lanes (zeros enter from
// outside a row), then the row totals travel down the rows.
__device__ __forceinline__ int wave_incl_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);    // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);    // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);    // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);    // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

// The ranked lists travel from the workgroups that rank to the one that expands through memory, within one launch and
// between compute dies whose L2 caches do not see each other: they are written and read as relaxed device-scope
// atomics, which go through to memory, and the writer waits for its stores before it counts itself as done.
__device__ __forceinline__ void publish(u64 *top_row, int r, u64 key)        // probability bits << 32 | token
{
    __hip_atomic_store(top_row + r, (key & 0xFFFFFFFF00000000ull) | (0xFFFFFFFFu - (uint32_t)key), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr u64 NO_TOKEN = 0xFFFFFFFFull;      // the key of probability 0, token 0: what stands behind the K best of a list

// ------------------------------------------------------------------------------------------------
// Step 1: per-thread maxima.  Workgroup (chunk, row) scans the chunk's 256 << LGE elements of the row; thread t looks
// at elements 4t..4t+3 of every 1024 (its slot, elements numbered k = 4 * piece + element) and keeps the largest
// probability it saw, where it saw it, and the second largest:
// part[row][chunk][t] = { bits of the largest, bits of the second largest with k of the largest in the low 5 bits }.
// The second largest is only ever compared with a bound whose low 19 bits are zero, so the 5 bits cost nothing.
// Among equal probabilities the first one counts as the largest and the next as the second largest.
// ------------------------------------------------------------------------------------------------
struct TbCounters { int done; };            // zero between calls

// STREAM: read with the non-temporal hint.
template <int LGE, bool STREAM>
__global__ __launch_bounds__(256) void tb_thread_max(const float *marg, int V, int chunks, uint2 *part)
{
    const int tid = threadIdx.x, chunk = blockIdx.x, row = blockIdx.y;
    const float *src = marg + (size_t)row * V;
    uint32_t m1 = 0u, m2 = 0u, k1 = 0u;
    auto see = [&](uint32_t b, int k) {
        m2 = umax(m2, b < m1 ? b : m1);                          // the smaller of the newcomer and the best so far
        k1 = b > m1 ? (uint32_t)k : k1;
        m1 = umax(m1, b);
    };
    // All of a thread's loads are in flight at once: none lies behind a branch that its lanes may take apart, for which the compiler would wait each time
    // (8 round trips, 32 where the row is not aligned to 16 bytes: the whole call for 16 x 128256 marginals and 16 nodes 12.7 us, then 11.7; 16 x 128255 15.2 and 11.7).  A load of four floats needs the
    // alignment of one.  The row's last chunk, a sixteenth of the workgroups, ends with the others so: by single floats, four times as many loads,
    // it was what the launch waited for (16 x 128256 and 16 nodes 11.6 -> 11.0 us, 256 nodes 25.0 -> 24.3; 128 rows of 128256 4 us less).
    constexpr int PIECES = (1 << LGE) / 4;
    typedef float Four __attribute__((ext_vector_type(4)));
    typedef Four Four_any __attribute__((aligned(4)));
    auto load = [&](int at) {
        const Four_any *x = reinterpret_cast<const Four_any *>(src + at);
        if constexpr (STREAM) return (Four)__builtin_nontemporal_load(x);
        else return (Four)*x;
    };
    const int first = slot_first(LGE, chunk, tid);               // coalesced: a wave reads 1 KiB per load
    if ((chunk + 1) << (8 + LGE) <= V) {                         // (uniform)
        Four a[PIECES];
#pragma unroll
        for (int j = 0; j < PIECES; ++j) a[j] = load(first + j * 1024);
#pragma unroll
        for (int j = 0; j < PIECES; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) see(prob_bits(a[j][i]), 4 * j + i);
    } else {                                                     // the row's last chunk: as many loads, the last of them moved back into the row
        Four a[PIECES];
#pragma unroll
        for (int j = 0; j < PIECES; ++j) a[j] = load(min(first + j * 1024, V - 4));      // (V > 4096 here)
#pragma unroll
        for (int j = 0; j < PIECES; ++j) {
            const int past = first + j * 1024 - (V - 4);         // so many places forward
            float x[4] = { a[j][0], a[j][1], a[j][2], a[j][3] };
            if (past > 0) {                                      // (0 changes nothing)
                if (past & 1) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; x[3] = 0.f; }
                if (past & 2) { x[0] = x[2]; x[1] = x[3]; x[2] = x[3] = 0.f; }
                if (past > 3) x[0] = x[1] = x[2] = x[3] = 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) see(prob_bits(x[i]), 4 * j + i);
        }
    }
    part[((size_t)row * chunks + chunk) * 256 + tid] = make_uint2(m1, (m2 & ~31u) | k1);
}

// The ranking workgroup: its chain of short steps is bound by the issue of instructions, so the 4096 slots of a position are 4 to a thread.  With 256
// threads and 16 to a thread the whole call (16 positions x 128256 tokens, sigma 5) took 20.8 us for 64 nodes and 28.7 for 256, with 1024 19.0 and 27.1.
constexpr int RANK_T = 1024, RANK_W = RANK_T / 64, PER = 4096 / RANK_T;

constexpr int TBINS = 4096;

// ------------------------------------------------------------------------------------------------
// Step 2 (inside tb_rank_expand): the bound and the candidates of one position.  Every per-thread maximum of
// step 1 is a different token of the row, so the K-th largest of them (K <= 256 <= their number) is a lower bound
// of the row's K-th largest probability, and a tight one: it only falls short by the few tokens of the K best
// that share a slot with a better one.  The workgroup finds the 12-bit bin (sign-less float bits [30:19]: an
// eighth of a binade) that holds it from a histogram of the chunks*256 maxima and takes the lower edge of that bin
// as the bound; only slots whose maximum reaches the bound can hold candidates (about K of the chunks*256).  Where
// the slot's second largest stays below the bound, the maximum is the slot's one candidate and goes to the list
// from what step 1 recorded; the other slots, a handful, are read again, 32 elements each, and their elements at
// or above the bound join the list in LDS: K plus a few.
// Step 3, part A: the candidates are ranked by counting the candidates above each (order: probability desc, token
// id asc) and the K best go to the position's top list.  More than SELCAP candidates (heavily tied or otherwise
// degenerate probabilities): the K-th largest key of the whole row is found by radix selection, one byte of the
// key per pass (histogram of 256 bins, one wavefront), and the K keys at or above it are ranked the same way.
// ------------------------------------------------------------------------------------------------
constexpr int SELCAP = 512;
constexpr int SLOTCAP = 1024;

// One of four registers for a lane-dependent i.  The values pass through an empty asm one by one, which hides from the compiler that they are the
// elements of one array: it would turn the selects into an indexed load and move the array into scratch memory.
__device__ __forceinline__ uint32_t pick4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, int i)
{
    asm volatile("" : "+v"(x0)); asm volatile("" : "+v"(x1)); asm volatile("" : "+v"(x2)); asm volatile("" : "+v"(x3));
    const uint32_t a = (i & 2) ? x2 : x0, b = (i & 2) ? x3 : x1;
    return (i & 1) ? b : a;
}

struct alignas(16) RankLds {                // bound and ranking of one position
    union {
        alignas(16) int bins[TBINS];        // histogram of the per-thread maxima (before the candidates exist)
        struct {
            alignas(16) u64 sel[SELCAP + 64];   // the candidates (+ a place per lane for the stores that store nothing)
            uint16_t slot[SLOTCAP + 64];        // slots (chunk * 256 + thread) whose maximum reaches the bound
        };
    };
    alignas(16) int first[2048];            // rank_keys_binned: RANK_BINS bins; SELCAP keys
    alignas(16) int at[2048];
    u64 sorted[SELCAP];
    int hist[256];
    int wsum[RANK_W];
    int sel_bin;
    int nslot;
    int nsel;
    int last;
};

struct alignas(16) ExpandLds {              // the expansion
    float q[MAXB * BTV_MAX_NODES + 64];     // q[k*KP + r]: probability of rank r at position k (+ padding: q[..][r+1] is
                                            // fetched, not used, also for the last rank of the last position)
    double cost[BTV_MAX_NODES];             // adaptive budget: estimated cycle latency at budget n + 1
    uint32_t tok[MAXB * BTV_MAX_NODES];     // token ids of the same lists (fetched with q: a read from memory per emitted
                                            // node at the end of the expansion would be one more round trip)
};

// The level-by-level expansion (expand_sweep).
constexpr int SW_CAP = 4096;                // candidates of all levels together
constexpr int SW_COARSE = 512;              // bins of a score during the sweep: 4 per binade of fp32 (what is above 2 shares the last)
constexpr int SW_BINS = 2048;               // bins when the tree is put in order: 16 per binade
constexpr int SW_KEEP = 512;                // candidates that reach the last threshold (N and what shares its bin)
constexpr int SW_FANS = 12;                 // fans wider than four that one wavefront walks alone
// Probability of the greedy chain's second node from which the sweep starts from the chain.  With / without, 16 positions x 30000 tokens: one
// token of probability 0.9 x 0.93^k at position k: N = 64 1.8, N = 256 5.1 us less; 0.7: 0.9 and 2.1 less; 0.6 x 0.9^k (a second node of
// 0.32): 0.6 and 1.3 less; 0.5: 0.1 less and 0.1 more; softmax of 3 N(0, 1): 0.5 and 0.8 more.
constexpr float SW_CHAIN = 0.3f;
constexpr int SW_THIN = 96;                 // nodes up to which a level is one wavefront's work
struct alignas(16) SweepLds {
    // score bits << 32 | depth, parent and rank of a candidate (sweep_meta); a level's candidates lie in lexicographic
    // order of their rank paths.  At the end the upper half takes the candidate's place in the tree.
    uint2 cand[SW_CAP + 4];                 // (and four places for what sweep_thin writes past the last)
    alignas(16) int coarse[SW_COARSE];      // candidates per bin
    alignas(16) int hist[SW_BINS];          // candidates that are left, per bin; then those in the bins above
    int at[SW_BINS];                        // next place of the bin in `key`
    u64 key[SW_KEEP];                       // score bits << 32 | ~candidate, bin after bin
    uint16_t order[SW_KEEP];                // places in `key`, in the tree's order
    alignas(16) int cnt[2][BTV_MAX_NODES];  // children per node of a block of 256
    int wsum[4];
    int d, a, b, th;                        // where the sweep stands
    int kept;
    double wd[4];
    int n_stop;
};

struct Batch {                              // several requests in one launch (n_nodes == nullptr: one request)
    const int32_t *n_nodes;                 // [batch] budget of each request (device)
    const int32_t *q_offset;                // [batch + 1] first output row of each request (device)
    uint32_t *flag;
};

struct Adaptive {                           // Algorithm 1's early stop (cost == nullptr: fixed budget)
    const double *cost;
    double L_AR;
    double *s_best;
    uint32_t *flag;
};

// sel[0 .. n): distinct keys; those of rank < K (rank = number of keys above) go to the position's list.  A key belongs to T
// neighbouring lanes, which take the list's pairs in turn (lane `part` reads pairs part, part + T, ...), two keys per LDS read and U reads in
// flight; the shares meet by moves within the row of 16 lanes.  Every address is the trip's base plus a constant (a compare, a select and
// an address sum per read had been half of the loop's instructions), none of the reads is conditional (the compiler
// would wait for each conditional read on its own), and they run past the end of the list into zero keys, which are above nothing.
template <int T, int U>
__device__ __forceinline__ void rank_keys(u64 *sel, int n, int K, u64 *top_row, int tid)
{
    static_assert(T <= 16, "a key's lanes are of one row");
    const int i = tid / T, part = tid % T, trips = (n + 2 * T * U - 1) / (2 * T * U);      // (uniform)
    if (n + tid < trips * 2 * T * U) sel[n + tid] = 0ull;
    __syncthreads();
    const u64 mine = sel[min(i, n - 1)];
    const ulonglong2 *at = reinterpret_cast<const ulonglong2 *>(sel) + part;
    int cnt = 0;
    for (int r = 0; r < trips; ++r, at += U * T) {
        ulonglong2 kk[U];
#pragma unroll
        for (int u = 0; u < U; ++u) kk[u] = at[u * T];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cnt += kk[u].x > mine ? 1 : 0;
            cnt += kk[u].y > mine ? 1 : 0;
        }
    }
    if (T >= 2) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0xB1, 0xF, 0xF, false);     // quad_perm [1,0,3,2]
    if (T >= 4) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x4E, 0xF, 0xF, false);     // quad_perm [2,3,0,1]
    if (T >= 8) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x141, 0xF, 0xF, false);    // row_half_mirror
    if (T >= 16) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x140, 0xF, 0xF, false);   // row_mirror
    if (part == 0 && i < n && cnt < K) publish(top_row, cnt, mine);
}

// How many of keys[lo .. hi - 1] are above `mine`: eight reads in flight.
__device__ __forceinline__ int count_above(const u64 *keys, int lo, int hi, u64 mine)
{
    int n = 0;
    for (int j = lo; j < hi; j += 8) {
        u64 k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = keys[min(j + u, hi - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) n += j + u < hi && k[u] > mine ? 1 : 0;
    }
    return n;
}

// More keys: into bins of a 64th of a binade above the bound (a key's bin falls as its probability does), an
// exclusive sum of the bins from the top gives their first ranks, and a key is counted only against those of its bin: six barriers
// instead of n^2 comparisons (the whole call with 256 nodes, a confident drafter: 27.8 us by counting, 26.3 by bins).
constexpr int RANK_FEW = 256;               // vocabularies up to this size are ranked whole
constexpr int RANK_BINS = 2048, RANK_SHIFT = 17;
__device__ __forceinline__ void rank_keys_binned(const u64 *sel, u64 *sorted, int *first, int *at, int *wsum, uint32_t tau, int n, int K, u64 *top_row, int tid,
                                                 int lane, int w)
{
    static_assert(RANK_BINS == 2 * RANK_T && SELCAP <= RANK_T, "two bins and at most one key per thread");
    const u64 key = sel[min(tid, n - 1)];
    const int bin = min((int)(((uint32_t)(key >> 32) - tau) >> RANK_SHIFT), RANK_BINS - 1);
    reinterpret_cast<int2 *>(first)[tid] = make_int2(0, 0);
    __syncthreads();
    if (tid < n) atomicAdd(&first[bin], 1);
    __syncthreads();
    {                                                          // thread t: bins 2 t and 2 t + 1
        const int2 x = reinterpret_cast<const int2 *>(first)[tid];
        const int own = x.x + x.y, incl = wave_incl_scan(own), total = __builtin_amdgcn_readlane(incl, 63);
        if (lane == 0) wsum[w] = total;
        __syncthreads();
        const int others = wave_incl_scan(lane < RANK_W && lane > w ? wsum[lane & (RANK_W - 1)] : 0);
        const int up = total - incl + __builtin_amdgcn_readlane(others, RANK_W - 1);
        reinterpret_cast<int2 *>(first)[tid] = reinterpret_cast<int2 *>(at)[tid] = make_int2(up + x.y, up);
    }
    __syncthreads();
    if (tid < n) sorted[atomicAdd(&at[bin], 1)] = key;
    __syncthreads();
    if (tid < n) {
        const int lo = first[bin], rank = lo + count_above(sorted, lo, at[bin], key);
        if (rank < K) publish(top_row, rank, key);
    }
}

template <typename ForEach>
__device__ __forceinline__ u64 wave_kth_largest(ForEach for_each, int K, int *hist, int lane)
{
    u64 prefix = 0;
    int krem = K;
    for (int byte = 7; byte >= 0; --byte) {
        *reinterpret_cast<int4 *>(&hist[lane * 4]) = make_int4(0, 0, 0, 0);
        __builtin_amdgcn_wave_barrier();
        const int sh = 8 * byte;
        for_each([&](u64 key) {
            if (byte == 7 || (key >> (sh + 8)) == (prefix >> (sh + 8))) atomicAdd(&hist[(int)((key >> sh) & 255)], 1);
        });
        __builtin_amdgcn_wave_barrier();
        const int4 h = *reinterpret_cast<const int4 *>(&hist[lane * 4]);
        const int own = h.x + h.y + h.z + h.w;
        int suf = own;                         // inclusive suffix sum over the higher lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_down(suf, off);
            if (lane + off < 64) suf += o;
        }
        const int above = suf - own;
        int sel = 0, kn = 0;
        const bool here = above < krem && above + own >= krem;
        if (here) {
            int cum = above;
            const int hb[4] = { h.x, h.y, h.z, h.w };
#pragma unroll
            for (int b = 3; b >= 0; --b) {
                if (kn == 0 && cum + hb[b] >= krem) { sel = lane * 4 + b; kn = krem - cum; }
                cum += hb[b];
            }
        }
        const int srcl = __builtin_ctzll(__builtin_amdgcn_ballot_w64(here));
        sel = __builtin_amdgcn_readlane(sel, srcl);
        krem = __builtin_amdgcn_readlane(kn, srcl);
        prefix |= (u64)sel << sh;
        __builtin_amdgcn_wave_barrier();
    }
    return prefix;
}

template <typename ForEach>
__device__ __forceinline__ void wave_select(ForEach for_each, int K, int *hist, u64 *sel, int *nsel, int lane)
{
    const u64 kth = wave_kth_largest(for_each, K, hist, lane);
    if (lane == 0) *nsel = 0;
    __builtin_amdgcn_wave_barrier();
    for_each([&](u64 key) {
        if (key >= kth) {
            const int pos = atomicAdd(nsel, 1);
            if (pos < SELCAP) sel[pos] = key;                  // exactly K keys: they are distinct
        }
    });
}

// ------------------------------------------------------------------------------------------------
// Step 3, part B: the expansion, one wavefront, the frontier in registers.
// A single wavefront issues an instruction every few cycles at best, so the loop is written for few instructions
// per emitted node rather than for parallel work.
// A frontier entry stands for "the children of one node, from rank r on".  The entry for the children of node i
// lives in slot i + 1 (slot 0: the children of the root), slot s = lane s % 64 of register row s / 64; slots are
// never reused, so no search for a free one is needed and the parent of an entry is its slot number minus one.
// Per entry: key = bits(rho of rank r) + 1 (0 = empty or exhausted), rho of the parent, x = LDS address of
// q[depth-1][r] (depth and r are read back from it: KP is a power of two), and qn = q[depth-1][r+1], the
// probability of the next sibling (every lane re-reads qn after every pop: one gather, whose latency is off the
// critical path because qn is used one pop later at the earliest).  Popping an entry emits (parent, depth, r)
// and advances the entry in place to rank r + 1; the emitted node's own children become the entry of the next
// slot.  Emitted node i is kept in lane i % 64 of row i / 64 as rec = index of q[depth-1][r] | slot << 13.
// Order of emission: rho desc, depth asc, rank path lexicographic asc.  The wave maximum of the keys decides
// almost always; on ties the depth decides, then the rank paths, rebuilt by walking the parents of the tied
// entries through the emitted nodes.
// ------------------------------------------------------------------------------------------------
// ADAPT: the budget is chosen online (Sec. 3.4, Eq. 6): with Ahat summed in fp64 in emission order, the popped node
// is kept only while Ahat(N) * L_AR / C(N) strictly improves, compared as Ahat(N) * C(N*) > Ahat(N*) * C(N).
// An empty volatile asm in the body of a wave-uniform `if` keeps it a real (scalar) branch: with several register
// rows the compiler would otherwise turn the row selection into select chains over every row, which costs more
// instructions than the branches do.
#define BTV_KEEP_BRANCH() asm volatile("" ::: "memory")

template <int R, bool ADAPT>
__device__ __forceinline__ void expand_wave(ExpandLds &S, int B, int K, int KP, int N, int lane, int32_t *parent, int32_t *token,
                                            int32_t *depth, float *rho, int32_t *n_out, float *ahat, const Adaptive &ad)
{
    const float *q_s = S.q;
    const uint32_t q_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)q_s;
    const int lg = 31 - __builtin_clz((unsigned)KP);           // KP = 1 << lg
    const float qfirst = lane < B ? q_s[lane * KP] : 0.f;      // lane k: probability of the best token at position k
    uint32_t e_key[R], e_x[R], o_rec[R];
    float e_prho[R], e_qn[R], o_rho[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { e_key[r] = 0u; e_prho[r] = 0.f; e_qn[r] = 0.f; e_x[r] = q_base; o_rec[r] = 0u; o_rho[r] = 0.f; }
    if (lane == 0) {       // slot 0: the children of the root
        e_key[0] = __float_as_uint(__fmul_rn(1.0f, q_s[0])) + 1u;
        e_qn[0] = q_s[1];                                      // padding when K == 1: never used
        e_prho[0] = 1.0f;
    }
    int n = 0;
    double run_a = 1.0, best_a = 0.0, best_c = 0.0;            // Ahat so far; Ahat and cost at the best budget so far
    auto phase = [&](auto ra_c, int n_end) {
        constexpr int RA = decltype(ra_c)::value;
        while (n < n_end) {
            double c_n = 0.0;
            if (ADAPT) c_n = S.cost[n];                            // fetched early: used after the wave maximum
            uint32_t lm = e_key[0];
    #pragma unroll
            for (int r = 1; r < RA; ++r) lm = umax(lm, e_key[r]);
            const uint32_t m = wave_max_u32(lm);
            if (__builtin_expect(m == 0u, 0)) break;     // frontier empty: the lattice is exhausted
            if (ADAPT) {
                const double a_new = run_a + (double)__uint_as_float(m - 1u);
                if (__builtin_expect(!(c_n > 0.0), 0)) {           // invalid cost: stop here and tell
                    if (lane == 0) atomicOr(ad.flag, 4u);
                    break;
                }
                if (n > 0 && !(a_new * best_c > best_a * c_n)) break;   // the estimated speedup did not improve
                run_a = a_new; best_a = a_new; best_c = c_n;
            }
            u64 al[RA];
            int cnt = 0;
    #pragma unroll
            for (int r = 0; r < RA; ++r) { al[r] = __builtin_amdgcn_ballot_w64(e_key[r] == m); cnt += __builtin_popcountll(al[r]); }
            if (__builtin_expect(cnt > 1, 0)) {
                // ties on rho: shallower first (x grows with the depth) ...
                uint32_t cl = 0u;
    #pragma unroll
                for (int r = 0; r < RA; ++r)
                    if ((al[r] >> lane) & 1ull) cl = umax(cl, 0x100u - ((e_x[r] - q_base) >> (2 + lg)));
                const uint32_t cm = wave_max_u32(cl);
                cnt = 0;
    #pragma unroll
                for (int r = 0; r < RA; ++r) {
                    al[r] = __builtin_amdgcn_ballot_w64(((al[r] >> lane) & 1ull) && 0x100u - ((e_x[r] - q_base) >> (2 + lg)) == cm);
                    cnt += __builtin_popcountll(al[r]);
                }
                if (cnt > 1) {
                    // ... then the smaller rank path: one byte per position, first position in the most significant
                    // byte of word 0; the walk fetches the emitted ancestors from the lanes that hold them
                    uint32_t path[RA][4];
    #pragma unroll
                    for (int r = 0; r < RA; ++r) {
    #pragma unroll
                        for (int w = 0; w < 4; ++w) path[r][w] = 0u;
                    }
    #pragma unroll
                    for (int r = 0; r < RA; ++r) {                  // every lane walks, tied or not: the fetches are wave-wide
                        uint32_t idx = (e_x[r] - q_base) >> 2;     // index of q[depth-1][rank]
                        int node = r * 64 + lane - 1;              // the entry's parent
                        bool live = (al[r] >> lane) & 1ull;
                        while (__builtin_amdgcn_ballot_w64(live) != 0ull) {
                            const int pos = (int)(idx >> lg), sh = 24 - 8 * (pos & 3);
                            const uint32_t byte = (idx & (uint32_t)(KP - 1)) << sh;
                            if (live) {
    #pragma unroll
                                for (int w = 0; w < 4; ++w) if (w == (pos >> 2)) path[r][w] |= byte;
                            }
                            live = live && node >= 0;
                            const int src = node >= 0 ? node : 0;
                            uint32_t rec = 0u;
    #pragma unroll
                            for (int rr = 0; rr < RA; ++rr) {
                                const uint32_t got = (uint32_t)__shfl((int)o_rec[rr], src & 63);
                                if (rr == (src >> 6)) rec = got;
                            }
                            idx = rec & 0x1FFFu;
                            node = (int)(rec >> 13) - 1;
                        }
                    }
    #pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        if (cnt <= 1) break;
                        uint32_t pl = 0u;
    #pragma unroll
                        for (int r = 0; r < RA; ++r)
                            if ((al[r] >> lane) & 1ull) pl = umax(pl, ~path[r][w]);
                        const uint32_t pm = wave_max_u32(pl);
                        cnt = 0;
    #pragma unroll
                        for (int r = 0; r < RA; ++r) {
                            al[r] = __builtin_amdgcn_ballot_w64(((al[r] >> lane) & 1ull) && ~path[r][w] == pm);
                            cnt += __builtin_popcountll(al[r]);
                        }
                    }
                }
            }
            int wr = 0;
    #pragma unroll
            for (int r = RA - 1; r >= 1; --r) if (al[r] != 0ull) wr = r;
            if (al[0] != 0ull) wr = 0;
            u64 alw = al[0];
            uint32_t s_x = e_x[0];
    #pragma unroll
            for (int r = 1; r < RA; ++r)
                if (r == wr) { alw = al[r]; s_x = e_x[r]; }
            const int wl = __builtin_ctzll(alw);
            const uint32_t u_idx = (__builtin_amdgcn_readlane(s_x, wl) - q_base) >> 2;
            const float u_rho = __uint_as_float(m - 1u);
            const int d = (int)(u_idx >> lg) + 1, rank = u_idx & (uint32_t)(KP - 1);
            // emit node n into its lane
            {
                const uint32_t rec = u_idx | ((uint32_t)(wr * 64 + wl) << 13);     // parent + 1 = the entry's slot
    #pragma unroll
                for (int r = 0; r < RA; ++r)
                    if (r == (n >> 6)) {                           // wave-uniform
                        BTV_KEEP_BRANCH();
                        const bool me = lane == (n & 63);
                        o_rec[r] = me ? rec : o_rec[r];
                        o_rho[r] = me ? u_rho : o_rho[r];
                    }
            }
            // the entry moves on to the next sibling, in its own lane
            const bool has_next = rank + 1 < K;
    #pragma unroll
            for (int r = 0; r < RA; ++r)
                if (r == wr) {                                     // wave-uniform
                    BTV_KEEP_BRANCH();
                    const bool me = lane == wl;
                    const uint32_t nk = has_next ? __float_as_uint(__fmul_rn(e_prho[r], e_qn[r])) + 1u : 0u;
                    e_key[r] = me ? nk : e_key[r];
                    e_x[r] += me ? 4u : 0u;
                }
            // the emitted node's children: the entry of slot n + 1 (a slot past the last row is simply not written)
            if (d < B) {
                const int cs = n + 1;
                const float q_child = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(qfirst), d));
                const uint32_t key_child = __float_as_uint(__fmul_rn(u_rho, q_child)) + 1u;
                const uint32_t x_child = q_base + ((uint32_t)d << (2 + lg));
    #pragma unroll
                for (int r = 0; r < RA; ++r)
                    if (r == (cs >> 6)) {                          // wave-uniform
                        BTV_KEEP_BRANCH();
                        const bool me = lane == (cs & 63);
                        e_key[r] = me ? key_child : e_key[r];
                        e_prho[r] = me ? u_rho : e_prho[r];
                        e_x[r] = me ? x_child : e_x[r];
                    }
            }
    #pragma unroll
            for (int r = 0; r < RA; ++r)
                e_qn[r] = *reinterpret_cast<const __attribute__((address_space(3))) float *>((uintptr_t)(e_x[r] + 4u));
            ++n;
        }
    };
    phase(std::integral_constant<int, R>{}, N);
    double a = 0.0;                  // the surrogate: summed in fp64 and rounded once
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * 64 + lane;
        if (i < n) {
            const uint32_t idx = o_rec[r] & 0x1FFFu;
            token[i] = (int32_t)S.tok[idx];
            parent[i] = (int32_t)(o_rec[r] >> 13) - 1;
            if (depth) depth[i] = (int)(idx >> lg) + 1;
            if (rho) rho[i] = o_rho[r];
            a += (double)o_rho[r];
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off);
    if (lane == 0) {
        *n_out = n;
        if (ahat) *ahat = ADAPT ? (float)run_a : (float)(1.0 + a);
        if (ADAPT && ad.s_best) *ad.s_best = n > 0 ? best_a * ad.L_AR / best_c : -INFINITY;
    }
}

// ------------------------------------------------------------------------------------------------
// Step 3, part B'': the same tree, level by level, on the whole workgroup.
// The emission order (rho desc, depth asc, rank path asc) is a total order of the lattice in which a node comes
// after its parent and after its elder siblings, so the tree is the set of the N first prefixes of that order, and nothing
// about it needs the frontier, nor any order before the end.  The levels are swept once with a threshold that only
// rises: level d's candidates are the children of level d-1's candidates that score above it (a node deeper than N nodes that
// score at least as much cannot be among the first N).  Where the draft is confident (SW_CHAIN) it begins at the N-th best of a set of
// prefixes that need no sweep (sweep_bound), which as a rule leaves so few candidates, in thin levels, that one wavefront goes through them all with the threshold as it is (sweep_thin): N = 256 of a
// confident drafter, 13 levels: 600 candidates instead of 1480 without it, the sweep 14.8 -> 10.1 us.  Elsewhere, and where they are many all
// the same, the levels are swept with a threshold that moves up, after a level, to the lower edge of the bin that holds the N-th best
// candidate so far (a histogram of the scores' bits, 4 bins per binade, to which every candidate is added once; a suffix sum
// finds the bin).  A child of rank r is not needed either where the product of
// (rank + 1) along its path exceeds N: that many prefixes of its own level come before it (kept per node as the most
// children it can have: floor(N / product) = floor(floor(N / parent's product) / (r + 1))).
// Children take their places in their parents' order, so that a candidate's index grows with the depth and, within a level, with
// the rank path: score and index are the emission order's whole key.  At the end the candidates of the bins that
// are left, N of them and the few that share the last bin, are put in order: bin after bin by a finer histogram (16 per
// binade), and within a bin by counting.
// A thin level is one wavefront's work, 64 nodes at a time: what it costs is the length of its chain of steps, of which workgroup
// barriers and the LDS words around them would be a good part.  A wide one (the second level of a flat tree, all levels of
// a small vocabulary's) is the whole workgroup's, 256 nodes at a time, which go to the wavefronts in turn (node 4 l + w to
// lane l of wavefront w), since the wide fans come first.  A node writes its first four children from the registers that it
// tested them in; the rest of a wide fan is tested and written by its wavefront together.  If the candidates outgrow
// the LDS (marginals that are no probabilities can do that), nothing has been written yet and the frontier loop builds
// the tree.
// Measured (16 x 128256 marginals, whole call replayed from a HIP graph): see the rule in tb_rank_expand.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ int sweep_bin(uint32_t bits) { return (int)min(bits >> 19, (uint32_t)SW_BINS - 1u); }
__device__ __forceinline__ int sweep_coarse(uint32_t bits) { return (int)min(bits >> 21, (uint32_t)SW_COARSE - 1u); }

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x)                // 0 where no lane is the source
{
    const u64 b = __builtin_bit_cast(u64, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xF, CTRL < 0x142);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xF, CTRL < 0x142);
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
}
__device__ __forceinline__ double wave_incl_sum(double x)
{
    x += dpp_f64<0x111, 0xF>(x);
    x += dpp_f64<0x112, 0xF>(x);
    x += dpp_f64<0x114, 0xF>(x);
    x += dpp_f64<0x118, 0xF>(x);
    x += dpp_f64<0x142, 0xA>(x);
    x += dpp_f64<0x143, 0xC>(x);
    return x;
}
__device__ __forceinline__ float row_incl_sum(float x)             // within the rows of 16 lanes
{
    auto step = [&](auto ctrl) { x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(ctrl)::value, 0xF, 0xF, true)); };
    step(std::integral_constant<int, 0x111>{}); step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{}); step(std::integral_constant<int, 0x118>{});
    return x;
}

// parent (0xFFFF: the root) | rank << 16 is what identifies a node; depth - 1 takes 4 bits and `cap` - 1, the most children, 8:
// parent 12 bits, rank 8, depth 4, cap 8.
__device__ __forceinline__ uint32_t sweep_meta(uint32_t par, uint32_t rank, int dep1, int cap) { return par | (rank << 12) | ((uint32_t)dep1 << 20) | ((uint32_t)(cap - 1) << 24); }
constexpr uint32_t SW_ROOT = 0xFFFu;        // parent of the first level's nodes (no candidate that has children has this number)
static_assert(SW_CAP <= 4096, "a parent's number takes 12 bits");

// whole numbers: cap / (r + 1), cap <= 256
__device__ __forceinline__ int sweep_share(int cap, int r) { return (int)(((float)cap + 0.5f) * __builtin_amdgcn_rcpf((float)(r + 1))); }

__device__ __forceinline__ void sweep_put(SweepLds &L, int at, uint32_t score, uint32_t meta)
{
    L.cand[at] = make_uint2(meta, score);
    atomicAdd(&L.coarse[sweep_coarse(score)], 1);
}

// Children of one wavefront's nodes that score above the threshold: how many (first four in sc).
__device__ __forceinline__ int sweep_count(float rp, int most, const float (&qr)[4], const float *qd, int K, int th, int lane, uint32_t (&sc)[4])
{
    int c = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        sc[r] = __float_as_uint(__fmul_rn(rp, qr[r]));
        c += r < most && (int)sc[r] > th ? 1 : 0;              // (the scores fall with the rank)
    }
    u64 wide = __builtin_amdgcn_ballot_w64(c == 4 && most > 4);
    if (wide == 0ull) return c;
    if (__builtin_popcountll(wide) <= 8) {                     // a few: the wavefront tests 64 ranks of each
        while (wide != 0ull) {
            const int src = __builtin_ctzll(wide);
            wide &= wide - 1ull;
            const float wr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(rp), src));
            const int wm = __builtin_amdgcn_readlane(most, src);
            int cnt = 4;
            for (int r0 = 4; r0 < wm; r0 += 64) {
                const int r = r0 + lane;
                const int got = __builtin_popcountll(__builtin_amdgcn_ballot_w64(r < wm && (int)__float_as_uint(__fmul_rn(wr, qd[min(r, K - 1)])) > th));
                cnt += got;
                if (got < 64) break;
            }
            c = lane == src ? cnt : c;
        }
    } else {
        int lo = 4, hi = c == 4 ? most : 4;
        while (__builtin_amdgcn_ballot_w64(lo < hi) != 0ull) {
            const int mid = (lo + hi) >> 1;
            const bool ok = (int)__float_as_uint(__fmul_rn(rp, qd[min(mid, K - 1)])) > th, open = lo < hi;
            lo = open && ok ? mid + 1 : lo;
            hi = open && !ok ? mid : hi;
        }
        c = c == 4 ? lo : c;
    }
    return c;
}

// ... and their entries, from place `off` on.  i: the lane's node; lane src of the wavefront holds node i0 + src * step.
__device__ __forceinline__ void sweep_write(SweepLds &L, int c, int off, int i, int i0, int step, uint32_t rb, int cap, int dep1, const float *qd, int lane,
                                            const uint32_t (&sc)[4])
{
    const int part[4] = { cap, cap >> 1, (cap * 171) >> 9, cap >> 2 };      // cap / (r + 1)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (__builtin_amdgcn_ballot_w64(r < c) == 0ull) return;
        if (r < c) sweep_put(L, off + r, sc[r], sweep_meta((uint32_t)i, (uint32_t)r, dep1, part[r]));
    }
    u64 left = __builtin_amdgcn_ballot_w64(c > 4);
    while (left != 0ull) {
        const int src = __builtin_ctzll(left);
        left &= left - 1ull;
        const int wc = __builtin_amdgcn_readlane(c, src), wo = __builtin_amdgcn_readlane(off, src), wp = __builtin_amdgcn_readlane(cap, src);
        const float wr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)rb, src));
        for (int r = 4 + lane; r < wc; r += 64)
            sweep_put(L, wo + r, __float_as_uint(__fmul_rn(wr, qd[r])), sweep_meta((uint32_t)(i0 + src * step), (uint32_t)r, dep1, sweep_share(wp, r)));
    }
}

// The threshold, by one wavefront: lower edge of the coarse bin of the N-th best candidate (lane l: bins 8 l .. 8 l + 7).
__device__ __forceinline__ int sweep_raise(const SweepLds &L, int N, int lane)
{
    const int4 x = reinterpret_cast<const int4 *>(L.coarse)[2 * lane], y = reinterpret_cast<const int4 *>(L.coarse)[2 * lane + 1];
    const int s6 = y.w + y.z, s5 = s6 + y.y, s4 = s5 + y.x, s3 = s4 + x.w, s2 = s3 + x.z, s1 = s2 + x.y, own = s1 + x.x;
    const int incl = wave_incl_scan(own), need = N - (__builtin_amdgcn_readlane(incl, 63) - incl);      // that many of this lane's best
    const int sel = (y.w < need) + (s6 < need) + (s5 < need) + (s4 < need) + (s3 < need) + (s2 < need) + (s1 < need);
    const u64 here = __builtin_amdgcn_ballot_w64(need > 0 && own >= need);
    if (here == 0ull) return -1;                               // fewer than N of them
    const int src = __builtin_ctzll(here);
    return (8 * src + 7 - __builtin_amdgcn_readlane(sel, src)) << 21;
}

// A threshold to start from, by the whole workgroup: the greedy chain's nodes and the 64 best siblings of each are prefixes, and so
// are all first tokens; the N-th best of them is no better than the N-th best of all.  Lower edge of its bin less one (a
// score on the edge counts: it may be that of a lesser depth), -1 if there are fewer.  Not where the marginals are no
// probabilities: a child may then be better than its parent.  (The chain's scores by a scan, a little less than they are: a score's exact
// rounding does not matter here.  Scores fall from lane to lane, so one lane counts for all of a bin's: atomics of many lanes on
// few bins took 2.4 us in all.)
__device__ __forceinline__ int sweep_bound(const ExpandLds &S, SweepLds &L, int B, int K, int KP, int N, int lane, int w)
{
    const int tid = w * 64 + lane, K1 = min(K, N), most = min(K1, 64);
    if (tid < SW_COARSE / 4) reinterpret_cast<int4 *>(L.coarse)[tid] = make_int4(0, 0, 0, 0);
    const float first = S.q[min(tid, K - 1)], best = lane < B ? S.q[lane * KP] : 1.0f;
    float own[MAXB / 4];                                       // wavefront w: positions w + 1, w + 5, ..
#pragma unroll
    for (int u = 0; u < MAXB / 4; ++u) own[u] = S.q[min(4 * u + w + 1, B - 1) * KP + min(lane, K - 1)];
    const int least = K >= N ? (int)__float_as_uint(__fmul_rn(1.0f, S.q[N - 1])) - 1 : -1;      // (N first tokens are that good)
    const bool sound = __builtin_amdgcn_ballot_w64(!(best <= 1.0f)) == 0ull;
    float chain = best;                                        // lane k: of the chain's node at depth k + 1
    auto step = [&](auto ctrl) {
        const float o = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0x3F800000, (int)__float_as_uint(chain), decltype(ctrl)::value, 0xF, 0xF, false));
        chain *= o;
    };
    step(std::integral_constant<int, 0x111>{}); step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{}); step(std::integral_constant<int, 0x118>{});
    chain *= 0.99999f;
    __syncthreads();
    auto count = [&](uint32_t score, int n) {
        const int more = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n && (int)score > least));
        const int bin = sweep_coarse(score), bin1 = __builtin_amdgcn_update_dpp(0, bin, 0x101, 0xF, 0xF, false);      // row_shl:1
        const int at = (lane & 15) + 1;                        // (rows of 16 lanes, each for itself)
        const bool last = lane == more - 1 || at == 16;
        if (lane < more && (last || bin != bin1)) {
            atomicAdd(&L.coarse[bin], at);
            if (!last) atomicAdd(&L.coarse[bin1], -at);
        }
    };
    count(__float_as_uint(__fmul_rn(1.0f, first)), K1 - w * 64);
#pragma unroll
    for (int u = 0; u < MAXB / 4; ++u)
        if (4 * u + w + 1 < B)
            count(__float_as_uint(__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(chain), min(4 * u + w, 15))) * own[u]), most);
    __syncthreads();
    return sound ? max(sweep_raise(L, N, lane) - 1, -1) : -1;
}

// Levels 1, 2, .. by one wavefront, with the threshold as it is.  What a level costs is one instruction after the other, some 7 cycles
// each: the next level's probabilities are asked for a level ahead; a node that has children writes four, the last first, so that those that
// it does not have are overwritten by the nodes behind it; the rest of a wide fan is tested and written with one probability per
// lane; no histogram is kept.  Stops (d, a, b as in sweep_levels) at a level that is wide, or where the candidates become many, or the
// wide fans (about 0.25 us each here, one after the other; a limit of 8 or of 16 is slower on peaked marginals of 1000 to 128256 tokens).
__device__ __forceinline__ void sweep_thin(const ExpandLds &S, SweepLds &L, int B, int K, int KP, int N, int lane, int bound, int th, int &d, int &a, int &b)
{
    const int K1 = min(K, N);
    d = 2; a = 0; b = 0;
    for (int t0 = 0; t0 < K1; t0 += 64) {                      // level 1: the best tokens of position 0, already in order
        const int t = t0 + lane;
        const uint32_t score = __float_as_uint(__fmul_rn(1.0f, S.q[min(t, K - 1)]));
        const bool in = t < K1 && (int)score > bound;          // (the first is kept whatever the floor)
        if (in) L.cand[t] = make_uint2(sweep_meta(SW_ROOT, (uint32_t)t, 0, sweep_share(N, t)), score);
        const int got = __builtin_popcountll(__builtin_amdgcn_ballot_w64(in));
        b += got;
        if (got < 64) break;
    }
    const float inv_rank = __builtin_amdgcn_rcpf((float)(lane + 5));     // (sweep_share of rank 4 + lane)
    const int r1 = min(1, K - 1), r2 = min(2, K - 1), r3 = min(3, K - 1), rv = min(4 + lane, K - 1);
    float q[5], nq[5];                                         // ranks 0 .. 3, and 4 + lane, of position d - 1
    auto fetch = [&](int dd, float (&x)[5]) {
        const float *qd = S.q + (min(dd, B) - 1) * KP;
        x[0] = qd[0]; x[1] = qd[r1]; x[2] = qd[r2]; x[3] = qd[r3]; x[4] = qd[rv];
    };
    fetch(2, q);
    const uint32_t cand = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)L.cand;
    int fans = 0;
    uint32_t level = 1u << 20;                                 // what sweep_meta adds for depth - 1
    while (d <= B && a < b && b - a <= 2 * SW_THIN && b <= SW_CAP / 4) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint2 x = L.cand[min(a + lane, b - 1)];
        fetch(d + 1, nq);
        int nb = b;
        for (int a0 = a; a0 < b; a0 += 64) {
            const int i = a0 + lane;
            const float rp = __uint_as_float(x.y);
            const int cap = (int)(x.x >> 24) + 1, most = i < b ? min(cap, K) : 0;
            if (a0 + 64 < b) x = L.cand[min(i + 64, b - 1)];
            uint32_t sc[4];
            int c = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sc[r] = __float_as_uint(__fmul_rn(rp, q[r]));
                c += (int)sc[r] > th ? 1 : 0;                  // (the scores fall with the rank)
            }
            c = min(c, most);
            const u64 wide = __builtin_amdgcn_ballot_w64(min(c, most - 1) >= 4);
            fans += __builtin_popcountll(wide);
            if (fans > SW_FANS) return;
            for (u64 left = wide; left != 0ull; left &= left - 1ull) {
                const int src = __builtin_ctzll(left), wm = __builtin_amdgcn_readlane(most, src);
                const float wr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(rp), src));
                int cnt = 4 + __builtin_popcountll(__builtin_amdgcn_ballot_w64(4 + lane < wm && (int)__float_as_uint(__fmul_rn(wr, q[4])) > th));
                for (int r0 = 68; __builtin_expect(cnt == r0 && r0 < wm, 0); r0 += 64) {
                    const int r = r0 + lane;
                    cnt += __builtin_popcountll(__builtin_amdgcn_ballot_w64(r < wm && (int)__float_as_uint(__fmul_rn(wr, S.q[(d - 1) * KP + min(r, K - 1)])) > th));
                }
                c = lane == src ? cnt : c;
            }
            const int incl = wave_incl_scan(c), total = __builtin_amdgcn_readlane(incl, 63), off = nb + incl - c;
            if (__builtin_expect(nb + total > SW_CAP, 0)) { b = SW_CAP + 1; return; }        // (marginals that are no probabilities)
            const uint32_t meta = (uint32_t)i + level - (1u << 24);
            const uint32_t part[4] = { (uint32_t)cap, (uint32_t)cap >> 1, ((uint32_t)cap * 171u) >> 9, (uint32_t)cap >> 2 };     // cap / (r + 1)
            if (c > 0) {                                       // (these nodes' first places are all different; raw writes, which stay in this order)
                const uint32_t at = cand + 8u * (uint32_t)off;
#define BTV_PUT(R)                                                                                                                \
    {                                                                                                                             \
        const u64 e_ = ((u64)sc[R] << 32) | (meta + ((uint32_t)R << 12) + (part[R] << 24));                                       \
        asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(at), "v"(e_), "n"(8 * R) : "memory");                                  \
    }
                BTV_PUT(3) BTV_PUT(2) BTV_PUT(1) BTV_PUT(0)
#undef BTV_PUT
            }
            for (u64 left = wide; left != 0ull; left &= left - 1ull) {
                const int src = __builtin_ctzll(left);
                const int wc = __builtin_amdgcn_readlane(c, src), wo = __builtin_amdgcn_readlane(off, src), wp = __builtin_amdgcn_readlane(cap, src);
                const float wr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(rp), src));
                const uint32_t wm = (uint32_t)(a0 + src) + level - (1u << 24);
                if (4 + lane < wc)
                    L.cand[wo + 4 + lane] = make_uint2(wm + ((uint32_t)(4 + lane) << 12) + ((uint32_t)(((float)wp + 0.5f) * inv_rank) << 24), __float_as_uint(__fmul_rn(wr, q[4])));
                if (__builtin_expect(wc > 68, 0))
                    for (int r = 68 + lane; r < wc; r += 64)
                        L.cand[wo + r] = make_uint2(sweep_meta((uint32_t)(a0 + src), (uint32_t)r, d - 1, sweep_share(wp, r)),
                                                    __float_as_uint(__fmul_rn(wr, S.q[(d - 1) * KP + r])));
            }
            nb += total;
        }
        a = b; b = nb;
        ++d;
        level += 1u << 20;
#pragma unroll
        for (int r = 0; r < 5; ++r) q[r] = nq[r];
    }
}

// Whole sweep.  Returns the number of candidates, -1 if they do not fit.
__device__ __forceinline__ int sweep_levels(const ExpandLds &S, SweepLds &L, int B, int K, int KP, int N, int lane, int w, int floor)
{
    const int tid = w * 64 + lane;
    const bool chain = B > 1 && __builtin_amdgcn_ballot_w64(__fmul_rn(S.q[0], S.q[KP]) >= SW_CHAIN) != 0ull;
    int d = 2, a = 0, b = min(K, N), th = floor, buf = 0;      // a .. b - 1: the candidates of the level before
    if (chain) {
        // (the early stop's floor takes the bound's place: within 64 nodes it leaves hardly more, without the bound's 1.4 us)
        const int bound = floor >= 0 ? -1 : sweep_bound(S, L, B, K, KP, N, lane, w);
        th = max(floor, bound);
        if (w == 0) {
            sweep_thin(S, L, B, K, KP, N, lane, bound, th, d, a, b);
            if (lane == 0) { L.d = d; L.a = a; L.b = b; }
        }
        __syncthreads();
        d = __builtin_amdgcn_readfirstlane(L.d); a = __builtin_amdgcn_readfirstlane(L.a); b = __builtin_amdgcn_readfirstlane(L.b);
        if (b > SW_CAP) return -1;
        if (d > B || a == b) return b;
        __syncthreads();
    }
    // ---- wide levels, or many candidates: with a threshold that rises ------------------------------------------------------
    if (tid < SW_COARSE / 4) reinterpret_cast<int4 *>(L.coarse)[tid] = make_int4(0, 0, 0, 0);
    __syncthreads();
    if (chain)
        for (int c = tid; c < b; c += 256) atomicAdd(&L.coarse[sweep_coarse(L.cand[c].y)], 1);
    else if (tid < b)                                          // level 1: the best tokens of position 0, already in order
        sweep_put(L, tid, __float_as_uint(__fmul_rn(1.0f, S.q[tid])), sweep_meta(SW_ROOT, (uint32_t)tid, 0, sweep_share(N, tid)));
    __syncthreads();
    floor = th;
    bool raised = false;
    for (;;) {
        if (w == 0) {
            int seen = 0;                                      // candidates when the threshold was last moved
            while (d <= B && a < b) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const float *qd = S.q + (d - 1) * KP;
                const float qr[4] = { qd[0], qd[min(1, K - 1)], qd[min(2, K - 1)], qd[min(3, K - 1)] };
                uint2 x = L.cand[min(a + lane, b - 1)];
                // (a few more candidates since then hardly move it)
                if (b >= N && (!raised || b - seen > (N >> 2))) { th = max(floor, sweep_raise(L, N, lane)); seen = b; raised = true; }
                if (b - a > SW_THIN) break;
                int nb = b;
                for (int a0 = a; a0 < b; a0 += 64) {
                    const int i = a0 + lane;
                    if (a0 != a) x = L.cand[min(i, b - 1)];
                    const int cap = (int)(x.x >> 24) + 1;
                    uint32_t sc[4];
                    const int c = sweep_count(__uint_as_float(x.y), i < b ? min(cap, K) : 0, qr, qd, K, th, lane, sc);
                    const int incl = wave_incl_scan(c), total = __builtin_amdgcn_readlane(incl, 63);
                    if (nb + total > SW_CAP) { d = 0; break; }
                    sweep_write(L, c, nb + incl - c, i, a0, 1, x.y, cap, d - 1, qd, lane, sc);
                    nb += total;
                }
                if (d == 0) break;
                a = b; b = nb;
                ++d;
            }
            if (lane == 0) { L.d = d; L.a = a; L.b = b; L.th = th; }
        }
        __syncthreads();
        d = __builtin_amdgcn_readfirstlane(L.d); a = __builtin_amdgcn_readfirstlane(L.a); b = __builtin_amdgcn_readfirstlane(L.b);
        th = __builtin_amdgcn_readfirstlane(L.th);
        if (d == 0) return -1;
        if (d > B || a == b) return b;
        // ---- a wide level, by the whole workgroup ----------------------------------------------------------------------
        const float *qd = S.q + (d - 1) * KP;
        const float qr[4] = { qd[0], qd[min(1, K - 1)], qd[min(2, K - 1)], qd[min(3, K - 1)] };
        int nb = b;
        for (int a0 = a; a0 < b; a0 += 256, buf ^= 1) {
            const int i = a0 + 4 * lane + w;
            const uint2 x = L.cand[min(i, b - 1)];
            const int cap = (int)(x.x >> 24) + 1;
            uint32_t sc[4];
            const int c = sweep_count(__uint_as_float(x.y), i < b ? min(cap, K) : 0, qr, qd, K, th, lane, sc);
            L.cnt[buf][4 * lane + w] = c;
            __syncthreads();
            const int4 c4 = reinterpret_cast<const int4 *>(L.cnt[buf])[lane];
            const int sum = c4.x + c4.y + c4.z + c4.w, incl = wave_incl_scan(sum), total = __builtin_amdgcn_readlane(incl, 63);
            if (nb + total > SW_CAP) return -1;                // (uniform)
            sweep_write(L, c, nb + incl - sum + (w > 0 ? c4.x : 0) + (w > 1 ? c4.y : 0) + (w > 2 ? c4.z : 0), i, a0 + w, 4, x.y, cap, d - 1, qd, lane, sc);
            nb += total;
        }
        __syncthreads();
        a = b; b = nb;
        ++d;
    }
}

// star: the tree is the N best tokens of the first position.  floor: nodes that score no more (bits; -1: none) are not wanted.
// more: nothing is written, and false returned, if the early stop has not come within N nodes.
__device__ __forceinline__ bool expand_sweep(ExpandLds &S, SweepLds &L, int B, int K, int KP, int N, bool star, bool adapt, bool more, int floor, int tid, int32_t *parent,
                                             int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                                             const Adaptive &ad)
{
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int np = min(K, N), rank = tid, dep = 1;
    float r;
    uint32_t par = SW_ROOT;
    if (__builtin_expect(star, 1)) {                           // (0.1 us of 7: what follows is 50 KB of code)
        r = tid < np ? __fmul_rn(1.0f, S.q[tid]) : 0.f;
    } else {
#pragma unroll
    for (int i = 0; i < SW_BINS / 1024; ++i) reinterpret_cast<int4 *>(L.hist)[i * 256 + tid] = make_int4(0, 0, 0, 0);
    // ---- the N first of the candidates, in order ---------------------------------------------------------------------
    const int b = sweep_levels(S, L, B, K, KP, N, lane, w, floor);
    if (b < 0) return false;                                   // (uniform)
    np = min(b, N);
    for (int c = tid; c < b; c += 256) atomicAdd(&L.hist[sweep_bin(L.cand[c].y)], 1);
    if (tid == 0) L.kept = b;
    __syncthreads();
    int kept;                                                  // candidates in the bins of the first N
    {                                                          // thread t: bins 8 t .. 8 t + 7, and what lies above them
        const int4 x = reinterpret_cast<const int4 *>(L.hist)[2 * tid], y = reinterpret_cast<const int4 *>(L.hist)[2 * tid + 1];
        const int s7 = y.w, s6 = s7 + y.z, s5 = s6 + y.y, s4 = s5 + y.x, s3 = s4 + x.w, s2 = s3 + x.z, s1 = s2 + x.y, own = s1 + x.x;
        const int incl = wave_incl_scan(own), total = __builtin_amdgcn_readlane(incl, 63);
        if (lane == 0) L.wsum[w] = total;
        __syncthreads();
        const int t0 = L.wsum[0], t1 = L.wsum[1], t2 = L.wsum[2], t3 = L.wsum[3];
        const int up = total - incl + (w < 1 ? t1 : 0) + (w < 2 ? t2 : 0) + (w < 3 ? t3 : 0);
        const int4 p = make_int4(up + s1, up + s2, up + s3, up + s4), q = make_int4(up + s5, up + s6, up + s7, up);
        reinterpret_cast<int4 *>(L.hist)[2 * tid] = p;
        reinterpret_cast<int4 *>(L.hist)[2 * tid + 1] = q;
        reinterpret_cast<int4 *>(L.at)[2 * tid] = p;
        reinterpret_cast<int4 *>(L.at)[2 * tid + 1] = q;
        if (up < N && up + own >= N)                           // the bin of the N-th is one of these: what is above it, and it
            L.kept = q.z + y.z >= N ? (q.w + y.w >= N ? q.w + y.w : q.z + y.z) : q.y + y.y >= N ? q.y + y.y : q.x + y.x >= N ? q.x + y.x :
                     p.w + x.w >= N ? p.w + x.w : p.z + x.z >= N ? p.z + x.z : p.y + x.y >= N ? p.y + x.y : p.x + x.x;
    }
    __syncthreads();
    kept = L.kept;
    if (kept > SW_KEEP) return false;                          // (uniform) scores that are nearly all the same
    for (int c = tid; c < b; c += 256) {
        const uint32_t r = L.cand[c].y;
        const int bin = sweep_bin(r);
        if (L.hist[bin] < N) L.key[atomicAdd(&L.at[bin], 1)] = ((u64)r << 32) | (u64)(0xFFFFFFFFu - (uint32_t)c);
    }
    __syncthreads();
    for (int p = tid; p < kept; p += 256) {
        const u64 k = L.key[p];
        const int bin = sweep_bin((uint32_t)(k >> 32)), lo = L.hist[bin], hi = L.at[bin];
        const int place = lo + count_above(L.key, lo, hi, k);
        const uint32_t c = 0xFFFFFFFFu - (uint32_t)k;
        L.cand[c].y = (uint32_t)place;
        L.order[place] = (uint16_t)p;
    }
    __syncthreads();
    const u64 k = L.key[tid < np ? L.order[tid] : 0];
    const uint32_t mt = L.cand[0xFFFFFFFFu - (uint32_t)k].x;
    r = tid < np ? __uint_as_float((uint32_t)(k >> 32)) : 0.f;
    rank = (int)((mt >> 12) & 0xFFu); dep = (int)((mt >> 20) & 0xFu) + 1;
    par = mt & 0xFFFu;
    }
    int n = np;
    if (adapt) {
        // Sec. 3.4, Eq. 6: the budget stops at the first node that does not improve Ahat(n) * L_AR / C(n); all nodes before
        // it improved, so a node is compared with the one before it (fp64 prefix sums in emission order)
        double sum = wave_incl_sum((double)r);
        if (lane == 63) L.wd[w] = sum;
        if (tid == 0) L.n_stop = np;
        __syncthreads();
        const double w0 = L.wd[0], w1 = L.wd[1], w2 = L.wd[2];
        const double an = 1.0 + ((w > 0 ? w0 : 0.0) + (w > 1 ? w1 : 0.0) + (w > 2 ? w2 : 0.0) + sum), before = an - (double)r;
        const double cn = tid < np ? S.cost[tid] : 1.0, cb = tid > 0 && tid < np ? S.cost[tid - 1] : 1.0;
        // (one lane of each wavefront: the compiler takes the lanes of an atomic to one address one after the other, 5000 cycles)
        const u64 stops = __builtin_amdgcn_ballot_w64(tid < np && (!(cn > 0.0) || (tid > 0 && !(an * cb > before * cn))));
        if (lane == 0 && stops != 0ull) atomicMin(&L.n_stop, w * 64 + (int)__builtin_ctzll(stops));
        __syncthreads();
        n = L.n_stop;
        if (more && n == N) return false;                      // (uniform) still improving: the caller goes on to a larger budget
        if (tid == n && n < np && !(cn > 0.0)) atomicOr(ad.flag, 4u);
        if (tid == max(n - 1, 0)) {
            *n_out = n;
            if (ahat) *ahat = n > 0 ? (float)an : 1.0f;
            if (ad.s_best) *ad.s_best = n > 0 ? an * ad.L_AR / cn : -INFINITY;
        }
    }
    if (tid < n) {
        token[tid] = (int32_t)S.tok[(dep - 1) * KP + rank];
        parent[tid] = par == SW_ROOT ? -1 : (int32_t)L.cand[par].y;
        if (depth) depth[tid] = dep;
        if (rho) rho[tid] = r;
    }
    if (!adapt) {
        const double sum = wave_incl_sum((double)r);
        if (lane == 63) L.wd[w] = sum;
        __syncthreads();
        if (tid == 0) {
            *n_out = n;
            if (ahat) *ahat = (float)(1.0 + ((L.wd[0] + L.wd[1]) + (L.wd[2] + L.wd[3])));
        }
    }
    return true;
}

// Workgroup `row` ranks the candidates of its position into top_q / top_tok (global, [B][KP]); the workgroup that
// finishes last then runs the expansion on its first wavefront.
// ------------------------------------------------------------------------------------------------
// Step 3, part B': the beam-search tree (Sec. 4.3's comparison topology): depth by depth, the `width` extensions
// with the largest path score among all extensions of the prefixes kept at the previous depth.  Only the `width`
// best tokens of a position can be kept (an extension of rank r is preceded by r extensions of the same prefix),
// so a depth has at most width * width <= 256 candidates: one per thread, ranked by counting.  Order within a
// depth: rho desc, then the parent's place in the previous depth, then the token's rank.
// ------------------------------------------------------------------------------------------------
constexpr int MAXW = 16;

struct BeamLds {
    u64 key[MAXW * MAXW];
    float rho[2][MAXW];
    int node[2][MAXW];
    double part[4];
};

__device__ __forceinline__ void beam_block(const ExpandLds &S, BeamLds &Bm, int depth_max, int K, int KP, int width, int tid,
                                           int32_t *parent, int32_t *token, int32_t *depth, float *rho, int32_t *n_out,
                                           float *ahat)
{
    int n = 0, kept = 1;                                    // nodes so far, prefixes kept at the previous depth
    double mine_sum = 0.0;
    if (tid == 0) { Bm.rho[0][0] = 1.f; Bm.node[0][0] = -1; }
    __syncthreads();
    for (int k = 0; k < depth_max; ++k) {
        const int cur = k & 1, nc = kept * K, keep = min(nc, width);
        const int b = tid / K, rk = tid - b * K;            // candidate tid = (kept prefix b, rank rk)
        float r = 0.f;
        u64 mine = 0;
        if (tid < nc) {
            r = __fmul_rn(Bm.rho[cur][b], S.q[k * KP + rk]);
            mine = ((u64)__float_as_uint(r) << 32) | (u64)(0xFFFFFFFFu - (uint32_t)tid);
            Bm.key[tid] = mine;
        }
        __syncthreads();
        if (tid < nc) {
            int rank = 0;
            for (int j = 0; j < nc; ++j) rank += Bm.key[j] > mine ? 1 : 0;
            if (rank < keep) {
                const int nd = n + rank;
                parent[nd] = Bm.node[cur][b];
                token[nd] = (int32_t)S.tok[k * KP + rk];
                if (depth) depth[nd] = k + 1;
                if (rho) rho[nd] = r;
                Bm.rho[cur ^ 1][rank] = r;
                Bm.node[cur ^ 1][rank] = nd;
                mine_sum += (double)r;
            }
        }
        n += keep;
        kept = keep;
        __syncthreads();
    }
    for (int off = 32; off >= 1; off >>= 1) mine_sum += __shfl_xor(mine_sum, off);
    if ((tid & 63) == 0) Bm.part[tid >> 6] = mine_sum;
    __syncthreads();
    if (tid == 0) {
        *n_out = n;
        if (ahat) *ahat = (float)(1.0 + ((Bm.part[0] + Bm.part[1]) + (Bm.part[2] + Bm.part[3])));
    }
}

// All positions of a request with few marginals, by one workgroup: no list goes through memory, and nobody counts workgroups in.
// solo: log2 of the keys that a position has room for, and log2 of the lanes that share a key << 8.
__device__ __forceinline__ void rank_alone(ExpandLds &S, u64 *keys, const float *marg, int V, int B, int K, int KP, int solo, int tid)
{
    const int lgv = solo & 255, lgt = (solo >> 8) & 255, Vp = 1 << lgv, T = 1 << lgt;
    {
        const int pos = tid >> lgv, v = tid & (Vp - 1);
        const bool in = pos < B && v < V;
        const u64 key = make_key(marg[in ? (size_t)pos * V + v : 0], (uint32_t)v);
        keys[tid] = in ? key : 0ull;                           // (a key of zero is above nothing)
    }
    for (int e = tid; e < B * KP; e += RANK_T)
        if ((e & (KP - 1)) >= K) { S.q[e] = 0.f; S.tok[e] = 0u; }
    __syncthreads();
    const int pos = tid >> (lgv + lgt), v = (tid >> lgt) & (Vp - 1), part = tid & (T - 1);
    const u64 mine = keys[(pos << lgv) + v];
    const ulonglong2 *at = reinterpret_cast<const ulonglong2 *>(keys + (pos << lgv)) + part;
    int cnt = 0;
    for (int r = 0; r < 1 << (lgv - lgt - 1); r += 8, at += 8 * T) {         // (uniform; a lane has 8 pairs or more)
        ulonglong2 kk[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) kk[u] = at[u * T];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            cnt += kk[u].x > mine ? 1 : 0;
            cnt += kk[u].y > mine ? 1 : 0;
        }
    }
    if (T >= 2) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0xB1, 0xF, 0xF, false);     // quad_perm [1,0,3,2]
    if (T >= 4) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x4E, 0xF, 0xF, false);     // quad_perm [2,3,0,1]
    if (T >= 8) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x141, 0xF, 0xF, false);    // row_half_mirror
    if (T >= 16) cnt += __builtin_amdgcn_update_dpp(0, cnt, 0x140, 0xF, 0xF, false);   // row_mirror
    if (part == 0 && pos < B && v < V && cnt < K) {
        S.q[pos * KP + cnt] = __uint_as_float((uint32_t)(mine >> 32));
        S.tok[pos * KP + cnt] = 0xFFFFFFFFu - (uint32_t)mine;
    }
}

// SOLO: a workgroup takes all positions of a request (solo_plan; a kernel of its own: in one with the other the others took 0.2 us longer).
template <bool SOLO>
__global__ __launch_bounds__(RANK_T) void tb_rank_expand(const float *marg, int V, int B, int K, int KP, int N, int chunks, int lge,
                                                      TbCounters *ctr, const uint2 *part, u64 *top, int32_t *parent,
                                                      int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                                                      Adaptive ad, int beam_width, Batch bt, int algo, int solo)
{
    __shared__ union RankOrLevels { RankLds rank; SweepLds lev; } U;     // the ranking is over when the expansion starts
    __shared__ ExpandLds S;
    __shared__ BeamLds BM;
    __shared__ int use_levels, L_floor[2];
    RankLds &RL = U.rank;
    // Fetch every argument in one round trip: left to the compiler the scalar loads follow the code in four
    // dependent steps over an argument block of several cache lines that is cold in every launch.
    asm volatile("" ::"s"(marg), "s"(V), "s"(B), "s"(K), "s"(KP), "s"(N), "s"(chunks), "s"(lge), "s"(ctr), "s"(part), "s"(top),
                 "s"(parent), "s"(token), "s"(depth), "s"(rho), "s"(n_out), "s"(ahat), "s"(ad.cost), "s"(ad.L_AR),
                 "s"(ad.s_best), "s"(ad.flag), "s"(beam_width), "s"(bt.n_nodes), "s"(bt.q_offset), "s"(bt.flag), "s"(solo));
    // Workgroup `row` = position row % B of request row / B; marginals, per-thread maxima and top lists are laid out
    // request after request, outputs start at the request's q_offset.
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), row = blockIdx.x;
    const int req = SOLO ? row : row / B;
    double cost_mine = 1.0;
    if constexpr (SOLO) {                      // the whole request by this workgroup (see solo_plan)
        rank_alone(S, reinterpret_cast<u64 *>(RL.bins), marg + (size_t)req * B * V, V, B, K, KP, solo, tid);
        if (ad.cost && tid < N) cost_mine = ad.cost[tid];
    } else {
    u64 *top_row = top + (size_t)row * KP;
    const float *src = marg + (size_t)row * V;
    const bool aligned = (((size_t)row * V) & 3) == 0 && (reinterpret_cast<uintptr_t>(marg) & 15) == 0;
    const int slots = lge == 0 ? V : chunks * 256;             // slot e: chunk e / 256, thread e % 256 of the scan (or marginal e)
    const uint2 *pr = part + (size_t)row * chunks * 256;
    // ---- the bound: K-th largest per-thread maximum of the row, down to the lower edge of its histogram bin ---
    uint32_t pv[PER], pw[PER];                                 // the loads are in flight while the histogram is cleared
#pragma unroll
    for (int j = 0; j < PER; ++j) {                            // no load behind a branch: all of them in flight at once
        const int e = j * RANK_T + tid, at = e < slots ? e : 0;
        if (lge == 0) { pv[j] = prob_bits(src[at]); pw[j] = 0u; }
        else { const uint2 x = pr[at]; pv[j] = x.x; pw[j] = x.y; }
    }
    if (tid == 0) { RL.nsel = 0; RL.nslot = 0; }
    // A row of so few marginals that all of them can be ranked needs no bound.
    const bool few = V <= RANK_FEW;                            // (uniform)
    if (!few) {
        for (int b = tid; b < TBINS / 4; b += RANK_T) reinterpret_cast<int4 *>(RL.bins)[b] = make_int4(0, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) if (j * RANK_T + tid < slots) atomicAdd(&RL.bins[(int)(pv[j] >> 19)], 1);
        for (int e = PER * RANK_T + tid; e < slots; e += RANK_T) atomicAdd(&RL.bins[(int)(pr[e].x >> 19)], 1);
        __syncthreads();
        {
            const int4 hb = reinterpret_cast<const int4 *>(RL.bins)[tid];                  // thread t owns bins 4 t .. 4 t + 3
            const int own = hb.x + hb.y + hb.z + hb.w, incl = wave_incl_scan(own), wtot = __builtin_amdgcn_readlane(incl, 63);
            if (lane == 0) RL.wsum[w] = wtot;
            __syncthreads();
            const int others = wave_incl_scan(lane < RANK_W && lane > w ? RL.wsum[lane & (RANK_W - 1)] : 0);
            const int above = wtot - incl + __builtin_amdgcn_readlane(others, RANK_W - 1);  // in the bins of the higher threads
            if (above < K && above + own >= K) {
                const int s3 = above + hb.w, s2 = s3 + hb.z, s1 = s2 + hb.y;
                RL.sel_bin = tid * 4 + (s3 >= K ? 3 : s2 >= K ? 2 : s1 >= K ? 1 : 0);
            }
            __syncthreads();                                       // the histogram is dead from here on: sel[] takes its place
        }
    }
    const uint32_t tau = few ? 0u : (uint32_t)RL.sel_bin << 19;
    // ---- the candidates.  A slot whose maximum reaches the bound holds a candidate; when its second largest stays
    // below the bound, which is the rule (K of thousands of slots are taken), that maximum is the slot's only one
    // and goes to the list as it stands, with the token id that its place in the slot gives.  The other slots
    // are listed and read again, one 16-byte piece of a slot per thread.
    // Places in the lists are handed out per wavefront: every lane counts what it has, a scan places the lanes,
    // one lane takes the wavefront's range from the shared counter (one LDS round trip, not one per entry).
    // A lane rarely holds more than one entry: it keeps its entries as a bit mask and the wavefront loops until
    // every mask is empty, each lane storing one entry per trip (to a place of its own behind the list when it has
    // none left), which costs less than a branch or a store per possible entry. ----------------------------------
    auto wave_range = [&](int mine, int *counter) {            // first place of this lane's `mine` entries
        const int incl = wave_incl_scan(mine), total = __builtin_amdgcn_readlane(incl, 63);
        int first = 0;
        if (total > 0) {                                       // (wave-uniform)
            if (lane == 0) first = atomicAdd(counter, total);
            first = __builtin_amdgcn_readfirstlane(first);
        }
        return first + incl - mine;
    };
    if (few) {
        if (tid < V) RL.sel[tid] = ((u64)pv[0] << 32) | (u64)(0xFFFFFFFFu - (uint32_t)tid);
        if (tid == 0) RL.nsel = V;
    } else {
        uint32_t one = 0u, more = 0u;                           // records whose slot holds one candidate / maybe several
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (j * RANK_T + tid < slots && pv[j] >= tau) {
                if (pw[j] >= tau && lge != 0) more |= 1u << j; else one |= 1u << j;
            }
        if (__builtin_amdgcn_ballot_w64(one != 0u) != 0ull) {
            int pos = wave_range(__builtin_popcount(one), &RL.nsel);
            do {
                const bool has = one != 0u;
                const int j = has ? __builtin_ctz(one) : 0, e = j * RANK_T + tid;
                const uint32_t k = pick4(pw[0], pw[1], pw[2], pw[3], j) & 31u;
                const uint32_t v = (uint32_t)slot_first(lge, e >> 8, e & 255) + (k >> 2) * 1024u + (k & 3u);
                RL.sel[has && pos < SELCAP ? pos : SELCAP + lane] = ((u64)pick4(pv[0], pv[1], pv[2], pv[3], j) << 32) | (u64)(0xFFFFFFFFu - v);
                pos += has ? 1 : 0;
                one &= one - 1u;
            } while (__builtin_amdgcn_ballot_w64(one != 0u) != 0ull);
        }
        int mine = __builtin_popcount(more);
        if (chunks <= 256)                                      // (a place of the list takes 16 bits)
            for (int e = PER * RANK_T + tid; e < slots; e += RANK_T) mine += pr[e].x >= tau ? 1 : 0;
        if (__builtin_amdgcn_ballot_w64(mine != 0) != 0ull) {
            int pos = wave_range(mine, &RL.nslot);
            while (__builtin_amdgcn_ballot_w64(more != 0u) != 0ull) {
                const bool has = more != 0u;
                const int j = has ? __builtin_ctz(more) : 0;
                RL.slot[has && pos < SLOTCAP ? pos : SLOTCAP + lane] = (uint16_t)(j * RANK_T + tid);
                pos += has ? 1 : 0;
                more &= more - 1u;
            }
            if (chunks <= 256)
                for (int e = PER * RANK_T + tid; e < slots; e += RANK_T)
                    if (pr[e].x >= tau) {
                        if (pos < SLOTCAP) RL.slot[pos] = (uint16_t)e;
                        ++pos;
                    }
        }
    }
    __syncthreads();
    const int nslot = RL.nslot;
    if (nslot == 0 && chunks <= 256) {
        // nothing to read again
    } else if (nslot <= SLOTCAP && chunks <= 256) {
        const int lgp = lge - 2, pmask = (1 << lgp) - 1;       // 16-byte pieces per slot (lge >= 2 here)
        const int total = nslot << lgp;
        const bool whole = aligned && (V & 3) == 0;            // every piece that starts inside the row ends inside it
        for (int base = 0; base < total; base += RANK_T) {
            const int i = base + tid, sl = RL.slot[(i < total ? i : 0) >> lgp];
            const int v = slot_first(lge, sl >> 8, sl & 255) + (i & pmask) * 1024, v0 = i < total && v < V ? v : -1;
            float pe[4] = { 0.f, 0.f, 0.f, 0.f };
            uint32_t ok = 0u;                                   // bit e: element e of the piece is a candidate
            if (whole) {
                const float4 a = *reinterpret_cast<const float4 *>(src + (v0 < 0 ? 0 : v0));
                pe[0] = a.x; pe[1] = a.y; pe[2] = a.z; pe[3] = a.w;
            } else if (v0 >= 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) pe[e] = src[min(v0 + e, V - 1)];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (v0 >= 0 && v0 + e < V && prob_bits(pe[e]) >= tau) ok |= 1u << e;
            if (__builtin_amdgcn_ballot_w64(ok != 0u) == 0ull) continue;
            int pos = wave_range(__builtin_popcount(ok), &RL.nsel);
            while (__builtin_amdgcn_ballot_w64(ok != 0u) != 0ull) {
                const bool has = ok != 0u;
                const int e = has ? __builtin_ctz(ok) : 0;
                const float pq = __uint_as_float(pick4(__float_as_uint(pe[0]), __float_as_uint(pe[1]), __float_as_uint(pe[2]), __float_as_uint(pe[3]), e));
                RL.sel[has && pos < SELCAP ? pos : SELCAP + lane] = make_key(pq, (uint32_t)(v0 + e));
                pos += has ? 1 : 0;
                ok &= ok - 1u;
            }
        }
    } else if (tid == 0) {
        RL.nsel = SELCAP + 1;                                  // too many slots tie at the bound: select from the row
    }
    __syncthreads();
    int nc = RL.nsel;
    if (nc > SELCAP) {                         // rare: one wavefront selects the K best of the row first
        __syncthreads();
        if (w == 0) wave_select([&](auto f) { for (int v = lane; v < V; v += 64) f(make_key(src[v], (uint32_t)v)); }, K, RL.hist, RL.sel, &RL.nsel, lane);
        nc = K;
        __syncthreads();
    }
    if (nc <= 64) rank_keys<16, 2>(RL.sel, nc, K, top_row, tid);
    else if (nc <= 128) rank_keys<8, 8>(RL.sel, nc, K, top_row, tid);
    else if (few) rank_keys<4, 8>(RL.sel, nc, K, top_row, tid);
    else rank_keys_binned(RL.sel, RL.sorted, RL.first, RL.at, RL.wsum, tau, nc, K, top_row, tid, lane, w);
    if (K + tid < KP) publish(top_row, K + tid, NO_TOKEN);     // (KP <= 256)
    // ---- the workgroup that finishes last expands -------------------------------------------------------------
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this thread's part of the lists has reached memory
    __syncthreads();
    if (tid == 0) {
        RL.last = __hip_atomic_fetch_add(&ctr[req].done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == B - 1;
        if (RL.last) __hip_atomic_store(&ctr[req].done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // ready for the next call
    }
    __syncthreads();
    if (!RL.last) return;
    if (ad.cost && tid < N) cost_mine = ad.cost[tid];         // (on its way together with the lists)
    {   // all of a thread's loads are issued before the first is stored (a load and its store per loop trip would
        // make every trip a round trip to memory)
        const u64 *lists = top + (size_t)req * B * KP;
        const int n = B * KP;                                  // (4096 at most)
        u64 x[MAXB * BTV_MAX_NODES / RANK_T];
#pragma unroll
        for (int i = 0; i < MAXB * BTV_MAX_NODES / RANK_T; ++i)
            if (i * RANK_T < n) x[i] = __hip_atomic_load(lists + min(tid + i * RANK_T, n - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < MAXB * BTV_MAX_NODES / RANK_T; ++i) {
            const int e = tid + i * RANK_T;
            if (e < n) { S.q[e] = __uint_as_float((uint32_t)(x[i] >> 32)); S.tok[e] = (uint32_t)x[i]; }
        }
    }
    }

    if (bt.n_nodes) {                          // this request's budget and output rows
        const int o0 = bt.q_offset[req], room = bt.q_offset[req + 1] - o0, want = bt.n_nodes[req];
        const bool bad = o0 < 0 || want < 0 || want > N || want > room;
        if (bad && tid == 0) atomicOr(bt.flag, 16u);
        N = bad ? 0 : want;
        parent += o0; token += o0;
        if (depth) depth += o0;
        if (rho) rho += o0;
        n_out += req;
        if (ahat) ahat += req;
        if (N == 0) {
            if (tid == 0) { *n_out = 0; if (ahat) *ahat = 1.0f; }
            return;
        }
    }
    if (ad.cost && tid < N) S.cost[tid] = cost_mine;           // (N <= 256)
    __syncthreads();
    if (w >= 4) return;                        // the expansions are written for four wavefronts (those that have ended count at no barrier)
    if (beam_width > 0) {                      // B rows = depths of the beam tree, K = min(V, width)
        beam_block(S, BM, B, K, KP, beam_width, tid, parent, token, depth, rho, n_out, ahat);
        return;
    }
    // Which expansion: the sweep pays per level (0.4 us and 1.4 us for its threshold where it starts from the chain, 0.9 us elsewhere, and 2 us at
    // the end), the one-wavefront loop per node (0.24 us up to 64 nodes, 0.5 us at 256), so the loop is left with the smallest
    // trees that may be deep.  The tree cannot be deeper
    // than the greedy chain stays above the N-th best token of the first position (every node scores at least as much as
    // the tree's last one, which scores at least that).
    // 16 positions x 128256 tokens, HIP-graph replays, sweep / loop: a confident drafter (depth 8 .. 13) N = 16: 17.7 / 15.0 us, N = 32: 19.9 /
    // 19.3, N = 48: 20.7 / 23.1, N = 64: 21.4 / 27.1, N = 256: 26.8 / 137; depth 4 .. 5: N = 16: 14.8 / 15.0, N = 24: 15.6 / 16.9, N = 64:
    // 18.1 / 27.1; 4 positions x 64 tokens, N = 16: 10.0 / 11.2.
    if (w == 0) {
        const int k = min(lane, B - 1);
        const float chain = row_incl_sum(lane < B ? __log2f(S.q[k * KP]) : -1e30f);      // (an estimate: the choice changes no result)
        const float g_est = __log2f(S.q[min(K, N) - 1]);
        const int reach = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < B && chain >= g_est));
        // a star: no child of the best first token comes before the N-th best first token (a tie goes to the lesser depth)
        const bool star = K >= N && (B == 1 || __fmul_rn(__fmul_rn(1.0f, S.q[0]), S.q[KP]) <= __fmul_rn(1.0f, S.q[N - 1]));
        if (ad.cost && !star) {
            // The early stop takes a node only if rho(n) C(n-1) > Ahat(n-1) (C(n) - C(n-1)); Ahat(n-1) is at least 1 and the
            // sum of the greedy chain's n - 1 best scores, so no wanted node scores less than the least of these bounds over n
            // (up to 64 nodes, the first budget; up to N).  Not with costs that are no costs
            // or marginals that are no probabilities.
            const float own = lane < B ? __builtin_amdgcn_exp2f(chain) : 0.f, sums = row_incl_sum(own);
            const float first = 1.0f + __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(own), 0));
            const float whole = 1.0f + __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(sums), 15));
            bool good = lane >= B || S.q[k * KP] <= 1.0f;
            uint32_t inv[2];                            // ~bits of the least: the greatest of them is wanted
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = u * 64 + lane, at = min(e, N - 1);
                const double c = S.cost[at], cb = S.cost[max(at - 1, 0)];
                good = good && c > 0.0 && c < 1e300;
                const float l = (float)(c - cb) * __builtin_amdgcn_rcpf((float)cb) * (at > B ? whole : first);
                const uint32_t x = e == 0 || e >= N ? 0u : l > 0.f ? ~__float_as_uint(l) : 0xFFFFFFFFu;
                if (u < 2) inv[u] = x; else inv[1] = umax(inv[1], x);
            }
            const uint32_t a0 = wave_max_u32(inv[0]), a1 = umax(a0, wave_max_u32(inv[1]));
            const bool ok = __builtin_amdgcn_ballot_w64(!good) == 0ull;
            auto floor_of = [&](uint32_t a) {
                const float l = __uint_as_float(~a);
                return ok && l > 0.f && l < 1.0f ? (int)__float_as_uint(l * 0.999f) : -1;
            };
            if (lane == 0) { L_floor[0] = floor_of(a0); L_floor[1] = floor_of(a1); }
        }
        if (lane == 0)
            use_levels = algo == 0 && star ? 2 : algo == 2 || (algo == 0 && (N > 64 || 0.7f + 0.5f * (float)min(reach, N) < 0.22f * (float)N)) ? 1 : 0;
    }
    __syncthreads();
    if (use_levels) {
        // with the early stop: it comes within the first 64 nodes as a rule, and their tree is a prefix of the larger one
        const bool adapt = ad.cost != nullptr, star = use_levels == 2;
        bool done = false;
        for (int budget = adapt && !star ? min(N, 64) : N;; budget = N) {
            done = expand_sweep(S, U.lev, B, K, KP, budget, star, adapt, budget < N, adapt && !star ? L_floor[budget < N ? 0 : 1] : -1, tid, parent, token, depth, rho, n_out, ahat, ad);
            if (done || budget == N) break;
            __syncthreads();
        }
        if (done) return;
    }
    if (w != 0) return;
    if (ad.cost) {
        if (N <= 64) expand_wave<1, true>(S, B, K, KP, N, lane, parent, token, depth, rho, n_out, ahat, ad);
        else expand_wave<4, true>(S, B, K, KP, N, lane, parent, token, depth, rho, n_out, ahat, ad);
    } else {
        if (N <= 64) expand_wave<1, false>(S, B, K, KP, N, lane, parent, token, depth, rho, n_out, ahat, ad);
        else expand_wave<4, false>(S, B, K, KP, N, lane, parent, token, depth, rho, n_out, ahat, ad);
    }
}

int next_pow2(int x) { int p = 1; while (p < x) p <<= 1; return p; }

struct TopkPlan { int K, KP, lge, chunks; size_t ctr_bytes, part_bytes, top_bytes; };

constexpr int MAX_BATCH = 1024;

TopkPlan topk_plan(int batch, int B, int V, int N)
{
    TopkPlan t;
    t.K = std::min(V, N);
    t.KP = std::max(next_pow2(t.K), 1);
    t.lge = V <= 16 * 256 ? 0 : 2;
    while (t.lge > 0 && t.lge < LGE_MAX && V > 16 * (256 << t.lge)) ++t.lge;
    t.chunks = (V + (256 << t.lge) - 1) / (256 << t.lge);
    // (the counters stay zero from call to call, so their place must not depend on the call's sizes)
    t.ctr_bytes = btv_align_up((size_t)MAX_BATCH * sizeof(TbCounters), BTV_WS_ALIGN);
    t.part_bytes = t.lge == 0 ? 0 : btv_align_up((size_t)batch * B * t.chunks * 256 * sizeof(uint2), BTV_WS_ALIGN);
    t.top_bytes = btv_align_up((size_t)batch * B * t.KP * sizeof(u64), BTV_WS_ALIGN);
    return t;
}

// One workgroup for all positions of a request where its threads hold all marginals twice, positions and vocabulary rounded up to powers of two
// (16 marginals at least, so that a lane of those that share a key has eight pairs of keys to look at).  4 x 64 marginals, 16 nodes: 8.2 us with a workgroup
// per position, whose lists the last one to finish fetches from memory, 6.5 alone; 4 x 128, 64 nodes: 12.4 and 11.3; 4 x 200, a thread per marginal: 12.7 and 15.2.
int solo_plan(int B, int V)
{
    const int Vp = std::max(16, next_pow2(V)), Bp = next_pow2(B);
    if (2 * Vp * Bp > RANK_T) return 0;
    const int T = std::min(std::min(RANK_T / (Vp * Bp), Vp / 16), 16);
    return __builtin_ctz(Vp) | __builtin_ctz(T) << 8;
}

size_t tree_build_ws(int batch, int B, int V, int N)
{
    if (batch < 1 || batch > MAX_BATCH || B < 1 || B > MAXB || V < 1 || N < 1 || N > BTV_MAX_NODES) return 0;
    TopkPlan t = topk_plan(batch, B, V, N);
    return BTV_WS_HEADER + t.ctr_bytes + t.part_bytes + t.top_bytes;
}

}  // namespace

extern "C" {

size_t btv_tree_build_workspace(int B, int V, int N) { return tree_build_ws(1, B, V, N); }

size_t btv_tree_build_batch_workspace(int batch, int B, int V, int N_max) { return tree_build_ws(batch, B, V, N_max); }

static int tree_build_launch(const float *marginals, int batch, int B, int V, int N, const Adaptive &ad_in, int beam_width,
                             Batch bt, int algo, int32_t *parent, int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                             void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(marginals && parent && token && n_out, "null pointer");
    BTV_REQUIRE(batch >= 1 && batch <= MAX_BATCH, "batch=%d outside [1,%d]", batch, MAX_BATCH);
    BTV_REQUIRE(B >= 1 && B <= MAXB, "B=%d outside [1,%d]", B, MAXB);
    BTV_REQUIRE(V >= 1, "V=%d", V);
    BTV_REQUIRE(N >= 1 && N <= BTV_MAX_NODES, "N=%d outside [1,%d]", N, BTV_MAX_NODES);
    int rc = btv_check_ws(ws, ws_bytes, tree_build_ws(batch, B, V, N));
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    TopkPlan t = topk_plan(batch, B, V, N);
    unsigned char *base = static_cast<unsigned char *>(ws);
    TbCounters *ctr = reinterpret_cast<TbCounters *>(base + BTV_WS_HEADER);
    uint2 *part = reinterpret_cast<uint2 *>(base + BTV_WS_HEADER + t.ctr_bytes);
    u64 *top = reinterpret_cast<u64 *>(base + BTV_WS_HEADER + t.ctr_bytes + t.part_bytes);
    Adaptive ad = ad_in;
    ad.flag = reinterpret_cast<uint32_t *>(base);
    bt.flag = reinterpret_cast<uint32_t *>(base);
    const dim3 scan_grid(t.chunks, B * batch);
    auto scan = [&](auto lge) {
        constexpr int LGE = decltype(lge)::value;
        // Marginals that the last-level cache (256 MB) cannot hold are read past it: read through it, rows that are still there make way for others.  us, through it / past it,
        // behind the softmax that wrote them | a pass over them in place | other buffers in between | the same marginals again at once: 312 MB 90.0 / 80.5 | 96.7 / 75.4 | 82.8 / 80.3 |
        // 81.3 / 79.4; 394 MB 118 / 98 | 138 / 94 | 102 / 97 | 103 / 98; 525 MB 163 / 131 | 180 / 129 | 138 / 129 | 138 / 127.  Just above the cache's size much of them is still there, and
        // some calls lose: 271 MB 75.1 / 73.2 | 67.0 / 68.9 | 74.0 / 71.9 | 66.9 / 71.8; 279 MB 77.4 / 73.1 | 66.5 / 67.1 | 75.2 / 72.0 | 68.2 / 72.1; 296 MB 84.7 / 78.4 | 83.7 / 71.0 | 79.7 / 76.1 |
        // 73.1 / 75.2.  Below: 131 MB 36.9 / 38.2 | - | 39.2 / 38.2 | 35.1 / 37.7; 263 MB 69.7 / 69.8 | 64.6 / 64.5 | 71.7 / 69.6 | 63.3 / 69.3.
        const bool stream_read = (unsigned long long)batch * B * V * sizeof(float) > (288ull << 20);
        const auto kern = stream_read ? tb_thread_max<LGE, true> : tb_thread_max<LGE, false>;
        hipLaunchKernelGGL(kern, scan_grid, dim3(256), 0, st, marginals, V, t.chunks, part);
    };
    if (t.lge == 2) scan(std::integral_constant<int, 2>{});
    else if (t.lge == 3) scan(std::integral_constant<int, 3>{});
    else if (t.lge == 4) scan(std::integral_constant<int, 4>{});
    else if (t.lge == 5) scan(std::integral_constant<int, 5>{});
    BTV_HIP(hipGetLastError());
    const int solo = solo_plan(B, V);
    const auto rank_expand = solo ? tb_rank_expand<true> : tb_rank_expand<false>;
    hipLaunchKernelGGL(rank_expand, dim3(solo ? batch : B * batch), dim3(RANK_T), 0, st, marginals, V, B, t.K, t.KP, N, t.chunks, t.lge, ctr, part, top,
                       parent, token, depth, rho, n_out, ahat, ad, beam_width, bt, algo, solo);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

static const Batch kOneRequest = { nullptr, nullptr, nullptr };

int btv_tree_build(const float *marginals, int B, int V, int N, int32_t *parent, int32_t *token, int32_t *depth,
                   float *rho, int32_t *n_out, float *ahat, void *ws, size_t ws_bytes, void *stream)
{
    const Adaptive none = { nullptr, 0.0, nullptr, nullptr };
    return tree_build_launch(marginals, 1, B, V, N, none, 0, kOneRequest, 0, parent, token, depth, rho, n_out, ahat, ws, ws_bytes, stream);
}

int btv_tree_build_beam(const float *marginals, int B, int V, int width, int depth_max, int32_t *parent, int32_t *token,
                        int32_t *depth, float *rho, int32_t *n_out, float *ahat, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(width >= 1 && width <= MAXW, "width=%d outside [1,%d]", width, MAXW);
    BTV_REQUIRE(B >= 1 && B <= MAXB, "B=%d outside [1,%d]", B, MAXB);
    BTV_REQUIRE(depth_max >= 1 && depth_max <= B, "depth=%d outside [1,B=%d]", depth_max, B);
    // the first depth_max positions are ranked for their `width` best tokens; the rest of the path is shared
    const Adaptive none = { nullptr, 0.0, nullptr, nullptr };
    return tree_build_launch(marginals, 1, depth_max, V, width, none, width, kOneRequest, 0, parent, token, depth, rho, n_out, ahat,
                             ws, ws_bytes, stream);
}

int btv_tree_build_adaptive(const float *marginals, int B, int V, int N_max, const double *cost, double L_AR,
                            int32_t *parent, int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                            double *s_best, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(cost != nullptr, "null pointer");
    BTV_REQUIRE(L_AR > 0.0, "L_AR must be positive");
    const Adaptive ad = { cost, L_AR, s_best, nullptr };
    return tree_build_launch(marginals, 1, B, V, N_max, ad, 0, kOneRequest, 0, parent, token, depth, rho, n_out, ahat, ws, ws_bytes, stream);
}

int btv_tree_build_tuned(const float *marginals, int B, int V, int N, const double *cost, double L_AR, int algo,
                         int32_t *parent, int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                         double *s_best, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(algo >= 0 && algo <= 2, "algo=%d outside [0,2]", algo);
    BTV_REQUIRE(cost == nullptr || L_AR > 0.0, "L_AR must be positive");
    const Adaptive ad = { cost, L_AR, cost ? s_best : nullptr, nullptr };
    return tree_build_launch(marginals, 1, B, V, N, ad, 0, kOneRequest, algo, parent, token, depth, rho, n_out, ahat, ws, ws_bytes,
                             stream);
}

int btv_tree_build_batch(const float *marginals, int batch, int B, int V, const int32_t *n_nodes, const int32_t *q_offset,
                         int N_max, int32_t *parent, int32_t *token, int32_t *depth, float *rho, int32_t *n_out, float *ahat,
                         void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(n_nodes && q_offset, "null pointer");
    const Adaptive none = { nullptr, 0.0, nullptr, nullptr };
    const Batch bt = { n_nodes, q_offset, nullptr };
    return tree_build_launch(marginals, batch, B, V, N_max, none, 0, bt, 0, parent, token, depth, rho, n_out, ahat, ws, ws_bytes,
                             stream);
}

}  // extern "C"
