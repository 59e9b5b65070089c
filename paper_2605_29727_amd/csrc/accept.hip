// Greedy acceptance on the GPU (gfx950): target argmax per tree row and the walk; also straight from the hidden states.
// (The rejection walk at temperature 1 is in stochastic.hip.)
//
// App. C "Acceptance" / Sec. 3.1: the committed tokens are the longest root-to-node path the
// target itself would have produced.  Rows of `logits`: 0 = root, 1+i = node i.
#include "btv_common.h"
#include "lm_head.h"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace {

constexpr int ACHUNK = 8192;     // vocabulary elements per argmax workgroup

using Best = LmBest;

__device__ __forceinline__ void best_take(Best &b, float v, int i)
{   // larger value wins; equal values: lower index wins; NaN never wins
    if (v > b.v || (v == b.v && i < b.i)) { b.v = v; b.i = i; }
}

__device__ __forceinline__ Best best_wave(Best b)
{
    for (int off = 32; off >= 1; off >>= 1) {
        float ov = __shfl_xor(b.v, off);
        int oi = __shfl_xor(b.i, off);
        best_take(b, ov, oi);
    }
    return b;
}

template <bool BF16>
__device__ __forceinline__ float load_one(const void *logits, size_t idx)
{
    if (BF16) return __uint_as_float((uint32_t)static_cast<const uint16_t *>(logits)[idx] << 16);
    return static_cast<const float *>(logits)[idx];
}

// Best of elements v0 .. v1 - 1 of a row (its first at element `base` of the logits), as seen by thread tid of T.  What lies in whole 16-byte pieces
// of memory is read by 16-byte loads, U per thread in flight before the first is looked at, wherever the row begins (a vocabulary that is no multiple of
// eight leaves most rows unaligned); the few elements before and behind those pieces one per thread, by a load that is under way with the others.
// Loads past the last piece are redirected to it, so that none lies behind a branch that the threads may take apart: the compiler would wait for each.
// A thread meets its elements in rising index order, so "larger than the best so far" alone keeps the first of equal values, and the place is kept as
// the number of the element within the trip (a constant in the instruction): three instructions per element against eight for best_take, by which the scan was
// bound.  Elements equal to the start value, -inf, are not taken that way: where a thread ends without a place its wavefront goes through them again.
// us, before (rows of unaligned vocabularies by one element per load) -> now: 65 rows of 128255 bf16 12.8 -> 8.4, 21 of 30001 10.4 -> 5.9; batches of 8 requests: 520 rows
// of 128255 89.8 -> 27.6, 168 of 20001 14.2 -> 6.6 (and aligned: 65 of 128256 8.9 -> 8.2, 520 of them 29.8 -> 27.6).
// STREAM: read with the non-temporal hint.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ __forceinline__ u32x4 load_piece(const u32x4 *x)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(x);
    else return *x;
}
template <bool BF16, int T, int U, bool STREAM>
__device__ __forceinline__ Best span_scan(const void *logits, size_t base, int v0, int v1, int tid)
{
    constexpr int ES = BF16 ? 2 : 4, PER = 16 / ES;              // element size, elements per piece
    const unsigned char *first = static_cast<const unsigned char *>(logits) + (base + v0) * ES;
    const int n = v1 - v0, head = min((PER - (int)((reinterpret_cast<uintptr_t>(first) & 15) / ES)) & (PER - 1), n);
    const int P = (n - head) / PER, tail = n - head - P * PER;
    const u32x4 *x = reinterpret_cast<const u32x4 *>(first + head * ES);
    const int ve = tid < head ? v0 + tid : tid < head + tail ? v1 - tail + tid - head : v0;
    const float edge = load_one<BF16>(logits, base + ve);
    Best b = { -INFINITY, INT_MAX };
    auto pass = [&](auto exact) {
        for (int h = 0; h < P; h += U * T) {                     // (uniform)
            u32x4 q[U];
            if (h + U * T <= P) {
#pragma unroll
                for (int j = 0; j < U; ++j) q[j] = load_piece<STREAM>(x + h + j * T + tid);
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) q[j] = load_piece<STREAM>(x + min(h + j * T + tid, P - 1));
            }
            auto place = [&](int k) { return v0 + head + min(h + k / PER * T + tid, P - 1) * PER + k % PER; };
            float bv = b.v;
            int bk = -1;
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t wds[4] = { q[j][0], q[j][1], q[j][2], q[j][3] };
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const float f = !BF16 ? __uint_as_float(wds[e & 3]) : e & 1 ? __uint_as_float(wds[e / 2] & 0xFFFF0000u) : __uint_as_float(wds[e / 2] << 16);
                    if constexpr (decltype(exact)::value) best_take(b, f, place(j * PER + e));
                    else if (f > bv) { bv = f; bk = j * PER + e; }
                }
            }
            if (bk >= 0) { b.v = bv; b.i = place(bk); }
        }
    };
    pass(std::false_type{});
    if (P > 0 && __builtin_amdgcn_ballot_w64(b.i == INT_MAX) != 0ull) {
        b = Best{ -INFINITY, INT_MAX };
        pass(std::true_type{});
    }
    if (tid < head + tail) best_take(b, edge, ve);
    return b;
}

// grid = (chunks, rows).  part[(row*chunks + chunk)] = best of the chunk.
template <bool BF16, bool STREAM>
__global__ __launch_bounds__(256) void argmax_chunks(const void *logits, int V, Best *part)
{
    __shared__ Best wb[4];
    const int tid = threadIdx.x, chunk = blockIdx.x, row = blockIdx.y;
    Best b = best_wave(span_scan<BF16, 256, BF16 ? 4 : 8, STREAM>(logits, (size_t)row * V, chunk * ACHUNK, min(chunk * ACHUNK + ACHUNK, V), tid));
    if ((tid & 63) == 0) wb[tid >> 6] = b;
    __syncthreads();
    if (tid == 0) {
        Best r = wb[0];
        best_take(r, wb[1].v, wb[1].i); best_take(r, wb[2].v, wb[2].i); best_take(r, wb[3].v, wb[3].i);
        part[(size_t)row * gridDim.x + chunk] = r;
    }
}

// ------------------------------------------------------------------------------------------------
// Greedy acceptance of one request in one launch.  A wavefront scans one unit of WCHUNK vocabulary elements of one
// row; the waves of a workgroup fold the units that belong to the same row and leave one 64-bit key per row they
// touched in the workgroup's own slots of the workspace.  The workgroup with the highest index (the last one to be
// placed on the chip) then collects: it takes every slot with an atomic exchange against zero, again while a slot
// is still empty, merges the keys per row and walks the tree on its first wavefront.  Nobody else waits for
// anything, so every wait of the collector ends as soon as the other workgroups have run; a wall-clock limit
// (s_memrealtime) bounds it all the same, and running into it raises the workspace's flag.  The exchange leaves the
// slots at zero for the next call.
// The L2 caches of the 8 XCDs are not coherent with each other, and a device-scope fence writes back and
// invalidates a whole cache; the only words other workgroups must see are the slots, moved by relaxed device-scope
// atomics (executed at the memory side).  Counting the workgroups in instead (each waits for its key updates to be
// acknowledged, adds itself to a counter, the last one reads the keys) puts three dependent round trips to the
// memory side, about 2 us each, behind the scan; here it is the flight of a store and one exchange.
// Key = value bits made monotonic << 32 | ~index: the larger value wins, then the lower index; a key's upper half is
// never zero, so 1 stands for "only NaN seen": a row without a key has argmax 0, as in the two-launch path.
// The walk keeps node c in lane c % 64, register row c / 64: `ok` = the node's token is the target's argmax at its
// parent; a step is a ballot over "child of the current node and ok" per row, lowest node index first.
// ------------------------------------------------------------------------------------------------
constexpr int WALK_ROWS = (BTV_MAX_NODES + 63) / 64;
constexpr int WCHUNK = 4096;     // vocabulary elements per wavefront unit of the one-launch kernel
constexpr int OL_WAVES = 8;      // wavefronts per workgroup of the one-launch kernel (16: 8.7 us at 65 rows, 8: 7.7 us)
static_assert(OL_WAVES * 64 > BTV_MAX_NODES, "the collector gives every logit row a thread");
constexpr unsigned long long OL_NO_KEY = 1ull;
constexpr long long OL_WAIT_TICKS = 100000000ll;    // collector's limit: one second of the 100 MHz wall clock

// The walk, by one wavefront: t[r] = argmax of row r (in LDS), lane l holds nodes l, 64 + l, ... (par INT_MIN: none).
__device__ __forceinline__ void walk_tree(const int *t, const int (&par)[WALK_ROWS], const int (&tok)[WALK_ROWS], int M, int lane, int32_t *path,
                                          int32_t *n_acc, int32_t *bonus)
{
    bool ok[WALK_ROWS];
#pragma unroll
    for (int r = 0; r < WALK_ROWS; ++r) {
        const int c = r * 64 + lane;
        ok[r] = c < M && par[r] >= -1 && par[r] < M && tok[r] == t[par[r] + 1];
    }
    int cur = -1, n = 0;
    while (n < M) {
        int nx = -1;
#pragma unroll
        for (int r = WALK_ROWS - 1; r >= 0; --r) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(ok[r] && par[r] == cur);
            if (m != 0ull) nx = r * 64 + __builtin_ctzll(m);
        }
        if (nx < 0) break;
        if (lane == 0) path[n] = nx;
        cur = nx;
        ++n;
    }
    if (lane == 0) { *n_acc = n; *bonus = t[cur + 1]; }
}

// Rows that OL_WAVES consecutive units can touch: the slots a workgroup owns.
__host__ __device__ inline int ol_slots_per_wg(int chunks)
{
    const int r = (OL_WAVES - 1) / chunks + 2;
    return r < OL_WAVES ? r : OL_WAVES;
}

__device__ __forceinline__ unsigned long long best_key(Best b)
{
    if (b.i == INT_MAX) return 0ull;
    const uint32_t u = __float_as_uint(b.v + 0.0f);              // -0 counts as +0
    const uint32_t mono = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)mono << 32) | (uint32_t)~(uint32_t)b.i;
}

template <bool BF16>
__global__ __launch_bounds__(OL_WAVES * 64) void accept_greedy_one_launch(
    const void *logits, int V, int chunks, unsigned long long *slot, uint32_t *flag, const int32_t *parent,
    const int32_t *token, int M, int32_t *path, int32_t *n_acc, int32_t *bonus, int32_t *argmax_out, long long wait_ticks)
{
    __shared__ Best wbest[OL_WAVES];
    __shared__ int wrow[OL_WAVES];
    __shared__ int t[BTV_MAX_NODES + 1];
    __shared__ unsigned long long rowmax[BTV_MAX_NODES + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, units = (M + 1) * chunks;
    const int RS = ol_slots_per_wg(chunks);
    const bool collector = blockIdx.x == gridDim.x - 1;
    // the collector's walk needs the tree: asked for now, used after the scan
    int par[WALK_ROWS], tok[WALK_ROWS];
#pragma unroll
    for (int r = 0; r < WALK_ROWS; ++r) {
        const int c = r * 64 + lane;
        const bool mine = collector && wave == 0 && c < M;
        par[r] = mine ? parent[c] : INT_MIN;
        tok[r] = mine ? token[c] : -1;
    }
    {
        const int u = blockIdx.x * OL_WAVES + wave;              // (the grid covers the units exactly once)
        Best b = { -INFINITY, INT_MAX };
        int row = -1;
        if (u < units) {
            row = u / chunks;
            const int chunk = u - row * chunks;
            b = best_wave(span_scan<BF16, 64, 8, false>(logits, (size_t)row * V, chunk * WCHUNK, min(chunk * WCHUNK + WCHUNK, V), lane));
        }
        if (lane == 0) { wbest[wave] = b; wrow[wave] = row; }
        if (collector)
            for (int i = tid; i <= M; i += OL_WAVES * 64) rowmax[i] = 0ull;
        __syncthreads();
        if (tid < OL_WAVES && wrow[tid] >= 0 && (tid == 0 || wrow[tid - 1] != wrow[tid])) {
            // first unit of a row within this workgroup: fold the row's other units, leave the key
            Best r = wbest[tid];
            for (int j = tid + 1; j < OL_WAVES && wrow[j] == wrow[tid]; ++j) best_take(r, wbest[j].v, wbest[j].i);
            const unsigned long long key = best_key(r);
            __hip_atomic_store(slot + (size_t)blockIdx.x * RS + (wrow[tid] - wrow[0]), key != 0ull ? key : OL_NO_KEY,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (!collector) return;
    // workgroup w owns units OL_WAVES w .. OL_WAVES (w + 1) - 1 (as far as they exist); its slot j belongs to row
    // (OL_WAVES w) / chunks + j
    {
        const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
        bool late = wait_ticks < 0;                              // (a negative limit: give up at once, for tests of this path)
        for (int s = tid; s < (int)gridDim.x * RS && !late; s += OL_WAVES * 64) {
            const int w = s / RS, j = s - w * RS;
            const int r0 = (w * OL_WAVES) / chunks, r1 = min(w * OL_WAVES + OL_WAVES - 1, units - 1) / chunks;
            if (j > r1 - r0) continue;
            unsigned long long key = 0ull;
            for (;;) {
                key = __hip_atomic_exchange(slot + s, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (key != 0ull) break;
                if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > wait_ticks) { late = true; break; }
                __builtin_amdgcn_s_sleep(8);
            }
            if (key > 0xFFFFFFFFull) atomicMax(&rowmax[r0 + j], key);
        }
        if (late) atomicOr(flag, 128u);
    }
    __syncthreads();
    if (tid <= M) {
        const unsigned long long key = rowmax[tid];
        t[tid] = key == 0ull ? 0 : (int)~(uint32_t)key;
        if (argmax_out) argmax_out[tid] = t[tid];
    }
    __syncthreads();
    if (tid >= 64) return;
    walk_tree(t, par, tok, M, lane, path, n_acc, bonus);
}

// The same where one workgroup takes all rows at once: vocabularies of up to 4 LPR tokens, LPR neighbouring lanes per row and up to
// SMALL_PASSES rows per lane, all loads in flight before the first is looked at.  The maxima meet in LDS, so nothing goes through the
// workspace and nobody waits: what remains is a launch, a memory round trip and the walk (17 x 64 fp32: 4.8 us by accept_greedy_one_launch,
// 2.6 by this).  A pass is 0.9 us, so that three passes are the most that gain (us by one launch / by this, at one, two, three and
// four passes: 64 tokens 4.7 / 2.6, 4.9 / 3.5, 4.6 / 4.3, 5.1 / 5.2; 128 tokens 4.5 / 2.7, 4.6 / 3.6, 4.6 / 4.5, 4.8 / 5.6; 256 tokens 4.5 / 2.8 at
// one, 4.8 / 4.8 at three, 4.6 / 5.9 at four).  More than 4 tokens per lane gain for a handful of rows only: 512 tokens, 17 rows 5.0 / 7.3.
constexpr int SMALL_PASSES = 3, SMALL_THREADS = 512;
template <bool BF16, int LPR>
__global__ __launch_bounds__(SMALL_THREADS) void accept_greedy_small(const void *logits, int V, const int32_t *parent, const int32_t *token, int M,
                                                                     int32_t *path, int32_t *n_acc, int32_t *bonus, int32_t *argmax_out)
{
    constexpr int RPP = SMALL_THREADS / LPR;                     // rows per pass
    __shared__ int t[BTV_MAX_NODES + 1];
    const int tid = threadIdx.x, lane = tid & 63, l = tid % LPR, r0 = tid / LPR;
    int par[WALK_ROWS], tok[WALK_ROWS];
#pragma unroll
    for (int r = 0; r < WALK_ROWS; ++r) {
        const int c = r * 64 + lane;
        const bool mine = tid < 64 && c < M;
        par[r] = mine ? parent[c] : INT_MIN;
        tok[r] = mine ? token[c] : -1;
    }
    float x[SMALL_PASSES][4];
#pragma unroll
    for (int p = 0; p < SMALL_PASSES; ++p)
        if (p * RPP <= M)                                        // (uniform)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = p * RPP + r0, v = l + LPR * i;
                x[p][i] = load_one<BF16>(logits, row <= M && v < V ? (size_t)row * V + v : 0);
            }
#pragma unroll
    for (int p = 0; p < SMALL_PASSES; ++p)
        if (p * RPP <= M) {
            const int row = p * RPP + r0;
            Best b = { -INFINITY, INT_MAX };
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (l + LPR * i < V) best_take(b, x[p][i], l + LPR * i);
            for (int off = LPR / 2; off >= 1; off >>= 1) {
                const float ov = __shfl_xor(b.v, off);
                const int oi = __shfl_xor(b.i, off);
                best_take(b, ov, oi);
            }
            if (l == 0 && row <= M) {
                t[row] = b.i == INT_MAX ? 0 : b.i;
                if (argmax_out) argmax_out[row] = t[row];
            }
        }
    __syncthreads();
    if (tid >= 64) return;
    walk_tree(t, par, tok, M, lane, path, n_acc, bonus);
}

// Lanes per row of accept_greedy_small, 0 where it does not take a call.
int small_lanes(int M, int V)
{
    const int lpr = V <= 64 ? 16 : V <= 128 ? 32 : V <= 256 ? 64 : 0;
    return lpr && M + 1 <= SMALL_PASSES * (SMALL_THREADS / lpr) ? lpr : 0;
}

template <bool BF16>
void small_launch(int lpr, const void *logits, int V, const int32_t *parent, const int32_t *token, int M, int32_t *path, int32_t *n_acc,
                  int32_t *bonus, int32_t *argmax_out, hipStream_t st)
{
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(1), dim3(SMALL_THREADS), 0, st, logits, V, parent, token, M, path, n_acc, bonus, argmax_out); };
    if (lpr == 16) go(accept_greedy_small<BF16, 16>);
    else if (lpr == 32) go(accept_greedy_small<BF16, 32>);
    else go(accept_greedy_small<BF16, 64>);
}

// One workgroup per request of a batch: finish the argmax of every row, then walk the tree.  Request r owns nodes
// q_offset[r] .. q_offset[r+1] - 1 and logit rows q_offset[r] + r .. q_offset[r+1] + r (its root row first).
// A row's partials are read by as many lanes as there are of them (64 at most), eight or four reads in flight per lane; what
// is left is latency (a wavefront per request that walked with workgroup barriers after a thread per row: 5.4 us, now 3.6 at 65 rows).
constexpr int GW_WAVES = 16;
__global__ __launch_bounds__(GW_WAVES * 64) void greedy_walk(const Best *part, int chunks, const int32_t *parent,
                                                   const int32_t *token, int M, int32_t *path, int32_t *n_acc,
                                                   int32_t *bonus, int32_t *argmax_out, const int32_t *q_offset,
                                                   int total_M, uint32_t *flag)
{
    __shared__ int t[BTV_MAX_NODES + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rq = blockIdx.x, o0 = q_offset[rq], m = q_offset[rq + 1] - o0;
    n_acc += rq; bonus += rq;
    // M = the largest request the caller announced; a request may not reach past the total_M rows of the arrays
    if (o0 < 0 || m < 1 || m > M || (long long)o0 + m > (long long)total_M) {
        if (tid == 0) { atomicOr(flag, 32u); *n_acc = 0; *bonus = 0; }
        return;
    }
    M = m;
    part += (size_t)(o0 + rq) * chunks;
    parent += o0; token += o0; path += o0;
    if (argmax_out) argmax_out += o0 + rq;
    int par[WALK_ROWS], tok[WALK_ROWS];
#pragma unroll
    for (int r = 0; r < WALK_ROWS; ++r) {
        const int c = r * 64 + lane;
        const bool mine = wave == 0 && c < M;
        par[r] = mine ? parent[c] : INT_MIN;
        tok[r] = mine ? token[c] : -1;
    }
    const int lg = chunks >= 64 ? 6 : chunks <= 1 ? 0 : 32 - __builtin_clz(chunks - 1);
    const int per = 1 << lg, sub = lane & (per - 1), rsub = lane >> lg, step = GW_WAVES * (64 >> lg);    // lanes per row; rows per pass
    auto finish = [&](Best b, int row) {
        for (int off = 1; off < per; off <<= 1) {
            const float ov = __shfl_xor(b.v, off);
            const int oi = __shfl_xor(b.i, off);
            best_take(b, ov, oi);
        }
        if (sub == 0 && row <= M) {
            const int a = b.i == INT_MAX ? 0 : b.i;
            t[row] = a;
            if (argmax_out) argmax_out[row] = a;
        }
    };
    const int first = wave * (64 >> lg);
    if (chunks <= 64) {
        for (int r0 = first; r0 <= M; r0 += 4 * step) {        // four passes' reads in flight
            Best b[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) b[k] = part[(size_t)min(r0 + k * step + rsub, M) * chunks + min(sub, chunks - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                Best x = { -INFINITY, INT_MAX };
                best_take(x, b[k].v, b[k].i);
                if (r0 + k * step <= M) finish(x, r0 + k * step + rsub);
            }
        }
    } else {
        for (int r0 = first; r0 <= M; r0 += step) {            // (one row per wavefront)
            const Best *row = part + (size_t)r0 * chunks;
            Best x = { -INFINITY, INT_MAX };
            for (int c0 = 0; c0 < chunks; c0 += 8 * 64) {
                Best b[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) b[u] = row[min(c0 + u * 64 + lane, chunks - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) best_take(x, b[u].v, b[u].i);
            }
            finish(x, r0);
        }
    }
    __syncthreads();
    if (wave == 0) walk_tree(t, par, tok, M, lane, path, n_acc, bonus);
}

// part[chunk][row]: best of every row's per-chunk partials, 16 rows per workgroup (a line of 128 bytes per chunk), then the walk, by the
// workgroup that is done last (a launch of its own for that: 2 us more).  The rows' results cross the XCDs as relaxed device-scope
// atomics, which go through to memory; a workgroup counts itself in when its own have arrived.  done: 0 between calls.
constexpr int MERGE_ROWS = 16, MERGE_THREADS = 1024, MERGE_SUBS = MERGE_THREADS / MERGE_ROWS;
__global__ __launch_bounds__(MERGE_THREADS) void argmax_merge_walk(const Best *part, int chunks, unsigned long long *out, uint32_t *done, const int32_t *parent,
                                                                   const int32_t *token, int M, int32_t *path, int32_t *n_acc, int32_t *bonus,
                                                                   int32_t *argmax_out)
{
    __shared__ Best wb[MERGE_THREADS / 64][MERGE_ROWS];
    __shared__ int t[BTV_MAX_NODES + 1];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane % MERGE_ROWS, row = blockIdx.x * MERGE_ROWS + r, sub = tid / MERGE_ROWS;
    int par[WALK_ROWS], tok[WALK_ROWS];                        // (asked for now, by every workgroup; used by the last)
#pragma unroll
    for (int k = 0; k < WALK_ROWS; ++k) {
        const int c = k * 64 + lane;
        const bool mine = wave == 0 && c < M;
        par[k] = mine ? parent[c] : INT_MIN;
        tok[k] = mine ? token[c] : -1;
    }
    Best b = { -INFINITY, INT_MAX };
    for (int c0 = 0; c0 < chunks; c0 += 4 * MERGE_SUBS) {
        Best x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = part[(size_t)min(c0 + u * MERGE_SUBS + sub, chunks - 1) * (M + 1) + min(row, M)];
#pragma unroll
        for (int u = 0; u < 4; ++u) best_take(b, x[u].v, x[u].i);
    }
    auto over_subs = [&]() {                                   // of the lanes that have the same row
#pragma unroll
        for (int o = MERGE_ROWS; o < 64; o <<= 1) {
            const float ov = __shfl_xor(b.v, o);
            const int oi = __shfl_xor(b.i, o);
            best_take(b, ov, oi);
        }
    };
    over_subs();
    if (lane < MERGE_ROWS) wb[wave][lane] = b;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) best_take(b, wb[lane / MERGE_ROWS * 4 + k][r].v, wb[lane / MERGE_ROWS * 4 + k][r].i);
        over_subs();
        const int a = b.i == INT_MAX ? 0 : b.i;
        if (lane < MERGE_ROWS && row <= M) {
            if (argmax_out) argmax_out[row] = a;
            if (gridDim.x == 1) t[row] = a;
            else __hip_atomic_store(out + row, (unsigned long long)(uint32_t)a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (gridDim.x > 1) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) {
                last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
                if (last) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    __syncthreads();
    if (gridDim.x > 1) {
        if (!last) return;
        for (int k = tid; k <= M; k += MERGE_THREADS) t[k] = (int)(uint32_t)__hip_atomic_load(out + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
    if (wave == 0) walk_tree(t, par, tok, M, lane, path, n_acc, bonus);
}

constexpr int LM_DONE_WORD = 20;            // of the workspace's header: workgroups that have merged (0 between calls)

// workgroups of the one-launch greedy kernel: OL_WAVES units each, every unit once
int greedy_wgs(int M, int V)
{
    const long long chunks = (V + WCHUNK - 1) / WCHUNK;
    return (int)(((long long)(M + 1) * chunks + OL_WAVES - 1) / OL_WAVES);
}

int check_accept(const void *logits, int dtype, const int32_t *parent, const int32_t *token, int M, int V,
                 int32_t *path, int32_t *n_acc, int32_t *bonus)
{
    BTV_REQUIRE(logits && parent && token && path && n_acc && bonus, "null pointer");
    BTV_REQUIRE(dtype == BTV_F32 || dtype == BTV_BF16, "dtype=%d unsupported", dtype);
    BTV_REQUIRE(M >= 1 && M <= BTV_MAX_NODES, "M=%d outside [1,%d]", M, BTV_MAX_NODES);
    BTV_REQUIRE(V >= 1, "V=%d", V);
    return BTV_OK;
}

}  // namespace

extern "C" {

size_t btv_tree_accept_workspace(int M, int V, int stochastic)
{
    if (M < 1 || M > BTV_MAX_NODES || V < 1) return 0;
    if (stochastic) return btv_stochastic_workspace(V);
    const int chunks = (V + WCHUNK - 1) / WCHUNK;
    return BTV_WS_HEADER + btv_align_up((size_t)greedy_wgs(M, V) * ol_slots_per_wg(chunks) * sizeof(unsigned long long), BTV_WS_ALIGN);
}

int btv_tree_accept_greedy_tuned(const void *logits, int dtype, const int32_t *parent, const int32_t *token, int M, int V,
                                 int32_t *path, int32_t *n_acc, int32_t *bonus, int32_t *argmax_out, void *ws,
                                 size_t ws_bytes, void *stream, long long wait_ticks)
{
    int rc = check_accept(logits, dtype, parent, token, M, V, path, n_acc, bonus);
    if (rc) return rc;
    rc = btv_check_ws(ws, ws_bytes, btv_tree_accept_workspace(M, V, 0));
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned long long *slot = reinterpret_cast<unsigned long long *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER);
    uint32_t *flag = static_cast<uint32_t *>(ws);
    const int chunks = (V + WCHUNK - 1) / WCHUNK, wgs = greedy_wgs(M, V), lpr = small_lanes(M, V);
    if (lpr) {
        if (dtype == BTV_BF16) small_launch<true>(lpr, logits, V, parent, token, M, path, n_acc, bonus, argmax_out, st);
        else small_launch<false>(lpr, logits, V, parent, token, M, path, n_acc, bonus, argmax_out, st);
    } else if (dtype == BTV_BF16)
        hipLaunchKernelGGL(accept_greedy_one_launch<true>, dim3(wgs), dim3(OL_WAVES * 64), 0, st, logits, V, chunks, slot,
                           flag, parent, token, M, path, n_acc, bonus, argmax_out, wait_ticks);
    else
        hipLaunchKernelGGL(accept_greedy_one_launch<false>, dim3(wgs), dim3(OL_WAVES * 64), 0, st, logits, V, chunks, slot,
                           flag, parent, token, M, path, n_acc, bonus, argmax_out, wait_ticks);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

int btv_tree_accept_greedy(const void *logits, int dtype, const int32_t *parent, const int32_t *token, int M, int V,
                           int32_t *path, int32_t *n_acc, int32_t *bonus, int32_t *argmax_out, void *ws,
                           size_t ws_bytes, void *stream)
{
    return btv_tree_accept_greedy_tuned(logits, dtype, parent, token, M, V, path, n_acc, bonus, argmax_out, ws, ws_bytes, stream,
                                        OL_WAIT_TICKS);
}

size_t btv_tree_accept_lm_head_workspace(int M, int V)
{
    if (M < 1 || M > BTV_MAX_NODES || V < 1) return 0;
    const size_t rows = (size_t)M + 1;
    return BTV_WS_HEADER + btv_align_up(rows * ((V + 31) / 32) * sizeof(Best), BTV_WS_ALIGN) +
           btv_align_up(rows * sizeof(Best), BTV_WS_ALIGN);
}

int btv_tree_accept_greedy_lm_head(const void *hidden, const void *W, int h, const int32_t *parent, const int32_t *token,
                                   int M, int V, int32_t *path, int32_t *n_acc, int32_t *bonus, int32_t *argmax_out,
                                   void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(hidden && W && parent && token && path && n_acc && bonus, "null pointer");
    BTV_REQUIRE(M >= 1 && M <= BTV_MAX_NODES, "M=%d outside [1,%d]", M, BTV_MAX_NODES);
    BTV_REQUIRE(V >= 1, "V=%d", V);
    BTV_REQUIRE(h >= 128 && h % 128 == 0, "h=%d must be a positive multiple of 128", h);
    BTV_REQUIRE((reinterpret_cast<uintptr_t>(hidden) & 15) == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0,
                "hidden and W must be 16-byte aligned");
    int rc = btv_check_ws(ws, ws_bytes, btv_tree_accept_lm_head_workspace(M, V));
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int R = M + 1;
    const LmShares p = lm_shares(R, V);
    Best *part = reinterpret_cast<Best *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER);
    unsigned long long *best = reinterpret_cast<unsigned long long *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER +
                                          btv_align_up((size_t)R * ((V + 31) / 32) * sizeof(Best), BTV_WS_ALIGN));
    rc = lm_head_launch(p, hidden, W, R, h, V, part, st);
    if (rc) return rc;
    hipLaunchKernelGGL(argmax_merge_walk, dim3((R + MERGE_ROWS - 1) / MERGE_ROWS), dim3(MERGE_THREADS), 0, st, part, p.chunks, best,
                       static_cast<uint32_t *>(ws) + LM_DONE_WORD, parent, token, M, path, n_acc, bonus, argmax_out);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

size_t btv_tree_accept_batch_workspace(int batch, int total_M, int V)
{
    if (batch < 1 || total_M < 1 || V < 1) return 0;
    int chunks = (V + ACHUNK - 1) / ACHUNK;
    return BTV_WS_HEADER + btv_align_up(((size_t)total_M + batch) * chunks * sizeof(Best), BTV_WS_ALIGN);
}

int btv_tree_accept_greedy_batch(const void *logits, int dtype, const int32_t *parent, const int32_t *token,
                                 const int32_t *q_offset, int batch, int total_M, int M_max, int V, int32_t *path,
                                 int32_t *n_acc, int32_t *bonus, int32_t *argmax_out, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(logits && parent && token && q_offset && path && n_acc && bonus, "null pointer");
    BTV_REQUIRE(dtype == BTV_F32 || dtype == BTV_BF16, "dtype=%d unsupported", dtype);
    BTV_REQUIRE(batch >= 1 && total_M >= batch, "batch=%d, total_M=%d", batch, total_M);
    BTV_REQUIRE(M_max >= 1 && M_max <= BTV_MAX_NODES, "M_max=%d outside [1,%d]", M_max, BTV_MAX_NODES);
    BTV_REQUIRE(V >= 1, "V=%d", V);
    int rc = btv_check_ws(ws, ws_bytes, btv_tree_accept_batch_workspace(batch, total_M, V));
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Best *part = reinterpret_cast<Best *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER);
    const int chunks = (V + ACHUNK - 1) / ACHUNK, rows = total_M + batch;
    // Logits of 64 to 160 MiB, and of more than 288, are read past the caches.  us, through them / past them.  The product that wrote the logits has put its weights through the
    // last-level cache (256 MB) since, and most of them come from memory: 90 MB 24.4 / 24.2, 130 MB 29.7 / 29.5, 150 MB 33.8 / 32.3, 165 MB 36.0 / 34.4 (a vocabulary of 32000: 38.2 / 33.5), 310 MB
    // 62.7 / 54.9, 410 MB 78.1 / 71.9.  Passes over them in place in between (a scale, a bias, a mask, a cap) leave what fits in the cache: 90 MB 23.8 / 23.3, 165 MB 34.1 / 33.7, 310 MB 70.3 to 75.5 / 54.2
    // to 64.5.  From 190 to 285 MB it is a matter of the pass, which the call cannot know: behind the product 43.2 / 40.5 (210 MB), 52.3 / 47.4 (260 MB), but behind a scale or a division that follows it
    // 42.9 / 45.7 (230 MB), 46.9 / 54.6 (260 MB), 49.2 / 58.5 (275 MB), fp32 35.6 / 40.1 (190 MB), and where they are met again at once 35.5 / 37.0 (200 MB, 32000).  Below 64 MiB nothing is gained
    // behind the product (51 MB 18.1 / 18.4; 64 MB 20.2 / 20.0).  One request's logits (257 rows of 128256 floats are 132 MB) gained nothing behind it either.
    const unsigned long long bytes = (unsigned long long)rows * V * (dtype == BTV_BF16 ? 2 : 4);
    const bool stream_read = (bytes > (64ull << 20) && bytes <= (160ull << 20)) || bytes > (288ull << 20);
    const auto scan = dtype == BTV_BF16 ? (stream_read ? argmax_chunks<true, true> : argmax_chunks<true, false>)
                                        : (stream_read ? argmax_chunks<false, true> : argmax_chunks<false, false>);
    hipLaunchKernelGGL(scan, dim3(chunks, rows), dim3(256), 0, st, logits, V, part);
    BTV_HIP(hipGetLastError());
    hipLaunchKernelGGL(greedy_walk, dim3(batch), dim3(GW_WAVES * 64), 0, st, part, chunks, parent, token, M_max, path, n_acc, bonus,
                       argmax_out, q_offset, total_M, static_cast<uint32_t *>(ws));
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

}  // extern "C"
