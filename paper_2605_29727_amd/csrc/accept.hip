// Greedy acceptance on the GPU (gfx950): target argmax per tree row and the walk; also straight from the hidden states.
// (The rejection walk at temperature 1 is in stochastic.hip.)
//
// App. C "Acceptance" / Sec. 3.1: the committed tokens are the longest root-to-node path the
// target itself would have produced.  Rows of `logits`: 0 = root, 1+i = node i.
#include "btv_common.h"

#include <atomic>

#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>

namespace {

constexpr int ACHUNK = 8192;     // vocabulary elements per argmax workgroup

struct alignas(8) Best { float v; int i; };


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
template <bool BF16, int T, int U>
__device__ __forceinline__ Best span_scan(const void *logits, size_t base, int v0, int v1, int tid)
{
    constexpr int ES = BF16 ? 2 : 4, PER = 16 / ES;              // element size, elements per piece
    const unsigned char *first = static_cast<const unsigned char *>(logits) + (base + v0) * ES;
    const int n = v1 - v0, head = min((PER - (int)((reinterpret_cast<uintptr_t>(first) & 15) / ES)) & (PER - 1), n);
    const int P = (n - head) / PER, tail = n - head - P * PER;
    const uint4 *x = reinterpret_cast<const uint4 *>(first + head * ES);
    const int ve = tid < head ? v0 + tid : tid < head + tail ? v1 - tail + tid - head : v0;
    const float edge = load_one<BF16>(logits, base + ve);
    Best b = { -INFINITY, INT_MAX };
    auto pass = [&](auto exact) {
        for (int h = 0; h < P; h += U * T) {                     // (uniform)
            uint4 q[U];
            if (h + U * T <= P) {
#pragma unroll
                for (int j = 0; j < U; ++j) q[j] = x[h + j * T + tid];
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) q[j] = x[min(h + j * T + tid, P - 1)];
            }
            auto place = [&](int k) { return v0 + head + min(h + k / PER * T + tid, P - 1) * PER + k % PER; };
            float bv = b.v;
            int bk = -1;
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t wds[4] = { q[j].x, q[j].y, q[j].z, q[j].w };
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
template <bool BF16>
__global__ __launch_bounds__(256) void argmax_chunks(const void *logits, int V, Best *part)
{
    __shared__ Best wb[4];
    const int tid = threadIdx.x, chunk = blockIdx.x, row = blockIdx.y;
    Best b = best_wave(span_scan<BF16, 256, BF16 ? 4 : 8>(logits, (size_t)row * V, chunk * ACHUNK, min(chunk * ACHUNK + ACHUNK, V), tid));
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
            b = best_wave(span_scan<BF16, 64, 8>(logits, (size_t)row * V, chunk * WCHUNK, min(chunk * WCHUNK + WCHUNK, V), lane));
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

// One workgroup per request: finish the argmax of every row, then walk the tree.  With q_offset (a batch),
// request r owns nodes q_offset[r] .. q_offset[r+1] - 1 and logit rows q_offset[r] + r .. q_offset[r+1] + r (its
// root row first); without, there is one request of M nodes.
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
    if (q_offset) {
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
    }
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

// ------------------------------------------------------------------------------------------------
// LM head fused with the argmax (App. E: 2*s*h*V FLOPs and s*V activation elements for the logits;
// App. C "Acceptance": only their top-1 is used).  logit[r, v] = sum_k H[r, k] W[v, k] is formed on the
// matrix cores and reduced to one (value, token) pair per row and workgroup: the logits never reach
// memory, the 2*V*h bytes of W are streamed once.
//
// Transposed product, C^T = W_tile * H^T (v_mfma_f32_32x32x16_bf16): a wave owns 32
// vocabulary rows and every row of H, so a lane's accumulator registers run over vocabulary rows of
// one H row and the argmax is a per-lane scan.  The operand layout wants lane l to hold row l % 32,
// which as a direct load would touch 64 cache lines per instruction and use 16 bytes of each;
// instead every load instruction fetches whole row segments (8 or 16 lanes per row), and the block
// is turned round through a wave-private LDS tile.  H blocks [rows, KB] are shared by the waves
// through a double-buffered LDS slab.  All tiles store the 16-byte chunks of a row XOR-permuted by
// the row number, so operand reads (ds_read_b128, 16 lanes = 16 different rows) are conflict-free.
// ------------------------------------------------------------------------------------------------
typedef __bf16 lm_bf16x8 __attribute__((ext_vector_type(8)));
typedef float lm_f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int lm_u32x4 __attribute__((ext_vector_type(4)));

// VW waves side by side over the vocabulary times KW over the contraction (each takes every KW-th block of it, with a
// slab of H of its own; the sums meet in LDS at the end).
template <int RT, int VW, int KW, int KB>
struct LmShape {
    static constexpr int WAVES = VW * KW, THREADS = WAVES * 64, ROWS = RT * 32;
    static constexpr int GT = VW * 64;                    // threads that share a slab
    static constexpr int VROWS = 32;                      // vocabulary rows of a wave
    static constexpr int RB = KB * 2;                     // bytes of a tile row
    static constexpr int CPR = RB / 16;                   // 16-byte chunks per row
    static constexpr int WTILE = VROWS * RB, SLAB = ROWS * RB;
    static constexpr int LDS_BYTES = WAVES * WTILE + KW * 2 * SLAB;
    static constexpr int WLD = VROWS * CPR / 64;          // load instructions per wave and block for W
    static constexpr int HLD = (ROWS * CPR + GT - 1) / GT;             // chunks of the H slab per thread and block
    static constexpr bool HEVEN = ROWS * CPR % GT == 0;
    static constexpr int SUMS = (KW - 1) * VW * RT * 16 * 64 * 4; // accumulators handed over at the end
    static_assert(CPR == 8 || CPR == 16, "KB is 64 or 128");
    static_assert(LDS_BYTES <= 160 * 1024 && SUMS <= LDS_BYTES, "LDS of a CU");
    // byte offset of 16-byte chunk `col` of tile row `row`: 16 lanes reading one chunk index of 16 consecutive
    // rows must land in 16 different 16-byte bank groups of the 256-byte bank line
    __device__ static constexpr int at(int row, int col)
    {
        return row * RB + ((col ^ (CPR == 16 ? (row & 15) : ((row >> 1) & 7))) << 4);
    }
};

// One block of the contraction for a wave: KB / 16 steps of 1 + RT operand reads and RT MFMAs.  Here the
// reads are raw instructions with hand-placed waits (as ordinary loads each is waited for right before its MFMA,
// which leaves the matrix core idle for an LDS round trip): the reads of step j + 1 are issued before the MFMAs
// of step j, and the in-order counter tells when step j's have landed.
template <int RT>
__device__ __forceinline__ void lm_read_step(uint32_t wt, uint32_t hb, int tile_bytes, lm_u32x4 &a, lm_u32x4 (&b)[RT])
{
    asm volatile("ds_read_b128 %0, %1" : "=v"(a) : "v"(wt) : "memory");
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
        asm volatile("ds_read_b128 %0, %1" : "=v"(b[rt]) : "v"(hb + (uint32_t)(rt * tile_bytes)) : "memory");
}

template <int RT, int YOUNGER>
__device__ __forceinline__ void lm_wait_step(lm_u32x4 &a, lm_u32x4 (&b)[RT])
{
    static_assert(YOUNGER >= 0 && YOUNGER <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(YOUNGER) : "memory");
    asm volatile("" : "+v"(a));                                         // uses below may not move above the wait
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) asm volatile("" : "+v"(b[rt]));
}

// ob = offset of this lane's operand chunk at step 0 within a 32-row tile; step j sits at ob ^ (j << 5)
template <int RT, int KB, int RB>
__device__ __forceinline__ void lm_multiply(uint32_t wt, uint32_t hb, uint32_t ob, lm_f32x16 (&acc)[RT])
{
    constexpr int STEPS = KB / 16, N = 1 + RT;
    static_assert(N <= 15, "lgkmcnt range");
    lm_u32x4 a[2], b[2][RT];
    lm_read_step<RT>(wt + ob, hb + ob, 32 * RB, a[0], b[0]);
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (j + 1 < STEPS) {
            const uint32_t o = ob ^ (uint32_t)((j + 1) << 5);
            lm_read_step<RT>(wt + o, hb + o, 32 * RB, a[(j + 1) & 1], b[(j + 1) & 1]);
            lm_wait_step<RT, N>(a[j & 1], b[j & 1]);
        } else {
            lm_wait_step<RT, 0>(a[j & 1], b[j & 1]);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(lm_bf16x8, a[j & 1]),
                                                              __builtin_bit_cast(lm_bf16x8, b[j & 1][rt]), acc[rt], 0, 0, 0);
    }
}

// The same block with ordinary loads, scheduled by the compiler: leaner in registers, used when the accumulators
// of many row tiles leave no room for a second set of operands.
template <int RT, int KB, int RB>
__device__ __forceinline__ void lm_multiply_plain(const unsigned char *wt, const unsigned char *hb, uint32_t ob,
                                                  lm_f32x16 (&acc)[RT])
{
#pragma unroll
    for (int j = 0; j < KB / 16; ++j) {
        const uint32_t o = ob ^ (uint32_t)(j << 5);
        const lm_u32x4 a = *reinterpret_cast<const lm_u32x4 *>(wt + o);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const lm_u32x4 b = *reinterpret_cast<const lm_u32x4 *>(hb + rt * 32 * RB + o);
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(lm_bf16x8, a), __builtin_bit_cast(lm_bf16x8, b), acc[rt], 0, 0, 0);
        }
    }
}

template <int RT, int VW, int KW, int KB, bool RAW>
__global__ __launch_bounds__(VW * KW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void lm_head_argmax(
    const uint16_t *__restrict__ H, const uint16_t *__restrict__ W, int R, int h, int V, int chunks, int groups, Best *__restrict__ part)
{
    using S = LmShape<RT, VW, KW, KB>;
    extern __shared__ __align__(16) unsigned char lm_lds[];
    // Workgroup = a chunk of the vocabulary times a group of rows; the groups of one chunk stream the same weights and
    // get ids that are congruent mod 8, i.e. one XCD's L2.
    const int group = (int)(blockIdx.x >> 3) % groups, chunk = (int)(blockIdx.x >> 3) / groups * 8 + (int)(blockIdx.x & 7);
    if (chunk >= chunks) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r32 = lane & 31, half = lane >> 5;
    const int vw = wave % VW, kw = __builtin_amdgcn_readfirstlane(wave / VW), gtid = tid - kw * S::GT, r0 = group * S::ROWS;
    const int vwg = chunk * VW * S::VROWS, v0 = vwg + vw * S::VROWS;
    unsigned char *wtile = lm_lds + wave * S::WTILE;
    unsigned char *slab = lm_lds + S::WAVES * S::WTILE + kw * 2 * S::SLAB;
    const int nkb = h / KB, rounds = (nkb + KW - 1) / KW;
    const int own = KW == 1 ? nkb : (nkb - kw + KW - 1) / KW;      // this wave's blocks of the contraction: kw, kw + KW, ... (may be none)

    // Addresses are a wave-uniform base (block of the contraction, first row of the workgroup) plus a 32-bit
    // per-lane offset that never changes.
    // W: instruction i moves rows i*(64/CPR) .. of the wave's tile, CPR lanes per row
    constexpr int RPI = 64 / S::CPR;                       // rows per load instruction
    const int wcol = lane % S::CPR, wrow0 = lane / S::CPR;
    const unsigned char *wbase = reinterpret_cast<const unsigned char *>(W) + (size_t)vwg * h * 2 + (own ? kw : 0) * (KB * 2);
    const unsigned char *hbase = reinterpret_cast<const unsigned char *>(H) + (own ? kw : 0) * (KB * 2);
    uint32_t woff[S::WLD], hoff[S::HLD];
    // LDS destinations: rows 16 apart share the swizzle, so only the first 16 / RPI of a tile's store addresses
    // differ by more than a constant
    constexpr int WDN = 16 / RPI < S::WLD ? 16 / RPI : S::WLD;
    int wdst[WDN];
#pragma unroll
    for (int i = 0; i < S::WLD; ++i) {
        const int row = i * RPI + wrow0;
        woff[i] = (uint32_t)(min(v0 + row, V - 1) - vwg) * (uint32_t)(h * 2) + wcol * 16;
        if (i < WDN) wdst[i] = S::at(row, wcol);
    }
    // H: chunk c of the slab -> row c / CPR, column c % CPR
#pragma unroll
    for (int i = 0; i < S::HLD; ++i) {
        const int c = gtid + i * S::GT, row = c / S::CPR, col = c % S::CPR;
        hoff[i] = (uint32_t)min(r0 + row, R - 1) * (uint32_t)(h * 2) + col * 16;
    }
    // a thread's chunks are GT / CPR rows apart; where that is no multiple of 16 (whose swizzle is the same), each has its place
    constexpr int HSTEP = S::GT / S::CPR;
    constexpr bool HEVENLY = HSTEP % 16 == 0;
    const int hrow0 = gtid / S::CPR, hcol0 = gtid % S::CPR, hdst0 = S::at(hrow0, hcol0);
    // operand reads: step j of a block uses chunk 2j + half of row r32 (same chunk on both sides), which sits at
    // at(r32, half) ^ (j << 5): the swizzle is an XOR and 2j + half = 2j ^ half
    const uint32_t ob = (uint32_t)S::at(r32, half);

    lm_f32x16 acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[rt][e] = 0.f;

    // Workgroups start at different blocks of the contraction and wrap round: rows of W are a multiple of 4 KB
    // apart, so workgroups marching in step would all hit the same few memory channels.
    const int wrap = own ? own : 1;
    int curw = (chunk * 5) % wrap, curh = curw;
    // (staging arrays are of a native vector type: arrays of the uint4 struct were left in scratch memory)
#define LM_FETCH_W(w)                                                                                      \
    {                                                                                                      \
        const unsigned char *b_ = wbase + (size_t)curw * (KW * KB * 2);                                         \
        curw = curw + 1 == wrap ? 0 : curw + 1;                                                             \
        _Pragma("unroll") for (int i = 0; i < S::WLD; ++i) w[i] = *reinterpret_cast<const lm_u32x4 *>(b_ + woff[i]); \
    }
#define LM_FETCH_H(x)                                                                                      \
    {                                                                                                      \
        const unsigned char *b_ = hbase + (size_t)curh * (KW * KB * 2);                                         \
        curh = curh + 1 == wrap ? 0 : curh + 1;                                                             \
        _Pragma("unroll") for (int i = 0; i < S::HLD; ++i) x[i] = *reinterpret_cast<const lm_u32x4 *>(b_ + hoff[i]); \
    }
#define LM_STORE_W(w)                                                                                   \
    {                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < S::WLD; ++i)                                              \
            *reinterpret_cast<lm_u32x4 *>(wtile + wdst[i % WDN] + (i / WDN) * 16 * S::RB) = w[i];       \
    }
#define LM_STORE_H(x, dst)                                                                              \
    {                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < S::HLD; ++i)                                              \
            if (S::HEVEN || hrow0 + i * HSTEP < S::ROWS)   /* past the slab: fetched, never stored */   \
                *reinterpret_cast<lm_u32x4 *>((dst) + (HEVENLY ? hdst0 + i * HSTEP * S::RB : S::at(hrow0 + i * HSTEP, hcol0))) = x[i]; \
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) void *)lm_lds);
    const uint32_t wt_addr = lds0 + wave * S::WTILE, slab_addr = lds0 + S::WAVES * S::WTILE + kw * 2 * S::SLAB;
#define LM_MULTIPLY(sl)                                                                                      \
    {                                                                                                        \
        if constexpr (RAW) lm_multiply<RT, KB, S::RB>(wt_addr, slab_addr + (sl) * S::SLAB, ob, acc);         \
        else lm_multiply_plain<RT, KB, S::RB>(wtile, slab + (sl) * S::SLAB, ob, acc);                        \
    }

    // While block t is multiplied from LDS, the weights of blocks t + 1 and t + 2 are in registers or on their way
    // (they come from HBM); H comes from the L2 and is fetched one block ahead.  Fetches past the end wrap round to
    // blocks already seen; they land where nobody reads.
    lm_u32x4 w0[S::WLD], w1[S::WLD], x[S::HLD];
    LM_FETCH_W(w0)
    LM_FETCH_H(x)
    LM_FETCH_W(w1)
    LM_STORE_H(x, slab)
    LM_STORE_W(w0)
    __syncthreads();
    for (int kb = 0; kb + 1 < rounds; kb += 2) {
        // even round: slab 0 and the W tile hold block kb, w1 block kb + 1
        LM_FETCH_H(x)                                   // block kb + 1
        LM_FETCH_W(w0)                                  // block kb + 2
        if (KW == 1 || kb < own) LM_MULTIPLY(0)
        LM_STORE_H(x, slab + S::SLAB)                   // slab 1 is idle in this round
        LM_STORE_W(w1)                                  // own W tile: consumed by the multiply above
        __syncthreads();
        LM_FETCH_H(x)                                   // block kb + 2
        LM_FETCH_W(w1)                                  // block kb + 3
        if (KW == 1 || kb + 1 < own) LM_MULTIPLY(1)
        LM_STORE_H(x, slab)
        LM_STORE_W(w0)
        __syncthreads();
    }
    if (rounds & 1) {                                   // the last block of an odd count sits in slab 0
        if (KW == 1 || rounds - 1 < own) LM_MULTIPLY(0)
        __syncthreads();
    }
#undef LM_MULTIPLY
#undef LM_FETCH_W
#undef LM_FETCH_H
#undef LM_STORE_W
#undef LM_STORE_H

    // per-lane scan over the 16 vocabulary rows of a tile that it holds (ascending), other half, then the waves
    if constexpr (KW > 1) {                                 // the sums of the other parts of the contraction
        float *ex = reinterpret_cast<float *>(lm_lds) + vw * (RT * 16 * 64) + lane;
        constexpr int PLANE = VW * RT * 16 * 64;
        if (kw > 0) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int e = 0; e < 16; ++e) ex[(kw - 1) * PLANE + (rt * 16 + e) * 64] = acc[rt][e];
        }
        __syncthreads();
        if (kw == 0) {
#pragma unroll
            for (int k = 0; k < KW - 1; ++k)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[rt][e] += ex[k * PLANE + (rt * 16 + e) * 64];
        }
        __syncthreads();
    }
    Best *wb = reinterpret_cast<Best *>(lm_lds);            // [VW][ROWS]
    static_assert(S::LDS_BYTES >= VW * S::ROWS * (int)sizeof(Best), "exchange area must fit");
    if (KW == 1 || kw == 0)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        Best b = { -INFINITY, INT_MAX };
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int v = v0 + (e >> 2) * 8 + half * 4 + (e & 3);
            if (v < V) best_take(b, acc[rt][e], v);
        }
        const float ov = __shfl_xor(b.v, 32);
        const int oi = __shfl_xor(b.i, 32);
        best_take(b, ov, oi);
        if (half == 0) wb[vw * S::ROWS + rt * 32 + r32] = b;
    }
    __syncthreads();
    for (int row = tid; row < min(R - r0, S::ROWS); row += S::THREADS) {
        Best b = wb[row];
#pragma unroll
        for (int w = 1; w < VW; ++w) best_take(b, wb[w * S::ROWS + row].v, wb[w * S::ROWS + row].i);
        part[(size_t)(r0 + row) * chunks + chunk] = b;
    }
}

// grid = rows: best of a row's per-workgroup partials -> out[row]; the workgroup that is done last walks the tree (a launch of
// its own for that: 2 us more).  The rows' results cross the XCDs as relaxed device-scope atomics, which go through to
// memory; a workgroup counts itself in when its own has arrived.  done: 0 between calls.
__global__ __launch_bounds__(256) void argmax_merge_walk(const Best *part, int chunks, unsigned long long *out, uint32_t *done, const int32_t *parent,
                                                         const int32_t *token, int M, int32_t *path, int32_t *n_acc, int32_t *bonus,
                                                         int32_t *argmax_out)
{
    __shared__ Best wb[4];
    __shared__ int t[BTV_MAX_NODES + 1];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, row = blockIdx.x;
    int par[WALK_ROWS], tok[WALK_ROWS];                        // (asked for now, by every workgroup; used by the last)
#pragma unroll
    for (int r = 0; r < WALK_ROWS; ++r) {
        const int c = r * 64 + lane;
        const bool mine = tid < 64 && c < M;
        par[r] = mine ? parent[c] : INT_MIN;
        tok[r] = mine ? token[c] : -1;
    }
    Best b = { -INFINITY, INT_MAX };
    for (int c = tid; c < chunks; c += 256) best_take(b, part[(size_t)row * chunks + c].v, part[(size_t)row * chunks + c].i);
    b = best_wave(b);
    if (lane == 0) wb[tid >> 6] = b;
    __syncthreads();
    if (tid == 0) {
        Best r = wb[0];
        best_take(r, wb[1].v, wb[1].i); best_take(r, wb[2].v, wb[2].i); best_take(r, wb[3].v, wb[3].i);
        const int a = r.i == INT_MAX ? 0 : r.i;
        if (argmax_out) argmax_out[row] = a;
        __hip_atomic_store(out + row, (unsigned long long)(uint32_t)a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (last) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last) return;
    for (int r = tid; r <= M; r += 256) t[r] = (int)(uint32_t)__hip_atomic_load(out + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (tid < 64) walk_tree(t, par, tok, M, lane, path, n_acc, bonus);
}

constexpr int LM_ONE_WG = 3000;
constexpr int LM_DONE_WORD = 20;            // of the workspace's header: rows that are merged (0 between calls)

// Shape of the LM-head kernel for R rows of H: row tiles per workgroup (R may take several groups of them), waves over the
// vocabulary and over the contraction, contraction block, raw or compiler-scheduled operand reads (pipelined raw reads pay only
// while a second set of operands fits beside the accumulators).
struct LmPlan { int rt, vw, kw, kb, raw; };

// The shape with the least estimated time: what a workgroup's blocks of the contraction take (alone on a CU, and where the
// chip is full), times the rounds, no less than the stream of W, some of the smaller of the two on top, and the merge of
// what the workgroups leave.  Fitted to 84 problems (h = 1024 to 4096, V = 8k to 128k, 2 to 256 rows) times all shapes: half a
// percent behind the best shape on average.  The rule by the number of rows alone that it replaces (all rows in one workgroup, 4 or
// 8 waves side by side) was 34 % behind: it left most CUs without a workgroup at small vocabularies (196 rows, h = 4096,
// V = 8000: 32 workgroups, 138 us; 42 in four groups of rows) and streamed with few waves (h = 4096, V = 16k, one row: 40 us, 32
// with two waves over the contraction).
inline LmPlan lm_plan(int R, int h, int V)
{
    static constexpr struct { LmPlan p; float alone, full; int per_cu; } SHAPES[] = {      // us per 128 of the contraction
        { { 1, 4, 1, 128, 1 }, 0.622f, 1.045f, 2 }, { { 1, 2, 2, 128, 1 }, 0.670f, 1.237f, 2 },
        { { 2, 4, 1, 128, 1 }, 0.836f, 1.338f, 2 }, { { 2, 2, 2, 128, 1 }, 1.053f, 1.186f, 1 },
        { { 3, 4, 1, 128, 0 }, 0.993f, 1.850f, 2 }, { { 3, 8, 1, 128, 0 }, 1.628f, 1.802f, 1 },
        { { 4, 4, 1, 128, 0 }, 1.274f, 1.361f, 1 }, { { 4, 8, 1, 128, 0 }, 1.946f, 2.107f, 1 },
        { { 5, 8, 1, 128, 0 }, 2.185f, 2.354f, 1 }, { { 6, 8, 1, 128, 0 }, 2.579f, 2.787f, 1 },
        { { 7, 8, 1, 64, 0 }, 3.420f, 3.716f, 1 }, { { 8, 8, 1, 64, 0 }, 3.500f, 3.792f, 1 },
        { { 9, 8, 1, 64, 0 }, 3.900f, 4.250f, 1 },
    };
    const int tiles = (R + 31) / 32;
    const float mem = 2.0f * V * h / 7.0e6f;
    LmPlan best = SHAPES[0].p;
    float best_t = 0.f;
    for (const auto &s : SHAPES) {
        if (s.p.rt > tiles) continue;
        const int chunks = (V + s.p.vw * 32 - 1) / (s.p.vw * 32), groups = (tiles + s.p.rt - 1) / s.p.rt, wgs = (chunks + 7) / 8 * 8 * groups;
        const float blocks = (float)((h / s.p.kb + s.p.kw - 1) / s.p.kw * s.p.kb) / 128.f, fill = wgs / (256.f * s.per_cu);
        const float rounds = 0.45f * std::ceil(fill) + 0.55f * std::max(1.f, fill);
        const float comp = rounds * blocks * (wgs <= 256 ? s.alone : s.full);
        const float t = std::max(comp, mem) + 0.45f * std::min(comp, mem) + 1.1e-4f * chunks * R;
        if (!best_t || t < best_t) { best = s.p; best_t = t; }
    }
    return best;
}

inline int lm_chunks(const LmPlan &p, int V) { return (V + p.vw * 32 - 1) / (p.vw * 32); }

template <int RT, int VW, int KW, int KB, bool RAW>
int lm_head_launch(const uint16_t *H, const uint16_t *W, int R, int h, int V, Best *part, hipStream_t st)
{
    using S = LmShape<RT, VW, KW, KB>;
    static std::atomic<bool> configured{false};         // (one GPU per process: the attribute is set once)
    auto kern = lm_head_argmax<RT, VW, KW, KB, RAW>;
    if (!configured.load(std::memory_order_acquire)) {
        BTV_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    S::LDS_BYTES));
        configured.store(true, std::memory_order_release);
    }
    const int chunks = (V + VW * S::VROWS - 1) / (VW * S::VROWS), groups = (R + S::ROWS - 1) / S::ROWS;
    hipLaunchKernelGGL(kern, dim3((chunks + 7) / 8 * 8 * groups), dim3(S::THREADS), S::LDS_BYTES, st, H, W, R, h, V, chunks, groups, part);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

int lm_head_dispatch(const LmPlan &p, const uint16_t *H, const uint16_t *W, int R, int h, int V, Best *part, hipStream_t st)
{
#define LM_CASE(rt_, vw_, kw_, kb_, raw_)                                                             \
    if (p.rt == rt_ && p.vw == vw_ && p.kw == kw_ && p.kb == kb_ && p.raw == raw_)                    \
        return lm_head_launch<rt_, vw_, kw_, kb_, raw_ != 0>(H, W, R, h, V, part, st);
    LM_CASE(1, 4, 1, 128, 1) LM_CASE(2, 4, 1, 128, 1)
    LM_CASE(1, 2, 2, 128, 1) LM_CASE(2, 2, 2, 128, 1)
    LM_CASE(3, 4, 1, 128, 0) LM_CASE(4, 4, 1, 128, 0)
    LM_CASE(3, 8, 1, 128, 0)
    LM_CASE(4, 8, 1, 128, 0) LM_CASE(5, 8, 1, 128, 0) LM_CASE(6, 8, 1, 128, 0)
    LM_CASE(7, 8, 1, 64, 0) LM_CASE(8, 8, 1, 64, 0) LM_CASE(9, 8, 1, 64, 0)
#undef LM_CASE
    return btv_fail(BTV_EINVAL, "no LM-head kernel for %d rows", R);
}

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
    const LmPlan pl = lm_plan(R, h, V);
    const int chunks = lm_chunks(pl, V);
    Best *part = reinterpret_cast<Best *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER);
    unsigned long long *best = reinterpret_cast<unsigned long long *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER +
                                          btv_align_up((size_t)R * ((V + 31) / 32) * sizeof(Best), BTV_WS_ALIGN));
    const uint16_t *Hp = static_cast<const uint16_t *>(hidden), *Wp = static_cast<const uint16_t *>(W);
    rc = lm_head_dispatch(pl, Hp, Wp, R, h, V, part, st);
    if (rc) return rc;
    // one workgroup reads few partials itself; many take one per row (65000 took one workgroup 16 us)
    if ((long long)R * chunks > LM_ONE_WG)
        hipLaunchKernelGGL(argmax_merge_walk, dim3(R), dim3(256), 0, st, part, chunks, best, static_cast<uint32_t *>(ws) + LM_DONE_WORD, parent, token, M,
                           path, n_acc, bonus, argmax_out);
    else
        hipLaunchKernelGGL(greedy_walk, dim3(1), dim3(GW_WAVES * 64), 0, st, part, chunks, parent, token, M, path, n_acc, bonus, argmax_out,
                           static_cast<const int32_t *>(nullptr), 0, static_cast<uint32_t *>(nullptr));
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
    if (dtype == BTV_BF16) hipLaunchKernelGGL(argmax_chunks<true>, dim3(chunks, rows), dim3(256), 0, st, logits, V, part);
    else hipLaunchKernelGGL(argmax_chunks<false>, dim3(chunks, rows), dim3(256), 0, st, logits, V, part);
    BTV_HIP(hipGetLastError());
    hipLaunchKernelGGL(greedy_walk, dim3(batch), dim3(GW_WAVES * 64), 0, st, part, chunks, parent, token, M_max, path, n_acc, bonus,
                       argmax_out, q_offset, total_M, static_cast<uint32_t *>(ws));
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

}  // extern "C"
