// Stochastic acceptance on the GPU (gfx950): token-level rejection walk at temperature 1 (App. C "Acceptance", Sec. 2.1).
//
// The scalar form of a node.  With e[v] = exp(logit[v] - max), q[v] = the draft marginal of the depth and T = the draft
// mass not tried yet, the target distribution after some rejections is  p[v] = max(e[v] - s q[v], 0) / G(s)  with
//     G(s) = sum_v max(e[v] - s q[v], 0)        (s = 0 at first: the softmax)
// and the draft distribution of the untried tokens q[v] / T (a rejected token has p < q / T, so its residual is zero
// from then on and the same formula covers it).  A child with token x and uniform u is accepted iff
// u q[x] / T < p[x]; a rejection takes max(p - q / T, 0), which is  s <- s + G(s) / T,  T <- T - q[x]  (s stays where
// the new residual would be all zero).  All of s, G, T and the sums behind them are fp64; e is one fp32 exponential per token.
//
// One launch of G workgroups walks the tree together: workgroup w owns a contiguous slice of the vocabulary, and a
// thread keeps the (e, q) of its own tokens in registers for as long as the walk stays at a node.  What a node needs from
// all of them (row maximum and sums, one G(s) per rejection) is exchanged in the workspace: every workgroup leaves
// its part in words of its own, (tag << 32 | 32 bits of payload) so that a word says by itself whether it is this
// exchange's, and every workgroup reads all parts and does the same arithmetic on them in the same order, so that they
// all take the same decisions and nobody has to be told.  An exchange is one store and one load at the memory side
// (relaxed device-scope atomics: the L2s of the 8 XCDs are not coherent with each other), 1.5 us; two sets of words in turn are
// enough, because a workgroup writes exchange i + 2 only after it has read all of exchange i + 1, which everybody
// wrote after reading exchange i.  Tags count on from call to call (`base` in the workspace), so words are never cleared.
//
// The exchanges need all workgroups on the chip at once.  There are no more of them than CUs that the stream may use (the LDS
// holds one on a CU), and longer slices where those are few; but other work may hold the CUs, so nothing depends on it: a
// wait ends after `wait_ticks` of the wall clock, its workgroup leaves the exchanges, and the first to do so (it finds no claim
// of these tags in the workspace) walks the tree once more alone, over the whole vocabulary, and writes every result (workgroups
// that do get through write the same).  Then it moves `base` past all tags that a call can use.  A workgroup that only starts
// after that takes the new tags, finds nobody and does the same again, so whoever has written words under some tags, `base` is
// past them when the kernel ends, and the next call takes none of them for its own.  Alone the walk takes 4 to 12 ms at
// V = 128256, which is where the limit lies: 10 ms, so that waiting costs no more than it can save.
//
// A wide fan is not walked one exchange per rejection.  s_{k+1} = s_k + G(s_k) / T_k is a recurrence in one scalar, T_k is known
// beforehand, and G is convex and piecewise linear, G(s) = E - s Q with E, Q the sums of e and q over the tokens with
// e / q > s.  So all of s_1 .. s_K are found at once by Newton's method on the whole sequence: E and Q are evaluated at
// guesses for all s_k in one exchange, after which the recurrence is affine and is solved by a prefix scan; the guesses come from a table of
// G at 256 points (one exchange).  The error squares with every exchange (measured on normal logits and marginals:
// 5e-5 after the table, 1e-9 after one, rounding after two), and the sequence is taken when no s_k moved by more than
// 1e-7 of itself: what is left is second order then, below 1e-13, except for tokens whose kink (e = s q) lies within that
// last move, which E and Q count on the wrong side; such a token leaves at most 1e-7 of s times q / T, of the size of the
// rounding of e.  Anything that does not converge is walked one by one.
// For the evaluations a workgroup sorts its slice once by e / q into bins with prefix sums.
//
// What bounds it is latency: an exchange (1.5 us for one double, 2.5 for a chain's rows or for the sums at
// 128 points), the row loads in front of it (2 us), code that runs once per call.  Measured
// at V = 128256 (MI355X, one call after the other): 127 children under the root, all rejected, fp32: 124 -> 39 us against
// one workgroup that walked a row sorted by four launches ahead of it; a drafter whose target follows it for 7 to 12
// levels, bf16: 860 .. 1280 -> 29 .. 33 us against that workgroup's passes over every row (110 us per level).  Slices of 4096
// tokens instead of 2048 (half the workgroups): 52 and 48 .. 52 us at the same two.
#include "btv_common.h"

#include <algorithm>
#include <climits>

namespace {

typedef unsigned long long u64;

constexpr int SA_T = 1024, SA_WAVES = SA_T / 64;
constexpr int SA_MAX_WGS = 64;                          // slices: one lane of a wavefront per workgroup when parts are collected
constexpr int SA_BINS = 1024;                           // bins of e / q, 32 per binade upwards from the current s
constexpr int SA_GRID = 256;                            // points of the table that the first guesses come from
constexpr int SA_POINTS = BTV_MAX_NODES;                // points of an exchange
constexpr int SA_WORDS = 4 * SA_POINTS;                 // words of one workgroup's part: point k's two doubles at 4 k
constexpr int SA_CHAIN = 4;                             // rows of a first-child chain that are read and exchanged together
constexpr int SA_CHAIN_FAN = 8;                         // children up to which a node's first child is worth reading ahead (it is one of
                                                        // several that the draft likes about as well, otherwise)
// Up to so many workgroups run on one XCD (a grid eight times as large, of which all others but the stand-ins below leave at once), and their exchanges
// stay in its L2.  us, over memory / in the L2: 11 workgroups 39 children rejected 38.7 / 34.5, 16 of them 100 rejected 38.9 / 34.9, a followed draft 28.4 / 28.4 and
// 34.1 / 33.6 (what the exchanges gain its rows lose, which come through one XCD's share of the memory); 32 workgroups 37.8 / 34.0.
// A workgroup takes a CU for itself, of which an XCD has 32, and other work may hold them, another stream's walk for one.  So each slice has a
// stand-in as well, a workgroup on one of the seven other XCDs: it leaves when it sees that its slice has been taken, and takes it if that has not
// happened SA_START after its own start.  The first of the two that counts itself in (a word per slice; both of them do in every call, so that an even
// number is there at its start) has the slice, and the other one leaves whenever it starts.  A walk with a stand-in in it exchanges through memory.  The
// counting costs 0.5 us of 18 to 28 where the draft is followed and up to 0.3 of 35 in a fan; four streams of walks of 24 workgroups that meet on one XCD take 44 us
// a call instead of 62.  (The words on lines of their own: no gain.  The count looked at only behind the first rows' loads, for which it has to be held in a
// register through the loop: 1 us more.)
constexpr int SA_NEAR = 24;
constexpr int SA_BASE_WORD = 16, SA_TURN_WORD = 32;     // of the workspace's header: `base`; one word per slice
static_assert(SA_TURN_WORD + SA_NEAR <= BTV_WS_HEADER / 4, "the header holds them");
constexpr long long SA_START = 500ll;                   // 5 us
constexpr int SA_DIRECT = 3;                            // rejections that are walked one by one in any case, one less per 32 children
                                                        // (a node of many children has no likely one among its first)
constexpr int SA_BATCH_MIN = 10;                        // children left from which the rest is solved at once (the price of ten exchanges)
constexpr long long SA_WAIT_TICKS = 1000000ll;          // 10 ms of the 100 MHz wall clock
constexpr uint32_t SA_SPAN = 1u << 20;                  // more tags than a call can use (256 nodes of at most 18 + 256 exchanges)
static_assert(SA_GRID <= SA_POINTS, "all points of an exchange fit");

struct SaParams {
    const void *logits;
    const float *marg, *uniforms;
    const int32_t *parent, *token;
    int32_t *path, *n_acc, *bonus;
    uint32_t *flag, *base;
    u64 *claim;                                         // 1 << 32 | the tags' base of the last walk that was done alone
    u64 *slots;                                         // [2][G][SA_WORDS]
    int B, M, V, G, per;                                // per: tokens of a slice
    long long wait_ticks;
};

// Sum of x over the wavefront, returned in every lane: quad swaps, row mirrors, then the row totals travel down the
// rows (DPP moves of the two halves; lanes a step does not write add zero).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, true);
    return x + __longlong_as_double(((long long)(uint32_t)hi << 32) | (long long)(uint32_t)lo);
}
__device__ __forceinline__ double wave_sum(double x)
{
    x = dpp_add<0xB1, 0xF>(x);      // quad_perm [1,0,3,2]
    x = dpp_add<0x4E, 0xF>(x);      // quad_perm [2,3,0,1]
    x = dpp_add<0x141, 0xF>(x);     // row_half_mirror
    x = dpp_add<0x140, 0xF>(x);     // row_mirror: every lane holds its row's total
    x = dpp_add<0x142, 0xA>(x);     // row_bcast15 into rows 1 and 3
    x = dpp_add<0x143, 0xC>(x);     // row_bcast31 into rows 2 and 3: lane 63 holds the total
    const long long b = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (long long)lo);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max(float x)
{
    return fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp((int)0xFF800000u, __float_as_int(x), CTRL, ROW_MASK, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float x)
{
    x = dpp_max<0xB1, 0xF>(x);
    x = dpp_max<0x4E, 0xF>(x);
    x = dpp_max<0x141, 0xF>(x);
    x = dpp_max<0x140, 0xF>(x);
    x = dpp_max<0x142, 0xA>(x);
    x = dpp_max<0x143, 0xC>(x);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
// Inclusive prefix sums over the lanes: of a row of 16 lanes by its shifts, then the rows before.
__device__ __forceinline__ double wave_scan(double x)
{
    x = dpp_add<0x111, 0xF>(x);     // row_shr:1, 2, 4, 8
    x = dpp_add<0x112, 0xF>(x);
    x = dpp_add<0x114, 0xF>(x);
    x = dpp_add<0x118, 0xF>(x);
    x = dpp_add<0x142, 0xA>(x);     // row_bcast15 into rows 1 and 3
    return dpp_add<0x143, 0xC>(x);  // row_bcast31 into rows 2 and 3
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_add(int x) { return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROW_MASK, 0xF, true); }
__device__ __forceinline__ int wave_scan(int x)
{
    x = dpp_add<0x111, 0xF>(x); x = dpp_add<0x112, 0xF>(x); x = dpp_add<0x114, 0xF>(x); x = dpp_add<0x118, 0xF>(x);
    x = dpp_add<0x142, 0xA>(x);
    return dpp_add<0x143, 0xC>(x);
}
// x of another lane of the row, or of a row before; `none` where there is no such lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_of(float x, float none)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)__float_as_uint(none), (int)__float_as_uint(x), CTRL, ROW_MASK, 0xF, false));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_of(double x, double none)
{
    const u64 b = (u64)__double_as_longlong(x), n = (u64)__double_as_longlong(none);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)n, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(n >> 32), (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
// Composition of the affine maps of lanes 0 .. lane - 1 (lane 0 first): x -> A x + B.  (By moves between the lanes: through
// LDS, six round trips one after the other, the table's solution took 3.1 us instead of 2.6, a Newton step 1.4 instead of 1.2.)
template <typename F>
__device__ __forceinline__ void wave_affine_before(F a, F b, int lane, F &A, F &B)
{
#define BTV_STEP(CTRL, ROWS) { const F ao = dpp_of<CTRL, ROWS>(a, (F)1), bo = dpp_of<CTRL, ROWS>(b, (F)0); b = a * bo + b; a = a * ao; }
    BTV_STEP(0x111, 0xF) BTV_STEP(0x112, 0xF) BTV_STEP(0x114, 0xF) BTV_STEP(0x118, 0xF) BTV_STEP(0x142, 0xA) BTV_STEP(0x143, 0xC)
#undef BTV_STEP
    A = __shfl_up(a, 1); B = __shfl_up(b, 1);
    if (lane == 0) { A = (F)1; B = (F)0; }
}
// Sum over the 2^lg (up to 16) neighbouring lanes of a group.
__device__ __forceinline__ double group_sum(double x, int lg)
{
    x = dpp_add<0xB1, 0xF>(x);
    x = dpp_add<0x4E, 0xF>(x);
    if (lg > 2) x = dpp_add<0x141, 0xF>(x);
    if (lg > 3) x = dpp_add<0x140, 0xF>(x);
    return x;
}
// Sum of the first n (uniform) of one value per wavefront, in their order; all are read at once (one after the other they made the
// sort of a fan 5.3 us, with the scans through LDS; 3.9 now).
template <typename F>
__device__ __forceinline__ F sum_before(const F *x, int n)
{
    F t = (F)0;
#pragma unroll
    for (int i = 0; i < SA_WAVES; ++i) t += i < n ? x[i] : (F)0;
    return t;
}

template <bool BF16>
__device__ __forceinline__ float load_logit(const void *logits, size_t idx)
{
    if (BF16) return __uint_as_float((uint32_t)static_cast<const uint16_t *>(logits)[idx] << 16);
    return static_cast<const float *>(logits)[idx];
}

// N tokens of a row and of its marginals in pieces of four, v + step * i .. + 3 for i < N / 4; logits from v1 on come as -inf, marginals from
// vq on as 0.  v is a multiple of four, and so are v1 and vq unless they are the row's end: there the piece that the end cuts is loaded from V - 4 on
// and moved into place.  A row may begin at any element (the hardware takes such addresses).  All loads are issued before the first is looked at.
// A chain's rows are bound by how many loads 16 wavefronts issue: pieces are of the compiler's own vector types, because of float4, a structure, it
// takes the four floats, and merged their loads with those of a path by single tokens, four of 4 bytes for one of 16 (a draft followed over 7
// to 12 levels, 128256 tokens: bf16 35.8 -> 32.7 us, fp32 40.4 -> 32.9; a fan of 127 39.4 -> 38.8).  Rows of 128255 tokens by single tokens / by
// pieces: bf16 33.5 / 27.6, fp32 34.4 / 27.5; 60002 32.8 / 26.1; 3001 21.8 / 19.3; and with no second path 128256 took 31.0 / 30.1.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));
template <bool BF16, int N>
__device__ __forceinline__ void load_tokens(const void *row, const float *marg, int v, int step, int v1, int vq, int V, float (&e)[N], float (&q)[N])
{
    if (__builtin_expect(V >= 4, 1)) {                          // (uniform)
        u32x2 wb[N / 4];
        f32x4 wf[N / 4], wq[N / 4];
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const int at = v + step * i < v1 ? min(v + step * i, V - 4) : 0;
            if constexpr (BF16) wb[i] = *reinterpret_cast<const u32x2_any *>(static_cast<const uint16_t *>(row) + at);
            else wf[i] = *reinterpret_cast<const f32x4_any *>(static_cast<const float *>(row) + at);
        }
#pragma unroll
        for (int i = 0; i < N / 4; ++i) wq[i] = *reinterpret_cast<const f32x4_any *>(marg + (v + step * i < vq ? min(v + step * i, V - 4) : 0));
        const bool ragged = (V & 3) != 0 && v1 == V;           // (uniform) the row's last piece was loaded from V - 4 on
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const int at = v + step * i;
            float x[4], y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (BF16) x[k] = __uint_as_float(k & 1 ? wb[i][k / 2] & 0xFFFF0000u : wb[i][k / 2] << 16);
                else x[k] = wf[i][k];
                y[k] = wq[i][k];
            }
            if (ragged) {
#pragma unroll
                for (int s = 4; s > 1; --s)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const bool on = at + s > V;
                        x[k] = on ? x[k + 1] : x[k];
                        y[k] = on ? y[k + 1] : y[k];
                    }
#pragma unroll
                for (int k = 1; k < 4; ++k) {
                    x[k] = at + k < v1 ? x[k] : -INFINITY;
                    y[k] = at + k < vq ? y[k] : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e[4 * i + k] = at < v1 ? x[k] : -INFINITY;
                q[4 * i + k] = at < vq ? y[k] : 0.f;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int t = v + step * (i / 4) + i % 4;
            const float x = load_logit<BF16>(row, t < v1 ? t : 0), y = marg[t < vq ? t : 0];
            e[i] = t < v1 ? x : -INFINITY;
            q[i] = t < vq ? y : 0.f;
        }
    }
}

// e^x for x <= 0 to about one ulp: 2^(x log2(e)) with the rounding of the product, and of the constant, brought back in to
// first order (expf spends two thirds of its instructions on arguments that do not occur here).  Below 2^-126: 0.
__device__ __forceinline__ float exp_neg(float x)
{
    const float t = x * 1.44269502f;                    // log2(e) = 1.44269502 + 1.925963e-8
    const float lo = fmaf(x, 1.44269502f, -t) + x * 1.92596299e-8f;
    const float y = __builtin_amdgcn_exp2f(t);
    return t > -1000.f ? fmaf(y, lo * 0.693147182f, y) : 0.f;
}

// Bin of a ratio e / q, descending: bin 0 holds the largest (NaN and inf too), 32 bins per binade upwards from b0; what lies
// below b0 comes out from SA_BINS on.
__device__ __forceinline__ int sa_bin(float r, int b0)
{
    return SA_BINS - 1 - min((int)((__float_as_uint(r) & 0x7FFFFFFFu) >> 18) - b0, SA_BINS - 1);
}

__device__ __forceinline__ uint32_t this_xcd() { return (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11)); }     // HW_REG_XCC_ID, bits 3:0

// near: all workgroups run on one XCD, and the word need not go further than its L2.
__device__ __forceinline__ void put_u32(u64 *p, uint32_t tag, uint32_t x, bool near)
{
    if (near) __hip_atomic_store(p, ((u64)tag << 32) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, ((u64)tag << 32) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_f64(u64 *lo, u64 *hi, uint32_t tag, double x, bool near)
{
    const u64 b = (u64)__double_as_longlong(x);
    put_u32(lo, tag, (uint32_t)b, near);
    put_u32(hi, tag, (uint32_t)(b >> 32), near);
}
__device__ __forceinline__ double get_f64(u64 lo, u64 hi)
{
    return __longlong_as_double((long long)(((hi & 0xFFFFFFFFull) << 32) | (lo & 0xFFFFFFFFull)));
}
// Two words of each of R workgroups' parts, R loads in flight, once they all carry the tag: workgroup first + k * step,
// k < R, from offset `at` (even) of its part on; workgroups from G on (and lanes with want = false) are left out.  False: the limit
// has passed.  What this costs is the number of requests, whatever their size: both words come with one load (each has its own tag, so
// nothing depends on their coming together), and lanes that want neighbouring words share a request (a chain's exchange, five words
// of each of 63 workgroups by four wavefronts: 3.1 -> 2.4 us against a load per word with one lane per workgroup; the words of all
// workgroups side by side instead, which reads still fewer lines, has them all write to the same ones: 2.7 us for one double
// instead of 1.7).  A wavefront sleeps between two looks.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <int R>
__device__ __forceinline__ bool take(const u64 *set, int first, int step, int G, int at, bool want, uint32_t tag, ulong2 (&w)[R], long long wait_ticks)
{
    const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
    for (;;) {
        u32x4 x[R];
        const u64 *p[R];
#pragma unroll
        for (int k = 0; k < R; ++k) p[k] = set + (want && first + k * step < G ? (size_t)(first + k * step) * SA_WORDS + at : 0);
        static_assert(R == 1 || R == 4, "what is written out here");
        if constexpr (R == 1)
            asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(x[0]) : "v"(p[0]) : "memory");
        else
            asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                         "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                         : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]) : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]) : "memory");
        bool ok = true;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const bool in = want && first + k * step < G;
            ok = ok && (!in || (x[k][1] == tag && x[k][3] == tag));
            w[k] = make_ulong2(((u64)x[k][1] << 32) | x[k][0], ((u64)x[k][3] << 32) | x[k][2]);
        }
        if (__builtin_amdgcn_ballot_w64(!ok) == 0ull) return true;
        if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > wait_ticks) return false;
        __builtin_amdgcn_s_sleep(2);
    }
}

template <int PT>
struct SaShared {
    static constexpr int BT = PT < 4 ? 4 : PT;
    int par[BTV_MAX_NODES], tok[BTV_MAX_NODES];
    int2 kids[BTV_MAX_NODES + 1];                       // first child of node c (INT_MAX: none), and how many, at c + 1
    float uni[BTV_MAX_NODES + 1];
    int kcnt[SA_CHAIN][BTV_MAX_NODES / 64];             // children of chain row r among the nodes of wavefront w
    int kid_node[BTV_MAX_NODES], kid_slice[BTV_MAX_NODES];
    float kid_x[BTV_MAX_NODES];                         // the chain rows' children, row after row, in node order
    double kid_q[BTV_MAX_NODES], kid_e[BTV_MAX_NODES];
    float wm[SA_WAVES];
    double wz[SA_WAVES], wq[SA_WAVES];
    double z[SA_CHAIN], tq[SA_CHAIN], g, s_hi;
    float Mx[SA_CHAIN][SA_MAX_WGS];                     // the slices' maxima, exp(slice maximum - maximum), parts of G
    double F[SA_CHAIN][SA_MAX_WGS], GW[SA_CHAIN + 1][SA_MAX_WGS];
    alignas(16) int acc0[SA_CHAIN];
    int wsum[SA_WAVES];
    int dead, status, acc, pick, last, late;
    float2 tab[SA_GRID];                                // slope and intercept of G / G_cur over s / s_cur between two points
    double pt[BTV_MAX_NODES], ptG[BTV_MAX_NODES], invT[BTV_MAX_NODES];
    double sE[SA_POINTS], sQ[SA_POINTS], part[SA_T];
    int bin_at[SA_BINS + 1];                            // where bin b (0 = largest ratios) starts
    double cE[SA_T + 1], cQ[SA_T + 1];                  // sums over the sorted positions before PT * c
    float2 sorted[SA_T * BT];                           // (e, q) of the slice, e / q descending by bin (behind the rest: what lies
                                                        // below 64 KB is addressed with the instructions' own offsets)
    static constexpr bool KEEP = BT == 4;               // (e, q) in the row's order, kept through a fan (8 tokens a thread leave no room for it)
    float2 row[KEEP ? SA_T * BT : 1];
    int koff[SA_CHAIN + 1];                             // where the children of chain row r begin
    int near;                                           // (last: the places of the others matter, 8 bytes further on they cost 0.4 us of 37)
};

// A walk that goes down mostly takes first children (they have the largest draft probability), so the rows of a node, its
// first child, that one's first child and so on, SA_CHAIN of them, are read and exchanged together: wavefronts 4 r ..
// 4 r + 3 hold row r of the chain, PT * 4 tokens per lane.  OVER: the slices are longer than those registers; what
// is beyond a lane's first PT * 4 tokens is computed again from the row wherever it is needed (vocabularies above
// 64 x 8192 tokens), and fans are walked one by one.
// The next call's tags begin `used` further on, unless another workgroup has moved them already.
__device__ __forceinline__ void sa_move_on(uint32_t *word, uint32_t base, uint32_t used)
{
    __hip_atomic_compare_exchange_strong(word, &base, base + used, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t *sa_turn(const SaParams &p, int slice) { return p.base + (SA_TURN_WORD - SA_BASE_WORD) + slice; }

// ALONE: one workgroup (me = 0) with the whole vocabulary for a slice.  NEAR: the workgroups are dealt out so that they run on one XCD; if the first
// exchange, which goes through memory, says so of all of them, the others stay in its L2; a workgroup whose slice has been taken leaves.  Returns whether a
// wait has passed its limit (the same in all threads; results may then be missing).
template <bool BF16, int PT, bool OVER, bool ALONE, bool NEAR>
__device__ __forceinline__ bool sa_walk(const SaParams &p, SaShared<PT> &L, int me, uint32_t &base)
{
    static_assert(OVER || !ALONE, "a slice of any length");
    constexpr int TG = 4 * PT;                          // tokens of its chain row that a lane keeps
    constexpr int BT = SaShared<PT>::BT;                // tokens of the slice that a thread sorts
    constexpr int KW = BTV_MAX_NODES / 64;              // wavefronts that hold nodes
    const int M = p.M, V = p.V, G = ALONE ? 1 : p.G, per = ALONE ? V : p.per;
    int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The compiler takes everything that depends on the thread alone out of the walk's loop, dozens of registers, and
    // spills them; what tid is, it has to find out again at every node, and at every fan.
    auto forget = [&]() {
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
        wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    };
    const int v0 = min(me * per, V), v1 = min(v0 + per, V);
    for (int c = tid; c <= BTV_MAX_NODES; c += SA_T) {
        L.kids[c] = make_int2(INT_MAX, 0);
        if (c < BTV_MAX_NODES) { L.par[c] = c < M ? p.parent[c] : INT_MIN; L.tok[c] = c < M ? p.token[c] : -1; }
        if (c <= M) L.uni[c] = p.uniforms[c];
    }
    if (tid == 0) {
        L.dead = 0; L.late = 0;
    }
    if (NEAR && tid == 0) L.near = __hip_atomic_fetch_add(sa_turn(p, me), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u ? -1 : 0;
    base = G > 1 ? __hip_atomic_load(p.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    uint32_t seq = 0;
    int cur = -1, n = 0, ui = 0, d = 0;
    bool dead = false, near = false;
    __syncthreads();
    if (tid < M && L.par[tid] >= -1 && L.par[tid] < M) {
        atomicMin(&L.kids[L.par[tid] + 1].x, tid);
        atomicAdd(&L.kids[L.par[tid] + 1].y, 1);
    }
    __syncthreads();
    if (NEAR && __builtin_expect(__builtin_amdgcn_readfirstlane(L.near) < 0, 0)) return false;
    for (;;) {
        forget();
        // ---- the chain from cur, this wavefront group's row of it --------------------------------------------------
        int node[SA_CHAIN], nch = 1;
        node[0] = cur;
#pragma unroll
        for (int r = 1; r < SA_CHAIN; ++r) {
            node[r] = INT_MAX;
            if (nch == r && d + r - 1 < p.B) {
                const int2 k = L.kids[node[r - 1] + 1];
                const int first = __builtin_amdgcn_readfirstlane(k.x), fan = __builtin_amdgcn_readfirstlane(k.y);
                node[r] = fan <= SA_CHAIN_FAN ? first : INT_MAX;
            }
            if (node[r] != INT_MAX) ++nch;
            else node[r] = cur;
        }
        const int grp = wv / (SA_WAVES / SA_CHAIN), gt = tid & (SA_T / SA_CHAIN - 1);
        const bool has_row = grp < nch;
        const size_t row_at = (size_t)((grp == 0 ? node[0] : grp == 1 ? node[1] : grp == 2 ? node[2] : node[3]) + 1) * V;
        const void *xrow = BF16 ? static_cast<const void *>(static_cast<const uint16_t *>(p.logits) + row_at)
                                : static_cast<const void *>(static_cast<const float *>(p.logits) + row_at);
        const bool row_q = d + grp < p.B;
        const float *q0 = p.marg + (size_t)(row_q ? d + grp : 0) * V;
        // piece i of a lane: tokens tv + TS * i .. + 3, so that a wave instruction reads a stretch; up to vr from registers, from
        // there to ve (OVER) from memory
        constexpr int TS = SA_T / SA_CHAIN * 4;
        int tv = v0 + gt * 4;
        const int ve = has_row ? v1 : v0, vr = OVER ? min(v0 + TS * PT, ve) : ve;
        float e[TG], q[TG];
        auto load_row = [&]() {
            load_tokens<BF16, TG>(xrow, q0, tv, TS, vr, row_q ? vr : v0, V, e, q);
        };
        load_row();
        // this lane's node, if it is a child of a chain row's: what it needs of the rows is asked for behind them
        u64 bal[SA_CHAIN];
        float kid_q = 0.f, kid_x = -INFINITY;
        int kid_tok = -1, kid_slice = 0;
        if (wv < KW) {
            int at = -1, above = cur;
#pragma unroll
            for (int r = 0; r < SA_CHAIN; ++r) {
                const bool child = r < nch && d + r < p.B && L.par[tid & (BTV_MAX_NODES - 1)] == node[r];
                bal[r] = __builtin_amdgcn_ballot_w64(child);
                if (child) { at = d + r; above = node[r]; }
                if (lane == 0) L.kcnt[r][wv] = __builtin_popcountll(bal[r]);
            }
            kid_tok = L.tok[tid & (BTV_MAX_NODES - 1)];
            kid_slice = (int)((uint32_t)kid_tok / (uint32_t)per);
            if (at >= 0 && kid_tok >= 0 && kid_tok < V) {
                kid_q = p.marg[(size_t)at * V + kid_tok];
                kid_x = load_logit<BF16>(p.logits, (size_t)(above + 1) * V + kid_tok);
            }
        }
        float mx = e[0];
#pragma unroll
        for (int i = 1; i < TG; ++i) mx = fmaxf(mx, e[i]);
        if (OVER)
            for (int v = v0 + TS * PT + gt; v < ve; v += SA_T / SA_CHAIN) mx = fmaxf(mx, load_logit<BF16>(xrow, v));
        mx = wave_max(mx);
        if (lane == 0) L.wm[wv] = mx;
        __syncthreads();
        // What all 16 wavefronts do between two exchanges is bound by issue, four on a SIMD at some 5 cycles an instruction: the children's offsets are worked out by
        // the four that hold nodes, first children that are taken are counted by one ballot, a node's first child and its fan are one read (each by
        // all, and in steps: a followed draft 32.7 -> 31.0 us, fp32 32.9 -> 30.9; with the padding by pieces 29.9; 30 nodes, 32000 tokens 25.9 -> 24.6).
        int koff[SA_CHAIN + 1];
        koff[0] = 0;
        if (wv < KW) {
#pragma unroll
            for (int r = 0; r < SA_CHAIN; ++r) {
                const int4 c = *reinterpret_cast<const int4 *>(L.kcnt[r]);
                static_assert(KW == 4, "four counts");
                if ((bal[r] >> lane) & 1) {
                    const int j = koff[r] + (wv > 0 ? c.x : 0) + (wv > 1 ? c.y : 0) + (wv > 2 ? c.z : 0) + __builtin_popcountll(bal[r] & ((1ull << lane) - 1ull));
                    const bool ok = kid_tok >= 0 && kid_tok < V;      // not a vocabulary id: rejected, its uniform spent, nothing indexed
                    L.kid_node[j] = ok ? tid : -1 - tid;
                    L.kid_slice[j] = ok ? kid_slice : 0;
                    L.kid_q[j] = (double)kid_q;
                    L.kid_x[j] = kid_x;
                }
                koff[r + 1] = __builtin_amdgcn_readfirstlane(koff[r] + c.x + c.y + c.z + c.w);
            }
            if (tid <= SA_CHAIN) L.koff[tid] = tid == 0 ? 0 : tid == 1 ? koff[1] : tid == 2 ? koff[2] : tid == 3 ? koff[3] : koff[4];
        }
        float m_own;
        {
            const float4 t = *reinterpret_cast<const float4 *>(L.wm + grp * 4);
            m_own = fmaxf(fmaxf(t.x, t.y), fmaxf(t.z, t.w));
        }
        const bool none = m_own == -INFINITY;           // nothing but -inf in this slice: it has no part in anything
        double z = 0.0, tq = 0.0;
#pragma unroll
        for (int i = 0; i < TG; ++i) {
            e[i] = none ? 0.f : exp_neg(e[i] - m_own);   // (past the end: -inf, which gives 0)
            z += (double)e[i]; tq += (double)q[i];
        }
        auto e_at = [&](int v) { return none ? 0.f : exp_neg(load_logit<BF16>(xrow, v) - m_own); };
        if (OVER)
            for (int v = v0 + TS * PT + gt; v < ve; v += SA_T / SA_CHAIN) { z += (double)e_at(v); tq += row_q ? (double)q0[v] : 0.0; }
        z = wave_sum(z); tq = wave_sum(tq);
        if (lane == 0) { L.wz[wv] = z; L.wq[wv] = tq; }
        __syncthreads();
        ++seq;
        if (wv < nch) {                                 // wavefront r exchanges row r
            const int r = wv;
            z = (L.wz[4 * r] + L.wz[4 * r + 1]) + (L.wz[4 * r + 2] + L.wz[4 * r + 3]);
            tq = (L.wq[4 * r] + L.wq[4 * r + 1]) + (L.wq[4 * r + 2] + L.wq[4 * r + 3]);
            const float m_row = fmaxf(fmaxf(L.wm[4 * r], L.wm[4 * r + 1]), fmaxf(L.wm[4 * r + 2], L.wm[4 * r + 3]));
            float mw = lane == 0 ? m_row : -INFINITY;
            double zw = lane == 0 ? z : 0.0, tw = lane == 0 ? tq : 0.0;
            if (G > 1) {
                u64 *set = p.slots + (size_t)(seq & 1) * G * SA_WORDS;
                const uint32_t tag = base + seq;
                if (lane < 6) {                         // z, the draft mass, the maximum (NEAR: where this workgroup runs; else the maximum again, for whole pairs of words)
                    const u64 b = (u64)__double_as_longlong(lane < 2 ? z : tq);
                    put_u32(set + (size_t)me * SA_WORDS + 8 * r + lane, tag, NEAR && lane == 5 ? this_xcd() : lane >= 4 ? __float_as_uint(m_row) : (uint32_t)(lane & 1 ? b >> 32 : b), near);
                }
                // four lanes read a part's row, which lies in one line, and hand it to the lane that has the part
                ulong2 w[4];
                if (!take<4>(set, lane >> 2, 16, G, 8 * r + 2 * (lane & 3), (lane & 3) < 3, tag, w, p.wait_ticks) && lane == 0) L.dead = 1;
                uint32_t *x = reinterpret_cast<uint32_t *>(L.sorted) + r * (SA_MAX_WGS * 9);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t *o = x + ((lane >> 2) + 16 * k) * 9 + 2 * (lane & 3);
                    o[0] = (uint32_t)w[k].x;
                    o[1] = (uint32_t)w[k].y;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                x += lane * 9;
                mw = lane < G ? __uint_as_float(x[4]) : -INFINITY;
                zw = lane < G ? get_f64(x[0], x[1]) : 0.0;
                tw = lane < G ? get_f64(x[2], x[3]) : 0.0;
                // (all workgroups read the same words: they all find the same)
                if (NEAR && r == 0 && seq == 1 && __builtin_amdgcn_ballot_w64(lane < G && x[5] != this_xcd()) == 0ull) L.near = 1;
            }
            const float m = wave_max(mw);
            const double F = mw == -INFINITY ? 0.0 : exp((double)mw - (double)m);
            const double gw = zw * F;
            L.Mx[r][lane] = mw; L.F[r][lane] = F; L.GW[r][lane] = gw;
            z = wave_sum(gw); tq = wave_sum(tw);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int k0 = r == 0 ? koff[0] : r == 1 ? koff[1] : r == 2 ? koff[2] : koff[3];
            const int k1 = r == 0 ? koff[1] : r == 1 ? koff[2] : r == 2 ? koff[3] : koff[4];
            bool acc0 = false;                          // is the first child accepted, if the rows above took theirs?
#pragma nounroll
            for (int j = k0 + lane; j < k1; j += 64) {  // a child's e exactly as its slice's owner has it
                const int w = L.kid_slice[j];
                const float x = L.kid_x[j];
                const double ek = x == -INFINITY ? 0.0 : L.F[r][w] * (double)exp_neg(x - L.Mx[r][w]);
                L.kid_e[j] = ek;
                if (j == k0) acc0 = L.kid_node[j] >= 0 && (double)L.uni[min(ui + r, M)] * (L.kid_q[j] * (tq > 0.0 ? 1.0 / tq : 0.0)) * z < ek;
            }
            if (lane == 0) { L.z[r] = z; L.tq[r] = tq; L.acc0[r] = acc0 ? 1 : 0; }
        }
        __syncthreads();
        if (L.dead) { dead = true; break; }
        if (NEAR) near = __builtin_amdgcn_readfirstlane(L.near) != 0;
        // ---- first children, as far as they are accepted -------------------------------------------------------------
        int r;
        {
            const int next = __builtin_amdgcn_readfirstlane(L.kids[(nch > 3 ? node[3] : nch > 2 ? node[2] : nch > 1 ? node[1] : node[0]) + 1].x);
            const uint32_t taken = (uint32_t)__builtin_amdgcn_ballot_w64(L.acc0[lane & (SA_CHAIN - 1)] != 0);
            r = min(min(__builtin_ctz(~taken | 1u << SA_CHAIN), nch), M - n);
            auto below = [&](int k) { return k >= nch ? next : k == 1 ? node[1] : k == 2 ? node[2] : node[3]; };     // chain row k - 1's first child
            if (r > 0) {
                if (me == 0 && tid < r) p.path[n + tid] = below(tid + 1);
                cur = __builtin_amdgcn_readfirstlane(below(r));
                n += r; d += r; ui += r;
            }
        }
        if (r == nch) continue;
        // ---- row r: its first child is rejected, or it has none ---------------------------------------------------------
        const int k0 = __builtin_amdgcn_readfirstlane(L.koff[r]);
        const int nk = __builtin_amdgcn_readfirstlane(L.koff[r + 1]) - k0;
        const bool here = grp == r;                     // this wavefront holds the row's tokens
        double s = 0.0, Gs = L.z[r], T = L.tq[r];
        const double f = L.F[r][me], invf = f > 0.0 ? 1.0 / f : 0.0;
        int gbuf = r, galt = SA_CHAIN;                  // GW[gbuf]: the parts of G(s)
        bool batch_ok = !OVER;
        int accepted = -1, j = 0;
        for (; j < nk; ++j) {
            const int c = L.kid_node[k0 + j];
            if (c < 0) {
                if (me == 0 && tid == 0) atomicOr(p.flag, 64u);
                continue;
            }
            const double qx = L.kid_q[k0 + j], invT = T > 0.0 ? 1.0 / T : 0.0;
            const double px = L.kid_e[k0 + j] - s * qx;      // G(s) times the target probability of the child's token
            if ((double)L.uni[min(ui + j, M)] * (qx * invT) * Gs < (px > 0.0 ? px : 0.0)) { accepted = c; ++j; break; }
            double s1 = s + Gs * invT;
            bool all = false;
            // (expected not to happen, which keeps the fan's code out of the way of the chain's: a followed draft takes 1.7 us of 36 less)
            if (__builtin_expect(batch_ok && j + (nk >> 5) >= SA_DIRECT && nk - j >= SA_BATCH_MIN && s > 0.0, 0)) {
                // ---- child j is rejected, K - 1 more follow: s_1 .. s_K at once (pt[i] is s_{i+1}, ptG[i] its G) ---------
                forget();
                const int K = nk - j, kj = k0 + j;
                {
                    // the row's tokens, from its four wavefronts to all of them
                    float2 *row = SaShared<PT>::KEEP ? L.row : L.sorted;
                    if (here) {
#pragma unroll
                        for (int i = 0; i < TG; ++i) row[(tv - v0) + TS * (i / 4) + i % 4] = make_float2(e[i], q[i]);
                    }
                    __syncthreads();
                    const int bv = v0 + tid * BT;
                    float be[BT], bq[BT];
#pragma unroll
                    for (int i = 0; i < BT; ++i) { const float2 x = row[tid * BT + i]; be[i] = x.x; bq[i] = x.y; }
                    const int b0 = (int)(__float_as_uint((float)(s * invf)) >> 18);
                    L.bin_at[tid] = 0;
                    if (wv == 0) {                      // 1 / T_k, and how far s can come
                        double own[4], sum = 0.0, ht = 0.0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) { const int k = 4 * lane + i; own[i] = k < K ? L.kid_q[kj + k] : 0.0; sum += own[i]; }
                        double t = T - (wave_scan(sum) - sum);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int k = 4 * lane + i;
                            const double it = k < K && L.kid_node[kj + k] >= 0 && t > 0.0 ? 1.0 / t : 0.0;
                            L.invT[k] = it; ht += it;
                            t -= own[i];
                        }
                        ht = wave_sum(ht);
                        if (lane == 0) L.s_hi = s + Gs * ht;
                    }
                    __syncthreads();
                    int rank[BT], bin[BT];
#pragma unroll
                    for (int i = 0; i < BT; ++i) {      // (ratios below the current s never count again: left out)
                        bin[i] = bv + i < v1 && f > 0.0 ? sa_bin(__fdiv_rn(be[i], bq[i]), b0) : SA_BINS;
                        rank[i] = bin[i] < SA_BINS ? atomicAdd(&L.bin_at[bin[i]], 1) : 0;
                    }
                    __syncthreads();
                    {   // exclusive scan of the bin counts (one bin per thread)
                        static_assert(SA_BINS == SA_T, "one bin per thread");
                        const int c0 = L.bin_at[tid];
                        const int ci = wave_scan(c0);
                        if (lane == 63) L.wsum[wv] = ci;
                        __syncthreads();
                        const int cb = sum_before(L.wsum, wv);
                        L.bin_at[tid] = cb + ci - c0;
                        if (tid == SA_T - 1) L.bin_at[SA_BINS] = cb + ci;
                    }
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < BT; ++i)
                        if (bin[i] < SA_BINS) L.sorted[L.bin_at[bin[i]] + rank[i]] = make_float2(be[i], bq[i]);
                    __syncthreads();
                    {   // prefix sums over the sorted positions, BT of them per thread
                        const int cnt = L.bin_at[SA_BINS];
                        double ce = 0.0, cq = 0.0;
#pragma unroll
                        for (int i = 0; i < BT; ++i)
                            if (BT * tid + i < cnt) { const float2 x = L.sorted[BT * tid + i]; ce += (double)x.x; cq += (double)x.y; }
                        const double ie = wave_scan(ce), iq = wave_scan(cq);
                        if (lane == 63) { L.wz[wv] = ie; L.wq[wv] = iq; }
                        __syncthreads();
                        const double se = sum_before(L.wz, wv), sq = sum_before(L.wq, wv);
                        L.cE[tid] = se + (ie - ce); L.cQ[tid] = sq + (iq - cq);
                        if (tid == SA_T - 1) { L.cE[SA_T] = se + ie; L.cQ[SA_T] = sq + iq; }
                    }
                    __syncthreads();
                }
                const int b0 = (int)(__float_as_uint((float)(s * invf)) >> 18);
                const float span = __log2f((float)(L.s_hi / s)), step = span / (float)(SA_GRID - 1);
                int status = 0;
                // pass -1: the table at SA_GRID points and the guesses from it; then Newton on the true sums
#pragma nounroll
                for (int pass = -1; pass < 8; ++pass) {
                    forget();
                    const int np = pass < 0 ? SA_GRID : K;
                    const int lkp = np > 128 ? 8 : np > 64 ? 7 : 6;      // points, a power of two
                    const int LP = SA_T >> lkp, k = tid >> (10 - lkp), sub = tid & (LP - 1);      // LP neighbouring lanes per point
                    {   // E and Q of this slice at point k, by LP neighbouring lanes
                        const double sv = pass < 0 ? s * (double)exp2f(step * (float)k) : L.pt[k];
                        double E = 0.0, Q = 0.0;
                        if (f > 0.0) {
                            const double sl = sv * invf;
                            const int b = min(max(sa_bin((float)sl, b0), 0), SA_BINS - 1);
                            const int p0 = L.bin_at[b] / BT, p1 = L.bin_at[b + 1];
#pragma nounroll
                            for (int i = p0 * BT + sub; i < p1; i += LP) {
                                const float2 x = L.sorted[i];
                                if ((double)x.x - sl * (double)x.y > 0.0) { E += (double)x.x; Q += (double)x.y; }
                            }
                            if (sub == 0) { E += L.cE[p0]; Q += L.cQ[p0]; }
                        }
                        E = group_sum(E, 10 - lkp); Q = group_sum(Q, 10 - lkp);
                        E *= f;
                        ++seq;
                        if (G > 1) {
                            if (sub < 4 && k < np) {    // four lanes a point: consecutive words by consecutive lanes
                                const u64 b = (u64)__double_as_longlong(sub & 2 ? Q : E);
                                put_u32(p.slots + ((size_t)(seq & 1) * G + me) * SA_WORDS + 4 * k + sub, base + seq, (uint32_t)(sub & 1 ? b >> 32 : b), near);
                            }
                        } else if (sub == 0) {
                            L.sE[k] = E; L.sQ[k] = Q;
                        }
                    }
                    if (G > 1) {
                        // summed in two exchanges: each workgroup adds up 2^lgp neighbouring points of all workgroups, and everybody
                        // reads the sums (with everybody reading every part instead, 4 MB for 32 workgroups, a pass took 3 us
                        // longer).  What an exchange of this size costs is the number of its requests, loads and stores alike: a
                        // thread has one double of one part and neighbouring threads neighbouring doubles, so that 16 lanes share
                        // a request where they read 8 points of a part (256 points, 63 workgroups: 9.3 -> 4.0 us both exchanges, 128
                        // points 4.1 .. 5.8 -> 2.6 .. 3.2, against a lane that read all four words of its point, every lane in
                        // another part; the same words written 256 bytes apart instead: 17 us).
                        const int lgp = G >= np ? 0 : 32 - __builtin_clz((np - 1) / G), lgd = lgp + 1, lgw = min(lgd, 6);
                        const u64 *set = p.slots + (size_t)(seq & 1) * G * SA_WORDS;
                        ulong2 x[1];
                        bool fine = true;
                        const int mine = min(np - (me << lgp), 1 << lgp) * 2;      // doubles that this workgroup adds up
                        ++seq;
                        if (mine > 0) {
                            const int w = tid >> lgd, dd = tid & ((1 << lgd) - 1);
                            if ((wv * 64 >> lgd) < G) {
                                const bool in = w < G && dd < mine;
                                fine = take<1>(set, w, 0, G, ((me << lgp) * 2 + dd) * 2, in, base + seq - 1, x, p.wait_ticks);
                                double y = in ? get_f64(x[0].x, x[0].y) : 0.0;
#pragma nounroll
                                for (int off = 1 << lgw; off < 64; off <<= 1) y += __shfl_xor(y, off);
                                if (lane < 1 << lgw) L.part[(wv << lgw) + lane] = y;
                                if (!fine && lane == 0) L.dead = 1;
                            }
                            __syncthreads();
                            if (L.dead) break;
                            if (tid < mine) {
                                double y = 0.0;
#pragma nounroll
                                for (int i = tid; i < ((((G << lgd) + 63) >> 6) << lgw); i += 1 << lgd) y += L.part[i];
                                u64 *o = p.slots + ((size_t)(seq & 1) * G + me) * SA_WORDS + 2 * tid;
                                put_f64(o, o + 1, base + seq, y, near);
                            }
                        }
                        set = p.slots + (size_t)(seq & 1) * G * SA_WORDS;
                        if (wv * 64 < 2 * np) {
                            const int k = min(tid >> 1, np - 1);
                            fine = take<1>(set, k >> lgp, 0, G, 4 * (k & ((1 << lgp) - 1)) + 2 * (tid & 1), tid < 2 * np, base + seq, x, p.wait_ticks);
                            if (tid < 2 * np) (tid & 1 ? L.sQ : L.sE)[k] = get_f64(x[0].x, x[0].y);
                        }
                        // (not L.dead: another wavefront may not have looked at that yet)
                        if (!fine && lane == 0) L.late = 1;
                    }
                    __syncthreads();
                    if (L.late) break;
                    if (pass < 0) {
                        if (tid < SA_GRID) {
                            const int kk = min(tid, SA_GRID - 2);
                            const double ig = 1.0 / Gs;
                            const float r0 = exp2f(step * (float)kk), r1 = exp2f(step * (float)(kk + 1));
                            const float g0 = fmaxf((float)((L.sE[kk] - s * (double)r0 * L.sQ[kk]) * ig), 0.f);
                            const float g1 = fmaxf((float)((L.sE[kk + 1] - s * (double)r1 * L.sQ[kk + 1]) * ig), 0.f);
                            const float sl = r1 > r0 ? (g1 - g0) / (r1 - r0) : 0.f;
                            L.tab[tid] = make_float2(sl, g0 - sl * r0);
                        }
                        __syncthreads();
                        if (wv == 0) {                  // the recurrence solved on the table (fp32, s / s_cur and G / G_cur)
                            float kap[4], nx[4];
                            const double scale = Gs / s;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                kap[i] = (float)(scale * L.invT[4 * lane + i]);
                                nx[i] = exp2f(0.5f * span * (float)(4 * lane + i + 1) / (float)K);
                            }
                            const float per_step = step > 0.f ? 1.f / step : 0.f;
#pragma nounroll
                            for (int it = 0; it < 16; ++it) {
                                float at = __shfl_up(nx[3], 1), a = 1.f, b = 0.f, ai[4], bi[4];
                                at = lane == 0 ? 1.f : at;
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const int kk = min(max((int)(__log2f(at) * per_step), 0), SA_GRID - 2);
                                    const float2 t = L.tab[kk];
                                    ai[i] = 1.f + t.x * kap[i]; bi[i] = t.y * kap[i];
                                    b = ai[i] * b + bi[i]; a = ai[i] * a;
                                    at = nx[i];
                                }
                                float A, Bv;
                                wave_affine_before(a, b, lane, A, Bv);
                                float x = A + Bv, moved = 0.f;
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    x = fmaxf(ai[i] * x + bi[i], 1.f);
                                    if (4 * lane + i < K) moved = fmaxf(moved, fabsf(x - nx[i]) / x);
                                    nx[i] = x;
                                }
                                if (__builtin_amdgcn_ballot_w64(!(moved < 3e-5f)) == 0ull) break;
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) L.pt[4 * lane + i] = s * (double)nx[i];
                        }
                        __syncthreads();
                        continue;
                    }
                    if (wv == 0) {
                        double ai[4], bi[4], a = 1.0, b = 0.0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int kk = 4 * lane + i;
                            const double it = L.invT[kk];
                            ai[i] = kk > 0 && kk < K ? 1.0 - L.sQ[kk - 1] * it : 1.0;
                            bi[i] = kk < K ? (kk > 0 ? L.sE[kk - 1] : Gs) * it : 0.0;
                            b = ai[i] * b + bi[i]; a = ai[i] * a;
                        }
                        double A, Bv;
                        wave_affine_before(a, b, lane, A, Bv);
                        double x = A * s + Bv;
                        bool close = true, good = true;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int kk = 4 * lane + i;
                            x = ai[i] * x + bi[i];
                            if (kk < K) {
                                const double g = L.sE[kk] - x * L.sQ[kk];
                                close = close && fabs(x - L.pt[kk]) <= 1e-7 * x;
                                good = good && g > 0.0;
                                L.pt[kk] = x; L.ptG[kk] = g;
                            }
                        }
                        const bool all_close = __builtin_amdgcn_ballot_w64(!close) == 0ull, all_good = __builtin_amdgcn_ballot_w64(!good) == 0ull;
                        // (a residual that is all zero keeps s where it is, which the recurrence does not say: walked one by one)
                        if (lane == 0) L.status = all_close ? (all_good ? 1 : 2) : 0;
                        if (all_close && all_good) {    // child j + k is tried at s_k
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                            int first = INT_MAX;
#pragma nounroll
                            for (int kk = 1 + lane; kk < K; kk += 64) {
                                const double qk = L.kid_q[kj + kk], pk = L.kid_e[kj + kk] - L.pt[kk - 1] * qk;
                                const bool acc = L.kid_node[kj + kk] >= 0 &&
                                                 (double)L.uni[min(ui + j + kk, M)] * (qk * L.invT[kk]) * L.ptG[kk - 1] < (pk > 0.0 ? pk : 0.0);
                                if (acc) first = min(first, kk);
                            }
                            for (int off = 32; off >= 1; off >>= 1) first = min(first, __shfl_xor(first, off));
                            if (lane == 0) L.acc = first;
#pragma nounroll
                            for (int kk = 1 + lane; kk < min(K, first); kk += 64)
                                if (L.kid_node[kj + kk] < 0 && me == 0) atomicOr(p.flag, 64u);
                        }
                    }
                    __syncthreads();
                    status = L.status;
                    if (status != 0) break;
                }
                if (L.dead | L.late) { dead = true; break; }
                if (status == 1 && L.acc < K) {
                    accepted = L.kid_node[kj + L.acc];
                    j += L.acc + 1;
                    break;
                }
                forget();
                asm volatile("" : "+v"(tv));
                if constexpr (SaShared<PT>::KEEP) {     // (the row's registers were given up for the fan; from memory: 0.9 us more)
#pragma unroll
                    for (int i = 0; i < TG; ++i) {
                        const float2 x = L.row[(tv - v0) + TS * (i / 4) + i % 4];
                        e[i] = x.x; q[i] = x.y;
                    }
                } else {
                    load_row();
#pragma unroll
                    for (int i = 0; i < TG; ++i) e[i] = none ? 0.f : exp_neg(e[i] - m_own);
                }
                if (status == 1) { s1 = L.pt[K - 1]; all = true; }      // all rejected: the parts of G(s_K) are still to be had
                batch_ok = false;                       // not converged, or a residual that is all zero
            }
            // ---- one rejection: G at the next s --------------------------------------------------------------------
            if (here) {
                double a = 0.0;
                if (f > 0.0) {
                    const double sl = s1 * invf;
#pragma unroll
                    for (int i = 0; i < TG; ++i) {
                        asm volatile("" : "+v"(e[i]), "+v"(q[i]));     // (or all of them are kept as doubles through the loop)
                        const double x = (double)e[i] - sl * (double)q[i];
                        a += x > 0.0 ? x : 0.0;
                    }
                    if (OVER)
                        for (int v = v0 + TS * PT + gt; v < ve; v += SA_T / SA_CHAIN) {
                            const double x = (double)e_at(v) - sl * (double)q0[v];
                            a += x > 0.0 ? x : 0.0;
                        }
                }
                a = wave_sum(a);
                if (lane == 0) L.wz[wv & 3] = a;
            }
            __syncthreads();
            ++seq;
            if (wv == 0) {
                const double a = ((L.wz[0] + L.wz[1]) + (L.wz[2] + L.wz[3])) * f;
                double gw = lane == 0 ? a : 0.0;
                if (G > 1) {
                    u64 *set = p.slots + (size_t)(seq & 1) * G * SA_WORDS;
                    const uint32_t tag = base + seq;
                    const u64 b = (u64)__double_as_longlong(a);
                    if (lane < 2) put_u32(set + (size_t)me * SA_WORDS + lane, tag, (uint32_t)(lane ? b >> 32 : b), near);
                    ulong2 w[1];
                    if (!take<1>(set, lane, 0, G, 0, true, tag, w, p.wait_ticks) && lane == 0) L.dead = 1;
                    gw = lane < G ? get_f64(w[0].x, w[0].y) : 0.0;
                }
                L.GW[galt][lane] = gw;
                gw = wave_sum(gw);
                if (lane == 0) L.g = gw;
            }
            __syncthreads();
            if (L.dead) { dead = true; break; }
            if (L.g > 0.0) { s = s1; Gs = L.g; const int t = gbuf; gbuf = galt; galt = t; }
            T -= qx;                                    // drafted without replacement
            if (all) { j = nk; break; }
        }
        if (dead) break;
        ui += j;                                        // one uniform per child tried
        if (accepted >= 0 && n < M) {
            cur = __builtin_amdgcn_readfirstlane(accepted);
            if (me == 0 && tid == 0) p.path[n] = cur;
            ++n; ++d;
            continue;
        }
        // ---- bonus: smallest v with cumsum(p)[v] > u ---------------------------------------------------------------
        const double target = (double)L.uni[min(ui, M)] * Gs;
        const double gw = L.GW[gbuf][lane], incl = wave_scan(gw);
        const u64 over = __builtin_amdgcn_ballot_w64(incl > target && gw > 0.0);
        const int owner = over != 0ull ? __builtin_ctzll(over) : -1;
        if (owner == me || owner < 0) {
            // this slice holds the crossing (or rounding put it past the end: then every slice's last token with mass)
            if (tid == 0) { L.pick = INT_MAX; L.last = -1; }
            const double sl = s * invf;
            auto mass = [&](float ev, float qv) { const double x = ((double)ev - sl * (double)qv) * f; return x > 0.0 ? x : 0.0; };
            // tokens in order: piece after piece, in a piece lane after lane (OVER: the rest the same way, one token per lane)
            double run = owner >= 0 ? __shfl(incl - gw, owner) : 0.0;
            const int trips = (v1 - v0 + TS - 1) / TS, rest = OVER ? max(v1 - v0 - TS * PT + SA_T / SA_CHAIN - 1, 0) / (SA_T / SA_CHAIN) : 0;
#pragma nounroll
            for (int t = 0; t < (OVER ? PT + rest : min(trips, PT)); ++t) {
                double x[4] = { 0.0, 0.0, 0.0, 0.0 };
                int v = tv + TS * t;
                if (here) {
                    if (!OVER || t < PT) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            float ev = e[k], qv = q[k];
#pragma unroll
                            for (int i = 1; i < PT; ++i) { ev = t == i ? e[4 * i + k] : ev; qv = t == i ? q[4 * i + k] : qv; }
                            x[k] = mass(ev, qv);
                        }
                    } else {
                        v = v0 + TS * PT + (t - PT) * (SA_T / SA_CHAIN) + gt;
                        if (v < ve) x[0] = mass(e_at(v), row_q ? q0[v] : 0.f);
                    }
                }
                const double own = (x[0] + x[1]) + (x[2] + x[3]), iw = wave_scan(own);
                if (here && lane == 63) L.wz[wv & 3] = iw;
                __syncthreads();
                if (here) {
                    double at = run + (iw - own);
#pragma unroll
                    for (int w = 0; w < 3; ++w) at += w < (wv & 3) ? L.wz[w] : 0.0;
                    int hit = INT_MAX, last = -1;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        at += x[k];
                        if (x[k] > 0.0) { last = v + k; hit = at > target ? min(hit, v + k) : hit; }
                    }
                    if (last >= 0) atomicMax(&L.last, last);
                    if (owner >= 0 && hit != INT_MAX) atomicMin(&L.pick, hit);
                }
                run += (L.wz[0] + L.wz[1]) + (L.wz[2] + L.wz[3]);
                __syncthreads();
            }
            __syncthreads();
            if (owner >= 0 && tid == 0) *p.bonus = L.pick != INT_MAX ? L.pick : max(L.last, 0);
        }
        if (owner < 0) {
            ++seq;
            if (wv == 0) {
                int last = lane == 0 ? L.last : -1;
                if (G > 1) {
                    u64 *set = p.slots + (size_t)(seq & 1) * G * SA_WORDS;
                    const uint32_t tag = base + seq;
                    if (lane < 2) put_u32(set + (size_t)me * SA_WORDS + lane, tag, (uint32_t)L.last, near);
                    ulong2 w[1];
                    if (!take<1>(set, lane, 0, G, 0, true, tag, w, p.wait_ticks) && lane == 0) L.dead = 1;
                    last = lane < G ? (int)(uint32_t)w[0].x : -1;
                }
                for (int off = 32; off >= 1; off >>= 1) last = max(last, __shfl_xor(last, off));
                if (me == 0 && lane == 0) *p.bonus = max(last, 0);
            }
            __syncthreads();
            if (L.dead) dead = true;
        }
        break;
    }
    if (!dead && me == 0 && tid == 0) {
        *p.n_acc = n;
        if (G > 1) sa_move_on(p.base, base, seq);
    }
    return dead;
}

// The walk alone, in a function of its own that reads the arguments again: what is next to never needed is not to cost the walk above
// registers, nor to lie in the way of its code (inlined, with the arguments held: 0.5 to 1 us of 25 to 45).
typedef const __attribute__((address_space(4))) SaParams *SaArgs;
template <int PT> using SaLds = __attribute__((address_space(3))) SaShared<PT> *;
template <bool BF16, int PT>
__device__ __attribute__((noinline, cold)) void sa_walk_alone(SaArgs args, SaLds<PT> L)
{
    uint32_t none;
    sa_walk<BF16, PT, true, true, false>(*(const SaParams *)args, *(SaShared<PT> *)L, 0, none);
}

template <bool BF16, int PT, bool OVER, bool NEAR>
__global__ __launch_bounds__(SA_T) void stochastic_walk(SaParams p)
{
    __shared__ SaShared<PT> L;
    uint32_t base;
    const int me = NEAR ? blockIdx.x >> 3 : blockIdx.x;
    if constexpr (NEAR) {                               // (ids that are congruent mod 8 run on one XCD)
        const int from = blockIdx.x & 7;
        if (from != 0 && from != 1 + me % 7) return;
        if (from != 0) {                                // a stand-in
            if (threadIdx.x < 64) {
                const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
                __builtin_amdgcn_s_sleep(72);           // (2 us, by which a slice is taken as a rule)
                while (!(__hip_atomic_load(sa_turn(p, me), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u) && (long long)__builtin_amdgcn_s_memrealtime() - t0 < SA_START)
                    __builtin_amdgcn_s_sleep(16);
            }
            __syncthreads();
        }
    }
    if (!sa_walk<BF16, PT, OVER, false, NEAR>(p, L, me, base)) return;
    auto again = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(again));
    const SaArgs args = (SaArgs)again;
    const u64 call = 1ull << 32 | base;
    if (threadIdx.x == 0) L.status = __hip_atomic_exchange(args->claim, call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != call;
    __syncthreads();
    if (!L.status) return;
    sa_walk_alone<BF16, PT>(args, (SaLds<PT>)&L);
    if (threadIdx.x == 0) sa_move_on(args->base, base, SA_SPAN);
}

// Slices for a vocabulary of V tokens on at most `most` workgroups (no more than CUs that the stream may use: with 32 of them the two
// walks named at the top take 52 and 48 .. 52 us, with 16 110 and 101 .. 118): of 2048 tokens (two per thread) as long as those cover the
// vocabulary, of 4096, of 8192, longer ones above.
struct SaPlan { int G, per, pt; bool over, near; };
SaPlan sa_plan(int V, int most)
{
    SaPlan a;
    a.pt = V <= most * SA_T * 2 ? 2 : V <= most * SA_T * 4 ? 4 : 8;
    a.over = V > most * SA_T * 8;
    const int slice = SA_T * a.pt;
    a.G = a.over ? most : (V + slice - 1) / slice;
    a.per = (int)((((long long)V + a.G - 1) / a.G + 3) / 4 * 4);
    a.near = false;
    return a;
}

template <bool BF16>
void sa_launch(const SaPlan &a, const SaParams &p, hipStream_t st)
{
    if (a.over) hipLaunchKernelGGL((stochastic_walk<BF16, 8, true, false>), dim3(a.G), dim3(SA_T), 0, st, p);
    else if (a.pt == 8) hipLaunchKernelGGL((stochastic_walk<BF16, 8, false, false>), dim3(a.G), dim3(SA_T), 0, st, p);
    else if (a.pt == 4) hipLaunchKernelGGL((stochastic_walk<BF16, 4, false, false>), dim3(a.G), dim3(SA_T), 0, st, p);
    else if (a.near) hipLaunchKernelGGL((stochastic_walk<BF16, 2, false, true>), dim3(8 * a.G), dim3(SA_T), 0, st, p);
    else hipLaunchKernelGGL((stochastic_walk<BF16, 2, false, false>), dim3(a.G), dim3(SA_T), 0, st, p);
}

}  // namespace

size_t btv_stochastic_workspace(int V)
{
    return BTV_WS_HEADER + btv_align_up((size_t)2 * sa_plan(V, SA_MAX_WGS).G * SA_WORDS * sizeof(u64), BTV_WS_ALIGN);   // (fewer workgroups: fewer slices)
}

extern "C" int btv_tree_accept_stochastic_tuned(const void *logits, int dtype, const float *marginals, int B, const int32_t *parent,
                                                const int32_t *token, int M, int V, const float *uniforms, int32_t *path,
                                                int32_t *n_acc, int32_t *bonus, void *ws, size_t ws_bytes, void *stream,
                                                int max_workgroups, long long wait_ticks)
{
    BTV_REQUIRE(logits && parent && token && path && n_acc && bonus, "null pointer");
    BTV_REQUIRE(dtype == BTV_F32 || dtype == BTV_BF16, "dtype=%d unsupported", dtype);
    BTV_REQUIRE(M >= 1 && M <= BTV_MAX_NODES, "M=%d outside [1,%d]", M, BTV_MAX_NODES);
    BTV_REQUIRE(V >= 1, "V=%d", V);
    BTV_REQUIRE(marginals && uniforms, "null pointer");
    BTV_REQUIRE(B >= 1 && B <= BTV_MAX_DEPTH, "B=%d outside [1,%d]", B, BTV_MAX_DEPTH);
    BTV_REQUIRE(max_workgroups >= 0 && max_workgroups <= SA_MAX_WGS, "max_workgroups=%d outside [0,%d]", max_workgroups, SA_MAX_WGS);
    const int rc = btv_check_ws(ws, ws_bytes, btv_stochastic_workspace(V));
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    SaPlan a = sa_plan(V, max_workgroups ? max_workgroups : SA_MAX_WGS);
    if (!max_workgroups && a.G > 1) {
        const int cus = btv_usable_cus(st);
        a = sa_plan(V, std::min(SA_MAX_WGS, cus));
        a.near = a.pt == 2 && !a.over && a.G > 1 && a.G <= SA_NEAR && cus >= 256;
    }
    SaParams p;
    p.logits = logits; p.marg = marginals; p.uniforms = uniforms; p.parent = parent; p.token = token;
    p.path = path; p.n_acc = n_acc; p.bonus = bonus;
    p.flag = static_cast<uint32_t *>(ws);
    p.base = static_cast<uint32_t *>(ws) + SA_BASE_WORD; p.claim = static_cast<u64 *>(ws) + 9;
    p.slots = reinterpret_cast<u64 *>(static_cast<unsigned char *>(ws) + BTV_WS_HEADER);
    p.B = B; p.M = M; p.V = V; p.G = a.G; p.per = a.per; p.wait_ticks = wait_ticks;
    if (dtype == BTV_BF16) sa_launch<true>(a, p, st);
    else sa_launch<false>(a, p, st);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

extern "C" int btv_tree_accept_stochastic(const void *logits, int dtype, const float *marginals, int B, const int32_t *parent,
                                          const int32_t *token, int M, int V, const float *uniforms, int32_t *path,
                                          int32_t *n_acc, int32_t *bonus, void *ws, size_t ws_bytes, void *stream)
{
    return btv_tree_accept_stochastic_tuned(logits, dtype, marginals, B, parent, token, M, V, uniforms, path, n_acc, bonus, ws,
                                            ws_bytes, stream, 0, SA_WAIT_TICKS);
}
