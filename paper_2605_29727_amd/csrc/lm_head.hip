// LM head fused with the argmax (App. E: 2*s*h*V FLOPs and s*V activation elements for the logits; App. C "Acceptance": only
// their top-1 is used).  logit[r, v] = sum_k H[r, k] W[v, k] is formed on the matrix cores, a workgroup leaves the best
// (value, token) of its part of the vocabulary for every row of H, and the logits never reach memory.
//
// The vocabulary is shared out evenly: as many workgroups as CUs, each with V / 256 tokens (or a half, a third, ... of them,
// one after the other, where a CU cannot hold the sums), whatever number of whole tiles that is.  A workgroup takes all rows
// of H, so W is read once and by all CUs at the same rate to the end; what a tile has beyond its share is multiplied for
// nothing, which costs no memory traffic.  (Workgroups of whole tiles of 128 or 256 tokens, as this was before, leave up to
// half of the CUs idle in the last round: 193 of h = 3712, V = 80815, 316 workgroups of 256 tokens, 231 us, now 142.)
//
// Both operands come by 16-byte loads to LDS into a ring of stages (64 or 128 of the contraction): the loads of a chunk's
// first stages are under way while the chunk before it ends, no registers hold what is on its way, and there is one barrier
// per stage.  The transposed product C^T = W_tile * H^T (v_mfma_f32_16x16x32_bf16) keeps a lane's sums on one row of H, so
// the argmax is a scan in registers.  Tiles store the 16-byte chunks of a row XOR-permuted by the row number, so operand
// reads (16 lanes = 16 different rows) are conflict-free.
//
// What bounds it: with up to some 60 rows the rate of memory (64 rows, h = 4096, V = 128256: 1.05 GB in 162 us, 6.5 TB/s,
// 191 before; 4 rows, V = 50000: 72 -> 64 us), in short calls the chain of one stage, the merge and the walk (7 rows,
// h = 1024, V = 8000 11.5 -> 8.8). With more rows what a CU can get into LDS, some 33 KB per us: all of H (from the L2) for
// each of its chunks besides W, and the operand reads from LDS (256 rows, h = 4096, V = 128256 329 -> 261).  Tried without
// gain: rings of their own for H (short) and W (long), loaded by waves of their own, 64 rows 183 -> 220; stages of 32
// (64-byte pieces of W), 247 rows at V = 26424 61 -> 72; leaving out the loads of rows that are not there (their branches
// cost more), 163 rows at V = 10203 31 -> 36.
#include "btv_common.h"
#include "lm_head.h"

#include <algorithm>
#include <atomic>
#include <climits>
#include <numeric>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define LM_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

constexpr int LDS_MOST = 160 * 1024;
constexpr int MOST_ROWS = (BTV_MAX_NODES + 1 + 15) / 16 * 16;

// 8 waves: VW over the vocabulary, RW over the rows, KW over the contraction (their sums meet at the end); a wave holds VT x RT tiles of 16 x 16.
template <int VT, int RT, int VW, int RW, int KW, int KB>
struct Share {
    static constexpr int WAVES = VW * RW * KW, THREADS = WAVES * 64;
    static constexpr int VROWS = VW * VT * 16, ROWS = RW * RT * 16;
    static constexpr int RB = KB * 2, CPR = RB / 16, RPI = 64 / CPR;      // bytes and 16-byte chunks of a row, rows of a load instruction
    static constexpr int HROWS = ROWS < MOST_ROWS ? ROWS : MOST_ROWS;    // rows of H that are loaded; what lies behind them belongs to rows that are not there
    static constexpr int WI = VROWS / RPI, INSTR = (VROWS + HROWS) / RPI, STAGE = (VROWS + HROWS) * RB;
    static constexpr int LPW = (INSTR + WAVES - 1) / WAVES, REM = INSTR - (LPW - 1) * WAVES;     // waves below REM issue LPW loads, the others one less
    // (one word per row for the best of all waves: with one per row and wave 153 rows, h = 2688, V = 52200 have room for two stages and take 77 us, so 68)
    static constexpr int BEST = ROWS * 8, SPARE = (ROWS - HROWS) * RB > BEST ? (ROWS - HROWS) * RB : BEST;
    static constexpr int ROOM = (LDS_MOST - SPARE) / STAGE, SLOTS = ROOM < 4 ? ROOM : 4;
    static constexpr int LDS_BYTES = SLOTS * STAGE + SPARE;
    static constexpr int STEPS = KB / 32 / KW;
    static constexpr bool PIPE = KW == 1 && STEPS == 2;
    static_assert(WAVES == 8 && SLOTS >= 2 && (CPR == 8 || CPR == 16) && STEPS >= 1, "shape");
    static_assert(KW == 1 || WAVES * VT * 1024 <= STAGE, "the sums of a row tile fit a slot");
    static_assert((SLOTS - 2) * LPW <= 63, "vmcnt range");
    __device__ static constexpr int swizzle(int row) { return CPR == 16 ? row & 15 : (row >> 1) & 7; }
};

__device__ __forceinline__ void take(float &v, int &i, float ov, int oi)
{
    if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}
// (value, token) as a number that is larger for the larger value and, of equals, the smaller token; 0: none.  (x + 0: -0 becomes 0.)
__device__ __forceinline__ unsigned long long packed(float v, int i)
{
    const uint32_t b = __float_as_uint(v + 0.f), key = b & 0x80000000u ? ~b : b | 0x80000000u;
    return i == INT_MAX ? 0 : (unsigned long long)key << 32 | ~(uint32_t)i;
}
__device__ __forceinline__ LmBest unpacked(unsigned long long x)
{
    const uint32_t key = (uint32_t)(x >> 32);
    return x ? LmBest{ __uint_as_float(key & 0x80000000u ? key & 0x7FFFFFFFu : ~key), (int)~(uint32_t)x } : LmBest{ -INFINITY, INT_MAX };
}

// 16 bytes per lane to LDS, lane after lane from `to`.  STREAM: marked as read once (2: non-temporal).
template <bool STREAM>
__device__ __forceinline__ void load_1k(const unsigned char *from, unsigned char *to)
{
    __builtin_amdgcn_global_load_lds(from, LM_LDS_PTR(to), 16, 0, STREAM ? 2 : 0);
}
__device__ __forceinline__ const unsigned char *uniform(const unsigned char *p)
{
    const unsigned long long x = reinterpret_cast<unsigned long long>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return reinterpret_cast<const unsigned char *>((unsigned long long)hi << 32 | lo);
}
template <int N>
__device__ __forceinline__ void lgkm_wait()
{
    static_assert(N >= 0 && N <= 15, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void vm_wait()
{
    static_assert(N >= 0 && N <= 63, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// All but the youngest min(younger, MOST) stages of EACH loads have landed.
template <int MOST, int EACH>
__device__ __forceinline__ void stages_wait(int younger)
{
    if constexpr (MOST > 0) {
        if (younger < MOST) return stages_wait<MOST - 1, EACH>(younger);
    }
    vm_wait<MOST * EACH>();
}

// Operands of 16 rows and 32 of the contraction; tile i lies 16 rows further.  The reads are raw instructions with waits placed by hand.
template <int RB>
__device__ __forceinline__ void read_tile(u32x4 &x, uint32_t at, int i)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(x) : "v"(at), "n"(i * 16 * RB) : "memory");
}
template <int N, int RB>
__device__ __forceinline__ void read_tiles(u32x4 (&x)[N], uint32_t at)
{
#pragma unroll
    for (int i = 0; i < N; ++i) read_tile<RB>(x[i], at, i);
}
// The uses of operands may not move above the wait that covers them.
template <int N>
__device__ __forceinline__ void landed(u32x4 (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}
__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <int VT, int RT, int VW, int RW, int KW, int KB, bool STREAM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lm_head_shares(
    const unsigned char *__restrict__ H, const unsigned char *__restrict__ W, int R, int h, int V, int share, int chunks, int stride, LmBest *__restrict__ part)
{
    using S = Share<VT, RT, VW, RW, KW, KB>;
    extern __shared__ __align__(256) unsigned char lm_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave / (VW * RW), vw = wave % VW, rw = wave / VW % RW, l16 = lane & 15, q = lane >> 4;
    const int nkb = h / KB, row_bytes = h * 2;
    const int mine = (chunks - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x, total = mine * nkb;     // (the grid is no larger than chunks)

    // Loads: instruction i * WAVES + wave of a stage fills 1 KB; the swizzle is on the side of the addresses.
    // Workgroups start at different blocks of the contraction and wrap round: rows of W may be a multiple of 4 KB apart, and in step
    // they would all read the same few memory channels (all from the first block: 64 rows, h = 4096, V = 128256 239 us, so 182).  The
    // stride shares no factor with the number of blocks, so the 32 workgroups of an XCD are spread evenly.
    auto first = [&](int c) { return ((c >> 3) * stride + (c & 7) * 2) % nkb; };
    uint32_t off[S::LPW];
    int lchunk = blockIdx.x, lk = 0, lcur = first(lchunk), issued = 0, lslot = 0;
    const unsigned char *wbase = nullptr;
    const int sub = lane / S::CPR, col = lane % S::CPR;
    auto start = [&]() {
        const int c0 = lchunk * share, n = min(share, V - c0);
        wbase = W + (size_t)c0 * row_bytes;
#pragma unroll
        for (int i = 0; i < S::LPW; ++i) {
            const int in = i * S::WAVES + wave, lrow = in * S::RPI + sub, hr = lrow - S::VROWS;
            const int row = in < S::WI ? min(lrow, n - 1) : min(hr, R - 1);
            off[i] = (uint32_t)row * (uint32_t)row_bytes + (uint32_t)((col ^ S::swizzle(lrow)) << 4);
        }
    };
    const unsigned char *fromW, *fromH;
    unsigned char *to;
    bool more;
    auto begin = [&]() {
        more = issued < total;
        fromW = uniform(wbase + (size_t)lcur * S::RB); fromH = uniform(H + (size_t)lcur * S::RB);
        to = lm_smem + lslot * S::STAGE + wave * 1024;
    };
    auto load = [&](int i) {
        const bool ofW = (i + 1) * S::WAVES <= S::WI || (i * S::WAVES < S::WI && i * S::WAVES + wave < S::WI);    // (mostly a constant)
        if (i < S::LPW - 1 || S::REM == S::WAVES || wave < S::REM) {
            if (ofW) load_1k<STREAM>(fromW + off[i], to + i * S::WAVES * 1024);
            else load_1k<false>(fromH + off[i], to + i * S::WAVES * 1024);
        }
    };
    auto end = [&]() {
        ++issued;
        lslot = lslot + 1 == S::SLOTS ? 0 : lslot + 1;
        lcur = lcur + 1 == nkb ? 0 : lcur + 1;
        if (++lk == nkb) {
            lk = 0; lchunk += gridDim.x;
            if (issued < total) { lcur = first(lchunk); start(); }
        }
    };
    auto issue = [&]() {
        begin();
        if (!more) return;
#pragma unroll
        for (int i = 0; i < S::LPW; ++i) load(i);
        end();
    };
    // own loads of a stage have landed, with at most `left` stages after it in the queue
    auto arrived = [&](int left) {
        if (S::REM == S::WAVES || wave < S::REM) stages_wait<S::SLOTS - 2, S::LPW>(left);
        else stages_wait<S::SLOTS - 2, S::LPW - 1>(left);
    };

    const uint32_t ring = (uint32_t)(uintptr_t)LM_LDS_PTR(lm_smem), best = ring + S::SLOTS * S::STAGE;
    const uint32_t lane_at = (uint32_t)(l16 * S::RB + ((q ^ S::swizzle(l16)) << 4));
    const uint32_t wrow = (uint32_t)(vw * VT * 16 * S::RB), hrow = (uint32_t)((S::VROWS + rw * RT * 16) * S::RB);
    f32x4 acc[VT][RT];
    int slot = 0;
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < VT; ++i)
#pragma unroll
            for (int j = 0; j < RT; ++j) acc[i][j] = f32x4{ 0.f, 0.f, 0.f, 0.f };
    };
    auto wat = [&](int slot, int step) { return ring + slot * S::STAGE + wrow + (lane_at ^ (uint32_t)(step << 6)); };
    auto hat = [&](int slot, int step) { return ring + slot * S::STAGE + hrow + (lane_at ^ (uint32_t)(step << 6)); };
    // A row's best of the vocabulary rows that 16 x 4 lanes hold goes into its word of LDS.
    auto leave = [&](float v, int i, int row) {
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            const float ov = __shfl_xor(v, o);
            const int oi = __shfl_xor(i, o);
            take(v, i, ov, oi);
        }
        if (q == 0) asm volatile("ds_max_u64 %0, %1" ::"v"(best + (uint32_t)(row + l16) * 8), "v"(packed(v, i)) : "memory");
    };
    auto finish = [&](int chunk) {
        const int c0 = chunk * share, n = min(share, V - c0), r0 = vw * VT * 16 + q * 4;
        if constexpr (KW == 1) {
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                float v = -INFINITY;
                int at = INT_MAX;
#pragma unroll
                for (int i = 0; i < VT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (i * 16 + e < n - r0) take(v, at, acc[i][j][e], i * 16 + e);
                leave(v, at == INT_MAX ? at : at + c0 + r0, (rw * RT + j) * 16);
            }
        } else {
            // the waves' sums meet in the slot of the stage that has just been read, a row tile of each at a time
            const uint32_t sums = ring + slot * S::STAGE + (uint32_t)((rw * VW + vw) * VT * 1024 + lane * 16);
            constexpr int PLANE = RW * VW * VT * 1024;
            lgkm_wait<0>();
            __builtin_amdgcn_s_barrier();                        // everybody has read the stage
#pragma unroll
            for (int j = 0; j < RT; ++j) {
#pragma unroll
                for (int i = 0; i < VT; ++i)                     // (ordinary stores: ahead of one in inline assembly the compiler would not wait for acc)
                    *(__attribute__((address_space(3))) f32x4 *)(uintptr_t)(sums + (uint32_t)(kw * PLANE + i * 1024)) = acc[i][j];
                lgkm_wait<0>();
                __builtin_amdgcn_s_barrier();
                for (int i = kw; i < VT; i += KW) {
                    f32x4 x[KW];
#pragma unroll
                    for (int k = 0; k < KW; ++k) asm volatile("ds_read_b128 %0, %1" : "=v"(x[k]) : "v"(sums + (uint32_t)(k * PLANE + i * 1024)) : "memory");
                    lgkm_wait<0>();
#pragma unroll
                    for (int k = 0; k < KW; ++k) asm volatile("" : "+v"(x[k]));
#pragma unroll
                    for (int k = 1; k < KW; ++k) x[0] += x[k];
                    float v = -INFINITY;
                    int at = INT_MAX;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (i * 16 + e < n - r0) take(v, at, x[0][e], c0 + r0 + i * 16 + e);
                    leave(v, at, (rw * RT + j) * 16);
                }
                if (j + 1 < RT) { lgkm_wait<0>(); __builtin_amdgcn_s_barrier(); }
            }
        }
        lgkm_wait<0>();
        __builtin_amdgcn_s_barrier();
        if (tid < min(R, S::ROWS)) {
            unsigned long long x;
            asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(x) : "v"(best + (uint32_t)tid * 8) : "memory");
            asm volatile("ds_write_b64 %0, %1" ::"v"(best + (uint32_t)tid * 8), "v"(0ull) : "memory");   // (for the next chunk, a stage's barrier away)
            part[(size_t)chunk * R + tid] = unpacked(x);
        }
    };

    for (int i = tid; i < S::ROWS; i += S::THREADS) asm volatile("ds_write_b64 %0, %1" ::"v"(best + (uint32_t)i * 8), "v"(0ull) : "memory");
    start();
#pragma unroll
    for (int i = 0; i < S::SLOTS - 1; ++i) issue();
    clear();
    int chunk = blockIdx.x, k = 0;
    auto next = [&]() { slot = slot + 1 == S::SLOTS ? 0 : slot + 1; };
    if constexpr (S::PIPE) {
        // The reads of a step run one step ahead: those of W into a second set, those of H each into the registers that the tiles of the
        // row before it have just been multiplied with.  What is read past the last stage is not used.
        u32x4 a0[VT], a1[VT], b[RT];
        arrived(total - 1);
        __builtin_amdgcn_s_barrier();
        issue();
        read_tiles<VT, S::RB>(a0, wat(0, 0));
        read_tiles<RT, S::RB>(b, hat(0, 0));
        for (int g = 0; g < total; ++g) {
            read_tiles<VT, S::RB>(a1, wat(slot, 1));
            const uint32_t h1 = hat(slot, 1);
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                lgkm_wait<VT + RT - 1>();
                if (j == 0) landed(a0);
                asm volatile("" : "+v"(b[j]));
#pragma unroll
                for (int i = 0; i < VT; ++i) acc[i][j] = mfma(a0[i], b[j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
                read_tile<S::RB>(b[j], h1, j);
            }
            lgkm_wait<0>();
            landed(a1);
            landed(b);
            next();
            if (g + 1 < total) {
                arrived(total - 2 - g);
                __builtin_amdgcn_s_barrier();                    // ... of everybody, and everybody has read stage g
            }
            begin();
            read_tiles<VT, S::RB>(a0, wat(slot, 0));
            const uint32_t h0 = hat(slot, 0);
#pragma unroll
            for (int j = 0; j < RT; ++j) {
#pragma unroll
                for (int i = 0; i < VT; ++i) acc[i][j] = mfma(a1[i], b[j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
                read_tile<S::RB>(b[j], h0, j);
                // (a load to LDS holds its wave for some hundred cycles: they go between the matrix instructions; all of them ahead of those:
                // 256 rows, h = 4096, V = 10000 48.3 us, so 45.7)
                if (more) {
#pragma unroll
                    for (int i = j * S::LPW / RT; i < (j + 1) * S::LPW / RT; ++i) load(i);
                }
            }
            if (more) end();
            if (++k == nkb) {
                lgkm_wait<0>();                                  // (the next chunk's first operands: landed before anything may move them)
                landed(a0);
                landed(b);
                finish(chunk);
                clear();
                k = 0; chunk += gridDim.x;
            }
        }
    } else {
        for (int g = 0; g < total; ++g) {
            arrived(total - 1 - g);
            __builtin_amdgcn_s_barrier();
#pragma unroll
            for (int t = 0; t < S::STEPS; ++t) {
                u32x4 a[VT], b[RT];
                read_tiles<VT, S::RB>(a, wat(slot, kw * S::STEPS + t));
                read_tiles<RT, S::RB>(b, hat(slot, kw * S::STEPS + t));
                if (t == 0) issue();
                lgkm_wait<0>();
                landed(a);
                landed(b);
#pragma unroll
                for (int j = 0; j < RT; ++j)
#pragma unroll
                    for (int i = 0; i < VT; ++i) acc[i][j] = mfma(a[i], b[j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);               // (one set of operands)
            }
            if (++k == nkb) {
                finish(chunk);
                clear();
                k = 0; chunk += gridDim.x;
            }
            next();
        }
    }
}

template <int VT, int RT, int VW, int RW, int KW, int KB, bool STREAM>
int launch(const void *H, const void *W, int R, int h, int V, int share, int chunks, LmBest *part, hipStream_t st)
{
    using S = Share<VT, RT, VW, RW, KW, KB>;
    static std::atomic<bool> configured{false};         // (one GPU per process: the attribute is set once)
    auto kern = lm_head_shares<VT, RT, VW, RW, KW, KB, STREAM>;
    if (!configured.load(std::memory_order_acquire)) {
        BTV_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES));
        configured.store(true, std::memory_order_release);
    }
    if (R > S::ROWS || share > S::VROWS) return btv_fail(BTV_EINVAL, "no LM-head kernel for %d rows and shares of %d", R, share);
    int stride = 17;
    while (std::gcd(stride, h / KB) > 1) stride += 2;
    hipLaunchKernelGGL(kern, dim3(std::min(chunks, 256)), dim3(S::THREADS), S::LDS_BYTES, st, static_cast<const unsigned char *>(H),
                       static_cast<const unsigned char *>(W), R, h, V, share, chunks, stride, part);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

template <int RT, int VW, int RW, int KW, int KB, int LEAST, int VT>
int pick(int vt, const void *H, const void *W, int R, int h, int V, int share, int chunks, LmBest *part, hipStream_t st)
{
    if constexpr (VT > LEAST)
        if (vt < VT) return pick<RT, VW, RW, KW, KB, LEAST, VT - 1>(vt, H, W, R, h, V, share, chunks, part, st);
    // Weights of more than half of the last-level cache (256 MB) are read past it.  A step that follows another has read all layers' weights and caches in
    // between, and then the hint gains at every size; up to half, a caller that comes back sooner finds them in the cache, and loses by the hint more than
    // the other gains.  us, without / with it, the matrix met again at once | two others of its size in between | 1 GB of other data in between: 65 rows, 82 MB 24.0 / 26.1
    // | 24.0 / 27.4 | 29.0 / 28.6; 102 MB 27.1 / 27.4 | 27.8 / 28.0 | 30.9 / 29.2; 131 MB 28.2 / 30.2 | 32.4 / 30.6 | 34.3 / 32.2; 164 MB 33.2 / 39.0 | 41.0 / 39.6
    // | 42.6 / 41.2; 262 MB 47.1 / 48.3 | 53.0 / 48.4 | 54.9 / 50.7; 328 MB 64.3 / 58.2 | 63.8 / 58.4 | 65.6 / 60.6.
    if ((size_t)V * h * 2 > ((size_t)128 << 20)) return launch<VT, RT, VW, RW, KW, KB, true>(H, W, R, h, V, share, chunks, part, st);
    return launch<VT, RT, VW, RW, KW, KB, false>(H, W, R, h, V, share, chunks, part, st);
}

// Which arrangement, by the rows and by the tokens of a CU (`rows`):
//   LM_FEW   waves over the contraction: all waves have all rows, which is the fewest operand reads for few rows, and 256-byte pieces of memory
//   LM_WIDE  4 waves over the vocabulary, 2 over the rows
//   LM_TALL  2 and 4: fewer operand reads where a share is narrow and the rows are many
// us, FEW / WIDE: 40 rows, h = 2944, V = 12933 20.2 / 25.7; 65 at h = 2560, V = 22326 26.6 / 29.2; 77 at h = 3328, V = 24774 49 / 40.8; 55
// at h = 2176, V = 41403 47 / 39.8; 91 at h = 3840, V = 8110 24.1 / 31.3; 81 at h = 1024, V = 16000 16.8 / 15.1.  WIDE / TALL: 247 at h = 2304,
// V = 20296 43.9 / 39.5; 116 at h = 2048, V = 24000 27.6 / 26.1; 154 at h = 3328, V = 78883 116 / 145.
// As many tokens at once as the sums leave room for.  LM_FEW also leaves room for a ring of three stages (one row, V = 44928, h = 1920: 176 at once,
// in two stages, 36.0, two times 88 34.5).  LM_WIDE does not: its widest shares (up to 320 tokens, above 96 rows) have two stages, and from 193 rows
// on some operands in scratch memory, and are faster so than in two rounds.  us, as it is / 256 tokens at most above 96 rows / no more than three stages leave room for: h = 4096, V = 72000,
// 100 rows 134 / 147 / 147, 120 rows 134 / 140 / 136, 160 rows 144 / 164 / 160, 250 rows 187 / 204 / 213; h = 2048, V = 80000, 120 rows 74.4 / 73.7 / 74.4, 250 rows 106 / 117 / 122;
// h = 4096, V = 128256, 257 rows 290 / 296 / 327.
constexpr LmShares shares_of(int R, int V)
{
    const int rt = (R + 15) / 16, rows = (V + 255) / 256;
    LmShares p = {};
    p.form = rt > 6 ? rows <= 128 ? LM_TALL : LM_WIDE : rt > 5 ? rows <= 48 ? LM_FEW : LM_WIDE : rt > 2 && rows > 96 ? LM_WIDE : LM_FEW;
    const int tile = p.form == LM_WIDE ? 64 : 32;
    const int most = tile * (p.form == LM_TALL ? 4 : p.form == LM_WIDE ? (rt > 16 ? 4 : 5) : rt <= 2 ? 4 : rt <= 5 ? 3 : 2);
    const int rounds = (rows + most - 1) / most;
    p.share = std::max((V + 256 * rounds - 1) / (256 * rounds), std::min(V, 32));
    p.vt = (p.share + tile - 1) / tile;
    p.chunks = (V + p.share - 1) / p.share;
    return p;
}

// The fewest tiles of 16 tokens a wave that shares of this form come to, for lo to hi tiles of 16 rows.
constexpr int least_tiles(LmForm form, int lo, int hi)
{
    int least = INT_MAX;
    for (int rt = lo; rt <= hi; ++rt)
        for (int rows = 1; rows <= 1024; ++rows) {               // (per CU; more of them are cut into several rounds, of half of what fits at least)
            const LmShares p = shares_of(rt * 16, rows * 256);
            if (p.form == form) least = std::min(least, p.vt);
        }
    return least;
}

}  // namespace

LmShares lm_shares(int R, int V) { return shares_of(R, V); }

int lm_head_launch(const LmShares &p, const void *H, const void *W, int R, int h, int V, LmBest *part, hipStream_t st)
{
    const int t = (R + 15) / 16;
#define LM_SHARES(form_, lo, rows, rt, vw, rw, kw, kb, least, vts)                                                                      \
    if (t <= rows) {                                                                                                                 \
        static_assert(least_tiles(form_, lo, rows) == least, "every kernel can be reached");                                         \
        return pick<rt, vw, rw, kw, kb, least, vts>(p.vt, H, W, R, h, V, p.share, p.chunks, part, st);                               \
    }
    if (p.form == LM_TALL) {
#define LM_ROWS(lo, rows, rt, least, vts) LM_SHARES(LM_TALL, lo, rows, rt, 2, 4, 1, 64, least, vts)
        LM_ROWS(7, 8, 2, 1, 4) LM_ROWS(9, 12, 3, 1, 4) LM_ROWS(13, 16, 4, 1, 4) LM_ROWS(17, 20, 5, 1, 4)
#undef LM_ROWS
    } else if (p.form == LM_WIDE) {
#define LM_ROWS(lo, rows, rt, least, vts) LM_SHARES(LM_WIDE, lo, rows, rt, 4, 2, 1, 64, least, vts)
        LM_ROWS(3, 4, 2, 2, 5) LM_ROWS(5, 6, 3, 1, 5) LM_ROWS(7, 8, 4, 3, 5) LM_ROWS(9, 10, 5, 3, 5) LM_ROWS(11, 12, 6, 3, 5)
        LM_ROWS(13, 14, 7, 3, 5) LM_ROWS(15, 16, 8, 3, 5) LM_ROWS(17, 18, 9, 3, 4)
#undef LM_ROWS
    } else {
#define LM_ROWS(rows, least, vts) LM_SHARES(LM_FEW, rows, rows, rows, 2, 1, 4, 128, least, vts)
        LM_ROWS(1, 1, 4) LM_ROWS(2, 1, 4) LM_ROWS(3, 1, 3) LM_ROWS(4, 1, 3) LM_ROWS(5, 1, 3) LM_ROWS(6, 1, 2)
#undef LM_ROWS
    }
#undef LM_SHARES
    return btv_fail(BTV_EINVAL, "no LM-head kernel for %d rows", R);
}
