// Tree-masked attention for gfx950 (MI355X): ancestor bitmask, bf16 MFMA split-K kernels (one request, batches of short
// requests, batches whose workgroups share the work out; bf16 or FP8 K/V), fp32 reference-precision kernel, split-K
// combine, and their C-ABI entry points.
//
// What is computed (App. C, "Linearization and verification mask"): node i attends to the L
// prefix rows of the KV cache and to the tree rows of its ancestors and itself.
//
// bf16 kernel layout.  For one KV head the G = Hq/Hkv query heads of every node are packed
// into rows r = i*G + j, so the whole GQA group shares each K/V byte that is streamed.
// A workgroup (4 or 8 wavefronts of 64 lanes) owns WR rows and a range of 32-key tiles; K and V
// tiles are staged through LDS once per workgroup (ring of stages filled by direct-to-LDS loads).
// Scores are computed transposed, S^T = K . Q^T with 32x32x16 bf16 MFMA: in the accumulator
// layout a lane then holds ONE query column and 16 keys, so the running max / sum of the
// online softmax are per-lane scalars (one cross-half exchange per tile), the P^T tile is
// already in B-operand layout for O^T += V^T . P^T, and the O^T accumulator is rescaled by a
// per-lane factor.  V^T operands come from transposing LDS reads.  The tree mask is applied only on tiles
// that touch tree rows, from a 32-bit visibility word per (query, tile) built from the node's
// ancestor bitmask.
#include "btv_common.h"

#include <atomic>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int TK = 32;          // keys per tile = per LDS stage
constexpr float NEG_BIG = -1.0e30f;

struct AttnParams {
    const void *Q, *K, *V;
    void *O;
    const int32_t *parent;        // [total_M], indices local to each request
    const int32_t *block_table;   // paged only
    const int32_t *q_offset;      // paged only, [batch+1]
    const int32_t *prefix_len;    // paged only, [batch]
    _Float16 *Opart;              // [nsplit][total_rows][D]: split partial of O^T's row, divided by its largest magnitude
    float *ML;                    // [nsplit][total_rows][4]: reference max, row sum, that magnitude, unused
    uint32_t *flag;
    unsigned long long *sync;     // one request: words of the merge inside the attention kernel (null: tv_combine_bf16 merges)
    int wait_ticks;               // ... how long a workgroup waits for the others of its group
    int M, L;                     // contiguous: actual sizes; paged: host upper bounds
    int Hq, Hkv, G;
    int ginv;                     // ceil(2^16 / G): (x * ginv) >> 16 = x / G for every packed row x < 4096 (G <= 16)
    int max_blocks, num_blocks;
    int total_rows;               // rows of the partial buffers (>= total_M * Hq)
    int total_M;
    int sps;                      // one request: whole tiles per split (`longer` of them take a round more); batch: tiles per part
    int longer;
    int nsplit;                   // key splits (batch: of the longest request)
    int row_blocks, units;        // row blocks per (split, head, request) unit; number of units
    uint32_t inv_row_blocks, inv_nsplit, inv_sps, inv_Hkv;    // for quotient()
    long long *plan;              // batch only: [batch + 2], where the requests' work starts (see Stretch)
    int batch, teams_log2, pairing, wmin, wr_log2;   // batch only: requests, teams of workgroups, whether a team is a pair, smallest share, rows per block
    float scale;                  // softmax scale
    float scale_log2;             // scale * log2(e) (times the key scale of an FP8 cache)
    float out_scale;              // 1, or the value scale of an FP8 cache
};

// n / d for n >= 0, with inv = reciprocal(d).  (A division by a number that the compiler does not know takes some 30 instructions, and a workgroup
// has three to five of them ahead of its first load.)
__host__ constexpr uint32_t reciprocal(int d) { return d <= 1 ? 0u : (uint32_t)((0x100000000ull + (unsigned)d - 1) / (unsigned)d); }
__device__ __forceinline__ int quotient(int n, int d, uint32_t inv)
{
    const int q = (int)__umulhi((uint32_t)n, inv);      // at most one too many
    return d == 1 ? n : q - (q * d > n);
}

__device__ __forceinline__ uint32_t float_to_bf16_bits(float f)
{   // round to nearest even; inputs here are finite
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Request geometry: contiguous calls have one request; paged calls read it from device arrays
// and clamp against the host-provided bounds so that no access can leave its buffer.
struct Req { int q0, M, L; bool ok; };

template <bool PAGED>
__device__ __forceinline__ Req load_req(const AttnParams &p, int r)
{
    Req q;
    if (!PAGED) { q.q0 = 0; q.M = p.M; q.L = p.L; q.ok = true; return q; }
    q.q0 = p.q_offset[r];
    q.M = p.q_offset[r + 1] - q.q0;
    q.L = p.prefix_len[r];
    q.ok = q.M >= 1 && q.M <= p.M && q.L >= 0 && q.L <= p.L && q.q0 >= 0 &&
           q.q0 + q.M <= p.total_M && (long long)q.L + q.M <= (long long)p.max_blocks * BTV_PAGE;
    return q;
}

// Visibility of keys kb..kb+31 for a node: bit c set iff key kb+c is a prefix row, or a tree
// row L+a with a in anc(node).  Bits of anc past the request's node count are zero.
// AncT is either a pointer to the node's BTV_ANC_WORDS words or a register array of them.
template <typename AncT>
__device__ __forceinline__ uint32_t anc_word(const AncT &anc, int w)
{
    uint32_t r = 0u;
#pragma unroll
    for (int k = 0; k < BTV_ANC_WORDS; ++k) r = (k == w) ? anc[k] : r;
    return r;
}

template <typename AncT>
__device__ __forceinline__ uint32_t vis_word(const AncT &anc, int kb, int L)
{
    int off = kb - L;
    if (off <= -32) return 0xFFFFFFFFu;
    if (off < 0) {
        int n = -off;
        return ((1u << n) - 1u) | (anc_word(anc, 0) << n);
    }
    int w = off >> 5, sh = off & 31;
    uint32_t lo = anc_word(anc, w), hi = anc_word(anc, w + 1);
    return sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
}

// ------------------------------------------------------------------------------------------------
// Ancestor bitmask: anc[i] = {i} u anc[parent[i]].  One workgroup, one thread per node,
// each walking its own chain (parents are strictly decreasing, so the walk ends; an out-of-range
// parent is treated as -1 and flagged).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void anc_mask_kernel(const int32_t *parent, int M, uint32_t *anc, uint32_t *flag)
{
    __shared__ int32_t par[BTV_MAX_NODES];
    int i = threadIdx.x;
    bool bad = false;
    if (i < M) {
        int pa = parent[i];
        if (pa < -1 || pa >= i) { bad = true; pa = -1; }
        par[i] = pa;
    }
    __syncthreads();
    if (i < M) {
        uint32_t w[BTV_ANC_WORDS];
#pragma unroll
        for (int k = 0; k < BTV_ANC_WORDS; ++k) w[k] = 0u;
        for (int a = i; a >= 0; a = par[a]) {
#pragma unroll
            for (int k = 0; k < BTV_ANC_WORDS; ++k)
                if ((a >> 5) == k) w[k] |= 1u << (a & 31);
        }
        uint4 *dst = reinterpret_cast<uint4 *>(anc + (size_t)i * BTV_ANC_WORDS);
        dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
        dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
    if (bad) atomicOr(flag, 1u);
}

// ------------------------------------------------------------------------------------------------
// bf16 MFMA kernel
//
// LDS holds a ring of NT stages; a stage is one 32-key tile: the K rows and the V rows exactly as
// they lie in memory ([key][channel], 2*D bytes per row).  Stages are filled by direct-to-LDS
// global loads (each lane moves 16 bytes, a wave instruction fills 1 KiB of LDS), so no staging
// registers and no VALU work are spent on data movement and up to NT-1 stages stay in flight.
// Bank conflicts are avoided by choosing which 16-byte chunk of a row each lane fetches: the chunk
// stored at physical position pc of LDS row r is chunk pc ^ f(r) of the source row.
//   K: LDS row i holds key kb + swap_bits_2_3(i) (the MFMA A-row order that makes a lane's 16 score
//      registers two runs of 8 consecutive keys); A operands are 16-byte LDS reads.
//   V: LDS row r holds key kb + r; the V^T A operand (one channel, 8 consecutive keys per lane) comes
//      from two transposing LDS reads (ds_read_b64_tr_b16): a 16-lane group reads 4 keys x 16 channels
//      and every lane receives the 4 keys of its own channel.
// ------------------------------------------------------------------------------------------------
// EB = bytes per K/V element in memory and in LDS: 2 (bf16) or 1 (FP8 E4M3, converted to bf16 in registers after
// the operand reads: every E4M3 number is a bf16 number, so the conversion is exact).
template <int D, int EB = 2>
struct Lds {
    static constexpr int ROWB = EB * D;                      // bytes per K or V row
    static constexpr int TILEB = 32 * ROWB;                  // one K (or V) tile
    static constexpr int STAGE = 2 * TILEB;                  // K tile then V tile
    static constexpr int INSTR = STAGE / 1024;               // wave-wide 1 KiB fills per tile
    static constexpr int CHUNKS = ROWB / 16;                 // 16-byte chunks per row
};

__device__ __forceinline__ int swap_bits_2_3(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }

// bf16 rows (2*D bytes): consecutive rows start on the same bank, so the chunk is rotated by the row number.
// FP8 rows of 128 bytes: even and odd rows already sit in different halves of the 64 banks, so pairs of rows share a
// rotation.
template <int D, int EB = 2> __device__ __forceinline__ int swz_k(int row)
{
    return EB == 2 ? (row & (D / 8 - 1)) : ((row >> 1) & (Lds<D, EB>::CHUNKS - 1));
}
// V rows, bf16: the four rows a 16-lane group of a transposing read touches (row % 4 = 0..3) are moved 64 bytes
// apart.  FP8: a group touches 8 rows x 16 bytes and two groups (32 bytes per row) are served together; the four
// even (and the four odd) rows among them are moved 32 bytes apart.
template <int D, int EB = 2> __device__ __forceinline__ int swz_v(int row)
{
    return EB == 2 ? (((row & 3) << 2) & (D / 8 - 1)) : ((((row >> 1) & 3) << 1) & (Lds<D, EB>::CHUNKS - 1));
}

#define BTV_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// 16 bytes of every lane straight to LDS, lane after lane from dst on (uniform)
__device__ __forceinline__ void fill_lds(const unsigned char *src, unsigned char *dst)
{
    __builtin_amdgcn_global_load_lds(src, BTV_LDS_PTR(dst), 16, 0, 0);
}

// Per-wave, loop-invariant part of the ring fills.  A wave issues LPW fills per tile; fill jj of wave w is
// instruction j = w*LPW + jj of the tile (K part first).  Lane l of it fills LDS row r, physical chunk pc, with
// source row key_off (relative to the tile's first key) and source chunk pc ^ swizzle(r).  A wave's fills of a tile are ROWS rows of K
// or of V, all in the same half of the tile (the permutation of the K rows stays within 16), so in a paged cache of one page.
template <int D, int WAVES, bool PAGED, int EB = 2>
struct Fill {
    static constexpr int LPW = Lds<D, EB>::INSTR / WAVES, ROWS = 64 / WAVES;
    static_assert(LPW >= 1 && LPW * WAVES == Lds<D, EB>::INSTR, "fills must divide evenly over the waves");
    static_assert(ROWS <= 16 && BTV_PAGE == 16, "a wave's rows are of one half of the tile: of one page");
    const unsigned char *base;      // K or V of this KV head (wave-uniform)
    const int32_t *block_table;     // row of this request (paged)
    uint32_t pages;                 // paged, lane l: page of this wave's rows in tile l of a window of 32 (PGV)
    int num_blocks, S, half;
    uint32_t row_bytes;             // Hkv * D * EB: distance between consecutive keys
    uint32_t lane_off[LPW];         // contiguous: key_off*row_bytes + chunk*16;  paged: (key_off & 15)*row_bytes + chunk*16
    // where the 16 rows of a page begin (an id from the block table is clamped, so that no access can leave the pool)
    __device__ __forceinline__ int valid_page(int id) const { return min(max(id, 0), num_blocks - 1); }
    // The page of the wave's rows in tile st (constant space: a scalar load, so that the vector-memory counter only ever counts the LDS
    // fills).  Past the end it is the last page: rows of the tile's upper half re-read the lower half's last row then.
    __device__ __forceinline__ int page_id(int st) const
    {
        typedef const __attribute__((address_space(4))) int32_t *const_i32;
        const const_i32 bt = reinterpret_cast<const_i32>(reinterpret_cast<uintptr_t>(block_table));
        return bt[__builtin_amdgcn_readfirstlane(min(2 * st + half, (S - 1) >> 4))];
    }
    __device__ __forceinline__ const unsigned char *page(int id) const { return base + (size_t)(uint32_t)id * (BTV_PAGE * row_bytes); }
};

template <int D, int WAVES, bool PAGED, int EB = 2>
__device__ __forceinline__ Fill<D, WAVES, PAGED, EB> make_fill(const void *K, const void *V, const int32_t *bt, int num_blocks,
                                                               int Hkv, int g, int S, int w, int l)
{
    using LD = Lds<D, EB>;
    constexpr int CH = LD::CHUNKS, RPI = 1024 / LD::ROWB;
    Fill<D, WAVES, PAGED, EB> f;
    const bool isv = w >= WAVES / 2;                 // (uniform)
    f.base = static_cast<const unsigned char *>(isv ? V : K) + (size_t)g * D * EB;
    f.block_table = bt; f.num_blocks = num_blocks; f.S = S;
    f.half = (w * f.ROWS & 16) >> 4;
    f.row_bytes = (uint32_t)Hkv * D * EB;
#pragma unroll
    for (int jj = 0; jj < f.LPW; ++jj) {
        const int r = (w * f.LPW + jj) * RPI % 32 + l / CH, pc = l % CH;
        const int key_off = isv ? r : swap_bits_2_3(r);
        const int chunk = pc ^ (isv ? swz_v<D, EB>(r) : swz_k<D, EB>(r));
        f.lane_off[jj] = (uint32_t)(PAGED ? (key_off & 15) : key_off) * f.row_bytes + chunk * 16;
    }
    return f;
}

// Source row (relative to the tile's first key) of lane l in fill jj of wave w: recomputed where it is needed (the
// clamped last tile) rather than kept in registers through the main loop.
template <int D, int WAVES, int EB>
__device__ __forceinline__ int fill_key_off(int w, int jj, int l)
{
    using LD = Lds<D, EB>;
    constexpr int CH = LD::CHUNKS, RPI = 1024 / LD::ROWB, LPW = LD::INSTR / WAVES;
    const int r = (w * LPW + jj) * RPI % 32 + l / CH;
    return w >= WAVES / 2 ? r : swap_bits_2_3(r);
}

// Issue this wave's share of the direct-to-LDS loads of tile `st` (keys 32*st ..) into ring slot `slot`.
// Keys past the end of the sequence re-read the last valid row (finite data; their scores are masked).
// JB .. JE - 1: which of the wave's LPW fills (all by default; the pipelined loop issues them one by one, each behind a
// group of MFMAs, because an issue holds its wave for about a hundred cycles).
// PGV: the page comes from lane `at` of the window in f.pages, else from a scalar load.
template <int D, int WAVES, bool PAGED, int EB = 2, int JB = 0, int JE = Lds<D, EB>::INSTR / WAVES, bool PGV = false>
__device__ __forceinline__ void issue_tile(const Fill<D, WAVES, PAGED, EB> &f, unsigned char *smem, int slot, int st, int w, int l, int at = 0)
{
    using LD = Lds<D, EB>;
    const int kb = st * 32;
    const bool whole = kb + 32 <= f.S;       // uniform: no key of this tile needs clamping
    const unsigned char *src;                // uniform
    if constexpr (!PAGED) src = f.base + (size_t)kb * f.row_bytes;
    else if constexpr (PGV) src = f.page(__builtin_amdgcn_readlane((int)f.pages, at));
    else {
        src = f.page(f.valid_page(f.page_id(st)));
    }
    uint32_t off[JE];
#pragma unroll
    for (int jj = JB; jj < JE; ++jj) off[jj] = f.lane_off[jj];
    if (!whole) {
#pragma unroll
        for (int jj = JB; jj < JE; ++jj) {
            const int ko = fill_key_off<D, WAVES, EB>(w, jj, l), kc = min(kb + ko, f.S - 1) - kb;
            off[jj] += (uint32_t)(PAGED ? (kc & 15) - (ko & 15) : kc - ko) * f.row_bytes;
        }
    }
#pragma unroll
    for (int jj = JB; jj < JE; ++jj) {
        asm volatile("" : "+v"(off[jj]));    // (one branch for all of them: else there is one for each)
        fill_lds(src + off[jj], smem + slot * LD::STAGE + (w * f.LPW + jj) * 1024);
    }
}

// ---- LDS operand reads ---------------------------------------------------------------------------
// All operand reads are raw instructions with explicit counter waits: as ordinary loads / builtins the
// compiler would drain the whole vector-memory queue (the ring fills still in flight) in front of every tile.
// Each wait takes the registers it covers as in/out operands, so no use can be scheduled above it.
//
// K A-operands: lane (c = l%32, h = l/32) reads chunk (2s+h) ^ swz_k(c) of LDS row c for s = 0..D/16-1.  Row
// starts are 2*D-byte aligned, so the address is  (tile + lane part) ^ (s << 5).
template <int D> __device__ __forceinline__ uint32_t lane_k_off(int l)
{
    const int c = l & 31, h = l >> 5;
    return (uint32_t)(c * Lds<D>::ROWB + ((h ^ swz_k<D>(c)) << 4));
}

template <int D> __device__ __forceinline__ void lds_read_k(uint32_t a, u32x4 (&ka)[D / 16])
{
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
        const uint32_t addr = a ^ (uint32_t)(s << 5);
        asm volatile("ds_read_b128 %0, %1" : "=v"(ka[s]) : "v"(addr));
    }
}

template <int DS, int YOUNGER> __device__ __forceinline__ void lds_wait_k(u32x4 (&ka)[DS])
{
    static_assert(DS == 4 || DS == 8, "D in {64,128}");
    if constexpr (DS == 8)
        asm volatile("s_waitcnt lgkmcnt(%8)"
                     : "+v"(ka[0]), "+v"(ka[1]), "+v"(ka[2]), "+v"(ka[3]), "+v"(ka[4]), "+v"(ka[5]), "+v"(ka[6]), "+v"(ka[7])
                     : "n"(YOUNGER));
    else
        asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(ka[0]), "+v"(ka[1]), "+v"(ka[2]), "+v"(ka[3]) : "n"(YOUNGER));
}

// V^T A-operands (ds_read_b64_tr_b16): lane l sits in 16-lane group l/16 = 2h + dhalf; for (dt, mm, i) it
// supplies the address of key row 16mm + 8h + 4i + (l%16)/4, channels 32dt + 16dhalf + 4(l%4) .. +3, and
// receives keys 16mm + 8h + 4i .. +3 of channel 32dt + (l%32).  With the V swizzle the address is
// ((tile + lane part) ^ (dt << 6)) + (16mm + 4i) * row bytes, the last term an immediate offset.
template <int D> __device__ __forceinline__ uint32_t lane_v_off(int l)
{
    const int h = l >> 5, dhalf = (l >> 4) & 1, rr = (l & 15) >> 2, q = l & 3;
    const int x = 2 * dhalf + (q >> 1);
    return (uint32_t)((8 * h + rr) * Lds<D>::ROWB + ((swz_v<D>(rr) ^ x) << 4) + ((q & 1) << 3));
}

// The reads for keys 16*MM .. 16*MM + 15 (the operands of the PV MFMAs with index mm = MM): 2*D/32 instructions.
template <int D, int MM> __device__ __forceinline__ void lds_read_vt(uint32_t a, bf16x4 (&va)[D / 32][2][2])
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        const uint32_t addr = a ^ (uint32_t)(dt << 6);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                         : "=v"(va[dt][MM][i])
                         : "v"(addr), "n"((16 * MM + 4 * i) * Lds<D>::ROWB));
    }
}

template <int DT>
__device__ __forceinline__ void lds_wait_vt(bf16x4 (&va)[DT][2][2])
{
    static_assert(DT == 2 || DT == 4, "D in {64,128}");
    if constexpr (DT == 4)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(va[0][0][0]), "+v"(va[0][0][1]), "+v"(va[0][1][0]), "+v"(va[0][1][1]), "+v"(va[1][0][0]),
                       "+v"(va[1][0][1]), "+v"(va[1][1][0]), "+v"(va[1][1][1]), "+v"(va[2][0][0]), "+v"(va[2][0][1]),
                       "+v"(va[2][1][0]), "+v"(va[2][1][1]), "+v"(va[3][0][0]), "+v"(va[3][0][1]), "+v"(va[3][1][0]),
                       "+v"(va[3][1][1]));
    else
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(va[0][0][0]), "+v"(va[0][0][1]), "+v"(va[0][1][0]), "+v"(va[0][1][1]), "+v"(va[1][0][0]),
                       "+v"(va[1][0][1]), "+v"(va[1][1][0]), "+v"(va[1][1][1]));
}

// ---- the arithmetic steps of one 32-key tile of one wave (32 query rows) ---------------------------------
// S^T = K . Q^T
template <int DS>
__device__ __forceinline__ f32x16 qk_tile(const u32x4 (&ka)[DS], const bf16x8 (&qreg)[DS], f32x16 s)
{
#pragma unroll
    for (int k = 0; k < DS; ++k)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[k]), qreg[k], s, 0, 0, 0);
    return s;
}

// largest score of the lane's query over the 32 keys (the other half of the wave holds the other 16)
__device__ __forceinline__ float tile_max(const f32x16 &s)
{
    float t = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, s[v]);
    auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// Scores arrive in log2 units: the queries were multiplied by scale * log2(e) once, in the prologue, so a
// probability is exp2(score - reference) with no multiply per element.
//
// One half (keys 8 mm .. 8 mm + 7 of the lane's 16) of a tile whose scores already are relative to the reference:
// P = exp2(x) as a B operand, its rounded values added to `sum`.
__device__ __forceinline__ void exp_half(const f32x16 &x, int mm, bf16x8 &pbm, float &sum)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = { (__bf16)1.0f, (__bf16)1.0f };
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(x[mm * 8 + e]);
        const float p1 = __builtin_amdgcn_exp2f(x[mm * 8 + e + 1]);
        const bf16x2 pp = { (__bf16)p0, (__bf16)p1 };
        pbm[e] = pp[0];
        pbm[e + 1] = pp[1];
        sum = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, sum, false);
    }
}

// The reference of the step-by-step tiles enters through the matrix cores as well: the score accumulator starts from
// -base (negb: the same value in all 16 registers), base being the running maximum once there is one (0 before), so
// the scores arrive relative to it and a probability is exp2 of the accumulator as it stands.  The reference only moves where
// the tile's maximum exceeds it by more than LAZY, so that probabilities stay below 2^LAZY and most tiles rescale nothing; the
// result is the same, numerator and denominator refer to the same m_run.  Where it moves the tile's scores are shifted by hand.
template <int DT>
__device__ __forceinline__ void rebase_tile(f32x16 &srel, float &base, f32x16 &negb, float &m_run, float &l_run, f32x16 (&oacc)[DT])
{
    constexpr float LAZY = 8.0f;
    const float rmax = tile_max(srel);
    const bool grow = (rmax + base) - m_run > LAZY;
    if (__builtin_amdgcn_ballot_w64(grow) != 0ull) {
        const float mnew = grow ? rmax + base : m_run;
        const float alpha = __builtin_amdgcn_exp2f(m_run - mnew);
        m_run = mnew;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
        const float nb = m_run > 0.5f * NEG_BIG ? m_run : 0.f;
        const float d = nb - base;
        base = nb;
#pragma unroll
        for (int v = 0; v < 16; ++v) { srel[v] -= d; negb[v] = -nb; }
    }
}

// Probabilities of a tile whose scores are relative to the reference.  The reference has to follow the scores up (rebase_tile)
// where there is none yet or the tile is masked (`exact`); otherwise nothing stands between the scores and their
// exponentials, and the tile's sum tells afterwards whether one of them exceeded 16: then it is done again, against a new one.  (The
// maximum, its exchange between the halves of the wave and the branch on it are 150 cycles of a tile's 1300 to 1800.)
constexpr float GROW = 1048576.0f;       // 2^20: a sum of 16 terms above it means some score > 16
template <int DT>
__device__ __forceinline__ void probabilities(f32x16 &x, bool exact, float &base, f32x16 &negb, float &m_run, float &l_run, f32x16 (&oacc)[DT],
                                              bf16x8 (&pb)[2])
{
    if (exact) rebase_tile<DT>(x, base, negb, m_run, l_run, oacc);
    float ts[2] = { 0.f, 0.f };
    exp_half(x, 0, pb[0], ts[0]);
    exp_half(x, 1, pb[1], ts[1]);
    float sum = ts[0] + ts[1];
    if (!exact && __builtin_amdgcn_ballot_w64(!(sum <= GROW)) != 0ull) {
        rebase_tile<DT>(x, base, negb, m_run, l_run, oacc);
        ts[0] = ts[1] = 0.f;
        exp_half(x, 0, pb[0], ts[0]);
        exp_half(x, 1, pb[1], ts[1]);
        sum = ts[0] + ts[1];
    }
    l_run += sum;
}

// O^T += V^T . P^T
template <int DT>
__device__ __forceinline__ void pv_tile(const bf16x4 (&va)[DT][2][2], const bf16x8 (&pb)[2], f32x16 (&oacc)[DT])
{
#pragma unroll
    for (int mm = 0; mm < 2; ++mm)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const bf16x8 a = __builtin_shufflevector(va[dt][mm][0], va[dt][mm][1], 0, 1, 2, 3, 4, 5, 6, 7);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[mm], oacc[dt], 0, 0, 0);
        }
}

// tree mask of a tile that touches tree rows (or the end of the sequence)
__device__ __forceinline__ void mask_tile(f32x16 &s, uint32_t vis, int h)
{
    vis >>= 8 * h;
    asm volatile("" : "+v"(vis));            // (what follows from the lane alone would be worked out ahead of the loop, in calls without a mask too)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int bit = 16 * (v >> 3) + (v & 7);
        if (!((vis >> bit) & 1u)) s[v] = -INFINITY;
    }
}

// One whole tile, step after step (no overlap between the steps): used for the tiles that need the mask and
// by the workgroup shapes whose wave pairs alternate over the tiles.  PLAIN: prefix rows only, and not the wave's first tile;
// `exact` (see probabilities) else.
template <int D, bool PLAIN>
__device__ __forceinline__ void do_tile(uint32_t stage, int kb, int Lr, int l,
                                        const uint32_t (&anc_i)[BTV_ANC_WORDS],
                                        const bf16x8 (&qreg)[D / 16], float &m_run, float &l_run, f32x16 (&oacc)[D / 32],
                                        float &base, f32x16 &negb, bool exact)
{
    constexpr int DS = D / 16, DT = D / 32;
    u32x4 ka[DS];
    bf16x4 va[DT][2][2];
    const uint32_t va_addr = stage + Lds<D>::TILEB + lane_v_off<D>(l);
    lds_read_k<D>(stage + lane_k_off<D>(l), ka);
    lds_read_vt<D, 0>(va_addr, va);
    lds_wait_k<DS, DT * 2>(ka);          // the counter completes in order: K has landed when 2*DT reads remain
    lds_read_vt<D, 1>(va_addr, va);
    f32x16 s = qk_tile<DS>(ka, qreg, negb);
    if (!PLAIN && kb + 32 > Lr) mask_tile(s, vis_word(anc_i, kb, Lr), l >> 5);
    bf16x8 pb[2];
    probabilities<DT>(s, !PLAIN && exact, base, negb, m_run, l_run, oacc, pb);
    lds_wait_vt<DT>(va);
    pv_tile<DT>(va, pb, oacc);
}

// ---- FP8 (E4M3) K/V: operand reads and exact conversion to bf16 ---------------------------------------
// K: a lane reads 16 consecutive channels (16 bytes) of its key row, channels 32 s + 16 h .. + 15 for s = 0 .. D/32-1,
// and uses the first 8 for contraction step 2s, the last 8 for step 2s+1.  The contraction steps thus take the
// channels in another order than the bf16 layout; the query operands are loaded in the same order, so the sum is
// over the same products.  Address: (tile + lane part) ^ (s << 5), as for bf16 with 128-byte rows.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int D> __device__ __forceinline__ uint32_t lane_k8_off(int l)
{
    const int c = l & 31, h = l >> 5;
    return (uint32_t)(c * Lds<D, 1>::ROWB + ((h ^ swz_k<D, 1>(c)) << 4));
}

template <int D> __device__ __forceinline__ void lds_read_k8(uint32_t a, u32x4 (&k8)[D / 32])
{
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        const uint32_t addr = a ^ (uint32_t)(s << 5);
        asm volatile("ds_read_b128 %0, %1" : "=v"(k8[s]) : "v"(addr));
    }
}

template <int YOUNGER> __device__ __forceinline__ void lds_wait_k8(u32x4 (&k8)[4])
{
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(k8[0]), "+v"(k8[1]), "+v"(k8[2]), "+v"(k8[3]) : "n"(YOUNGER));
}

// Two E4M3 codes (one 16-bit half of a register) to two bf16, scale 1: exact for every code.
__device__ __forceinline__ uint32_t fp8x2_to_bf16x2(uint32_t w, bool high)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 r = high ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true)
                          : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    return __builtin_bit_cast(uint32_t, r);
}

// eight consecutive codes (two registers) -> one bf16 MFMA operand
__device__ __forceinline__ bf16x8 fp8x8_to_bf16x8(uint32_t w0, uint32_t w1)
{
    const u32x4 r = { fp8x2_to_bf16x2(w0, false), fp8x2_to_bf16x2(w0, true), fp8x2_to_bf16x2(w1, false),
                      fp8x2_to_bf16x2(w1, true) };
    return __builtin_bit_cast(bf16x8, r);
}

// V^T operands (ds_read_b64_tr_b8): a 16-lane group reads 8 key rows x 16 channels; lane j of the group supplies
// the address of row j/2, bytes 8 (j%2) .. + 7 of the group's 16 channels, and receives the 8 keys of channel j.
// Lane l sits in group l/16 = 2h + dhalf; for (dt, mm) the group reads keys 16mm + 8h .. + 7, channels
// 32dt + 16dhalf .. + 15, so the lane receives keys 16mm + 8h .. + 7 of channel 32dt + (l%32): one whole operand
// of the PV MFMA with index mm.  With the V swizzle the address is ((tile + lane part) ^ (dt << 5)) + 16mm * row
// bytes, the last term an immediate offset.
template <int D> __device__ __forceinline__ uint32_t lane_v8_off(int l)
{
    const int h = l >> 5, dhalf = (l >> 4) & 1, j = l & 15;
    const int row = 8 * h + (j >> 1);
    return (uint32_t)(row * Lds<D, 1>::ROWB + ((swz_v<D, 1>(row) ^ dhalf) << 4) + ((j & 1) << 3));
}

template <int D, int MM> __device__ __forceinline__ void lds_read_vt8(uint32_t a, u32x2 (&v8)[D / 32][2])
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        const uint32_t addr = a ^ (uint32_t)(dt << 5);
        asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(v8[dt][MM]) : "v"(addr), "n"(16 * MM * Lds<D, 1>::ROWB));
    }
}

__device__ __forceinline__ void lds_wait_vt8(u32x2 (&v8)[4][2])
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v8[0][0]), "+v"(v8[0][1]), "+v"(v8[1][0]), "+v"(v8[1][1]), "+v"(v8[2][0]), "+v"(v8[2][1]),
                   "+v"(v8[3][0]), "+v"(v8[3][1]));
}

// One whole tile of an FP8 cache: the same steps as do_tile with half the operand reads and the conversions.
template <int D, bool PLAIN>
__device__ __forceinline__ void do_tile8(uint32_t stage, int kb, int Lr, int l,
                                         const uint32_t (&anc_i)[BTV_ANC_WORDS],
                                         const bf16x8 (&qreg)[D / 16], float &m_run, float &l_run, f32x16 (&oacc)[D / 32],
                                         float &base, f32x16 &negb, bool exact)
{
    static_assert(D == 128, "FP8 K/V: head dimension 128 only");
    constexpr int DS = D / 16, DT = D / 32;
    u32x4 k8[DS / 2];
    u32x2 v8[DT][2];
    const uint32_t va_addr = stage + Lds<D, 1>::TILEB + lane_v8_off<D>(l);
    lds_read_k8<D>(stage + lane_k8_off<D>(l), k8);
    lds_read_vt8<D, 0>(va_addr, v8);
    lds_wait_k8<DT>(k8);                 // the counter completes in order: K has landed when DT reads remain
    lds_read_vt8<D, 1>(va_addr, v8);
    f32x16 s = negb;
#pragma unroll
    for (int k = 0; k < DS / 2; ++k) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp8x8_to_bf16x8(k8[k][0], k8[k][1]), qreg[2 * k], s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp8x8_to_bf16x8(k8[k][2], k8[k][3]), qreg[2 * k + 1], s, 0, 0, 0);
    }
    if (!PLAIN && kb + 32 > Lr) mask_tile(s, vis_word(anc_i, kb, Lr), l >> 5);
    bf16x8 pb[2];
    probabilities<DT>(s, !PLAIN && exact, base, negb, m_run, l_run, oacc, pb);
    lds_wait_vt8(v8);
#pragma unroll
    for (int mm = 0; mm < 2; ++mm)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp8x8_to_bf16x8(v8[dt][mm][0], v8[dt][mm][1]), pb[mm],
                                                               oacc[dt], 0, 0, 0);
}

// ---- half-tile operand buffers of the software-pipelined loop ----------------------------------------------
// The loop keeps 16 registers of K operands and 16 of V^T operands (D = 128): half a tile each, refilled right
// after the MFMAs that consumed the previous contents were issued.  Addresses are loop-invariant registers (one
// per contraction step / channel block, the XOR of the swizzle already applied); the ring slot is an immediate
// offset, which reaches SPB slots from one base (the offset field has 16 bits).
template <int OFF> __device__ __forceinline__ void ds_read_k_imm(uint32_t a, u32x4 &r)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset range");
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
}
template <int OFF> __device__ __forceinline__ void ds_read_vt_imm(uint32_t a, bf16x4 &r)
{
    static_assert(OFF >= 0 && OFF < 65536, "immediate offset range");
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
}

// K operands of contraction steps HALF * DS/2 .. + DS/2 - 1 of the tile in slot SLOT (relative to the base in ak).
template <int D, int SLOT, int HALF> __device__ __forceinline__ void read_k_half(const uint32_t (&ak)[D / 16], u32x4 (&kh)[D / 32])
{
#pragma unroll
    for (int s = 0; s < D / 32; ++s) ds_read_k_imm<SLOT * Lds<D>::STAGE>(ak[HALF * (D / 32) + s], kh[s]);
}
// V^T operands of keys 16 MM .. 16 MM + 15 (the PV MFMAs with index MM), all channel blocks.
template <int D, int SLOT, int MM> __device__ __forceinline__ void read_v_half(const uint32_t (&av)[D / 32], bf16x4 (&vh)[D / 32][2])
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        ds_read_vt_imm<SLOT * Lds<D>::STAGE + (16 * MM) * Lds<D>::ROWB>(av[dt], vh[dt][0]);
        ds_read_vt_imm<SLOT * Lds<D>::STAGE + (16 * MM + 4) * Lds<D>::ROWB>(av[dt], vh[dt][1]);
    }
}
// the same reads with the stage address in a register (prologue and epilogue of the loop)
template <int D, int HALF> __device__ __forceinline__ void read_k_half_at(uint32_t a, u32x4 (&kh)[D / 32])
{
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        const uint32_t addr = a ^ (uint32_t)((HALF * (D / 32) + s) << 5);
        asm volatile("ds_read_b128 %0, %1" : "=v"(kh[s]) : "v"(addr));
    }
}
template <int D, int MM> __device__ __forceinline__ void read_v_half_at(uint32_t a, bf16x4 (&vh)[D / 32][2])
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        const uint32_t addr = a ^ (uint32_t)(dt << 6);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(vh[dt][i]) : "v"(addr), "n"((16 * MM + 4 * i) * Lds<D>::ROWB));
    }
}
// Wait until at most YOUNGER LDS reads issued after these are still in flight (the counter completes in order).
template <int KH, int YOUNGER> __device__ __forceinline__ void wait_k_half(u32x4 (&kh)[KH])
{
    static_assert((KH == 2 || KH == 4) && YOUNGER >= 0 && YOUNGER < 16, "D in {64,128}");
    if constexpr (KH == 4) asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(kh[0]), "+v"(kh[1]), "+v"(kh[2]), "+v"(kh[3]) : "n"(YOUNGER));
    else asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(kh[0]), "+v"(kh[1]) : "n"(YOUNGER));
}
template <int DT, int YOUNGER> __device__ __forceinline__ void wait_v_half(bf16x4 (&vh)[DT][2])
{
    static_assert((DT == 2 || DT == 4) && YOUNGER >= 0 && YOUNGER < 16, "D in {64,128}");
    if constexpr (DT == 4)
        asm volatile("s_waitcnt lgkmcnt(%8)"
                     : "+v"(vh[0][0]), "+v"(vh[0][1]), "+v"(vh[1][0]), "+v"(vh[1][1]), "+v"(vh[2][0]), "+v"(vh[2][1]),
                       "+v"(vh[3][0]), "+v"(vh[3][1])
                     : "n"(YOUNGER));
    else
        asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(vh[0][0]), "+v"(vh[0][1]), "+v"(vh[1][0]), "+v"(vh[1][1]) : "n"(YOUNGER));
}
// half of S^T = K . Q^T: contraction steps HALF * DS/2 .. on top of c
template <int DS, int HALF>
__device__ __forceinline__ f32x16 qk_half(const u32x4 (&kh)[DS / 2], const bf16x8 (&qreg)[DS], f32x16 c)
{
#pragma unroll
    for (int k = 0; k < DS / 2; ++k)
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kh[k]), qreg[HALF * (DS / 2) + k], c, 0, 0, 0);
    return c;
}
// half of O^T += V^T . P^T: the keys of one P operand
template <int DT> __device__ __forceinline__ void pv_half(const bf16x4 (&vh)[DT][2], const bf16x8 &pbm, f32x16 (&oacc)[DT])
{
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        const bf16x8 a = __builtin_shufflevector(vh[dt][0], vh[dt][1], 0, 1, 2, 3, 4, 5, 6, 7);
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pbm, oacc[dt], 0, 0, 0);
    }
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Wait until at most `tiles` (wave-uniform, clamped to [0, MAXT]) tiles of LPW fills each are in flight.
template <int LPW, int MAXT> __device__ __forceinline__ void wait_tiles(int tiles)
{
    static_assert(MAXT * LPW < 64, "vmcnt range");
    if constexpr (MAXT > 0) {
        if (tiles >= MAXT) { wait_vmcnt<MAXT * LPW>(); return; }
        wait_tiles<LPW, MAXT - 1>(tiles);
    } else {
        wait_vmcnt<0>();
    }
}

// LDS map of one workgroup: the ring of NT stages; the query tiles (one per row-wave: its 32 rows as they lie in
// memory, 2*D bytes each, chunk-rotated like a bf16 K tile) in the top of the ring when the prologue's fills leave
// that free, else behind them; 9 KiB for parent[] and the ancestor sets (see PAROFF).  Queries are consumed before the main
// loop's first barrier, after which the ring owns every stage, and so are the sets where they lie in one.  The merge of the
// key-waves re-uses the same memory after the loop.
template <int D, int RW, int KW, int NT, int EB>
struct WgLds {
    static constexpr int STAGE = Lds<D, EB>::STAGE;
    static constexpr int PREFILL = KW == 1 ? (NT - 1 < 3 ? NT - 1 : 3) : NT - KW;   // tiles issued before the main loop
    static constexpr int RING = NT * STAGE;
    static constexpr int QTILE = 32 * D * 2;
    static constexpr int QBYTES = RW * QTILE;
    static constexpr int PRE_B = PREFILL * STAGE;
    static constexpr int QOFF = RING - QBYTES > PRE_B ? RING - QBYTES : PRE_B;
    // parent[] and the ancestor sets.  Shapes with two key-waves read them before the main loop: in stages the prologue leaves free, or
    // behind the query tiles where those leave less than 9 KiB of them (64 channels in the 64-row bf16 shape).  The pipelined shape reads
    // the sets after the plain prefix tiles: behind the ring.
    static constexpr int PARENTS = BTV_MAX_NODES * 4, TREEB = PARENTS + BTV_MAX_NODES * BTV_ANC_WORDS * 4;
    static constexpr int PAROFF = KW == 1 ? (RING > QOFF + QBYTES ? RING : QOFF + QBYTES) : (QOFF - PRE_B >= TREEB ? PRE_B : QOFF + QBYTES);
    static constexpr int USED = (PAROFF + TREEB > QOFF + QBYTES ? PAROFF + TREEB : QOFF + QBYTES) > RING
                                    ? (PAROFF + TREEB > QOFF + QBYTES ? PAROFF + TREEB : QOFF + QBYTES) : RING;
    static_assert(KW == 1 || KW == 2, "the merge is between two key-waves");
    static constexpr int MERGE = KW == 2 ? RW * 2 * ((D / 64) * 16 + 3) * 64 * 4 : 0;    // they exchange half a row each (+ m, l, bound)
    static constexpr int BYTES = USED > MERGE ? USED : MERGE;
    static_assert(QOFF % 1024 == 0 && PAROFF % 1024 == 0 && BYTES <= 160 * 1024, "LDS budget");
};

// Wait until at most n (wave-uniform, clamped to [0, MAXN]) vector-memory operations are in flight.
template <int MAXN> __device__ __forceinline__ void wait_vm_ops(int n)
{
    if constexpr (MAXN > 0) {
        if (n >= MAXN) { wait_vmcnt<MAXN>(); return; }
        wait_vm_ops<MAXN - 1>(n);
    } else {
        wait_vmcnt<0>();
    }
}

// A lane's query row: row r of a KV head's packed rows is node r / G, query head r % G of the group.  Worked out where
// it is needed (mask construction, final store) rather than held in registers through the main loop.  Padding rows
// (r >= rows_g) recompute row 0 and are never written.
struct LaneRow { bool valid; int node; long long orow; };
__device__ __forceinline__ LaneRow lane_row(const AttnParams &p, int r, int rows_g, int g, int q0)
{
    LaneRow x;
    x.valid = r < rows_g;
    const int rr = x.valid ? r : 0;
    x.node = (rr * p.ginv) >> 16;
    x.orow = (long long)(q0 + x.node) * p.Hq + g * p.G + (rr - x.node * p.G);       // row of Q/O as [total_M*Hq, D]
    return x;
}

// Ancestor sets of the request's nodes, set[i] = {i} u set[parent[i]], by the threads of the workgroup, one per node: a thread
// takes over what its node's ancestor has found so far and goes on from where that one has got to, so that what it knows doubles from
// turn to turn: log2 of the depth turns of some 200 cycles, where a walk along parent[] takes as many as the tree is deep (270 each; 2.8 us for a
// random tree of 33 nodes in a workgroup that all others of its group wait for, 7 for one of 60 levels).  The wavefronts do not wait for
// each other: a thread writes its set before the place to go on from, and reads the place before the set (the LDS operations of a wavefront are in
// order), so what it takes is never less than the ancestors down to that place, whoever is ahead.  Every turn moves down: places strictly decrease.
// par: parent[] as staged (entries are checked here), then the places; sets: BTV_ANC_WORDS words per node, the upper half only where
// there are more than 128 nodes.  The sets may be read behind the next barrier.
__device__ __forceinline__ void find_ancestors(const AttnParams &p, uint32_t par, uint32_t sets, int M, int tid)
{
    static_assert(BTV_ANC_WORDS == 8 && BTV_MAX_NODES <= 256, "two 16-byte pieces per set, a thread per node");
    const bool mine = tid < M, big = M > 128;                    // (big: uniform)
    const uint32_t pa = par + 4u * (uint32_t)tid, sa = sets + 32u * (uint32_t)tid;
    int at = -1;
    u32x4 lo, hi;
#pragma unroll
    for (int k = 0; k < 4; ++k) { lo[k] = tid >> 5 == k ? 1u << (tid & 31) : 0u; hi[k] = tid >> 5 == k + 4 ? 1u << (tid & 31) : 0u; }
    if (mine) {
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(at) : "v"(pa) : "memory");
        if (at < -1 || at >= tid) { atomicOr(p.flag, 1u); at = -1; }
    }
    auto put = [&]() {                                           // the set, then the place
        if (big) asm volatile("ds_write_b128 %0, %1 offset:16" ::"v"(sa), "v"(hi) : "memory");
        asm volatile("ds_write_b128 %0, %1\n\tds_write_b32 %2, %3" ::"v"(sa), "v"(lo), "v"(pa), "v"(at) : "memory");
    };
    if (mine) put();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                                // all entries are checked, all sets hold their node
    while (at >= 0) {                                            // (a wavefront: while any of its lanes goes on)
        const uint32_t pb = par + 4u * (uint32_t)at, sb = sets + 32u * (uint32_t)at;
        int next;
        u32x4 l2, h2 = { 0u, 0u, 0u, 0u };
        if (big) asm volatile("ds_read_b32 %0, %3\n\tds_read_b128 %1, %4\n\tds_read_b128 %2, %4 offset:16\n\ts_waitcnt lgkmcnt(0)"
                              : "=&v"(next), "=&v"(l2), "=&v"(h2) : "v"(pb), "v"(sb) : "memory");
        else asm volatile("ds_read_b32 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(next), "=&v"(l2) : "v"(pb), "v"(sb) : "memory");
        lo |= l2; hi |= h2;
        at = next;
        put();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// The same for up to 64 nodes, by each wavefront for itself: lane i has node i, sets and places stay in registers and move between the lanes
// (log2 of the depth turns of some 100 cycles, no barrier).  lo, hi: the set of `node`.
__device__ __forceinline__ void wave_ancestors(const AttnParams &p, uint32_t par, int M, int l, int node, uint32_t &lo, uint32_t &hi)
{
    int at;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(at) : "v"(par + 4u * (uint32_t)l) : "memory");
    if (l < M && (at < -1 || at >= l)) atomicOr(p.flag, 1u);
    if (l >= M || at >= l) at = -1;
    uint32_t a = l < 32 ? 1u << l : 0u, b = l < 32 ? 0u : 1u << (l & 31);
    while (__builtin_amdgcn_ballot_w64(at >= 0) != 0ull) {
        uint32_t a2, b2;
        int next;
        asm volatile("ds_bpermute_b32 %0, %3, %4\n\tds_bpermute_b32 %1, %3, %5\n\tds_bpermute_b32 %2, %3, %6\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(a2), "=&v"(b2), "=&v"(next) : "v"(at < 0 ? 4 * l : 4 * at), "v"(a), "v"(b), "v"(at));
        a |= a2; b |= b2;                                        // (a lane that is done takes its own)
        at = next;
    }
    asm volatile("ds_bpermute_b32 %0, %2, %3\n\tds_bpermute_b32 %1, %2, %4\n\ts_waitcnt lgkmcnt(0)" : "=&v"(lo), "=&v"(hi) : "v"(4 * node), "v"(a), "v"(b));
}

// Largest finite magnitude of a lane's values: what its row's partials are divided by.  (An infinite one, from a value in the
// cache or a sum past the end of fp32, would leave nothing of the row's other channels.)
template <int B> __device__ __forceinline__ float finite_max(f32x16 (&x)[B])
{
    float a = 0.f;
    // x may be the result of matrix instructions that are still under way, and the compiler puts no wait states ahead of inline assembly
    // (ahead of a vector instruction of its own 12 for a 32x32x16).  The maxima follow these by way of a, the x by being passed through.
#pragma unroll
    for (int b = 1; b < B; ++b) asm volatile("" : "+v"(x[b]));
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(x[0]), "+v"(a));
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int v = 0; v < 16; v += 2)              // (fmaxf of fabsf's takes three instructions a value: each is made canonical first)
            asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(a) : "v"(x[b][v]), "v"(x[b][v + 1]));
    if (__builtin_amdgcn_ballot_w64(a > FLT_MAX) != 0ull) {        // (rare)
        a = 0.f;
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) a = fabsf(x[b][v]) <= FLT_MAX ? fmaxf(a, fabsf(x[b][v])) : a;
    }
    return fmaxf(a, __shfl_xor(a, 32));             // the other half of the wave holds the row's other channels
}

// What one workgroup does in one go: rows of row block `by` of (request, KV head g) against the tiles st0 .. st1 - 1.
struct Piece {
    int rq, g, by, st0, st1;
    int bx;                       // which partial of its rows this is
    int direct;                   // the only one: O is written
    int grouped;                  // its partial is `pitch` rows on end in the place of the group (merge_group)
    int group, pitch;
};

// A page window (32 tiles' page ids) per 256 bytes, four of them in turn, behind everything else; not where two workgroups
// fill the LDS of a CU to the last byte.
template <int D, int RW, int KW, int NT, bool PAGED, int EB>
struct PageLds {
    static constexpr int BASE = WgLds<D, RW, KW, NT, EB>::BYTES;
    static constexpr int PER_CU = RW * KW <= 4 ? 2 : 1;          // workgroups that are to share a CU
    static constexpr bool USED = PAGED && (BASE + 1024) * PER_CU <= 160 * 1024;
    static constexpr int BYTES = BASE + (USED ? 1024 : 0);
};

// Workgroup = RW row-waves x KW key-waves; wave (rw, kw) owns query rows [32 rw, 32 rw + 32) of the block and,
// in every round of KW consecutive tiles, tile number kw.  LDS ring of NT tiles; one barrier per round.
// begun(): called once the first loads are on their way (by all threads).
template <int D, int RW, int KW, int NT, bool PAGED, int EB, typename Begun>
__device__ __forceinline__ void attn_piece(const AttnParams &p, unsigned char *smem, int tid, const Req &rq_, const Piece &pc_, Begun begun)
{
    static_assert(EB == 2 || (EB == 1 && KW >= 2), "FP8 K/V runs in the shapes whose waves alternate over the tiles");
    constexpr int WAVES = RW * KW;
    constexpr int WR = RW * 32;
    constexpr int DS = D / 16;
    constexpr int DT = D / 32;
    constexpr int LPW = Lds<D, EB>::INSTR / WAVES;       // fill instructions per wave and tile
    constexpr int AHEAD = NT - 2 * KW;            // tiles still in flight when a round's tiles have landed
    static_assert(AHEAD >= 0 && AHEAD * LPW < 64, "ring too small or too deep for the counter");
    using LD = Lds<D, EB>;
    using PL = PageLds<D, RW, KW, NT, PAGED, EB>;
    constexpr bool PGV = PL::USED;
    const int w = tid >> 6, l = tid & 63, c = l & 31, h = l >> 5;
    const int kw = w % KW, rw = w / KW;
    const int rq = pc_.rq, g = pc_.g, by = pc_.by, bx = pc_.bx;
    const int Mr = rq_.M, Lr = rq_.L, S = Lr + Mr;
    const int rows_g = Mr * p.G;
    const int st0 = pc_.st0;
    int st1 = pc_.st1;
    {   // tree rows past the last node of this row block are invisible to all of its rows: their tiles are dropped
        const int node_hi = ((min((by + 1) * WR, rows_g) - 1) * p.ginv) >> 16;
        st1 = min(st1, max((Lr + node_hi + 1 + 31) / 32, st0 + 1));
    }

    using WL = WgLds<D, RW, KW, NT, EB>;

    // ---- prologue loads, oldest first: the first two page windows, parent[] (one entry per thread), this wave's share of
    // its row-wave's query tile, the first ring tiles.  All are raw instructions counted by hand.
    const int32_t *bt_row = PAGED ? p.block_table + (long long)rq * p.max_blocks : nullptr;
    auto load_window = [&](int g_) {                     // page ids of tiles st0 + 32 g_ .. + 31 (by the first wave)
        const int32_t *src = bt_row + min(2 * (st0 + 32 * g_) + l, (S - 1) >> 4);
        __builtin_amdgcn_global_load_lds(src, BTV_LDS_PTR(smem + PL::BASE + (g_ & 3) * 256), 4, 0, 0);
    };
    if (PGV && __builtin_amdgcn_readfirstlane(w) == 0) { load_window(0); load_window(1); }
    // parent[]: every wave moves 64 entries straight into LDS (index clamped to the request's nodes), whether or not
    // the workgroup reaches the tree rows; entries are checked where they are read.
#pragma unroll
    for (int i0 = 0; i0 < BTV_MAX_NODES; i0 += WAVES * 64)
        if (tid + i0 < BTV_MAX_NODES) {              // wave-uniform: whole waves
            const int32_t *pp = p.parent + rq_.q0 + min(tid + i0, Mr - 1);
            const int dst = __builtin_amdgcn_readfirstlane(WL::PAROFF + ((tid + i0) >> 6) * 256);
            __builtin_amdgcn_global_load_lds(pp, BTV_LDS_PTR(smem + dst), 4, 0, 0);
        }
    // Query tile: direct-to-LDS like a K tile (each wave instruction moves 1 KiB: whole rows, coalesced); as
    // per-lane operand loads the same bytes cost 64 separate 16-byte pieces per instruction and held the ring fills
    // back by about two microseconds.  The KW waves of a row-wave share the tile's instructions.
    constexpr int QCH = D / 8, QRPI = 1024 / (2 * D), QINSTR = WL::QTILE / 1024, QPW = QINSTR / KW;
    static_assert(QPW * KW == QINSTR, "query tile instructions must divide over the key-waves");
#pragma unroll
    for (int jj = 0; jj < QPW; ++jj) {
        const int j = kw * QPW + jj;
        const int qrow = j * QRPI + l / QCH, pc = l % QCH;
        const int rf = by * WR + rw * 32 + qrow;
        const long long of = lane_row(p, rf, rows_g, g, rq_.q0).orow;
        const unsigned char *src = static_cast<const unsigned char *>(p.Q) + of * (D * 2) + ((pc ^ swz_k<D, 2>(qrow)) << 4);
        // the destination must be wave-uniform: rw and kw are, but the compiler cannot know
        const int dst = __builtin_amdgcn_readfirstlane(WL::QOFF + rw * WL::QTILE + j * 1024);
        __builtin_amdgcn_global_load_lds(src, BTV_LDS_PTR(smem + dst), 16, 0, 0);
    }

    // ---- start filling the ring ------------------------------------------------------------------------
    const int wu = __builtin_amdgcn_readfirstlane(w);
    Fill<D, WAVES, PAGED, EB> fill = make_fill<D, WAVES, PAGED, EB>(p.K, p.V, bt_row, p.num_blocks, p.Hkv, g, S, wu, l);
    // KW == 1: three tiles up front (the first compute needs two), the rest of the ring fills during the first
    // rounds; an issue holds its wave for about a hundred cycles, so a full prefill would only delay the start.
    constexpr int PREFILL = WL::PREFILL;
    int issued = st0, islot = 0;
#pragma unroll
    for (int k = 0; k < PREFILL; ++k)
        if (issued < st1) {
            issue_tile<D, WAVES, PAGED, EB>(fill, smem, islot, issued, wu, l);
            ++issued; ++islot;
        }
    if (islot >= NT) islot -= NT;

    // ---- parent[] and the query tile have landed when only the ring fills are in flight ------------------------
    wait_vm_ops<PREFILL * LPW>((issued - st0) * LPW);
    // A bare barrier, and raw LDS reads below: with the fence of a full synchronisation, or with ordinary reads of
    // memory that direct-to-LDS loads wrote, the compiler drains the ring fills first.
    __builtin_amdgcn_s_barrier();                    // query tiles (filled by KW waves), parent[] and the page windows are visible
    // The window that tile `issued` belongs to, once per 32 tiles; the first wave asks for the one after it, which is there long
    // before it is read: the ring's waits cover every older load, and a barrier follows each of them.
    auto turn_window = [&]() {
        if constexpr (PGV) {
            const int g_ = (issued - st0) >> 5;
            int v;
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)"
                         : "=v"(v) : "v"((uint32_t)(uintptr_t)BTV_LDS_PTR(smem) + PL::BASE + (uint32_t)((g_ & 3) * 256 + (l & 31) * 8 + fill.half * 4)) : "memory");
            fill.pages = (uint32_t)fill.valid_page(v);
            if (g_ > 0 && wu == 0) load_window(g_ + 1);
        }
    };
    auto next_window = [&]() { if (PGV && ((issued - st0) & 31) == 0) turn_window(); };
    // Where tiles follow each other of which all keys exist, a fill is a scalar base, the lane's fixed offset and a stage's address: nothing is tested
    // and, with a page per wave and tile, one id is looked up.  With a test for every fill and both pages of a tile worked out for each, fills
    // were 90 of a trip's 250 instructions in the pipelined loop of a paged cache and several branches (8 requests of 1k to 16k, a layer 163 -> 146 us; FP8
    // 171 -> 149), and 60 of a round's 300 in the contiguous shapes with two key-waves (64 nodes, 2048 keys 11.0 -> 10.6 us; FP8, 5000 keys 14.7 -> 13.5).
    const uint32_t tile_bytes = 32 * fill.row_bytes;
    const unsigned char *ahead = nullptr;                // contiguous: tile `issued`, where whole tiles follow each other
    int ids[KW] = {};                                    // paged without a window: the pages of the next KW tiles, asked for a round ahead
    auto whole_src = [&]() {                             // where this wave's rows of tile `issued` lie, if all of its keys exist
        if constexpr (!PAGED) {
            const unsigned char *src = ahead;
            ahead += tile_bytes;
            asm volatile("" : "+s"(src));                // (a scalar base and the lane's offset; else a pointer per fill and lane is carried along)
            return src;
        } else if constexpr (PGV) {
            const unsigned char *src = fill.page(__builtin_amdgcn_readlane((int)fill.pages, (issued - st0) & 31));
            asm volatile("" : "+s"(src));
            return src;
        } else {
            const unsigned char *src = fill.page(fill.valid_page(ids[0]));
            if (KW > 1) ids[0] = ids[KW - 1];
            ids[KW - 1] = fill.page_id(issued + KW);
            return src;
        }
    };
    auto whole_tiles = [&]() {                           // ahead of the first of a row of them
        if constexpr (!PAGED) ahead = fill.base + (size_t)issued * tile_bytes;
        else if constexpr (!PGV)
#pragma unroll
            for (int k = 0; k < KW; ++k) ids[k] = fill.page_id(issued + k);
    };
    turn_window();
    begun();
    const bool tree_wg = st1 * 32 > Lr;              // this workgroup's keys reach the tree rows
    const uint32_t par_lds = (uint32_t)(uintptr_t)BTV_LDS_PTR(smem) + WL::PAROFF, sets_lds = par_lds + WL::PARENTS;
    static_assert(WAVES * 64 >= BTV_MAX_NODES, "find_ancestors: a thread per node");
    if (tree_wg && Mr > 64) find_ancestors(p, par_lds, sets_lds, Mr, tid);
    // Operand s holds the 8 channels that contraction step s takes from this lane's half: 16 s + 8 h .. + 7 for
    // bf16 K, 32 (s/2) + 16 h + 8 (s%2) .. + 7 for FP8 K (the order of its 16-byte operand reads).
    u32x4 qv[DS];
    {
        const uint32_t qa = (uint32_t)(uintptr_t)BTV_LDS_PTR(smem) + WL::QOFF + rw * WL::QTILE + c * (2 * D);
        const int sw = swz_k<D, 2>(c);
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            const int chunk = EB == 2 ? 2 * s + h : 4 * (s / 2) + 2 * h + (s % 2);
            const uint32_t addr = qa + (uint32_t)((chunk ^ sw) << 4);
            asm volatile("ds_read_b128 %0, %1" : "=v"(qv[s]) : "v"(addr));
        }
    }

    // ---- ancestor bitmask of this lane's node, only in workgroups whose keys reach the tree rows ----------
    // Shapes whose waves alternate over the tiles keep the sets inside the ring and read theirs before the main loop; the pipelined
    // shape keeps them behind the ring and reads them after the plain prefix tiles, so that they are not live through that loop.
    uint32_t anc_i[BTV_ANC_WORDS];
#pragma unroll
    for (int k = 0; k < BTV_ANC_WORDS; ++k) anc_i[k] = 0u;
    auto read_mask = [&]() {
        if (!tree_wg) return;
        const int node = lane_row(p, by * WR + rw * 32 + c, rows_g, g, rq_.q0).node;
        if (Mr <= 64) {
            wave_ancestors(p, par_lds, Mr, l, node, anc_i[0], anc_i[1]);
            return;
        }
        const uint32_t a = sets_lds + (uint32_t)node * (BTV_ANC_WORDS * 4);
        u32x4 lo, hi = { 0u, 0u, 0u, 0u };
        if (Mr > 128) asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" : "=&v"(lo), "=&v"(hi) : "v"(a) : "memory");
        else asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(lo) : "v"(a) : "memory");
#pragma unroll
        for (int k = 0; k < 4; ++k) { anc_i[k] = lo[k]; anc_i[k + 4] = hi[k]; }
    };
    if constexpr (KW > 1) {
        if (tree_wg && Mr > 64) __builtin_amdgcn_s_barrier();    // every wave's sets are there
        read_mask();
    }

    float m_run = NEG_BIG, l_run = 0.f;
    float base = 0.f;                 // what the step-by-step tiles' scores are relative to (rebase_tile)
    f32x16 negb;
#pragma unroll
    for (int v = 0; v < 16; ++v) negb[v] = 0.f;
    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;

    bf16x8 qreg[DS];
    if constexpr (DS == 8)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(qv[0]), "+v"(qv[1]), "+v"(qv[2]), "+v"(qv[3]), "+v"(qv[4]), "+v"(qv[5]), "+v"(qv[6]), "+v"(qv[7]));
    else
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(qv[0]), "+v"(qv[1]), "+v"(qv[2]), "+v"(qv[3]));
    const uint32_t ring = (uint32_t)(uintptr_t)BTV_LDS_PTR(smem);
    auto issue_one = [&]() {                             // the next tile of this split, if there is one
        if (issued < st1) {
            next_window();
            issue_tile<D, WAVES, PAGED, EB, 0, LPW, PGV>(fill, smem, islot, issued, wu, l, (issued - st0) & 31);
            ++issued;
            if (++islot == NT) islot = 0;
        }
    };
    // one half of the wave's fills of the next tile (LPW = 2 in the pipelined shape); the caller advances the counters
    auto issue_part = [&](auto part) {
        constexpr int P = decltype(part)::value;
        constexpr int MID = (LPW + 1) / 2, JB = P == 0 ? 0 : MID, JE = P == 0 ? MID : LPW;
        if constexpr (JB < JE)
            issue_tile<D, WAVES, PAGED, EB, JB, JE, PGV>(fill, smem, islot, issued, wu, l, (issued - st0) & 31);
    };
    // the same of a tile whose 32 keys all exist; src: its first row, or that of the wave's page of it
    auto issue_whole = [&](auto part, auto parts, int slot, const unsigned char *src) {
        constexpr int P = decltype(part)::value, N = decltype(parts)::value;
#pragma unroll
        for (int jj = 0; jj < LPW; ++jj)
            if (N == 1 || (P == 0) == (jj < (LPW + 1) / 2))
                fill_lds(src + fill.lane_off[jj], smem + slot * LD::STAGE + (wu * LPW + jj) * 1024);
    };
    if constexpr (KW == 1) {
        // Every wave has its queries in registers (parent[] and the sets lie behind the ring): the ring owns all stages from here on.
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int k = PREFILL; k < NT - 1; ++k) issue_one();
    }
    // At the top of the round starting at tile st (KW > 1), tiles st+KW .. issued-1 may still be in flight.  The
    // barrier also tells that every wave is done with the previous round, whose KW ring slots the next
    // issues overwrite (in front of the first round: with the queries' tiles and the ancestor sets).
    auto begin_round = [&](int st) {
        if (issued - st - KW == AHEAD) wait_vmcnt<AHEAD * LPW>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int k = 0; k < KW; ++k) issue_one();
    };
    // The first round, of which the queries' scaling (160 instructions) hides the wait or the loads: with four waves the next fills are four to a wave and
    // go out after it (32 nodes over 8192 keys 15.8 -> 15.6 us, 1500 keys 8.9 -> 8.7; FP8, 33 over 12003 18.3 -> 18.0), with eight two and ahead of it
    // (64 and 100 nodes 0.5 % slower the other way).
    constexpr bool SCALED_FIRST = KW > 1 && RW == 2;
    if constexpr (KW > 1 && !SCALED_FIRST) begin_round(st0);
    // The queries take the softmax scale and the change of base once (rounded to bf16 again, to nearest even: a
    // relative 2^-9 per element, as if the caller's projection had produced the scaled queries): scores then
    // are in log2 units and a probability costs no multiply.
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const float qs = p.scale_log2;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            u32x4 r;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t wd = qv[s][j];
                const bf16x2 pr = { (__bf16)(__uint_as_float(wd << 16) * qs), (__bf16)(__uint_as_float(wd & 0xFFFF0000u) * qs) };
                r[j] = __builtin_bit_cast(uint32_t, pr);
            }
            qreg[s] = __builtin_bit_cast(bf16x8, r);
            if constexpr (SCALED_FIRST) asm volatile("" : "+v"(qreg[s]));
        }
    }
    if constexpr (SCALED_FIRST) begin_round(st0);
    if constexpr (KW == 1 && EB == 2) {
        // ---- main loop, one tile per round, software-pipelined over the plain prefix tiles ------------------------
        // Local tile j = tile st0 + j lives in ring slot j % NT.  Tiles whose 32 keys all are prefix rows ("plain":
        // no mask) run through a pipeline in which iteration i issues
        //     the PV MFMAs of tile i-1 among the exponentials of tile i,  then the score MFMAs of tile i+1.
        // Scores come out of the matrix cores relative to the running reference (the accumulator starts at minus
        // the reference), so P = exp2(x) with no other arithmetic per element.  The reference is the maximum of
        // the split's first tile and moves only when a tile's row sum shows that some x exceeded 16 (checked on
        // the sum: no maximum per tile); then the tile is redone against its own maximum and everything rescaled.
        // K and V^T operands live in two half-tile buffers, each refilled right after the MFMAs that read it.
        static_assert(NT == 8, "the pipelined loop is written for a ring of 8 stages");
        constexpr int KH = DS / 2;                               // LDS reads per K half (a V^T half takes 2 * DT)
        int Tf = min(st1, Lr / 32) - st0;                        // plain tiles at the start of this split
        if (Tf < 3) Tf = 0;
        int j0 = 0;                                              // first local tile the step-by-step loop below takes
        // A wave whose 32 rows all lie past the request's last row has nothing to compute: it takes its share of the fills and
        // its part in every barrier, and leaves its SIMD to the other wave there.
        if (by * WR + __builtin_amdgcn_readfirstlane(rw) * 32 >= rows_g) {
            if (Tf > 0) {
                wait_tiles<LPW, NT - 4>(issued - st0 - 3);
                __builtin_amdgcn_s_barrier();
                for (int i = 1; i <= Tf - 2; ++i) {
                    wait_tiles<LPW, 3>(issued - st0 - i - 3);
                    __builtin_amdgcn_s_barrier();
                    issue_one();
                }
            }
            for (int j = Tf; j < st1 - st0; ++j) {
                wait_tiles<LPW, NT - 1>(issued - st0 - j - 1);
                __builtin_amdgcn_s_barrier();
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (issued - st0 - j < NT) issue_one();
            }
            wait_vmcnt<0>();
            return;
        }
        if (Tf > 0) {
            const uint32_t kbase = ring + lane_k_off<D>(l), vbase = ring + LD::TILEB + lane_v_off<D>(l);
            auto slot_off = [](int j) { return (uint32_t)((j & (NT - 1)) * LD::STAGE); };      // wave-uniform
            u32x4 kh[KH];
            bf16x4 vh[DT][2];
            f32x16 x;
            bf16x8 pa[2], pc[2];
            float negm;                                          // minus the reference: what the score accumulator starts from
            f32x16 negm16;                                       // ... kept splatted: the first score MFMA of a tile takes it as its
                                                                 // addend and writes x, so no tile pays sixteen moves for it
            // the tile's probabilities against a new reference: its own maximum joins the old one; sums, accumulator follow
            auto regrow = [&](bf16x8 (&pn)[2], float &ts) {
                const float dlt = fmaxf(tile_max(x), 0.f), alpha = __builtin_amdgcn_exp2f(-dlt);
                negm -= dlt;
#pragma unroll
                for (int v = 0; v < 16; ++v) negm16[v] = negm;
                l_run *= alpha;
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] -= dlt;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
                ts = 0.f;
                exp_half(x, 0, pn[0], ts);
                exp_half(x, 1, pn[1], ts);
            };
            // tiles 0 .. 2 have landed when at most the later ones are in flight
            wait_tiles<LPW, NT - 4>(issued - st0 - 3);
            __builtin_amdgcn_s_barrier();
            // ---- prologue: scores of tile 0 set the reference; its probabilities; scores of tile 1 ----
            {
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] = 0.f;
                read_k_half_at<D, 0>(kbase, kh); wait_k_half<KH, 0>(kh); x = qk_half<DS, 0>(kh, qreg, x);
                read_k_half_at<D, 1>(kbase, kh); wait_k_half<KH, 0>(kh); x = qk_half<DS, 1>(kh, qreg, x);
                read_k_half_at<D, 0>(kbase + slot_off(1), kh);
                negm = -tile_max(x);
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] += negm;
                exp_half(x, 0, pa[0], l_run);                    // x <= 0 here: no growth check
                exp_half(x, 1, pa[1], l_run);
#pragma unroll
                for (int v = 0; v < 16; ++v) negm16[v] = negm;
                wait_k_half<KH, 0>(kh); x = qk_half<DS, 0>(kh, qreg, negm16);
                read_k_half_at<D, 1>(kbase + slot_off(1), kh); wait_k_half<KH, 0>(kh); x = qk_half<DS, 1>(kh, qreg, x);
                read_v_half_at<D, 0>(vbase, vh);                 // queue: V(0) first half, K(2) low half
                read_k_half_at<D, 0>(kbase + slot_off(2), kh);
            }
            // ---- iteration i (1 <= i <= Tf - 2): x holds the scores of tile i, pprev the probabilities of tile i-1, pcur
            // receives those of tile i ----
            // On entry the LDS queue holds [V(i-1) first half, K(i+1) low half].
            // Loop-invariant operand addresses for the trips whose ring slots are known at compile time (eight trips
            // unrolled, one per slot): the slot is an immediate offset then, which reaches four slots from one base,
            // and a trip needs no address arithmetic at all (20 instructions of it otherwise).
            uint32_t ak[DS], akh[DS], av[DT], avh[DT];
#pragma unroll
            for (int s2 = 0; s2 < DS; ++s2) { ak[s2] = kbase ^ (uint32_t)(s2 << 5); akh[s2] = ak[s2] + 4u * LD::STAGE; }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) { av[dt] = vbase ^ (uint32_t)(dt << 6); avh[dt] = av[dt] + 4u * LD::STAGE; }
            auto rk = [&](auto slot, auto half) {
                constexpr int S = decltype(slot)::value & 7, H = decltype(half)::value;
                if constexpr (S < 4) read_k_half<D, S, H>(ak, kh); else read_k_half<D, S - 4, H>(akh, kh);
            };
            auto rv = [&](auto slot, auto mm) {
                constexpr int S = decltype(slot)::value & 7, MM = decltype(mm)::value;
                if constexpr (S < 4) read_v_half<D, S, MM>(av, vh); else read_v_half<D, S - 4, MM>(avh, vh);
            };
            // ph: the trip's tile number modulo 8 as a constant, or -1 for a trip with its addresses in registers
            // steady: the tile that this trip asks for exists, and so do all of its keys
            auto iter = [&](bf16x8 (&pprev)[2], bf16x8 (&pcur)[2], int i, auto ph, auto steady) {
                constexpr int PH = decltype(ph)::value;
                constexpr bool STEADY = decltype(steady)::value;
                using C0 = std::integral_constant<int, 0>;
                using C1 = std::integral_constant<int, 1>;
                // tiles <= i+2 are read in this iteration; the barrier also tells that every wave is done with
                // iteration i-1, i.e. with tile i-2, whose slot the next fill takes
                const unsigned char *src = nullptr;
                bool fill_now = true;                            // tile i+6 goes into the slot tile i-2 left
                if constexpr (STEADY) {
                    wait_vmcnt<3 * LPW>();
                    __builtin_amdgcn_s_barrier();
                    if constexpr (((PH + 6) & 7) == 0) next_window();
                    src = whole_src();
                } else {
                    wait_tiles<LPW, 3>(issued - st0 - i - 3);
                    __builtin_amdgcn_s_barrier();
                    fill_now = issued < st1;
                    if (fill_now) next_window();
                }
                auto fill_half = [&](auto part) {
                    if constexpr (STEADY) issue_whole(part, std::integral_constant<int, 2>{}, (PH + 6) & 7, src);
                    else if (fill_now) issue_part(part);
                };
                uint32_t k1 = 0, k2 = 0, v0 = 0, v1 = 0;
                if constexpr (PH < 0) {
                    k1 = kbase + slot_off(i + 1); k2 = kbase + slot_off(i + 2);
                    v0 = vbase + slot_off(i - 1); v1 = vbase + slot_off(i);
                }
                float ts = 0.f;
                wait_v_half<DT, KH>(vh);                          // V(i-1) first half
                pv_half<DT>(vh, pprev[0], oacc);
                fill_half(C0{});                                  // behind four MFMAs: its issue stall is covered
                if constexpr (PH < 0) read_v_half_at<D, 1>(v0, vh);                     // V(i-1) second half  queue: K(i+1)lo, V(i-1)b
                else rv(std::integral_constant<int, PH + 7>{}, C1{});
                __builtin_amdgcn_sched_barrier(0);
                exp_half(x, 0, pcur[0], ts);
                asm volatile("" : "+v"(pcur[0]), "+v"(ts));       // (the exponentials stay between the reads and their wait)
                __builtin_amdgcn_sched_barrier(0);
                wait_v_half<DT, 0>(vh);                           // V(i-1) second half (and K(i+1) low)
                pv_half<DT>(vh, pprev[1], oacc);
                fill_half(C1{});
                if constexpr (PH < 0) read_v_half_at<D, 0>(v1, vh);                     // V(i) first half     queue: V(i)a
                else rv(std::integral_constant<int, PH>{}, C0{});
                __builtin_amdgcn_sched_barrier(0);
                exp_half(x, 1, pcur[1], ts);
                asm volatile("" : "+v"(pcur[1]), "+v"(ts));
                __builtin_amdgcn_sched_barrier(0);
                if (__builtin_amdgcn_ballot_w64(!(ts <= GROW)) != 0ull) regrow(pcur, ts);     // rare
                l_run += ts;
                wait_k_half<KH, 2 * DT>(kh);                      // K(i+1) low (landed above; binds the registers)
                x = qk_half<DS, 0>(kh, qreg, negm16);
                if constexpr (PH < 0) read_k_half_at<D, 1>(k1, kh);                     // K(i+1) high         queue: V(i)a, K(i+1)hi
                else rk(std::integral_constant<int, PH + 1>{}, C1{});
                wait_k_half<KH, 0>(kh);                           // K(i+1) high (and V(i) first half)
                x = qk_half<DS, 1>(kh, qreg, x);
                if constexpr (PH < 0) read_k_half_at<D, 0>(k2, kh);                     // K(i+2) low          queue: K(i+2)lo (V(i)a has landed)
                else rk(std::integral_constant<int, PH + 2>{}, C0{});
                if constexpr (STEADY) ++issued;
                else if (fill_now) { ++issued; if (++islot == NT) islot = 0; }
            };
            // ---- epilogue: tile e = Tf - 1 has its scores, tile e-1 its probabilities (pp); nothing left to overlap ----
            auto drain = [&](bf16x8 (&pp)[2], bf16x8 (&pn)[2]) {
                const int e = Tf - 1;
                const uint32_t ve1 = vbase + slot_off(e - 1), ve = vbase + slot_off(e);
                wait_k_half<KH, 0>(kh);                          // (the low half of tile e+1's K: not used)
                wait_v_half<DT, 0>(vh);                          // V(e-1) first half
                pv_half<DT>(vh, pp[0], oacc);
                read_v_half_at<D, 1>(ve1, vh);
                float ts = 0.f;
                exp_half(x, 0, pn[0], ts);
                exp_half(x, 1, pn[1], ts);
                wait_v_half<DT, 0>(vh);
                pv_half<DT>(vh, pp[1], oacc);
                read_v_half_at<D, 0>(ve, vh);
                if (__builtin_amdgcn_ballot_w64(!(ts <= GROW)) != 0ull) regrow(pn, ts);
                l_run += ts;
                wait_v_half<DT, 0>(vh);
                pv_half<DT>(vh, pn[0], oacc);
                read_v_half_at<D, 1>(ve, vh);
                wait_v_half<DT, 0>(vh);
                pv_half<DT>(vh, pn[1], oacc);
                m_run = -negm;
            };
            // One iteration per trip, the new probabilities copied into place at its end (8 moves): with the roles of
            // two register sets alternating over an unrolled pair the allocator shuffles tuples and spills.
            int i = 1;
            // (the two probability buffers swap roles from trip to trip: no copies inside a group of eight)
            // (one barrier for two trips, with the fills one tile less ahead, measured the same)
#define BTV_TRIP(k, slot, from, to) iter(from, to, i + k, std::integral_constant<int, slot>{}, steady);
#define BTV_TRIPS                                                                                                             \
            BTV_TRIP(0, 1, pa, pc) BTV_TRIP(1, 2, pc, pa) BTV_TRIP(2, 3, pa, pc) BTV_TRIP(3, 4, pc, pa)                       \
            BTV_TRIP(4, 5, pa, pc) BTV_TRIP(5, 6, pc, pa) BTV_TRIP(6, 7, pa, pc) BTV_TRIP(7, 0, pc, pa)
            const int whole = min(st1, S / 32) - st0;            // tiles of this split with all keys
            whole_tiles();
            for (; i + 7 <= Tf - 2 && i + 13 < whole; i += 8) {  // tile i is in ring slot 1 here: eight trips, one per slot
                constexpr std::true_type steady;
                BTV_TRIPS
            }
            for (; i + 7 <= Tf - 2; i += 8) {
                constexpr std::false_type steady;
                BTV_TRIPS
            }
#undef BTV_TRIPS
#undef BTV_TRIP
            for (; i <= Tf - 2; ++i) {
                iter(pa, pc, i, std::integral_constant<int, -1>{}, std::false_type{});
#pragma unroll
                for (int mm = 0; mm < 2; ++mm) pa[mm] = pc[mm];
            }
            drain(pa, pc);
            j0 = Tf;
        }
        // ---- the remaining tiles (those that touch tree rows, or all of a short split), step by step ----
        if (j0 > 0) {                                            // (m_run is a real maximum after the pipelined part)
            base = m_run;
#pragma unroll
            for (int v = 0; v < 16; ++v) negb[v] = -m_run;
        }
        read_mask();                                             // (barriers since the sets were written: those of the prologue)
        for (int j = j0; j < st1 - st0; ++j) {
            wait_tiles<LPW, NT - 1>(issued - st0 - j - 1);       // tile j has landed
            __builtin_amdgcn_s_barrier();                        // ... for every wave, and all are done with tile j-1
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (issued - st0 - j < NT) issue_one();
            do_tile<D, false>(ring + (j & 7) * LD::STAGE, (st0 + j) * 32, Lr, l, anc_i, qreg, m_run, l_run, oacc, base, negb, true);
        }
        if constexpr (PAGED) wait_vmcnt<0>();
    } else {
        // ---- main loop: one barrier per round of KW tiles, wave kw takes tile number kw of the round ------
        // (a wave whose 32 rows all lie past the last one only fills)
        const bool live = by * WR + __builtin_amdgcn_readfirstlane(rw) * 32 < rows_g;
        const int kwu = wu % KW;                                 // (kw, as a scalar)
        int cslot = kwu, st = st0;
        auto tile = [&](auto plain) {                            // this wave's tile of the round
            constexpr bool PLAIN = decltype(plain)::value;
            const bool exact = !PLAIN && (st == st0 || (st + kwu) * 32 + 32 > Lr);      // (constant in the first round)
            if constexpr (EB == 2)
                do_tile<D, PLAIN>(ring + cslot * LD::STAGE, (st + kwu) * 32, Lr, l, anc_i, qreg, m_run, l_run, oacc, base, negb, exact);
            else
                do_tile8<D, PLAIN>(ring + cslot * LD::STAGE, (st + kwu) * 32, Lr, l, anc_i, qreg, m_run, l_run, oacc, base, negb, exact);
        };
        auto next_round = [&]() {
            st += KW;
            cslot += KW;
            if (cslot >= NT) cslot -= NT;
        };
        // Rounds that ask for KW tiles of the prefix with all their keys, and so only take such, have nothing to test for.
        const int plain = min(st1, Lr / 32);
        if (live && st + kwu < st1) tile(std::false_type{});     // (on its own: nothing has to be cleared ahead of it)
        next_round();
        whole_tiles();
        for (; issued + KW <= plain; next_round()) {
            wait_vmcnt<AHEAD * LPW>();
            __builtin_amdgcn_s_barrier();
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                next_window();
                issue_whole(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, islot, whole_src());
                ++issued;
                if (++islot == NT) islot = 0;
            }
            if (live) tile(std::true_type{});
        }
        for (; st < st1; next_round()) {
            begin_round(st);
            if (live && st + kwu < st1) tile(std::false_type{});
        }
    }
    const LaneRow lrow = lane_row(p, by * WR + rw * 32 + c, rows_g, g, rq_.q0);
    const bool rvalid = lrow.valid;
    const long long orow = lrow.orow;
    // both halves of a wave hold partial row sums of the same queries
    l_run += __shfl_xor(l_run, 32);

    // ---- merge the key-waves of each row-wave through LDS ---------------------------------------------------
    // Two key-waves: each keeps one half of the channels and hands the other half to its partner, so both merge,
    // scale and store half a row.  dt0 .. dt0 + DTK - 1 are the channel blocks this wave ends up with.
    int dt0 = 0;
    constexpr int DTK = KW == 2 ? DT / 2 : DT;
    float fin[DTK][16];                             // what this wave stores: its rows times `factor`
    float amax;                                     // bound on the row's largest magnitude (for the fp16 partials)
    // Partials travel as fp16 relative to (a bound within a factor two of) the row's largest magnitude, kept in fp32 beside m and l:
    // half the bytes of fp32 to write, flush at the end of the kernel and read back, at a relative error of at most 2^-10 of that
    // magnitude, below the final bf16 rounding.  (The bound stays above LEAST, so that its reciprocal is finite.)
    constexpr float LEAST = 1.0e-36f;
    auto factor = [&]() { return pc_.direct ? p.out_scale / l_run : 1.0f / amax; };
    if constexpr (KW == 2) {
        constexpr int QUADS = DTK * 4, SLOT = (DTK * 16 + 3) * 64;      // floats a wave hands over: groups of four, then m, l, bound
        float *mg = reinterpret_cast<float *>(smem) + rw * 2 * SLOT;
        amax = finite_max<DT>(oacc);
        wait_vmcnt<0>();
        __syncthreads();                            // every wave is done with the ring
        float *out = mg + kw * SLOT;
        auto give = [&](auto first) {               // the channel blocks first .. first + DTK - 1 go to the partner
            constexpr int F = decltype(first)::value;
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                const f32x16 &o = oacc[F + q / 4];
                const f32x4 x = { o[4 * (q & 3)], o[4 * (q & 3) + 1], o[4 * (q & 3) + 2], o[4 * (q & 3) + 3] };
                reinterpret_cast<f32x4 *>(out)[q * 64 + l] = x;
            }
        };
        if (kw == 0) give(std::integral_constant<int, DTK>{}); else give(std::integral_constant<int, 0>{});
        out[(DTK * 16) * 64 + l] = m_run;
        out[(DTK * 16 + 1) * 64 + l] = l_run;
        out[(DTK * 16 + 2) * 64 + l] = amax;
        __syncthreads();
        const float *in = mg + (kw ^ 1) * SLOT;
        const float m1 = in[(DTK * 16) * 64 + l], l1 = in[(DTK * 16 + 1) * 64 + l], x1 = in[(DTK * 16 + 2) * 64 + l];
        f32x4 other[QUADS];
#pragma unroll
        for (int q = 0; q < QUADS; ++q) other[q] = reinterpret_cast<const f32x4 *>(in)[q * 64 + l];
        const float mn = fmaxf(m_run, m1);
        float a0 = __builtin_amdgcn_exp2f(m_run - mn);
        float a1 = __builtin_amdgcn_exp2f(m1 - mn);
        // both waves must arrive at the same l and bound: sums of the same two products, order fixed by kw
        const float la = kw == 0 ? l_run * a0 : l1 * a1, lb = kw == 0 ? l1 * a1 : l_run * a0;
        const float xa = kw == 0 ? amax * a0 : x1 * a1, xb = kw == 0 ? x1 * a1 : amax * a0;
        m_run = mn;
        l_run = la + lb;
        amax = fminf(fmaxf(xa + xb, LEAST), FLT_MAX);     // >= the merged row's largest (finite) magnitude, at most twice it
        const float f = factor();
        a0 *= f; a1 *= f;
        auto take = [&](auto first) {
            constexpr int F = decltype(first)::value;
#pragma unroll
            for (int dt = 0; dt < DTK; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) fin[dt][v] = fmaf(oacc[F + dt][v], a0, other[dt * 4 + v / 4][v & 3] * a1);
        };
        if (kw == 0) take(std::integral_constant<int, 0>{}); else take(std::integral_constant<int, DTK>{});
        dt0 = kw * DTK;                             // the kept blocks now sit in oacc[0 .. DTK)
    }
    if (!rvalid) return;
    if constexpr (KW == 1) {
        amax = fmaxf(finite_max<DT>(oacc), LEAST);
        const float f = factor();
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) fin[dt][v] = oacc[dt][v] * f;
    }

    // ---- write: final bf16 rows when this request has a single split, scaled fp16 partials otherwise ---
    // A lane holds channels 8 q + 4 h .. + 3 of its row, the other half of the wave the other four: they exchange every second
    // group, so that each has 8 neighbouring channels and a store instruction touches half as many pieces of rows (there
    // are 32 rows per instruction whatever its width; the stores of a 256-row workgroup took 3 us).
    auto store_rows = [&](unsigned char *row, auto pack) {
#pragma unroll
        for (int dt = 0; dt < DTK; ++dt)
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const uint2 a = pack(dt, q), b = pack(dt, q + 1);
                const auto x = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false), y = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
                *reinterpret_cast<uint4 *>(row + (dt * 32 + (q + h) * 8) * 2) = make_uint4(x[0], y[0], x[1], y[1]);
            }
    };
    if (pc_.direct) {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        auto pack = [&](int dt, int q) {
            const b2 lo = { (__bf16)fin[dt][q * 4 + 0], (__bf16)fin[dt][q * 4 + 1] }, hi = { (__bf16)fin[dt][q * 4 + 2], (__bf16)fin[dt][q * 4 + 3] };
            return make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
        };
        store_rows(static_cast<unsigned char *>(p.O) + (orow * D + dt0 * 32) * 2, pack);
    } else {
        const size_t prow = pc_.grouped ? (size_t)((pc_.group * p.nsplit + bx) * pc_.pitch + rw * 32 + c) : (size_t)bx * p.total_rows + orow;
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        auto pack = [&](int dt, int q) {
            const h2 lo = { (_Float16)fin[dt][q * 4 + 0], (_Float16)fin[dt][q * 4 + 1] }, hi = { (_Float16)fin[dt][q * 4 + 2], (_Float16)fin[dt][q * 4 + 3] };
            return make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
        };
        store_rows(reinterpret_cast<unsigned char *>(p.Opart) + (prow * D + dt0 * 32) * 2, pack);
        if (h == 0 && kw == 0) *reinterpret_cast<float4 *>(p.ML + prow * 4) = make_float4(m_run, l_run, amax, 0.f);
    }
}

// Fetch every argument now, in one round trip.  Left to the compiler the scalar loads follow the early-exit tests
// in five dependent steps, three of which miss the cache (the argument block spans three lines and is cold in every
// launch): about two microseconds before the first fill is issued.
#define BTV_FETCH_ARGS(p)                                                                                                     \
    asm volatile("" ::"s"(p.Q), "s"(p.K), "s"(p.V), "s"(p.O), "s"(p.parent), "s"(p.block_table), "s"(p.q_offset),              \
                 "s"(p.prefix_len), "s"(p.Opart), "s"(p.ML), "s"(p.flag), "s"(p.sync), "s"(p.M), "s"(p.L), "s"(p.Hq), "s"(p.Hkv), "s"(p.G), "s"(p.ginv), \
                 "s"(p.max_blocks), "s"(p.num_blocks), "s"(p.total_rows), "s"(p.total_M), "s"(p.sps), "s"(p.longer), "s"(p.nsplit), \
                 "s"(p.inv_row_blocks), "s"(p.inv_nsplit), "s"(p.row_blocks), "s"(p.units), "s"(p.scale_log2), "s"(p.out_scale))

// ---- the merge inside the attention kernel --------------------------------------------------------------------------------
// A group = the workgroups whose partials belong to the same rows: the key splits of one (KV head, row block).  Where the
// launch gives every group workgroup ids that are congruent mod 8 they run on one XCD, their partials meet in that XCD's L2, and each of
// them, once all have stored theirs, merges its share of the rows (every nsplit-th) and writes O.  That takes the place of a second
// launch: the write-back of the partials between the kernels, a launch and tv_combine_bf16's own round trips.
//
// Nothing depends on where workgroups run or on whether they run at once:
// * A workgroup writes the XCD it runs on (the hardware's register) beside the call's tag when it starts, and reads its peers' words
//   at its end.  Only if all have started, and on its own XCD, it relies on the L2 ("together"); otherwise its partials are
//   released to the whole device first, and the others' acquired.  A workgroup that is together knows that all its peers are
//   on this XCD, whatever they know themselves.
// * A workgroup says that its partials are stored in a word in the L2 (near; a store of workgroup scope, which stays there), and if it is
//   not together in a word at the memory side as well (far).  It waits until all have, for `wait_ticks` at most.  If that passes it says
//   so in the same words, looks once more, at near and far words alike, and leaves if somebody still is missing.  Whoever stores
//   last sees all words, and who has left among them (each writes its own word, and has it acknowledged, before it looks at the others'), and
//   merges their shares too.  Two that do the same share write the same values.
// * "Not started": where other streams' work holds compute units, a peer may wait for the very units that the waiting workgroups hold.  So after
//   5 us it counts whether all have started, and leaves if not.  A call of 64 nodes over 8192 keys, 21 us alone, beside a kernel that holds
//   64, 128 or 192 of the 256 units: 81, 73 and 151 us with 20 us for all, 65, 58 and 106 with 5 (and 62, 54 and 97 with 2); beside the same
//   calls on another stream, whose workgroups come one after the other: 34 us with 20 or 5, but 46 with 2, as the last one then merges alone
//   what a little more patience has merged by all.  (By a second launch: 32 beside the same calls; beside such a kernel its calls
//   did not run at all until that kernel had ended.)
// * Words carry the call's tag (one more than `epoch`, which every workgroup reads at its start and whoever has seen all of the group
//   moves on), so they are never cleared and a workspace may change its sizes from call to call.
// An exchange between 32 workgroups takes 930 cycles through the L2 and 2300 at the memory side (MI355X, store to all have read).
constexpr int MERGE_GROUPS = 128, MERGE_SPLITS = 32;
typedef unsigned long long u64;
struct MergeWords {                                     // of one group
    u64 started[MERGE_SPLITS];                          // tag << 8 | XCD
    u64 near[MERGE_SPLITS], far[MERGE_SPLITS];          // tag << 8 | 1 if it has left
    u64 epoch, pad[31];
};
static_assert(sizeof(MergeWords) == 1024, "whole cache lines per group");
constexpr int MERGE_WAIT_TICKS = 2000;                  // 20 us of the 100 MHz wall clock
constexpr int MERGE_START_TICKS = 500;                  // (see "not started" above)

__device__ __forceinline__ uint32_t this_xcd() { return (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11)); }     // HW_REG_XCC_ID, bits 3:0

// One of the group's shares: rows of, of + n, .. of the block's `rows`.  16 lanes take a row's partial of one split with one load each
// (a load holds its wave for some 80 cycles whatever its width), 4, 2 or 1 such sets of lanes of a wavefront share a row's splits out,
// by how many rows there are.  Loads go past the L1, to which the group's other workgroups do not write.  The arithmetic is combine_row's, the
// sums over the splits in another order.  What a wavefront spends its time on is one instruction after the other (two wavefronts
// on a SIMD, some 7 cycles each): offsets are worked out before the wait for the others, sums are multiply-adds on the fp16 values as they are.
template <int D, int WAVES> struct Share {
    static constexpr int E = D / 16, SETS = WAVES * 4;  // values per lane; sets of 16 lanes
    int of, count, lp;                                  // first row, number of rows, log2 of the sets per row
    int k, row, ml, part[8];                            // a set's row: which of the share's, of O; byte offsets of what it loads
    __device__ __forceinline__ void begin(int of_, int n, int rows, int tid)
    {
        of = of_;
        count = (rows - of + n - 1) / n;
        lp = 4 * count <= SETS ? 2 : 2 * count <= SETS ? 1 : 0;
        k = (tid >> 4) >> lp;
    }
    __device__ __forceinline__ void find(const AttnParams &p, const Piece &pc, int n, int wr, int tid)
    {
        const int r = of + n * k, rr = pc.by * wr + r, node = (rr * p.ginv) >> 16;
        row = node * p.Hq + pc.g * p.G + (rr - node * p.G);
        ml = (min(tid & ((16 << lp) - 1), n - 1) * pc.pitch + r) * 16;
#pragma unroll
        for (int b = 0; b < 8; ++b) part[b] = part_at(pc, b, 0, n, tid);
    }
    __device__ __forceinline__ int part_at(const Piece &pc, int b, int at, int n, int tid) const
    {
        const int s = at + ((tid >> 4) & ((1 << lp) - 1)) + (b << lp);
        return (min(s, n - 1) * pc.pitch + of + n * k) * (D * 2) + (tid & 15) * (E * 2);
    }
};

template <int D, int WAVES>
__device__ __forceinline__ void merge_share(const AttnParams &p, const Piece &pc, Share<D, WAVES> sh, int n, int wr, float *weights, int tid)
{
    constexpr int E = Share<D, WAVES>::E, PAST_L1 = 16;                 // SC1
    typedef _Float16 hvec __attribute__((ext_vector_type(E)));
    typedef __bf16 bvec __attribute__((ext_vector_type(E)));
    const int lp = sh.lp, set = tid >> 4, sub = set & ((1 << lp) - 1);
    float *wsh = weights + (set >> lp << lp) * MERGE_SPLITS;           // (by the row's first set: no other wavefront's, whatever lp is)
    const uint32_t pitch = (uint32_t)pc.pitch, first = (uint32_t)(pc.group * n) * pitch;
    const auto ml_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.ML + (size_t)first * 4, 0, (int)(n * pitch * 16), 0x00027000);
    const auto part_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.Opart + (size_t)first * D, 0, (int)(n * pitch * D * 2), 0x00027000);
    const int s0 = tid & ((16 << lp) - 1), s1 = s0 + 16;                // splits whose weights this lane works out (s1: one set per row)
    while (sh.k < sh.count) {
        auto load_ml = [&](int off) { return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(ml_rsrc, off, 0, PAST_L1)); };
        const float4 m0 = load_ml(sh.ml);
        float4 m1 = make_float4(NEG_BIG, 0.f, 0.f, 0.f);
        if (lp == 0 && n > 16) m1 = load_ml((min(s1, n - 1) * pc.pitch + sh.of + n * sh.k) * 16);
        hvec part[8];
        auto load_parts = [&]() {
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if constexpr (E == 8) part[b] = __builtin_bit_cast(hvec, __builtin_amdgcn_raw_buffer_load_b128(part_rsrc, sh.part[b], 0, PAST_L1));
                else part[b] = __builtin_bit_cast(hvec, __builtin_amdgcn_raw_buffer_load_b64(part_rsrc, sh.part[b], 0, PAST_L1));
            }
        };
        load_parts();
        auto over_row = [&](float x, auto op) {                         // over the row's 16, 32 or 64 lanes
            x = op(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xF, 0xF, false)));      // quad_perm [1,0,3,2]
            x = op(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xF, 0xF, false)));      // quad_perm [2,3,0,1]
            x = op(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xF, 0xF, false)));     // row_half_mirror
            x = op(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x140, 0xF, 0xF, false)));     // row_mirror
            if (lp >= 1) {
                const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                x = op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            if (lp == 2) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                x = op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            return x;
        };
        const float x0 = s0 < n ? m0.x : NEG_BIG, x1 = s1 < n ? m1.x : NEG_BIG;
        const float mmax = over_row(lp == 0 ? fmaxf(x0, x1) : x0, [](float u, float v) { return fmaxf(u, v); });
        const float w0 = s0 < n ? __builtin_amdgcn_exp2f(x0 - mmax) : 0.f, w1 = lp == 0 && s1 < n ? __builtin_amdgcn_exp2f(x1 - mmax) : 0.f;
        // weight times the partial's magnitude; 0 past the last split.  (The row's lanes are of one wavefront: no barrier needed.)
        if (s0 < MERGE_SPLITS) wsh[s0] = s0 < n ? w0 * m0.z : 0.f;
        if (lp == 0) wsh[s1] = s1 < n ? w1 * m1.z : 0.f;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const float den = over_row((s0 < n ? w0 * m0.y : 0.f) + (lp == 0 && s1 < n ? w1 * m1.y : 0.f), [](float u, float v) { return u + v; });
        float inv = p.out_scale / den;
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.f;
        for (int at = 0;;) {
            float wg[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) wg[b] = wsh[(at + sub + (b << lp)) & (MERGE_SPLITS - 1)];
#pragma unroll
            for (int b = 0; b < 8; ++b)
                if (at + (b << lp) < n) {                               // (a set past the last split: weight 0)
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[e] = fmaf(wg[b], (float)part[b][e], acc[e]);
                }
            at += 8 << lp;
            if (at >= n) break;
#pragma unroll
            for (int b = 0; b < 8; ++b) sh.part[b] = sh.part_at(pc, b, at, n, tid);
            load_parts();
        }
        bvec o;
#pragma unroll
        for (int e = 0; e < E; ++e) {                                   // the row's sets
            if (lp >= 1) {
                const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[e]), __float_as_uint(acc[e]), false, false);
                acc[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            }
            if (lp == 2) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[e]), __float_as_uint(acc[e]), false, false);
                acc[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            }
            o[e] = (__bf16)(acc[e] * inv);
        }
        if (sub == 0) *reinterpret_cast<bvec *>(static_cast<__bf16 *>(p.O) + (size_t)sh.row * D + (tid & 15) * E) = o;
        sh.k += sh.SETS >> lp;
        if (sh.k < sh.count) sh.find(p, pc, n, wr, tid);
    }
}

// The rest of a workgroup whose partials have been stored (by its threads; not necessarily acknowledged yet).
template <int D, int WAVES, int WR>
__device__ __forceinline__ void merge_group(const AttnParams &p, MergeWords &m, unsigned char *smem, int tid, const Piece &pc, int n, u64 tag)
{
    const int split = pc.bx;
    uint32_t *said = reinterpret_cast<uint32_t *>(smem) + WAVES * 4 * MERGE_SPLITS;      // what the first wavefront has seen (behind merge_share's weights)
    const int lane = tid & 63, peer = min(lane, n - 1), rows = min(WR, p.M * p.G - pc.by * WR);
    u64 begun = 0;
    if (tid < 64) begun = __hip_atomic_load(&m.started[peer], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Share<D, WAVES> own;                                // found ahead of the wait
    own.begin(split, n, rows, tid);
    own.find(p, pc, n, WR, tid);
    asm volatile("" : "+v"(own.k), "+v"(own.row), "+v"(own.ml), "+v"(own.part[0]), "+v"(own.part[1]), "+v"(own.part[2]), "+v"(own.part[3]),
                 "+v"(own.part[4]), "+v"(own.part[5]), "+v"(own.part[6]), "+v"(own.part[7]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wavefront's partials are in the L2 ...
    __syncthreads();                                    // ... and all the workgroup's
    if (tid < 64) {
        const bool together = __builtin_amdgcn_ballot_w64(begun != (tag << 8 | this_xcd())) == 0ull;
        if (!together) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        auto say = [&](u64 word) {
            if (lane == 0) __hip_atomic_store(&m.near[split], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (!together) {
                if (lane == 0) __hip_atomic_store(&m.far[split], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        };
        u64 left = 0;
        auto look = [&](bool both) {                    // are all there?  Which have left?
            const u64 a = __hip_atomic_load(&m.near[peer], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u64 b = both ? __hip_atomic_load(&m.far[peer], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : a;
            const bool in_a = a >> 8 == tag, in_b = b >> 8 == tag;
            left = __builtin_amdgcn_ballot_w64(lane < n && ((in_a && (a & 1)) || (in_b && (b & 1))));
            return __builtin_amdgcn_ballot_w64(!in_a && !in_b) == 0ull;
        };
        say(tag << 8);
        bool all = look(!together);
        if (!all) {
            const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
            int limit = min(p.wait_ticks, MERGE_START_TICKS);
            do {
                if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > limit) {
                    if (limit < p.wait_ticks) {         // have all started by now?
                        limit = p.wait_ticks;
                        const u64 now = __hip_atomic_load(&m.started[peer], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (__builtin_amdgcn_ballot_w64(now >> 8 != tag) == 0ull) continue;
                    }
                    say(tag << 8 | 1);
                    all = look(true);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                all = look(!together);
            } while (!all);
        }
        if (all && !together) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane == 0) *reinterpret_cast<uint2 *>(said) = make_uint2(all, (uint32_t)left);
    }
    __syncthreads();
    const uint2 seen = *reinterpret_cast<const uint2 *>(said);
    if (!__builtin_amdgcn_readfirstlane(seen.x)) return;
    merge_share<D, WAVES>(p, pc, own, n, WR, reinterpret_cast<float *>(smem), tid);
    uint32_t left = __builtin_amdgcn_readfirstlane(seen.y) & ~(1u << split);
    while (left) {                                      // (rare) the shares of those that have left
        own.begin(__builtin_ctz(left), n, rows, tid);
        own.find(p, pc, n, WR, tid);
        merge_share<D, WAVES>(p, pc, own, n, WR, reinterpret_cast<float *>(smem), tid);
        left &= left - 1;
    }
    if (tid == 0) __hip_atomic_store(&m.epoch, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One request: a workgroup per (key split, KV head, row block).  MERGE: the workgroups merge the splits (a kernel of its own: with
// both in one, those that do not merge took 0.2 us longer).
template <int D, int RW, int KW, int NT, int EB, bool MERGE>
__global__ __launch_bounds__(RW * KW * 64, 2) void tv_attn_bf16(AttnParams p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    BTV_FETCH_ARGS(p);
    // Workgroups go to the 8 XCDs round-robin by their linear id.  The row blocks of one (key split, KV head) stream the same K/V
    // bytes, so they get ids that are congruent mod 8 and share one L2; where the merge is done here, so do all splits of a group
    // (p.units counts the (split, head) pairs, or the heads, or the groups that are dealt out to the XCDs; 0: the pairs are dealt
    // out although the merge is done here, so that tests meet a group on several XCDs).
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    Piece pc = {};
    if constexpr (!MERGE) {
        const int q = quotient(slot, p.row_blocks, p.inv_row_blocks), unit = q * 8 + xcd;
        if (unit >= p.units) return;
        pc.by = slot - q * p.row_blocks; pc.g = quotient(unit, p.nsplit, p.inv_nsplit); pc.bx = unit - pc.g * p.nsplit;
    } else if (p.units == p.Hkv) {
        const int q = quotient(slot, p.row_blocks, p.inv_row_blocks), u = quotient(q, p.nsplit, p.inv_nsplit);
        pc.by = slot - q * p.row_blocks; pc.g = u * 8 + xcd; pc.bx = q - u * p.nsplit;
        if (pc.g >= p.Hkv) return;
    } else if (p.units) {
        const int u = quotient(slot, p.nsplit, p.inv_nsplit), q = u * 8 + xcd;
        pc.g = quotient(q, p.row_blocks, p.inv_row_blocks); pc.by = q - pc.g * p.row_blocks; pc.bx = slot - u * p.nsplit;
        if (pc.g >= p.Hkv) return;
    } else {
        const int q = quotient(slot, p.row_blocks, p.inv_row_blocks), unit = q * 8 + xcd;
        pc.by = slot - q * p.row_blocks; pc.g = quotient(unit, p.nsplit, p.inv_nsplit); pc.bx = unit - pc.g * p.nsplit;
        if (pc.g >= p.Hkv) return;
    }
    const Req rq = load_req<false>(p, 0);
    const int tiles = (rq.L + rq.M + 31) / 32;
    pc.st0 = pc.bx * p.sps + KW * min(pc.bx, p.longer);
    pc.st1 = min(pc.st0 + p.sps + (pc.bx < p.longer ? KW : 0), tiles);
    pc.direct = p.nsplit == 1;
    pc.grouped = MERGE;
    pc.group = pc.g * p.row_blocks + pc.by;
    pc.pitch = min(RW * 32, rq.M * p.G) + 1;            // (rows of the same number lie in different channels)
    if constexpr (MERGE) {
        MergeWords *m = reinterpret_cast<MergeWords *>(p.sync) + pc.group;
        // (a scalar load: nothing writes it before every workgroup of the group has read it)
        const u64 tag = *reinterpret_cast<const __attribute__((address_space(4))) u64 *>(reinterpret_cast<uintptr_t>(&m->epoch)) + 1;
        attn_piece<D, RW, KW, NT, false, EB>(p, smem, threadIdx.x, rq, pc, [&] {
            if (threadIdx.x == 0)
                __hip_atomic_store(&m->started[pc.bx], tag << 8 | this_xcd(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        merge_group<D, RW * KW, RW * 32>(p, *m, smem, threadIdx.x, pc, p.nsplit, tag);
    } else {
        attn_piece<D, RW, KW, NT, false, EB>(p, smem, threadIdx.x, rq, pc, [] {});
    }
}

// A batch of short requests: a workgroup per (part of at most sps tiles, KV head, request, row block) of the largest request;
// those that a request has no use for leave at once.
template <int D, int RW, int KW, int NT, int EB>
__global__ __launch_bounds__(RW * KW * 64, 2) void tv_attn_short(AttnParams p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    BTV_FETCH_ARGS(p);
    asm volatile("" ::"s"(p.inv_sps), "s"(p.inv_Hkv));
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int uq = quotient(slot, p.row_blocks, p.inv_row_blocks), by = slot - uq * p.row_blocks, unit = uq * 8 + xcd;
    if (unit >= p.units) return;
    Piece pc = {};
    // The part is rotated by the request (and the head).  Without it part i of a head is on the same XCD in every request, or on the
    // same few, and as all requests have a first part and only the longest a last one, some XCDs have most of the work: rotated by the
    // (request, head) number, which comes to the same for an even number of parts, 29 requests of up to 2347 keys with 30 nodes took
    // 69 us, now 61; 31 of up to 3181 with 10 65.5 and 58.
    const int bz = quotient(unit, p.nsplit, p.inv_nsplit);
    pc.rq = quotient(bz, p.Hkv, p.inv_Hkv); pc.g = bz - pc.rq * p.Hkv; pc.by = by;
    const int turned = unit - bz * p.nsplit + 3 * pc.g + pc.rq;
    pc.bx = turned - quotient(turned, p.nsplit, p.inv_nsplit) * p.nsplit;
    const Req rq = load_req<true>(p, pc.rq);
    if (!rq.ok) {
        if (threadIdx.x == 0 && by == 0 && pc.bx == 0 && pc.g == 0) atomicOr(p.flag, 2u);
        return;
    }
    const int tiles = (rq.L + rq.M + 31) >> 5, parts = quotient(tiles + p.sps - 1, p.sps, p.inv_sps);
    if (by * RW * 32 >= rq.M * p.G || pc.bx >= parts) return;
    pc.st0 = pc.bx * p.sps;
    pc.st1 = min(pc.st0 + p.sps, tiles);
    pc.direct = parts == 1;
    attn_piece<D, RW, KW, NT, true, EB>(p, smem, threadIdx.x, rq, pc, [] {});
}

// ---- ragged batches ---------------------------------------------------------------------------------------------------
// The host knows bounds on the requests' sizes only, so the workgroups share the work out themselves: as many as the CUs
// hold, all with about the same time to spend, whatever the lengths.  A request's work for one KV head is a row of
// stretches, one per row block, START + weight * t long for t tiles (START: what starting on a row block and storing its
// rows costs; the weight is WHOLE, or PART where no more than half of the block's rows exist, as a tile goes faster then).
// The stretches lie one after the other, request after request, KV head after KV head (so an XCD keeps to one head or
// two), and team k takes what lies between k w and (k + 1) w; where that cuts a stretch, tv_combine_batch
// merges the parts.  A cut less than MARGIN tiles from where a stretch's tiles begin or end moves there.  A stretch of up to
// SMALL tiles is not cut: the team that its beginning falls to does all of it.  Both make shares uneven by as much as they are long, and that costs
// more than the pieces they save (with 8 and 16 tiles the fullest share of 32 requests of 100 to 4000 tokens was 242 of 174 on average; times below).
// Where trees may take several row blocks a team is a pair of workgroups (neighbours on one XCD, running side by side): a
// stretch stands for two row blocks then, one for each member, over the same tiles, so that the second finds the K/V of the
// first in their L2; an odd last row block is a stretch of half its tiles, each member taking half of every part
// (if it is small, one of them takes it alone).
// Bound by the tiles (0.84 to 0.91 us each in bf16 pieces of more than 128 rows, 0.58 to 0.61 below; FP8 0.49 to 0.51 in pieces of more than 64 rows, 0.32 to 0.34 below), and
// by the pieces: 6 (FP8) to 10.5 us each beyond its tiles (the plan and finding it 1.2 to 1.8, page ids and first tiles 2 to 2.7, the rest of the prologue 1.1, merging
// and storing 1.3 to 2, waiting for the other waves 0.1 to 0.8, the way into and out of the loop 0.5 to 3.2), START comes from that.  us, with START, MARGIN and SMALL of 8, 8 and 16 tiles / 8, 2 and 8 / 10, 2 and 8:
// 8 requests of 1k to 16k, bf16 156 / 155 / 152; 32 of 100 to 4000, FP8 59.7 / 52.8 / 50.9; 5 of up to 8k with 83 nodes 58.5 / 51.8 / 53.8; 9 of up to 9k with
// 12 42.0 / 39.7 / 39.9; 14 of up to 6k, FP8 67.4 / 65.4 / 65.0.  The figures beside the choice of the form
// (short_batch) are the whole call's.
constexpr int WHOLE = 3, PART = 2, START = 10 * WHOLE, MARGIN = 2, SMALL = 8;
// A halved stretch of an odd number of tiles has half a step less for its second member.  A cut one step ahead of its end would leave that
// member's last part empty, nobody would write it, and tv_combine_batch counts it: cuts stay two steps away from the end.
static_assert(MARGIN >= 2, "both members have tiles in every part");
struct Stretch { int t, du, wt, sl, len; };             // tiles; whole stretches; weight of the last; length of the halved one; all
__device__ __forceinline__ Stretch stretch_of(const AttnParams &p, const Req &q)
{
    Stretch s;
    s.t = q.ok ? (q.L + q.M + 31) >> 5 : 0;
    const int rows = q.ok ? q.M * p.G : 0, rb = (rows + (1 << p.wr_log2) - 1) >> p.wr_log2;
    s.du = rb >> p.pairing;
    s.wt = rows - ((rb - 1) << p.wr_log2) <= 1 << p.wr_log2 >> 1 ? PART : WHOLE;
    s.sl = p.pairing && (rb & 1) ? (s.t <= SMALL ? (s.t * s.wt + START + 1) >> 1 : ((s.t + 1) >> 1) * s.wt + START) : 0;
    s.len = s.du * (s.t * (p.pairing ? WHOLE : s.wt) + START) + s.sl;
    return s;
}
__device__ __forceinline__ int wave_incl_scan(int x)
{
    // (rows of 16 by shifts, then the last lane of each row into the rows behind it)
#define BTV_SCAN_STEP(ctrl, rows) x += __builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xF, ctrl < 0x142)
    BTV_SCAN_STEP(0x111, 0xF); BTV_SCAN_STEP(0x112, 0xF); BTV_SCAN_STEP(0x114, 0xF); BTV_SCAN_STEP(0x118, 0xF);
    BTV_SCAN_STEP(0x142, 0xA); BTV_SCAN_STEP(0x143, 0xC);
#undef BTV_SCAN_STEP
    return x;
}
// 64 lengths: their low and high halves on their own, so that no sum leaves 32 bits
__device__ __forceinline__ long long wave_incl_scan_len(int x)
{
    return ((long long)wave_incl_scan(x >> 16) << 16) + wave_incl_scan(x & 0xFFFF);
}
// Where a team stands.  Every wavefront of its workgroups works this out for itself.
struct Walk {
    long long first, end;                               // the team's share
    long long pos, head;                                // what comes next; where its KV head's work begins
    long long wh;                                       // one head's work
    int h, w;                                           // that KV head; a share
};

// A chunk of 64 requests, one per lane: their stretches, and where they end in a head's work (cum: where the chunk begins).
struct Chunk { Stretch s; long long incl; bool bad; };
__device__ __forceinline__ Chunk load_chunk(const AttnParams &p, int c0, int lane, long long cum)
{
    Chunk c;
    const bool in = c0 + lane < p.batch;
    const Req q = load_req<true>(p, min(c0 + lane, p.batch - 1));
    c.s = stretch_of(p, q);
    c.bad = in && !q.ok;
    c.incl = wave_incl_scan_len(in ? c.s.len : 0) + cum;
    return c;
}
// The first chunk is kept in LDS from one piece to the next.  Loaded again it cost 1.1 us a piece (1.4 to 1.8 pieces a workgroup): its loads
// wait behind the last piece's stores; from LDS 0.5.  8 requests of 1k to 16k, two layers and trees, 303 -> 299 us; 32 of 100 to 4000, FP8, 119.4 -> 115.9; 20 of 1k to
// 6k with 64 channels 181 -> 176.  (Looking for the next piece during this one's first loads, by one wavefront that tells the others: +-1 %.)  Raw
// instructions: ahead of ordinary reads the compiler waits for the stores as well.
constexpr int CHUNK_BYTES = 64 * 32;
__device__ __forceinline__ void keep_chunk(uint32_t kept, int lane, const Chunk &c)
{
    const u32x4 a = { (uint32_t)c.s.t, (uint32_t)c.s.du, (uint32_t)c.s.wt, (uint32_t)c.s.sl }, b = { (uint32_t)c.s.len, (uint32_t)c.incl, (uint32_t)(c.incl >> 32), 0 };
    asm volatile("ds_write_b128 %0, %1\n\tds_write_b128 %0, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" :: "v"(kept + (uint32_t)lane * 32), "v"(a), "v"(b) : "memory");
}
__device__ __forceinline__ Chunk kept_chunk(uint32_t kept, int lane)
{
    u32x4 a, b;
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" : "=&v"(a), "=&v"(b) : "v"(kept + (uint32_t)lane * 32) : "memory");
    Chunk c;
    c.s.t = (int)a[0]; c.s.du = (int)a[1]; c.s.wt = (int)a[2]; c.s.sl = (int)a[3]; c.s.len = (int)b[0];
    c.incl = (long long)((unsigned long long)b[2] << 32 | b[1]);
    c.bad = false;
    return c;
}
__device__ __forceinline__ long long last_lane(long long x)
{
    return (long long)(((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), 63) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)x, 63));
}

// The share of a team (the `nth` on its XCD), and the first chunk of requests.  The very first workgroup leaves the plan for the merge.
__device__ __forceinline__ Walk share_out(const AttnParams &p, int xcd, int nth, int lane, bool leader, Chunk &c)
{
    Walk k;
    long long begin = 0;
    bool bad = false;
    for (int c0 = ((p.batch - 1) >> 6) << 6; c0 >= 0; c0 -= 64) {         // (the first chunk last; sums of the others do not matter yet)
        c = load_chunk(p, c0, lane, 0);
        bad = bad || c.bad;
        begin += last_lane(c.incl);
    }
    k.wh = begin;
    const long long all = k.wh * p.Hkv;
    const long long w = max((all + (1 << p.teams_log2) - 1) >> p.teams_log2, (long long)p.wmin);
    if (leader) {
        long long cum = 0;
        for (int c0 = 0; c0 < p.batch; c0 += 64) {
            const Chunk d = c0 ? load_chunk(p, c0, lane, cum) : c;
            if (c0 + lane < p.batch) p.plan[2 + c0 + lane] = d.incl - d.s.len;
            cum = last_lane(d.incl);
        }
        if (lane == 0) { p.plan[0] = w; p.plan[1] = k.wh; }
        if (bad) atomicOr(p.flag, 2u);
    }
    k.w = (int)min(w, (long long)INT_MAX);
    // neighbouring shares on one XCD, as many on each: where the work is for a part of the teams, all XCDs have some
    long long per_xcd = (1 << p.teams_log2) >> 3;
    if (w == p.wmin) per_xcd = min(per_xcd, ((all + w - 1) / w + 7) >> 3);
    k.first = k.pos = nth < per_xcd ? min((xcd * per_xcd + nth) * w, all) : all;
    k.end = min(k.first + w, all);
    k.head = 0; k.h = 0;
    return k;
}

// The member's next piece; the walk moves behind it.  False: none left.  c holds the first chunk of requests.
__device__ __forceinline__ bool next_piece(const AttnParams &p, Walk &k, int member, int lane, const Chunk &c, Piece &pc)
{
    while (k.pos < k.end) {
        while (k.pos - k.head >= k.wh) { k.head += k.wh; ++k.h; }
        const long long x = k.pos - k.head;
        Chunk d = c;
        int r0 = 0;
        unsigned long long beyond;
        while ((beyond = __builtin_amdgcn_ballot_w64(x < d.incl)) == 0ull) {
            r0 += 64;
            if (r0 >= p.batch) return false;            // (cannot be: x lies within the head's work)
            d = load_chunk(p, r0, lane, last_lane(d.incl));
        }
        const int src = __builtin_ctzll(beyond);
        Stretch s;
        s.t = __builtin_amdgcn_readlane(d.s.t, src); s.du = __builtin_amdgcn_readlane(d.s.du, src);
        s.wt = __builtin_amdgcn_readlane(d.s.wt, src); s.sl = __builtin_amdgcn_readlane(d.s.sl, src);
        s.len = __builtin_amdgcn_readlane(d.s.len, src);
        const int y = s.len + __builtin_amdgcn_readlane((int)(x - d.incl), src);       // place in the request's work
        const int whole = s.t * (p.pairing ? WHOLE : s.wt) + START, u = min(y / whole, s.du);
        const bool halved = u == s.du;
        const int y0 = y - u * whole;                   // ... in the stretch
        const long long us = k.pos - y0;                // where the stretch begins
        pc.rq = r0 + src;
        pc.g = k.h;
        pc.by = p.pairing ? (halved ? 2 * u : 2 * u + member) : u;
        pc.bx = 0; pc.direct = 1; pc.st0 = 0; pc.st1 = s.t;
        if (s.t <= SMALL) {
            k.pos = us + (halved ? s.sl : whole);
            if (y0 == 0 && (!halved || ((pc.rq ^ k.h) & 1) == member)) return true;
            continue;
        }
        const int wt = halved || !p.pairing ? s.wt : WHOLE;
        const int tl = halved ? (s.t + 1) >> 1 : s.t, cl = tl * wt, cm = MARGIN * wt;  // tiles of the stretch; their length
        const long long ts = us + START;                // they begin here
        int c0 = y0 - START, c1 = (int)min(k.end - ts, (long long)cl);
        if (c0 < cm) c0 = 0; else if (c0 > cl - cm) c0 = cl;
        if (c1 < cm) c1 = 0; else if (c1 > cl - cm) c1 = cl;
        k.pos = c1 < cl ? k.end : ts + cl;
        if (c0 >= c1) continue;
        const int cut = c0 == 0 ? 0 : (c0 - cm) / k.w + 1;
        const int x0 = c0 / wt, x1 = c1 / wt;
        if (!halved) {
            pc.st0 = x0; pc.st1 = x1; pc.bx = cut; pc.direct = c0 == 0 && c1 == cl;
            return true;
        }
        pc.bx = 2 * cut + member; pc.direct = 0;
        pc.st0 = member ? x0 + x1 : 2 * x0;
        pc.st1 = member ? min(2 * x1, s.t) : x0 + x1;
        if (pc.st0 < pc.st1) return true;
    }
    return false;
}

template <int D, int RW, int KW, int NT, int EB>
__global__ __launch_bounds__(RW * KW * 64, 2) void tv_attn_batch(AttnParams p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    BTV_FETCH_ARGS(p);
    asm volatile("" ::"s"(p.plan), "s"(p.batch), "s"(p.teams_log2), "s"(p.pairing), "s"(p.wmin), "s"(p.wr_log2));
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, member = slot & p.pairing;
    Chunk c;
    Walk k = share_out(p, xcd, slot >> p.pairing, threadIdx.x & 63, blockIdx.x == 0 && threadIdx.x < 64, c);
    const uint32_t kept = (uint32_t)(uintptr_t)BTV_LDS_PTR(smem) + PageLds<D, RW, KW, NT, true, EB>::BYTES;
    if (threadIdx.x < 64) keep_chunk(kept, threadIdx.x, c);     // (barriers before it is read: those of the first piece)
    for (bool again = false;; again = true) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                   // keeps what derives from it (all addresses) from being carried across pieces
        if (again) {
            if (k.pos >= k.end) break;
            c = kept_chunk(kept, tid & 63);
        }
        Piece pc = {};
        if (!next_piece(p, k, member, tid & 63, c, pc)) break;
        attn_piece<D, RW, KW, NT, true, EB>(p, smem, tid, load_req<true>(p, pc.rq), pc, [] {});
        // every wave is done with this piece's LDS, its own fills have landed; the stores may still be on their way
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    }
}

// Split-K combine: O[row] = sum_s w_s a_s O'_s / sum_s w_s l_s with w_s = exp2((m_s - max m) * scale*log2 e), O'_s the
// fp16 partial and a_s the magnitude it was divided by.
// 8 rows per workgroup, 32 lanes per row, each lane owns D/32 consecutive channels.  Lane j of a row fetches the
// (m, l) pairs of splits j, j + 32, ... and computes their weights; the partial rows of up to 32 splits are fetched
// by independent loads issued before anything is waited for, so the kernel costs about one memory round trip
// whatever the number of splits.  What happens between the lanes of a row stays off the LDS crossbar where it can:
// maximum and sum over the 32 lanes are DPP steps within the rows of 16 and one swap between the two rows (they were
// five dependent ds_bpermute round trips each), and the 32 weights reach every lane through one LDS store and eight
// 16-byte reads of the same address (they were 32 shuffles, each waited for before its multiply-adds).
__device__ __forceinline__ float row32_max(float x, int lane)
{
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xF, 0xF, false)));    // quad_perm [1,0,3,2]
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xF, 0xF, false)));    // quad_perm [2,3,0,1]
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xF, 0xF, false)));   // row_half_mirror
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x140, 0xF, 0xF, false)));   // row_mirror
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(x, __uint_as_float((lane & 16) ? sw[0] : sw[1]));                                               // the other row of 16
}

__device__ __forceinline__ float row32_sum(float x, int lane)
{
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xF, 0xF, false));
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xF, 0xF, false));
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xF, 0xF, false));
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x140, 0xF, 0xF, false));
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return x + __uint_as_float((lane & 16) ? sw[0] : sw[1]);
}

// Over the N = 8, 16 or 32 lanes of a row.
template <int N>
__device__ __forceinline__ float lanes_max(float x)
{
    if (N == 32) return row32_max(x, (int)threadIdx.x);
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xF, 0xF, false)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xF, 0xF, false)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xF, 0xF, false)));
    return N == 8 ? x : fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x140, 0xF, 0xF, false)));
}
template <int N>
__device__ __forceinline__ float lanes_sum(float x)
{
    if (N == 32) return row32_sum(x, (int)threadIdx.x);
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xF, 0xF, false));
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xF, 0xF, false));
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xF, 0xF, false));
    return N == 8 ? x : x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x140, 0xF, 0xF, false));
}

// E = 2, 4 or 8 channels per lane
template <int D, int E>
__device__ __forceinline__ void store_row(const AttnParams &p, size_t row, int lane, const float (&acc)[E], float inv)
{
    uint16_t *dst = static_cast<uint16_t *>(p.O) + row * D + lane * E;
    uint32_t x[E / 2];
#pragma unroll
    for (int e = 0; e < E / 2; ++e) x[e] = float_to_bf16_bits(acc[2 * e] * inv) | (float_to_bf16_bits(acc[2 * e + 1] * inv) << 16);
    if constexpr (E == 8) *reinterpret_cast<uint4 *>(dst) = make_uint4(x[0], x[1], x[2], x[3]);
    else if constexpr (E == 4) *reinterpret_cast<uint2 *>(dst) = make_uint2(x[0], x[1]);
    else *reinterpret_cast<uint32_t *>(dst) = x[0];
}

template <int D>
__device__ __forceinline__ void combine_row(const AttnParams &p, size_t row, int nsplit_r, float (&wsh)[8][32])
{
    constexpr int E = D / 32;
    typedef _Float16 hvec __attribute__((ext_vector_type(E)));
    const int rin = threadIdx.x >> 5, lane = threadIdx.x & 31;
    const size_t sstride = (size_t)p.total_rows;
    // reference maximum over all splits: with more than 32 of them it takes a round trip of its own
    float mmax = NEG_BIG;
    for (int s = lane + 32; s < nsplit_r; s += 32) mmax = fmaxf(mmax, p.ML[(s * sstride + row) * 4]);
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    float den = 0.f;
    for (int s0 = 0; s0 < nsplit_r; s0 += 32) {     // one pass for up to 32 splits
        const int s_mine = s0 + lane;
        const float4 mlr = *reinterpret_cast<const float4 *>(p.ML + ((size_t)min(s_mine, nsplit_r - 1) * sstride + row) * 4);
        const float4 ml = s_mine < nsplit_r ? mlr : make_float4(NEG_BIG, 0.f, 0.f, 0.f);
        hvec part[32];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (s0 + 8 * g < nsplit_r) {             // uniform within the row's lanes: whole groups of 8 loads
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const int s = min(s0 + 8 * g + b, nsplit_r - 1);
                    part[8 * g + b] = *reinterpret_cast<const hvec *>(p.Opart + (s * sstride + row) * D + lane * E);
                }
            }
        if (s0 == 0) mmax = row32_max(fmaxf(mmax, ml.x), (int)threadIdx.x);
        const float w = s_mine < nsplit_r ? __builtin_amdgcn_exp2f(ml.x - mmax) : 0.f;
        den += w * ml.y;
        wsh[rin][lane] = w * ml.z;                              // weight times the partial's magnitude; 0 past the last split
        // (the row's 32 lanes are one half of a wavefront: its LDS operations complete in order, no barrier needed)
        float wgt[32];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(&wsh[rin][4 * q]);
            wgt[4 * q] = x.x; wgt[4 * q + 1] = x.y; wgt[4 * q + 2] = x.z; wgt[4 * q + 3] = x.w;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (s0 + 8 * g < nsplit_r) {
#pragma unroll
                for (int b = 0; b < 8; ++b) {
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[e] += wgt[8 * g + b] * (float)part[8 * g + b][e];
                }
            }
    }
    den = row32_sum(den, (int)threadIdx.x);
    const float inv = p.out_scale / den;
    store_row<D, E>(p, row, lane, acc, inv);
}

template <int D>
__global__ __launch_bounds__(256) void tv_combine_bf16(AttnParams p)
{
    __shared__ __attribute__((aligned(16))) float wsh[8][32];
    // every argument in one round trip (the argument block is cold in every launch)
    asm volatile("" ::"s"(p.O), "s"(p.Opart), "s"(p.ML), "s"(p.M), "s"(p.L), "s"(p.Hq), "s"(p.total_rows), "s"(p.nsplit), "s"(p.out_scale));
    const int row = blockIdx.x * 8 + (threadIdx.x >> 5);
    if (row >= p.M * p.Hq) return;
    combine_row<D>(p, (size_t)row, p.nsplit, wsh);
}

// The same for a batch: how many parts a row has follows from where its request's work lies (the plan that the attention's first
// workgroup left).  What bounds it is the chain of the request's place, the parts and the sums: lanes of E channels, the first PARTS
// parts all asked for at once.  With 8 channels a lane has 16-byte loads and half of the wavefronts do, so those of many rows are under way
// together (8 requests of up to 128 nodes, 32 heads: attention and merge 156 -> 153 us, 150 to 156 from run to run; 32 of up to 24, FP8, 51.1 -> 49.1); few rows leave the
// chip room, and D / 32 channels with 16 parts at once are faster (7 requests of 33 nodes, 16 heads, in up to 20 parts: 23.8 and 25.6).
template <int D, int E, int PARTS>
__global__ __launch_bounds__(256) void tv_combine_batch(AttnParams p)
{
    constexpr int LPR = D / E, ROWS = 256 / LPR;             // lanes of a row, rows of a workgroup
    __shared__ __attribute__((aligned(16))) float wsh[ROWS][LPR];
    asm volatile("" ::"s"(p.O), "s"(p.q_offset), "s"(p.prefix_len), "s"(p.Opart), "s"(p.ML), "s"(p.M), "s"(p.L), "s"(p.Hq), "s"(p.G),
                 "s"(p.max_blocks), "s"(p.total_rows), "s"(p.total_M), "s"(p.plan), "s"(p.Hkv), "s"(p.pairing), "s"(p.wr_log2), "s"(p.sps), "s"(p.out_scale));
    const int r = blockIdx.y;
    const Req q = load_req<true>(p, r);
    long long w = 0, wh = 0, at = 0;
    if (!p.sps) { w = p.plan[0]; wh = p.plan[1]; at = p.plan[2 + r]; }
    if (!q.ok) return;
    const int lr = blockIdx.x * ROWS + threadIdx.x / LPR;
    if (lr >= q.M * p.Hq) return;
    int n = 1;
    if (p.sps) {                                        // short requests: equal parts
        n = (((q.L + q.M + 31) >> 5) + p.sps - 1) / p.sps;
    } else {
        const Stretch s = stretch_of(p, q);
        const int node = lr / p.Hq, hq = lr - node * p.Hq, h = hq / p.G, by = (node * p.G + hq - h * p.G) >> p.wr_log2;
        if (s.t <= SMALL) return;                           // written by the attention kernel
        const int u = by >> p.pairing;
        const bool halved = u == s.du;
        const int wt = halved || !p.pairing ? s.wt : WHOLE;
        const int cl = (halved ? (s.t + 1) >> 1 : s.t) * wt, cm = MARGIN * wt;
        const long long ts = h * wh + at + (long long)u * (s.t * WHOLE + START) + START;   // (u = 0 where a team is one workgroup)
        const long long lo = ts + cm, hi = ts + cl - cm;    // where a cut counts
        if (hi >= lo) n += wh * p.Hkv < INT_MAX ? (int)hi / (int)w - ((int)lo - 1) / (int)w : (int)(hi / w - (lo - 1) / w);
        if (halved) n *= 2;
    }
    if (n == 1) return;
    // The first PARTS parts, in groups of four, are all asked for before the first is looked at.
    typedef _Float16 hvec __attribute__((ext_vector_type(E)));
    constexpr int GROUPS = PARTS / 4, TURNS = PARTS > LPR ? PARTS / LPR : 1;
    const int rin = threadIdx.x / LPR, lane = threadIdx.x % LPR;
    const size_t row = (size_t)q.q0 * p.Hq + lr, sstride = (size_t)p.total_rows;
    auto magnitudes = [&](int s) {
        const float4 x = *reinterpret_cast<const float4 *>(p.ML + (min(s, n - 1) * sstride + row) * 4);
        return s < n ? x : make_float4(NEG_BIG, 0.f, 0.f, 0.f);
    };
    const _Float16 *Pp = p.Opart + row * D + lane * E;
    hvec part[GROUPS][4];
    auto load = [&](hvec (&x)[4], int s0) {
#pragma unroll
        for (int b = 0; b < 4; ++b) x[b] = *reinterpret_cast<const hvec *>(Pp + min(s0 + b, n - 1) * sstride * D);
    };
    float4 ml[TURNS];
#pragma unroll
    for (int k = 0; k < TURNS; ++k) ml[k] = magnitudes(k * LPR + lane);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        if (g == 0 || n > 4 * g) load(part[g], 4 * g);
    float mmax = ml[0].x, den = 0.f;
#pragma unroll
    for (int k = 1; k < TURNS; ++k) mmax = fmaxf(mmax, ml[k].x);
    for (int s = lane + TURNS * LPR; s < n; s += LPR) mmax = fmaxf(mmax, p.ML[(s * sstride + row) * 4]);     // (rare)
    mmax = lanes_max<LPR>(mmax);
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    auto weights = [&](const float4 &m, int s0) {           // of the LPR parts from s0 on, one per lane
        const float w = s0 + lane < n ? __builtin_amdgcn_exp2f(m.x - mmax) : 0.f;
        den += w * m.y;
        wsh[rin][lane] = w * m.z;                           // weight times the part's magnitude; 0 past the last part
        // (the row's lanes are in one wavefront: its LDS operations complete in order, no barrier needed)
    };
    auto add = [&](const hvec (&x)[4], int at) {
        const float4 wg = *reinterpret_cast<const float4 *>(&wsh[rin][at]);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += wg.x * (float)x[0][e] + wg.y * (float)x[1][e] + wg.z * (float)x[2][e] + wg.w * (float)x[3][e];
    };
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        if (g == 0 || n > 4 * g) {
            if (4 * g % LPR == 0) weights(ml[4 * g / LPR], 4 * g);
            add(part[g], 4 * g % LPR);
        }
#pragma unroll 1
    for (int s0 = PARTS; s0 < n; s0 += 4) {
        if ((s0 & (LPR - 1)) == 0) weights(magnitudes(s0 + lane), s0);
        load(part[0], s0);
        add(part[0], s0 & (LPR - 1));
    }
    const float inv = p.out_scale / lanes_sum<LPR>(den);
    store_row<D, E>(p, row, lane, acc, inv);
}

// ------------------------------------------------------------------------------------------------
// fp32 kernel: one workgroup per (node, query head), over the keys in chunks of CH = 256 (D = 64) or 128 (D = 128; 512
// threads for 256 keys measured the same).
// Precision path, not the fast one; the shapes it sees are small, so what it costs is its chain of steps, a launch for
// the ancestor masks among them once.  A key's score takes D / 64 neighbouring threads, 64 channels each; its
// probability goes to LDS; then a thread owns one channel of 64 of the chunk's keys, whose values are on their way since
// before the scores (one memory round trip per chunk).  The node's ancestors are walked by one thread over parent[] in
// LDS while the keys arrive.  144 keys, 16 nodes, one head: 5.3 us; with a private softmax state of all channels per
// thread, merged by D * 6 shuffles, and the masks' launch it was 12.3.
// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void tv_attn_f32(AttnParams p)
{
    constexpr int TPK = D / 64, CH = 256 / TPK, GROUPS = 256 / D, WAVES = 4;   // threads per key, keys per chunk, groups of 64 keys
    static_assert(GROUPS * 64 == CH, "a thread of each group takes 64 of the chunk's keys");
    __shared__ __attribute__((aligned(16))) float qs[D], prob[CH], red[GROUPS][D];
    __shared__ float wmax[WAVES], wsum[WAVES];
    __shared__ int par[BTV_MAX_NODES];
    __shared__ unsigned char seen[BTV_MAX_NODES];
    asm volatile("" ::"s"(p.Q), "s"(p.K), "s"(p.V), "s"(p.O), "s"(p.parent), "s"(p.flag), "s"(p.M), "s"(p.L), "s"(p.Hq), "s"(p.Hkv), "s"(p.G), "s"(p.scale));
    const int i = blockIdx.x, hq = blockIdx.y, tid = threadIdx.x, g = hq / p.G;
    const float *Q = static_cast<const float *>(p.Q) + ((size_t)i * p.Hq + hq) * D;
    const float *K = static_cast<const float *>(p.K) + (size_t)g * D, *V = static_cast<const float *>(p.V) + (size_t)g * D;
    const size_t pitch = (size_t)p.Hkv * D;
    const int S = p.L + p.M;
    const int kk = tid / TPK, part = (tid % TPK) * 64;                         // scores: this thread's key of the chunk, its channels
    const int d = tid % D, kg = tid / D;                                       // values: its channel, its group of keys
    if (tid < D) qs[tid] = Q[tid];
    if (tid < p.M) par[tid] = p.parent[tid];
    seen[tid] = 0;
    float m = NEG_BIG, lsum = 0.f, o = 0.f;
    for (int j0 = 0; j0 < S; j0 += CH) {
        float4 kv[16];
        float vv[64];
        const float *kr = K + (size_t)min(j0 + kk, S - 1) * pitch + part;
#pragma unroll
        for (int u = 0; u < 16; ++u) kv[u] = *reinterpret_cast<const float4 *>(kr + 4 * u);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (j0 + kg * 64 + b * 16 < S)                                     // (uniform in a wavefront)
#pragma unroll
                for (int u = 0; u < 16; ++u) vv[b * 16 + u] = V[(size_t)min(j0 + kg * 64 + b * 16 + u, S - 1) * pitch + d];
        __syncthreads();                                                       // (also: the last chunk's probabilities have been read)
        if (j0 == 0) {                                                         // the node's ancestors, and every parent's check
            if (tid < p.M && (par[tid] < -1 || par[tid] >= tid)) atomicOr(p.flag, 1u);
            if (tid == 255)
                for (int a = i; a >= 0;) {
                    seen[a] = 1;
                    const int pa = par[a];
                    a = pa < -1 || pa >= a ? -1 : pa;                          // an invalid entry ends the walk (flagged above)
                }
        }
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float4 q4 = *reinterpret_cast<const float4 *>(&qs[part + 4 * u]);
            s = fmaf(q4.x, kv[u].x, s); s = fmaf(q4.y, kv[u].y, s);
            s = fmaf(q4.z, kv[u].z, s); s = fmaf(q4.w, kv[u].w, s);
        }
        if (TPK == 2) s += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(s), 0xB1, 0xF, 0xF, false));   // the pair's other half
        s *= p.scale;
        __syncthreads();                                                       // seen[]
        const int j = j0 + kk;
        const bool visible = j < p.L || (j < S && seen[j - p.L] != 0);
        float mx = visible ? s : NEG_BIG;
        mx = row32_max(mx, tid);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if ((tid & 63) == 0) wmax[tid >> 6] = mx;
        __syncthreads();
        float mn = m;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) mn = fmaxf(mn, wmax[k]);
        const float alpha = expf(m - mn), pj = visible ? expf(s - mn) : 0.f;
        m = mn;
        lsum = lsum * alpha + pj;
        if (part == 0) prob[kk] = pj;
        __syncthreads();
        o *= alpha;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (j0 + kg * 64 + b * 16 < S)
#pragma unroll
                for (int u = 0; u < 16; u += 4) {
                    const float4 pr = *reinterpret_cast<const float4 *>(&prob[kg * 64 + b * 16 + u]);
                    o = fmaf(pr.x, vv[b * 16 + u], o); o = fmaf(pr.y, vv[b * 16 + u + 1], o);
                    o = fmaf(pr.z, vv[b * 16 + u + 2], o); o = fmaf(pr.w, vv[b * 16 + u + 3], o);
                }
    }
    lsum = row32_sum(lsum, tid);
    lsum += __shfl_xor(lsum, 32);
    if ((tid & 63) == 0) wsum[tid >> 6] = lsum;
    red[kg][d] = o;
    __syncthreads();
    if (tid < D) {
        float x = red[0][tid];
#pragma unroll
        for (int k = 1; k < GROUPS; ++k) x += red[k][tid];
        float den = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) den += wsum[k];
        den *= 1.0f / TPK;                                                     // (every thread of a key counted it)
        static_cast<float *>(p.O)[((size_t)i * p.Hq + hq) * D + tid] = x / den;
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
// ---- scratch of the entry point that allocates nothing ---------------------------------------------------------
// One array per GPU, part of the loaded code object (zero until first used), held until the process ends.  Host code
// never uses the array's name as an address: the device address is asked for once per device and kept.
constexpr size_t SCRATCH_BYTES = (size_t)32 << 20;
constexpr size_t MOST_PARTIALS = (size_t)31 << 20;      // bytes of partials that a plan of one request may take: they and the words fit the array
constexpr int SCRATCH_MAX_DEVICES = 64;
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];
void *g_scratch_ptr[SCRATCH_MAX_DEVICES];
std::atomic<bool> g_scratch_known[SCRATCH_MAX_DEVICES];

// Device address of the current device's copy of `scratch` (looked up on the first call per device).
int scratch_address(void **out)
{
    int dev = -1;
    BTV_HIP(hipGetDevice(&dev));
    BTV_REQUIRE(dev >= 0 && dev < SCRATCH_MAX_DEVICES, "device index %d outside [0,%d)", dev, SCRATCH_MAX_DEVICES);
    if (!g_scratch_known[dev].load(std::memory_order_acquire)) {
        void *ptr = nullptr;
        BTV_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        BTV_REQUIRE(ptr != nullptr, "no device address for the scratch array");
        g_scratch_ptr[dev] = ptr;                   // (two racing first calls store the same address)
        g_scratch_known[dev].store(true, std::memory_order_release);
    }
    *out = g_scratch_ptr[dev];
    return BTV_OK;
}

// Clears the first `words` 32-bit words at p (a kernel rather than a memset node, so that the call can be captured).
__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t *p, int words)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < words) p[i] = 0u;
}

constexpr int MOST_SPLITS = 64;                         // that the library chooses by itself
struct Plan { int rw, kw, nt, wr, row_blocks, stages, sps, longer, nsplit; float bytes; };      // (bytes of K and V)

// Whether the workgroups of a plan merge their partials themselves (merge_group): few enough splits and groups for its words; all
// groups' workgroups congruent mod 8, and as many on each XCD; and the chip takes all at once.  Where the KV heads do not share out
// evenly over the XCDs the groups do, and a head's row blocks, on up to 8 XCDs, each read its K/V: 2 .. 4 % faster than the two
// launches for up to 64 MB of such reading (330 plans of 1 to 6 KV heads), 1 .. 3 % slower on average above, 25 % at 140 .. 200 MB.
bool merges_inside(const Plan &pl, int Hkv)
{
    const int groups = Hkv * pl.row_blocks;
    return pl.nsplit > 1 && pl.nsplit <= MERGE_SPLITS && groups <= MERGE_GROUPS &&
           (Hkv % 8 == 0 || (groups % 8 == 0 && pl.bytes * (float)(std::min(8, pl.row_blocks) - 1) <= 64e6f)) &&
           pl.nsplit * groups <= (pl.rw == 2 ? 512 : 256);
}

// Rows of one split's partials, by either merge.
size_t partial_rows(const Plan &pl, int M, int Hq, int Hkv)
{
    return std::max<size_t>((size_t)M * Hq, (size_t)Hkv * pl.row_blocks * (std::min(pl.wr, M * (Hq / Hkv)) + 1));
}

// Splits of `want` parts for a shape: whole rounds of KW tiles, as evenly as they go.
void split_plan(Plan &pl, int L, int want)
{
    // The last split has the tree rows: its workgroups find the ancestor sets and mask tiles (in the pipelined loop those also lose
    // the overlap).  Shared out as if there were `extra` more rounds at the end, it is that much shorter.
    const int tree_tiles = pl.stages - L / TK, rounds = (pl.stages + pl.kw - 1) / pl.kw;
    pl.nsplit = std::max(1, std::min(want, rounds));
    const int extra = std::min(pl.kw == 1 ? (7 * tree_tiles + 9) / 10 : 1, rounds / pl.nsplit - 1);
    const int all = rounds + (pl.nsplit > 1 ? extra : 0);
    pl.sps = all / pl.nsplit * pl.kw;
    pl.longer = all % pl.nsplit;
}

// Shape of the workgroups (64, 128 or 256 packed rows of a KV head; 32 rows per wave, pairs of waves alternating over the
// tiles in the first two, the software-pipelined loop in the third) and number of key splits of one request: those with
// the least estimated time.  The estimate: what a workgroup takes, its start and its tiles (two workgroups of the 64-row shape
// share a CU at 1.3 times the time each), times the rounds in which the CUs of the fullest XCD take the workgroups, but no less than the
// K/V bytes need, some of the smaller of the two on top; and for more than one split the merge.  Its constants are a fit to
// 1200 shapes with splits of equal length, as they were cut then (fitted again to splits that differ by a round: 0.2 %; prefixes of 64 to 32k, 4 to 256 nodes, 2 to 8 KV heads, all three K/V types and head sizes) times all shapes
// and 28 split counts, of the choice and of the time: the choice is 1.2 % behind the best one found on average (fitted to 700 of
// them, 1.1 % on the other 500; with the constants of the merge by a second launch 2.0 %), a rule by row count alone (always
// 256 workgroups where the tiles allow it) was 15 % behind, 70 % for many rows over a short prefix (860 rows over 450 keys: 21 us
// in 256-row blocks and 2 splits, 12 us in 64-row blocks and 5).
// `force_split` > 0 and `force_shape` in 1..3 replace the choice (the tuning entry point passes them).
Plan make_plan(int M, int L, int Hq, int Hkv, int D, int eb = 2, int force_split = 0, int force_shape = 0)
{
    static constexpr struct { int rw, kw, nt; float start, tile[3]; } SHAPES[3] = {      // us; tile: bf16 D = 128, D = 64, FP8
        { 2, 2, 5, 1.90f, { 0.420f, 0.271f, 0.372f } },
        { 4, 2, 8, 2.47f, { 0.494f, 0.294f, 0.495f } },
        { 8, 1, 8, 2.22f, { 0.675f, 0.433f, 0.0f } },
    };
    static constexpr float SHARED_TILE[3] = { 0.596f, 0.337f, 0.517f };                   // two 64-row workgroups on a CU
    static constexpr int SPLITS[] = { 1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 64 };
    const int rows_g = Hq / Hkv * M, kind = eb == 1 ? 2 : D == 64 ? 1 : 0;
    const float bytes = 2.0f * ((float)L + M) * Hkv * D * eb, mem = bytes / 6.73e6f, part = 2.0f * M * Hq * D * 1e-6f;
    Plan best = {};
    float best_t = 0.f;
    for (int k = 0; k < 3; ++k) {
        if (force_shape ? force_shape != k + 1 && !(eb == 1 && force_shape == 3 && k == 1) : eb == 1 && k == 2) continue;
        Plan pl;
        pl.rw = SHAPES[k].rw; pl.kw = SHAPES[k].kw; pl.nt = SHAPES[k].nt;
        pl.wr = pl.rw * 32; pl.bytes = bytes;
        pl.row_blocks = (rows_g + pl.wr - 1) / pl.wr;
        pl.stages = (L + M + TK - 1) / TK;
        auto consider = [&](int want) {
            split_plan(pl, L, want);
            const int n = pl.nsplit, wgs = (n * Hkv + 7) / 8 * 8 * pl.row_blocks;         // (as many as the fullest XCD has, times 8)
            const float cap = k == 0 ? 512.f : 256.f, fill = wgs / cap;
            const float rounds = 0.31f * std::ceil(fill) + 0.69f * std::max(1.f, fill);
            const float comp = rounds * (SHAPES[k].start + (pl.sps + (pl.longer ? pl.kw : 0)) * (k == 0 && wgs > 256 ? SHARED_TILE[kind] : SHAPES[k].tile[kind]));
            float t = std::max(comp, mem) + 0.123f * std::min(comp, mem);
            if (n > 1) t += merges_inside(pl, Hkv) ? 1.67f + 0.70f * n * part : 1.78f + 0.83f * n * part + 0.095f * std::max(0, n - 32);
            if (!best_t || t < best_t) { best = pl; best_t = t; }
        };
        if (force_split > 0) { consider(force_split); continue; }
        // no more splits than tiles, nor partials than the built-in scratch array holds (32 MB are 6 us to write and read)
        const int most = (int)std::min<long long>(std::min(MOST_SPLITS, pl.stages),
                                                  std::max<long long>(1, (long long)(MOST_PARTIALS / (partial_rows(pl, M, Hq, Hkv) * (D * 2 + 16)))));
        for (int want : SPLITS)
            if (want <= most) consider(want);
        for (int cap = 256; cap <= (k == 0 ? 1024 : 512); cap *= 2) {                     // as many as whole rounds take
            const int want = cap / (8 * pl.row_blocks) * 8 / Hkv;
            if (want >= 1 && want <= most) consider(want);
        }
    }
    return best;
}

// A batch: shape of the workgroups by the largest tree's packed rows; in how many parts a row's partials may come; whether a
// merge can be needed at all.  Then either (sps > 0) a workgroup per part of sps tiles, or the plan that the workgroups make
// themselves: how many teams of them the chip holds and the smallest share (slots: a stretch of the longest request gets that
// many parts where the average one is 2.5 times shorter; longer ones larger parts).
struct PlanB { int rw, wr_log2, pairing, teams_log2, slots, wmin, sps, row_blocks; bool merge; };
// The plan that the workgroups make themselves pays where they have much to do (64-row tiles per CU at most, of 128 channels; t: tiles of the longest
// request); below, its larger row blocks and the longer way to the first tile cost more than an even load gives.  us, a grid of parts / the plan.  128 channels: 35
// tiles per CU, t = 142 22.5 / 33.5; 45, t = 242 30.0 / 26.3; 58, t = 124 35.2 / 33.7; 61, t = 63 27.2 / 32.4; 62, t = 333 37.0 / 28.4; 75, t = 240 42.1 / 35.4; 86, t = 185
// 30.4 / 36.9; 101, t = 294 67.6 / 59.9; 104, t = 119 47.5 / 38.0; 115, t = 123 41.0 / 36.2; 150, t = 89 39.2 / 39.4; 178, t = 127 53.2 / 51.7.  64 channels: 60, t = 192
// 21.4 / 26.7; 88, t = 378 27.1 / 30.7; 107, t = 229 27.1 / 26.9; 106, t = 310 28.0 / 24.8; 147, t = 91 33.9 / 28.5; 154, t = 176 35.9 / 29.2; 160, t = 214 28.1 / 29.0; 226, t = 259
// 44.8 / 33.5.  What decides besides is how uneven the lengths are, which the host does not know: of 190 batches the choice is 3.0 % slower than the better form on
// average with 128 channels and 1.1 % with 64, 31 and 19 % at most.  (A line at 60 tiles and t = 80 for 128 channels: 1.5 %, but up to 20 % slower than this one for some.)
bool short_batch(int rows_g, int t, int Hkv, int D, int batch)
{
    const long long tiles_cu = (long long)Hkv * batch * ((rows_g + 63) >> 6) * t / 256;
    return tiles_cu * D < 220 * 128 && !(t >= 90 && tiles_cu * D * t >= 13000ll * 128);
}

PlanB make_batch_plan(int M_max, int L_max, int Hq, int Hkv, int D, int batch, int eb)
{
    PlanB b = {};
    const int G = Hq / Hkv, rows_g = G * M_max, t = (L_max + M_max + TK - 1) / TK;
    if (short_batch(rows_g, t, Hkv, D, batch)) {
        b.rw = 2; b.wr_log2 = 6;
        b.row_blocks = (rows_g + 63) >> 6;
        const int base = Hkv * batch * b.row_blocks;
        // One request: as in the contiguous form.  More: parts of 32 tiles even out the lengths, or of 24 where the workgroups of the
        // whole requests are few (17 requests of up to 1.8k keys with 22 nodes 35.5 us in one part and 26.8 in two, 31 of up to 2.6k
        // with 49, D = 64, 32.6 in two and 27.7 in three; but 30 of up to 2k with 40 49 and 61).  Where that leaves the chip room (it
        // takes 512 of these workgroups at once, but two that share a CU take longer), parts of 4 tiles or more for a workgroup per
        // CU, of 8 or more for two of the longest request, of 16 or more for two rounds of those (2 requests of up to 2.4k with 26
        // nodes took 31 us in 2 parts and take 15 in 9; 7 of up to 1k with 8 13.8 in 3 and 12.0 in 4; 2 of up to 5.7k with 66 26.5
        // in 6 and 23.1 in 8), if a part is more than 10 tiles shorter than the whole: the partials and their merge cost as much
        // (6 of up to 463, D = 64, 9.4 in one and 8.4 in 4; 10 of up to 270 8.7 in one and 10.0 in 3).
        int want = batch == 1 ? std::min((rows_g <= 64 ? 512 : 256) / base, t / 8) : std::min(8, t / (base < 512 ? 24 : 32));
        if (batch > 1 && base < 256) {
            const int one = std::min(256 / base, (t + 3) / 4), two = std::min(512 / base, t / 8);
            const int by = std::min(32, std::max(2 * two >= 3 * one ? two : one, std::min(1024 / base, t / 16)));
            if (by > 1 && t - (t + by - 1) / by > 10) want = std::max(want, by);
        }
        b.sps = ((t + std::max(1, want) - 1) / std::max(1, want) + 1) & ~1;                // whole rounds of two tiles
        b.slots = (t + b.sps - 1) / b.sps;
        b.merge = b.slots > 1;
        return b;
    }
    b.rw = rows_g <= 64 && eb == 1 ? 2 : rows_g <= 128 || eb == 1 ? 4 : 8;
    b.wr_log2 = b.rw == 2 ? 6 : b.rw == 4 ? 7 : 8;
    b.row_blocks = (rows_g + (1 << b.wr_log2) - 1) >> b.wr_log2;
    b.pairing = b.row_blocks > 1;
    b.teams_log2 = (b.rw == 2 ? 9 : 8) - b.pairing;     // (one workgroup per CU, or two of the small ones)
    const long long stretches = (long long)Hkv * batch * ((b.row_blocks + b.pairing) >> b.pairing);
    b.slots = std::min(32, std::max(8, 4 + (int)((5 << b.teams_log2) / (b.pairing ? stretches : 2 * stretches))));
    b.wmin = std::max(2 * START, (t + b.slots - 5) / (b.slots - 4) * WHOLE);
    b.merge = t > SMALL;
    return b;
}

// The merge's words lie at the same place in every workspace of attention calls that hold partials: other calls leave them alone.
struct WsLayout { size_t sync, plan, ml, opart, total; };

WsLayout ws_layout(size_t rows, int D, int nsplit, int batch = 0)
{
    WsLayout w;
    size_t off = BTV_WS_HEADER;
    w.sync = off; off += batch || nsplit > 1 ? MERGE_GROUPS * sizeof(MergeWords) : 0;
    w.plan = off; off += batch ? btv_align_up((size_t)(batch + 2) * sizeof(long long), BTV_WS_ALIGN) : 0;
    size_t ns = nsplit > 1 ? nsplit : 0;
    w.ml = off; off += btv_align_up(ns * rows * 4 * 4, BTV_WS_ALIGN);
    w.opart = off; off += btv_align_up(ns * rows * D * 2, BTV_WS_ALIGN);
    w.total = off;
    return w;
}

// What the workspace queries of one request answer: enough for every call of up to M nodes over up to L keys.  The plan's own need
// is no answer to that: a shorter context or a smaller tree may be cut into more parts, or rows padded to larger blocks (32 nodes of an
// 8B shape: 8.8 MB at 32768 keys, 9.1 at 10208).  No plan of these sizes has more splits than there are tiles, nor than MOST_SPLITS, nor more than
// MOST_PARTIALS bytes in more than one split; partial_rows grows with M.  64 nodes over 8192 keys: 32.6 MB where that call's plan takes 8.6.
size_t enough_for(int M, int L, int Hq, int Hkv, int D, int eb, int force_split = 0, int force_shape = 0)
{
    size_t most = 0;
    const int n = std::min(force_split > 0 ? force_split : MOST_SPLITS, (L + M + TK - 1) / TK);
    for (int k = 1; k <= 3 && n > 1; ++k) {
        if (force_shape ? std::min(force_shape, eb == 1 ? 2 : 3) != k : eb == 1 && k == 3) continue;
        Plan pl = {};
        pl.wr = 32 << k;
        pl.row_blocks = (Hq / Hkv * M + pl.wr - 1) / pl.wr;
        const size_t part = partial_rows(pl, M, Hq, Hkv) * (D * 2 + 16);
        most = std::max(most, force_split > 0 ? n * part : std::min(n * part, MOST_PARTIALS));
    }
    // (the two arrays are aligned one by one)
    static_assert(MOST_PARTIALS + BTV_WS_HEADER + MERGE_GROUPS * sizeof(MergeWords) + 2 * BTV_WS_ALIGN <= SCRATCH_BYTES, "a plan's need fits the built-in array");
    return ws_layout(0, D, n).total + btv_align_up(most, BTV_WS_ALIGN) + (n > 1 ? BTV_WS_ALIGN : 0);
}

// The same for a batch: up to `batch` requests, M_max nodes, L_max keys.  Fewer or smaller requests are cut into more parts, so their
// partials may be the more.  Of make_batch_plan's forms: a short batch takes up to 8 parts of 24 tiles or more; where its grid is
// small, up to 32 parts of 4 tiles or more in no more than 256 workgroups of 64 rows, or of 8 tiles or more in no more than 1024
// (one request: 512 parts in 512); the others 8 parts, or 4 and their share of (5 << teams_log2) pieces, which is 640 row blocks, 1280
// where they go in pairs.  All of it grows with the sizes, and so does what makes a batch one of the others.  8 x 128 nodes over 16k
// keys 124.9 MB, which is that plan's own need.
size_t enough_for_batch(int batch, int M_max, int L_max, int Hq, int Hkv, int D, int eb)
{
    const int rows_g = Hq / Hkv * M_max, t = (L_max + M_max + TK - 1) / TK;
    const long long rows = (long long)batch * M_max * Hq, one = (long long)M_max * Hq;
    long long most = 0;
    if (t >= 48) most = rows * std::min(8, t / 24);
    if (t >= 12) most = std::max(most, std::min<long long>(rows * std::min(32, (t + 3) / 4), 256 * 64));
    if (t >= 16) most = std::max({ most, std::min<long long>(rows * std::min(32, t / 8), 1024 * 64), std::min<long long>(one * std::min(512, t / 8), 512 * 64) });
    if (!short_batch(rows_g, t, Hkv, D, batch)) {
        const long long spread = 640 * 128 * (rows_g <= 128 ? 1 : eb == 1 || rows_g <= 256 ? 2 : 4);
        most = std::max(most, std::min(rows * 32, std::max(rows * 8, rows * 4 + spread)));
    }
    return ws_layout(0, D, 1, batch).total + (most ? btv_align_up((size_t)most * (D * 2 + 16), BTV_WS_ALIGN) + BTV_WS_ALIGN : 0);
}

enum Form { ONE_REQUEST, ONE_MERGED, SHORT_BATCH, LONG_BATCH };

template <int D, int RW, int KW, int NT, Form FORM, int EB = 2>
int launch_bf16(const AttnParams &p, dim3 grid, hipStream_t st)
{
    constexpr int LDS_BYTES = PageLds<D, RW, KW, NT, (FORM > ONE_MERGED), EB>::BYTES + (FORM == LONG_BATCH ? CHUNK_BYTES : 0);
    static_assert(LDS_BYTES * (RW * KW <= 4 ? 2 : 1) <= 160 * 1024, "LDS budget");
    static std::atomic<bool> configured{false};         // (one GPU per process: the attribute is set once)
    void (*kern)(AttnParams);
    if constexpr (FORM == LONG_BATCH) kern = tv_attn_batch<D, RW, KW, NT, EB>;
    else if constexpr (FORM == SHORT_BATCH) kern = tv_attn_short<D, RW, KW, NT, EB>;
    else kern = tv_attn_bf16<D, RW, KW, NT, EB, FORM == ONE_MERGED>;
    if (!configured.load(std::memory_order_acquire)) {
        BTV_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    LDS_BYTES));
        configured.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, grid, dim3(RW * KW * 64), LDS_BYTES, st, p);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

template <Form FORM>
int dispatch_bf16(const AttnParams &p, int rw, int D, int eb, dim3 grid, hipStream_t st)
{
    if (eb == 1) {      // FP8 K/V
        if (D == 128 && rw == 2) return launch_bf16<128, 2, 2, 5, FORM, 1>(p, grid, st);
        if constexpr (FORM != SHORT_BATCH)
            if (D == 128 && rw == 4) return launch_bf16<128, 4, 2, 8, FORM, 1>(p, grid, st);
        return btv_fail(BTV_EINVAL, "no FP8-KV kernel for D=%d", D);
    }
#define BTV_CASE(DD, RR, KK, NN) \
    if (D == DD && rw == RR) return launch_bf16<DD, RR, KK, NN, FORM>(p, grid, st);
    if constexpr (FORM != LONG_BATCH) { BTV_CASE(128, 2, 2, 5) BTV_CASE(64, 2, 2, 5) }
    if constexpr (FORM != SHORT_BATCH) {
        BTV_CASE(128, 4, 2, 8) BTV_CASE(128, 8, 1, 8) BTV_CASE(64, 4, 2, 8) BTV_CASE(64, 8, 1, 8)
    }
#undef BTV_CASE
    return btv_fail(BTV_EINVAL, "no kernel for D=%d", D);
}

int check_shape(int M, int L, int Hq, int Hkv, int D)
{
    BTV_REQUIRE(M >= 1 && M <= BTV_MAX_NODES, "M=%d outside [1,%d]", M, BTV_MAX_NODES);
    BTV_REQUIRE(L >= 0 && (long long)L + M < (1ll << 30), "L=%d out of range", L);
    BTV_REQUIRE(Hq >= 1 && Hkv >= 1 && Hq % Hkv == 0 && Hq / Hkv <= 16, "bad heads Hq=%d Hkv=%d", Hq, Hkv);
    BTV_REQUIRE(D == 64 || D == 128, "D=%d not in {64,128}", D);
    return BTV_OK;
}

int check_fp8(int D, float k_scale, float v_scale)
{
    BTV_REQUIRE(D == 128, "FP8 K/V: D=%d, only 128 is built", D);
    BTV_REQUIRE(k_scale > 0.f && k_scale <= 3.0e38f && v_scale > 0.f && v_scale <= 3.0e38f,
                "FP8 K/V scales must be positive and finite");
    return BTV_OK;
}

bool aligned16(const void *a) { return (reinterpret_cast<uintptr_t>(a) & 15u) == 0; }

// eb = bytes per K/V element (2: the dtype's own; 1: E4M3 codes, bf16 Q and O).  The key scale multiplies every
// score, so it joins the softmax scale; the value scale multiplies the weighted sum, so it joins the final division.
void set_scales(AttnParams &p, int D, float scale, float k_scale, float v_scale)
{
    p.scale = (scale > 0.f ? scale : 1.0f / sqrtf((float)D)) * k_scale;
    p.scale_log2 = p.scale * 1.4426950408889634f;
    p.out_scale = v_scale;
}

int attn_contiguous(const void *Q, const void *K, const void *V, const int32_t *parent, int M, int L, int Hq, int Hkv,
                    int D, int dtype, int eb, float scale, float k_scale, float v_scale, void *O, void *ws,
                    size_t ws_bytes, void *stream, int force_split = 0, int force_shape = 0, uint32_t *flag_out = nullptr,
                    int merge = 0, int wait_ticks = MERGE_WAIT_TICKS)
{
    BTV_REQUIRE(Q && K && V && parent && O, "null pointer");
    BTV_REQUIRE(aligned16(Q) && aligned16(K) && aligned16(V) && aligned16(O), "Q, K, V and O must be 16-byte aligned");
    int rc = check_shape(M, L, Hq, Hkv, D);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Plan pl = make_plan(M, L, Hq, Hkv, D, eb, force_split, force_shape);
    if (dtype == BTV_F32) pl.nsplit = 1;
    WsLayout wl = ws_layout(partial_rows(pl, M, Hq, Hkv), D, pl.nsplit);
    rc = btv_check_ws(ws, ws_bytes, wl.total);
    if (rc) return rc;
    unsigned char *w8 = static_cast<unsigned char *>(ws);
    AttnParams p = {};
    p.Q = Q; p.K = K; p.V = V; p.O = O;
    p.ML = reinterpret_cast<float *>(w8 + wl.ml);
    p.Opart = reinterpret_cast<_Float16 *>(w8 + wl.opart);
    p.flag = flag_out ? flag_out : reinterpret_cast<uint32_t *>(w8);
    p.M = M; p.L = L; p.Hq = Hq; p.Hkv = Hkv; p.G = Hq / Hkv; p.ginv = (65536 + p.G - 1) / p.G;
    p.total_rows = M * Hq; p.total_M = M;
    p.sps = pl.sps; p.longer = pl.longer; p.nsplit = pl.nsplit; p.inv_nsplit = reciprocal(pl.nsplit);
    set_scales(p, D, scale, k_scale, v_scale);
    p.parent = parent;
    if (dtype == BTV_F32) {
        if (D == 64) hipLaunchKernelGGL(tv_attn_f32<64>, dim3(M, Hq), dim3(256), 0, st, p);
        else hipLaunchKernelGGL(tv_attn_f32<128>, dim3(M, Hq), dim3(256), 0, st, p);
        BTV_HIP(hipGetLastError());
        return BTV_OK;
    }
    p.row_blocks = pl.row_blocks; p.inv_row_blocks = reciprocal(pl.row_blocks);
    const bool inside = merge != 1 && merges_inside(pl, Hkv) && (merge || btv_usable_cus(st) >= 256);
    int wgs;
    if (inside) {
        p.sync = reinterpret_cast<unsigned long long *>(w8 + wl.sync);
        p.wait_ticks = wait_ticks;
        p.units = merge == 3 ? 0 : Hkv % 8 == 0 ? Hkv : Hkv * pl.row_blocks;
        wgs = merge == 3 ? (pl.nsplit * Hkv + 7) / 8 * 8 * pl.row_blocks : pl.nsplit * Hkv * pl.row_blocks;
    } else {
        p.units = pl.nsplit * Hkv;
        wgs = ((p.units + 7) / 8) * pl.row_blocks * 8;
    }
    rc = inside ? dispatch_bf16<ONE_MERGED>(p, pl.rw, D, eb, dim3(wgs), st) : dispatch_bf16<ONE_REQUEST>(p, pl.rw, D, eb, dim3(wgs), st);
    if (rc) return rc;
    if (pl.nsplit > 1 && !inside) {
        dim3 cg((M * Hq + 7) / 8, 1);
        if (D == 64) hipLaunchKernelGGL(tv_combine_bf16<64>, cg, dim3(256), 0, st, p);
        else hipLaunchKernelGGL(tv_combine_bf16<128>, cg, dim3(256), 0, st, p);
        BTV_HIP(hipGetLastError());
    }
    return BTV_OK;
}

int attn_paged(const void *Q, const void *Kpool, const void *Vpool, int num_blocks, const int32_t *block_table,
               int max_blocks, const int32_t *q_offset, const int32_t *prefix_len, const int32_t *parent, int batch,
               int total_M, int M_max, int L_max, int Hq, int Hkv, int D, int eb, float scale, float k_scale,
               float v_scale, void *O, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(Q && Kpool && Vpool && block_table && q_offset && prefix_len && parent && O, "null pointer");
    BTV_REQUIRE(aligned16(Q) && aligned16(Kpool) && aligned16(Vpool) && aligned16(O),
                "Q, K, V and O must be 16-byte aligned");
    BTV_REQUIRE(batch >= 1 && batch <= 4096, "batch=%d outside [1,4096]", batch);
    int rc = check_shape(M_max, L_max, Hq, Hkv, D);
    if (rc) return rc;
    BTV_REQUIRE(total_M >= 1 && total_M <= batch * M_max, "total_M=%d inconsistent with batch*M_max", total_M);
    BTV_REQUIRE(num_blocks >= 1 && max_blocks >= 1, "bad block counts");
    BTV_REQUIRE((long long)max_blocks * BTV_PAGE >= (long long)L_max + 1, "max_blocks too small for L_max");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const PlanB pl = make_batch_plan(M_max, L_max, Hq, Hkv, D, batch, eb);
    WsLayout wl = ws_layout((size_t)batch * M_max * Hq, D, pl.slots, batch);
    rc = btv_check_ws(ws, ws_bytes, wl.total);
    if (rc) return rc;
    unsigned char *w8 = static_cast<unsigned char *>(ws);
    AttnParams p = {};
    p.Q = Q; p.K = Kpool; p.V = Vpool; p.O = O;
    p.ML = reinterpret_cast<float *>(w8 + wl.ml);
    p.Opart = reinterpret_cast<_Float16 *>(w8 + wl.opart);
    p.flag = reinterpret_cast<uint32_t *>(w8);
    p.block_table = block_table; p.q_offset = q_offset; p.prefix_len = prefix_len;
    p.max_blocks = max_blocks; p.num_blocks = num_blocks;
    p.M = M_max; p.L = L_max; p.Hq = Hq; p.Hkv = Hkv; p.G = Hq / Hkv; p.ginv = (65536 + p.G - 1) / p.G;
    p.total_rows = batch * M_max * Hq;    // partial buffers are sized for the bound; rows index by q_offset
    p.total_M = total_M;
    p.plan = reinterpret_cast<long long *>(w8 + wl.plan);
    p.batch = batch; p.teams_log2 = pl.teams_log2; p.pairing = pl.pairing; p.wmin = pl.wmin; p.wr_log2 = pl.wr_log2;
    set_scales(p, D, scale, k_scale, v_scale);
    p.parent = parent;
    p.sps = pl.sps; p.row_blocks = pl.row_blocks; p.inv_row_blocks = reciprocal(pl.row_blocks);
    if (pl.sps) {
        p.nsplit = pl.slots; p.inv_nsplit = reciprocal(pl.slots); p.inv_sps = reciprocal(pl.sps); p.inv_Hkv = reciprocal(Hkv);
        p.units = pl.slots * Hkv * batch;
        rc = dispatch_bf16<SHORT_BATCH>(p, pl.rw, D, eb, dim3(((p.units + 7) / 8) * pl.row_blocks * 8), st);
    } else {
        rc = dispatch_bf16<LONG_BATCH>(p, pl.rw, D, eb, dim3(1 << (pl.teams_log2 + pl.pairing)), st);
    }
    if (rc || !pl.merge) return rc;
    const int rows = M_max * Hq;
    auto combine = [&](auto kern, int per) { hipLaunchKernelGGL(kern, dim3((rows + per - 1) / per, batch), dim3(256), 0, st, p); };
    const bool many = (long long)rows * batch > 12288;
    if (D == 64) many ? combine(tv_combine_batch<64, 8, 8>, 32) : combine(tv_combine_batch<64, 2, 16>, 8);
    else many ? combine(tv_combine_batch<128, 8, 8>, 16) : combine(tv_combine_batch<128, 4, 16>, 8);
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

}  // namespace

extern "C" {

int btv_tree_ancestor_mask(const int32_t *parent, int M, uint32_t *anc, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(parent && anc, "null pointer");
    BTV_REQUIRE(M >= 1 && M <= BTV_MAX_NODES, "M=%d outside [1,%d]", M, BTV_MAX_NODES);
    int rc = btv_check_ws(ws, ws_bytes, BTV_WS_HEADER);
    if (rc) return rc;
    hipLaunchKernelGGL(anc_mask_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), parent, M, anc, static_cast<uint32_t *>(ws));
    BTV_HIP(hipGetLastError());
    return BTV_OK;
}

size_t btv_tree_verify_attn_workspace(int M, int L, int Hq, int Hkv, int D, int dtype)
{
    if (check_shape(M, L, Hq, Hkv, D) != BTV_OK) return 0;
    return dtype == BTV_BF16 ? enough_for(M, L, Hq, Hkv, D, 2) : ws_layout(0, D, 1).total;
}

int btv_tree_verify_attn(const void *Q, const void *K, const void *V, const int32_t *parent, int M, int L, int Hq,
                         int Hkv, int D, int dtype, float scale, void *O, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(dtype == BTV_F32 || dtype == BTV_BF16, "dtype=%d unsupported", dtype);
    return attn_contiguous(Q, K, V, parent, M, L, Hq, Hkv, D, dtype, 2, scale, 1.0f, 1.0f, O, ws, ws_bytes, stream);
}

int btv_tree_verify_attn_noalloc(const void *Q, const void *K, const void *V, const int32_t *parent, int M, int L, int Hq,
                                 int Hkv, int D, int dtype, float scale, void *O, uint32_t *status, void *stream)
{
    BTV_REQUIRE(dtype == BTV_F32 || dtype == BTV_BF16, "dtype=%d unsupported", dtype);
    int rc = check_shape(M, L, Hq, Hkv, D);
    if (rc) return rc;
    void *ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    // the header (data flag, counters) must start at zero whatever an earlier call left behind
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint32_t *>(ws), (int)(BTV_WS_HEADER / 4));
    BTV_HIP(hipGetLastError());
    return attn_contiguous(Q, K, V, parent, M, L, Hq, Hkv, D, dtype, 2, scale, 1.0f, 1.0f, O, ws, SCRATCH_BYTES, stream, 0, 0,
                           status);
}

size_t btv_tree_verify_attn_fp8kv_workspace(int M, int L, int Hq, int Hkv, int D)
{
    if (check_shape(M, L, Hq, Hkv, D) != BTV_OK || D != 128) return 0;
    return enough_for(M, L, Hq, Hkv, D, 1);
}

int btv_tree_verify_attn_fp8kv(const void *Q, const void *K8, const void *V8, float k_scale, float v_scale,
                               const int32_t *parent, int M, int L, int Hq, int Hkv, int D, float scale, void *O,
                               void *ws, size_t ws_bytes, void *stream)
{
    int rc = check_fp8(D, k_scale, v_scale);
    if (rc) return rc;
    return attn_contiguous(Q, K8, V8, parent, M, L, Hq, Hkv, D, BTV_BF16, 1, scale, k_scale, v_scale, O, ws, ws_bytes,
                           stream);
}

size_t btv_tree_verify_attn_tuned_workspace(int M, int L, int Hq, int Hkv, int D, int kv_fp8, int nsplit, int shape)
{
    if (check_shape(M, L, Hq, Hkv, D) != BTV_OK || (kv_fp8 && D != 128) || nsplit < 0 || shape < 0 || shape > 3) return 0;
    return enough_for(M, L, Hq, Hkv, D, kv_fp8 ? 1 : 2, nsplit, shape);
}

int btv_tree_verify_attn_tuned(const void *Q, const void *K, const void *V, int kv_fp8, float k_scale, float v_scale,
                               const int32_t *parent, int M, int L, int Hq, int Hkv, int D, float scale, int nsplit,
                               int shape, void *O, void *ws, size_t ws_bytes, void *stream)
{
    return btv_tree_verify_attn_merge_tuned(Q, K, V, kv_fp8, k_scale, v_scale, parent, M, L, Hq, Hkv, D, scale, nsplit, shape, 0,
                                            MERGE_WAIT_TICKS, O, ws, ws_bytes, stream);
}

int btv_tree_verify_attn_merge_tuned(const void *Q, const void *K, const void *V, int kv_fp8, float k_scale, float v_scale,
                                     const int32_t *parent, int M, int L, int Hq, int Hkv, int D, float scale, int nsplit,
                                     int shape, int merge, int wait_ticks, void *O, void *ws, size_t ws_bytes, void *stream)
{
    BTV_REQUIRE(merge >= 0 && merge <= 3, "merge=%d outside [0,3]", merge);
    BTV_REQUIRE(nsplit >= 0 && shape >= 0 && shape <= 3, "nsplit=%d or shape=%d out of range", nsplit, shape);
    if (kv_fp8) {
        int rc = check_fp8(D, k_scale, v_scale);
        if (rc) return rc;
        BTV_REQUIRE(shape != 3, "shape 3 is not built for an FP8 cache");
    }
    return attn_contiguous(Q, K, V, parent, M, L, Hq, Hkv, D, BTV_BF16, kv_fp8 ? 1 : 2, scale, kv_fp8 ? k_scale : 1.0f,
                           kv_fp8 ? v_scale : 1.0f, O, ws, ws_bytes, stream, nsplit, shape, nullptr, merge, wait_ticks);
}

size_t btv_tree_verify_attn_paged_workspace(int batch, int M_max, int L_max, int Hq, int Hkv, int D)
{
    if (batch < 1 || batch > 4096 || check_shape(M_max, L_max, Hq, Hkv, D) != BTV_OK) return 0;
    return enough_for_batch(batch, M_max, L_max, Hq, Hkv, D, 2);
}

int btv_tree_verify_attn_paged(const void *Q, const void *Kpool, const void *Vpool, int num_blocks,
                               const int32_t *block_table, int max_blocks, const int32_t *q_offset,
                               const int32_t *prefix_len, const int32_t *parent, int batch, int total_M, int M_max,
                               int L_max, int Hq, int Hkv, int D, float scale, void *O, void *ws, size_t ws_bytes,
                               void *stream)
{
    return attn_paged(Q, Kpool, Vpool, num_blocks, block_table, max_blocks, q_offset, prefix_len, parent, batch, total_M,
                      M_max, L_max, Hq, Hkv, D, 2, scale, 1.0f, 1.0f, O, ws, ws_bytes, stream);
}

size_t btv_tree_verify_attn_paged_fp8kv_workspace(int batch, int M_max, int L_max, int Hq, int Hkv, int D)
{
    if (batch < 1 || batch > 4096 || check_shape(M_max, L_max, Hq, Hkv, D) != BTV_OK || D != 128) return 0;
    return enough_for_batch(batch, M_max, L_max, Hq, Hkv, D, 1);
}

int btv_tree_verify_attn_paged_fp8kv(const void *Q, const void *K8pool, const void *V8pool, float k_scale,
                                     float v_scale, int num_blocks, const int32_t *block_table, int max_blocks,
                                     const int32_t *q_offset, const int32_t *prefix_len, const int32_t *parent,
                                     int batch, int total_M, int M_max, int L_max, int Hq, int Hkv, int D, float scale,
                                     void *O, void *ws, size_t ws_bytes, void *stream)
{
    int rc = check_fp8(D, k_scale, v_scale);
    if (rc) return rc;
    return attn_paged(Q, K8pool, V8pool, num_blocks, block_table, max_blocks, q_offset, prefix_len, parent, batch,
                      total_M, M_max, L_max, Hq, Hkv, D, 1, scale, k_scale, v_scale, O, ws, ws_bytes, stream);
}

}  // extern "C"
