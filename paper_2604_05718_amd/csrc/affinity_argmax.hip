// Fused cosine affinity + self-masked row argmax (Eq. 1 and the nearest
// neighbour of Sec. 3.2) for gfx950.
//
// For image b with n tokens, every query i gets
//     nb[i] = argmax_{j != i, j < n} (x_i . x_j) * inv_j,   inv_j = 1 / max(||x_j||, 1e-12),
// with the lowest j kept among equal scores. Dividing the dot product by
// ||x_i|| as well would not move a row's argmax, so only the candidate norm is
// applied. The dot products come from MFMA on the stored values (bfloat16
// products are exact in float32, accumulation is float32); normalising first
// and rounding the unit vectors back to bfloat16 would cost about three
// decimal digits of the cosine, so the inputs are never rescaled.
//
// Tiling. A work item is a block of QT queries against a tile of CT candidates
// of one image; the N x N affinity only ever lives in MFMA accumulators. The K
// dimension (D) of both is staged through LDS in 128-byte chunks,
// double-buffered: the global loads of the next chunk are in flight while the
// current one feeds the MFMAs.
// In the 32x32 MFMA the candidate is the row operand and the query the column
// operand, so each lane's 16 accumulator values belong to ONE query and 16
// different candidates: the running (max, index) reduction is per lane, in
// registers, in ascending candidate order, and lanes/waves are merged
// lexicographically (larger score, then smaller index) only once at the end.
// The norms are summed from the same LDS rows that feed the MFMAs, so X is read
// once per tile and no separate normalisation pass exists.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/mpm.h"
#include "mpm_device.h"
#include "mpm_launch.h"
#include "mpm_work.h"

namespace mpm {
namespace {

template <class S>
struct Mfma;

template <>
struct Mfma<Bf16> {
    // 16 bytes per lane = 8 bfloat16 values along k: one 32x32x16 MFMA.
    static __device__ __forceinline__ void mma(f32x16& acc, u32x4 a, u32x4 b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                      __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
    // Sum of squares of the 8 values, accumulated into s: one v_dot2c_f32_bf16 per pair
    // (both squares and the running sum in one instruction, a quarter of the vector ALU
    // work of unpacking and two FMAs; its relative error on 768-value rows is at most
    // 1.6e-6 against float64, below the FMA chain's 3.5e-6). The words are copied to
    // scalars first: a bit cast of a subscripted element a[e] of the 4-word vector
    // compiled to four reads of its first word, and a cast of the whole fragment to 8
    // values cost 15-20 more VGPRs in the persistent kernels.
    static __device__ __forceinline__ float sumsq(u32x4 a, float s)
    {
        const uint32_t w0 = a.x, w1 = a.y, w2 = a.z, w3 = a.w;
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w0), __builtin_bit_cast(bf16x2, w0), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w1), __builtin_bit_cast(bf16x2, w1), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w2), __builtin_bit_cast(bf16x2, w2), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w3), __builtin_bit_cast(bf16x2, w3), s, false);
        return s;
    }
};

template <>
struct Mfma<F32> {
    // 16 bytes per lane = 4 float32 values along k: four 32x32x2 MFMAs. Lane l
    // feeds k-slot l/32 of the instruction; both operands use the same
    // lane -> k assignment, so the sum runs over all 8 k of the 32-byte group.
    static __device__ __forceinline__ void mma(f32x16& acc, u32x4 a, u32x4 b)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]),
                                                       acc, 0, 0, 0);
    }
    static __device__ __forceinline__ float sumsq(u32x4 a, float s)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) s = fmaf(__uint_as_float(a[e]), __uint_as_float(a[e]), s);
        return s;
    }
};

constexpr int kChunkBytes = 128;  // bytes of each row per LDS stage
constexpr int kSplitRows = 256;   // block rows of the symmetric schedule that has a half-block launch
// Fewest bfloat16 chunks of K from which a batch of single-block images with two slots for each
// runs as half blocks only (float32 blocks: any): half of a round has to outweigh the second
// launch. Images of more blocks would run their other blocks in the first launch and the halves
// after them. Neighbour queries of 1 to 128 images of at most 256 rows, whole / half blocks:
// bfloat16 rows of 768 bytes 15.7 / 13.9 us, of 2048 bytes 27.8 / 19.7, float32 rows of 3072
// bytes 181 / 96; bfloat16 rows of 128 and 384 bytes are 8 to 20% and 9% faster whole.
constexpr int kLoneSplitChunks = 6;
template <class S>
__host__ __device__ constexpr bool splits_lone(int nchunks, int blocks)  // of an image
{
    return blocks == 1 && (S::kBytes == 4 || nchunks >= kLoneSplitChunks);
}
constexpr int kXcds = 8;  // MI355X: workgroups are dealt round-robin to 8 XCDs, each with its own L2

// Workgroup barrier that waits only for this wave's LDS operations (not for
// outstanding global loads, which keep streaming into other LDS buffers).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt unconstrained
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The locality constraint of Sec. 5 (candidates restricted to a window on the token
// grid): a token's position is a raster index on a grid of grid_w columns (pos packed
// like x; null: the token's index in its image); j is a candidate of i when both lie
// within radius rows and columns of each other. Positions are non-decreasing in row
// along an image (raster order, which the left-to-right ids keep for merged tokens).
struct Window {
    const int32_t* pos;
    FixedDiv grid_w;  // row of a position: grid_w(pos)
    int radius;
};

// Lane exchanges for the reverse-direction argmax of the symmetric schedule.
// Each DPP pattern used is an involution on the lanes of a 16-lane row.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int32_t dpp_i(int32_t x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
// x + the value of the lane 32 away.
__device__ __forceinline__ float half_sum(float x)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// The larger values (of finite or infinite ones; a NaN loses).
__device__ __forceinline__ float max_of(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max_of(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// (v, i) = the lexicographic maximum of (av, ai) and (bv, bi): larger score, then
// smaller index (as unsigned, so -1 loses every tie). Branch-free.
__device__ __forceinline__ void merge_pair(float& v, int32_t& i, float av, int32_t ai, float bv, int32_t bi)
{
    const bool c = (bv > av) | ((bv == av) & ((uint32_t)bi < (uint32_t)ai));
    v = c ? bv : av;
    i = c ? bi : ai;
}
// One reduce-scatter step over the H slot pairs (k, k+H): the partner lane (DPP
// pattern CTRL) keeps the other half. Lanes with `upper` keep slots k+H, the others
// slots k; each kept slot is merged with the partner's copy of it into slot k.
template <int CTRL, int H>
__device__ __forceinline__ void exchange_half(float* v, int32_t* ix, int upper)
{
#pragma unroll
    for (int k = 0; k < H; ++k) {
        const float kv = upper ? v[k + H] : v[k];
        const int32_t ki = upper ? ix[k + H] : ix[k];
        const float sv = upper ? v[k] : v[k + H];
        const int32_t si = upper ? ix[k] : ix[k + H];
        merge_pair(v[k], ix[k], kv, ki, dpp_f<CTRL>(sv), dpp_i<CTRL>(si));
    }
}

// Persistent kernel for rows (bfloat16 or float32) of any whole number of 16-byte
// pieces; everything below is laid out in bytes, and Mfma<S> consumes the same 16-byte
// fragments for either type. Work item = (image, query block of QT, candidate tile of
// CT); an item streams its two operand blocks in 128-byte chunks of the rows through
// two LDS stages filled by direct global->LDS loads (global_load_lds_dwordx4), runs the
// K loop on MFMA, then reduces its tile to one (score, index) partial per query.
//
// Scheduling for the 8 per-XCD L2 caches: workgroups are dealt round-robin to the XCDs,
// so workgroup w serves XCD group w % xcds, and each group takes a contiguous share of the
// batch's items (mpm_work.h). The items of an image run at the same time on one XCD, in
// lockstep over K, and each block of rows is fetched from HBM once and re-read from that
// XCD's L2 by the other items that use it, instead of being refetched once per candidate
// tile. Packed images are counted by their own lengths: the workgroup tabulates the block
// counts of up to kMaxCountedImages images first (one image a thread: by one wave, 64 images
// at a time, 402 images took 5 us of a launch of 17).
//
// Pipeline. The chunks of all the workgroup's items form one stream. The barrier before
// chunk c makes chunk c visible and retires chunk c-1's stage; chunk c's first fragments
// are requested, then chunk c+1's loads into the retired stage, so loads run one chunk
// ahead. Within a chunk the MFMA fragments are double-buffered: the fragments of the next
// k-group are requested before the current k-group's MFMAs issue, so LDS latency hides
// behind the matrix cores. Each load instruction reads whole 128-byte lines; 64-byte
// chunks in four stages had twice the barriers and half the load rate (95.5 against 85.6
// us on 64 images of 1024 rows of 1536 bytes).
// The global->LDS loads are written as assembly: the compiler cannot tell which
// ring slot they fill and would otherwise wait for all of them before every LDS
// read; their completion is waited for explicitly (vmcnt) instead.
//
// TAIL: rows that are no whole number of chunks. A row's last chunk is loaded with its
// columns past the row's end clamped to the row's last 16 bytes (in bounds for the last
// row of x too), and each lane overwrites the pieces it loaded there with zeros in LDS
// before the barrier that makes the chunk visible, so the chunk loop itself is the same.
// Zero pieces add nothing to the products or norms: the scores are bit-identical to a
// K loop that ends with the row. Of a last chunk that ends in its first half only that half is
// computed, which a uniform branch a chunk decides: computed whole, 64-byte float32 rows, half
// of a chunk, took 1.3 times as long (1903 images of 400: 288 us). 24
// packed images of 346 to 990 rows of 400 bytes: 20 us, against 59 us for a kernel that
// staged such rows through registers, one workgroup per query block.
//
// LDS layout of one stage: CB = 128 bytes of K per row, rows of an operand stored one
// after the other, with the 16-byte columns of a row permuted by an XOR swizzle: column c
// of row r sits in slot c ^ swz(r), swz(r) = ((r % 8) / 2) | (((r / 8) % 2) << 2).
// One load instruction fills 1 KB = 1024/CB consecutive rows: lane l reads 16
// bytes of row l / (CB/16) (the lanes of a row cover its CB contiguous bytes of
// global memory) and lands at 16*l. An MFMA fragment read (one 16-byte column
// of 32 consecutive rows per lane half) then touches 16 distinct 16-byte bank
// groups in every 16-lane group, so it is free of bank conflicts on the
// 64-bank LDS. Load groups are dealt to the waves round-robin.
// Rows past the image are clamped to its last row (their scores are masked).
//
// Symmetric schedule (SYM). S = X X^T of an image is symmetric (Eq. 1), so only
// the blocks with query block <= candidate tile are computed: nb(nb+1)/2 items
// per image instead of nb^2. An off-diagonal item also yields the reverse
// direction: each candidate row j of the tile gets its best query q of the block,
// scored (x_j . x_q) * inv_q from the same accumulators, and writes the partial of
// row j for tile slot "query block". Every (row, slot) partial is still written
// exactly once, so the reduction over slots is unchanged. The products and sums
// are the same as in the item that would compute block (j's tile, q's block)
// directly, so the partials are bit-identical to the full schedule's. Items are
// taken image by image, the blocks of an image row by row, so all the items of
// an image still run together on one XCD and share its L2.
//
// HALVES: the second launch of a symmetric schedule on 256-row blocks. The first
// launch (SYM) leaves out the last diagonal blocks of its XCD group's share, as many as its
// last round would hold on at most half of the slots (work_share()), so that its slots
// take whole rounds; this launch runs each deferred block as two items of the block's
// 256 candidates and one half of its queries (QT = CT/2). A diagonal block needs no
// reverse direction, so the two halves write disjoint query partials, and each score
// comes from the same MFMA sequence as in a whole block.
//
// LOCAL: the locality constraint of Sec. 5, on the symmetric schedule. A work item is a query
// block with the candidate tiles its window band reaches from its own on ([tlo, thi] is the
// whole band, found from the positions at the block and tile boundaries); the item runs them
// one after the other through the same ring (one K loop per tile), keeps each query's running
// best across them in registers, sets scores outside the window to -inf, and writes one partial
// per query (the block's own tile slot) beside the reverse direction's of each tile; the slots
// no item writes for the block's rows hold -inf. Positions (win.pos, null: the token's index)
// are fetched per tile while its K loop runs, as given norms are.
//
// GIVEN (bfloat16 rows only): xinv holds the inverse row norms 1 / max(||x_j||, 1e-12),
// one float per row packed like x, which the kernel then takes instead of summing them
// from the fragments in the K loop (vector ALU work in the K loop adds to its time about
// one for one). Otherwise xinv is unused and every k-group's norm sums run without a
// branch; each case is its own build.
template <class S, int WC, int WQ, int MT, int NT, bool SYM, bool HALVES, bool LOCAL, bool GIVEN, bool TAIL,
          bool COUNTED>
__global__ __launch_bounds__(WC * WQ * kWave, 2) void affinity_partial_kernel(  // 2 waves per SIMD
    const uint8_t* __restrict__ x, const int32_t* __restrict__ x_off, int B, int N, int D, int T, int log_xcds,
    int slots, WorkShape shape, float* __restrict__ pv, int32_t* __restrict__ pi, const float* __restrict__ xinv, Window win,
    Clear clear)
{
    constexpr int THREADS = WC * WQ * kWave;
    constexpr int WAVES = WC * WQ;
    constexpr int CT = WC * MT * 32;
    constexpr int QT = WQ * NT * 32;
    constexpr int CB = kChunkBytes;
    constexpr int NS = CB / 16;                       // 16-byte slots per row
    constexpr int RPI = 64 / NS;                      // rows per load instruction (1 KB)
    // Rows a stage holds: the candidate tile, then the query block (none for a half item,
    // whose queries are rows of its own candidate tile).
    constexpr int QROWS = HALVES ? 0 : QT;
    constexpr int GROUPS = (CT + QROWS) / RPI;        // load instructions per stage
    constexpr int LOADS = GROUPS / WAVES;             // ... per wave
    constexpr int STAGE_BYTES = (CT + QROWS) * CB;
    constexpr int KG = CB / 32;                       // 32-byte k-groups (one MFMA k-step each) per chunk
    static_assert(GROUPS % WAVES == 0 && CT % RPI == 0 && CT % 32 == 0 && QT % 32 == 0, "stage/wave mismatch");
    static_assert(KG % 2 == 0, "the fragment double buffer alternates over an even number of k-groups");

    __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * STAGE_BYTES];
    __shared__ __attribute__((aligned(16))) float inv_all[CT + (SYM ? QT : 0)];  // of the candidates, then the queries
    float* const inv_c = inv_all;
    float* const inv_q = inv_all + (SYM ? CT : 0);
    __shared__ float red_v[WC][QT];
    __shared__ int32_t red_i[WC][QT];
    __shared__ float red_cv[SYM ? WQ : 1][SYM ? CT : 1];
    __shared__ int32_t red_ci[SYM ? WQ : 1][SYM ? CT : 1];
    // LOCAL: grid row [0] and column [1] of the item's candidates (0 .. CT-1) and queries (CT ..).
    __shared__ __attribute__((aligned(16))) int32_t win_rc[2][LOCAL ? CT + QT : 1];
    __shared__ int32_t win_pos[LOCAL ? CT + QT : 1];  // ... their positions as given
    static_assert(!LOCAL || (SYM && !HALVES && QT == CT && CT + QT <= WC * WQ * kWave),
                  "window items: symmetric, square blocks, one position per thread");
    static_assert(!SYM || QT == CT, "the symmetric schedule pairs equal blocks");
    static_assert(!GIVEN || S::kBytes == 2, "given norms: bfloat16 rows");
    constexpr bool given = GIVEN;

    const int tid = threadIdx.x;
    // The words the compaction counts in start at zero, whatever the workspace held.
    if (!HALVES && blockIdx.x == 0)
        for (int k = tid; k < clear.words; k += THREADS) clear.p[k] = 0;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform: scalar registers and branches
    const int wc = wave % WC;
    const int wq = wave / WC;
    const int lrow = lane & 31;
    const int khalf = lane >> 5;

    static_assert(!HALVES || (!SYM && 2 * QT == CT), "half items: forward only, half a block of queries");
    static_assert(HALVES || QT == CT, "square blocks");
    constexpr bool SPLIT = SYM && !LOCAL && CT == kSplitRows;  // the blocks the second launch exists for
    constexpr WorkOrder ORDER = LOCAL ? kOrderBand : (SYM || HALVES) ? kOrderSymmetric : kOrderFull;
    __shared__ int32_t items_tab[COUNTED ? kMaxCountedImages + 1 : 1], diags_tab[COUNTED ? kMaxCountedImages + 1 : 1];
    const WorkCounts<COUNTED> counts{shape, items_tab, diags_tab};
    if constexpr (COUNTED) {
        // One image a thread: inclusive sums over the wave, then over the waves before it.
        __shared__ int32_t part[2][WAVES];
        int items = 0, diags = 0;  // of the images of earlier passes
        for (int b0 = 0; b0 < B; b0 += THREADS) {
            const int b = b0 + tid;
            const int im = work_place(b, shape.run);
            const int nb = b < B ? (x_off[im + 1] - x_off[im] + CT - 1) / CT : 0;
            int si = work_items(ORDER, nb), sd = nb;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int yi = __shfl_up(si, o), yd = __shfl_up(sd, o);
                si += lane >= o ? yi : 0;
                sd += lane >= o ? yd : 0;
            }
            if (b0 > 0) __syncthreads();  // the last pass's sums are read
            if (lane == kWave - 1) {
                part[0][wave] = si;
                part[1][wave] = sd;
            }
            __syncthreads();
            int pi0 = items, pd0 = diags;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const int ci = part[0][w], cd = part[1][w];
                pi0 += w < wave ? ci : 0;
                pd0 += w < wave ? cd : 0;
                items += ci;
                diags += cd;
            }
            if (b < B) {
                items_tab[b + 1] = pi0 + si;
                diags_tab[b + 1] = pd0 + sd;
            }
        }
        if (tid == 0) items_tab[0] = diags_tab[0] = 0;
        __syncthreads();
    }
    const int group = blockIdx.x & ((1 << log_xcds) - 1);
    const int slot = blockIdx.x >> log_xcds;
    const long rowbytes = (long)D * S::kBytes;
    const int nchunks = (int)((rowbytes + CB - 1) / CB);
    const WorkShare share =
        work_share(counts, B, group, log_xcds, slots, SPLIT || HALVES, !COUNTED && splits_lone<S>(nchunks, (int)shape.nb.d));
    const int nitems = HALVES ? 2 * share.ndef : share.cnt - share.ndef;
    if (slot >= nitems) return;  // uniform over the workgroup

    // Item cursor; all fields are uniform over the workgroup.
    struct Item {
        int k, b, place, qbase, cbase, n, row0;
        int tlo, thi;  // LOCAL: the item's band of candidate tiles (cbase walks up to thi)
    };
    auto find = [&](int k, int from) {
        Item it;
        for (; k < nitems; k += slots) {
            const WorkBlock w = HALVES ? work_deferred(counts, B, share, k >> 1) : work_block<ORDER, SPLIT>(counts, share, k, from);
            const int b = work_place(w.b, shape.run), t = w.t;
            const int qbase = HALVES ? w.q * CT + (k & 1) * QT : w.q * QT;  // half item: query half k % 2
            const int row0 = x_off ? x_off[b] : b * N;
            const int n = x_off ? x_off[b + 1] - row0 : N;
            if (qbase < n && t * CT < n) {
                it.k = k; it.b = b; it.place = w.b; it.qbase = qbase; it.cbase = t * CT; it.n = n; it.row0 = row0;
                it.tlo = t;
                it.thi = t;
                if constexpr (LOCAL) {
                    // Candidate tiles whose grid rows can meet the block's window rows.
                    auto grid_row = [&](int i) { return win.grid_w(win.pos ? win.pos[row0 + i] : i); };
                    const int r_first = grid_row(qbase), r_last = grid_row(min(qbase + QT, n) - 1);
                    int tlo = 0, thi = (n - 1) / CT;
                    while (tlo < thi && grid_row(min((tlo + 1) * CT, n) - 1) < r_first - win.radius) ++tlo;
                    while (thi > tlo && grid_row(thi * CT) > r_last + win.radius) --thi;
                    // The symmetric schedule starts at the block's own tile: the tiles before
                    // it reach this block through their own items' reverse direction.
                    it.cbase = t * CT;
                    it.tlo = tlo;
                    it.thi = thi;
                }
                return it;
            }
            if constexpr (!COUNTED && !HALVES) {
                // An item past its image's end, in a batch whose images are not counted: the
                // slot's next item inside its image, 64 of them at a time. One after the other
                // took half a microsecond each: 1380 images of up to 3487 rows, a twentieth of
                // them filled, 566 items a slot.
                int k0 = k + slots;
                for (; k0 < nitems; k0 += kWave * slots) {
                    const int kl = k0 + lane * slots;
                    bool inside = false;
                    if (kl < nitems) {
                        const WorkBlock v = work_block<ORDER, SPLIT>(counts, share, kl, 0);
                        const int bv = work_place(v.b, shape.run);
                        const int nv = x_off[bv + 1] - x_off[bv];  // with offsets: dense items are never past the end
                        inside = v.q * QT < nv && v.t * CT < nv;
                    }
                    const uint64_t found = __ballot(inside);
                    if (found != 0) {
                        k0 += (int)__builtin_ctzll(found) * slots;
                        break;
                    }
                }
                k = k0 - slots;
            }
        }
        it.k = nitems; it.b = 0; it.place = 0; it.qbase = 0; it.cbase = 0; it.n = 1; it.row0 = 0; it.tlo = 0; it.thi = 0;
        return it;
    };
    // The work after `it`: its next band tile (LOCAL), else the slot's next item.
    auto next_of = [&](const Item& it) {
        if constexpr (LOCAL) {
            if (it.cbase < it.thi * CT) {
                Item nx = it;
                nx.cbase += CT;
                return nx;
            }
        }
        return find(it.k + slots, it.place);
    };

    // Swizzle of the 16-byte column slot for a row (see the layout note above).
    auto swz = [](int r) { return ((r & 7) >> 1) | (((r >> 3) & 1) << 2); };
    const int lrowi = lane / NS;                          // row inside a load group
    const int lslot = lane % NS;                          // column slot this lane fills
    // The byte column of a chunk this lane loads: the swizzle of its rows is the same in every
    // load group of a wave (groups of a wave are a whole number of 16-row periods apart).
    static_assert(RPI * WAVES % 16 == 0 && CT % 16 == 0, "one column per lane");
    const int lcol = (lslot ^ swz((wave * RPI + lrowi) & 15)) << 4;
    // Load group u = wave + WAVES * i covers rows u*RPI .. u*RPI+RPI-1 of [cand; query].
    // Byte offsets (from the image's first row) of this lane's 16-byte pieces for
    // the issue cursor's item; they change per item, not per chunk.
    struct Offsets {
        uint32_t v[LOADS];
    };
    auto offsets_of = [&](const Item& it) {
        Offsets o;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int u = wave + WAVES * i;
            const bool is_q = u * RPI >= CT;
            const int r = u * RPI - (is_q ? CT : 0) + lrowi;   // row inside its operand block
            int row = (is_q ? it.qbase : it.cbase) + r;
            row = row < it.n ? row : it.n - 1;
            o.v[i] = (uint32_t)row * (uint32_t)rowbytes + (uint32_t)lcol;
        }
        return o;
    };

    Item ii = find(slot, work_image(counts, B, share.lo));  // issue cursor
    Item inext = ii;  // the item of the chunk issued last
    if (ii.k >= nitems) return;  // no work for this slot (uniform over the workgroup)
    Offsets ioff = offsets_of(ii);
    int ichunk = 0;
    int issued = 0;
    // The loads of a chunk are issued one at a time between the MFMAs of the chunk before
    // (issue_part, from mma_issue). Issued together after the barrier, a chunk's loads filled
    // the load queue and the wave stalled at issue with its MFMAs waiting behind them.
    uint8_t* isb = lds;
    const uint8_t* ibase = x;
    bool iact = false;
    uint32_t iback = 0;  // TAIL: how far this lane's column lies past its row's last 16 bytes
    auto issue_begin = [&]() {
        iact = ii.k < nitems;
        isb = lds + (issued & 1) * STAGE_BYTES;
        if constexpr (TAIL) iback = (uint32_t)max(0, ichunk * CB + lcol - (int)(rowbytes - 16));
        ibase = x + (long)ii.row0 * rowbytes + (long)ichunk * CB;   // uniform
    };
    // Once the issue cursor is past its last item the loads go on, unconditionally (no branch
    // per load in the K loop): they re-read rows of the last item (valid addresses) into the
    // ring slot after the last chunk, which nothing reads any more.
    auto issue_part = [&](int i) {
        const uint32_t off = TAIL ? ioff.v[i] - iback : ioff.v[i];
        const uint32_t m0 =
            (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)(isb + (wave + WAVES * i) * RPI * CB);
        // The LDS destination goes in M0, which the instruction reads implicitly: an input
        // operand bound to M0, so the compiler sets it and knows the asm reads it.
        asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(ibase), "{m0}"(m0) : "memory");
    };
    // The issue cursor's next item, once its chunks are all requested: before the next chunk's
    // loads, or, for window items, behind the last loads (their next tile is found in a few
    // instructions; before the loads it delayed every one of a lone workgroup's, 2538 images of
    // 24 rows of 2048 bytes 103 us against 97. Found behind the loads, the next item of 128 x 128
    // dense blocks cost 5%: 32 images of 900 rows of 1536 bytes 42.2 us against 40.3).
    auto advance = [&]() {
        if (ichunk < nchunks) return;
        ichunk = 0;
        ii = next_of(ii);
        if (ii.k < nitems) ioff = offsets_of(ii);
    };
    auto issue_end = [&]() {
        inext = ii;
        if (!iact) return;
        ++issued;
        ++ichunk;
        if constexpr (LOCAL) advance();
    };
    auto issue_next = [&]() {
        issue_begin();
#pragma unroll
        for (int i = 0; i < LOADS; ++i) issue_part(i);
        issue_end();
    };

    // Row lrow of every 32-row fragment has the same swizzle (32 is a multiple of 16).
    const int sw = swz(lrow & 15);
    const int lc_off = (wc * MT * 32 + lrow) * CB;
    // A half item's queries are rows qbase - cbase.. of its candidate tile. Its first value
    // comes from the issue cursor's first item, which is the compute cursor's first item; a
    // slot runs at most one half item (2 * ndef <= slots).
    int lq_off = (HALVES ? ii.qbase - ii.cbase : CT) * CB + (wq * NT * 32 + lrow) * CB;
    u32x4 fa0[MT], fq0[NT], fa1[MT], fq1[NT];
    auto read_frags = [&](u32x4 (&fa)[MT], u32x4 (&fq)[NT], int chunk, int g) {
        const uint8_t* sb = lds + (chunk & 1) * STAGE_BYTES;
        const int col = ((2 * g + khalf) ^ sw) << 4;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) fa[mt] = *reinterpret_cast<const u32x4*>(sb + lc_off + mt * 32 * CB + col);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) fq[nt] = *reinterpret_cast<const u32x4*>(sb + lq_off + nt * 32 * CB + col);
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x16{};
    // Norm sums (rows not given): wave (wc, wq) sums candidate m-tiles wq, wq + WQ, ... and,
    // in the symmetric schedule, query n-tiles wc, wc + WC, ... It reads those fragments from
    // LDS a second time, before each k-group's MFMAs (own_c / own_q: their offsets in a stage,
    // before the k column), and sums them after the MFMAs. Picking them out of its registers
    // by wave index instead took a branch per tile in the K loop, which cost 5-8% of the
    // launch. An index past the wave's tiles reads its last tile, whose sum is unused.
    constexpr int NSC = (MT + WQ - 1) / WQ;
    constexpr int NSQ = SYM ? (NT + WC - 1) / WC : 1;
    float ss[NSC], sq[NSQ];
    int own_c[NSC], own_q[NSQ];
#pragma unroll
    for (int j = 0; j < NSC; ++j) {
        ss[j] = 0.0f;
        own_c[j] = lc_off + min(wq + j * WQ, MT - 1) * 32 * CB;
    }
#pragma unroll
    for (int j = 0; j < NSQ; ++j) {
        sq[j] = 0.0f;
        own_q[j] = min(wc + j * WC, NT - 1) * 32 * CB;  // from lq_off
    }
    // TAIL: whether the last chunk of a row ends in its first half.
    // (Large window blocks of bfloat16 rows have no registers left for the branch, and in a chunk
    // of small blocks it costs more than half a chunk of them saves: 4 images of 2 rows of 3312
    // bytes 15.4 us with it, 14.4 without.)
    constexpr bool CUT = TAIL && (S::kBytes == 4 || (MT * NT > 1 && !(LOCAL && MT * NT >= 8)));
    const bool half_tail = CUT && rowbytes - (long)(nchunks - 1) * CB <= CB / 2;
    // One load part before every PSTEP-th MFMA of a chunk, over the first half of its MFMAs (the
    // loads must land before the chunk ends).
    constexpr int PGROUPS = KG * MT * NT;  // MFMAs per chunk
    constexpr int PSPAN = PGROUPS / 2;
    static_assert(PSPAN >= 1, "load parts per MFMA");
    constexpr int PSTEP = PSPAN >= LOADS ? PSPAN / LOADS : 1;              // MFMAs between load slots
    constexpr int PPER = PSPAN >= LOADS ? 1 : (LOADS + PSPAN - 1) / PSPAN;  // loads per slot (small tiles)
    static_assert((LOADS - 1) / PPER * PSTEP < PSPAN, "every load in the first half");
    auto mma_issue = [&](const u32x4 (&fa)[MT], const u32x4 (&fq)[NT], int chunk, int g) {
        u32x4 oc[NSC], oq[NSQ];
        if constexpr (!given) {
            const uint8_t* sb = lds + (chunk & 1) * STAGE_BYTES;
            const int col = ((2 * g + khalf) ^ sw) << 4;
#pragma unroll
            for (int j = 0; j < NSC; ++j) oc[j] = *reinterpret_cast<const u32x4*>(sb + own_c[j] + col);
            if constexpr (SYM) {
#pragma unroll
                for (int j = 0; j < NSQ; ++j) oq[j] = *reinterpret_cast<const u32x4*>(sb + lq_off + own_q[j] + col);
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int p = (g * MT + mt) * NT + nt;
                if (p % PSTEP == 0) {
#pragma unroll
                    for (int q = 0; q < PPER; ++q)
                        if ((p / PSTEP) * PPER + q < LOADS) issue_part((p / PSTEP) * PPER + q);
                }
                Mfma<S>::mma(acc[mt][nt], fa[mt], fq[nt]);
            }
        }
        if constexpr (!given) {
#pragma unroll
            for (int j = 0; j < NSC; ++j) ss[j] = Mfma<S>::sumsq(oc[j], ss[j]);
            if constexpr (SYM) {
#pragma unroll
                for (int j = 0; j < NSQ; ++j) sq[j] = Mfma<S>::sumsq(oq[j], sq[j]);
            }
        }
    };
    Item ci = ii;  // compute cursor
    issue_next();  // prologue: the first chunk
    // Values of the compute cursor's rows (one per candidate row, then one per query row) that
    // its epilogue reads, loaded straight to LDS once the first chunk's barrier has retired
    // them there: given inverse norms, given grid positions (LOCAL). They land before the next
    // chunk's barrier, behind that chunk's MFMAs; loaded to a register before the chunk's own
    // wait, they held every item up for their latency.
    constexpr int VALUES = CT + (SYM ? QT : 0);
    static_assert(VALUES % kWave == 0 && VALUES <= THREADS, "one value per thread at most");
    auto fetch_rows = [&](const Item& it, const void* values, void* to) {
        if (wave * kWave >= VALUES) return;  // uniform
        const int r = min(tid < CT ? it.cbase + tid : it.qbase + tid - CT, it.n - 1);
        const uint8_t* base = static_cast<const uint8_t*>(values) + 4L * it.row0;  // uniform
        const uint32_t m0 =
            (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)(static_cast<uint8_t*>(to) + wave * kWave * 4);
        asm volatile("global_load_lds_dword %0, %1" ::"v"(4 * r), "s"(base), "{m0}"(m0) : "memory");
    };
    auto fetch_item = [&](const Item& it) {
        if constexpr (given) fetch_rows(it, xinv, inv_all);
        if constexpr (LOCAL)
            if (win.pos) fetch_rows(it, win.pos, win_pos);
    };
    // The partials of an item are merged over the waves and stored at the next item's first
    // chunk (after the loop for the last one): the chunk's barrier makes the waves' shares
    // visible, so the epilogue has no barrier of its own for them, and the stores complete
    // behind that chunk's MFMAs instead of ahead of its wait.
    bool pend_fwd = false, pend_rev = false;
    Item done = ci;
    auto flush = [&]() {
        const int n = done.n;
        if (pend_fwd && tid < QT && done.qbase + tid < n) {
            // The query block's partial: its tile's slot (LOCAL: the block's own slot, whose
            // earlier slots take the reverse direction).
            const int t = LOCAL ? done.qbase / QT : done.cbase / CT;
            const int qi = done.qbase + tid;
            float v = red_v[0][tid];
            int32_t i = red_i[0][tid];
#pragma unroll
            for (int w = 1; w < WC; ++w) merge_pair(v, i, v, i, red_v[w][tid], red_i[w][tid]);
            const long o = ((long)done.b * T + t) * N + qi;
            pv[o] = v;
            pi[o] = i;
        }
        if constexpr (SYM) {
            // Candidate rows of the tile over the query block (the block's tile slot), on the
            // threads without a query.
            static_assert(THREADS >= CT + QT, "a thread per candidate row besides the queries'");
            const int jl = tid - (THREADS - CT);
            if (pend_rev && jl >= 0 && done.cbase + jl < n) {
                float v = red_cv[0][jl];
                int32_t i = red_ci[0][jl];
#pragma unroll
                for (int w = 1; w < WQ; ++w) merge_pair(v, i, v, i, red_cv[w][jl], red_ci[w][jl]);
                // A row with no query of the block inside its window: -inf, and no index.
                if (LOCAL && v == -__builtin_inff()) i = -1;
                const long o = ((long)done.b * T + done.qbase / QT) * N + done.cbase + jl;
                pv[o] = v;
                pi[o] = i;
            }
        }
        pend_fwd = pend_rev = false;
    };
    // LOCAL: each query's best so far over the item's earlier tiles (this lane's n-tiles).
    float bv_run[LOCAL ? NT : 1];
    int32_t bi_run[LOCAL ? NT : 1];
#pragma unroll
    for (int nt = 0; nt < (LOCAL ? NT : 1); ++nt) {
        bv_run[nt] = -__builtin_inff();
        bi_run[nt] = -1;
    }
    int cchunk = 0;
    int consumed = 0;
    while (ci.k < nitems) {
        // Chunk c has landed for this wave (and its LDS writes are done); after the barrier for
        // every wave, and every wave is done with chunk c-1, whose stage then takes chunk c+1.
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0)
        if constexpr (TAIL) {
            if (cchunk == nchunks - 1) {
                if (cchunk * CB + lcol >= rowbytes) {
                    uint8_t* sb = lds + (consumed & 1) * STAGE_BYTES + lane * 16;
#pragma unroll
                    for (int i = 0; i < LOADS; ++i) store16(sb + (wave + WAVES * i) * RPI * CB, u32x4{0u, 0u, 0u, 0u});
                }
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            }
        }
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_frags(fa0, fq0, consumed, 0);
        if (cchunk == 0) {
            flush();
            fetch_item(ci);
        }
        if constexpr (!LOCAL) advance();
        issue_begin();
        auto groups = [&](int g0, int g1) {
#pragma unroll
            for (int g = g0; g < g1; ++g) {
                if (g + 1 < KG) {
                    if ((g & 1) == 0) read_frags(fa1, fq1, consumed, g + 1);
                    else read_frags(fa0, fq0, consumed, g + 1);
                }
                if ((g & 1) == 0) mma_issue(fa0, fq0, consumed, g);
                else mma_issue(fa1, fq1, consumed, g);
            }
        };
        if constexpr (CUT) {
            groups(0, KG / 2);  // with all of the next chunk's loads
            if (cchunk < nchunks - 1 || !half_tail) groups(KG / 2, KG);
        } else {
            groups(0, KG);
        }
        issue_end();
        ++consumed;
        if (++cchunk < nchunks) continue;

        // ---- end of an item: norms, scores, per-query partial argmax ----
        if (nchunks == 1 && (given || LOCAL)) __builtin_amdgcn_s_waitcnt(0x0F70);  // the item's own values have landed
        if constexpr (!given) {
#pragma unroll
            for (int j = 0; j < NSC; ++j) {
                const int mt = wq + j * WQ;
                if (mt >= MT) break;
                const float t = half_sum(ss[j]);  // lanes l, l+32: the two k halves
                if (khalf == 0) inv_c[wc * MT * 32 + mt * 32 + lrow] = 1.0f / fmaxf(sqrtf(t), 1e-12f);
            }
            if constexpr (SYM) {
#pragma unroll
                for (int j = 0; j < NSQ; ++j) {
                    const int nt = wc + j * WC;
                    if (nt >= NT) break;
                    const float t = half_sum(sq[j]);
                    if (khalf == 0) inv_q[wq * NT * 32 + nt * 32 + lrow] = 1.0f / fmaxf(sqrtf(t), 1e-12f);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NSC; ++j) ss[j] = 0.0f;
#pragma unroll
        for (int j = 0; j < NSQ; ++j) sq[j] = 0.0f;
        if constexpr (LOCAL) {
            if (tid < CT + QT) {
                const int p = win.pos ? win_pos[tid] : min(tid < CT ? ci.cbase + tid : ci.qbase + tid - CT, ci.n - 1);
                const int row = win.grid_w(p);
                win_rc[0][tid] = row;
                win_rc[1][tid] = p - row * (int)win.grid_w.d;
            }
        }
        // Given norms are visible since the second chunk's barrier.
        if (!given || LOCAL || nchunks == 1) lds_barrier();
        const float* iv = inv_c;
        const int n = ci.n;
        const int cb = ci.cbase;
        // 32-row tiles of this wave that hold at least one token of the image (uniform);
        // the others are computed on clamped rows and skipped here.
        const int mt_lim = min(MT, max(0, (n - (cb + wc * MT * 32) + 31) / 32));
        const int nt_lim = min(NT, max(0, (n - (ci.qbase + wq * NT * 32) + 31) / 32));
        // Query blocks are aligned and no larger than candidate tiles, so a query's own
        // index is a candidate of this item only when its block lies inside the tile;
        // it then sits in candidate 32-row tile (qbase - cb)/32 + (query 32-row tile).
        static_assert(CT % QT == 0, "query blocks must nest in candidate tiles");
        const bool diag = ci.qbase >= cb && ci.qbase < cb + CT;
        const int self_tile0 = (ci.qbase - cb) / 32;
        // Accumulator element r = 4g+e of this lane is candidate row 8g + 4*khalf + e of
        // its 32-row tile, so rows ascend with r. The 32 values of two tiles are reduced together:
        // first their maximum, by value alone (two to three values an instruction), then the
        // first value equal to it, so the lowest index wins among equal scores; pairs of tiles
        // are merged into the running best in ascending order with a strict >. A tournament that
        // carried an index through every comparison took a compare and two selects a value and
        // waited for most of its compares: whole schedules were 1.4 to 2.4% slower with it, the
        // neighbour query of 16 images of 1024 768-byte rows 3.8%.
        float bv[NT];
        int32_t bi[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            bv[nt] = LOCAL ? bv_run[LOCAL ? nt : 0] : -__builtin_inff();
            bi[nt] = LOCAL ? bi_run[LOCAL ? nt : 0] : -1;
        }
        // LOCAL: this lane's query's grid row and column per n-tile; the window test is
        // |row_j - row_q| <= radius and |col_j - col_q| <= radius, as unsigned compares.
        int q_r[LOCAL ? NT : 1], q_c[LOCAL ? NT : 1];
        if constexpr (LOCAL) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                q_r[nt] = win_rc[0][CT + wq * NT * 32 + nt * 32 + lrow] - win.radius;
                q_c[nt] = win_rc[1][CT + wq * NT * 32 + nt * 32 + lrow] - win.radius;
            }
        }
        const uint32_t wspan = 2u * (uint32_t)win.radius;
        // This lane's own row inside a 32-row tile, as an accumulator element (if it holds it).
        const int self_r = (((lrow >> 2) & 1) == khalf) ? 4 * (lrow >> 3) + (lrow & 3) : -1;
        if constexpr (LOCAL) {
            // Both directions read the accumulators: pairs outside the window become -inf
            // there (the inverse norms that scale them are positive).
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int jl = wc * MT * 32 + mt * 32 + 8 * g + 4 * khalf;
                    const int4 cr = *reinterpret_cast<const int4*>(&win_rc[0][jl]);
                    const int4 cc = *reinterpret_cast<const int4*>(&win_rc[1][jl]);
                    const int crv[4] = {cr.x, cr.y, cr.z, cr.w}, ccv[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const bool in = (uint32_t)(crv[e] - q_r[nt]) <= wspan && (uint32_t)(ccv[e] - q_c[nt]) <= wspan;
                            acc[mt][nt][4 * g + e] = in ? acc[mt][nt][4 * g + e] : -__builtin_inff();
                        }
                }
        }
        // Candidate tiles reduced together (one where the window's state leaves no registers for two).
        constexpr int MP = MT >= 2 && !(LOCAL && MT * NT >= 8) ? 2 : 1;
        constexpr int SC = MP * 16, GR = SC / 4;
#pragma unroll
        for (int mp = 0; mp < MT; mp += MP) {
            if (mp >= mt_lim) break;
            const int jt = cb + wc * MT * 32 + mp * 32 + 4 * khalf;  // candidate of r = 0
            f32x4 ivv[4 * MP];
#pragma unroll
            for (int g = 0; g < 4 * MP; ++g)
                ivv[g] = *reinterpret_cast<const f32x4*>(&iv[wc * MT * 32 + mp * 32 + 8 * g + 4 * khalf]);
            const bool partial = cb + wc * MT * 32 + mp * 32 + MP * 32 > n;  // some rows of these tiles are past the image
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (nt >= nt_lim) break;
                float sc[SC];
#pragma unroll
                for (int r = 0; r < SC; ++r) sc[r] = acc[mp + r / 16][nt][r % 16] * ivv[r / 4][r % 4];
                if (partial) {
#pragma unroll
                    for (int r = 0; r < SC; ++r) sc[r] = jt + 8 * (r >> 2) + (r & 3) < n ? sc[r] : -__builtin_inff();
                }
#pragma unroll
                for (int m = 0; m < MP; ++m) {
                    if (diag && wc * MT + mp + m == self_tile0 + wq * NT + nt) {  // the tile holding each lane's own query
#pragma unroll
                        for (int r = 0; r < 16; ++r) sc[16 * m + r] = r == self_r ? -__builtin_inff() : sc[16 * m + r];
                    }
                }
                // The best of each group of four, then of the groups, by value alone; then the first
                // group that holds it and the first of its four.
                float gm[GR];
#pragma unroll
                for (int k = 0; k < GR; ++k) gm[k] = max_of(max_of(sc[4 * k], sc[4 * k + 1], sc[4 * k + 2]), sc[4 * k + 3]);
                float v1 = max_of(gm[0], gm[1], gm[2]);
#pragma unroll
                for (int k = 3; k + 1 < GR; k += 2) v1 = max_of(v1, gm[k], gm[k + 1]);
                static_assert(GR % 2 == 0, "the last group alone");
                v1 = max_of(v1, gm[GR - 1]);
                float x[4] = {sc[SC - 4], sc[SC - 3], sc[SC - 2], sc[SC - 1]};
                int r1 = SC - 4;
#pragma unroll
                for (int k = GR - 2; k >= 0; --k) {
                    const bool c = gm[k] == v1;
#pragma unroll
                    for (int e = 0; e < 3; ++e) x[e] = c ? sc[4 * k + e] : x[e];
                    r1 = c ? 4 * k : r1;
                }
                const int e1 = x[0] == v1 ? 0 : x[1] == v1 ? 1 : x[2] == v1 ? 2 : 3;
                r1 += e1;
                // Materialise the winning index before the merge: otherwise the compiler moves
                // the index selection into a divergent branch per tile, which serialises the
                // tiles' reductions (measured slower).
                asm volatile("" : "+v"(r1));
                const bool up = v1 > bv[nt];
                bv[nt] = up ? v1 : bv[nt];
                bi[nt] = up ? jt + r1 + 4 * (r1 >> 2) : bi[nt];  // row 8*(r/4) + r%4 from the first tile's
            }
        }
        // Reverse direction of an off-diagonal item (query block before the candidate
        // tile). A candidate row's queries of one n-tile sit in the 32 lanes of one lane
        // half (one per lane), so after an in-lane merge over the NT n-tiles the best of
        // each row is found by a reduce-scatter across the half: exchanges with lane
        // l^16, l^15, l^7, l^2 and l^1 (XOR masks spanning all five lane bits) each
        // halve the rows a lane carries, until lanes 2r and 2r+1 hold row r's best.
        // Merges are lexicographic (larger score, then smaller query), so the lowest
        // query wins ties, as in the forward direction.
        const bool rev = SYM && !diag;
        if (rev) {
            float ivq[NT];
            bool qok[NT];
            int32_t qidx[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int ql = wq * NT * 32 + nt * 32 + lrow;
                ivq[nt] = inv_q[ql];
                qidx[nt] = ci.qbase + ql;
                qok[nt] = qidx[nt] < n;
            }
            const bool all_q = ci.qbase + (wq + 1) * NT * 32 <= n;  // every query of this wave is a token (uniform)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (mt >= mt_lim) break;
                // This lane's best query for each of its 16 accumulator rows (a strict >
                // keeps the lower n-tile, i.e. the lower query, on ties).
                float v[16];
                int32_t ix[16];
                if (all_q) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        v[r] = acc[mt][0][r] * ivq[0];
                        ix[r] = qidx[0];
#pragma unroll
                        for (int nt = 1; nt < NT; ++nt) {
                            const float s2 = acc[mt][nt][r] * ivq[nt];
                            const bool c = s2 > v[r];
                            v[r] = c ? s2 : v[r];
                            ix[r] = c ? qidx[nt] : ix[r];
                        }
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        v[r] = qok[0] ? acc[mt][0][r] * ivq[0] : -__builtin_inff();
                        ix[r] = qidx[0];
#pragma unroll
                        for (int nt = 1; nt < NT; ++nt) {
                            const float s2 = qok[nt] ? acc[mt][nt][r] * ivq[nt] : -__builtin_inff();
                            const bool c = s2 > v[r];
                            v[r] = c ? s2 : v[r];
                            ix[r] = c ? qidx[nt] : ix[r];
                        }
                    }
                }
                // l^16 with v_permlane16_swap: slots k and k+8 of the two 16-lane rows of a
                // half trade places, and the lower row keeps rows k, the upper rows k+8.
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const auto sv = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[k]), __float_as_uint(v[k + 8]),
                                                                     false, false);
                    const auto si = __builtin_amdgcn_permlane16_swap((uint32_t)ix[k], (uint32_t)ix[k + 8], false, false);
                    merge_pair(v[k], ix[k], __uint_as_float(sv[0]), (int32_t)si[0], __uint_as_float(sv[1]),
                               (int32_t)si[1]);
                }
                exchange_half<0x140, 4>(v, ix, (lane >> 3) & 1);  // l^15 (row mirror), split on lane bit 3
                exchange_half<0x141, 2>(v, ix, (lane >> 2) & 1);  // l^7 (half-row mirror), bit 2
                exchange_half<0x4E, 1>(v, ix, (lane >> 1) & 1);   // l^2 (quad permutation 2,3,0,1), bit 1
                merge_pair(v[0], ix[0], v[0], ix[0], dpp_f<0xB1>(v[0]), dpp_i<0xB1>(ix[0]));  // l^1 (1,0,3,2)
                // Lanes 2r, 2r+1 of half h: accumulator row r = candidate row 8(r/4) + 4h + r%4.
                if ((lane & 1) == 0) {
                    const int r = (lrow >> 1) & 15;
                    const int jl = wc * MT * 32 + mt * 32 + 8 * (r >> 2) + 4 * khalf + (r & 3);
                    red_cv[wq][jl] = v[0];
                    red_ci[wq][jl] = ix[0];
                }
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x16{};  // the next item starts from zero
        // LOCAL: between the tiles of an item only the running best is kept; the lanes,
        // waves and the partial are merged and written after its last tile.
        bool item_end = true;
        if constexpr (LOCAL) {
            item_end = ci.cbase >= ci.thi * CT;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                bv_run[nt] = item_end ? -__builtin_inff() : bv[nt];
                bi_run[nt] = item_end ? -1 : bi[nt];
            }
        }
        if (item_end) {
            // Merge the two lane halves (larger score, then smaller index); the waves' merge follows
            // in flush(). Two n-tiles at a time: after the swap, a lane holds one half's entry of
            // the first tile (lanes 0-31) or the second (32-63) and the other half's.
            static_assert(NT == 1 || NT % 2 == 0, "n-tiles in pairs");
#pragma unroll
            for (int nt = 0; nt < NT; nt += 2) {
                const int n2 = NT == 1 ? nt : nt + 1;
                const auto sv = __builtin_amdgcn_permlane32_swap(__float_as_uint(bv[nt]), __float_as_uint(bv[n2]), false, false);
                const auto si = __builtin_amdgcn_permlane32_swap((uint32_t)bi[nt], (uint32_t)bi[n2], false, false);
                float v;
                int32_t i;
                merge_pair(v, i, __uint_as_float(sv[0]), (int32_t)si[0], __uint_as_float(sv[1]), (int32_t)si[1]);
                const int ql = wq * NT * 32 + nt * 32 + (NT == 1 ? lrow : lane);
                if (NT > 1 || khalf == 0) {
                    red_v[wc][ql] = v;
                    red_i[wc][ql] = i;
                }
            }
        }
        if constexpr (LOCAL) {
            // The slots no item writes for this block's rows: tiles before the band and after
            // the block (the band relation is symmetric, so the items that write slot q for
            // these rows are exactly the blocks q of the band before it).
            if (item_end && tid < QT && ci.qbase + tid < n) {
                const int nq = (n + QT - 1) / QT, own = ci.qbase / QT;
                for (int q = 0; q < nq; ++q) {
                    if (q >= ci.tlo && q <= own) continue;
                    const long oq = ((long)ci.b * T + q) * N + ci.qbase + tid;
                    pv[oq] = -__builtin_inff();
                    pi[oq] = -1;
                }
            }
        }
        pend_fwd = item_end;
        pend_rev = rev;
        done = ci;
        cchunk = 0;
        ci = inext;  // loads run one chunk ahead: the chunk issued last is the next item's first
        if constexpr (HALVES) lq_off = (ci.qbase - ci.cbase + wq * NT * 32 + lrow) * CB;
    }
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    flush();
    // (The waits above also cover the trailing loads, which land before the LDS is released.)
}

// Block shapes. 256 x 256 on 8 waves (two 64 KB stages, one workgroup per CU): the full
// schedule splits the tile over 2 candidate x 4 query waves (128 x 64 each), the symmetric
// one over 4 x 2 (64 x 128 each), so that its reverse direction merges 4 queries inside
// each lane before the cross-lane steps and carries half as many rows through them.
constexpr int kPWC = 2, kPWQ = 4, kPMT = 4, kPNT = 2, kPWGS = 1;
constexpr int kSWC = 4, kSWQ = 2, kSMT = 2, kSNT = 4;
constexpr int kPCT = kPWC * kPMT * 32;
static_assert(kPCT == kSplitRows, "the half-block launch splits the large blocks");
// Small batches use 64 x 64 blocks on 4 waves of one 32 x 32 tile each, up to four
// workgroups per CU, so a single image of 1024 tokens still spreads over 256 CUs.
constexpr int kTWC = 2, kTWQ = 2, kTMT = 1, kTNT = 1, kTWGS = 4;
constexpr int kTCT = kTWC * kTMT * 32;
static_assert(kTWQ * kTNT * 32 == kTCT && kPCT % kTCT == 0, "square small blocks that nest in the large ones");
static_assert(kSWC * kSMT * 32 == kPCT && kSWQ * kSNT * 32 == kPCT && kPWQ * kPNT * 32 == kPCT,
              "both schedules use 256 x 256 tiles, so their partials share one layout");

// Rows that are a whole number of 64 bytes: the ones the schedule and block-size arguments
// and given norms apply to.
bool whole_64(int D, int dt) { return ((long)D * (dt == kBf16 ? 2 : 4)) % 64 == 0; }

}  // namespace

bool affinity_takes_norms(int D, int dt) { return dt == kBf16 && whole_64(D, dt); }

namespace {

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

// Whether a symmetric launch may defer diagonal blocks in any XCD group (images whose
// lengths only the device knows: any may).
bool defers_diagonals(bool counted, int B, int N, int log_xcds, int slots, bool lone)
{
    if (counted) return true;
    const int nb = (N + kPCT - 1) / kPCT;
    const WorkShape shape(kOrderSymmetric, B, nb);
    const WorkCounts<false> counts{shape, nullptr, nullptr};
    for (int g = 0; g < 1 << log_xcds; ++g)
        if (work_share(counts, B, g, log_xcds, slots, true, lone).ndef > 0) return true;
    return false;
}

struct AffinityArgs {
    const void* x;
    const int32_t* x_off;
    const float* xinv;
    int B, N, D, T, cus, xcds;
    float* pv;
    int32_t* pi;
    hipStream_t stream;
    hipEvent_t start, stop;
    Window win;
    Clear clear;
};

template <class S>
constexpr int chunks_of(int D)
{
    return (int)(((long)D * S::kBytes + kChunkBytes - 1) / kChunkBytes);
}

template <class S, int WC, int WQ, int MT, int NT, bool SYM, bool LOCAL, bool GIVEN, bool TAIL, bool COUNTED>
void launch_counted(const AffinityArgs& a, int slots, const WorkShape& shape)
{
    const uint8_t* xb = static_cast<const uint8_t*>(a.x);
    const int log_xcds = a.xcds == 1 ? 0 : 3;
    static_assert(kXcds == 8, "the groups of mpm_work.h");
    const dim3 grid(slots * a.xcds), block(WC * WQ * kWave);
    // The symmetric schedule's deferred diagonal blocks, as half blocks, in a second launch
    // (one item per slot); the timing events then span both.
    constexpr bool SPLIT = SYM && !LOCAL && WC * MT * 32 == kSplitRows;
    const bool lone = splits_lone<S>(chunks_of<S>(a.D), (int)shape.nb.d);
    const bool halves = SPLIT && defers_diagonals(COUNTED, a.B, a.N, log_xcds, slots, lone);
    hipExtLaunchKernelGGL((affinity_partial_kernel<S, WC, WQ, MT, NT, SYM, false, LOCAL, GIVEN, TAIL, COUNTED>), grid,
                          block, 0, a.stream, a.start, halves ? nullptr : a.stop, 0, xb, a.x_off, a.B, a.N, a.D, a.T,
                          log_xcds, slots, shape, a.pv, a.pi, a.xinv, a.win, a.clear);
    if constexpr (SPLIT) {
        if (halves)
            hipExtLaunchKernelGGL((affinity_partial_kernel<S, WC, WQ, MT, NT / 2, false, true, false, GIVEN, TAIL, COUNTED>),
                                  grid, block, 0, a.stream, nullptr, a.stop, 0, xb, a.x_off, a.B, a.N, a.D, a.T,
                                  log_xcds, slots, shape, a.pv, a.pi, a.xinv, a.win, Clear{});
    }
}

template <class S, int WC, int WQ, int MT, int NT, bool SYM, bool LOCAL, bool GIVEN, bool TAIL>
void launch_persistent_as(AffinityArgs a, int groups)
{
    // No more slots than a group can have items (images of N tokens; two a diagonal block that
    // may run as halves), and no count of the images' own blocks when every item has its slot
    // (the count costs each workgroup 0.8 us).
    constexpr int CT = WC * MT * 32;
    constexpr bool SPLIT = SYM && !LOCAL && CT == kSplitRows;
    constexpr WorkOrder ORDER = LOCAL ? kOrderBand : SYM ? kOrderSymmetric : kOrderFull;
    const int nb = (a.N + CT - 1) / CT;
    const long total = (long)a.B * work_items(ORDER, nb);
    const bool counted = a.x_off != nullptr && a.B <= kMaxCountedImages && total > groups / a.xcds * (long)a.xcds;
    // Fewer images than XCDs: one group, so that the share is the chip's, where blocks may run as
    // halves, past a round. An early share of a large image has too few diagonal blocks to defer
    // and takes another round: one image of 5835 rows of 2048 bytes, 276 blocks on 256 slots, in 8
    // groups / one 84.5 / 58.5 us. Elsewhere one group is slower (every row passes through every
    // L2): seven images of 2027 rows of 3440 bytes 88 / 97, seven packed ones of 140 to 400
    // 3024-byte rows on small blocks 17.9 / 21.7; only a few very uneven images, the longest one's
    // items all on its share's XCDs, would gain (1288 and 80 float32 rows of 4096 bytes 81 / 45).
    if (SPLIT && a.B < kXcds && total > a.cus) a.xcds = 1;
    const int most = groups / a.xcds;
    const long each = (total + a.xcds - 1) / a.xcds;
    const int slots = (int)std::min<long>(most, SPLIT && splits_lone<S>(chunks_of<S>(a.D), nb) ? 2 * each : each);
    const WorkShape shape(ORDER, a.B, nb);
    if (counted)
        launch_counted<S, WC, WQ, MT, NT, SYM, LOCAL, GIVEN, TAIL, true>(a, slots, shape);
    else
        launch_counted<S, WC, WQ, MT, NT, SYM, LOCAL, GIVEN, TAIL, false>(a, slots, shape);
}

// Given norms (bfloat16 only) and norms summed in the K loop are separate builds: with one
// build and a run-time flag, the flag's branch per k-group cost the summing launches 2-4%,
// and two builds alternating between insertions showed no instruction-cache penalty.
template <class S, int WC, int WQ, int MT, int NT, bool SYM, bool LOCAL>
void launch_blocks(const AffinityArgs& a, int groups)
{
    const bool tail = ((long)a.D * S::kBytes) % kChunkBytes != 0;
    if constexpr (S::kBytes == 2) {
        if (a.xinv != nullptr) {
            if (tail) launch_persistent_as<S, WC, WQ, MT, NT, SYM, LOCAL, true, true>(a, groups);
            else launch_persistent_as<S, WC, WQ, MT, NT, SYM, LOCAL, true, false>(a, groups);
            return;
        }
    }
    if (tail) launch_persistent_as<S, WC, WQ, MT, NT, SYM, LOCAL, false, true>(a, groups);
    else launch_persistent_as<S, WC, WQ, MT, NT, SYM, LOCAL, false, false>(a, groups);
}

template <int WC, int WQ, int MT, int NT, bool SYM, bool LOCAL = false>
void launch_persistent(int dt, const AffinityArgs& a, int groups)
{
    if (dt == kBf16) launch_blocks<Bf16, WC, WQ, MT, NT, SYM, LOCAL>(a, groups);
    else launch_blocks<F32, WC, WQ, MT, NT, SYM, LOCAL>(a, groups);
}

}  // namespace

// Partial slots reserved per token: enough for the smallest block width any schedule uses.
int partial_tiles(int N) { return (N + kTCT - 1) / kTCT; }

bool valid_schedule(int schedule)
{
    return schedule == kScheduleAuto || schedule == kScheduleFull || schedule == kScheduleSymmetric ||
           schedule == kScheduleFull64;
}

namespace {

// The locality-constrained schedule's two block sizes: 256 x 256 blocks on 8 waves, one
// workgroup per CU (the dense symmetric shape), or 128 x 128 blocks on 4 waves of 64 x 64,
// two workgroups per CU. Smaller blocks cut a query block's window band more finely and
// give twice the items; each small block costs about 0.357 of a large one (a quarter of
// its matrix work at about 70% of its efficiency: half the flops per byte loaded), of float32
// rows 0.29 (they are bound by the matrix work).
constexpr int kLWC = 2, kLWQ = 2, kLMT = 2, kLNT = 2, kLWGS = 2;
constexpr int kLCT = kLWC * kLMT * 32;
static_assert(kLWQ * kLNT * 32 == kLCT && kPCT % kLCT == 0 && kLCT % kTCT == 0, "square small window blocks");
constexpr double kLSmallBlockCost = 0.357, kLSmallBlockCostF32 = 0.29;

// Estimated duration (in large-block times) of a locality-constrained launch with ts x ts
// blocks, on a full raster grid (positions = token indices): per XCD group, the blocks of
// its images are dealt to the slots in order, each costing the tiles of its band from its
// own on. With two workgroups per CU, the busiest slot is taken to share its CU with a
// typical (median) one.
double local_cost(int B, int N, int grid_w, int radius, int ts, int xcds, int slots, int wgs_per_cu, double block_cost)
{
    const int nblk = (N + ts - 1) / ts;
    std::vector<int> tiles(nblk);
    long total = 0;
    for (int t = 0; t < nblk; ++t) {
        const long r_last = (long)(std::min((t + 1) * ts, N) - 1) / grid_w;
        const long thi = std::min<long>(nblk - 1, ((r_last + radius + 1) * (long)grid_w - 1) / ts);
        tiles[t] = (int)(thi - t + 1);
        total += tiles[t];
    }
    const long items = ((long)B * nblk + xcds - 1) / xcds;  // of the largest group
    if (items > 64L * slots) return (double)items * total / nblk / slots * wgs_per_cu * block_cost;  // many rounds: balanced
    std::vector<long> load(slots, 0);
    for (long k = 0; k < items; ++k) load[k % slots] += tiles[k % nblk];
    std::sort(load.begin(), load.end());
    const long busiest = load[slots - 1];
    const long typical = load[slots / 2];
    return (double)(wgs_per_cu == 1 ? busiest : busiest + typical) * block_cost;
}

}  // namespace

bool valid_local_block_rows(int requested) { return requested == 0 || requested == kLCT || requested == kPCT; }

namespace {

// The block rows a windowed launch runs (local_block_rows reports N for rows the argument
// does not apply to).
int local_rows(int B, int N, int D, int dt, int grid_w, int radius, int requested)
{
    if (requested != 0 && whole_64(D, dt)) return requested;
    const int cus = device_cus();
    if (cus <= 0) return kPCT;
    const int xcds = cus % kXcds == 0 ? kXcds : 1;
    const double large = local_cost(B, N, grid_w, radius, kPCT, xcds, cus * kPWGS / xcds, kPWGS, 1.0);
    const double small = local_cost(B, N, grid_w, radius, kLCT, xcds, cus * kLWGS / xcds, kLWGS,
                                    dt == kBf16 ? kLSmallBlockCost : kLSmallBlockCostF32);
    return small < large ? kLCT : kPCT;
}

}  // namespace

int local_block_rows(int B, int N, int D, int dt, int grid_w, int radius, int requested)
{
    if (!whole_64(D, dt)) return N;
    return local_rows(B, N, D, dt, grid_w, radius, requested);
}

int local_tile_width(int B, int N, int D, int dt, int grid_w, int radius, int requested)
{
    return local_rows(B, N, D, dt, grid_w, radius, requested);
}

namespace {

// Block shape and schedule of a launch: 64 x 64 full, 128 x 128 symmetric (the shape of the
// small window blocks: 4 waves, two workgroups per CU), 256 x 256 full and symmetric.
enum Blocks : int { kBlocks64, kBlocks128, kBlocks256, kBlocksSym256 };

// Estimated duration (us) of a dense launch's items on c 128-byte chunks of K: a fixed part,
// and a round of the workgroup slots. Fitted to launches of 1 to 64 images of 100 to 4096
// bfloat16 rows of 128 to 2048 bytes (495 shapes, replayed from a graph): the pick it gives is
// 0.2% slower than the fastest of the four shapes over the dense ones, 0.5% over packed
// batches, and 15% (dense) and 19% (packed) faster than 64 x 64 blocks for at most 32 large
// blocks and 256 x 256 ones elsewhere. Examples, 64 / 128 / 256 full / 256 symmetric, dense rows
// of 1536 bytes: 8 images of 400 rows 10.0 / 13.5 / 21.2 / 24.2 us; 12 of 1024 rows 35.8 /
// 18.0 / 22.6 / 24.7; 24 of 1024 rows 67.7 / 32.3 / 41.9 / 27.1; 16 of 1024 rows of 384 bytes
// - / 15.7 / 11.3 / 14.6.
// Dense batches past those, up to 1000 images (215 shapes of rows of 64 to 2048 bytes): after some
// rounds of large symmetric blocks the workgroups no longer start theirs together, and a round
// costs a tenth less: 500 images of 400 rows of 768 bytes, 128 / 256 symmetric, 86.5 / 78.5 us.
// Packed ones keep the estimate above: their lengths are only guessed, and where they fall short
// of the guess a large block costs four times a middling one (1000 packed images of at most 196
// rows of 128 bytes, 128 / 256 full: 25.4 / 18.6 us as long as guessed, twice as slow the other
// way round at a tenth of it).
double round_us(double fixed, double round, double rounds) { return fixed + round * rounds; }

double settled(double rounds) { return std::min(rounds, 4.0) + 0.9 * std::max(0.0, rounds - 4.0); }

double estimate_us(Blocks k, double blocks64, double blocks128, double full256, double sym256, double c, double cus,
                   bool counted)
{
    // Rounds of whole slots; a packed batch's lengths are only guessed, so a part of a round is
    // taken to cost its mean there.
    switch (k) {
    case kBlocks64: {
        const double per_cu = blocks64 / cus;  // up to four workgroups share a CU
        return 3.5 + 0.29 * c + std::max(0.0, per_cu - 1.0) * (0.68 + 0.20 * c);
    }
    case kBlocks128: {
        const double round = 5.3 + 0.79 * c, r = blocks128 / (2 * cus);
        // The last round's workgroups run alone on their CU up to half of the slots.
        auto part = [](double f) { return f <= 0 ? 0.0 : f <= 0.5 ? 0.6 : 0.6 + 0.4 * (2 * f - 1); };
        if (counted) return round_us(4.4, round, 1.1 * r <= 1 ? part(1.1 * r) : r + 0.31);
        return round_us(4.4, round, std::floor(r) + part(r - std::floor(r)));
    }
    case kBlocks256: return round_us(2.5, 4.3 + 1.43 * c, std::ceil(full256 / cus));
    default: {
        const double round = 9.0 + 1.31 * c, r = sym256 / cus;
        if (counted) return round_us(2.0, round, 1.1 * r <= 1 ? 1 : r + 0.62) + (1.1 * r <= 1 ? 0 : 3.0);
        const double f = r - std::floor(r);  // a short last round runs as half blocks
        return round_us(2.0, round, settled(std::floor(r) + (f <= 0 ? 0 : r > 1 && f <= 0.5 ? 0.82 : 1.0)));
    }
    }
}

// float32 rows: a block's matrix work outweighs the rest of it, so only the rounds count, in
// units of a round of 128 x 128 symmetric blocks (two per CU); one of 256 x 256 blocks takes
// 1.8. Up to four 64 x 64 blocks a CU run as fast as the rest of the chip allows (they are whole
// rounds of a quarter of the work). Timed on 170 dense and 170 packed shapes, 1 to 64 images of
// 100 to 4096 rows of 192 to 4096 bytes: 0.6% slower than the fastest of the four shapes, against
// 59% for 64 x 64 blocks of at most 32 large blocks and 256 x 256 ones elsewhere. Examples, 64 /
// 128 / 256 full / 256 symmetric, dense rows of 768 bytes: 4 images of 1024 rows 19.1 / 19.5 /
// 49.0 / 52.5 us; 16 of 1024 rows 60.3 / 44.5 / 50.0 / 52.6; 32 of 1024 rows - / 78.9 / 106.4 /
// 86.7; 46 of 1924 rows of 832 bytes - / 420.6 / 660.8 / 384.5.
// Dense rows of at most one and a half chunks (c, in halves) are too narrow for that: their items'
// fixed parts count, and a single round of full 256 x 256 blocks is the fastest of the large
// shapes. 64-byte rows, 128 / 256 full / 256 symmetric: 16 images of 1024 rows 13.2 / 10.3 / 13.0
// us, 128 of them 57.7 / 58.8 / 47.8. Packed rows keep to rounds (lengths far from the guess).
Blocks pick_blocks_f32(double blocks64, double blocks128, double full256, double sym256, double c, double cus,
                       bool packed)
{
    if (blocks64 <= 4 * cus) return kBlocks64;
    const double r = blocks128 / (2 * cus), s = sym256 / cus;
    double rounds128, rounds256;
    if (packed) {  // lengths are only guessed: a part of a round is taken to cost its mean
        rounds128 = 1.1 * r <= 0.5 ? 0.6 : 1.1 * r <= 1 ? 1.0 : r + 0.3;
        rounds256 = 1.1 * s <= 1 ? 1.0 : s + 0.6;
    } else {
        const double f = r - std::floor(r), g = s - std::floor(s);
        // The last round: alone on their CUs up to half of the slots; as half blocks.
        rounds128 = std::floor(r) + (f <= 0 ? 0.0 : f <= 0.5 ? 0.6 : 0.95);
        rounds256 = std::floor(s) + (g <= 0 ? 0.0 : s > 1 && g <= 0.5 ? 0.6 : 1.0);
    }
    if (packed || c > 1.5) return rounds128 <= 1.8 * rounds256 ? kBlocks128 : kBlocksSym256;
    const double us128 = round_us(2.5, 4.6 + 3.5 * c, rounds128), us256 = round_us(2.0, 6.0 + 7.1 * c, rounds256);
    if (round_us(2.5, 3.4 + 7.05 * c, std::ceil(full256 / cus)) < std::min(us128, us256)) return kBlocks256;
    return us128 <= us256 ? kBlocks128 : kBlocksSym256;
}

Blocks pick_blocks(int B, int N, int D, int dt, int schedule, bool packed, int device_cu_count)
{
    if (whole_64(D, dt)) {
        if (schedule == kScheduleFull) return kBlocks256;
        if (schedule == kScheduleSymmetric) return kBlocksSym256;
        if (schedule == kScheduleFull64) return kBlocks64;
    }
    const int cus = std::max(1, device_cu_count);
    auto blocks = [&](int w, WorkOrder order, int percent) {  // of images of at least one token
        return (double)B * work_items(order, (int)((std::max(1L, (long)N * percent / 100) + w - 1) / w));
    };
    const double capacity64 = blocks(kTCT, kOrderFull, 100);
    // A small block a CU is the fastest by every estimate below (host time of the smallest calls);
    // and images of at most 64 tokens have one block of any size (1000 of 64 rows of 2048 bytes, 64 /
    // 128: 21.8 / 36.1 us; 1400 one-token images of float32 rows of 768 bytes 9.9 / 19.4).
    if (capacity64 <= cus || N <= kTCT) return kBlocks64;
    const double full256 = blocks(kPCT, kOrderFull, 100);
    const double c = std::ceil(2.0 * D / kChunkBytes);
    double b64 = capacity64, b128 = blocks(kLCT, kOrderSymmetric, 100), s256 = blocks(kPCT, kOrderSymmetric, 100);
    if (packed) {  // images as an earlier insertion leaves them: 80 to 90% of N tokens
        b64 = b128 = s256 = 0;
        for (int percent : {80, 85, 90}) {
            b64 += blocks(kTCT, kOrderFull, percent) / 3;
            b128 += blocks(kLCT, kOrderSymmetric, percent) / 3;
            s256 += blocks(kPCT, kOrderSymmetric, percent) / 3;
        }
    }
    if (dt != kBf16)
        return pick_blocks_f32(b64, b128, full256, s256, std::ceil(4.0 * D / (kChunkBytes / 2)) / 2, cus, packed);
    Blocks best = kBlocks128;
    double us = estimate_us(kBlocks128, b64, b128, full256, s256, c, cus, packed);
    for (Blocks k : {kBlocks64, kBlocks256, kBlocksSym256}) {
        if (k == kBlocks64 && capacity64 > 2.5 * cus) continue;  // beyond, 128 x 128 blocks are as fast
        if (k == kBlocks256 && packed && full256 > cus) continue;  // a round of whole images or the symmetric blocks
        const double e = estimate_us(k, b64, b128, full256, s256, c, cus, packed);
        if (e < us) {
            us = e;
            best = k;
        }
    }
    return best;
}

int block_rows(Blocks k) { return k == kBlocks64 ? kTCT : k == kBlocks128 ? kLCT : kPCT; }

}  // namespace

int partial_tile_width(int B, int D, int dt, int N, int schedule, bool packed)
{
    return block_rows(pick_blocks(B, N, D, dt, schedule, packed, device_cus()));
}

hipError_t affinity_plan(int B, int N, int D, int dt, int schedule, bool packed, int* used, int* rows)
{
    const int cus = device_cus();
    if (cus <= 0) return hipErrorInvalidDevice;
    const Blocks k = pick_blocks(B, N, D, dt, schedule, packed, cus);
    *used = k == kBlocks64 ? kScheduleFull64 : k == kBlocks256 ? kScheduleFull : kScheduleSymmetric;
    *rows = block_rows(k);
    return hipSuccess;
}

hipError_t affinity_schedule(int B, int N, int D, int dt, int schedule, int* used)
{
    *used = kScheduleFull;
    if (!whole_64(D, dt)) return hipSuccess;  // no choice of schedule
    int rows = 0;
    return affinity_plan(B, N, D, dt, schedule, false, used, &rows);
}

hipError_t launch_affinity(const void* x, const int32_t* x_off, int B, int N, int D, int dt, int schedule, float* pv,
                           int32_t* pi, hipStream_t stream, hipEvent_t start, hipEvent_t stop, const float* xinv,
                           Clear clear, int* tile_width)
{
    const int T = partial_tiles(N);
    if (xinv && !affinity_takes_norms(D, dt)) return hipErrorInvalidValue;  // those kernels sum their own norms
    const int cus = device_cus();
    if (cus <= 0) return hipErrorInvalidDevice;
    const int xcds = cus % kXcds == 0 ? kXcds : 1;
    const AffinityArgs a{x, x_off, dt == kBf16 ? xinv : nullptr, B, N, D, T, cus, xcds, pv, pi, stream, start, stop,
                         Window{nullptr, FixedDiv(1), 0}, clear};
    const Blocks blocks = pick_blocks(B, N, D, dt, schedule, x_off != nullptr, cus);
    *tile_width = block_rows(blocks);
    switch (blocks) {
    case kBlocks64: launch_persistent<kTWC, kTWQ, kTMT, kTNT, false>(dt, a, cus * kTWGS); break;
    case kBlocks128: launch_persistent<kLWC, kLWQ, kLMT, kLNT, true>(dt, a, cus * kLWGS); break;
    case kBlocksSym256: launch_persistent<kSWC, kSWQ, kSMT, kSNT, true>(dt, a, cus * kPWGS); break;
    default: launch_persistent<kPWC, kPWQ, kPMT, kPNT, false>(dt, a, cus * kPWGS); break;
    }
    return hipGetLastError();
}

hipError_t launch_affinity_local(const void* x, const int32_t* x_off, const float* xinv, const int32_t* pos,
                                 int grid_w, int radius, int block_rows,
                                 int B, int N, int D, int dt, float* pv, int32_t* pi, hipStream_t stream,
                                 hipEvent_t start, hipEvent_t stop, Clear clear)
{
    // The persistent kernel on the symmetric schedule, one item per query block and the
    // tiles of its band from its own on (given norms: bf16 only), with blocks of block_rows.
    const int T = partial_tiles(N);
    const int cus = device_cus();
    if (cus <= 0) return hipErrorInvalidDevice;
    const int xcds = cus % kXcds == 0 ? kXcds : 1;
    // No two cells of a grid are further apart (the kernel adds the radius to a row).
    const int reach = std::min(radius, MPM_MAX_N);
    const AffinityArgs a{x, x_off, dt == kBf16 ? xinv : nullptr, B, N, D, T, cus, xcds, pv, pi, stream, start, stop,
                         Window{pos, FixedDiv((uint32_t)grid_w), reach}, clear};
    if (block_rows == kLCT) launch_persistent<kLWC, kLWQ, kLMT, kLNT, true, true>(dt, a, cus * kLWGS);
    else launch_persistent<kSWC, kSWQ, kSMT, kSNT, true, true>(dt, a, cus * kPWGS);
    return hipGetLastError();
}

}  // namespace mpm
