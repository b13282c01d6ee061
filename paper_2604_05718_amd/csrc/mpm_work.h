// How the affinity's work items are dealt to the workgroups (host and device; no HIP
// calls, so it compiles for the CPU too).
//
// The items of a batch stand in one order: image by image, and inside an image its
// blocks row by row (query block, then candidate tile). XCD group g of G takes the
// contiguous share [total*g/G, total*(g+1)/G) of that order, and its slot s (one
// workgroup) the share's items s, s + slots, ... So every group has the same number of
// items, give or take one, whatever the batch size and the images' lengths, the items of
// an image run together on one XCD (two at a share's ends) and re-read its rows from
// that XCD's L2. Dealing whole images to the groups instead (image b to group b mod 8)
// left groups idle when the batch was no multiple of 8, and counting every image as N
// tokens long left slots idle on ragged images.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define MPM_HD __host__ __device__ __forceinline__
#else
#define MPM_HD inline
#endif

namespace mpm {

// Full: every (query block, candidate tile) pair; symmetric: those on and above the block
// diagonal; band: one item per query block (it walks its own tiles).
enum WorkOrder : int { kOrderFull, kOrderSymmetric, kOrderBand };

// Images whose own block counts are tabulated (8 bytes of LDS each, beside the stages of up to
// four workgroups a CU); larger packed batches count every image as N tokens and skip the items
// past its end. Not counted / counted, launches in us: 32 images of 820 to 920 rows of 768 bytes
// 25.2 / 23.2, of 360 to 1024 23.5 / 19.1; 400 of them 237 / 230 and 198 / 164, of 820 to 920
// 128-byte rows 109 / 115, of at most 256 11.6 / 13.2 (the count is most of the difference).
// Past the line, counted up to 1024, 700 of them 413 / 402 and 339 / 290, 190 / 200, 16.2 / 18.8.
constexpr int kMaxCountedImages = 512;

// Division of values below 2^31 by a value fixed at the launch (scalar instructions only; a
// plain integer division is a vector sequence of some 40).
struct FixedDiv {
    uint32_t d, m;
    MPM_HD explicit FixedDiv(uint32_t v) : d(v), m(v > 1 ? (uint32_t)((UINT64_C(1) << 32) / v) : UINT32_MAX) {}
    MPM_HD int operator()(int v) const
    {
        const uint32_t q = (uint32_t)((uint64_t)(uint32_t)v * m >> 32);  // at most one too small
        return (int)(q + ((uint32_t)v - q * d >= d ? 1u : 0u));
    }
};

// The image at place i of the batch's order: eight interleaved runs (image 0, 8, 16, ...,
// then 1, 9, ...), so that the eight groups work on neighbouring images at a time.
MPM_HD int work_place(int i, const FixedDiv& run)  // run: max(1, B / 8)
{
    const int k = run(i);
    return k < 8 ? k + 8 * (i - k * (int)run.d) : i;
}

MPM_HD int work_items(WorkOrder order, int nb)
{
    return order == kOrderBand ? nb : order == kOrderSymmetric ? nb * (nb + 1) / 2 : nb * nb;
}

MPM_HD int uniform(int v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(v);
#else
    return v;
#endif
}

// A batch of equal images of nb blocks, as the launch passes it.
struct WorkShape {
    FixedDiv per, nb, rest, run;  // items of an image, its blocks, its items but the diagonal ones, B / 8
    MPM_HD WorkShape(WorkOrder order, int B, int blocks)
        : per((uint32_t)work_items(order, blocks)), nb((uint32_t)blocks),
          rest((uint32_t)(work_items(order, blocks) > blocks ? work_items(order, blocks) - blocks : 1)),
          run((uint32_t)(B >= 8 ? B / 8 : 1))
    {
    }
};

// Items and block rows (diagonal blocks) of the images before place b: tabulated (TAB), or
// of equal images.
template <bool TAB>
struct WorkCounts {
    const WorkShape& shape;
    const int32_t* items_tab;
    const int32_t* diags_tab;
    MPM_HD int items(int b) const { return TAB ? uniform(items_tab[b]) : b * (int)shape.per.d; }
    MPM_HD int diags(int b) const { return TAB ? uniform(diags_tab[b]) : b * (int)shape.nb.d; }
};

// A group's share, and the diagonal blocks it leaves to the half-block launch: those with
// index dstart and up (counted over the batch), the share's last ndef.
struct WorkShare {
    int lo, cnt;
    int dstart, ndef;
};

// The image that holds position p of the order (p below the batch's total).
template <bool TAB>
MPM_HD int work_image(const WorkCounts<TAB>& c, int B, int p)
{
    if constexpr (!TAB) return c.shape.per(p);
    int lo = 0, hi = B - 1;
    while (lo < hi) {  // the last image that starts at or before p holds it (empty ones before it start there too)
        const int mid = (lo + hi + 1) / 2;
        if (c.items(mid) <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Diagonal blocks at positions below p (symmetric order: each row starts with its own).
template <bool TAB>
MPM_HD int work_diags_before(const WorkCounts<TAB>& c, int B, int p)
{
    if (p >= c.items(B)) return c.diags(B);
    const int b = work_image(c, B, p);
    const int nb = c.diags(b + 1) - c.diags(b);
    int w = p - c.items(b), q = 0;
    while (w > 0) {
        w -= nb - q;
        ++q;
    }
    return c.diags(b) + q;
}

// Group g of 2^log_groups. When the share's items leave a last round of 0 < 2m <= slots
// after at least one whole round (`lone`, and every share has two slots an item: or are m
// diagonal blocks and no more), and it has at least m diagonal blocks, its last m are deferred
// (`split`).
template <bool TAB>
MPM_HD WorkShare work_share(const WorkCounts<TAB>& c, int B, int g, int log_groups, int slots, bool split,
                            bool lone = false)
{
    const int64_t total = c.items(B);
    WorkShare s;
    s.lo = (int)(total * g >> log_groups);
    const int hi = (int)(total * (g + 1) >> log_groups);
    s.cnt = hi - s.lo;
    s.ndef = 0;
    s.dstart = 0;
    lone = lone && 2 * ((total + (1 << log_groups) - 1) >> log_groups) <= slots;
    if (split && (lone || s.cnt > slots)) {
        const int m = s.cnt % slots;
        if (m > 0 && 2 * m <= slots) {
            const int dhi = work_diags_before(c, B, hi);
            if (dhi - work_diags_before(c, B, s.lo) >= m) {
                s.ndef = m;
                s.dstart = dhi - m;
            }
        }
    }
    return s;
}

struct WorkBlock {
    int b, q, t;  // image, query block, candidate tile (band order: the block's own)
};

constexpr int kWaveLanes = 64;

// The r-th item of the share that is not deferred (r < cnt - ndef). `from`: an image at or
// before the item's, to start looking at. On the device a whole wave calls it with the same
// arguments where images are tabulated; elsewhere each lane may ask for another item.
template <WorkOrder ORDER, bool SPLIT, bool TAB>
MPM_HD WorkBlock work_block(const WorkCounts<TAB>& c, const WorkShare& s, int r, int from)
{
    // Item r of a share with deferred diagonals stands at position lo + r of the order
    // without them; image b starts there at items(b) less the deferred blocks before it.
    const int p = s.lo + r;
    const bool defers = SPLIT && s.ndef > 0;
    WorkBlock k;
    int w;
    const int per = (int)c.shape.per.d, nbs = (int)c.shape.nb.d;
    if constexpr (!TAB) {
        if (!defers) {
            k.b = c.shape.per(p);
            w = p - k.b * per;
        } else {
            const int bs = c.shape.nb(s.dstart);  // the image with the first deferred block
            const int after = (bs + 1) * per - ((bs + 1) * nbs - s.dstart);  // start of image bs + 1
            if (p < after) {
                const int b = c.shape.per(p);
                k.b = b < bs ? b : bs;
                w = p - k.b * per;
            } else {  // images without any of their diagonals (at least one item each: p is one)
                const int past = c.shape.rest(p - after);
                k.b = bs + 1 + past;
                w = p - after - past * (int)c.shape.rest.d;
            }
        }
    } else {
        int b = from;
        int start;
#if defined(__HIP_DEVICE_COMPILE__)
        // 64 images at a time, one a lane (one after the other, a batch of one-block images cost
        // each item as many reads as its group has slots). The entry past the last image lies
        // past p, so the first one that does is found before any entry that was never written.
        const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        for (;;) {
            const int i = b + lane < kMaxCountedImages ? b + lane : kMaxCountedImages;
            const int di = c.diags_tab[i];
            const int at = c.items_tab[i] - (defers && di > s.dstart ? di - s.dstart : 0);
            const uint64_t past = __ballot(at > p);
            if (past != 0) {
                const int f = (int)__builtin_ctzll(past);
                b += f - 1;
                start = __builtin_amdgcn_readlane(at, f - 1);  // f >= 1: `from` starts at or before p
                break;
            }
            b += kWaveLanes - 1;
        }
#else
        start = c.items(b) - (defers && c.diags(b) > s.dstart ? c.diags(b) - s.dstart : 0);
        for (;;) {
            const int next = c.items(b + 1) - (defers && c.diags(b + 1) > s.dstart ? c.diags(b + 1) - s.dstart : 0);
            if (p < next) break;
            start = next;
            ++b;
        }
#endif
        k.b = b;
        w = p - start;
    }
    const int nb = TAB ? c.diags(k.b + 1) - c.diags(k.b) : nbs;
    if constexpr (ORDER == kOrderBand) {
        k.q = k.t = w;
    } else if constexpr (ORDER == kOrderFull) {
        k.q = TAB ? w / nb : c.shape.nb(w);
        k.t = w - k.q * nb;
    } else {
        const int q0 = defers ? s.dstart - c.diags(k.b) : nb;  // rows from q0 on are without their diagonal
        int q = 0;
        for (;;) {
            const int len = nb - q - (q >= q0 ? 1 : 0);
            if (w < len) break;
            w -= len;
            ++q;
        }
        k.q = q;
        k.t = q + w + (q >= q0 ? 1 : 0);
    }
    return k;
}

// Deferred diagonal block e of the share (e < ndef).
template <bool TAB>
MPM_HD WorkBlock work_deferred(const WorkCounts<TAB>& c, int B, const WorkShare& s, int e)
{
    const int d = s.dstart + e;
    WorkBlock k;
    if constexpr (!TAB) {
        k.b = c.shape.nb(d);
    } else {
        int lo = 0, hi = B - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (c.diags(mid) <= d) lo = mid;
            else hi = mid - 1;
        }
        k.b = lo;
    }
    k.q = k.t = d - c.diags(k.b);
    return k;
}

}  // namespace mpm
