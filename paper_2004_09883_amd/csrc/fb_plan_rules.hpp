// fb_plan_rules.hpp -- compile-time and host-side rules of the plan: the radix
// list of an axis length and the launch geometry of a pencil pass.
//
// Radix list of n = 2^a 3^b, in the order the stages are applied to the data:
// b threes, then floor(a/4) sixteens, then 2^(a mod 4) when a mod 4 > 0
// (e.g. 512 -> 16,16,2; 768 -> 3,16,16; 64 -> 16,4; 2304 -> 3,3,16,16).
// A 3D axis may have any such length up to 4096.
#pragma once
#include <stdint.h>

namespace fb {

struct RadixPlan {
    int count;
    int r[16];
    int ns[16];     // product of the radices before stage s
    int twoff[16];  // offset of stage s in the per-axis twiddle table
    int twlen;      // total twiddle entries
};

constexpr RadixPlan radix_plan(int n)
{
    RadixPlan p{};
    p.count = 0;
    int a = 0, b = 0, m = n;
    while (m > 1 && m % 3 == 0) { m /= 3; b++; }
    while (m > 1 && m % 2 == 0) { m /= 2; a++; }
    if (m != 1 || n < 1) { p.count = -1; return p; }
    for (int i = 0; i < b; i++) p.r[p.count++] = 3;
    for (int i = 0; i < a / 4; i++) p.r[p.count++] = 16;
    if (a % 4) p.r[p.count++] = 1 << (a % 4);
    int ns = 1, off = 0;
    for (int s = 0; s < p.count; s++) {
        p.ns[s] = ns;
        p.twoff[s] = off;
        if (ns > 1) off += (p.r[s] - 1) * ns;  // entries w_{ns r}^(q k), 1<=q<r, k<ns
        ns *= p.r[s];
    }
    p.twlen = off;
    return p;
}

// True when n is an axis length the 3D passes support: 2^a 3^b, 1..4096.
constexpr bool supported_length(int64_t n)
{
    if (n < 1 || n > 4096) return false;
    int64_t m = n;
    while (m % 3 == 0) m /= 3;
    while (m % 2 == 0) m /= 2;
    return m == 1;
}

// True for the lengths 2^a and 3 * 2^a (the batched form's pass lengths).
constexpr bool supported_length_b1(int64_t n)
{
    if (n < 1 || n > 4096) return false;
    int64_t m = n;
    if (m % 3 == 0) m /= 3;
    while (m % 2 == 0) m /= 2;
    return m == 1;
}

// Threads that cooperate on one pencil: each holds about 16 elements (n/16
// threads when 16 divides n; one thread for the short lengths up to 32;
// otherwise ceil(n/16), and the stages whose butterfly count is not a
// multiple of it leave the last round part-filled).  Lengths with repeated
// radix-3 stages take the count of their stage groups instead (group_plan).
constexpr int threads_per_pencil(int n) { return (n % 16 == 0) ? n / 16 : n <= 32 ? 1 : (n + 15) / 16; }

// Whether a pass works its stages in groups (group_plan): the lengths whose
// radix list repeats the radix 3, on the vector units.  54 and 72 points stay
// stage by stage in contiguous passes: as groups they take 3 threads instead
// of 4 and 5, whose loads lie further apart (72: 16.8 -> 19.0 us); the shorter
// ones move their tiles as one block, where that does not matter.
constexpr bool grouped(int n, bool contig, bool mx) { return n % 9 == 0 && !mx && (!contig || n <= 48 || n >= 81); }

// Stages worked together in registers.  A group of consecutive stages of
// radices R_s .. R_e and product G is a set of N/G independent butterflies of
// G elements (butterfly b reads x[b + g N/G], g < G), so a thread that holds
// those G elements runs all the group's stages without an exchange; the
// operations and their order on every element are the stages' own.
//
// Why: with one group per stage, 216 = 3,3,3,8 makes three LDS exchanges of
// three- or eight-element butterflies; as (3,3),(3,8) it makes one.  The
// groups are the fewest whose products, and whose elements per thread, stay
// within 27 (108 registers of complex128 or of a complex64 pair); among the
// splits of that many groups the rule takes one that wastes at most a fifth of
// the lanes' work, if it can with whole rounds of loads (a part-filled round
// is a branch, and its loads wait behind the others: 216 points on 9 threads,
// 24 butterflies in 3 rounds, took 31 us where 12 threads take 23), and then
// the one nearest 18 elements per thread.  One group per stage (fuse = false)
// everywhere else: the lengths 2^a and 3 2^a exchange between radix-16 stages,
// and matrix-core stages work on one stage at a time.
//
// Measured on 64 MiB complex128 grids against one group per stage, same bits:
// strided 81 points 21.9 -> 14.3 us, 144: 20.8 -> 14.5, 216: 29.3 -> 22.6,
// 1458: 35.7 -> 25.3; contiguous 162: 26.2 -> 18.3; complex64 contiguous 729
// (32 MiB): 20.0 -> 11.7.
constexpr int kMaxGroupElems = 27;
constexpr int kGoodGroupElems = 18;
struct GroupPlan {
    int count;
    int first[16];  // first stage of the group
    int nst[16];    // stages of the group
    int g[16];      // product of their radices
    int ns[16];     // product of the radices before the group
    int threads;    // threads per pencil
    int elems;      // largest number of elements one thread holds
};

constexpr GroupPlan groups_of_mask(const RadixPlan &rp, unsigned mask)   // bit i: a group ends after stage i
{
    GroupPlan p{};
    p.count = 0;
    for (int s = 0; s < rp.count; s++) {
        if (s == 0 || (mask >> (s - 1) & 1)) {
            p.first[p.count] = s;
            p.nst[p.count] = 0;
            p.g[p.count] = 1;
            p.ns[p.count] = rp.ns[s];
            p.count++;
        }
        p.nst[p.count - 1]++;
        p.g[p.count - 1] *= rp.r[s];
    }
    return p;
}

constexpr GroupPlan group_plan(int n, bool fuse)
{
    const RadixPlan rp = radix_plan(n);
    GroupPlan best = groups_of_mask(rp, ~0u);
    best.threads = threads_per_pencil(n);
    for (int i = 0; i < best.count; i++) {
        const int u = (n / best.g[i] + best.threads - 1) / best.threads;
        if (u * best.g[i] > best.elems) best.elems = u * best.g[i];
    }
    if (!fuse) return best;
    best.threads = 0;
    int best_key[4] = {0, 0, 0, 0};
    for (unsigned mask = 0; mask < (1u << (rp.count - 1)); mask++) {
        GroupPlan p = groups_of_mask(rp, mask);
        bool fits = true;
        for (int i = 0; i < p.count; i++) fits = fits && p.g[i] <= kMaxGroupElems;
        if (!fits || (best.threads && p.count > best.count)) continue;
        for (int t = (n + kMaxGroupElems - 1) / kMaxGroupElems; t <= n / 2 || t == 1; t++) {
            int elems = 0, work = 0;
            for (int i = 0; i < p.count; i++) {
                const int u = (n / p.g[i] + t - 1) / t;
                if (u * p.g[i] > elems) elems = u * p.g[i];
                work += u * p.g[i] * t;
            }
            if (elems > kMaxGroupElems) continue;
            const int waste = work / p.count * 1000 / n - 1000;   // per mille
            const int ragged = (n / p.g[0]) % t != 0 && n / p.g[0] > t ? 1 : 0;
            const int off = elems > kGoodGroupElems ? elems - kGoodGroupElems : kGoodGroupElems - elems;
            // in this order: few wasted lanes, distance, all wasted lanes, more threads
            const int key[4] = {waste > 200 ? waste : ragged, off, waste, -t};
            if (best.threads && p.count == best.count) {
                int c = 0;
                while (c < 3 && key[c] == best_key[c]) c++;
                if (key[c] >= best_key[c]) continue;
            }
            p.threads = t;
            p.elems = elems;
            best = p;
            for (int c = 0; c < 4; c++) best_key[c] = key[c];
        }
    }
    return best;
}

// Pencils that one pass can have: their numbers, a tile's overhang included,
// fit 32 bits.  A batch of more images than that splits them over groups
// (2^31 images of 2 x 2 are 64 GiB).
#ifndef FB_MAX_PENCILS
#define FB_MAX_PENCILS ((int64_t(1) << 32) - (1 << 16))
#endif
constexpr int64_t batch_images_per_group(int64_t side) { return (FB_MAX_PENCILS - 1) / side; }

// LDS row of one pencil: one pad element every 16 (breaks the stride-R
// pattern of the first exchange) and an odd total (consecutive pencils land
// on different banks).
constexpr int lds_pencil_stride(int n)
{
    int s = n + n / 16;
    return (s % 2 == 0) ? s + 1 : s;
}

// Build-time tuning knobs (defaults are the measured best on MI355X).
#ifndef FB_LDS_CONTIG_KB
#define FB_LDS_CONTIG_KB 40   // contiguous complex64 passes
#endif
#ifndef FB_LDS_CONTIG16_KB
#define FB_LDS_CONTIG16_KB 20   // contiguous complex128 passes: one wavefront per tile at n = 128, 256
#endif
#ifndef FB_LDS_CONTIG_MX_KB
#define FB_LDS_CONTIG_MX_KB 20   // contiguous complex64 matrix-core passes
#endif
// Complex128 vector-unit passes exchange real and imaginary parts through
// LDS one after the other (FB_SPLIT_EXCHANGE = 1): half the LDS per tile, so
// more tiles fit a CU; their budgets are then FB_LDS_SPLIT_*_KB.
#ifndef FB_SPLIT_EXCHANGE
#define FB_SPLIT_EXCHANGE 1
#endif
#ifndef FB_SPLIT_MAX_N
#define FB_SPLIT_MAX_N 256   // longer passes keep the one-round exchange
#endif
#ifndef FB_LDS_SPLIT_CONTIG_KB
#define FB_LDS_SPLIT_CONTIG_KB 10
#endif
#ifndef FB_LDS_SPLIT_STRIDED_KB
#define FB_LDS_SPLIT_STRIDED_KB 36
#endif
#ifndef FB_LDS_STRIDED_KB
#define FB_LDS_STRIDED_KB 72
#endif
#ifndef FB_LDS_STRIDED_MX_KB
#define FB_LDS_STRIDED_MX_KB 36   // strided complex64 matrix-core passes: half-size tiles
#endif
#ifndef FB_STRIDED_P16
#define FB_STRIDED_P16 16   // target pencils per workgroup, strided complex128
#endif
#ifndef FB_STRIDED_P8
#define FB_STRIDED_P8 32    // target pencils per workgroup, strided complex64
#endif
#ifndef FB_CONTIG_THREADS
#define FB_CONTIG_THREADS 256
#endif

constexpr int lds_budget_bytes(bool contig, int esize, bool mx = false)
{
    return !contig     ? (mx ? FB_LDS_STRIDED_MX_KB : FB_LDS_STRIDED_KB) * 1024
           : esize == 16 ? FB_LDS_CONTIG16_KB * 1024
           : mx          ? FB_LDS_CONTIG_MX_KB * 1024
                         : FB_LDS_CONTIG_KB * 1024;
}

constexpr int gcd_int(int a, int b) { return b == 0 ? a : gcd_int(b, a % b); }

// split: the tile's LDS holds one real part per element (8 bytes) at a time
constexpr bool pencils_fit(int P, int n, bool contig, int esize, bool mx = false, bool split = false)
{
    const int elem = split ? 8 : esize;
    const int budget = split ? (contig ? FB_LDS_SPLIT_CONTIG_KB : FB_LDS_SPLIT_STRIDED_KB) * 1024
                             : lds_budget_bytes(contig, esize, mx);
    return P * threads_per_pencil(n) <= 1024 && P * lds_pencil_stride(n) * elem <= budget;
}

// Pencils per workgroup.  Contiguous passes aim for 256 threads; strided
// passes aim for 16 (c128) / 32 (c64) adjacent pencils so that every row
// access is a 256-byte segment.  P is then moved to a multiple of
// 64 / gcd(T, 64) so that the workgroup is whole wavefronts, when that fits;
// finally it is capped by 1024 threads and by the LDS budget.  A
// matrix-core pass (mx) takes the budget of its own kind only where the tile
// stays whole wavefronts (which the matrix-core stages need); otherwise that
// of the vector-unit pass.
constexpr int pencils_per_wg_b(int n, bool contig, int esize, bool mx, bool split)
{
    const int T = threads_per_pencil(n);
    int P = contig ? (FB_CONTIG_THREADS / T > 0 ? FB_CONTIG_THREADS / T : 1)
                   : (esize == 16 ? FB_STRIDED_P16 : FB_STRIDED_P8);
    if (!contig && T == 1) P = 64;
    const int m = 64 / gcd_int(T, 64);
    if (P % m) {
        const int down = (P / m) * m, up = down + m;
        if (down > 0) P = down;
        else if (pencils_fit(up, n, contig, esize, mx, split)) P = up;
    }
    while (P > 1 && !pencils_fit(P, n, contig, esize, mx, split)) P /= 2;
    return P;
}
// Pencils per workgroup of a pass with stage groups, whose thread counts are
// odd: the count that leaves the fewest lanes of the tile's last wavefront
// idle, within the LDS budget and 256 (contiguous) or 512 threads.  Strided
// tiles keep whole 128-byte row segments, two of them where that fits (as
// the other strided passes, which lose a tenth with one).
constexpr int grouped_pencils(int n, int threads, bool contig, int esize, bool split)
{
    const int elem = split ? 8 : esize;
    const int budget = (contig ? 20 : split ? FB_LDS_SPLIT_STRIDED_KB : FB_LDS_STRIDED_KB) * 1024;
    const int max_threads = contig ? 256 : 512;
    for (int step = contig ? 1 : 256 / esize; step >= 1; step /= 2) {
        int best = 0, best_idle = 0;   // idle lanes per mille
        for (int p = step; p * threads <= max_threads && p * lds_pencil_stride(n) * elem <= budget;
             p += contig ? 1 : 128 / esize) {
            const int lanes = (p * threads + 63) / 64 * 64;
            const int idle = (lanes - p * threads) * 1000 / lanes / 20 * 20;
            if (best == 0 || idle < best_idle) {
                best = p;
                best_idle = idle;
            }
        }
        if (best) return best;
    }
    return 1;
}

// Wavefronts of a contiguous pass from which its tiles move as one block
// (block_to_rows in fb_pass.hpp) instead of pencil by pencil; 0: never.  A pass
// with few wavefronts per CU is one latency after another, and the LDS round
// trips of a block add theirs; with more of them the accesses count, and they
// count most where they are non-temporal.  one_group: all stages in registers.
//
// Measured (block / pencil-wise time; 1 to 500 MiB; repeated on the same grid /
// on grids that come from memory):
//  - non-temporal complex128: 6 to 36 points 0.9 to 1.5 / 0.5 to 1.0 at 256
//    wavefronts (24 and 32 points 1.1 to 1.5 / 1.05), 0.3 to 0.9 / 0.2 to 0.7 at
//    1024; 48 to 72: 0.85 to 1.06 / 0.73 to 1.0 at 1024; up to 243 points 1.0 to
//    1.5 below 2048, 0.5 to 0.95 from there; 288, 324: 1.05 at 5462, 0.9 from
//    8192; 432, 486: 1.0 at 8192, 0.93 to 0.99 from 16384.  2 points 1.1 at 2048,
//    0.8 at 4096; 3: 0.85 at 2048; 4: 1.0 / 0.9 at 1024;
//  - non-temporal complex64: 6 to 16 points 0.7 to 1.2 / 0.4 to 1.0 at 1024; 18 to
//    48: 0.5 to 1.3 / 0.4 to 0.7 at 512, 54 to 72 and 96: 0.7 to 1.0 at 768; up to
//    243 points 1.2 to 1.5 at 600, 0.8 to 1.1 at 1536, 0.6 to 0.9 from 2300 on;
//    288 to 486: 1.0 to 1.4 at 2048, 0.85 to 1.1 from 4096.  2 points 1.1 to 1.2 at
//    any size, 3: 1.0, 4: 0.8 to 1.0 from 4096;
//  - cached complex128: 8 to 27 points in one group 1.0 to 1.5 at 512, 0.6 to 0.9
//    from 1024 (16 points 0.92 and 0.99 at 512); 24 and 36: 1.1 to 1.2 at 1024, 0.8 to 0.98 from 2048; 3: 1.1 at
//    2048, 0.9 at 4096; 2, 32 and 48: 1.0 to 1.4 at any size;
//  - cached complex64: 0.65 to 0.96 from 2048 on (9 and 36 points 1.1 to 1.4 at
//    512, 16 and 32 points 0.9 to 1.0 at 1024; 18: 1.1 to 1.2 at 2048, 1.0 and 0.93 at 4096); 2, 3, 4 and 27: 1.0 to
//    1.8 at any size;
//  - cached passes with several outputs, which store more than they load: 5 steps
//    as a whole 0.92 to 1.0 from 512 (complex128, up to 18 points; longer ones 1.0
//    to 1.08) and 1024 (complex64, 0.93 to 1.0; 9, 18 and 36 points 0.94 to 0.99
//    from 512).
constexpr int block_waves(int n, int esize, bool one_group, bool nt, bool multi)
{
    if (esize == 16) {
        if (nt && n <= 4) return n == 2 ? 4096 : n == 3 ? 2048 : 1024;
        if (nt && n <= 36) return n == 24 || n == 32 ? 512 : 256;
        if (nt) return n <= 72 ? 1024 : n <= 243 ? 2048 : n < 400 ? 8192 : 16384;
        if (multi) return n == 2 || n > 18 ? 0 : 512;
        if (n > 36 || n == 2 || n == 32) return 0;
        return n == 3 ? 4096 : n == 4 ? 2048 : n == 16 ? 512 : one_group || n <= 16 ? 1024 : 2048;
    }
    if (nt && n <= 48) return n <= 3 ? 0 : n == 4 ? 4096 : n <= 16 ? 1024 : multi && n == 27 ? 256 : 512;
    if (nt) return n <= 72 || n == 96 ? 768 : n <= 243 ? 1536 : 4096;
    if (n <= 4 || n > 48) return 0;
    if (multi) return n == 9 || n == 18 || n == 36 ? 512 : 1024;
    return n == 27 ? 0 : n == 18 ? 4096 : n == 16 || n == 32 ? 1024 : 2048;
}

// Pencils per workgroup of the long strided complex128 passes (has_wide
// below): 8, a whole 128-byte line per row, while the workgroup's LDS (one
// real part per element) and threads allow it, then 4.  More than 512 threads
// leave 128 registers each, enough for 18 elements per thread.
constexpr int wide_pencils(int n, int threads, int elems)
{
    int p = 8;
    while (p > 1 && (p * threads > (elems <= 18 ? 1024 : 512) || p * lds_pencil_stride(n) * 8 > 150 * 1024)) p /= 2;
    return p;
}

// Long strided complex128 passes have a second instance, with tiles of whole
// 128-byte lines per row (wide_pencils).  With the 72 KB of one-round tiles a
// row segment is 64 bytes at 1024 points and 16 at 4096, and the lines that
// neighbouring tiles share have left the L2 before their turn.  A two-round
// exchange halves the tile's LDS, and one tile may take most of a CU's.
constexpr bool has_wide(int n, bool contig) { return FB_SPLIT_EXCHANGE && !contig && n > 512; }

// Whether a pass of `npencils` pencils takes its wide instance (`pencils` per
// tile); `inner` pencils lie side by side, rows `inner` elements apart or more;
// nt: non-temporal accesses.  The wide tiles are fewer and larger: they need
// enough of them for the 256 CUs, and whole lines (rows that start inside a
// line make two of every segment, and the caches join narrow segments well).
//
// Measured (wide / narrow time; 22 lengths, 16 to 65536 pencils, x and y passes,
// grids in the caches and out of them):
//  - fewer than 128 tiles: 1.0 to 2.5 everywhere;
//  - up to 1024 points, where narrow rows are 64 bytes: 0.9 to 1.8 with cached
//    accesses and 1.0 to 1.6 with rows inside lines.  Non-temporal 0.67 to 0.94
//    for 648 and 729 points from 160 tiles on, 0.70 to 0.98 for 972 and 1024 from
//    360; 576, 768 and 864 points 0.86 to 1.10 from 480, above the last-level
//    cache 1.04 to 1.17, and 0.80 to 1.05 from 288 MiB on with rows 64 KB apart;
//  - past 1024 points, whole lines: non-temporal 0.35 to 0.97 from 160 tiles on
//    (128 for 2187 and 2916 points, 0.81 to 0.88).  Cached, 1536, 1728 and 2048
//    points 0.41 to 0.99 from 128 MiB on, 0.89 to 1.01 where the tiles are one
//    per CU (2048 x 2048: 35 -> 31 us), else 0.9 to 1.4; the others 0.28 to 1.0,
//    but 1.0 to 1.4 between 300 and 800 tiles while the caches hold the grid
//    (1152 x 3072: 27.6 / 32.9 us there and 32 / 25 us from memory at 2048);
//  - rows inside lines: 0.77 to 0.91 for 1152, 1296, 1458, 2048 and 3072 points
//    from 192 MiB on (1.1 to 1.6 below), 0.9 to 1.4 for 1536 and 1728 points at
//    any size, for the others 0.45 to 0.95, with a few of up to 1.27 around 300
//    and 550 tiles; rows of fewer than 9 (1152 .. 3072) or 4 pencils 1.1 to 1.4.
constexpr bool wide_pays(int n, int pencils, int64_t npencils, int64_t inner, bool nt)
{
    constexpr int64_t MiB = 1 << 20;
    const int64_t tiles = (npencils + pencils - 1) / pencils, bytes = npencils * n * 16;
    const bool whole = inner % 8 == 0;
    if (n <= 1024) {
        if (!whole || !nt) return false;
        if (n % 96 == 0) return tiles >= 480 && (bytes < 192 * MiB || (bytes >= 288 * MiB && inner >= 4096));
        return tiles >= (n < 900 ? 160 : 360);
    }
    const int64_t least = n % 729 == 0 ? 128 : 160;
    if (whole) {
        if (!nt && (n == 1536 || n == 1728 || n == 2048))
            return bytes >= 128 * MiB || (tiles >= 224 && tiles <= 256);
        return tiles >= least;
    }
    if (n < 1500 || n == 2048 || n == 3072) return bytes >= 192 * MiB && inner >= 9;
    return n >= 1944 && tiles >= least && inner >= 4;
}

// Whether a complex128 pass exchanges real and imaginary parts in two rounds:
// up to 256 points it lets more tiles share a CU (at 257 .. 512 points one
// round was faster, the 512-point x pass 196 against 215 us); the wide strided
// tiles always do.
constexpr bool split_exchange(int n) { return FB_SPLIT_EXCHANGE && n <= FB_SPLIT_MAX_N; }

constexpr int pencils_per_wg(int n, bool contig, int esize, bool mx = false, bool split = false, bool groups = true)
{
    if (split && !contig && n > 512) {
        const GroupPlan gp = group_plan(n, grouped(n, contig, mx));
        return wide_pencils(n, gp.threads, gp.elems);
    }
    if (groups && grouped(n, contig, mx)) return grouped_pencils(n, group_plan(n, true).threads, contig, esize, split);
    if (mx) {
        const int P = pencils_per_wg_b(n, contig, esize, true, split);
        if ((P * threads_per_pencil(n)) % 64 == 0) return P;
    }
    return pencils_per_wg_b(n, contig, esize, false, split);
}

}  // namespace fb
