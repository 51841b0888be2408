// Encoder for long rows (the ones that neither row-resident kernel takes): every pass over a row is spread
// over many workgroups, the per-row state lives in the workspace, and the stages are five launches on the
// caller's stream:
//
//   sample    per row: up to 4096 evenly spread 16-byte chunks.  Their histogram gives a lower bound that a
//             little more than k elements reach, and a table that maps the elements above it to at
//             most 2048 "fine bins" of about equal population
//   compact   per tile of up to 16384 elements: ordered compaction of everything at or above the bound into a list
//             segment, the tile's histogram over the fine bins (as "entries at or above the bin"), and the
//             list positions arranged by fine bin
//   bounds    per row, by up to eight workgroups: the tiles' histograms are summed; the top-K cut (ATKF, Sec. 3.1) and the first and last
//             element of every block (MS, Sec. 3.2) are order statistics whose fine bin is found in the sums and
//             which are resolved among the few members of that bin, or by a sort of a bin of many; rows that do not fit are redone by the
//             generic encoder, in the row's last workgroup to find that out
//   split     per tile: block of every entry, stable split by block (ascending index inside a block), integer
//             ABQ sums (Sec. 3.2.1); the last workgroup of a row chooses the bitwidths and bit offsets
//   pack      one window of stream words per workgroup, written straight to its place in the stream when
//             the batch has at most 256 rows (every workgroup adds up the word counts of the rows before its own)
//
// A sample decides only how long the list is and how full the bins are, never the result: the counts are exact.
//
// What bounds it: launches and the latency of dependent loads, not bandwidth.  Every launch costs 2.5 to 4 us
// before it does anything and a workgroup lives three to six memory round trips, so the stages were
// chosen for their number: counting exactly before compacting, separate block counts, sums and choice, and a
// final gather made ten launches.  One atomic per entry on a table in memory is no way to
// join the tiles' histograms (29 G atomics/s: 100 us for 3 M of them); the per-tile tables cost 8 KB
// per tile, written once.  Inside a stage the lanes' LDS lookups are written as straight-line code for several
// entries at once: behind branches they wait for each other (split kernel 68 -> 41 us on 32 maps of 401408 at the time, together with four instead of
// eight entries per thread, which spill nothing, and the choice of the guard taken outside the entry loop).
// Measured (us, fp32 [1 x 200704] and [32 x 401408] keep 0.2, 16 + 16 blocks; every step on inputs that no cache holds): sample 12.4 and 14.9,
// compact 6.5 and 21.6, bounds 11.3 and 17.8, split 14.0 and 36.2, pack 6.3 and 22.4.  Where the row is in a cache the sample takes 6 and 10; the
// calls then take 43.1 and 111.7, with CSR blocks and decode 142.  Before the changes that the stages' comments name (in a cache): sample 9.5 and
// 13, compact 6 and 29, bounds 15.7 and 24, split 15 and 41; the calls 53 and 135, with CSR blocks and decode 165.
//
// Order: comp = key << w | (2^w - 1 - index): larger comp = larger magnitude, then lower index.  c32 is
// its leading 31 (fp32: the key) or 32 bits (bf16: the key and the first 17 bits of the inverted
// index), so that bins can cut through a run of equal bf16 keys.
#pragma once

#include <algorithm>

#include "slicer_common.hpp"
#include "slicer_encode_generic.hpp"

namespace slicer {

constexpr int kTileThreads = 512;   // a compact / split workgroup handles a tile of up to 16384 elements
constexpr int kMaxTab = 510, kTabSize = kMaxTab + 2;        // sample bins with fine bins of their own: 16 octaves above the bound
// Fine bins per row, a template parameter (FB) of the stages.  A batch of up to 256 rows has a CU for every row and takes the
// many bins, few members each, and 1024 threads per row where a stage works on whole rows; there a row's latency counts.
// In a larger batch the rows wait for each other and what counts is a row's cost.  4096 bins had half the members a bin and tables of
// twice the size: the bounds stage's sums of fp32 [32 x 401408] took 5.5 us instead of 3.5, and compact's LDS let three workgroups on a CU instead
// of four, 768 of 800 at once.
constexpr int kFBWide = 2048, kFBNarrow = 1024;
constexpr int lr_row_threads(int FB) { return FB == kFBWide ? 1024 : 256; }    // of the per-row stages
constexpr int kSampleBins = 8192;   // 32 bins per octave
// members of the bins that hold order statistics, per row (BIG: for lists of many entries, at one row a CU)
constexpr int lr_mem_cap(int FB, bool BIG) { return FB == kFBWide ? (BIG ? 16384 : 6144) : 1536; }
constexpr int kPackWords = 1024;    // stream words per pack workgroup
constexpr u64 kTop = 1ull << 63;

struct LargeArgs {
    const void* x;
    int64_t R, N, k;
    int M, Mn, w, nq;       // blocks of the positive / negative class
    int qlist[kMaxQ];
    double beta;
    u64 cap_words;
    u32 sample_target;      // see lr_sample_plan
    float sample_scale;
    int tile, S;            // elements of a tile, tiles per row
    bool dense;             // most wavefronts of the compact stage have more entries than kLrEntries
    int parts;              // workgroups that share a row in the bounds stage,
    int part_step;          // and how far apart they are in its grid
    u32 capL;               // list capacity per row
    uint16_t* tab;          // [R][kTabSize]  first fine bin of a sample bin | log2 of its number of fine bins << 12; one guard at either end
    u32* cum;               // [R][S][FB]     entries of the tile at or above the bin: positive | negative << 16
    u32* seg;               // [R][S][2]      list position of the tile's segment, positive | negative entries << 16
    uint8_t* L;             // [R][8 capL]    a row's list, see LrList (the generic encoder's list of the row has the same place)
    u32* rowst;             // [R][16]        see kSt*
    u32* redo;              // [R]            the row is left to the generic encoder (narrow tables only)
    u64* thr;               // [R][B2]        comp of the block's last element
    u32* vminb;             // [R][B2]        keys
    u32* vmaxb;
    u32* blk_start;         // [R][B2 + 1]
    u32* pair;              // [R][B2][S]     entries of the tile in this block and the blocks of its class before it
    u64* sums;              // [R][B2][nq + 1]  ABQ sums
    u32* qsel;              // [R][B2]
    float* inv_sel;         // [R][B2]
    u64* code_off;          // [R][B2 + 1]
    u32* bo_idx;            // [R][k]
    u32* bo_val;            // [R][k]
    u64* row_words;
    u32* slots;
    MetaView mv;
    Ladder lad;             // fixed multi-level mode
    int guard;              // 0: relative squared-error budget; 1: DS mismatch, greedy descent (beta = delta)
    // pack
    int pack_words;         // stream words per pack workgroup in the index section (<= kPackWords)
    int pack_words_code;    // ... from the first word with code bits on (fields there are short: fewer words per workgroup)
    int pack_words_ptr;     // ... up to the first word with column bits, where row pointers have windows of their own
    int nwin_ptr, nwin_idx, nwin;     // windows of row pointers alone; those and the ones that may lie in the index section; windows per row
    int direct;             // 1: words go to their place in the stream, 0: to the row's slot
    u32* stream;
    void* meta;
    // two-dimensional instances (n_cols > 0): row pointers and columns instead of flat indices
    int64_t n_rows, n_cols;
    int wp, wc;
};

// Elements per tile of the long-row stages, a multiple of 512 from 4608 to 16384: 8192 while these do
// not fill the chip, and in large batches where they leave out a quarter or more of what long tiles would cover (bf16 [4096 x 8192] 461 -> 428 us, fp32
// [4096 x 20480] 529 -> 510; with a sixth left out the added tiles cost more: bf16 [4096 x 33001] 758 -> 826).  Between the two as many tiles as
// can run at once, four a CU, but no more than tiles of 8192 would be.  Rows of many tiles are cut so that every CU has as many as
// the next one: fp32 [32 x 401408], 32 tiles a row, 120.5 us, with 49 tiles 126.0, with 25 134.7; [16 x 401408] 32 tiles 84.5 us, 49 92,
// 25 97; [4 x 401408] 64 tiles 61.6, 49 65.2 (rows of few tiles gain less by it than they lose: [32 x 100352] 8 tiles 58.5, 13 54.3).  A
// row has at most 128 tiles where these are no longer than 16384: one workgroup adds up their tables ([1 x 2000000] 245 tiles
// 89 us, 128 76).
inline int large_tile(int64_t rows, int64_t row_len)
{
    const int64_t n8 = (row_len + 8191) / 8192, n16 = (row_len + 16383) / 16384;
    auto of = [&](int64_t S) { return (int)((row_len + 512 * S - 1) / (512 * S) * 512); };
    if (rows > kScanRows) return n8 == 1 || n8 == 3 ? 8192 : of(n16);
    const int64_t most = std::max<int64_t>(128, n16);
    auto even = [&](int64_t per_cu, int64_t shortest) {          // tiles of a row where every CU has per_cu of them; 0: they would be too short, too long or few
        const int64_t S = 256 * per_cu / rows;
        return S >= 24 && S <= most && of(S) >= shortest && of(S) <= 16384 ? S : 0;
    };
    if (const int64_t S = even(4, 8192)) return of(S);
    if (const int64_t S = even(2, 8192)) return of(S);
    if (rows * n8 <= 256) {
        if (const int64_t S = even(1, 6144)) return of(S);       // (below the 8192 that the workspace's tables are sized for)
        return n8 <= most ? 8192 : of(most);
    }
    return of(std::max(n16, std::min({1024 / rows, n8, most})));
}

constexpr int kLrEntries = 640;      // room for a wavefront's entries in the compact stage

// What the sample stage aims at: how many of the sample's elements must reach the bound, i.e. the expected number of the k kept ones plus
// four standard deviations, taken as if the elements of a chunk were all alike; and the row's elements per sampled one.  (Of the
// row's chunks counted from its start: one that starts inside a chunk may have one more, which the margin covers.)
inline void lr_sample_plan(LargeArgs& a, int fine_bins, int epc)
{
    const int64_t Q = (a.N + epc - 1) / epc, room = fine_bins == kFBWide ? 4096 : 2048;
    const double G = (double)(Q < room ? Q : room), f = (double)a.k / (double)a.N;
    a.sample_target = (u32)(f * G * epc + 4.0 * epc * sqrt(G * f * (1.0 - f))) + 1u;
    a.sample_scale = (float)((double)a.N / (G * epc));
    // the line: fp32 [316 x 126280], expected 551 entries a wavefront, dense 783 us, else 768, [64 x 630000] 246 and 239; 591 entries 280 and 303, 252 and 284
    a.dense = (double)a.sample_target / (G * epc) * (a.tile / (kTileThreads / kWave)) > 0.9 * kLrEntries;
}

// words of a row's state.  kStFlag (encoded generically): written by compact, and by the bounds stage when no part of the row reads it any more
enum { kStT = 0, kStBlo, kStNb, kStCursor, kStTicket, kStFlag, kStNpos, kStNneg, kStLeft };

struct LrList {
    u32* raw;               // [capL]  fp32: the raw word; bf16: the raw half in the high 16 bits
    uint16_t* idx;          // [capL]  index relative to the tile
    uint16_t* pos;          // [capL]  positions inside the segment by fine bin, highest first, positive class first
    __device__ inline LrList(const LargeArgs& a, int64_t r)
    {
        raw = (u32*)(a.L + (size_t)r * 8u * a.capL);
        idx = (uint16_t*)(raw + a.capL);
        pos = idx + a.capL;
    }
};

template <int DT> struct LrOrder;
template <> struct LrOrder<0> { static constexpr int kSh = 18; static constexpr u32 kLeast = 1u; };
template <> struct LrOrder<1> { static constexpr int kSh = 19; static constexpr u32 kLeast = 1u << 17; };

template <int DT>
__device__ inline u32 lr_c32(u32 key, u32 idx, int w)
{
    if (DT == 0) return key;
    const u32 inv = ((1u << w) - 1u) - idx;
    return (key << 17) | (w >= 17 ? inv >> (w - 17) : inv << (17 - w));
}

// fine bin of an element at or above the bound: its sample bin's first one plus the leading bits inside the sample
// bin (the guards at the table's ends catch elements beyond its reach); no branch, so that the lookups of several entries overlap
template <int DT>
__device__ inline u32 lr_fine_bin(u32 cc, const uint16_t* tab, u32 Blo, u32 nb)
{
    constexpr int SH = LrOrder<DT>::kSh;
    const int d = (int)(cc >> SH) - (int)Blo + 1, hi = (int)nb + 1;
    const u32 t = tab[d < 0 ? 0 : d < hi ? d : hi];
    return (t & 0xFFFu) + (((cc << (32 - SH)) >> 1) >> (31u - (t >> 12)));
}

// raw element e of a 16-byte chunk (fp32: 0..3, bf16: 0..7)
template <int DT>
__device__ inline u32 chunk_elem(const uint4& v, int e)
{
    const int d = DT == 0 ? e : e >> 1;
    const u32 wd = d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
    return DT == 0 ? wd : ((e & 1) ? wd >> 16 : wd & 0xFFFFu);
}

__device__ inline u64 lr_comp(u32 key, u32 idx, int w) { return ((u64)key << w) | (u64)(((1u << w) - 1u) - idx); }

// ---- 1. sample ------------------------------------------------------------------------------------
template <int DT, int FB>
__global__ __launch_bounds__(lr_row_threads(FB)) __attribute__((amdgpu_waves_per_eu(FB == kFBWide ? 4 : DT == 0 ? 6 : 5))) void lr_sample_kernel(LargeArgs a)
{
    typedef Elem<DT> E;
    constexpr int TH = lr_row_threads(FB), NU = FB == kFBWide ? 4 : 8, LG = FB == kFBWide ? 12 : 11;     // 4096 or 2048 chunks
    constexpr int EPC = RowChunks<DT>::EPC, SH = LrOrder<DT>::kSh, SUB = FB == kFBWide ? 11 : 10;
    static_assert(TH * NU == 1 << LG && FB == 1 << SUB && TH * NU * EPC < 65536, "16-bit counters");
    constexpr bool kHalf = FB != kFBWide;            // two counters per word (more rows per CU; a single row is 0.4 us faster with words)
    __shared__ u32 h[kHalf ? kSampleBins / 2 : kSampleBins];
    __shared__ u32 h2[FB];
    __shared__ u32 scr[TH / kWave + 1];
    __shared__ u32 s_v[8];
    const int tid = threadIdx.x, w = a.w;
    const int64_t r = blockIdx.x;
    const RowChunks<DT> row(a.x, r, a.N);
    const u32 Q = (u32)(row.Nh + EPC - 1) / EPC, G = Q < (u32)(TH * NU) ? Q : (u32)(TH * NU);      // chunks of the row, of the sample
    const bool rg = row.ragged();
    // one chunk from every G-th of the row, at a hashed place: even spread without a period
    uint4 v[NU];
    u32 qs[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const u32 g = (u32)u * (u32)TH + (u32)tid;
        v[u] = make_uint4(0, 0, 0, 0);
        qs[u] = 0;
        if (g < G) {
            const u32 lo = G == Q ? g : (u32)(((u64)g * Q) >> LG), len = G == Q ? 1u : (u32)(((u64)(g + 1u) * Q) >> LG) - lo;
            u32 hs = g * 0x9E3779B1u;
            hs ^= hs >> 15; hs *= 0x85EBCA77u; hs ^= hs >> 13;
            qs[u] = lo + __umulhi(hs, len);
            if (!rg || row.whole((int)qs[u])) v[u] = row.base[qs[u]];       // (a partial chunk at either end is left out)
        }
    }
    {
        uint4* h4 = (uint4*)h;
        for (int i = tid; i < (kHalf ? kSampleBins / 8 : kSampleBins / 4); i += TH) h4[i] = make_uint4(0, 0, 0, 0);
        if (tid < FB / 4) ((uint4*)h2)[tid] = make_uint4(0, 0, 0, 0);
        if (tid < 8) s_v[tid] = tid == 5 ? (u32)kSampleBins - 1u : 0u;
    }
    auto count_of = [&](u32 bin) -> u32 { return kHalf ? (h[bin >> 1] >> (16u * (bin & 1u))) & 0xFFFFu : h[bin]; };
    u32* st = a.rowst + (size_t)r * 16;
    if (tid == 0) { st[kStCursor] = 0; st[kStTicket] = 0; st[kStFlag] = 0; st[kStLeft] = 0; }
    __syncthreads();
    auto c32_of = [&](int u, int e) -> u32 {
        const u32 key = E::key((typename E::raw_t)chunk_elem<DT>(v[u], e));
        return key ? lr_c32<DT>(key, (u32)((int)qs[u] * EPC + e - row.head), w) : 0u;
    };
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const u32 c = c32_of(u, e), bin = c >> SH;
            if (c) atomicAdd(&h[kHalf ? bin >> 1 : bin], kHalf ? 1u << (16u * (bin & 1u)) : 1u);
        }
    __syncthreads();
    // how many of the sample's elements must reach the bound; a complete sample needs no margin
    const bool whole = G == Q && !rg;
    const u32 target = whole ? (a.k > 0 ? (u32)a.k : 1u) : a.sample_target;
    constexpr int BPT = kSampleBins / TH;
    const int hi = kSampleBins - tid * BPT;         // thread t owns the BPT bins below kSampleBins - BPT t
    u32 cs[BPT];
    constexpr int PER = kHalf ? 8 : 4;              // bins per 16 bytes
#pragma unroll
    for (int j = 0; j < BPT / PER; ++j) {
        const uint4 t = ((const uint4*)h)[hi / PER - 1 - j];
        const u32 wd[4] = { t.w, t.z, t.y, t.x };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (kHalf) { cs[PER * j + 2 * i] = wd[i] >> 16; cs[PER * j + 2 * i + 1] = wd[i] & 0xFFFFu; }
            else cs[PER * j + i] = wd[i];
        }
    }
    u32 local = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) local += cs[j];
    u32 tot;
    {
        u32 acc = block_excl_scan<TH>(local, scr, &tot);
#pragma unroll
        for (int j = 0; j < BPT; ++j) {
            if (acc < target && target <= acc + cs[j]) { s_v[0] = (u32)(hi - 1 - j); s_v[1] = acc; s_v[2] = 1u; }
            acc += cs[j];
        }
        // the sample's largest and smallest bin: one lane of a wavefront knows its own (an LDS atomic of every lane, all at one address, took 3 us:
        // stage on fp32 [1 x 200704] 9.5 -> 6.5)
        const u64 some = __ballot(local != 0u);
        const int ln = (int)lane_id();
        if (local && ln == __ffsll((unsigned long long)some) - 1) {
            int topj = 0;
#pragma unroll
            for (int j = BPT - 1; j >= 0; --j) if (cs[j]) topj = j;
            atomicMax(&s_v[3], (u32)(hi - 1 - topj));
        }
        if (local && ln == 63 - __clzll((long long)some)) {
            int botj = 0;
#pragma unroll
            for (int j = 0; j < BPT; ++j) if (cs[j]) botj = j;
            atomicMin(&s_v[5], (u32)(hi - 1 - botj));
        }
    }
    __syncthreads();
    u32 T = LrOrder<DT>::kLeast;                    // every non-zero element, unless the sample holds more than wanted
    if (s_v[2]) {                                    // uniform
        const u32 B = s_v[0];
        T = B << SH;
        if (!whole && count_of(B) * 16u > target) {  // a full bin: the bound inside it
            const u32 rem = target - s_v[1];
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    const u32 c = c32_of(u, e);
                    if (c && (c >> SH) == B) atomicAdd(&h2[(c >> (SH - SUB)) & (u32)(FB - 1)], 1u);
                }
            __syncthreads();
            constexpr int BPT2 = FB / TH;
            const int hi2 = FB - tid * BPT2;
            u32 c2[BPT2], sum2 = 0;
#pragma unroll
            for (int j = 0; j < BPT2; ++j) { c2[j] = h2[hi2 - 1 - j]; sum2 += c2[j]; }
            u32 tot2;
            u32 acc = block_excl_scan<TH>(sum2, scr, &tot2);
#pragma unroll
            for (int j = 0; j < BPT2; ++j) {
                if (acc < rem && rem <= acc + c2[j]) s_v[4] = (u32)(hi2 - 1 - j);
                acc += c2[j];
            }
            __syncthreads();
            T |= s_v[4] << (SH - SUB);
        }
        if (T < LrOrder<DT>::kLeast) T = LrOrder<DT>::kLeast;
    }
    // fine bins: a sample bin that should hold c list entries is cut into the largest power of two up to c / per, with
    // `per` such that all of them fit; elements in sample bins above the sample's largest element share the last fine
    // bin, elements below its smallest one (or below the table's reach, when nearly all non-zeros are wanted) the first
    u32 Blo = T >> SH;
    Blo = Blo > s_v[5] ? Blo : s_v[5];
    u32 Btop = s_v[3] > Blo ? s_v[3] : Blo;
    if (Btop - Blo > (u32)kMaxTab - 1u) Btop = Blo + (u32)kMaxTab - 1u;
    const u32 nb = Btop - Blo + 1u;
    const float scale = a.sample_scale;
    const u32 room = (u32)FB - 2u - nb;
    float per = scale * (float)((tot < target ? tot : target) + count_of(Blo)) / (float)room + 1.0f;
    per = per < 8.0f ? 8.0f : per;
    constexpr int VPT = TH >= 512 ? 1 : 512 / TH;    // thread i: sample bins Blo + VPT i, ...
    u32 lg[VPT], sub = 0;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const u32 i = (u32)(tid * VPT + j);
        lg[j] = 0;
        if (i < nb) {
            const u32 c = (u32)((float)count_of(Blo + i) * scale / per);
            lg[j] = c > 1u ? 31u - (u32)__clz((int)c) : 0u;
            lg[j] = lg[j] < (u32)SUB ? lg[j] : (u32)SUB;
            sub += 1u << lg[j];
        }
    }
    u32 nbins;
    u32 base = block_excl_scan<TH>(sub, scr, &nbins);
    const bool over = nbins > (u32)FB - 2u;          // cannot happen by more than rounding: one fine bin each
    if (over) { nbins = nb; base = (u32)(tid * VPT); }
    uint16_t* tab = a.tab + (size_t)r * kTabSize;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const u32 i = (u32)(tid * VPT + j), l = over ? 0u : lg[j];
        if (i < nb) tab[i + 1u] = (uint16_t)((base + 1u) | (l << 12));
        base += 1u << l;
    }
    if (tid == 0) { tab[0] = 0; tab[nb + 1u] = (uint16_t)(nbins + 1u); }
    if (tid == 0) { st[kStT] = T; st[kStBlo] = Blo; st[kStNb] = nb; }
}

// ---- 2. compact -----------------------------------------------------------------------------------
// A wavefront owns up to NR * 512 consecutive elements, all of them on their way to its registers from the start, and squeezes the entries
// above the bound into its own piece of LDS (index order) as they arrive; then every lane takes whole entries.  With a fifth of the
// elements above the bound the work per entry (fine bin, atomics, stores) would otherwise run with a fifth of the lanes.
// The lanes hold consecutive 32-bit words, so that the order of the elements is that of (word of the lane, lane) and an entry's place
// follows from the ballot of its word's flags.  With 16 bytes a lane the places took prefix sums of per-lane counts, behind a count
// of everything; with the fine bins of all entries kept in registers from the histogram to the positions, up to 49 of them spilled.
// A tile with a wavefront of more than kLrEntries entries is read again, 512 elements at a time.
// DENSE: for lists with more entries than that in most wavefronts, where reading again took half the stage's time (encode, fp32 [40 x 985624] keep
// 0.8 729 -> 573 us, [316 x 126280] keep 0.3 353 -> 293).  The elements stay in registers and give way, 512 at a time, to the bins and places of their entries.
template <int DT, int NR, int FB, bool DENSE>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(DENSE && NR > 2 ? 6 : 8))) void lr_compact_kernel(LargeArgs a)
{
    constexpr int EPW = DT == 0 ? 1 : 2, WPR = 8 / EPW;              // elements of a word, words per lane and round
    constexpr int NW = NR * WPR, NWV = kTileThreads / kWave, RE = 8 * kWave, NS = kLrEntries / kWave;       // words of a lane; elements of a round; entries of a lane
    constexpr int kRoom = DENSE ? RE : kLrEntries;   // entries of a wavefront's piece of LDS
    constexpr int kBuf = DENSE && NR * RE * NWV * 2 > NWV * kRoom * 6 ? NR * RE * NWV * 2 : NWV * kRoom * 6;
    typedef typename Elem<DT>::raw_t raw_t;
    __shared__ u32 hist[FB];                         // positive | negative << 16; later the place of the bin's next entry
    __shared__ __align__(4) uint16_t tab[kTabSize];
    __shared__ __align__(16) unsigned char buf[kBuf];
    __shared__ u32 wtot[NWV];
    __shared__ u32 scr[NWV + 1];
    __shared__ u32 s_base;
    const int tid = threadIdx.x, s = blockIdx.x, w = a.w, wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    u32* braw = (u32*)buf + wv * kRoom;              // entries of this wavefront
    uint16_t* bidx = (uint16_t*)(buf + NWV * kRoom * 4) + wv * kRoom;
    uint16_t* bpos = (uint16_t*)buf;                 // in the end: list positions by fine bin
    const u32 lane = lane_id();
    const int64_t r = blockIdx.y;
    u32* st = a.rowst + (size_t)r * 16;
    const u32 WE = (u32)a.tile / NWV, tile0 = (u32)s * (u32)a.tile, we0 = (u32)wv * WE;       // elements of a wavefront; first one of the tile, of the wavefront in the tile
    // Buffer loads: what lies behind the wavefront's share or the row's end reads as zeros, which are below every bound.  Words where
    // the row consists of whole ones; bf16 rows of odd length or at odd places by halves.
    const raw_t* row = (const raw_t*)a.x + (size_t)r * (size_t)a.N;
    const u32 first = tile0 + we0, behind = first < (u32)a.N ? (u32)a.N - first : 0u, mine = behind < WE ? behind : WE;
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<raw_t*>(row) + (behind ? first : 0u), 0, (int)(mine * (u32)sizeof(raw_t)), 0x00020000);
    const bool words = DT == 0 || ((a.N & 1) == 0 && ((uintptr_t)row & 3) == 0);
    auto load = [&](auto& v, int at) {
        constexpr int n = sizeof(v) / 4;
        if (words) {
#pragma unroll
            for (int c = 0; c < n; ++c) v[c] = __builtin_amdgcn_raw_buffer_load_b32(rs, at + c * (4 * kWave), 0, 0);
        } else {
#pragma unroll
            for (int c = 0; c < n; ++c) {
                const u32 lo = __builtin_amdgcn_raw_buffer_load_b16(rs, at + c * (4 * kWave), 0, 0);
                v[c] = lo | ((u32)__builtin_amdgcn_raw_buffer_load_b16(rs, at + c * (4 * kWave) + 2, 0, 0) << 16);
            }
        }
    };
    u32 v[NW];
    load(v, (int)(lane * 4u));
    const u32 T = st[kStT], Blo = st[kStBlo], nb = st[kStNb];
    {
        uint4* h4 = (uint4*)hist;
        for (int i = tid; i < FB / 4; i += kTileThreads) h4[i] = make_uint4(0, 0, 0, 0);
        const u32* tg = (const u32*)(a.tab + (size_t)r * kTabSize);
        if (tid < kTabSize / 2) ((u32*)tab)[tid] = tg[tid];
    }
    // bf16: 17 bits of the inverted index (an element behind the row's end has key 0 and stays below the least bound, 2^17)
    const u32 inv0 = (1u << w) - 1u - (tile0 + we0 + lane * (u32)EPW);
    const int up = w < 17 ? 17 - w : 0, down = w < 17 ? 0 : w - 17;
    // the entries of word c (elements c * 64 * EPW ... of the wavefront) to its piece, behind `run` others; or only their number
    auto squeeze = [&](u32 x, u32 c, u32& run, auto store) {
        constexpr bool kStore = decltype(store)::value;
        const u32 e = (c * (u32)kWave + lane) * (u32)EPW;
        if (DT == 0) {
            const bool in = (x & 0x7FFFFFFFu) >= T;
            const u64 m = __ballot(in);
            const u32 pos = run + mask_rank(m);
            run += (u32)__popcll(m);
            if (kStore && run <= (u32)kRoom && in) { braw[pos] = x; bidx[pos] = (uint16_t)e; }
        } else {
            const u32 k0 = (x << 16) & 0x7FFF0000u, k1 = x & 0x7FFF0000u, inv = inv0 - c * (u32)(kWave * EPW);
            const bool in0 = ((k0 << 1) | __builtin_amdgcn_ubfe(inv << up, (u32)down, 17u)) >= T;
            const bool in1 = ((k1 << 1) | __builtin_amdgcn_ubfe((inv - 1u) << up, (u32)down, 17u)) >= T;
            const u64 m0 = __ballot(in0), m1 = __ballot(in1);
            const u32 pos = run + mask_rank(m0) + mask_rank(m1), pos1 = pos + (in0 ? 1u : 0u);
            run += (u32)__popcll(m0) + (u32)__popcll(m1);
            if (kStore && run <= (u32)kRoom) {
                if (in0) { braw[pos] = x << 16; bidx[pos] = (uint16_t)e; }
                if (in1) { braw[pos1] = x & 0xFFFF0000u; bidx[pos1] = (uint16_t)(e + 1u); }
            }
        }
    };
    typedef std::true_type yes;
    auto bin_of = [&](u32 raw, u32 ix) -> u32 {      // fine bin | negative << 31
        const u32 key = DT == 0 ? raw & 0x7FFFFFFFu : (raw >> 16) & 0x7FFFu;
        return lr_fine_bin<DT>(lr_c32<DT>(key, first + ix, w), tab, Blo, nb) | (raw & 0x80000000u);
    };
    auto one = [&](u32 b) -> u32 { return b >> 31 ? 0x10000u : 1u; };
    u32 wn = 0;
#pragma unroll
    for (int c = 0; c < NW; ++c) squeeze(v[c], (u32)c, wn, std::integral_constant<bool, !DENSE>());
    if (lane == 0) wtot[wv] = wn;
    __syncthreads();
    u32 wbase = 0, ntile = 0, most = 0;              // entries of the wavefronts before this one, of the tile
#pragma unroll
    for (int i = 0; i < NWV; ++i) { const u32 t = wtot[i]; if (i < wv) wbase += t; ntile += t; most = t > most ? t : most; }
    const bool dense = !DENSE && most > (u32)kLrEntries;     // uniform
    if (tid == 0) {
        u32 b = atomicAdd(&st[kStCursor], ntile);
        if (b > a.capL || ntile > a.capL - b) { b = 0xFFFFFFFFu; st[kStFlag] = 1u; }     // the list is full: the row is redone generically
        s_base = b;
    }
    // a dense tile's entries, 512 elements of every wavefront at a time: f(entries before, entry, raw, index in the wavefront)
    auto rounds = [&](auto&& f) {
        u32 before = 0;
#pragma unroll 1
        for (int g = 0; g < NR; ++g) {
            u32 t[WPR], run = 0;
            load(t, (int)(lane * 4u) + g * (RE * (int)sizeof(raw_t)));
#pragma unroll
            for (int j = 0; j < WPR; ++j) squeeze(t[j], (u32)(g * WPR + j), run, yes());
            wave_sync();
#pragma unroll 1
            for (u32 i = lane; i < run; i += kWave) f(before + i, braw[i], (u32)bidx[i]);
            wave_sync();
            before += run;
        }
    };
    u32 bf[DENSE ? NR * 8 : NS], nr[NR];             // bins, and DENSE: | entries of the bin before this one << 12; entries of a round
    if (DENSE) __syncthreads();                      // s_base
    const u32 seg0d = DENSE ? s_base : 0u;
    if (DENSE) {
        u32* __restrict__ Lraw = LrList(a, r).raw + seg0d + wbase;
        uint16_t* __restrict__ Lidx = LrList(a, r).idx + seg0d + wbase;
        u32 before = 0;
#pragma unroll
        for (int g = 0; g < NR; ++g) {
            u32 run = 0;
#pragma unroll
            for (int j = 0; j < WPR; ++j) squeeze(v[g * WPR + j], (u32)(g * WPR + j), run, yes());
            nr[g] = run;
            wave_sync();
#pragma unroll
            for (int h = 0; h < 8; h += 2) {         // two entries per lane at a time, their lookups side by side
                bf[DENSE ? g * 8 + h : 0] = bf[DENSE ? g * 8 + h + 1 : 0] = 0;
                if ((u32)(h * kWave) >= run) continue;       // uniform in the wavefront
                u32 raw[2], ix[2], b[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) { const u32 i = (u32)((h + e) * kWave) + lane; raw[e] = braw[i]; ix[e] = (u32)bidx[i]; }
#pragma unroll
                for (int e = 0; e < 2; ++e) b[e] = bin_of(raw[e], ix[e]);
#pragma unroll
                for (int e = 0; e < 2; ++e) {        // (lanes without an entry add nothing, each to a bin of its own)
                    const u32 i = (u32)((h + e) * kWave) + lane;
                    const bool in = i < run;
                    const u32 old = atomicAdd(&hist[in ? b[e] & 0xFFFu : lane], in ? one(b[e]) : 0u);
                    bf[DENSE ? g * 8 + h + e : 0] = b[e] | ((b[e] >> 31 ? old >> 16 : old & 0xFFFFu) << 12);
                    if (in && seg0d != 0xFFFFFFFFu) { Lraw[before + i] = raw[e]; Lidx[before + i] = (uint16_t)(we0 + ix[e]); }
                }
            }
            wave_sync();
            before += run;
        }
    } else if (dense) rounds([&](u32, u32 raw, u32 ix) { const u32 b = bin_of(raw, ix); atomicAdd(&hist[b & 0xFFFu], one(b)); });
    else {
#pragma unroll
        for (int h = 0; h < (DENSE ? 0 : NS); h += 2) {            // two entries per lane at a time, their lookups side by side
            if ((u32)(h * kWave) >= wn) break;       // uniform in the wavefront
            u32 raw[2], ix[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const u32 i = (u32)((h + e) * kWave) + lane;
                raw[e] = braw[i]; ix[e] = (u32)bidx[i];
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) bf[h + e] = bin_of(raw[e], ix[e]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {            // (lanes without an entry add nothing, each to a bin of its own)
                const bool in = (u32)((h + e) * kWave) + lane < wn;
                atomicAdd(&hist[in ? bf[h + e] & 0xFFFu : lane], in ? one(bf[h + e]) : 0u);
            }
        }
    }
    __syncthreads();
    const u32 seg0 = s_base;
    const bool full = seg0 == 0xFFFFFFFFu;
    const LrList list(a, r);
    u32* __restrict__ Lraw = list.raw + seg0 + wbase;
    uint16_t* __restrict__ Lidx = list.idx + seg0 + wbase;
    uint16_t* __restrict__ Lpos = list.pos + seg0;
    u32* seg = a.seg + ((size_t)r * a.S + s) * 2;
    {
        // bins per thread from the top, 4 or 2; the halves add up separately: no sum reaches 2^16
        constexpr int BPT = FB / kTileThreads;
        typedef u32 bins_t __attribute__((ext_vector_type(BPT)));
        bins_t* h4 = (bins_t*)hist + (FB / BPT - 1 - tid);
        const bins_t t = *h4;
        u32 local = 0;
#pragma unroll
        for (int j = 0; j < BPT; ++j) local += t[j];
        u32 tot;
        u32 at = block_excl_scan<kTileThreads>(local, scr, &tot);
        const u32 off = (tot & 0xFFFFu) << 16;       // the negative entries follow the positive ones
        bins_t up, st0;                              // entries at or above the bin; place of the bin's first one
#pragma unroll
        for (int j = BPT - 1; j >= 0; --j) { st0[j] = at + off; at += t[j]; up[j] = at; }
        ((bins_t*)(a.cum + ((size_t)r * a.S + s) * FB))[FB / BPT - 1 - tid] = up;
        *h4 = st0;
        if (tid == 0) { seg[0] = seg0; seg[1] = tot; }
    }
    if (full || ntile == 0u) return;                 // uniform
    if (DENSE) {
        __syncthreads();
        u32 before = 0;
#pragma unroll
        for (int g = 0; g < NR; ++g) {
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                if ((u32)(h * kWave) >= nr[g]) continue;     // uniform in the wavefront
                const u32 i = (u32)(h * kWave) + lane, t = bf[DENSE ? g * 8 + h : 0], at = hist[t & 0xFFFu];
                if (i < nr[g]) bpos[(t >> 31 ? at >> 16 : at & 0xFFFFu) + ((t >> 12) & 0x7FFFu)] = (uint16_t)(wbase + before + i);
            }
            before += nr[g];
        }
        __syncthreads();
        for (u32 i = (u32)tid; i < ntile; i += kTileThreads) Lpos[i] = bpos[i];
        return;
    }
    if (dense) {
        __syncthreads();
        rounds([&](u32 i, u32 raw, u32 ix) {
            Lraw[i] = raw; Lidx[i] = (uint16_t)(we0 + ix);
            const u32 b = bin_of(raw, ix), at = atomicAdd(&hist[b & 0xFFFu], one(b));
            Lpos[b >> 31 ? at >> 16 : at & 0xFFFFu] = (uint16_t)(wbase + i);
        });
        return;
    }
#pragma unroll
    for (int h = 0; h < (DENSE ? 0 : NS); ++h) {
        const u32 i = (u32)(h * kWave) + lane;
        if ((u32)(h * kWave) >= wn) break;
        if (i < wn) { Lraw[i] = braw[i]; Lidx[i] = (uint16_t)(we0 + (u32)bidx[i]); }
    }
    __syncthreads();                                 // the entries have been read: their storage takes the positions
#pragma unroll
    for (int h = 0; h < (DENSE ? 0 : NS); ++h) {
        if ((u32)(h * kWave) >= wn) break;
        const u32 i = (u32)(h * kWave) + lane;
        if (i < wn) {
            const u32 at = atomicAdd(&hist[bf[h] & 0xFFFu], one(bf[h]));
            bpos[bf[h] >> 31 ? at >> 16 : at & 0xFFFFu] = (uint16_t)(wbase + i);
        }
    }
    __syncthreads();
    for (u32 i = (u32)tid; i < ntile; i += kTileThreads) Lpos[i] = bpos[i];
}

// ---- bitwidths, bit offsets and the row's length ----------------------------------------------------
// Thread b holds block b's bitwidth q and flag (0x80: none feasible); everything the pack stage and meta need follows.
template <int DT>
__device__ inline void lr_finish_row(const LargeArgs& a, int64_t r, u32 n_pos, u32 n_neg, bool on, u32 q, u32 flag, u32 cnt, float vmin, float vmax,
                                     u64* bits_s)
{
    const int b = threadIdx.x, B2 = a.M + a.Mn;
    if (on) {
        float inv = 0.f;
        const float rng = vmax - vmin;
        if (cnt && rng > 0.f) inv = (float)((1u << q) - 1u) / unit_range(rng, range_exp(rng));
        a.qsel[r * B2 + b] = q;
        a.inv_sel[r * B2 + b] = inv;
        const size_t mi = (size_t)r * (size_t)B2 + b;
        a.mv.vmin[mi] = vmin; a.mv.vmax[mi] = vmax; a.mv.q[mi] = (uint8_t)(q | flag);
        bits_s[b] = (u64)cnt * (u64)q;
    }
    __syncthreads();
    if (on) {
        u64 acc = 0;
        for (int i = 0; i < b; ++i) acc += bits_s[i];
        a.code_off[(size_t)r * (B2 + 1) + b] = acc;
        if (b == B2 - 1) {
            acc += bits_s[b];
            a.code_off[(size_t)r * (B2 + 1) + B2] = acc;
            const u64 n = (u64)n_pos + n_neg;
            const u64 bits = a.n_cols > 0 ? (u64)B2 * (u64)(a.n_rows + 1) * (u64)a.wp + n * (u64)a.wc + acc : n * (u64)a.w + acc;
            u64 words = (bits + 31) >> 5;
            if (words > a.cap_words) words = a.cap_words;            // cannot happen: the capacity is the worst case
            a.row_words[r] = words;
            a.mv.n_pos[r] = n_pos;
            a.mv.n_neg[r] = n_neg;
        }
    }
}

// ---- 3. bounds ------------------------------------------------------------------------------------
constexpr int kMaxTargets = 2 * kMaxB2;

// a member: comp in the low 55 bits (31 of the key, up to 24 of the index), its group, its class
constexpr int kMemGroup = 55;
constexpr u64 kMemComp = (1ull << kMemGroup) - 1ull;
// Largest bin whose members are compared with each other; with a larger one in the row they are sorted.  Encode us, 1024 / 512: fp32 [1 x 200704]
// in steps of 1/40 133 / 117, [1 x 4000000] keep 0.3 209 / 150, [32 x 401408] clipped at 3 sigma 137 / 121.
constexpr u32 kLrSortBin = 512;

template <int FB, bool BIG>
struct LrBoundsLds {
    static constexpr int kMemCap = lr_mem_cap(FB, BIG);
    u32 at_p[FB + 4], at_n[FB + 4];                // list entries at or above the bin
    u64 mem[kMemCap + 4];                            // members of the bins that hold a target
    u32 tg_bin[kMaxTargets], tg_rem[kMaxTargets];    // target 2 b: first element of block b, 2 b + 1: its last one
    u64 tg_comp[kMaxTargets];
    u32 g_bin[kMaxTargets], g_cls[kMaxTargets];      // groups of consecutive targets in one bin; class 2: both
    u32 g_start[kMaxTargets + 1], g_fill[kMaxTargets], g_t0[kMaxTargets + 1];
    u32 v[8];
};

template <int DT, int FB, bool BIG>
__global__ __launch_bounds__(lr_row_threads(FB)) void lr_bounds_kernel(LargeArgs a, EncArgs ea)
{
    constexpr int TH = lr_row_threads(FB), kMemCap = lr_mem_cap(FB, BIG);
    constexpr bool kRedo = FB == kFBWide;            // rows that do not fit are redone here (else: after the pack stage)
    constexpr size_t kOwn = sizeof(LrBoundsLds<FB, BIG>), kRedoLds = kRedo ? sizeof(GenericLds<1024>) : 0;
    __shared__ __align__(16) unsigned char lds[kOwn > kRedoLds ? kOwn : kRedoLds];
    LrBoundsLds<FB, BIG>& L = *(LrBoundsLds<FB, BIG>*)lds;
    const int tid = threadIdx.x, w = a.w, M = a.M, Mn = a.Mn, B2 = M + Mn, S = a.S;
    // P workgroups share a row: all of them sum the tables and find the bins, each resolves its share of these.  A bin's members lie one or two
    // to a cache line, a thousand lines and more for a row, at the end of three dependent loads: one workgroup of fp32 [32 x 401408] took
    // 18 us to gather and compare them, eight take 5.
    const int P = a.parts, part = (int)(blockIdx.x / (u32)a.part_step);
    const int64_t r = blockIdx.x % (u32)a.part_step;
    if (r >= a.R) return;
    u32* st = a.rowst + (size_t)r * 16;
    const u32 k = (u32)a.k;
    const u32* __restrict__ cum = a.cum + (size_t)r * S * FB;
    const u32* __restrict__ seg = a.seg + (size_t)r * S * 2;
    const LrList list(a, r);
    const u32* __restrict__ Lraw = list.raw;
    const uint16_t* __restrict__ Lidx = list.idx;
    const uint16_t* __restrict__ Lpos = list.pos;
    u32* pair = a.pair + (size_t)r * B2 * S;
    bool bad = st[kStFlag] != 0u;                    // uniform
    if (part == 0) for (int i = tid; i < B2 * (a.nq + 1); i += TH) a.sums[(size_t)r * B2 * (a.nq + 1) + i] = 0;
    const u32 T = st[kStT];

    // sums of the tiles' tables: a thread takes four bins of every GT-th tile, eight of them in flight
    {
        constexpr int GT = 4 * TH / FB;
        static_assert(GT == 1 || GT == 2, "the groups' sums meet in one step");
        const int gt = tid / (FB / 4), c4 = tid - gt * (FB / 4);
        u32 p[4] = { 0, 0, 0, 0 }, n[4] = { 0, 0, 0, 0 };
        for (int s0 = gt; s0 < S; s0 += 8 * GT) {
            uint4 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = s0 + u * GT < S ? ((const uint4*)(cum + (size_t)(s0 + u * GT) * FB))[c4] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                p[0] += t[u].x & 0xFFFFu; p[1] += t[u].y & 0xFFFFu; p[2] += t[u].z & 0xFFFFu; p[3] += t[u].w & 0xFFFFu;
                n[0] += t[u].x >> 16; n[1] += t[u].y >> 16; n[2] += t[u].z >> 16; n[3] += t[u].w >> 16;
            }
        }
        uint4* ap = (uint4*)L.at_p + c4;
        uint4* an = (uint4*)L.at_n + c4;
        if (GT > 1) {
            if (gt) { *ap = make_uint4(p[0], p[1], p[2], p[3]); *an = make_uint4(n[0], n[1], n[2], n[3]); }
            __syncthreads();
        }
        if (!gt) {
            if (GT > 1) {
                const uint4 tp = *ap, tn = *an;
                p[0] += tp.x; p[1] += tp.y; p[2] += tp.z; p[3] += tp.w;
                n[0] += tn.x; n[1] += tn.y; n[2] += tn.z; n[3] += tn.w;
            }
            *ap = make_uint4(p[0], p[1], p[2], p[3]); *an = make_uint4(n[0], n[1], n[2], n[3]);
        }
        if (tid == 0) { L.at_p[FB] = 0; L.at_n[FB] = 0; }
        if (tid < 8) L.v[tid] = 0;
    }
    __syncthreads();
    const u32 nL = L.at_p[0] + L.at_n[0];
    if (nL < k && T > LrOrder<DT>::kLeast) bad = true;       // the sample's bound was too high

    auto at_c = [&](u32 cls, u32 b) -> u32 { return cls == 0u ? L.at_p[b] : cls == 1u ? L.at_n[b] : L.at_p[b] + L.at_n[b]; };
    // members of the bins of groups ga .. gb - 1 (g_start: room per group), tile by tile; up to eight threads share a tile's
    // members while there are threads to spare, and more of them where a bin is crowded
    auto gather = [&](int ga, int gb, bool crowded) {
        const int ng = gb - ga;
        const u32 m0 = L.g_start[ga];
        int lp = 0;                                  // log2 of the threads that share
        while (lp < (crowded ? 8 : 3) && (ng * S << (lp + 1)) <= TH) ++lp;
        for (int i = tid; i < ng * S << lp; i += TH) {
            const int gs = i >> lp, share_of = i - (gs << lp), gi = gs / S, s = gs - gi * S, g = ga + gi;
            const u32 cls = L.g_cls[g], b = L.g_bin[g];
            const u32 c0 = cum[(size_t)s * FB + b], c1 = b + 1u < (u32)FB ? cum[(size_t)s * FB + b + 1u] : 0u;
            const u32 seg0 = seg[2 * s], np = seg[2 * s + 1] & 0xFFFFu;
#pragma unroll
            for (u32 h = 0; h < 2u; ++h) {
                if (cls != 2u && cls != h) continue;
                const u32 n0 = h ? c0 >> 16 : c0 & 0xFFFFu, n1 = h ? c1 >> 16 : c1 & 0xFFFFu, cn = n0 - n1;
                if (cls != 2u && share_of == 0)          // entries of the tile above the bin: the start of the blocks' counts
                    for (u32 t = L.g_t0[g]; t < L.g_t0[g + 1]; ++t) if (t & 1u) pair[(size_t)(t >> 1) * S + s] = n1;
                const u32 share = (cn + (1u << lp) - 1u) >> lp, p0 = (u32)share_of * share, p1 = p0 + share < cn ? p0 + share : cn;
                if (p0 >= p1) continue;
                const u32 slot = L.g_start[g] - m0 + atomicAdd(&L.g_fill[g], p1 - p0) - p0;
                for (u32 j0 = p0; j0 < p1; j0 += 4) {
                    u32 lp[4], rw[4], ix[4];
#pragma unroll
                    for (u32 u = 0; u < 4; ++u) lp[u] = seg0 + (j0 + u < p1 ? (u32)Lpos[seg0 + (h ? np : 0u) + n1 + j0 + u] : 0u);
#pragma unroll
                    for (u32 u = 0; u < 4; ++u) { rw[u] = Lraw[lp[u]]; ix[u] = Lidx[lp[u]]; }
#pragma unroll
                    for (u32 u = 0; u < 4; ++u) {
                        if (j0 + u < p1) {
                            const u32 key = DT == 0 ? rw[u] & 0x7FFFFFFFu : (rw[u] >> 16) & 0x7FFFu;
                            L.mem[slot + j0 + u] = lr_comp(key, (u32)(s * a.tile) + ix[u], w) | ((u64)g << kMemGroup) | (h ? kTop : 0ull);
                        }
                    }
                }
            }
        }
        __syncthreads();
    };

    u32 n_pos = L.at_p[0], n_neg = L.at_n[0];
    if (!bad && nL > k) {
        if (n_neg == 0u || k == 0u) { n_pos = k; n_neg = 0; }
        else if (n_pos == 0u) n_neg = k;
        else {                                       // ATKF cut: overall rank k - 1
#pragma unroll
            for (u32 j = 0; j < (u32)(FB / TH); ++j) {
                const u32 b = (u32)tid * (u32)(FB / TH) + j;
                if (at_c(2, b) > k - 1u && at_c(2, b + 1u) <= k - 1u) {
                    L.g_bin[0] = b; L.g_cls[0] = 2; L.g_start[0] = 0; L.g_start[1] = at_c(2, b) - at_c(2, b + 1u);
                    L.g_fill[0] = 0;
                }
            }
            __syncthreads();
            const u32 cn = L.g_start[1], cb = L.g_bin[0];
            if (cn > (u32)kMemCap) bad = true;
            else {
                const bool crowded = cn > kLrSortBin;
                gather(0, 1, crowded);
                const u32 rem = k - 1u - at_c(2, cb + 1u);
                if (__builtin_expect(crowded, 0)) {
                    block_sort<TH>(L.mem, cn, [](u64 m) { return m & ~kTop; });
                    for (u32 i0 = 0; i0 <= rem; i0 += TH) {
                        const u32 i = i0 + (u32)tid, in_n = (u32)__popcll(__ballot(i <= rem && (L.mem[i <= rem ? i : 0u] & kTop)));
                        const u32 in = (u32)__popcll(__ballot(i <= rem));
                        if (lane_id() == 0u && in) { atomicAdd(&L.v[0], in - in_n); atomicAdd(&L.v[1], in_n); }
                    }
                } else for (u32 i = (u32)tid; i < cn; i += TH) {
                    const u64 me = L.mem[i] & ~kTop;
                    u32 gt = 0;
                    for (u32 j = 0; j < cn; j += 4) {
                        u64 m4[4];
#pragma unroll
                        for (u32 u = 0; u < 4; ++u) m4[u] = L.mem[j + u] & ~kTop;
#pragma unroll
                        for (u32 u = 0; u < 4; ++u) gt += (u32)(j + u < cn) & (u32)(m4[u] > me);
                    }
                    if (gt <= rem) atomicAdd(&L.v[(L.mem[i] & kTop) ? 1 : 0], 1u);
                }
                __syncthreads();
                n_pos = L.at_p[cb + 1u] + L.v[0];
                n_neg = L.at_n[cb + 1u] + L.v[1];
                __syncthreads();
            }
        }
    }
    const u32 Kc0 = n_pos / (u32)M, Kc1 = n_neg / (u32)Mn;
    if (!bad) {
        // the bin of every target, sixteen lanes a target: the last one with more than `rank` entries at or above it
        for (int t0 = 0; t0 < 2 * B2; t0 += TH / 16) {
            const int t = t0 + tid / 16, b = t >> 1, c = b >= M ? 1 : 0, m = b - c * M, Ms = c ? Mn : M;
            const u32 K = c ? Kc1 : Kc0, cnt = t >= 2 * B2 ? 0u : m < Ms - 1 ? K : (c ? n_neg : n_pos) - K * (u32)(Ms - 1);
            const u32 rank = (u32)m * K + ((t & 1) && cnt ? cnt - 1u : 0u);
            const u32* at = c ? L.at_n : L.at_p;
            u32 lo = 0;                              // (an empty block's search finds nothing of use)
#pragma unroll
            for (int step = FB > 256 ? (FB + 255) / 256 * 16 : 16; step; step = step > 16 ? 16 : step > 1 ? 1 : 0) {
                const u32 b2 = lo + (u32)((tid & 15) * step);
                const u64 above = __ballot(b2 < (u32)FB && at[b2 < (u32)FB ? b2 : 0u] > rank);
                const u32 mine = (u32)(above >> (tid & 48)) & 0xFFFFu;
                lo += (mine ? 31u - (u32)__clz((int)mine) : 0u) * (u32)step;
            }
            if (t < 2 * B2 && (tid & 15) == 0) {
                L.tg_bin[t] = cnt ? lo : 0xFFFFFFFFu;        // an empty block has no elements
                L.tg_rem[t] = cnt ? rank - at[lo + 1u] : 0u;
                L.tg_comp[t] = ~0ull;
            }
        }
        __syncthreads();
        if (tid < kWave) {                           // groups: a target opens one unless the target before it lies in the same bin
            const int TL = (2 * B2 + kWave - 1) / kWave;     // targets a lane
            u32 lead = 0, room = 0, most = 0;
            for (int j = 0; j < TL; ++j) {
                const int t = tid * TL + j;
                if (t >= 2 * B2) break;
                const u32 b = L.tg_bin[t], c = (t >> 1) >= M ? 1u : 0u;
                const bool same = t > 0 && L.tg_bin[t - 1] == b && (((t - 1) >> 1) >= M ? 1u : 0u) == c;
                if (b != 0xFFFFFFFFu && !same) {
                    const u32 n = at_c(c, b) - at_c(c, b + 1u);
                    lead |= 1u << j; room += n; most = n > most ? n : most;
                }
            }
            if (__any(most > kLrSortBin) && tid == 0) L.v[3] = 1u;
            const u32 nl = (u32)__popc(lead);
            const u32 incl = wave_scan_dpp(nl), incr = wave_scan_dpp(room);
            u32 g = incl - nl, at = incr - room;
            for (int j = 0; j < TL; ++j) {
                const int t = tid * TL + j;
                if (!((lead >> j) & 1u)) continue;
                const u32 b = L.tg_bin[t], c = (t >> 1) >= M ? 1u : 0u;
                L.g_bin[g] = b; L.g_cls[g] = c; L.g_start[g] = at; L.g_fill[g] = 0; L.g_t0[g] = (u32)t;
                at += at_c(c, b) - at_c(c, b + 1u);
                ++g;
            }
            if (tid == kWave - 1) { L.g_start[incl] = incr; L.g_t0[incl] = (u32)(2 * B2); L.v[2] = incl; }
        }
        __syncthreads();
        const int ng = (int)L.v[2];
        const int lgP = __builtin_ctz((u32)P);       // (P is a power of two)
        if (__builtin_expect(L.g_start[ng] > (u32)kMemCap, 0))
            for (int i = 0; i < P; ++i) bad |= L.g_start[ng * (i + 1) >> lgP] - L.g_start[ng * i >> lgP] > (u32)kMemCap;
        if (!bad) {
            const int ga = ng * part >> lgP, gb = ng * (part + 1) >> lgP;
            const u32 m0 = L.g_start[ga], nm = L.g_start[gb] - m0;
            const bool crowded = L.v[3] != 0u;       // uniform
            gather(ga, gb, crowded);
            if (__builtin_expect(crowded, 0)) {
                // Groups in their order, the members of each from the largest comp down: a target is found by its rank.  All against all grew with
                // the square of the bin: fp32 [1 x 140000] keep 0.5, 64 + 64 blocks, 16000 equal values of either sign 4.2 ms, now 0.28 (by the generic
                // encoder 9.4); 16000 of one sign for the cut alone 18.9 ms; [1 x 200704] in steps of 1/20 338 us, now 110.
                block_sort<TH>(L.mem, nm, [](u64 m) { return m ^ ~kMemComp; });
                const int lane = (int)lane_id();
                for (int g = ga + tid / kWave; g < gb; g += TH / kWave)
                    for (int t = (int)L.g_t0[g] + lane; t < (int)L.g_t0[g + 1]; t += kWave)
                        if (L.tg_bin[t] == L.g_bin[g]) L.tg_comp[t] = L.mem[L.g_start[g] - m0 + L.tg_rem[t]] & kMemComp;
                __syncthreads();
                // per tile: entries of the class from the block's last element up.  Equal values of a tile follow each other: one addition a run
                for (u32 i0 = (u32)(tid / kWave * kWave); i0 < nm; i0 += TH) {
                    const u32 i = i0 + (u32)lane;
                    const u64 me = L.mem[i < nm ? i : nm - 1u];
                    const u32 g = (u32)(me >> kMemGroup) & 0xFFu, t0 = L.g_t0[g], t1 = L.g_t0[g + 1];
                    const u32 s = ((1u << w) - 1u - ((u32)me & ((1u << w) - 1u))) / (u32)a.tile, run = s | (g << 16);
                    const u32 before = (u32)__shfl_up((int)run, 1);          // (by all lanes)
                    const bool head = lane == 0 || before != run;
                    const u64 heads = __ballot(head), above = heads & ~((2ull << lane) - 1ull);       // (lane 63: none)
                    const u64 mine = (above ? (1ull << __builtin_ctzll(above)) - 1ull : ~0ull) & ~((1ull << lane) - 1ull);
                    const u32 ta = bcast(t0, 0), tb = bcast(t1, kWave - 1);
                    for (u32 t = ta | 1u; t < tb; t += 2u) {
                        const u64 from = __ballot(i < nm && t >= t0 && t < t1 && (me & kMemComp) >= L.tg_comp[t]);
                        const u32 n = (u32)__popcll(from & mine);
                        if (head && n) atomicAdd(&pair[(size_t)(t >> 1) * S + s], n);
                    }
                }
            } else {
                // rank of every member in its group, by up to sixteen lanes a member (one lane: 2.7 us of a row's 13 with 90 members a group)
                int lr = 0;
                while (lr < 4 && (nm << (lr + 1)) <= (u32)TH) ++lr;
                const u32 sl = (u32)tid & ((1u << lr) - 1u), lanes = 1u << lr;
                for (u32 i0 = 0; i0 < nm; i0 += (u32)TH >> lr) {
                    const u32 i = i0 + ((u32)tid >> lr);
                    const u64 me = i < nm ? L.mem[i] : 0ull;
                    const u32 g = i < nm ? (u32)(me >> kMemGroup) & 0xFFu : (u32)ga, m1 = L.g_start[g + 1] - m0, t1 = L.g_t0[g + 1], gb_bin = L.g_bin[g];
                    u32 gt = 0;
                    for (u32 j = L.g_start[g] - m0 + sl; j < m1; j += 4 * lanes) {
                        u64 m4[4];
#pragma unroll
                        for (u32 u = 0; u < 4; ++u) m4[u] = L.mem[j + u * lanes < m1 ? j + u * lanes : m1 - 1u];
#pragma unroll
                        for (u32 u = 0; u < 4; ++u) gt += (u32)(j + u * lanes < m1) & (u32)(m4[u] > me);
                    }
                    for (int d = 1; d < (int)lanes; d <<= 1) gt += (u32)__shfl_xor((int)gt, d);
                    for (u32 t = L.g_t0[g] + sl; i < nm && t < t1; t += lanes)
                        if (L.tg_bin[t] == gb_bin && L.tg_rem[t] == gt) L.tg_comp[t] = me & kMemComp;
                }
                __syncthreads();
                // per tile: entries of the class from the block's last element up
                for (u32 i = (u32)tid; i < nm; i += TH) {
                    const u32 g = (u32)(L.mem[i] >> kMemGroup) & 0xFFu;
                    const u64 me = L.mem[i] & kMemComp;
                    const u32 s = ((1u << w) - 1u - ((u32)me & ((1u << w) - 1u))) / (u32)a.tile;      // its tile
                    for (u32 t = L.g_t0[g]; t < L.g_t0[g + 1]; ++t)
                        if ((t & 1u) && me >= L.tg_comp[t]) atomicAdd(&pair[(size_t)(t >> 1) * S + s], 1u);
                }
            }
            for (int t = tid; t < 2 * B2; t += TH) {
                const u64 c = L.tg_comp[t];
                const size_t rb = (size_t)r * B2 + (t >> 1);
                const bool empty = L.tg_bin[t] == 0xFFFFFFFFu;
                if (empty ? part != 0 : c == ~0ull) continue;            // (another workgroup's)
                const u32 key = empty ? 0u : (u32)(c >> w);
                if (t & 1) { a.thr[rb] = c; a.vminb[rb] = key; } else a.vmaxb[rb] = key;
            }
            if (part == 0) {
                for (int b = tid; b <= B2; b += TH) {  // K, ..., K, K + remainder per class
                    const int c = b >= M ? 1 : 0, m = b - c * M;
                    a.blk_start[(size_t)r * (B2 + 1) + b] = b == B2 ? n_pos + n_neg : (c ? n_pos : 0u) + (u32)m * (c ? Kc1 : Kc0);
                }
                if (tid == 0) { st[kStNpos] = n_pos; st[kStNneg] = n_neg; }
            }
        }
    }
    if (!bad && part != 0) return;
    if constexpr (!kRedo) {                          // (one workgroup a row)
        if (tid == 0) {
            a.redo[r] = bad ? 1u : 0u;
            if (bad) { st[kStFlag] = 1u; a.row_words[r] = 0; a.blk_start[(size_t)r * (B2 + 1) + B2] = 0; }     // (nothing for the pack stage)
        }
    } else if (bad) {                                // rare: the row goes to its slot by the generic encoder
        // The generic encoder's list takes the place of the row's, which other parts may be reading for the cut, as they may the flag.  All
        // parts come to the same decision; the last one to have made it, behind everybody's reads, has the row.
        __syncthreads();
        if (P > 1) {
            if (tid == 0) L.v[4] = __hip_atomic_fetch_add(&st[kStLeft], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (L.v[4] != (u32)P - 1u) return;       // uniform
            __syncthreads();                         // (the encoder's LDS is the same)
        }
        if (tid == 0) st[kStFlag] = 1u;
        enc_generic_rows<DT, 1024>(ea, r, r + 1, *(GenericLds<1024>*)lds);
        __syncthreads();
        // its block-ordered arrays, counts, ranges and bitwidths are what the pack stage reads
        const u32 gp = a.mv.n_pos[r], gn = a.mv.n_neg[r], K0 = gp / (u32)M, K1 = gn / (u32)Mn;
        const bool on = tid < B2;
        u32 q = 0, cnt = 0;
        float vmin = 0.f, vmax = 0.f;
        if (on) {
            const int c = tid >= M ? 1 : 0, m = tid - c * M, Ms = c ? Mn : M;
            const u32 K = c ? K1 : K0;
            cnt = m < Ms - 1 ? K : (c ? gn : gp) - K * (u32)(Ms - 1);
            a.blk_start[(size_t)r * (B2 + 1) + tid] = (c ? gp : 0u) + (u32)m * K;
            if (tid == B2 - 1) a.blk_start[(size_t)r * (B2 + 1) + B2] = gp + gn;
            const size_t mi = (size_t)r * B2 + tid;
            q = a.mv.q[mi];
            vmin = a.mv.vmin[mi]; vmax = a.mv.vmax[mi];
        }
        __syncthreads();
        lr_finish_row<DT>(a, r, gp, gn, on, q & 0x7Fu, q & 0x80u, cnt, vmin, vmax, L.mem);
    }
}

// ---- 4. split -------------------------------------------------------------------------------------
constexpr int kSplitNE = 4;          // entries per thread and step (eight spill)
// LDS carve-up (bytes)
struct LrSplitLds { int thr, sums, place, val, tk, gbase, lstart, cnt, inv, vmin, e, er, lidx, wcnt, blk, total; };
// log2 of the places of a class's thresholds: its blocks and at least one more
__host__ __device__ inline int lr_split_steps(int M, int Mn)
{
    int n = 1;
    while ((1 << n) <= (M > Mn ? M : Mn)) ++n;
    return n;
}
// room for a step's entries with every block padded to whole groups of kSplitNE
__host__ __device__ inline int lr_split_room(int B2) { return (kTileThreads + B2 + 1) * kSplitNE; }     // (and one group for what is not kept)
__host__ __device__ inline LrSplitLds lr_split_carve(int M, int Mn, int nq)
{
    LrSplitLds o;
    const int B2 = M + Mn, EC = lr_split_room(B2);
    int p = 0;
    o.thr = p;    p += 8 * B2;
    o.sums = p;   p += 8 * B2 * (nq + 1);
    o.place = p;  p += 8 * B2;
    o.val = (p + 15) & ~15; p = o.val + 4 * EC;
    o.tk = p;     p += 8 << lr_split_steps(M, Mn);
    o.gbase = p;  p += 4 * B2;
    o.lstart = p; p += 4 * (B2 + 1);
    o.cnt = p;    p += 4 * B2;
    o.inv = p;    p += 4 * B2 * nq;
    o.vmin = p;   p += 4 * B2;
    o.e = p;      p += 4 * B2;
    o.er = p;     p += 4 * B2;
    o.lidx = p;   p += 2 * EC;
    o.wcnt = p;   p += 2 * (kTileThreads / kWave) * B2;
    o.blk = p;    p += EC / kSplitNE;
    o.total = (p + 15) & ~15;
    return o;
}

// loads of what other workgroups of the launch have written, past the caches of one XCD
__device__ inline u64 agent_load(const u64* p) { return __hip_atomic_load(const_cast<u64*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// ABQ sums of the first `left` of kSplitNE values of one block (keys as fp32 patterns): acc[t] += squared residual (or DS mismatch) at the
// t-th bitwidth; returns the energy.  inv15: 2^15 L / (range brought to [1, 2)) per bitwidth, 0 for a block of range 0.
// MODE 0: squared error, bitwidths up to 8; 1: squared error, any bitwidth; 2: Eq. "DS"
template <int DT, int NQ, int MODE>
__device__ inline u64 lr_abq_entries(const LargeArgs& a, int nq, const u32 (&vv)[kSplitNE], u32 left, float vmin, int e, int er, const float* inv15,
                                     u32 (&acc)[NQ ? NQ : kMaxQ])
{
    constexpr int QN = NQ ? NQ : kMaxQ;
    float inv[QN];
#pragma unroll
    for (int t = 0; t < QN; ++t) inv[t] = (NQ || t < nq) ? inv15[t] : 0.f;
    float inv_top = 0.f;
    const int top = nq - 1, qtop = a.qlist[top];
    if (MODE == 2) inv_top = inv15[top] * 0x1p-15f;
    u64 accE = 0;
#pragma unroll
    for (int j = 0; j < kSplitNE; ++j) {
        const bool in = (u32)j < left;
        const float av = in ? __uint_as_float(vv[j]) : vmin;   // (an offset of zero adds nothing to any residual)
        const u64 A = in ? (u64)(u32)rintf(ldexpf(av, 20 - e)) : 0ull;     // 20-bit energy grid scaled to vmax
        accE += A * A;
        const float d = to_unit(av - vmin, er);                // (range 0: every offset is zero)
        if (MODE == 2) {
            // | (code at q_bit >> (q_bit - q)) - code at q | for every lower bitwidth
            const u32 c0 = (u32)rintf(d * inv_top);               // within [0, 2^q - 1]: no clamp needed
#pragma unroll
            for (int t = 0; t < QN; ++t) {
                if ((NQ || t < nq) && t < top) {
                    const u32 c = (u32)rintf(d * (inv[t] * 0x1p-15f));
                    const u32 ref = c0 >> (u32)(qtop - a.qlist[t]);
                    acc[t] += ref > c ? ref - c : c - ref;
                }
            }
        } else {
            // residual on the 2^-15 grid: rint(y * 2^15) reduced to 15 signed bits (Sec. 3.2.1 metric
            // in the code domain); bitwidths up to 8 keep y * 2^15 below 2^23, where adding 2^23
            // rounds to the integer grid with the same round-half-even
#pragma unroll
            for (int t = 0; t < QN; ++t) {
                if (NQ || t < nq) {
                    const u32 zi = MODE == 0 ? __float_as_uint(d * inv[t] + 8388608.0f) : (u32)rintf(d * inv[t]);
                    const int rho = __builtin_amdgcn_sbfe((int)zi, 0u, 15u);
                    acc[t] += (u32)(rho * rho);
                }
            }
        }
    }
    return accE;
}

// NQ > 0: the number of allowed bitwidths is known at compile time; NQ == 0: any number up to 16.
template <int DT, int NQ>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(8))) void lr_split_kernel(LargeArgs a)
{
    typedef Elem<DT> E;
    constexpr int QN = NQ ? NQ : kMaxQ, NWV = kTileThreads / kWave, NE = kSplitNE, EC = kTileThreads * NE;
    static_assert(NE <= 8, "u32 partial sums hold 8 residuals of 2^28");
    extern __shared__ __align__(16) unsigned char smem8[];
    const int tid_in = threadIdx.x, tid = tid_in, s = blockIdx.x, wv = tid / kWave, w = a.w, M = a.M, Mn = a.Mn, B2 = M + Mn, S = a.S;
    const int nq = NQ ? NQ : a.nq;
    const u32 lane = lane_id();
    const int64_t r = blockIdx.y;
    u32* st = a.rowst + (size_t)r * 16;
    const u32 seg0 = a.seg[((size_t)r * S + s) * 2], ntp = a.seg[((size_t)r * S + s) * 2 + 1];
    if (st[kStFlag]) return;                         // encoded by the bounds stage
    const u32 nt = (ntp & 0xFFFFu) + (ntp >> 16);
    const LrSplitLds o = lr_split_carve(M, Mn, nq);
    u64* thr = (u64*)(smem8 + o.thr);
    u64* sums = (u64*)(smem8 + o.sums);
    u32* val = (u32*)(smem8 + o.val);
    u32* gbase = (u32*)(smem8 + o.gbase);
    u32* lstart = (u32*)(smem8 + o.lstart);
    float* invt = (float*)(smem8 + o.inv);
    float* vminf = (float*)(smem8 + o.vmin);
    int* e_tab = (int*)(smem8 + o.e);
    int* er_tab = (int*)(smem8 + o.er);
    uint16_t* lidx = (uint16_t*)(smem8 + o.lidx);
    uint16_t* wcnt = (uint16_t*)(smem8 + o.wcnt);
    uint8_t* blk = (uint8_t*)(smem8 + o.blk);        // block of every group of NE places
    u32* cntb = (u32*)(smem8 + o.cnt);
    uint2* place = (uint2*)(smem8 + o.place);        // position of a block's entry in the row minus its place here; end of its places
    constexpr u32 kNone = 0xFFu;                     // not kept
    constexpr int kMaskBlocks = 32;
    const int room = lr_split_room(B2);
    static_assert(8 * (kTileThreads / kWave) * (kMaskBlocks + 1) <= 4 * kTileThreads + 4 * kMaskBlocks, "the masks fit the sorted entries");
    u32* tk = (u32*)(smem8 + o.tk);                  // thresholds as c32, one class after the other
    const int steps = lr_split_steps(M, Mn);
    const LrList list(a, r);
    const u32* __restrict__ Lraw = list.raw + seg0;
    const uint16_t* __restrict__ Lidx = list.idx + seg0;
    const u32 tile0 = (u32)(s * a.tile);             // index of the tile's element 0
    const bool want_sums = !a.lad.on;

    u32 rw[NE], ix[NE];
    auto fetch = [&](u32 e0) {
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const u32 p = e0 + (u32)(wv * NE + j) * kWave + lane;
            rw[j] = p < nt ? Lraw[p] : 0u;
            ix[j] = p < nt ? (u32)Lidx[p] : 0u;
        }
    };
    fetch(0);
    // the tile's place in every block: the entries of the tiles before it, sixteen lanes a block and a scan
    for (int b0 = 0; b0 < B2; b0 += kTileThreads / 16) {
        const int b = b0 + tid / 16;
        const u32* pr = a.pair + ((size_t)r * B2 + (b < B2 ? b : 0)) * S;
        u32 n = 0;
        for (int t0 = tid & 15; t0 < s; t0 += 64) {
            u32 c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = t0 + 16 * u < s ? pr[t0 + 16 * u] : 0u;
            n += (c[0] + c[1]) + (c[2] + c[3]);
        }
        n = row_scan_dpp(n);
        if (b < B2 && (tid & 15) == 15) cntb[b] = n;     // with the blocks of its class before it (an empty block's is not looked at)
    }
    float* rngf = (float*)val;
    for (int i = tid; i < 2 << steps; i += kTileThreads) {
        const int c = i >> steps, m = i - (c << steps);
        u32 t = 0;                                   // (behind a class's blocks: below everything)
        if (m < (c ? Mn : M)) {
            const int b = c * M + m;
            const size_t rb = (size_t)r * B2 + b;
            const u64 cx = a.thr[rb];
            t = cx == ~0ull ? ~0u : lr_c32<DT>((u32)(cx >> w), (1u << w) - 1u - ((u32)cx & ((1u << w) - 1u)), w);
            thr[b] = cx;
            gbase[b] = a.blk_start[(size_t)r * (B2 + 1) + b];
            const u32 lo = E::value_bits(a.vminb[rb]), hi = E::value_bits(a.vmaxb[rb]);
            const float vmin = __uint_as_float(lo), rng = __uint_as_float(hi) - vmin;
            vminf[b] = vmin;
            rngf[b] = rng;
            er_tab[b] = rng > 0.f ? range_exp(rng) : 0;              // only a range of exactly 0 is degenerate
            e_tab[b] = cx != ~0ull ? ilogb_bits(hi) + 1 : 0;
        }
        tk[i] = t;
    }
    for (int i = tid; i < B2 * (nq + 1); i += kTileThreads) sums[i] = 0;
    __syncthreads();
    for (int i = tid; i < B2 * nq; i += kTileThreads) {              // quantiser scales 2^15 L / (range brought to [1, 2))
        const int b = i / nq, t = i - b * nq;
        const float rng = rngf[b];
        invt[i] = rng > 0.f ? (float)((1u << a.qlist[t]) - 1u) / unit_range(rng, er_tab[b]) * 32768.0f : 0.f;      // (times 2^15: exact)
    }
    if (tid < B2) {
        const bool first = tid == 0 || tid == M || thr[tid - 1] == ~0ull;
        gbase[tid] += cntb[tid] - (first ? 0u : cntb[tid - 1]);
    }
    int nbits = 0;
    while ((1 << nbits) < B2) ++nbits;
    const int mode = a.guard == 1 ? 2 : a.qlist[nq - 1] > 8 ? 1 : 0;      // (the bitwidths ascend)
    u32* __restrict__ bo_idx = a.bo_idx + (size_t)r * (size_t)a.k;
    u32* __restrict__ bo_val = a.bo_val + (size_t)r * (size_t)a.k;

    for (u32 e0 = 0; e0 < nt; e0 += EC) {
        // (an opaque copy: the addresses below are cheap, and hoisting all of them out of this loop, which runs once or
        //  twice, spilled up to 50 registers: 68 against 64 us on a batch of 32 maps)
        int tid = tid_in;
        asm volatile("" : "+v"(tid));
        const u32 lane = (u32)tid & (u32)(kWave - 1);
        const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
        for (int i = tid; i < NWV * B2 / 2; i += kTileThreads) ((u32*)wcnt)[i] = 0;      // (16 * B2 counters)
        __syncthreads();
        // (a) block of every entry: how many of its class's thresholds lie above it, by bisection over their leading bits (they
        // descend; empty blocks, whose threshold is the largest, come first).  Straight-line code: the lookups of a lane's entries
        // overlap.  A table of blocks by fine bin took twice the instructions, and 5 KB a workgroup to load: the first 6.6 us of a workgroup's 27 on
        // fp32 [32 x 401408], now 3.5 of 22.
        u32 bk[NE], rank[NE];
        {
            u32 c32[NE], pos[NE];
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const u32 key = DT == 0 ? rw[j] & 0x7FFFFFFFu : (rw[j] >> 16) & 0x7FFFu;
                c32[j] = lr_c32<DT>(key, tile0 + ix[j], w);
                pos[j] = (rw[j] >> 31) << steps;
            }
#pragma unroll
            for (int n = 7; n > 0; --n) {
                if (n > steps) continue;             // uniform
                const u32 step = 1u << (n - 1);
#pragma unroll
                for (int j = 0; j < NE; ++j) pos[j] += tk[pos[j] + step - 1u] > c32[j] ? step : 0u;
            }
            bool tie = false;
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const u32 neg = rw[j] >> 31, m = pos[j] - (neg << steps), b = m + (neg ? (u32)M : 0u);
                const bool in = e0 + (u32)(wv * NE + j) * kWave + lane < nt && m < (u32)(neg ? Mn : M);
                tie |= in && tk[pos[j]] == c32[j];
                bk[j] = in ? b : kNone;
            }
            if (__any(tie)) {                        // leading bits alike: the whole order decides
#pragma unroll
                for (int j = 0; j < NE; ++j) {
                    const u32 c1 = rw[j] >> 31 ? (u32)B2 : (u32)M;
                    const u32 key = DT == 0 ? rw[j] & 0x7FFFFFFFu : (rw[j] >> 16) & 0x7FFFu;
                    const u64 cx = lr_comp(key, tile0 + ix[j], w);
                    while (bk[j] != kNone && thr[bk[j]] > cx) bk[j] = bk[j] + 1u < c1 ? bk[j] + 1u : kNone;
                }
            }
        }
        // (b) stable rank inside the wavefront's 64 * NE consecutive entries: a bit mask of the lanes per block and slot
        // (in the storage of the sorted entries; row B2 takes what is not kept), or with many blocks one ballot per bit of
        // the block number
        if (B2 <= kMaskBlocks) {
            const int MB = B2 + 1;
            u64* mk = (u64*)val + wv * NE * MB;
            uint16_t* pf = lidx + wv * NE * MB;
            for (int i = (int)lane; i < NE * MB; i += kWave) mk[i] = 0;
            wave_sync();
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const int b = bk[j] != kNone ? (int)bk[j] : B2;
                atomicOr((u32*)(mk + j * MB + b) + (lane >> 5), 1u << (lane & 31u));
            }
            wave_sync();
            if ((int)lane < B2) {
                u64 m[NE];
                u32 run = 0;
#pragma unroll
                for (int j = 0; j < NE; ++j) m[j] = mk[j * MB + (int)lane];
#pragma unroll
                for (int j = 0; j < NE; ++j) { pf[j * MB + (int)lane] = (uint16_t)run; run += (u32)__popcll(m[j]); }
                wcnt[wv * B2 + (int)lane] = (uint16_t)run;
            }
            wave_sync();
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const int b = bk[j] != kNone ? (int)bk[j] : B2;
                rank[j] = (u32)pf[j * MB + b] + mask_rank(mk[j * MB + b]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const bool kept = bk[j] != kNone;
                const u32 b = kept ? bk[j] : 0u;
                const u64 km = __ballot(kept);
                u32 plo = (u32)km, phi = (u32)(km >> 32);
                for (int bit = 0; bit < nbits; ++bit) {
                    const u32 onm = (u32)__builtin_amdgcn_sbfe((int)b, (u32)bit, 1u);
                    const u64 bal = __ballot(onm != 0u);
                    plo &= ~((u32)bal ^ onm);
                    phi &= ~((u32)(bal >> 32) ^ onm);
                }
                const u32 before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
                u32 run = 0;
                if (kept) run = wcnt[wv * B2 + (int)b];
                wave_sync();
                if (kept && before == 0) wcnt[wv * B2 + (int)b] = (uint16_t)(run + (u32)__popc(plo) + (u32)__popc(phi));
                wave_sync();
                rank[j] = run + before;
            }
        }
        __syncthreads();
        if (wv == 0) {                               // per block: the wavefronts' places, then the blocks' places (two blocks per lane)
            u32 tot[2] = { 0, 0 };
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int b = 2 * (int)lane + h;
                if (b < B2) {
                    u32 c[NWV];
#pragma unroll
                    for (int v = 0; v < NWV; ++v) c[v] = wcnt[v * B2 + b];
#pragma unroll
                    for (int v = 0; v < NWV; ++v) { wcnt[v * B2 + b] = (uint16_t)tot[h]; tot[h] += c[v]; }
                }
            }
            constexpr u32 PM = (u32)NE - 1u;         // every block starts on a whole group of NE places
            const u32 pad[2] = { (tot[0] + PM) & ~PM, (tot[1] + PM) & ~PM };
            const u32 incl = wave_scan_dpp(pad[0] + pad[1]);
            const u32 ex = incl - pad[0] - pad[1];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int b = 2 * (int)lane + h;
                if (b < B2) {
                    const u32 at = ex + (h ? pad[0] : 0u);
                    lstart[b] = at; cntb[b] = tot[h];
                    for (u32 g = at / NE; g < (at + pad[h]) / NE; ++g) blk[g] = (uint8_t)b;
                }
            }
            if (lane == kWave - 1) lstart[B2] = incl;
        }
        __syncthreads();
        const u32 n_it = lstart[B2];
        if (tid < B2) place[tid] = make_uint2(gbase[tid] - lstart[tid], lstart[tid] + cntb[tid]);
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const bool kept = bk[j] != kNone;
            const u32 b = kept ? bk[j] : 0u;
            const u32 at = kept ? lstart[b] + (u32)wcnt[wv * B2 + (int)b] + rank[j] : (u32)(room - 1);
            val[at] = DT == 0 ? rw[j] & 0x7FFFFFFFu : rw[j] & 0x7FFF0000u;
            lidx[at] = (uint16_t)ix[j];
        }
        __syncthreads();
        if (e0 + EC < nt) fetch(e0 + EC);
        // (c) to the block-ordered arrays, in runs
        for (u32 i1 = 0; i1 < n_it; i1 += 4 * kTileThreads) {
#pragma unroll
            for (u32 u = 0; u < 4; ++u) {
                const u32 i = i1 + u * kTileThreads + (u32)tid, ic = i < n_it ? i : 0u;
                const uint2 pl = place[blk[ic / NE]];
                const u32 g = pl.x + ic, ixv = tile0 + (u32)lidx[ic], vv = val[ic];
                if (i < n_it && i < pl.y && (int64_t)g < a.k) {      // (the last test always holds)
                    bo_idx[g] = ixv;
                    bo_val[g] = vv;
                }
            }
        }
        // (d) ABQ sums: a thread takes a group of NE places, all of one block; the lanes of one block inside each
        // row of sixteen are added up by a segmented scan, and the last lane of a segment adds to the table
        if (want_sums) {
            for (u32 i0 = (u32)tid * NE; i0 < n_it + (u32)(kWave * NE); i0 += kTileThreads * NE) {
                if ((i0 & ~(u32)(kWave * NE - 1)) >= n_it) break;        // uniform in the wavefront
                const bool on = i0 < n_it;
                const u32 b = on ? (u32)blk[i0 / NE] : 0xFFFFu, bb = on ? b : 0u;
                const u32 left = on ? cntb[bb] - (i0 - lstart[bb]) : 0u;
                u32 vv[NE];
#pragma unroll
                for (int j = 0; j < NE; j += 4) {
                    uint4 t = make_uint4(0, 0, 0, 0);
                    if (on) t = *(const uint4*)(val + i0 + j);
                    vv[j] = t.x; vv[j + 1] = t.y; vv[j + 2] = t.z; vv[j + 3] = t.w;
                }
                u32 acc[QN];
#pragma unroll
                for (int t = 0; t < QN; ++t) acc[t] = 0;
                u64 accE;
                if (mode == 0) accE = lr_abq_entries<DT, NQ, 0>(a, nq, vv, left, vminf[bb], e_tab[bb], er_tab[bb], invt + bb * nq, acc);
                else if (mode == 1) accE = lr_abq_entries<DT, NQ, 1>(a, nq, vv, left, vminf[bb], e_tab[bb], er_tab[bb], invt + bb * nq, acc);
                else accE = lr_abq_entries<DT, NQ, 2>(a, nq, vv, left, vminf[bb], e_tab[bb], er_tab[bb], invt + bb * nq, acc);
                // low 28 bits of every sum, and what is above them four to a word (at most 16 * 8 each)
                u32 hi4[(QN + 3) / 4];
#pragma unroll
                for (int t = 0; t < (QN + 3) / 4; ++t) hi4[t] = 0;
#pragma unroll
                for (int t = 0; t < QN; ++t) { hi4[t / 4] |= (acc[t] >> 28) << (8 * (t & 3)); acc[t] &= 0xFFFFFFFu; }
                u32 e0 = (u32)accE & 0xFFFFFFFu, e1 = (u32)(accE >> 28);
                u32 m[4];                                // all ones where the lane 1, 2, 4, 8 below is of the same block
                m[0] = dpp_get<0x111, 0xf, 0xf>(b + 1u) == b + 1u ? ~0u : 0u;
                m[1] = dpp_get<0x112, 0xf, 0xf>(b + 1u) == b + 1u ? ~0u : 0u;
                m[2] = dpp_get<0x114, 0xf, 0xf>(b + 1u) == b + 1u ? ~0u : 0u;
                m[3] = dpp_get<0x118, 0xf, 0xf>(b + 1u) == b + 1u ? ~0u : 0u;
                auto seg_scan = [&](u32 v) -> u32 {      // (lanes outside the row read zero)
                    v += dpp_get<0x111, 0xf, 0xf>(v) & m[0];
                    v += dpp_get<0x112, 0xf, 0xf>(v) & m[1];
                    v += dpp_get<0x114, 0xf, 0xf>(v) & m[2];
                    v += dpp_get<0x118, 0xf, 0xf>(v) & m[3];
                    return v;
                };
                const u32 nxt = dpp_get<0x101, 0xf, 0xf>(b + 1u);        // row_shl:1 (zero for a row's last lane)
                const bool last = on && nxt != b + 1u;
#pragma unroll
                for (int t = 0; t < (QN + 3) / 4; ++t) hi4[t] = seg_scan(hi4[t]);
#pragma unroll
                for (int t = 0; t < QN; ++t) {
                    if (NQ || t < nq) {
                        const u32 lo = seg_scan(acc[t]);
                        if (last) atomicAdd(&sums[bb * (u32)(nq + 1) + (u32)t], (u64)lo + ((u64)((hi4[t / 4] >> (8 * (t & 3))) & 0xFFu) << 28));
                    }
                }
                e0 = seg_scan(e0); e1 = seg_scan(e1);
                if (last) atomicAdd(&sums[bb * (u32)(nq + 1) + (u32)nq], (u64)e0 + ((u64)e1 << 28));
            }
        }
        __syncthreads();
        if (tid < B2) gbase[tid] += cntb[tid];
    }
    // the tile's sums leave the workgroup; the row's last workgroup chooses
    __syncthreads();
    const int ns = B2 * (nq + 1);
    u64* rs = a.sums + (size_t)r * ns;
    if (want_sums && S > 1) for (int i = tid; i < ns; i += kTileThreads) if (sums[i]) __hip_atomic_fetch_add(&rs[i], sums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // The sums alone must be seen by the row's last workgroup: they are added where all XCDs meet and waited for before the
    // ticket is drawn, and are loaded from there.  A ticket with release and acquire order writes back the whole L2, dirty with the
    // block-ordered entries, once per workgroup: encode of 32 maps of 401408 with a ladder 113 -> 133 us, DS guard 123 -> 138.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the additions have been made ...
    __syncthreads();
    if (tid == 0) lstart[0] = S > 1 ? __hip_atomic_fetch_add(&st[kStTicket], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;   // ... before the ticket
    __syncthreads();
    if (lstart[0] != (u32)S - 1u) return;
    if (want_sums && S > 1) {
        for (int i = tid; i < ns; i += kTileThreads) sums[i] = agent_load(&rs[i]);
    }
    __syncthreads();
    const int b = tid;
    const bool on = b < B2;
    u32 q = 0, flag = 0, cnt = 0;
    float vmin = 0.f, vmax = 0.f;
    if (on) {
        cnt = a.blk_start[(size_t)r * (B2 + 1) + b + 1] - a.blk_start[(size_t)r * (B2 + 1) + b];
        int chosen = 0;
        if (cnt) {
            const u32 hi = E::value_bits(a.vmaxb[r * B2 + b]);
            vmin = vminf[b];
            vmax = __uint_as_float(hi);
            const float rng = vmax - vmin;
            if (rng > 0.f && a.guard == 0 && !a.lad.on) {
                const double rhs = a.beta * ldexp((double)sums[b * (nq + 1) + nq], 2 * e_tab[b] - 40);
                chosen = -1;
                for (int t = 0; t < nq && chosen < 0; ++t) {
                    const float ostep = rng / (float)((1u << a.qlist[t]) - 1u);
                    const double lhs = ((double)ostep * (double)ostep) * (double)sums[b * (nq + 1) + t] * 0x1p-30;
                    if (lhs <= rhs) chosen = t;
                }
                if (chosen < 0) { chosen = nq - 1; flag = 0x80u; }
            }
            if (a.guard == 1) {                      // greedy descent from q_bit while the mismatch stays within delta
                chosen = nq - 1;
                for (int t = nq - 2; t >= 0; --t) {
                    if ((double)sums[b * (nq + 1) + t] <= a.beta * (double)cnt) chosen = t; else break;
                }
            }
        }
        if (a.lad.on) chosen = (int)ladder_index(a.lad, b < M ? b : b - M);      // given, also for empty and degenerate blocks
        q = (u32)a.qlist[chosen];
    }
    __syncthreads();                                 // the sums have been read: their storage takes the blocks' code bits
    lr_finish_row<DT>(a, r, st[kStNpos], st[kStNneg], on, q, flag, cnt, vmin, vmax, sums);
}

// ---- 5. pack --------------------------------------------------------------------------------------
// A thread packs a run of consecutive fields into whole words in registers and writes each
// word of the window image once: the first and the last word of a run may be shared with the
// neighbouring runs (atomic OR), the words between belong to this run alone (plain store).
struct RunPacker {
    u32* stage;
    int nwords;          // words of the window
    u64 acc;
    int fill, wi;
    bool first;
    __device__ inline void begin(u32* st, int nw, int rel)      // rel: first bit, relative to the window (may be negative)
    {
        stage = st; nwords = nw;
        wi = rel >> 5; fill = rel & 31; acc = 0; first = true;
    }
    __device__ inline void put(u32 wd, bool shared)
    {
        if (wi >= 0 && wi < nwords) {
            if (shared) atomicOr(&stage[wi], wd); else stage[wi] = wd;
        }
    }
    __device__ inline void append(u32 v, int nb)                 // nb <= 32, v < 2^nb
    {
        acc |= (u64)v << fill;
        fill += nb;
        if (fill >= 32) {
            put((u32)acc, first);
            first = false;
            acc >>= 32; fill -= 32; ++wi;
        }
    }
    __device__ inline void finish() { if (fill > 0) put((u32)acc, true); }
};

constexpr int kPackPtrs = 4096;                   // row pointers of one window at most

// CSR: row pointers and columns instead of flat indices (Sec. 3.2 step 3)
template <int DT, bool CSR>
__global__ __launch_bounds__(256) void lr_pack_kernel(LargeArgs a, FinishArgs fa)
{
    constexpr int RUN = 8;                        // consecutive entries per thread and run
    __shared__ u32 sA[kPackWords];
    __shared__ u32 bs[kMaxB2 + 1], qsel[kMaxB2];
    __shared__ u32 crel[kMaxB2];                  // first code bit of the block relative to the window, modulo 2^32
    __shared__ float vminf[kMaxB2], invs[kMaxB2];
    __shared__ int ers[kMaxB2];
    __shared__ u32 s_rng[2];
    __shared__ u64 s_off[2];
    __shared__ u32 ptrs[CSR ? kPackPtrs : 1];
    const int tid = threadIdx.x;
    const int64_t r = blockIdx.y;
    const int B2 = a.M + a.Mn, wi = CSR ? a.wc : a.w;
    // Windows of row pointers alone, which take longest, are started first, then those with code fields, which hold the most
    // entries.  (As windows of 1024 words behind the others the pointers made the tail of the launch: fp32 32 x [512 x 784] pack
    // 52 us, now 29.)
    const int nwp = CSR ? a.nwin_ptr : 0, nwc = a.nwin - a.nwin_idx, wx = (int)blockIdx.x - nwp;
    const int win = wx < 0 ? (int)blockIdx.x : wx < nwc ? a.nwin_idx + wx : nwp + wx - nwc;
    const u64 row_words = a.row_words[r];
    const u32 n = a.blk_start[(size_t)r * (B2 + 1) + B2];
    const u64 ptr_bits = CSR ? (u64)B2 * (u64)(a.n_rows + 1) * (u64)a.wp : 0ull;
    const u64 idx_bits = ptr_bits + (u64)n * (u64)wi;       // first code bit
    // windows of pack_words words up to the first word that holds code bits, then of pack_words_code words
    u64 c0, c1;
    {
        const u64 wb = idx_bits >> 5, wq = nwp ? ptr_bits >> 5 : 0ull;
        if (CSR && win < nwp) {
            c0 = (u64)win * (u64)a.pack_words_ptr;
            c1 = c0 + (u64)a.pack_words_ptr < wq ? c0 + (u64)a.pack_words_ptr : wq;
        } else if (win < a.nwin_idx) {
            c0 = wq + (u64)(win - nwp) * (u64)a.pack_words;
            c1 = c0 + (u64)a.pack_words < wb ? c0 + (u64)a.pack_words : wb;
        } else {
            c0 = wb + (u64)(win - a.nwin_idx) * (u64)a.pack_words_code;
            c1 = c0 + (u64)a.pack_words_code;
        }
        c1 = c1 < row_words ? c1 : row_words;
    }
    const bool lead = win == 0;                      // also the row's offset; of row 0 also the header
    if (c1 <= c0 && !lead) return;
    const int cw = c1 > c0 ? (int)(c1 - c0) : 0;
    const u64 lo = c0 << 5, hi = lo + ((u64)cw << 5);
    const u32* __restrict__ bo_idx = a.bo_idx + (size_t)r * (size_t)a.k;
    const u32* __restrict__ bo_val = a.bo_val + (size_t)r * (size_t)a.k;
    // index fields that meet the window; their first run is in flight while the tables arrive
    u32 iq0 = 0, iq1 = 0;
    if (cw && lo < idx_bits && hi > ptr_bits) {
        iq0 = lo > ptr_bits ? (u32)((lo - ptr_bits) / (u64)wi) : 0u;
        const u64 t1 = (hi - ptr_bits + (u64)wi - 1) / (u64)wi;
        iq1 = t1 > (u64)n ? n : (u32)t1;
    }
    u32 vi[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) { const u32 p = iq0 + (u32)tid * RUN + (u32)u; vi[u] = p < iq1 ? bo_idx[p] : 0u; }
    if (a.direct && tid < kWave) {                   // words of the rows before this one (at most 256 rows)
        u64 before = 0, total = 0;
#pragma unroll
        for (int j = 0; j < kScanRows / kWave; ++j) {
            const int64_t i = (int64_t)j * kWave + tid;
            const u64 t = i < a.R ? a.row_words[i] : 0ull;
            total += t;
            if (i < r) before += t;
        }
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) { before += __shfl_xor(before, d); total += __shfl_xor(total, d); }
        if (tid == 0) { s_off[0] = before; s_off[1] = total; }
    }
    if (tid == 0) { s_rng[0] = n; s_rng[1] = 0; }
    __syncthreads();
    for (int b = tid; b < B2; b += 256) {
        const size_t rb = (size_t)r * B2 + b;
        const u32 b0 = a.blk_start[(size_t)r * (B2 + 1) + b], q = a.qsel[rb];
        bs[b] = b0;
        if (b == B2 - 1) bs[B2] = n;
        qsel[b] = q;
        invs[b] = a.inv_sel[rb];
        vminf[b] = a.mv.vmin[rb];
        const float rng = a.mv.vmax[rb] - vminf[b];
        ers[b] = rng > 0.f ? range_exp(rng) : 0;          // blocks of range 0 have inv = 0 and are not scaled
        const u64 cs = idx_bits + a.code_off[(size_t)r * (B2 + 1) + b], ce = idx_bits + a.code_off[(size_t)r * (B2 + 1) + b + 1];
        crel[b] = (u32)(cs - lo);
        if (ce > cs && ce > lo && cs < hi) {              // the block's entries whose code field meets the window (fewer than 2^31 bits)
            const u32 dlo = (u32)((lo > cs ? lo : cs) - cs), dhi = (u32)((hi < ce ? hi : ce) - cs);
            atomicMin(&s_rng[0], b0 + dlo / q);
            atomicMax(&s_rng[1], b0 + (dhi + q - 1) / q);
        }
    }
    for (int i = tid; i < cw; i += 256) sA[i] = 0;
    __syncthreads();
    if (a.direct && lead && tid == 0) {
        a.mv.row_off[r] = s_off[0];
        if (r == 0) {
            write_header(fa, s_off[1]);
            if (CSR) { u32* h32 = (u32*)a.meta; h32[11] = (u32)a.wc; h32[15] = (u32)a.n_cols; }
        }
    }
    if (!cw) return;
    const u32 cq0 = s_rng[0], cq1 = s_rng[1];
    u32 vc[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) { const u32 p = cq0 + (u32)tid * RUN + (u32)u; vc[u] = p < cq1 ? bo_val[p] : 0u; }
    const u32 ncols = (u32)a.n_cols, rcp = CSR ? (ncols > 1u ? (u32)((1ull << 32) / ncols) : 0xFFFFFFFFu) : 0u;
    auto tensor_row = [&](u32 idx) -> u32 {          // idx / n_cols: the scaled reciprocal is at most one too low for idx < 2^31
        u32 q = __umulhi(idx, rcp);
        if (idx - q * ncols >= ncols) ++q;
        return q;
    };
    RunPacker rp;
    // Bit positions are taken relative to the window in 32-bit arithmetic: the true value of
    // every position handled here lies within a few bits of the window, so the wrapped
    // difference is exact.
    const u32 lo32 = (u32)lo;
    if (CSR && lo < ptr_bits) {
        // Pointer j of a block = number of its entries in tensor rows before j.  Either every pointer is searched for, a
        // lane each, over the pointers of all such blocks in the window at once, or the block's entries are walked: an
        // entry settles the pointers from the row after its predecessor's to its own; the last one also those behind it.
        // The walk is for blocks with about as many entries as pointers.  With an eighth of them or fewer a lane writes
        // long runs; with more than sixteen a pointer most entries settle nothing.  Encode call with every block walked
        // whole by every window, and now: fp32 32 x [1 x 401408] 246 -> 127 us, 8 x [401408 x 1] in one block 288 -> 114 us,
        // 1 x [64 x 3136] 81 -> 58 us; 32 x [512 x 784] 157 -> 150 us.
        const u32 np1 = (u32)a.n_rows + 1u;
        const u64 n_ptr = (u64)B2 * np1;
        const u64 f0 = lo / (u64)a.wp, fe = (hi + (u64)a.wp - 1) / (u64)a.wp, f1 = fe < n_ptr ? fe : n_ptr;
        const u32 bl0 = (u32)(f0 / np1), bl1 = (u32)((f1 - 1) / np1), first = (u32)(f0 - (u64)bl0 * np1);
        const float rnp = 1.0f / (float)np1;
        auto walked = [&](u32 cnt) -> bool { return cnt * 8u >= np1 && cnt <= 16u * np1; };
        auto search = [&](u32 p0, u32 cnt, u32 j) -> u32 {
            const u64 target = (u64)j * ncols;
            u32 l = 0, h = cnt;
            while (l < h) { const u32 mid = (l + h) >> 1; if ((u64)bo_idx[p0 + mid] < target) l = mid + 1; else h = mid; }
            return l;
        };
        if (bl1 > bl0) {                             // pointers of several blocks, at most 128
            const u32 bt = bl0 + (u32)tid;
            if (__syncthreads_or(bt <= bl1 && bs[bt + 1] > bs[bt] && !walked(bs[bt + 1] - bs[bt]))) {
                for (u32 i = (u32)tid; i < (u32)(f1 - f0); i += 256) {
                    const u32 f = first + i;
                    u32 db = (u32)((float)f * rnp);  // f / np1, at most kPackPtrs: the float quotient is off by at most one
                    if (db * np1 > f) --db;
                    if ((db + 1u) * np1 <= f) ++db;
                    const u32 p0 = bs[bl0 + db], cnt = bs[bl0 + db + 1] - p0;
                    if (cnt && !walked(cnt)) ptrs[i] = search(p0, cnt, f - db * np1);
                }
            }
        }
        for (u32 b = bl0; b <= bl1; ++b) {
            const u64 fb = (u64)b * np1;
            const u32 j0 = f0 > fb ? (u32)(f0 - fb) : 0u, j1 = f1 < fb + np1 ? (u32)(f1 - fb) : np1;     // pointers [j0, j1)
            u32* out = ptrs + (fb + j0 - f0);        // pointer j0
            const u32 p0 = bs[b], cnt = bs[b + 1] - p0;
            if (!walked(cnt)) {                      // (uniform)
                if (bl1 == bl0 || !cnt) for (u32 j = j0 + (u32)tid; j < j1; j += 256) out[j - j0] = search(p0, cnt, j);      // (empty: zeros)
                continue;
            }
            // entries in tensor rows before j: 256 probes at once
            auto before = [&](u32 j) -> u32 {
                const u64 target = (u64)j * ncols;
                u32 l = 0, n = cnt;
                while (n) {
                    const u32 step = (n + 255u) / 256u, at = (u32)tid * step;
                    const u32 c = (u32)__syncthreads_count(at < n && (u64)bo_idx[p0 + l + at] < target);
                    if (!c) break;
                    const u32 up = (c - 1u) * step + 1u;
                    l += up;
                    n = step - 1u < n - up ? step - 1u : n - up;
                }
                return l;
            };
            // the walk starts at the first entry that settles a pointer of this window and ends at the last one (a short
            // block is walked whole: four steps take no longer than the probes)
            const bool part = cnt > 1024u;
            u32 i0 = part && j0 ? before(j0) : 0u;
            i0 = i0 < cnt ? i0 : cnt - 1u;
            u32 i1 = part && j1 < np1 ? before(j1 - 1u) + 1u : cnt;
            i1 = i1 < cnt ? i1 : cnt;
            for (u32 ib = i0 + (u32)tid; ib < i1; ib += 4 * 256) {      // the entries of four steps in flight
                u32 at[4], bef[4];
#pragma unroll
                for (u32 u = 0; u < 4; ++u) {
                    const u32 i = ib + 256u * u < i1 ? ib + 256u * u : ib;
                    at[u] = bo_idx[p0 + i];
                    bef[u] = i ? bo_idx[p0 + i - 1u] : 0u;
                }
#pragma unroll
                for (u32 u = 0; u < 4; ++u) {
                    const u32 i = ib + 256u * u;
                    if (i >= i1) break;
                    const u32 row = tensor_row(at[u]), prev = i ? tensor_row(bef[u]) + 1u : 0u;
                    const u32 x1 = row + 1u < j1 ? row + 1u : j1;
                    for (u32 j = prev > j0 ? prev : j0; j < x1; ++j) out[j - j0] = i;
                    if (i == cnt - 1u) for (u32 j = row + 1u > j0 ? row + 1u : j0; j < j1; ++j) out[j - j0] = cnt;
                }
            }
        }
        __syncthreads();
        const u32 nf = (u32)(f1 - f0);
        for (u32 p0 = (u32)tid * RUN; p0 < nf; p0 += 256 * RUN) {
            rp.begin(sA, cw, (int)((u32)f0 * (u32)a.wp + p0 * (u32)a.wp - lo32));
#pragma unroll
            for (int u = 0; u < RUN; ++u)
                if (p0 + (u32)u < nf) rp.append(ptrs[p0 + (u32)u], a.wp);
            rp.finish();
        }
    }
    for (u32 p0 = iq0 + (u32)tid * RUN; p0 < iq1; p0 += 256 * RUN) {
        if (p0 != iq0 + (u32)tid * RUN) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) { const u32 p = p0 + (u32)u; vi[u] = p < iq1 ? bo_idx[p] : 0u; }
        }
        rp.begin(sA, cw, (int)((u32)ptr_bits + p0 * (u32)wi - lo32));
#pragma unroll
        for (int u = 0; u < RUN; ++u)
            if (p0 + (u32)u < iq1) rp.append(CSR ? vi[u] - tensor_row(vi[u]) * ncols : vi[u], wi);
        rp.finish();
    }
    {
        // the block's constants stay in registers until the position leaves the block; the code
        // sections of consecutive blocks are contiguous in the stream, so a run may cross blocks
        int b = 0;
        for (u32 p0 = cq0 + (u32)tid * RUN; p0 < cq1; p0 += 256 * RUN) {
            if (p0 != cq0 + (u32)tid * RUN) {
#pragma unroll
                for (int u = 0; u < RUN; ++u) { const u32 p = p0 + (u32)u; vc[u] = p < cq1 ? bo_val[p] : 0u; }
            }
            while (b < B2 - 1 && p0 >= bs[b + 1]) ++b;
            u32 b_end = b < B2 - 1 ? bs[b + 1] : 0xFFFFFFFFu;
            int q = (int)qsel[b];
            float inv = invs[b], vmin = vminf[b], qmaxf = (float)((1u << q) - 1u);
            int er = ers[b];
            rp.begin(sA, cw, (int)(crel[b] + (p0 - bs[b]) * (u32)q));
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const u32 p = p0 + (u32)u;
                if (p >= cq1) break;
                if (p >= b_end) {
                    while (b < B2 - 1 && p >= bs[b + 1]) ++b;
                    b_end = b < B2 - 1 ? bs[b + 1] : 0xFFFFFFFFu;
                    q = (int)qsel[b]; inv = invs[b]; vmin = vminf[b]; qmaxf = (float)((1u << q) - 1u); er = ers[b];
                }
                u32 c = 0;
                if (inv != 0.f) {
                    const float y = to_unit(__uint_as_float(vc[u]) - vmin, er) * inv;
                    c = (u32)fminf(fmaxf(rintf(y), 0.f), qmaxf);
                }
                rp.append(c, q);
            }
            rp.finish();
        }
    }
    __syncthreads();
    u32* __restrict__ dst = a.direct ? a.stream + s_off[0] : a.slots + (size_t)r * (size_t)a.cap_words;
    for (int i = tid; i < cw; i += 256) dst[c0 + i] = sA[i];
}

}  // namespace slicer
