// Row-resident encoder for short rows: ONE WAVEFRONT PER ROW, the row held in
// registers, every list in LDS, no workgroup barrier anywhere.
//
// All ordering is done on one integer per element, the "comp": magnitude key in the high
// bits, inverted index in the low bits (larger comp = larger magnitude, then lower index:
// the tie rule of the top-K filter and of the block ranks), and the sign class as the top
// bit, positive class on top.  Comps are distinct, so a comp is a complete rank threshold.
//
//   1. load the row (16-byte coalesced loads, whatever its length and alignment); its largest magnitude key; a 2048-bin
//      histogram in LDS over a window that hangs from that key (bf16: one key per bin);
//      two-level scan from the top -> the bin B1 that holds rank k-1;
//   2. ordered compaction of everything at or above B1 into a short list L
//      (ascending index: the kept set plus the undecided bin);
//   3. L is bucketed into 1024 fine bins, linear in the key from the list's lower
//      bound, both sign classes counted in one packed table; an exclusive scan from
//      the top gives every bin's places in the list S, which holds the positive class
//      and then the negative one, each arranged by bin.  Order statistics (rank k-1
//      overall for the top-K cut of Sec. 3.1; ranks j*K-1 per class for the block
//      boundaries of Sec. 3.2) are resolved among the members of their bin, and the bin
//      of a class rank is that of the entry of S at this place;
//   4. an entry's block is the number of boundaries above it (plus one for the negative
//      class); a stable split by block id (wave ballots) restores ascending index inside
//      each block;
//   5. ABQ sums on integer grids, bitwidth choice, bit offsets, packing through an
//      LDS image of the row's stream segment.
//
// Rows whose list would not fit (many equal or nearly equal values around the threshold) take the exact cut, found by narrower
// histograms, and list the kept elements alone: no row is left to another kernel.  (With lists of that
// kind flagged and redone by the generic kernel, every call paid for a launch that looks for flags.)
#pragma once

#include <type_traits>

#include "slicer_common.hpp"

namespace slicer {

struct SmallArgs {
    const void* x;
    int64_t R, N, k;
    int M, Mn, w, nq;   // blocks of the positive / negative class
    int qlist[kMaxQ];
    double beta;
    u64 cap_words;
    u64* row_words;     // [R] workgroup-per-row kernel
    u32* row_words32;   // [R] one-wavefront kernel
    u32* slots;         // [R][cap_words]
    u32* fallback;      // [R] workgroup-per-row kernel: 1 = redo this row with the generic kernel
    u32* stream;        // one-wavefront kernel, a single row: its words go straight to the stream, and the header with them; else null
    void* meta;
    u32 bit_set;
    MetaView mv;
    int cap;            // list capacity, multiple of 64, < 2048
    int region0_words;  // fine histogram, later block-ordered indices + stream image
    Ladder lad;         // fixed multi-level mode: no sums, no search
    int guard;          // 0: relative squared-error budget; 1: DS mismatch of Eq. "DS", greedy descent (beta = delta)
    float one_plus, one_minus;   // asymmetric thresholds of Sec. 3.1 (ASYM kernels): 1 + lambda, 1 - lambda in fp32
    int nbits, lg;      // bits of a block number; log2 of the lanes per boundary
    int lpb, cl, es, nc;    // ABQ: lanes per block, those of them with candidate bitwidths of their own, slices of a block, candidates of a lane
    u32* hint;          // [kHintSlots] cut keys of rows encoded earlier with this workspace (any contents are safe)
};

// how the lanes of the one-wavefront kernel are dealt to B2 blocks and nq bitwidths
inline void small_split_lanes(SmallArgs& a)
{
    const int B2 = a.M + a.Mn, ntg = B2 - 2;
    a.nbits = 0;
    while ((1 << a.nbits) < B2) ++a.nbits;
    a.lg = ntg > 32 ? 0 : ntg > 16 ? 1 : ntg > 8 ? 2 : ntg > 4 ? 3 : ntg > 2 ? 4 : 5;
    a.lpb = kWave / (B2 < kWave ? B2 : kWave);
    // Up to eight lanes with candidates of their own; blocks of sixteen lanes or more are sliced among such groups.  Where such blocks are long,
    // a lane takes up to four candidates instead, and there are as many more slices: a walk of fewer steps, but more lanes that add
    // to a sum.  Encode us, eight lanes / four candidates: fp32 [8192 x 4096] keep 0.4, one block a class, 328 / 304, one class alone,
    // DS guard, 448 / 386 (417 when every lane had a share of the block for all candidates); at 409 kept elements equal, at 204
    // up to 6 % longer, below 100 up to 20 %.
    a.cl = a.lpb < 8 ? a.lpb : a.lpb < 16 || a.k < 512 ? 8 : a.nq <= 4 ? 1 : a.nq <= 8 ? 2 : 4;
    a.es = a.lpb >= 16 ? a.lpb / a.cl : 1;
    a.nc = (a.nq + a.cl - 1) / a.cl;
}

// Threshold hints.  Rows of one tensor (tokens of one sequence, successive decode steps) have their
// top-K cut at nearly the same magnitude, so a wave first tries the cut key some earlier row left in
// the workspace, lowered by kHintDelta steps of the key's top 15 bits: if the number of keys at or
// above it lies in [k, k + kHintSlack] the list is built from it directly, and the row's largest key,
// the 2048-bin histogram and its scan are skipped.  The count decides, not the hint: a stale,
// foreign or garbage value only sends the row down the histogram path, and the output never depends on it.
constexpr int kHintSlots = 512;
constexpr u32 kHintDelta = 8;
constexpr u32 kHintSlack = 120;

constexpr int kCoarseBits = 11;
constexpr int kCoarseBins = 1 << kCoarseBits;
constexpr int kFineBins = 1024;
// Fine bins of the one-wavefront kernel: lists of up to 256 entries need fewer of them (fp32 [12608 x 768], 115 kept: kernel
// 37.7 us with 1024 bins, 36.9 with 512, 38.6 with 256, where the bins fill up).
__host__ __device__ constexpr int small_fine_bins(int maxs) { return maxs == 4 ? 512 : kFineBins; }

// LDS carve-up of one wave (word offsets); small_lds_words() on the host must match.
// The coarse histogram (2048 16-bit counters) overlays everything: nothing else is live before the
// compaction.  Region 0 is the fine histogram and fp32's list positions first; once the boundaries are known it holds
// the block-ordered indices, the stream image, the ABQ sums and the quantiser scales.  With the positions in a place of their
// own and room for sums that lanes keep in registers, long fp32 lists cost a CU one or two of its wavefronts: fp32 [2048 x 4096]
// keep 0.25, 16 + 16 blocks, all 16 bitwidths 88.4 us of encode at seven a CU, 56.7 at eleven.
struct SmallLds {
    u32* hist;      // [region0]   fine histogram and a word for the bin above it, Sp; later bo_idx, stream image, sums, invt
    u32* S;         // [cap + 4]   entries arranged by class and fine bin (bf16: comp; fp32: its key word), then zeros; later bo_val
    uint16_t* Sp;   // [cap + 4]   fp32 only, in region 0: the list position of the entry in S
    u32* thr;       // [B2]        block boundaries (class-extended comps; fp32: their key words), positive class first
    u32* thr_lo;    // [B2]        fp32 only: the low words
    u32* Lent;      // [cap]       MAXS = 0 only: list entries, ascending index (as `ent` in the kernel)
    uint16_t* Lidx; // [cap]       MAXS = 0 and fp32 only: index of the entry
    u32* qtab;      // [16]        allowed bitwidths
    u32* blk_start; // [B2 + 1]
    u32* vminb;     // [B2] key of the block's smallest / largest element
    u32* vmaxb;     // [B2]
    u32* run;       // [B2]        next free position of the block; later the chosen bitwidth index
};

// 64-bit sums of a block in LDS: the energy, and one for each bitwidth where several lanes add to it (blocks of sixteen lanes or more)
__host__ __device__ inline int small_block_sums(int B2, int nq) { return kWave / B2 >= 16 ? nq + 1 : 1; }

// words of region 0: the row's bit mask (at most 2 * 128 words) and list positions, then the fine histogram and fp32's Sp, then
// indices + stream image + sums + scales
__host__ __device__ inline int small_region0_words(int dt, int64_t k, u64 cap_words, int B2, int nq, int cap, int bins)
{
    const int64_t late = (((k + 1) / 2 + (int64_t)cap_words + 1) & ~(int64_t)1) + 2 * B2 * small_block_sums(B2, nq) + B2 * nq;
    const int64_t early = 2 * 128 + 4 + cap / 2, fine = bins + 4 + (dt == 0 ? (cap + 4) / 2 : 0);
    int64_t r0 = late > fine ? late : fine;
    r0 = r0 > early ? r0 : early;
    return (int)((r0 + 3) & ~(int64_t)3);
}

__host__ __device__ inline int small_lds_words(int dt, int cap, int region0, int B2, int maxs)
{
    int wds = region0 + (cap + 4);
    wds += B2 + (dt == 0 ? B2 : 0);
    wds += maxs ? 0 : cap + (dt == 0 ? cap / 2 : 0);
    wds += 16 + (B2 + 1) + B2 * 3;
    if (wds < kCoarseBins / 2) wds = kCoarseBins / 2;      // 16-bit counters of the coarse histogram
    return wds;
}

// The block-ordered values are read four at a time, by lanes that all walk as many as the longest block has: a lane whose block
// is shorter reads on behind it.  Where that can pass the end of the list, the group of four starts at `cap` at the latest:
// S has cap + 4 words, and a group that starts higher holds no entry.
__host__ __device__ inline u32 small_group_at(u32 at, int cap) { return at < (u32)cap ? at : (u32)cap; }

// A lane's part of its block for the sums: slice sl of `per` entries of the block of cnt entries at bs0; nothing: at place 0, where
// as many steps as any block has entries stay inside the list
struct AbqSlice { u32 q0, qn; };
__host__ __device__ inline AbqSlice small_abq_slice(u32 bs0, u32 cnt, u32 per, u32 sl, bool active)
{
    const u32 end = bs0 + cnt, q0 = bs0 + sl * per < end ? bs0 + sl * per : end, q1 = q0 + per < end ? q0 + per : end;
    const u32 qn = active ? q1 - q0 : 0u;
    return { qn ? q0 : 0u, qn };
}

__device__ inline SmallLds small_carve(u32* base, int dt, int cap, int region0, int B2, int maxs)
{
    SmallLds L;
    u32* p = base;
    L.hist = p;            p += region0;           // a multiple of four words
    L.S = p;               p += cap + 4;
    L.Sp = (uint16_t*)(base + small_fine_bins(maxs) + 4);
    L.thr = p;             p += B2;
    L.thr_lo = p;          p += dt == 0 ? B2 : 0;
    L.Lent = p;            p += maxs ? 0 : cap;
    L.Lidx = (uint16_t*)p; p += (dt == 0 && !maxs) ? cap / 2 : 0;
    L.qtab = p;            p += 16;
    L.blk_start = p;       p += B2 + 1;
    L.vminb = p;           p += B2;
    L.vmaxb = p;           p += B2;
    L.run = p;             p += B2;
    return L;
}

// LDS by byte offset: dynamic shared memory starts at offset 0 when the kernel has no static
// LDS (checked at run time), so an address computed as an integer needs no base register.
typedef __attribute__((address_space(3))) u32 lds_u32;
__device__ inline lds_u32* lds_at(u32 byte_off) { return (lds_u32*)(uintptr_t)byte_off; }
__device__ inline u32 lds_add(u32 byte_off, u32 v)
{
    return __hip_atomic_fetch_add(lds_at(byte_off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline void lds_inc(u32 byte_off, u32 v)
{
    __hip_atomic_fetch_add(lds_at(byte_off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// NQ > 0: the number of allowed bitwidths is known at compile time (loops over the
// candidate bitwidths unroll without predicates); NQ == 0: any number up to 16.
// MAXS > 0: the list has at most 64 * MAXS entries and lives in registers (fp32 with MAXS = 20: one of its two arrays in scratch, 96
// bytes a lane).
// ASYM: the asymmetric thresholds of Sec. 3.1 with lambda > 0.  The kept set is not a
// plain top-K then: after the first selection has given tau, the strict set is counted, a second
// selection over a subset of the row (the fill candidates, or the strict set when it is too large)
// gives the last key taken, and the list is built from that rule; the equal keys at the end are cut
// in index order.  Both selections need the exact key of their rank, i.e. one key per histogram bin:
// ranks that lie below the 2048-key window are found bit by bit over the row in registers.
// Wavefronts per SIMD the register allocator must leave room for.  The variants that hold the row in at most
// 32 registers come out at 65 to 89 VGPRs and are asked for five wavefronts (96).  fp32 rows of more than 2048 elements (64
// registers for the row, 138 to 154 in all) are asked for three (168); bf16 rows of more than 4096 come out at 143 to 153.  No
// variant spills.  (With the exact cut found bit by bit over the row, whose masked words were then held from bit to bit, fp32 rows
// of more than 2048 elements spilled 28 to 30 registers: [2048 x 4096] keep 0.10 encode 26.7 us, now 24.0.)
constexpr int small_min_waves(int dt, int epl, int nq, int maxs, bool asym)
{
    const int row_regs = dt == 0 ? epl : epl / 2;
    return row_regs <= 32 ? 5 : (dt == 0 && row_regs == 64) ? 3 : 1;
}

template <int DT, int EPL, int NQ, int MAXS, bool ASYM = false>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(small_min_waves(DT, EPL, NQ, MAXS, ASYM)))) void enc_small_kernel(SmallArgs a)
{
    typedef Elem<DT> E;
    constexpr int kRegThr = 14;                                              // boundaries held in registers
    constexpr int QN = NQ ? NQ : kMaxQ;
    constexpr int EPC = DT == 0 ? 4 : 8;            // elements per 16-byte chunk
    constexpr int NCH = EPL / EPC;                  // chunks per lane
    constexpr int FB = small_fine_bins(MAXS);
    extern __shared__ u32 smem[];

    const u32 lane = lane_id();
    const int64_t r = xcd_row((int64_t)blockIdx.x, a.R);        // neighbouring rows stay on one XCD
    if (r >= a.R) return;
    const int M = a.M, Mn = a.Mn, w = a.w, B2 = a.M + a.Mn, nq = NQ ? NQ : a.nq, cap = a.cap;
    const int k = (int)a.k;
    SmallLds L = small_carve(smem, DT, cap, a.region0_words, B2, MAXS);
    if (__builtin_amdgcn_groupstaticsize() != 0u) __builtin_trap();      // integer LDS addresses assume offset 0: the kernel has no static LDS
    // ---- list entry accessors ---------------------------------------------------------------
    // Entry p of the list (ascending index): the class as the top bit (set for the positive one), the magnitude key below it
    // and, for bf16, the inverted index in the low half: the whole class-extended comp.  fp32 entries have ~p as their low
    // word where equal keys must be told apart (list positions rise with the index).
    constexpr u32 kPos = 0x80000000u, kMag = 0x7FFFFFFFu;
    constexpr int SLN = MAXS ? MAXS : 32;          // slots of 64 entries (cap < 2048)
    u32 ent[MAXS ? MAXS : 1], eix[(MAXS && DT == 0) ? MAXS : 1];
    auto ent_word = [&](int s) -> u32 { return MAXS ? ent[MAXS ? s : 0] : L.Lent[s * kWave + (int)lane]; };
    auto ent_index = [&](int s) -> u32 {
        if (DT == 1) return ~ent_word(s) & 0xFFFFu;
        return MAXS ? eix[(MAXS && DT == 0) ? s : 0] : (u32)L.Lidx[s * kWave + (int)lane];
    };
    auto word_key = [&](u32 e) -> u32 { return DT == 0 ? e & kMag : (e >> 16) & 0x7FFFu; };

    // ---- 1. load the row, coarse histogram ------------------------------------------
    const RowChunks<DT> row(a.x, r, a.N);           // element i of the row is element head + i of its chunks
    const int head = row.head, Nh = row.Nh;
    uint4 v[NCH];
    row.template load<NCH, kWave>(v, (int)lane);
    auto word_of = [&](int c, int d) -> u32 { return d == 0 ? v[c].x : d == 1 ? v[c].y : d == 2 ? v[c].z : v[c].w; };
    constexpr bool kHint = !ASYM && MAXS > 0;       // (the list must be in registers: its largest key is taken from there)
    const u32 hslot = (u32)blockIdx.x & (u32)(kHintSlots - 1);
    u32 hint_key = 0;
    if (kHint) hint_key = a.hint[hslot] & (DT == 0 ? 0x7FFFFFFFu : 0x7FFFu);

    // Largest magnitude key of the row: the histogram window hangs from it.
    u32 kmax = 0;
    auto row_kmax = [&]() {
        u32 mx = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const u32 wd = word_of(c, d);
                if (DT == 0) mx = max(mx, wd & 0x7FFFFFFFu);
                else mx = pk_max_u16(mx, wd & 0x7FFF7FFFu);
            }
        }
        if (DT == 1) mx = max(mx & 0xFFFFu, mx >> 16);
        kmax = wave_max_dpp(mx);
    };

    // Coarse histogram over a window of 2048 bins that hangs from `wtop`: bin = (wtop - key) >> S,
    // bin 0 on top.  First pass: S = 0 (bf16: one key per bin) or 16 (fp32: the same 128 bins per
    // octave), i.e. 16 octaves below the largest key, everything further down in the last bin.
    // Values of one row crowd into a few octaves, so bins this fine keep the lanes of an LDS
    // atomic on different addresses, and the bin of rank k-1 holds little beyond the kept set.
    // If rank k-1 lies below the window, a second pass with 16 times wider bins hangs from the
    // window's lower end and reaches key 0.
    constexpr int S1 = DT == 0 ? 16 : 0;
    u32 wtop = 0, above = 0;                        // above = number of keys > wtop
    int S = S1;
    u32 B1 = 0, c_gt = 0, cnt1 = 0;
    bool found = false;
    u32 rank_t = k > 0 ? (u32)(k - 1) : 0u;         // the rank the pass looks for (among the keys the functor lets through)
    auto all_keys = [](u32 wd) -> u32 { return wd & (DT == 0 ? 0x7FFFFFFFu : 0x7FFF7FFFu); };   // fp32: one key; bf16: a pair
    // skip0: keys that the functor turned into 0 are not counted at all (they would all meet on one
    // LDS address); the pass then reports found = false when the rank lies beyond the counted keys
    // windowed (fp32 narrowing passes): keys above the window or below its 2048 bins are not counted at all
    // (they would all meet on the first or the last bin's LDS address); `above` then only enters the rank
    auto hist_pass = [&](auto shift, auto key_pair, auto skip0, auto windowed) __attribute__((always_inline)) {
        constexpr int SH = decltype(shift)::value;
        constexpr bool kSkip0 = decltype(skip0)::value;
        constexpr bool kWindowed = decltype(windowed)::value;
        constexpr int SHB = SH >= 2 ? SH - 2 : 0;      // fp32: shift that leaves the bin number times 4
        // two 16-bit counters per word (a row has fewer than 2^16 elements): bin b is half b & 1 of word b >> 1
        auto bin_inc = [](u32 b4) { lds_inc((b4 >> 1) & ~3u, 1u << ((b4 & 4u) << 2)); };
        {
            uint4* h4 = (uint4*)smem;
#pragma unroll
            for (int i = 0; i < kCoarseBins / 8 / kWave; ++i) h4[i * kWave + lane] = make_uint4(0, 0, 0, 0);
        }
        wave_sync();
        const u32 wt2 = wtop * 0x10001u;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if ((c * kWave + (int)lane) * EPC < Nh) {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32 wd = word_of(c, d);
                    if (DT == 0) {
                        const u32 key = key_pair(wd);
                        const u32 df = wtop > key ? wtop - key : 0u;
                        const u32 b4 = SH >= 2 ? min((df >> SHB) & ~3u, (u32)(4 * kCoarseBins - 4))
                                               : (min(df >> SH, (u32)(kCoarseBins - 1)) << 2);
                        if (kWindowed) {
                            if ((!kSkip0 || key) && key <= wtop && (df >> SH) < (u32)kCoarseBins) bin_inc(b4);
                        } else if (!kSkip0 || key) {
                            bin_inc(b4);
                        }
                    } else {
                        const u32 kp = key_pair(wd);
                        u32 b = pk_sub_sat_u16(wt2, kp);
                        if (SH) b = pk_shr_u16(b, SH);
                        b = pk_shl_u16(pk_min_u16(b, (u32)(kCoarseBins - 1) * 0x10001u), 2);
                        if (!kSkip0 || (kp & 0xFFFFu)) bin_inc(b & 0xFFFFu);
                        if (!kSkip0 || (kp >> 16)) bin_inc(b >> 16);
                    }
                }
            }
        }
        wave_sync();
        if (!kWindowed && above && lane == 0) smem[0] -= above;   // keys above the window were counted in bin 0
        wave_sync();
        // Scan from the top in two levels: every lane sums 32 bins, the lane that holds the rank
        // is then opened bin by bin.
        constexpr int BPL = kCoarseBins / kWave;       // 32 bins = 16 words
        const uint4* h4 = (const uint4*)(smem + (int)lane * (BPL / 2));
        u32 both = 0;                                  // the halves add up separately: no sum reaches 2^16
#pragma unroll
        for (int j = 0; j < BPL / 8; ++j) {
            const uint4 t = h4[j];
            both += (t.x + t.y) + (t.z + t.w);
        }
        const u32 local = (both & 0xFFFFu) + (both >> 16);
        const u32 incl = wave_scan_dpp(local), excl = incl - local;
        const u32 rem = rank_t - above;
        const u64 m_src = __ballot(local > 0 && excl <= rem && rem < incl);
        const int src = m_src ? (int)__builtin_ctzll(m_src) : 0;
        const u32 ex_src = bcast(excl, src);
        const u32 w2 = lane < (u32)BPL ? smem[src * (BPL / 2) + (int)(lane >> 1)] : 0u;
        const u32 c2 = (lane & 1u) ? w2 >> 16 : w2 & 0xFFFFu;
        const u32 inc2 = wave_scan_dpp(c2);            // lanes 0..31: running count inside lane `src`
        const u64 m_b1 = __ballot(lane < (u32)BPL && ex_src + inc2 > rem);
        found = m_src && m_b1;
        if (found) {
            const int j1 = (int)__builtin_ctzll(m_b1);
            B1 = (u32)(src * BPL + j1);
            cnt1 = bcast(c2, j1);
            c_gt = ex_src + bcast(inc2, j1) - cnt1;
        }
        wave_sync();
    };
    // Which elements go to the list: a bit mask of the row.  Every lane flags the elements of its own chunks (8 or 4 bits a
    // chunk: the flags are the words' sign bits, gathered by one byte permutation and one dot product per four of them), the
    // chunks' bits meet in LDS, and every lane takes the bits of EPL consecutive elements: one prefix sum over the lanes then
    // gives the list positions in index order.
    constexpr int NM = EPL >= 32 ? EPL / 32 : 1;    // words of a lane's mask
    uint16_t* plist = (MAXS || DT == 1) ? (uint16_t*)(smem + 2 * EPL + 4) : L.Lidx;      // row positions of the list's entries
    u32 t_lo = 1u, nL = 0, mk[NM], pos0 = 0;        // pos0: entries of the lanes below
    // flag(word): bf16: bits 15 and 31 set where the word's elements are taken; fp32: bit 31
    auto row_mask = [&](auto flag) __attribute__((always_inline)) {
        unsigned char* mb = (unsigned char*)smem;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            u32 f[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) f[d] = flag(word_of(c, d));
            // selectors 8 to 11 of the byte permutation: the sign of a 16-bit half as a byte of ones or zeros; 12: zero
            const u32 p0 = __builtin_amdgcn_perm(f[1], f[0], DT == 0 ? 0x0C0C0B09u : 0x0B0A0908u);
            const u32 p1 = __builtin_amdgcn_perm(f[3], f[2], DT == 0 ? 0x0B090C0Cu : 0x0B0A0908u);
            // -1 times weights -1, -2, -4, ...
            int m = __builtin_amdgcn_sdot4((int)p0, DT == 0 ? 0x0000FEFF : (int)0xF8FCFEFFu, 0, false);
            m = __builtin_amdgcn_sdot4((int)p1, DT == 0 ? (int)0xF8FC0000u : (int)0x80C0E0F0u, m, false);
            if (DT == 0) {                          // two lanes share a byte
                const u32 up = (u32)__builtin_amdgcn_update_dpp(0, m, 0xF5, 0xf, 0xf, true);      // quad_perm 1 1 3 3
                if (!(lane & 1u)) mb[(c * kWave + (int)lane) >> 1] = (unsigned char)((u32)m | (up << 4));
            } else {
                mb[c * kWave + (int)lane] = (unsigned char)m;
            }
        }
        wave_sync();
        if (EPL >= 32) {
#pragma unroll
            for (int i = 0; i < NM; ++i) mk[i] = smem[(int)lane * NM + i];
        } else {                                    // (the word after the mask is readable; its bits are masked off)
            const u32 at = lane * (u32)EPL;
            mk[0] = __builtin_amdgcn_alignbit(smem[(at >> 5) + 1], smem[at >> 5], at & 31u) & ((1u << (EPL & 31)) - 1u);
        }
        wave_sync();
    };
    auto scan_mask = [&]() __attribute__((always_inline)) {
        u32 n1 = 0;
#pragma unroll
        for (int i = 0; i < NM; ++i) n1 += (u32)__popc(mk[i]);
        const u32 incl = wave_scan_dpp(n1);
        nL = bcast(incl, kWave - 1);
        pos0 = incl - n1;
    };
    // sign bits: the word's keys that are at or above t <=> the sign bit of key + (2^31 - t), or of both halves with 2^15
    auto key_flag = [&](u32 wd, u32 t) -> u32 {
        return (wd & (DT == 0 ? 0x7FFFFFFFu : 0x7FFF7FFFu)) + (DT == 0 ? 0x80000000u - t : (0x8000u - t) * 0x10001u);
    };
    auto mask_plain = [&]() __attribute__((always_inline)) {                       // every key at or above t_lo
        row_mask([&](u32 wd) -> u32 { return key_flag(wd, t_lo); });
        scan_mask();
    };
    // of the elements flagged by `ties`, all in the mask, only the first `need` stay there
    auto keep_first = [&](u32 need, auto ties) __attribute__((always_inline)) {
        u32 all[NM];
#pragma unroll
        for (int i = 0; i < NM; ++i) all[i] = mk[i];
        row_mask(ties);
        scan_mask();
        u32 left = need > pos0 ? need - pos0 : 0u;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            u32 e = mk[i], stay = 0;
            for (; e && left; --left) { stay |= e & (0u - e); e &= e - 1u; }
            mk[i] = (all[i] & ~mk[i]) | stay;
        }
    };
    // The exact key of rank rank_t among the keys a functor lets through, by histogram passes over narrowing windows, each of
    // them inside the bin that the one before it found: on success wtop - B1 is the key, above + c_gt the number of counted
    // keys above it, cnt1 its multiplicity.  single_keys() goes on from a pass whose bins have 2^S1 keys, or 2^(S1 + 4) (wide: after the
    // values spread over more than 16 octaves): fp32 bins of 2^5 keys (2^9), then single keys; bf16 single keys from
    // wide bins, where a pass without them has found the key already.
    auto narrow = [&](int sh_done) { above += c_gt; wtop -= B1 << sh_done; };
    // A bin of up to 64 members, as nearly all are, is resolved at once: its members meet in LDS and every lane counts those above its own
    // (encode of fp32 [12608 x 768], lambda = 0.1: 61.8 us with four more histogram passes, now 54.7).
    auto few_members = [&](int sh, auto key_fn, auto skip0) __attribute__((always_inline)) {
        constexpr bool kSkip0 = decltype(skip0)::value;
        narrow(sh);
        const u32 rem = rank_t - above, n = cnt1;
        u32 at = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c * kWave * EPC >= Nh) break;        // uniform (the row's unused chunks: [1 x 2060], 32 + 32 blocks 42.8 us with them, 38.9 without)
            const bool on = (c * kWave + (int)lane) * EPC < Nh;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const u32 key = key_fn(word_of(c, d));
                const bool in = on && (!kSkip0 || key) && key <= wtop && ((wtop - key) >> sh) == 0u;
                const u64 m = __ballot(in);
                const u32 pos = at + mask_rank(m);
                if (in && pos < (u32)kWave) smem[pos] = key;
                at += (u32)__popcll(m);
            }
        }
        wave_sync();
        const u32 me = lane < n ? smem[lane] : 0u;
        u32 gt = 0, ge = 0;
        for (u32 j = 0; j < n; ++j) {
            const u32 other = bcast(me, (int)j);
            gt += other > me ? 1u : 0u;
            ge += other >= me ? 1u : 0u;
        }
        const u64 hit = __ballot(lane < n && gt <= rem && rem < ge);
        const int src = hit ? (int)__builtin_ctzll(hit) : 0;
        wtop = bcast(me, src); B1 = 0;
        c_gt = bcast(gt, src); cnt1 = bcast(ge, src) - c_gt;
        wave_sync();
    };
    auto single_keys = [&](bool wide, auto key_fn, auto skip0) __attribute__((always_inline)) {
        if constexpr (DT == 0) {
            if (cnt1 <= (u32)kWave) {                // uniform
                few_members(wide ? 20 : 16, key_fn, skip0);
                return;
            }
        }
        if (DT == 0) {
            if (wide) {
                narrow(20);
                hist_pass(std::integral_constant<int, 9>(), key_fn, skip0, std::true_type());
                if (!found) return;
                narrow(9);
            } else {
                narrow(16);
                hist_pass(std::integral_constant<int, 5>(), key_fn, skip0, std::true_type());
                if (!found) return;
                narrow(5);
            }
            hist_pass(std::integral_constant<int, 0>(), key_fn, skip0, std::true_type());
        } else if (wide) {
            narrow(4);
            hist_pass(std::integral_constant<int, 0>(), key_fn, skip0, std::false_type());
        }
    };
    // from wtop with above = 0
    auto exact_select = [&](auto key_fn, auto skip0) __attribute__((always_inline)) {
        hist_pass(std::integral_constant<int, S1>(), key_fn, skip0, std::false_type());
        const bool wide = found && B1 == (u32)(kCoarseBins - 1) && (wtop >> S1) > (u32)(kCoarseBins - 1);
        if (wide) {
            narrow(S1);
            hist_pass(std::integral_constant<int, S1 + 4>(), key_fn, skip0, std::integral_constant<bool, DT == 0>());
        }
        if (found) single_keys(wide, key_fn, skip0);
    };
    // the hinted bound: accepted when it keeps at least k keys and not many more
    bool hinted = false;
    if (kHint && k > 0) {
        const u32 dlt = kHintDelta << (DT == 0 ? 16 : 0);
        t_lo = hint_key > dlt ? hint_key - dlt : 1u;
        mask_plain();
        hinted = nL >= (u32)k && nL <= (u32)k + kHintSlack && (int)nL <= cap;
    }
    if (!hinted && ASYM && DT == 0) row_kmax();      // (its selections run further down)
    if (!hinted && !(ASYM && DT == 0)) {
        row_kmax();
        wtop = kmax;
        hist_pass(std::integral_constant<int, S1>(), all_keys, std::false_type(), std::false_type());
        if (found && B1 == (u32)(kCoarseBins - 1) && (wtop >> S1) > (u32)(kCoarseBins - 1)) {
            narrow(S1);
            S = S1 + 4;
            hist_pass(std::integral_constant<int, S1 + 4>(), all_keys, std::false_type(), std::false_type());
        }
    }

    // ---- asymmetric thresholds: strict set, second selection ------------------------------------
    // Everything per pair of keys (packed 16-bit lanes): st = 1 where the element is strictly
    // retained, inF = 1 where it is a fill candidate (not strict, at or below tau).
    constexpr u32 kOne2 = 0x00010001u;
    u32 tau2 = 0, tp2 = 0, dthr2 = 0, t2_2 = 0;     // tau, tau+ and (tau- minus tau+), last key taken: duplicated in both halves
    u32 t2_key = 0, need_ties = 0, cnt_ties = 0, tn_key = 0;
    bool trim = false;
    auto gt01 = [&](u32 a2, u32 b2) -> u32 { return pk_min_u16(pk_sub_sat_u16(a2, b2), kOne2); };   // a > b, per half
    // (each use starts from an opaque copy of the word: the flags are recomputed where they are needed
    //  instead of being held in registers for the whole row from one phase to the next)
    auto strict01 = [&](u32 wd) -> u32 {
        asm volatile("" : "+v"(wd));
        const u32 neg01 = (wd >> 15) & kOne2;
        return gt01(wd & 0x7FFF7FFFu, pk_add_u16(tp2, pk_mul_lo_u16(neg01, dthr2)));
    };
    auto fill01 = [&](u32 wd, u32 st) -> u32 {
        asm volatile("" : "+v"(wd));
        return (st ^ kOne2) & (gt01(wd & 0x7FFF7FFFu, tau2) ^ kOne2);
    };
    u32 tp_key32 = 0, tau_key32 = 0;
    auto strict32 = [&](u32 wd) -> bool { return (wd & 0x7FFFFFFFu) > ((wd >> 31) ? tn_key : tp_key32); };
    auto fill32 = [&](u32 wd) -> bool { return !strict32(wd) && (wd & 0x7FFFFFFFu) <= tau_key32; };
    if (ASYM && DT == 0 && k > 0) {
        // tau = the k-th largest magnitude, exactly (the first pass above has run on the same window: redo it
        // as the first level of the exact selection)
        wtop = kmax; above = 0; S = 0;
        exact_select(all_keys, std::false_type());     // (finds it: every key is counted)
        tau_key32 = wtop - B1;
        const float tau = __uint_as_float(tau_key32);
        tp_key32 = __float_as_uint(__fmul_rn(a.one_plus, tau));
        tn_key = __float_as_uint(__fmul_rn(a.one_minus, tau));
        u32 accS = 0, accF = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if ((c * kWave + (int)lane) * EPC < Nh) {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32 wd = word_of(c, d);
                    accS += strict32(wd) ? 1u : 0u;
                    accF += fill32(wd) ? 1u : 0u;
                }
            }
        }
        const u32 tot = bcast(wave_scan_dpp(accS | (accF << 16)), kWave - 1);
        const u32 c_strict = tot & 0xFFFFu, f_fill = tot >> 16;
        trim = c_strict >= (u32)k;
        const u32 D = trim ? 0u : (u32)k - c_strict;
        if (trim || f_fill > D) {
            rank_t = trim ? (u32)(k - 1) : D - 1u;
            wtop = trim ? kmax : tau_key32;
            above = 0;
            if (trim) exact_select([&](u32 wd) -> u32 { return strict32(wd) ? wd & 0x7FFFFFFFu : 0u; }, std::true_type());
            else exact_select([&](u32 wd) -> u32 { return fill32(wd) ? wd & 0x7FFFFFFFu : 0u; }, std::true_type());
            if (found) {
                t2_key = wtop - B1;
                need_ties = rank_t + 1u - (above + c_gt);
                cnt_ties = cnt1;
            }                                            // else: the rank lies among zeros, every non-zero candidate is taken
        }
        if (t2_key == 0) { t2_key = 1; need_ties = 0; cnt_ties = 0; }
        S = 0; B1 = 0;
    }
    if (ASYM && DT == 1 && k > 0) {
        // (the bins of a second pass hold several keys)
        if (S != S1) single_keys(true, all_keys, std::false_type());
        const u32 tau_key = wtop - B1;
        const float tau = __uint_as_float(tau_key << 16);
        const u32 tp_key = __float_as_uint(__fmul_rn(a.one_plus, tau)) >> 16;    // (key << 16) > T  <=>  key > (T >> 16)
        tn_key = __float_as_uint(__fmul_rn(a.one_minus, tau)) >> 16;
        tau2 = tau_key * 0x10001u; tp2 = tp_key * 0x10001u; dthr2 = ((tn_key - tp_key) & 0xFFFFu) * 0x10001u;
        u32 accS = 0, accF = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if ((c * kWave + (int)lane) * EPC < Nh) {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32 wd = word_of(c, d);
                    const u32 st = strict01(wd);
                    accS = pk_add_u16(accS, st);
                    accF = pk_add_u16(accF, fill01(wd, st));
                }
            }
        }
        const u32 both = ((accS & 0xFFFFu) + (accS >> 16)) | (((accF & 0xFFFFu) + (accF >> 16)) << 16);
        const u32 tot = bcast(wave_scan_dpp(both), kWave - 1);
        const u32 c_strict = tot & 0xFFFFu, f_fill = tot >> 16;
        trim = c_strict >= (u32)k;
        const u32 D = trim ? 0u : (u32)k - c_strict;
        if (trim || f_fill > D) {
            // rank k-1 of the strict set, or rank D-1 of the fill candidates: the other keys count as 0
            rank_t = trim ? (u32)(k - 1) : D - 1u;
            wtop = trim ? kmax : tau_key;
            above = 0;
            if (trim) exact_select([&](u32 wd) -> u32 { return pk_mul_lo_u16(wd & 0x7FFF7FFFu, strict01(wd)); }, std::true_type());
            else exact_select([&](u32 wd) -> u32 { return pk_mul_lo_u16(wd & 0x7FFF7FFFu, fill01(wd, strict01(wd))); }, std::true_type());
            if (found) {
                t2_key = wtop - B1;
                need_ties = rank_t + 1u - (above + c_gt);
                cnt_ties = cnt1;
            }                                            // else: the rank lies among zeros, every non-zero candidate is taken
        }
        if (t2_key == 0) { t2_key = 1; need_ties = 0; cnt_ties = 0; }     // the rank falls on zeros (never sent) or every candidate is taken
        t2_2 = t2_key * 0x10001u;
    }

    // the list takes every non-zero key from bin B1 up (a bin that reaches key 0 also counts the
    // zeros, which never enter the list: its length is known after the counting pass below)
    if (!hinted) {
        const long long lowk = (long long)wtop - ((long long)(B1 + 1u) << S) + 1;
        t_lo = lowk > 1 ? (u32)lowk : 1u;                        // smallest non-zero key of bin B1
        if (ASYM && k > 0) t_lo = trim ? t2_key : min(t2_key, tn_key + 1u);   // smallest key the list can hold
    }

    // ---- 2. ordered compaction into L -------------------------------------------------
    // The list's row positions first (a lane writes its set bits one after the other), then its values, fetched again from
    // the row: consecutive entries lie close together, so these loads touch a few cache lines each, and they hit the L2.
    // Storing from registers instead costs 12 instructions per pair of elements, flagged or not.  Up to the list in registers a
    // row of 4096 bf16 elements took 757 vector instructions and takes 352 (kernel, 16384 rows: 95.1 -> 87.2 us); fp32
    // [12608 x 768]: 281 and 213 (44.2 -> 43.6 us).
    if (k == 0) nL = 0;
    if (k > 0) {
        if (ASYM) {
            // taken: the strict set or its largest part, and the fill candidates down to the last key taken; of several
            // elements with that key the first need_ties stay
            auto taken = [&](u32 wd, bool ties) -> u32 {         // ties: only the candidates with the last key taken
                if (DT == 1) {
                    const u32 st = strict01(wd);
                    u32 wk = wd;
                    asm volatile("" : "+v"(wk));
                    const u32 ge = gt01(t2_2, wk & 0x7FFF7FFFu) ^ kOne2;              // key >= last key taken
                    if (ties) return ((trim ? st : fill01(wd, st)) & ge & (gt01(wk & 0x7FFF7FFFu, t2_2) ^ kOne2)) << 15;
                    return (trim ? (st & ge) : (st | (fill01(wd, st) & ge))) << 15;
                }
                const u32 key = wd & 0x7FFFFFFFu;
                const bool st = strict32(wd), ge = key >= t2_key;
                if (ties) return (trim ? st : fill32(wd)) && key == t2_key ? 0x80000000u : 0u;
                return (trim ? (st && ge) : (st || (fill32(wd) && ge))) ? 0x80000000u : 0u;
            };
            row_mask([&](u32 wd) -> u32 { return taken(wd, false); });
            if (need_ties < cnt_ties) keep_first(need_ties, [&](u32 wd) -> u32 { return taken(wd, true); });     // uniform
            scan_mask();
        } else {
            if (!hinted) mask_plain();
            if (__builtin_expect((int)nL > cap, 0)) {       // uniform, rare: the exact cut
                single_keys(S != S1, all_keys, std::false_type());
                t_lo = wtop - B1;
                mask_plain();
                if (nL > (u32)k)
                    keep_first((u32)k - (above + c_gt), [&](u32 wd) -> u32 { return key_flag(wd, t_lo) & ~key_flag(wd, t_lo + 1u); });
                scan_mask();
            }
        }
        const u32 pl_off = (u32)((u32*)plist - smem) * 4u;
        typedef __attribute__((address_space(3))) uint16_t lds_u16;
        u32 wa = pl_off + 2u * pos0;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const u32 i0 = lane * (u32)EPL + 32u * (u32)i - (u32)head;
            u32 m = mk[i];
            while (m) {
                *(lds_u16*)(uintptr_t)wa = (uint16_t)(i0 + (u32)__builtin_ctz(m));
                wa += 2u;
                m &= m - 1u;
            }
        }
        wave_sync();
    }
    const typename E::raw_t* __restrict__ xr = (const typename E::raw_t*)a.x + (size_t)r * (size_t)a.N;
    if (MAXS) {
        // the list moves straight into registers, four slots at a time with all their loads in flight
        u32 ix[MAXS ? MAXS : 1];
#pragma unroll
        for (int s = 0; s < SLN; ++s) { ix[MAXS ? s : 0] = 0; ent[MAXS ? s : 0] = 0; }
#pragma unroll
        for (int g = 0; g < SLN; g += 4) {
            if ((u32)(g * kWave) >= nL) continue;   // uniform
#pragma unroll
            for (int s = g; s < g + 4 && s < SLN; ++s) ix[MAXS ? s : 0] = (u32)plist[s * kWave + lane];
#pragma unroll
            for (int s = g; s < g + 4 && s < SLN; ++s)      // (element 0 exists; its copies behind the list's end are not looked at)
                ent[MAXS ? s : 0] = (u32)xr[ix[MAXS ? s : 0] = (int)lane < (int)nL - s * kWave ? ix[MAXS ? s : 0] : 0u];
        }
#pragma unroll
        for (int s = 0; s < SLN; ++s) {
            asm volatile("" : "+v"(ent[MAXS ? s : 0]));     // (the shift stays behind all of the loads)
            if (DT == 1) ent[MAXS ? s : 0] = ((ent[MAXS ? s : 0] << 16) | ix[MAXS ? s : 0]) ^ (kPos | 0xFFFFu);
            else { ent[MAXS ? s : 0] ^= kPos; eix[(MAXS && DT == 0) ? s : 0] = ix[MAXS ? s : 0]; }
        }
        wave_sync();
    } else {
        for (u32 p = lane; p < nL; p += kWave) {    // fp32: the row positions stay where they are
            const u32 i = plist[p], raw = (u32)xr[i];
            L.Lent[p] = DT == 1 ? ((raw << 16) | i) ^ (kPos | 0xFFFFu) : raw ^ kPos;
        }
        wave_sync();
    }
    if (MAXS) {
        if (kHint && hinted) {                        // the row's largest key is the list's largest
            u32 mx = 0;
#pragma unroll
            for (int s = 0; s < SLN; ++s) mx = max(mx, ent[MAXS ? s : 0] & kMag);
            kmax = wave_max_dpp(mx);
            if (DT == 1) kmax >>= 16;
        }
    }
    {
        uint4* h4 = (uint4*)L.hist;
#pragma unroll
        for (int i = 0; i < FB / 4 / kWave; ++i) h4[i * kWave + lane] = make_uint4(0, 0, 0, 0);
    }
    if (lane == 0) {
#pragma unroll
        for (int t = 0; t < QN; ++t)
            if (NQ || t < nq) L.qtab[t] = (u32)a.qlist[t];
    }
    wave_sync();

    // ---- 3. fine bins ---------------------------------------------------------------------
    // FB bins, linear in (key - t_lo) >> sh; sh from the row's largest key.  A bin's word counts the positive class
    // in its high half and the negative one in its low half; after the scan the halves are the places in S where the bin's
    // members of the class go, and adding an entry moves them on: in the end they are the ends of the bin's places, which
    // begin where those of the bin above end.
    const int nslots = (int)((nL + kWave - 1) / kWave);
    const u32 range = kmax > t_lo ? kmax - t_lo : 0u;
    const int sh = range < (u32)FB ? 0 : (32 - __clz((int)range)) - (FB == 512 ? 9 : 10);
    auto in_list = [&](int s) -> bool { return (int)lane < (int)nL - s * kWave; };      // this lane has an entry in slot s
    auto key_bin = [&](u32 key) -> u32 { return (key - t_lo) >> sh; };
    // Place of a bin's word.  A lane scans 16 consecutive bins of 1024 in four 16-byte pieces; lanes four apart would meet on
    // the same banks, so the pieces of every fourth lane are swapped (bf16 [16384 x 4096] kernel 68.3 -> 67.6 us).
    auto bin_word = [](u32 b) -> u32 { return b ^ ((b >> 4) & (FB == 512 ? 4u : 12u)); };
    auto half_of = [](u32 e) -> u32 { return (e >> 27) & 16u; };                     // shift of the class's half
    u32 b4[MAXS ? MAXS : 1];                        // byte offset of the entry's bin
#pragma unroll(MAXS ? MAXS : 1)
    for (int s = 0; s < SLN; ++s) {
        if (s >= nslots) break;
        if (in_list(s)) {
            const u32 e = ent_word(s), at = bin_word(key_bin(word_key(e))) << 2;
            if (MAXS) b4[MAXS ? s : 0] = at;
            lds_inc(at, 1u << half_of(e));
        }
    }
    wave_sync();
    u32 nLp, n_pos, n_neg;                          // positive entries of the list; class sizes of the kept set
    int cut_lane = 0;
    constexpr int BPL = FB / kWave;          // bins per lane, from the top
    {
        const int hi = FB - (int)lane * BPL;
        u32 cs[BPL];
        uint4* h4 = (uint4*)(L.hist + hi - BPL);
        auto piece = [&](int j) -> int { return j ^ (((hi - BPL) >> 6) & (FB == 512 ? 1 : 3)); };
#pragma unroll
        for (int j = 0; j < BPL / 4; ++j) {
            const uint4 t = h4[piece(BPL / 4 - 1 - j)];
            cs[4 * j + 0] = t.w; cs[4 * j + 1] = t.z; cs[4 * j + 2] = t.y; cs[4 * j + 3] = t.x;
        }
        u32 local = 0;                              // (the list has fewer than 2048 entries: the halves never carry)
#pragma unroll
        for (int j = 0; j < BPL; ++j) local += cs[j];
        const u32 incl = wave_scan_dpp(local);
        const u32 tot = bcast(incl, kWave - 1);
        nLp = tot >> 16;
        n_pos = nLp; n_neg = tot & 0xFFFFu;
        // the lane whose bins hold overall rank k-1 (meaningful when nL > k)
        const u32 ov_in = (incl >> 16) + (incl & 0xFFFFu), ov_ex = ov_in - (local >> 16) - (local & 0xFFFFu);
        const u64 mc = __ballot(k > 0 && ov_ex <= (u32)(k - 1) && (u32)(k - 1) < ov_in);
        cut_lane = mc ? (int)__builtin_ctzll(mc) : 0;
        u32 acc = incl - local + nLp;               // the negative class follows the positive one
        u32 o[BPL];
#pragma unroll
        for (int j = 0; j < BPL; ++j) {
            o[j] = acc;
            acc += cs[j];
        }
#pragma unroll
        for (int j = 0; j < BPL / 4; ++j) h4[piece(BPL / 4 - 1 - j)] = make_uint4(o[4 * j + 3], o[4 * j + 2], o[4 * j + 1], o[4 * j + 0]);
        if (lane == 0) L.hist[FB] = nLp;     // the bin above all others ends where the classes begin
        if (lane < 4u) L.S[nL + lane] = 0;          // (read behind the last entry by the loops that take four at a time)
    }
    wave_sync();
#pragma unroll(MAXS ? MAXS : 1)
    for (int s = 0; s < SLN; ++s) {
        if (s >= nslots) break;
        if (in_list(s)) {
            const u32 e = ent_word(s), hf = half_of(e);
            const u32 old = lds_add(MAXS ? b4[MAXS ? s : 0] : bin_word(key_bin(word_key(e))) << 2, 1u << hf);
            const u32 at = __builtin_amdgcn_ubfe(old, hf, 16u);
            L.S[at] = e;
            if (DT == 0) L.Sp[at] = (uint16_t)(s * kWave + (int)lane);
        }
    }
    wave_sync();
    auto low_of = [&](u32 at) -> u32 { return DT == 0 ? ~(u32)L.Sp[at] : 0u; };      // fp32: low word of the comp at place `at`
    auto beats = [&](u32 x, u32 xl, u32 y, u32 yl) -> bool { return DT == 0 ? x > y || (x == y && xl > yl) : x > y; };
    // The member of rank `rem` of the c0 places from a0 and the c1 places from a1, all of one bin, by the whole wavefront: for bins
    // of many members (equal or nearly equal values), where comparing all pairs would take c^2 steps.  Its key bit by bit, over
    // the bits in which the members' keys differ; then, of the list's entries with this key and class (classes: the class bits
    // that count), which come in the order of their ranks, the one that is left.  Equal values, as constant or coarsely
    // quantised rows have them, need no bit and one pass over the list (a bit of key and list position at a time: fp32 [1 x 4096] of one value,
    // 8 + 8 blocks, 314 us, now 44).
    auto wave_select = [&](u32 a0, u32 c0, u32 a1, u32 c1, u32 rem, u32 classes, u32 cls, u32& hi, u32& lo) __attribute__((always_inline)) {
        auto key_at = [&](u32 i) -> u32 { return word_key(L.S[i < c0 ? a0 + i : a1 + (i - c0)]); };
        auto count = [&](auto take) -> u32 {
            u32 n = 0;
            for (u32 i = lane; i < c0 + c1; i += kWave) n += take(key_at(i)) ? 1u : 0u;
            return wave_sum(n);
        };
        u32 mx = 0, inv = 0;                        // largest key, complement of the smallest
        for (u32 i = lane; i < c0 + c1; i += kWave) { const u32 x = key_at(i); mx = max(mx, x); inv = max(inv, ~x); }
        u32 key = wave_max_dpp(mx), left = rem;
        const u32 differ = key ^ ~wave_max_dpp(inv);
        if (differ) {
            u32 bit = 0x80000000u >> __clz((int)differ);
            key &= ~(2u * bit - 1u);
            for (; bit; bit >>= 1) {
                const u32 t = key | bit;
                if (count([&](u32 x) -> bool { return x >= t; }) > rem) key = t;
            }
            left -= count([&](u32 x) -> bool { return x > key; });
        }
        hi = 0; lo = 0;
        u32 entries = nL;
        asm volatile("" : "+s"(entries));           // (or the slots' lane masks would be held for the whole row)
#pragma unroll(MAXS ? MAXS : 1)
        for (int s = 0; s < SLN; ++s) {
            if (s >= nslots) break;
            const u32 x = ent_word(s);
            const bool is = (int)lane < (int)entries - s * kWave && word_key(x) == key && (x & classes) == cls;
            const u64 m = __ballot(is);
            const u32 c = (u32)__popcll(m);
            if (left < c) {
                const int l = (int)__builtin_ctzll(__ballot(is && mask_rank(m) == left));
                hi = bcast(x, l); lo = ~(u32)(s * kWave + l);
                break;
            }
            left -= c;
        }
    };

    // ---- top-K cut: the comp of overall rank k-1 (ATKF) -----------------------------------------
    u32 thrK = 0, thrK_lo = 0;                      // without the class bit; every entry of L is kept when nL <= k
    bool eq_cut = false;                            // fp32: equal keys on both sides of the cut: the low words decide
    if (nL > (u32)k) {
        // open the bins of the lane found by the scan: the first one that ends behind rank k-1
        const int hi = FB - cut_lane * BPL;
        const u32 wj = lane < (u32)BPL ? L.hist[bin_word((u32)hi - 1u - lane)] : 0u;
        const u64 mj = __ballot(lane < (u32)BPL && (wj >> 16) + (wj & 0xFFFFu) - nLp > (u32)(k - 1));
        const int fj = (int)__builtin_ctzll(mj), lo = hi - 1 - fj;
        const u32 wd = bcast(wj, fj), wu = (u32)__builtin_amdgcn_readfirstlane((int)L.hist[bin_word((u32)lo + 1u)]);
        const u32 sp = wu >> 16, sn = wu & 0xFFFFu, cp = (wd >> 16) - sp, cnt = cp + (wd & 0xFFFFu) - sn;
        const u32 rem = (u32)(k - 1) - (sp + sn - nLp);
        u32 kp, kn;                                 // members that stay
        if (__builtin_expect(cnt <= (u32)kWave, 1)) {
            const bool in = lane < cnt;
            const u32 at = in ? (lane < cp ? sp + lane : sn + lane - cp) : 0u;
            const u32 me = in ? L.S[at] & kMag : 0u, ml = in ? low_of(at) : 0u;
            u32 gt = 0;
            for (u32 j = 0; j < cnt; ++j) gt += beats(bcast(me, (int)j), bcast(ml, (int)j), me, ml) ? 1u : 0u;
            const u64 stay = __ballot(in && gt <= rem);
            kn = (u32)__popcll(stay);
            kp = (u32)__popcll(stay & ((cp < 64u ? 1ull << cp : 0ull) - 1ull));
            kn -= kp;
            const int hl = (int)__builtin_ctzll(__ballot(in && gt == rem));
            thrK = bcast(me, hl);
            if (DT == 0) { thrK_lo = bcast(ml, hl); eq_cut = __popcll(__ballot(in && me == thrK)) > 1; }
        } else {
            wave_select(sp, cp, sn, cnt - cp, rem, 0u, 0u, thrK, thrK_lo);
            thrK &= kMag;
            eq_cut = true;
            u32 n = 0;
            for (u32 i = lane; i < cp; i += kWave) n += beats(thrK, thrK_lo, L.S[sp + i] & kMag, low_of(sp + i)) ? 0u : 1u;
            kp = wave_sum(n);
            kn = rem + 1u - kp;
        }
        n_pos = sp + kp; n_neg = sn - nLp + kn;
    }
    const u32 n = n_pos + n_neg;
    const u32 Kc[2] = { (u32)__builtin_amdgcn_readfirstlane((int)udiv16(n_pos, (u32)M)), (u32)__builtin_amdgcn_readfirstlane((int)udiv16(n_neg, (u32)Mn)) };

    // ---- block boundaries: comps of class ranks j*K-1 ----------------------------------------------
    // M-1 boundaries for the positive class, then Mn-1 for the negative one, a few lanes each.  A class with fewer than M
    // members has K = 0 and every member in its last block: its boundaries sit above every comp of the class.
    // S holds the bin of a class rank at this very place; a search over the bins' first ranks, one lane a boundary, and
    // lanes dealt to (boundary, member) pairs took 356 vector instructions a row of 16 blocks (bf16 [16384 x 4096]), this takes 118.
    const int ntg = B2 - 2;
    u32* thr = L.thr;
    u64 eq_thr = 0;                                 // fp32: boundaries with equal keys on both sides (bit t << lg): the low words decide
    if (ntg > 0) {
        constexpr u32 kWide = 32;                   // members from which on wave_select takes fewer steps
        const int lg = a.lg;                        // log2 of the lanes per boundary
        const u32 t = lane >> lg, sub = lane & ((1u << lg) - 1u);
        const bool mine = (int)t < ntg;
        const int cls = (int)t >= M - 1 ? 1 : 0;
        const u32 j = t - (cls ? (u32)(M - 1) : 0u) + 1u, K = cls ? Kc[1] : Kc[0];
        const bool act = mine && K > 0;
        const u32 R = act ? j * K - 1u + (cls ? nLp : 0u) : 0u;         // its place
        const u32 bin = act ? key_bin(word_key(L.S[R])) : 0u;
        const u32 hf = cls ? 0u : 16u;
        const u32 st = __builtin_amdgcn_ubfe(L.hist[bin_word(bin + 1u)], hf, 16u);
        const u32 cn = act ? __builtin_amdgcn_ubfe(L.hist[bin_word(bin)], hf, 16u) - st : 0u, rem = R - st;
        if (mine && !act && sub == 0) { thr[t] = cls ? kMag : ~0u; if (DT == 0) L.thr_lo[t] = ~0u; }
        bool eq = DT == 0 && mine && !act && kmax == kMag;      // (no finite value is equal to the boundary above a class)
        if (cn <= kWide) {
            // entries behind the bin's end belong to lower bins or to the negative class or are zeros: none lies above a member
            for (u32 i = sub; i < cn; i += 1u << lg) {
                const u32 me = L.S[st + i], ml = low_of(st + i);
                u32 gt = 0, same = 0;
                for (u32 jj = 0; jj < cn; jj += 4) {
#pragma unroll
                    for (u32 u = 0; u < 4; ++u) {
                        const u32 x = L.S[st + jj + u];
                        gt += beats(x, low_of(st + jj + u), me, ml) ? 1u : 0u;
                        if (DT == 0) same += x == me ? 1u : 0u;
                    }
                }
                if (gt == rem) { thr[t] = me; if (DT == 0) { L.thr_lo[t] = ml; eq = same > 1u; } }
            }
        }
        for (u64 wide = __ballot(sub == 0 && cn > kWide); __builtin_expect(wide != 0ull, 0); wide &= wide - 1ull) {
            const int l = (int)__builtin_ctzll(wide);
            u32 vh, vl;
            wave_select(bcast(st, l), bcast(cn, l), 0u, 0u, bcast(rem, l), kPos, bcast(cls ? 0u : kPos, l), vh, vl);
            if (lane == 0) { thr[l >> lg] = vh; if (DT == 0) L.thr_lo[l >> lg] = vl; }
            eq = eq || (DT == 0 && (int)lane == l);
        }
        // (a boundary's lanes: the one that found its member, moved to the lowest)
        if (DT == 0)
            for (u64 found_by = __ballot(eq); __builtin_expect(found_by != 0ull, 0); found_by &= found_by - 1ull) eq_thr |= 1ull << (__builtin_ctzll(found_by) >> lg << lg);
    }

    // block starts in closed form (K, ..., K, K + remainder per class)
    const bool one_key = sh == 0;                    // a bin holds one key: S has a block's largest and smallest key at its ends
    if ((int)lane < B2) {
        const int s = (int)lane >= M ? 1 : 0, m = (int)lane - s * M;
        const u32 K = s ? Kc[1] : Kc[0], st = (s ? n_pos : 0u) + (u32)m * K;
        L.blk_start[lane] = st;
        L.run[lane] = st;
        u32 lo = 0xFFFFFFFFu, hi = 0;
        if (one_key) {
            const u32 at = st + (s ? nLp - n_pos : 0u), cnt = m < (s ? Mn : M) - 1 ? K : (s ? n : n_pos) - st;
            hi = word_key(L.S[at]);
            lo = word_key(L.S[cnt ? at + cnt - 1u : at]);
        }
        L.vminb[lane] = lo; L.vmaxb[lane] = hi;
    }
    if (lane == 0) L.blk_start[B2] = n;
    wave_sync();

    // ---- 4. blocks, stable split by block, block-ordered arrays -----------------------------------
    // S and the fine bins are dead (boundaries are resolved): S's storage takes the
    // block-ordered values, the histogram region the indices and the stream image
    u32* bo_val = L.S;
    uint16_t* bo_idx = (uint16_t*)(L.hist);
    u32* stage = L.hist + (k + 1) / 2;
    // An entry's block = number of boundaries above it, plus one for the negative class: a
    // positive entry is above every negative boundary, a negative entry below every positive
    // one.  Up to kRegThr boundaries are held in registers.
    u32 tx[kRegThr];
#pragma unroll
    for (int j = 0; j < kRegThr; ++j) tx[j] = j < ntg ? thr[j] : 0u;
    // plo, phi: the kept lanes of this slot in the same block
    auto place = [&](int s, u32 cx, bool kept, u32 b, u32 plo, u32 phi) __attribute__((always_inline)) {
        const u32 before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        if (kept) {
            const u32 key = word_key(cx), base = L.run[b];
            if (!one_key) { atomicMin(&L.vminb[b], key); atomicMax(&L.vmaxb[b], key); }
            wave_sync();                            // every lane of the block has read run[b] before one moves it on
            if (before == 0) L.run[b] = base + (u32)__popc(plo) + (u32)__popc(phi);
            bo_val[base + before] = E::value_bits(key);
            bo_idx[base + before] = (uint16_t)ent_index(s);
        }
        wave_sync();                                // the next slot reads the moved places
    };
    auto is_kept = [&](int s, u32 cx) -> bool {
        bool kept = in_list(s) && (cx & kMag) >= thrK;
        if (DT == 0 && __builtin_expect(eq_cut, 0)) kept = kept && !beats(thrK, thrK_lo, cx & kMag, ~(u32)(s * kWave + (int)lane));
        return kept;
    };
    if (M == 8 && Mn == 8 && !(DT == 0 && eq_thr)) {
        // 8 + 8 blocks: the 14 boundaries and the class bit are 15 separators in descending order; four compares walk them
        // as a binary tree (the first is the class bit itself).  Their outcomes are the bits of the block number, and
        // the compares' lane masks the ballots that the ranks inside a block need (split 604 -> 503 vector instructions a row,
        // kernel 74.1 -> 68.3 us, with the block ranges read from S and no nested conditions).
#pragma unroll(MAXS ? MAXS : 1)
        for (int s = 0; s < SLN; ++s) {
            if (s >= nslots) break;
            const u32 cx = ent_word(s);
            const bool kept = is_kept(s, cx);
            const bool c1 = !(cx & kPos);
            u32 m = c1 ? tx[10] : tx[3];
            const bool c2 = m > cx;
            m = c1 ? (c2 ? tx[12] : tx[8]) : (c2 ? tx[5] : tx[1]);
            const bool c3 = m > cx;
            const u32 lo4 = c3 ? (c2 ? tx[6] : tx[2]) : (c2 ? tx[4] : tx[0]);
            const u32 hi4 = c3 ? (c2 ? tx[13] : tx[9]) : (c2 ? tx[11] : tx[7]);
            m = c1 ? hi4 : lo4;
            const bool c4 = m > cx;
            const u64 km = __ballot(kept);
            u32 b = 0, plo = (u32)km, phi = (u32)(km >> 32);
            auto bit = [&](bool c, u32 value) __attribute__((always_inline)) {
                const u64 bal = __ballot(c);
                const u32 onm = c ? ~0u : 0u;
                b |= onm & value;
                plo &= ~((u32)bal ^ onm);
                phi &= ~((u32)(bal >> 32) ^ onm);
            };
            bit(c1, 8u); bit(c2, 4u); bit(c3, 2u); bit(c4, 1u);
            place(s, cx, kept, b, plo, phi);
        }
    } else {
#pragma unroll(MAXS ? MAXS : 1)
        for (int s = 0; s < SLN; ++s) {
            if (s >= nslots) break;
            const u32 cx = ent_word(s);
            const bool kept = is_kept(s, cx);
            u32 b = (cx & kPos) ? 0u : 1u;
#pragma unroll
            for (int j = 0; j < kRegThr; ++j) b += tx[j] > cx ? 1u : 0u;
            for (int j = kRegThr; j < ntg; ++j) b += thr[j] > cx ? 1u : 0u;
            if (DT == 0)                             // boundaries of the same key, one or two in most rows that have any
                for (u64 m = eq_thr; __builtin_expect(m != 0ull, 0); m &= m - 1ull) {
                    const int j = (int)__builtin_ctzll(m) >> a.lg;
                    b += thr[j] == cx && L.thr_lo[j] > ~(u32)(s * kWave + (int)lane) ? 1u : 0u;
                }
            // one ballot per bit of the block number
            const u64 km = __ballot(kept);
            u32 plo = (u32)km, phi = (u32)(km >> 32);
            for (int bit = 0; bit < a.nbits; ++bit) {
                const u32 onm = (u32)__builtin_amdgcn_sbfe((int)b, (u32)bit, 1u);   // all ones if the bit is set
                const u64 bal = __ballot(onm != 0u);
                plo &= ~((u32)bal ^ onm);
                phi &= ~((u32)(bal >> 32) ^ onm);
            }
            place(s, cx, kept, b, plo, phi);
        }
    }
    wave_sync();

    // ---- 5. ABQ -----------------------------------------------------------------------------------
    // A block has lpb = kWave / B2 lanes.  For the sums each of them takes some of the candidate bitwidths and walks the whole
    // block (a slice of it where a block has sixteen lanes or more): the sums stay in registers and the lane decides on
    // its bitwidths by itself.  Lanes that walked a share of the block for all bitwidths had to add their sums up with 64-bit
    // LDS atomics, four lanes on an address: 312 of a row's 1486 busy cycles of the LDS (16 blocks) and 645 * 4 cycles of
    // waiting (kernel, bf16 [16384 x 4096]: 80.4 -> 75.8 us, fp32 [12608 x 768]: 42.6 -> 39.8).  The energy, and later the packing, share the block's entries out.
    u64* sums = (u64*)(L.hist + ((((k + 1) / 2 + (int)a.cap_words) + 1) & ~1));
    const int ns = small_block_sums(B2, nq);         // a block's sums; the last one is its energy
    float* invt = (float*)(sums + B2 * ns);
    const u32 lpb = (u32)a.lpb;
    const u32 myb = udiv16(lane, lpb), sub = lane - myb * lpb;
    const bool lane_on = myb < (u32)B2;
    u32 r0 = 0, r1 = 0, bs0 = 0, mycnt = 0;
    float vmin = 0.f, rng = 0.f, rng1 = 1.f;
    int e = 0, dg = 1, er = 0;
    u32 vmaxbits = 0;
    if (lane_on) {
        bs0 = L.blk_start[myb];
        const u32 be = L.blk_start[myb + 1];
        mycnt = be - bs0;
        const u32 perb = udiv16(mycnt + lpb - 1, lpb);
        r0 = bs0 + sub * perb; r0 = r0 < be ? r0 : be;
        r1 = r0 + perb < be ? r0 + perb : be;
        if (mycnt) {
            const u32 lo = E::value_bits(L.vminb[myb]);
            vmaxbits = E::value_bits(L.vmaxb[myb]);
            vmin = __uint_as_float(lo);
            rng = __uint_as_float(vmaxbits) - vmin;
            dg = !(rng > 0.f);                       // only a range of exactly 0 is degenerate
            if (!dg) { er = range_exp(rng); rng1 = unit_range(rng, er); }
            e = ilogb_bits(vmaxbits) + 1;
        }
    }
    // longest run of any lane: the largest block holds K + (n mod M) entries
    const u32 mc0 = n_pos - Kc[0] * (u32)(M - 1), mc1 = n_neg - Kc[1] * (u32)(Mn - 1);
    const u32 maxb = mc0 > mc1 ? mc0 : mc1;
    const u32 T = udiv16(maxb + lpb - 1, lpb);
    // quantiser scales L / (range brought to [1, 2)): the lanes of a block share the divisions through LDS
    if (lane_on) {
        for (u32 t = sub; t < (u32)nq; t += lpb) {
            const float Lq = (float)((1u << L.qtab[t]) - 1u);
            invt[myb * (u32)nq + t] = dg ? 0.f : Lq / rng1;
        }
        if (sub == 0) {
            sums[myb * ns + ns - 1] = 0;
            // budget guard: index of the chosen bitwidth, nq = none feasible yet; DS guard: mask of violations
            L.run[myb] = (mycnt && !dg && a.guard == 0) ? (u32)nq : 0u;
        }
    }
    wave_sync();
    if (a.lad.on) {
        if (lane_on && sub == 0) L.run[myb] = ladder_index(a.lad, (int)(myb >= (u32)M ? myb - (u32)M : myb));
    } else {
        const u32 cl = (u32)a.cl, es = (u32)a.es;    // lanes with candidates of their own; slices of the block
        const u32 ct = es > 1u ? sub & (cl - 1u) : sub, sl = es > 1u ? sub >> __builtin_ctz(cl) : 0u;     // (cl: a power of two then)
        const bool active = lane_on && ct < cl && sl < es;
        const u32 per = es > 1u ? udiv16(mycnt + es - 1u, es) : mycnt, T2 = es > 1u ? udiv16(maxb + es - 1u, es) : maxb;
        const AbqSlice slice = small_abq_slice(bs0, mycnt, per, sl, active);
        const u32 q0 = slice.q0, qn = slice.qn;
        if (es > 1u && active) for (u32 t = ct + cl * sl; t < (u32)nq; t += cl * es) sums[myb * ns + t] = 0;
        double rhs = 0.0;
        if (a.guard == 0) {
            u64 accE = 0;
            for (u32 i = 0; i < T; i += 4) {
                u32 v[4];                            // (beyond the lane's share: not used)
                const u32 at = small_group_at(r0 + i, cap);
#pragma unroll
                for (u32 j = 0; j < 4; ++j) v[j] = bo_val[at + j];
#pragma unroll
                for (u32 j = 0; j < 4; ++j) {
                    u32 A = (u32)rintf(ldexpf(__uint_as_float(v[j]), 20 - e));      // 20-bit energy grid scaled to vmax
                    A = r0 + i + j < r1 ? A & 0x1FFFFFu : 0u;    // (at most 2^20: 24-bit products)
                    accE += (u64)A * (u64)A;
                }
            }
            if (accE) atomicAdd(&sums[myb * ns + ns - 1], accE);
            wave_sync();
            if (lane_on) rhs = a.beta * ldexp((double)sums[myb * ns + ns - 1], 2 * e - 40);
        }
        auto decide = [&](u32 t, u64 sum) __attribute__((always_inline)) {          // (mycnt > 0 and a range above 0)
            if (a.guard == 1) {
                if (t + 1u < (u32)nq && !((double)sum <= a.beta * (double)mycnt)) atomicOr(&L.run[myb], 1u << t);
            } else {
                const float Lq = (float)((1u << L.qtab[t]) - 1u);
                const float o = rng / Lq;
                if (((double)o * (double)o) * (double)sum * 0x1p-30 <= rhs) atomicMin(&L.run[myb], t);
            }
        };
        bool small_q = true;
#pragma unroll
        for (int t = 0; t < QN; ++t)
            if ((NQ || t < nq) && a.qlist[t] > 8) small_q = false;
        // MODE 0: squared error, bitwidths up to 8; 1: squared error, any bitwidth; 2: Eq. "DS"
        u32 least = 0;
        if (es == 1u) {
            const u32 l0 = Kc[0] ? Kc[0] : n_pos ? n_pos : ~0u, l1 = Kc[1] ? Kc[1] : n_neg ? n_neg : ~0u;
            least = l0 < l1 ? l0 : l1;
        }
        // FOLD: the scaling by 2^-er is part of the scales (exact: the same products, as long as nothing leaves the normal range)
        auto walk = [&](auto mode, auto fold, auto ncand, u32 c0) __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode)::value, NCU = decltype(ncand)::value;
            constexpr bool FOLD = decltype(fold)::value;
            // Residual of a code on the 2^-15 grid, rho = rint((y - rint(y)) * 2^15) with y = d * inv:
            // z = d * (inv * 2^15) equals y * 2^15 exactly, rint(y) * 2^15 is a multiple of 2^15, and
            // |rho| <= 2^14, so rho is rint(z) reduced to 15 signed bits (for |rho| = 2^14 the sign is
            // lost, the square is not).  Bitwidths up to 8 keep z below 2^23, where adding 2^23 rounds
            // to the integer grid with the same round-half-even.
            float inv[NCU];
            u32 tt[NCU], shq[NCU];
            u64 tot[NCU];
            const int top = nq - 1, qtop = (int)L.qtab[top];
            const float inv_top = MODE == 2 && lane_on ? invt[myb * (u32)nq + (u32)top] : 0.f;
#pragma unroll
            for (int u = 0; u < NCU; ++u) {
                tt[u] = ct + (c0 + (u32)u) * cl;
                const bool has = active && tt[u] < (u32)nq;
                inv[u] = has ? invt[myb * (u32)nq + tt[u]] : 0.f;
                if (MODE == 0) inv[u] = FOLD ? ldexpf(inv[u], 15 - er) : inv[u] * 32768.0f;
                shq[u] = MODE == 2 && has ? (u32)(qtop - (int)L.qtab[tt[u]]) : 0u;
                if (!has) tt[u] = ~0u;
                tot[u] = 0;
            }
            auto four = [&](u32 i, u32 (&acc)[NCU], auto tail) __attribute__((always_inline)) {
                u32 v[4];                            // (beyond the block's end: not used)
                const u32 at = decltype(tail)::value ? small_group_at(q0 + i, cap) : q0 + i;
#pragma unroll
                for (u32 j = 0; j < 4; ++j) v[j] = bo_val[at + j];
#pragma unroll
                for (u32 j = 0; j < 4; ++j) {
                    float d = __uint_as_float(v[j]) - vmin;
                    if (!FOLD) d = to_unit(d, er);
                    if (decltype(tail)::value) d = i + j < qn ? d : 0.f;    // (an offset of zero adds nothing)
                    const u32 ref0 = MODE == 2 ? (u32)rintf(d * inv_top) : 0u;      // within [0, 2^q - 1]: no clamp needed
#pragma unroll
                    for (int u = 0; u < NCU; ++u) {
                        if (MODE == 2) {
                            // | (code at q_bit >> (q_bit - q)) - code at q |
                            const u32 c = (u32)rintf(d * inv[u]), ref = ref0 >> shq[u];
                            acc[u] += ref > c ? ref - c : c - ref;
                        } else {
                            // (wider bitwidths: y first, then the exact scaling, so that nothing overflows)
                            const u32 zi = MODE == 0 ? __float_as_uint(d * inv[u] + 8388608.0f) : (u32)rintf((d * inv[u]) * 32768.0f);
                            const int rho = __builtin_amdgcn_sbfe((int)zi, 0u, 15u);
                            asm("v_mad_i32_i24 %0, %1, %1, %0" : "+v"(acc[u]) : "v"(rho));      // (as sums of products: half as many again)
                        }
                    }
                }
            };
            // every block that is not empty has at least `least` entries: no look at the block's end before that
            u32 i = 0;
            for (; i < T2; i += 8) {                 // u32 partial sums hold 8 residuals of 2^28
                u32 acc[NCU];
#pragma unroll
                for (int u = 0; u < NCU; ++u) acc[u] = 0;
                if (i + 8 <= least) {
                    four(i, acc, std::false_type());
                    four(i + 4, acc, std::false_type());
                } else {
                    four(i, acc, std::true_type());
                    if (i + 4 < T2) four(i + 4, acc, std::true_type());
                }
#pragma unroll
                for (int u = 0; u < NCU; ++u) tot[u] += acc[u];
            }
            if (active && mycnt && !dg) {
#pragma unroll
                for (int u = 0; u < NCU; ++u) {
                    if (tt[u] == ~0u) continue;
                    if (es > 1u) atomicAdd(&sums[myb * ns + tt[u]], tot[u]); else decide(tt[u], tot[u]);
                }
            }
        };
        auto walk_all = [&](auto mode, auto fold) __attribute__((always_inline)) {
            const u32 nc = (u32)a.nc;                // candidates of a lane
            if (nc == 1u) walk(mode, fold, std::integral_constant<int, 1>(), 0u);
            else if (nc == 2u) walk(mode, fold, std::integral_constant<int, 2>(), 0u);
            else for (u32 c0 = 0; c0 < nc; c0 += 4u) walk(mode, fold, std::integral_constant<int, 4>(), c0);
        };
        wave_sync();
        if (a.guard == 1) walk_all(std::integral_constant<int, 2>(), std::false_type());
        else if (!small_q) walk_all(std::integral_constant<int, 1>(), std::false_type());
        else if (__ballot(er < -60 || er > 60)) walk_all(std::integral_constant<int, 0>(), std::false_type());
        else walk_all(std::integral_constant<int, 0>(), std::true_type());
        wave_sync();
        if (es > 1u) {
            if (active && sl == 0u && mycnt && !dg) for (u32 t = ct; t < (u32)nq; t += cl) decide(t, sums[myb * ns + t]);
            wave_sync();
        }
        if (a.guard == 1) {
            // greedy descent: the chosen index is one above the highest violating candidate below q_bit
            if (lane_on && sub == 0) {
                const u32 viol = L.run[myb];
                L.run[myb] = viol ? 32u - (u32)__clz((int)viol) : 0u;
            }
        }
    }
    wave_sync();
    u32 myq = 0, flag = 0;
    float my_inv = 0.f;
    if (lane_on) {
        u32 tb = L.run[myb];
        if (tb == (u32)nq) { flag = 0x80u; tb = (u32)nq - 1u; }   // none feasible: the largest bitwidth, flagged
        myq = L.qtab[tb];
        my_inv = invt[myb * (u32)nq + tb];
    }
    if (lane_on && sub == 0) {
        const size_t mi = (size_t)r * (size_t)B2 + myb;
        a.mv.vmin[mi] = mycnt ? vmin : 0.f;
        a.mv.vmax[mi] = mycnt ? __uint_as_float(vmaxbits) : 0.f;
        a.mv.q[mi] = (uint8_t)(myq | flag);
    }
    // bit offsets of the blocks' code sections: scan over one lane per block
    const u32 mybits = (lane_on && sub == 0) ? mycnt * myq : 0u;
    const u32 incl_bits = wave_scan_dpp(mybits);
    const u32 code_bits = bcast(incl_bits, kWave - 1);
    const u32 my_off = incl_bits - mybits;              // valid in the block's first lane ...
    const u32 coff = (u32)__shfl((int)my_off, (int)(myb * lpb));   // ... fetched by its other lanes
    const u32 idx_bits = n * (u32)w;
    const u32 row_bits = idx_bits + code_bits;
    u32 row_words = (row_bits + 31u) >> 5;
    if ((u64)row_words > a.cap_words) row_words = (u32)a.cap_words;   // cannot happen (worst-case capacity)
    for (u32 i = lane; i < row_words; i += kWave) stage[i] = 0;
    wave_sync();

    // ---- packing ----------------------------------------------------------------------------------
    {
        // two neighbouring entries of a block at a time: their index fields (at most 13 bits) are one field of 2 w bits, their
        // codes one of 2 q bits; a field is put in by two atomic ORs on neighbouring words (an odd end adds
        // zeros).  One entry at a time took 262 vector instructions a row instead of 167 (75.8 -> 74.1 us).
        auto put = [&](u32 bit, u32 v) {
            const u64 f = (u64)v << (bit & 31u);
            u32* at = stage + (bit >> 5);
            atomicOr(at, (u32)f);
            atomicOr(at + 1, (u32)(f >> 32));
        };
        for (u32 p = r0, i = 0; i < T; i += 2, p += 2) {
            if (p < r1) {
                const bool two = p + 1u < r1;
                u32 c[2];
#pragma unroll
                for (u32 j = 0; j < 2; ++j) {
                    const float y = to_unit(__uint_as_float(bo_val[p + j]) - vmin, er) * my_inv;
                    c[j] = (u32)rintf(y);             // already within [0, 2^q - 1] (range 0: a scale and a code of 0)
                }
                put(__umul24(p, (u32)w), (u32)bo_idx[p] | (two ? (u32)bo_idx[p + 1u] << w : 0u));
                put(idx_bits + coff + __umul24(p - bs0, myq), c[0] | (two ? c[1] << myq : 0u));
            }
        }
    }
    wave_sync();
    u32* __restrict__ slot = a.stream ? a.stream : a.slots + (size_t)r * (size_t)a.cap_words;
    for (u32 i = lane; i < row_words; i += kWave) slot[i] = stage[i];
    if (lane == 0) {
        a.mv.n_pos[r] = n_pos;
        a.mv.n_neg[r] = n_neg;
        if (a.stream) {                              // a single row: its offset is known (bf16 [1 x 4096] ladder 14.2 -> 10.6 us)
            a.mv.row_off[r] = 0;
            write_header(a.meta, DT, M, Mn, a.R, a.N, a.k, a.bit_set, w, row_words);
        } else {
            a.row_words32[r] = row_words;
        }
        if (kHint && k > 0) a.hint[hslot] = nL > (u32)k ? word_key(thrK) : t_lo;    // this row's cut key, for a later row
    }
}

}  // namespace slicer
