// C ABI of the SLICER IF codec for MI355X (see include/slicer.h): argument
// checks, workspace carving and kernel launches.  No device memory is allocated.
#include "../../include/slicer.h"

#include <hip/hip_runtime.h>
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>

#include "slicer_common.hpp"
#include "slicer_encode_generic.hpp"
#include "slicer_launch.hpp"
#include "slicer_encode_wg.hpp"
#include "slicer_encode_large.hpp"
#include "slicer_decode.hpp"
#include "slicer_csr.hpp"

using namespace slicer;

// Scratch of slicer_encode_static: the workspace of an encode call for callers that cannot
// allocate.  Every GPU the library runs on holds its own copy until the process ends.
static __device__ __align__(256) unsigned char scratch[SLICER_STATIC_SCRATCH_BYTES];

namespace {

thread_local int g_last_hip_error = 0;
thread_local hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;

inline int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return SLICER_EHIP;
}

#define SLICER_HIP(call)                                   \
    do {                                                   \
        hipError_t e_ = (call);                            \
        if (e_ != hipSuccess) return hip_fail(e_);         \
    } while (0)

int check_shape(int dt, int64_t rows, int64_t row_len, int n_blocks)
{
    if (dt != SLICER_F32 && dt != SLICER_BF16) return SLICER_EUNSUPPORTED;
    if (rows <= 0 || row_len <= 0 || row_len >= ((int64_t)1 << 31)) return SLICER_EINVAL;
    if (n_blocks < 1 || n_blocks > SLICER_MAX_BLOCKS) return SLICER_EINVAL;
    return SLICER_OK;
}

int check_args(int dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks, uint32_t bit_set)
{
    int rc = check_shape(dt, rows, row_len, n_blocks);
    if (rc) return rc;
    if (!(keep_ratio >= 0.0 && keep_ratio <= 1.0)) return SLICER_EINVAL;
    if (bit_set == 0 || (bit_set & ~0x1FFFEu)) return SLICER_EINVAL;
    return SLICER_OK;
}

int index_bits(int64_t N)
{
    int w = 1;
    while (((int64_t)1 << w) < N) ++w;
    return w;
}

struct Plan {
    int64_t k, kept_stride;
    int w, qmax;
    u64 cap_words;          // per row
    size_t off_row_words, off_slots, off_kept, off_bo_idx, off_bo_val, off_fallback, off_row_local, off_chunk_tot, off_hint, total;
    // row-resident fast path (0 = not eligible)
    int small_epl, small_cap, small_region0, small_lds_bytes, small_maxs;
    // workgroup-per-row path for rows of up to 32768 bf16 or 16384 fp32 elements (0 = not eligible)
    int wg_ept, wg_nw, wg_cap, wg_region0, wg_lds_bytes;
    bool one_wave;          // a row that either row-resident kernel holds goes to one wavefront (lambda = 0)
    // long-row path (large_S == 0: not eligible)
    int large_S, large_fb;  // tiles per row, fine bins
    u32 large_capL;
    size_t lo_tab, lo_cum, lo_seg, lo_rowst, lo_thr, lo_vminb, lo_vmaxb, lo_blk_start, lo_pair, lo_sums,
           lo_qsel, lo_inv_sel, lo_code_off;
};

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int count_bits(int64_t k)      // bits that hold any value in 0..k
{
    int w = 1;
    while (((int64_t)1 << w) <= k) ++w;
    return w;
}

// Members of the fine bins that hold a block's first or last element (two per block, most of them shared), about: a bin is filled
// with 8 to 16 entries, or with the list's share and up to twice as many, and all of them together cannot hold more than the list, about 1.4 k.
int64_t large_members(int fine_bins, int64_t k, int B2)
{
    return std::min<int64_t>((B2 + 2) * std::max<int64_t>(12, k * 3 / (fine_bins * 7 / 5)), k * 14 / 10 + 100);
}

// Fine bins per row of the long-row stages.  Few of them in large batches (encode with 4096 and with 1024: fp32 [4096 x 20480]
// 821 and 529 us, bf16 [9494 x 8738] keep 0.01 M 64 2367 and 1146, bf16 [512 x 8193] M 40 113 and 108), where the members
// should fit a row's room of 1536.
int large_fine_bins(int64_t rows, int64_t k, int B2)
{
    return rows > kScanRows && large_members(kFBNarrow, k, B2) <= 1200 ? kFBNarrow : kFBWide;
}

// the bounds stage with the larger room
bool large_many_members(int64_t k, int B2) { return large_members(kFBWide, k, B2) > 4800; }

// Room for the stages' tables.  It is what they took with 4096 bins, a block for every bin, sums per tile and tiles of 8192 or 16384 elements,
// which is never less than they take now: the size of a workspace is part of what callers plan and store, and does not follow the stages' tuning.
size_t large_table_room(size_t R, int64_t row_len, int epc, int64_t k, size_t B2, size_t nq)
{
    const int64_t n8 = (row_len + 8191) / 8192, tile = (int64_t)R * n8 <= 256 || (R > kScanRows && (n8 == 1 || n8 == 3)) ? 8192 : 16384;
    const size_t S = (size_t)((row_len + epc - 1 + tile - 1) / tile);
    const int64_t members = std::min<int64_t>((int64_t)(B2 + 2) * std::max<int64_t>(12, k * 3 / 1400), k * 14 / 10 + 100);
    const size_t bins = R > kScanRows && members <= 1200 ? 1024 : 4096;
    size_t o = 0;
    for (size_t bytes : { 2 * R * kTabSize, 4 * R * S * bins, 8 * R * S, 4 * R * 16, 8 * R * B2, 2 * R * bins, 4 * R * B2, 4 * R * B2, 4 * R * (B2 + 1),
                          4 * R * B2 * S, 8 * R * S * B2 * (nq + 1), 4 * R * B2, 4 * R * B2, 8 * R * (B2 + 1) })
        o = align256(o + bytes);
    return o;
}

// aligned: x starts on a 16-byte boundary (the workspace layout does not depend on it, only the choice of kernel)
// long_rows: the long-row stages may serve the call; without them (the generic kernel) it needs less workspace
Plan make_plan(int dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks, int n_blocks_neg, uint32_t bit_set,
               bool aligned = true, bool long_rows = true)
{
    const int B2_all = n_blocks + n_blocks_neg;          // blocks per row
    Plan p;
    p.k = (int64_t)std::floor(keep_ratio * (double)row_len);   // ATKF: k = floor((1-s) N)
    p.w = index_bits(row_len);
    p.qmax = 16;
    while (!((bit_set >> p.qmax) & 1u)) --p.qmax;
    p.cap_words = ((u64)p.k * (u64)(p.w + p.qmax) + 31) / 32;

    size_t o = 0;
    p.off_row_words = o; o = align256(o + 8 * (size_t)rows);
    p.off_slots = o;     o = align256(o + 4 * (size_t)rows * (size_t)p.cap_words);
    p.kept_stride = p.k;
    p.off_bo_idx = o;    o = align256(o + 4 * (size_t)rows * (size_t)p.k);
    p.off_bo_val = o;    o = align256(o + 4 * (size_t)rows * (size_t)p.k);
    p.off_fallback = o;  o = align256(o + 4 * (size_t)rows);
    p.off_row_local = o; o = align256(o + 8 * (size_t)rows);
    p.off_chunk_tot = o; o = align256(o + 8 * (size_t)((rows + kScanRows - 1) / kScanRows));
    p.off_hint = o;      o = align256(o + 4 * (size_t)kHintSlots);
    const int epc = dt == SLICER_F32 ? 4 : 8;
    const bool whole_len = row_len % epc == 0, whole = whole_len && aligned;
    const int64_t span = row_len + (whole ? 0 : epc - 1);     // elements of the row's 16-byte chunks

    int nq = 0;
    for (int q = 1; q <= 16; ++q) nq += (bit_set >> q) & 1u;

    // The one-wave-per-row kernel holds the row in registers (64 * EPL elements) and
    // its lists in LDS; it needs 16-bit indices, one lane per
    // block and a list capacity below 2048 entries (11-bit rank fields).
    // A row that does not consist of whole aligned chunks may start anywhere in its first one.
    p.small_epl = 0; p.small_cap = 0; p.small_region0 = 0; p.small_lds_bytes = 0; p.small_maxs = 0;
    const int64_t margin = std::max<int64_t>(64, row_len / (dt == SLICER_F32 ? 16 : 32));  // room for the undecided coarse bin
    const int64_t cap = std::min<int64_t>(1984, (p.k + margin + 63) / 64 * 64);   // ranks are 11-bit fields
    const bool lists_fit = B2_all <= kWave && p.k + 64 <= cap;
    const int maxs = cap <= 256 ? 4 : cap <= 640 ? 10 : cap <= 1280 ? 20 : 0;             // list held in registers
    const int64_t region0 = lists_fit ? small_region0_words(dt, p.k, p.cap_words, B2_all, nq, (int)cap, small_fine_bins(maxs)) : 0;
    const int64_t wg_region0 = lists_fit ? wg_region0_words(p.k, p.cap_words, B2_all, nq) : 0;
    const int64_t small_lds = lists_fit ? 4 * (int64_t)small_lds_words(dt, (int)cap, (int)region0, B2_all, maxs) : 0;
    auto small_holds = [&](int64_t elements) { return lists_fit && elements <= (dt == SLICER_F32 ? 4096 : 8192) && small_lds <= 64 * 1024; };
    if (small_holds(span)) {
        int epl = epc;
        while ((int64_t)epl * kWave < span) epl *= 2;
        // fp32 rows of the common transformer widths 768 and 1280: three and five chunks per lane instead of four and eight
        if (dt == SLICER_F32 && span > 512 && span <= 768) epl = 12;
        if (dt == SLICER_F32 && span > 1024 && span <= 1280) epl = 20;
        p.small_epl = epl; p.small_cap = (int)cap; p.small_region0 = (int)region0; p.small_lds_bytes = (int)small_lds;
        p.small_maxs = maxs;
    }
    // One workgroup per row (the wavefronts of a workgroup share the row): every row of more than 4096 and up to
    // 32768 bf16 / 16384 fp32 elements, but for bf16 rows of up to 8192 whose list has at most 768 entries, in large batches.  One
    // wavefront per row does less work in all, and takes longer for a single row: the longer, the longer the list and the more
    // blocks.  Encode us, workgroup / wavefront, 8 + 8 blocks: [300 x 5120], 256 kept, 20.4 / 15.2, [512 x 8192], 409 kept, 21.5 / 18.3,
    // [2048 x 8192] 39 / 24; but [256 x 8192] 18 / 21, and lists of more entries [512 x 8192] 24.1 / 26.9, [4096 x 6144], 1228 kept, 80 / 81.
    // 16 + 16 blocks: [512 x 8192], 163 kept, 0.88 of the workgroup's time, 327 kept 1.14, and with 1024 rows 0.96; 24 + 24 and 32 + 32 blocks:
    // [257 x 5120], 51 kept, 0.95 and 0.99, 256 kept 1.20; [1500 x 6144], 245 kept, 0.97, 430 kept 1.03 and 1.08; with 2048 rows 0.60 to 0.84.
    p.wg_ept = 0; p.wg_nw = 0; p.wg_cap = 0; p.wg_region0 = 0; p.wg_lds_bytes = 0;
    const int64_t wg_lds = lists_fit ? 4 * (int64_t)wg_lds_words(dt, (int)cap, (int)wg_region0, B2_all) : 0;
    auto wg_holds = [&](int64_t elements) {
        return lists_fit && elements > 4096 && elements <= (dt == SLICER_F32 ? 16384 : 32768) && wg_lds <= 64 * 1024;
    };
    const int64_t few = B2_all <= 16 || (B2_all <= 32 && p.k <= 256) || p.k <= 64 ? kScanRows
                      : B2_all <= 32 ? 768 : p.k <= 256 ? 1024 : 2047;            // rows up to which the workgroup is faster
    p.one_wave = p.small_epl && (!wg_holds(span) || (cap <= 768 && rows > few));
    if (wg_holds(span)) {
        // wavefronts per row: sixteen for the smallest batches (more wavefronts per SIMD hide each other's
        // latencies: 4 % less latency per call), four otherwise (a 256-row batch on sixteen leaves no room
        // for a neighbouring stream's kernels: 20 % less throughput when steps overlap)
        p.wg_nw = rows <= 128 ? 16 : 4;
        const int64_t chunks = ((span + epc - 1) / epc + 64 * p.wg_nw - 1) / (64 * p.wg_nw);     // 16-byte chunks per thread
        p.wg_ept = (int)(chunks <= 1 ? 1 : chunks <= 2 ? 2 : chunks <= 4 ? 4 : chunks <= 8 ? 8 : 16);    // (kept as a chunk count)
        p.wg_cap = (int)cap; p.wg_region0 = (int)wg_region0; p.wg_lds_bytes = (int)wg_lds;
    }

    // Long rows: every pass is spread over many workgroups (slicer_encode_large.hpp).  A row that starts or ends
    // inside a 16-byte chunk takes them from 8192 elements on: below, one workgroup of the generic kernel is as fast.
    // The workspace holds the stages' tables (8 KB a tile and more) only where some row of this length can reach the
    // stages: not where a row-resident kernel holds the row wherever it starts.
    p.large_S = 0; p.large_capL = 0; p.large_fb = 0;
    auto row_kernel_holds = [&](int64_t elements) { return small_holds(elements) || wg_holds(elements); };
    auto held = [&] { return (!whole_len || row_kernel_holds(row_len)) && row_kernel_holds(row_len + epc - 1); };
    if (long_rows && row_len > 4096 && rows <= 65535 && (whole_len || row_len > 8192) && !held()) {      // (a call for short rows divides nothing here)
        const int64_t tile = large_tile(rows, row_len);
        const int64_t S = (row_len + tile - 1) / tile;       // rows of up to 2^23 elements
        const int64_t capL = (p.k + std::max<int64_t>(4096, row_len / 16) + 7) & ~(int64_t)7;
        if (S <= 512) {
            const size_t R = (size_t)rows, B2 = (size_t)B2_all, Sz = (size_t)S;
            if (whole || row_len > 8192) p.large_S = (int)S;
            p.large_capL = (u32)capL;
            p.large_fb = large_fine_bins(rows, p.k, B2_all);
            p.kept_stride = capL;
            const size_t tables = o;
            p.lo_tab = o;       o = align256(o + 2 * R * kTabSize);
            p.lo_cum = o;       o = align256(o + 4 * R * Sz * (size_t)p.large_fb);
            p.lo_seg = o;       o = align256(o + 8 * R * Sz);
            p.lo_rowst = o;     o = align256(o + 4 * R * 16);
            p.lo_thr = o;       o = align256(o + 8 * R * B2);
            p.lo_vminb = o;     o = align256(o + 4 * R * B2);
            p.lo_vmaxb = o;     o = align256(o + 4 * R * B2);
            p.lo_blk_start = o; o = align256(o + 4 * R * (B2 + 1));
            p.lo_pair = o;      o = align256(o + 4 * R * B2 * Sz);
            p.lo_sums = o;      o = align256(o + 8 * R * B2 * (size_t)(nq + 1));
            p.lo_qsel = o;      o = align256(o + 4 * R * B2);
            p.lo_inv_sel = o;   o = align256(o + 4 * R * B2);
            p.lo_code_off = o;  o = align256(o + 8 * R * (B2 + 1));
            o = std::max(o, tables + large_table_room(R, row_len, epc, p.k, B2, (size_t)nq));
        }
    }
    // the generic kernel's list of a row (8 bytes an entry) and the long-row list (a word and two halves) share their place
    p.off_kept = o;      o = align256(o + 8 * (size_t)rows * (size_t)p.kept_stride);
    p.total = o ? o : 256;
    return p;
}

template <int DT>
hipError_t launch_small_any(const SmallArgs& sa, const SmallLaunch& p, bool asym, hipStream_t st)
{
    if (asym) return sa.nq == 7 ? launch_small<DT, true, 7>(sa, p, st) : launch_small<DT, true, 0>(sa, p, st);
    return sa.nq == 7 ? launch_small<DT, false, 7>(sa, p, st) : launch_small<DT, false, 0>(sa, p, st);
}

template <int DT, int FB>
void launch_large_stages(const LargeArgs& la, const EncArgs& ea, const FinishArgs& fa, hipStream_t st)
{
    const dim3 gT((unsigned)la.S, (unsigned)la.R), gR((unsigned)la.R), gB((unsigned)(la.part_step * la.parts)), gW((unsigned)la.nwin, (unsigned)la.R), bT(kTileThreads);
    const dim3 bR((unsigned)lr_row_threads(FB));
    hipLaunchKernelGGL((lr_sample_kernel<DT, FB>), gR, bR, 0, st, la);
    if (la.dense) {
        if (la.tile <= 8192) hipLaunchKernelGGL((lr_compact_kernel<DT, 2, FB, true>), gT, bT, 0, st, la);
        else hipLaunchKernelGGL((lr_compact_kernel<DT, 4, FB, true>), gT, bT, 0, st, la);
    } else if (la.tile <= 8192) hipLaunchKernelGGL((lr_compact_kernel<DT, 2, FB, false>), gT, bT, 0, st, la);
    else hipLaunchKernelGGL((lr_compact_kernel<DT, 4, FB, false>), gT, bT, 0, st, la);
    if (FB == kFBWide && large_many_members(la.k, la.M + la.Mn))
        hipLaunchKernelGGL((lr_bounds_kernel<DT, FB, FB == kFBWide>), gB, bR, 0, st, la, ea);
    else hipLaunchKernelGGL((lr_bounds_kernel<DT, FB, false>), gB, bR, 0, st, la, ea);
    const size_t lds = (size_t)lr_split_carve(la.M, la.Mn, la.nq).total;
    if (la.nq == 7) hipLaunchKernelGGL((lr_split_kernel<DT, 7>), gT, bT, lds, st, la);   // {2..8}: the benchmarked set
    else hipLaunchKernelGGL((lr_split_kernel<DT, 0>), gT, bT, lds, st, la);
    if (la.n_cols > 0) hipLaunchKernelGGL((lr_pack_kernel<DT, true>), gW, dim3(256), 0, st, la, fa);
    else hipLaunchKernelGGL((lr_pack_kernel<DT, false>), gW, dim3(256), 0, st, la, fa);
}

template <int DT>
int launch_large(const LargeArgs& la, int fine_bins, const EncArgs& ea, const FinishArgs& fa, hipStream_t st)
{
    if (fine_bins == kFBNarrow) launch_large_stages<DT, kFBNarrow>(la, ea, fa, st);
    else launch_large_stages<DT, kFBWide>(la, ea, fa, st);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SLICER_OK : hip_fail(e);
}

template <int DT>
int launch_encode(const EncArgs& ea, hipStream_t st)
{
    const bool timed = g_ev_start && g_ev_stop && !ea.only_flagged;
    if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
    const unsigned grid = (unsigned)((ea.R + ea.rows_per_wg - 1) / ea.rows_per_wg);
    if (ea.N >= 32768)
        hipLaunchKernelGGL((enc_generic_kernel<DT, 1024>), dim3(grid), dim3(1024), 0, st, ea);
    else
        hipLaunchKernelGGL((enc_generic_kernel<DT, 256>), dim3(grid), dim3(256), 0, st, ea);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
    return SLICER_OK;
}

int launch_decode(const void* stream, const void* meta, void* y, int dt, int64_t rows, int64_t row_len,
                  int n_blocks, int n_blocks_neg, hipStream_t st)
{
    DecArgs da;
    da.stream = (const u32*)stream;
    da.y = y;
    da.R = rows; da.N = row_len; da.M = n_blocks; da.Mn = n_blocks_neg; da.w = index_bits(row_len);
    const int64_t dec_chunk = kDecChunkBytes / (dt == SLICER_F32 ? 4 : 2);
    da.chunks_per_row = (int)((row_len + dec_chunk - 1) / dec_chunk);
    da.mv = meta_view(const_cast<void*>(meta), rows, n_blocks + n_blocks_neg);
    da.total_words = (const u64*)meta + 6;
    // the stream segment of a row at keep ratios up to about 0.2 (longer segments are read from global memory)
    da.stage_words = (int)std::min<int64_t>(1020, (row_len / 16 + 3) / 4 * 4);
    da.xcd_map = (rows >= 32 && da.chunks_per_row > 1) ? 1 : 0;
    const u64 grid = (u64)(da.xcd_map ? xcd_grid(rows) : rows) * (u64)da.chunks_per_row;
    if (grid >= (1ull << 31)) return SLICER_EINVAL;
    const bool timed = g_ev_start && g_ev_stop;
    if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
    // short rows: one wavefront per row, the row assembled in LDS (16 KB per wave, and up to two more chunks for a
    // row that starts or ends inside a 16-byte chunk)
    const int64_t esz = dt == SLICER_F32 ? 4 : 2, row_bytes = row_len * esz;
    const int64_t image16 = (row_bytes % 16 == 0 && ((uintptr_t)y & 15) == 0) ? row_bytes / 16 : (row_bytes + 2 * (16 - esz)) / 16;
    if (row_bytes <= 16 * 1024 && n_blocks + n_blocks_neg <= kWave && (uintptr_t)y % (uintptr_t)esz == 0) {
        // one wave per workgroup: the LDS of a row (image + stream segment) is the unit of occupancy
        const size_t lds = 16 * (size_t)image16 + 16 * (size_t)((da.stage_words + 4) / 4);
        if (dt == SLICER_F32)
            hipLaunchKernelGGL((dec_small_kernel<0>), dim3((unsigned)xcd_grid(rows)), dim3(kWave), lds, st, da);
        else
            hipLaunchKernelGGL((dec_small_kernel<1>), dim3((unsigned)xcd_grid(rows)), dim3(kWave), lds, st, da);
    } else if (grid <= 256) {       // a workgroup per CU at most: more threads shorten its chain (fp32 [1 x 200704] 5.9 -> 5.5 us; a full chip, [32 x 401408]: 20.5 -> 24.2)
        if (dt == SLICER_F32) hipLaunchKernelGGL((dec_kernel<0, 512>), dim3((unsigned)grid), dim3(512), 0, st, da);
        else hipLaunchKernelGGL((dec_kernel<1, 512>), dim3((unsigned)grid), dim3(512), 0, st, da);
    } else {
        if (dt == SLICER_F32) hipLaunchKernelGGL((dec_kernel<0, 256>), dim3((unsigned)grid), dim3(256), 0, st, da);
        else hipLaunchKernelGGL((dec_kernel<1, 256>), dim3((unsigned)grid), dim3(256), 0, st, da);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
    return SLICER_OK;
}

}  // namespace

extern "C" {

int slicer_sizes_pn(slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks,
                    int n_blocks_neg, uint32_t bit_set, size_t* stream_capacity_bytes, size_t* meta_bytes_out,
                    size_t* workspace_bytes)
{
    int rc = check_args((int)dt, rows, row_len, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    if (n_blocks_neg < 1 || n_blocks_neg > SLICER_MAX_BLOCKS) return SLICER_EINVAL;
    Plan p = make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks_neg, bit_set);
    if (stream_capacity_bytes) *stream_capacity_bytes = (size_t)(p.cap_words * 4ull * (u64)rows);
    if (meta_bytes_out) *meta_bytes_out = meta_bytes(rows, n_blocks + n_blocks_neg);
    if (workspace_bytes) *workspace_bytes = p.total;
    return SLICER_OK;
}

int slicer_sizes(slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks,
                 uint32_t bit_set, size_t* stream_capacity_bytes, size_t* meta_bytes_out,
                 size_t* workspace_bytes)
{
    return slicer_sizes_pn(dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, stream_capacity_bytes,
                           meta_bytes_out, workspace_bytes);
}

int slicer_encode_path(slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks,
                       uint32_t bit_set)
{
    int rc = check_args((int)dt, rows, row_len, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    Plan p = make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set);
    return p.one_wave ? 1 : p.wg_ept ? 3 : p.large_S ? 2 : 0;
}

// two-dimensional instances whose stream the long-row stages write in CSR form themselves
struct CsrShape {
    int64_t n_rows, n_cols;
    int wp, wc;
    u64 cap_words;
};

static int encode_impl(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                       int n_blocks, int n_blocks_neg, uint32_t bit_set, double distortion_budget, const Ladder& lad, int guard,
                       void* stream, void* meta, void* workspace, void* hip_stream, double lambda = 0.0, const CsrShape* csr = nullptr,
                       bool long_rows = true)
{
    if (!(lambda >= 0.0 && lambda < 1.0)) return SLICER_EINVAL;
    const bool asym = (float)lambda > 0.0f;      // lambda = 0 is the plain top-K filter: every fast path applies
    int rc = check_args((int)dt, rows, row_len, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    if (!x || !stream || !meta || !workspace) return SLICER_EINVAL;
    if (!(distortion_budget >= 0.0)) return SLICER_EINVAL;
    if (rows >= ((int64_t)1 << 31)) return SLICER_EINVAL;
    if (n_blocks_neg < 1 || n_blocks_neg > SLICER_MAX_BLOCKS) return SLICER_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const bool aligned = ((uintptr_t)x & 15) == 0, on_elements = ((uintptr_t)x & (dt == SLICER_F32 ? 3 : 1)) == 0;
    Plan p = make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks_neg, bit_set, aligned, long_rows);
    char* ws = (char*)workspace;

    EncArgs ea;
    ea.x = x;
    ea.R = rows; ea.N = row_len; ea.k = p.k;
    ea.M = n_blocks; ea.Mn = n_blocks_neg; ea.w = p.w;
    ea.nq = 0;
    for (int q = 1; q <= 16; ++q)
        if ((bit_set >> q) & 1u) ea.qlist[ea.nq++] = q;
    for (int t = ea.nq; t < kMaxQ; ++t) ea.qlist[t] = 0;
    ea.beta = distortion_budget;
    ea.cap_words = p.cap_words;
    ea.kept_stride = p.kept_stride;
    ea.row_words = (u64*)(ws + p.off_row_words);
    ea.slots = (u32*)(ws + p.off_slots);
    ea.kept = (u64*)(ws + p.off_kept);
    ea.bo_idx = (u32*)(ws + p.off_bo_idx);
    ea.bo_val = (u32*)(ws + p.off_bo_val);
    ea.mv = meta_view(meta, rows, n_blocks + n_blocks_neg);
    ea.only_flagged = nullptr;
    ea.rows_per_wg = 1;
    ea.lad = lad;
    ea.guard = guard;
    ea.asym = asym ? 1 : 0;
    ea.one_plus = 1.0f + (float)lambda;
    ea.one_minus = 1.0f - (float)lambda;

    // asymmetric thresholds need a second selection over a subset of the row: the row-resident kernels have it for every row that
    // they hold, the generic kernel for every shape.  One wavefront takes long for two selections over a row of more than 4096 elements, so
    // the workgroup has all of these but, of large batches, the narrower ones with short lists and the longer ones whose list one wavefront has in
    // registers.  Encode us, wavefront / workgroup, lambda = 0.1, 8 + 8 blocks: bf16 [1 x 8192] 42 / 23, [256 x 8192] 49 / 29, [300 x 4160] 39 / 27,
    // [4000 x 8192] 101 / 88 (409 kept), [8000 x 8192] 275 / 194 (1228 kept), [5040 x 5952] 118 / 115 (595 kept); but [13000 x 4160] 195 / 210, and
    // [8000 x 8192] 156 / 156 (409 kept), 239 / 270 where the values are multiples of 1/8.
    const bool one_wave = asym ? rows > 4096 && (row_len <= 6144 ? p.one_wave : p.small_epl && p.small_maxs) : p.one_wave;
    const bool use_wg = p.wg_ept && on_elements && !one_wave;
    if (use_wg) {
        // one workgroup per row; rows it cannot hold are flagged and redone by the generic kernel
        SmallArgs sa;
        sa.x = x; sa.R = rows; sa.N = row_len; sa.k = p.k;
        sa.M = n_blocks; sa.Mn = n_blocks_neg; sa.w = p.w; sa.nq = ea.nq;
        for (int t = 0; t < kMaxQ; ++t) sa.qlist[t] = ea.qlist[t];
        sa.beta = distortion_budget;
        sa.cap_words = p.cap_words;
        sa.row_words = ea.row_words; sa.row_words32 = nullptr; sa.slots = ea.slots;
        sa.fallback = (u32*)(ws + p.off_fallback);
        sa.stream = nullptr; sa.meta = meta; sa.bit_set = bit_set;
        sa.mv = ea.mv;
        sa.cap = p.wg_cap; sa.region0_words = p.wg_region0;
        sa.lad = lad;
        sa.guard = guard;
        sa.one_plus = ea.one_plus; sa.one_minus = ea.one_minus;
        sa.hint = (u32*)(ws + p.off_hint);
        const bool timed = g_ev_start && g_ev_stop;
        if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
        const WgLaunch wl = { p.wg_nw, p.wg_ept, p.wg_lds_bytes };
        if (asym) SLICER_HIP((dt == SLICER_F32 ? launch_wg<0, true> : launch_wg<1, true>)(sa, wl, st));
        else SLICER_HIP((dt == SLICER_F32 ? launch_wg<0, false> : launch_wg<1, false>)(sa, wl, st));
        if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
        ea.only_flagged = sa.fallback;
    }
    const bool use_small = !use_wg && p.small_epl && on_elements;
    if (use_small) {                                // one wavefront per row, whatever the row holds
        SmallArgs sa;
        sa.x = x; sa.R = rows; sa.N = row_len; sa.k = p.k;
        sa.M = n_blocks; sa.Mn = n_blocks_neg; sa.w = p.w; sa.nq = ea.nq;
        for (int t = 0; t < kMaxQ; ++t) sa.qlist[t] = ea.qlist[t];
        sa.beta = distortion_budget;
        sa.cap_words = p.cap_words;
        sa.row_words = nullptr; sa.row_words32 = (u32*)(ws + p.off_row_words); sa.slots = ea.slots;
        sa.fallback = nullptr;
        sa.stream = rows == 1 ? (u32*)stream : nullptr; sa.meta = meta; sa.bit_set = bit_set;
        sa.mv = ea.mv;
        sa.cap = p.small_cap; sa.region0_words = p.small_region0;
        sa.lad = lad;
        sa.guard = guard;
        sa.one_plus = ea.one_plus; sa.one_minus = ea.one_minus;
        sa.hint = (u32*)(ws + p.off_hint);
        const bool timed = g_ev_start && g_ev_stop;
        if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
        small_split_lanes(sa);
        const SmallLaunch sl = { p.small_epl, p.small_lds_bytes, p.small_maxs };
        SLICER_HIP(dt == SLICER_F32 ? launch_small_any<0>(sa, sl, asym, st) : launch_small_any<1>(sa, sl, asym, st));
        if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
        if (rows == 1) return SLICER_OK;
    }
    FinishArgs fa;
    fa.R = rows; fa.N = row_len; fa.k = p.k;
    fa.M = n_blocks; fa.Mn = n_blocks_neg; fa.w = p.w; fa.dt = (int)dt;
    fa.bit_set = bit_set;
    fa.row_words = ea.row_words;
    fa.row_off_local = (u64*)(ws + p.off_row_local);
    fa.chunk_tot = (u64*)(ws + p.off_chunk_tot);
    fa.slots = ea.slots;
    fa.cap_words = p.cap_words;
    fa.chunks_per_row = (int)std::max<u64>(1, (p.cap_words + kGatherWords - 1) / kGatherWords);
    fa.stream = (u32*)stream;
    fa.meta = meta;
    fa.mv = ea.mv;
    fa.row_words32 = (const u32*)(ws + p.off_row_words);
    bool done = use_small;                          // every row is in its slot
    if (!done && !asym && !ea.only_flagged && p.large_S && on_elements) {
        // long rows: stages of many workgroups per row; rows they cannot hold are redone by the generic encoder inside the third one
        LargeArgs la;
        la.x = x; la.R = rows; la.N = row_len; la.k = p.k;
        la.M = n_blocks; la.Mn = n_blocks_neg; la.w = p.w; la.nq = ea.nq;
        for (int t = 0; t < kMaxQ; ++t) la.qlist[t] = ea.qlist[t];
        la.beta = distortion_budget; la.cap_words = csr ? csr->cap_words : p.cap_words;
        const int epc = dt == SLICER_F32 ? 4 : 8;
        la.tile = large_tile(rows, row_len);
        la.S = (int)((row_len + la.tile - 1) / la.tile);
        la.capL = p.large_capL;
        // workgroups that share a row in the bounds stage: as many as there are CUs for
        la.parts = rows <= 32 ? 8 : rows <= 64 ? 4 : rows <= 128 ? 2 : 1;
        // a row's workgroups on one XCD, rows on one after the other: its L2 serves their tables, and where a row is redone the row (five
        // rows of 597761 that are: 1897 us where their last workgroups ran, two of them on one XCD, 1390 now; [3 x 401408] 60.4 -> 56.7)
        la.part_step = la.parts == 1 || rows == 1 ? (int)rows : (int)((rows + 7) / 8 * 8);
        lr_sample_plan(la, p.large_fb, epc);
        la.n_rows = csr ? csr->n_rows : 0; la.n_cols = csr ? csr->n_cols : 0;
        la.wp = csr ? csr->wp : 0; la.wc = csr ? csr->wc : 0;
        // pack windows: index fields are w bits, code fields as short as one bit, so the windows
        // from the first code bit on are a quarter of the others; all are smaller while the launch is small
        la.pack_words = kPackWords;
        while (la.pack_words > 128 && (u64)rows * ((la.cap_words + (u64)la.pack_words - 1) / (u64)la.pack_words) < 1024) la.pack_words /= 2;
        const u64 ptr_bits = csr ? (u64)(n_blocks + n_blocks_neg) * (u64)(csr->n_rows + 1) * (u64)csr->wp : 0, ptr_words = ptr_bits / 32;
        // Row pointers have windows of their own, 256 words each and started first, where these are few (a workgroup per CU), or
        // not many (five) and a block has as many entries as pointers: then a window's walk or searches are long, and windows as long as the others'
        // made the tail of the launch.  Elsewhere the window's tables cost more than that tail.  Encode us, windows of their own / not:
        // fp32 32 x [64 x 3136] keep 0.2, 32 blocks 95 / 101, 32 x [512 x 784] 8 blocks 120 / 143, 32 blocks 128 / 151; but 32 x [256 x 196] 128 blocks
        // 96 / 91, 32 x [2048 x 49] 128 blocks 169 / 128, 8 x [401408 x 1] 584 / 365.  (At the line's foot, with as many entries as
        // pointers, [256 x 196] 32 blocks 64 / 70, [2048 x 49] 8 blocks 75 / 73.)
        const u64 ptr_wins = csr ? (u64)rows * ((ptr_words + 255) / 256) : 0;
        const bool ptr_own = csr && (ptr_wins <= 256 || (ptr_wins <= 1280 && p.k >= (int64_t)(n_blocks + n_blocks_neg) * (csr->n_rows + 1)));
        la.pack_words_ptr = std::min(la.pack_words, 256);      // at most 1026 pointers: slicer_encode_csr refuses this route to widths below eight bits
        if (csr && !ptr_own) while (la.pack_words * 32 / csr->wp + 2 > kPackPtrs) la.pack_words /= 2;
        la.pack_words_code = std::max(64, la.pack_words / 4);
        {
            // largest first word with code bits; words from there to the end
            const u64 own_words = ptr_own ? ptr_words : 0, idx_words_max = (ptr_bits + (u64)p.k * (u64)(csr ? csr->wc : p.w)) / 32 - own_words;
            la.nwin_ptr = (int)((own_words + (u64)la.pack_words_ptr - 1) / (u64)la.pack_words_ptr);
            la.nwin_idx = la.nwin_ptr + (int)((idx_words_max + (u64)la.pack_words - 1) / (u64)la.pack_words);
            const u64 code_words_max = ((u64)p.k * (u64)p.qmax + 31) / 32 + 2;
            la.nwin = la.nwin_idx + (int)((code_words_max + (u64)la.pack_words_code - 1) / (u64)la.pack_words_code);
        }
        la.tab = (uint16_t*)(ws + p.lo_tab);      la.cum = (u32*)(ws + p.lo_cum);
        la.seg = (u32*)(ws + p.lo_seg);
        la.L = (uint8_t*)(ws + p.off_kept);
        la.rowst = (u32*)(ws + p.lo_rowst);       la.thr = (u64*)(ws + p.lo_thr);
        la.vminb = (u32*)(ws + p.lo_vminb);       la.vmaxb = (u32*)(ws + p.lo_vmaxb);
        la.blk_start = (u32*)(ws + p.lo_blk_start); la.pair = (u32*)(ws + p.lo_pair);
        la.sums = (u64*)(ws + p.lo_sums);
        la.qsel = (u32*)(ws + p.lo_qsel);         la.inv_sel = (float*)(ws + p.lo_inv_sel);
        la.code_off = (u64*)(ws + p.lo_code_off);
        la.bo_idx = ea.bo_idx; la.bo_val = ea.bo_val;
        la.row_words = ea.row_words; la.slots = ea.slots;
        la.mv = ea.mv;
        la.lad = lad;
        la.guard = guard;
        la.direct = rows <= kScanRows ? 1 : 0;
        la.stream = (u32*)stream; la.meta = meta;
        la.redo = p.large_fb == kFBNarrow ? (u32*)(ws + p.off_fallback) : nullptr;
        const bool timed = g_ev_start && g_ev_stop;
        if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
        rc = dt == SLICER_F32 ? launch_large<0>(la, p.large_fb, ea, fa, st) : launch_large<1>(la, p.large_fb, ea, fa, st);
        if (rc) return rc;
        if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
        if (la.direct) return SLICER_OK;
        if (la.redo) {                              // flagged rows, spread over the chip (data with many equal values flags all of them)
            EncArgs ra = ea;
            ra.only_flagged = la.redo;
            ra.rows_per_wg = (int)((rows + 1023) / 1024);
            rc = dt == SLICER_F32 ? launch_encode<0>(ra, st) : launch_encode<1>(ra, st);
            if (rc) return rc;
        }
        done = true;
    }
    if (csr && !done) return SLICER_EINVAL;         // (callers ask for this form only where the long-row stages apply)
    if (!ea.only_flagged && !done) {
        rc = dt == SLICER_F32 ? launch_encode<0>(ea, st) : launch_encode<1>(ea, st);
        if (rc) return rc;
    }

    const u64 grid = (u64)xcd_grid((int64_t)(((u64)rows * (u64)fa.chunks_per_row + 3) / 4));     // four wavefronts per workgroup
    if (grid >= (1ull << 31)) return SLICER_EINVAL;
    if (rows <= kScanRows) {        // small batches: repair, offsets, header and gather in one launch
        if (use_small) hipLaunchKernelGGL((enc_finish_small_kernel<0, false>), dim3((unsigned)grid), dim3(kScanRows), 0, st, ea, fa);
        else if (dt == SLICER_F32) hipLaunchKernelGGL((enc_finish_small_kernel<0, true>), dim3((unsigned)grid), dim3(kScanRows), 0, st, ea, fa);
        else hipLaunchKernelGGL((enc_finish_small_kernel<1, true>), dim3((unsigned)grid), dim3(kScanRows), 0, st, ea, fa);
        hipError_t e1 = hipGetLastError();
        return e1 == hipSuccess ? SLICER_OK : hip_fail(e1);
    }
    if (use_small && rows <= kJoinRows) {
        // rows per wavefront: enough workgroups for every CU first, then fewer of them, each of which adds up all counts before its rows
        const int rpw = rows <= 4096 ? 1 : rows <= 8192 ? 2 : 4;
        const dim3 gj((unsigned)xcd_grid((rows + 8 * rpw - 1) / (8 * rpw))), bj(kJoinThreads);
        if (rpw == 1) hipLaunchKernelGGL((enc_join_kernel<1>), gj, bj, 0, st, fa);
        else if (rpw == 2) hipLaunchKernelGGL((enc_join_kernel<2>), gj, bj, 0, st, fa);
        else hipLaunchKernelGGL((enc_join_kernel<4>), gj, bj, 0, st, fa);
        hipError_t e1 = hipGetLastError();
        return e1 == hipSuccess ? SLICER_OK : hip_fail(e1);
    }
    const dim3 gscan((unsigned)((rows + kScanRows - 1) / kScanRows));
    if (use_small)
        hipLaunchKernelGGL((enc_rowscan_kernel<true>), gscan, dim3(kScanRows), 0, st, fa);
    else if (!ea.only_flagged)
        hipLaunchKernelGGL((enc_rowscan_kernel<false>), gscan, dim3(kScanRows), 0, st, fa);
    else if (dt == SLICER_F32)      // rows a fast path flagged are redone here, just before the scan of their chunk
        hipLaunchKernelGGL((enc_fix_rowscan_kernel<0>), gscan, dim3(kScanRows), 0, st, ea, fa);
    else
        hipLaunchKernelGGL((enc_fix_rowscan_kernel<1>), gscan, dim3(kScanRows), 0, st, ea, fa);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    if (use_small) hipLaunchKernelGGL((enc_gather_kernel<true>), dim3((unsigned)grid), dim3(256), 0, st, fa);
    else hipLaunchKernelGGL((enc_gather_kernel<false>), dim3((unsigned)grid), dim3(256), 0, st, fa);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    return SLICER_OK;
}

int slicer_encode(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                  int n_blocks, uint32_t bit_set, double distortion_budget, void* stream, void* meta,
                  void* workspace, void* hip_stream)
{
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, distortion_budget, none, 0,
                       stream, meta, workspace, hip_stream);
}

// Address of this device's copy of `scratch`, looked up once per device.  The array's name is a
// host-side stand-in: only the pointer hipGetSymbolAddress returns is usable as a kernel argument.
static int static_scratch(void** out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = 0;
    SLICER_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return SLICER_EINVAL;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        SLICER_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return SLICER_EHIP;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return SLICER_OK;
}

int slicer_encode_static(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                         int n_blocks, uint32_t bit_set, double distortion_budget, void* stream, void* meta,
                         void* hip_stream)
{
    int rc = check_args((int)dt, rows, row_len, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    // rows whose long-row tables do not fit the array go to the generic kernel, which needs none
    bool long_rows = true;
    if (make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set).total > (size_t)SLICER_STATIC_SCRATCH_BYTES) {
        long_rows = false;
        const Plan p = make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, true, false);
        if (p.total > (size_t)SLICER_STATIC_SCRATCH_BYTES) return SLICER_ETOOBIG;
    }
    if (!x || !stream || !meta) return SLICER_EINVAL;
    void* ws = nullptr;
    rc = static_scratch(&ws);
    if (rc) return rc;
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, distortion_budget, none, 0,
                       stream, meta, ws, hip_stream, 0.0, nullptr, long_rows);
}

int slicer_encode_pn(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                     int n_blocks, int n_blocks_neg, uint32_t bit_set, double distortion_budget, void* stream,
                     void* meta, void* workspace, void* hip_stream)
{
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks_neg, bit_set, distortion_budget, none, 0,
                       stream, meta, workspace, hip_stream);
}

static int check_csr_shape(int64_t n_rows, int64_t n_cols)
{
    if (n_rows <= 0 || n_cols <= 0 || n_cols >= ((int64_t)1 << 31) || n_rows > (((int64_t)1 << 31) - 1) / n_cols) return SLICER_EINVAL;
    return SLICER_OK;
}

// Two-dimensional instances: the long-row stages write the CSR form themselves; elsewhere the flat encode (any kernel
// family) writes its stream into the workspace and the repack kernels turn it into the CSR form.  Workspace: the flat plan's, then the flat stream, then its offsets.
struct CsrPlan {
    Plan flat;
    int wc, wp;
    u64 cap_words;          // per instance, CSR form
    size_t off_tmp, off_flat_off, total;
};

static CsrPlan make_csr_plan(int dt, int64_t instances, int64_t n_rows, int64_t n_cols, double keep_ratio, int n_blocks,
                             uint32_t bit_set)
{
    CsrPlan c;
    c.flat = make_plan(dt, instances, n_rows * n_cols, keep_ratio, n_blocks, n_blocks, bit_set);
    c.wc = index_bits(n_cols); c.wp = count_bits(c.flat.k);
    c.cap_words = ((u64)(2 * n_blocks) * (u64)(n_rows + 1) * (u64)c.wp + (u64)c.flat.k * (u64)(c.wc + c.flat.qmax) + 31) / 32;
    size_t o = align256(c.flat.total);
    c.off_tmp = o;      o = align256(o + 4 * (size_t)instances * (size_t)c.flat.cap_words + 8);   // (+ one readable word)
    c.off_flat_off = o; o = align256(o + 8 * (size_t)instances);
    c.total = o;
    return c;
}

int slicer_sizes_csr(slicer_dtype dt, int64_t instances, int64_t n_rows, int64_t n_cols, double keep_ratio, int n_blocks,
                     uint32_t bit_set, size_t* stream_capacity_bytes, size_t* meta_bytes_out, size_t* workspace_bytes)
{
    int rc = check_csr_shape(n_rows, n_cols);
    if (rc) return rc;
    rc = check_args((int)dt, instances, n_rows * n_cols, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    const CsrPlan c = make_csr_plan((int)dt, instances, n_rows, n_cols, keep_ratio, n_blocks, bit_set);
    if (stream_capacity_bytes) *stream_capacity_bytes = (size_t)(c.cap_words * 4ull * (u64)instances);
    if (meta_bytes_out) *meta_bytes_out = meta_bytes(instances, 2 * n_blocks);
    if (workspace_bytes) *workspace_bytes = c.total;
    return SLICER_OK;
}

int slicer_encode_csr(const void* x, slicer_dtype dt, int64_t instances, int64_t n_rows, int64_t n_cols, double keep_ratio,
                      int n_blocks, uint32_t bit_set, double distortion_budget, void* stream, void* meta, void* workspace,
                      void* hip_stream)
{
    int rc = check_csr_shape(n_rows, n_cols);
    if (rc) return rc;
    rc = check_args((int)dt, instances, n_rows * n_cols, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    if (!x || !stream || !meta || !workspace) return SLICER_EINVAL;
    const CsrPlan c = make_csr_plan((int)dt, instances, n_rows, n_cols, keep_ratio, n_blocks, bit_set);
    const u64 nwin = std::max<u64>(1, (c.cap_words + kCsrWin - 1) / kCsrWin);
    if ((u64)instances * nwin >= (1ull << 31)) return SLICER_EINVAL;
    char* ws = (char*)workspace;
    hipStream_t st = (hipStream_t)hip_stream;
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    // the long-row stages write the CSR form themselves
    if (c.flat.large_S && !c.flat.wg_ept && !c.flat.small_epl && instances <= kScanRows && c.wp >= 8 && ((uintptr_t)x & 15) == 0) {
        const CsrShape cs = { n_rows, n_cols, c.wp, c.wc, c.cap_words };
        return encode_impl(x, dt, instances, n_rows * n_cols, keep_ratio, n_blocks, n_blocks, bit_set, distortion_budget, none, 0,
                           stream, meta, workspace, hip_stream, 0.0, &cs);
    }
    // flat encode: kept set, blocks, ranges, bitwidths, codes, flat indices (its stream goes to the workspace)
    rc = encode_impl(x, dt, instances, n_rows * n_cols, keep_ratio, n_blocks, n_blocks, bit_set, distortion_budget, none, 0,
                     ws + c.off_tmp, meta, workspace, hip_stream);
    if (rc) return rc;
    CsrArgs ca;
    ca.R = instances; ca.n_rows = n_rows; ca.n_cols = n_cols; ca.k = c.flat.k;
    ca.M = n_blocks; ca.Mn = n_blocks; ca.w = c.flat.w; ca.wc = c.wc; ca.wp = c.wp; ca.dt = (int)dt;
    ca.bit_set = bit_set;
    ca.nwin = (int)nwin;
    ca.flat = (const u32*)(ws + c.off_tmp);
    ca.flat_off = (u64*)(ws + c.off_flat_off);
    ca.row_words = (u64*)(ws + c.flat.off_row_words);
    ca.row_off_local = (const u64*)(ws + c.flat.off_row_local);
    ca.chunk_tot = (const u64*)(ws + c.flat.off_chunk_tot);
    ca.stream = (u32*)stream; ca.meta = meta;
    ca.mv = meta_view(meta, instances, 2 * n_blocks);
    hipLaunchKernelGGL(csr_sizes_kernel, dim3((unsigned)((instances + 255) / 256)), dim3(256), 0, st, ca);
    FinishArgs fa;                                           // the row-offset scan, now over the CSR segment lengths
    fa.R = instances; fa.N = n_rows * n_cols; fa.k = c.flat.k;
    fa.M = n_blocks; fa.Mn = n_blocks; fa.w = c.flat.w; fa.dt = (int)dt; fa.bit_set = bit_set;
    fa.row_words = ca.row_words;
    fa.row_off_local = (u64*)(ws + c.flat.off_row_local);
    fa.chunk_tot = (u64*)(ws + c.flat.off_chunk_tot);
    fa.row_words32 = nullptr; fa.slots = nullptr; fa.cap_words = c.cap_words; fa.chunks_per_row = 1;
    fa.stream = (u32*)stream; fa.meta = meta; fa.mv = ca.mv;
    hipLaunchKernelGGL((enc_rowscan_kernel<false>), dim3((unsigned)((instances + kScanRows - 1) / kScanRows)), dim3(kScanRows), 0, st, fa);
    hipLaunchKernelGGL(csr_repack_kernel, dim3((unsigned)((u64)instances * nwin)), dim3(256), 0, st, ca);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SLICER_OK : hip_fail(e);
}

static int launch_decode_csr(const void* stream, const void* meta, void* y, int dt, int64_t instances, int64_t n_rows,
                             int64_t n_cols, int n_blocks, int n_blocks_neg, hipStream_t st)
{
    DecCsrArgs da;
    da.stream = (const u32*)stream; da.y = y;
    da.R = instances; da.n_rows = n_rows; da.n_cols = n_cols;
    da.M = n_blocks; da.Mn = n_blocks_neg; da.wc = index_bits(n_cols);
    da.mv = meta_view(const_cast<void*>(meta), instances, n_blocks + n_blocks_neg);
    da.k_keep = (const u64*)meta + 4;
    // several short tensor rows per workgroup, as long as about a thousand workgroups remain
    da.rows_per_wg = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(kCsrRows, instances * n_rows / 1024), kCsrImage / n_cols));
    da.image = (int)std::min<int64_t>(kCsrImage, da.rows_per_wg * n_cols);
    da.groups = (n_rows + da.rows_per_wg - 1) / da.rows_per_wg;
    const u64 grid = (u64)xcd_grid(instances * da.groups);
    if ((u64)instances * (u64)da.groups >= (1ull << 31) || grid >= (1ull << 31)) return SLICER_EINVAL;
    const bool timed = g_ev_start && g_ev_stop;
    if (timed) SLICER_HIP(hipEventRecord(g_ev_start, st));
    const size_t lds = dec_csr_lds_bytes(dt == SLICER_F32 ? 4 : 2, da.image, n_blocks + n_blocks_neg, da.rows_per_wg);
    if (dt == SLICER_F32) hipLaunchKernelGGL((dec_csr_kernel<0>), dim3((unsigned)grid), dim3(kCsrThreads), lds, st, da);
    else hipLaunchKernelGGL((dec_csr_kernel<1>), dim3((unsigned)grid), dim3(kCsrThreads), lds, st, da);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    if (timed) SLICER_HIP(hipEventRecord(g_ev_stop, st));
    return SLICER_OK;
}

int slicer_decode_as_csr(const void* stream, const void* meta, void* y, slicer_dtype dt, int64_t instances, int64_t n_rows,
                         int64_t n_cols, int n_blocks, void* hip_stream)
{
    int rc = check_csr_shape(n_rows, n_cols);
    if (rc) return rc;
    rc = check_shape((int)dt, instances, n_rows * n_cols, n_blocks);
    if (rc) return rc;
    if (!stream || !meta || !y) return SLICER_EINVAL;
    return launch_decode_csr(stream, meta, y, (int)dt, instances, n_rows, n_cols, n_blocks, n_blocks, (hipStream_t)hip_stream);
}

int slicer_encode_atkf(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio, double lambda,
                       int n_blocks, int n_blocks_neg, uint32_t bit_set, double distortion_budget, void* stream,
                       void* meta, void* workspace, void* hip_stream)
{
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks_neg, bit_set, distortion_budget, none, 0,
                       stream, meta, workspace, hip_stream, lambda);
}

int slicer_encode_ds(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                     int n_blocks, uint32_t bit_set, double delta, void* stream, void* meta, void* workspace,
                     void* hip_stream)
{
    Ladder none;
    none.on = 0;
    for (int j = 0; j < kMaxBlocks / 8; ++j) none.nib[j] = 0;
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, delta, none, 1,
                       stream, meta, workspace, hip_stream);
}

uint32_t slicer_ladder_bit_set(const uint8_t* ladder, int n_blocks)
{
    if (!ladder || n_blocks < 1 || n_blocks > kMaxBlocks) return 0;
    uint32_t bs = 0;
    for (int m = 0; m < n_blocks; ++m) {
        if (ladder[m] < 1 || ladder[m] > 16) return 0;
        bs |= 1u << ladder[m];
    }
    return bs;
}

int slicer_encode_ladder(const void* x, slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio,
                         int n_blocks, const uint8_t* ladder, void* stream, void* meta, void* workspace,
                         void* hip_stream)
{
    const uint32_t bit_set = slicer_ladder_bit_set(ladder, n_blocks);
    if (!bit_set) return SLICER_EINVAL;
    Ladder lad;
    lad.on = 1;
    for (int j = 0; j < kMaxBlocks / 8; ++j) lad.nib[j] = 0;
    for (int m = 0; m < n_blocks; ++m) {
        uint32_t t = 0;                                  // position of ladder[m] among the set's bitwidths, ascending
        for (int q = 1; q < ladder[m]; ++q) t += (bit_set >> q) & 1u;
        lad.nib[m >> 3] |= t << ((m & 7) * 4);
    }
    return encode_impl(x, dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set, 0.0, lad, 0, stream, meta, workspace,
                       hip_stream);
}

int slicer_bound(slicer_dtype dt, int64_t rows, int64_t row_len, double keep_ratio, int n_blocks,
                 uint32_t bit_set, uint64_t* value_bits, uint64_t* index_bits_out, uint64_t* header_bits)
{
    int rc = check_args((int)dt, rows, row_len, keep_ratio, n_blocks, bit_set);
    if (rc) return rc;
    const Plan p = make_plan((int)dt, rows, row_len, keep_ratio, n_blocks, n_blocks, bit_set);
    const u64 R = (u64)rows, k = (u64)p.k;
    if (value_bits) *value_bits = R * k * (u64)p.qmax;
    if (index_bits_out) *index_bits_out = R * k * (u64)p.w;
    if (header_bits) *header_bits = 8ull * (u64)meta_bytes(rows, 2 * n_blocks) + R * (32ull * p.cap_words - k * (u64)(p.w + p.qmax));
    return SLICER_OK;
}

int slicer_decode_as_pn(const void* stream, const void* meta, void* y, slicer_dtype dt, int64_t rows,
                        int64_t row_len, int n_blocks, int n_blocks_neg, void* hip_stream)
{
    int rc = check_shape((int)dt, rows, row_len, n_blocks);
    if (rc) return rc;
    if (n_blocks_neg < 1 || n_blocks_neg > SLICER_MAX_BLOCKS) return SLICER_EINVAL;
    if (!stream || !meta || !y) return SLICER_EINVAL;
    return launch_decode(stream, meta, y, (int)dt, rows, row_len, n_blocks, n_blocks_neg, (hipStream_t)hip_stream);
}

int slicer_decode_as(const void* stream, const void* meta, void* y, slicer_dtype dt, int64_t rows,
                     int64_t row_len, int n_blocks, void* hip_stream)
{
    return slicer_decode_as_pn(stream, meta, y, dt, rows, row_len, n_blocks, n_blocks, hip_stream);
}

// Copies of a header on their way to the host: a slot of page-locked memory that a one-wavefront kernel fills, word by word
// and then the ticket, while the caller polls the ticket.  A copy into the caller's memory and a wait for the stream took 18 us
// (decode of fp32 [1 x 200704] 26.6 us in all, 12.5 now).  32 calls can be under way at once, on any threads, streams and GPUs; one more, a
// stream under capture, and a system that gives no page-locked memory take the copy and the wait.
struct HeaderSlot { u32 words[kHeaderBytes / 4]; u32 ticket; u32 pad[15]; };
constexpr int kHeaderSlots = 32;

static __global__ __launch_bounds__(kWave) void header_copy_kernel(const u32* meta, HeaderSlot* slot, u32 ticket)
{
    if (threadIdx.x < kHeaderBytes / 4)
        __hip_atomic_store(&slot->words[threadIdx.x], meta[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();                          // (one wavefront: waits for the words of all its lanes)
    if (threadIdx.x == 0) __hip_atomic_store(&slot->ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

static HeaderSlot* header_slots()                    // allocated once, 4 KB, kept until the process ends
{
    static std::once_flag once;
    static HeaderSlot* slots = nullptr;
    std::call_once(once, [] {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;      // (another thread may be capturing)
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        void* p = nullptr;
        if (hipHostMalloc(&p, sizeof(HeaderSlot) * kHeaderSlots, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) {
            memset(p, 0, sizeof(HeaderSlot) * kHeaderSlots);
            slots = (HeaderSlot*)p;
        } else {
            (void)hipGetLastError();
        }
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    });
    return slots;
}

static int check_header(const uint32_t* h32) { return h32[0] == kMagic && h32[1] == kVersion ? SLICER_OK : SLICER_EFORMAT; }

static int read_header(const void* meta, hipStream_t st, uint32_t* h32)
{
    SLICER_HIP(hipMemcpyAsync(h32, meta, kHeaderBytes, hipMemcpyDeviceToHost, st));
    SLICER_HIP(hipStreamSynchronize(st));
    return check_header(h32);
}

// For slicer_decode alone: its own kernels read meta on the same stream right after.  slicer_stream_words keeps the copy: it
// serves any meta that a copy can reach, also that of another GPU.
static int poll_header(const void* meta, hipStream_t st, uint32_t* h32)
{
    static std::atomic<u32> busy[kHeaderSlots];
    static u32 tickets[kHeaderSlots];                // of the slot's last call; touched only while the slot is held
    // An error that some earlier call of this thread left would be taken for one of the launch below: the copy leaves it to be
    // reported where the decode kernel is launched.
    if (hipPeekAtLastError() != hipSuccess) return read_header(meta, st, h32);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    HeaderSlot* slots = nullptr;
    if (hipStreamIsCapturing(st, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone) slots = header_slots();
    int s = slots ? 0 : kHeaderSlots;
    for (; s < kHeaderSlots; ++s) {
        u32 idle = 0;
        if (busy[s].compare_exchange_strong(idle, 1u, std::memory_order_acquire)) break;
    }
    if (s == kHeaderSlots) return read_header(meta, st, h32);
    HeaderSlot* slot = slots + s;
    const u32 ticket = ++tickets[s];
    hipLaunchKernelGGL(header_copy_kernel, dim3(1), dim3(kWave), 0, st, (const u32*)meta, slot, ticket);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {                           // nothing was launched that could write to the slot
        busy[s].store(0u, std::memory_order_release);
        return hip_fail(e);
    }
    const auto t0 = std::chrono::steady_clock::now();
    bool there = false;
    for (u32 i = 0; !there; ++i) {
        there = __atomic_load_n(&slot->ticket, __ATOMIC_ACQUIRE) == ticket;
        if (!there && (i & 255u) == 255u && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(1)) break;
    }
    if (!there) {                                    // much work before it, or an error: wait in the ordinary way
        e = hipStreamSynchronize(st);
        there = __atomic_load_n(&slot->ticket, __ATOMIC_ACQUIRE) == ticket;
        // a copy that has not come may still be under way: its slot is not used again
        if (e != hipSuccess || !there) {
            if (there) busy[s].store(0u, std::memory_order_release);
            return hip_fail(e != hipSuccess ? e : hipErrorUnknown);
        }
    }
    memcpy(h32, slot->words, kHeaderBytes);
    busy[s].store(0u, std::memory_order_release);
    return check_header(h32);
}

int slicer_decode(const void* stream, const void* meta, void* y, void* hip_stream)
{
    if (!stream || !meta || !y) return SLICER_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    alignas(8) uint32_t h32[kHeaderBytes / 4];
    int rc = poll_header(meta, st, h32);
    if (rc) return rc;
    const uint64_t* h64 = (const uint64_t*)h32;
    const int dt = (int)h32[2], M = (int)h32[3];
    const int64_t rows = (int64_t)h64[2], row_len = (int64_t)h64[3];
    const int Mn = h32[14] ? (int)h32[14] : M;           // 0: the negative class has M blocks too
    rc = check_shape(dt, rows, row_len, M);
    if (rc || Mn < 1 || Mn > SLICER_MAX_BLOCKS) return SLICER_EFORMAT;
    if (h32[15]) {                                        // two-dimensional instances: blocks stored as CSR triples
        const int64_t n_cols = (int64_t)h32[15];
        if (row_len % n_cols || (int)h32[11] != index_bits(n_cols)) return SLICER_EFORMAT;
        return launch_decode_csr(stream, meta, y, dt, rows, row_len / n_cols, n_cols, M, Mn, st);
    }
    if ((int)h32[11] != index_bits(row_len)) return SLICER_EFORMAT;
    return launch_decode(stream, meta, y, dt, rows, row_len, M, Mn, st);
}

int slicer_stream_words(const void* meta, uint64_t* words, void* hip_stream)
{
    if (!meta || !words) return SLICER_EINVAL;
    alignas(8) uint32_t h32[kHeaderBytes / 4];
    int rc = read_header(meta, (hipStream_t)hip_stream, h32);
    if (rc) return rc;
    *words = ((const uint64_t*)h32)[6];
    return SLICER_OK;
}

int slicer_check(const void* meta, uint64_t stream_words, slicer_dtype dt, int64_t rows, int64_t row_len,
                 int n_blocks, void* scratch, void* hip_stream)
{
    return slicer_check_pn(meta, stream_words, dt, rows, row_len, n_blocks, n_blocks, scratch, hip_stream);
}

static int check_impl(const void* meta, uint64_t stream_words, slicer_dtype dt, int64_t rows, int64_t row_len,
                      int n_blocks, int n_blocks_neg, int64_t csr_cols, void* scratch, void* hip_stream);

int slicer_check_pn(const void* meta, uint64_t stream_words, slicer_dtype dt, int64_t rows, int64_t row_len,
                    int n_blocks, int n_blocks_neg, void* scratch, void* hip_stream)
{
    return check_impl(meta, stream_words, dt, rows, row_len, n_blocks, n_blocks_neg, 0, scratch, hip_stream);
}

int slicer_check_csr(const void* meta, uint64_t stream_words, slicer_dtype dt, int64_t instances, int64_t n_rows,
                     int64_t n_cols, int n_blocks, void* scratch, void* hip_stream)
{
    int rc = check_csr_shape(n_rows, n_cols);
    if (rc) return rc;
    return check_impl(meta, stream_words, dt, instances, n_rows * n_cols, n_blocks, n_blocks, n_cols, scratch, hip_stream);
}

static int check_impl(const void* meta, uint64_t stream_words, slicer_dtype dt, int64_t rows, int64_t row_len,
                      int n_blocks, int n_blocks_neg, int64_t csr_cols, void* scratch, void* hip_stream)
{
    int rc = check_shape((int)dt, rows, row_len, n_blocks);
    if (rc) return rc;
    if (n_blocks_neg < 1 || n_blocks_neg > SLICER_MAX_BLOCKS) return SLICER_EINVAL;
    if (!meta || !scratch) return SLICER_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    CheckArgs ca;
    ca.meta = meta; ca.R = rows; ca.N = row_len; ca.M = n_blocks; ca.Mn = n_blocks_neg; ca.dt = (int)dt;
    ca.csr_cols = csr_cols;
    ca.w = csr_cols > 0 ? index_bits(csr_cols) : index_bits(row_len);
    ca.avail_words = stream_words;
    ca.flag = (u32*)scratch;
    hipLaunchKernelGGL(meta_flag_clear_kernel, dim3(1), dim3(64), 0, st, ca.flag);
    hipLaunchKernelGGL(meta_check_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st, ca);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    u32 flag = 0;
    SLICER_HIP(hipMemcpyAsync(&flag, scratch, 4, hipMemcpyDeviceToHost, st));
    SLICER_HIP(hipStreamSynchronize(st));
    return flag ? SLICER_EFORMAT : SLICER_OK;
}

int slicer_profile_events(void* start_event, void* stop_event)
{
    if ((start_event == nullptr) != (stop_event == nullptr)) return SLICER_EINVAL;
    g_ev_start = (hipEvent_t)start_event;
    g_ev_stop = (hipEvent_t)stop_event;
    return SLICER_OK;
}

int slicer_last_hip_error(void) { return g_last_hip_error; }

const char* slicer_strerror(int code)
{
    switch (code) {
        case SLICER_OK: return "ok";
        case SLICER_EINVAL: return "invalid argument";
        case SLICER_EUNSUPPORTED: return "unsupported dtype";
        case SLICER_EHIP: return "HIP call failed (see slicer_last_hip_error)";
        case SLICER_EFORMAT: return "meta header is not a version-1 SLICER header";
        case SLICER_ETOOBIG: return "shape needs more scratch than the library's static buffer holds";
        default: return "unknown error";
    }
}

}  // extern "C"
