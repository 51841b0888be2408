// Host check of the row kernel's reads of block-ordered values (S, cap + 4 words of LDS): walks the sums' and the energy's loops as
// the kernel's lanes do and looks at every address; and how many rows a CU's LDS holds.  Prints the number of layouts looked at; ends with 1 at the first bad read.
#include <cmath>
#include <cstdio>

#include "../paper_2511_11608_amd/csrc/slicer_encode_small.hpp"

using namespace slicer;

static int bad(const char* what, int cap, int n_pos, int n_neg, int M, int Mn, int nq, u32 lane, u32 at)
{
    printf("%s: cap %d, %d + %d entries, %d + %d blocks, %d bitwidths, lane %u reads %u..%u of %d words\n", what, cap, n_pos, n_neg, M, Mn, nq, lane, at,
           at + 3, cap + 4);
    return 1;
}

static int check(int k, int cap, int n_pos, int n_neg, int M, int Mn, int nq)
{
    SmallArgs a = {};
    a.k = k; a.M = M; a.Mn = Mn; a.nq = nq;
    small_split_lanes(a);
    const int B2 = M + Mn, n = n_pos + n_neg;
    const u32 K0 = n_pos / M, K1 = n_neg / Mn, lpb = a.lpb, es = a.es, cl = a.cl;
    const u32 mc0 = n_pos - K0 * (M - 1), mc1 = n_neg - K1 * (Mn - 1), maxb = mc0 > mc1 ? mc0 : mc1;
    const u32 T = (maxb + lpb - 1) / lpb, T2 = es > 1 ? (maxb + es - 1) / es : maxb;
    const u32 l0 = K0 ? K0 : n_pos ? n_pos : ~0u, l1 = K1 ? K1 : n_neg ? n_neg : ~0u;
    const u32 least = es > 1 ? 0u : l0 < l1 ? l0 : l1;
    for (u32 lane = 0; lane < kWave; ++lane) {
        const u32 myb = lane / lpb, sub = lane - myb * lpb;
        const bool on = myb < (u32)B2;
        const bool neg = myb >= (u32)M;
        const u32 m = neg ? myb - M : myb, K = neg ? K1 : K0, Ms = neg ? Mn : M, nc = neg ? n_neg : n_pos;
        const u32 bs0 = on ? (neg ? n_pos : 0) + m * K : 0u, cnt = on ? (m < Ms - 1 ? K : nc - m * K) : 0u;
        // energy: the block's entries dealt to its lanes
        const u32 perb = (cnt + lpb - 1) / lpb, be = bs0 + cnt, r0 = on ? (bs0 + sub * perb < be ? bs0 + sub * perb : be) : 0u, r1 = r0 + perb < be ? r0 + perb : be;
        for (u32 i = 0; i < T; i += 4) {
            const u32 at = small_group_at(r0 + i, cap);
            if (at + 3 >= (u32)cap + 4 || (r0 + i < r1 && at != r0 + i)) return bad("energy", cap, n_pos, n_neg, M, Mn, nq, lane, at);
        }
        // sums
        const u32 ct = es > 1 ? sub % cl : sub, sl = es > 1 ? sub / cl : 0u;
        const bool active = on && ct < cl && sl < es;
        const AbqSlice s = small_abq_slice(bs0, cnt, es > 1 ? (cnt + es - 1) / es : cnt, sl, active);
        if (s.qn && s.q0 + s.qn > (u32)n) return bad("slice", cap, n_pos, n_neg, M, Mn, nq, lane, s.q0);
        for (u32 i = 0; i < T2; i += 8) {
            const bool whole = i + 8 <= least;
            for (u32 g = i; g < i + 8 && (g == i || whole || g < T2); g += 4) {
                const u32 at = whole ? s.q0 + g : small_group_at(s.q0 + g, cap);
                if (at + 3 >= (u32)cap + 4 || (g < s.qn && at != s.q0 + g)) return bad("sums", cap, n_pos, n_neg, M, Mn, nq, lane, at);
            }
        }
    }
    return 0;
}

// fp32 rows of 4096 elements whose LDS decides how many of them a CU holds (160 KB, dealt in units of 1280 bytes); the list positions,
// the sums and the scales lie inside region 0
static int check_lds(int k, int cap, int maxs, int M, int nq, int qmax, int per_cu)
{
    const int B2 = 2 * M;
    const u64 cap_words = ((u64)k * (u64)(12 + qmax) + 31) / 32;
    const int region0 = small_region0_words(0, k, cap_words, B2, nq, cap, small_fine_bins(maxs)), words = small_lds_words(0, cap, region0, B2, maxs);
    const int held = 160 * 1024 / ((4 * words + 1279) / 1280 * 1280);
    const int sums = (((k + 1) / 2 + (int)cap_words) + 1) & ~1;
    if (held >= per_cu && small_fine_bins(maxs) + 4 + (cap + 4) / 2 <= region0 && sums + 2 * B2 * small_block_sums(B2, nq) + B2 * nq <= region0) return 0;
    printf("%d of 4096, %d + %d blocks, %d bitwidths: %d words, region 0 %d, %d rows a CU, not %d\n", k, M, M, nq, words, region0, held, per_cu);
    return 1;
}

int main()
{
    if (check_lds(1024, 1280, 20, 16, 16, 16, 8) || check_lds(1228, 1536, 0, 16, 7, 8, 6) || check_lds(1228, 1536, 0, 1, 7, 8, 7) ||
        check_lds(1024, 1280, 20, 16, 7, 8, 10)) return 1;
    long seen = 0;
    const int ks[] = { 1, 2, 63, 115, 204, 409, 512, 819, 1024, 1500, 1856, 1920 };
    const int blocks[] = { 1, 2, 3, 4, 5, 8, 11, 16, 31, 32 };
    const int nqs[] = { 1, 2, 3, 4, 7, 9, 16 };
    for (int k : ks)
        for (int margin : { 64, 128, 512 }) {
            const int up = (k + margin + 63) / 64 * 64, cap = up < 1984 ? up : 1984;      // as the plan's list capacity
            if (k + 64 > cap) continue;
            for (int M : blocks)
                for (int Mn : blocks)
                    for (int nq : nqs)
                        for (int n : { 1, k / 3 + 1, k - 1, k })
                            for (int n_neg : { 0, 1, n / 2, n - 1, n }) {
                                if (n <= 0 || n > k || n_neg < 0 || n_neg > n) continue;
                                if (check(k, cap, n - n_neg, n_neg, M, Mn, nq)) return 1;
                                ++seen;
                            }
        }
    printf("%ld layouts\n", seen);
    return 0;
}
