// Neighbor-list build, list-based energy/gradient sweep and FP64 verify.
//
// One workgroup per instance throughout: an instance (n <= 1024 circles,
// 8 KB of positions) is staged in LDS once and every access after that is
// on chip.
#include "pecc_device.hpp"
#include "pecc_launch.hpp"
#include "pecc_lbfgs.hpp"

#include <type_traits>

namespace pecc {

constexpr int kBuildBlock = 256;

// Positions of one instance into LDS (coalesced float2 loads).
template <int BLOCK>
__device__ __forceinline__ void stage_positions(const float *xy, int off, int n, float2 *pos)
{
    const float2 *src = reinterpret_cast<const float2 *>(xy) + off;
    for (int i = threadIdx.x; i < n; i += BLOCK) pos[i] = src[i];
}

// Circle range of instance b.  False when the offsets are not a valid
// range inside [0, total_n] or the instance has more than kMaxN circles.
__device__ __forceinline__ bool instance_range(const int32_t *offset, int b, int64_t total_n,
                                               int *off, int *n)
{
    const int a = offset[b], e = offset[b + 1];
    *off = a;
    *n = e - a;
    return a >= 0 && e >= a && (int64_t)e <= total_n && e - a <= kMaxN;
}

// True when circles off .. off+n-1 may be written for an invalid instance.
__device__ __forceinline__ bool writable_range(int off, int n, int64_t total_n)
{
    return off >= 0 && n > 0 && (int64_t)off + n <= total_n;
}

// ---------------------------------------------------------------------------
// Neighbor lists (CSR, rows ascending).  One launch over the instances: a
// workgroup sorts its circles into cells, finds every circle's neighbors,
// and needs the number of entries of all instances before it to know where
// its own go.  It takes its instance by a ticket, publishes its count, and
// looks back over the counts of the earlier instances until one that already
// knows its prefix (all of them were taken by workgroups that run or have
// ended, and none waits for a later one, so every wait ends).
//
// Bound by vector issue: 9 cells of candidates per circle.  A thread takes
// the circles of sorted slots tid + 256 u, so that a wave's circles are
// neighbors in space and their runs have similar lengths; the candidates
// cost an FP32 distance and a mask bit (neighbor_masks); the neighbors of two
// circles are collected in one set of registers as 16-bit halves and sorted
// by a network (packed 16-bit minimum and maximum), 8, 12 or 16 entries (at
// packing density and the packing cutoff of 2.3 a row has 4 to 8, rarely 16).
// Longer rows, and those of circles with more candidates than a mask holds (32
// in a cell row, 64 in all), are written from bits in LDS, half a wave per row:
// 32 words hold the circles of an instance in ascending order.  They stand
// behind branches that are taken for the wave and laid out of the way: code in
// the path of the short rows costs its instruction fetches, 9 us of the first
// workgroups' 27.  The instance's segment is staged in LDS and stored in order
// (stores of 8 bytes), as is the row table.
// One pass instead of a count pass, a one-workgroup scan and a fill pass that
// sorted rows in global memory: 4096 x n = 1000 at cutoff 2.3 in 112 us (442 us
// before), at cutoff 4 in 317 us (1656 us, and 1723 us while long rows were
// taken candidate by candidate by their threads), at cutoff 4 in cells of 8 in
// 884 us (2074, 3790), at cutoff 8 in 0.98 ms (19.5, 21.3); of the 112 about 85
// are vector issue, and about 14 the tickets of the first generation, all on
// one word.  Looks
// back of 256 or 1024 words per turn were slower (172 and 193 us with the
// energy against 168): words read while they are about to be written.
// ---------------------------------------------------------------------------
constexpr int kBuildCpt = kMaxN / kBuildBlock;
constexpr int kBuildNc = 32;            // cells per axis at most
constexpr int kRowRegs = 16;            // neighbors of a row sorted in registers
constexpr int kStage = 6144;            // entries of an instance staged in LDS
// A state word: an instance's count or prefix under its flag.  Word 0 counts
// the tickets as well, above the 20 bits that the first instance's count takes.
constexpr unsigned long long kHasCount = 1ull << 62, kHasPrefix = 2ull << 62;
constexpr int kTicketShift = 24;
static_assert(kMaxN * (kMaxN - 1) < (1 << kTicketShift), "count of one instance");

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Ascending sort of two sets of 16-bit keys (the halves of a[0 .. N)) by
// Batcher's odd-even merge network.
template <int N>
__device__ __forceinline__ void sort_pairs(u16x2 (&a)[kRowRegs])
{
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j <= N - 1 - k; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const u16x2 u = a[i + j], v = a[i + j + k];
                        a[i + j] = __builtin_elementwise_min(u, v);
                        a[i + j + k] = __builtin_elementwise_max(u, v);
                    }
}

// State words of a build, cleared.  The last instance's word is nobody's to
// read and is left out (see launch_build), except where it is the only one.
__device__ __host__ __forceinline__ int state_words(int B) { return B > 1 ? B - 1 : 1; }

__global__ __launch_bounds__(kBuildBlock) void build_clear_kernel(unsigned long long *state, int B)
{
    const int64_t i = (int64_t)blockIdx.x * kBuildBlock + threadIdx.x;
    if (i < state_words(B)) state[i] = 0ull;
}

template <int FORMAT>
__global__ __launch_bounds__(kBuildBlock, 5) void build_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ R,
    const float *__restrict__ xy, int B, int64_t total_n, double c2, float h_req,
    int32_t *__restrict__ row, void *__restrict__ col_v, int64_t capacity,
    int64_t *num_pairs, unsigned long long *state)
{
    constexpr bool kLocal = FORMAT == kListLocal16, kHalf = FORMAT == kListHalf;
    using Idx = std::conditional_t<kLocal, uint16_t, int32_t>;
    Idx *__restrict__ col = static_cast<Idx *>(col_v);
    __shared__ int cell_start[kBuildNc * kBuildNc + 1];
    __shared__ uint16_t cell_circ[kMaxN];
    __shared__ int scan_tmp[kBuildBlock / kWave];
    __shared__ int start_s[kMaxN];              // row lengths, then row starts, by circle
    __shared__ unsigned bits_s[kBuildBlock];    // per wave: two rows as bits
    // positions in cell order and the sort's scratch, then the staged segment
    __shared__ union {
        struct {
            float2 psort[kMaxN + 8];
            uint16_t slot_tmp[kMaxN];
        };
        uint16_t stage[kStage];
    } sh;
    float2 *const psort = sh.psort;
    uint16_t *const stage = sh.stage;
    __shared__ int inst_s;
    __shared__ long long base_s;

    const int tid = threadIdx.x;
    if (tid == 0)
        inst_s = (int)((atomicAdd(&state[0], 1ull << kTicketShift) & ~(3ull << 62)) >> kTicketShift);
    __syncthreads();
    const int b = inst_s;
    int off, n;
    const bool valid = instance_range(offset, b, total_n, &off, &n);
    const int nn = valid ? n : 0;               // circles to list (an invalid instance has empty rows)

    float2 x[kBuildCpt];
#pragma unroll
    for (int u = 0; u < kBuildCpt; ++u) {
        const int i = tid + u * kBuildBlock;
        x[u] = i < nn ? reinterpret_cast<const float2 *>(xy)[off + i] : make_float2(0.f, 0.f);
        // NaN is no neighbor of anything, and neither is infinity
        if (x[u].x != x[u].x) x[u].x = HUGE_VALF;
        if (x[u].y != x[u].y) x[u].y = HUGE_VALF;
        start_s[i] = 0;
    }
    const Grid g = make_grid<kBuildNc>(R[b], h_req);
    {
        int own[kBuildCpt];
        sort_cells<kBuildBlock, kBuildCpt>(tid, x, nn, g, cell_start, cell_circ, sh.slot_tmp, psort,
                                           scan_tmp, own);
    }
    // The long rows (bit u of `slow`): more neighbors than a row's registers, or
    // runs too long for a mask.  Half a wave takes one, 32 candidates a turn.
    // at(slot, circle) gives a position; f(i, on, turns) is called by the wave
    // with each half's circle (on: there is one), and turns(v) calls v(has, j)
    // with every candidate.
    unsigned slow = 0, far = 0;                 // far: runs too long for a mask
    const int lane = tid & (kWave - 1);
    const float c2f = (float)c2, band = c2f * 1e-6f + 1e-30f;
    auto long_rows = [&](auto &&at, auto &&f) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(slow != 0) == 0, 1)) return;
#pragma unroll 1
        for (int u = 0; u < kBuildCpt; ++u) {
            unsigned long long left = __builtin_amdgcn_ballot_w64((slow >> u & 1) != 0);
            while (left) {
                const int l0 = __builtin_ctzll(left);
                left &= left - 1;
                const bool two = left != 0;
                const int l1 = two ? __builtin_ctzll(left) : l0;
                left &= left - 1;
                const bool on = lane < 32 || two;
                const int s = tid - lane + u * kBuildBlock + (lane < 32 ? l0 : l1);
                const int i = cell_circ[s];
                const float2 q = at(s, i);
                int ra[3], rl[3], self;
                cell_rows(q, on, s, g, cell_start, ra, rl, self);
                const int n0 = rl[0], n1 = n0 + rl[1], all = n1 + rl[2];
                const int longest = max(__builtin_amdgcn_readlane(all, 0), __builtin_amdgcn_readlane(all, 32));
                f(i, on, [&](auto &&v) {
                    for (int k0 = 0; k0 < longest; k0 += 32) {
                        const int k = k0 + (lane & 31);
                        const bool in = k < all;
                        const int t = in ? k + (k < n0 ? ra[0] : k < n1 ? ra[1] - n0 : ra[2] - n1) : s;
                        const int j = cell_circ[t];
                        // (as neighbor_masks: the FP64 predicate within the band)
                        const float2 p = at(t, j);
                        const float dx = q.x - p.x, dy = q.y - p.y;
                        const float d = fmaf(dx, dx, fmaf(dy, dy, -c2f));
                        bool has = d < 0.f;
                        if (__builtin_amdgcn_ballot_w64(!(fabsf(d) > band))) has = near64(q, p, c2);
                        v(in && t != s && has, j);
                    }
                });
            }
        }
    };
    auto at_slot = [&](int s, int) { return psort[s]; };
    // A thread's circle with runs too long for a mask: f(w, first) gets 32
    // candidates at a time, bit b of w for a neighbor at slot first + b.
    auto wide_words = [&](float2 q, bool on, int own, auto &&f) {
        const int cx = cell_coord(q.x, g), cy = cell_coord(q.y, g);
        const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx < g.nc - 1 ? cx + 1 : cx;
#pragma unroll 1
        for (int r = -1; r <= 1; ++r) {
            const int y = cy + r;
            const bool row = on && y >= 0 && y < g.nc;
            int first = row ? cell_start[y * g.nc + x0] : 0;
            int len = row ? cell_start[y * g.nc + x1 + 1] - first : 0;
            const int longest = wave_max_dpp(max(len, 0));
            constexpr int kTurn = 4;
#pragma unroll 1
            for (int k0 = 0; k0 < longest; k0 += 32, first += 32, len -= 32) {
                unsigned w;
                float dmin = 3.0e38f;
                auto scan = [&](auto exact) {
                    w = 0;
                    // downwards, so that the bit shifted in last is the first candidate
#pragma unroll 1
                    for (int k = min(32, (longest - k0 + kTurn - 1) / kTurn * kTurn) - kTurn; k >= 0; k -= kTurn) {
                        float2 c[kTurn];
                        const float2 *src = psort + min(first + k, kMaxN);
#pragma unroll
                        for (int v = 0; v < kTurn; ++v) c[v] = src[v];
#pragma unroll
                        for (int v = kTurn - 1; v >= 0; --v) {
                            if constexpr (decltype(exact)::value) {
                                w = w << 1 | (near64(q, c[v], c2) ? 1u : 0u);
                            } else {
                                const float dx = q.x - c[v].x, dy = q.y - c[v].y;
                                const float t = fmaf(dx, dx, fmaf(dy, dy, -c2f));
                                w = __builtin_amdgcn_alignbit(w, __float_as_uint(t), 31);
                                dmin = fminf(dmin, fabsf(t));
                            }
                        }
                    }
                };
                scan(std::false_type{});
                if (__builtin_amdgcn_ballot_w64(dmin <= band)) scan(std::true_type{});
                w &= len >= 32 ? ~0u : len > 0 ? (1u << len) - 1u : 0u;
                const unsigned place = (unsigned)(own - first);
                if (place < 32u) w &= ~(1u << place);
                f(w, first);
            }
        }
    };
    // ---- neighbor masks of the circles of slots tid + 256 u, two at a time ---
    unsigned long long mask[kBuildCpt];
    unsigned firsts[kBuildCpt], lens[kBuildCpt];        // the three runs, 10 bits each (a first slot of 1024 is an empty run, and so are those after it)
    int ci[kBuildCpt], mine = 0;
#pragma unroll
    for (int h = 0; h < kBuildCpt / 2; ++h) {
        float2 q[2];
        bool on[2], fits[2];
        int ra[2][3], rl[2][3], self[2], kmax[3] = {0, 0, 0};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int s = tid + (2 * h + e) * kBuildBlock;
            on[e] = s < nn;
            q[e] = psort[on[e] ? s : 0];
            ci[2 * h + e] = cell_circ[on[e] ? s : 0];
            cell_rows(q[e], on[e], s, g, cell_start, ra[e], rl[e], self[e]);
            // infinity has no neighbors: its runs are emptied
            if (!(fabsf(q[e].x) < HUGE_VALF && fabsf(q[e].y) < HUGE_VALF)) {
#pragma unroll
                for (int r = 0; r < 3; ++r) rl[e][r] = 0;
                on[e] = false;
            }
            fits[e] = max(rl[e][0], max(rl[e][1], rl[e][2])) <= 32 && rl[e][0] + rl[e][1] + rl[e][2] <= 64;
            // a circle with too many candidates stands aside (empty runs)
            far |= on[e] && !fits[e] ? 1u << (2 * h + e) : 0u;
            on[e] = on[e] && fits[e];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                rl[e][r] = fits[e] ? rl[e][r] : 0;
                kmax[r] = max(kmax[r], rl[e][r]);
            }
            firsts[2 * h + e] = (unsigned)(ra[e][0] | ra[e][1] << 10 | ra[e][2] << 20);
            lens[2 * h + e] = (unsigned)(rl[e][0] | rl[e][1] << 10 | rl[e][2] << 20);
        }
#pragma unroll
        for (int r = 0; r < 3; ++r) kmax[r] = wave_max_dpp(kmax[r]);
        unsigned long long mk[2];
        neighbor_masks<2, 4, kMaxN, true>(q, on, self, ra, rl, kmax, psort, c2, mk);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int u = 2 * h + e, pop = __builtin_popcountll(mk[e]);
            mine += pop;
            mask[u] = pop <= kRowRegs ? mk[e] : 0ull;
            slow |= pop <= kRowRegs ? 0u : 1u << u;
            if (!kHalf && pop > kRowRegs) start_s[ci[u]] = pop;
        }
    }
    slow |= far;
    // lengths of the long rows that no mask gave (a half list's rows hold only
    // the circles above their own)
    const unsigned uncounted = kHalf ? slow : far;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(uncounted != 0) != 0, 0)) {
#pragma unroll 1
        for (int u = 0; u < kBuildCpt; ++u) {
            const bool on = (uncounted >> u & 1) != 0;
            const int own = tid + u * kBuildBlock, i = cell_circ[on ? own : 0];
            int pop = 0, len = 0;
            wide_words(psort[on ? own : 0], on, own, [&](unsigned w, int first) {
                pop += __builtin_popcount(w);
                if (kHalf)
                    for (; w; w &= w - 1) len += cell_circ[first + __builtin_ctz(w)] > i ? 1 : 0;
            });
            mine += (far >> u & 1) ? pop : 0;
            if (on) start_s[i] = kHalf ? len : pop;
        }
    }
    // The instance's count, published before the rows are collected: the
    // workgroups behind wait for it (a half list holds half: the predicate is
    // symmetric)
    int total = block_sum<kBuildBlock>(mine, scan_tmp);
    if (kHalf) total /= 2;
    if (tid == 0) {
        if (b == 0)
            atomicAdd(&state[0], kHasPrefix | (unsigned long long)total);
        else if (b < state_words(B))
            __hip_atomic_store(&state[b], kHasCount | (unsigned long long)total, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    // ---- the rows, sorted, two at a time ---------------------------------------
    u16x2 nb[kBuildCpt / 2][kRowRegs];
    int cnt[kBuildCpt], used[kBuildCpt / 2];    // used: longest of the wave
#pragma unroll
    for (int h = 0; h < kBuildCpt / 2; ++h) {
        int m = 0, most = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned l = lens[2 * h + e];
            m = max(m, __builtin_popcountll(mask[2 * h + e]));
            most = max(most, (int)((l & 1023) + (l >> 10 & 1023) + (l >> 20)));
            cnt[2 * h + e] = 0;
        }
        m = wave_max_dpp(m);
        most = wave_max_dpp(most);
        used[h] = m;
        auto collect = [&](auto word) {
            using M = decltype(word);
            M mk[2];
            int n0[2], n1[2], s0[2], s1[2], s2[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const unsigned l = lens[2 * h + e], f = firsts[2 * h + e];
                mk[e] = (M)mask[2 * h + e];
                n0[e] = l & 1023;
                n1[e] = n0[e] + (l >> 10 & 1023);
                s0[e] = f & 1023;
                s1[e] = (int)(f >> 10 & 1023) - n0[e];
                s2[e] = (int)(f >> 20) - n1[e];
            }
#pragma unroll
            for (int k = 0; k < kRowRegs; ++k) {
                nb[h][k] = u16x2{0xffff, 0xffff};
                if (k < m) {                     // wave-uniform
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        int j;
                        bool has = next_neighbor(mk[e], n0[e], n1[e], s0[e], s1[e], s2[e], cell_circ, j);
                        if (kHalf) has = has && j > ci[2 * h + e];
                        cnt[2 * h + e] += has ? 1 : 0;
                        nb[h][k][e] = has ? (unsigned short)j : (unsigned short)0xffff;
                    }
                }
            }
        };
        if (most <= 32) collect(0u);
        else collect(0ull);
        if (m <= 8) sort_pairs<8>(nb[h]);
        else if (m <= 12) sort_pairs<12>(nb[h]);
        else sort_pairs<16>(nb[h]);
    }
#pragma unroll
    for (int u = 0; u < kBuildCpt; ++u) {
        const int s = tid + u * kBuildBlock;
        if (s < nn && !(slow >> u & 1)) start_s[ci[u]] = cnt[u];
    }
    __syncthreads();
    // ---- row starts: thread t holds circles 4 t .. 4 t + 3 -------------------
    int len4[kBuildCpt], sum = 0;
#pragma unroll
    for (int u = 0; u < kBuildCpt; ++u) {
        len4[u] = start_s[kBuildCpt * tid + u];
        sum += len4[u];
    }
    int sum_all;
    int run = block_exclusive_scan<kBuildBlock>(sum, scan_tmp, &sum_all);
#pragma unroll
    for (int u = 0; u < kBuildCpt; ++u) {
        start_s[kBuildCpt * tid + u] = run;
        run += len4[u];
    }
    __syncthreads();
    // A long row in ascending order: its circles as bits in LDS, a word per lane
    // of the half, and every lane's places from a prefix sum over the words.
    // put(place in the segment, circle).
    auto put_long_rows = [&](auto &&at, auto &&put) {
        unsigned *const word = bits_s + (tid - lane);
        long_rows(at, [&](int i, bool on, auto &&turns) {
            word[lane] = 0;
            wave_sync();
            turns([&](bool has, int j) {
                if (has) atomicOr(&word[(lane & 32) + (j >> 5)], 1u << (j & 31));
            });
            wave_sync();
            unsigned w = word[lane];
            if (kHalf) {
                const int first = i + 1 - 32 * (lane & 31);      // bits below it are not listed
                w = first >= 32 ? 0u : first > 0 ? w & (~0u << first) : w;
            }
            int before = __builtin_popcount(w);
            const int own = before;
            before += dppi<0x111>(before);                       // row_shr 1, 2, 4, 8
            before += dppi<0x112>(before);
            before += dppi<0x114>(before);
            before += dppi<0x118>(before);
            before += dppi<kDppBcast15, 0xa>(before);            // a half is two rows
            int place = start_s[i] + before - own;
            while (on && w) {
                put(place++, 32 * (lane & 31) + __builtin_ctz(w));
                w &= w - 1;
            }
            wave_sync();
        });
    };
    // ---- the segment into LDS -----------------------------------------------
    const bool staged = total <= kStage;
    if (staged) {
#pragma unroll
        for (int u = 0; u < kBuildCpt; ++u) {
            if (tid + u * kBuildBlock >= nn) continue;
            uint16_t *dst = stage + start_s[ci[u]];
#pragma unroll
            for (int k = 0; k < kRowRegs; ++k)
                if (k < used[u / 2] && k < cnt[u]) dst[k] = nb[u / 2][k][u % 2];
        }
        // (the sorted positions are overwritten by now)
        put_long_rows([&](int, int j) { return reinterpret_cast<const float2 *>(xy)[off + j]; },
                      [&](int place, int j) { stage[place] = (uint16_t)j; });
    }
    // ---- where the segment goes: the counts of the instances before ----------
    // One wave looks, a word per lane, so that little is read of words that
    // others are about to write.
    if (tid < kWave) {
        long long base = 0;
        for (int hi = b; hi > 0; hi -= kWave) {
            // a word before the first instance stands for a prefix of 0
            const int k = hi - 1 - tid;
            unsigned long long v = kHasPrefix;
            if (k >= 0) {
                while (((v = __hip_atomic_load(&state[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 62) == 0)
                    __builtin_amdgcn_s_sleep(1);
                if (k == 0) v = kHasPrefix | (v & ((1ull << kTicketShift) - 1));
            }
            const unsigned long long known = __builtin_amdgcn_ballot_w64((v >> 62) == 2);
            const int first = known ? __builtin_ctzll(known) : kWave;      // nearest prefix
            long long part = tid <= first ? (long long)(v & ~(3ull << 62)) : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, kWave);
            base += part;
            if (known) break;
        }
        if (tid == 0) {
            if (b > 0 && b < state_words(B))
                __hip_atomic_store(&state[b], kHasPrefix | (unsigned long long)(base + total),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            base_s = base;
        }
    }
    __syncthreads();                             // base, and the staged segment
    const long long base = base_s;
    auto clip = [](long long r) { return (int32_t)(r < 0x7fffffffLL ? r : 0x7fffffffLL); };
    if (tid == 0 && b == B - 1) {
        row[0] = 0;
        row[total_n] = clip(base + total);
        num_pairs[0] = base + total;
    }
    if (!valid) {
        // not a valid instance: an empty row for each circle it may write
        if (writable_range(off, n, total_n))
            for (int i = tid; i < n; i += kBuildBlock) row[off + i] = clip(base);
        return;
    }
    for (int i = tid; i < n; i += kBuildBlock) row[off + i] = clip(base + start_s[i]);
    const int add = kLocal ? 0 : off;
    if (staged) {
        // entries that fit, in order: single ones up to 8-byte (uint16) or
        // 16-byte (int32) alignment, then four per store
        const int len = (int)min((long long)total, max(capacity - base, 0LL));
        Idx *dst = col + base;
        const int mis = (int)((reinterpret_cast<uintptr_t>(dst) / sizeof(Idx)) & 3);
        const int head = min(len, (4 - mis) & 3);
        const int quads = (len - head) / 4;
        if (tid < head) dst[tid] = (Idx)(add + stage[tid]);
        for (int k = tid; k < quads; k += kBuildBlock) {
            const uint16_t *src = stage + head + 4 * k;
            if constexpr (kLocal)
                *reinterpret_cast<ushort4 *>(dst + head + 4 * k) = make_ushort4(src[0], src[1], src[2], src[3]);
            else
                *reinterpret_cast<int4 *>(dst + head + 4 * k) =
                    make_int4(add + src[0], add + src[1], add + src[2], add + src[3]);
        }
        const int done = head + 4 * quads;
        if (tid < len - done) dst[done + tid] = (Idx)(add + stage[done + tid]);
        return;
    }
    // a segment too long for LDS: rows from registers by their threads
#pragma unroll
    for (int u = 0; u < kBuildCpt; ++u) {
        if (tid + u * kBuildBlock >= nn) continue;
        const long long a = base + start_s[ci[u]];
#pragma unroll
        for (int k = 0; k < kRowRegs; ++k)
            if (k < cnt[u] && a + k < capacity) col[a + k] = (Idx)(add + nb[u / 2][k][u % 2]);
    }
    put_long_rows(at_slot, [&](int place, int j) {
        if (base + place < capacity) col[base + place] = (Idx)(add + j);
    });
}

// ---------------------------------------------------------------------------
// Energy and gradient over a list with both orientations (Def. 3.1,
// Def. 3.2), in one of two index forms: int32 global circle indices or
// uint16 instance-local ones (the compact form: 2 bytes per entry, so the
// list costs 4 bytes per pair).  Each thread owns circles and sums their
// pair terms in list order: no atomics.  One workgroup of 256 threads per
// instance; positions (8 KB) and the instance's list segment (when it fits,
// up to 6123 entries) are staged in LDS with coalesced streaming
// (non-temporal) 16-byte loads, the segment held as 16-bit byte offsets into
// the staged positions, so global memory sees each byte once, and the
// gradient leaves with streaming 8-byte stores.  An entry past a row's end
// reads a sentinel that points at a position far outside every container,
// so the pair loop needs no tests of its own.  The LDS footprint (20,464
// bytes) lets eight workgroups (32 waves) stay resident per CU, overlapping
// one instance's loads with another's arithmetic, and each thread walks the
// lists of two circles at once so that their LDS reads overlap.
// ---------------------------------------------------------------------------
constexpr int kSweepBlock = 256;
constexpr int kColLds = 6124;   // 8200 + 2 * 6124 + 16 bytes of LDS fit 8 workgroups per CU
constexpr uint16_t kFarOff = kMaxN * sizeof(float2);   // byte offset of the far position

template <typename Idx>
__global__ __launch_bounds__(kSweepBlock) void energy_grad_full_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ R,
    const float *__restrict__ xy, int64_t total_n, const int32_t *__restrict__ row,
    const Idx *__restrict__ col, int64_t col_len, float rad,
    float *__restrict__ energy, float *__restrict__ grad)
{
    // entries per 16-byte load; a local index needs no offset
    constexpr int kIV = 16 / (int)sizeof(Idx);
    constexpr bool kLocal = sizeof(Idx) == 2;
    __shared__ float2 pos[kMaxN + 1];         // + the far position
    __shared__ uint16_t col_s[kColLds];
    __shared__ float sum_tmp[kSweepBlock / kWave];

    const int b = blockIdx.x;
    int off, n;
    if (!instance_range(offset, b, total_n, &off, &n)) {
        if (threadIdx.x == 0) energy[b] = __builtin_nanf("");
        return;
    }
    // list entries outside [0, col_len) are never read
    const int r0 = row[off], r1 = row[off + n];
    const int len = r1 - r0;
    const bool sane = r0 >= 0 && len >= 0 && (int64_t)r1 <= col_len;
    if (!sane) {
        if (threadIdx.x == 0) energy[b] = __builtin_nanf("");
        return;
    }
    const bool staged = len < kColLds;         // room for the sentinel
    // One batch of streaming loads per thread -- positions as float4 where
    // the instance start is 16-byte aligned, the list segment as int4 -- all
    // issued before the first is used, so the workgroup waits for memory
    // once; then the LDS writes (list entries as 16-bit local indices).
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef int v4i __attribute__((ext_vector_type(4)));
    constexpr int kPV = (kMaxN / 2 + kSweepBlock - 1) / kSweepBlock;   // float4 per thread
    constexpr int kCV = (kColLds / kIV + kSweepBlock - 1) / kSweepBlock; // 16-byte loads per thread
    const bool pos_al = (reinterpret_cast<uintptr_t>(xy + 2 * (int64_t)off) & 15) == 0;
    const int npv = pos_al ? n / 2 : 0;
    const v4f *psrc = reinterpret_cast<const v4f *>(xy + 2 * (int64_t)off);
    const int mis = (int)((reinterpret_cast<uintptr_t>(col + r0) & 15) / sizeof(Idx));
    const int head = staged ? min(len, (kIV - mis) & (kIV - 1)) : 0;
    const int nv = staged ? (len - head) / kIV : 0;
    const v4i *csrc = reinterpret_cast<const v4i *>(col + r0 + head);
    // unconditional loads (indices clamped into range; the extra lanes'
    // values are dropped below), so nothing waits between them
    v4f pv[kPV];
    v4i cv[kCV];
    if (npv > 0) {
#pragma unroll
        for (int u = 0; u < kPV; ++u) {
            const int k = threadIdx.x + u * kSweepBlock;
            pv[u] = __builtin_nontemporal_load(psrc + (k < npv ? k : 0));
        }
    }
    if (nv > 0) {
#pragma unroll
        for (int u = 0; u < kCV; ++u) {
            const int v = threadIdx.x + u * kSweepBlock;
            cv[u] = __builtin_nontemporal_load(csrc + (v < nv ? v : 0));
        }
    }
    // row bounds of this thread's circles tid + 256 c (indices clamped to n)
    constexpr int kRC = kMaxN / kSweepBlock;
    int rw[kRC + 1];
#pragma unroll
    for (int c = 0; c <= kRC; ++c) {
        const int i = threadIdx.x + c * kSweepBlock;
        rw[c] = row[off + (i < n ? i : n)];
    }
    int rw1[kRC];
#pragma unroll
    for (int c = 0; c < kRC; ++c) {
        const int i = threadIdx.x + c * kSweepBlock + 1;
        rw1[c] = row[off + (i < n ? i : n)];
    }
    // an entry as the byte offset of its position; one outside the
    // instance as the far position (a pair that does not overlap)
    auto put = [&](int k, int v) {
        const int jj = kLocal ? v : v - off;
        col_s[k] = (unsigned)jj < (unsigned)n ? (uint16_t)(jj * (int)sizeof(float2)) : kFarOff;
    };
    if (!pos_al) {
        stage_positions<kSweepBlock>(xy, off, n, pos);
    } else if ((n & 1) && threadIdx.x == 0) {
        pos[n - 1] = reinterpret_cast<const float2 *>(xy)[off + n - 1];
    }
    if (staged) {
        if (threadIdx.x == 0) {
            col_s[len] = kFarOff;                         // sentinel past the last row
            pos[kMaxN] = make_float2(1e18f, 1e18f);       // squared distances stay finite
        }
        if ((int)threadIdx.x < head) put(threadIdx.x, col[r0 + threadIdx.x]);
        for (int k = head + kIV * nv + threadIdx.x; k < len; k += kSweepBlock) put(k, col[r0 + k]);
    }
#pragma unroll
    for (int u = 0; u < kPV; ++u) {
        const int k = threadIdx.x + u * kSweepBlock;
        if (k < npv) reinterpret_cast<float4 *>(pos)[k] = make_float4(pv[u].x, pv[u].y, pv[u].z, pv[u].w);
    }
#pragma unroll
    for (int u = 0; u < kCV; ++u) {
        const int v = threadIdx.x + u * kSweepBlock;
        if (v < nv) {
            const int k = head + kIV * v;
            if constexpr (kLocal) {
                // eight 16-bit entries, low half first
                const int w4[4] = {cv[u].x, cv[u].y, cv[u].z, cv[u].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    put(k + 2 * q, w4[q] & 0xffff);
                    put(k + 2 * q + 1, (int)((unsigned)w4[q] >> 16));
                }
            } else {
                put(k, cv[u].x); put(k + 1, cv[u].y); put(k + 2, cv[u].z); put(k + 3, cv[u].w);
            }
        }
    }
    __syncthreads();
    const float Rb = R[b];
    const float two_r = 2.0f * rad, four_r2 = two_r * two_r;
    float e = 0.0f;
    const bool g_al = (reinterpret_cast<uintptr_t>(grad) & 7) == 0;
#pragma unroll
    for (int pass = 0; pass < kRC / 2; ++pass) {
      const int i0 = threadIdx.x + 2 * kSweepBlock * pass;
      if (i0 >= n) break;
      // two circles per pass (i0 and i0 + kSweepBlock): their list and
      // position reads overlap; each keeps its own order of terms
      float gxA[2], gyA[2], eiA[2];
      int aA[2], zA[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
          const int i = i0 + h * kSweepBlock;
          gxA[h] = gyA[h] = eiA[h] = 0.f;
          aA[h] = 0; zA[h] = 0;
          if (i < n) {
              int a = rw[2 * pass + h] - r0, z = rw1[2 * pass + h] - r0;
              aA[h] = a < 0 ? 0 : a;
              zA[h] = z > len ? len : z;
          }
      }
      const int span = max(zA[0] - aA[0], zA[1] - aA[1]);
      const float2 piA[2] = {pos[i0], i0 + kSweepBlock < n ? pos[i0 + kSweepBlock] : make_float2(0.f, 0.f)};
      // one pass over the rows, branch-free: an entry past its row or
      // outside the instance is the far position, a pair that does not
      // overlap.  Per pair side: kf' = d / l (the factor -2 of the gradient
      // term is applied to the sums at the end, exactly), and d^2 of every
      // side (each pair counted twice, halved at the end); 1/l from
      // l^2 + FLT_MIN (exactly l^2 above 2^-100), so coincident centres (l =
      // 0, dx = dy = 0) give d = 2 rad and no gradient without a test of
      // their own.
      auto rows_pass = [&](auto staged_c) {
          constexpr bool ST = decltype(staged_c)::value;
#pragma unroll 1
          for (int t = 0; t < span; ++t) {
              float2 pjA[2];
              bool realA[2];
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                  const int k = aA[h] + t;
                  if constexpr (ST) {
                      // past the row: the sentinel at col_s[len]
                      const int off8 = col_s[k < zA[h] ? k : len];
                      pjA[h] = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(pos) + off8);
                      realA[h] = true;
                  } else {
                      int j = 0xFFFF;
                      if (k < zA[h]) j = kLocal ? (int)col[r0 + k] : col[r0 + k] - off;
                      realA[h] = (unsigned)j < (unsigned)n;
                      pjA[h] = pos[realA[h] ? j : 0];
                  }
              }
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                  const float2 pi = piA[h], pj = pjA[h];
                  const float dx = pi.x - pj.x, dy = pi.y - pj.y;
                  const float l2r = dx * dx + dy * dy;
                  const float l2 = ST || realA[h] ? l2r : four_r2;
                  const float il = __builtin_amdgcn_rsqf(l2 + 1.17549435e-38f);
                  const float d = l2 < four_r2 ? two_r - l2 * il : 0.f;
                  eiA[h] = fmaf(d, d, eiA[h]);
                  const float kf = d * il;
                  gxA[h] = fmaf(kf, dx, gxA[h]);
                  gyA[h] = fmaf(kf, dy, gyA[h]);
              }
          }
      };
      if (staged) rows_pass(std::true_type{});
      else rows_pass(std::false_type{});
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = i0 + h * kSweepBlock;
        if (i >= n) break;
        const float2 pi = piA[h];
        // the sums of the pair sides: gradient times -2, energy halved
        float gx = -2.f * gxA[h], gy = -2.f * gyA[h], ei = 0.5f * eiA[h];
        const float r2 = pi.x * pi.x + pi.y * pi.y;
        const float ir = r2 > 0.f ? __builtin_amdgcn_rsqf(r2) : 0.f;
        const float d0 = fmaxf(r2 * ir + rad - Rb, 0.f);
        ei += d0 * d0;
        const float kc = 2.f * d0 * ir;
        gx += kc * pi.x;
        gy += kc * pi.y;
        // E sums over every circle: a non-finite position makes it NaN
        if (!(isfinite(pi.x) && isfinite(pi.y))) ei = __builtin_nanf("");
        e += ei;
        if (grad) {
            if (g_al) {
                typedef float v2f __attribute__((ext_vector_type(2)));
                const v2f t = {gx, gy};
                __builtin_nontemporal_store(t, reinterpret_cast<v2f *>(grad) + (off + i));
            } else {
                __builtin_nontemporal_store(gx, &grad[2 * (int64_t)(off + i)]);
                __builtin_nontemporal_store(gy, &grad[2 * (int64_t)(off + i) + 1]);
            }
        }
      }
    }
    const float tot = block_sum<kSweepBlock>(e, sum_tmp);
    if (threadIdx.x == 0) energy[b] = tot;
}

// ---------------------------------------------------------------------------
// Energy and gradient over a neighbor list that holds each pair once
// (Def. 3.1, Def. 3.2; rows ascending, entries j > i).  One workgroup of 512
// threads per instance, three passes over the list segment staged in LDS:
//   * staging: coalesced streaming (non-temporal) 16-byte loads of the
//     segment, every entry stored as the pair (i, j) of 16-bit local indices
//     (j from the loads, i filled in by the thread that owns row i), so
//     global memory sees each list entry once;
//   * the pair pass, entry-parallel (every thread the same number of
//     pairs): the pair term of Def. 3.1 once per pair, its energy added to
//     the thread's sum and its gradient term for circle i stored in place of
//     the entry; the entry is also counted and placed in circle j's bucket
//     (a counting sort by j in LDS: 16-bit counters two per word, a block
//     scan, a scatter, each bucket then sorted by entry, as the scatter's
//     order depends on atomic arrival);
//   * the gather, one thread per circle: the terms of its partners below it
//     (its bucket, negated: the term for j is minus the term for i, bit for
//     bit) and then above it (its own row), in ascending order of the other
//     circle.  No atomics on the sums, so the result is bitwise
//     reproducible.
// A segment longer than the LDS chunk is taken in consecutive chunks: every
// partner i < j of circle j sits in a row before row j, so a circle's terms
// are still added in ascending order of the other circle.  Four workgroups
// (32 waves) stay resident per CU, overlapping one instance's loads with
// another's on-chip work.
// ---------------------------------------------------------------------------
constexpr int kHalfBlock = 512;
constexpr int kHalfWaves = kHalfBlock / kWave;
constexpr int kHalfChunk = 3024;    // list entries per chunk (a multiple of 8)

union SweepEntry {
    struct { uint16_t j, i; } h;   // staged pair: local indices of the partner and of the row
    uint32_t ij;
    float2 f;                      // after the pair pass: the pair's gradient term for circle i
};

__global__ __launch_bounds__(kHalfBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void energy_grad_half_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ R,
    const float *__restrict__ xy, int64_t total_n, const int32_t *__restrict__ row,
    const int32_t *__restrict__ col, int64_t col_len, float rad,
    float *__restrict__ energy, float *__restrict__ grad)
{
    __shared__ float2 pos[kMaxN];
    __shared__ SweepEntry ent[kHalfChunk];
    __shared__ uint16_t rev[kHalfChunk];        // entries grouped by the higher circle j
    __shared__ uint32_t rcur[kMaxN / 2];    // per circle a 16-bit count / cursor, two per word
    __shared__ int scan_tmp[kHalfWaves];
    __shared__ float sum_tmp[kHalfWaves];

    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    int off, n;
    if (!instance_range(offset, b, total_n, &off, &n)) {
        if (tid == 0) energy[b] = __builtin_nanf("");
        return;
    }
    // list entries outside [0, col_len) are never read
    const int r0 = row[off], r1 = row[off + n];
    const int len = r1 - r0;
    if (!(r0 >= 0 && len >= 0 && (int64_t)r1 <= col_len)) {
        if (tid == 0) energy[b] = __builtin_nanf("");
        return;
    }
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef int v4i __attribute__((ext_vector_type(4)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    constexpr int kPV = (kMaxN / 2 + kHalfBlock - 1) / kHalfBlock;   // float4 per thread
    constexpr int kCV = (kHalfChunk / 4 + kHalfBlock - 1) / kHalfBlock;  // int4 per thread
    constexpr int kEV = (kHalfChunk + kHalfBlock - 1) / kHalfBlock;      // entries per thread
    constexpr int kRC = kMaxN / kHalfBlock;                           // circles per thread
    const bool pos_al = (reinterpret_cast<uintptr_t>(xy + 2 * (int64_t)off) & 15) == 0;
    const int npv = pos_al ? n / 2 : 0;
    const v4f *psrc = reinterpret_cast<const v4f *>(xy + 2 * (int64_t)off);

    // One batch of streaming loads of the chunk starting at entry c0 (cl
    // entries): a scalar head up to 16-byte alignment, int4 loads, a tail.
    // The int4 loads are unconditional (indices clamped into range, the
    // extra lanes' values dropped when stored), so nothing waits between them.
    v4i cv[kCV];
    int head = 0, nv = 0;
    auto load_chunk = [&](int c0, int cl) {
        const int32_t *src = col + r0 + c0;
        const int mis = (int)((reinterpret_cast<uintptr_t>(src) & 15) >> 2);
        head = min(cl, (4 - mis) & 3);
        nv = (cl - head) >> 2;
        const v4i *csrc = reinterpret_cast<const v4i *>(src + head);
        if (nv > 0) {
#pragma unroll
            for (int u = 0; u < kCV; ++u) {
                const int v = tid + u * kHalfBlock;
                cv[u] = __builtin_nontemporal_load(csrc + (v < nv ? v : 0));
            }
        }
    };
    auto put = [&](int k, int v) {
        const int jj = v - off;
        ent[k].h.j = (unsigned)jj < (unsigned)n ? (uint16_t)jj : (uint16_t)0xFFFF;
    };
    auto store_chunk = [&](int c0, int cl) {
        const int32_t *src = col + r0 + c0;
        if (tid < head) put(tid, src[tid]);
        for (int k = head + 4 * nv + tid; k < cl; k += kHalfBlock) put(k, src[k]);
#pragma unroll
        for (int u = 0; u < kCV; ++u) {
            const int v = tid + u * kHalfBlock;
            if (v < nv) {
                const int k = head + 4 * v;
                put(k, cv[u].x); put(k + 1, cv[u].y); put(k + 2, cv[u].z); put(k + 3, cv[u].w);
            }
        }
    };

    v4f pv[kPV];
    if (npv > 0) {
#pragma unroll
        for (int u = 0; u < kPV; ++u) {
            const int k = tid + u * kHalfBlock;
            pv[u] = __builtin_nontemporal_load(psrc + (k < npv ? k : 0));
        }
    }
    int cl = len < kHalfChunk ? len : kHalfChunk;
    load_chunk(0, cl);
    // row bounds of this thread's circles tid + 512 c, relative to r0
    // (indices clamped to n); rows must be non-decreasing inside [r0, r1]
    int ra[kRC], rz[kRC];
    int bad = 0;
#pragma unroll
    for (int c = 0; c < kRC; ++c) {
        const int i = tid + c * kHalfBlock;
        ra[c] = row[off + (i < n ? i : n)];
        rz[c] = row[off + (i + 1 < n ? i + 1 : n)];
        if (i < n && !(r0 <= ra[c] && ra[c] <= rz[c] && rz[c] <= r1)) bad = 1;
        ra[c] -= r0;
        rz[c] -= r0;
    }
    // the row of every entry of the chunk, from the thread that owns it
    auto fill_rows = [&](int tid, int c0, int cl) {
#pragma unroll
        for (int c = 0; c < kRC; ++c) {
            const int i = tid + c * kHalfBlock;
            const int a = max(ra[c] - c0, 0), z = min(rz[c] - c0, cl);
            for (int k = a; k < z; ++k) ent[k].h.i = (uint16_t)i;
        }
    };
    if (!pos_al) {
        stage_positions<kHalfBlock>(xy, off, n, pos);
    } else if ((n & 1) && tid == 0) {
        pos[n - 1] = reinterpret_cast<const float2 *>(xy)[off + n - 1];
    }
#pragma unroll
    for (int u = 0; u < kPV; ++u) {
        const int k = tid + u * kHalfBlock;
        if (k < npv) reinterpret_cast<float4 *>(pos)[k] = make_float4(pv[u].x, pv[u].y, pv[u].z, pv[u].w);
    }
    store_chunk(0, cl);
    if (!bad) fill_rows(tid, 0, cl);
    for (int q = tid; q < kMaxN / 2; q += kHalfBlock) rcur[q] = 0u;
    if (__syncthreads_or(bad)) {
        if (tid == 0) energy[b] = __builtin_nanf("");
        return;
    }

    const float Rb = R[b];
    const float two_r = 2.0f * rad, four_r2 = two_r * two_r;
    float e = 0.0f;                 // this thread's energy terms
    float gxA[kRC], gyA[kRC];       // gradient of this thread's circles
#pragma unroll
    for (int c = 0; c < kRC; ++c) gxA[c] = gyA[c] = 0.f;
    auto cur16 = [&](int j) -> int { return (int)((rcur[j >> 1] >> ((j & 1) * 16)) & 0xffffu); };

    for (int c0 = 0;;) {
        // an opaque copy of the thread id: addresses and circle indices are
        // recomputed inside the loop instead of being hoisted and kept live
        int tid_l = (int)threadIdx.x;
        asm volatile("" : "+v"(tid_l));
        const int tid = tid_l;
        // ---- count the listed pairs (i < j < n) of every circle j ----------
#pragma unroll
        for (int u = 0; u < kEV; ++u) {
            const int k = tid + u * kHalfBlock;
            if (k < cl) {
                const uint32_t ij = ent[k].ij;
                const int i = (int)(ij >> 16), j = (int)(ij & 0xffffu);
                if (j < n && j > i) atomicAdd(&rcur[j >> 1], 1u << ((j & 1) * 16));
            }
        }
        __syncthreads();
        // exclusive scan: thread t holds the counts of circles 2t and 2t + 1
        // (word t; every count is below kHalfChunk)
        const uint32_t w = rcur[tid];
        const int k0 = (int)(w & 0xffffu), k1 = (int)(w >> 16);
        const int t2 = k0 + k1;
        int inc = t2;                     // inclusive scan over the wave
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int v = __shfl_up(inc, o, kWave);
            if ((tid & (kWave - 1)) >= o) inc += v;
        }
        if ((tid & (kWave - 1)) == kWave - 1) scan_tmp[tid / kWave] = inc;
        __syncthreads();
        int s0 = inc - t2;                // plus the totals of the waves before
#pragma unroll
        for (int q = 0; q < kHalfWaves - 1; ++q) s0 += q < tid / kWave ? scan_tmp[q] : 0;
        rcur[tid] = (uint32_t)s0 | ((uint32_t)(s0 + k0) << 16);
        __syncthreads();
        // ---- the pair pass: every listed pair once --------------------------
#pragma unroll
        for (int u = 0; u < kEV; ++u) {
            const int k = tid + u * kHalfBlock;
            if (k < cl) {
                const uint32_t ij = ent[k].ij;
                const int i = (int)(ij >> 16), j = (int)(ij & 0xffffu);
                float2 f = make_float2(0.f, 0.f);
                if (j < n && j > i) {
                    const float2 pi = pos[i], pj = pos[j];
                    const float dx = pi.x - pj.x, dy = pi.y - pj.y;
                    const float l2 = dx * dx + dy * dy;
                    const bool ov = l2 < four_r2;
                    const float il = (ov && l2 > 0.f) ? __builtin_amdgcn_rsqf(l2) : 0.f;
                    const float d = ov ? two_r - l2 * il : 0.f;
                    e += d * d;
                    const float kf = -2.f * d * il;
                    f = make_float2(kf * dx, kf * dy);
                    const uint32_t sh = (j & 1) * 16;
                    const uint32_t old = atomicAdd(&rcur[j >> 1], 1u << sh);
                    rev[(old >> sh) & 0xffffu] = (uint16_t)k;
                }
                ent[k].f = f;
            }
        }
        __syncthreads();
        // ---- the gather: partners below (bucket), then above (own row) ------
        // cursors now hold bucket ends: circle j's bucket is rev[e(j-1) .. e(j))
        int aA[kRC], nrA[kRC], fA[kRC], totA[kRC];
#pragma unroll
        for (int c = 0; c < kRC; ++c) {
            const int i = tid + c * kHalfBlock;
            aA[c] = i > 0 ? cur16(i - 1) : 0;
            const int z = i < n ? cur16(i) : aA[c];
            nrA[c] = z - aA[c];
            for (int q = aA[c] + 1; q < z; ++q) {        // sort the bucket by entry
                const uint16_t key = rev[q];
                int t = q - 1;
                while (t >= aA[c] && rev[t] > key) { rev[t + 1] = rev[t]; --t; }
                rev[t + 1] = key;
            }
            fA[c] = max(ra[c] - c0, 0);
            const int fz = min(rz[c] - c0, cl);
            totA[c] = nrA[c] + (fz > fA[c] ? fz - fA[c] : 0);
        }
        const int span = max(totA[0], totA[1]);
        for (int t = 0; t < span; ++t) {
            float2 fv[kRC];
            bool below[kRC];
#pragma unroll
            for (int c = 0; c < kRC; ++c) {
                below[c] = t < nrA[c];
                const int k = below[c] ? (int)rev[aA[c] + t] : fA[c] + t - nrA[c];
                fv[c] = t < totA[c] ? ent[k].f : make_float2(0.f, 0.f);
            }
#pragma unroll
            for (int c = 0; c < kRC; ++c) {
                if (t < totA[c]) {
                    if (below[c]) { gxA[c] -= fv[c].x; gyA[c] -= fv[c].y; }
                    else { gxA[c] += fv[c].x; gyA[c] += fv[c].y; }
                }
            }
        }
        c0 += cl;
        if (c0 >= len) break;
        // next chunk: every thread has finished with this one
        cl = len - c0 < kHalfChunk ? len - c0 : kHalfChunk;
        __syncthreads();
        load_chunk(c0, cl);
        store_chunk(c0, cl);
        fill_rows(tid, c0, cl);
        for (int q = tid; q < kMaxN / 2; q += kHalfBlock) rcur[q] = 0u;
        __syncthreads();
    }

    // containment terms; a non-finite position makes E NaN
    const bool g_al = (reinterpret_cast<uintptr_t>(grad) & 7) == 0;
#pragma unroll
    for (int c = 0; c < kRC; ++c) {
        const int i = tid + c * kHalfBlock;
        if (i >= n) break;
        const float2 pi = pos[i];
        float gx = gxA[c], gy = gyA[c];
        const float r2 = pi.x * pi.x + pi.y * pi.y;
        const float ir = r2 > 0.f ? __builtin_amdgcn_rsqf(r2) : 0.f;
        const float d0 = fmaxf(r2 * ir + rad - Rb, 0.f);
        e += d0 * d0;
        const float kc = 2.f * d0 * ir;
        gx += kc * pi.x;
        gy += kc * pi.y;
        if (!(isfinite(pi.x) && isfinite(pi.y))) e = __builtin_nanf("");
        if (grad) {
            if (g_al) {
                const v2f t = {gx, gy};
                __builtin_nontemporal_store(t, reinterpret_cast<v2f *>(grad) + (off + i));
            } else {
                __builtin_nontemporal_store(gx, &grad[2 * (int64_t)(off + i)]);
                __builtin_nontemporal_store(gy, &grad[2 * (int64_t)(off + i) + 1]);
            }
        }
    }
    const float tot = block_sum<kHalfBlock>(e, sum_tmp);
    if (tid == 0) energy[b] = tot;
}

// ---------------------------------------------------------------------------
// FP64 verify: the overlap energy of every pair and every circle, each pair
// once.  Only pairs closer than 2 contribute, so the circles are sorted into
// cells of side >= 2 and a circle at slot s meets the slots after it in its
// own cell row (its cell and the next) and the three cells of the row above:
// two runs of consecutive positions, about five candidates in all at the
// densities of packings.  An FP32 distance (within 4e-7) passes the
// candidates within 1e-5 of an overlap to FP64, in which every term is formed
// and summed; the others' terms are exactly zero.  Slots are in cell order,
// then circle order (sort_cells), so every sum has a fixed order.  No
// contraction: products and sums round as written, like the oracle's.
// Up to kVerifyBrute circles every pair is tested without a grid: circle i
// with the next floor((n-1)/2) circles cyclically (and, for even n, with
// i+n/2 when i < n/2); the positions sit in LDS twice in a row, so partner
// i + t needs no wrap.
// With R_tight set it also forms the smallest container of the unit
// circles, rho_max = max_i fl(|c_i| + 1): at any radius R >= rho_max every
// containment term (fl(|c_i| + 1) - R) is <= 0, so the layout is feasible
// there exactly when its pair energy is below tol.  R_tight[b] receives
// rho_max rounded up to FP32 when that holds and the value is below the
// instance's radius, else the instance's FP32 radius; feas_tight[b] is
// feasibility at R_tight[b].
// 256 threads and 17 KB of LDS per instance: eight workgroups per CU, so one
// instance's sort (a chain of LDS round trips and barriers) runs beside the
// others' distances.  2048 x n = 1000: 26 us, against 277 us with every pair
// tested in FP64 from LDS; 256 x n = 1000 53 -> 10 us.
// ---------------------------------------------------------------------------
constexpr int kVerifyBlock = 256;
constexpr int kVerifyCpt = kMaxN / kVerifyBlock;
constexpr int kVerifyNc = 32;            // cells per axis at most (side 2.2 at n = 1024, R = 35)
// Candidates of a circle from which its wave takes them all in FP64 (packings
// have about five, layouts compressed to a third of their width 45).  500 of
// 1000 circles in a box of 4 x 4, 256 instances: 106 us, 148 with a branch per
// overlap and 111 with every pair tested in FP64 from LDS; all 1000 in it 281,
// 401 and 162; 512 layouts at a third of their width 53.5, 65 and 254.
constexpr int kVerifyCrowd = 32;
constexpr int kVerifyBrute = 64;         // 2048 instances of 96: 14.8 us tested pair by pair, of 200 sorted 12.9

__global__ __launch_bounds__(kVerifyBlock) void verify_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ R,
    const double *__restrict__ R64, const float *__restrict__ xy, int64_t total_n, double tol,
    double *__restrict__ energy64, double *__restrict__ max_pair,
    double *__restrict__ max_cont, int32_t *__restrict__ feasible, float *__restrict__ R_tight,
    int32_t *__restrict__ feas_tight)
{
#pragma clang fp contract(off)
    __shared__ float2 psort[kMaxN + 4];
    __shared__ int cell_start[kVerifyNc * kVerifyNc + 1];
    __shared__ uint16_t cell_circ[kMaxN];
    __shared__ uint16_t slot_tmp[kMaxN];
    __shared__ int scan_tmp[kVerifyBlock / kWave];
    __shared__ double part[kVerifyBlock / kWave][5];

    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    int off, n;
    if (!instance_range(offset, b, total_n, &off, &n)) {
        if (tid == 0) {
            if (energy64) energy64[b] = __builtin_nan("");
            if (max_pair) max_pair[b] = __builtin_nan("");
            if (max_cont) max_cont[b] = __builtin_nan("");
            if (feasible) feasible[b] = 0;
            if (R_tight) R_tight[b] = R[b];
            if (feas_tight) feas_tight[b] = 0;
        }
        return;
    }
    float2 p[kVerifyCpt];
#pragma unroll
    for (int u = 0; u < kVerifyCpt; ++u) {
        const int i = tid + u * kVerifyBlock;
        p[u] = i < n ? reinterpret_cast<const float2 *>(xy)[off + i] : make_float2(0.f, 0.f);
    }
    const double Rb = R64 ? R64[b] : (double)R[b];
    double sp = 0.0, sc = 0.0, mp = 0.0, mc = 0.0, rm = 0.0;
    // the FP64 term of a pair
    auto pair = [&](float2 pi, float2 pj) {
#pragma clang fp contract(off)
        const double dx = (double)pi.x - (double)pj.x;
        const double dy = (double)pi.y - (double)pj.y;
        const double l2 = dx * dx + dy * dy;
        if (l2 < 4.0) {
            const double d = 2.0 - sqrt(l2);
            sp = sp + d * d;
            mp = fmax(mp, d);
        }
    };
    // FP32 tests: a pair that may overlap, a circle that may reach past R
    const float near2 = 4.0f * (1.0f + 1e-5f);
    const double inner = Rb - 1.0;
    const float lim2 = inner > 0.0 ? (float)(inner * inner * (1.0 - 1e-5)) : -1.0f;

    if (n <= kVerifyBrute) {
        if (tid < n) {
            psort[tid] = p[0];
            psort[tid + n] = p[0];
        }
        __syncthreads();
        const int cnt = (n - 1) / 2 + (((n & 1) == 0 && tid < n / 2) ? 1 : 0);
        if (tid < n)
            for (int t = 1; t <= cnt; ++t) {
                const float2 pj = psort[tid + t];
                const float dx = p[0].x - pj.x, dy = p[0].y - pj.y;
                if (dx * dx + dy * dy < near2) pair(p[0], pj);
            }
    } else {
        const Grid g = make_grid<kVerifyNc>(R[b], 2.0f * (1.0f + kCellSafety));
        int own[kVerifyCpt];
        if (tid == 0) psort[kMaxN] = make_float2(HUGE_VALF, HUGE_VALF);       // overlaps nothing
        sort_cells<kVerifyBlock, kVerifyCpt>(tid, p, n, g, cell_start, cell_circ, slot_tmp, psort,
                                             scan_tmp, own);
#pragma unroll
        for (int u = 0; u < kVerifyCpt; ++u) {
            const int s = tid + u * kVerifyBlock;
            const bool on = s < n;
            p[u] = psort[on ? s : 0];                 // from here on: the circle of slot s
            const int cx = cell_coord(p[u].x, g), cy = cell_coord(p[u].y, g);
            const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx < g.nc - 1 ? cx + 1 : g.nc - 1;
            const int up = cy < g.nc - 1 ? cy + 1 : cy;
            const int a1 = cell_start[up * g.nc + x0], z1 = cell_start[up * g.nc + x1 + 1];
            const int z0 = cell_start[cy * g.nc + x1 + 1];
            const int run0 = on ? z0 - (s + 1) : 0, run1 = on && up > cy ? z1 - a1 : 0;
            const int run = run0 + run1;
            // a crowded neighborhood, where most candidates overlap: the FP64
            // terms of four side by side, without the FP32 test
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(run > kVerifyCrowd) != 0, 0)) {
                const int longest = wave_max_dpp(run);
                const double xi = p[u].x, yi = p[u].y;
                for (int k0 = 0; k0 < longest; k0 += 4) {
                    double d[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int k = k0 + q;
                        const float2 pj = psort[k < run0 ? s + 1 + k : k < run ? a1 + (k - run0) : kMaxN];
                        const double dx = xi - (double)pj.x, dy = yi - (double)pj.y;
                        d[q] = 2.0 - sqrt(dx * dx + dy * dy);
                        asm volatile("" : "+v"(d[q]));
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        d[q] = fmax(d[q], 0.0);       // no overlap, and NaN, add zero
                        sp = sp + d[q] * d[q];
                        mp = fmax(mp, d[q]);
                    }
                }
                continue;
            }
            // both runs as one, four candidates in flight
            for (int k0 = 0; k0 < run; k0 += 4) {
                float2 pj[4];
                bool hit[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int k = k0 + q;
                    pj[q] = psort[k < run0 ? s + 1 + k : k < run ? a1 + (k - run0) : 0];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float dx = p[u].x - pj[q].x, dy = p[u].y - pj[q].y;
                    hit[q] = k0 + q < run && dx * dx + dy * dy < near2;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (hit[q]) pair(p[u], pj[q]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kVerifyCpt; ++u) {
        if (tid + u * kVerifyBlock >= n) continue;
        const float2 q = p[u];
        // (a non-finite coordinate fails the test)
        if (R_tight == nullptr && q.x * q.x + q.y * q.y < lim2) continue;
        const double xi = q.x, yi = q.y;
        const double rho = sqrt(xi * xi + yi * yi);
        rm = fmax(rm, rho + 1.0);
        const double d0 = (rho + 1.0) - Rb;
        if (d0 > 0.0) {
            sc = sc + d0 * d0;
            mc = fmax(mc, d0);
        }
        if (!(isfinite(xi) && isfinite(yi))) sc = __builtin_nan("");
    }
    const double v[5] = {wave_sum_dpp(sp), wave_sum_dpp(sc), wave_max_dpp(mp), wave_max_dpp(mc), wave_max_dpp(rm)};
    if ((tid & (kWave - 1)) == 0)
#pragma unroll
        for (int q = 0; q < 5; ++q) part[tid / kWave][q] = v[q];
    __syncthreads();
    if (tid == 0) {
        double Ep = part[0][0], Ec = part[0][1], Mp = part[0][2], Mc = part[0][3], Rm = part[0][4];
#pragma unroll
        for (int w = 1; w < kVerifyBlock / kWave; ++w) {
            Ep += part[w][0];
            Ec += part[w][1];
            Mp = fmax(Mp, part[w][2]);
            Mc = fmax(Mc, part[w][3]);
            Rm = fmax(Rm, part[w][4]);
        }
        const double E = Ep + Ec;
        const bool bad = E != E;     // a non-finite coordinate
        if (energy64) energy64[b] = E;
        if (max_pair) max_pair[b] = bad ? E : Mp;
        if (max_cont) max_cont[b] = bad ? E : Mc;
        if (feasible) feasible[b] = E < tol ? 1 : 0;
        if (R_tight) {
            const float rt = __double2float_ru(Rm);     // smallest FP32 value >= Rm
            const bool use = !bad && n > 0 && Ep < tol && (double)rt < Rb;
            R_tight[b] = use ? rt : R[b];
            if (feas_tight) feas_tight[b] = (use || E < tol) ? 1 : 0;
        }
    }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
hipError_t launch_build(const int32_t *offset, const float *R, const float *xy, int B,
                        int64_t total_n, double cutoff, float h_req, int format,
                        int32_t *row, void *col, int64_t capacity, int64_t *num_pairs,
                        int64_t *inst_state, hipStream_t s)
{
    const double c2 = cutoff * cutoff;
    // the caller's workspace may start at any byte: the atomics need 8-byte
    // words, of which at least B - 1 follow in its 8 B bytes (B = 1: its 256)
    unsigned long long *state =
        reinterpret_cast<unsigned long long *>((reinterpret_cast<uintptr_t>(inst_state) + 7) & ~(uintptr_t)7);
    build_clear_kernel<<<(state_words(B) - 1) / kBuildBlock + 1, kBuildBlock, 0, s>>>(state, B);
    if (format == kListLocal16)
        build_kernel<kListLocal16><<<B, kBuildBlock, 0, s>>>(offset, R, xy, B, total_n, c2, h_req, row,
                                                             col, capacity, num_pairs, state);
    else if (format == kListHalf)
        build_kernel<kListHalf><<<B, kBuildBlock, 0, s>>>(offset, R, xy, B, total_n, c2, h_req, row, col,
                                                          capacity, num_pairs, state);
    else
        build_kernel<kListFull><<<B, kBuildBlock, 0, s>>>(offset, R, xy, B, total_n, c2, h_req, row, col,
                                                          capacity, num_pairs, state);
    return hipGetLastError();
}

hipError_t launch_energy_grad(const int32_t *offset, const float *R, const float *xy, int B,
                              int64_t total_n, const int32_t *row, const void *col,
                              int64_t col_len, int format, float rad, float *energy, float *grad,
                              hipStream_t s)
{
    if (format == kListHalf)
        energy_grad_half_kernel<<<B, kHalfBlock, 0, s>>>(
            offset, R, xy, total_n, row, static_cast<const int32_t *>(col), col_len, rad, energy, grad);
    else if (format == kListFull)
        energy_grad_full_kernel<int32_t><<<B, kSweepBlock, 0, s>>>(
            offset, R, xy, total_n, row, static_cast<const int32_t *>(col), col_len, rad, energy, grad);
    else
        energy_grad_full_kernel<uint16_t><<<B, kSweepBlock, 0, s>>>(
            offset, R, xy, total_n, row, static_cast<const uint16_t *>(col), col_len, rad, energy, grad);
    return hipGetLastError();
}

hipError_t launch_verify(const int32_t *offset, const float *R, const double *R64,
                         const float *xy, int B, int64_t total_n, double tol, double *e64,
                         double *mp, double *mc, int32_t *feas, hipStream_t s)
{
    verify_kernel<<<B, kVerifyBlock, 0, s>>>(offset, R, R64, xy, total_n, tol, e64, mp, mc, feas,
                                             nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_verify_tighten(const int32_t *offset, const float *R, const double *R64,
                                 const float *xy, int B, int64_t total_n, double tol,
                                 float *R_out, int32_t *feas, hipStream_t s)
{
    verify_kernel<<<B, kVerifyBlock, 0, s>>>(offset, R, R64, xy, total_n, tol, nullptr, nullptr,
                                             nullptr, nullptr, R_out, feas);
    return hipGetLastError();
}

}  // namespace pecc
