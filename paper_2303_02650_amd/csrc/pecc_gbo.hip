// Geometric batch descent (Alg. 1 with the limited-memory reading of
// Eq. 8-11 and the batch energy of Eq. 7) for batches of instances, one
// persistent launch.
//
// Mapping (one workgroup of 512 threads = 8 waves per instance):
//   * the circles are partitioned once, at the start, into the blocks of a
//     blocks x blocks grid over [-R, R]^2 (computed in FP64 on the input
//     positions); block (bx, by) has colour (bx mod 2) + 2 (by mod 2), so
//     blocks of one colour never touch;
//   * an outer iteration visits the colours 0..3 in turn; inside a colour
//     the 8 waves take its batches, one batch per wave at a time, and run one
//     quasi-Newton iteration each, entirely inside the wave: the batch's
//     circles sit on the lanes (up to 128, two per lane), its curvature
//     history is loaded into registers, its Gram matrix into a wave-private
//     LDS area, and every reduction is a wave reduction -- no workgroup
//     barrier inside a visit;
//   * the other circles are seen at their positions from the start of the
//     colour (the batches of a colour run concurrently); the batch's own
//     trial positions live in a separate LDS array;
//   * neighbor lists (cutoff 2 rad + 2 skin) are rebuilt after a colour once
//     some circle has moved more than skin / 2 from the positions of the
//     last rebuild, so every circle starts a colour within skin / 2 of them.
//     A trial that keeps the batch's circles within skin of those positions
//     is evaluated over the lists; a longer trial (the step of Alg. 1 is not
//     limited) over the cell grid of the last rebuild for the other circles
//     (still within skin / 2 of their cells' positions, so the 3 x 3 cells
//     around the trial position hold every partner closer than 2 rad) and
//     over all of the batch's own circles;
//   * per-batch history (a ring of m pairs) and Gram matrix persist between
//     visits in the caller's workspace (L2-resident per instance).
// Results are bitwise reproducible: membership, list order and every sum
// are functions of the positions only.
//
// Bound by latency: a wave or two per SIMD on as many CUs as there are
// instances, whose visits are serial chains of LDS reads, global loads
// (history) and dependent arithmetic.  So loads that do not depend on each
// other are issued together (history, Gram matrix, six list neighbors of a
// circle, a thread's circles outside the visits), what a wave keeps in LDS is
// one array indexed by offsets (an access through a chosen pointer becomes a
// flat one, which waits for every counter), and the lists are built from mask
// bits.  Eight waves take up to eight batches of a colour at once, and share
// the lists, energies and moves; the instance's sums keep the order of four
// waves of four circles per thread.  64 instances of n = 1000 in 4 x 4 blocks,
// 300 outer iterations: 16.7 ms; with four waves 17.8 ms, and 24.5 ms with one
// load or neighbor at a time.  64 instances of n = 900 in 6 x 6 blocks, 100
// outer iterations: 7.05 ms, 10.5 ms with four waves.  Loading the next visit's
// history ahead gained under 1 % more (not kept).
// Neighbors per turn were chosen by time alone, at n = 1000 in 4 x 4 blocks: 16.9
// ms with three, 17.6 with four, 16.7 with six, 17.3 with eight, 18.3 with
// twelve (a list has five to twelve, so places past its end cost their terms,
// but that does not order these figures).  At two waves per SIMD a visit does
// not fit its 256 registers: 112 bytes per lane are spilled (with three to
// eight neighbors; 144 with twelve), 164 with FP64 sweeps; four waves of the
// same code had room for all of it.
#include "pecc_device.hpp"
#include "pecc_host.hpp"
#include "pecc_launch.hpp"
#include "pecc_lbfgs.hpp"

namespace pecc {

constexpr int kGT = 512;                    // threads per workgroup
constexpr int kGW = kGT / kWave;            // waves
constexpr int kGCPB = 2;                    // circles per lane inside a batch
constexpr int kGEll = 24;                   // neighbor slots per circle
constexpr int kMaxGboBatch = kWave * kGCPB; // circles per batch at most
constexpr int kMaxGboBatches = 64;          // blocks x blocks, blocks <= 8
constexpr int kGU = kMaxN / kGT;            // circles per thread outside the visits
constexpr int kGSum = 4;                    // waves whose order the instance's sums keep
constexpr int kInBatch = kMaxN * (int)sizeof(float2);      // list entries: the trial position
constexpr int kNowhere = 2 * kInBatch;                     // and the place beyond everything

constexpr int kTot = 2 * kNB * kNB;         // slot totals in a wave's array

struct GboShared {
    // positions at the start of the colour, trial positions of the visited
    // batches, a place beyond everything; a list entry is a byte offset here
    float2 xy[2 * kMaxN + 1];
    float2 npos[kMaxN];                     // positions after the colour
    float2 xref[kMaxN];                     // positions at the last rebuild
    int cell_start[kMaxCells + 1];
    uint16_t cell_circ[kMaxN];
    uint16_t slot_tmp[kMaxN];
    float2 psort[kMaxN + 8];                // positions in cell order
    uint16_t code[kMaxN];                   // and there, circle + batch << 10
    uint16_t list[kGEll][kMaxN];            // kInBatch set: a circle of the same batch
    uint8_t list_n[kMaxN];
    uint8_t batch_of[kMaxN];
    uint16_t members[kMaxN];                // circles grouped by batch, ascending
    int bstart[kMaxGboBatches + 1];
    uint8_t colour_batches[4][kMaxGboBatches];
    int ncolour[4];
    // per wave: Gram matrix, double-buffered, and the slot totals (one array,
    // so that an entry's source is an offset and every access stays an LDS one)
    alignas(8) float wave[kGW][kTot + kWave];
    float gn[4][kMaxGboBatches];            // gradient norms of the visits, by colour
    uint16_t bsrc[2][kNB * kNB];
    float redf[2][kGW], redg[2][kGSum];
    double redd[2][kGW];
    int scan_tmp[kGW + 1];
    int bk[kMaxGboBatches], bhead[kMaxGboBatches];   // pairs and ring position of every batch
    int evw[kGW];                           // per-wave evaluation counts at the end
    int flag, over, bad, work;
};

// Workspace of one instance: history S and Y (rings of kMM pairs of up to
// kMaxGboBatch circles) and Gram matrices of every batch.
__host__ __device__ inline size_t gbo_instance_bytes(int nbat)
{
    const size_t b = (size_t)nbat * (2 * (size_t)kMM * kMaxGboBatch * sizeof(float2) +
                                     (size_t)kNB * kNB * sizeof(float));
    return (b + 255) & ~(size_t)255;
}

// Neighbor lists at the current positions: the circles sorted into cells, and
// of every circle the neighbors (predicate near64 with c2) in the order of the
// cells.  Mask bits over the sorted positions (neighbor_masks), the two circles
// of a thread side by side; a wave with a circle that has more candidates than
// a mask holds goes through them one by one.  Returns whether some list is too long.
__device__ __forceinline__ bool gbo_build(GboShared &sh, int tid, int n, const Grid &grid, double c2)
{
    {
        float2 x[kGU];
        int own[kGU];
#pragma unroll
        for (int u = 0; u < kGU; ++u) x[u] = sh.xy[tid + u * kGT];
        sort_cells<kGT, kGU>(tid, x, n, grid, sh.cell_start, sh.cell_circ, sh.slot_tmp, sh.psort,
                             sh.scan_tmp, own);
#pragma unroll
        for (int u = 0; u < kGU; ++u)
            if (tid + u * kGT < n)
                sh.code[own[u]] = (uint16_t)(tid + u * kGT + (sh.batch_of[tid + u * kGT] << 10));
    }
    if (tid == 0) sh.over = 0;
    __syncthreads();
    bool over = false;
    float2 q[kGU];
    bool on[kGU], fits = true;
    int ci[kGU], bi[kGU], ra[kGU][3], rl[kGU][3], self[kGU], kmax[3] = {0, 0, 0};
#pragma unroll
    for (int e = 0; e < kGU; ++e) {
        const int s = tid + e * kGT;
        on[e] = s < n;
        q[e] = sh.psort[on[e] ? s : 0];
        const int code = sh.code[on[e] ? s : 0];
        ci[e] = code & 1023;
        bi[e] = code >> 10;
    }
#pragma unroll
    for (int e = 0; e < kGU; ++e) {
        cell_rows(q[e], on[e], tid + e * kGT, grid, sh.cell_start, ra[e], rl[e], self[e]);
        fits = fits && max(rl[e][0], max(rl[e][1], rl[e][2])) <= 32 && rl[e][0] + rl[e][1] + rl[e][2] <= 64;
#pragma unroll
        for (int r = 0; r < 3; ++r) kmax[r] = max(kmax[r], rl[e][r]);
    }
    // list entry of the circle of a code
    auto entry = [&](int code, int batch) {
        return (uint16_t)((code & 1023) * (int)sizeof(float2) + (code >> 10 == batch ? kInBatch : 0));
    };
    if (__builtin_amdgcn_ballot_w64(!fits)) {
#pragma unroll
        for (int e = 0; e < kGU; ++e) {
            if (!on[e]) continue;
            int m = 0;
            for (int r = 0; r < 3; ++r)
                for (int t = ra[e][r]; t < ra[e][r] + rl[e][r]; ++t) {
                    if (t == tid + e * kGT || !near64(q[e], sh.psort[t], c2)) continue;
                    if (m < kGEll) sh.list[m][ci[e]] = entry(sh.code[t], bi[e]);
                    ++m;
                }
            over = over || m > kGEll;
            sh.list_n[ci[e]] = (uint8_t)min(m, kGEll);
        }
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r) kmax[r] = wave_max_dpp(kmax[r]);
        unsigned long long mask[kGU];
        neighbor_masks<kGU, 4, kMaxN>(q, on, self, ra, rl, kmax, sh.psort, c2, mask);
        int cut[kGU], s1[kGU], s2[kGU], code[kGU], m = 0;
        bool has[kGU];
#pragma unroll
        for (int e = 0; e < kGU; ++e) {
            cut[e] = rl[e][0] + rl[e][1];
            s1[e] = ra[e][1] - rl[e][0];
            s2[e] = ra[e][2] - cut[e];
            const int cnt = __builtin_popcountll(mask[e]);
            over = over || cnt > kGEll;
            if (on[e]) sh.list_n[ci[e]] = (uint8_t)min(cnt, kGEll);
            m = max(m, cnt);
        }
        m = min(wave_max_dpp(m), kGEll);
        // the next neighbors' codes are read before the current ones are stored
#pragma unroll
        for (int e = 0; e < kGU; ++e)
            has[e] = next_neighbor(mask[e], rl[e][0], cut[e], ra[e][0], s1[e], s2[e], sh.code, code[e]);
        for (int k = 0; k < m; ++k) {
            int cur[kGU];
            bool put[kGU];
#pragma unroll
            for (int e = 0; e < kGU; ++e) { cur[e] = code[e]; put[e] = has[e]; }
#pragma unroll
            for (int e = 0; e < kGU; ++e)
                has[e] = next_neighbor(mask[e], rl[e][0], cut[e], ra[e][0], s1[e], s2[e], sh.code, code[e]);
#pragma unroll
            for (int e = 0; e < kGU; ++e)
                if (put[e]) sh.list[k][ci[e]] = entry(cur[e], bi[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < kGU; ++e)
        if (on[e]) sh.xref[ci[e]] = q[e];
    if (over) sh.over = 1;
    if (tid == 0) sh.flag = 0;
    __syncthreads();
    return sh.over != 0;
}

__device__ __forceinline__ float2 at_offset(const GboShared &sh, int byte_offset)
{
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(sh.xy) + byte_offset);
}

template <bool F64>
__global__ __launch_bounds__(kGT) void gbo_descend_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ Rv,
    const double *__restrict__ Rv64, float *__restrict__ xy, int B, int64_t total_n,
    DescentArgs A, int blocks, DescentResultDev *__restrict__ out, int32_t *__restrict__ queue,
    unsigned char *__restrict__ wsb)
{
    __shared__ GboShared sh;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = tid / kWave;
    const int nbat = blocks * blocks;
    for (int q = tid; q < 2 * kNB * kNB; q += kGT)
        sh.bsrc[q / (kNB * kNB)][q % (kNB * kNB)] = gram_source(q % (kNB * kNB), q >= kNB * kNB);
    if (tid == 0) sh.xy[2 * kMaxN] = make_float2(kFarCoord, kFarCoord);

    for (;;) {
        __syncthreads();
        if (tid == 0) sh.work = atomicAdd(&queue[0], 1);
        __syncthreads();
        const int slot = sh.work;
        if (slot >= B) break;
        const int b = queue[1 + slot];
        const int off = offset[b], n = offset[b + 1] - off;
        const float R = Rv[b];
        const double R64 = Rv64 ? Rv64[b] : (double)R;
        auto bad_instance = [&]() {
            if (tid == 0) {
                DescentHead r = {};
                r.status = 7;
                r.E32 = __builtin_nanf("");
                r.gnorm = __builtin_nanf("");
                r.E64 = -1.0;
                store_result(out, b, r, 0);
            }
        };
        if (!(off >= 0 && n >= 0 && n <= kMaxN && (int64_t)off + n <= total_n)) {
            bad_instance();
            continue;
        }
        const float rad = A.rad, two_r = 2.0f * rad, four_r2 = two_r * two_r;
        const double two_r64 = 2.0 * (double)rad, four_r2_64 = two_r64 * two_r64;
        const Grid grid = make_grid(R, A.h_req);
        unsigned char *wsi = wsb + (size_t)b * gbo_instance_bytes(nbat);
        float2 *histS = reinterpret_cast<float2 *>(wsi);
        float2 *histY = histS + (size_t)nbat * kMM * kMaxGboBatch;
        float *gram = reinterpret_cast<float *>(histY + (size_t)nbat * kMM * kMaxGboBatch);

        // ---- load, partition (FP64, from the input positions) ------------------
        if (tid == 0) { sh.bad = 0; sh.flag = 1; }
        for (int i = tid; i < n; i += kGT) {
            const float2 p = reinterpret_cast<const float2 *>(xy)[off + i];
            sh.xy[i] = p;
            sh.npos[i] = p;
            const double S = 2.0 * (double)R / blocks;
            const double tx = floor(((double)p.x + (double)R) / S), ty = floor(((double)p.y + (double)R) / S);
            int bx = tx >= 0.0 ? (tx < blocks - 1 ? (int)tx : blocks - 1) : 0;
            int by = ty >= 0.0 ? (ty < blocks - 1 ? (int)ty : blocks - 1) : 0;
            sh.batch_of[i] = (uint8_t)(by * blocks + bx);
        }
        for (int e = tid; e < nbat * kNB * kNB; e += kGT) gram[e] = 0.f;
        for (int p = tid; p < nbat; p += kGT) { sh.bk[p] = 0; sh.bhead[p] = 0; }
        for (int q = tid; q < 4 * kMaxGboBatches; q += kGT) sh.gn[q / kMaxGboBatches][q % kMaxGboBatches] = 0.f;
        __syncthreads();
        // members, ascending inside a batch: one thread per batch
        for (int p = tid; p < nbat; p += kGT) {
            int c = 0;
            for (int i = 0; i < n; ++i) c += sh.batch_of[i] == p;
            sh.bstart[p + 1] = c;
        }
        __syncthreads();
        if (tid == 0) {
            sh.bstart[0] = 0;
            for (int p = 0; p < nbat; ++p) {
                sh.bstart[p + 1] += sh.bstart[p];
                if (sh.bstart[p + 1] - sh.bstart[p] > kMaxGboBatch) sh.bad = 1;
            }
            for (int c = 0; c < 4; ++c) sh.ncolour[c] = 0;
            for (int p = 0; p < nbat; ++p) {
                if (sh.bstart[p + 1] == sh.bstart[p]) continue;
                const int c = (p % blocks & 1) + 2 * ((p / blocks) & 1);
                sh.colour_batches[c][sh.ncolour[c]++] = (uint8_t)p;
            }
        }
        __syncthreads();
        for (int p = tid; p < nbat; p += kGT) {
            int w = sh.bstart[p];
            for (int i = 0; i < n; ++i)
                if (sh.batch_of[i] == p) sh.members[w++] = (uint16_t)i;
        }
        __syncthreads();
        if (sh.bad) {   // a batch larger than kMaxGboBatch circles
            bad_instance();
            continue;
        }

        int rebuilds = 0, evals = 0, status = 0, outer = 0;
        int cell_mine = 0;      // this wave's evaluations over the cell grid
        int64_t pair_mine = 0;
        bool overflow = false;
        double ehist = 0.0, E64t = -1.0;
        float Ew = 0.f, gs_all = 0.f;
        const int window = A.ftol_window;

        constexpr int kGramTurns = (kNB * kNB + kWave - 1) / kWave;
        // entry of a turn; the last turn's spare lanes repeat the last entry
        auto gram_entry = [&](int t) { return min(lane + t * kWave, kNB * kNB - 1); };
        // A turn is a colour; the energies and stop tests come before colour 0.
        for (int colour = 0;; colour = (colour + 1) & 3) {
            // ---- neighbor lists at the current positions when flagged -------------
            if (sh.flag) {
                overflow = gbo_build(sh, tid, n, grid, A.c2);
                ++rebuilds;
            }

            // ---- whole-instance energies and the stop tests ------------------------
            if (colour == 0) {
                float *const e_of = &sh.wave[0][0];
                double *const et_of = reinterpret_cast<double *>(e_of + kMaxN);
                static_assert(sizeof(sh.wave) >= kMaxN * (sizeof(float) + sizeof(double)), "energies fit the scratch");
                float2 qv[kGU];
                float ec[kGU];
                double etc[kGU];
                int mc[kGU], mmax = 0;
#pragma unroll
                for (int u = 0; u < kGU; ++u) {
                    const int i = tid + u * kGT;
                    qv[u] = sh.xy[i];
                    mc[u] = i < n ? sh.list_n[i] : 0;
                    mmax = max(mmax, mc[u]);
                    ec[u] = 0.f;
                    etc[u] = 0.0;
                }
                // every pair once, at its lower circle; a thread's two circles
                // side by side, two neighbors each in flight (a neighbor that
                // does not count stands beyond everything and adds zeros)
                auto visit_pair = [&](float2 q, float2 pj, float &ecu, double &etu) {
                    float e1 = 0.f, gx = 0.f, gy = 0.f;
                    double eo = 0.0;
                    pair_term32(q, pj, true, two_r, four_r2, ecu, e1, gx, gy);
                    const float l2 = dot2(q.x - pj.x, q.x - pj.x, q.y - pj.y, q.y - pj.y);
                    const float il = l2 > 0.f ? __builtin_amdgcn_rsqf(l2) : 0.f;
                    pair_term64s(q, pj, l2 * il, il, two_r64, four_r2_64, eo, etu);
                };
                if (!overflow) {
                    mmax = wave_max_dpp(mmax);
                    for (int t0 = 0; t0 < mmax; t0 += 2) {
                        int o[2][kGU];
                        float2 pj[2][kGU];
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int u = 0; u < kGU; ++u) o[t][u] = sh.list[t0 + t][tid + u * kGT];
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int u = 0; u < kGU; ++u) {
                                const int j = o[t][u] & ~kInBatch;
                                const bool use = t0 + t < mc[u] && j > (tid + u * kGT) * (int)sizeof(float2);
                                pj[t][u] = at_offset(sh, use ? j : kNowhere);
                            }
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int u = 0; u < kGU; ++u) visit_pair(qv[u], pj[t][u], ec[u], etc[u]);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < kGU; ++u) {
                        const int i = tid + u * kGT;
                        if (i < n)
                            for_each_candidate(i, qv[u], grid, sh.cell_start, sh.cell_circ, [&](int j) {
                                if (j > i) visit_pair(qv[u], sh.xy[j], ec[u], etc[u]);
                            });
                    }
                }
#pragma unroll
                for (int u = 0; u < kGU; ++u) {
                    const float2 q = qv[u];
                    const float r2 = q.x * q.x + q.y * q.y;
                    const float ir = r2 > 0.f ? __builtin_amdgcn_rsqf(r2) : 0.f;
                    const float d0 = fmaxf(r2 * ir + rad - R, 0.f);
                    ec[u] += d0 * d0;
                    const double r64 = sqrt(dot2((double)q.y, (double)q.y, (double)q.x, (double)q.x));
                    const double ct = r64 + 1.0 - R64;
                    if (ct > 0.0) etc[u] += ct * ct;
                    if (!(isfinite(q.x) && isfinite(q.y))) { ec[u] = __builtin_nanf(""); etc[u] = __builtin_nan(""); }
                    // (the waves' scratch is free here)
                    const bool on = tid + u * kGT < n;
                    e_of[tid + u * kGT] = on ? ec[u] : 0.f;
                    et_of[tid + u * kGT] = on ? etc[u] : 0.0;
                }
                __syncthreads();
                const int par = outer & 1;
                if (wv < kGSum) {
                    // the sums of 256 threads of four circles each, and of the
                    // visits of four waves, whatever the workgroup's size
                    float e = 0.f, gs = 0.f;
                    double et = 0.0;
#pragma unroll
                    for (int q = 0; q < kMaxN / (kGSum * kWave); ++q) {
                        e += e_of[tid + q * kGSum * kWave];
                        et += et_of[tid + q * kGSum * kWave];
                    }
                    for (int c = 0; c < 4; ++c)
                        for (int r = wv; r < sh.ncolour[c]; r += kGSum) gs += sh.gn[c][r];
                    e = wave_sum(e);
                    et = wave_sum(et);
                    if (lane == 0) {
                        sh.redf[par][wv] = e;
                        sh.redd[par][wv] = et;
                        sh.redg[par][wv] = gs;
                    }
                }
                __syncthreads();
                Ew = 0.f;
                float gs = 0.f;
                double ett = 0.0;
#pragma unroll
                for (int w = 0; w < kGSum; ++w) {
                    Ew += sh.redf[par][w];
                    ett += sh.redd[par][w];
                    gs += sh.redg[par][w];
                }
                gs_all = gs;
                E64t = ett;
                const double Eacc = (double)Ew;
                if (!isfinite(Ew)) { status = 6; break; }
                if (E64t < A.e_feasible) { status = 1; break; }
                if (outer > 0 && gs <= A.g_tol) { status = 2; break; }
                if (A.ftol > 0.f && outer >= window) {
                    const int src = (outer - window) % (window + 1);
                    const long long bits = __builtin_bit_cast(long long, ehist);
                    const int lo = __builtin_amdgcn_readlane((int)(bits & 0xffffffffLL), src);
                    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), src);
                    const double eold = __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
                    if (eold - Eacc <= (double)A.ftol * eold) { status = 3; break; }
                }
                if (lane == outer % (window + 1)) ehist = Eacc;
                if (outer >= A.max_iter) { status = 5; break; }
                ++outer;
            }

            // ---- the colour's batches ---------------------------------------------
            {
                for (int r = wv; r < sh.ncolour[colour]; r += kGW) {
                    const int p = sh.colour_batches[colour][r];
                    const int m0 = sh.bstart[p], np = sh.bstart[p + 1] - m0;
                    // ---- visit batch p: registers <- its circles and history --
                    int k = __builtin_amdgcn_readfirstlane(sh.bk[p]);
                    int head = __builtin_amdgcn_readfirstlane(sh.bhead[p]);
                    bool act[kGCPB];
                    int ci[kGCPB];
                    float2 x[kGCPB], g[kGCPB], pd[kGCPB];
                    // history and Gram matrix, every load in flight (a slot that
                    // holds no pair is read and dropped; the second circles'
                    // only where the batch has them)
                    float2 S[kGCPB][kMM] = {}, Y[kGCPB][kMM] = {};
                    float gv[kGramTurns];
                    {
                        const float2 *hS = histS + (size_t)p * kMM * kMaxGboBatch;
                        const float2 *hY = histY + (size_t)p * kMM * kMaxGboBatch;
                        const float *gp = gram + (size_t)p * kNB * kNB;
#pragma unroll
                        for (int t = 0; t < kGramTurns; ++t) gv[t] = gp[gram_entry(t)];
#pragma unroll
                        for (int c = 0; c < kGCPB; ++c) {
                            if (c * kWave >= np) break;
#pragma unroll
                            for (int j = 0; j < kMM; ++j) {
                                // logical j (newest at kMM-1) is ring slot head - (kMM-1-j)
                                const int sl = head - (kMM - 1 - j) + (head < kMM - 1 - j ? kMM : 0);
                                S[c][j] = hS[(size_t)sl * kMaxGboBatch + lane + c * kWave];
                                Y[c][j] = hY[(size_t)sl * kMaxGboBatch + lane + c * kWave];
                            }
                        }
                    }
#pragma unroll
                    for (int c = 0; c < kGCPB; ++c) {
                        const int q = lane + c * kWave;
                        act[c] = q < np;
                        ci[c] = act[c] ? sh.members[m0 + q] : 0;
                        x[c] = act[c] ? sh.xy[ci[c]] : make_float2(0.f, 0.f);
                        g[c] = make_float2(0.f, 0.f);
                        pd[c] = make_float2(0.f, 0.f);
                    }
#pragma unroll
                    for (int c = 0; c < kGCPB; ++c)
#pragma unroll
                        for (int j = 0; j < kMM; ++j) {
                            const bool valid = act[c] && j >= kMM - k;
                            S[c][j] = valid ? S[c][j] : make_float2(0.f, 0.f);
                            Y[c][j] = valid ? Y[c][j] : make_float2(0.f, 0.f);
                        }
                    float *const W = sh.wave[wv];
                    int cur = 0;            // offset of the current Gram matrix
#pragma unroll
                    for (int t = 0; t < kGramTurns; ++t) W[gram_entry(t)] = gv[t];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

                    // one evaluation of the batch energy (Eq. 7) at xt: returns the
                    // slot total of this lane; gt gets the batch gradient
                    float Ep = 0.f;
                    double Ep64 = 0.0;
                    auto evaluate = [&](const float2 (&xt)[kGCPB], const float2 (&sc)[kGCPB],
                                        float2 (&gt)[kGCPB], float2 (&yc)[kGCPB], double &e64,
                                        bool far) -> float {
#pragma unroll
                        for (int c = 0; c < kGCPB; ++c)
                            if (act[c]) sh.xy[kMaxN + ci[c]] = xt[c];
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        float e = 0.f, e1_unused = 0.f;
                        double ed = 0.0;
                        int pe = 0;
#pragma unroll
                        for (int c = 0; c < kGCPB; ++c) {
                            float gx = 0.f, gy = 0.f;
                            double gxd = 0.0, gyd = 0.0;
                            {
                                const int i = ci[c];
                                const float2 q = xt[c];
                                auto term_at = [&](float2 pj, bool ce) {
                                    pe += ce;
                                    if (F64) {
                                        const double dx = (double)q.x - (double)pj.x;
                                        const double dy = (double)q.y - (double)pj.y;
                                        const double l2 = dx * dx + dy * dy;
                                        if (l2 < four_r2_64) {
                                            const double l = sqrt(l2);
                                            const double d = two_r64 - l;
                                            if (ce) ed += d * d;
                                            if (l > 0.0) {
                                                const double kf = -2.0 * d / l;
                                                gxd += kf * dx;
                                                gyd += kf * dy;
                                            }
                                        }
                                    } else {
                                        pair_term32(q, pj, ce, two_r, four_r2, e, e1_unused, gx, gy);
                                    }
                                };
                                auto term = [&](int j) {
                                    const bool inb = sh.batch_of[j] == p;
                                    term_at(sh.xy[j + (inb ? kMaxN : 0)], inb ? j < i : true);   // Eq. 7
                                };
                                if (c * kWave < np && !far && !overflow) {
                                    // the wave's longest list, six neighbors in
                                    // flight; past a list's end a place that adds
                                    // zeros
                                    const int mc = act[c] ? sh.list_n[i] : 0;
                                    const int mmax = wave_max_dpp(mc);
                                    constexpr int kTurn = 6;
                                    static_assert(kGEll % kTurn == 0, "whole turns");
                                    for (int t0 = 0; t0 < mmax; t0 += kTurn) {
                                        int o[kTurn];
                                        float2 pj[kTurn];
#pragma unroll
                                        for (int t = 0; t < kTurn; ++t) o[t] = sh.list[t0 + t][i];
#pragma unroll
                                        for (int t = 0; t < kTurn; ++t) {
                                            o[t] = t0 + t < mc ? o[t] : kNowhere;
                                            pj[t] = at_offset(sh, o[t]);
                                        }
#pragma unroll
                                        for (int t = 0; t < kTurn; ++t)      // Eq. 7: a pair of the batch once
                                            term_at(pj[t], o[t] < kInBatch + i * (int)sizeof(float2));
                                    }
                                }
                                if (act[c] && (far || overflow)) {
                                    // lists that do not fit: all circles from the cell
                                    // grid.  A circle of the batch that left the skin:
                                    // the other circles from the cell grid, the batch's
                                    // own from its member list
                                    for_each_candidate(i, q, grid, sh.cell_start, sh.cell_circ, [&](int j) {
                                        if (!far || sh.batch_of[j] != p) term(j);
                                    });
                                    for (int t = 0; t < (far ? np : 0); ++t) {
                                        const int j = sh.members[m0 + t];
                                        if (j != i) term(j);
                                    }
                                }
                            }
                            if (act[c]) {
                                const float2 q = xt[c];
                                if (F64) {
                                    const double r64 = sqrt((double)q.x * q.x + (double)q.y * q.y);
                                    const double d0 = r64 + (double)rad - R64;
                                    if (d0 > 0.0) {
                                        ed += d0 * d0;
                                        if (r64 > 0.0) {
                                            gxd += 2.0 * d0 * q.x / r64;
                                            gyd += 2.0 * d0 * q.y / r64;
                                        }
                                    }
                                    gx = (float)gxd;
                                    gy = (float)gyd;
                                } else {
                                    const float r2 = q.x * q.x + q.y * q.y;
                                    const float ir = r2 > 0.f ? __builtin_amdgcn_rsqf(r2) : 0.f;
                                    const float d0 = fmaxf(r2 * ir + rad - R, 0.f);
                                    e += d0 * d0;
                                    const float kc = 2.f * d0 * ir;
                                    gx += kc * q.x;
                                    gy += kc * q.y;
                                }
                                if (!(isfinite(q.x) && isfinite(q.y))) {
                                    e = __builtin_nanf("");
                                    ed = __builtin_nan("");
                                }
                            }
                            gt[c] = make_float2(gx, gy);
                            yc[c] = make_float2(gx - g[c].x, gy - g[c].y);
                        }
                        if (F64) e = (float)ed;
                        e64 = F64 ? wave_sum(ed) : 0.0;
                        ++evals;
                        cell_mine += (far || overflow) ? 1 : 0;
                        pair_mine += pe;
                        return wave_reduce_scatter<false>(gt, sc, yc, S, Y, e, 0.f);
                    };

                    auto gram_update = [&](bool push) {
                        int src[kGramTurns];
                        float v[kGramTurns];
#pragma unroll
                        for (int t = 0; t < kGramTurns; ++t) src[t] = sh.bsrc[push ? 1 : 0][gram_entry(t)];
#pragma unroll
                        for (int t = 0; t < kGramTurns; ++t) {
                            v[t] = W[(src[t] & 0x8000) ? kTot + (src[t] & 0x7fff) : cur + src[t]];
                        }
#pragma unroll
                        for (int t = 0; t < kGramTurns; ++t) W[kNB * kNB - cur + gram_entry(t)] = v[t];
                        cur = kNB * kNB - cur;
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    };
                    // ---- the gradient at the start of the visit (Alg. 1), then the
                    // backtracking line search on E(x_p), over one copy of the
                    // evaluation ----------------------------------------------------
                    bool accepted = false, push = false;
                    float2 xt[kGCPB], sc[kGCPB], gt[kGCPB], yc[kGCPB];
                    double e64 = 0.0;
                    float gp = 0.f, alpha = 0.f;
#pragma unroll
                    for (int c = 0; c < kGCPB; ++c) { xt[c] = x[c]; sc[c] = make_float2(0.f, 0.f); }
                    // (every circle starts a colour within skin / 2 of its list
                    // position, so the visit's first point is in range of the lists)
                    bool far = false;
                    for (int h = -1;;) {
                        const float tot = evaluate(xt, sc, gt, yc, e64, far);
                        // slot totals are lane-indexed by lane_slot(); stage them
                        W[kTot + lane_slot(lane)] = tot;
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        if (h >= 0) {
                            const float Et = W[kTot + sE];
                            const bool ok = F64 ? e64 <= Ep64 + (double)A.c1 * (double)alpha * (double)gp
                                                : Et <= Ep + A.c1 * alpha * gp;
                            if (ok) {
                                accepted = true;
                                push = W[kTot + sScYc] > A.eps_curv * W[kTot + sYcYc];
                            }
                        }
                        if (h < 0 || accepted) gram_update(push);
                        if (accepted) break;
                        if (h < 0) {
                            Ep = W[kTot + sE];
                            Ep64 = e64;
#pragma unroll
                            for (int c = 0; c < kGCPB; ++c) g[c] = gt[c];
                            const float gg = W[cur + kG * kNB + kG];
                            const float gn = sqrtf(fmaxf(gg, 0.f));
                            if (lane == 0) sh.gn[colour][r] = gn;

                            // ---- direction: two-loop on the batch's Gram matrix -----------
                            float Bc[kNB];
#pragma unroll
                            for (int a2 = 0; a2 < kNB; ++a2) Bc[a2] = W[cur + a2 * kNB + min(lane, kNB - 1)];
#pragma unroll
                            for (int a2 = 0; a2 < kNB; ++a2) Bc[a2] = lane < kNB ? Bc[a2] : 0.f;
                            // two-loop on the Gram matrix: lane l keeps (B q)_l, the Gram
                            // product of the current q with basis vector l (q = g at the
                            // start), so each step is one readlane and one FMA
                            const int jp = lane < kMM ? lane : lane - kMM;
                            const bool live = lane < 2 * kMM && jp >= kMM - k;
                            float rho_v = 0.f;              // 1 / s_j'y_j at lanes j and kMM + j
                            if (live) rho_v = 1.f / W[cur + (lane < kMM ? kMM + lane : lane - kMM) * kNB + lane];
                            float acc = Bc[kG];
                            float cf = 0.f;                 // a_j at lane kMM + j, coefficient of s_j at lane j
                            two_loop_down(Bc + kMM, rho_v, acc, cf);               // a_j = rho_j s_j'q
                            float gam = 1.f;
                            if (k > 0) gam = lane_value(Bc[kMM - 1], 2 * kMM - 1) / lane_value(Bc[2 * kMM - 1], 2 * kMM - 1);
                            acc *= gam;
                            two_loop_up(Bc, rho_v, acc, cf);                       // a_j - rho_j y_j'r
                            gp = -lane_value(acc, kG);                               // g'p = -g'r
                            {
                                float cs[kMM], cy[kMM];
#pragma unroll
                                for (int j = 0; j < kMM; ++j) { cs[j] = lane_value(cf, j); cy[j] = -gam * lane_value(cf, kMM + j); }
#pragma unroll
                                for (int c = 0; c < kGCPB; ++c) {
                                    float px = -gam * g[c].x, py = -gam * g[c].y;
#pragma unroll
                                    for (int j = 0; j < kMM; ++j) {
                                        px -= cs[j] * S[c][j].x + cy[j] * Y[c][j].x;
                                        py -= cs[j] * S[c][j].y + cy[j] * Y[c][j].y;
                                    }
                                    pd[c] = make_float2(px, py);
                                }
                            }
                            if (k > 0 && !(gp < 0.f)) {
                                k = 0;
#pragma unroll
                                for (int c = 0; c < kGCPB; ++c) pd[c] = make_float2(-g[c].x, -g[c].y);
                                gp = -gg;
                            }
                            alpha = k > 0 ? 1.f : 1.f / fmaxf(1.f, gn);
                        } else {
                            alpha *= 0.5f;
                        }
                        if (++h > A.max_halvings) break;
                        bool out = false;
#pragma unroll
                        for (int c = 0; c < kGCPB; ++c) {
                            xt[c] = make_float2(fmaf(alpha, pd[c].x, x[c].x), fmaf(alpha, pd[c].y, x[c].y));
                            sc[c] = make_float2(xt[c].x - x[c].x, xt[c].y - x[c].y);
                            if (act[c]) {
                                const float2 rf = sh.xref[ci[c]];
                                const double dx = (double)xt[c].x - (double)rf.x, dy = (double)xt[c].y - (double)rf.y;
                                out |= dx * dx + dy * dy > A.skin2;
                            }
                        }
                        far = __builtin_amdgcn_ballot_w64(out) != 0;
                    }
                    if (accepted) {
                        if (push) {
                            const int sl = (head + 1) % kMM;
#pragma unroll
                            for (int c = 0; c < kGCPB; ++c) {
                                const int q = lane + c * kWave;
                                if (act[c]) {
                                    histS[((size_t)p * kMM + sl) * kMaxGboBatch + q] = sc[c];
                                    histY[((size_t)p * kMM + sl) * kMaxGboBatch + q] = yc[c];
                                }
                            }
                            head = sl;
                            k = k + 1 > A.m ? A.m : k + 1;
                        }
#pragma unroll
                        for (int c = 0; c < kGCPB; ++c)
                            if (act[c]) sh.npos[ci[c]] = xt[c];
                    }
                    // ---- persist the batch's Gram matrix and ring ----------------
                    float *gdst = gram + (size_t)p * kNB * kNB;
#pragma unroll
                    for (int t = 0; t < kGramTurns; ++t) gdst[gram_entry(t)] = W[cur + gram_entry(t)];
                    if (lane == 0) { sh.bk[p] = k; sh.bhead[p] = head; }
                }
                // ---- end of the colour: commit, maybe rebuild --------------------
                __syncthreads();
                int moved = 0;
                {
                    float2 q[kGU], rf[kGU];
#pragma unroll
                    for (int u = 0; u < kGU; ++u) {
                        q[u] = sh.npos[tid + u * kGT];
                        rf[u] = sh.xref[tid + u * kGT];
                    }
#pragma unroll
                    for (int u = 0; u < kGU; ++u) {
                        if (tid + u * kGT >= n) continue;
                        sh.xy[tid + u * kGT] = q[u];
                        const double dx = (double)q[u].x - (double)rf[u].x, dy = (double)q[u].y - (double)rf[u].y;
                        moved |= dx * dx + dy * dy > 0.25 * A.skin2;
                    }
                }
                if (moved) sh.flag = 1;
                __syncthreads();
            }
        }

        // ---- write back ----------------------------------------------------------
        for (int i = tid; i < n; i += kGT) reinterpret_cast<float2 *>(xy)[off + i] = sh.xy[i];
        {
            unsigned long long pm = (unsigned long long)pair_mine;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) pm += __shfl_xor(pm, o, kWave);
            __syncthreads();
            if (lane == 0) sh.redd[0][wv] = __builtin_bit_cast(double, pm);
            __syncthreads();
            pm = 0;
            for (int w = 0; w < kGW; ++w) pm += __builtin_bit_cast(unsigned long long, sh.redd[0][w]);
            pair_mine = (int64_t)pm;
        }
        {
            // every wave's batch evaluations, and those over the cell grid
            __syncthreads();
            if (lane == 0) { sh.scan_tmp[wv] = cell_mine; sh.evw[wv] = evals; }
            __syncthreads();
            cell_mine = 0;
            evals = 0;
            for (int w = 0; w < kGW; ++w) {
                cell_mine += sh.scan_tmp[w];
                evals += sh.evw[w];
            }
        }
        if (tid == 0) {
            DescentHead r;
            r.status = status;
            r.iters = outer;
            r.evals = evals;
            r.rebuilds = rebuilds;
            r.pair_evals = pair_mine;
            r.E32 = Ew;
            r.gnorm = gs_all;
            r.E64 = E64t;
            store_result(out, b, r, cell_mine);
        }
    }
}

size_t gbo_workspace_bytes(int B, int blocks)
{
    return sizeof(int32_t) * ((size_t)B + 1 + 64) + (size_t)B * gbo_instance_bytes(blocks * blocks);
}

int gbo_grid(int B)
{
    const int cus = current_device_cus();
    return B < cus ? B : cus;
}

hipError_t launch_queue_init(const int32_t *offset, int B, int32_t *queue, hipStream_t s);

hipError_t launch_gbo(const int32_t *offset, const float *R, const double *R64, float *xy, int B,
                      int64_t total_n, const DescentArgs &a, int blocks, int sweep_fp64, void *out,
                      void *ws, hipStream_t s)
{
    int32_t *queue = reinterpret_cast<int32_t *>(ws);
    unsigned char *wsb = reinterpret_cast<unsigned char *>(ws) +
                         ((sizeof(int32_t) * ((size_t)B + 1 + 64) + 255) & ~(size_t)255);
    hipError_t e = launch_queue_init(offset, B, queue, s);
    if (e != hipSuccess) return e;
    const int grid = gbo_grid(B);
    if (sweep_fp64)
        gbo_descend_kernel<true><<<grid, kGT, 0, s>>>(offset, R, R64, xy, B, total_n, a, blocks,
                                                      reinterpret_cast<DescentResultDev *>(out), queue, wsb);
    else
        gbo_descend_kernel<false><<<grid, kGT, 0, s>>>(offset, R, R64, xy, B, total_n, a, blocks,
                                                       reinterpret_cast<DescentResultDev *>(out), queue, wsb);
    return hipGetLastError();
}

}  // namespace pecc
