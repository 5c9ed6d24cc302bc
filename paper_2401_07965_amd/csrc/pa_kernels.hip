// HIP kernels of the population-annealing hot path for gfx950 (MI355X).
//
// Spins are multi-spin coded: bit b of word [w][s] is replica 64w+b at site s,
// 1 meaning sigma = -1.  One workgroup owns one 64-replica word column: the
// whole lattice of its 64 replicas (N words) sits in LDS while it is swept.
//
// Every kernel serves a batch of runs through a block map (PaBlk: run, index
// within the run); a run's population size, ping-pong index, temperature and
// step are read from its device record, so launches need no host knowledge
// of the state and a whole anneal can be captured in a graph.  Grids cover
// each run's capacity; workgroups past the live population return at once.
#include "pa_sweep.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>

namespace {

// ------------------------------------------------------------------ helpers
__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

int grid_for(int64_t n, int threads = kThreads, int cap = 4096)
{
    int64_t g = (n + threads - 1) / threads;
    if (g < 1)
        g = 1;
    return (int)(g > cap ? cap : g);
}

// ------------------------------------------------------------------ step 1: init
// Record of a fresh run at beta_0 = 0: ln Z_0 = N ln 2, every move accepted.
__global__ void k_init_rec(const PaRunDesc *__restrict__ runs)
{
    const PaRunDesc &rd = runs[blockIdx.x];
    for (int k = threadIdx.x; k < PA_CALL_SLOTS; k += blockDim.x)
        rd.dv.calls[k] = 0;
    if (threadIdx.x != 0)
        return;
    PaRecord *rec = rd.dv.rec;
    rec->cur = 0;
    rec->status = 0;
    rec->skip = 0;
    rec->step = 0;
    rec->sweeps = 0;
    rec->gather = 0;
    rec->Rcur = (uint64_t)rd.R0;
    rec->beta = 0.0;
    rec->lnQ = 0.0;
    rec->lnZ = (double)rd.N * 0x1.62e42fefa39efp-1; // N * RN(ln 2)
    rec->sv = 0.0;
    for (int k = 0; k < 3; ++k)
        rec->T[k] = rec->Tn[k] = 1ull << 32;
    rec->site_updates = 0;
    rec->attempts = 0;
    rec->accE = rec->accE2 = rec->accAbsM = rec->accM2 = rec->accC2 = rec->accFam = 0;
    rec->accE3[0] = rec->accE3[1] = 0;
    rec->lnq_hist[0] = rec->lnq_hist[1] = rec->lnq_hist[2] = 0.0;
    rec->S_f = log((double)rd.R0);
    rec->weighted = 0;
    rec->keep = 0;
    rec->resamplings = 0;
    rec->ess = (double)rd.R0;
}

// The site words of the sweeps' table walk: word c N/2 + k is site k of colour
// c (row = y + L z = k div (L/2), x = 2 (k mod L/2) + (y + z + c) mod 2).
// Workgroups (run, kThreads sites): one for a run's whole table kept the
// creation of a 2D L = 128 run waiting, with couplings 252 -> 227 us.
__global__ __launch_bounds__(kThreads) void k_sites(const PaRunDesc *__restrict__ runs)
{
    const PaRunDesc &rd = runs[blockIdx.x];
    const int L = rd.L, half = L >> 1, nh = rd.N >> 1;
    const int i = blockIdx.y * blockDim.x + threadIdx.x;
    if (i < rd.N) {
        const int c = i >= nh ? 1 : 0, k = i - c * nh;
        const int row = k / half, z = row / L, y = row - z * L;
        const int x = 2 * (k - row * half) + ((y + z + c) & 1), s = x + L * row;
        rd.dv.sites[i] = site_word(s, rd.J ? (uint32_t)rd.dv.jmask[s] : 0u, x, y, L);
    }
}

// Replica 64w+b, site s: bit b of x0 | x1<<32 of Philox(s, w, 0, INIT<<28).
__global__ __launch_bounds__(kThreads) void k_init_spins(const PaRunDesc *__restrict__ runs,
                                                         const PaBlk *__restrict__ map)
{
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    const uint32_t w = b.idx;
    if ((int64_t)w * 64 >= rd.R0)
        return;
    uint64_t *g = rd.dv.spins[0] + (size_t)w * rd.N;
    for (int s = threadIdx.x; s < rd.N; s += blockDim.x) {
        const pa_philox_out o = pa_philox(rd.seed, rd.run_id, (uint32_t)s, w, 0u, PA_PURPOSE_INIT << 28);
        g[s] = (uint64_t)o.x0 | ((uint64_t)o.x1 << 32);
    }
}

__global__ __launch_bounds__(kThreads) void k_init_labels(const PaRunDesc *__restrict__ runs,
                                                          const PaBlk *__restrict__ map)
{
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    const int64_t beg = (int64_t)b.idx * PA_CHUNK;
    for (int64_t j = beg + threadIdx.x; j < beg + PA_CHUNK && j < rd.R0; j += blockDim.x) {
        rd.dv.label[0][j] = (uint32_t)j;
        rd.dv.fam[j] = 0; // family counts start at zero; k_obs_fam returns them to zero
    }
}


// ------------------------------------------------------------------ cluster updates
// The cluster-update driver (Sec. 1 names cluster updates among the update
// algorithms the scheme can use): nsteps Wolff single-cluster updates of
// every replica at the run's current beta.  For replica b of column w at
// (step i, update t):
//  - seed site floor(x0 N / 2^32), x0 of Philox(b, w, i, WSEED<<28 | t<<8);
//  - bond (s, mu) to s + e_mu active iff satisfied and u < T_p, T_p =
//    min(2^32, floor(2^32 (1 - pa_exp(-2 beta)))), u's bits from the planes
//    of Philox(s, w, i, WBOND<<28 | t<<8 | mu<<4 | q), q = 0..15, decided
//    from the most significant bit as for the Metropolis thresholds;
//  - the cluster is every site joined to the seed by active bonds; it flips.
// Every bond's activity is decided first, for all 64 replicas of its owner's
// word at once (a replica's bond depends on its counters and threshold alone,
// not on when the cluster reaches it), so the growth itself draws nothing: it
// floods the active bonds until no word changes.  The component does not
// depend on the order of growth.
//
// What bounds it: the decisions are VALU (Philox, about a sweep's work), the
// growth the number of passes, as many as the deepest of the 64 clusters
// needs, times a pass's LDS reads and logic.  So a lane owns a patch of PX PY
// PZ sites and keeps their cluster words and bonds in registers; a pass reads
// the words around the patch, floods the patch forwards and backwards and
// writes what changed.  At the 2D critical point (L = 64) the deepest cluster
// is about 230 bonds deep: some 57 passes with patches of 4 x 4 against 150
// with strips of 4 and 230 site by site.  Waves do not wait for each other
// between passes (words only gain bits, so an old one costs a pass and no
// more); every kGrowPasses-th pass ends at a barrier that tells whether any
// word changed.  Two words per site of LDS, so two workgroups share a CU at
// N = 4096.
// 2D L = 64, R = 10^5 at the critical point, per update: 8.2 ms with bonds
// decided as the growth reached them and a barrier a pass, 1.29 ms with strips of
// four, 0.45 ms now.  Two or eight passes to a barrier ran 3 % and 1 % slower.
constexpr int kGrowPasses = 4;

// Most lanes of a workgroup: N <= 4096 sites in patches of 16, of 4 (2D) or of 8 (3D); twice as many
// as there can be patches of 16 for the decisions of few columns (cluster_launch).
constexpr int cluster_lanes(int d, int patch) { return patch == 16 ? 512 : (d == 2 ? 1024 : 512); }

// T_p at the run's beta.
__device__ __forceinline__ uint64_t wolff_threshold(const PaRecord *rec)
{
    const double p = 1.0 - pa_exp(-(2.0 * rec->beta));
    const double tf = floor(ldexp(p, 32));
    uint64_t T = (uint64_t)tf;
    if (T > (1ull << 32))
        T = 1ull << 32;
    return uni64(T);
}

// The seed site of replica b.
__device__ __forceinline__ uint32_t wolff_seed(const PlaneCtx &pc, uint32_t b, int N)
{
    const pa_philox_out o =
        pa_philox(pc.seed, pc.run_id, b, pc.w, pc.step, (PA_PURPOSE_WSEED << 28) | (pc.t << 8));
    return (uint32_t)(((uint64_t)o.x0 * (uint64_t)N) >> 32);
}

// Activity of bond (owner, mu) for the replicas in cnd.
__device__ __forceinline__ uint64_t wolff_bond(const PlaneCtx &pc, uint32_t owner, uint32_t mu, uint64_t cnd,
                                               uint64_t T)
{
    if (T >= (1ull << 32))
        return cnd;
    if (T == 0)
        return 0;
    constexpr int kFirst = 3; // as the sweeps: nearly every word needs three pairs, their chains interleaved
    const uint32_t x3 = (PA_PURPOSE_WBOND << 28) | (pc.t << 8) | (mu << 4);
    const pa_philox_shared sh = pa_philox_share(pc.seed, pc.run_id, owner, pc.w, pc.step);
    uint64_t und = cnd, acc = 0;
    pa_philox_out o[kFirst];
    pa_philox_k<kFirst>(pc.seed, pc.run_id, sh, pc.w, pc.step, x3, o);
#pragma unroll
    for (int q = 0; q < kFirst; ++q)
        pair_core<false>(o[q], tbit((uint32_t)T, 31 - 2 * q), tbit((uint32_t)T, 30 - 2 * q), und, und, acc);
    for (uint32_t q = kFirst; q < 16u && und != 0; ++q) {
        const int b0 = 31 - 2 * (int)q;
        pair_core<false>(pa_philox_with(pc.seed, pc.run_id, sh, pc.w, pc.step, x3 | q), tbit((uint32_t)T, b0),
                         tbit((uint32_t)T, b0 - 1), und, und, acc);
    }
    return acc;
}

// The same for replica b alone.
__device__ __forceinline__ bool wolff_bond_of(const PlaneCtx &pc, uint32_t owner, uint32_t mu, uint32_t b, uint64_t T)
{
    if (T >= (1ull << 32))
        return true;
    constexpr int kFirst = 3;
    const uint32_t x3 = (PA_PURPOSE_WBOND << 28) | (pc.t << 8) | (mu << 4);
    const pa_philox_shared sh = pa_philox_share(pc.seed, pc.run_id, owner, pc.w, pc.step);
    uint32_t u = 0; // the uniform's leading bits
    auto bits = [&](const pa_philox_out &o) {
        u = (u << 2) | ((((b < 32u ? o.x0 : o.x1) >> (b & 31u)) & 1u) << 1) | (((b < 32u ? o.x2 : o.x3) >> (b & 31u)) & 1u);
    };
    pa_philox_out o[kFirst];
    pa_philox_k<kFirst>(pc.seed, pc.run_id, sh, pc.w, pc.step, x3, o);
#pragma unroll
    for (int q = 0; q < kFirst; ++q)
        bits(o[q]);
    int left = 32 - 2 * kFirst; // bits to come
    for (uint32_t q = kFirst; left > 0 && u == (uint32_t)T >> left; ++q, left -= 2)
        bits(pa_philox_with(pc.seed, pc.run_id, sh, pc.w, pc.step, x3 | q));
    return u < (uint32_t)T >> left;
}

// PX, PY (and in 3D PZ) divide L; a workgroup has a lane for each of the N / (PX PY PZ) patches, and
// more that only decide bonds, recount and copy.  REST: the updates that k_cluster_list left.
template <int D, bool J, int PX, int PY, int PZ, bool REST>
__global__ __launch_bounds__(cluster_lanes(D, PX * PY * PZ)) void k_cluster(const PaRunDesc *__restrict__ runs,
                                                                          const PaBlk *__restrict__ map, int nsteps,
                                                                          uint32_t t0)
{
    static_assert(D == 3 || PZ == 1, "flat patches in 2D");
    // dynamic LDS: lattice, then cluster, [N] | one axis's bonds [N] (at least 32 per wave, reused by
    // the recount) | jmask [N] bytes
    extern __shared__ uint64_t lat[];
    const PaBlk blk = map[blockIdx.x];
    const PaRunDesc &rd = runs[blk.run];
    PaRecord *rec = rd.dv.rec;
    const uint32_t w = blk.idx;
    const int64_t Rlive = (int64_t)rec->Rcur;
    if ((int64_t)w * 64 >= Rlive || frozen(rec))
        return;
    const int first = REST ? uni((int)rd.dv.r[w]) : 0;
    if (REST && first >= nsteps)
        return;
    const int L = uni(rd.L), N = uni(rd.N), LL = L * L;
    const int cur = uni(rec->cur);
    const int tid = threadIdx.x, bs = blockDim.x, nw = bs >> 6;
    uint64_t *xb = lat + N;
    uint8_t *jl = reinterpret_cast<uint8_t *>(xb + max(N, 32 * nw));
    uint64_t *g = rd.dv.spins[cur] + (size_t)w * N;
    load_column(lat, g, N);
    if (J)
        load_jmask(jl, rd.dv.jmask, N);
    const uint32_t mL = uni((uint32_t)(((1ull << 32) + (uint64_t)L - 1) / (uint64_t)L));
    const uint64_t T = wolff_threshold(rec);
    PlaneCtx pc;
    pc.seed = uni(rd.seed);
    pc.run_id = uni(rd.run_id);
    pc.w = w;
    pc.step = uni(rec->step);
    // the lane's patch: its first site, and the steps from its faces to the words beyond them
    const int px = L / PX, py = L / PY;
    const bool own = tid * (PX * PY * PZ) < N;
    const int q = own ? tid : 0;
    const int qx = q % px, qr = q / px, qy = qr % py, qz = qr / py;
    const int s0 = qx * PX + L * (qy * PY) + LL * (qz * PZ);
    const int oxm = qx == 0 ? L - 1 : -1, oxp = qx == px - 1 ? 1 - L : 1;
    const int oym = qy == 0 ? L * (L - 1) : -L, oyp = qy == py - 1 ? -L * (L - 1) : L;
    const int ozm = qz == 0 ? LL * (L - 1) : -LL, ozp = (qz + 1) * PZ == L ? -LL * (L - 1) : LL;
    __syncthreads();
    for (int step = first; step < nsteps; ++step) {
        pc.t = t0 + (uint32_t)step;
        // the patch's own bonds (towards +e_mu), and those its neighbours own into its low faces
        uint64_t bx[PZ][PY][PX], by[PZ][PY][PX], bz[PZ][PY][PX], fx[PZ][PY], fy[PZ][PX], fz[PY][PX];
#pragma unroll
        for (int mu = 0; mu < D; ++mu) {
            for (int s = tid; s < N; s += bs) {
                const int row = (int)__umulhi((uint32_t)s, mL);
                const int x = s - row * L;
                const int z = (D == 2) ? 0 : (int)__umulhi((uint32_t)row, mL);
                const int y = row - z * L;
                const int c = mu == 0 ? x : (mu == 1 ? y : z), st = mu == 0 ? 1 : (mu == 1 ? L : LL);
                const uint64_t n = lat[c == L - 1 ? s - st * (L - 1) : s + st];
                // active where satisfied and drawn
                xb[s] = wolff_bond(pc, (uint32_t)s, (uint32_t)mu, ~bond<J>(lat[s], n, J ? (uint32_t)jl[s] : 0u, mu), T);
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PZ; ++k)
#pragma unroll
                for (int j = 0; j < PY; ++j)
#pragma unroll
                    for (int i = 0; i < PX; ++i) {
                        const int s = s0 + i + L * j + LL * k;
                        if (mu == 0) {
                            bx[k][j][i] = own ? xb[s] : 0ull;
                            if (i == 0)
                                fx[k][j] = own ? xb[s + oxm] : 0ull;
                        } else if (mu == 1) {
                            by[k][j][i] = own ? xb[s] : 0ull;
                            if (j == 0)
                                fy[k][i] = own ? xb[s + oym] : 0ull;
                        } else {
                            bz[k][j][i] = own ? xb[s] : 0ull;
                            if (k == 0)
                                fz[j][i] = own ? xb[s + ozm] : 0ull;
                        }
                    }
            __syncthreads(); // before the next axis's bonds; after the last, the lattice's words are not needed
        }
        for (int s = tid; s < N; s += bs)
            lat[s] = 0;
        __syncthreads();
        if (tid < 64) { // the seed of replica tid
            atomicOr((unsigned long long *)&lat[wolff_seed(pc, (uint32_t)tid, N)], 1ull << tid);
        }
        __syncthreads();
        uint64_t c[PZ][PY][PX];
#pragma unroll
        for (int k = 0; k < PZ; ++k)
#pragma unroll
            for (int j = 0; j < PY; ++j)
#pragma unroll
                for (int i = 0; i < PX; ++i)
                    c[k][j][i] = own ? lat[s0 + i + L * j + LL * k] : 0ull;
        __syncthreads(); // every lane has its words before any writes
        // every round that continues has added a (site, replica) pair: at most 64 N rounds
        constexpr int kAndOr = PA_T3((PA_A & PA_B) | PA_C);
        for (int round = 0; round <= 64 * N; ++round) {
            int any = 0;
            for (int pass = 0; pass < kGrowPasses; ++pass) {
                if (own) {
                    uint64_t n[PZ][PY][PX];
#pragma unroll
                    for (int k = 0; k < PZ; ++k)
#pragma unroll
                        for (int j = 0; j < PY; ++j)
#pragma unroll
                            for (int i = 0; i < PX; ++i) {
                                const int s = s0 + i + L * j + LL * k;
                                uint64_t v = c[k][j][i];
                                if (i == 0)
                                    v = pa_bop3<kAndOr>(lat[s + oxm], fx[k][j], v);
                                if (i == PX - 1)
                                    v = pa_bop3<kAndOr>(lat[s + oxp], bx[k][j][i], v);
                                if (j == 0)
                                    v = pa_bop3<kAndOr>(lat[s + oym], fy[k][i], v);
                                if (j == PY - 1)
                                    v = pa_bop3<kAndOr>(lat[s + oyp], by[k][j][i], v);
                                if (D == 3 && k == 0)
                                    v = pa_bop3<kAndOr>(lat[s + ozm], fz[j][i], v);
                                if (D == 3 && k == PZ - 1)
                                    v = pa_bop3<kAndOr>(lat[s + ozp], bz[k][j][i], v);
                                // forwards through the patch
                                if (i > 0)
                                    v = pa_bop3<kAndOr>(n[k][j][i > 0 ? i - 1 : 0], bx[k][j][i > 0 ? i - 1 : 0], v);
                                if (j > 0)
                                    v = pa_bop3<kAndOr>(n[k][j > 0 ? j - 1 : 0][i], by[k][j > 0 ? j - 1 : 0][i], v);
                                if (k > 0)
                                    v = pa_bop3<kAndOr>(n[k > 0 ? k - 1 : 0][j][i], bz[k > 0 ? k - 1 : 0][j][i], v);
                                n[k][j][i] = v;
                            }
                    uint64_t ch = 0;
#pragma unroll
                    for (int k = PZ - 1; k >= 0; --k)
#pragma unroll
                        for (int j = PY - 1; j >= 0; --j)
#pragma unroll
                            for (int i = PX - 1; i >= 0; --i) { // and backwards
                                uint64_t v = n[k][j][i];
                                if (i < PX - 1)
                                    v = pa_bop3<kAndOr>(n[k][j][i < PX - 1 ? i + 1 : 0], bx[k][j][i], v);
                                if (j < PY - 1)
                                    v = pa_bop3<kAndOr>(n[k][j < PY - 1 ? j + 1 : 0][i], by[k][j][i], v);
                                if (k < PZ - 1)
                                    v = pa_bop3<kAndOr>(n[k < PZ - 1 ? k + 1 : 0][j][i], bz[k][j][i], v);
                                n[k][j][i] = v;
                                ch = pa_bop3<PA_T3(PA_A | (PA_B ^ PA_C))>(ch, v, c[k][j][i]);
                                c[k][j][i] = v;
                            }
                    if (ch != 0) {
                        any = 1;
#pragma unroll
                        for (int k = 0; k < PZ; ++k)
#pragma unroll
                            for (int j = 0; j < PY; ++j)
#pragma unroll
                                for (int i = 0; i < PX; ++i)
                                    lat[s0 + i + L * j + LL * k] = c[k][j][i];
                    }
                }
                asm volatile("" ::: "memory"); // the next pass reads the neighbours' words again
            }
            if (!__syncthreads_or(any))
                break;
        }
        // flip: the lattice's words are still in memory
        for (int s = tid; s < N; s += bs) {
            const uint64_t v = g[s] ^ lat[s];
            lat[s] = v;
            if (step + 1 < nsteps)
                g[s] = v;
        }
        __syncthreads();
    }
    if (tid == 0 && w == 0) // once per run; no block reads it during the launch
        rec->sweeps = t0 + (uint32_t)nsteps;
    recount_column<D, J, false>(lat, [&](int t, int, int, int) -> uint32_t { return jl[t]; }, g, xb, rd, cur, w, Rlive, L, N,
                         LL, mL, 0ull);
}

// The same updates where few bonds are active, one workgroup per column: the
// clusters grow pair by pair (site, replica), level by level, from a list in
// LDS; a lane decides one bond of a listed pair.  Deciding every bond of the
// lattice would be most of such an update.  An update whose list overflows is
// left, with those after it, to k_cluster: r[w] holds the first one left (the
// copy numbers are scratch between resamplings).  Bound by the column's load
// and recount and the latency of a few levels.  3D L = 12, R = 10^5, (2 d - 1) p =
// 0.2: 180 us with the bonds decided as passes over the lattice reached them,
// 165 with all decided first, 41 now.
constexpr int kListed = 1024;
template <int D, bool J>
__global__ __launch_bounds__(1024) void k_cluster_list(const PaRunDesc *__restrict__ runs,
                                                       const PaBlk *__restrict__ map, int nsteps, uint32_t t0)
{
    // dynamic LDS: lattice [N] | cluster [N] (at least 32 per wave, reused by the recount) | jmask [N] bytes
    extern __shared__ uint64_t lat[];
    __shared__ uint32_t item[kListed], listed; // site << 6 | replica; how many
    const PaBlk blk = map[blockIdx.x];
    const PaRunDesc &rd = runs[blk.run];
    PaRecord *rec = rd.dv.rec;
    const uint32_t w = blk.idx;
    const int64_t Rlive = (int64_t)rec->Rcur;
    if ((int64_t)w * 64 >= Rlive || frozen(rec))
        return;
    const int L = uni(rd.L), N = uni(rd.N), LL = L * L;
    const int cur = uni(rec->cur);
    const int tid = threadIdx.x, bs = blockDim.x, nw = bs >> 6;
    uint64_t *cl = lat + N;
    uint8_t *jl = reinterpret_cast<uint8_t *>(cl + max(N, 32 * nw));
    uint64_t *g = rd.dv.spins[cur] + (size_t)w * N;
    load_column(lat, g, N);
    if (J)
        load_jmask(jl, rd.dv.jmask, N);
    const uint32_t mL = uni((uint32_t)(((1ull << 32) + (uint64_t)L - 1) / (uint64_t)L));
    const uint64_t T = wolff_threshold(rec);
    PlaneCtx pc;
    pc.seed = uni(rd.seed);
    pc.run_id = uni(rd.run_id);
    pc.w = w;
    pc.step = uni(rec->step);
    int step = 0;
    for (; step < nsteps; ++step) {
        pc.t = t0 + (uint32_t)step;
        for (int s = tid; s < N; s += bs)
            cl[s] = 0;
        if (tid == 0)
            listed = 64;
        __syncthreads();
        if (tid < 64) {
            const uint32_t sd = wolff_seed(pc, (uint32_t)tid, N);
            atomicOr((unsigned long long *)&cl[sd], 1ull << tid);
            item[tid] = (sd << 6) | (uint32_t)tid;
        }
        __syncthreads();
        int lo = 0, hi = T == 0 ? 0 : 64;
        while (lo < hi && hi <= kListed) { // every level adds pairs or is the last
            for (int t = tid; t < (hi - lo) * 2 * D; t += bs) {
                const int k = t / (2 * D), dir = t - k * 2 * D, mu = dir % D;
                const uint32_t it = item[lo + k], b = it & 63u;
                const int s = (int)(it >> 6), row = (int)__umulhi((uint32_t)s, mL);
                const int x = s - row * L;
                const int z = (D == 2) ? 0 : (int)__umulhi((uint32_t)row, mL);
                const int y = row - z * L;
                const int c = mu == 0 ? x : (mu == 1 ? y : z), st = mu == 0 ? 1 : (mu == 1 ? L : LL);
                const int n = dir < D ? (c == L - 1 ? s - st * (L - 1) : s + st) : (c == 0 ? s + st * (L - 1) : s - st);
                const int owner = dir < D ? s : n;
                const uint64_t out = bond<J>(lat[s], lat[n], J ? (uint32_t)jl[owner] : 0u, mu) | cl[n];
                if (((out >> b) & 1ull) == 0 && wolff_bond_of(pc, (uint32_t)owner, (uint32_t)mu, b, T) &&
                    ((atomicOr((unsigned long long *)&cl[n], 1ull << b) >> b) & 1ull) == 0) {
                    const uint32_t slot = atomicAdd(&listed, 1u);
                    if (slot < (uint32_t)kListed)
                        item[slot] = ((uint32_t)n << 6) | b;
                }
            }
            __syncthreads();
            lo = hi;
            hi = uni((int)listed);
            __syncthreads(); // every lane has the number before it grows
        }
        if (lo < hi)
            break; // the list is full
        for (int s = tid; s < N; s += bs)
            lat[s] ^= cl[s];
        __syncthreads();
    }
    if (tid == 0) {
        rd.dv.r[w] = (uint32_t)step;
        if (w == 0) // once per run; no block reads it during the launch
            rec->sweeps = t0 + (uint32_t)nsteps;
    }
    __syncthreads();
    recount_column<D, J, false>(lat, [&](int t, int, int, int) -> uint32_t { return jl[t]; }, g, cl, rd, cur, w, Rlive, L, N,
                         LL, mL, 0ull);
}

// ------------------------------------------------------------------ step 2: Q
// Energy levels h = (E + dN) / 4: all energies of a run share E mod 4, since a
// flip changes E by a multiple of 4.
__global__ void k_hist_prep(const PaRunDesc *__restrict__ runs)
{
    const PaRunDesc &rd = runs[blockIdx.x];
    for (int i = threadIdx.x; i < rd.H; i += blockDim.x)
        rd.dv.hist[i] = 0;
    if (threadIdx.x == 0) {
        rd.dv.rec->emin = INT_MAX;
        rd.dv.rec->emax = INT_MIN;
    }
}

// The workgroup's lowest and highest of its threads' energies, in every thread
// (s_lo, s_hi: a word per wave).
__device__ __forceinline__ void block_energy_range(int &lo, int &hi, int *s_lo, int *s_hi)
{
    lo = (int)pa_wave_min_i64(lo);
    hi = (int)pa_wave_max_i64(hi);
    if ((threadIdx.x & 63) == 0) {
        s_lo[threadIdx.x >> 6] = lo;
        s_hi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) {
        lo = min(lo, s_lo[k]);
        hi = max(hi, s_hi[k]);
    }
}

// Adds a tile's replicas to the run's level histogram: the tile's energies into
// registers, counts in LDS for the levels of their range, and one atomic per
// populated level.  Counters for every level of the lattice, cleared and
// scanned by each tile, cost more than the counting where the levels are
// many: 2D L = 128, R = 2 10^4 12 -> 4.4 us, 3D L = 8, R = 10^6 10.5 -> 9.6.
__global__ __launch_bounds__(kThreads) void k_hist(const PaRunDesc *__restrict__ runs,
                                                   const PaBlk *__restrict__ map)
{
    extern __shared__ uint32_t lh[]; // the lattice's levels at most
    __shared__ int s_lo[kThreads / 64], s_hi[kThreads / 64];
    constexpr int kVec = 4; // 16-byte loads a thread: tiles of up to 16 kThreads replicas
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    const int64_t R = (int64_t)rec->Rcur;
    const int64_t tile = pa_counts_tile(rd.cap), beg = (int64_t)b.idx * tile;
    if (beg >= R || frozen(rec))
        return;
    const int DN = rd.d * rd.N;
    const int32_t *E = rd.dv.E[rec->cur];
    const int64_t end = beg + tile < R ? beg + tile : R;
    const int nv = (int)(tile / (4 * kThreads));
    alignas(16) int32_t e[kVec][4];
    int lo = INT_MAX, hi = INT_MIN;
#pragma unroll
    for (int v = 0; v < kVec; ++v) {
        const int64_t j = beg + 4 * (threadIdx.x + (int64_t)v * kThreads);
        if (v < nv && j + 4 <= end) {
            *reinterpret_cast<uint4 *>(e[v]) = *reinterpret_cast<const uint4 *>(E + j);
        } else if (v < nv) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                e[v][k] = E[j + k < end ? j + k : end - 1]; // past the end: not counted
        }
    }
#pragma unroll
    for (int v = 0; v < kVec; ++v)
        if (v < nv)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lo = min(lo, e[v][k]);
                hi = max(hi, e[v][k]);
            }
    block_energy_range(lo, hi, s_lo, s_hi);
    const int hlo = (lo + DN) >> 2, nl = ((hi + DN) >> 2) - hlo + 1;
    for (int i = threadIdx.x; i < nl; i += blockDim.x)
        lh[i] = 0;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kVec; ++v) {
        const int64_t j = beg + 4 * (threadIdx.x + (int64_t)v * kThreads);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (v < nv && j + k < end)
                atomicAdd(&lh[((e[v][k] + DN) >> 2) - hlo], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nl; i += blockDim.x)
        if (lh[i])
            atomicAdd(&rd.dv.hist[hlo + i], lh[i]);
    if (threadIdx.x == 0) {
        atomicMin(&rec->emin, lo);
        atomicMax(&rec->emax, hi);
    }
}

__device__ __forceinline__ pa_u128 block_sum_u128(pa_u128 v, uint64_t *su)
{
    pa_u128 t = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t limb = (uint64_t)(v >> (32 * k)) & 0xFFFFFFFFull;
        t += (pa_u128)pa_block_sum_u64(limb, su) << (32 * k);
    }
    return t;
}

// One workgroup per run: weights per level above the lowest, the Q sum in a
// fixed order (contiguous chunk per thread, then the block's fixed tree), S
// and sum_h n_h W_h^2 exactly, ln Q and the Metropolis thresholds of the next
// beta.  A weighted population only gets dbeta and the thresholds here; its
// per-replica passes (k_rw_max, k_rw_sum, k_rw_final) do the rest.
// T: 1024 lanes for few runs (a chain of latencies), 256 for more than a run
// per CU, where most levels of a small lattice leave most of 1024 lanes idle
// but started: 1024 runs of 2D L = 16 15.5 -> 5.9 us.  The sums are of the same 16 waves' chunks
// either way.
template <int T>
__device__ __forceinline__ void reweight_run(const PaRunDesc &rd, PaRecord *rec, double beta_next)
{
    __shared__ uint64_t su[16 * 6];
    const int DN = rd.d * rd.N;
    const double dbeta = beta_next - rec->beta;
    const int32_t emin = rec->emin, emax = rec->emax;
    // the resampling that follows starts with clean tile flags, tickets and status
    const int64_t ntiles = 2 * pa_tiles_per_sum(rd.cap);
    for (int64_t t = threadIdx.x; t < ntiles; t += blockDim.x)
        rd.dv.tiles[t].word = 0ull;
    const int hmin = (emin + DN) >> 2, hmax = (emax + DN) >> 2;
    const int nlev = hmax - hmin + 1;
    if (rec->weighted) {
        __syncthreads(); // every thread has read the record before thread 0 writes it
        // the level histogram is not needed any more: back to zero for the next build
        for (int k = threadIdx.x; k < nlev; k += blockDim.x)
            rd.dv.hist[hmin + k] = 0;
        if (threadIdx.x == 0) {
            rec->emin = INT_MAX;
            rec->emax = INT_MIN;
            rec->ticket[0] = rec->ticket[1] = 0u;
            rec->status = 0;
            rec->skip = 0;
            rec->keep = 0;
            rec->wemin = emin;
            rec->dbeta = dbeta;
            rec->beta_next = beta_next;
            rec->S = 0;
            rec->Q2[0] = rec->Q2[1] = 0;
            rec->xmag = ~0ull;
            rec->Tn[0] = pa_threshold(beta_next, 4);
            rec->Tn[1] = pa_threshold(beta_next, 8);
            rec->Tn[2] = pa_threshold(beta_next, 12);
        }
        return;
    }
    // 16 waves' worth of chunks, T lanes at a time up to the last level
    const int chunk = (nlev + 1023) / 1024, nwaves = (nlev + 64 * chunk - 1) / (64 * chunk);
    for (int w0 = 0; w0 < nwaves; w0 += T / 64) {
        const int lo = (w0 * 64 + (int)threadIdx.x) * chunk;
        const int hi = lo + chunk < nlev ? lo + chunk : nlev;
        double q = 0.0;
        uint64_t s = 0;
        pa_u128 s2 = 0;
        for (int k = lo; k < hi; ++k) {
            const uint32_t n = rd.dv.hist[hmin + k];
            const double wv = pa_exp(-(dbeta * (double)(4 * k)));
            const uint64_t W = (uint64_t)floor(ldexp(wv, 40));
            rd.dv.wtab[k] = W;
            q = q + (double)n * wv;
            s += (uint64_t)n * W;
            s2 += (pa_u128)((uint64_t)n * W) * W;
        }
        // one exchange through LDS for all block sums: Q (a double, the waves'
        // butterfly totals added in wave order, so the same bits every run), S
        // and the four 32-bit limbs of sum n W^2 (a limb's block total stays
        // below 2^42)
        uint64_t x[6] = {s, (uint64_t)s2 & 0xFFFFFFFFull, (uint64_t)(s2 >> 32) & 0xFFFFFFFFull,
                         (uint64_t)(s2 >> 64) & 0xFFFFFFFFull, (uint64_t)(s2 >> 96),
                         (uint64_t)__double_as_longlong(pa_wave_sum_f64(q))};
#pragma unroll
        for (int i = 0; i < 5; ++i)
            x[i] = pa_wave_sum_u64(x[i]);
        const int wave = w0 + (int)(threadIdx.x >> 6);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int i = 0; i < 6; ++i)
                su[wave * 6 + i] = x[i];
    }
    __syncthreads(); // also: every level has been read
    double Q = 0.0;
    uint64_t t[5] = {0, 0, 0, 0, 0};
    for (int k = 0; k < nwaves; ++k) {
#pragma unroll
        for (int i = 0; i < 5; ++i)
            t[i] += su[k * 6 + i];
        Q = Q + __longlong_as_double((long long)su[k * 6 + 5]);
    }
    const uint64_t S = t[0];
    const pa_u128 S2 = (pa_u128)t[1] + ((pa_u128)t[2] << 32) + ((pa_u128)t[3] << 64) + ((pa_u128)t[4] << 96);
    // back to zero for the next build of the level histogram
    for (int k = threadIdx.x; k < nlev; k += blockDim.x)
        rd.dv.hist[hmin + k] = 0;
    // the record's new values, the exponentials on separate lanes
    if (threadIdx.x == 0) {
        rec->emin = INT_MAX;
        rec->emax = INT_MIN;
        rec->ticket[0] = rec->ticket[1] = 0u;
        rec->status = 0;
        rec->skip = 0;
        rec->keep = 0;
        rec->wemin = emin;
        rec->qsum = Q;
        rec->S = S;
        rec->Q2[0] = (uint64_t)S2;
        rec->Q2[1] = (uint64_t)(S2 >> 64);
        rec->dbeta = dbeta;
        rec->beta_next = beta_next;
        rec->lnQ = -dbeta * (double)emin + log(Q / (double)rec->Rcur);
    } else if (threadIdx.x < 4) {
        rec->Tn[threadIdx.x - 1] = pa_threshold(beta_next, 4 * (int)threadIdx.x);
    }
}

template <int T>
__global__ __launch_bounds__(T) void k_reweight(const PaRunDesc *__restrict__ runs, double beta_next)
{
    const PaRunDesc &rd = runs[blockIdx.x];
    if (!frozen(rd.dv.rec))
        reweight_run<T>(rd, rd.dv.rec, beta_next);
}

// ------------------------------------------------------------------ adaptive step
// Overlap of the population with its reweighting by dbeta, with the integer
// weights the resampling uses: W_h = floor(2^40 pa_exp(-dbeta 4(h - hmin)))
// per energy level, S = sum_h n_h W_h, and
//   alpha = sum_h n_h min(S, R W_h) / (R S)
// exactly (integer sums, so any order gives the same numbers).  The bisection
// keeps the largest dbeta in [0, dbeta_max] with 2^32 num >= A R S, A the
// target overlap in units of 2^-32.
__device__ __forceinline__ double u128_to_double(pa_u128 x)
{
    return (double)(uint64_t)(x >> 64) * 18446744073709551616.0 + (double)(uint64_t)x;
}

struct Overlap {
    pa_u128 num, den;
};

// The whole workgroup's overlap at dbeta: every thread takes every
// blockDim-th level (with a contiguous range each, the lanes' reads of counts
// and weights lay apart: 60 halvings over 16000 levels 1370 -> 1196 us, over
// 4000 399 -> 353).
__device__ Overlap rule_overlap(const uint32_t *__restrict__ hist, int hmin, int nlev, uint64_t R, double dbeta,
                                uint64_t *wcache, uint64_t *su)
{
    const int bs = (int)blockDim.x;
    uint64_t s = 0;
    for (int k = threadIdx.x; k < nlev; k += bs) {
        const uint64_t W = pa_weight(dbeta, 4 * k);
        if (k < kRuleCache)
            wcache[k] = W;
        s += (uint64_t)hist[hmin + k] * W;
    }
    const uint64_t S = pa_block_sum_u64(s, su);
    pa_u128 a = 0;
    for (int k = threadIdx.x; k < nlev; k += bs) {
        const uint64_t W = k < kRuleCache ? wcache[k] : pa_weight(dbeta, 4 * k);
        const uint64_t RW = R * W;
        a += (pa_u128)hist[hmin + k] * (RW < S ? RW : S);
    }
    Overlap o;
    o.num = block_sum_u128(a, su);
    o.den = (pa_u128)R * S;
    return o;
}

__device__ __forceinline__ bool qualifies(const Overlap &o, uint64_t A) { return (o.num << 32) >= (pa_u128)A * o.den; }

// Sum of v over the wave in every lane, for lane values below 2^26 (the sum
// stays below 2^32): butterflies by lane permutations within rows of 16, then
// by exchanges of whole rows and halves.
__device__ __forceinline__ uint32_t wave_sum_26(uint32_t v)
{
    v += xlane<1>(v);
    v += xlane<2>(v);
    v += xlane<4>(v);
    v += xlane<8>(v);
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] + a[1];
    const auto c = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return uni(c[0] + c[1]);
}

// A wave's sum of lane values below 2^(26 LIMBS), in 26-bit limbs.
template <int LIMBS>
__device__ __forceinline__ pa_u128 wave_sum_u128(pa_u128 v)
{
    pa_u128 t = 0;
#pragma unroll
    for (int k = 0; k < LIMBS; ++k)
        t += (pa_u128)wave_sum_26((uint32_t)(v >> (26 * k)) & 0x3FFFFFFu) << (26 * k);
    return t;
}

// The rule's search.  An overlap is a sum over some hundred populated levels:
// little work, so one evaluation at a time by the whole workgroup spent its
// time on the barriers of the block sums.  Here each of kRuleWaves waves
// evaluates a point of its own, with no barrier, and the workgroup takes
// several halvings a round: either the seven midpoints of the next three
// halvings (a tree, right whatever the outcome), or the midpoints of the next
// seven along the path to the secant root of the overlap between lo and hi,
// used as far as the outcomes follow that path.  The path is tried once the
// bracket has shrunk and dropped for a round when it gained less than a tree
// would (below about 2^-40 of dbeta_max the integer weights make the overlap
// a staircase); 60 halvings take about 12 rounds.  The result is the plain bisection's, bit for bit.
// Above kRuleLevels levels the evaluations bound the search and the whole
// workgroup takes one at a time.
// 3D L = 8, R = 10^5 (about 400 levels, 60 halvings): 258 -> 41 us.
constexpr int kRuleWaves = 8;
constexpr int kRuleLevels = 2048, kRuleHeld = 16; // held: levels per lane whose weights stay in registers

struct RuleLds {
    uint64_t su[16];
    uint64_t wcache[kRuleCache];
    uint32_t count[kRuleLevels]; // replicas per level
    // the points of a round (two rounds' worth: one barrier a round): their overlaps, what those
    // exceed the target by, and whether they qualify
    double x[2][kRuleWaves], f[2][kRuleWaves];
    pa_u128 num[2][kRuleWaves], den[2][kRuleWaves];
    uint32_t ok[2][kRuleWaves];
};

struct RuleSearch {
    RuleLds *l;
    const uint32_t *hist;
    int hmin, nlev, buf;
    uint64_t R, A;
    bool waves; // a wave per point

    // Starts a search over the run's populated levels (all threads).
    // most: levels up to which a wave takes a point of its own
    __device__ __forceinline__ RuleSearch(RuleLds *lds, const PaRunDesc &rd, const PaRecord *rec, double alpha_star,
                                          int most = kRuleLevels)
        : l(lds), hist(rd.dv.hist), buf(0)
    {
        const int DN = rd.d * rd.N;
        hmin = (rec->emin + DN) >> 2;
        nlev = uni(((rec->emax + DN) >> 2) - hmin + 1);
        R = uni64(rec->Rcur);
        A = uni64((uint64_t)rint(ldexp(alpha_star, 32)));
        waves = nlev <= most;
        if (waves)
            for (int k = threadIdx.x; k < nlev; k += blockDim.x)
                l->count[k] = hist[hmin + k];
        __syncthreads();
    }

    // The wave's overlap at x (the same in every lane).
    __device__ Overlap wave_overlap(double x) const
    {
        const int lane = threadIdx.x & 63;
        uint64_t W[kRuleHeld], s = 0;
        uint32_t n[kRuleHeld];
#pragma unroll
        for (int i0 = 0; i0 < kRuleHeld; i0 += 4) // four levels at a time: independent chains
            if (64 * i0 < nlev)
#pragma unroll
                for (int i = i0; i < i0 + 4; ++i) {
                    const int k = 64 * i + lane;
                    W[i] = pa_weight(x, 4 * k);
                    n[i] = k < nlev ? l->count[k] : 0u;
                    s += (uint64_t)n[i] * W[i];
                }
        for (int k = 64 * kRuleHeld + lane; k < nlev; k += 64)
            s += (uint64_t)l->count[k] * pa_weight(x, 4 * k);
        const uint64_t S = (uint64_t)wave_sum_u128<3>(s);
        pa_u128 a = 0;
#pragma unroll
        for (int i0 = 0; i0 < kRuleHeld; i0 += 4)
            if (64 * i0 < nlev)
#pragma unroll
                for (int i = i0; i < i0 + 4; ++i) {
                    const uint64_t RW = R * W[i];
                    a += (pa_u128)n[i] * (RW < S ? RW : S);
                }
        for (int k = 64 * kRuleHeld + lane; k < nlev; k += 64) {
            const uint64_t RW = R * pa_weight(x, 4 * k);
            a += (pa_u128)l->count[k] * (RW < S ? RW : S);
        }
        Overlap o;
        o.num = wave_sum_u128<4>(a); // below 2^88: counts below 2^24, S below 2^64
        o.den = (pa_u128)R * S;
        return o;
    }

    // One round: wave v's overlap at its x (NaN: none) into slot v; afterwards slot(v), x(v) hold them.
    __device__ __forceinline__ void round(double x)
    {
        const int v = threadIdx.x >> 6;
        buf ^= 1;
        if (x == x) {
            const Overlap o = wave_overlap(x);
            const double f = excess(o);
            const bool ok = qualifies(o, A);
            if ((threadIdx.x & 63) == 0) {
                l->x[buf][v] = x;
                l->f[buf][v] = f;
                l->ok[buf][v] = ok ? 1u : 0u;
                l->num[buf][v] = o.num;
                l->den[buf][v] = o.den;
            }
        }
        __syncthreads();
    }

    __device__ __forceinline__ Overlap slot(int v) const { return {l->num[buf][v], l->den[buf][v]}; }

    // Prepares the overlaps at up to kRuleWaves points, to be read by at() before the next round.
    template <int n>
    __device__ __forceinline__ void points(const double (&x)[n])
    {
        static_assert(n <= kRuleWaves, "a wave per point");
        if (!waves)
            return;
        double mine = __longlong_as_double(-1ll);
#pragma unroll
        for (int k = 0; k < n; ++k)
            if (k == (int)(threadIdx.x >> 6))
                mine = x[k];
        round(mine);
    }

    // The overlap at x, prepared as point k (without a wave per point: computed now).
    __device__ __forceinline__ Overlap at(int k, double x)
    {
        return waves ? slot(k) : rule_overlap(hist, hmin, nlev, R, x, l->wcache, l->su);
    }

    __device__ __forceinline__ double excess(const Overlap &o) const
    {
        return u128_to_double(o.num) / u128_to_double(o.den) - (double)A * (1.0 / 4294967296.0);
    }

    // `iterations` halvings of [lo, hi] keeping lo qualified: lo (overlap olo) qualifies, hi (ohi) does not.
    __device__ void bisect(double &lo, Overlap &olo, double hi, const Overlap &ohi, int iterations)
    {
        const int v = threadIdx.x >> 6;
        double flo = excess(olo), fhi = excess(ohi);
        bool path = false;
        for (int it = 0; it < iterations;) {
            const double mid = 0.5 * (lo + hi);
            if (mid == lo || mid == hi)
                break; // nothing lies between: every further halving keeps lo
            if (!waves) {
                const Overlap om = rule_overlap(hist, hmin, nlev, R, mid, l->wcache, l->su);
                if (qualifies(om, A)) {
                    lo = mid;
                    olo = om;
                } else {
                    hi = mid;
                }
                ++it;
                continue;
            }
            // this wave's point: midpoint v (1..7) of the tree, in heap order, or the v-th along the path
            const double root = lo + (hi - lo) * (flo / (flo - fhi));
            double a = lo, b = hi, x = __longlong_as_double(-1ll);
            if (v > 0) {
                const int depth = path ? v - 1 : 31 - __builtin_clz(v);
                for (int d = 0; d < depth; ++d) {
                    const double m = 0.5 * (a + b);
                    const bool up = path ? m <= root : ((v >> (depth - 1 - d)) & 1) != 0;
                    a = up ? m : a;
                    b = up ? b : m;
                }
                x = 0.5 * (a + b);
            }
            round(x);
            int n = 1, gained = 0, kept = 0;
            for (const int most = path ? kRuleWaves - 1 : 3; gained < most && it < iterations;) {
                const double m = l->x[buf][n], f = l->f[buf][n];
                const bool ok = l->ok[buf][n] != 0u;
                ++gained;
                ++it;
                if (ok) {
                    lo = m;
                    flo = f;
                    kept = n;
                } else {
                    hi = m;
                    fhi = f;
                }
                if (path && ok != (m <= root))
                    break;
                n = path ? n + 1 : 2 * n + (ok ? 1 : 0);
            }
            if (kept)
                olo = slot(kept);
            path = path ? gained >= 3 : true;
        }
    }
};

__global__ __launch_bounds__(kRuleWaves * 64) void k_rule(const PaRunDesc *__restrict__ runs, double alpha_star,
                                                          double dbeta_max, int iterations, int bisect)
{
    __shared__ RuleLds lds;
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec))
        return;
    // a single point of many levels: the workgroup's lanes outweigh its barriers (2000 levels 23.8 -> 17.8 us
    // with the call's copy and wait)
    RuleSearch rs(&lds, rd, rec, alpha_star, bisect ? kRuleLevels : 64 * kRuleHeld);
    const double xs[1] = {dbeta_max};
    rs.points(xs);
    const Overlap top = rs.at(0, dbeta_max);
    double best = dbeta_max;
    Overlap obest = top;
    if (bisect && !qualifies(top, rs.A)) {
        best = 0.0;
        obest.num = obest.den = 1; // alpha(0) = 1
        rs.bisect(best, obest, dbeta_max, top, iterations);
    }
    if (threadIdx.x == 0) {
        rec->rule_dbeta = best;
        rec->rule_alpha = u128_to_double(obest.num) / u128_to_double(obest.den);
    }
}

// Inputs of the learned step model from the energy histogram (moments in
// float64, fixed chunks and tree), the record's ln Q history and the family
// entropy of the latest observables: beta, <E>/N, sd(E)/sqrt(N), skewness,
// ln Q_{i-2..i}/N, S_f / ln R.
__global__ __launch_bounds__(kRuleThreads) void k_features(const PaRunDesc *__restrict__ runs)
{
    __shared__ double sd[16];
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec))
        return;
    const int DN = rd.d * rd.N;
    const int32_t emin = rec->emin;
    const int hmin = (emin + DN) >> 2, hmax = (rec->emax + DN) >> 2;
    const int nlev = hmax - hmin + 1;
    const double R = (double)rec->Rcur;
    const int chunk = (nlev + (int)blockDim.x - 1) / (int)blockDim.x;
    const int lo = (int)threadIdx.x * chunk;
    const int hi = lo + chunk < nlev ? lo + chunk : nlev;
    double s1 = 0.0;
    for (int k = lo; k < hi; ++k)
        s1 = s1 + (double)rd.dv.hist[hmin + k] * (double)(emin + 4 * k);
    const double mean = pa_block_sum_f64(s1, sd) / R;
    double s2 = 0.0, s3 = 0.0;
    for (int k = lo; k < hi; ++k) {
        const double dx = (double)(emin + 4 * k) - mean, n = (double)rd.dv.hist[hmin + k];
        s2 = s2 + n * dx * dx;
        s3 = s3 + n * dx * dx * dx;
    }
    const double var = pa_block_sum_f64(s2, sd) / R;
    const double m3 = pa_block_sum_f64(s3, sd) / R;
    if (threadIdx.x == 0) {
        const double N = (double)rd.N;
        rec->feat[0] = (float)rec->beta;
        rec->feat[1] = (float)(mean / N);
        rec->feat[2] = (float)(sqrt(var) / sqrt(N));
        rec->feat[3] = (float)(var > 0.0 ? m3 / (var * sqrt(var)) : 0.0);
        rec->feat[4] = (float)(rec->lnq_hist[0] / N);
        rec->feat[5] = (float)(rec->lnq_hist[1] / N);
        rec->feat[6] = (float)(rec->lnq_hist[2] / N);
        rec->feat[7] = (float)(R > 1.0 ? rec->S_f / log(R) : 0.0);
    }
}

// The learned proposal is kept if it passes the exact overlap check;
// otherwise the bisection of the rule decides (fallback).
// The learned step's exact check: the model's proposal c (clamped to
// dbeta_max) is kept only where alpha >= alpha*.  With refine > 0 it seeds a
// short search instead of being taken as it is: if c qualifies, the bracket
// [c, min(bracket c, dbeta_max)] (whose top is taken if it qualifies), else
// [c / bracket, c] if its bottom qualifies, is halved `refine` times keeping
// the lower end qualified.  Where neither applies (or c <= 0) the rule itself
// decides: the bisection of k_rule over [0, dbeta_max] (the fallback).
// Every value returned has alpha >= alpha*, tested exactly.
__global__ __launch_bounds__(kRuleWaves * 64) void k_check_candidate(const PaRunDesc *__restrict__ runs,
                                                                     double alpha_star, double dbeta_max,
                                                                     int iterations, double bracket, int refine)
{
    __shared__ RuleLds lds;
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec))
        return;
    RuleSearch rs(&lds, rd, rec, alpha_star);
    const double cand = rec->cand_dbeta;
    auto publish = [&](double db, const Overlap &o, uint32_t fb) {
        if (threadIdx.x == 0) {
            rec->rule_dbeta = db;
            rec->rule_alpha = u128_to_double(o.num) / u128_to_double(o.den);
            rec->fallback = fb;
        }
    };
    // the candidate and the points that may be asked for next, in one round:
    // the bracket's top and bottom, and the rule's first
    const double up = bracket * cand < dbeta_max ? bracket * cand : dbeta_max;
    const double xs[4] = {cand, up, cand / bracket, dbeta_max};
    rs.points(xs);
    if (cand > 0.0) {
        const Overlap oc = rs.at(0, cand);
        const bool ok = qualifies(oc, rs.A);
        if (ok && (refine == 0 || cand >= dbeta_max)) {
            publish(cand, oc, 0u);
            return;
        }
        if (refine > 0) {
            double lo = ok ? cand : xs[2], hi = ok ? up : cand;
            Overlap olo = oc, ohi = oc;
            bool bracketed = true;
            if (ok) {
                ohi = rs.at(1, up);
                if (qualifies(ohi, rs.A)) {
                    publish(up, ohi, 0u);
                    return;
                }
            } else {
                olo = rs.at(2, lo);
                bracketed = qualifies(olo, rs.A);
            }
            if (bracketed) {
                rs.bisect(lo, olo, hi, ohi, refine);
                publish(lo, olo, 0u);
                return;
            }
        }
    }
    const Overlap top = rs.at(3, dbeta_max);
    double best = dbeta_max;
    Overlap obest = top;
    if (!qualifies(top, rs.A)) {
        best = 0.0;
        obest.num = obest.den = 1;
        rs.bisect(best, obest, dbeta_max, top, iterations);
    }
    publish(best, obest, 1u);
}

// ------------------------------------------------------------------ resampling
__device__ __forceinline__ uint64_t weight_of(int32_t e, int DN, int hmin, const uint64_t *wtab)
{
    return wtab[((e + DN) >> 2) - hmin];
}

// Per-replica resampling kernels: chunk b.idx of run b.run, replicas
// [idx*CHUNK, ...) below the pre-resampling size.
struct RepCtx {
    const PaRunDesc *rd;
    PaRecord *rec;
    int64_t beg, end;
};

__device__ __forceinline__ bool rep_ctx(const PaRunDesc *runs, const PaBlk *map, RepCtx *c)
{
    const PaBlk b = map[blockIdx.x];
    c->rd = runs + b.run;
    c->rec = c->rd->dv.rec;
    const int64_t R = (int64_t)c->rec->Rcur;
    c->beg = (int64_t)b.idx * PA_CHUNK;
    c->end = c->beg + PA_CHUNK < R ? c->beg + PA_CHUNK : R;
    return c->beg < R && !frozen(c->rec);
}

// The kernels of a resampling proper: idle when a conditional resampling
// decided to keep the population.
__device__ __forceinline__ bool rs_ctx(const PaRunDesc *runs, const PaBlk *map, RepCtx *c)
{
    return rep_ctx(runs, map, c) && !c->rec->keep;
}

// Integer weight of replica j for the resampling: per energy level for a
// uniform population, per replica (k_rw_sum) for a weighted one.
__device__ __forceinline__ uint64_t rep_weight(const RepCtx &c, bool wt, const int32_t *E, int64_t j, int DN,
                                               int hmin)
{
    return wt ? c.rd->dv.Wj[j] : weight_of(E[j], DN, hmin, c.rd->dv.wtab);
}

// ------------------------------------------------------------------ weighted populations
// Sec. 3 allows keeping the population, with importance weights, while their
// variance is small.  Replica j then carries a log-weight lw_j <= 0 (largest
// 0) and weighs exp(lw_j - dbeta E_j) at the next beta.  With
//   x_j = lw_j + (-(dbeta (E_j - E_min)))   (every x_j <= 0)
// and m = min_j |x_j| (so max_j x_j = -m), the integer weights are
// W_j = floor(2^40 pa_exp(x_j + m)) and
//   ln Q = -dbeta E_min - m + ln sum_j exp(x_j + m) - ln sum_j exp(lw_j),
// Eq. (1) for weighted replicas.  A uniform population is the case lw = 0
// (x_j is then the argument of its per-level weights and m = 0).
__device__ __forceinline__ double wx(const PaDev &dv, const PaRecord *rec, int cur, bool wt, int64_t j)
{
    const double g = (double)(dv.E[cur][j] - rec->wemin);
    const double lw = wt ? dv.lw[j] : 0.0;
    return lw + (-(rec->dbeta * g));
}

__device__ __forceinline__ double xmag_value(const PaRecord *rec) { return __longlong_as_double((long long)rec->xmag); }

// m: the smallest |x_j| (IEEE bits of non-negative doubles order as integers).
__global__ __launch_bounds__(kThreads) void k_rw_max(const PaRunDesc *__restrict__ runs,
                                                     const PaBlk *__restrict__ map)
{
    RepCtx c;
    if (!rep_ctx(runs, map, &c) || !c.rec->weighted)
        return;
    const PaDev &dv = c.rd->dv;
    const int cur = c.rec->cur;
    int64_t mag = INT64_MAX;
    for (int64_t j = c.beg + threadIdx.x; j < c.end; j += blockDim.x) {
        const int64_t b = __double_as_longlong(wx(dv, c.rec, cur, true, j)) & INT64_MAX;
        mag = b < mag ? b : mag;
    }
    mag = pa_wave_min_i64(mag);
    if ((threadIdx.x & 63) == 0)
        atomicMin(&c.rec->xmag, (unsigned long long)mag);
}

// Per-replica integer weights, S and sum W^2 exactly (order-free atomics),
// and per chunk the fixed-order sums of pa_exp(x_j + m) and pa_exp(lw_j).
__global__ __launch_bounds__(kThreads) void k_rw_sum(const PaRunDesc *__restrict__ runs,
                                                     const PaBlk *__restrict__ map)
{
    __shared__ double sd[16];
    __shared__ uint64_t su[16];
    RepCtx c;
    if (!rep_ctx(runs, map, &c) || !c.rec->weighted)
        return;
    const PaDev &dv = c.rd->dv;
    const int cur = c.rec->cur;
    const double m = xmag_value(c.rec);
    uint64_t s = 0;
    pa_u128 s2 = 0;
    double q = 0.0, l = 0.0;
    for (int64_t j = c.beg + threadIdx.x; j < c.end; j += blockDim.x) {
        const double wv = pa_exp(wx(dv, c.rec, cur, true, j) + m);
        const uint64_t W = (uint64_t)floor(ldexp(wv, 40));
        dv.Wj[j] = W;
        s += W;
        s2 += (pa_u128)W * W;
        q = q + wv;
        l = l + pa_exp(dv.lw[j]);
    }
    s = pa_block_sum_u64(s, su);
    s2 = block_sum_u128(s2, su);
    q = pa_block_sum_f64(q, sd);
    l = pa_block_sum_f64(l, sd);
    if (threadIdx.x == 0) {
        atomicAdd((unsigned long long *)&c.rec->S, (unsigned long long)s);
        const unsigned long long lo = (uint64_t)s2, hi = (uint64_t)(s2 >> 64);
        const unsigned long long old = atomicAdd(&c.rec->Q2[0], lo);
        atomicAdd(&c.rec->Q2[1], hi + (old + lo < old ? 1ull : 0ull));
        const int64_t chunks = (c.rd->cap + PA_CHUNK - 1) / PA_CHUNK, k = c.beg / PA_CHUNK;
        dv.wpart[k] = q;
        dv.wpart[chunks + k] = l;
    }
}

// ln Q of a weighted population from the chunk sums in chunk order.
__global__ __launch_bounds__(kThreads) void k_rw_final(const PaRunDesc *__restrict__ runs)
{
    __shared__ double sd[16];
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec) || !rec->weighted)
        return;
    const int64_t chunks = (rd.cap + PA_CHUNK - 1) / PA_CHUNK;
    const int nlive = (int)(((int64_t)rec->Rcur + PA_CHUNK - 1) / PA_CHUNK);
    double q = 0.0, l = 0.0;
    for (int k = threadIdx.x; k < nlive; k += blockDim.x) {
        q = q + rd.dv.wpart[k];
        l = l + rd.dv.wpart[chunks + k];
    }
    q = pa_block_sum_f64(q, sd);
    l = pa_block_sum_f64(l, sd);
    if (threadIdx.x == 0) {
        rec->qsum = q;
        rec->lnQ = ((-rec->dbeta * (double)rec->wemin - xmag_value(rec)) + log(q)) - log(l);
    }
}

// Conditional resampling: resample only if the effective sample size of the
// step's weights, ESS = S^2 / sum_j W_j^2, is below kappa R_cur.  Decided
// exactly as 2^16 S^2 < kq R_cur sum_j W_j^2 (kq = kappa 2^16) on 192-bit
// integers: S^2 < 2^128, sum W^2 < 2^104, kq R_cur < 2^41.
__device__ __forceinline__ bool ess_below(const PaRecord *rec, uint32_t kq)
{
    const uint64_t S = rec->S;
    const pa_u128 S2 = (pa_u128)S * S;
    const uint64_t a0 = (uint64_t)(S2 << 16), a1 = (uint64_t)((S2 << 16) >> 64), a2 = (uint64_t)(S2 >> 112);
    const uint64_t f = (uint64_t)kq * rec->Rcur;
    const pa_u128 p0 = (pa_u128)rec->Q2[0] * f, p1 = (pa_u128)rec->Q2[1] * f;
    const pa_u128 mid = (p0 >> 64) + (pa_u128)(uint64_t)p1;
    const uint64_t r0 = (uint64_t)p0, r1 = (uint64_t)mid, r2 = (uint64_t)(p1 >> 64) + (uint64_t)(mid >> 64);
    return a2 != r2 ? a2 < r2 : (a1 != r1 ? a1 < r1 : a0 < r0);
}

// Whether a run's population is kept (kq < 0: never).  Every workgroup of the
// resampling's first pass decides it from the same sums, which that pass does
// not change; the run's first one records it, and the kept size for the
// capacity and extinction checks, for the passes after it.  (As a launch of its
// own the decision took 4.6 us of a step.)
__device__ __forceinline__ bool decide_kept(PaRecord *rec, int kq, uint32_t block)
{
    if (kq < 0 || ess_below(rec, (uint32_t)kq))
        return false;
    if (block == 0 && threadIdx.x == 0) {
        rec->keep = 1u;
        rec->Rnew = rec->Rcur;
    }
    return true;
}

// Sampling variance, Eq. (5): each chunk sums (r_j - tauhat_j)^2 over its
// replicas in a fixed order (per thread, then the block's fixed tree) into
// partial[chunk]; k_commit adds the partials in chunk order.
__device__ __forceinline__ double sv_term(uint32_t r, uint64_t W, double S, double Rt)
{
    const double tau = ((double)W / S) * Rt;
    const double dlt = (double)r - tau;
    return dlt * dlt;
}

__device__ __forceinline__ void sv_store(const RepCtx &c, double acc, double *sd)
{
    const double t = pa_block_sum_f64(acc, sd);
    if (threadIdx.x == 0)
        c.rd->dv.partial[c.beg / PA_CHUNK] = t;
}

// Poisson by inversion: tauhat = R W / S; tauhat > 32 is cut into
// ceil(tauhat/32) equal pieces, piece p using u from Philox(j, p, i, RS_POIS<<28).
__device__ __forceinline__ uint32_t poisson_copies(const PaRunDesc &rd, uint64_t W, uint64_t S, uint64_t Rt,
                                                   int64_t j, uint32_t step)
{
    const double tau = ((double)W / (double)S) * (double)Rt;
    uint32_t m = 1;
    if (tau > 32.0)
        m = (uint32_t)ceil(tau / 32.0);
    const double mu = tau / (double)m;
    uint32_t tot = 0;
    for (uint32_t p = 0; p < m; ++p) {
        const pa_philox_out o = pa_philox(rd.seed, rd.run_id, (uint32_t)j, p, step, PA_PURPOSE_RS_POIS << 28);
        const double u = ((double)(o.x0 >> 5) * 67108864.0 + (double)(o.x1 >> 6)) * (1.0 / 9007199254740992.0);
        uint32_t k = 0;
        double pr = pa_exp(-mu);
        double F = pr;
        while (u >= F) {
            k += 1;
            pr = (pr * mu) / (double)k;
            const double Fn = F + pr;
            if (Fn == F)
                break;
            F = Fn;
        }
        tot += k;
    }
    return tot;
}

// Systematic: #points (k + U/2^32) S/R below c, k < R, is
// min(R, q + [rho 2^32 > U S]) with c R = q S + rho.
__device__ __forceinline__ uint64_t sys_below(uint64_t c, uint64_t Rt, uint64_t S, uint32_t U)
{
    const pa_u128 cR = (pa_u128)c * Rt;
    uint64_t q = (uint64_t)floor(((double)c * (double)Rt) / (double)S);
    if (q > Rt)
        q = Rt;
    while (q > 0 && (pa_u128)q * S > cR)
        --q;
    while ((pa_u128)(q + 1) * S <= cR)
        ++q;
    const uint64_t rho = (uint64_t)(cR - (pa_u128)q * S);
    const uint64_t n = q + ((((pa_u128)rho) << 32) > ((pa_u128)U * S) ? 1u : 0u);
    return n < Rt ? n : Rt;
}

// Multinomial: U_k = floor(r S / 2^128), r = 128 bits of Philox(k, 0, i,
// RS_MULT<<28), k < R; the box of replica j is [C_{j-1}, C_j).  The chunks of
// the map cover the draws k (capacity >= R).
__global__ __launch_bounds__(kThreads) void k_counts_multinomial(const PaRunDesc *__restrict__ runs,
                                                                 const PaBlk *__restrict__ map)
{
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    const int64_t Rt = rd.R0, Rprev = (int64_t)rec->Rcur;
    const int64_t beg = (int64_t)b.idx * PA_CHUNK;
    if (beg >= Rt || frozen(rec) || rec->keep)
        return;
    const int64_t end = beg + PA_CHUNK < Rt ? beg + PA_CHUNK : Rt;
    const uint64_t S = rec->S;
    const uint32_t step = rec->step + 1;
    const uint64_t *C = rd.dv.C;
    for (int64_t k = beg + threadIdx.x; k < end; k += blockDim.x) {
        const pa_philox_out o = pa_philox(rd.seed, rd.run_id, (uint32_t)k, 0u, step, PA_PURPOSE_RS_MULT << 28);
        const uint64_t lo = (uint64_t)o.x0 | ((uint64_t)o.x1 << 32);
        const uint64_t hi = (uint64_t)o.x2 | ((uint64_t)o.x3 << 32);
        const pa_u128 A = (pa_u128)lo * S, B = (pa_u128)hi * S;
        const uint64_t U = (uint64_t)((B + (A >> 64)) >> 64);
        int64_t a = 0, z = Rprev - 1;
        while (a < z) {
            const int64_t mid = a + ((z - a) >> 1);
            if (C[mid] > U)
                z = mid;
            else
                a = mid + 1;
        }
        atomicAdd(&rd.dv.r[a], 1u);
    }
}

// Sampling variance of the multinomial scheme (its copy numbers are complete
// only after k_counts_multinomial).
__global__ __launch_bounds__(kThreads) void k_sv_partial(const PaRunDesc *__restrict__ runs,
                                                          const PaBlk *__restrict__ map)
{
    __shared__ double sd[16];
    RepCtx c;
    if (!rs_ctx(runs, map, &c))
        return;
    const PaRunDesc &rd = *c.rd;
    const bool wt = c.rec->weighted != 0u;
    const int DN = rd.d * rd.N;
    const int hmin = (c.rec->wemin + DN) >> 2;
    const double S = (double)c.rec->S, Rt = (double)rd.R0;
    const int32_t *E = rd.dv.E[c.rec->cur];
    double acc = 0.0;
    for (int64_t j = c.beg + threadIdx.x; j < c.end; j += blockDim.x)
        acc = acc + sv_term(rd.dv.r[j], rep_weight(c, wt, E, j, DN, hmin), S, Rt);
    sv_store(c, acc, sd);
}

// Decoupled look-back (Merrill & Garland 2016), run by a tile's first wave:
// the tile publishes its aggregate, looks back over up to 64 preceding tiles
// at once (one flag per lane; the nearest tile with an inclusive prefix ends
// the look-back, the aggregates of the tiles after it add up), then
// publishes its own inclusive prefix.  Returns the exclusive prefix in every
// lane of the wave.  The workgroups of a run take their tile index from the
// run's own atomic ticket, so every tile a tile waits on (same run, lower
// index) belongs to a workgroup that is already running; a wait past the
// spin limit sets the run's timeout status and gives up (the resampling is
// then not applied).
__device__ __forceinline__ unsigned long long tile_lookback(PaScanTile *tiles, uint32_t tile,
                                                            unsigned long long agg, PaRecord *rec)
{
    const int lane = threadIdx.x & 63;
    unsigned long long *me = &tiles[tile].word;
    unsigned long long excl = 0;
    if (lane == 0) // tile 0's aggregate is its inclusive prefix
        __hip_atomic_store(me, (tile == 0 ? PA_TILE_INCL : PA_TILE_AGG) | agg, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    if (tile == 0)
        return 0;
    int64_t top = (int64_t)tile - 1; // the window: tiles top - lane
    uint32_t spins = 0;
    for (;;) {
        const int64_t p = top - lane;
        unsigned long long word = PA_TILE_INCL; // before tile 0: an inclusive prefix of 0
        if (p >= 0)
            word = __hip_atomic_load(&tiles[p].word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t f = (uint32_t)(word >> 62);
        const unsigned long long val = word & PA_TILE_VALUE;
        const uint64_t inc = __ballot(f == 2u), pending = __ballot(f == 0u);
        const int first = inc ? __ffsll((long long)inc) - 1 : 64;
        const uint64_t need = first >= 63 ? ~0ull : ((2ull << first) - 1ull); // lanes 0..first
        if (pending & need) { // a tile the prefix needs has not published yet
            if (++spins > (1u << 26)) {
                if (lane == 0)
                    atomicOr(&rec->status, PA_ST_SCAN_TIMEOUT);
                break; // gave up; the status bit is set
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        excl += pa_wave_sum_u64(((need >> lane) & 1ull) ? val : 0ull);
        if (first < 64)
            break;
        top -= 64;
    }
    // a prefix too wide for the word stays unpublished: later tiles then
    // add this tile's aggregate themselves
    if (lane == 0 && excl + agg <= PA_TILE_VALUE)
        __hip_atomic_store(me, PA_TILE_INCL | (excl + agg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return excl;
}

// Exclusive prefix of each thread's `run` within the workgroup (waves by
// shuffles, then the waves' totals through LDS); *agg: the workgroup total.
template <int THREADS>
__device__ __forceinline__ unsigned long long block_excl_scan(unsigned long long run, unsigned long long *s_wave,
                                                              unsigned long long *agg)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long incl = pa_wave_scan_u64(run);
    if (lane == 63)
        s_wave[wave] = incl;
    __syncthreads();
    unsigned long long wave_off = 0, a = 0;
    for (int k = 0; k < THREADS / 64; ++k) {
        if (k < wave)
            wave_off += s_wave[k];
        a += s_wave[k];
    }
    *agg = a;
    return wave_off + incl - run;
}

// The ancestor map of one tile: slot k of thread t (replica tile0 + ITEMS t +
// k) gets the r[k] entries from its offset on, the tile's entries being
// [o0, o1) and the thread's first offset o0 + first.  Entries at or past the
// capacity are not written (a resampling that overflows is not applied).
// The workgroup expands the copy numbers together: over windows of kTile
// entries every slot with copies marks the entry it starts at in LDS, a
// running maximum over the window gives each entry its slot, and the entries
// go out as 16-byte stores.  A thread that wrote its own slots' entries held
// its whole workgroup back where few replicas take most copies (steps of the
// width of the energy distribution): 3D L = 16, R = 10^6, dbeta = 0.02 114 ->
// 29 us for the systematic pass, 3D L = 10, R = 2 x 5 10^5, dbeta = 0.05 101 ->
// 25 us, 32 uneven runs 94 -> 17 us.
// Called by every thread of the workgroup with the same o0, o1, tile0.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void write_ancestors(uint32_t *anc, int64_t cap, uint64_t o0, uint64_t o1, uint64_t first,
                                                const uint32_t (&r)[ITEMS], int64_t tile0,
                                                uint32_t *mark /* THREADS ITEMS, 16-byte aligned */,
                                                uint32_t *s_max /* THREADS / 64 */)
{
    constexpr int kTile = THREADS * ITEMS;
    static_assert(ITEMS % 4 == 0, "items of a thread are whole 16-byte vectors");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t end = o1 < (uint64_t)cap ? o1 : (uint64_t)cap;
    uint32_t carry = 0; // 1 + the tile's slot that covers the window's first entry
    for (uint64_t w0 = o0 & ~3ull; w0 < end; w0 += kTile) { // (o0 rounded down: aligned stores)
#pragma unroll
        for (int k = 0; k < ITEMS / 4; ++k)
            reinterpret_cast<uint4 *>(mark)[tid + k * THREADS] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        uint64_t st = o0 + first;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (r[k] != 0u && st >= w0 && st < w0 + kTile)
                mark[st - w0] = (uint32_t)(tid * ITEMS + k) + 1u;
            st += r[k];
        }
        __syncthreads();
        uint32_t v[ITEMS], top = 0;
#pragma unroll
        for (int k = 0; k < ITEMS / 4; ++k) {
            const uint4 q = reinterpret_cast<const uint4 *>(mark)[tid * (ITEMS / 4) + k];
            v[4 * k] = q.x;
            v[4 * k + 1] = q.y;
            v[4 * k + 2] = q.z;
            v[4 * k + 3] = q.w;
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            top = v[k] > top ? v[k] : top;
            v[k] = top;
        }
        const uint32_t incl = pa_wave_scanmax_u32(top); // running maximum over the wave's lanes
        if (lane == 63)
            s_max[wave] = incl;
        uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x138, 0xF, 0xF, false); // wave_shr 1
        before = carry > before ? carry : before;
        __syncthreads(); // also: the marks have been read
        for (int k = 0; k < THREADS / 64; ++k) {
            const uint32_t m = s_max[k];
            if (k < wave)
                before = m > before ? m : before;
            carry = m > carry ? m : carry;
        }
        const uint64_t d0 = w0 + (uint64_t)(tid * ITEMS);
        const uint32_t a0 = (uint32_t)tile0 - 1u;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            v[k] = a0 + (v[k] > before ? v[k] : before);
        if (d0 >= o0 && d0 + ITEMS <= end) {
#pragma unroll
            for (int k = 0; k < ITEMS / 4; ++k)
                reinterpret_cast<uint4 *>(anc + d0)[k] = make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2],
                                                                    v[4 * k + 3]);
        } else {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k)
                if (d0 + k >= o0 && d0 + k < end)
                    anc[d0 + k] = v[k];
        }
    }
}

// Multinomial copy numbers' exclusive prefix sum, written only as the
// ancestor map: each run's first Rcur copy numbers (entries past Rcur count
// as 0), PA_SCAN_ITEMS consecutive ones per thread, tiles of PA_SCAN_TILE.
__global__ __launch_bounds__(PA_SCAN_THREADS) void k_scan_counts(const PaRunDesc *__restrict__ runs,
                                                                 const PaBlk *__restrict__ map)
{
    static_assert(PA_SCAN_ITEMS % 4 == 0, "items of a thread are whole 16-byte vectors");
    __shared__ uint32_t s_tile;
    __shared__ unsigned long long s_wave[PA_SCAN_THREADS / 64];
    __shared__ unsigned long long s_excl;
    __shared__ alignas(16) uint32_t s_mark[PA_SCAN_TILE];
    __shared__ uint32_t s_max[PA_SCAN_THREADS / 64];
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec) || rec->keep)
        return; // every tile of a frozen (or kept) run returns: none waits
    if (threadIdx.x == 0)
        s_tile = atomicAdd(&rec->ticket[1], 1u);
    __syncthreads();
    const uint32_t tile = s_tile;
    const int64_t n = (int64_t)rec->Rcur;
    const int64_t ntiles = (rd.cap + PA_SCAN_TILE - 1) / PA_SCAN_TILE;
    PaScanTile *tiles = rd.dv.tiles + pa_tiles_per_sum(rd.cap);
    const int64_t base = (int64_t)tile * PA_SCAN_TILE + (int64_t)threadIdx.x * PA_SCAN_ITEMS;
    alignas(16) uint32_t v[PA_SCAN_ITEMS]; // entries past the population count as 0
    if (base + PA_SCAN_ITEMS <= n) {
#pragma unroll
        for (int k = 0; k < PA_SCAN_ITEMS / 4; ++k)
            reinterpret_cast<uint4 *>(v)[k] = reinterpret_cast<const uint4 *>(rd.dv.r + base)[k];
    } else {
#pragma unroll
        for (int k = 0; k < PA_SCAN_ITEMS; ++k)
            v[k] = base + k < n ? rd.dv.r[base + k] : 0u;
    }
    unsigned long long run = 0;
#pragma unroll
    for (int k = 0; k < PA_SCAN_ITEMS; ++k)
        run += v[k];
    unsigned long long agg;
    const unsigned long long thread_excl = block_excl_scan<PA_SCAN_THREADS>(run, s_wave, &agg);
    if ((threadIdx.x >> 6) == 0) {
        const unsigned long long excl = tile_lookback(tiles, tile, agg, rec);
        if ((threadIdx.x & 63) == 0) {
            s_excl = excl;
            if ((int64_t)tile == ntiles - 1)
                rec->Rnew = excl + agg;
        }
    }
    __syncthreads();
    write_ancestors<PA_SCAN_THREADS, PA_SCAN_ITEMS>(rd.dv.anc, rd.cap, s_excl, s_excl + agg, thread_excl, v,
                                                    (int64_t)tile * PA_SCAN_TILE, s_mark, s_max);
}

// The chunk sums of the sampling-variance terms: a wave's slots are one
// chunk when it holds PA_CHUNK of them (ITEMS = 16), else four waves' are
// (ITEMS = 4).  Chunk c goes to out[c]; the barriers publish it to the
// workgroup where out is LDS, and what the first wave wrote to LDS before.
template <int ITEMS>
__device__ __forceinline__ void store_chunk_sv(double *out, int64_t cap, uint32_t tile, double sv, double *sd)
{
    static_assert(64 * ITEMS == PA_CHUNK || kThreads * ITEMS == PA_CHUNK, "chunks of one or of four whole waves");
    const int tid = threadIdx.x, nwaves = (int)(blockDim.x >> 6);
    const double t = pa_wave_sum_f64(sv);
    if (64 * ITEMS == PA_CHUNK) {
        const int64_t chunk = (int64_t)tile * nwaves + (tid >> 6);
        if ((tid & 63) == 0 && chunk * PA_CHUNK < cap)
            out[chunk] = t;
    } else {
        if ((tid & 63) == 0)
            sd[tid >> 6] = t;
        __syncthreads();
        if (tid < nwaves / 4) {
            double c = 0.0;
            for (int k = 0; k < 4; ++k)
                c = c + sd[4 * tid + k];
            out[(int64_t)tile * (nwaves / 4) + tid] = c;
        }
    }
    __syncthreads();
}

// The integer weights of the slots [base, base + ITEMS), 0 past the population.
template <int ITEMS>
__device__ __forceinline__ void load_weights(const PaRunDesc &rd, const PaRecord *rec, int64_t base, int64_t n,
                                             uint64_t (&v)[ITEMS])
{
    const bool wt = rec->weighted != 0u;
    const int DN = rd.d * rd.N;
    const int hmin = (rec->wemin + DN) >> 2;
    const int32_t *E = rd.dv.E[rec->cur];
    if (base + ITEMS <= n && !wt) {
        alignas(16) int32_t e[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS / 4; ++k)
            reinterpret_cast<uint4 *>(e)[k] = reinterpret_cast<const uint4 *>(E + base)[k];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            v[k] = weight_of(e[k], DN, hmin, rd.dv.wtab);
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            v[k] = base + k < n ? (wt ? rd.dv.Wj[base + k] : weight_of(E[base + k], DN, hmin, rd.dv.wtab)) : 0ull;
    }
}

// The systematic copies of a tile's replicas (weights v, their prefix C before
// the thread's first one): N(c) = #points (k + U/2^32) S/R below c, k < R, so
// replica j's copies are [N(C_{j-1}), N(C_j)).  Writes them into the ancestor
// map, the new size (the tile of the last replica) and the chunk sums of the
// sampling variance into `part`.  Called after a barrier past the last use of
// s_wave.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void systematic_copies(const PaRunDesc &rd, PaRecord *rec, uint32_t tile, int64_t n,
                                                  unsigned long long acc, const uint64_t (&v)[ITEMS], double *part,
                                                  unsigned long long *s_wave, double *sd, uint32_t *s_mark,
                                                  uint32_t *s_max)
{
    constexpr int kTile = THREADS * ITEMS;
    const int64_t base = (int64_t)tile * kTile + (int64_t)threadIdx.x * ITEMS;
    const uint64_t S = rec->S, Rt = (uint64_t)rd.R0;
    const uint32_t U = pa_philox(rd.seed, rd.run_id, 0u, 0u, rec->step + 1, PA_PURPOSE_RS_SYS << 28).x0;
    uint64_t lo = sys_below(acc, Rt, S, U); // N(C_{base-1}); N(0) = 0
    const uint64_t first = lo;
    uint32_t r[ITEMS];
    double sv = 0.0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t j = base + k;
        r[k] = 0;
        if (j < n) {
            acc += v[k];
            const uint64_t hi = sys_below(acc, Rt, S, U);
            r[k] = (uint32_t)(hi - lo);
            if (j == n - 1)
                rec->Rnew = hi; // N(S) = Rt: the size is kept
            sv = sv + sv_term(r[k], v[k], (double)S, (double)Rt);
            lo = hi;
        }
    }
    // the tile's range of copies (the barriers of store_chunk_sv publish it)
    if (threadIdx.x == 0)
        s_wave[0] = first;
    if (threadIdx.x == THREADS - 1)
        s_wave[1] = lo;
    store_chunk_sv<ITEMS>(part, rd.cap, tile, sv, sd);
    const uint64_t o0 = s_wave[0], o1 = s_wave[1];
    write_ancestors<THREADS, ITEMS>(rd.dv.anc, rd.cap, o0, o1, first - o0, r, (int64_t)tile * kTile, s_mark, s_max);
}

// Integer weights and their inclusive prefix sums C in one pass: tile t (the
// run's ticket order) holds replica slots [T t, T (t + 1)), T = kThreads
// ITEMS = pa_counts_tile(cap), ITEMS consecutive ones per thread; each weight
// is taken from the replica's energy level (or a weighted population's own)
// as the tile is loaded.  MULTINOMIAL: writes C and returns the copy numbers
// to zero for the draws.  SYSTEMATIC: writes no C but each replica's copy
// range [N(C_{j-1}), N(C_j)) straight into the ancestor map (the points
// below C_{j-1} are the copies of the replicas before j), the new size
// N(C_{R-1}) and the sampling variance per chunk.
constexpr int PA_SCAN_SYSTEMATIC = 0, PA_SCAN_MULTINOMIAL = 1;
template <int MODE, int ITEMS>
__device__ __forceinline__ void weights_scan_tile(const PaRunDesc &rd, PaRecord *rec, uint32_t tile,
                                                  unsigned long long *s_wave, unsigned long long *s_excl,
                                                  double *sd, uint32_t *s_mark, uint32_t *s_max)
{
    constexpr int kTile = kThreads * ITEMS;
    const int64_t n = (int64_t)rec->Rcur;
    const int64_t ntiles = (rd.cap + kTile - 1) / kTile;
    PaScanTile *tiles = rd.dv.tiles;
    const int64_t base = (int64_t)tile * kTile + (int64_t)threadIdx.x * ITEMS;
    const bool whole = base + ITEMS <= n; // the thread's slots are all live
    uint64_t v[ITEMS];
    load_weights<ITEMS>(rd, rec, base, n, v);
    if (MODE == PA_SCAN_MULTINOMIAL) {
        if (whole) {
#pragma unroll
            for (int k = 0; k < ITEMS / 4; ++k)
                reinterpret_cast<uint4 *>(rd.dv.r + base)[k] = make_uint4(0u, 0u, 0u, 0u);
        } else {
            for (int k = 0; k < ITEMS; ++k)
                if (base + k < n)
                    rd.dv.r[base + k] = 0u;
        }
    }
    unsigned long long run = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        run += v[k];
    unsigned long long agg;
    const unsigned long long thread_excl = block_excl_scan<kThreads>(run, s_wave, &agg);
    if ((threadIdx.x >> 6) == 0) {
        const unsigned long long excl = tile_lookback(tiles, tile, agg, rec);
        if ((threadIdx.x & 63) == 0) {
            *s_excl = excl;
            if ((int64_t)tile == ntiles - 1)
                rec->Ctot = excl + agg;
        }
    }
    if (MODE == PA_SCAN_MULTINOMIAL) {
        __syncthreads();
        unsigned long long acc = *s_excl + thread_excl;
        alignas(16) uint64_t o[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            acc += v[k];
            o[k] = acc;
        }
        if (whole) {
#pragma unroll
            for (int k = 0; k < ITEMS / 2; ++k)
                reinterpret_cast<uint4 *>(rd.dv.C + base)[k] = reinterpret_cast<const uint4 *>(o)[k];
        } else {
            for (int k = 0; k < ITEMS; ++k)
                if (base + k < n)
                    rd.dv.C[base + k] = o[k];
        }
        return;
    }
    __syncthreads(); // s_excl
    systematic_copies<kThreads, ITEMS>(rd, rec, tile, n, *s_excl + thread_excl, v, rd.dv.partial, s_wave, sd, s_mark,
                                       s_max);
}

template <int MODE>
__global__ __launch_bounds__(kThreads) void k_weights_scan(const PaRunDesc *__restrict__ runs,
                                                           const PaBlk *__restrict__ map, int kq)
{
    __shared__ uint32_t s_tile;
    __shared__ unsigned long long s_wave[kThreads / 64];
    __shared__ unsigned long long s_excl;
    __shared__ double sd[16];
    __shared__ alignas(16) uint32_t s_mark[MODE == PA_SCAN_SYSTEMATIC ? kThreads * 16 : 4];
    __shared__ uint32_t s_max[kThreads / 64];
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec) || decide_kept(rec, kq, b.idx))
        return; // every tile of a frozen (or kept) run returns: none waits
    if (threadIdx.x == 0)
        s_tile = atomicAdd(&rec->ticket[0], 1u);
    __syncthreads();
    static_assert(kThreads * 16 == 4096 && kThreads * 4 == 1024, "the tiles of pa_counts_tile");
    if (pa_counts_tile(rd.cap) == 4096)
        weights_scan_tile<MODE, 16>(rd, rec, s_tile, s_wave, &s_excl, sd, s_mark, s_max);
    else
        weights_scan_tile<MODE, 4>(rd, rec, s_tile, s_wave, &s_excl, sd, s_mark, s_max);
}

// The copy numbers of the slots [base, base + ITEMS) and their sum: nearest
// integer (SCHEME 2: floor(tauhat) + [u S < (R W mod S) 2^32], u = x0 of
// Philox(j, 0, i, RS_NI<<28)) or Poisson (SCHEME 1); *sv: their
// sampling-variance terms' sum.
template <int SCHEME, int ITEMS>
__device__ __forceinline__ unsigned long long draw_copies(const PaRunDesc &rd, const PaRecord *rec, int64_t base,
                                                          int64_t n, uint32_t (&r)[ITEMS], double *sv)
{
    const bool wt = rec->weighted != 0u;
    const int DN = rd.d * rd.N;
    const int hmin = (rec->wemin + DN) >> 2;
    const uint64_t S = rec->S, Rt = (uint64_t)rd.R0;
    const uint32_t step = rec->step + 1;
    const int32_t *E = rd.dv.E[rec->cur];
    alignas(16) int32_t e[ITEMS];
    if (base + ITEMS <= n && !wt) {
#pragma unroll
        for (int k = 0; k < ITEMS / 4; ++k)
            reinterpret_cast<uint4 *>(e)[k] = reinterpret_cast<const uint4 *>(E + base)[k];
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            e[k] = (!wt && base + k < n) ? E[base + k] : 0;
    }
    *sv = 0.0;
    unsigned long long run = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t j = base + k;
        r[k] = 0;
        if (j >= n)
            continue;
        const uint64_t W = wt ? rd.dv.Wj[j] : weight_of(e[k], DN, hmin, rd.dv.wtab);
        if (SCHEME == 2) {
            const uint64_t a = Rt * W;
            const uint64_t qt = a / S;
            const uint64_t rho = a - qt * S;
            const pa_philox_out o = pa_philox(rd.seed, rd.run_id, (uint32_t)j, 0u, step, PA_PURPOSE_RS_NI << 28);
            const bool extra = ((pa_u128)o.x0 * S) < ((pa_u128)rho << 32);
            r[k] = (uint32_t)qt + (extra ? 1u : 0u);
        } else {
            r[k] = poisson_copies(rd, W, S, Rt, j, step);
        }
        *sv = *sv + sv_term(r[k], W, (double)S, (double)Rt);
        run += r[k];
    }
    return run;
}

// Nearest-integer (SCHEME 2) or Poisson (SCHEME 1) copy numbers drawn and
// summed in one pass: tile t (the run's ticket order) holds replica slots
// [T t, T (t + 1)), T = kThreads ITEMS = pa_counts_tile(cap), ITEMS
// consecutive ones per thread.  Each thread draws its replicas' copy
// numbers, the workgroup sums them, the look-back gives the tile's offset,
// and the ancestor map is written from it.  The sampling-variance terms of
// chunk c (PA_CHUNK slots) go to partial[c].
template <int SCHEME, int ITEMS>
__device__ __forceinline__ void counts_scan_tile(const PaRunDesc &rd, PaRecord *rec, uint32_t *s_tile,
                                                 unsigned long long *s_wave, unsigned long long *s_excl,
                                                 double *sd, uint32_t *s_mark, uint32_t *s_max)
{
    constexpr int kTile = kThreads * ITEMS;
    const uint32_t tile = *s_tile;
    const int64_t n = (int64_t)rec->Rcur;
    const int64_t ntiles = (rd.cap + kTile - 1) / kTile;
    PaScanTile *tiles = rd.dv.tiles + pa_tiles_per_sum(rd.cap);
    const int64_t base = (int64_t)tile * kTile + (int64_t)threadIdx.x * ITEMS;
    uint32_t r[ITEMS];
    double sv;
    const unsigned long long run = draw_copies<SCHEME, ITEMS>(rd, rec, base, n, r, &sv);
    unsigned long long agg;
    const unsigned long long thread_excl = block_excl_scan<kThreads>(run, s_wave, &agg);
    if ((threadIdx.x >> 6) == 0) {
        const unsigned long long excl = tile_lookback(tiles, tile, agg, rec);
        if ((threadIdx.x & 63) == 0) {
            *s_excl = excl;
            if ((int64_t)tile == ntiles - 1)
                rec->Rnew = excl + agg;
        }
    }
    store_chunk_sv<ITEMS>(rd.dv.partial, rd.cap, tile, sv, sd);
    write_ancestors<kThreads, ITEMS>(rd.dv.anc, rd.cap, *s_excl, *s_excl + agg, thread_excl, r,
                                     (int64_t)tile * kTile, s_mark, s_max);
}

template <int SCHEME>
__global__ __launch_bounds__(kThreads) void k_counts_scan(const PaRunDesc *__restrict__ runs,
                                                          const PaBlk *__restrict__ map, int kq)
{
    __shared__ uint32_t s_tile;
    __shared__ unsigned long long s_wave[kThreads / 64];
    __shared__ unsigned long long s_excl;
    __shared__ double sd[16];
    __shared__ alignas(16) uint32_t s_mark[kThreads * 16];
    __shared__ uint32_t s_max[kThreads / 64];
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec) || decide_kept(rec, kq, b.idx))
        return; // every tile of a frozen (or kept) run returns: none waits
    if (threadIdx.x == 0)
        s_tile = atomicAdd(&rec->ticket[1], 1u);
    __syncthreads();
    static_assert(kThreads * 16 == 4096 && kThreads * 4 == 1024, "the tiles of pa_counts_tile");
    if (pa_counts_tile(rd.cap) == 4096)
        counts_scan_tile<SCHEME, 16>(rd, rec, &s_tile, s_wave, &s_excl, sd, s_mark, s_max);
    else
        counts_scan_tile<SCHEME, 4>(rd, rec, &s_tile, s_wave, &s_excl, sd, s_mark, s_max);
}

// A new resampling starts with a clean status (a frozen run stays frozen),
// cleared tile flags for both prefix sums (weights, copy numbers) and their
// tile tickets.  The reweighting prepares its resampling the same way; this
// launch serves a resampling retried after a failed one.
__global__ void k_resample_prep(const PaRunDesc *__restrict__ runs)
{
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    const int64_t ntiles = 2 * pa_tiles_per_sum(rd.cap);
    for (int64_t t = threadIdx.x; t < ntiles; t += blockDim.x)
        rd.dv.tiles[t].word = 0ull;
    if (threadIdx.x == 0) {
        rec->ticket[0] = rec->ticket[1] = 0u;
        if (!frozen(rec)) {
            rec->status = 0;
            rec->skip = 0;
            rec->keep = 0;
        }
    }
}

// Capacity and extinction: a resampling that would not fit (or leave no
// replica), a non-finite ln Q or an unfinished prefix sum is not applied.
// Every kernel after the copy-number scan evaluates this from the same record
// fields, so they agree without a separate pass; k_commit records it.
__device__ __forceinline__ uint32_t resample_status(const PaRecord *rec, int64_t cap)
{
    const uint64_t Rn = rec->Rnew;
    uint32_t st = rec->status & PA_ST_SCAN_TIMEOUT;
    if (Rn > (uint64_t)cap)
        st |= PA_ST_CAPACITY;
    if (Rn == 0)
        st |= PA_ST_EXTINCT;
    const double q = rec->lnQ;
    if (!(q == q) || q - q != 0.0)
        st |= PA_ST_NONFINITE;
    return st;
}

// ------------------------------------------------------------------ apply

// The replicas [beg, end) of a kept population take their new log-weights
// x_j + m (m = 0 if it was uniform).
__device__ __forceinline__ void keep_weights(const PaRunDesc &rd, const PaRecord *rec, int64_t beg, int64_t end)
{
    const bool wt = rec->weighted != 0u;
    const double m = wt ? xmag_value(rec) : 0.0;
    for (int64_t j = beg + threadIdx.x; j < end; j += blockDim.x)
        rd.dv.lw[j] = wx(rd.dv, rec, rec->cur, wt, j) + m;
}

// A resampled population's energies, magnetisations and labels, from their
// ancestors into the other buffer (before the commit swaps the buffers).  Its
// spins follow later (PaRecord::gather): in the next sweep's column load, or
// in k_gather_spins when something else reads them first.  A kept population
// gets its new log-weights here.
__global__ __launch_bounds__(kThreads) void k_gather_meta(const PaRunDesc *__restrict__ runs,
                                                          const PaBlk *__restrict__ map)
{
    const PaBlk blk = map[blockIdx.x];
    const PaRunDesc &rd = runs[blk.run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec) || resample_status(rec, rd.cap) != 0u)
        return;
    const int64_t Rnew = (int64_t)rec->Rnew; // kept: the population's size
    const int64_t beg = (int64_t)blk.idx * PA_CHUNK, end = beg + PA_CHUNK < Rnew ? beg + PA_CHUNK : Rnew;
    if (rec->keep)
        return keep_weights(rd, rec, beg, end);
    const int cur = rec->cur;
    for (int64_t d = beg + threadIdx.x; d < end; d += blockDim.x) {
        const uint32_t a = rd.dv.anc[d];
        rd.dv.E[cur ^ 1][d] = rd.dv.E[cur][a];
        rd.dv.M[cur ^ 1][d] = rd.dv.M[cur][a];
        rd.dv.label[cur ^ 1][d] = rd.dv.label[cur][a];
    }
}

// Word column w of a resampled population from its ancestors.  PRE: before
// the commit swaps the buffers, from the current buffer into the other one,
// with the energies, magnetisations and labels (every run's spins move now).
// Otherwise: after the commit, the spins a resampling left for the sweeps
// (PaRecord::gather), from the other buffer into the current one.
// kGatherThreads lanes with up to eight site pairs each: an item's bookkeeping
// (its scalars and branches) is spread over 16 words a lane; 256 lanes
// with four or eight pairs ran 2 % and 15 % slower at 3D L = 16, R = 10^6,
// dbeta = 0.01.
constexpr int kGatherThreads = 128;
template <bool PRE>
__global__ __launch_bounds__(kGatherThreads) void k_gather_spins(const PaRunDesc *__restrict__ runs,
                                                           const PaBlk *__restrict__ map)
{
    __shared__ uint32_t g_word[64], g_code[64], g_mask[64];
    __shared__ int g_n;
    // an output word takes bits of the source words its ancestors lie in, the
    // same words as its neighbours: neighbouring words go to one XCD
    const PaBlk blk = map[xcd_contiguous(blockIdx.x, gridDim.x)];
    const PaRunDesc &rd = runs[blk.run];
    PaRecord *rec = rd.dv.rec;
    const int64_t R = PRE ? (int64_t)rec->Rnew : (int64_t)rec->Rcur;
    const uint32_t w = blk.idx;
    if (frozen(rec) || (int64_t)w * 64 >= R)
        return;
    if (PRE ? resample_status(rec, rd.cap) != 0u : rec->gather == 0u)
        return;
    if (PRE && rec->keep) // kept: its new log-weights
        return keep_weights(rd, rec, 64 * (int64_t)w, min(64 * (int64_t)w + 64, R));
    const int N = rd.N;
    const int cur = rec->cur;
    const int from = PRE ? cur : cur ^ 1;
    if (PRE && threadIdx.x < 64) { // the replicas' energies, magnetisations and labels
        const int64_t d = 64 * (int64_t)w + threadIdx.x;
        if (d < R) {
            const uint32_t a = rd.dv.anc[d];
            rd.dv.E[cur ^ 1][d] = rd.dv.E[cur][a];
            rd.dv.M[cur ^ 1][d] = rd.dv.M[cur][a];
            rd.dv.label[cur ^ 1][d] = rd.dv.label[cur][a];
        }
    }
    const GatherItems G = {g_word, g_code, g_mask, &g_n};
    gather_items(rd.dv.anc, w, R, G);
    __syncthreads();
    __attribute__((address_space(1))) pa_u64x2 *dst =
        (__attribute__((address_space(1))) pa_u64x2 *)(rd.dv.spins[from ^ 1] + (size_t)w * N);
    auto put = [&](int p, pa_u64x2 v) { dst[p] = v; };
    if (N > 8 * (int)blockDim.x) // more than four site pairs per thread
        gather_sites<8>(rd.dv.spins[from], N, G, put);
    else
        gather_sites<4>(rd.dv.spins[from], N, G, put);
}

// The record after an applied resampling (one thread).
__device__ __forceinline__ void commit_resampled(PaRecord *rec, double sv, uint64_t Rnew, bool gather)
{
    rec->sv = sv;
    rec->lnZ = rec->lnZ + rec->lnQ;
    rec->lnq_hist[0] = rec->lnq_hist[1];
    rec->lnq_hist[1] = rec->lnq_hist[2];
    rec->lnq_hist[2] = rec->lnQ;
    rec->T[0] = rec->Tn[0];
    rec->T[1] = rec->Tn[1];
    rec->T[2] = rec->Tn[2];
    rec->Rprev = rec->Rcur;
    rec->Rcur = Rnew;
    rec->cur ^= 1;
    rec->gather = gather ? 1 : 0; // the spins wait in the other buffer
    rec->beta = rec->beta_next;
    rec->step += 1;
    rec->sweeps = 0;
    rec->weighted = 0;
    rec->resamplings += 1;
}

// Completes an applied resampling: SV (Eq. (5)) from the partials in fixed
// order, ln Z_hat += ln Q (Eq. (7)), the new beta and its thresholds, the
// buffer swap and the step count.  A kept population advances the same way
// with its members in place, its new log-weights and SV = 0 (nothing drawn).
// spins_moved: the spins were gathered before the commit (k_gather_spins<true>).
__global__ __launch_bounds__(kThreads) void k_commit(const PaRunDesc *__restrict__ runs, int freeze,
                                                     int spins_moved)
{
    __shared__ double sd[16];
    const PaRunDesc &rd = runs[blockIdx.x];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec))
        return;
    const uint32_t st = resample_status(rec, rd.cap);
    __syncthreads(); // every thread has read the status before thread 0 writes it
    if (st != 0u) {
        if (threadIdx.x == 0) {
            rec->skip = 1;
            rec->status = freeze ? (st | PA_ST_FROZEN) : st;
            rec->gather = 0;
        }
        return;
    }
    if (rec->keep) {
        if (threadIdx.x == 0) {
            rec->gather = 0;
            rec->sv = 0.0;
            rec->lnZ = rec->lnZ + rec->lnQ;
            rec->lnq_hist[0] = rec->lnq_hist[1];
            rec->lnq_hist[1] = rec->lnq_hist[2];
            rec->lnq_hist[2] = rec->lnQ;
            rec->T[0] = rec->Tn[0];
            rec->T[1] = rec->Tn[1];
            rec->T[2] = rec->Tn[2];
            rec->Rprev = rec->Rcur;
            rec->beta = rec->beta_next;
            rec->step += 1;
            rec->sweeps = 0;
            rec->weighted = 1;
        }
        return;
    }
    const int64_t Rprev = (int64_t)rec->Rcur;
    const int nlive = (int)((Rprev + PA_CHUNK - 1) / PA_CHUNK);
    double v = 0.0;
    for (int k = threadIdx.x; k < nlive; k += blockDim.x)
        v = v + rd.dv.partial[k];
    const double t = pa_block_sum_f64(v, sd);
    if (threadIdx.x == 0)
        commit_resampled(rec, t / (double)Rprev, rec->Rnew, spins_moved == 0);
}

// The whole resampling of a small run (capacity up to PA_SMALL_CAP) by one
// workgroup: copy numbers (SCHEME as above, 3: systematic), ancestor map,
// energies, magnetisations and labels, and the commit.  Its spins follow as a
// large run's that the sweeps gather (PaRecord::gather).  Bound by its chain of
// dependent loads; three launches (copy numbers, gather, commit) with a chain
// each become one: R = 1000 6.2 + 3.8 + 2.6 us -> 9.5 and two launches less,
// 1024 runs of R = 100 8.1 + 4.7 + 4.8 -> 9.6.  Every sum keeps the large
// runs' order and every number their definition, so a run's results depend
// neither on T (256 only where the run fits one chunk: small_launches) nor on
// the launches of its batch.
template <int T, int SCHEME>
__device__ __forceinline__ void resample_small_run(const PaRunDesc &rd, PaRecord *rec, int freeze)
{
    constexpr int kItems = 4, kPer = PA_SMALL_CAP / 1024;
    static_assert(kPer * 256 >= PA_CHUNK && kThreads * kItems == PA_CHUNK, "every slot has a lane's item");
    __shared__ unsigned long long s_wave[T / 64];
    __shared__ double sd[16], part[T / kThreads];
    __shared__ alignas(16) uint32_t s_mark[T * kItems];
    __shared__ uint32_t s_max[T / 64];
    const int tid = threadIdx.x, cur = rec->cur;
    const int64_t n = (int64_t)rec->Rcur, base = (int64_t)tid * kItems;
    unsigned long long agg;
    if (SCHEME == 3) {
        uint64_t v[kItems];
        load_weights<kItems>(rd, rec, base, n, v);
        unsigned long long run = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            run += v[k];
        const unsigned long long before = block_excl_scan<T>(run, s_wave, &agg);
        __syncthreads(); // the waves' totals have been read
        systematic_copies<T, kItems>(rd, rec, 0u, n, before, v, part, s_wave, sd, s_mark, s_max);
        agg = s_wave[1]; // the copies end at N(S)
    } else {
        uint32_t r[kItems];
        double sv;
        const unsigned long long run = draw_copies<SCHEME, kItems>(rd, rec, base, n, r, &sv);
        const unsigned long long before = block_excl_scan<T>(run, s_wave, &agg);
        store_chunk_sv<kItems>(part, rd.cap, 0u, sv, sd);
        write_ancestors<T, kItems>(rd.dv.anc, rd.cap, 0u, agg, before, r, 0, s_mark, s_max);
        if (tid == 0)
            rec->Rnew = agg;
    }
    __syncthreads(); // the ancestor map and the new size
    const uint32_t st = resample_status(rec, rd.cap);
    const int64_t Rnew = (int64_t)agg;
    if (st == 0u) {
        uint32_t a[kPer];
        int32_t e[kPer], m[kPer];
        uint32_t l[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) { // a slot past the end loads the last one's
            const int64_t d = tid + k * T;
            a[k] = rd.dv.anc[d < Rnew ? d : Rnew - 1];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            e[k] = rd.dv.E[cur][a[k]];
            m[k] = rd.dv.M[cur][a[k]];
            l[k] = rd.dv.label[cur][a[k]];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t d = tid + k * T;
            if (d < Rnew) {
                rd.dv.E[cur ^ 1][d] = e[k];
                rd.dv.M[cur ^ 1][d] = m[k];
                rd.dv.label[cur ^ 1][d] = l[k];
            }
        }
    }
    __syncthreads(); // every thread has read the record before thread 0 writes it
    if (st != 0u) {
        if (tid == 0) {
            rec->skip = 1;
            rec->status = freeze ? (st | PA_ST_FROZEN) : st;
            rec->gather = 0;
        }
        return;
    }
    if (tid < 64) {
        const int nlive = (int)((n + PA_CHUNK - 1) / PA_CHUNK);
        const double t = pa_wave_sum_f64(tid < nlive ? part[tid] : 0.0);
        if (tid == 0)
            commit_resampled(rec, t / (double)n, (uint64_t)Rnew, true);
    }
}

template <int T, int SCHEME>
__global__ __launch_bounds__(T) void k_resample_small(const PaRunDesc *__restrict__ runs,
                                                      const uint32_t *__restrict__ list, int freeze)
{
    const PaRunDesc &rd = runs[list ? list[blockIdx.x] : blockIdx.x];
    if (!frozen(rd.dv.rec))
        resample_small_run<T, SCHEME>(rd, rd.dv.rec, freeze);
}

// The reweighting (of a uniform population) and the resampling of a small run
// in one launch, for steps that nobody looks into in between: 1024 runs of 2D
// L = 16, R = 100 5.9 + 9.8 us -> 13.3.
template <int T, int SCHEME>
__global__ __launch_bounds__(T) void k_advance_small(const PaRunDesc *__restrict__ runs,
                                                     const uint32_t *__restrict__ list, double beta_next, int freeze)
{
    const PaRunDesc &rd = runs[list ? list[blockIdx.x] : blockIdx.x];
    if (frozen(rd.dv.rec))
        return;
    reweight_run<T>(rd, rd.dv.rec, beta_next);
    __syncthreads(); // the record, the level weights and the cleared histogram
    resample_small_run<T, SCHEME>(rd, rd.dv.rec, freeze);
}

// ------------------------------------------------------------------ step 4: observables
// Counters of the level histogram a block of the observables pass keeps in
// LDS: its energies' levels, from its lowest; a wider spread (high
// temperatures, large lattices) goes to the run's histogram directly.
constexpr int kObsLevels = 2048;

__global__ __launch_bounds__(kThreads) void k_obs_rep(const PaRunDesc *__restrict__ runs,
                                                      const PaBlk *__restrict__ map, int build_hist)
{
    __shared__ uint64_t su[16 * 5];
    __shared__ double sd[16 * PA_WPARTS];
    __shared__ uint32_t lh[kObsLevels];
    __shared__ int s_lo[kThreads / 64], s_hi[kThreads / 64];
    // pa_counts_tile replica slots per workgroup: four chunks where the run
    // fills the chip so (fewer workgroups merge their level counts and sums
    // into the run's, on the same addresses), else one (R = 20011 on five
    // workgroups took 19.4 us, on twenty 10.9; R = 10^5 19.9 -> 12.4)
    RepCtx c;
    {
        const PaBlk b = map[blockIdx.x];
        c.rd = runs + b.run;
        c.rec = c.rd->dv.rec;
        const int64_t R = (int64_t)c.rec->Rcur;
        const int64_t tile = pa_counts_tile(c.rd->cap);
        c.beg = (int64_t)b.idx * tile;
        c.end = c.beg + tile < R ? c.beg + tile : R;
        if (c.beg >= R || frozen(c.rec))
            return;
    }
    const PaDev &dv = c.rd->dv;
    const int cur = c.rec->cur;
    const int DN = c.rd->d * c.rd->N;
    // the level histogram of the population (for the next reweighting, the
    // step rule and the step model): the block's energy range first, then
    // per-block counts in LDS merged with one atomic per populated level
    int hlo = 0, nlh = 0;
    if (build_hist) {
        int blo = INT_MAX, bhi = INT_MIN;
        for (int64_t d = c.beg + threadIdx.x; d < c.end; d += blockDim.x) {
            const int e = dv.E[cur][d];
            blo = min(blo, e);
            bhi = max(bhi, e);
        }
        block_energy_range(blo, bhi, s_lo, s_hi);
        hlo = (blo + DN) >> 2;
        nlh = ((bhi + DN) >> 2) - hlo + 1;
        if (nlh <= kObsLevels)
            for (int k = threadIdx.x; k < nlh; k += blockDim.x)
                lh[k] = 0;
        if (threadIdx.x == 0) {
            atomicMin(&c.rec->emin, blo);
            atomicMax(&c.rec->emax, bhi);
        }
        __syncthreads();
    }
    uint64_t sE = 0, sE2 = 0, sA = 0, sM2 = 0, sE3 = 0; // sE3: int64 bits (|sum| < 2^63 per block)
    const int lane = threadIdx.x & 63;
    // a weighted population: sums of w, wE, wE^2, wE^3, w|M|, wM^2, w^2 with w = pa_exp(lw)
    const bool wt = c.rec->weighted != 0u;
    double ws[PA_WPARTS] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    static_assert(PA_CHUNK % kThreads == 0, "whole chunks of whole passes");
    const int64_t chunks = (c.rd->cap + PA_CHUNK - 1) / PA_CHUNK;
    // kPre passes' loads are issued before the first pass's atomics (which
    // the compiler would not let later loads pass); a slot past the end loads
    // the last slot again and is not counted
    constexpr int kPre = 4;
    for (int64_t base0 = c.beg; base0 < c.end; base0 += kPre * (int64_t)blockDim.x) {
        int32_t pe[kPre], pm[kPre];
        uint32_t pl[kPre];
        double plw[kPre];
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int64_t d = base0 + k * (int64_t)blockDim.x + threadIdx.x;
            const int64_t dc = d < c.end ? d : c.end - 1;
            pe[k] = dv.E[cur][dc];
            pm[k] = dv.M[cur][dc];
            pl[k] = dv.label[cur][dc];
            plw[k] = wt ? dv.lw[dc] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int64_t base = base0 + k * (int64_t)blockDim.x;
            if (base >= c.end)
                break;
            const int64_t d = base + threadIdx.x;
            const bool valid = d < c.end;
            uint32_t lab = 0xFFFFFFFFu;
            if (valid) {
                const int64_t e = pe[k], m = pm[k];
                if (build_hist) {
                    const int h = ((int)e + DN) >> 2;
                    if (nlh <= kObsLevels)
                        atomicAdd(&lh[h - hlo], 1u);
                    else
                        atomicAdd(&dv.hist[h], 1u);
                }
                sE += (uint64_t)e;
                sE2 += (uint64_t)(e * e);
                sE3 += (uint64_t)(e * e * e);
                sA += (uint64_t)(m < 0 ? -m : m);
                sM2 += (uint64_t)(m * m);
                lab = pl[k];
                if (wt) {
                    const double w = pa_exp(plw[k]), ef = (double)e, mf = (double)(m < 0 ? -m : m);
                    ws[0] = ws[0] + w;
                    ws[1] = ws[1] + w * ef;
                    ws[2] = ws[2] + w * (ef * ef);
                    ws[3] = ws[3] + w * (ef * ef * ef);
                    ws[4] = ws[4] + w * mf;
                    ws[5] = ws[5] + w * (mf * mf);
                    ws[6] = ws[6] + w * w;
                }
            }
            // family counts: one atomic per run of equal labels in the wave (the
            // resampling keeps copies adjacent, so runs are long)
            const uint32_t prev = (uint32_t)__shfl_up((int)lab, 1, 64);
            const bool start = valid && (lane == 0 || lab != prev);
            const uint64_t sm = __ballot(start), vm = __ballot(valid);
            if (start) {
                const uint64_t above = lane == 63 ? 0ull : ((sm | ~vm) & ~((2ull << lane) - 1ull));
                const int stop = above ? __ffsll((long long)above) - 1 : 64;
                atomicAdd(&dv.fam[lab], (uint32_t)(stop - lane));
            }
            // a weighted population's sums per chunk of PA_CHUNK slots, in the
            // fixed order of the block sum
            if (wt && ((base + (int64_t)blockDim.x) % PA_CHUNK == 0 || base + (int64_t)blockDim.x >= c.end)) {
                pa_block_sum_f64x(ws, sd);
                if (threadIdx.x == 0)
#pragma unroll
                    for (int f = 0; f < PA_WPARTS; ++f)
                        dv.wpart[f * chunks + base / PA_CHUNK] = ws[f];
#pragma unroll
                for (int f = 0; f < PA_WPARTS; ++f)
                    ws[f] = 0.0;
            }
        }
    }
    uint64_t sums[5] = {sE, sE2, sA, sM2, sE3};
    pa_block_sum_u64x(sums, su); // (its barriers also end the LDS counting)
    sE = sums[0];
    sE2 = sums[1];
    sA = sums[2];
    sM2 = sums[3];
    sE3 = sums[4];
    if (build_hist && nlh <= kObsLevels)
        for (int k = threadIdx.x; k < nlh; k += blockDim.x)
            if (lh[k])
                atomicAdd(&dv.hist[hlo + k], lh[k]);
    if (threadIdx.x == 0) {
        // 128-bit add of the block's signed sum: low word, then the high word
        // with the carry out of the low word (order-free, hence exact)
        const unsigned long long lo = sE3, hi = (long long)sE3 < 0 ? ~0ull : 0ull;
        const unsigned long long old = atomicAdd(&c.rec->accE3[0], lo);
        atomicAdd(&c.rec->accE3[1], hi + (old + lo < old ? 1ull : 0ull));
        atomicAdd(&c.rec->accE, (unsigned long long)sE);
        atomicAdd(&c.rec->accE2, (unsigned long long)sE2);
        atomicAdd(&c.rec->accAbsM, (unsigned long long)sA);
        atomicAdd(&c.rec->accM2, (unsigned long long)sM2);
    }
}

// Family statistics over PA_HCHUNK family slots per workgroup: sum of c^2,
// the number of families and sum of c ln c (partial[block], in the block's
// fixed order; k_obs_final adds them in block order); the counts return to
// zero for the next pass.
__global__ __launch_bounds__(kThreads) void k_obs_fam(const PaRunDesc *__restrict__ runs,
                                                      const PaBlk *__restrict__ map)
{
    __shared__ uint64_t su[16 * 2];
    __shared__ double sd[16];
    const PaBlk b = map[blockIdx.x];
    const PaRunDesc &rd = runs[b.run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec))
        return;
    const int64_t beg = (int64_t)b.idx * PA_HCHUNK;
    const int64_t end = beg + PA_HCHUNK < rd.R0 ? beg + PA_HCHUNK : rd.R0;
    uint64_t c2 = 0, nf = 0;
    double cl = 0.0;
    // four passes' loads before their stores (a slot past the end loads the
    // last slot again and is not counted)
    constexpr int kPre = 4;
    for (int64_t f0 = beg; f0 < end; f0 += kPre * (int64_t)blockDim.x) {
        uint32_t pc[kPre];
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int64_t f = f0 + k * (int64_t)blockDim.x + threadIdx.x;
            pc[k] = rd.dv.fam[f < end ? f : end - 1];
        }
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int64_t f = f0 + k * (int64_t)blockDim.x + threadIdx.x;
            const uint64_t c = pc[k];
            if (f < end && c) {
                c2 += c * c;
                rd.dv.fam[f] = 0;
                nf += 1;
                cl = cl + (double)c * log((double)c);
            }
        }
    }
    uint64_t sums[2] = {c2, nf};
    pa_block_sum_u64x(sums, su);
    cl = pa_block_sum_f64(cl, sd);
    if (threadIdx.x == 0) {
        atomicAdd(&rec->accC2, (unsigned long long)sums[0]);
        atomicAdd(&rec->accFam, (unsigned long long)sums[1]);
        rd.dv.partial[b.idx] = cl;
    }
}

// A signed 128-bit integer (two's complement words) to double: magnitude
// from its two non-negative words, so no cancellation between them.
__device__ __forceinline__ double i128_to_double(unsigned long long lo, unsigned long long hi)
{
    const bool neg = (long long)hi < 0;
    if (neg) {
        lo = ~lo + 1ull;
        hi = ~hi + (lo == 0ull ? 1ull : 0ull);
    }
    const double m = (double)hi * 18446744073709551616.0 + (double)lo;
    return neg ? -m : m;
}

// The exact sums of a population and its families.
struct ObsSums {
    uint64_t E, E2, absM, M2, E3lo, E3hi, C2, families;
};

// Averages of step 4 and the family statistics, written to the record: rho_t =
// sum_k c_k^2 / R (Eq. (6) with n_k = c_k / R), S_f = ln R - (1/R) sum_k c_k ln
// c_k (clnc).  A weighted population reports weighted averages sum_j w_j O_j /
// sum_j w_j and ESS = (sum w)^2 / sum w^2 (the integer sums and family
// statistics stay those of the members).
__device__ __forceinline__ void publish_averages(PaRecord *rec, int N, const ObsSums &s, double clnc, bool wt,
                                                 const double (&ws)[PA_WPARTS])
{
    rec->sumE = s.E;
    rec->sumE2 = s.E2;
    rec->sumAbsM = s.absM;
    rec->sumM2 = s.M2;
    rec->sumC2 = s.C2;
    rec->families = s.families;
    rec->sumE3[0] = s.E3lo;
    rec->sumE3[1] = s.E3hi;
    const double n = (double)N, r = (double)rec->Rcur;
    rec->e3 = i128_to_double(s.E3lo, s.E3hi) / (n * n * n * r);
    rec->sumClnC = clnc;
    rec->e = (double)(long long)s.E / (n * r);
    rec->e2 = (double)(long long)s.E2 / (n * n * r);
    rec->abs_m = (double)(long long)s.absM / (n * r);
    rec->m2 = (double)(long long)s.M2 / (n * n * r);
    rec->rho_t = (double)s.C2 / r;
    rec->S_f = log(r) - clnc / r;
    rec->ess = r;
    if (wt) {
        rec->e = ws[1] / ws[0] / n;
        rec->e2 = ws[2] / ws[0] / (n * n);
        rec->e3 = ws[3] / ws[0] / (n * n * n);
        rec->abs_m = ws[4] / ws[0] / n;
        rec->m2 = ws[5] / ws[0] / (n * n);
        rec->ess = ws[0] * ws[0] / ws[6];
    }
}

// The row of temperature point `point` of a batched anneal.
__device__ __forceinline__ void write_step_record(const PaRecord *rec, PaStepRecord *o, int point)
{
    o->beta = rec->beta;
    o->lnQ = point > 0 ? rec->lnQ : 0.0;
    o->lnZ = rec->lnZ;
    o->sv = rec->sv;
    o->e = rec->e;
    o->e2 = rec->e2;
    o->abs_m = rec->abs_m;
    o->m2 = rec->m2;
    o->rho_t = rec->rho_t;
    o->S_f = rec->S_f;
    o->R = (long long)rec->Rcur;
    o->sumE = (long long)rec->sumE;
    o->sumE2 = (long long)rec->sumE2;
    o->sumAbsM = (long long)rec->sumAbsM;
    o->sumM2 = (long long)rec->sumM2;
    o->sumC2 = (long long)rec->sumC2;
    o->families = (long long)rec->families;
    o->status = rec->status;
    o->pad = 0;
}

// Publishes the averages of the runs whose passes were k_obs_rep and k_obs_fam
// (the large ones), from their accumulators and partial sums.
__global__ __launch_bounds__(kThreads) void k_obs_final(const PaRunDesc *__restrict__ runs,
                                                        const uint32_t *__restrict__ list, PaStepRecord *steprec,
                                                        int npoints, int point)
{
    __shared__ double sd[16 * PA_WPARTS];
    const uint32_t run = list[blockIdx.x];
    const PaRunDesc &rd = runs[run];
    PaRecord *rec = rd.dv.rec;
    const bool fz = frozen(rec);
    const bool wt = !fz && rec->weighted != 0u;
    const int nparts = (int)((rd.R0 + PA_HCHUNK - 1) / PA_HCHUNK); // k_obs_fam's workgroups
    double v = 0.0;
    if (!fz)
        for (int k = threadIdx.x; k < nparts; k += blockDim.x)
            v = v + rd.dv.partial[k];
    const double t = pa_block_sum_f64(v, sd);
    double ws[PA_WPARTS] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (wt) {
        const int64_t chunks = (rd.cap + PA_CHUNK - 1) / PA_CHUNK;
        const int nlive = (int)(((int64_t)rec->Rcur + PA_CHUNK - 1) / PA_CHUNK);
        for (int k = threadIdx.x; k < nlive; k += blockDim.x)
#pragma unroll
            for (int f = 0; f < PA_WPARTS; ++f)
                ws[f] = ws[f] + rd.dv.wpart[f * chunks + k];
        pa_block_sum_f64x(ws, sd);
    }
    if (threadIdx.x != 0)
        return;
    if (!fz) {
        const ObsSums s = {rec->accE, rec->accE2, rec->accAbsM, rec->accM2,
                           rec->accE3[0], rec->accE3[1], rec->accC2, rec->accFam};
        rec->accE = rec->accE2 = rec->accAbsM = rec->accM2 = rec->accC2 = rec->accFam = 0;
        rec->accE3[0] = rec->accE3[1] = 0;
        publish_averages(rec, rd.N, s, t, wt, ws);
    }
    if (steprec)
        write_step_record(rec, steprec + (size_t)run * npoints + point, point);
}

// The whole observables pass of a small run (capacity up to PA_SMALL_CAP) by
// one workgroup: energy range, level histogram, sums, families (counted in
// LDS) and averages.  The three passes of a large run cost a small one their
// launches and their chains of dependent loads: R = 1000 9.1 + 4.0 + 3.0 us ->
// 7.2, 1024 runs of R = 100 10.3 + 5.4 + 6.2 -> 9.4.  A group of 256 lanes takes
// each chunk (its replicas are loaded once, before anything waits); with
// several chunks a group, R = 20011 took 30 us in one workgroup, as long as in
// three passes.  Every floating-point sum keeps the large runs' order, so a
// run's numbers depend neither on T (256 only where the run fits one chunk:
// small_launches) nor on which side of PA_SMALL_CAP it is.
template <int T>
__global__ __launch_bounds__(T) void k_obs_small(const PaRunDesc *__restrict__ runs,
                                                 const uint32_t *__restrict__ list, int build_hist,
                                                 PaStepRecord *steprec, int npoints, int point)
{
    constexpr int kPer = PA_CHUNK / kThreads;
    static_assert(PA_SMALL_CAP <= PA_HCHUNK && PA_SMALL_CAP <= 4 * PA_CHUNK, "one chunk a group, one chunk of families");
    __shared__ uint32_t fam[PA_SMALL_CAP];
    __shared__ uint32_t lh[kObsLevels];
    __shared__ uint64_t su[7][kThreads], tot[7];
    __shared__ double sw[T / 64][PA_WPARTS], sf[4], logs[64];
    __shared__ int s_lo[T / 64], s_hi[T / 64];
    const uint32_t run = list ? list[blockIdx.x] : blockIdx.x;
    const PaRunDesc &rd = runs[run];
    PaRecord *rec = rd.dv.rec;
    if (frozen(rec)) {
        if (threadIdx.x == 0 && steprec)
            write_step_record(rec, steprec + (size_t)run * npoints + point, point);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = tid / kThreads, t = tid % kThreads;
    const int R = (int)rec->Rcur, R0 = (int)rd.R0, cur = rec->cur;
    const int DN = rd.d * rd.N;
    const PaDev &dv = rd.dv;
    const bool wt = rec->weighted != 0u;
    int32_t pe[kPer], pm[kPer];
    uint32_t pl[kPer];
    double plw[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) { // a slot past the end loads the last one again and is not counted
        const int d = min(chunk * PA_CHUNK + k * kThreads + t, R - 1);
        pe[k] = dv.E[cur][d];
        pm[k] = dv.M[cur][d];
        pl[k] = dv.label[cur][d];
        plw[k] = wt ? dv.lw[d] : 0.0;
    }
    for (int f = tid; f < R0; f += T)
        fam[f] = 0;
    for (int k = tid; k < 7 * kThreads; k += T)
        (&su[0][0])[k] = 0;
    if (tid < 64) // ln of the small family sizes (most of them)
        logs[tid] = tid > 1 ? log((double)tid) : 0.0;
    int hlo = 0, nlh = 0;
    if (build_hist) {
        int lo = pe[0], hi = pe[0];
#pragma unroll
        for (int k = 1; k < kPer; ++k) {
            lo = min(lo, pe[k]);
            hi = max(hi, pe[k]);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            lo = min(lo, __shfl_xor(lo, m, 64));
            hi = max(hi, __shfl_xor(hi, m, 64));
        }
        if (lane == 0) {
            s_lo[wave] = lo;
            s_hi[wave] = hi;
        }
        __syncthreads();
        for (int k = 0; k < T / 64; ++k) {
            lo = min(lo, s_lo[k]);
            hi = max(hi, s_hi[k]);
        }
        hlo = (lo + DN) >> 2;
        nlh = ((hi + DN) >> 2) - hlo + 1;
        if (nlh <= kObsLevels)
            for (int k = tid; k < nlh; k += T)
                lh[k] = 0;
        if (tid == 0) {
            rec->emin = lo;
            rec->emax = hi;
        }
    }
    __syncthreads();
    uint64_t sums[7] = {0, 0, 0, 0, 0, 0, 0}; // E, E^2, |M|, M^2, E^3 (int64 bits), c^2, families
    double ws[PA_WPARTS] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const bool valid = chunk * PA_CHUNK + k * kThreads + t < R;
        uint32_t lab = 0xFFFFFFFFu;
        if (valid) {
            const int64_t e = pe[k], m = pm[k];
            if (build_hist) {
                const int h = ((int)e + DN) >> 2;
                if (nlh <= kObsLevels)
                    atomicAdd(&lh[h - hlo], 1u);
                else
                    atomicAdd(&dv.hist[h], 1u);
            }
            sums[0] += (uint64_t)e;
            sums[1] += (uint64_t)(e * e);
            sums[2] += (uint64_t)(m < 0 ? -m : m);
            sums[3] += (uint64_t)(m * m);
            sums[4] += (uint64_t)(e * e * e);
            lab = pl[k];
            if (wt) {
                const double w = pa_exp(plw[k]), ef = (double)e, mf = (double)(m < 0 ? -m : m);
                ws[0] = ws[0] + w;
                ws[1] = ws[1] + w * ef;
                ws[2] = ws[2] + w * (ef * ef);
                ws[3] = ws[3] + w * (ef * ef * ef);
                ws[4] = ws[4] + w * mf;
                ws[5] = ws[5] + w * (mf * mf);
                ws[6] = ws[6] + w * w;
            }
        }
        // family counts: one atomic per run of equal labels in the wave
        const uint32_t prev = (uint32_t)__shfl_up((int)lab, 1, 64);
        const bool start = valid && (lane == 0 || lab != prev);
        const uint64_t sm = __ballot(start), vm = __ballot(valid);
        if (start) {
            const uint64_t above = lane == 63 ? 0ull : ((sm | ~vm) & ~((2ull << lane) - 1ull));
            const int stop = above ? __ffsll((long long)above) - 1 : 64;
            atomicAdd(&fam[lab], (uint32_t)(stop - lane));
        }
    }
    if (wt) {
#pragma unroll
        for (int f = 0; f < PA_WPARTS; ++f) {
            const double v = pa_wave_sum_f64(ws[f]);
            if (lane == 0)
                sw[wave][f] = v;
        }
    }
    __syncthreads(); // the counts in LDS are complete
    if (build_hist && nlh <= kObsLevels)
        for (int k = tid; k < nlh; k += T)
            if (lh[k])
                dv.hist[hlo + k] = lh[k]; // the histogram was zero
    if (wave < 4) { // families: the 256 lanes of a large run's one workgroup
        double cl = 0.0;
        for (int f = tid; f < R0; f += kThreads) {
            const uint64_t c = fam[f];
            if (c) {
                sums[5] += c * c;
                sums[6] += 1;
                if (c > 1)
                    cl = cl + (double)c * (c < 64 ? logs[c] : log((double)c));
            }
        }
        cl = pa_wave_sum_f64(cl);
        if (lane == 0)
            sf[wave] = cl;
    }
    // the block's sums: lane t's of every group meet in LDS, then 32 lanes add each quantity's 256
#pragma unroll
    for (int q = 0; q < 7; ++q)
        atomicAdd((unsigned long long *)&su[q][t], (unsigned long long)sums[q]);
    __syncthreads();
    if (tid < 7 * 32) {
        uint64_t v = 0;
        for (int k = tid & 31; k < kThreads; k += 32)
            v += su[tid >> 5][k];
        for (int m = 16; m >= 1; m >>= 1)
            v += pa_shfl_xor_u64(v, m);
        if ((tid & 31) == 0)
            tot[tid >> 5] = v;
    }
    __syncthreads();
    if (tid != 0)
        return;
    const double clnc = ((sf[0] + sf[1]) + sf[2]) + sf[3];
    // the chunks' sums (their four waves in order) as the large runs add them: a butterfly over up to 4 lanes
    if (wt)
        for (int f = 0; f < PA_WPARTS; ++f) {
            double c[4] = {0.0, 0.0, 0.0, 0.0};
            for (int q = 0; q < T / kThreads; ++q)
                if (q * PA_CHUNK < R)
                    c[q] = ((sw[4 * q][f] + sw[4 * q + 1][f]) + sw[4 * q + 2][f]) + sw[4 * q + 3][f];
            ws[f] = (c[0] + c[2]) + (c[1] + c[3]);
        }
    const ObsSums s = {tot[0], tot[1], tot[2], tot[3], tot[4], (int64_t)tot[4] < 0 ? ~0ull : 0ull, tot[5], tot[6]};
    publish_averages(rec, rd.N, s, clnc, wt, ws);
    if (steprec)
        write_step_record(rec, steprec + (size_t)run * npoints + point, point);
}

// ------------------------------------------------------------------ overlap
// Pairs replica d of run a with replica d of run b: per word column, the
// bit-sliced count of differing sites per replica, then q-histogram entry
// N - count.
__global__ __launch_bounds__(kThreads) void k_overlap(const PaRunDesc *__restrict__ A,
                                                      const PaRunDesc *__restrict__ B, unsigned long long *hist)
{
    __shared__ uint64_t red[kThreads / 64][16];
    const uint32_t w = blockIdx.x;
    const PaRecord *ra = A->dv.rec, *rb = B->dv.rec;
    const int64_t R = ra->Rcur < rb->Rcur ? (int64_t)ra->Rcur : (int64_t)rb->Rcur;
    if ((int64_t)w * 64 >= R)
        return;
    const int N = A->N;
    const uint64_t *a = A->dv.spins[ra->cur] + (size_t)w * N;
    const uint64_t *b = B->dv.spins[rb->cur] + (size_t)w * N;
    uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    uint64_t c16[16];
    // up to 64 sites per thread with 256 threads and N <= 16384: fits 8 planes
    for (int s = threadIdx.x; s < N; s += 2 * blockDim.x) {
        const int t = s + blockDim.x;
        vadd2_at<0>(v, a[s] ^ b[s], t < N ? a[t] ^ b[t] : 0ull);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
        c16[k] = k < 8 ? v[k] : 0;
    wave_vsum16(c16);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == 0)
        for (int k = 0; k < 16; ++k)
            red[wave][k] = c16[k];
    __syncthreads();
    if (wave == 0) {
        uint32_t cnt = 0;
        for (int q = 0; q < nw; ++q)
            for (int k = 0; k < 16; ++k)
                cnt += (uint32_t)((red[q][k] >> lane) & 1u) << k;
        const int64_t d = 64 * (int64_t)w + lane;
        if (d < R)
            atomicAdd(&hist[N - (int)cnt], 1ull);
    }
}

// Free-energy-weighted combination of runs (Eqs. (9)-(10)), one workgroup per
// group g: over the runs m with group_of[m] == g, l_m = ln R_i^(m) + ln
// Z_hat_i^(m), omega_m = exp(l_m - l_max) / sum exp(l - l_max); ln Z of the
// pooled population = l_max + ln sum exp(l - l_max) - ln sum R^(m); moments
// are weighted averages and c, chi follow Eqs. (11)-(12).  Every thread takes
// every 256th run and the block sums keep a fixed order.  Latency of the
// record reads: one thread per group that walked through its runs took 2067 us
// for 1024 runs in one group, the workgroup 18 us.
__global__ __launch_bounds__(kThreads) void k_combine(const PaStepRecord *__restrict__ steprec, int npoints, int point,
                                                      const int32_t *__restrict__ group_of, int nruns,
                                                      const int32_t *__restrict__ Ns,
                                                      double *__restrict__ out /* [ngroups][PA_COMBINE_FIELDS] */)
{
    __shared__ double sd[16 * 8];
    __shared__ int64_t s_last[kThreads / 64];
    const int g = blockIdx.x, wave = threadIdx.x >> 6;
    double lmax = -INFINITY;
    int64_t last = -1; // the group's last run (its N and beta are the group's), -1: none
    for (int m = threadIdx.x; m < nruns; m += kThreads) {
        if (group_of[m] != g)
            continue;
        const PaStepRecord &r = steprec[(size_t)m * npoints + point];
        if (r.status & PA_ST_FROZEN)
            continue;
        const double l = log((double)r.R) + r.lnZ;
        lmax = l > lmax ? l : lmax;
        last = m;
    }
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) {
        const double o = pa_shfl_xor_f64(lmax, k);
        lmax = o > lmax ? o : lmax;
    }
    last = pa_wave_max_i64(last);
    if ((threadIdx.x & 63) == 0) {
        sd[wave] = lmax;
        s_last[wave] = last;
    }
    __syncthreads();
    for (int k = 0; k < kThreads / 64; ++k) {
        lmax = sd[k] > lmax ? sd[k] : lmax;
        last = s_last[k] > last ? s_last[k] : last;
    }
    const int N = last >= 0 ? Ns[last] : 0;
    const double beta = last >= 0 ? steprec[(size_t)last * npoints + point].beta : 0.0;
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}; // weighted sums of 1, e, e2, |m|, m2, w, c, chi
    double p[5] = {0.0, 0.0, 0.0, 0.0, 0.0};                // plain sums of 1, R, e, c, chi
    for (int m = threadIdx.x; m < nruns; m += kThreads) {
        if (group_of[m] != g)
            continue;
        const PaStepRecord &r = steprec[(size_t)m * npoints + point];
        if (r.status & PA_ST_FROZEN)
            continue;
        const double w = exp(log((double)r.R) + r.lnZ - lmax);
        const double c_m = beta * beta * (double)N * (r.e2 - r.e * r.e); // the run's own c and chi
        const double chi_m = beta * (double)N * (r.m2 - r.abs_m * r.abs_m);
        a[0] = a[0] + w;
        a[1] = a[1] + w * r.e;
        a[2] = a[2] + w * r.e2;
        a[3] = a[3] + w * r.abs_m;
        a[4] = a[4] + w * r.m2;
        a[5] = a[5] + w * w;
        a[6] = a[6] + w * c_m;
        a[7] = a[7] + w * chi_m;
        p[0] = p[0] + 1.0;
        p[1] = p[1] + (double)r.R;
        p[2] = p[2] + r.e;
        p[3] = p[3] + c_m;
        p[4] = p[4] + chi_m;
    }
    pa_block_sum_f64x(a, sd);
    pa_block_sum_f64x(p, sd);
    if (threadIdx.x != 0)
        return;
    const double n = p[0], den = a[0];
    const double e = a[1] / den, e2 = a[2] / den, am = a[3] / den, m2 = a[4] / den;
    double *o = out + (size_t)g * PA_COMBINE_FIELDS;
    const bool any = last >= 0;
    o[0] = any ? lmax + log(den) - log(p[1]) : NAN;
    o[1] = any ? e : 0.0;
    o[2] = any ? e2 : 0.0;
    o[3] = any ? am : 0.0;
    o[4] = any ? m2 : 0.0;
    o[5] = any ? beta * beta * (double)N * (e2 - e * e) : 0.0;
    o[6] = any ? beta * (double)N * (m2 - am * am) : 0.0;
    o[7] = any ? den * den / a[5] : 0.0;
    o[8] = n;
    o[9] = beta;
    o[10] = any ? a[6] / den : 0.0;
    o[11] = any ? a[7] / den : 0.0;
    o[12] = any ? p[2] / n : NAN;
    o[13] = any ? p[3] / n : NAN;
    o[14] = any ? p[4] / n : NAN;
}

// Imported state: thresholds of its beta and the scalars.
__global__ void k_set_beta(const PaRunDesc *__restrict__ runs, double beta, double lnZ, uint32_t step,
                           uint32_t sweeps, uint64_t R)
{
    PaRecord *rec = runs[blockIdx.x].dv.rec;
    if (threadIdx.x == 0) {
        rec->T[0] = pa_threshold(beta, 4);
        rec->T[1] = pa_threshold(beta, 8);
        rec->T[2] = pa_threshold(beta, 12);
        rec->beta = beta;
        rec->lnZ = lnZ;
        rec->step = step;
        rec->sweeps = sweeps;
        rec->Rcur = R;
        rec->sv = 0.0;
        rec->status = 0;
        rec->skip = 0;
        rec->weighted = 0;
        rec->keep = 0;
        rec->gather = 0;
    }
}

// Metropolis thresholds of every run set to those of `beta` (the autotuner
// times sweeps at a temperature of the anneal; the populations are drawn
// again afterwards).
__global__ void k_tune_beta(const PaRunDesc *__restrict__ runs, double beta)
{
    PaRecord *rec = runs[blockIdx.x].dv.rec;
    if (threadIdx.x == 0) {
        rec->T[0] = pa_threshold(beta, 4);
        rec->T[1] = pa_threshold(beta, 8);
        rec->T[2] = pa_threshold(beta, 12);
    }
}

// Generator throughput probe: Metropolis-purpose counters as the sweep forms
// them, three independent chains per thread, outputs folded into one word.
__global__ __launch_bounds__(kThreads) void k_philox_probe(uint32_t *__restrict__ out, int iters)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t acc = 0;
    for (int i = 0; i < iters; ++i) {
        pa_philox_out o[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
            o[q] = pa_philox(1u, 2u, t, (uint32_t)i, 7u, (PA_PURPOSE_METRO << 28) | (uint32_t)q);
#pragma unroll
        for (int q = 0; q < 3; ++q)
            acc ^= o[q].x0 ^ o[q].x1 ^ o[q].x2 ^ o[q].x3;
    }
    out[t] = acc;
}

constexpr int kLdsPerCu = 163840, kWavesPerCu = 16; // gfx950 LDS; four sweep waves per SIMD (<= 128 VGPRs)

// Dynamic LDS of a sweep workgroup with walk `walk`.
size_t sweep_lds(int N, int d, int threads, bool J, int walk)
{
    const size_t sites = walk == kWalkTable ? (size_t)N * 4 : (J ? (((size_t)N + 7) & ~(size_t)7) : 0);
    return (size_t)N * 8 + (size_t)(threads / 64) * kQueue * (3 * 8 + 4) +
           (size_t)(d == 2 ? ttab_words<2>() : ttab_words<3>()) * 4 + sites;
}

// Sweep waves per CU for that LDS.
int sweep_waves(size_t lds, int threads)
{
    const int w = threads / 64, blocks = (int)(kLdsPerCu / lds);
    return (blocks < kWavesPerCu / w ? blocks : kWavesPerCu / w) * w;
}

// Whether the sweeps claim registers for four waves per SIMD (k_sweep4): more
// than 16 waves to a CU only for workgroups of one or two waves, and only
// where LDS holds at least six waves per SIMD.  With 17 to 23 the SIMDs hold
// four, five or six of them, and a column on the fullest is late: ten sweeps
// of 4000 columns of 2D L = 32 (128 lanes, 20 waves) 395 us against 341 with
// 16, of 8000 of 2D L = 24 (64 lanes, 18 waves) 498 against 419, of 5000 of 3D
// L = 8 (64 lanes, 18 waves) 287 against 254.  From 24 on k_sweep is the
// faster: 2D L = 16 (64 lanes, 27) 0 to 3 %, 2D L = 8 (128 lanes, 40) 8 %.
bool sweep_four(size_t lds, int threads)
{
    const int w = threads / 64, blocks = (int)(kLdsPerCu / lds);
    return w > 2 || blocks * w < 24;
}

// The walk a sweep of this shape takes: coordinates that stay from pass to
// pass where the workgroup size allows it, else the site table unless its LDS
// costs resident waves (a wave lost costs more than the index arithmetic).
int sweep_walk(int N, int d, int threads, bool J)
{
    int L = 2;
    while ((d == 2 ? L * L : L * L * L) < N)
        ++L;
    if (threads % (d == 2 ? L : L * L) == 0)
        return d == 3 && (L * L / 2) % 64 == 0 ? kWalkZ : kWalkFix;
    const size_t plain = sweep_lds(N, d, threads, J, kWalkIndex), table = sweep_lds(N, d, threads, J, kWalkTable);
    return table <= (size_t)kLdsPerCu && sweep_waves(table, threads) >= sweep_waves(plain, threads) ? kWalkTable
                                                                                                    : kWalkIndex;
}

// Whether group g's sweeps take in the spins a resampling left in the other
// buffer (their column load gathers them) or a k_gather_spins pass of the
// resampling moves them: the gather in the load keeps the workgroup off the
// VALU for longer, which the other resident workgroups hide only when each
// SIMD holds four sweep waves (measured: 3D L = 10 and the uneven batch gain
// 2-6 %, 3D L = 16 at 256 lanes, three waves per SIMD, loses 1.3 %).  A
// function of the group's workgroup size, which the host keeps fixed between
// a resampling and the sweep after it.
bool sweep_gathers(const PaBatchView &v, int g)
{
    const int threads = v.gthreads[g];
    return sweep_waves(pa_sweep_lds_bytes(v.gN[g], v.gd[g], threads, v.gJ[g] != 0), threads) >= kWavesPerCu;
}

hipError_t sweep_launch(const PaBatchView &v, int g, int theta, int threads, uint32_t t0, hipStream_t st,
                        int gather)
{
    if (v.gncol[g] == 0)
        return hipSuccess;
    const size_t lds = pa_sweep_lds_bytes(v.gN[g], v.gd[g], threads, v.gJ[g] != 0);
    const int walk = sweep_walk(v.gN[g], v.gd[g], threads, v.gJ[g] != 0);
    if (gather && !sweep_gathers(v, g)) // gathered after the resampling
        gather = 0;
    const bool four = sweep_four(lds, threads);
    if (v.gd[g] == 3)
        return pa_sweep3_launch(v.runs, v.gcol[g], v.gncol[g], threads, lds, st, v.gJ[g] != 0, theta, t0, gather, walk,
                                four);
    return v.gJ[g] ? sweep_start<2, true>(v.runs, v.gcol[g], v.gncol[g], threads, lds, st, theta, t0, gather, walk, four)
                   : sweep_start<2, false>(v.runs, v.gcol[g], v.gncol[g], threads, lds, st, theta, t0, gather, walk,
                                           four);
}

} // namespace

// ====================================================================== launchers
size_t pa_sweep_lds_bytes(int N, int d, int threads, bool J)
{
    return sweep_lds(N, d, threads, J, sweep_walk(N, d, threads, J));
}

int pa_sweep_walk(int N, int d, int threads, bool J) { return sweep_walk(N, d, threads, J); }

int pa_sweep_waves_cap(int N, int d, int threads, bool J)
{
    return sweep_four(pa_sweep_lds_bytes(N, d, threads, J), threads) ? kWavesPerCu : 4 * (d == 3 ? 5 : 7);
}

namespace {

// Where (2 d - 1) p, p = 1 - exp(-2 beta), the most active bonds a site of the
// cluster can have towards new ones on average, is below kListBelow, clusters
// are small enough for k_cluster_list: an update at 0.2, 0.6, 1.2, 1.4 and 1.6 takes
// 23, 26, 36, 47, 202 us against 100, 102, 113, 122, 147 at 3D L = 16, R = 2
// 10^4, and 13, 15, 27, 40, 66 against 22, 22, 26, 29, 38 at 2D L = 32, R = 5000.
// Deciding every bond is no more work where the lattice has few sites (2D L =
// 16, R = 5000 14 us by the list, 12 by the flood at 0.2).
constexpr double kListBelow = 1.2;
constexpr int kListSites = 512;
constexpr int kFewColumns = 256; // no more columns than CUs: each has a CU to itself

size_t cluster_lds(int N, int threads, bool J)
{
    return ((size_t)N + (size_t)std::max(N, threads / 2)) * 8 + (J ? (((size_t)N + 7) & ~(size_t)7) : 0);
}

static_assert(PA_CLUSTER_SITES / 16 <= cluster_lanes(2, 16) && PA_CLUSTER_SITES / 4 <= cluster_lanes(2, 4) &&
                  PA_CLUSTER_SITES / 8 <= cluster_lanes(3, 8),
              "a lane for each patch");

template <int D, bool J, int PX, int PY, int PZ, bool REST>
hipError_t cluster_launch(const PaBatchView &v, int g, int nsteps, uint32_t t0)
{
    constexpr int kMost = cluster_lanes(D, PX * PY * PZ);
    const int N = v.gN[g];
    int threads = (N / (PX * PY * PZ) + 63) / 64 * 64;
    if (threads > kMost)
        return hipErrorInvalidValue;
    // more lanes decide a column's bonds sooner where it has a CU to itself: 2D L = 32, R = 5000 at the
    // critical point 69 -> 49 us, 3D L = 16 180 -> 169
    if (v.gncol[g] <= kFewColumns)
        threads = std::max(threads, std::min(kMost, (N + 63) / 64 * 64));
    k_cluster<D, J, PX, PY, PZ, REST>
        <<<v.gncol[g], threads, cluster_lds(N, threads, J), v.stream>>>(v.runs, v.gcol[g], nsteps, t0);
    return hipGetLastError();
}

// Patches of 16 sites (4 x 4 or 4 x 2 x 2) where L allows it and they fill at least a wave, else of
// two sites each way: with fewer than 64 patches the lanes without one idle through the growth.
template <int D, bool J>
hipError_t cluster_launch(const PaBatchView &v, int g, int nsteps, uint32_t t0, double beta)
{
    const int N = v.gN[g];
    int L = 2;
    while ((D == 2 ? L * L : L * L * L) < N)
        ++L;
    if (N > kListSites && (2 * D - 1) * -std::expm1(-2.0 * beta) < kListBelow) {
        const int threads = std::min(v.gncol[g] <= kFewColumns ? 1024 : 512, (N / 4 + 63) / 64 * 64);
        k_cluster_list<D, J>
            <<<v.gncol[g], threads, cluster_lds(N, threads, J), v.stream>>>(v.runs, v.gcol[g], nsteps, t0);
        return cluster_launch<D, J, 2, 2, D == 2 ? 1 : 2, true>(v, g, nsteps, t0);
    }
    if (L % 4 == 0 && N >= 16 * 64)
        return cluster_launch<D, J, 4, D == 2 ? 4 : 2, D == 2 ? 1 : 2, false>(v, g, nsteps, t0);
    return cluster_launch<D, J, 2, 2, D == 2 ? 1 : 2, false>(v, g, nsteps, t0);
}

} // namespace

hipError_t pa_b_cluster(const PaBatchView &v, int nsteps, uint32_t t0, double beta)
{
    for (int g = 0; g < v.ngroups; ++g) {
        if (v.gncol[g] == 0)
            continue;
        hipError_t e;
        if (v.gd[g] == 2)
            e = v.gJ[g] ? cluster_launch<2, true>(v, g, nsteps, t0, beta) : cluster_launch<2, false>(v, g, nsteps, t0, beta);
        else
            e = v.gJ[g] ? cluster_launch<3, true>(v, g, nsteps, t0, beta) : cluster_launch<3, false>(v, g, nsteps, t0, beta);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

size_t pa_cluster_lds_bytes(int N, bool J) { return cluster_lds(N, 1024, J) + (kListed + 1) * sizeof(uint32_t); }

hipError_t pa_query_lds(int *max_lds)
{
    int dev = 0, v = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e == hipSuccess)
        *max_lds = v;
    return e;
}

hipError_t pa_b_sites(const PaBatchView &v)
{
    const int most = *std::max_element(v.gN, v.gN + v.ngroups);
    k_sites<<<dim3(v.nruns, (most + kThreads - 1) / kThreads), kThreads, 0, v.stream>>>(v.runs);
    return hipGetLastError();
}

hipError_t pa_b_init(const PaBatchView &v)
{
    k_init_rec<<<v.nruns, 64, 0, v.stream>>>(v.runs);
    k_hist_prep<<<v.nruns, kThreads, 0, v.stream>>>(v.runs);
    k_init_spins<<<v.ncol, kThreads, 0, v.stream>>>(v.runs, v.col);
    k_init_labels<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
    hipError_t e = hipGetLastError();
    for (int g = 0; g < v.ngroups && e == hipSuccess; ++g)
        e = sweep_launch(v, g, 0, v.gthreads[g], 0u, v.stream, 0);
    return e;
}

hipError_t pa_b_sweep_group(const PaBatchView &v, int g, int theta, int threads)
{
    return sweep_launch(v, g, theta, threads, 0u, v.stream, 0);
}

hipError_t pa_b_gather(const PaBatchView &v)
{
    for (int g = 0; g < v.ngroups; ++g)
        if (v.gncol[g] && sweep_gathers(v, g))
            k_gather_spins<false><<<v.gncol[g], kGatherThreads, 0, v.stream>>>(v.runs, v.gcol[g]);
    return hipGetLastError();
}

hipError_t pa_b_sweep(const PaBatchView &v, int theta, uint32_t t0, int gather)
{
    hipError_t e = hipSuccess;
    if (v.ngroups < 2 || !v.fork) {
        for (int g = 0; g < v.ngroups && e == hipSuccess; ++g)
            e = sweep_launch(v, g, theta, v.gthreads[g], t0, v.stream, gather);
        return e;
    }
    // the groups are independent: each on its own stream, so that one group's
    // last partly filled round of workgroups overlaps the others' work, the
    // longest columns first (a launch that starts last ends last)
    e = hipEventRecord(v.fork, v.stream);
    for (int i = 0; i < v.ngroups && e == hipSuccess; ++i) {
        const int g = v.gorder[i];
        e = hipStreamWaitEvent(v.gstream[g], v.fork, 0);
        if (e == hipSuccess)
            e = sweep_launch(v, g, theta, v.gthreads[g], t0, v.gstream[g], gather);
        if (e == hipSuccess)
            e = hipEventRecord(v.join[g], v.gstream[g]);
    }
    for (int g = 0; g < v.ngroups && e == hipSuccess; ++g)
        e = hipStreamWaitEvent(v.stream, v.join[g], 0);
    return e;
}

// The level histogram of the current populations, from the state the host
// tracks: valid (nothing to do), zero (build it) or stale (clear, then build).
static hipError_t hist_launch(const PaBatchView &v, int state)
{
    if (state == PA_HIST_VALID)
        return hipSuccess;
    if (state == PA_HIST_STALE)
        k_hist_prep<<<v.nruns, kThreads, 0, v.stream>>>(v.runs);
    k_hist<<<v.ncrep, kThreads, (size_t)v.maxH * 4, v.stream>>>(v.runs, v.crep);
    return hipGetLastError();
}


hipError_t pa_b_reweight(const PaBatchView &v, double beta_next, int hist_state)
{
    hipError_t e = hist_launch(v, hist_state);
    if (e != hipSuccess)
        return e;
    if (v.nruns > 256) // more than one run per CU
        k_reweight<256><<<v.nruns, 256, 0, v.stream>>>(v.runs, beta_next);
    else
        k_reweight<1024><<<v.nruns, 1024, 0, v.stream>>>(v.runs, beta_next);
    if (v.weights) { // runs that may hold a weighted population
        k_rw_max<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
        k_rw_sum<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
        k_rw_final<<<v.nruns, kThreads, 0, v.stream>>>(v.runs);
    }
    return hipGetLastError();
}

hipError_t pa_b_rule(const PaBatchView &v, double alpha_star, double dbeta_max, int iterations, int bisect,
                     int hist_state)
{
    hipError_t e = hist_launch(v, hist_state);
    if (e != hipSuccess)
        return e;
    k_rule<<<v.nruns, kRuleWaves * 64, 0, v.stream>>>(v.runs, alpha_star, dbeta_max, iterations, bisect);
    return hipGetLastError();
}

hipError_t pa_b_features(const PaBatchView &v, int hist_state)
{
    hipError_t e = hist_launch(v, hist_state);
    if (e != hipSuccess)
        return e;
    k_features<<<v.nruns, kRuleThreads, 0, v.stream>>>(v.runs);
    return hipGetLastError();
}

// after pa_b_features and the model's proposal (the histogram is current)
hipError_t pa_b_check_candidate(const PaBatchView &v, double alpha_star, double dbeta_max, int iterations,
                                double bracket, int refine)
{
    k_check_candidate<<<v.nruns, kRuleWaves * 64, 0, v.stream>>>(v.runs, alpha_star, dbeta_max, iterations, bracket,
                                                              refine);
    return hipGetLastError();
}

// The spins of the groups whose sweeps do not gather them, after the commit.
static hipError_t gather_rest(const PaBatchView &v)
{
    for (int g = 0; g < v.ngroups; ++g)
        if (v.gncol[g] && !sweep_gathers(v, g))
            k_gather_spins<false><<<v.gncol[g], kGatherThreads, 0, v.stream>>>(v.runs, v.gcol[g]);
    return hipGetLastError();
}

// Whether a step's resampling takes one workgroup per run.
static bool resamples_small(const PaBatchView &v, int scheme, int kq)
{
    return v.nlarge == 0 && kq < 0 && scheme >= 1 && scheme <= 3;
}

// Calls f(lanes, list of the runs (null: all of the batch), n) for the small
// runs: workgroups of 1024 lanes, or of 256 where every run is tiny.  Where tiny
// runs outnumber the CUs and all small runs are more than two to a CU (what
// 1024-lane workgroups fill), the middle and the tiny ones start apart: 1024
// lanes for a tiny run leave most idle but take their place.  2D L = 8, R = 100
// with one run of R = 2000, a step: 4001 runs 327 us in one launch each, 153 in
// two, 1001 runs 94 and 68, 501 runs 59 and 59, 301 runs 55 and 59.
constexpr uint32_t kSplitTiny = 256, kSplitAll = 512;
template <typename F>
static void small_launches(const PaBatchView &v, F f)
{
    const uint32_t *list = v.list + v.nlarge;
    const uint32_t n = v.nruns - v.nlarge, tiny = n - v.nmid;
    if (v.nmid && tiny > kSplitTiny && n > kSplitAll) {
        f(std::integral_constant<int, 1024>{}, list, v.nmid);
        f(std::integral_constant<int, 256>{}, list + v.nmid, tiny);
        return;
    }
    if (v.nlarge == 0)
        list = nullptr; // all runs: no load of the index first
    if (v.nmid)
        f(std::integral_constant<int, 1024>{}, list, n);
    else if (n)
        f(std::integral_constant<int, 256>{}, list, n);
}

bool pa_advances_at_once(const PaBatchView &v, int scheme) { return resamples_small(v, scheme, -1) && !v.weights; }

hipError_t pa_b_advance(const PaBatchView &v, double beta_next, int hist_state, int scheme, int freeze)
{
    hipError_t e = hist_launch(v, hist_state);
    if (e != hipSuccess)
        return e;
    small_launches(v, [&](auto lanes, const uint32_t *list, uint32_t n) {
        constexpr int T = decltype(lanes)::value;
        if (scheme == 1)
            k_advance_small<T, 1><<<n, T, 0, v.stream>>>(v.runs, list, beta_next, freeze);
        else if (scheme == 2)
            k_advance_small<T, 2><<<n, T, 0, v.stream>>>(v.runs, list, beta_next, freeze);
        else
            k_advance_small<T, 3><<<n, T, 0, v.stream>>>(v.runs, list, beta_next, freeze);
    });
    return gather_rest(v);
}

// Launches per scheme (after the reweighting): where every run is small and
// resampled, one workgroup per run for all of it (k_resample_small; a large
// run needs the whole chip, and conditional or multinomial steps have passes
// of their own).  Otherwise: nearest integer and Poisson draw the copy numbers
// and sum them into the ancestor map in one pass; systematic sums the weights
// and writes the ancestor map from each replica's closed-form copy range in
// the same pass; multinomial sums the weights, draws, adds the sampling
// variance and sums the copy numbers.  Then the energies, magnetisations and
// labels move to the ancestors' order (a kept population takes its new
// log-weights in the same launch) and the commit swaps the buffers; the spins follow at once for groups whose
// sweeps do not gather them, else in the next sweep or pa_b_gather.
hipError_t pa_b_resample(const PaBatchView &v, int scheme, int freeze, int kq, bool prepped)
{
    hipError_t e;
    if (!prepped)
        k_resample_prep<<<v.nruns, kThreads, 0, v.stream>>>(v.runs);
    if (resamples_small(v, scheme, kq)) {
        small_launches(v, [&](auto lanes, const uint32_t *list, uint32_t n) {
            constexpr int T = decltype(lanes)::value;
            if (scheme == 1)
                k_resample_small<T, 1><<<n, T, 0, v.stream>>>(v.runs, list, freeze);
            else if (scheme == 2)
                k_resample_small<T, 2><<<n, T, 0, v.stream>>>(v.runs, list, freeze);
            else
                k_resample_small<T, 3><<<n, T, 0, v.stream>>>(v.runs, list, freeze);
        });
        return gather_rest(v);
    }
    switch (scheme) {
    case 2:
        k_counts_scan<2><<<v.ncrep, kThreads, 0, v.stream>>>(v.runs, v.crep, kq);
        break;
    case 1:
        k_counts_scan<1><<<v.ncrep, kThreads, 0, v.stream>>>(v.runs, v.crep, kq);
        break;
    case 3:
    case 0:
        if (scheme == 3) {
            k_weights_scan<PA_SCAN_SYSTEMATIC><<<v.ncrep, kThreads, 0, v.stream>>>(v.runs, v.crep, kq);
        } else {
            k_weights_scan<PA_SCAN_MULTINOMIAL><<<v.ncrep, kThreads, 0, v.stream>>>(v.runs, v.crep, kq);
            k_counts_multinomial<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
            k_sv_partial<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
            k_scan_counts<<<v.ntile, PA_SCAN_THREADS, 0, v.stream>>>(v.runs, v.tile);
        }
        break;
    default:
        return hipErrorInvalidValue;
    }
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    // with no group whose sweeps gather, every spin moves now in the same pass
    // as the energies, magnetisations and labels; otherwise those move now and
    // the spins of the other groups right after the commit
    bool any = false;
    for (int g = 0; g < v.ngroups; ++g)
        any = any || (v.gncol[g] && sweep_gathers(v, g));
    if (any)
        k_gather_meta<<<v.nrep, kThreads, 0, v.stream>>>(v.runs, v.rep);
    else
        k_gather_spins<true><<<v.ncol, kGatherThreads, 0, v.stream>>>(v.runs, v.col);
    k_commit<<<v.nruns, kThreads, 0, v.stream>>>(v.runs, freeze, any ? 0 : 1);
    return any ? gather_rest(v) : hipGetLastError();
}

hipError_t pa_b_observables(const PaBatchView &v, int point, int hist_state)
{
    const int build = hist_state != PA_HIST_VALID;
    PaStepRecord *rows = point >= 0 ? v.steprec : nullptr;
    if (hist_state == PA_HIST_STALE)
        k_hist_prep<<<v.nruns, kThreads, 0, v.stream>>>(v.runs);
    if (v.nlarge) {
        k_obs_rep<<<v.ncrep_large, kThreads, 0, v.stream>>>(v.runs, v.crep, build);
        k_obs_fam<<<v.nfam_large, kThreads, 0, v.stream>>>(v.runs, v.fam);
        k_obs_final<<<v.nlarge, kThreads, 0, v.stream>>>(v.runs, v.list, rows, v.npoints, point);
    }
    small_launches(v, [&](auto lanes, const uint32_t *list, uint32_t n) {
        constexpr int T = decltype(lanes)::value;
        k_obs_small<T><<<n, T, 0, v.stream>>>(v.runs, list, build, rows, v.npoints, point);
    });
    return hipGetLastError();
}

hipError_t pa_b_set_beta(const PaBatchView &v, double beta, double lnZ, uint32_t step, uint32_t sweeps,
                         uint64_t R)
{
    k_set_beta<<<v.nruns, 64, 0, v.stream>>>(v.runs, beta, lnZ, step, sweeps, R);
    return hipGetLastError();
}

hipError_t pa_b_tune_beta(const PaBatchView &v, double beta)
{
    k_tune_beta<<<v.nruns, 64, 0, v.stream>>>(v.runs, beta);
    return hipGetLastError();
}

hipError_t pa_launch_combine(const PaBatchView &v, int point, const int32_t *group_of, int ngroups,
                             const int32_t *Ns, double *out)
{
    k_combine<<<ngroups, kThreads, 0, v.stream>>>(v.steprec, v.npoints, point, group_of, (int)v.nruns, Ns, out);
    return hipGetLastError();
}

hipError_t pa_launch_philox_probe(uint32_t *out, int64_t nthreads, int iters, hipStream_t st)
{
    k_philox_probe<<<(unsigned)(nthreads / kThreads), kThreads, 0, st>>>(out, iters);
    return hipGetLastError();
}

hipError_t pa_launch_overlap(const PaRunDesc *a, const PaRunDesc *b, int N, uint32_t ncols_a,
                             unsigned long long *hist, hipStream_t st)
{
    k_fill_u32<<<grid_for((int64_t)(N + 1) * 2), kThreads, 0, st>>>(reinterpret_cast<uint32_t *>(hist),
                                                                     (int64_t)(N + 1) * 2, 0u);
    k_overlap<<<ncols_a, kThreads, 0, st>>>(a, b, hist);
    return hipGetLastError();
}

// ------------------------------------------------------------------ allocation-free overlap
// The overlap histogram of pa_overlap_noalloc lives in this file-scope device
// array instead of a run's workspace: PA_NOALLOC_HIST_MAX counters (the
// largest lattice's N + 1), 128 KiB per device, held until the process ends.
// Every call on a device shares that device's copy.  In host code `scratch`
// names a host-side stand-in, never the device memory: the device address
// comes from hipGetSymbolAddress, taken once per device with that device
// current, and only that address is passed to kernels.
static __device__ __align__(256) unsigned long long scratch[PA_NOALLOC_HIST_MAX];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
} // namespace

hipError_t pa_noalloc_scratch(int device, unsigned long long **out)
{
    if (device < 0 || device >= kMaxDevices)
        return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int prev = 0;
        hipError_t e = hipGetDevice(&prev);
        if (e != hipSuccess)
            return e;
        if (prev != device && (e = hipSetDevice(device)) != hipSuccess)
            return e;
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (prev != device) {
            const hipError_t e2 = hipSetDevice(prev);
            if (e == hipSuccess)
                e = e2;
        }
        if (e != hipSuccess)
            return e;
        g_scratch_ptr[device] = ptr;
    }
    *out = static_cast<unsigned long long *>(g_scratch_ptr[device]);
    return hipSuccess;
}
