// No-Time-Counter pair selection (section "Cell partition and collision-pair
// selection").  Candidates are generated for all cells at once, one lane per
// candidate, so the work is balanced however uneven the cell populations are:
//   count M_k per cell, with each tile of cells' sum -> candidate offsets
//   (a workgroup adds the sums of the tiles before its own), the cell of each
//   64-candidate round's first candidate and the overflow decision -> decide
//   pass: each wave takes a chunk of candidates, walks its cells forward,
//   draws and decides the candidates and stages the accepted pairs compactly
//   in the chunk's own slots, with each cell's offset inside the chunk -> one
//   workgroup's scan of the chunk counts -> copy pass: the staged pairs of
//   every chunk to their dense, cell-major place -> per cell offsets and
//   counts.
// Six launches; with general scans the stage took twelve, at some 4 us each.
// The decision arithmetic (g, the candidate count) uses explicitly rounded
// FP64 operations so it is the same on every launch shape.
#include <math.h>

#include "common.hpp"

namespace dsmc {

struct XsLaw {
    double C, e;  // sigma(g) g = C g^e
};

static int xs_law(const dsmc_xs& xs, XsLaw* out)
{
    constexpr double KB = 1.380649e-23;
    constexpr double PI = 3.14159265358979323846;
    if (xs.kind == DSMC_XS_VHS) {
        if (!(xs.m > 0) || !(xs.d_ref > 0) || !(xs.T_ref > 0) || !(xs.omega > 0.5) ||
            !(xs.omega < 1.0))
            return arg_error("dsmc_xs: bad VHS parameters");
        const double mr = xs.m / 2.0;
        out->C = PI * xs.d_ref * xs.d_ref * pow(2.0 * KB * xs.T_ref / mr, xs.omega - 0.5) /
                 tgamma(2.5 - xs.omega);
        out->e = 2.0 - 2.0 * xs.omega;
        return DSMC_OK;
    }
    if (xs.kind == DSMC_XS_CONST) {
        if (!(xs.sigma > 0)) return arg_error("dsmc_xs: sigma must be > 0");
        out->C = xs.sigma;
        out->e = 1.0;
        return DSMC_OK;
    }
    return arg_error("dsmc_xs: kind %d", xs.kind);
}

__device__ __forceinline__ int32_t cand_count(int32_t N, double lam, XsLaw law, double cmax,
                                              const dsmc_rng& rng, int32_t k)
{
    if (N < 2) return 0;
    const double ghat = 2.0 * cmax;
    const double sgmax = law.C * pow(ghat, law.e);
    const U4 r = draw(rng, 0u, (uint32_t)k, SLOT_COUNT);
    const double U = unif53(r.a, r.b);
    double x = __dmul_rn(0.5, (double)N);
    x = __dmul_rn(x, (double)(N - 1));
    x = __dmul_rn(x, lam);
    x = __dmul_rn(x, sgmax);
    x = __dadd_rn(x, U);
    if (!(x >= 0.0) || !(x < 2147483647.0)) return 0;
    return (int32_t)floor(x);
}

// Candidates (NTC) or trials (SBT: N - 1) of every cell, and their sum over
// each tile of `tile` cells (one workgroup per tile).
enum { SEL_NTC = 0, SEL_SBT = 1 };

constexpr int CNT_THREADS = 256;
constexpr int CNT_TILES = 4096;   // most tiles: the offsets pass adds this many sums

__device__ __forceinline__ int64_t block_sum_i64(int64_t x)
{
    __shared__ int64_t ws_[CNT_THREADS / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) ws_[threadIdx.x >> 6] = x;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int w = 0; w < CNT_THREADS / 64; ++w) t += ws_[w];
    return t;
}

template <int SEL>
__global__ void __launch_bounds__(CNT_THREADS)
k_cand_count(const int32_t* __restrict__ cell_start, int32_t n_cells, int32_t tile,
             const double* __restrict__ lambda, const double* __restrict__ mom, XsLaw law,
             dsmc_rng rng, int32_t* __restrict__ cnt, int64_t* __restrict__ tile_sum)
{
    const int64_t k0 = (int64_t)blockIdx.x * tile;
    const int64_t k1 = k0 + tile < n_cells ? k0 + tile : n_cells;
    int64_t sum = 0;
    for (int64_t k = k0 + threadIdx.x; k < k1; k += CNT_THREADS) {
        const int32_t N = cell_start[k + 1] - cell_start[k];
        int32_t c;
        if (SEL == SEL_NTC)
            c = cand_count(N, lambda[k], law, mom[6 * (size_t)k + 4], rng, (int32_t)k);
        else
            c = N >= 2 ? N - 1 : 0;
        cnt[k] = c;
        sum += c;
    }
    sum = block_sum_i64(sum);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = sum;
}

constexpr int CAND_GROUP = 4;
constexpr int CAND_WIN = 4;      // scalar cell window of a group (see k_cand_decide)

// Rounds of 64 candidates per chunk (one chunk per wave at a time): few, so a
// small selection spreads over the chip's waves, until there are candidates
// enough to give every wave a long chunk; then 16, whose staged runs are
// longer and whose counts are fewer (53 million candidates: decide 0.46 ms
// against 0.63 ms with 4, copy 0.07 against 0.14 ms; 17 000 candidates:
// decide 13 us with 4 against 32 us with 16).  The stage with 4 and with 16
// around the line: 3.1 million candidates 77 and 84 us, 4.7 million 100 and
// 106, 6.2 million 126 and 123, 9.3 million 175 and 169, 74 million 1 287 and
// 1 245.
constexpr int CHUNK_MIN = 64 * CAND_GROUP;
constexpr int64_t CHUNK_LONG_FROM = (int64_t)1 << 23;
__device__ __forceinline__ int cand_rounds(int64_t total)
{
    return total < CHUNK_LONG_FROM ? CAND_GROUP : 4 * CAND_GROUP;
}

// What the passes after the count share.
struct SelTotals {
    int64_t n_use;      // candidates processed (0 on overflow)
    int64_t n_chunks;
    int32_t ok;
    int32_t chunk;      // candidates per chunk
};

// Offsets of a tile's cells: the sums of the tiles before it, then a running
// scan over its cells; the cell owning the first candidate of each
// 64-candidate round (written by that cell's thread); the overflow decision.
__global__ void __launch_bounds__(CNT_THREADS)
k_cand_offsets(int32_t n_cells, int32_t tile, const int32_t* __restrict__ cnt,
               const int64_t* __restrict__ tile_sum, int64_t cap, int32_t* __restrict__ cand_off,
               int32_t* __restrict__ round_cell, SelTotals* __restrict__ tot, dsmc_status* st)
{
    int64_t before = 0, all = 0;
    for (int t = threadIdx.x; t < (int)gridDim.x; t += CNT_THREADS) {
        const int64_t x = tile_sum[t];
        all += x;
        before += t < (int)blockIdx.x ? x : 0;
    }
    before = block_sum_i64(before);
    all = block_sum_i64(all);
    const bool fits = all <= cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        tot->n_use = fits ? all : 0;
        const int chunk = 64 * cand_rounds(all);
        tot->n_chunks = fits ? (all + chunk - 1) / chunk : 0;
        tot->ok = fits ? 1 : 0;
        tot->chunk = chunk;
        if (st) {
            st->n_cand = all;
            if (!fits) atomicOr(&st->flags, (uint32_t)DSMC_ST_PAIR_OVERFLOW);
        }
    }
    if (!fits) return;
    __shared__ int32_t wsum[CNT_THREADS / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t k0 = (int64_t)blockIdx.x * tile;
    const int64_t k1 = k0 + tile < n_cells ? k0 + tile : n_cells;
    int32_t run = (int32_t)before;
    for (int64_t b = k0; b < k1; b += CNT_THREADS) {
        const int64_t k = b + threadIdx.x;
        const int32_t x = k < k1 ? cnt[k] : 0;
        int32_t inc = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        __syncthreads();
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        int32_t pre = run;
#pragma unroll
        for (int q = 0; q < CNT_THREADS / 64; ++q) {
            if (q < w) pre += wsum[q];
            run += wsum[q];
        }
        if (k < k1) {
            const int64_t a = pre + inc - x, e = a + x;
            cand_off[k] = (int32_t)a;
            for (int64_t r = (a + 63) / 64; r * 64 < e; ++r) round_cell[r] = (int32_t)k;
        }
    }
}

// Candidate t of cell k: indices (Lemire multiply-shift, j != i) and the
// acceptance uniform.
struct CandDraw {
    int32_t i, j;   // sorted slots
    double U;
};

__device__ __forceinline__ CandDraw cand_draw(int32_t s0, int32_t N, int32_t k, int32_t t,
                                              const dsmc_rng& rng)
{
    const U4 r = draw(rng, (uint32_t)t, (uint32_t)k, SLOT_CAND);
    int32_t i = (int32_t)(((uint64_t)r.a * (uint64_t)N) >> 32);
    int32_t j = (int32_t)(((uint64_t)r.b * (uint64_t)(N - 1)) >> 32);
    if (j >= i) j += 1;
    return CandDraw{s0 + i, s0 + j, unif53(r.c, r.d)};
}

// Acceptance test U < (g / g_hat)^e on the pre-step velocities.
template <typename T>
__device__ __forceinline__ bool cand_accept(const CandDraw& d, const V3<const T>& v, double ghat,
                                            double e)
{
    const double dx = (double)v.x[d.i] - (double)v.x[d.j];
    const double dy = (double)v.y[d.i] - (double)v.y[d.j];
    const double dz = (double)v.z[d.i] - (double)v.z[d.j];
    const double g2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)),
                                __dmul_rn(dz, dz));
    const double g = sqrt(g2);
    const double ratio = g / ghat;
    const double p = (e == 1.0) ? ratio : pow(ratio, e);
    return d.U < p;
}

// Simplified Bernoulli Trials (Stefanov 2011): trial t of cell k is the
// particle in slot t; its partner is drawn uniformly among the m = N-1-t
// later slots and the pair collides with probability P = m lambda_k sigma(g) g
// (values above 1 act as 1 and are counted).
__device__ __forceinline__ CandDraw sbt_draw(int32_t s0, int32_t N, int32_t k, int32_t t,
                                             const dsmc_rng& rng, int32_t& m)
{
    m = N - 1 - t;
    const U4 r = draw(rng, (uint32_t)t, (uint32_t)k, SLOT_SBT);
    const int32_t j = t + 1 + (int32_t)(((uint64_t)r.a * (uint64_t)m) >> 32);
    return CandDraw{s0 + t, s0 + j, unif53(r.c, r.d)};
}

template <typename T>
__device__ __forceinline__ bool sbt_accept(const CandDraw& d, int32_t m, const V3<const T>& v,
                                           double lam, double C, double e, bool& clamped)
{
    const double dx = (double)v.x[d.i] - (double)v.x[d.j];
    const double dy = (double)v.y[d.i] - (double)v.y[d.j];
    const double dz = (double)v.z[d.i] - (double)v.z[d.j];
    const double g2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)),
                                __dmul_rn(dz, dz));
    const double g = sqrt(g2);
    const double sg = __dmul_rn(C, (e == 1.0) ? g : pow(g, e));
    const double P = __dmul_rn(__dmul_rn((double)m, lam), sg);
    clamped = P > 1.0;
    return d.U < P;
}

// Decide every candidate of a chunk; accepted pairs go to the chunk's slots
// [ch * chunk, ...) of the staging arrays in candidate order; loc[k] = number
// of accepted pairs of the chunk before cell k's first candidate (for every
// cell whose candidates start inside the chunk; empty cells take the value of
// the next candidate).
template <typename T, int SEL>
__global__ void __launch_bounds__(256)
k_cand_decide(const int32_t* __restrict__ cell_start, int32_t n_cells,
              const int32_t* __restrict__ cand_off, const SelTotals* __restrict__ tot,
              const int32_t* __restrict__ round_cell, const double* __restrict__ mom,
              const double* __restrict__ lambda, double C, double e, dsmc_rng rng,
              V3<const T> v, int32_t* __restrict__ chunk_cnt, int32_t* __restrict__ chunk_clamped,
              int32_t* __restrict__ si, int32_t* __restrict__ sj, int32_t* __restrict__ sc,
              int32_t* __restrict__ loc)
{
    const int64_t total = tot->n_use;
    const int64_t nch = tot->n_chunks;
    const int chunk = tot->chunk, rounds = chunk / 64;
    const int lane = threadIdx.x & 63;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t ch = wave; ch < nch; ch += nwaves) {
        const int64_t cbase = ch * chunk;
        int32_t acc = 0, clamped_n = 0;
        // CAND_GROUP rounds at a time.  Cells are looked up in two ways:
        //  - when the group's candidates lie in the CAND_WIN cells from the
        //    cell of its first candidate (cells of many candidates), those
        //    cells are read once by scalar loads and a lane's cell is the
        //    number of their starts at or below its candidate;
        //  - otherwise each round of 64 candidates reads a window of 64 cells
        //    from the cell of its first candidate (one coalesced load per
        //    lane and field), a lane finds its cell by a binary search over
        //    the window's candidate offsets with lane shuffles, and a round
        //    that crosses more than 63 cell starts (runs of cells without
        //    candidates) walks on from the window's last cell.
        for (int r0 = 0; r0 < rounds; r0 += CAND_GROUP) {
            const int64_t gfirst = cbase + r0 * 64;
            if (gfirst >= total) break;
            int32_t kk[CAND_GROUP], s0u[CAND_GROUP], nu[CAND_GROUP], au[CAND_GROUP];
            double gu[CAND_GROUP];
            bool val[CAND_GROUP];
            int64_t cc[CAND_GROUP];
            const int32_t kw = __builtin_amdgcn_readfirstlane(round_cell[gfirst >> 6]);
            const int64_t glast = (gfirst + CAND_GROUP * 64 < total ? gfirst + CAND_GROUP * 64
                                                                      : total) - 1;
            int32_t wb[CAND_WIN];
#pragma unroll
            for (int q = 0; q < CAND_WIN; ++q)
                wb[q] = kw + 1 + q < n_cells ? cand_off[kw + 1 + q] : INT32_MAX;
            if (glast < (int64_t)wb[CAND_WIN - 1]) {
                int32_t ws0[CAND_WIN + 1];
                double wg[CAND_WIN];
#pragma unroll
                for (int q = 0; q <= CAND_WIN; ++q)
                    ws0[q] = cell_start[kw + q <= n_cells ? kw + q : n_cells];
#pragma unroll
                for (int q = 0; q < CAND_WIN; ++q) {
                    const int32_t kq = kw + q < n_cells ? kw + q : n_cells - 1;
                    wg[q] = SEL == SEL_NTC ? 2.0 * mom[6 * (size_t)kq + 4] : lambda[kq];
                }
                const int32_t wa0 = cand_off[kw];
#pragma unroll
                for (int u = 0; u < CAND_GROUP; ++u) {
                    cc[u] = gfirst + u * 64 + lane;
                    val[u] = cc[u] < total;
                    int32_t w = 0;
#pragma unroll
                    for (int q = 0; q < CAND_WIN - 1; ++q) w += cc[u] >= wb[q] ? 1 : 0;
                    int32_t s0 = ws0[0], s1 = ws0[1], a = wa0;
                    double g = wg[0];
#pragma unroll
                    for (int q = 1; q < CAND_WIN; ++q)
                        if (w == q) { s0 = ws0[q]; s1 = ws0[q + 1]; g = wg[q]; a = wb[q - 1]; }
                    kk[u] = kw + w;
                    au[u] = a;
                    s0u[u] = s0;
                    nu[u] = s1 - s0;
                    gu[u] = g;
                }
            } else {
#pragma unroll
                for (int u = 0; u < CAND_GROUP; ++u) {
                    cc[u] = gfirst + u * 64 + lane;
                    val[u] = cc[u] < total;
                    const int64_t rfirst = gfirst + u * 64;
                    const int32_t kr =
                        rfirst < total ? __builtin_amdgcn_readfirstlane(round_cell[rfirst >> 6])
                                       : 0;
                    const int32_t kl = kr + lane;
                    const int32_t A = kl < n_cells ? cand_off[kl] : INT32_MAX;
                    const int32_t An = kl + 1 < n_cells ? cand_off[kl + 1] : INT32_MAX;
                    const int32_t S = cell_start[kl < n_cells ? kl : n_cells];
                    const int32_t Sn = cell_start[kl < n_cells ? kl + 1 : n_cells];
                    const int32_t kq = kl < n_cells ? kl : n_cells - 1;
                    const double G = SEL == SEL_NTC ? 2.0 * mom[6 * (size_t)kq + 4] : lambda[kq];
                    // largest window index l with A[l] <= cc (A[0] <= cc holds)
                    int32_t l = 0;
#pragma unroll
                    for (int stp = 32; stp > 0; stp >>= 1) {
                        const int32_t c = l + stp;
                        const int32_t Ac = __shfl(A, c < 64 ? c : 63, 64);
                        if (c < 64 && (int64_t)Ac <= cc[u]) l = c;
                    }
                    int32_t k = kr + l;
                    int32_t a = __shfl(A, l, 64);
                    int32_t s0 = __shfl(S, l, 64), s1 = __shfl(Sn, l, 64);
                    double g = __shfl(G, l, 64);
                    const int32_t an = __shfl(An, l, 64);
                    if (val[u] && (int64_t)an <= cc[u]) {
                        // beyond the window
                        while (k + 1 < n_cells && cand_off[k + 1] <= cc[u]) ++k;
                        a = cand_off[k];
                        s0 = cell_start[k];
                        s1 = cell_start[k + 1];
                        g = SEL == SEL_NTC ? 2.0 * mom[6 * (size_t)k + 4] : lambda[k];
                    }
                    kk[u] = k;
                    au[u] = a;
                    s0u[u] = s0;
                    nu[u] = s1 - s0;
                    gu[u] = g;
                }
            }
            CandDraw dr[CAND_GROUP];
            int32_t mm[CAND_GROUP];
#pragma unroll
            for (int u = 0; u < CAND_GROUP; ++u) {
                const int32_t t = (int32_t)(cc[u] - au[u]);
                mm[u] = 0;
                if (!val[u]) dr[u] = CandDraw{0, 0, 1.0};
                else if (SEL == SEL_NTC) dr[u] = cand_draw(s0u[u], nu[u], kk[u], t, rng);
                else dr[u] = sbt_draw(s0u[u], nu[u], kk[u], t, rng, mm[u]);
            }
            bool take[CAND_GROUP];
#pragma unroll
            for (int u = 0; u < CAND_GROUP; ++u) {
                if (SEL == SEL_NTC) {
                    take[u] = val[u] && cand_accept<T>(dr[u], v, gu[u], e);
                } else {
                    bool cl = false;
                    take[u] = val[u] && sbt_accept<T>(dr[u], mm[u], v, gu[u], C, e, cl);
                    clamped_n += (int32_t)__popcll(__ballot(val[u] && cl));
                }
            }
#pragma unroll
            for (int u = 0; u < CAND_GROUP; ++u) {
                const uint64_t ab = __ballot(take[u]);
                const int32_t p = acc + (int32_t)__popcll(ab & lt);
                if (take[u]) {
                    si[cbase + p] = dr[u].i;
                    sj[cbase + p] = dr[u].j;
                    sc[cbase + p] = kk[u];
                }
                if (val[u] && cc[u] == au[u]) {
                    loc[kk[u]] = p;
                    for (int32_t q = kk[u] - 1; q >= 0 && cand_off[q] == cc[u]; --q) loc[q] = p;
                }
                acc += (int32_t)__popcll(ab);
            }
        }
        if (lane == 0) {
            chunk_cnt[ch] = acc;
            if (SEL == SEL_SBT) chunk_clamped[ch] = clamped_n;
        }
    }
}

// Exclusive scan of the chunk counts by one workgroup, 16 384 counts a step
// (chunk_off[n_chunks] = all pairs), and the sum of the trials whose
// probability was clamped.  52 000 counts take 15 us.  (Sums added
// atomically by the decide pass instead, one address per 64 chunks, cost it
// more than this launch; its waves' atomic counts of clamped trials on the one
// status word took 40 of its 55 us for a million trials.)
template <int SEL>
__global__ void __launch_bounds__(SCAN1_THREADS)
k_chunk_scan(const SelTotals* __restrict__ tot, const int32_t* __restrict__ cnt,
             const int32_t* __restrict__ clamped, int32_t* __restrict__ off, dsmc_status* st)
{
    __shared__ int32_t csum[SCAN1_THREADS / 64];
    const int64_t n = tot->n_chunks;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t nclamp = 0;
    scan_one<true>(cnt, off, n, [&](int64_t b) {
        if (SEL == SEL_SBT)
            for (int64_t i = b + threadIdx.x; i < n && i < b + SCAN1_STEP; i += SCAN1_THREADS)
                nclamp += clamped[i];
    });
    if (SEL == SEL_SBT && st) {
        nclamp = wave_sum_i(nclamp);
        if (lane == 0) csum[w] = nclamp;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t c = 0;
            for (int u = 0; u < SCAN1_THREADS / 64; ++u) c += csum[u];
            if (c > 0) {
                atomicAdd(&st->prob_clamped, c);
                atomicOr(&st->flags, (uint32_t)DSMC_ST_PROB_CLAMP);
            }
        }
    }
}

// Staged pairs of each chunk to their dense place (one wave per chunk).
__global__ void __launch_bounds__(256)
k_stage_copy(const SelTotals* __restrict__ tot, const int32_t* __restrict__ chunk_cnt,
             const int32_t* __restrict__ chunk_off, const int32_t* __restrict__ si,
             const int32_t* __restrict__ sj, const int32_t* __restrict__ sc,
             int32_t* __restrict__ pi, int32_t* __restrict__ pj, int32_t* __restrict__ pc)
{
    const int64_t nch = tot->n_chunks;
    const int chunk = tot->chunk;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t ch = wave; ch < nch; ch += nwaves) {
        const int32_t n = chunk_cnt[ch], o = chunk_off[ch];
        const int64_t src = ch * chunk;
        for (int32_t q = lane; q < n; q += 64) {
            pi[o + q] = si[src + q];
            pj[o + q] = sj[src + q];
            pc[o + q] = sc[src + q];
        }
    }
}

// Pair offsets and counts per cell; cells whose candidates would start at or
// after the last candidate (none left) get the total as offset.
__global__ void __launch_bounds__(256)
k_pair_counts(int32_t n_cells, const int32_t* __restrict__ cand_off,
              const SelTotals* __restrict__ tot, const int32_t* __restrict__ chunk_off,
              const int32_t* __restrict__ loc, int32_t* __restrict__ off,
              int32_t* __restrict__ cnt, dsmc_status* st)
{
    const bool fits = tot->ok != 0;
    const int64_t total = tot->n_use;
    const int32_t npairs = fits ? chunk_off[tot->n_chunks] : 0;
    const int chunk = tot->chunk;
    for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n_cells;
         k += gridDim.x * blockDim.x) {
        if (!fits) {
            off[k] = 0;
            cnt[k] = 0;
            continue;
        }
        const int64_t ca = cand_off[k];
        const int32_t a = ca >= total ? npairs : chunk_off[ca / chunk] + loc[k];
        int32_t b = npairs;
        if (k + 1 < n_cells) {
            const int64_t cb = cand_off[k + 1];
            b = cb >= total ? npairs : chunk_off[cb / chunk] + loc[k + 1];
        }
        off[k] = a;
        cnt[k] = b - a;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && st) st->n_pairs = npairs;
}

struct SelectWs {
    int32_t* cand_cnt;    // [n_cells]
    int32_t* cand_off;    // [n_cells]
    int32_t* loc;         // [n_cells]
    int64_t* tile_sum;    // [CNT_TILES]
    SelTotals* tot;
    int32_t* round_cell;  // [max chunks * CAND_GROUP]
    int32_t* chunk_cnt;   // [max chunks]
    int32_t* chunk_clamped; // [max chunks]
    int32_t* chunk_off;   // [max chunks + 1]
    int32_t* si;          // staging [max chunks * CHUNK_MIN]
    int32_t* sj;
    int32_t* sc;
    size_t bytes;
};

static int64_t max_chunks(int64_t cap) { return (cap + CHUNK_MIN - 1) / CHUNK_MIN + 1; }

static SelectWs select_ws_layout(void* base, int32_t n_cells, int64_t cap)
{
    SelectWs w{};
    // (the queried size has 256 spare bytes for the alignment of the base)
    uint8_t* p = reinterpret_cast<uint8_t*>(align_up(reinterpret_cast<uintptr_t>(base)));
    size_t o = 0;
    auto take = [&](size_t b) { uint8_t* r = p ? p + o : nullptr; o += align_up(b); return r; };
    const int64_t mc = max_chunks(cap);
    w.cand_cnt = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)n_cells));
    w.cand_off = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)n_cells));
    w.loc = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)n_cells));
    w.tile_sum = reinterpret_cast<int64_t*>(take(sizeof(int64_t) * CNT_TILES));
    w.tot = reinterpret_cast<SelTotals*>(take(sizeof(SelTotals)));
    w.round_cell = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)mc * CAND_GROUP));
    w.chunk_cnt = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)mc));
    w.chunk_clamped = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)mc));
    w.chunk_off = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * ((size_t)mc + 1)));
    const size_t stage = sizeof(int32_t) * (size_t)mc * CHUNK_MIN;
    w.si = reinterpret_cast<int32_t*>(take(stage));
    w.sj = reinterpret_cast<int32_t*>(take(stage));
    w.sc = reinterpret_cast<int32_t*>(take(stage));
    w.bytes = o;
    return w;
}

template <typename T, int SEL>
static int select_impl(int32_t n_cells, const int32_t* cell_start, dsmc_vec3 v, XsLaw law,
                       const double* lambda, const double* mom, dsmc_rng rng,
                       dsmc_pairs pairs, void* ws, dsmc_status* st, hipStream_t s)
{
    SelectWs w = select_ws_layout(ws, n_cells, pairs.cap);
    const int pb = persistent_blocks(256);
    int cb = (n_cells + 255) / 256;
    cb = cb < 1 ? 1 : (cb > pb ? pb : cb);
    // tiles of one workgroup-width of cells, larger only beyond CNT_TILES of them
    const int64_t widths = ((int64_t)n_cells + CNT_THREADS - 1) / CNT_THREADS;
    const int32_t tile = (int32_t)((widths + CNT_TILES - 1) / CNT_TILES * CNT_THREADS);
    const int tiles = (int)(((int64_t)n_cells + tile - 1) / tile);
    k_cand_count<SEL><<<tiles, CNT_THREADS, 0, s>>>(cell_start, n_cells, tile, lambda, mom, law,
                                                    rng, w.cand_cnt, w.tile_sum);
    DSMC_LAUNCH_CHECK("select:count");
    k_cand_offsets<<<tiles, CNT_THREADS, 0, s>>>(n_cells, tile, w.cand_cnt, w.tile_sum, pairs.cap,
                                                 w.cand_off, w.round_cell, w.tot, st);
    DSMC_LAUNCH_CHECK("select:offsets");
    // no more workgroups than chunks fit the capacity
    const int64_t ch_max = max_chunks(pairs.cap);
    const int db = (int)((ch_max + 3) / 4 < pb ? (ch_max + 3) / 4 : pb);
    k_cand_decide<T, SEL><<<db, 256, 0, s>>>(cell_start, n_cells, w.cand_off, w.tot, w.round_cell,
                                             mom, lambda, law.C, law.e, rng, v3<const T>(v),
                                             w.chunk_cnt, w.chunk_clamped, w.si, w.sj, w.sc, w.loc);
    DSMC_LAUNCH_CHECK("select:decide");
    k_chunk_scan<SEL><<<1, SCAN1_THREADS, 0, s>>>(w.tot, w.chunk_cnt, w.chunk_clamped, w.chunk_off,
                                                  st);
    DSMC_LAUNCH_CHECK("select:scan");
    k_stage_copy<<<db, 256, 0, s>>>(w.tot, w.chunk_cnt, w.chunk_off, w.si, w.sj, w.sc, pairs.i,
                                    pairs.j, pairs.cell);
    DSMC_LAUNCH_CHECK("select:copy");
    k_pair_counts<<<cb, 256, 0, s>>>(n_cells, w.cand_off, w.tot, w.chunk_off, w.loc, pairs.off,
                                     pairs.cnt, st);
    DSMC_LAUNCH_CHECK("select:counts");
    return DSMC_OK;
}

}  // namespace dsmc

using namespace dsmc;

extern "C" size_t dsmc_select_pairs_ntc_ws(int32_t n_cells, int64_t cap)
{
    if (n_cells < 1 || cap < 0) return 0;
    return select_ws_layout(nullptr, n_cells, cap).bytes + 256;
}

extern "C" int dsmc_select_pairs_ntc(int32_t n_cells, const int32_t* cell_start, int32_t dtype,
                                     dsmc_vec3 v, dsmc_xs xs, const double* lambda,
                                     const double* mom, dsmc_rng rng, dsmc_pairs pairs,
                                     void* ws, size_t ws_bytes, dsmc_status* st,
                                     dsmc_stream_t stream)
{
    if (n_cells < 1) return arg_error("dsmc_select_pairs_ntc: n_cells=%d", n_cells);
    if (!cell_start || !lambda || !mom || !ws || !v.x || !v.y || !v.z || !pairs.off ||
        !pairs.cnt || (pairs.cap > 0 && (!pairs.i || !pairs.j || !pairs.cell)))
        return arg_error("dsmc_select_pairs_ntc: null pointer");
    if (pairs.cap < 0 || pairs.cap >= (int64_t)INT32_MAX - 2)
        return arg_error("dsmc_select_pairs_ntc: cap %lld out of range", (long long)pairs.cap);
    if (ws_bytes < dsmc_select_pairs_ntc_ws(n_cells, pairs.cap))
        return arg_error("dsmc_select_pairs_ntc: workspace %zu < %zu", ws_bytes,
                         dsmc_select_pairs_ntc_ws(n_cells, pairs.cap));
    XsLaw law;
    int rc = xs_law(xs, &law);
    if (rc) return rc;
    hipStream_t s = as_stream(stream);
    if (dtype == DSMC_F64)
        return select_impl<double, SEL_NTC>(n_cells, cell_start, v, law, lambda, mom, rng, pairs,
                                            ws, st, s);
    if (dtype == DSMC_F32)
        return select_impl<float, SEL_NTC>(n_cells, cell_start, v, law, lambda, mom, rng, pairs,
                                           ws, st, s);
    return arg_error("dsmc_select_pairs_ntc: dtype %d", dtype);
}

extern "C" size_t dsmc_select_pairs_sbt_ws(int32_t n_cells, int64_t cap)
{
    return dsmc_select_pairs_ntc_ws(n_cells, cap);
}

extern "C" int dsmc_select_pairs_sbt(int32_t n_cells, const int32_t* cell_start, int32_t dtype,
                                     dsmc_vec3 v, dsmc_xs xs, const double* lambda,
                                     dsmc_rng rng, dsmc_pairs pairs, void* ws, size_t ws_bytes,
                                     dsmc_status* st, dsmc_stream_t stream)
{
    if (n_cells < 1) return arg_error("dsmc_select_pairs_sbt: n_cells=%d", n_cells);
    if (!cell_start || !lambda || !ws || !v.x || !v.y || !v.z || !pairs.off || !pairs.cnt ||
        (pairs.cap > 0 && (!pairs.i || !pairs.j || !pairs.cell)))
        return arg_error("dsmc_select_pairs_sbt: null pointer");
    if (pairs.cap < 0 || pairs.cap >= (int64_t)INT32_MAX - 2)
        return arg_error("dsmc_select_pairs_sbt: cap %lld out of range", (long long)pairs.cap);
    if (ws_bytes < dsmc_select_pairs_sbt_ws(n_cells, pairs.cap))
        return arg_error("dsmc_select_pairs_sbt: workspace %zu < %zu", ws_bytes,
                         dsmc_select_pairs_sbt_ws(n_cells, pairs.cap));
    XsLaw law;
    int rc = xs_law(xs, &law);
    if (rc) return rc;
    hipStream_t s = as_stream(stream);
    if (dtype == DSMC_F64)
        return select_impl<double, SEL_SBT>(n_cells, cell_start, v, law, lambda, nullptr, rng,
                                            pairs, ws, st, s);
    if (dtype == DSMC_F32)
        return select_impl<float, SEL_SBT>(n_cells, cell_start, v, law, lambda, nullptr, rng,
                                           pairs, ws, st, s);
    return arg_error("dsmc_select_pairs_sbt: dtype %d", dtype);
}

namespace dsmc {
// Shared with the fused step kernel.
int xs_law_public(const dsmc_xs& xs, double* C, double* e)
{
    XsLaw l;
    int rc = xs_law(xs, &l);
    *C = l.C;
    *e = l.e;
    return rc;
}
}  // namespace dsmc
