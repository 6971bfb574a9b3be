// The MU inner loop row by row. With the other factors fixed, row i of Phi
// depends only on row i of B and on row i's nonzeros, so the iterations of a row
// need no other row: a workgroup forms the pi rows of its rows' nonzeros once,
// keeps them in registers and runs all the inner iterations
//   m_k = b . pi_k,  phi = sum_k x_k / max(m_k, eps) pi_k,  b <- b .* phi
// on them. The Phi kernel's limit is the gather of the other factors' rows
// (every iteration again); here each row is gathered once per inner loop.
//
// The only coupling between rows is the KKT stop (one violation for the whole
// mode). With tol > 0 the light and team rows run a chunk of iterations
// speculatively and record each iteration's violation; the heavy rows, for which
// every iteration costs the gathers again, follow one iteration at a time and
// halt at the first one whose violation over all rows is below tol. decide_kernel
// finds that iteration, and if there is one the others go back to it: by a copy
// if it was the chunk's last, else the light rows run again from their saved
// start and the team rows are taken from their history (all on the device, no
// host round trip).
//
// Rows by length (a plan-time counting sort of the rows into classes):
//  * up to K nonzeros: one group of G lanes per row (each lane holds C rank
//    columns, R <= G * C, of up to K pi rows); 64 / G rows per wave;
//  * longer: 2, 4, .. 64 / G groups of a wave, then 2 or 4 waves of a workgroup;
//  * longer than 4 waves' registers, in a mode with few nonzeros in such rows: team
//    rows, each shared by several workgroups of 4 waves that meet once per iteration
//    and sum their partial rows in a fixed order (single loops: while all members
//    fit the device at once; batches: always);
//  * longer: heavy rows. Their nonzeros are cut into chunks of one row each; every
//    iteration gathers again (heavy_kernel), the last workgroup of a row to finish
//    sums the chunks' partial rows in order and takes the MU step of that row. With
//    three or four modes their nonzeros may be split by a second mode's longest
//    rows, which a workgroup keeps in LDS (hot_kernel).
// Every sum has a fixed order, so results repeat bit for bit while the same path
// is taken: the row of a team whose members were not all running in time is summed
// by one workgroup, in other pieces.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "internal.hpp"

namespace cpapr {
namespace {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// x / m for finite m > 0: reciprocal estimate and one Newton step (the Phi
// kernel's quotient, within a few ulps).
__device__ __forceinline__ double div_pos(double x, double m)
{
    double r = __builtin_amdgcn_rcp(m);
    r = __builtin_fma(r, __builtin_fma(-m, r, 1.0), r);
    return x * r;
}

__device__ __forceinline__ double wave_max(double v)
{
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    return v;
}

// quad_perm controls broadcasting lane j of each quad
template <int J>
__device__ __forceinline__ double quad_bcast(double v) { return dpp_f64<J * 0x55>(v); }
template <int J>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, J * 0x55, 0xF, 0xF, false);
}

// One block of four nonzeros of a lane group: every lane holds its C columns
// of the four pi rows and of b, and the value x of the nonzero whose slot is
// its lane's place in the quad. The four dot products are reduce-scattered
// over the quad (7 instead of 8 adds, and every lane ends with one nonzero), summed
// over the group's quads by mirrors, so that a lane divides once for the four,
// and the four scales come back as quad broadcasts. A mirror pairs place i
// with place 3 - i of another quad, so lanes of odd quads (G >= 8) hold the
// block's nonzeros in reverse order; everything else is the same for all lanes.
template <int G, int C>
__device__ __forceinline__ void block4(const double (&pi)[4][C], double x, const double (&b)[C], double eps, bool odd1,
                                       bool odd2, double (&acc)[C])
{
    double d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        d[j] = b[0] * pi[j][0];
#pragma unroll
        for (int c = 1; c < C; ++c) d[j] = __builtin_fma(b[c], pi[j][c], d[j]);
    }
    const double a0 = (odd1 ? d[1] : d[0]) + dpp_f64<0xB1>(odd1 ? d[0] : d[1]);
    const double a1 = (odd1 ? d[3] : d[2]) + dpp_f64<0xB1>(odd1 ? d[2] : d[3]);
    double m = (odd2 ? a1 : a0) + dpp_f64<0x4E>(odd2 ? a0 : a1);
    if constexpr (G >= 8) m += dpp_f64<0x141>(m);
    if constexpr (G >= 16) m += dpp_f64<0x140>(m);
    const double s = div_pos(x, __builtin_fmax(m, eps));
    const double s0 = quad_bcast<0>(s), s1 = quad_bcast<1>(s), s2 = quad_bcast<2>(s), s3 = quad_bcast<3>(s);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        acc[c] = __builtin_fma(s0, pi[0][c], acc[c]);
        acc[c] = __builtin_fma(s1, pi[1][c], acc[c]);
        acc[c] = __builtin_fma(s2, pi[2][c], acc[c]);
        acc[c] = __builtin_fma(s3, pi[3][c], acc[c]);
    }
}

// Columns [colbase, colbase + C) of the row at element offset `off`.
template <int C, typename L>
__device__ __forceinline__ void load_cols(const L* fac, uint32_t off, int colbase, double (&v)[C])
{
    const L* f = fac + (uint64_t)off + colbase;
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = (double)f[c];
}

// Sum of the two values v of lanes i and i ^ 16 (i ^ 32), in both.
__device__ __forceinline__ double sum_xor16(double v)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double sum_xor32(double v)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Place among its group's columns of a lane: groups with an odd number hold
// them in reverse, so that the mirrors below pair equal columns.
template <int G>
__device__ __forceinline__ int column_lane(int lane)
{
    if constexpr (G == 4) return (lane & 3) ^ (lane & 4 ? 3 : 0);
    if constexpr (G == 8) return (lane & 7) ^ (lane & 8 ? 7 : 0);
    return lane % G;
}

// Sum over the S lane groups (aligned, S a power of two up to 64 / G) of one
// row, every lane receiving its column's total, on the vector unit alone
// (shuffles through LDS made this most of a short iteration).
template <int G>
__device__ __forceinline__ double sum_groups(double v, int S)
{
    if constexpr (G == 4) {
        if (S >= 2) v += dpp_f64<0x141>(v);
        if (S >= 4) v += dpp_f64<0x140>(v);
    }
    if constexpr (G == 8)
        if (S >= 2) v += dpp_f64<0x140>(v);
    if (S * G >= 32) v = sum_xor16(v);
    if (S * G >= 64) v = sum_xor32(v);
    return v;
}

struct Entry {
    int32_t block0;  // first workgroup of the class
    int32_t row0;    // first position in `order`
    int32_t count;   // rows
    int32_t groups;  // lane groups per row (> 64 / G: several waves)
};
constexpr int kEntries = 16;

struct ResArgs {
    const uint32_t* cofs;
    const double* vals;
    const int32_t* row_ptr;
    const int32_t* order;
    const void* fac[kMaxOther];
    double* B;
    double* B0;     // saved start of the chunk (tol > 0), else nullptr
    double* B1;     // b before the chunk's last update (or nullptr)
    double* Phi;
    const int32_t* done;       // the inner loop has stopped: no work
    const int32_t* rerun;      // iteration to run again to (-1: none)
    unsigned long long* iv;    // [iv_slots x kInnerChunk] violations
    int iv_slots;
    int slot;                  // batch slot
    int teams;                 // team rows that run as teams
    double tol;
    double* heavy_hist;  // heavy rows: B, then Phi of their last iteration (restored on a stop)
    double* hist;        // team rows: B and Phi per iteration
    int64_t nnz;
    double eps;
    int R;
    int NM1;
    int n_it;       // iterations (rerun: read from the state)
    int each;       // 1: record every iteration's violation, 0: the last one's
    int nentries;
    int heavy0, nheavy;  // positions of the heavy rows in `order`, the rows that run as teams last
    int light_blocks;
    // team rows: workgroups (members) of one row that meet after every iteration
    int team_blocks;             // members of all teams
    int team0;                   // first team's heavy row
    const int32_t* team_begin;   // [teams + 1] first member of each team
    const int32_t* team_row;     // [members] team of each member
    double* team_part;           // [3 x members x R] members' partial rows, by iteration mod 3
    unsigned int* team_count;    // [teams] arrivals (kAbandoned: the team never met); zero between launches
    unsigned int* team_ticket;   // next member; zero between launches
    long long team_wait;         // clock ticks a member waits for its team to meet
    Entry entry[kEntries];
};

constexpr int kResBlock = 256;
constexpr int kCountStride = 32;  // u32 words between counters: one 128-byte line each (their atomics and polls serialise per line)

constexpr unsigned int kAbandoned = 0x80000000u;

// Members of a team exchange their partial rows after every iteration: a
// member stores its row in memory and reads everybody's, waiting for entries
// that still hold kNotYet. Three buffers in turn: in iteration l a member
// clears its row of l + 1 (read last in l - 2, which all have left) before it
// computes, and stores its row of l once that has arrived, so whoever sees the
// row of l never finds an old one in l + 1. One trip through memory per
// iteration; counting the members in and then reading took three (teams of up
// to 128 for all long rows of the 20M-nonzero three-way tensor: 1.34 against
// 1.69 ms per inner loop; with the counters on one cache line 3.4 ms).
//
// First the members must be running at all: in iteration 0 they count
// themselves in, their rows stored, and wait a bounded time for the team to be
// complete. A member that gives up marks the team abandoned (only while it is
// incomplete, so either all members meet or none); *last tells the last member to
// arrive at an abandoned team.
constexpr unsigned long long kNotYet = 0x7ff8a5a5c3c35a5aull;

__device__ __forceinline__ bool team_meet(unsigned int* count, unsigned int T, long long wait, bool* last)
{
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned int seen = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
    *last = seen == (kAbandoned | T);
    const long long t0 = wall_clock64();
    while (true) {
        if (seen & kAbandoned) return false;
        if (seen >= T) return true;
        if (wall_clock64() - t0 > wait) {
            unsigned int expect = seen;
            if (__hip_atomic_compare_exchange_strong(count, &expect, seen | kAbandoned, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                return false;
            seen = expect;
            continue;
        }
        __builtin_amdgcn_s_sleep(1);
        seen = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int G, int C, int K, bool MIXED, bool TEAM>
__device__ __forceinline__ void resident_rows(const ResArgs& a, int at, bool rerun, int n_it)
{
    using L = typename std::conditional<MIXED, float, double>::type;
    constexpr int NG = 64 / G;     // lane groups per wave
    constexpr int KB = K / 4;      // blocks of four nonzeros per lane group
    constexpr int W = kResBlock / 64;
    constexpr int RP = 4 * G;      // columns of a partial row, padded
    __shared__ double red[2][W][RP];
    __shared__ unsigned long long vmax[kInnerChunk];
    __shared__ int sh_ok, sh_last;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int gl = column_lane<G>(lane), g = lane / G;
    const int R = a.R;
    if (t < kInnerChunk) vmax[t] = 0ull;

    int row, S, sub, WR, member = 0, h = 0;
    int T = 1, nseg = 1;  // members of the team; pieces the row is taken in (an abandoned team's)
    uint32_t p0, p1;
    bool valid = true;
    uint32_t seg0 = 0, seg1 = 0;  // the whole row, for an abandoned team
    if constexpr (TEAM) {
        member = at;
        h = a.team_row[member];
        const int m0 = a.team_begin[h];
        T = a.team_begin[h + 1] - m0;
        row = a.order[a.heavy0 + a.team0 + h];
        seg0 = (uint32_t)a.row_ptr[row];
        seg1 = (uint32_t)a.row_ptr[row + 1];
        const uint32_t per = ((seg1 - seg0 + T - 1) / T + 3) / 4 * 4;
        p0 = seg0 + (uint32_t)(member - m0) * per;
        p1 = min(p0 + per, seg1);
        S = W * NG;
        WR = W;
        sub = wave * NG + g;
    } else {
        int e = 0;
        while (e + 1 < a.nentries && at >= a.entry[e + 1].block0) ++e;
        const int row0 = a.entry[e].row0, count = a.entry[e].count;
        S = a.entry[e].groups;
        WR = S > NG ? S / NG : 1;  // waves per row
        const int local = at - a.entry[e].block0;
        // position of this lane group's row in the class, and its place among the row's groups
        int pos;
        if (WR > 1) {
            pos = local * (W / WR) + wave / WR;
            sub = (wave % WR) * NG + g;
        } else {
            pos = (local * W + wave) * (NG / S) + g / S;
            sub = g % S;
        }
        valid = pos < count;
        row = a.order[row0 + (valid ? pos : count - 1)];
        p0 = (uint32_t)a.row_ptr[row];
        p1 = (uint32_t)a.row_ptr[row + 1];
    }
    bool lead = valid && sub == 0 && (!TEAM || p0 == seg0);  // writes the row

    const int colbase = min(gl * C, R - C);
    bool own[C];
#pragma unroll
    for (int c = 0; c < C; ++c) own[c] = colbase + c >= gl * C && colbase + c < R;
    const bool odd1 = lane & 1, odd2 = lane & 2;
    const int q = (lane & 3) ^ (G >= 8 && (lane & 4) ? 3 : 0);  // nonzero of the block this lane holds

    double b[C];
    {
        const double* src = (rerun ? a.B0 : a.B) + (int64_t)row * R + colbase;
#pragma unroll
        for (int c = 0; c < C; ++c) b[c] = own[c] ? src[c] : 0.0;
        if (!TEAM && !rerun && a.B0 != nullptr && lead)
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (own[c]) a.B0[(int64_t)row * R + colbase + c] = b[c];
    }

    // pi rows of [p0, p1): slots past the end repeat its last nonzero with value 0
    double pi[KB][4][C];
    double x[KB];
    int nb = 0;  // blocks this wave runs (the longest of its rows)
    auto gather = [&]() {
        nb = ((int)(p1 - p0) + 4 * S - 1) / (4 * S);
#pragma unroll
        for (int o = G; o < 64; o <<= 1) nb = max(nb, __shfl_xor(nb, o));
        nb = min(__builtin_amdgcn_readfirstlane(nb), KB);
        uint32_t off[KB];
        auto at = [&](int kb) { return p0 + (uint32_t)((kb * S + sub) * 4 + q); };
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            x[kb] = 0.0;
            off[kb] = 0;
            if (kb < nb) {
                x[kb] = at(kb) < p1 ? a.vals[min(at(kb), p1 - 1)] : 0.0;
                off[kb] = a.cofs[min(at(kb), p1 - 1)];
            }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[kb][j][c] = 1.0;
        for (int m = 0; m < a.NM1; ++m) {
            const L* fac = (const L*)a.fac[m];
            uint32_t next[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)  // the next factor's offsets before this one's rows are used
                next[kb] = kb < nb && m + 1 < a.NM1 ? a.cofs[(int64_t)(m + 1) * a.nnz + min(at(kb), p1 - 1)] : 0u;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb < nb) {
                    double f[4][C];
                    load_cols<C>(fac, quad_bcast<0>(off[kb]), colbase, f[0]);
                    load_cols<C>(fac, quad_bcast<1>(off[kb]), colbase, f[1]);
                    load_cols<C>(fac, quad_bcast<2>(off[kb]), colbase, f[2]);
                    load_cols<C>(fac, quad_bcast<3>(off[kb]), colbase, f[3]);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int c = 0; c < C; ++c) pi[kb][j][c] *= f[j][c];
                }
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) off[kb] = next[kb];
        }
    };

    double acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.0;
    __syncthreads();  // vmax is cleared
    for (int l = 0; l < n_it; ++l) {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = 0.0;
        if (TEAM && T > 1 && wave == 0 && g == 0)
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (own[c])
                    __hip_atomic_store((unsigned long long*)a.team_part +
                                           ((int64_t)((l + 1) % 3) * a.team_blocks + member) * R + colbase + c,
                                       kNotYet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int sg = 0; sg < nseg; ++sg) {
            if (TEAM && nseg > 1) {  // an abandoned team's row, piece by piece in every iteration
                p0 = seg0 + (uint32_t)sg * (uint32_t)(K * NG * W);
                p1 = min(p0 + (uint32_t)(K * NG * W), seg1);
            }
            if (l == 0 || (TEAM && nseg > 1)) gather();
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                if (kb < nb) block4<G, C>(pi[kb], x[kb], b, a.eps, odd1, odd2, acc);
        }
        // the row's other lane groups of this wave
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = sum_groups<G>(acc[c], S);
        if (WR > 1) {  // uniform over the workgroup
            double(*rd)[RP] = red[l & 1];
            if (g == 0)
#pragma unroll
                for (int c = 0; c < C; ++c) rd[wave][gl * C + c] = acc[c];
            __syncthreads();
            const int w0 = wave / WR * WR;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                double v = 0.0;
                for (int w = 0; w < WR; ++w) v += rd[w0 + w][gl * C + c];
                acc[c] = v;
            }
        }
        if (TEAM && T > 1) {  // a team: the members' partial rows, summed by every member in the same order
            double* part = a.team_part + (int64_t)(l % 3) * a.team_blocks * R;
            if (wave == 0 && g == 0) {
                __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the next meeting's row is cleared
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (own[c]) {
                        // a value with the bits of "not there yet" can only be a NaN of the inputs
                        const double v = acc[c] == acc[c] ? acc[c] : __builtin_nan("");
                        __hip_atomic_store(&part[(int64_t)member * R + colbase + c], v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    }
            }
            if (l == 0) {
                if (t == 0) {
                    bool last = false;
                    sh_ok = team_meet(a.team_count + h * kCountStride, (unsigned int)T, a.team_wait, &last);
                    sh_last = last;
                }
                __syncthreads();
                if (!__builtin_amdgcn_readfirstlane(sh_ok)) {
                    // Nobody else works on this row: its last member does, alone.
                    if (!__builtin_amdgcn_readfirstlane(sh_last)) return;
                    __syncthreads();
                    T = 1;
                    lead = sub == 0;
                    nseg = (int)((seg1 - seg0 + K * NG * W - 1) / (uint32_t)(K * NG * W));
                    l = -1;
                    continue;
                }
            }
            const int m0 = a.team_begin[h];
            const int c1 = lane % RP, k0 = wave * (64 / RP) + lane / RP;
            constexpr int KS = W * (64 / RP);
            double v = 0.0;
            if (c1 < R) {
                const double* src = part + (int64_t)m0 * R + c1;
                for (int k = k0; k < T; k += 4 * KS) {
                    unsigned long long u[4];
                    bool wait;
                    do {  // every member is running: its row comes
                        wait = false;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            u[i] = k + i * KS < T ? __hip_atomic_load((const unsigned long long*)&src[(int64_t)(k + i * KS) * R],
                                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                  : 0ull;
#pragma unroll
                        for (int i = 0; i < 4; ++i) wait = wait || u[i] == kNotYet;
                    } while (wait);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v += __longlong_as_double((long long)u[i]);
                }
            }
            if constexpr (RP <= 16) v = sum_xor16(v);
            if constexpr (RP <= 32) v = sum_xor32(v);
            double(*rd)[RP] = red[(l & 1) ^ 1];
            if (lane < RP) rd[wave][lane] = v;
            __syncthreads();
#pragma unroll
            for (int c = 0; c < C; ++c) {
                double w = 0.0;
#pragma unroll
                for (int u = 0; u < W; ++u) w += rd[u][colbase + c];
                acc[c] = w;
            }
            __syncthreads();
        }
        if (!rerun && (a.each || l + 1 == n_it)) {
            double v = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const double r = 1.0 - acc[c];
                if (own[c]) v = fmax(v, fabs(b[c] < r ? b[c] : r));
            }
            v = wave_max(valid ? v : 0.0);
            if (lane == 0) atomicMax(&vmax[a.each ? l : 0], (unsigned long long)__double_as_longlong(v));
            if (TEAM && a.each && lead)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (own[c]) {
                        const int64_t n = (int64_t)a.teams * R;
                        double* hist = a.hist + 2 * l * n + (int64_t)h * R + colbase + c;
                        hist[0] = b[c];
                        hist[n] = acc[c];
                    }
        }
        if (l + 1 < n_it)
#pragma unroll
            for (int c = 0; c < C; ++c) b[c] *= acc[c];
    }
    if (lead)
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (own[c]) {
                const int64_t e = (int64_t)row * R + colbase + c;
                if (!TEAM && !rerun && a.B1 != nullptr) a.B1[e] = b[c];
                a.B[e] = rerun ? b[c] : b[c] * acc[c];
                a.Phi[e] = acc[c];
            }
    if (!rerun) {
        __syncthreads();
        const int nv = a.each ? n_it : 1;
        if (t < nv) atomicMax(&a.iv[blockIdx.x % a.iv_slots * kInnerChunk + t], vmax[t]);
    }
}

// Next team member: members in the order in which workgroups start, so that the
// oldest team is always the first to be complete.
__device__ __forceinline__ int next_member(unsigned int* ticket)
{
    __shared__ int sh;
    if (threadIdx.x == 0) sh = (int)__hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(sh);
}

// Team members and light workgroups alternate in launch order, so that a
// compute unit has light rows to work on while a team meets. Returns whether
// workgroup b is a team's; *light: its place among the light ones.
__device__ __forceinline__ bool team_turn(int b, int members, int lights, int* light)
{
    const int both = min(members, lights);
    *light = b < 2 * both ? b >> 1 : b - members;
    return b < 2 * both ? (b & 1) == 0 : members > lights;
}

// Heavy and team rows from their history after a stop at iteration l.
__device__ __forceinline__ void restore_rows(const ResArgs& a, int l, int at, int blocks)
{
    const int64_t nh = (int64_t)(a.nheavy - a.teams) * a.R, nt = (int64_t)a.teams * a.R;
    for (int64_t i = (int64_t)at * kResBlock + threadIdx.x; i < nh + nt; i += (int64_t)blocks * kResBlock) {
        const int64_t e = (int64_t)a.order[a.heavy0 + i / a.R] * a.R + i % a.R;
        const double* hist = i < nh ? a.heavy_hist + i : a.hist + 2 * l * nt + (i - nh);
        a.B[e] = hist[0];
        a.Phi[e] = hist[i < nh ? nh : nt];
    }
}

// The light rows back to before the chunk's last update, after a stop there
// (Phi is that iteration's already).
__device__ __forceinline__ void restore_last(const ResArgs& a, int n_it, int at)
{
    const double* src = n_it == 1 ? a.B0 : a.B1;
    for (int64_t i = (int64_t)at * kResBlock + threadIdx.x; i < (int64_t)a.heavy0 * a.R;
         i += (int64_t)a.light_blocks * kResBlock) {
        const int64_t e = (int64_t)a.order[i / a.R] * a.R + i % a.R;
        a.B[e] = src[e];
    }
}

// After a stop at iteration l of n_it: block `at` of the light rows' or, after
// them, of the others'.
template <int G, int C, int K, bool MIXED>
__device__ __forceinline__ void back_to(const ResArgs& a, int l, int n_it, int at, int blocks)
{
    if (at >= a.light_blocks)
        restore_rows(a, l, at - a.light_blocks, blocks - a.light_blocks);
    else if (l + 1 == n_it && (n_it == 1 || a.B1 != nullptr))
        restore_last(a, n_it, at);
    else
        resident_rows<G, C, K, MIXED, false>(a, at, true, l + 1);
}

// Two waves per SIMD: the pi rows take most of a lane's 256 registers.
template <int G, int C, int K, bool MIXED>
__global__ __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void resident_kernel(ResArgs a)
{
    if (*a.done) return;
    int light;
    if (team_turn((int)blockIdx.x, a.team_blocks, a.light_blocks, &light))
        resident_rows<G, C, K, MIXED, true>(a, next_member(a.team_ticket), false, a.n_it);
    else
        resident_rows<G, C, K, MIXED, false>(a, light, false, a.n_it);
}

// After a stop at iteration *rerun of the chunk: all rows back to it.
template <int G, int C, int K, bool MIXED>
__global__ __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void rerun_kernel(ResArgs a)
{
    const int l = *a.rerun;
    if (l < 0) return;
    back_to<G, C, K, MIXED>(a, l, a.n_it, (int)blockIdx.x, (int)gridDim.x);
}

// Item of `n` (prefix [n + 1] of counts) that holds place `at`: one load per
// thread instead of a chain of them (called by the whole workgroup).
__device__ __forceinline__ int item_at(const int32_t* __restrict__ prefix, int n, int at)
{
    int found = 0;
    for (int i0 = 0; i0 < n; i0 += kResBlock) {
        const int i = i0 + (int)threadIdx.x;
        found += __syncthreads_count(i < n && prefix[i] <= at);
    }
    return __builtin_amdgcn_readfirstlane(found - 1);
}

// The same for the slots of a batch that share a launch shape.
template <int G, int C, int K, bool MIXED>
__global__ __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void batch_resident_kernel(
    const ResArgs* __restrict__ items, const int32_t* __restrict__ lights, const int32_t* __restrict__ members, int n,
    int nlight, int nmembers, unsigned int* ticket, int n_it)
{
    int light;
    if (team_turn((int)blockIdx.x, nmembers, nlight, &light)) {
        const int m = next_member(ticket);
        const int i = item_at(members, n, m);
        if (*items[i].done) return;
        resident_rows<G, C, K, MIXED, true>(items[i], m - members[i], false, n_it);
    } else {
        const int i = item_at(lights, n, light);
        if (*items[i].done) return;
        resident_rows<G, C, K, MIXED, false>(items[i], light - lights[i], false, n_it);
    }
}

template <int G, int C, int K, bool MIXED>
__global__ __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void batch_rerun_kernel(
    const ResArgs* __restrict__ items, const int32_t* __restrict__ blocks, int n, int n_it)
{
    const int i = item_at(blocks, n, (int)blockIdx.x);
    const int l = *items[i].rerun;
    if (l < 0) return;
    back_to<G, C, K, MIXED>(items[i], l, n_it, (int)blockIdx.x - blocks[i], blocks[i + 1] - blocks[i]);
}

// A heavy row has added its violation of iteration l to the slots (one wave; lane
// 0 did): the last of the nrows rows knows the iteration's violation over all
// rows of the mode and halts the chunk's further heavy iterations if it is below
// tol. The counters are spread (one row after the other on a single one would
// take longer than the rows' sums) and are zero again afterwards.
__device__ __forceinline__ void row_finished(DevState* st, unsigned int* finished, int h, int nrows, int l, double tol)
{
    static_assert(kInnerSlots == 64, "a slot per lane");
    int last = 0;
    if ((threadIdx.x & 63) == 0) {
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int slot = h % kInnerSlots;
        unsigned int* c = finished + (1 + slot) * kCountStride;
        const unsigned int n = (unsigned int)((nrows - slot + kInnerSlots - 1) / kInnerSlots);
        if (__hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == n) {
            __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = __hip_atomic_fetch_add(finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                   (unsigned int)min(nrows, kInnerSlots);
            if (last) __hip_atomic_store(finished, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    const double v = wave_max(__longlong_as_double((long long)__hip_atomic_load(
        &st->iv[threadIdx.x & 63][l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
    if ((threadIdx.x & 63) == 0 && v < tol)
        __hip_atomic_store(&st->halt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct HeavyArgs {
    const uint32_t* cofs[kMaxOther];  // offsets into fac[m]
    const double* vals;
    const int32_t* row_ptr;
    const int32_t* rows;         // heavy rows (in `order`)
    const int32_t* chunk_begin;  // [nheavy + 1] first chunk of each heavy row
    const int32_t* chunk_row;    // [chunks] heavy row of each chunk
    const void* fac[kMaxOther];
    double* B;
    double* Phi;
    double* partial;             // [chunks x R]
    unsigned int* ticket;        // [nheavy], zero between launches
    DevState* st;
    double* hist;                // tol > 0: B, then Phi of this iteration, else nullptr
    unsigned int* finished;      // counters of row_finished
    int64_t nnz;
    double eps, tol;
    int nrows;                   // heavy rows
    int R;
    int NM1;
    int chunk;
    int l;                       // violation slot of this iteration, -1: not recorded
};

// One iteration of the heavy rows: a workgroup per chunk of one row, so b is
// loaded once and there is no row logic. A wave takes 4 * 64 / G consecutive
// nonzeros per step, four per lane group, their gathers in flight together.
template <int G, int C, int NM1, bool MIXED>
__global__ __launch_bounds__(kBlock) void heavy_kernel(HeavyArgs a)
{
    using L = typename std::conditional<MIXED, float, double>::type;
    constexpr int W = kBlock / 64;
    constexpr int STEP = 4 * (64 / G);
    __shared__ double red[W][G * C];
    __shared__ double fin[kBlock];
    __shared__ int last;
    if (a.st->done || a.st->halt) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int gl = lane % G, g = lane / G;
    const int R = a.R;
    const int ch = blockIdx.x;
    const int h = a.chunk_row[ch];
    const int row = a.rows[h];
    const int c0 = a.chunk_begin[h], nch = a.chunk_begin[h + 1] - c0;
    const uint32_t r1 = (uint32_t)a.row_ptr[row + 1];
    const uint32_t p0 = (uint32_t)a.row_ptr[row] + (uint32_t)((ch - c0) * a.chunk);
    const uint32_t p1 = min(p0 + (uint32_t)a.chunk, r1);
    const uint32_t per = (uint32_t)((a.chunk / W + STEP - 1) / STEP * STEP);
    const uint32_t w0 = p0 + (uint32_t)wave * per, w1 = min(w0 + per, p1);

    const int colbase = min(gl * C, R - C);
    const bool odd1 = lane & 1, odd2 = lane & 2;
    const int q = (lane & 3) ^ (G >= 8 && (lane & 4) ? 3 : 0);
    double b[C], acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const bool own = colbase + c >= gl * C && colbase + c < R;
        b[c] = own ? a.B[(int64_t)row * R + colbase + c] : 0.0;
        acc[c] = 0.0;
    }
    // Other modes: a.fac[0] is the one the row's nonzeros are ordered by. While a
    // step's nonzeros all share that coordinate (a fiber of the row), its factor
    // row multiplies b once instead of every nonzero, and is not gathered again:
    //   m = (b .* a) . f,  phi += a .* (sum of s f),  f the other factors' product.
    const int nm1 = NM1 > 0 ? NM1 : a.NM1;
    constexpr int NOFF = NM1 > 0 ? NM1 : 1;
    uint32_t off[NOFF];
    double x = 0.0;
    auto load_meta = [&](uint32_t base) {
        const uint32_t p = base + (uint32_t)(g * 4 + q);
        const uint32_t pc = min(p, w1 - 1);
        x = __builtin_nontemporal_load(a.vals + pc);
        if (p >= w1) x = 0.0;
#pragma unroll
        for (int m = 0; m < NOFF; ++m) off[m] = __builtin_nontemporal_load(a.cofs[m] + pc);
    };
    uint32_t cur = 0;
    double arow[C], bw[C], tacc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) arow[c] = bw[c] = tacc[c] = 0.0;
    bool have = false;
    if (w0 < w1) load_meta(w0);
    for (uint32_t base = w0; base < w1; base += STEP) {
        double pi[4][C];
        const double xc = x;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)off[0]);
        const bool fiber = NM1 != 1 && __ballot(off[0] != first) == 0ull;
        if (fiber && (!have || first != cur)) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                acc[c] = __builtin_fma(arow[c], tacc[c], acc[c]);
                tacc[c] = 0.0;
            }
            load_cols<C>((const L*)a.fac[0], first, colbase, arow);
#pragma unroll
            for (int c = 0; c < C; ++c) bw[c] = b[c] * arow[c];
            cur = first;
            have = true;
        }
        if constexpr (NM1 > 0) {
            double f[NM1][4][C];
            auto gather = [&](int m) {
                const L* fac = (const L*)a.fac[m];
                load_cols<C>(fac, quad_bcast<0>(off[m]), colbase, f[m][0]);
                load_cols<C>(fac, quad_bcast<1>(off[m]), colbase, f[m][1]);
                load_cols<C>(fac, quad_bcast<2>(off[m]), colbase, f[m][2]);
                load_cols<C>(fac, quad_bcast<3>(off[m]), colbase, f[m][3]);
            };
#pragma unroll
            for (int m = 1; m < NM1; ++m) gather(m);
            if (fiber) {
                if (base + STEP < w1) load_meta(base + STEP);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        pi[j][c] = f[NM1 - 1][j][c];
#pragma unroll
                        for (int m = 1; m < NM1 - 1; ++m) pi[j][c] *= f[m][j][c];
                    }
                block4<G, C>(pi, xc, bw, a.eps, odd1, odd2, tacc);
            } else {
                gather(0);
                if (base + STEP < w1) load_meta(base + STEP);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        pi[j][c] = f[0][j][c];
#pragma unroll
                        for (int m = 1; m < NM1; ++m) pi[j][c] *= f[m][j][c];
                    }
                block4<G, C>(pi, xc, b, a.eps, odd1, odd2, acc);
            }
        } else {
            const uint32_t pc = min(base + (uint32_t)(g * 4 + q), w1 - 1);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[j][c] = 1.0;
            for (int m = fiber ? 1 : 0; m < nm1; ++m) {
                const L* fac = (const L*)a.fac[m];
                const uint32_t o = m == 0 ? off[0] : a.cofs[m][pc];
                double f[4][C];
                load_cols<C>(fac, quad_bcast<0>(o), colbase, f[0]);
                load_cols<C>(fac, quad_bcast<1>(o), colbase, f[1]);
                load_cols<C>(fac, quad_bcast<2>(o), colbase, f[2]);
                load_cols<C>(fac, quad_bcast<3>(o), colbase, f[3]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < C; ++c) pi[j][c] *= f[j][c];
            }
            if (base + STEP < w1) load_meta(base + STEP);
            if (fiber)
                block4<G, C>(pi, xc, bw, a.eps, odd1, odd2, tacc);
            else
                block4<G, C>(pi, xc, b, a.eps, odd1, odd2, acc);
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = __builtin_fma(arow[c], tacc[c], acc[c]);
    // lane groups, then waves, in a fixed order
#pragma unroll
    for (int o = G; o < 64; o <<= 1)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] += __shfl_xor(acc[c], o);
    if (g == 0)
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (colbase + c >= gl * C && colbase + c < R) red[wave][colbase + c] = acc[c];
    __syncthreads();
    // The partial row goes out past the L2 of this die (other dies' workgroups
    // may finish the row); the ticket is taken once it has arrived.
    if (t < R) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) v += red[w][t];
        __hip_atomic_store(&a.partial[(int64_t)ch * R + t], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
        const unsigned int k = __hip_atomic_fetch_add(&a.ticket[h * kCountStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = k + 1 == (unsigned int)nch;
    }
    __syncthreads();
    if (!last) return;
    // this workgroup is the row's last: sum its chunks, kBlock / rp of them in parallel
    int rp = 1;
    while (rp < R) rp *= 2;
    const int lanes = kBlock / rp, c = t % rp, jj = t / rp;
    double v = 0.0;
    if (c < R) {
        const double* src = a.partial + (int64_t)c0 * R + c;
        int k = jj;
        for (; k + 7 * lanes < nch; k += 8 * lanes) {
            double u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                u[i] = __hip_atomic_load(&src[(int64_t)(k + i * lanes) * R], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int i = 0; i < 8; ++i) v += u[i];
        }
        for (; k < nch; k += lanes)
            v += __hip_atomic_load(&src[(int64_t)k * R], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    fin[t] = v;
    __syncthreads();
    for (int w = lanes / 2; w > 0; w >>= 1) {
        if (jj < w) fin[t] += fin[t + w * rp];
        __syncthreads();
    }
    double viol = 0.0;
    if (t < R) {
        const int64_t e = (int64_t)row * R + t;
        const double phi = fin[t], bb = a.B[e], r = 1.0 - phi;
        viol = fabs(bb < r ? bb : r);
        a.Phi[e] = phi;
        if (a.hist != nullptr) {
            a.hist[(int64_t)h * R + t] = bb;
            a.hist[(int64_t)(a.nrows + h) * R + t] = phi;
        }
        a.B[e] = bb * phi;
    }
    if (t == 0) a.ticket[h * kCountStride] = 0u;
    if (a.l >= 0 && t < 64) {
        viol = wave_max(viol);
        if (t == 0) atomicMax(&a.st->iv[h % kInnerSlots][a.l], (unsigned long long)__double_as_longlong(viol));
        if (a.hist != nullptr) row_finished(a.st, a.finished, h, a.nrows, a.l, a.tol);
    }
}

// ---- heavy rows with a second factor's hot rows in LDS ----

constexpr int kHotThreads = 1024;          // one workgroup per compute unit
constexpr int kHotLds = 140 * 1024;        // bytes of hot rows (the workgroup's sums take up to 16 KB more)
constexpr int kMaxHot = kHotLds / 8;       // places of hot rows, at every rank and width
constexpr uint16_t kCold = 0xffff;
static_assert(kMaxHot < kCold, "places fit 16 bits");

struct HotArgs {
    const uint32_t *s_lead, *s_hot, *s_third, *s_val;
    const double* vals;       // the sorted copy's, where s_val holds positions
    const int4* entry;
    const int32_t *xlist, *xbegin;
    const int32_t* rows;      // long rows (in `order`)
    const uint4* tab;         // the hot rows, in their places
    int tab_vecs;             // 16-byte words of them
    const void *lead, *hot, *third;
    const double* B;
    double* partial;          // [pieces x R]
    DevState* st;
    int R;
    double eps;
};

// A factor's hot rows in their places, once per inner loop.
template <typename L>
__global__ __launch_bounds__(kBlock) void hot_table_kernel(const L* __restrict__ fac, const int32_t* __restrict__ rows,
                                                           int nhot, int R, L* __restrict__ tab)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < nhot * R; i += gridDim.x * kBlock)
        tab[i] = fac[(int64_t)rows[i / R] * R + i % R];
}

template <int C, typename L>
__device__ __forceinline__ void load_lds(const L* tab, uint32_t at, double (&v)[C])
{
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = (double)tab[at + c];
}

// The partial rows of one iteration of the heavy rows, by workgroups that stay
// on their compute unit: each copies the hot rows of one factor to LDS once,
// then its waves take pieces of rows in turn, each on its own. In a hot piece
// every nonzero reads that factor from LDS; the gathers past L1 (the bound of
// heavy_kernel) are left to the other factors. The pieces of a long row go to
// the dies by their place in the row, and a die takes them in that order, so
// that the rows of the leading factor it gathers at a time stay in its L2.
template <int G, int C, bool THIRD, bool MIXED, bool EXACT>
__global__ __launch_bounds__(kHotThreads) void hot_kernel(HotArgs a)
{
    using L = typename std::conditional<MIXED, float, double>::type;
    constexpr int W = kHotThreads / 64;
    constexpr uint32_t STEP = 4 * (64 / G);
    extern __shared__ double2 dyn[];
    const L* tab = (const L*)dyn;
    if (a.st->done || a.st->halt) return;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int gl = lane % G, g = lane / G;
    const int R = a.R;
#pragma unroll 5
    for (int i = t; i < a.tab_vecs; i += kHotThreads) ((uint4*)dyn)[i] = a.tab[i];
    const int colbase = min(gl * C, R - C);
    const bool odd1 = lane & 1, odd2 = lane & 2;
    const int q = (lane & 3) ^ (G >= 8 && (lane & 4) ? 3 : 0);
    __syncthreads();
    const int die = (int)blockIdx.x % kXcds, nb = ((int)gridDim.x - die + kXcds - 1) / kXcds;  // workgroups of this die
    const int k1 = a.xbegin[die + 1];
    for (int k = a.xbegin[die] + wave * nb + (int)blockIdx.x / kXcds; k < k1; k += W * nb) {
        const int e = a.xlist[k];
        const int4 en = a.entry[e];
        const int row = a.rows[en.x];
        const uint32_t w0 = (uint32_t)en.y, w1 = (uint32_t)en.z;
        double b[C], acc[C], arow[C], bw[C], tacc[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const bool own = colbase + c >= gl * C && colbase + c < R;
            b[c] = own ? a.B[(int64_t)row * R + colbase + c] : 0.0;
            acc[c] = arow[c] = bw[c] = tacc[c] = 0.0;
        }
        auto run = [&](auto hotpart) {
            constexpr bool HOT = decltype(hotpart)::value;
            uint32_t ol = 0, oh = 0, o3 = 0, cur = 0, at = 0;
            double x = 0.0;
            bool have = false;
            const uint16_t* slot = (const uint16_t*)a.s_hot + (en.w - 1);
            if (!EXACT) at = a.s_val[min(w0 + (uint32_t)(g * 4 + q), w1 - 1)];
            auto load_meta = [&](uint32_t base) {
                const uint32_t p = base + (uint32_t)(g * 4 + q);
                const uint32_t pc = min(p, w1 - 1);
                if constexpr (EXACT) {
                    x = (double)__uint_as_float(__builtin_nontemporal_load(a.s_val + pc));
                } else {  // the position was loaded a step ahead
                    x = a.vals[at];
                    at = __builtin_nontemporal_load(a.s_val + min(p + STEP, w1 - 1));
                }
                if (p >= w1) x = 0.0;
                ol = __builtin_nontemporal_load(a.s_lead + pc);
                if constexpr (HOT)
                    oh = (uint32_t)__builtin_nontemporal_load(slot + pc) * (uint32_t)R;
                else
                    oh = __builtin_nontemporal_load(a.s_hot + pc);
                if constexpr (THIRD) o3 = __builtin_nontemporal_load(a.s_third + pc);
            };
            if (w0 < w1) load_meta(w0);
            for (uint32_t base = w0; base < w1; base += STEP) {
                const double xc = x;
                const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)ol);
                const bool fiber = __ballot(ol != first) == 0ull;
                if (fiber && (!have || first != cur)) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc[c] = __builtin_fma(arow[c], tacc[c], acc[c]);
                        tacc[c] = 0.0;
                    }
                    load_cols<C>((const L*)a.lead, first, colbase, arow);
#pragma unroll
                    for (int c = 0; c < C; ++c) bw[c] = b[c] * arow[c];
                    cur = first;
                    have = true;
                }
                double pi[4][C], f[4][C];
                if constexpr (THIRD) {
                    const L* fac = (const L*)a.third;
                    load_cols<C>(fac, quad_bcast<0>(o3), colbase, f[0]);
                    load_cols<C>(fac, quad_bcast<1>(o3), colbase, f[1]);
                    load_cols<C>(fac, quad_bcast<2>(o3), colbase, f[2]);
                    load_cols<C>(fac, quad_bcast<3>(o3), colbase, f[3]);
                }
                auto second = [&]() {
                    if constexpr (HOT) {
                        load_lds<C>(tab, quad_bcast<0>(oh) + colbase, pi[0]);
                        load_lds<C>(tab, quad_bcast<1>(oh) + colbase, pi[1]);
                        load_lds<C>(tab, quad_bcast<2>(oh) + colbase, pi[2]);
                        load_lds<C>(tab, quad_bcast<3>(oh) + colbase, pi[3]);
                    } else {
                        const L* fac = (const L*)a.hot;
                        load_cols<C>(fac, quad_bcast<0>(oh), colbase, pi[0]);
                        load_cols<C>(fac, quad_bcast<1>(oh), colbase, pi[1]);
                        load_cols<C>(fac, quad_bcast<2>(oh), colbase, pi[2]);
                        load_cols<C>(fac, quad_bcast<3>(oh), colbase, pi[3]);
                    }
                };
                auto times = [&]() {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int c = 0; c < C; ++c) pi[j][c] *= f[j][c];
                };
                if (fiber) {
                    second();
                    if (base + STEP < w1) load_meta(base + STEP);
                    if constexpr (THIRD) times();
                    block4<G, C>(pi, xc, bw, a.eps, odd1, odd2, tacc);
                } else {
                    second();
                    if constexpr (THIRD) times();
                    const L* fac = (const L*)a.lead;
                    load_cols<C>(fac, quad_bcast<0>(ol), colbase, f[0]);
                    load_cols<C>(fac, quad_bcast<1>(ol), colbase, f[1]);
                    load_cols<C>(fac, quad_bcast<2>(ol), colbase, f[2]);
                    load_cols<C>(fac, quad_bcast<3>(ol), colbase, f[3]);
                    if (base + STEP < w1) load_meta(base + STEP);
                    times();
                    block4<G, C>(pi, xc, b, a.eps, odd1, odd2, acc);
                }
            }
        };
        if (en.w)
            run(std::true_type{});
        else
            run(std::false_type{});
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = __builtin_fma(arow[c], tacc[c], acc[c]);
#pragma unroll
        for (int o = G; o < 64; o <<= 1)
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] += __shfl_xor(acc[c], o);
        if (g == 0)
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (colbase + c >= gl * C && colbase + c < R) a.partial[(int64_t)e * R + colbase + c] = acc[c];
    }
}

struct HotStep {
    const int32_t* entry_begin;
    const int32_t* rows;
    const double* partial;
    double* B;
    double* Phi;
    DevState* st;
    double* hist;
    unsigned int* finished;
    double tol;
    int nrows;
    int R;
    int l;
};

// After hot_kernel: a workgroup per long row sums its pieces' partial rows and
// takes the row's MU step.
__global__ __launch_bounds__(512) void hot_step_kernel(HotStep a)
{
    __shared__ double sum[8][64];
    if (a.st->done || a.st->halt) return;
    const int t = threadIdx.x, lane = t & 63, R = a.R, h = blockIdx.x;
    const int e0 = a.entry_begin[h], ne = a.entry_begin[h + 1] - e0;
    int rp = 1;
    while (rp < R) rp *= 2;
    const int lanes = 512 / rp, c = t % rp, jj = t / rp;
    double v = 0.0;
    if (c < R) {
        const double* src = a.partial + (int64_t)e0 * R + c;
        int k = jj;
        for (; k + 15 * lanes < ne; k += 16 * lanes) {  // sixteen loads in flight: the longest row is a chain of them
            double u[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) u[i] = src[(int64_t)(k + i * lanes) * R];
#pragma unroll
            for (int i = 0; i < 16; ++i) v += u[i];
        }
        for (; k < ne; k += lanes) v += src[(int64_t)k * R];
    }
    for (int o = rp; o < 64; o <<= 1) v += __shfl_xor(v, o);
    if (lane < rp) sum[t >> 6][lane] = v;
    __syncthreads();
    if (t >= 64) return;
    double viol = 0.0;
    if (t < R) {
        const int64_t x = (int64_t)a.rows[h] * R + t;
        double phi = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) phi += sum[w][t];
        const double b = a.B[x], r = 1.0 - phi;
        viol = fabs(b < r ? b : r);
        a.Phi[x] = phi;
        if (a.hist != nullptr) {
            a.hist[(int64_t)h * R + t] = b;
            a.hist[(int64_t)(a.nrows + h) * R + t] = phi;
        }
        a.B[x] = b * phi;
    }
    if (a.l >= 0) {
        viol = wave_max(viol);
        if (t == 0) atomicMax(&a.st->iv[h % kInnerSlots][a.l], (unsigned long long)__double_as_longlong(viol));
        if (a.hist != nullptr) row_finished(a.st, a.finished, h, a.nrows, a.l, a.tol);
    }
}

// End of a chunk of n iterations (one workgroup): the largest violation of each
// iteration, the slots cleared; the first iteration below tol stops the inner
// loop. Returns that iteration or -1, *viol the last violation that counts (thread 0).
__device__ __forceinline__ int decide(unsigned long long* iv, int slots, int n, bool each, double tol, double* viol)
{
    static_assert(kInnerChunk == 16 && kBlock == 256, "sixteen threads per iteration");
    __shared__ unsigned long long part[16][kInnerChunk], v[kInnerChunk];
    const int t = threadIdx.x, l0 = t % kInnerChunk;
    unsigned long long m = 0ull;
    for (int i = t; i < slots * kInnerChunk; i += kBlock) {
        const unsigned long long u = iv[i];
        m = u > m ? u : m;
        if (u) iv[i] = 0ull;
    }
    part[t / kInnerChunk][l0] = m;
    __syncthreads();
    if (t < kInnerChunk) {
        for (int k = 1; k < 16; ++k) m = part[k][t] > m ? part[k][t] : m;
        v[t] = m;
    }
    __syncthreads();
    int stop = -1;
    if (each)
        for (int l = 0; l < n && stop < 0; ++l)
            if (__longlong_as_double((long long)v[l]) < tol) stop = l;
    *viol = __longlong_as_double((long long)v[stop >= 0 ? stop : each ? n - 1 : 0]);
    return stop;
}

__global__ __launch_bounds__(kBlock) void decide_kernel(DevState* st, int mode, int n, int each, double tol,
                                                        unsigned int* team_ticket, unsigned int* team_count, int teams)
{
    const int t = threadIdx.x;
    for (int i = t; i < teams; i += kBlock) team_count[i * kCountStride] = 0u;
    if (t == 0) {
        *team_ticket = 0u;
        st->halt = 0;
    }
    if (st->done) {
        if (t == 0) {
            st->rerun = -1;
            st->mode_updates[mode] = st->updates;
        }
        return;
    }
    double viol;
    const int stop = decide(&st->iv[0][0], kInnerSlots, n, each != 0, tol, &viol);
    if (t != 0) return;
    const int upd = stop >= 0 ? stop : n;
    st->last_viol[mode] = viol;
    st->rerun = stop;
    if (stop >= 0) st->done = 1;
    st->updates += upd;
    st->sweep_updates += upd;
    st->total_updates += upd;
    st->phi_evals += stop >= 0 ? stop + 1 : n;
    st->mode_updates[mode] = st->updates;
}

// A workgroup per slot of a batch.
__global__ __launch_bounds__(kBlock) void batch_decide_kernel(const ResArgs* __restrict__ items, BatchState st,
                                                              int32_t* __restrict__ rerun, int n,
                                                              unsigned int* __restrict__ tickets)
{
    const ResArgs& a = items[blockIdx.x];
    const int t = threadIdx.x, slot = a.slot;
    for (int i = t; i < a.teams; i += kBlock) a.team_count[i * kCountStride] = 0u;
    if (blockIdx.x == 0 && t < kRowShapes) tickets[t * kCountStride] = 0u;
    if (st.done[slot]) {
        if (t == 0) rerun[slot] = -1;
        return;
    }
    double viol;
    const int stop = decide(a.iv, a.iv_slots, n, a.each != 0, a.tol, &viol);
    if (t != 0) return;
    st.viol[slot] = viol;
    st.updates[slot] += stop >= 0 ? stop : n;
    rerun[slot] = stop;
    if (stop >= 0) st.done[slot] = 1;
}

// ---- plan: rows by class ----

// Row classes of a launch shape: 0..KB blocks of four nonzeros for one lane
// group, then 2, 4, .. NG groups of a wave, then 2 and 4 waves, then heavy rows
// (more than kTeamMax workgroups' registers) and team rows.
struct ClassShape {
    int KB, NG;
};

__host__ __device__ inline int class_count(ClassShape c)
{
    int lg = 0;
    while ((1 << lg) < c.NG) ++lg;
    return c.KB + lg + 5;
}

__host__ __device__ inline int class_cap(ClassShape c) { return 4 * c.KB * c.NG * (kResBlock / 64); }

// Most members of a team: a quarter of the 512 workgroups that fit the device,
// so that a kernel on each of the process's four hardware queues still has a whole
// team running.
constexpr int kTeamMax = 128;
constexpr int kTeamMembers = 256;
constexpr int kTeamParts = 32768;   // members with room for their partial rows: of a batch slot's teams
constexpr int kSpreadBlocks = 256;  // one workgroup per compute unit

__device__ __forceinline__ int class_of(ClassShape c, int len)
{
    const int K = 4 * c.KB;
    if (len <= K) return (len + 3) / 4;
    int id = c.KB, g = 1;
    while (g < c.NG * (kResBlock / 64) && g * K < len) {
        g *= 2;
        ++id;
    }
    if (g * K >= len) return id;
    return len > kTeamMax * class_cap(c) ? id + 1 : id + 2;
}

// Bucket of a row length > 0, four per octave (longer rows in later buckets).
__host__ __device__ inline int len_bucket(int len)
{
    const int e = 31 - __builtin_clz((unsigned)len);
    return 4 * e + (e >= 2 ? (len >> (e - 2)) & 3 : (len << (2 - e)) & 3);
}

// What the kernels below need of every mode: each is one launch for all modes of a
// plan (blockIdx.y), as a mode's own share is a few microseconds.
struct ModeRows {
    const int32_t* rows;  // [nnz] sorted
    int64_t nrows;
    int32_t *row_ptr, *order, *chunk_begin, *chunk_row, *team_begin, *team_row;
    int* meta;            // class counts, the classes' cursors, pieces; rows and nonzeros per length bucket
};
struct AllModes {
    ModeRows m[CPAPR_MAX_MODES];
    int64_t nnz;
};

// First sorted position of every row (row_ptr[rows] = nnz), by binary search, and
// the counts of the classes and length buckets. A workgroup's last thread finds
// the end of the row before it.
__global__ __launch_bounds__(kBlock) void class_hist_kernel(AllModes a, ClassShape cs)
{
    const int32_t* __restrict__ rows = a.m[blockIdx.y].rows;
    int32_t* __restrict__ row_ptr = a.m[blockIdx.y].row_ptr;
    int* __restrict__ meta = a.m[blockIdx.y].meta;
    const int64_t nrows = a.m[blockIdx.y].nrows;
    __shared__ int h[kRowClasses], hr[kLenBuckets], hn[kLenBuckets], at[kBlock];
    const int t = threadIdx.x;
    if (t < kRowClasses) h[t] = 0;
    if (t < kLenBuckets) hr[t] = hn[t] = 0;
    for (int64_t r0 = blockIdx.x * (int64_t)(kBlock - 1); r0 < nrows; r0 += (int64_t)gridDim.x * (kBlock - 1)) {
        const int64_t r = r0 + t;
        int64_t lo = 0, hi = r <= nrows ? a.nnz : 0;
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            if (rows[mid] < r)
                lo = mid + 1;
            else
                hi = mid;
        }
        __syncthreads();
        at[t] = (int)lo;
        __syncthreads();
        if (r <= nrows && (t < kBlock - 1 || r == nrows)) row_ptr[r] = (int32_t)lo;
        if (t < kBlock - 1 && r < nrows) {
            const int len = at[t + 1] - (int)lo;
            atomicAdd(&h[class_of(cs, len)], 1);
            if (len > 0) {
                atomicAdd(&hr[len_bucket(len)], 1);
                atomicAdd(&hn[len_bucket(len)], len);
            }
        }
    }
    __syncthreads();
    if (t < kRowClasses && h[t]) atomicAdd(&meta[t], h[t]);
    if (t < kLenBuckets && hr[t]) {
        atomicAdd(&meta[64 + t], hr[t]);
        atomicAdd(&meta[64 + kLenBuckets + t], hn[t]);
    }
}

// Counting sort of the rows by class. meta: class counts, then the classes'
// cursors (zero before). A workgroup reserves its share of every class at
// once; the order inside a class does not matter to any row's result.
__global__ __launch_bounds__(kBlock) void class_scatter_kernel(AllModes a, ClassShape cs)
{
    const int32_t* __restrict__ row_ptr = a.m[blockIdx.y].row_ptr;
    int32_t* __restrict__ order = a.m[blockIdx.y].order;
    int* __restrict__ meta = a.m[blockIdx.y].meta;
    const int64_t nrows = a.m[blockIdx.y].nrows;
    __shared__ int h[kRowClasses], base[kRowClasses];
    for (int64_t r0 = blockIdx.x * (int64_t)kBlock; r0 < nrows; r0 += (int64_t)gridDim.x * kBlock) {
        if (threadIdx.x < kRowClasses) h[threadIdx.x] = 0;
        __syncthreads();
        const int64_t r = r0 + threadIdx.x;
        int id = -1, k = 0;
        if (r < nrows) {
            id = class_of(cs, row_ptr[r + 1] - row_ptr[r]);
            k = atomicAdd(&h[id], 1);
        }
        __syncthreads();
        if (threadIdx.x < kRowClasses) {
            int b = 0;
            for (int i = 0; i < (int)threadIdx.x; ++i) b += meta[i];
            if (h[threadIdx.x]) b += atomicAdd(&meta[kRowClasses + threadIdx.x], h[threadIdx.x]);
            base[threadIdx.x] = b;
        }
        __syncthreads();
        if (id >= 0) order[base[id] + k] = (int32_t)r;
        __syncthreads();
    }
}

// Rows of one class cut into pieces of at most `piece` nonzeros: the prefix of
// their counts (begin), the piece -> row map and the total. Block 0 of a mode: the
// long rows' chunks (and the longest class's share of them), block 1: the team
// rows' members.
struct Pieces {
    int cls, ncls, piece, max_rows, max_pieces;
};

__global__ __launch_bounds__(1024) void pieces_kernel(AllModes all, Pieces heavy, Pieces teams)
{
    const ModeRows& m = all.m[blockIdx.y];
    const int32_t *__restrict__ row_ptr = m.row_ptr, *__restrict__ order = m.order;
    int* __restrict__ meta = m.meta;
    const Pieces a = blockIdx.x == 0 ? heavy : teams;
    int32_t* const out_begin = blockIdx.x == 0 ? m.chunk_begin : m.team_begin;
    int32_t* const out_row = blockIdx.x == 0 ? m.chunk_row : m.team_row;
    __shared__ int scan[1024];
    const int t = threadIdx.x;
    int row0 = 0;
    for (int i = 0; i < a.cls; ++i) row0 += meta[i];
    int nheavy = 0;
    for (int i = 0; i < a.ncls; ++i) nheavy += meta[a.cls + i];
    nheavy = min(nheavy, a.max_rows);
    int run = 0;
    for (int h0 = 0; h0 < nheavy; h0 += 1024) {
        const int h = h0 + t;
        int n = 0;
        if (h < nheavy) {
            const int r = order[row0 + h];
            n = (row_ptr[r + 1] - row_ptr[r] + a.piece - 1) / a.piece;
        }
        scan[t] = n;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int v = t >= o ? scan[t - o] : 0;
            __syncthreads();
            scan[t] += v;
            __syncthreads();
        }
        const int begin = run + scan[t] - n;
        if (h < nheavy) out_begin[h] = begin;
        run += scan[1023];
        // the map: a wave per row
        const int lane = t & 63, w0 = t & ~63;
        for (int k = 0; k < 64; ++k) {
            const int b0 = __shfl(begin, k), nk = __shfl(n, k);
            for (int i = lane; i < nk; i += 64)
                if (b0 + i < a.max_pieces) out_row[b0 + i] = h0 + w0 + k;
        }
        __syncthreads();
    }
    if (t == 0) {
        out_begin[nheavy] = run;
        meta[2 * kRowClasses + blockIdx.x] = run;
        if (blockIdx.x == 0) meta[2 * kRowClasses + 2] = out_begin[min(meta[a.cls], nheavy)];
    }
}

// ---- plan: the long rows' nonzeros by hot and cold ----

// Places of a mode's hot rows: its rows in length buckets >= bucket, in any
// order. max_hot: their number, at most kMaxHot (hot_rows holds no more).
__global__ __launch_bounds__(kBlock) void hot_rows_kernel(const int32_t* __restrict__ row_ptr, int64_t nrows, int bucket,
                                                          int max_hot, int* __restrict__ counter,
                                                          uint16_t* __restrict__ hot_id, int32_t* __restrict__ hot_rows)
{
    for (int64_t r = blockIdx.x * (int64_t)kBlock + threadIdx.x; r < nrows; r += (int64_t)gridDim.x * kBlock) {
        const int len = row_ptr[r + 1] - row_ptr[r];
        uint16_t id = kCold;
        if (len > 0 && len_bucket(len) >= bucket) {
            const int k = atomicAdd(counter, 1);
            if (k < max_hot) {
                id = (uint16_t)k;
                hot_rows[k] = (int32_t)r;
            }
        }
        hot_id[r] = id;
    }
}

struct SplitArgs {
    const int32_t *row_ptr, *rows, *chunk_begin, *chunk_row;
    const uint32_t *lead, *hot, *third;  // the sorted copy's offsets
    const double* vals;
    const uint16_t* hot_id;
    uint32_t *s_lead, *s_hot, *s_third, *s_val;
    int exact32;
    int* hot_before;   // [chunks] hot nonzeros of the chunk, then of the row's chunks before it
    int* row_hot;      // [long rows] hot nonzeros
    int chunk;
    int piece;
    int R;
};

__device__ __forceinline__ void chunk_range(const SplitArgs& a, int ch, int* h, uint32_t* p0, uint32_t* p1)
{
    *h = a.chunk_row[ch];
    const int row = a.rows[*h];
    *p0 = (uint32_t)a.row_ptr[row] + (uint32_t)((ch - a.chunk_begin[*h]) * a.chunk);
    *p1 = min(*p0 + (uint32_t)a.chunk, (uint32_t)a.row_ptr[row + 1]);
}

__global__ __launch_bounds__(kBlock) void split_count_kernel(SplitArgs a)
{
    __shared__ int sum;
    int h;
    uint32_t p0, p1;
    chunk_range(a, blockIdx.x, &h, &p0, &p1);
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    int n = 0;
    for (uint32_t p = p0 + threadIdx.x; p < p1; p += kBlock) n += a.hot_id[a.hot[p] / (uint32_t)a.R] != kCold;
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if ((threadIdx.x & 63) == 0) atomicAdd(&sum, n);
    __syncthreads();
    if (threadIdx.x == 0) a.hot_before[blockIdx.x] = sum;
}

// A wave per long row: exclusive prefix of its chunks' hot counts.
__global__ __launch_bounds__(64) void split_scan_kernel(SplitArgs a)
{
    const int h = blockIdx.x, lane = threadIdx.x;
    const int c0 = a.chunk_begin[h], c1 = a.chunk_begin[h + 1];
    int run = 0;
    for (int c = c0; c < c1; c += 64) {
        const int v = c + lane < c1 ? a.hot_before[c + lane] : 0;
        int incl = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (c + lane < c1) a.hot_before[c + lane] = run + incl - v;
        run += __shfl(incl, 63);
    }
    if (lane == 0) a.row_hot[h] = run;
}

// Stable partition of a chunk's nonzeros into its row's hot and cold parts.
__global__ __launch_bounds__(kBlock) void split_scatter_kernel(SplitArgs a)
{
    __shared__ int wsum[kBlock / 64];
    int h;
    uint32_t p0, p1;
    chunk_range(a, blockIdx.x, &h, &p0, &p1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t start = (uint32_t)a.row_ptr[a.rows[h]];
    uint32_t hot_at = start + (uint32_t)a.hot_before[blockIdx.x];
    uint32_t cold_at = start + (uint32_t)a.row_hot[h] + (p0 - start) - (uint32_t)a.hot_before[blockIdx.x];
    for (uint32_t base = p0; base < p1; base += kBlock) {
        const uint32_t p = base + threadIdx.x;
        const bool in = p < p1;
        uint32_t off = 0;
        uint16_t id = kCold;
        if (in) {
            off = a.hot[p];
            id = a.hot_id[off / (uint32_t)a.R];
        }
        const bool ishot = id != kCold;
        const unsigned long long m = __ballot(ishot);
        const int below = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wsum[wave] = __popcll(m);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            if (w < wave) before += wsum[w];
            total += wsum[w];
        }
        before += below;
        if (in) {
            const uint32_t to = ishot ? hot_at + before : cold_at + (threadIdx.x - before);
            a.s_lead[to] = a.lead[p];
            if (ishot)
                ((uint16_t*)a.s_hot)[start + to] = id;
            else
                a.s_hot[to] = off;
            if (a.third != nullptr) a.s_third[to] = a.third[p];
            a.s_val[to] = a.exact32 ? __float_as_uint((float)a.vals[p]) : p;
        }
        const uint32_t n = min((uint32_t)kBlock, p1 - base);
        hot_at += total;
        cold_at += n - total;
        __syncthreads();
    }
}

// Inclusive scan over 1024 threads; *total receives the sum.
__device__ __forceinline__ int block_scan(int v, int* wsum, int* total)
{
    const int t = threadIdx.x, lane = t & 63;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[t >> 6] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < (t >> 6)) before += wsum[w];
        all += wsum[w];
    }
    __syncthreads();
    *total = all;
    return incl + before;
}

// Place of piece i of a part of np pieces of long row h among kPlaces: its
// position in the part, or (fewer pieces than dies) turned by the row.
constexpr int kPlaces = 256;
static_assert(kPlaces % kXcds == 0, "whole places per die");
__device__ __forceinline__ int piece_place(int i, int np, int h)
{
    const int at = (int)(((2 * (int64_t)i + 1) * kPlaces) / (2 * (int64_t)np));
    return np >= kXcds ? at : (at + 53 * h) % kPlaces;
}

// Pieces of the long rows' hot and cold parts (row by row), and their lists by
// die, in the order of their places (pass 0 counts the places' pieces, pass 1
// lists them).
__global__ __launch_bounds__(1024) void entries_kernel(SplitArgs a, int nlong, int max_entries, int4* __restrict__ entry,
                                                       int32_t* __restrict__ entry_begin, int32_t* __restrict__ xlist,
                                                       int32_t* __restrict__ xbegin)
{
    struct Row {
        int begin, n, nh;
        uint32_t p0, pm, p1;
    };
    __shared__ Row sh[1024];
    __shared__ int wsum[16], place_n[kPlaces], place_at[kPlaces], many[1024], nmany;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t < kPlaces) place_n[t] = 0;
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        int run = 0;
        for (int h0 = 0; h0 < nlong; h0 += 1024) {
            const int h = h0 + t;
            int n = 0, nh = 0;
            uint32_t p0 = 0, pm = 0, p1 = 0;
            if (h < nlong) {
                const int r = a.rows[h];
                p0 = (uint32_t)a.row_ptr[r];
                p1 = (uint32_t)a.row_ptr[r + 1];
                pm = p0 + (uint32_t)a.row_hot[h];
                nh = (int)((pm - p0 + a.piece - 1) / a.piece);
                n = nh + (int)((p1 - pm + a.piece - 1) / a.piece);
            }
            int all;
            const int begin = run + block_scan(n, wsum, &all) - n;
            if (h < nlong && pass == 0) entry_begin[h] = min(begin, max_entries);
            run += all;
            sh[t] = {begin, n, nh, p0, pm, p1};
            if (t == 0) nmany = 0;
            __syncthreads();
            if (n > 512) many[atomicAdd(&nmany, 1)] = t;
            __syncthreads();
            // Rows of many pieces by all waves, one row after the other, then a wave per row.
            const int rows = min(1024, nlong - h0), nm = nmany;
            for (int r = 0; r < nm + (rows - wave + 15) / 16; ++r) {
                const bool all16 = r < nm;
                const int k = all16 ? many[r] : wave + 16 * (r - nm);
                if (!all16 && sh[k].n > 512) continue;
                const int first = all16 ? wave * 64 : 0, step = all16 ? 1024 : 64;
                const int b0 = sh[k].begin, nk = min(sh[k].n, max_entries - b0), nhk = sh[k].nh, hk = h0 + k;
                const uint32_t q0 = sh[k].p0, qm = sh[k].pm, q1 = sh[k].p1;
                for (int i0 = first; i0 < nk; i0 += step) {
                    const int i = i0 + lane;
                    const bool in = i < nk, hot = i < nhk;
                    const int ip = hot ? i : i - nhk;
                    const int d = in ? piece_place(ip, hot ? nhk : sh[k].n - nhk, hk) : -1;
                    // neighbours of one place are counted together
                    const int prev = __shfl_up(d, 1);
                    const unsigned long long starts = __ballot(lane == 0 || d != prev);
                    const int lead = 63 - __clzll(starts & (~0ull >> (63 - lane)));
                    const unsigned long long after = lead < 63 ? starts >> (lead + 1) : 0ull;
                    const int len = after ? __ffsll(after) : 64 - lead;
                    int at = 0;
                    if (in && lane == lead) at = atomicAdd(pass == 0 ? &place_n[d] : &place_at[d], len);
                    at = __shfl(at, lead) + lane - lead;
                    if (!in) continue;
                    if (pass == 0) {
                        const uint32_t lo = (hot ? q0 : qm) + (uint32_t)(ip * a.piece);
                        entry[b0 + i] =
                            make_int4(hk, (int)lo, (int)min(lo + (uint32_t)a.piece, hot ? qm : q1), hot ? (int)q0 + 1 : 0);
                    } else if (at < max_entries) {
                        xlist[at] = b0 + i;
                    }
                }
            }
            __syncthreads();
        }
        __syncthreads();
        if (pass == 0 && t == 0) {
            entry_begin[nlong] = min(run, max_entries);
            int at = 0;
            for (int d = 0; d < kPlaces; ++d) {
                if (d % (kPlaces / kXcds) == 0) xbegin[d / (kPlaces / kXcds)] = at;
                place_at[d] = at;
                at += place_n[d];
            }
            xbegin[kXcds] = at;
        }
        __syncthreads();
    }
}

// Launch shape of the resident rows by rank: lanes per row and columns per
// lane so that few lanes idle, and as many nonzeros per lane group as leave the
// pi rows within 160 of a lane's 256 registers.
struct Shape {
    int G, C, K;
};

bool row_shape(int R, Shape* s)
{
    if (R <= 4)
        *s = {4, 1, 32};
    else if (R <= 8)
        *s = {4, 2, 32};
    else if (R <= 12)
        *s = {4, 3, 24};
    else if (R <= 16)
        *s = {4, 4, 20};
    else if (R <= 24)
        *s = {8, 3, 24};
    else if (R <= 32)
        *s = {8, 4, 20};
    else if (R <= 48)
        *s = {16, 3, 24};
    else if (R <= 64)
        *s = {16, 4, 20};
    else
        return false;
    return true;
}

template <typename F>
Error by_row_shape(const Shape& s, F&& f)
{
    using std::integral_constant;
#define CPAPR_ROW(GG, CC, KK)                   if (s.G == GG && s.C == CC)                     return f(integral_constant<int, GG>{}, integral_constant<int, CC>{}, integral_constant<int, KK>{});
    CPAPR_ROW(4, 1, 32)
    CPAPR_ROW(4, 2, 32)
    CPAPR_ROW(4, 3, 24)
    CPAPR_ROW(4, 4, 20)
    CPAPR_ROW(8, 3, 24)
    CPAPR_ROW(8, 4, 20)
    CPAPR_ROW(16, 3, 24)
    CPAPR_ROW(16, 4, 20)
#undef CPAPR_ROW
    return {CPAPR_EUNSUPPORTED, "no resident-row kernel for this rank"};
}

ClassShape class_shape(const Shape& s) { return {s.K / 4, 64 / s.G}; }

// Heavy rows' shape: the Phi kernel's lanes per nonzero (wider gathers), at
// columns per lane that fit the rank.
Shape heavy_shape(int R, bool mixed)
{
    if (R <= 4) return {4, 1, 0};
    if (R <= 8) return {8, 1, 0};
    if (R <= 16) return {4, 4, 0};
    if (R <= 24) return {8, 3, 0};
    if (R <= 32) return mixed ? Shape{8, 4, 0} : Shape{16, 2, 0};
    if (R <= 48) return {16, 3, 0};
    return {16, 4, 0};
}

template <bool MIXED, typename F>
Error by_heavy_shape(const Shape& s, F&& f)
{
    using std::integral_constant;
#define CPAPR_HVY(GG, CC)     if (s.G == GG && s.C == CC) return f(integral_constant<int, GG>{}, integral_constant<int, CC>{});
    CPAPR_HVY(4, 1)
    CPAPR_HVY(8, 1)
    CPAPR_HVY(4, 4)
    CPAPR_HVY(8, 3)
    if constexpr (MIXED) {
        CPAPR_HVY(8, 4)
    } else {
        CPAPR_HVY(16, 2)
    }
    CPAPR_HVY(16, 3)
    CPAPR_HVY(16, 4)
#undef CPAPR_HVY
    return {CPAPR_EUNSUPPORTED, "no heavy-row kernel for this rank"};
}

}  // namespace

// Nonzeros per heavy chunk: ~1000 chunks for a small tensor, 2048 for a large one.
int heavy_chunk(int64_t nnz)
{
    int c = 256;
    while (c < 2048 && (int64_t)c * 2 * 1024 <= nnz) c *= 2;
    return c;
}

namespace {

// Bounds on the rows longer than a workgroup's registers, the chunks of the
// heavy ones and the members of the teams.
int64_t max_long(int64_t nnz, const Shape& s) { return nnz / (class_cap(class_shape(s)) + 1); }
int64_t max_chunks(int64_t nnz, const Shape& s)
{
    return nnz / heavy_chunk(nnz) + max_long(nnz, s);
}
// Nonzeros a wave of hot_kernel takes at a time: about eight pieces per wave,
// so that the last round of pieces is a small part of the launch.
int hot_piece(int64_t nnz)
{
    int c = 256;
    while (c < 4096 && (int64_t)c * 2 * 32768 <= nnz) c *= 2;
    return c;
}
int64_t max_entries(int64_t nnz, const Shape& s) { return nnz / hot_piece(nnz) + 2 * max_long(nnz, s); }
int64_t max_partials(int64_t nnz, const Shape& s) { return std::max(max_chunks(nnz, s), max_entries(nnz, s)); }

// Tensors whose long rows may be split by hot rows: three- and four-way ones of
// at least 2^20 nonzeros (below, the launches weigh more than the gathers) and at
// most 2^28 (the split takes 12 and 16 bytes per nonzero and mode, 17 GB there).
bool hot_supported(int N, int64_t nnz, int R)
{
    Shape s;
    return (N == 3 || N == 4) && nnz >= (1 << 20) && nnz <= (1 << 28) && row_shape(R, &s);
}
constexpr int64_t kScheduled = int64_t(1) << 20;  // nonzeros from which chunks follow the last loop

int64_t max_members(int64_t nnz, const Shape& s) { return nnz / class_cap(class_shape(s)) + max_long(nnz, s); }

// Doubles of the long rows' history (tol > 0). A single loop keeps one iteration of
// its heavy rows, or, where it runs teams, kInnerChunk iterations of theirs (at
// most kTeamMembers / 2 rows: a team has two members or more) and one of the rows
// too long for a team. In a batch all long rows are teams: kInnerChunk iterations
// of theirs while that is no more than a double per nonzero and 64 MiB, else the
// batch takes shorter chunks (R = 64, every row just longer than a workgroup's
// registers: one iteration takes 3.2 bytes per nonzero).
int64_t hist_doubles(int64_t nnz, const Shape& s, int R)
{
    const int64_t nl = max_long(nnz, s), row = 2 * (int64_t)R;
    const int64_t longest = nnz / ((int64_t)kTeamMax * class_cap(class_shape(s)) + 1);
    const int64_t single = std::max(nl * row, (longest + std::min<int64_t>(nl, kTeamMembers / 2) * kInnerChunk) * row);
    return std::max(single, std::min({nl * row * kInnerChunk, nnz, int64_t(1) << 23}));
}

}  // namespace

// Up to 2^30 nonzeros: positions are 32-bit with room for a step past the end. The
// structures below lie where the plan's sort had its temporaries (44 bytes per
// nonzero), so that a plan takes, beyond one without them, 8 bytes per row of every
// mode and at most 0.065 bytes per nonzero and mode, except with three modes and R = 64
// below 2^23 nonzeros (up to 14) and with four modes and 2^20 to 2^28 nonzeros: 16 to
// 28 by rank (R = 32: 23 at 20M), up to 42 below 2^23 (R = 64).
bool rows_supported(int R, int64_t nnz)
{
    Shape s;
    return nnz <= (int64_t(1) << 30) && row_shape(R, &s);
}

size_t rows_mode_bind(RowPlan* r, char* base, int64_t nnz, int64_t dim, int R)
{
    Shape s;
    if (!row_shape(R, &s)) return 0;
    size_t at = 0;
    auto take = [&](int64_t n) {
        char* q = base != nullptr ? base + at : nullptr;
        at += align256((size_t)n * 4);
        return (int32_t*)q;
    };
    RowPlan o{};
    o.row_ptr = take(dim + 1);
    o.order = take(dim);
    o.chunk_begin = take(max_long(nnz, s) + 1);
    o.chunk_row = take(max_chunks(nnz, s) + 1);
    o.team_begin = take(max_long(nnz, s) + 1);
    o.team_row = take(max_members(nnz, s) + 1);
    if (r != nullptr) *r = o;
    return at;
}

size_t rows_state_bind(RowState* r, char* base, int64_t nnz, int64_t maxI, int R, bool stops)
{
    Shape s;
    if (!row_shape(R, &s)) return 0;
    const int64_t nl = max_long(nnz, s);
    size_t at = 0;
    auto take = [&](int64_t bytes) {
        char* q = base != nullptr ? base + at : nullptr;
        at += align256((size_t)bytes);
        return q;
    };
    RowState o{};
    o.partial = (double*)take(max_partials(nnz, s) * R * 8);
    o.team_part = (double*)take(3 * std::min<int64_t>(max_members(nnz, s), kTeamParts) * R * 8);
    o.tickets = (1 + 2 * nl + 1 + kInnerSlots) * kCountStride;
    o.ticket = (unsigned int*)take(o.tickets * 4);
    o.finished = o.ticket + (1 + 2 * nl) * kCountStride;
    o.split = (int*)take((max_chunks(nnz, s) + nl + CPAPR_MAX_MODES) * 4);
    o.hot_tab = (double*)take(kHotLds);
    if (stops) {
        o.B0 = (double*)take(maxI * R * 8);
        if (nnz >= kScheduled) o.B1 = (double*)take(maxI * R * 8);
        o.hist_n = hist_doubles(nnz, s, R);
        o.hist = (double*)take(o.hist_n * 8);
    }
    if (r != nullptr) *r = o;
    return at;
}

size_t rows_hot_bind(cpapr_plan* P, char* base, int N, int64_t nnz, const int64_t* dims, int R)
{
    if (!hot_supported(N, nnz, R)) return 0;
    Shape s;
    row_shape(R, &s);
    size_t at = 0;
    auto take = [&](int64_t bytes) {
        char* q = base != nullptr ? base + at : nullptr;
        at += align256((size_t)bytes);
        return q;
    };
    for (int n = 0; n < N; ++n) {
        uint32_t* lead = (uint32_t*)take(nnz * 4);
        uint32_t* hot = (uint32_t*)take(nnz * 4);
        uint32_t* third = N == 4 ? (uint32_t*)take(nnz * 4) : nullptr;
        uint32_t* val = (uint32_t*)take(nnz * 4);
        int32_t* xlist = (int32_t*)take((max_entries(nnz, s) + 1) * 4);
        int32_t* xbegin = (int32_t*)take((kXcds + 1) * 4);
        int4* entry = (int4*)take((max_entries(nnz, s) + 1) * 16);
        int32_t* begin = (int32_t*)take((max_long(nnz, s) + 1) * 4);
        uint16_t* id = (uint16_t*)take(dims[n] * 2);
        int32_t* rows = (int32_t*)take((int64_t)kMaxHot * 4);
        if (P != nullptr) {
            RowPlan& r = P->mode[n].rp;
            r.s_lead = lead;
            r.s_hot = hot;
            r.s_third = third;
            r.s_val = val;
            r.xlist = xlist;
            r.xbegin = xbegin;
            r.entry = entry;
            r.entry_begin = begin;
            r.hot_id = id;
            r.hot_rows = rows;
        }
    }
    return at;
}

Error rows_hot_choose(cpapr_plan* P)
{
    int dev = 0;
    CPAPR_HIP(hipGetDevice(&dev));
    CPAPR_HIP(hipDeviceGetAttribute(&P->rs.cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (P->params.method != CPAPR_METHOD_MU || !hot_supported(P->N, P->nnz, P->R)) return {CPAPR_OK, ""};
    const int word = P->params.precision == CPAPR_MIXED ? 4 : 8;
    const int fit = std::min(kHotLds / (P->R * word), kMaxHot);
    // every mode's hot rows: as many of its longest length buckets as fit
    double share[CPAPR_MAX_MODES];
    for (int m = 0; m < P->N; ++m) {
        RowPlan& r = P->mode[m].rp;
        r.bucket = kLenBuckets;
        r.nhot = 0;
        int64_t mass = 0;
        while (r.bucket > 0 && r.nhot + r.rows_in[r.bucket - 1] <= fit) {
            --r.bucket;
            r.nhot += r.rows_in[r.bucket];
            mass += r.nnz_in[r.bucket];
        }
        share[m] = (double)mass / (double)P->nnz;
    }
    for (int n = 0; n < P->N; ++n) {
        RowPlan& r = P->mode[n].rp;
        if (r.use_teams || r.nchunks_all == 0) continue;
        int lead = -1, hot = -1;
        for (int m = 0; m < P->N; ++m)
            if (m != n && (lead < 0 || P->dims[m] > P->dims[lead])) lead = m;
        for (int m = 0; m < P->N; ++m)
            if (m != n && m != lead && (hot < 0 || share[m] > share[hot])) hot = m;
        if (share[hot] < 0.25) continue;
        // Two gathered factors beside the table's and four columns per lane do not fit
        // hot_kernel's 128 registers (85 to 96 spilled): 4-way 5M Zipf nonzeros, 401
        // rows, ten iterations, R = 16 / 32 mixed / 64: 1.66 / 1.86 / 1.48 times the Phi
        // launches' time.
        if (P->N == 4 && heavy_shape(P->R, word == 4).C == 4) continue;
        r.lead = lead;
        r.hot = hot;
        r.third = -1;
        for (int m = 0; m < P->N; ++m)
            if (m != n && m != lead && m != hot) r.third = m;
    }
    return {CPAPR_OK, ""};
}

// The split of mode n, before its first inner loop (the caller holds the plan's
// row buffers): programs that run no inner loop of a mode pay nothing for it.
static Error rows_hot_make(cpapr_plan* P, int n, hipStream_t s)
{
    Shape sh;
    row_shape(P->R, &sh);
    const int ncls = class_count(class_shape(sh));
    RowPlan& r = P->mode[n].rp;
    RowPlan& rh = P->mode[r.hot].rp;
    Error e{CPAPR_OK, ""};
    if (!rh.hot_made) {
        e = launch_fill((double*)P->rs.split, 1, 0.0, nullptr, s);
        if (e.code) return e;
        hot_rows_kernel<<<(unsigned)std::min<int64_t>(cdiv(P->dims[r.hot], kBlock), 1024), kBlock, 0, s>>>(
            rh.row_ptr, P->dims[r.hot], rh.bucket, rh.nhot, P->rs.split, rh.hot_id, rh.hot_rows);
        CPAPR_LAUNCHED();
        rh.hot_made = true;
    }
    int first = 0;
    for (int i = 0; i < ncls - 2; ++i) first += r.count[i];
    SplitArgs a{};
    a.row_ptr = r.row_ptr;
    a.rows = r.order + first;
    a.chunk_begin = r.chunk_begin;
    a.chunk_row = r.chunk_row;
    for (int m = 0, k = 0; m < P->N; ++m) {
        if (m == n) continue;
        const uint32_t* c = P->mode[n].cofs + (int64_t)k++ * P->nnz;
        (m == r.lead ? a.lead : m == r.hot ? a.hot : a.third) = c;
    }
    a.vals = P->mode[n].vals;
    a.hot_id = rh.hot_id;
    a.s_lead = r.s_lead;
    a.s_hot = r.s_hot;
    a.s_third = r.s_third;
    a.s_val = r.s_val;
    a.exact32 = P->exact32 ? 1 : 0;
    a.hot_before = P->rs.split + CPAPR_MAX_MODES;
    a.row_hot = a.hot_before + max_chunks(P->nnz, sh);
    a.chunk = heavy_chunk(P->nnz);
    a.piece = hot_piece(P->nnz);
    a.R = P->R;
    split_count_kernel<<<r.nchunks_all, kBlock, 0, s>>>(a);
    CPAPR_LAUNCHED();
    split_scan_kernel<<<r.nlong, 64, 0, s>>>(a);
    CPAPR_LAUNCHED();
    split_scatter_kernel<<<r.nchunks_all, kBlock, 0, s>>>(a);
    CPAPR_LAUNCHED();
    entries_kernel<<<1, 1024, 0, s>>>(a, r.nlong, (int)max_entries(P->nnz, sh), r.entry, r.entry_begin,
                                       r.xlist, r.xbegin);
    CPAPR_LAUNCHED();
    auto allow = [&](auto M) -> Error {  // more than 64 KB of LDS is asked for
        constexpr bool MX = decltype(M)::value;
        return by_heavy_shape<MX>(heavy_shape(P->R, MX), [&](auto G, auto C) -> Error {
            constexpr int GG = decltype(G)::value, CC = decltype(C)::value;
            const void* f = P->exact32 ? (const void*)hot_kernel<GG, CC, false, MX, true>
                                       : (const void*)hot_kernel<GG, CC, false, MX, false>;
            if constexpr (CC < 4)
                if (r.third >= 0)
                    f = P->exact32 ? (const void*)hot_kernel<GG, CC, true, MX, true>
                                   : (const void*)hot_kernel<GG, CC, true, MX, false>;
            CPAPR_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kHotLds));
            return {CPAPR_OK, ""};
        });
    };
    e = P->params.precision == CPAPR_MIXED ? allow(std::true_type{}) : allow(std::false_type{});
    if (e.code) return e;
    r.split_made = true;
    return {CPAPR_OK, ""};
}

// Every mode's rows by class, from its sorted copy. meta: kRowMeta zeroed ints per
// mode on the device; rows_finish takes their host copy.
Error rows_build(const cpapr_plan* P, int* meta, hipStream_t s)
{
    Shape sh;
    if (!row_shape(P->R, &sh)) return {CPAPR_OK, ""};
    const ClassShape cs = class_shape(sh);
    AllModes a{};
    a.nnz = P->nnz;
    int64_t most = 0;
    for (int n = 0; n < P->N; ++n) {
        const RowPlan& r = P->mode[n].rp;
        a.m[n] = {P->mode[n].rows, P->dims[n], r.row_ptr, r.order, r.chunk_begin, r.chunk_row, r.team_begin, r.team_row,
                  meta + n * kRowMeta};
        most = std::max(most, P->dims[n]);
    }
    const dim3 grid((unsigned)std::min<int64_t>(cdiv(most, kBlock - 1), 2048), P->N);
    class_hist_kernel<<<grid, kBlock, 0, s>>>(a, cs);
    CPAPR_LAUNCHED();
    class_scatter_kernel<<<dim3(std::min(grid.x, 1024u), P->N), kBlock, 0, s>>>(a, cs);
    CPAPR_LAUNCHED();
    if (max_long(P->nnz, sh) > 0) {
        const int n = class_count(cs), nl = (int)max_long(P->nnz, sh);
        const Pieces heavy{n - 2, 2, heavy_chunk(P->nnz), nl, (int)max_chunks(P->nnz, sh)};
        const Pieces teams{n - 1, 1, class_cap(cs), nl, (int)max_members(P->nnz, sh)};
        pieces_kernel<<<dim3(2, P->N), 1024, 0, s>>>(a, heavy, teams);
        CPAPR_LAUNCHED();
    }
    return {CPAPR_OK, ""};
}

void rows_finish(cpapr_plan* P, int mode, const int* meta)
{
    Shape sh;
    if (!row_shape(P->R, &sh)) return;
    RowPlan& r = P->mode[mode].rp;
    const int n = class_count(class_shape(sh));
    for (int i = 0; i < kRowClasses; ++i) r.count[i] = i < n ? meta[i] : 0;
    r.nlong = r.count[n - 2] + r.count[n - 1];
    r.nchunks_all = meta[2 * kRowClasses];
    r.nmembers = meta[2 * kRowClasses + 1];
    // Teams where all their members fit the device at once (half of its 512
    // workgroups, the light rows beside them): then an iteration costs one
    // meeting instead of a launch (600k nonzeros: 92 us per inner loop of ten against
    // 195). With more members than that the heavy kernels are faster.
    r.use_teams = r.nmembers > 0 && r.nmembers <= kTeamMembers;
    r.nchunks = r.use_teams ? meta[2 * kRowClasses + 2] : r.nchunks_all;
    for (int i = 0; i < kLenBuckets; ++i) {
        r.rows_in[i] = meta[64 + i];
        r.nnz_in[i] = meta[64 + kLenBuckets + i];
    }
    // rows longer than a workgroup's registers (teams: than all members'), by length
    // bucket (one starts at either bound; rows of just that length count as longer)
    const int cap = class_cap(class_shape(sh)) * (r.use_teams ? kTeamMax : 1);
    int64_t longer = 0;
    for (int i = len_bucket(cap); i < kLenBuckets; ++i) longer += r.nnz_in[i];
    r.resident = P->nnz > 0 ? 1.0 - (double)longer / (double)P->nnz : 1.0;
    r.hot = -1;
    P->mode[mode].segments = P->dims[mode] - r.count[0];
}

namespace {

// Operands of the resident rows of one mode (without its flags).
void res_args(const cpapr_plan* P, int mode, double* B, const void* const* fac, double* Phi, bool teams, int max_spread,
              ResArgs* out, int ng = 0)
{
    Shape sh;
    row_shape(P->R, &sh);
    const ClassShape cs = class_shape(sh);
    const PlanMode& pm = P->mode[mode];
    const RowPlan& r = pm.rp;
    const int NG = ng > 0 ? ng : cs.NG, W = kResBlock / 64;  // ng: lane groups per wave of another launch
    ResArgs a{};
    a.cofs = pm.cofs;
    a.vals = pm.vals;
    a.row_ptr = r.row_ptr;
    a.order = r.order;
    a.B = B;
    a.Phi = Phi;
    a.nnz = P->nnz;
    a.eps = P->params.eps;
    a.R = P->R;
    a.NM1 = P->N - 1;
    a.tol = P->params.tol;
    a.each = P->params.tol > 0.0 ? 1 : 0;
    int j = 0;
    for (int m = 0; m < P->N; ++m)
        if (m != mode) a.fac[j++] = fac[m];
    // classes in launch order: the longest rows first
    const int ncls = class_count(cs), nlight = ncls - 2;
    int begin[kRowClasses] = {}, at = 0;
    for (int i = 0; i < ncls; ++i) {
        begin[i] = at;
        at += r.count[i];
    }
    // A tensor too small to fill the device spreads its rows over more lane
    // groups (fewer nonzeros per group one after the other), up to `spread` times.
    int64_t blocks = 0;
    auto list = [&](int spread) {
        blocks = 0;
        a.nentries = 0;
        for (int i = nlight - 1; i >= 0; --i) {
            if (r.count[i] == 0) continue;
            const int nb = i <= cs.KB ? i : cs.KB;  // blocks of four nonzeros per lane group
            int S = std::min(i <= cs.KB ? 1 : 1 << (i - cs.KB), W * NG);
            for (int f = 1; f < spread && f < nb && S < W * NG; f *= 2) S *= 2;
            const int per = std::max(1, W * NG / S);  // rows per workgroup
            a.entry[a.nentries++] = {(int32_t)blocks, begin[i], r.count[i], S};
            blocks += cdiv(r.count[i], per);  // < 2^31 rows
        }
    };
    int spread = 1;
    while (spread < max_spread) {
        list(2 * spread);
        if (blocks > kSpreadBlocks) break;
        spread *= 2;
    }
    list(spread);
    a.light_blocks = (int)blocks;
    a.heavy0 = begin[nlight];
    a.team0 = r.count[nlight];
    a.nheavy = r.count[nlight] + r.count[nlight + 1];
    a.team_blocks = teams ? r.nmembers : 0;
    a.teams = teams ? r.count[nlight + 1] : 0;
    a.team_begin = r.team_begin;
    a.team_row = r.team_row;
    a.team_part = P->rs.team_part;
    a.team_ticket = P->rs.ticket;
    a.team_count = P->rs.ticket + kCountStride;
    a.team_wait = P->team_wait;
    a.heavy_hist = P->rs.hist;
    a.hist = P->rs.hist + 2 * (int64_t)(a.nheavy - a.teams) * P->R;
    a.B0 = a.each ? P->rs.B0 : nullptr;
    a.B1 = a.each ? P->rs.B1 : nullptr;
    *out = a;
}

}  // namespace

// ---- line search of the row solves ----

namespace {

struct LsArgs {
    ResArgs r;  // sorted copy, rows by class, factors
    const double* D;
    const int32_t* live;
    double* T;
    const int* skip;
    const int32_t *chunk_begin, *chunk_row;
    double* partial;  // [chunks x 4]
    int chunk, nchunks;
};

// Four trial steps delta_k = max(b + alpha_k d, 0) - b, alpha = 1, 1/2, 1/4, 1/8
// of every live row: sums over its nonzeros of x log1p(dm_k / m), m = b . pi,
// dm_k = delta_k . pi (see delta_ratio in phi.hip for the cases at the floor).
// A row belongs to its lane groups alone, so b and the trial steps are formed
// once and four nonzeros go through the five dot products together, each
// reduce-scattered over the quad: a lane ends with all five of one nonzero. The
// group's quads share the four trials, so every lane takes 16 / G logarithms
// for the block instead of a fifth of the all-reduces and the quotients of
// every nonzero in every lane (the same sums by the Phi tile code: 1545 us on
// 20M nonzeros at R = 16).
template <int G, int C, int NM1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(C >= 3 ? 3 : 4))) void ls_rows_kernel(LsArgs a)
{
    constexpr int NG = 64 / G, W = kBlock / 64;
    constexpr int NQ = G / 4;                       // quads per lane group
    constexpr int TPQ = NQ >= 4 ? 1 : 4 / NQ;       // trials per quad
    __shared__ double red[W][4];
    if (*a.skip) return;
    const ResArgs& r = a.r;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int gl = lane % G, g = lane / G, qi = gl / 4;
    const int R = r.R;
    const bool odd1 = lane & 1, odd2 = lane & 2;
    const int q = (lane & 3) ^ (G >= 8 && (lane & 4) ? 3 : 0);
    int row, S, sub, WR;
    uint32_t p0, p1;
    bool valid = true;
    const bool heavy = (int)blockIdx.x < a.nchunks;
    if (heavy) {
        const int h = a.chunk_row[blockIdx.x];
        row = r.order[r.heavy0 + h];
        p0 = (uint32_t)r.row_ptr[row] + (uint32_t)(((int)blockIdx.x - a.chunk_begin[h]) * a.chunk);
        p1 = min(p0 + (uint32_t)a.chunk, (uint32_t)r.row_ptr[row + 1]);
        S = W * NG;
        WR = W;
        sub = wave * NG + g;
    } else {
        const int at = (int)blockIdx.x - a.nchunks;
        int e = 0;
        while (e + 1 < r.nentries && at >= r.entry[e + 1].block0) ++e;
        const int row0 = r.entry[e].row0, count = r.entry[e].count;
        S = r.entry[e].groups;
        WR = S > NG ? S / NG : 1;
        const int local = at - r.entry[e].block0;
        int pos;
        if (WR > 1) {
            pos = local * (W / WR) + wave / WR;
            sub = (wave % WR) * NG + g;
        } else {
            pos = (local * W + wave) * (NG / S) + g / S;
            sub = g % S;
        }
        valid = pos < count;
        row = r.order[row0 + (valid ? pos : count - 1)];
        p0 = (uint32_t)r.row_ptr[row];
        p1 = (uint32_t)r.row_ptr[row + 1];
    }
    valid = valid && a.live[row] == 1;
    if (!valid) p1 = p0;
    const int colbase = min(gl * C, R - C);
    double b[C], dk[4][C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const bool own = colbase + c >= gl * C && colbase + c < R;
        const int64_t e = (int64_t)row * R + colbase + c;
        b[c] = own && valid ? r.B[e] : 0.0;
        const double d = own && valid ? a.D[e] : 0.0;
        double alpha = 1.0;
#pragma unroll
        for (int k = 0; k < 4; ++k, alpha *= 0.5) {
            const double nb = b[c] + alpha * d;
            dk[k][c] = (nb > 0.0 ? nb : 0.0) - b[c];
        }
    }
    // dot products of the four nonzeros with u, the lane's nonzero's total
    auto dots = [&](const double (&pi)[4][C], const double (&u)[C]) {
        double d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = u[0] * pi[j][0];
#pragma unroll
            for (int c = 1; c < C; ++c) d[j] = __builtin_fma(u[c], pi[j][c], d[j]);
        }
        const double a0 = (odd1 ? d[1] : d[0]) + dpp_f64<0xB1>(odd1 ? d[0] : d[1]);
        const double a1 = (odd1 ? d[3] : d[2]) + dpp_f64<0xB1>(odd1 ? d[2] : d[3]);
        double m = (odd2 ? a1 : a0) + dpp_f64<0x4E>(odd2 ? a0 : a1);
        if constexpr (G >= 8) m += dpp_f64<0x141>(m);
        if constexpr (G >= 16) m += dpp_f64<0x140>(m);
        return m;
    };
    double sum[TPQ];
#pragma unroll
    for (int k = 0; k < TPQ; ++k) sum[k] = 0.0;
    constexpr int NOFF = NM1 > 0 ? NM1 : 1;
    uint32_t off[NOFF];
    double x = 0.0;
    auto load_meta = [&](uint32_t base) {
        const uint32_t p = base + (uint32_t)q, pc = min(p, p1 - 1);
        x = r.vals[pc];
        if (p >= p1) x = 0.0;
#pragma unroll
        for (int m = 0; m < NOFF; ++m) off[m] = r.cofs[(int64_t)m * r.nnz + pc];
    };
    const uint32_t step = (uint32_t)S * 4u;
    uint32_t base = p0 + (uint32_t)sub * 4u;
    if (base < p1) load_meta(base);
    for (; base < p1; base += step) {
        const double xc = x;
        double pi[4][C];
        const double* fac = (const double*)r.fac[0];
        load_cols<C>(fac, quad_bcast<0>(off[0]), colbase, pi[0]);
        load_cols<C>(fac, quad_bcast<1>(off[0]), colbase, pi[1]);
        load_cols<C>(fac, quad_bcast<2>(off[0]), colbase, pi[2]);
        load_cols<C>(fac, quad_bcast<3>(off[0]), colbase, pi[3]);
        const int nm1 = NM1 > 0 ? NM1 : r.NM1;
#pragma unroll
        for (int m = 1; m < nm1; ++m) {
            uint32_t o;
            if constexpr (NM1 > 0)
                o = off[m];
            else
                o = r.cofs[(int64_t)m * r.nnz + min(base + (uint32_t)q, p1 - 1)];
            const double* f2 = (const double*)r.fac[m];
            double f[4][C];
            load_cols<C>(f2, quad_bcast<0>(o), colbase, f[0]);
            load_cols<C>(f2, quad_bcast<1>(o), colbase, f[1]);
            load_cols<C>(f2, quad_bcast<2>(o), colbase, f[2]);
            load_cols<C>(f2, quad_bcast<3>(o), colbase, f[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[j][c] *= f[j][c];
        }
        const bool there = base + (uint32_t)q < p1;
        if (base + step < p1) load_meta(base + step);
        const double m = dots(pi, b);
        double dm[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) dm[k] = dots(pi, dk[k]);
#pragma unroll
        for (int k = 0; k < TPQ; ++k) {
            double d;
            if constexpr (NQ == 1)
                d = dm[k];
            else if constexpr (NQ == 2)
                d = qi ? dm[2 + k] : dm[k];
            else
                d = qi & 2 ? (qi & 1 ? dm[3] : dm[2]) : (qi & 1 ? dm[1] : dm[0]);
            const double m1 = m + d;
            double term;
            if (m > r.eps && m1 > r.eps)
                term = xc * log1p(div_pos(d, m));
            else
                term = m > r.eps ? -__builtin_inf() : xc * (log(m1 > r.eps ? m1 : r.eps) - log(r.eps));
            sum[k] += there ? term : 0.0;
        }
    }
    // the quad's nonzeros, the row's other lane groups, its other waves
#pragma unroll
    for (int k = 0; k < TPQ; ++k) {
        sum[k] += dpp_f64<0xB1>(sum[k]);
        sum[k] += dpp_f64<0x4E>(sum[k]);
#pragma unroll
        for (int o = G; o < 64; o <<= 1)
            if (o < G * S) sum[k] += __shfl_xor(sum[k], o);
    }
    if (WR > 1) {
        if (g == 0 && (gl & 3) == 0)
#pragma unroll
            for (int k = 0; k < TPQ; ++k)
                if (qi * TPQ + k < 4) red[wave][qi * TPQ + k] = sum[k];
        __syncthreads();
        const int w0 = wave / WR * WR;
        if (sub / NG == 0 && lane < 4) {
            double v = 0.0;
            for (int w = 0; w < WR; ++w) v += red[w0 + w][lane];
            if (heavy)
                a.partial[(int64_t)blockIdx.x * 4 + lane] = v;
            else if (valid)
                a.T[(int64_t)row * R + lane] = v;
        }
        return;
    }
    if (valid && sub == 0 && (gl & 3) == 0)
#pragma unroll
        for (int k = 0; k < TPQ; ++k) a.T[(int64_t)row * R + qi * TPQ + k] = sum[k];
}

// Long rows: the sums of their chunks, a wave per row.
__global__ __launch_bounds__(64) void ls_fold_kernel(LsArgs a)
{
    if (*a.skip) return;
    const int h = blockIdx.x, lane = threadIdx.x, k = lane & 3;
    const int row = a.r.order[a.r.heavy0 + h];
    const int c0 = a.chunk_begin[h], c1 = a.chunk_begin[h + 1];
    double v = 0.0;
#pragma unroll 8
    for (int c = c0 + lane / 4; c < c1; c += 16) v += a.partial[(int64_t)c * 4 + k];
    for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o);
    if (lane < 4 && a.live[row] == 1) a.T[(int64_t)row * a.r.R + lane] = v;
}

}  // namespace

Error launch_delta4_rows(const cpapr_plan* P, int mode, const double* B, const double* D, const int32_t* live,
                         const void* const* fac, double eps, double* out, const int* skip, hipStream_t s)
{
    const RowPlan& rp = P->mode[mode].rp;
    LsArgs a{};
    // few columns per lane: a lane holds five vectors of them beside the pi rows
    const Shape sh = P->R > 8 && P->R <= 16 ? Shape{8, 2, 0} : heavy_shape(P->R, false);
    res_args(P, mode, const_cast<double*>(B), fac, nullptr, false, 8, &a.r, 64 / sh.G);
    a.r.eps = eps;
    a.D = D;
    a.live = live;
    a.T = out;
    a.skip = skip;
    a.chunk_begin = rp.chunk_begin;
    a.chunk_row = rp.chunk_row;
    a.partial = P->rs.partial;
    a.chunk = heavy_chunk(P->nnz);
    a.nchunks = rp.nchunks_all;
    const int64_t blocks = (int64_t)a.nchunks + a.r.light_blocks;
    if (blocks == 0) return {CPAPR_OK, ""};
    if (blocks > 0x7fffffff) return {CPAPR_EUNSUPPORTED, "too many rows"};
    const dim3 grid((unsigned)blocks);
    auto launch = [&](auto G, auto C) -> Error {
        constexpr int GG = decltype(G)::value, CC = decltype(C)::value;
        switch (a.r.NM1) {
            case 1: ls_rows_kernel<GG, CC, 1><<<grid, kBlock, 0, s>>>(a); break;
            case 2: ls_rows_kernel<GG, CC, 2><<<grid, kBlock, 0, s>>>(a); break;
            case 3: ls_rows_kernel<GG, CC, 3><<<grid, kBlock, 0, s>>>(a); break;
            default: ls_rows_kernel<GG, CC, 0><<<grid, kBlock, 0, s>>>(a); break;
        }
        CPAPR_LAUNCHED();
        return {CPAPR_OK, ""};
    };
    using std::integral_constant;
    Error e = sh.G == 8 && sh.C == 2 ? launch(integral_constant<int, 8>{}, integral_constant<int, 2>{})
                                       : by_heavy_shape<false>(sh, launch);
    if (e.code || a.nchunks == 0) return e;
    ls_fold_kernel<<<rp.nlong, 64, 0, s>>>(a);
    CPAPR_LAUNCHED();
    return {CPAPR_OK, ""};
}

// ---- log-likelihood ----

namespace {

constexpr int kSumParts = 128;  // column-sum workgroups per factor

struct LoglikArgs {
    const int32_t* rows;
    const uint32_t* cofs;
    const double* vals;
    const double* fac[CPAPR_MAX_MODES];  // mode 0's factor, then the others'
    const double* all[CPAPR_MAX_MODES];  // every mode's factor, for the column sums
    int64_t dims[CPAPR_MAX_MODES];
    const double* lam;
    double* part;     // [term workgroups] sums of terms
    double* sums;     // [N x parts x R] column sums
    int64_t nnz;
    double eps;
    int R, N;
    int parts;        // column-sum workgroups per factor
    int per;          // nonzeros per wave
};

// x log(max(m, eps)) over the nonzeros of mode 0's copy, m = sum_r lambda_r
// prod_m A(m)[i_m, r]: four nonzeros per lane group, their sums
// reduce-scattered over the quad as in block4, so that a lane takes one
// logarithm for the four (an all-reduce with the logarithm in every lane
// spent 150 us on 5M three-way nonzeros at R = 16, Phi on the same tensor 85).
// While all nonzeros of a step lie in one row, that row is loaded once. The
// first workgroups sum the factors' columns.
template <int G, int C, int NM1>
__global__ __launch_bounds__(kBlock) void loglik_kernel(LoglikArgs a)
{
    constexpr int W = kBlock / 64;
    constexpr uint32_t STEP = 4 * (64 / G);
    __shared__ double sh[kBlock];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int R = a.R;
    if ((int)blockIdx.x < a.N * a.parts) {
        const int m = (int)blockIdx.x / a.parts, part = (int)blockIdx.x % a.parts;
        const int64_t per = (a.dims[m] + a.parts - 1) / a.parts;
        const int64_t r0 = part * per, r1 = min(r0 + per, a.dims[m]);
        const int Q = kBlock / R, c = t % R, q = t / R;
        double s = 0.0;
        if (q < Q) {
#pragma unroll 8
            for (int64_t i = r0 + q; i < r1; i += Q) s += a.all[m][i * R + c];
        }
        sh[t] = q < Q ? s : 0.0;
        __syncthreads();
        if (t < R) {
            double tot = 0.0;
            for (int k = 0; k < Q; ++k) tot += sh[k * R + t];
            a.sums[((int64_t)m * a.parts + part) * R + t] = tot;
        }
        return;
    }
    const int blk = (int)blockIdx.x - a.N * a.parts;
    const int gl = lane % G, g = lane / G;
    const int64_t p0 = ((int64_t)blk * W + wave) * a.per;
    const uint32_t w0 = (uint32_t)min(p0, a.nnz), w1 = (uint32_t)min(p0 + a.per, a.nnz);
    const int colbase = min(gl * C, R - C);
    const bool odd1 = lane & 1, odd2 = lane & 2;
    const int q = (lane & 3) ^ (G >= 8 && (lane & 4) ? 3 : 0);
    double lam[C];
#pragma unroll
    for (int c = 0; c < C; ++c) lam[c] = colbase + c >= gl * C && colbase + c < R ? a.lam[colbase + c] : 0.0;
    uint32_t off[NM1 > 0 ? NM1 : 1];
    uint32_t row = 0;
    double x = 0.0;
    auto load_meta = [&](uint32_t base) {
        const uint32_t p = base + (uint32_t)(g * 4 + q), pc = min(p, w1 - 1);
        x = a.vals[pc];
        if (p >= w1) x = 0.0;
        row = (uint32_t)a.rows[pc] * (uint32_t)R;
        if constexpr (NM1 > 0)
#pragma unroll
            for (int m = 0; m < NM1; ++m) off[m] = a.cofs[(int64_t)m * a.nnz + pc];
    };
    double ll = 0.0;
    if (w0 < w1) load_meta(w0);
    for (uint32_t base = w0; base < w1; base += STEP) {
        const double xc = x;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)row);
        const bool one = __ballot(row != first) == 0ull;
        double pi[4][C], f[4][C];
        auto times = [&](const double* fac, uint32_t o) {
            load_cols<C>(fac, quad_bcast<0>(o), colbase, f[0]);
            load_cols<C>(fac, quad_bcast<1>(o), colbase, f[1]);
            load_cols<C>(fac, quad_bcast<2>(o), colbase, f[2]);
            load_cols<C>(fac, quad_bcast<3>(o), colbase, f[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[j][c] *= f[j][c];
        };
        if (one) {
            load_cols<C>(a.fac[0], first, colbase, f[0]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[j][c] = f[0][c] * lam[c];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c) pi[j][c] = lam[c];
            times(a.fac[0], row);
        }
        if constexpr (NM1 > 0) {
#pragma unroll
            for (int m = 0; m < NM1; ++m) times(a.fac[1 + m], off[m]);
        } else {
            const uint32_t pc = min(base + (uint32_t)(g * 4 + q), w1 - 1);
            for (int m = 0; m < a.N - 1; ++m) times(a.fac[1 + m], a.cofs[(int64_t)m * a.nnz + pc]);
        }
        if (base + STEP < w1) load_meta(base + STEP);
        double d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = pi[j][0];
#pragma unroll
            for (int c = 1; c < C; ++c) d[j] += pi[j][c];
        }
        const double a0 = (odd1 ? d[1] : d[0]) + dpp_f64<0xB1>(odd1 ? d[0] : d[1]);
        const double a1 = (odd1 ? d[3] : d[2]) + dpp_f64<0xB1>(odd1 ? d[2] : d[3]);
        double m = (odd2 ? a1 : a0) + dpp_f64<0x4E>(odd2 ? a0 : a1);
        if constexpr (G >= 8) m += dpp_f64<0x141>(m);
        if constexpr (G >= 16) m += dpp_f64<0x140>(m);
        ll += xc * log(__builtin_fmax(m, a.eps));
    }
    if (gl >= 4) ll = 0.0;  // the group's other quads hold the same nonzeros
    for (int o = 32; o > 0; o >>= 1) ll += __shfl_xor(ll, o);
    if (lane == 0) sh[wave] = ll;
    __syncthreads();
    if (t == 0) a.part[blk] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Terms minus the model's mass sum_r lambda_r prod_m (column sums).
__global__ __launch_bounds__(1024) void loglik_sum_kernel(const double* __restrict__ part, int nparts,
                                                          const double* __restrict__ sums, int sum_parts,
                                                          const double* __restrict__ lam, int N, int R, DevState* st)
{
    __shared__ double sh[1024];
    __shared__ double mass[CPAPR_MAX_MODES * 64];
    const int t = threadIdx.x;
    // the columns of all factors, 1024 / (N R) threads each
    const int cols = N * R, Q = max(1, 1024 / cols);
    for (int c0 = 0; c0 < cols; c0 += 1024) {
        const int c = c0 + t % min(cols, 1024), q = t / min(cols, 1024);
        double s = 0.0;
        if (q < Q && c < cols) {
            const double* src = sums + (int64_t)(c / R) * sum_parts * R + c % R;
#pragma unroll 4
            for (int k = q; k < sum_parts; k += Q) s += src[(int64_t)k * R];
        }
        sh[t] = s;
        __syncthreads();
        if (q == 0 && c < cols) {
            double tot = 0.0;
            for (int k = 0; k < Q; ++k) tot += sh[k * min(cols, 1024) + t];
            mass[c] = tot;
        }
        __syncthreads();
    }
    double v = 0.0;
#pragma unroll 4
    for (int k = t; k < nparts; k += 1024) v += part[k];
    if (t < R) {
        double p = lam[t];
        for (int m = 0; m < N; ++m) p *= mass[m * R + t];
        v -= p;
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += sh[w];
        st->ll = s;
    }
}

}  // namespace

bool loglik_fused_supported(int R) { return R <= 64; }

Error launch_loglik_fused(const cpapr_plan* P, const double* lam, const double* const* A, double eps, hipStream_t s)
{
    LoglikArgs a{};
    a.rows = P->mode[0].rows;
    a.cofs = P->mode[0].cofs;
    a.vals = P->mode[0].vals;
    for (int m = 0; m < P->N; ++m) {
        a.fac[m] = a.all[m] = A[m];
        a.dims[m] = P->dims[m];
    }
    a.lam = lam;
    a.part = P->llpart;
    a.sums = P->partial;
    a.nnz = P->nnz;
    a.eps = eps;
    a.R = P->R;
    a.N = P->N;
    a.parts = std::min(kSumParts, kPartials / P->N);
    // 128 nonzeros per wave (512 per partial sum) at least; about 4096 waves
    int64_t per = 128;
    while (per < 2048 && per * 2 * 4096 <= P->nnz) per *= 2;
    a.per = (int)per;
    const int64_t blocks = cdiv(P->nnz, per * (kBlock / 64));
    const dim3 grid((unsigned)(blocks + (int64_t)a.N * a.parts));
    // four columns instead of three at R = 33 .. 48 as rank_columns has it
    const Shape sh = P->R > 32 && P->R <= 48 && (P->N == 3 || P->N == 4) ? Shape{16, 4, 0} : heavy_shape(P->R, false);
    Error e = by_heavy_shape<false>(sh, [&](auto G, auto C) -> Error {
        constexpr int GG = decltype(G)::value, CC = decltype(C)::value;
        switch (P->N) {
            case 2: loglik_kernel<GG, CC, 1><<<grid, kBlock, 0, s>>>(a); break;
            case 3: loglik_kernel<GG, CC, 2><<<grid, kBlock, 0, s>>>(a); break;
            case 4: loglik_kernel<GG, CC, 3><<<grid, kBlock, 0, s>>>(a); break;
            case 5: loglik_kernel<GG, CC, 4><<<grid, kBlock, 0, s>>>(a); break;
            default: loglik_kernel<GG, CC, 0><<<grid, kBlock, 0, s>>>(a); break;
        }
        CPAPR_LAUNCHED();
        return {CPAPR_OK, ""};
    });
    if (e.code) return e;
    loglik_sum_kernel<<<1, 1024, 0, s>>>(P->llpart, (int)blocks, P->partial, a.parts, lam, P->N, P->R, P->state);
    CPAPR_LAUNCHED();
    return {CPAPR_OK, ""};
}

// A batch slot can run row by row when its plan's single inner loop could, no row
// is longer than the largest team, and the teams' partial rows have room.
int rows_batch_shape(const cpapr_plan* P, int mode)
{
    Shape sh;
    if (!P->by_rows || P->params.method != CPAPR_METHOD_MU || !P->shape_auto ||
        P->params.variant != CPAPR_VARIANT_AUTO || !row_shape(P->R, &sh)) return -1;
    if (P->mode[mode].rp.count[class_count(class_shape(sh)) - 2] > 0 || P->mode[mode].rp.nmembers > kTeamParts) return -1;
    const int mixed = P->params.precision == CPAPR_MIXED ? 1 : 0;
    return 2 * (P->R <= 16 ? (P->R - 1) / 4 : P->R <= 32 ? 4 + (P->R - 17) / 8 : 6 + (P->R - 33) / 16) + mixed;
}

int rows_batch_chunk(const cpapr_plan* P, int mode)
{
    const int64_t per = 2 * (int64_t)P->mode[mode].rp.nlong * P->R;
    if (!(P->params.tol > 0.0) || per == 0) return kInnerChunk;
    return (int)std::max<int64_t>(1, std::min<int64_t>(kInnerChunk, P->rs.hist_n / per));
}

size_t rows_batch_item_bytes() { return sizeof(ResArgs); }

void rows_batch_item(const cpapr_plan* P, int mode, const double* B, const void* const* fac, double* Phi, int slot,
                     const int32_t* done, int32_t* rerun, unsigned long long* iv, void* out, int* light, int* again,
                     int* members)
{
    ResArgs a;
    res_args(P, mode, const_cast<double*>(B), fac, Phi, true, 1, &a);  // the batch fills the device
    a.slot = slot;
    a.done = done;
    a.rerun = rerun;
    a.iv = iv;
    a.iv_slots = kBatchInnerSlots;
    *light = a.light_blocks;
    *again = a.light_blocks + (int)cdiv((int64_t)a.nheavy * P->R, kResBlock);
    *members = a.team_blocks;
    std::memcpy(out, &a, sizeof(a));
}

Error launch_rows_batch(int shape, const RowsBatch& b, int n_it, bool again, hipStream_t s)
{
    const Shape shapes[kRowShapes / 2] = {{4, 1, 32}, {4, 2, 32}, {4, 3, 24}, {4, 4, 20},
                                          {8, 3, 24}, {8, 4, 20}, {16, 3, 24}, {16, 4, 20}};
    return by_row_shape(shapes[shape / 2], [&](auto G, auto C, auto K) -> Error {
        constexpr int GG = decltype(G)::value, CC = decltype(C)::value, KK = decltype(K)::value;
        const ResArgs* items = (const ResArgs*)b.items;
        const unsigned grid = (unsigned)(again ? b.nagain : b.nlight + b.nmembers);
        if (grid == 0) return {CPAPR_OK, ""};
        if (again && shape % 2)
            batch_rerun_kernel<GG, CC, KK, true><<<grid, kResBlock, 0, s>>>(items, b.again, b.n, n_it);
        else if (again)
            batch_rerun_kernel<GG, CC, KK, false><<<grid, kResBlock, 0, s>>>(items, b.again, b.n, n_it);
        else if (shape % 2)
            batch_resident_kernel<GG, CC, KK, true><<<grid, kResBlock, 0, s>>>(items, b.light, b.members, b.n, b.nlight,
                                                                              b.nmembers, b.ticket, n_it);
        else
            batch_resident_kernel<GG, CC, KK, false><<<grid, kResBlock, 0, s>>>(items, b.light, b.members, b.n, b.nlight,
                                                                               b.nmembers, b.ticket, n_it);
        CPAPR_LAUNCHED();
        return {CPAPR_OK, ""};
    });
}

Error launch_rows_batch_decide(const void* items, int n, BatchState st, int32_t* rerun, int n_it, unsigned int* tickets,
                               hipStream_t s)
{
    batch_decide_kernel<<<(unsigned)n, kBlock, 0, s>>>((const ResArgs*)items, st, rerun, n_it, tickets);
    CPAPR_LAUNCHED();
    return {CPAPR_OK, ""};
}

// What light rows compute past a stop is lost, and after a stop before the chunk's
// last iteration they gather again. From 2^20 nonzeros on, where that outweighs a
// launch or two, the first chunk is as long as the mode's last loop of this plan ran
// (the modes of a solve stop early in sweep after sweep once they have
// converged). Only the schedule depends on it, not the results.
// 8M uniform three-way nonzeros, R = 32, lmax = 10, stops at the first / second /
// sixth iteration: one chunk of all 1393 / 1395 / 1558 us, the Phi launches alone
// 443 / 659 / 1544, this 291 / 553 / 778; without a stop 1010 / 2427 / 1026. 20M
// nonzeros, Zipf rows, R = 16, stop at the first: 1905 / 471 / 381 (heavy rows ran
// all ten iterations).
static bool schedule_by_last(const cpapr_plan* P)
{
    return P->params.tol > 0.0 && P->nnz >= kScheduled;
}

// A loop that is expected to stop at its first iteration, or of which nothing is
// known yet, takes that one by the Phi launches, as one iteration alone does.
bool rows_first_alone(const cpapr_plan* P, int mode) { return schedule_by_last(P) && P->expect[mode] <= 1; }

static int first_chunk(const cpapr_plan* P, int mode, int lmax)
{
    const int e = P->expect[mode];
    return !schedule_by_last(P) || e <= 1 || e >= lmax ? inner_step(lmax) : std::min(e, kInnerChunk);
}

namespace {

// What an iteration of a mode's heavy rows takes, in units of the Phi launches'
// time for the same nonzeros: both gather every factor row again. Measured at 300k,
// 1.1M, 5M and 20M nonzeros, R = 8 .. 64, both precisions, uniform and Zipf(1.1)
// coordinates, modes of 53 to 40,003 rows:
//  * two modes: 0.55 to 1.1, rows of a few hundred nonzeros 1.2 to 1.5;
//  * split by hot rows, three modes: 0.6 to 0.9, above R = 32 to 1.06 at 5M;
//    four modes: 0.75 to 0.95 up to R = 32 at 20M, 0.9 to 1.1 below, 0.9 to 1.19 above;
//  * else, three modes: 0.8 to 1.0 up to 1.1M, from there 0.92 to 1.34, rows of up
//    to 1,000 nonzeros to 2.7;
//  * four modes: 0.86 to 1.0 at 300k, to 1.3 at 1.1M, 0.85 to 1.25 above, with four
//    columns per lane and FP32-stored factors to 1.6, short rows to 2.0;
//  * more modes: 0.7 to 1.0 at 300k, to 1.2 at 1.1M, 0.8 to 1.66 above, but R > 48 in
//    FP64 with long rows 0.7 to 1.0.
double heavy_cost(const cpapr_plan* P, const RowPlan& r)
{
    const int N = P->N, R = P->R;
    const bool mixed = P->params.precision == CPAPR_MIXED;
    const bool middle = P->nnz >= (int64_t(1) << 20), large = P->nnz >= (int64_t(1) << 21);
    const bool huge = P->nnz >= (int64_t(1) << 23);
    const bool brief = (1.0 - r.resident) * (double)P->nnz < 2048.0 * r.nlong;
    if (N == 2) return brief && huge ? 1.3 : 0.9;
    if (r.hot >= 0 && N == 3) return R <= 32 ? 0.85 : huge ? 0.95 : 1.02;
    if (r.hot >= 0) return R > 32 ? 1.1 : huge || (R <= 8 && !mixed) ? 0.95 : 1.05;
    if (!middle) return 0.95;
    if (N == 3) return !large ? 0.95 : brief ? 2.0 : 1.2;
    if (N == 4) return !large ? (mixed ? 1.3 : 1.1) : brief || (mixed && heavy_shape(R, true).C == 4) ? 1.6 : 1.25;
    return R <= 48 || mixed || brief ? 1.4 : large ? 0.95 : 1.05;
}

}  // namespace

// Row by row or by the Phi launches: resident nonzeros gather once per loop, at about
// the cost of one Phi, and then take about a tenth of it per iteration (8M uniform
// nonzeros, R = 32: 394 us for the first, Phi 224, and 70 for each further one);
// with FP32-stored factors at R > 24 the gather costs over two of that Phi once the
// factors' rows come from memory (20M nonzeros, lmax = 2: 1.13 to 1.2 times the Phi
// launches).
bool rows_pay(const cpapr_plan* P, int mode)
{
    const RowPlan& r = P->mode[mode].rp;
    const bool mixed = P->params.precision == CPAPR_MIXED;
    const double gather = mixed && P->R > 24 && P->nnz >= (int64_t(1) << 22) ? 2.2 : 1.0;
    const double resident = 0.1 + gather / P->params.lmax;
    return r.resident * resident + (1.0 - r.resident) * heavy_cost(P, r) <= 1.0;
}

Error enqueue_inner_rows(cpapr_plan* P, int mode, double* B, const void* const* fac, double* Phi, int lmax,
                         hipStream_t s)
{
    Shape sh;
    if (!row_shape(P->R, &sh)) return {CPAPR_EUNSUPPORTED, "no resident-row kernel for this rank"};
    const PlanMode& pm = P->mode[mode];
    const RowPlan& r = pm.rp;
    const bool mixed = P->params.precision == CPAPR_MIXED;
    const bool each = P->params.tol > 0.0;
    const int ncls = class_count(class_shape(sh)), nlight = ncls - 2;
    ResArgs a;
    res_args(P, mode, B, fac, Phi, r.use_teams, 8, &a);
    a.done = &P->state->done;
    a.rerun = &P->state->rerun;
    a.iv = &P->state->iv[0][0];
    a.iv_slots = kInnerSlots;
    const int64_t blocks = a.light_blocks;
    if (blocks + a.team_blocks > 0x7fffffff) return {CPAPR_EUNSUPPORTED, "too many rows"};

    HeavyArgs h{};
    h.vals = pm.vals;
    h.row_ptr = r.row_ptr;
    h.rows = r.order + a.heavy0;
    h.chunk_begin = r.chunk_begin;
    h.chunk_row = r.chunk_row;
    // the mode the rows are ordered by (the largest other one, the first on ties) leads
    int lead = 0, k = 0;
    int64_t most = -1;
    for (int m = 0; m < P->N; ++m)
        if (m != mode) {
            if (P->dims[m] > most) {
                most = P->dims[m];
                lead = k;
            }
            ++k;
        }
    for (int m = 0, at1 = 1; m < P->N - 1; ++m) {
        const int to = m == lead ? 0 : at1++;
        h.fac[to] = a.fac[m];
        h.cofs[to] = pm.cofs + (int64_t)m * P->nnz;
    }
    h.B = B;
    h.Phi = Phi;
    h.partial = P->rs.partial;
    h.ticket = P->rs.ticket + (1 + r.count[nlight + 1]) * kCountStride;
    h.st = P->state;
    h.hist = each ? a.heavy_hist : nullptr;
    h.finished = P->rs.finished;
    h.nrows = a.nheavy - a.teams;
    h.tol = P->params.tol;
    h.nnz = P->nnz;
    h.eps = P->params.eps;
    h.R = P->R;
    h.NM1 = P->N - 1;
    h.chunk = heavy_chunk(P->nnz);

    prof_begin(mode, s);  // one record for all iterations
    int n = each ? first_chunk(P, mode, lmax) : lmax;
    for (int l0 = 0; l0 < lmax; l0 += n, n = inner_step(lmax - l0)) {
        Error e{CPAPR_OK, ""};
        a.n_it = n;
        auto light = [&](bool rerun) {
            return by_row_shape(sh, [&](auto G, auto C, auto K) -> Error {
                constexpr int GG = decltype(G)::value, CC = decltype(C)::value, KK = decltype(K)::value;
                if (rerun) {
                    const dim3 grid((unsigned)(blocks + cdiv((int64_t)a.nheavy * P->R, kResBlock)));
                    if (mixed)
                        rerun_kernel<GG, CC, KK, true><<<grid, kResBlock, 0, s>>>(a);
                    else
                        rerun_kernel<GG, CC, KK, false><<<grid, kResBlock, 0, s>>>(a);
                } else if (mixed) {
                    resident_kernel<GG, CC, KK, true><<<(unsigned)(blocks + a.team_blocks), kResBlock, 0, s>>>(a);
                } else {
                    resident_kernel<GG, CC, KK, false><<<(unsigned)(blocks + a.team_blocks), kResBlock, 0, s>>>(a);
                }
                CPAPR_LAUNCHED();
                return {CPAPR_OK, ""};
            });
        };
        if (blocks + a.team_blocks > 0) e = light(false);
        if (e.code) return e;
        if (r.nchunks > 0 && r.hot >= 0) {
            if (!r.split_made) e = rows_hot_make(P, mode, s);
            if (e.code) return e;
            HotArgs k{};
            k.s_lead = r.s_lead;
            k.s_hot = r.s_hot;
            k.s_third = r.s_third;
            k.s_val = r.s_val;
            k.vals = pm.vals;
            k.entry = r.entry;
            k.xlist = r.xlist;
            k.xbegin = r.xbegin;
            k.rows = h.rows;
            k.tab = (const uint4*)P->rs.hot_tab;
            const int nhot = P->mode[r.hot].rp.nhot;
            k.tab_vecs = (int)cdiv((int64_t)nhot * P->R * (mixed ? 4 : 8), 16);
            k.lead = fac[r.lead];
            k.hot = fac[r.hot];
            k.third = r.third >= 0 ? fac[r.third] : nullptr;
            k.B = B;
            k.partial = h.partial;
            k.st = P->state;
            k.eps = h.eps;
            k.R = P->R;
            HotStep hs{r.entry_begin, h.rows, h.partial, B, Phi, P->state, h.hist, h.finished, h.tol, h.nrows, P->R, -1};
            const size_t lds = (size_t)k.tab_vecs * 16;
            if (l0 == 0) {
                const int32_t* rows = P->mode[r.hot].rp.hot_rows;
                const unsigned tg = (unsigned)cdiv((int64_t)nhot * P->R, kBlock);
                if (mixed)
                    hot_table_kernel<<<tg, kBlock, 0, s>>>((const float*)k.hot, rows, nhot, P->R, (float*)P->rs.hot_tab);
                else
                    hot_table_kernel<<<tg, kBlock, 0, s>>>((const double*)k.hot, rows, nhot, P->R, P->rs.hot_tab);
                CPAPR_LAUNCHED();
            }
            for (int l = 0; l < n; ++l) {
                auto launch = [&](auto M) -> Error {
                    constexpr bool MX = decltype(M)::value;
                    return by_heavy_shape<MX>(heavy_shape(P->R, mixed), [&](auto G, auto C) -> Error {
                        constexpr int GG = decltype(G)::value, CC = decltype(C)::value;
                        if (r.third >= 0) {
                            if constexpr (CC < 4) {
                                if (P->exact32)
                                    hot_kernel<GG, CC, true, MX, true><<<P->rs.cus, kHotThreads, lds, s>>>(k);
                                else
                                    hot_kernel<GG, CC, true, MX, false><<<P->rs.cus, kHotThreads, lds, s>>>(k);
                            } else {
                                return {CPAPR_EUNSUPPORTED, "no split of four modes with four columns per lane"};
                            }
                        } else if (P->exact32)
                            hot_kernel<GG, CC, false, MX, true><<<P->rs.cus, kHotThreads, lds, s>>>(k);
                        else
                            hot_kernel<GG, CC, false, MX, false><<<P->rs.cus, kHotThreads, lds, s>>>(k);
                        CPAPR_LAUNCHED();
                        return {CPAPR_OK, ""};
                    });
                };
                e = mixed ? launch(std::true_type{}) : launch(std::false_type{});
                if (e.code) return e;
                hs.l = each ? l : l + 1 == n ? 0 : -1;
                hot_step_kernel<<<r.nlong, 512, 0, s>>>(hs);
                CPAPR_LAUNCHED();
            }
        } else if (r.nchunks > 0) {
            const Shape hs = heavy_shape(P->R, mixed);
            for (int l = 0; l < n; ++l) {
                h.l = each ? l : l + 1 == n ? 0 : -1;
                auto launch = [&](auto M) -> Error {
                    constexpr bool MX = decltype(M)::value;
                    return by_heavy_shape<MX>(hs, [&](auto G, auto C) -> Error {
                        constexpr int GG = decltype(G)::value, CC = decltype(C)::value;
                        const dim3 grid((unsigned)r.nchunks);
                        switch (h.NM1) {
                            case 1: heavy_kernel<GG, CC, 1, MX><<<grid, kBlock, 0, s>>>(h); break;
                            case 2: heavy_kernel<GG, CC, 2, MX><<<grid, kBlock, 0, s>>>(h); break;
                            case 3: heavy_kernel<GG, CC, 3, MX><<<grid, kBlock, 0, s>>>(h); break;
                            default: heavy_kernel<GG, CC, 0, MX><<<grid, kBlock, 0, s>>>(h); break;
                        }
                        CPAPR_LAUNCHED();
                        return {CPAPR_OK, ""};
                    });
                };
                e = mixed ? launch(std::true_type{}) : launch(std::false_type{});
                if (e.code) return e;
            }
        }
        decide_kernel<<<1, kBlock, 0, s>>>(P->state, mode, n, each ? 1 : 0, P->params.tol, a.team_ticket,
                                          a.team_count, a.teams);
        CPAPR_LAUNCHED();
        if (each) e = light(true);
        if (e.code) return e;
    }
    prof_end(s);
    return {CPAPR_OK, ""};
}

}  // namespace cpapr
