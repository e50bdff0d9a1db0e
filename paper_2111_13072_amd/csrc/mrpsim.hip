// mrpsim: spectral kinetic simulation of the ideal Multipole Resonance Probe
// (Gong, Friedrichs, Oberrath, Brinkmann, arXiv:2111.13072) on one MI355X
// (gfx950).  C ABI declared in include/mrpsim.h.
//
// One time step (Sec. 3 field solver + Sec. 4 pusher) runs as these kernels:
//   sort:    key (r^2, id) -> bucket histogram -> bucket offsets -> scatter
//   moments: exact rank inside each bucket and the permuted SoA copy, then per
//            half tile of 32 radially consecutive particles the sums of
//            q R_lm (regular solid harmonics) and q I_lm (irregular ones)
//   carries: exclusive prefix of the interior sums and exclusive suffix of
//            the exterior sums over groups, totals T_lm, the boundary (image)
//            response, the surface charge, the hemisphere drive and Q_diff
//   field:   per particle, the far field of all other halves from its half's
//            coefficient vector, the near field of its own half pair by pair,
//            the self-image correction and the ion background; then the
//            leapfrog kick/drift, the wall rules and the next step's sort key
//            and bucket slot (the key kernel keys only what the push did not)
// A handle holds one or more independent simulations ("members") that share
// the probe geometry, the truncation l_max and the precision.  Each member
// owns a tile-aligned range of particle slots, a range of carry chunks and a
// range of sort buckets; every kernel maps its tile, chunk or bucket to the
// member through a device table, so one launch of each kernel steps all
// members, and members can be admitted and retired between steps.  A
// member's arithmetic does not depend on the others.  All work is on the
// handle's stream; one step is captured once into a HIP graph and replayed.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <type_traits>
#include <string>
#include <utility>
#include <vector>

#include "mrpsim.h"
#include "tables.h"

namespace {

constexpr double kQ = -1.0;   // electron charge, units of e (Sec. 4)
constexpr double kM = 1.0;    // electron mass, units of m_e
// A particle whose id has this bit set is an ion: charge +1, mass ion_mass.
constexpr uint32_t kIonBit = 0x80000000u;
constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxL = 64;
// A tile (one wave's 64 radially consecutive particles) is two halves of 32:
// the pair sums of the near field run inside a half, and the moments are
// summed per half.  A group is the four tiles of one workgroup of the moments
// and field kernels (256 slots): the carry scan runs over groups, and a
// member's particle slots are whole groups.
constexpr int kHalf = kWave / 2;
constexpr int kTilesPerGroup = kWavesPerBlock;
constexpr int kGroupSlots = kTilesPerGroup * kWave;
// Groups per chunk of the carry scan, per member: a power of two in
// [kChunkMin, kChunkMax], about a member's groups / kChunkTarget, so that small
// members get short serial chains and large ones few chunks.
constexpr int kChunkMin = 8, kChunkMax = 64, kChunkTarget = 256;
constexpr int kScanPerBlock = 1024;  // histogram entries per block of the bucket scan
constexpr int kBucketOccupancy = 8;  // mean particles per sort bucket

thread_local std::string g_last_error;

int fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

// ---------------------------------------------------------------------------
// Device-side structures
// ---------------------------------------------------------------------------

// Sorted state (this step's radial order), one array per component: the
// moments and field kernels read it with unit stride.
struct State {
    double *x, *y, *z, *vx, *vy, *vz;
    uint32_t *uid;
};

// Unsorted state (after the push, in the previous step's order): one 64-byte
// record per particle, so the sort's gather of a particle from its scattered
// source slot is a single cache line.
struct alignas(64) PRec {
    double x, y, z, vx, vy, vz;
    uint32_t uid, pad[3];
};

// Per-member control block in device memory.  A launch takes over next_step as
// its step in its first kernel that does not read step, and sets next_step in
// one that does not read it: no kernel is launched for that alone.
struct Ctl {
    int64_t next_step;  // absolute step of the state held in A
    int64_t step;       // the step being run or evaluated
    uint32_t records;   // records in A (some may be flagged absorbed); kKeyed: the
                        // last push already produced their sort keys, bucket slots
                        // and bucket counts (else the key kernel computes them)
    uint32_t n_live;    // alive particles sorted into B this step
    uint32_t n_dead;    // particles absorbed so far (graveyard fill)
    uint32_t n_dead_ion;  // of which ions
    double q_surface;   // Q_S used by this step's field
};
constexpr uint32_t kKeyed = 0x80000000u;   // a member has fewer than 2^31 particles

// Per-member description (device table, written by the host between steps).
struct Seg {
    uint32_t p0, cap;   // particle slots [p0, p0 + cap); p0 is a multiple of 256
    uint32_t t0, nt;    // tiles [t0, t0 + nt), t0 = p0 / 64
    uint32_t g0, ng;    // groups [g0, g0 + ng), g0 = p0 / 256
    uint32_t c0, nc;    // carry chunks [c0, c0 + nc)
    uint32_t cl;        // groups per chunk
    uint32_t b0, nb;    // sort buckets [b0, b0 + nb)
    double inv_vol;     // 1 / (r_out^3 - 1)
    double ntilde, inv_ntilde, ion_density, q_surface0, dt, r_out;
    uint64_t seed;
    int32_t probe_bc, wall_bc;
    int64_t n_steps;
    const double *u_asy;
    double *qdiff;
    // optional ion profile: densities at ion_k + 1 equally spaced radii from 1
    // to r_out, then the enclosed ion charge at those radii (super-particle units)
    const double *ion_tab;
    double ion_h, ion_inv_h;
    double ion_qm;      // charge / mass of ion particles (+1 / ion_mass)
    int32_t ion_k;
    int32_t near_w;     // particles of a near-field block: 32 (a half tile) or 64 (the tile)
    int32_t used;
    int32_t one_carry;  // the carries in one kernel, without chunks (carry_member)
};

constexpr uint32_t kNone = 0xffffffffu;

// Per-l and per-(l, m) constant tables (filled by fill_tables, read-only after it).
// The super-particle density 1 / ntilde is a per-member factor applied at use.
struct Tables {
    const double *ftil;     // image coefficient f_l, with f_0 = 0 (floating probe)
    const double *wl;       // 1 / (2l+1)
    const double *drive_w;  // c_l b^P_l sqrt(4 pi / (2l+1)) for odd l, else 0
    const double *self_w;   // f_l / (4 pi)
    const double *self_w1;  // (l+1) f_l / (4 pi)
    const double4 *nf4;     // {(2l+1)/(l+1), l/(l+1), 2l+1, l}, one wide load per l
    const int *chl;         // degree l of each channel in stream order
    // per channel: the factor that turns a sum of rescaled harmonics (Qh) into
    // a field coefficient, N_lm^2 / (2l+1) (times 1 / ntilde at use)
    const double *chg;
    // Legendre constants of the full near field, per l: {c_l, l c_l,
    // gamma_{l+1}, (2l+1) c_l}, where P_l = c_l Ph_l and the rescaled
    // polynomials obey Ph_{l+1} = u Ph_l - gamma_{l+1} Ph_{l-1}
    const double4 *lg4;
    // Rescaled harmonic recurrence in stream order of (m, l) (m outer,
    // l = m..L inner, so a loop over (m, l) reads consecutive entries): the
    // moments and the far field use Qh_l^m = Q_l^m / N_lm with Qh_m^m = 1,
    // Qh_l^m = z Qh_{l-1}^m - gamma_lm r^2 Qh_{l-2}^m; entries {gamma_lm,
    // l + 1/2, 0, 0}, one zero entry after the triangle.  The tile sums
    // are sums of Qh; the carries apply N_lm (chn, per channel) twice: once to
    // turn the sums into true moments, once for the field's Qh.
    const double4 *fq4;
    const double *chn;
    // FP32 copies of the field kernel's tables for the FP32-compensated mode
    const float4 *fq4_32;
    // FP32 near field's Legendre recurrence on E_l = l (P_l - P_{l-1}), per l:
    // {1 / (l+1), 0, 2l+1, l+1}
    const float4 *lw4_32;
};

// The moments kernel splits the orders m over the waves of its blocks, in up to
// this many slices (kWavesPerBlock per block of a group).
constexpr int kMaxMSlices = 16;

// Channels are kept in "stream order": m = 0..m_top outer, l = max(m,1)..L
// inner, cos then sin for m > 0.  l = 0 has no channel: its field is Gauss's
// law over the radial order (computed in the field kernel).
struct KParams {
    int L;          // l_max
    int C;          // channels: (L+1)^2 - 1 (full) or L (axisymmetric)
    int C2;         // 2C: interior then exterior
    int SW;         // C2 + 1: group sums also carry the group's total charge
    int HW;         // 4C + 2: a tile's row of H (interior and exterior sums
                    // of the group's other tiles, of its own halves, charges)
    int n_tiles;    // tile capacity (particle slots / 64, a multiple of 4)
    int n_groups;   // n_tiles / 4
    int n_chunks;   // chunk capacity
    int nb;         // bucket capacity
    int n_members;  // member table size
    int field_only; // evaluation without a step: every used member runs
    int fuse_keys;  // the push prepares the next step's sort records
    // moments kernel: slice s of m is [m_slice[s], m_slice[s + 1])
    uint8_t m_slice[kMaxMSlices + 1];
    // field kernel: the same in kWavesPerBlock slices, their ends packed in bytes
    // (an array here, indexed in a loop, would be copied to scratch memory)
    uint32_t f_ends;
};

// Device tables shared by the kernels.
struct Map {
    const Seg *seg;
    Ctl *ctl;
    const uint32_t *tile_member;   // [n_tiles], kNone for free tiles
    const uint32_t *chunk_member;  // [n_chunks], kNone for free chunks
};

// Charge of the immobile ions of a radial profile inside radius r, in
// super-particle units: the density is linear in r on each segment
// [r_j, r_j + h], integrated in closed form in the offset dd = r - r_j.
// (A uniform background enters the field kernel as its field directly.)
__device__ inline double ion_enclosed(const Seg &sg, double r, double r2)
{
    constexpr double kFourPi = 4.0 * 3.14159265358979323846;
    (void)r2;
    const int K = sg.ion_k;
    int j = (int)((r - 1.0) * sg.ion_inv_h);
    j = max(0, min(j, K - 1));
    const double rj = 1.0 + (double)j * sg.ion_h;
    const double dd = r - rj;
    const double nj = sg.ion_tab[j];
    const double beta = (sg.ion_tab[j + 1] - nj) * sg.ion_inv_h;
    const double d2 = dd * dd;
    const double seg = nj * (rj * rj * dd + rj * d2 + d2 * dd / 3.0) +
                       beta * (rj * rj * d2 / 2.0 + 2.0 * rj * d2 * dd / 3.0 + d2 * d2 / 4.0);
    return sg.ion_tab[K + 1 + j] + kFourPi * sg.ntilde * seg;
}

// A member takes part in this launch: it is in use and has steps left (or
// the launch only evaluates the field).
__device__ inline bool runs_step(const Seg &sg, int64_t step, const KParams &kp)
{
    return sg.used && (kp.field_only || step < sg.n_steps);
}
__device__ inline bool member_runs(const Seg &sg, const Ctl &c, const KParams &kp)
{
    return runs_step(sg, c.step, kp);
}

__device__ inline uint32_t uniform_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Blocks are placed on the 8 XCDs round-robin (block b on XCD b % 8), and
// each XCD has its own L2.  Kernels whose neighbouring blocks share cache
// lines renumber their blocks so that every XCD walks one contiguous range.
constexpr uint32_t kXcds = 8;

__device__ inline uint32_t xcd_block(uint32_t b, uint32_t nblocks)
{
    const uint32_t q = nblocks / kXcds, r = nblocks % kXcds;
    const uint32_t x = b % kXcds, k = b / kXcds;
    return x * q + min(x, r) + k;
}

// Read of a table that no kernel writes while it runs, through the constant
// address space: a wave-uniform index then becomes a scalar load through the
// scalar cache even where the kernel stores to global memory in between
// (which keeps the compiler from proving the read invariant).
template <typename T>
__device__ inline T ld_const(const T *p, int i)
{
    return reinterpret_cast<const __attribute__((address_space(4))) T *>(
        reinterpret_cast<uintptr_t>(p))[i];
}


// r^2 as (x*x + y*y) + z*z without contraction: the exact radial sort key.
// (HIP's __dadd_rn and __dmul_rn are plain operators, which the compiler fuses
// where it likes; the pragma keeps every operation rounded by itself.)
__device__ inline double key_r2(double x, double y, double z)
{
#pragma clang fp contract(off)
    return (x * x + y * y) + z * z;
}

// a + b c and a - b c with the product rounded first (the push).
__device__ inline double add_product(double a, double b, double c)
{
#pragma clang fp contract(off)
    return a + b * c;
}
__device__ inline double sub_product(double a, double b, double c)
{
#pragma clang fp contract(off)
    return a - b * c;
}
// a . b, every operation rounded by itself.
__device__ inline double dot3(double ax, double ay, double az, double bx, double by, double bz)
{
#pragma clang fp contract(off)
    return (ax * bx + ay * by) + az * bz;
}

// ---------------------------------------------------------------------------
// Sort: exact order by (r^2, id) through volume-uniform buckets
// ---------------------------------------------------------------------------

// Bucket of a key: a monotone non-decreasing map of r^2 to the member's
// buckets [b0, b0 + nb) by enclosed shell volume.  Every kernel that sorts or
// ranks uses this one expression, without contraction, so they agree bit for bit.
__device__ inline uint32_t bucket_of(double r2, double inv_vol, uint32_t b0, uint32_t nb)
{
#pragma clang fp contract(off)
    const double t = (r2 * sqrt(r2) - 1.0) * inv_vol * (double)nb;
    uint32_t lb;
    if (!(t < (double)(nb - 1))) lb = nb - 1;   // NaN too: its key sorts above every number's
    else if (!(t > 0.0)) lb = 0;
    else lb = (uint32_t)t;
    return b0 + lb;
}

// Sort records: (key, bucket, slot in the bucket) per particle slot, then
// (key, id, source slot) per position in bucket order; one 16-byte access each.
struct alignas(16) KeyRec {
    uint64_t key;
    uint32_t uid, sub;   // sub = kNone: not sorted this step
};
struct alignas(16) OrdRec {
    uint64_t key;
    uint32_t uid, idx;
};

// Orders this wave's LDS accesses at this point: LDS instructions of one wave
// complete in issue order, so rows a wave wrote are visible to its later
// reads without a block barrier; the fences keep the compiler from moving
// LDS accesses across.
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Slot inside bucket b, by the bucket's atomic count; all lanes of the wave call
// it, `on` marks those with a particle.  The lanes of a wave are neighbours in
// radius.  Where a step moves them little (cold plasma, ions, small time
// steps) they land in a few buckets, and their atomics on the few cache lines
// of those counts queue up: then the wave counts in LDS first and adds each
// bucket's count once, neighbouring counts from neighbouring lanes.  1e6
// electrons and ions at dt 0.01: the field and push kernel 130 -> 40 us, the
// key kernel 51 -> 20.  Spread wider than kSlotWindow buckets, the atomics
// already fall on distinct lines.
constexpr uint32_t kSlotWindow = 256;

__device__ inline uint32_t take_slot(int lane, bool on, uint32_t b, uint32_t *hist, uint32_t *cnt)
{
    const uint64_t any = __ballot(on);
    if (!any) return 0;
    const uint32_t mid =
        (uint32_t)__builtin_amdgcn_readlane((int)b, (int)__builtin_ctzll(any));
    const uint32_t base = mid - kSlotWindow / 2, d = b - base;
    if (__ballot(on && d >= kSlotWindow)) return on ? atomicAdd(&hist[b], 1u) : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kSlotWindow; k += kWave) cnt[k + lane] = 0u;
    wave_lds_sync();
    const uint32_t my = on ? atomicAdd(&cnt[d], 1u) : 0u;
    wave_lds_sync();
    uint32_t first[kSlotWindow / kWave];
#pragma unroll
    for (uint32_t k = 0; k < kSlotWindow / kWave; ++k) {
        const uint32_t c = cnt[k * kWave + lane];
        first[k] = c ? atomicAdd(&hist[base + k * kWave + lane], c) : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < kSlotWindow / kWave; ++k) cnt[k * kWave + lane] = first[k];
    wave_lds_sync();
    return on ? my + cnt[d] : 0u;
}

// Key, bucket and slot inside the bucket, over all particle slots.
// Members whose last push already produced this step's records (kKeyed)
// are skipped: the push kernel's tail does the same work for the particles
// it moves, where the field's arithmetic hides the atomics' latency.
__global__ __launch_bounds__(kBlock) void k_sort_key(Map mp, const PRec *A, const uint8_t *dead,
                                                     KeyRec *krec, uint32_t *hist, KParams kp)
{
    __shared__ uint32_t cnt[kWavesPerBlock][kSlotWindow];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t tile = i >> 6;
    if ((int)tile >= kp.n_tiles) return;   // whole waves: i < 64 * n_tiles
    const uint32_t mb = uniform_u32(mp.tile_member[tile]);
    bool live = false;
    double inv_vol = 0.0;
    uint32_t b0 = 0, nb = 1;
    if (mb != kNone) {
        const Seg &sg = mp.seg[mb];
        const Ctl &c = mp.ctl[mb];
        if (runs_step(sg, c.next_step, kp)) {
            const uint32_t records = c.records;
            if (records & kKeyed) return;   // wave-uniform
            live = (i - sg.p0) < records && !dead[i];
            inv_vol = sg.inv_vol;
            b0 = sg.b0;
            nb = sg.nb;
        }
    }
    KeyRec rec{0ull, 0u, kNone};
    uint32_t b = 0;
    if (live) {
        const double r2 = key_r2(A[i].x, A[i].y, A[i].z);
        rec.key = (uint64_t)__double_as_longlong(r2);
        rec.uid = A[i].uid;
        b = bucket_of(r2, inv_vol, b0, nb);
    }
    const uint32_t sub = take_slot(threadIdx.x & 63, live, b, hist, cnt[threadIdx.x >> 6]);
    if (live) rec.sub = sub;
    krec[i] = rec;
}

// Exclusive scan of a u32 array of length n into out[0..n], out[n] = total.
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wsum[kWavesPerBlock];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int k = 0; k < kWavesPerBlock; ++k) {
        if (k < w) off += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// The members take up their next step (by one block of a kernel that does not
// read their step).
__device__ inline void begin_step(const Map &mp, const KParams &kp)
{
    for (int s = threadIdx.x; s < kp.n_members; s += blockDim.x)
        if (mp.seg[s].used) mp.ctl[s].step = mp.ctl[s].next_step;
}

__global__ __launch_bounds__(kBlock) void k_scan_a(Map mp, KParams kp, const uint32_t *in,
                                                   uint32_t *bsum, int n)
{
    if (blockIdx.x == 0) begin_step(mp, kp);
    const int base = blockIdx.x * kScanPerBlock;
    uint32_t s = 0;
    for (int k = threadIdx.x; k < kScanPerBlock; k += kBlock) {
        int i = base + k;
        if (i < n) s += in[i];
    }
    uint32_t tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Offsets of the buckets: each block adds the sums of the blocks before it
// (at most a few thousand, read from L2) to the scan of its own entries.
// The histogram's last reader: it leaves the histogram zeroed for the next
// step (the handle zeroes it once at creation).
__global__ __launch_bounds__(kBlock) void k_scan_c(uint32_t *in, const uint32_t *bsum,
                                                   uint32_t *out, int n)
{
    uint32_t before = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kBlock) before += bsum[k];
    uint32_t carry;
    block_exclusive_scan(before, &carry);
    constexpr int per = kScanPerBlock / kBlock;
    const int base = blockIdx.x * kScanPerBlock + threadIdx.x * per;
    uint32_t v[per];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0u;
        s += v[k];
    }
#pragma unroll
    for (int k = 0; k < per; ++k)
        if (base + k < n) in[base + k] = 0u;
    uint32_t tot;
    uint32_t run = carry + block_exclusive_scan(s, &tot);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
        if (base + k == n - 1) out[n] = run;
    }
}

// Per member: alive count (its buckets' share of the global offsets) and the
// surface charge Q_S = q_surface0 + the charge absorbed so far, which enters
// the field as an interior l = 0 charge (Q_S / (4 pi r), Sec. 3).  Done by
// the first block of the kernel that ranks (after the offsets, before the carries).
__device__ inline void member_live(const Map &mp, const uint32_t *off, const KParams &kp)
{
    for (int s = threadIdx.x; s < kp.n_members; s += blockDim.x) {
        const Seg &sg = mp.seg[s];
        Ctl &c = mp.ctl[s];
        if (!member_runs(sg, c, kp)) continue;
        const uint32_t live = off[sg.b0 + sg.nb] - off[sg.b0];
        if (kp.field_only) {
            c.records &= ~kKeyed;   // the sort records are consumed
        } else {
            // what the next launch finds after this one's push (set here: a
            // store in the push kernel turns its table loads into vector loads)
            const int64_t next = c.step + 1;
            c.next_step = next;
            c.records = live | (kp.fuse_keys && next < sg.n_steps ? kKeyed : 0u);
        }
        c.n_live = live;
        c.q_surface =
            (sg.q_surface0 + kQ * (double)(c.n_dead - c.n_dead_ion)) + (double)c.n_dead_ion;
    }
}

// Bucket order (arbitrary inside a bucket): key, id and source slot.  Only
// the records of running members' first `records` slots count (the push writes
// records for the slots it moves, and slots past the alive count may hold
// older ones).
// SCAN, for histograms of up to kScanLdsBuckets buckets: every block scans the
// histogram for itself in LDS (the first one stores the offsets for the later
// kernels), which saves the launch of the offsets kernel: a step of 10,000
// particles at l_max 8 36.1 -> 35.2 us, with its share of the read-back
// (100 steps) 38.2 -> 35.8.  A later kernel clears the histogram.  At 16384
// buckets every block's scan of 64 KiB costs more than it saves (1e5 particles
// at l_max 16 83.3 -> 86.8 us per step).
constexpr int kScanLdsBuckets = 4096;

template <bool SCAN>
__global__ __launch_bounds__(kBlock) void k_sort_scatter(Map mp, const KeyRec *krec,
                                                         const uint32_t *hist, uint32_t *off,
                                                         OrdRec *orec, KParams kp)
{
    __shared__ uint32_t lds_off[SCAN ? kScanLdsBuckets : 1];
    const uint32_t i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const bool in = i < (uint32_t)kp.n_tiles * kWave;
    KeyRec r{0ull, 0u, kNone};
    if (in) r = krec[i];   // issued before the member's tables
    if constexpr (SCAN) {
        constexpr int per = kScanLdsBuckets / kBlock;
        const int base = (int)threadIdx.x * per;
        uint32_t v[per], s = 0, total;
#pragma unroll
        for (int k = 0; k < per; ++k) {
            v[k] = base + k < kp.nb ? hist[base + k] : 0u;
            s += v[k];
        }
        uint32_t run = block_exclusive_scan(s, &total);
#pragma unroll
        for (int k = 0; k < per; ++k) {
            lds_off[base + k] = run;
            if (blockIdx.x == 0 && base + k < kp.nb) off[base + k] = run;
            run += v[k];
        }
        if (blockIdx.x == 0) {
            if (threadIdx.x == 0) off[kp.nb] = total;
            begin_step(mp, kp);
        }
        __syncthreads();
    }
    if (!in) return;
    const uint32_t mb = uniform_u32(mp.tile_member[i >> 6]);
    if (mb == kNone) return;
    const Seg &sg = mp.seg[mb];
    const Ctl &c = mp.ctl[mb];
    if (!runs_step(sg, c.next_step, kp) || (i - sg.p0) >= (c.records & ~kKeyed)) return;
    if (r.sub == kNone) return;
    // the bucket again, from the key and the member of this slot's tile (the
    // same arithmetic as in the key kernel and the push, so the same bucket)
    const uint32_t b = bucket_of(__longlong_as_double((long long)r.key), sg.inv_vol, sg.b0, sg.nb);
    orec[(SCAN ? lds_off[b] : off[b]) + r.sub] = OrdRec{r.key, r.uid, i};
}

// Ranking in a kernel of its own, for large mean buckets (kPlaceMaxBucket).
// Final position = bucket start + number of bucket mates with a smaller
// (r^2, id) key (independent of the order inside the bucket), moved into the
// member's slot range; the particle's state moves there.  A block's positions
// cover a window of whole buckets, staged in LDS when it fits (12 KB; with
// 24 KB, six blocks per CU, the kernel took 5% longer).
constexpr int kRankWindow = 1024;

__device__ inline uint32_t bucket_of_rec(const Map &mp, const OrdRec &r)
{
    const Seg &sg = mp.seg[mp.tile_member[r.idx >> 6]];
    return bucket_of(__longlong_as_double((long long)r.key), sg.inv_vol, sg.b0, sg.nb);
}

__global__ __launch_bounds__(kBlock) void k_sort_rank_move(Map mp, const OrdRec *orec,
                                                           const uint32_t *off, const PRec *A,
                                                           State B,
                                                           KParams kp)
{
    __shared__ uint64_t wkey[kRankWindow];
    __shared__ uint32_t wuid[kRankWindow];
    if (blockIdx.x == 0) member_live(mp, off, kp);
    const uint32_t n = off[kp.nb];   // alive particles of all running members
    const uint32_t p0 = xcd_block(blockIdx.x, gridDim.x) * kBlock;
    if (p0 >= n) return;
    const uint32_t p_last = min(p0 + kBlock, n) - 1;
    const uint32_t p = p0 + threadIdx.x;
    const bool act = p < n;
    // This lane's record, then its member's tables, its bucket's bounds and
    // the gathered state: all issued before the block's window is staged, so
    // that their round trips overlap the window's (lanes past n take the
    // block's last record and leave after the barrier).
    const OrdRec me = orec[act ? p : p_last];
    const Seg &sg = mp.seg[mp.tile_member[me.idx >> 6]];
    const PRec a = A[me.idx];
    const uint32_t b = bucket_of(__longlong_as_double((long long)me.key), sg.inv_vol, sg.b0, sg.nb);
    const uint32_t lo = off[b], hi = off[b + 1];
    const uint32_t d0 = sg.p0 - off[sg.b0];   // the member's first slot, less its first offset
    const uint32_t w0 = off[bucket_of_rec(mp, orec[p0])];
    const uint32_t w1 = off[bucket_of_rec(mp, orec[p_last]) + 1];
    const bool staged = (w1 - w0) <= (uint32_t)kRankWindow;
    if (staged) {
        for (uint32_t j = w0 + threadIdx.x; j < w1; j += kBlock) {
            const OrdRec r = orec[j];
            wkey[j - w0] = r.key;
            wuid[j - w0] = r.uid;
        }
    }
    __syncthreads();
    if (!act) return;
    const uint64_t k = me.key;
    const uint32_t u = me.uid;
    uint32_t rank = 0;
    if (staged) {
        for (uint32_t j = lo - w0; j < hi - w0; ++j) {
            const uint64_t kj = wkey[j];
            rank += (kj < k) || (kj == k && wuid[j] < u);
        }
    } else {
        for (uint32_t j = lo; j < hi; ++j) {
            const OrdRec rj = orec[j];
            rank += (rj.key < k) || (rj.key == k && rj.uid < u);
        }
    }
    const uint32_t d = d0 + (lo + rank);
    B.x[d] = a.x;
    B.y[d] = a.y;
    B.z[d] = a.z;
    B.vx[d] = a.vx;
    B.vy[d] = a.vy;
    B.vz[d] = a.vz;
    B.uid[d] = u;
}

// ---------------------------------------------------------------------------
// Moments: per-tile sums of q R_lm and q I_lm
// ---------------------------------------------------------------------------
//
// Real solid harmonics through the polynomial Q_l^m(z, r^2) = r^l P~_l^m /
// (r sin th)^m and (x + i y)^m = C_m + i S_m:
//   R_lm^c = Q_l^m C_m,  R_lm^s = Q_l^m S_m,  I_lm = r^-(2l+1) R_lm,
// normalised so that sum_m Y_lm(a) Y_lm(b) = (2l+1)/(4 pi) P_l(a.b).  The
// kernel sums the rescaled Qh_l^m = Q_l^m / N_lm (a three-operation
// recurrence); the carries restore N_lm.

// A lane holds four consecutive particles of the group (lane i: slots 4 i ..
// 4 i + 3, so eight lanes hold a half tile) and adds its particles' terms in
// registers; the eight lanes of a half then meet in LDS.  kMomSlots channels
// make a batch: per channel and side (interior, exterior) one LDS row of the
// wave's 64 partial sums, the eight of a half at kMomHalfOff doubles.  A batch
// is read back with one (channel, side, half) per lane: its eight entries as
// four 16-byte reads, whose lanes fall on distinct banks by the 80-byte stride.
constexpr int kMomParts = kGroupSlots / kWave;     // particles per lane
constexpr int kMomSlots = 4;
constexpr int kMomLanes = kHalf / kMomParts;       // lanes of a half tile
constexpr int kMomHalves = kGroupSlots / kHalf;    // halves of a group
constexpr int kMomHalfOff = kMomLanes + 2;
constexpr int kMomRow = kMomHalves * kMomHalfOff;
static_assert(2 * kMomSlots * kMomHalves == kWave, "one lane per sum of a batch");

// The value of another lane of this lane's quad, through DPP: kPerm is a
// quad_perm control (0xB1: lane xor 1, 0x4E: lane xor 2).  A quad
// permutation has a source for every lane, so no "old" value is needed.
template <int kPerm>
__device__ inline double dpp_quad(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t plo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, kPerm, 0xF, 0xF, true);
    const uint32_t phi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), kPerm, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)phi << 32) | plo));
}

// The value of the lane four below within the upper half of every 8 lanes, zero
// in the lower (DPP row_shr:4 into banks 1 and 3 of a row of 16 lanes).
__device__ inline double dpp_shr4_odd_banks(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t plo =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x114, 0xF, 0xA, false);
    const uint32_t phi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x114, 0xF, 0xA, false);
    return __longlong_as_double((long long)(((uint64_t)phi << 32) | plo));
}

// A tile's row of H: per channel {interior sums of the group's tiles before
// this one, interior sum of half 0, exterior sums of the group's tiles after
// this one, exterior sum of half 1}, then the charge of the group's tiles
// before this one.
//
// One block per group and kWavesPerBlock slices of m: every wave goes through
// all 256 particles of the group for its slice's channels.  FP64 VALU is what
// bounds the kernel (9 operations per (l, m), particle and side pair); a
// layout with one particle per lane spent twice that on the cross-lane folds
// (v_permlane16_swap costs 1.5 FP64 FMAs, and v_mfma_f64_4x4x4 3.6, on the
// same unit).  Slicing m over the waves, not the particles, keeps the group's
// scan over its tiles inside a wave, without barriers, and lets a small launch
// spread one group over several blocks (21,347 particles at l_max 32: the
// evaluation 344 -> 222 us).  1.6e7 particles, l_max 16: 1.94 -> 1.29 ms, and
// 1.84 with the ranking (k_moments) that took 0.57 apart.
template <bool FULL>
__device__ inline void moment_sums(const double (&x)[kMomParts], const double (&y)[kMomParts],
                                   const double (&z)[kMomParts], const double (&q)[kMomParts],
                                   const uint64_t (&ions)[kMomParts], int count, int lane,
                                   int slice, uint32_t group, const Tables &tb, const KParams &kp,
                                   double *H, double *GS, double *wb)
{
    const int L = kp.L, C = kp.C;
    double *Hg = H + (size_t)group * kTilesPerGroup * kp.HW;
    double *Gs = GS + (size_t)group * kp.SW;
    if (slice == 0) {
        // charge of the group's tiles before each one, and of the group
        // (exact: counts of ions and electrons)
        double sq = 0.0;
        for (int t = 0; t < kTilesPerGroup; ++t) {
            const int n_val = min(max(count - t * kWave, 0), kWave);
            int n_ion = 0;
#pragma unroll
            for (int j = 0; j < kMomParts; ++j)
                n_ion += __popcll((ions[j] >> (t * (kWave / kMomParts))) & 0xffffull);
            if (lane == t) Hg[(size_t)t * kp.HW + 4 * C] = sq;
            sq += (double)n_ion + kQ * (double)(n_val - n_ion);
        }
        if (lane == 0) Gs[kp.C2] = sq;
    }
    const int m_begin = kp.m_slice[slice], m_end = kp.m_slice[slice + 1];
    if (m_begin >= m_end) return;

    double r2[kMomParts], inv_r2[kMomParts];
    double cq[kMomParts], sq[kMomParts], smm[kMomParts];   // q C_m, q S_m, r^-(2m+1)
#pragma unroll
    for (int j = 0; j < kMomParts; ++j) {
        r2[j] = fma(z[j], z[j], fma(y[j], y[j], x[j] * x[j]));
        inv_r2[j] = 1.0 / r2[j];
        smm[j] = 1.0 / sqrt(r2[j]);
        cq[j] = q[j];
        sq[j] = 0.0;
    }

    double *wr = wb + (lane >> 3) * kMomHalfOff + (lane & 7);
    // reader: channel rc of the batch, side rio, half h (in scan order: the
    // exterior sums are scanned from the last tile to the first)
    const int rc = lane >> 4, rio = (lane >> 3) & 1, ro = lane & 7;
    const int h = rio ? kMomHalves - 1 - ro : ro;
    const double2 *rd =
        reinterpret_cast<const double2 *>(wb + (2 * rc + rio) * kMomRow + h * kMomHalfOff);
    double *hdst = Hg + (size_t)(h >> 1) * kp.HW + 4 * rc + 2 * rio;
    double *gdst = Gs + rio * C + rc;
    const bool odd_tile = (lane & 2) != 0;
    // sums of the batch of n_ch channels from stream position ch0 on
    auto flush = [&](int ch0, int n_ch) {
        wave_lds_sync();
        double2 v[kMomLanes / 2];
#pragma unroll
        for (int k = 0; k < kMomLanes / 2; ++k) v[k] = rd[k];
        double own = 0.0;
        {
            double a[kMomLanes / 2];
#pragma unroll
            for (int k = 0; k < kMomLanes / 2; ++k) a[k] = v[k].x + v[k].y;
            own = (a[0] + a[1]) + (a[2] + a[3]);
        }
        // the tile's sum, then the exclusive scan over the group's four tiles
        const double t = own + dpp_quad<0xB1>(own);
        const double tx = dpp_quad<0x4E>(t);           // the pair's other tile
        const double pair = t + tx;
        const double below = dpp_shr4_odd_banks(pair);
        const double excl = below + (odd_tile ? tx : 0.0);
        if (rc < n_ch) {
            if ((lane & 1) == 0)
                *reinterpret_cast<double2 *>(hdst + 4 * ch0) = double2{excl, own};
            if (ro == 4) gdst[ch0] = below + pair;
        }
        wave_lds_sync();
    };
    // one channel's interior and exterior sums of this lane's particles
    auto put = [&](int slot, double r, double i) {
        wr[2 * slot * kMomRow] = r;
        wr[(2 * slot + 1) * kMomRow] = i;
    };
    // gamma_lm of the stream-order table, read one entry ahead of its use
    // through a running pointer (the read after the last entry lands on the
    // table's zero entry after the triangle; its value is never used)
    const double *ahead = reinterpret_cast<const double *>(
        tb.fq4 + (m_begin * (L + 1) - (m_begin * (m_begin - 1)) / 2));
    double ng = ld_const(ahead, 0);   // the next entry to use
    ahead += 4;
    auto next_gamma = [&]() {
        const double g = ng;
        ng = ld_const(ahead, 0);
        ahead += 4;
        return g;
    };
    // Qh_{l-1} -> Qh_l into the registers of Qh_{l-2}
    auto step_q = [&](const double *q1, double *q2) {
        const double g = next_gamma();
#pragma unroll
        for (int j = 0; j < kMomParts; ++j) q2[j] = fma(z[j], q1[j], -(g * r2[j]) * q2[j]);
    };
    int ch = 0;   // stream position of the batch's first channel
    int m = m_begin;
    if (m == 0) {
        // channels l = 1..L (Qh_0^0 = 1 only seeds the recurrence; l = 0 is
        // Gauss's law in the field kernel), the charge in the seed
        double qa[kMomParts], qb[kMomParts], sl[kMomParts];
#pragma unroll
        for (int j = 0; j < kMomParts; ++j) {
            qa[j] = q[j];
            qb[j] = 0.0;
            sl[j] = smm[j] * inv_r2[j];     // r^-(2l+1) at l = 1
        }
        (void)next_gamma();                 // l = 0
        int slot = 0;
        auto emit = [&](const double *qv) {
            double r = qv[0], i = qv[0] * sl[0];
#pragma unroll
            for (int j = 1; j < kMomParts; ++j) {
                r += qv[j];
                i = fma(qv[j], sl[j], i);
            }
#pragma unroll
            for (int j = 0; j < kMomParts; ++j) sl[j] *= inv_r2[j];
            put(slot, r, i);
            if (++slot == kMomSlots) {
                flush(ch, kMomSlots);
                ch += kMomSlots;
                slot = 0;
            }
        };
        int l = 1;
        for (; l < L; l += 2) {
            step_q(qa, qb);
            emit(qb);
            step_q(qb, qa);
            emit(qa);
        }
        if (l == L) {
            step_q(qa, qb);
            emit(qb);
        }
        if (slot > 0) flush(ch, slot);   // the other slots hold older values
        ch = L;
        m = 1;
    } else if (FULL) {
        ch = (m - 1) * (2 * L + 2 - m) + L;   // sum of 2 (L - k + 1), k = 1..m-1, after m = 0
        // powers m - 1 of x + i y and of r^-2, step by step (a member's sums
        // do not depend on how the orders are sliced)
        for (int k = 1; k < m; ++k) {
#pragma unroll
            for (int j = 0; j < kMomParts; ++j) {
                const double c = cq[j], s = sq[j];
                cq[j] = fma(x[j], c, -(y[j] * s));
                sq[j] = fma(x[j], s, y[j] * c);
                smm[j] *= inv_r2[j];
            }
        }
    }
    if (FULL) {
        bool second = false;   // the batch's second pair of channels is next
        for (; m < m_end; ++m) {
            double qa[kMomParts], qb[kMomParts], sl[kMomParts];
#pragma unroll
            for (int j = 0; j < kMomParts; ++j) {
                const double c = cq[j], s = sq[j];
                cq[j] = fma(x[j], c, -(y[j] * s));
                sq[j] = fma(x[j], s, y[j] * c);
                smm[j] *= inv_r2[j];
                sl[j] = smm[j];
                qa[j] = 1.0;
                qb[j] = 0.0;
            }
            // cos and sin of one (l, m) are two channels
            auto emit = [&](const double *qv) {
                double s0 = qv[0] * sl[0];
                double rcs = qv[0] * cq[0], rsn = qv[0] * sq[0];
                double ics = s0 * cq[0], isn = s0 * sq[0];
#pragma unroll
                for (int j = 1; j < kMomParts; ++j) {
                    s0 = qv[j] * sl[j];
                    rcs = fma(qv[j], cq[j], rcs);
                    rsn = fma(qv[j], sq[j], rsn);
                    ics = fma(s0, cq[j], ics);
                    isn = fma(s0, sq[j], isn);
                }
#pragma unroll
                for (int j = 0; j < kMomParts; ++j) sl[j] *= inv_r2[j];
                const int slot = second ? 2 : 0;
                put(slot, rcs, ics);
                put(slot + 1, rsn, isn);
                if (second) {
                    flush(ch, kMomSlots);
                    ch += kMomSlots;
                }
                second = !second;
            };
            (void)next_gamma();                     // l = m: Qh_m^m = 1
            emit(qa);
            int l = m + 1;
            for (; l < L; l += 2) {
                step_q(qa, qb);
                emit(qb);
                step_q(qb, qa);
                emit(qa);
            }
            if (l == L) {
                step_q(qa, qb);
                emit(qb);
            }
        }
        if (second) flush(ch, 2);
    }
}

// A group's particles in LDS.
struct __attribute__((aligned(16))) Parts {
    double x[kGroupSlots], y[kGroupSlots], z[kGroupSlots];
    float q[kGroupSlots];
    __device__ void put(int i, double xx, double yy, double zz, float qq)
    {
        x[i] = xx;
        y[i] = yy;
        z[i] = zz;
        q[i] = qq;
    }
    __device__ void load(int lane, double (&xx)[kMomParts], double (&yy)[kMomParts],
                         double (&zz)[kMomParts], double (&qq)[kMomParts],
                         uint64_t (&ions)[kMomParts]) const
    {
#pragma unroll
        for (int j = 0; j < kMomParts; ++j) {
            const int i = kMomParts * lane + j;
            xx[j] = x[i];
            yy[j] = y[i];
            zz[j] = z[i];
            qq[j] = (double)q[i];
            ions[j] = __ballot(qq[j] > 0.0);
        }
    }
};

// The ranking inside the moments kernel: each wave of a group's block places a
// tile, its records' gathers issued before the ranking.  A tile's window, the
// whole buckets around its positions, is ranked from LDS where it fits; where
// one of the block's four does not (the radial density well over the mean: 8
// records per bucket leave 80 in a window), every wave selects the records of its
// tile's slots from its window by counting digits of the key.  A step of 1e6
// particles at l_max 4, half of them at 10 / 30 / 100 / 1000 times the mean density:
// 209 / 241 / 275 / 404 us; with the ranking in a kernel of its own (windows of up
// to 1024 records per block in LDS, longer ones from memory) 247 / 324 / 762 / 3454, and
// with a counting pass per bit of the key past 320 records 272 / 658 / 881 / 2849.
// Windows of up to 144 or 420 records in LDS: 238 / 233 and 210 / 250 (290 at 20
// times), 320 records left to the last ranking instead of 96: 584 at 20 times (229).
constexpr int kPlaceWindow = 256;    // records of a window in LDS
constexpr int kPlaceMaxBucket = 32;  // larger mean buckets would not fit the window
constexpr int kPlaceRead = 4;        // keys a ranking reads at once (past its end, too)
constexpr int kDigitBits = 8, kDigits = 1 << kDigitBits;
constexpr int kPlaceSelect = 96;     // records left to a selecting wave for its last ranking

union PlaceLds {
    struct {
        uint64_t key[kPlaceWindow + kPlaceRead];
        uint32_t uid[kPlaceWindow];
    } win;
    uint32_t hist[2][kDigits];
    OrdRec sel[kPlaceSelect];
};

// Calls f(on, record) for the n records from rec on, all lanes in step, the loads
// of four records per lane issued ahead.
template <typename F>
__device__ inline void each_record(const OrdRec *__restrict__ rec, uint32_t n, int lane, F &&f)
{
    constexpr uint32_t kBatch = 4;
    for (uint32_t j0 = 0; j0 < n; j0 += kBatch * kWave) {
        OrdRec o[kBatch];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t j = j0 + k * kWave + (uint32_t)lane;
            o[k] = rec[min(j, n - 1)];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) f(j0 + k * kWave + (uint32_t)lane < n, o[k]);
    }
}

// One end of a tile's slots in its window's order: its class of records (those
// whose key, less the window's smallest, agrees with it above some bit, and, once
// keys are told apart, whose id does), and the records before and in the class.
struct PlaceEnd {
    uint64_t key = 0;
    uint32_t uid = 0, below = 0, count = 0;
};

// The records of the window of n from rec on that rank first .. first + tc - 1 in
// it, by store(rank - first, source slot); all lanes of the wave.  The classes of
// the two end ranks are narrowed digit by digit, one counting pass each (in all
// a pass for the smallest and largest key, one per digit and one that collects),
// until at most kPlaceSelect records lie between; these are ranked in LDS.  1 to 2
// digits where the density inside a bucket is smooth; the ids' digits count
// only where that many keys are equal.
template <typename Store>
__device__ inline void select_tile(const OrdRec *__restrict__ rec, uint32_t n, uint32_t first,
                                   uint32_t tc, int lane, PlaceLds &r, Store &&store)
{
    uint64_t least = ~0ull, most = 0ull;
    each_record(rec, n, lane, [&](bool, const OrdRec &o) {
        least = min(least, o.key);
        most = max(most, o.key);
    });
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        least = min(least, (uint64_t)__shfl_xor((unsigned long long)least, o));
        most = max(most, (uint64_t)__shfl_xor((unsigned long long)most, o));
    }
    // the bits of (key - least), then of the id, not yet told apart
    int kbits = most > least ? 64 - __builtin_clzll(most - least) : 0, ubits = 32;
    PlaceEnd lo, hi;   // of ranks first and first + tc - 1
    hi.count = n;
    auto low_mask = [](int bits) { return bits > 0 ? ~0ull >> (64 - bits) : 0ull; };
    while (hi.below + hi.count - lo.below > (uint32_t)kPlaceSelect && kbits + ubits > 0) {
        const bool ids = kbits == 0;
        int &bits = ids ? ubits : kbits;
        const uint64_t rest = low_mask(kbits), urest = low_mask(ubits);
        const int shift = max(bits - kDigitBits, 0);
        const bool one = lo.key == hi.key && lo.uid == hi.uid;   // one class for both ends
#pragma unroll
        for (int k = 0; k < 2 * kDigits / kWave; ++k) r.hist[0][k * kWave + lane] = 0u;
        wave_lds_sync();
        each_record(rec, n, lane, [&](bool on, const OrdRec &o) {
            const uint64_t key = o.key - least;
            auto in = [&](const PlaceEnd &e) {
                return (key & ~rest) == e.key && (!ids || (o.uid & ~(uint32_t)urest) == e.uid);
            };
            const uint32_t digit =
                (uint32_t)((ids ? (uint64_t)o.uid : key) >> shift) & (uint32_t)(kDigits - 1);
            if (on && in(lo)) atomicAdd(&r.hist[0][digit], 1u);
            if (on && !one && in(hi)) atomicAdd(&r.hist[1][digit], 1u);
        });
        wave_lds_sync();
        auto narrow = [&](PlaceEnd &e, const uint32_t *hist, uint32_t rank) {
            constexpr int per = kDigits / kWave;
            uint32_t c[per], sum = 0;
#pragma unroll
            for (int k = 0; k < per; ++k) {
                c[k] = hist[per * lane + k];
                sum += c[k];
            }
            uint32_t incl = sum;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t t = __shfl_up(incl, o);
                if (lane >= o) incl += t;
            }
            const uint32_t at = rank - e.below;   // in the class
            uint32_t digit = (uint32_t)(per * lane), before = incl - sum, count = c[0];
#pragma unroll
            for (int k = 1; k < per; ++k)
                if (before + count <= at) {
                    before += count;
                    count = c[k];
                    ++digit;
                }
            // the lane whose digits hold the rank
            const int src = (int)__builtin_ctzll(__ballot(at < incl) | 1ull << (kWave - 1));
            const uint64_t d = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)digit, src);
            e.below += (uint32_t)__builtin_amdgcn_readlane((int)before, src);
            e.count = (uint32_t)__builtin_amdgcn_readlane((int)count, src);
            if (ids) e.uid |= (uint32_t)(d << shift);
            else e.key |= d << shift;
        };
        narrow(lo, r.hist[0], first);
        narrow(hi, r.hist[one ? 0 : 1], first + tc - 1);
        bits = shift;
        wave_lds_sync();   // the counts are read
    }
    const uint64_t key1 = hi.key | low_mask(kbits);
    const uint32_t uid1 = hi.uid | (uint32_t)low_mask(ubits);
    uint32_t got = 0;
    each_record(rec, n, lane, [&](bool on, const OrdRec &o) {
        const uint64_t key = o.key - least;
        const bool in = on && (key > lo.key || (key == lo.key && o.uid >= lo.uid)) &&
                        (key < key1 || (key == key1 && o.uid <= uid1));
        const uint64_t v = __ballot(in);
        const uint32_t at = got + (uint32_t)__popcll(v & ((1ull << lane) - 1ull));
        if (in && at < (uint32_t)kPlaceSelect) r.sel[at] = o;
        got += (uint32_t)__popcll(v);
    });
    wave_lds_sync();
    const uint32_t m = min(got, (uint32_t)kPlaceSelect);
    for (uint32_t i0 = 0; i0 < m; i0 += kWave) {
        const uint32_t i = i0 + (uint32_t)lane;
        const OrdRec mine = r.sel[min(i, m - 1)];
        uint32_t rank = lo.below - first;   // wraps for records before the tile's
#pragma unroll 4
        for (uint32_t j = 0; j < m; ++j) {
            const OrdRec o = r.sel[j];
            rank += (o.key < mine.key) || (o.key == mine.key && o.uid < mine.uid);
        }
        if (i < m && rank < tc) store(rank, mine.idx);
    }
    wave_lds_sync();
}

// Places the tile's particles of the group (and, where the windows are ranked from
// LDS, what the tile's positions of the bucket order hold for the group's other
// tiles): p_group is the group's first position, count its particles, slot0 its
// first slot; q the tile; write: to the sorted state too.  All waves of the block.
__device__ inline void place_tile(const Seg &sg, const OrdRec *__restrict__ orec,
                                  const uint32_t *__restrict__ off, const PRec *__restrict__ A,
                                  const State &B, bool write, uint32_t p_group, int count,
                                  size_t slot0, int q, int lane, PlaceLds &r,
                                  uint32_t (&dense)[kWavesPerBlock], Parts &out)
{
    const int tc = min(max(count - q * kWave, 0), kWave);
    if (lane >= tc) out.put(q * kWave + lane, 0.0, 0.0, 2.0, 0.0f);
    auto store = [&](uint32_t slot, const PRec &a) {
        out.put((int)slot, a.x, a.y, a.z, (a.uid & kIonBit) ? 1.0f : (float)kQ);
        if (!write) return;
        const size_t d = slot0 + slot;
        B.x[d] = a.x;
        B.y[d] = a.y;
        B.z[d] = a.z;
        B.vx[d] = a.vx;
        B.vy[d] = a.vy;
        B.vz[d] = a.vz;
        B.uid[d] = a.uid;
    };
    const uint32_t pf = p_group + (uint32_t)(q * kWave), pl = pf + (uint32_t)tc - 1;
    const bool on = lane < tc;
    OrdRec me{0ull, 0u, 0u};
    PRec a;
    uint32_t lo = 0, hi = 0, w0 = 0, h0 = 0, l1 = 0, w1 = 0;
    if (tc > 0) {
        me = orec[on ? pf + (uint32_t)lane : pl];
        a = A[me.idx];
        const uint32_t b =
            bucket_of(__longlong_as_double((long long)me.key), sg.inv_vol, sg.b0, sg.nb);
        lo = off[b];
        hi = off[b + 1];
        w0 = (uint32_t)__builtin_amdgcn_readlane((int)lo, 0);
        h0 = (uint32_t)__builtin_amdgcn_readlane((int)hi, 0);
        l1 = (uint32_t)__builtin_amdgcn_readlane((int)lo, tc - 1);
        w1 = (uint32_t)__builtin_amdgcn_readlane((int)hi, tc - 1);
    }
    const uint32_t nw = w1 - w0;
    if (lane == 0) dense[q] = nw > (uint32_t)kPlaceWindow ? 1u : 0u;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) any |= dense[k];
    if (tc == 0) return;
    if (uniform_u32(any)) {
        select_tile(orec + w0, nw, pf - w0, (uint32_t)tc, lane, r,
                    [&](uint32_t i, uint32_t idx) { store((uint32_t)(q * kWave) + i, A[idx]); });
        return;
    }
    const uint32_t before = pf - w0, extra = before + (w1 - 1 - pl);
    // the window's records before and after the tile's positions
    auto extra_at = [&](uint32_t e) { return e < before ? w0 + e : pl + 1 + (e - before); };
    OrdRec ex{0ull, 0u, 0u};
    if ((uint32_t)lane < extra) ex = orec[extra_at(lane)];
    for (uint32_t e = (uint32_t)(lane + kWave); e < extra; e += kWave) {
        const OrdRec o = orec[extra_at(e)];
        r.win.key[extra_at(e) - w0] = o.key;
        r.win.uid[extra_at(e) - w0] = o.uid;
    }
    if (on) {
        r.win.key[before + lane] = me.key;
        r.win.uid[before + lane] = me.uid;
    }
    if ((uint32_t)lane < extra) {
        r.win.key[extra_at(lane) - w0] = ex.key;
        r.win.uid[extra_at(lane) - w0] = ex.uid;
    }
    wave_lds_sync();
    // slot in the group of a record whose bucket is [begin, end); the ids only
    // where another key is equal
    auto ranked = [&](uint64_t k, uint32_t u, uint32_t begin, uint32_t end) {
        uint32_t pos = begin, same = 0;
        for (uint32_t i = begin - w0; i < end - w0; i += kPlaceRead) {
            uint64_t key[kPlaceRead];
#pragma unroll
            for (uint32_t t = 0; t < (uint32_t)kPlaceRead; ++t) key[t] = r.win.key[i + t];
#pragma unroll
            for (uint32_t t = 0; t < (uint32_t)kPlaceRead; ++t) {
                const bool has = i + t < end - w0;
                pos += has && key[t] < k;
                same += has && key[t] == k;
            }
        }
        if (same > 1)
            for (uint32_t i = begin - w0; i < end - w0; ++i)
                pos += r.win.key[i] == k && r.win.uid[i] < u;
        return pos - p_group;   // wraps for positions before the group
    };
    const uint32_t slot = ranked(me.key, me.uid, lo, hi);
    if (on && slot < (uint32_t)count) store(slot, a);
    // records of other groups' positions that rank into this one: in the
    // buckets across the group's ends
    for (uint32_t e = (uint32_t)lane; __ballot(e < extra); e += kWave) {
        const uint32_t p = extra_at(e);
        const bool out_of_group = e < extra && p - p_group >= (uint32_t)count;
        if (!__ballot(out_of_group)) continue;
        if (out_of_group) {
            const OrdRec o = e < (uint32_t)kWave ? ex : orec[p];
            const bool low = e < before;
            const uint32_t es = ranked(o.key, o.uid, low ? w0 : l1, low ? h0 : w1);
            if (es < (uint32_t)count) store(es, A[o.idx]);
        }
    }
    wave_lds_sync();   // the window is read
}

// RANK: the block first puts its group in radial order (place_tile) and goes
// on with the particles it has in LDS.  Against a ranking kernel of its own
// this saves a launch and the reads of the sorted state.  Ranking and moments in
// kernels of their own and here, in us: 1.6e7 particles at l_max 1 711 / 710, 3 777 /
// 760, 4 836 / 789, 10 (6e6) 558 / 418 (the older moments kernel beside the ranking);
// evaluation of 120,011 particles at l_max 16 171 / 156.  Only mean buckets over
// kPlaceMaxBucket rank apart.
template <bool FULL, bool RANK>
__global__ __launch_bounds__(kBlock, 4) void k_moments(Map mp, const OrdRec *orec,
                                                       const uint32_t *off, const PRec *A, State B,
                                                       Tables tb, KParams kp, double *H, double *GS,
                                                       uint32_t *clear, int n_clear)
{
    __shared__ union {
        typename std::conditional<RANK, PlaceLds, double>::type place[kWavesPerBlock];
        double buf[kWavesPerBlock][2 * kMomSlots * kMomRow];
    } lds;
    __shared__ __attribute__((aligned(16))) typename std::conditional<RANK, Parts, double>::type part;
    __shared__ uint32_t dense[kWavesPerBlock];   // whose windows do not fit
    const int lane = threadIdx.x & 63;
    const int w = (int)uniform_u32(threadIdx.x >> 6);
    // (neighbouring groups share gathered lines)
    const uint32_t group = RANK ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    if constexpr (RANK) {
        if (blockIdx.x == 0 && blockIdx.y == 0) {
            member_live(mp, off, kp);
            // the histogram, where the scatter kernel scanned it
            for (int i = threadIdx.x; i < n_clear; i += kBlock) clear[i] = 0u;
        }
    }
    const uint32_t mb = uniform_u32(mp.tile_member[group * kTilesPerGroup]);
    if (mb == kNone || !member_runs(mp.seg[mb], mp.ctl[mb], kp)) return;
    double x[kMomParts], y[kMomParts], z[kMomParts], q[kMomParts];
    uint64_t ions[kMomParts];
    int count;   // the group's particles
    if constexpr (RANK) {
        const Seg &sg = mp.seg[mb];
        const uint32_t first = (group - sg.g0) * kGroupSlots;
        const uint32_t o0 = uniform_u32(off[sg.b0]);
        const uint32_t live = uniform_u32(off[sg.b0 + sg.nb]) - o0;
        count = live > first ? (int)min(live - first, (uint32_t)kGroupSlots) : 0;
        place_tile(sg, orec, off, A, B, blockIdx.y == 0, o0 + first, count,
                   (size_t)group * kGroupSlots, w, lane, lds.place[w], dense, part);
        __syncthreads();   // and the ranking's LDS is free for the sums from here on
        part.load(lane, x, y, z, q, ions);
    } else {
        const uint32_t first = (group - mp.seg[mb].g0) * kGroupSlots;
        const uint32_t n = mp.ctl[mb].n_live;
        count = n > first ? (int)min(n - first, (uint32_t)kGroupSlots) : 0;
        const size_t p = (size_t)group * kGroupSlots + kMomParts * lane;
#pragma unroll
        for (int j = 0; j < kMomParts; ++j) {
            const bool valid = kMomParts * lane + j < count;
            x[j] = valid ? B.x[p + j] : 0.0;
            y[j] = valid ? B.y[p + j] : 0.0;
            z[j] = valid ? B.z[p + j] : 2.0;
            const bool ion = valid && (B.uid[p + j] & kIonBit) != 0;
            q[j] = valid ? (ion ? 1.0 : kQ) : 0.0;
            ions[j] = __ballot(ion);
        }
    }
    const int turn = (int)(group & (kWavesPerBlock - 1));
    const int slice = (int)blockIdx.y * kWavesPerBlock + ((w + turn) & (kWavesPerBlock - 1));
    moment_sums<FULL>(x, y, z, q, ions, count, lane, slice, group, tb, kp, H, GS, lds.buf[w]);
}

// ---------------------------------------------------------------------------
// Carries: prefix/suffix scans over groups, totals, coefficients, Q_diff
// ---------------------------------------------------------------------------

// The chunk's member and its group range; false if the member does not run.
__device__ inline bool chunk_groups(const Map &mp, const KParams &kp, int j, uint32_t *mb,
                                    int *g0, int *g1)
{
    const uint32_t m = mp.chunk_member[j];
    if (m == kNone || !member_runs(mp.seg[m], mp.ctl[m], kp)) return false;
    const Seg &sg = mp.seg[m];
    if (sg.one_carry) return false;
    *mb = m;
    *g0 = (int)(sg.g0 + (uint32_t)(j - (int)sg.c0) * sg.cl);
    *g1 = min(*g0 + (int)sg.cl, (int)(sg.g0 + sg.ng));
    return true;
}

// The value that a DPP control brings to this lane, zero where it brings none
// (no source lane, or a row of 16 lanes outside kRows).
template <int kCtrl, int kRows = 0xF>
__device__ inline double dpp_or_zero(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, kRows, 0xF, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl, kRows, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// A lane's value to all.
__device__ inline double readlane(double v, int lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// A running FP64 sum that carries its own rounding error (Knuth's
// error-free TwoSum): the sum of n terms is good to about one rounding of
// the result instead of ~sqrt(n) of them.  The carries sum the group sums of
// up to ~6e4 groups per member; these kernels are bound by HBM, so the
// extra operations cost no time.
struct CompSum {
    double s = 0.0, e = 0.0;
    __device__ void add(double v)
    {
        const double t = s + v;
        const double z = t - s;
        e += (s - (t - z)) + (v - z);
        s = t;
    }
    __device__ double value() const { return s + e; }
};

// The group loops of the carry kernels issue the loads of kCarryBatch groups
// before using them (a chunk is 8-64 groups, or the tuned length, walked by
// one thread, and one HBM round trip per group would dominate); the sums
// keep the group order.
constexpr int kCarryBatch = 8;

// A channel's weights: interior sums of Qh = Q / N_lm to coefficients
// (carry * w + k) * nrm, with the image response of the exterior total and
// the drive in k; exterior ones carry * w_out.
struct ChannelWeights {
    double w, k, nrm, w_out;
};

__device__ inline ChannelWeights channel_weights(const Tables &tb, const Seg &sg, int c, int L,
                                                 double total, bool in_run, int64_t step)
{
    const int l = tb.chl[c];
    ChannelWeights cw;
    cw.nrm = tb.chn[c];
    cw.w = tb.wl[l] * sg.inv_ntilde * cw.nrm;
    cw.w_out = cw.w * cw.nrm;
    cw.k = -tb.ftil[l] * total * cw.w;
    if (c < L && in_run) cw.k += sg.u_asy[step] * tb.drive_w[l];
    return cw;
}

// All carries of a member of few groups in one kernel.  A block takes
// kOneChannels channels, both sides: their sums come to LDS in whole segments
// of lines, a wave scans a channel's two columns (the groups in 64 runs of scan
// order, one per lane, then the runs' sums across the wave), and the
// coefficients go back the same way.  One round trip of loads, where the
// chunked kernels' three launches take several: 100,117 particles (392 groups)
// at l_max 16 14.6 us for the three, 10.1 here (4.4 of either are the events
// around them).  Up to kOneCarryGroups groups, a
// run of eight per lane.  Steps of 5,000 / 30,000 / 128,000 particles, chunked
// and here, in us: l_max 16 43.7 / 53.8 / 90.3 and 38.0 / 48.1 / 88.5, l_max 32
// 66.0 / 90.9 / 177.8 and 59.9 / 84.9 / 177.9; room for 960 groups gained 3% at
// 200,000 particles and l_max 3, but cost the small ones 0.7 us.
constexpr int kOneCarryGroups = kWave * kCarryBatch;
constexpr int kOneChannels = kWavesPerBlock;   // channels per block
constexpr int kOneRow = kOneCarryGroups + 1;

// the channels' blocks, one for the charges, one for the response
__host__ __device__ inline int one_carry_blocks(int C)
{
    return (C + kOneChannels - 1) / kOneChannels + 2;
}

// One step of the wave's inclusive scan of compensated sums.
template <int kCtrl, int kRows = 0xF>
__device__ inline void comp_scan_step(CompSum &v)
{
    const double ts = dpp_or_zero<kCtrl, kRows>(v.s), te = dpp_or_zero<kCtrl, kRows>(v.e);
    v.add(ts);
    v.e += te;
}

// The compensated sums of the lanes below this one, from the lanes' own.
__device__ inline CompSum comp_sum_below(CompSum v, CompSum *total)
{
    comp_scan_step<0x111>(v);        // row_shr:1, 2, 4, 8
    comp_scan_step<0x112>(v);
    comp_scan_step<0x114>(v);
    comp_scan_step<0x118>(v);
    comp_scan_step<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    comp_scan_step<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    total->s = readlane(v.s, kWave - 1);
    total->e = readlane(v.e, kWave - 1);
    CompSum below;
    below.s = dpp_or_zero<0x138>(v.s);   // wave_shr:1
    below.e = dpp_or_zero<0x138>(v.e);
    return below;
}

__device__ inline void carry_member(const Seg &sg, const Ctl &ct, int block, const double *GS,
                                    const Tables &tb, const KParams &kp, double *CR, double *qpre)
{
    __shared__ double val[2 * kOneChannels][kOneRow];   // interior, exterior columns
    const int lane = threadIdx.x & 63;
    const int w = (int)uniform_u32(threadIdx.x >> 6);
    const int ng = (int)sg.ng, per = (ng + kWave - 1) / kWave;
    const int q0 = min(lane * per, ng), q1 = min(q0 + per, ng);   // this lane's run
    const size_t sw = (size_t)kp.SW;
    const double *src = GS + (size_t)sg.g0 * sw;
    const int64_t step = ct.step;
    const bool in_run = step >= 0 && step < sg.n_steps;
    const int n_blocks = one_carry_blocks(kp.C);
    // the sums before each group of this lane's run of a column, given by
    // get(group): run, and f(group, sum before it) over the run
    auto scan = [&](bool up, auto get, CompSum *run, CompSum *total) {
        CompSum part;
        for (int q = q0; q < q1; ++q) part.add(get(up ? q : ng - 1 - q));
        *run = comp_sum_below(part, total);
    };
    auto walk = [&](bool up, auto get, CompSum run, auto f) {
        for (int q = q0; q < q1; ++q) {
            const int g = up ? q : ng - 1 - q;
            const double v = get(g);
            f(g, run.value());
            run.add(v);
        }
    };
    CompSum run, total;
    if (block == n_blocks - 1) {
        // the probe response: totals of the m = 0 channels of odd l, a wave each
        double acc = 0.0;
        for (int l0 = 1; l0 <= kp.L; l0 += 2 * kWavesPerBlock) {
            const int l = l0 + 2 * w;
            double part = 0.0;
            if (l <= kp.L) {
                const double *col = src + kp.C + l - 1;
                scan(true, [&](int g) { return col[(size_t)g * sw]; }, &run, &total);
                part = tb.drive_w[l] * tb.chn[l - 1] * total.value();
            }
            __syncthreads();
            if (lane == 0) val[0][w] = part;
            __syncthreads();
            if (threadIdx.x == 0)
                for (int k = 0; k < kWavesPerBlock; ++k) acc += val[0][k];
        }
        if (threadIdx.x == 0 && in_run) sg.qdiff[step] = -acc / sg.ntilde;
        return;
    }
    if (block == n_blocks - 2) {   // charge of the member's particles before each group
        if (w != 0) return;
        auto get = [&](int g) { return src[(size_t)g * sw + kp.C2]; };
        scan(true, get, &run, &total);
        walk(true, get, run, [&](int g, double carry) { qpre[sg.g0 + g] = carry; });
        return;
    }
    // thread -> column (interior, then exterior) and group of the copies
    const int col = threadIdx.x & (2 * kOneChannels - 1), g_first = threadIdx.x / (2 * kOneChannels);
    constexpr int kStride = kBlock / (2 * kOneChannels);
    const int c0 = block * kOneChannels, cc = c0 + (col & (kOneChannels - 1));
    const int column = col < kOneChannels ? cc : kp.C + cc;
    if (cc < kp.C) {
        constexpr int kLoads = kOneCarryGroups / kStride;
        double v[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int g = g_first + k * kStride;
            if (g < ng) v[k] = src[(size_t)g * sw + column];
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int g = g_first + k * kStride;
            if (g < ng) val[col][g] = v[k];
        }
    }
    __syncthreads();
    const int c = c0 + w;
    if (c < kp.C) {
        double *in = val[w], *ex = val[kOneChannels + w];
        auto get_ex = [&](int g) { return ex[g]; };
        auto get_in = [&](int g) { return in[g]; };
        CompSum run_in, total_in;
        scan(false, get_ex, &run, &total);
        scan(true, get_in, &run_in, &total_in);
        const ChannelWeights cw = channel_weights(tb, sg, c, kp.L, total.value(), in_run, step);
        walk(false, get_ex, run, [&](int g, double carry) { ex[g] = carry * cw.w_out; });
        walk(true, get_in, run_in,
             [&](int g, double carry) { in[g] = (carry * cw.w + cw.k) * cw.nrm; });
    }
    __syncthreads();
    if (cc < kp.C) {
        double *dst = CR + (size_t)sg.g0 * kp.C2 + column;
        for (int g = g_first; g < ng; g += kStride) dst[(size_t)g * kp.C2] = val[col][g];
    }
}

__global__ __launch_bounds__(kBlock) void k_chunk_sums(Map mp, const double *__restrict__ GS,
                                                       double *__restrict__ chunkS, KParams kp)
{
    const int j = blockIdx.x;
    const int c = blockIdx.y * kBlock + threadIdx.x;
    if (c >= kp.SW) return;
    uint32_t mb;
    int g0, g1;
    if (!chunk_groups(mp, kp, j, &mb, &g0, &g1)) return;
    const size_t sw = (size_t)kp.SW;
    const double *src = GS + (size_t)g0 * sw + c;
    const int ng = g1 - g0;
    CompSum s;
    int g = 0;
    for (; g + kCarryBatch <= ng; g += kCarryBatch) {
        double v[kCarryBatch];
#pragma unroll
        for (int k = 0; k < kCarryBatch; ++k) v[k] = src[(size_t)(g + k) * sw];
#pragma unroll
        for (int k = 0; k < kCarryBatch; ++k) s.add(v[k]);
    }
    for (; g < ng; ++g) s.add(src[(size_t)g * sw]);
    chunkS[(size_t)j * kp.SW + c] = s.value();
}

// Per member (blockIdx.y) and channel (one wave each): exclusive prefix of the
// interior chunk sums and of the charge column, exclusive suffix of the
// exterior ones, and the totals T_lm.  The member's chunks, in scan order, are cut into 64 consecutive runs,
// one per lane: each lane sums its run, the wave scans the run sums, and each
// lane then writes its run's carries.
// The blocks past the n_cols of the columns carry the members of few groups
// (beside this kernel's few blocks and long chains they cost least).
__global__ __launch_bounds__(kBlock) void k_chunk_scan(Map mp, const double *chunkS,
                                                       double *chunkC, double *T, Tables tb,
                                                       KParams kp, int n_cols, const double *GS,
                                                       double *CR, double *qpre)
{
    const int s = blockIdx.y;
    if ((int)blockIdx.x >= n_cols) {
        const Seg &sg = mp.seg[s];
        if (!sg.one_carry || !member_runs(sg, mp.ctl[s], kp)) return;
        // (blocks of neighbouring columns share lines of GS and CR: one XCD)
        carry_member(sg, mp.ctl[s],
                     (int)xcd_block(blockIdx.x - (uint32_t)n_cols, gridDim.x - (uint32_t)n_cols),
                     GS, tb, kp, CR, qpre);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int c = (int)uniform_u32(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    if (c >= kp.SW) return;
    const Seg &sg = mp.seg[s];
    if (sg.one_carry || !member_runs(sg, mp.ctl[s], kp)) return;
    const int nc = (int)sg.nc;
    const bool interior = c < kp.C || c == kp.C2;
    const double *cS = chunkS + (size_t)sg.c0 * kp.SW + c;
    double *cC = chunkC + (size_t)sg.c0 * kp.SW + c;
    const int per = (nc + kWave - 1) / kWave;
    const int q0 = lane * per, q1 = min(q0 + per, nc);   // this lane's run in scan order
    auto chunk = [&](int q) { return interior ? q : nc - 1 - q; };
    CompSum part;
    for (int q = q0; q < q1; ++q) part.add(cS[(size_t)chunk(q) * kp.SW]);
    // inclusive scan of the runs' compensated sums (value and error term)
    CompSum incl = part;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const double ts = __shfl_up(incl.s, o), te = __shfl_up(incl.e, o);
        if (lane >= o) {
            incl.add(ts);
            incl.e += te;
        }
    }
    CompSum run;
    run.s = __shfl_up(incl.s, 1);
    run.e = __shfl_up(incl.e, 1);
    if (lane == 0) run = CompSum();
    for (int q = q0; q < q1; ++q) {
        const size_t at = (size_t)chunk(q) * kp.SW;
        cC[at] = run.value();
        run.add(cS[at]);
    }
    if (!interior && lane == kWave - 1) T[(size_t)s * kp.C + (c - kp.C)] = incl.value();
}

// Per-group coefficients of the field kernel (FP64, absolute).  Interior
// coefficient of group g: the carry of the groups before it, plus the
// constant part: the image response -f_l T_lm and the hemisphere drive (odd
// l, m = 0; stream positions 0..L-1 hold m = 0, l = 1..L).  Exterior: the
// carry of the groups after it.  The field kernel adds the sums of the
// group's own tiles and halves.  Column C2: the charge of the member's
// particles before the group.  The block of the member's first chunk also
// records the probe response Q_diff(t_step) from the totals.
__global__ __launch_bounds__(kBlock) void k_chunk_apply(Map mp, const double *__restrict__ GS,
                                                        const double *__restrict__ chunkC,
                                                        const double *__restrict__ T, Tables tb,
                                                        KParams kp, double *__restrict__ CR,
                                                        double *__restrict__ qpre)
{
    const int c = blockIdx.y * kBlock + threadIdx.x;
    const int j = blockIdx.x;
    uint32_t mb;
    int g0, g1;
    if (!chunk_groups(mp, kp, j, &mb, &g0, &g1)) return;
    const Seg &sg = mp.seg[mb];
    const int64_t step = mp.ctl[mb].step;
    const bool in_run = step >= 0 && step < sg.n_steps;
    const double *Ts = T + (size_t)mb * kp.C;
    if (c == 0 && blockIdx.y == 0 && j == (int)sg.c0 && in_run) {
        double acc = 0.0;
        // m = 0 channel l sits at stream position l - 1; its total is a sum of Qh
        for (int l = 1; l <= kp.L; l += 2) acc += tb.drive_w[l] * tb.chn[l - 1] * Ts[l - 1];
        sg.qdiff[step] = -acc / sg.ntilde;
    }
    if (c >= kp.SW) return;
    const size_t sw = (size_t)kp.SW;
    CompSum run;
    run.s = chunkC[(size_t)j * kp.SW + c];
    // Walks the chunk's groups in scan order (dir +1 from g0, -1 from g1 - 1),
    // calling f(g, carry before g) with the loads of kCarryBatch groups issued
    // ahead; the carry accumulates in group order, compensated.
    auto walk = [&](int dir, auto f) {
        const int ng = g1 - g0;
        const int first = dir > 0 ? g0 : g1 - 1;
        int i = 0;
        for (; i + kCarryBatch <= ng; i += kCarryBatch) {
            double v[kCarryBatch];
#pragma unroll
            for (int k = 0; k < kCarryBatch; ++k) v[k] = GS[(size_t)(first + dir * (i + k)) * sw + c];
#pragma unroll
            for (int k = 0; k < kCarryBatch; ++k) {
                f(first + dir * (i + k), run.value());
                run.add(v[k]);
            }
        }
        for (; i < ng; ++i) {
            const int g = first + dir * i;
            f(g, run.value());
            run.add(GS[(size_t)g * sw + c]);
        }
    };
    if (c == kp.C2) {   // charge of the member's particles before each group
        walk(1, [&](int g, double carry) { qpre[g] = carry; });
    } else if (c < kp.C) {
        const ChannelWeights cw = channel_weights(tb, sg, c, kp.L, Ts[c], in_run, step);
        walk(1, [&](int g, double carry) {
            CR[(size_t)g * kp.C2 + c] = (carry * cw.w + cw.k) * cw.nrm;
        });
    } else {
        const double w = channel_weights(tb, sg, c - kp.C, kp.L, 0.0, false, step).w_out;
        walk(-1, [&](int g, double carry) { CR[(size_t)g * kp.C2 + c] = carry * w; });
    }
}

// ---------------------------------------------------------------------------
// Counter-based generator for diffuse walls: Philox-4x64-10 (Salmon et al.,
// SC'11), counter (step, id, wall, 0), key (seed, 0).
// ---------------------------------------------------------------------------

__device__ inline void philox4x64(uint64_t c[4], uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0 = __umul64hi(M0, c[0]), lo0 = M0 * c[0];
        uint64_t hi1 = __umul64hi(M1, c[2]), lo1 = M1 * c[2];
        uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
        k0 += W0;
        k1 += W1;
    }
}

// Unit vector uniform on the hemisphere around the unit normal n.
__device__ inline void hemisphere_dir(uint64_t seed, uint32_t id, int64_t step, int wall,
                                      const double n[3], double d[3])
{
    uint64_t c[4] = {(uint64_t)step, (uint64_t)id, (uint64_t)wall, 0ull};
    philox4x64(c, seed, 0ull);
    const double inv53 = 1.0 / 9007199254740992.0;
    double ct = ((double)(c[0] >> 11) + 0.5) * inv53;
    double ph = 2.0 * kPi * (((double)(c[1] >> 11) + 0.5) * inv53);
    double st = sqrt(1.0 - ct * ct);
    double t[3] = {0.0, 0.0, 1.0};
    if (!(fabs(n[2]) < 0.9)) {
        t[0] = 1.0;
        t[2] = 0.0;
    }
    double ex[3] = {t[1] * n[2] - t[2] * n[1], t[2] * n[0] - t[0] * n[2], t[0] * n[1] - t[1] * n[0]};
    double inv = 1.0 / sqrt(ex[0] * ex[0] + ex[1] * ex[1] + ex[2] * ex[2]);
    ex[0] *= inv;
    ex[1] *= inv;
    ex[2] *= inv;
    double ey[3] = {n[1] * ex[2] - n[2] * ex[1], n[2] * ex[0] - n[0] * ex[2],
                    n[0] * ex[1] - n[1] * ex[0]};
    double cp = cos(ph), sp = sin(ph);
    for (int j = 0; j < 3; ++j) d[j] = ct * n[j] + st * (cp * ex[j] + sp * ey[j]);
}

// ---------------------------------------------------------------------------
// Field and push
// ---------------------------------------------------------------------------

struct Grave {
    double *x, *y, *z, *vx, *vy, *vz;
    uint32_t *uid;
};

// Double-double values (hi + lo, |lo| <= ulp(hi) / 2) for the l = 0 field,
// where two fields of ~N^(1/2) times the result cancel: error-free products
// through the FMA and error-free sums (Knuth's TwoSum).
struct DD {
    double hi, lo;
};

__device__ inline DD dd_from_sum(double a, double b)
{
    const double s = a + b;
    const double z = s - a;
    return DD{s, (a - (s - z)) + (b - z)};
}

__device__ inline DD dd_add(DD a, DD b)
{
    const DD s = dd_from_sum(a.hi, b.hi);
    return dd_from_sum(s.hi, s.lo + (a.lo + b.lo));
}

__device__ inline DD dd_mul(DD a, double b)
{
    const double p = a.hi * b;
    const double e = fma(a.hi, b, -p);
    return dd_from_sum(p, fma(a.lo, b, e));
}

__device__ inline DD dd_div(DD a, DD b)
{
    const double q = a.hi / b.hi;
    // remainder a - q b, its leading part exact through the FMA
    const double r = (fma(-q, b.hi, a.hi) + a.lo) - q * b.lo;
    return dd_from_sum(q, r / b.hi);
}

__device__ inline DD dd_mul_dd(DD a, DD b)
{
    const double p = a.hi * b.hi;
    const double e = fma(a.hi, b.hi, -p);
    return dd_from_sum(p, e + (a.hi * b.lo + a.lo * b.hi));
}

// x*x + y*y + z*z in double-double: error-free squares, compensated sums.
__device__ inline DD dd_norm2(double x, double y, double z)
{
    const double xx = x * x, yy = y * y, zz = z * z;
    DD s = dd_add(DD{xx, fma(x, x, -xx)}, DD{yy, fma(y, y, -yy)});
    return dd_add(s, DD{zz, fma(z, z, -zz)});
}

// The l = 0 field (radial component) of the charge enclosed by radius r:
// the surface charge and the particles below, `charge` (exact), and the
// uniform ion background n_i: charge / (4 pi ntilde r^2) + n_i (r^3 - 1) / (3 r^2),
// formed in double-double from the position itself and rounded once.  The
// two terms are ~N^(1/2) times their sum at N particles, and taking r from
// the rounded radial key shifts both the same way for every particle near
// that radius: a few 1e-13 of the RMS field at 1.6e7 particles.
__device__ inline double gauss_field_uniform(double charge, double ntilde, double ion_density,
                                             double x, double y, double z)
{
    const DD r2 = dd_norm2(x, y, z);
    // r = sqrt(r2) to double-double: one Newton correction of the FP64 root
    const double rh = sqrt(r2.hi);
    const DD r{rh, (fma(-rh, rh, r2.hi) + r2.lo) / (2.0 * rh)};
    const DD r3 = dd_mul_dd(r, r2);
    const DD num2 = dd_mul(dd_add(r3, DD{-1.0, 0.0}), ion_density);
    const DD den2 = dd_mul(r2, 3.0);
    const DD four_pi{4.0 * 3.141592653589793116, 4.0 * 1.2246467991473532e-16};
    const DD den1 = dd_mul_dd(dd_mul(r2, ntilde), four_pi);
    const DD f = dd_add(dd_div(DD{charge, 0.0}, den1), dd_div(num2, den2));
    return f.hi + f.lo;
}

// Far field of all other tiles through this tile's coefficient vector
// (interior alpha then exterior beta, stream order), evaluated at scaled
// coordinates xi = x / rho in the working precision R; returns grad_xi Phi.
//   Phi(xi) = sum_lm Qh_l^m(z, r^2) U_lm,
//   U_lm = (beta + s_l alpha)^c C_m + (beta + s_l alpha)^s S_m,  s_l = r^-(2l+1),
//   V_lm = alpha^c C_m + alpha^s S_m,
// with the rescaled Qh_l^m = Q_l^m / N_lm (the coefficients carry N_lm):
// Qh_m^m = 1, Qh_l^m = z Qh_{l-1}^m - gamma_lm r^2 Qh_{l-2}^m, and D_z Qh its
// z-derivative at fixed r^2, D_z Qh_l = Qh_{l-1} + z D_z Qh_{l-1} - gamma r^2
// D_z Qh_{l-2}.  Qh_l^m C_m is homogeneous of degree l, so the radial
// derivative is exact by Euler's relation and only D_z Qh enters the
// tangential part:
//   grad Phi = rhat (1/r) sum [(l - m) Qh U - (2l+1) s_l Qh V]
//              + (e_z - cos th rhat) sum U D_z Qh + (sum Qh dU/dx, sum Qh dU/dy, 0).
// (Assembling the radial part from the two partial derivatives of Q instead
// loses a factor ~l to cancellation.)  The radial bracket is summed as
// (l + 1/2) Qh W - (m + 1/2) Qh U with W_lm as U_lm but beta - s_l alpha: see
// far_order_zero.
// Where the far field reads the coefficients of channel k: interior and
// exterior side by side at p[2 (k - base)] and p[2 (k - base) + 1] (the
// channels of a few consecutive degrees lie within one LDS instruction's
// offset range of a single address).
template <typename R>
struct CfView {
    const R *p;
    int base;
    __device__ R a(int k) const { return p[2 * (k - base)]; }
    __device__ R b(int k) const { return p[2 * (k - base) + 1]; }
};

// stage(k0, k1) returns a view holding channels [k0, k1): the m = 0 block,
// then one m block at a time, in stream order.
//
// The coordinates come in FP64.  In FP32 (R = float) the far field is
// compensated: rounding the position to FP32 would shift every term of the
// recurrences coherently (a degree-l term by ~l ulps), and the terms of the
// tiles next to this one nearly cancel, which amplifies such shifts to
// ~1e-5 of the field.  So r^2 and z enter the Qh recurrence as hi + lo FP32
// pairs (the products with the lo parts are the first-order corrections,
// exact to O(ulp^2)), and the per-m quantities C_m, S_m, r^-(2m+1) and the
// directions are formed in FP64 and rounded once; what remains are the
// independent roundings of the FP32 arithmetic.
template <typename R>
struct FarPoint {
    double xd, yd, zd, inv_rd, inv_r2d;
    R r2, z, r2l, zl, inv_r2;
    __device__ FarPoint(double x, double y, double zz) : xd(x), yd(y), zd(zz)
    {
        constexpr bool kComp = sizeof(R) == 4;
        const double r2d = fma(zd, zd, fma(yd, yd, xd * xd));
        inv_r2d = 1.0 / r2d;
        inv_rd = kComp ? sqrt(inv_r2d) : 1.0 / sqrt(r2d);
        r2 = (R)r2d;
        z = (R)zd;
        r2l = kComp ? (R)(r2d - (double)r2) : (R)0;   // lo parts (zero in FP64)
        zl = kComp ? (R)(zd - (double)z) : (R)0;
        inv_r2 = (R)inv_r2d;
    }
    // gamma r^2 and one step of the recurrences, with the lo corrections
    __device__ R gam_r2(R g) const { return sizeof(R) == 4 ? fma(g, r2, g * r2l) : g * r2; }
    __device__ R rec_q(R Q1, R Q2, R gr2) const
    {
        const R t = -gr2 * Q2;
        return fma(z, Q1, sizeof(R) == 4 ? fma(zl, Q1, t) : t);
    }
    __device__ R rec_d(R Q1, R D1, R D2, R gr2) const
    {
        const R t = fma(z, D1, Q1);
        return fma(-gr2, D2, sizeof(R) == 4 ? fma(zl, D1, t) : t);
    }
};

// The sums over (l, m): radial, along D_z, and over d/dx, d/dy of C_m, S_m.
template <typename R>
struct FarSums {
    R a = 0, z = 0, x = 0, y = 0;
    __device__ void add(const FarSums &o)
    {
        a += o.a;
        z += o.z;
        x += o.x;
        y += o.y;
    }
};

// C_{m-1}, S_{m-1} and r^-(2m-1) of the order m that comes next.
template <typename R>
struct FarPower {
    double c = 1, s = 0, smm;
    __device__ explicit FarPower(const FarPoint<R> &pt) : smm(pt.inv_rd) {}
    __device__ void next(const FarPoint<R> &pt)
    {
        const double c1 = c, s1 = s;
        c = fma(pt.xd, c1, -(pt.yd * s1));
        s = fma(pt.xd, s1, pt.yd * c1);
        smm *= pt.inv_r2d;
    }
};

// Adds the order m = 0 to the sums.  With t = b + s_l a and
// w = b - s_l a (s_l = r^-(2l+1)), each (l, m) adds Qh t to the sum for d/dx,
// d/dy, t D_z Qh to the D_z sum, and to the radial sum
// Qh [(l - m) b - (l + m + 1) s_l a] = (l + 1/2) Qh w - (m + 1/2) Qh t:
// ten FMAs for the cos and the sin part (t, w and the three sums), and the
// (m + 1/2) part once per m from the sum of Qh t.  (With each sum taking its b
// and its a part by FMAs of their own: twelve and three more products; field
// kernel at 1.6e7 particles, l_max 16, FP32 2.80 -> 2.67 ms, FP64 at 2e6 0.557 ->
// 0.520 ms; errors against 64 bits the same, 1.2e-7 to 6e-7 in FP32.)
template <typename R, typename R4, typename Stage>
__device__ inline void far_order_zero(Stage &&stage, int L, const R4 *fq, const FarPoint<R> &pt,
                                      FarSums<R> &g)
{
    // cos channels only, stream position k = l - 1; l = 0 only seeds the
    // recurrence, its field is Gauss's law in the caller
    R Q1 = 1, Q2 = 0, D1 = 0, D2 = 0;           // Qh_{l-1}, Qh_{l-2} and their D_z
    R sl = (R)(pt.inv_rd * pt.inv_r2d);         // r^-(2l+1) at l = 1
    R T = 0, Wr = 0;
    const CfView<R> v = stage(0, L);
#pragma unroll 2
    for (int l = 1; l <= L; ++l) {
        const R4 e = fq[l];
        const R gr2 = pt.gam_r2(e.x);
        const R Qv = pt.rec_q(Q1, Q2, gr2);
        const R Dz = pt.rec_d(Q1, D1, D2, gr2);
        const R ac = v.a(l - 1), bc = v.b(l - 1);
        const R t = fma(sl, ac, bc), u = fma(-sl, ac, bc);
        T = fma(Qv, t, T);
        g.z = fma(Dz, t, g.z);
        Wr = fma(e.y * Qv, u, Wr);
        Q2 = Q1;
        Q1 = Qv;
        D2 = D1;
        D1 = Dz;
        sl *= pt.inv_r2;
    }
    g.a = fma((R)-0.5, T, g.a + Wr);
}

// The orders m0 <= m < m1, m0 >= 1, pw at m0.  Where m reaches a slice's end, the sums
// so far go to tot and a new slice begins: the slices' sums are added
// in their order whether one wave takes them all or four take one each.
template <typename R, typename R4, typename Stage>
__device__ inline void far_orders(Stage &&stage, int L, const R4 *fq, const FarPoint<R> &pt, int m0,
                                  int m1, uint32_t ends, FarPower<R> &pw, FarSums<R> &g,
                                  FarSums<R> &tot)
{
    int m = m0;
    int j = m * (L + 1) - (m * (m - 1)) / 2;   // stream index of (m, l = m)
    int k = L + (m - 1) * (2 * L + 2 - m);     // channel position of (m, l = m), cos then sin
    // C_m, S_m and C_{m-1}, S_{m-1} are common to all l of one m: the l
    // loop sums the cos and sin parts separately, combined once per m
    for (; m < m1; ++m) {
        if (m == (int)(ends & 0xffu)) {
            tot.add(g);
            g = FarSums<R>();
            ends >>= 8;
        }
        const R Cm1 = (R)pw.c, Sm1 = (R)pw.s;
        pw.next(pt);
        const R Cm = (R)pw.c, Sm = (R)pw.s;
        R sl = (R)pw.smm;
        // l = m: Qh = 1, D_z Qh = 0
        R Wc, Ws, Tc, Ts, Zc = 0, Zs = 0;
        const CfView<R> v = stage(k, k + 2 * (L - m + 1));
        {
            const R4 e = fq[j];
            const R ac = v.a(k), bc = v.b(k), as = v.a(k + 1), bs = v.b(k + 1);
            Tc = fma(sl, ac, bc);
            Ts = fma(sl, as, bs);
            Wc = e.y * fma(-sl, ac, bc);
            Ws = e.y * fma(-sl, as, bs);
            ++j;
            k += 2;
            sl *= pt.inv_r2;
        }
        R Q1 = 1, Q2 = 0, D1 = 0, D2 = 0;
#pragma unroll 2
        for (int l = m + 1; l <= L; ++l) {
            const R4 e = fq[j];
            const R ac = v.a(k), bc = v.b(k), as = v.a(k + 1), bs = v.b(k + 1);
            const R gr2 = pt.gam_r2(e.x);
            const R Qv = pt.rec_q(Q1, Q2, gr2);
            const R Dz = pt.rec_d(Q1, D1, D2, gr2);
            const R Qh = e.y * Qv;
            const R tc = fma(sl, ac, bc), uc = fma(-sl, ac, bc);
            const R ts = fma(sl, as, bs), us = fma(-sl, as, bs);
            Tc = fma(Qv, tc, Tc);
            Ts = fma(Qv, ts, Ts);
            Zc = fma(Dz, tc, Zc);
            Zs = fma(Dz, ts, Zs);
            Wc = fma(Qh, uc, Wc);
            Ws = fma(Qh, us, Ws);
            Q2 = Q1;
            Q1 = Qv;
            D2 = D1;
            D1 = Dz;
            ++j;
            k += 2;
            sl *= pt.inv_r2;
        }
        const R dm = (R)m, mh = (R)m + (R)0.5;
        g.a = fma(Cm, fma(-mh, Tc, Wc), fma(Sm, fma(-mh, Ts, Ws), g.a));
        g.z = fma(Cm, Zc, fma(Sm, Zs, g.z));
        g.x = fma(dm, fma(Tc, Cm1, Ts * Sm1), g.x);
        g.y = fma(dm, fma(Ts, Cm1, -(Tc * Sm1)), g.y);
    }
}

// grad_xi Phi from the sums.
template <typename R>
__device__ inline void far_gradient(const FarPoint<R> &pt, const FarSums<R> &g, R &gx, R &gy, R &gz)
{
    const R inv_r = (R)pt.inv_rd;
    const R xh = (R)(pt.xd * pt.inv_rd), yh = (R)(pt.yd * pt.inv_rd), c = (R)(pt.zd * pt.inv_rd);
    const R radial = fma(g.a, inv_r, -(c * g.z));
    gx = fma(xh, radial, g.x);
    gy = fma(yh, radial, g.y);
    gz = fma(c * g.a, inv_r, fma(xh, xh, yh * yh) * g.z);
}

// Near field: the direct part of G~_L between the particles of one block of
// W = 32 (a half tile) or 64 (the tile) radially consecutive particles (the
// pairs across blocks go through the coefficients), pair by pair.  For the
// pair (k, j) with rho = r_< / r_>, u = xh_k . xh_j and v = xh_other - u xh:
//   outer one: grad D = (1/r_>^2)       sum_l rho^l [-(l+1) P_l xh + P'_l v]
//   inner one: grad D = (1/(r_< r_>))   sum_l rho^l [ l P_l xh     + P'_l v]
// The three sums are symmetric in (k, j), so each pair is evaluated once: at
// step s lane k takes partner k + s (mod W, inside its block) and hands the
// partner's gradient to it through a lane rotation.  Each term carries the
// charge of its source (the other particle of the pair).  Pair terms in R,
// accumulated in FP64.  The rows hold each block twice (entries h + i and
// h + i + W for the i-th particle of the block starting at entry h = 2 W b),
// so the partner of every shift is a plain offset.

// Sums over the lanes of the wave below this one, and above it.  Each runs in
// its own direction and leaves the own lane out before it adds: the terms
// span r^l over the tile, so a total less a part would cancel.
__device__ inline double wave_sum_below(double v)
{
    v = dpp_or_zero<0x138>(v);            // wave_shr:1
    v += dpp_or_zero<0x111>(v);           // row_shr:1, 2, 4, 8
    v += dpp_or_zero<0x112>(v);
    v += dpp_or_zero<0x114>(v);
    v += dpp_or_zero<0x118>(v);
    v += dpp_or_zero<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ inline double wave_sum_above(double v, int lane)
{
    v = dpp_or_zero<0x130>(v);            // wave_shl:1
    v += dpp_or_zero<0x101>(v);           // row_shl:1, 2, 4, 8
    v += dpp_or_zero<0x102>(v);
    v += dpp_or_zero<0x104>(v);
    v += dpp_or_zero<0x108>(v);
    const double t3 = readlane(v, 48), t2 = t3 + readlane(v, 32), t1 = t2 + readlane(v, 16);
    return v + (lane < 16 ? t1 : lane < 32 ? t2 : lane < 48 ? t3 : 0.0);
}

// The whole field of the l >= 1, m = 0 channels (the axisymmetric kernel): with
// only l_max channels the tile's own pairs go through the radial scan too,
// carried on from the tile's coefficients lane by lane: about 60 instructions
// per degree where the pair sums took 18 per degree and pair shift (16 or 32
// shifts).  In FP64 in both precision modes.  1e6 particles, l_max 1: the field
// kernel 141 -> 130 us.
// Returns grad Phi; Ht is the tile's row of H, CRg the group's coefficients.
__device__ inline void axisym_field(int lane, int L, const Tables &tb, double inv_nt, const double *Ht,
                                    const double *CRg, double q, double x, double y, double z,
                                    double &gx, double &gy, double &gz)
{
    const double r2 = x * x + y * y + z * z;
    const double inv_r2 = 1.0 / r2, inv_r = 1.0 / sqrt(r2);
    double Ga = 0.0, Gz = 0.0;
    double Q1 = 1.0, Q2 = 0.0, D1 = 0.0, D2 = 0.0;   // Qh_{l-1}, Qh_{l-2} and their D_z
    double sl = inv_r * inv_r2;                      // r^-(2l+1) at l = 1
    for (int l = 1; l <= L; ++l) {
        const double gr2 = ld_const(reinterpret_cast<const double *>(tb.fq4 + l), 0) * r2;
        const double Qv = z * Q1 - gr2 * Q2;
        const double Dz = (Q1 + z * D1) - gr2 * D2;
        const double Qs = Qv * sl;
        // sums of the lanes before (interior) and after (exterior) this one
        const double below = wave_sum_below(q * Qv), above = wave_sum_above(q * Qs, lane);
        const double g = ld_const(tb.chg, l - 1) * inv_nt;
        const double a = ld_const(CRg, l - 1) + g * (ld_const(Ht, 4 * (l - 1)) + below);
        const double b =
            ld_const(CRg, L + l - 1) + g * (ld_const(Ht, 4 * (l - 1) + 2) + above);
        Ga = fma((double)l * Qv, b, Ga);
        Ga = fma(-(l + 1.0) * Qs, a, Ga);
        Gz = fma(Dz, b, Gz);
        Gz = fma(Dz * sl, a, Gz);
        Q2 = Q1;
        Q1 = Qv;
        D2 = D1;
        D1 = Dz;
        sl *= inv_r2;
    }
    const double xh = x * inv_r, yh = y * inv_r, c = z * inv_r;
    const double radial = Ga * inv_r - c * Gz;
    gx = xh * radial;
    gy = yh * radial;
    gz = c * Ga * inv_r + (xh * xh + yh * yh) * Gz;
}

// One wave's particles for the near field: each block's rows written twice
// (see above).
template <typename R>
struct NearRows {
    R xh[2 * kWave], yh[2 * kWave], zh[2 * kWave], r[2 * kWave], ir[2 * kWave], q[2 * kWave];
    // FP32 only: r / rho_t - 1 against the tile's reference radius rho_t
    R s[sizeof(R) == 4 ? 2 * kWave : 1];
};

__device__ inline double bpermute(int addr, double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ inline float bpermute(int addr, float v)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}

// Full near field.  Per pair (k, j), with rho = r_< / r_> and u = xh_k . xh_j:
//   S1 = sum_l rho^l P_l(u),  Sl = sum_l l rho^l P_l(u),  SB = sum_l rho^l P'_l(u)
// (l = 1..L) and, as above, S_in = Sl, S_out = -(Sl + S1).  For either particle
// the scale is 1 / (r_own r_>) whether it is the inner or the outer one, and
// grad D = (SA - SB u) xh_own + SB xh_other: a multiple of the own direction
// plus a multiple of the other's.  Each lane sums the multiples of its own
// direction in one number and the rest in a vector; the partner's two
// multiples go to it by a lane permutation, and it scales the sender's
// direction (read from LDS) itself.  Lanes without a particle carry charge 0,
// so their terms vanish without masks.  In FP64 the Legendre sums use the
// rescaled polynomials of the lg table (a two-operation recurrence; l = 1 is
// peeled); in FP32 a recurrence on P_l - P_{l-1} driven by 1 - u (lw table).
// The shifts come in kNearParts parts, each summed by itself and added in FP64
// in their order, so that a wave each may take them (the field kernel's SPLIT
// form) with the same result: this adds the parts p0 <= p < p1 to the sums.
constexpr int kNearParts = kWavesPerBlock;

struct NearSums {
    double ck = 0.0, bx = 0.0, by = 0.0, bz = 0.0;   // along the own direction; the rest
    __device__ void add(double c, double x, double y, double z)
    {
        ck += c;
        bx += x;
        by += y;
        bz += z;
    }
};

template <typename R, typename LG>
__device__ inline void near_field_full(int lane, int W, int L, const LG *lg, const NearRows<R> &nr,
                                       R xh, R yh, R zh, R r, R ir, R sk, R rho_t, R qk, int p0,
                                       int p1, NearSums &sum)
{
    R ck = 0, bx = 0, by = 0, bz = 0;
    const LG c1 = lg[1];
    // FP32: the constants of the first four degrees and of the last (L - 1) mod 4
    // stay in scalar registers over the shifts.  Loaded in each shift, the last
    // ones alone took two waits (4e6 particles, field kernel: l_max 4 233 -> 229
    // us, 8 306 -> 297, 16 599 -> 588).
    const int n_last = (L - 1) & 3;
    const LG f0 = lg[1], f1 = lg[min(2, L)], f2 = lg[min(3, L)], f3 = lg[min(4, L)];
    const LG e0 = lg[L - n_last], e1 = lg[min(L - n_last + 1, L)], e2 = lg[L - (n_last & 1)];
    const int hl = lane & (W - 1), hb = 2 * (lane & W);
    auto shift = [&](const int sft, R qk_s, bool last) {
        const int j = hb + hl + sft;   // partner, in the doubled block row
        const R xj = nr.xh[j], yj = nr.yh[j], zj = nr.zh[j];
        const R rj = nr.r[j], irj = nr.ir[j];
        const R qj = last && hl >= W / 2 ? (R)0 : nr.q[j];
        // a block's lanes are in radial order (key (r^2, id)): the partner
        // hl + sft (mod W) is the inner one when it wraps below this lane
        const bool k_outer = hl + sft >= W;
        const R irmx = k_outer ? ir : irj;   // 1 / r_>
        R u, S1, Sl, SB;
        if constexpr (sizeof(R) == 4) {
            // rho = r_< / r_> = 1 - del with del = (s_> - s_<) rho_t / r_>
            // from the offsets s = r / rho_t - 1 (FP64-exact, small): del
            // keeps its relative precision, and the powers rho^l are stepped
            // as rl - rl del, so no rounding of rho (an absolute 2^-24 near
            // 1) is raised to the l-th power.
            const R del = fabsf(sk - nr.s[j]) * (rho_t * irmx);
            const R rho = 1.0f - del;
            // FP32: w = 1 - u = |xh_j - xh_k|^2 / 2 (for nearly parallel
            // directions the difference is exact, so w keeps its relative
            // precision where a dot product would leave 1 - u an absolute
            // 2^-24), and the Legendre recurrence runs on the scaled
            // differences E_l = l (P_l - P_{l-1}): E_{l+1} = E_l - (2l+1) w P_l,
            // P_{l+1} = P_l + E_{l+1} / (l+1).  Near u = 1, where the sums of
            // rho^l P_l and rho^l P'_l amplify errors in u, this keeps P_l to
            // FP32 relative precision.
            const R dx = xj - xh, dy = yj - yh, dz = zj - zh;
            const R w = 0.5f * fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            u = 1.0f - w;
            S1 = rho * u;
            Sl = S1;
            SB = rho;
            // the registers of degree l and l + 1 trade roles: (Pa, Da, dPa)
            // hold P_l, E_l, P'_l and dPb P'_{l-1}, which the first of two
            // degrees overwrites with P'_{l+1}
            R Pa = u, Da = -w, dPa = 1, dPb = 0, rl = rho, Pb, Db;
            auto degree = [&](const LG c, R &P, R &D, R &dPm, R &Pn, R &Dn) {
                Dn = fmaf(-(c.z * w), P, D);
                Pn = fmaf(c.x, Dn, P);
                dPm = fmaf(c.z, P, dPm);   // P'_{l+1} = P'_{l-1} + (2l+1) P_l
                rl = fmaf(-rl, del, rl);
                const R t = rl * Pn;
                S1 += t;
                Sl = fmaf(c.w, t, Sl);
                SB = fmaf(rl, dPm, SB);
            };
            int l = 1;
            if (L > 4) {
                degree(f0, Pa, Da, dPb, Pb, Db);
                degree(f1, Pb, Db, dPa, Pa, Da);
                degree(f2, Pa, Da, dPb, Pb, Db);
                degree(f3, Pb, Db, dPa, Pa, Da);
                l = 5;
            }
#pragma unroll 1
            for (; l + 3 < L; l += 4) {   // four degrees: one wait for their constants
                const LG ca = lg[l], cb = lg[l + 1], cc = lg[l + 2], cd = lg[l + 3];
                degree(ca, Pa, Da, dPb, Pb, Db);   // degree l + 1
                degree(cb, Pb, Db, dPa, Pa, Da);   // degree l + 2
                degree(cc, Pa, Da, dPb, Pb, Db);
                degree(cd, Pb, Db, dPa, Pa, Da);
            }
            if (n_last & 2) {
                degree(e0, Pa, Da, dPb, Pb, Db);
                degree(e1, Pb, Db, dPa, Pa, Da);
            }
            if (n_last & 1) degree(e2, Pa, Da, dPb, Pb, Db);
        } else {
            const R rmin = k_outer ? rj : r;   // r_<
            const R rho = rmin * irmx;
            u = fma(zh, zj, fma(yh, yj, xh * xj));
            // l = 1: P_1 = u, P'_1 = 1.  Then two degrees per pass with the
            // registers of Ph_l and Ph_{l-1} (and of P'_l, P'_{l-1}) trading
            // roles
            S1 = rho * u;
            Sl = S1;
            SB = rho;
            R Pa = fma(u, u, -c1.z), Pb = u, dPa = c1.w * u, dPb = 1, rl = rho * rho;
            int l = 2;
            for (; l < L; l += 2) {
                const LG ca = lg[l], cb = lg[l + 1];
                R t = rl * Pa;   // degree l from Pa
                S1 = fma(ca.x, t, S1);
                Sl = fma(ca.y, t, Sl);
                SB = fma(rl, dPa, SB);
                Pb = fma(u, Pa, -(ca.z * Pb));   // Ph_{l+1}
                dPb = fma(ca.w, Pa, dPb);        // P'_{l+1}
                rl *= rho;
                t = rl * Pb;     // degree l + 1 from Pb
                S1 = fma(cb.x, t, S1);
                Sl = fma(cb.y, t, Sl);
                SB = fma(rl, dPb, SB);
                Pa = fma(u, Pb, -(cb.z * Pa));   // Ph_{l+2}
                dPa = fma(cb.w, Pb, dPa);        // P'_{l+2}
                rl *= rho;
            }
            if (l == L) {
                const LG ca = lg[l];
                const R t = rl * Pa;
                S1 = fma(ca.x, t, S1);
                Sl = fma(ca.y, t, Sl);
                SB = fma(rl, dPa, SB);
            }
        }
        const R S_out = -(Sl + S1), S_in = Sl;
        const R SAk = k_outer ? S_out : S_in, SAj = k_outer ? S_in : S_out;
        const R wk = qj * (ir * irmx), wj = qk_s * (irj * irmx);
        const R bk = wk * SB, bj = wj * SB;
        ck = fma(wk, SAk, ck);
        ck = fma(-bk, u, ck);
        bx = fma(bk, xj, bx);
        by = fma(bk, yj, by);
        bz = fma(bk, zj, bz);
        const R cj = fma(-bj, u, wj * SAj);
        // lane k's partner is k + sft (in its block), so lane k receives from
        // k - sft
        const int src_addr = 4 * ((lane & W) | ((hl - sft) & (W - 1)));
        const R cr = bpermute(src_addr, cj), br = bpermute(src_addr, bj);
        const int src = hb + hl + W - sft;   // in the doubled block row
        ck += cr;
        bx = fma(br, nr.xh[src], bx);
        by = fma(br, nr.yh[src], by);
        bz = fma(br, nr.zh[src], bz);
    };
    const int len = W / 2 / kNearParts;
    for (int part = p0; part < p1; ++part) {
        const int s1 = (part + 1) * len;
#pragma unroll 1
        for (int sft = part * len + 1; sft <= s1 && sft < W / 2; ++sft) shift(sft, qk, false);
        // the pairs (k, k + W/2) and (k + W/2, k) of a block are one pair: the
        // block's lanes below W/2 take it
        if (s1 == W / 2) shift(W / 2, hl >= W / 2 ? (R)0 : qk, true);
        sum.add((double)ck, (double)bx, (double)by, (double)bz);
        ck = 0;
        bx = 0;
        by = 0;
        bz = 0;
    }
}

// NEAR64: FP32 far field with the near field in FP64 (FP32 mode at high l_max).
// Waves per SIMD as the registers allow without spills: six in FP32, five for
// NEAR64 (four: 1e6 particles at l_max 32 670 us, five 640) and SPLIT (four:
// 1e5 particles at l_max 16, FP64, 41.0 us, five 38.6), four for FP64 in
// groups (five: ten registers spilled, 2e6 at l_max 4 157 -> 163 us).
// A block is a group, one tile per wave, or, for launches too small to fill the
// chip that way (SPLIT, split_max_tiles), one tile: each wave takes a slice of
// the orders m and a part of the pair shifts for all 64 particles, and the
// first wave adds the four and pushes.  Both forms add the same slices and
// parts in the same order: a member's results do not depend on the form.
template <bool FULL, bool FIELD_ONLY, bool FP32, bool NEAR64, bool SPLIT>
__global__ __launch_bounds__(kBlock, !FULL ? 8 : SPLIT || NEAR64 ? 5 : FP32 ? 6 : 4)
                                     void k_field_push(Map mp, State B, PRec *A, uint8_t *dead,
                                                       Grave G, const double *H,
                                                       const double *CR, const double *qpre,
                                                       Tables tb, KParams kp, double *Eout,
                                                       uint32_t *Eid, KeyRec *krec,
                                                       uint32_t *hist)
{
    // R, NF: the near field's precision; RF, NFF: the far field's
    using R = typename std::conditional<FP32 && !NEAR64, float, double>::type;
    using NF = typename std::conditional<FP32 && !NEAR64, float4, double4>::type;
    using RF = typename std::conditional<FP32, float, double>::type;
    using NFF = typename std::conditional<FP32, float4, double4>::type;
    // Per wave: the two halves' coefficients while the far field runs, then
    // the near field's rows.  The size is that of the FP64 rows, keeps the
    // block's LDS within a CU's 160 KB for up to six blocks and holds a window
    // of 192 FP64 channels or 384 FP32 ones; the second half's coefficients start kHalfPad bytes further, so that the two
    // addresses of a read fall on different banks.
    constexpr int kHalfPad = 16;
    constexpr int kLdsBytes = 6144 + kHalfPad;
    static_assert(sizeof(NearRows<R>) <= (size_t)kLdsBytes, "near-field rows exceed the wave's LDS");
    union WaveLds {
        NearRows<R> rows;
        RF cf[kLdsBytes / sizeof(RF)];
    };
    // (the axisymmetric kernel has neither; the push's slot counts come last)
    struct Counts {
        uint32_t c[kSlotWindow];
    };
    static_assert(sizeof(WaveLds) >= sizeof(Counts), "slot counts exceed the wave's LDS");
    __shared__ typename std::conditional<FULL, WaveLds, Counts>::type lds[kWavesPerBlock];

    const int lane = threadIdx.x & 63;
    const int w = (int)uniform_u32(threadIdx.x >> 6);
    const uint32_t tile = uniform_u32(SPLIT ? blockIdx.x : blockIdx.x * kTilesPerGroup + w);
    const uint32_t group = tile / kTilesPerGroup;
    const int tw = (int)(tile & (kTilesPerGroup - 1));   // the tile in its group
    // the tile's member: n = its alive count, pl = this lane's position in
    // its radial order
    uint32_t mb = kNone, n = 0, lt = 0;
    if ((int)tile < kp.n_tiles) {
        const uint32_t m = uniform_u32(mp.tile_member[tile]);
        if (m != kNone && member_runs(mp.seg[m], mp.ctl[m], kp)) {
            mb = m;
            n = mp.ctl[m].n_live;
            lt = tile - mp.seg[m].t0;
        }
    }
    const bool tile_live = mb != kNone && lt * kWave < n;
    const uint32_t p = tile * kWave + lane;
    const uint32_t pl = lt * kWave + lane;
    const bool valid = tile_live && pl < n;

    // (the velocities are read at the push, so that they hold no registers
    // through the field evaluation)
    double x = 0.0, y = 0.0, z = 2.0;
    uint32_t uid = 0xffffffffu;
    if (valid) {
        x = B.x[p];
        y = B.y[p];
        z = B.z[p];
        uid = B.uid[p];
    }
    const double r2 = key_r2(x, y, z);
    const double r = sqrt(r2);
    const double inv_r = 1.0 / r;
    const double inv_r2 = 1.0 / r2;
    const double xh = x * inv_r, yh = y * inv_r, zh = z * inv_r;
    const bool ion = valid && (uid & kIonBit);
    const double qk = ion ? 1.0 : kQ;   // this particle's charge
    if (!tile_live) return;

    const int L = kp.L;
    const Seg &sg = mp.seg[mb];
    Ctl &ct = mp.ctl[mb];
    const double ntilde = sg.ntilde, inv_nt = sg.inv_ntilde;
    // the rows of the group's tiles (half sums, half charges)
    const double *Hg = H + (size_t)group * kTilesPerGroup * kp.HW;
    // the near field's block: a half tile (the halves' coefficients differ by
    // the other half's sums) or the whole tile (they are the same)
    const int NW = (int)uniform_u32((uint32_t)sg.near_w);
    const bool split = NW == kHalf;

    // FP32: the tile's reference radius rho_t, its first particle's (the far
    // field's coordinates and coefficients are scaled by it; the near field
    // measures radii from it).
    double rho = 1.0;
    if (FP32) {
        const uint32_t p0 = tile * kWave;
        rho = sqrt(key_r2(B.x[p0], B.y[p0], B.z[p0]));
    }
    const double inv_rho = 1.0 / rho;

    double Ex, Ey, Ez;
    if constexpr (!FULL) {
        double gx, gy, gz;
        axisym_field(lane, L, tb, inv_nt, Hg + tw * kp.HW, CR + (size_t)group * kp.C2, valid ? qk : 0.0,
                     x, y, z, gx, gy, gz);
        Ex = -gx;
        Ey = -gy;
        Ez = -gz;
    } else {
        // ---- far field (all particles outside this lane's near-field block) ----
        FarSums<RF> far;
        // the field from the far sums (taken at once without SPLIT, so that the
        // point's factors hold no registers through the near field)
        auto far_field = [&](const FarPoint<RF> &pt) {
            RF gx, gy, gz;
            far_gradient(pt, far, gx, gy, gz);
            Ex = -(double)gx * inv_rho;
            Ey = -(double)gy * inv_rho;
            Ez = -(double)gz * inv_rho;
        };
        {
            const FarPoint<RF> pt(x * inv_rho, y * inv_rho, z * inv_rho);
            const NFF *fq;
            if constexpr (FP32) fq = tb.fq4_32;
            else fq = tb.fq4;
            // Coefficients of channel c for half h of this tile: the group's
            // (carries of the groups before and after it, the image response and
            // the drive) plus the sums of the group's own particles on each side:
            //   interior: the tiles before this one, and for h = 1 half 0;
            //   exterior: the tiles after this one, and for h = 0 half 1;
            // (the halves' own terms only with a near field per half tile)
            // as raw sums of Qh times N_lm^2 / ((2l+1) ntilde).  FP32: scaled to
            // the tile's coordinates x / rho (interior rho^-(l+1), exterior
            // rho^l) in FP64, then rounded once.  Every pass of every lane reads
            // them, so they go to LDS (the far field reads them as broadcasts, one
            // address per half), in windows of kWin channels (interior and
            // exterior of both halves) that hold whole m blocks; a window moves on
            // when the next block does not fit (never up to l_max 12 in FP64 and 18
            // in FP32, or where the waves share the orders, in a wave's slice of
            // that size; FP64 with room for l_max 16, 9216 B: 2e6 particles 555 / 564
            // us here, 560 / 552 with it).  An m block has at most 2 l_max <= 128
            // channels.
            constexpr int kWin = (kLdsBytes - kHalfPad) / (int)sizeof(RF) / 4;
            constexpr int kH1 = 2 * kWin + kHalfPad / (int)sizeof(RF);   // half 1's offset
            static_assert(kWin >= 2 * kMaxL, "an m block must fit a window");
            RF *cbuf = reinterpret_cast<RF *>(lds[w].cf);
            const int C = kp.C;
            const double *CRg = CR + (size_t)group * kp.C2;
            // FP32: rho^-(l+1) and rho^l of degree l = lane + 1, fetched per
            // channel from the lane of its degree
            double pw_in = 1.0, pw_out = 1.0;
            if (FP32) {
                // by squaring: 24 FP64 operations, log2 and exp2 took 124
                double sq = rho;
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    if ((lane + 1) >> k & 1) pw_out *= sq;
                    sq *= sq;
                }
                pw_in = 1.0 / (pw_out * rho);
            }
            int win0 = 0, win_len = -1;   // resident channels [win0, win0 + win_len)
            // Fills the window with channels [k0, k0 + len), U channels per lane at a
            // time with all their loads issued before the first use.  The first
            // window is filled before the far field starts (no other work of the
            // wave could hide its loads then, and few registers are live: U = 2);
            // a window moved inside the far field fills two channels at a time, one
            // in FP32 with the near field in FP32 (six waves per SIMD).
            auto fill = [&](int k0, int len, auto u_tag) {
                constexpr int U = decltype(u_tag)::value;
                const int n_iter = (len + kWave - 1) / kWave;
                for (int it0 = 0; it0 < n_iter; it0 += U) {
                    double yin[U], yout[U], hin[U], hout[U], ci[U], co[U], gsc[U];
                    int src[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = (it0 + u) * kWave + lane;
                        const int c = k0 + (i < len ? i : 0);
                        // the interior sums of the group's tiles before this one,
                        // the exterior sums of those after it, and the halves' own
                        // sums
                        const double *Ht = Hg + tw * kp.HW;
                        const double2 hi = reinterpret_cast<const double2 *>(Ht)[2 * c];
                        const double2 ho = reinterpret_cast<const double2 *>(Ht)[2 * c + 1];
                        yin[u] = hi.x;
                        yout[u] = ho.x;
                        hin[u] = split ? hi.y : 0.0;
                        hout[u] = split ? ho.y : 0.0;
                        ci[u] = CRg[c];
                        co[u] = CRg[C + c];
                        gsc[u] = tb.chg[c] * inv_nt;
                        src[u] = FP32 ? 4 * (tb.chl[c] - 1) : 0;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = (it0 + u) * kWave + lane;
                        double a0 = ci[u] + gsc[u] * yin[u], a1 = ci[u] + gsc[u] * (yin[u] + hin[u]);
                        double b1 = co[u] + gsc[u] * yout[u], b0 = co[u] + gsc[u] * (yout[u] + hout[u]);
                        if (FP32) {
                            // every lane takes part in the fetches
                            const double si = bpermute(src[u], pw_in), so = bpermute(src[u], pw_out);
                            a0 *= si;
                            a1 *= si;
                            b0 *= so;
                            b1 *= so;
                        }
                        if (i < len) {
                            cbuf[2 * i] = (RF)a0;
                            cbuf[2 * i + 1] = (RF)b0;
                            cbuf[kH1 + 2 * i] = (RF)a1;
                            cbuf[kH1 + 2 * i + 1] = (RF)b1;
                        }
                    }
                }
                wave_lds_sync();
                win0 = k0;
                win_len = len;
            };
            // this wave's orders, and their channels [c_begin, c_end)
            auto slice_end = [&](int sl) { return (int)((kp.f_ends >> (8 * sl)) & 0xffu); };
            const int m0 = SPLIT && w > 0 ? slice_end(w - 1) : 0;
            const int m1 = SPLIT ? slice_end(w) : L + 1;
            auto first_channel = [&](int m) { return m == 0 ? 0 : L + (m - 1) * (2 * L + 2 - m); };
            const int c_begin = first_channel(m0), c_end = first_channel(m1);
            fill(c_begin, min(kWin, c_end - c_begin), std::integral_constant<int, 2>());
            auto stage = [&](int k0, int k1) {
                if (k1 > win0 + win_len) {
                    wave_lds_sync();   // the old window's reads are done
                    // (the FP32 kernel at six waves per SIMD has no registers to spare)
                    fill(k0, min(kWin, c_end - k0), std::integral_constant<int, FP32 && !NEAR64 ? 1 : 2>());
                }
                return CfView<RF>{cbuf + (lane >= kHalf ? kH1 : 0), win0};
            };
            FarPower<RF> pw(pt);
            if constexpr (SPLIT) {
                for (int m = 1; m < m0; ++m) pw.next(pt);
                if (m0 == 0 && L > 0) far_order_zero<RF>(stage, L, fq, pt, far);
                FarSums<RF> unused;
                far_orders<RF>(stage, L, fq, pt, max(m0, 1), m1, 0u, pw, far, unused);
            } else {
                FarSums<RF> part;
                if (L > 0) far_order_zero<RF>(stage, L, fq, pt, part);
                far_orders<RF>(stage, L, fq, pt, 1, L + 1, kp.f_ends, pw, part, far);
                far.add(part);
                far_field(pt);
            }
            wave_lds_sync();   // read before the rows below overwrite them
        }

        // ---- near field (own block); E += -(1 / (4 pi nt)) sum_j q_j grad D ----
        NearRows<R> &nr = lds[w].rows;
        {
            const int e0 = 2 * (lane & NW) + (lane & (NW - 1));   // entries e0, e0 + NW
            for (int c = 0; c < 2; ++c) {
                const int i = e0 + c * NW;
                nr.xh[i] = (R)xh;
                nr.yh[i] = (R)yh;
                nr.zh[i] = (R)zh;
                nr.r[i] = (R)r;
                nr.ir[i] = (R)inv_r;
                nr.q[i] = valid ? (R)qk : (R)0;
                if constexpr (sizeof(R) == 4) nr.s[i] = (R)(r * inv_rho - 1.0);
            }
        }
        wave_lds_sync();   // the rows are this wave's own
        NearSums near;
        if (L >= 1) {   // else monopole only: Gauss's law below
            const NF *lg;
            if constexpr (std::is_same<R, float>::value) lg = tb.lw4_32;
            else lg = tb.lg4;
            near_field_full<R, NF>(lane, NW, L, lg, nr, (R)xh, (R)yh, (R)zh, (R)r, (R)inv_r,
                                   (R)(r * inv_rho - 1.0), (R)rho, valid ? (R)qk : (R)0,
                                   SPLIT ? w : 0, SPLIT ? w + 1 : kNearParts, near);
        }
        if constexpr (SPLIT) {
            // the waves' sums to the first wave
            constexpr int kSums = 8;
            static_assert(sizeof(WaveLds) >= kSums * kWave * sizeof(double), "sums exceed the wave's LDS");
            wave_lds_sync();   // the rows' reads are done
            double *mine = reinterpret_cast<double *>(&lds[w]) + lane;
            const double v[kSums] = {(double)far.a, (double)far.z, (double)far.x, (double)far.y,
                                     near.ck, near.bx, near.by, near.bz};
#pragma unroll
            for (int k = 0; k < kSums; ++k) mine[k * kWave] = v[k];
            __syncthreads();
            if (w != 0) return;
            far = FarSums<RF>();
            near = NearSums();
#pragma unroll 1
            for (int ww = 0; ww < kWavesPerBlock; ++ww) {
                const double *o = reinterpret_cast<const double *>(&lds[ww]) + lane;
                FarSums<RF> part;
                part.a = (RF)o[0];
                part.z = (RF)o[kWave];
                part.x = (RF)o[2 * kWave];
                part.y = (RF)o[3 * kWave];
                far.add(part);
                near.add(o[4 * kWave], o[5 * kWave], o[6 * kWave], o[7 * kWave]);
            }
            wave_lds_sync();
            far_field(FarPoint<RF>(x * inv_rho, y * inv_rho, z * inv_rho));
        }
        const double cn = -1.0 / (4.0 * kPi * ntilde);
        Ex = fma(cn, fma(near.ck, (double)xh, near.bx), Ex);
        Ey = fma(cn, fma(near.ck, (double)yh, near.by), Ey);
        Ez = fma(cn, fma(near.ck, (double)zh, near.bz), Ez);
    }

    // ---- self-image correction: the totals T_lm include the particle's own
    // image, which the pair sum i != k excludes ----
    {
        double sr = 0.0, sz = 0.0;   // radial and (e_z - c xh) parts of grad Phi_self
        double rl = inv_r2 * inv_r2 * inv_r;   // r^-(2l+3) at l = 1
        if (FULL) {
            for (int l = 1; l <= L; ++l) {
                // (by Horner's rule one operation fewer, but 16 VGPRs spilled
                // at six waves per SIMD: 4e6 particles at l_max 4, FP32, 233
                // -> 268 us, l_max 8 306 -> 327, 16 599 -> 610)
                sr = fma(tb.self_w1[l], rl, sr);
                rl *= inv_r2;
            }
            // grad Phi_self = -q sum f_l (l+1)/(4 pi nt) r^-(2l+3) xh; E = -grad
            const double e = qk * inv_nt * sr;
            Ex += e * xh;
            Ey += e * yh;
            Ez += e * zh;
        } else {
            double P0 = 1.0, P1 = zh, dP0 = 0.0, dP1 = 1.0;
            for (int l = 1; l <= L; ++l) {
                sr += tb.self_w[l] * rl * P1 * (-(l + 1.0) * P1);
                sz += tb.self_w[l] * rl * P1 * dP1;
                const double4 e = tb.nf4[l];
                const double P2 = e.x * zh * P1 - e.y * P0;
                const double dP2 = dP0 + e.z * P1;
                P0 = P1;
                P1 = P2;
                dP0 = dP1;
                dP1 = dP2;
                rl *= inv_r2;
            }
            // grad Phi_selfcorr = q sum (f_l/(4 pi nt)) r^-(2l+3) P_l [-(l+1) P_l xh + P'_l (e_z - c xh)]
            const double qn = qk * inv_nt;
            const double gx = qn * (sr * xh + sz * (-zh * xh));
            const double gy = qn * (sr * yh + sz * (-zh * yh));
            const double gz = qn * (sr * zh + sz * (1.0 - zh * zh));
            Ex -= gx;
            Ey -= gy;
            Ez -= gz;
        }
    }

    // ---- l = 0: Gauss's law.  The l = 0 part of G~ is 1/(4 pi r_>), so only
    // the charge enclosed by r_k pushes: Q_S, the particles before k in the
    // radial order (those of earlier tiles, carried by the scan, and the
    // lanes below in this tile), exact counts in super-particle units, and
    // the immobile ion background.  The particles' and the uniform
    // background's fields nearly cancel (to ~N^-1/2 of each), so they are
    // formed and added in double-double; a profile's enclosed charge is
    // tabulated and joins the count. ----
    {
        const uint64_t below = (1ull << lane) - 1ull;
        const int n_below = __popcll(__ballot(valid) & below);
        const int i_below = __popcll(__ballot(ion) & below);
        // the group's particles before this tile (exact counts)
        const double in_group = Hg[tw * kp.HW + 4 * kp.C];
        const double before =
            (qpre[group] + in_group) + ((double)i_below + kQ * (double)(n_below - i_below));
        double e;
        if (sg.ion_tab) {
            e = ((ct.q_surface + before) + ion_enclosed(sg, r, r2)) / (4.0 * kPi * ntilde * r2);
        } else if constexpr (FP32) {
            // FP64 rounding of the two opposing terms leaves ~1e-16 sqrt(N) of
            // the field, far below the FP32 mode's error
            const double q_enc = ct.q_surface + before;
            e = (q_enc / (4.0 * kPi * ntilde) + sg.ion_density * (r2 * r - 1.0) / 3.0) * inv_r2;
        } else {
            e = gauss_field_uniform(ct.q_surface + before, ntilde, sg.ion_density, x, y, z);
        }
        Ex += e * xh;
        Ey += e * yh;
        Ez += e * zh;
    }

    if (FIELD_ONLY) {
        if (valid) {   // by sorted position, or by id where no ids are asked for
            const size_t at = Eid ? (size_t)p : (size_t)uid;
            Eout[3 * at + 0] = Ex;
            Eout[3 * at + 1] = Ey;
            Eout[3 * at + 2] = Ez;
            if (Eid) Eid[p] = uid;
        }
        return;
    }
    // ---- leapfrog (Sec. 4 equations of motion) ----
    const double qm = ion ? sg.ion_qm : kQ / kM;
    const double dt = sg.dt;
    double vx = 0.0, vy = 0.0, vz = 0.0;
    if (valid) {
        vx = B.vx[p];
        vy = B.vy[p];
        vz = B.vz[p];
    }
    vx = add_product(vx, qm * Ex, dt);
    vy = add_product(vy, qm * Ey, dt);
    vz = add_product(vz, qm * Ez, dt);
    x = add_product(x, vx, dt);
    y = add_product(y, vy, dt);
    z = add_product(z, vz, dt);

    // ---- walls (tested on the new position) ----
    const double rn = sqrt(key_r2(x, y, z));
    uint8_t absorbed = 0;
    const int64_t step = ct.step;
    const double r_out = sg.r_out;
    if (valid && (rn <= 1.0 || rn >= r_out)) {
        const bool probe = rn <= 1.0;
        const int bc = probe ? sg.probe_bc : sg.wall_bc;
        if (probe && bc == SIM_BC_ABSORB) {
            absorbed = 1;
        } else {
            const double s = probe ? (2.0 - rn) / rn : (2.0 * r_out - rn) / rn;
            const double nrm[3] = {x / rn, y / rn, z / rn};
            x = x * s;
            y = y * s;
            z = z * s;
            if (bc == SIM_BC_DIFFUSE) {
                const double sp = sqrt(dot3(vx, vy, vz, vx, vy, vz));
                double inw[3] = {nrm[0], nrm[1], nrm[2]};
                if (!probe) {
                    inw[0] = -inw[0];
                    inw[1] = -inw[1];
                    inw[2] = -inw[2];
                }
                double d[3];
                hemisphere_dir(sg.seed, uid, step, probe ? 0 : 1, inw, d);
                vx = sp * d[0];
                vy = sp * d[1];
                vz = sp * d[2];
            } else {
                const double two_vn = 2.0 * dot3(vx, vy, vz, nrm[0], nrm[1], nrm[2]);
                vx = sub_product(vx, two_vn, nrm[0]);
                vy = sub_product(vy, two_vn, nrm[1]);
                vz = sub_product(vz, two_vn, nrm[2]);
            }
        }
    }
    if (valid) {
        PRec out;
        out.x = x;
        out.y = y;
        out.z = z;
        out.vx = vx;
        out.vy = vy;
        out.vz = vz;
        out.uid = uid;
        out.pad[0] = out.pad[1] = out.pad[2] = 0u;
        A[p] = out;
        dead[p] = absorbed;
    }
    // the next step's sort record of this slot, when the member runs then
    // (the same key, bucket and atomic slot as the key kernel would take;
    // the histogram was cleared by this step's offsets kernel, or by its moments
    // kernel where the scatter scanned it)
    if (kp.fuse_keys && step + 1 < sg.n_steps) {
        const bool live = valid && !absorbed;
        const double k2 = key_r2(x, y, z);
        const uint32_t sub = take_slot(lane, live, bucket_of(k2, sg.inv_vol, sg.b0, sg.nb), hist,
                                       reinterpret_cast<uint32_t *>(&lds[w]));
        KeyRec kr{0ull, 0u, kNone};
        if (live) {
            kr.key = (uint64_t)__double_as_longlong(k2);
            kr.uid = uid;
            kr.sub = sub;
        }
        if (valid) krec[p] = kr;
    }
    if (absorbed) {
        if (ion) atomicAdd(&ct.n_dead_ion, 1u);
        const uint32_t slot = sg.p0 + atomicAdd(&ct.n_dead, 1u);
        G.x[slot] = x;
        G.y[slot] = y;
        G.z[slot] = z;
        G.vx[slot] = vx;
        G.vy[slot] = vy;
        G.vz[slot] = vz;
        G.uid[slot] = uid;
    }
}

// The state of a member whose ids are its creation indices, in creation order:
// the records not flagged absorbed, and the graveyard.
__global__ __launch_bounds__(kBlock) void k_export_state(const PRec *A, const uint8_t *dead,
                                                         uint32_t n_cur, Grave G, uint32_t p0,
                                                         uint32_t n_dead, double *pos, double *vel,
                                                         uint8_t *alive)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n_cur && !dead[p0 + i]) {
        const PRec r = A[p0 + i];
        const size_t k = r.uid;
        pos[3 * k] = r.x;
        pos[3 * k + 1] = r.y;
        pos[3 * k + 2] = r.z;
        vel[3 * k] = r.vx;
        vel[3 * k + 1] = r.vy;
        vel[3 * k + 2] = r.vz;
        alive[k] = 1;
    }
    if (i < n_dead) {
        const size_t g = p0 + i, k = G.uid[g];
        pos[3 * k] = G.x[g];
        pos[3 * k + 1] = G.y[g];
        pos[3 * k + 2] = G.z[g];
        vel[3 * k] = G.vx[g];
        vel[3 * k + 1] = G.vy[g];
        vel[3 * k + 2] = G.vz[g];
        alive[k] = 0;
    }
}

constexpr unsigned kTableBlocks = 16;   // 4096 threads for up to 2146 entries (l_max 64)

__global__ __launch_bounds__(kBlock) void k_tables(TableDst t)
{
    fill_tables(t, (int)(blockIdx.x * kBlock + threadIdx.x), (int)(gridDim.x * kBlock));
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

enum KernelId {
    KN_SORT_KEY, KN_SCAN_A, KN_SCAN_C, KN_SORT_SCATTER, KN_SORT_RANK, KN_MOMENTS,
    KN_CHUNK_SUMS, KN_CHUNK_SCAN, KN_CHUNK_APPLY, KN_FIELD_PUSH, KN_STEP_FINISH, KN_COUNT
};

const char *kKernelNames[KN_COUNT] = {
    "sort_key", "bucket_sums", "bucket_offsets", "sort_scatter",
    "sort_rank_move", "moments", "carry_chunk_sums", "carry_chunk_scan", "carry_apply",
    "field_push", "step_finish"};

// What all members of a handle share, and the handle's capacities.
// The tunable launch sizes of sim_params, with 0 resolved to the built-in
// choice (bucket) or kept as "automatic" (chunk).
struct Tuning {
    int bucket = kBucketOccupancy;   // mean particles per sort bucket
    int chunk = 0;                   // groups per carry chunk, 0: by member size
    int keys = 0;                    // sort keys: 0 or 1 push, -1 own pass
    int split = 0;                   // near field: 1 half tiles, -1 whole tiles, 0 by member
};

Tuning tuning_of(const sim_params *p)
{
    Tuning t;
    if (p->sort_bucket > 0) t.bucket = p->sort_bucket;
    if (p->carry_chunk > 0) t.chunk = p->carry_chunk;
    t.keys = p->sort_keys;
    t.split = p->near_split;
    return t;
}

// Particles of a member's near-field block.  Half tiles halve the pair sums;
// the pairs across the halves then go through the coefficients.  In FP32 the
// coefficients carry the force of a close pair to a few ulps times l_max,
// while the pair's force is about l_max^2 / sqrt(n) of the RMS field (the
// collective field of n particles grows as sqrt(n)): half tiles are used
// where l_max^2 <= sqrt(n).  FP64 always splits.
int near_width(const Tuning &tu, bool fp32, int L, int64_t n)
{
    if (tu.split != 0) return tu.split > 0 ? kHalf : kWave;
    if (!fp32) return kHalf;
    return (double)L * (double)L <= std::sqrt((double)n) ? kHalf : kWave;
}

// In the FP32 mode the near field's FP32 error grows with l_max: a pair at
// nearly equal radius and angle contributes up to ~l_max^2 / (4 pi ntilde r^2)
// to the field, many times the field's RMS when the tile is sparse, and the
// FP32 evaluation of such a pair carries a few ulps of it.  With the radial
// powers stepped from 1 - rho and the Legendre recurrence driven by 1 - u it
// stays near 2-5e-6 of the RMS field up to l_max 19 on random shells of a few
// thousand particles; from this degree on the near field runs in FP64 while
// the far field stays FP32 (compensated).
constexpr int kNear64MinL = 20;

struct Layout {
    int L, C, C2;
    bool full, fp32;
    bool near64;     // FP32 mode with an FP64 near field (l_max >= kNear64MinL)
    int n_tiles;     // particle slots / 64 (whole groups)
    int n_groups;    // n_tiles / 4
    int n_chunks;
    int nb, nb_blocks;
    int n_members;
    Tuning tu;
};

// The part of the capacities in use: every member's tiles, chunks, buckets
// and table index lie below these (at least 1 each).  Launch grids cover the
// extent, not the capacity, so a large, sparsely filled handle steps at the
// cost of what it holds.
struct Extent {
    int n_tiles = kTilesPerGroup, n_chunks = 1, nb = 1, nb_blocks = 1, n_members = 1;
    bool one_carry = false, chunked = false;   // members of either kind of carries
    bool operator==(const Extent &o) const
    {
        return n_tiles == o.n_tiles && n_chunks == o.n_chunks && nb == o.nb &&
               n_members == o.n_members && one_carry == o.one_carry && chunked == o.chunked;
    }
};

// Per-member sizes: groups, tiles (4 per group), chunks, buckets, groups per chunk.
struct MemberShape {
    uint32_t ng, nt, nc, nb, cl;
};

uint32_t groups_for(int64_t n) { return (uint32_t)((n + kGroupSlots - 1) / kGroupSlots); }

MemberShape member_shape(int64_t n, const Tuning &tu)
{
    MemberShape m;
    m.ng = groups_for(n);
    m.nt = m.ng * kTilesPerGroup;
    if (tu.chunk > 0) {
        m.cl = (uint32_t)tu.chunk;
    } else {
        m.cl = kChunkMin;
        while (m.cl < (uint32_t)kChunkMax && (uint64_t)m.cl * kChunkTarget < m.ng) m.cl *= 2;
    }
    m.nc = (m.ng + m.cl - 1) / m.cl;
    m.nb = (uint32_t)std::max<int64_t>(1, n / tu.bucket);
    return m;
}

// Whether a member's carries run in one kernel (by the member alone: the two
// ways round differently).  A tuned chunk length asks for chunks.
bool takes_one_carry(const Tuning &tu, uint32_t ng)
{
    return tu.chunk == 0 && ng <= (uint32_t)kOneCarryGroups;
}

bool check_common(const sim_params *p, std::string *why)
{
    if (!p) { *why = "params is NULL"; return false; }
    if (p->struct_size != sizeof(sim_params)) { *why = "params struct_size mismatch"; return false; }
    if (p->l_max < 0 || p->l_max > kMaxL) { *why = "l_max must be in [0, 64]"; return false; }
    if (!(p->d > 0.0 && p->d < 1.0)) { *why = "d must be in (0, 1)"; return false; }
    if (!(p->eps_r > 0.0) || !std::isfinite(p->eps_r)) { *why = "eps_r must be > 0"; return false; }
    if (p->m_mode != SIM_M_FULL && p->m_mode != SIM_M_AXISYM) { *why = "bad m_mode"; return false; }
    if (p->precision != SIM_FP64 && p->precision != SIM_FP32_COMP) { *why = "bad precision"; return false; }
    if (p->tile != 0 && p->tile != kWave) { *why = "tile must be 0 or 64"; return false; }
    if (p->sort_bucket < 0 || p->sort_bucket > 256) { *why = "sort_bucket must be 0 or in [1, 256]"; return false; }
    if (p->sort_keys < -1 || p->sort_keys > 1) { *why = "sort_keys must be -1, 0 or 1"; return false; }
    if (p->near_split < -1 || p->near_split > 1) { *why = "near_split must be -1, 0 or 1"; return false; }
    if (p->carry_chunk != 0 && (p->carry_chunk < kChunkMin || p->carry_chunk > 1024)) {
        *why = "carry_chunk must be 0 or in [8, 1024]";
        return false;
    }
    return true;
}

// Scalar checks of a member (the particle arrays are checked at admission).
bool check_member_scalars(const sim_member *m, std::string *why)
{
    if (!m) { *why = "member is NULL"; return false; }
    if (m->struct_size != sizeof(sim_member)) { *why = "member struct_size mismatch"; return false; }
    if (m->n <= 0 || m->n > 0x7fffffffLL) { *why = "n must be in [1, 2^31)"; return false; }
    if (m->n_steps < 0) { *why = "n_steps < 0"; return false; }
    if (m->start_step < 0 || m->start_step > m->n_steps) {
        *why = "start_step outside [0, n_steps]";
        return false;
    }
    if (!(m->r_out > 1.0) || !std::isfinite(m->r_out)) { *why = "r_out must be > 1"; return false; }
    if (!(m->dt > 0.0) || !std::isfinite(m->dt)) { *why = "dt must be > 0"; return false; }
    if (!(m->ntilde > 0.0) || !std::isfinite(m->ntilde)) { *why = "ntilde must be > 0"; return false; }
    if (!(m->ion_density >= 0.0) || !std::isfinite(m->ion_density)) {
        *why = "ion_density must be >= 0";
        return false;
    }
    if (!std::isfinite(m->q_surface0)) { *why = "q_surface0 must be finite"; return false; }
    if (!(m->ion_mass >= 0.0) || !std::isfinite(m->ion_mass)) { *why = "ion_mass must be >= 0"; return false; }
    if (m->ion_profile && (m->ion_profile_len < 2 || m->ion_profile_len > (1 << 24))) {
        *why = "ion_profile_len must be in [2, 2^24]";
        return false;
    }
    if (m->probe_bc < SIM_BC_ABSORB || m->probe_bc > SIM_BC_DIFFUSE) { *why = "bad probe_bc"; return false; }
    if (m->wall_bc != SIM_BC_SPECULAR && m->wall_bc != SIM_BC_DIFFUSE) { *why = "bad wall_bc"; return false; }
    return true;
}

// chunks < 0: room for any mix of members (every tile in the shortest
// chunks, plus one partial chunk per member); else exactly that many.
bool make_layout(const sim_params *p, int64_t slots, int32_t max_members, int64_t chunks,
                 Layout *lo, std::string *why)
{
    if (!check_common(p, why)) return false;
    if (slots <= 0 || slots > 0x7fffffffLL - kGroupSlots) { *why = "slot capacity must be in [1, 2^31 - 256)"; return false; }
    if (max_members <= 0 || max_members > (1 << 20)) { *why = "max_members must be in [1, 2^20]"; return false; }
    lo->L = p->l_max;
    lo->full = p->m_mode == SIM_M_FULL;
    lo->fp32 = p->precision == SIM_FP32_COMP;
    lo->near64 = lo->fp32 && p->l_max >= kNear64MinL;
    lo->C = lo->full ? (p->l_max + 1) * (p->l_max + 1) - 1 : p->l_max;
    lo->C2 = 2 * lo->C;
    lo->n_groups = (int)groups_for(slots);
    lo->n_tiles = lo->n_groups * kTilesPerGroup;
    lo->n_members = max_members;
    lo->tu = tuning_of(p);
    // every member rounds its chunks and buckets up by at most one
    const int cl_min = lo->tu.chunk > 0 ? lo->tu.chunk : kChunkMin;
    lo->n_chunks = chunks >= 0 ? (int)std::max<int64_t>(1, chunks)
                               : (lo->n_groups + cl_min - 1) / cl_min + max_members;
    lo->nb = (int)std::max<int64_t>(1, slots / lo->tu.bucket) + (max_members > 1 ? max_members : 0);
    lo->nb_blocks = (lo->nb + kScanPerBlock - 1) / kScanPerBlock;
    return true;
}

struct Alloc {
    std::vector<std::pair<void **, size_t>> items;
    template <class T> void add(T **ptr, size_t count) { items.push_back({(void **)ptr, count * sizeof(T)}); }
    size_t total() const {
        size_t s = 0;
        for (auto &it : items) s += (it.second + 255) & ~size_t(255);
        return s;
    }
};

// Bytes of a member's arrays in the batch's data pool: drive and response
// (8 B per step each) and, with an ion profile of prof_len nodes, its node
// densities and enclosed charges (16 B per node), each 256-byte aligned.
constexpr size_t kPoolUnit = 256;

size_t align_unit(size_t b) { return (b + kPoolUnit - 1) & ~(kPoolUnit - 1); }

size_t member_bytes(int64_t n_steps, int64_t prof_len)
{
    return 2 * align_unit((size_t)std::max<int64_t>(n_steps, 1) * 8) +
           (prof_len > 0 ? align_unit((size_t)prof_len * 16) : 0);
}

// First-fit allocator of ranges [start, start + len) of a capacity.
class Ranges {
public:
    void reset(uint32_t capacity)
    {
        free_.clear();
        if (capacity) free_[0] = capacity;
    }
    bool take(uint32_t len, uint32_t *start)
    {
        for (auto it = free_.begin(); it != free_.end(); ++it) {
            if (it->second >= len) {
                *start = it->first;
                const uint32_t rest = it->second - len, at = it->first + len;
                free_.erase(it);
                if (rest) free_[at] = rest;
                return true;
            }
        }
        return false;
    }
    void give(uint32_t start, uint32_t len)
    {
        auto it = free_.emplace(start, len).first;
        auto nx = std::next(it);
        if (nx != free_.end() && it->first + it->second == nx->first) {
            it->second += nx->second;
            free_.erase(nx);
        }
        if (it != free_.begin()) {
            auto pv = std::prev(it);
            if (pv->first + pv->second == it->first) {
                pv->second += it->second;
                free_.erase(it);
            }
        }
    }

private:
    std::map<uint32_t, uint32_t> free_;
};

struct Member {
    bool used = false;
    Seg seg{};
    uint32_t md_start = 0, md_units = 0;   // the member's range of the data pool
    int64_t n = 0;
    int64_t step_host = 0;    // absolute step after all enqueued work
    int64_t start_step = 0;
    double q_surface0 = 0.0;
    std::vector<std::pair<uint32_t, int64_t>> id_index;  // (uid, creation index), sorted
    bool ids_are_indices = false;   // ids 0..n-1 in creation order
};

}  // namespace

struct sim {
    sim_params prm;
    Layout lo;
    Extent ext;
    KParams kp;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    hipStream_t cap_stream = nullptr;
    PRec *A = nullptr;
    State B{};
    Grave G{};
    uint8_t *dead = nullptr;
    KeyRec *krec = nullptr;
    OrdRec *orec = nullptr;
    uint32_t *hist = nullptr, *off = nullptr, *bsum = nullptr;
    double *H = nullptr, *GS = nullptr, *chunkS = nullptr, *chunkC = nullptr, *T = nullptr,
           *CR = nullptr, *tables = nullptr, *Eout = nullptr, *qpre = nullptr;
    int *chl = nullptr;
    double *chn = nullptr, *chg = nullptr;
    float *tables32 = nullptr;
    uint32_t *Eid = nullptr;
    Seg *seg = nullptr;
    Ctl *ctl = nullptr;
    uint32_t *tile_member = nullptr, *chunk_member = nullptr;
    Tables tb{};
    Map map{};
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    bool failed = false;
    bool keys_needed = true;   // some running member has no sort keys for its next step
    size_t shared_bytes = 0;
    // one device allocation holds every array, the members' data pool last
    sim_allocator alloc{};      // caller's callbacks, or all NULL (hipMalloc / hipFree)
    void *arena = nullptr;
    size_t arena_bytes = 0;
    char *mdata = nullptr;      // members' drive, response and ion-profile arrays
    std::vector<Member> members;
    Ranges groups, chunks, buckets, mdata_units;   // mdata_units: 256-byte units of mdata
};

namespace {

#define HIP_TRY(expr)                                                                 \
    do {                                                                              \
        hipError_t e_ = (expr);                                                       \
        if (e_ != hipSuccess) {                                                       \
            return fail(SIM_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
        }                                                                             \
    } while (0)

void plan_alloc(sim *h, Alloc &al, size_t pool_bytes)
{
    const Layout &lo = h->lo;
    const size_t n = (size_t)lo.n_tiles * kWave;
    al.add(&h->A, n);
    // (three columns in one array each: a state read uses them as one [3n]; see carve)
    al.add(&h->B.x, 3 * n);
    al.add(&h->B.vx, 3 * n);
    al.add(&h->B.uid, n);
    al.add(&h->G.x, n); al.add(&h->G.y, n); al.add(&h->G.z, n);
    al.add(&h->G.vx, n); al.add(&h->G.vy, n); al.add(&h->G.vz, n);
    al.add(&h->G.uid, n);
    al.add(&h->dead, n);
    al.add(&h->krec, n);
    al.add(&h->orec, n);
    al.add(&h->hist, (size_t)lo.nb + 1);
    al.add(&h->off, (size_t)lo.nb + 1);
    al.add(&h->bsum, (size_t)lo.nb_blocks + 1);
    al.add(&h->H, (size_t)lo.n_tiles * (4 * lo.C + 2));
    al.add(&h->GS, (size_t)lo.n_groups * (lo.C2 + 1));
    al.add(&h->CR, (size_t)lo.n_groups * std::max(lo.C2, 1));
    al.add(&h->qpre, (size_t)lo.n_groups);
    al.add(&h->tables32, tables32_len(lo.L));
    al.add(&h->chunkS, (size_t)lo.n_chunks * (lo.C2 + 1));
    al.add(&h->chunkC, (size_t)lo.n_chunks * (lo.C2 + 1));
    al.add(&h->T, (size_t)lo.n_members * std::max(lo.C, 1));
    al.add(&h->tables, tables_len(lo.L));
    al.add(&h->chl, (size_t)std::max(lo.C, 1));
    al.add(&h->chn, (size_t)std::max(lo.C, 1));
    al.add(&h->chg, (size_t)std::max(lo.C, 1));
    al.add(&h->Eout, 3 * n);
    al.add(&h->Eid, n);
    al.add(&h->seg, (size_t)lo.n_members);
    al.add(&h->ctl, (size_t)lo.n_members);
    al.add(&h->tile_member, (size_t)lo.n_tiles);
    al.add(&h->chunk_member, (size_t)lo.n_chunks);
    al.add(&h->mdata, std::max<size_t>(pool_bytes, kPoolUnit));
}

// Cuts the orders m = 0..top into ns slices [out[s], out[s + 1]) of near-equal
// work: the (l, m) pairs of an order (m = 0 has half the channels), and about
// one pair's worth for its start (the walk to a slice's first order, half a
// pair per step, is left out).
void cut_orders(int L, int top, int ns, uint8_t *out)
{
    auto cost = [&](int m) { return m == 0 ? 0.6 * L + 1.0 : L - m + 2.0; };
    auto cut = [&](double most, uint8_t *o) {
        int s = 0;
        double sum = 0.0;
        o[0] = 0;
        for (int m = 0; m <= top; ++m) {
            if (sum > 0.0 && sum + cost(m) > most) {
                if (++s >= ns) return false;
                o[s] = (uint8_t)m;
                sum = 0.0;
            }
            sum += cost(m);
        }
        while (s < ns) o[++s] = (uint8_t)(top + 1);
        return true;
    };
    double lo = 0.0, hi = 0.0;   // the smallest largest slice, by bisection
    for (int m = 0; m <= top; ++m) {
        lo = std::max(lo, cost(m));
        hi += cost(m);
    }
    uint8_t tmp[kMaxMSlices + 1];
    for (int it = 0; it < 12; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (cut(mid, tmp)) hi = mid;
        else lo = mid;
    }
    cut(hi, out);
}

// The moments kernel's slices; returns its blocks per group: a slice per wave
// of one block, and more blocks per group while the groups alone leave the
// chip's 256 CUs idle (each slice repeats the particles' loads and powers, so
// no more than that).
unsigned slice_orders(const Layout &lo, int n_groups, uint8_t *m_slice)
{
    const int top = lo.full ? lo.L : 0;   // the last order
    int ny = 1;
    while (lo.full && ny * kWavesPerBlock < kMaxMSlices && 2 * ny * kWavesPerBlock <= top &&
           n_groups * ny < 512)
        ny *= 2;
    cut_orders(lo.L, top, ny * kWavesPerBlock, m_slice);
    return (unsigned)ny;
}

// Up to this many tiles the field kernel takes a block per tile: a chip's worth
// of waves hides the latencies that one wave per SIMD cannot, until the
// repeated setup of four waves per tile costs more; later with a near field in
// FP64, whose groups' blocks hold fewer waves per SIMD.  Field kernel, blocks of
// groups and of tiles, in us.  FP64: l_max 3 85,000 particles 20.2 / 19.5,
// 100,000 21.0 / 22.0; l_max 8 200,000 42.3 / 40.4, 240,000 42.9 / 44.4; l_max 16
// 10,000 37.6 / 16.4, 300,000 96 / 86, 450,000 121 / 121; l_max 32 600,000 418 /
// 383, l_max 48 1,000,000 1444 / 1309; l_max 64 1,300,000 2939 / 2682.  FP32 with the near
// field in FP64: l_max 24 400,000 158 / 151, 600,000 219 / 224; l_max 32 700,000 476 / 452;
// l_max 48 1,000,000 1260 / 1232; l_max 64 1,300,000 2374 / 2420.  FP32: l_max 3 115,000 20.8 / 22.6; l_max 8
// 200,000 33.5 / 36.0; l_max 16 300,000 68.3 / 70.0.
int split_max_tiles(int L, bool near_fp32) { return near_fp32 ? 600 + 200 * L : 400 + 350 * L; }

// The push prepares the next step's sort keys unless told otherwise.
bool keys_in_push(const sim *h) { return h->lo.tu.keys >= 0; }

// The kernels' parameters for the extent in use.
KParams step_params(const sim *h, bool field_only)
{
    const Extent &ex = h->ext;
    KParams kp = h->kp;
    kp.field_only = field_only ? 1 : 0;
    kp.fuse_keys = keys_in_push(h) ? 1 : 0;
    kp.n_tiles = ex.n_tiles;
    kp.n_groups = ex.n_tiles / kTilesPerGroup;
    kp.n_chunks = ex.n_chunks;
    kp.nb = ex.nb;
    kp.n_members = ex.n_members;
    return kp;
}

// Sort keys of the members whose push did not prepare them.
void launch_keys(sim *h, hipStream_t s, const KParams &kp)
{
    const unsigned n = (unsigned)h->ext.n_tiles * kWave;
    k_sort_key<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(h->map, h->A, h->dead, h->krec, h->hist,
                                                            kp);
}

// An event before each kernel kind and after the last, and which kinds a step
// launched (between the events of one that it did not, only their own time passes).
struct Marks {
    hipEvent_t ev[KN_COUNT + 1];
    bool ran[KN_COUNT];
};

// One step (or field evaluation).  with_keys: the key kernel comes first; not
// needed where every running member's last push prepared its keys.
int launch_step(sim *h, hipStream_t s, bool field_only, bool with_keys, Marks *marks)
{
    const Layout &lo = h->lo;
    const Extent &ex = h->ext;
    KParams kp = step_params(h, field_only);
    const Map &mp = h->map;
    const unsigned n = (unsigned)ex.n_tiles * kWave;
    const unsigned gN = (n + kBlock - 1) / kBlock;
    const unsigned gT = (unsigned)(ex.n_tiles / kTilesPerGroup);   // one block per group
    const unsigned gC = (unsigned)((lo.C2 + 1 + kBlock - 1) / kBlock);   // group-sum columns
    int e = 0;
    auto mark = [&](int k, bool launched) {
        if (marks) (void)hipEventRecord(marks->ev[k], s);
        if (marks) marks->ran[k] = launched;
        return launched;
    };
    if (mark(KN_SORT_KEY, with_keys)) launch_keys(h, s, kp);
    const bool fused = lo.tu.bucket <= kPlaceMaxBucket;
    const bool lds_scan = fused && ex.nb <= kScanLdsBuckets;
    if (mark(KN_SCAN_A, !lds_scan))
        k_scan_a<<<ex.nb_blocks, kBlock, 0, s>>>(mp, kp, h->hist, h->bsum, ex.nb);
    if (mark(KN_SCAN_C, !lds_scan))
        k_scan_c<<<ex.nb_blocks, kBlock, 0, s>>>(h->hist, h->bsum, h->off, ex.nb);
    mark(KN_SORT_SCATTER, true);
    if (lds_scan)
        k_sort_scatter<true><<<gN, kBlock, 0, s>>>(mp, h->krec, h->hist, h->off, h->orec, kp);
    else
        k_sort_scatter<false><<<gN, kBlock, 0, s>>>(mp, h->krec, h->hist, h->off, h->orec, kp);
    if (mark(KN_SORT_RANK, !fused))
        k_sort_rank_move<<<gN, kBlock, 0, s>>>(mp, h->orec, h->off, h->A, h->B, kp);
    mark(KN_MOMENTS, true);
    const unsigned gS = slice_orders(lo, (int)gT, kp.m_slice);
#define MRP_MOMENTS(FULLV, RANKV)                                                       \
    k_moments<FULLV, RANKV><<<dim3(gT, gS), kBlock, 0, s>>>(mp, h->orec, h->off, h->A, h->B, \
                                                            h->tb, kp, h->H, h->GS, h->hist, \
                                                            lds_scan ? ex.nb : 0)
    if (lo.full) {
        if (fused) MRP_MOMENTS(true, true);
        else MRP_MOMENTS(true, false);
    } else {
        if (fused) MRP_MOMENTS(false, true);
        else MRP_MOMENTS(false, false);
    }
#undef MRP_MOMENTS
    if (mark(KN_CHUNK_SUMS, ex.chunked))
        k_chunk_sums<<<dim3(ex.n_chunks, gC), kBlock, 0, s>>>(mp, h->GS, h->chunkS, kp);
    const unsigned n_cols = ex.chunked ? (lo.C2 + 1 + kWavesPerBlock - 1) / kWavesPerBlock : 0;
    const unsigned n_one = ex.one_carry ? one_carry_blocks(lo.C) : 0;
    if (mark(KN_CHUNK_SCAN, n_cols + n_one > 0))   // none in a handle without members
        k_chunk_scan<<<dim3(n_cols + n_one, ex.n_members), kBlock, 0, s>>>(
            mp, h->chunkS, h->chunkC, h->T, h->tb, kp, (int)n_cols, h->GS, h->CR, h->qpre);
    if (mark(KN_CHUNK_APPLY, ex.chunked))
        k_chunk_apply<<<dim3(ex.n_chunks, gC), kBlock, 0, s>>>(mp, h->GS, h->chunkC, h->T, h->tb,
                                                               kp, h->CR, h->qpre);
    mark(KN_FIELD_PUSH, true);
    const bool split = lo.full && ex.n_tiles <= split_max_tiles(lo.L, lo.fp32 && !lo.near64);
    uint8_t cuts[kMaxMSlices + 1];
    cut_orders(lo.L, lo.L, kWavesPerBlock, cuts);
    kp.f_ends = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) kp.f_ends |= (uint32_t)cuts[i + 1] << (8 * i);
    auto field = [&](auto full, auto fo, auto f32, auto n64, auto spl) {
        constexpr bool kSplit = decltype(spl)::value;
        k_field_push<decltype(full)::value, decltype(fo)::value, decltype(f32)::value,
                     decltype(n64)::value, kSplit>
            <<<kSplit ? (unsigned)ex.n_tiles : gT, kBlock, 0, s>>>(
                mp, h->B, h->A, h->dead, h->G, h->H, h->CR, h->qpre, h->tb, kp, h->Eout, h->Eid,
                h->krec, h->hist);
    };
    const std::true_type yes;
    const std::false_type no;
    auto by_precision = [&](auto fo, auto spl) {
        if (lo.near64) field(yes, fo, yes, yes, spl);
        else if (lo.fp32) field(yes, fo, yes, no, spl);
        else field(yes, fo, no, no, spl);
    };
    auto by_form = [&](auto fo) {
        if (!lo.full) {
            if (lo.fp32) field(no, fo, yes, no, no);
            else field(no, fo, no, no, no);
        } else if (split) {
            by_precision(fo, yes);
        } else {
            by_precision(fo, no);
        }
    };
    if (field_only) by_form(yes);
    else by_form(no);
    mark(KN_STEP_FINISH, false);   // part of the sort and the moments
    if (marks) (void)hipEventRecord(marks->ev[KN_COUNT], s);
    hipError_t le = hipGetLastError();
    if (le != hipSuccess) e = fail(SIM_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(le));
    return e;
}

// Give a member's range of the data pool back (no device call).
void free_member_arrays(sim *h, Member &m)
{
    if (m.md_units) h->mdata_units.give(m.md_start, m.md_units);
    m.md_units = 0;
    m.seg.u_asy = nullptr;
    m.seg.qdiff = nullptr;
    m.seg.ion_tab = nullptr;
}

// The handle's work completes before its graph and memory go: the stream is
// drained first.
void release(sim *h)
{
    if (!h) return;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    if (h->graph) (void)hipGraphDestroy(h->graph);
    h->exec = nullptr;
    h->graph = nullptr;
    if (h->arena) {
        void *as = h->own_stream ? nullptr : (void *)h->stream;   // the stream given to alloc
        if (h->alloc.free) h->alloc.free(h->alloc.ctx, h->arena, h->arena_bytes, as);
        else (void)hipFree(h->arena);
    }
    h->arena = nullptr;
    if (h->cap_stream) (void)hipStreamDestroy(h->cap_stream);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    h->cap_stream = nullptr;
    h->stream = nullptr;
}

int check_handle(sim *h)
{
    if (!h) return fail(SIM_ESTATE, "NULL handle");
    if (h->failed) return fail(SIM_ESTATE, "handle is in the failed state");
    return SIM_OK;
}

int mark_failed(sim *h, int code)
{
    if (code == SIM_EDEVICE) h->failed = true;
    return code;
}

// A member's control block (the handle's stream is idle).
int read_ctl(sim *h, int32_t index, Ctl *c)
{
    if (hipMemcpy(c, h->ctl + index, sizeof(Ctl), hipMemcpyDeviceToHost) != hipSuccess)
        return mark_failed(h, fail(SIM_EDEVICE, "copy of control block failed"));
    return SIM_OK;
}

int check_member_index(sim *h, int32_t index)
{
    if (index < 0 || index >= (int32_t)h->members.size() || !h->members[index].used)
        return fail(SIM_ERANGE, "no member at index " + std::to_string(index));
    return SIM_OK;
}

TableDst table_dst(const sim *h, const sim_params &p)
{
    return TableDst{h->tables, h->tables32, h->chl, h->chn, h->chg, p.d, p.eps_r, h->lo.L, h->lo.C};
}

// Point the kernels' table, parameter and map views at the handle's carved
// arrays (its layout set).
void bind_device_tables(sim *h)
{
    const Layout &lo = h->lo;
    const int L = lo.L;
    double *tb = h->tables;
    h->tb.ftil = tb;
    h->tb.wl = tb + (L + 1);
    h->tb.drive_w = tb + 2 * (L + 1);
    h->tb.self_w = tb + 3 * (L + 1);
    h->tb.self_w1 = tb + 4 * (L + 1);
    h->tb.nf4 = reinterpret_cast<const double4 *>(tb + nf4_offset(L));
    h->tb.lg4 = reinterpret_cast<const double4 *>(tb + lg4_offset(L));
    h->tb.fq4 = reinterpret_cast<const double4 *>(tb + fq4_offset(L));
    h->tb.chn = h->chn;
    h->tb.chl = h->chl;
    h->tb.chg = h->chg;
    h->tb.fq4_32 = reinterpret_cast<const float4 *>(h->tables32 + fq4_32_offset(L));
    h->tb.lw4_32 = reinterpret_cast<const float4 *>(h->tables32 + lw4_32_offset(L));
    KParams &kp = h->kp;
    kp.L = lo.L;
    kp.C = lo.C;
    kp.C2 = lo.C2;
    kp.SW = lo.C2 + 1;
    kp.HW = 4 * lo.C + 2;
    kp.n_tiles = lo.n_tiles;
    kp.n_groups = lo.n_groups;
    kp.n_chunks = lo.n_chunks;
    kp.nb = lo.nb;
    kp.n_members = lo.n_members;
    kp.field_only = 0;
    kp.fuse_keys = 0;
    h->map.seg = h->seg;
    h->map.ctl = h->ctl;
    h->map.tile_member = h->tile_member;
    h->map.chunk_member = h->chunk_member;
}

// Carve the arrays of plan_alloc out of one block at base, in order, each
// 256-byte aligned.
void carve(sim *h, Alloc &al, void *base)
{
    char *at = static_cast<char *>(base);
    for (auto &it : al.items) {
        *it.first = at;
        at += align_unit(it.second);
    }
    const size_t n = (size_t)h->lo.n_tiles * kWave;
    h->B.y = h->B.x + n;
    h->B.z = h->B.y + n;
    h->B.vy = h->B.vx + n;
    h->B.vz = h->B.vy + n;
}

// Allocate the arena (the shared arrays and the members' data pool, in one
// allocation from the caller's allocator or hipMalloc), upload the tables.
int engine_init(sim *h, const sim_params *p, const Layout &lo, void *hip_stream,
                const sim_allocator *alloc, size_t pool_bytes)
{
    h->prm = *p;
    h->lo = lo;
    if (alloc) {
        if (!alloc->alloc || !alloc->free)
            return fail(SIM_EINVAL, "sim_allocator needs both alloc and free");
        h->alloc = *alloc;
    }
    Alloc al;
    plan_alloc(h, al, pool_bytes);
    h->shared_bytes = al.total();
    if (p->mem_limit_bytes && h->shared_bytes > p->mem_limit_bytes)
        return fail(SIM_ENOMEM, "footprint " + std::to_string(h->shared_bytes) +
                                    " B exceeds mem_limit_bytes");
    // the arena first (before any stream exists: a caller's allocator that
    // fails leaves no device state behind); its stream is the caller's, or
    // NULL when the handle runs on a stream of its own
    h->arena_bytes = h->shared_bytes;
    if (h->alloc.alloc) {
        h->arena = h->alloc.alloc(h->alloc.ctx, h->arena_bytes, hip_stream);
        if (!h->arena) return fail(SIM_ENOMEM, "the caller's allocator returned NULL");
        if (reinterpret_cast<uintptr_t>(h->arena) % kPoolUnit) {
            h->alloc.free(h->alloc.ctx, h->arena, h->arena_bytes, hip_stream);
            h->arena = nullptr;
            return fail(SIM_EINVAL, "the caller's allocator must return 256-byte aligned memory");
        }
    } else {
        hipError_t e = hipMalloc(&h->arena, h->arena_bytes);
        if (e != hipSuccess) {
            h->arena = nullptr;
            return fail(SIM_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        }
    }
    carve(h, al, h->arena);
    h->mdata_units.reset((uint32_t)(std::max<size_t>(pool_bytes, kPoolUnit) / kPoolUnit));
    if (hip_stream) {
        h->stream = (hipStream_t)hip_stream;
    } else {
        if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess)
            return fail(SIM_EDEVICE, "hipStreamCreate failed");
        h->own_stream = true;
    }
    if (hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking) != hipSuccess)
        return fail(SIM_EDEVICE, "hipStreamCreate failed");

    bind_device_tables(h);
    h->groups.reset((uint32_t)lo.n_groups);
    h->chunks.reset((uint32_t)lo.n_chunks);
    h->buckets.reset((uint32_t)lo.nb);
    h->members.assign((size_t)lo.n_members, Member());

    std::vector<Seg> segs((size_t)lo.n_members);   // used = 0
    std::vector<Ctl> ctls((size_t)lo.n_members);
    std::vector<uint32_t> none_t((size_t)lo.n_tiles, kNone), none_c((size_t)lo.n_chunks, kNone);
    k_tables<<<kTableBlocks, kBlock, 0, h->stream>>>(table_dst(h, *p));
    if (hipGetLastError() != hipSuccess ||
        hipMemcpy(h->seg, segs.data(), sizeof(Seg) * segs.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->ctl, ctls.data(), sizeof(Ctl) * ctls.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->tile_member, none_t.data(), 4 * none_t.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->chunk_member, none_c.data(), 4 * none_c.size(), hipMemcpyHostToDevice) ||
        hipMemset(h->dead, 0, (size_t)lo.n_tiles * kWave) ||
        hipMemset(h->hist, 0, sizeof(uint32_t) * ((size_t)lo.nb + 1)))
        return fail(SIM_EDEVICE, "upload failed");

    if (hipDeviceSynchronize() != hipSuccess) return fail(SIM_EDEVICE, "device sync failed");
    return SIM_OK;
}

// Recompute the extent in use and, when it changed (or no graph exists yet),
// capture one step into a new graph.  The handle's stream is idle here.
int update_graph(sim *h)
{
    Extent ex;
    for (int32_t k = 0; k < (int32_t)h->members.size(); ++k) {
        const Member &m = h->members[k];
        if (!m.used) continue;
        ex.n_tiles = std::max(ex.n_tiles, (int)(m.seg.t0 + m.seg.nt));
        ex.n_chunks = std::max(ex.n_chunks, (int)(m.seg.c0 + m.seg.nc));
        ex.nb = std::max(ex.nb, (int)(m.seg.b0 + m.seg.nb));
        ex.n_members = std::max(ex.n_members, k + 1);
        (m.seg.one_carry ? ex.one_carry : ex.chunked) = true;
    }
    ex.nb_blocks = (ex.nb + kScanPerBlock - 1) / kScanPerBlock;
    if (h->exec && ex == h->ext) return SIM_OK;
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    if (h->graph) (void)hipGraphDestroy(h->graph);
    h->exec = nullptr;
    h->graph = nullptr;
    h->ext = ex;
    if (hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return mark_failed(h, fail(SIM_EDEVICE, "hipStreamBeginCapture failed"));
    int le = launch_step(h, h->cap_stream, false, !keys_in_push(h), nullptr);
    hipError_t ce = hipStreamEndCapture(h->cap_stream, &h->graph);
    if (le != SIM_OK) return mark_failed(h, le);
    if (ce != hipSuccess)
        return mark_failed(h, fail(SIM_EDEVICE, std::string("capture: ") + hipGetErrorString(ce)));
    if (hipGraphInstantiate(&h->exec, h->graph, nullptr, nullptr, 0) != hipSuccess)
        return mark_failed(h, fail(SIM_EDEVICE, "hipGraphInstantiate failed"));
    return SIM_OK;
}

// A member's host-side data after validation: ids and the id -> creation
// index map.
struct Prepared {
    std::vector<uint32_t> uid;
    std::vector<std::pair<uint32_t, int64_t>> idx;
    bool ids_are_indices = false;
};

// Validate a member completely (no device work).
int prepare_member(const sim_member *m, Prepared *pr)
{
    std::string why;
    if (!check_member_scalars(m, &why)) return fail(SIM_EINVAL, why);
    const int64_t n = m->n;
    if (!m->pos || !m->vel) return fail(SIM_EINVAL, "pos and vel are required");
    if (m->n_steps > 0 && !m->u_asy) return fail(SIM_EINVAL, "u_asy is required when n_steps > 0");
    for (int64_t i = 0; i < n; ++i) {
        const double *x = m->pos + 3 * i, *v = m->vel + 3 * i;
        for (int j = 0; j < 3; ++j)
            if (!std::isfinite(x[j]) || !std::isfinite(v[j]))
                return fail(SIM_EINVAL, "non-finite particle state at index " + std::to_string(i));
        const double r = std::sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
        if (!(r > 1.0 && r < m->r_out))
            return fail(SIM_EINVAL, "particle " + std::to_string(i) + " not inside 1 < r < r_out");
    }
    for (int64_t s = 0; s < m->n_steps; ++s)
        if (!std::isfinite(m->u_asy[s])) return fail(SIM_EINVAL, "non-finite u_asy");
    if (m->ion_profile)
        for (int64_t j = 0; j < m->ion_profile_len; ++j)
            if (!std::isfinite(m->ion_profile[j]) || m->ion_profile[j] < 0.0)
                return fail(SIM_EINVAL, "ion_profile values must be finite and >= 0");
    pr->uid.resize((size_t)n);
    pr->ids_are_indices = true;
    for (int64_t i = 0; i < n; ++i) {
        pr->uid[i] = m->ids ? m->ids[i] : (uint32_t)i;
        if (pr->uid[i] != (uint32_t)i) pr->ids_are_indices = false;
    }
    if (!(m->ion_mass > 0.0))
        for (int64_t i = 0; i < n; ++i)
            if (pr->uid[i] & kIonBit) return fail(SIM_EINVAL, "ion ids (bit 31) need ion_mass > 0");
    pr->idx.resize((size_t)n);
    for (int64_t i = 0; i < n; ++i) pr->idx[i] = {pr->uid[i], i};
    std::sort(pr->idx.begin(), pr->idx.end());
    for (int64_t i = 1; i < n; ++i)
        if (pr->idx[i].first == pr->idx[i - 1].first) return fail(SIM_EINVAL, "ids are not distinct");
    return SIM_OK;
}

// Place and upload one validated member.  On failure the handle is unchanged
// (apart from the device contents of free ranges).
int engine_add(sim *h, const sim_member *m, Prepared &pr, int32_t *index)
{
    const int64_t n = m->n;
    std::vector<uint32_t> &uid = pr.uid;
    int32_t slot = -1;
    for (int32_t k = 0; k < (int32_t)h->members.size(); ++k)
        if (!h->members[k].used) { slot = k; break; }
    if (slot < 0) return fail(SIM_ENOMEM, "member table is full");
    const size_t mbytes = member_bytes(m->n_steps, m->ion_profile ? m->ion_profile_len : 0);
    const uint32_t md_units = (uint32_t)(mbytes / kPoolUnit);
    const MemberShape sh = member_shape(n, h->lo.tu);
    uint32_t g0 = 0, c0 = 0, b0 = 0, md0 = 0;
    if (!h->groups.take(sh.ng, &g0)) return fail(SIM_ENOMEM, "no free slot range for the member");
    if (!h->chunks.take(sh.nc, &c0)) {
        h->groups.give(g0, sh.ng);
        return fail(SIM_ENOMEM, "no free chunk range for the member");
    }
    if (!h->buckets.take(sh.nb, &b0)) {
        h->groups.give(g0, sh.ng);
        h->chunks.give(c0, sh.nc);
        return fail(SIM_ENOMEM, "no free bucket range for the member");
    }
    if (!h->mdata_units.take(md_units, &md0)) {
        h->groups.give(g0, sh.ng);
        h->chunks.give(c0, sh.nc);
        h->buckets.give(b0, sh.nb);
        return fail(SIM_ENOMEM, "the batch's member data pool has no room for the member's "
                                "drive and response arrays");
    }
    Member mb;
    mb.md_start = md0;
    mb.md_units = md_units;
    mb.used = true;
    mb.n = n;
    mb.step_host = m->start_step;
    mb.start_step = m->start_step;
    mb.q_surface0 = m->q_surface0;
    mb.id_index = std::move(pr.idx);
    mb.ids_are_indices = pr.ids_are_indices;
    Seg &sg = mb.seg;
    const uint32_t t0 = g0 * kTilesPerGroup;
    sg.p0 = g0 * kGroupSlots;
    sg.cap = sh.ng * kGroupSlots;
    sg.t0 = t0;
    sg.nt = sh.nt;
    sg.g0 = g0;
    sg.ng = sh.ng;
    sg.c0 = c0;
    sg.nc = sh.nc;
    sg.cl = sh.cl;
    sg.b0 = b0;
    sg.nb = sh.nb;
    sg.inv_vol = 1.0 / (m->r_out * m->r_out * m->r_out - 1.0);
    sg.ntilde = m->ntilde;
    sg.inv_ntilde = 1.0 / m->ntilde;
    sg.ion_density = m->ion_density;
    sg.q_surface0 = m->q_surface0;
    sg.dt = m->dt;
    sg.r_out = m->r_out;
    sg.seed = m->seed;
    sg.probe_bc = m->probe_bc;
    sg.wall_bc = m->wall_bc;
    sg.n_steps = m->n_steps;
    sg.ion_qm = m->ion_mass > 0.0 ? 1.0 / m->ion_mass : 0.0;
    sg.near_w = near_width(h->lo.tu, h->lo.fp32, h->lo.L, n);
    sg.one_carry = takes_one_carry(h->lo.tu, sh.ng) ? 1 : 0;
    sg.used = 1;
    auto undo = [&](int code) {
        free_member_arrays(h, mb);
        h->groups.give(g0, sh.ng);
        h->chunks.give(c0, sh.nc);
        h->buckets.give(b0, sh.nb);
        return code;
    };
    const size_t ns = (size_t)std::max<int64_t>(m->n_steps, 1);
    char *md = h->mdata + (size_t)md0 * kPoolUnit;
    double *u_dev = reinterpret_cast<double *>(md);
    double *q_dev = reinterpret_cast<double *>(md + align_unit(8 * ns));
    sg.u_asy = u_dev;
    sg.qdiff = q_dev;
    std::vector<double> ion_tab;
    if (m->ion_profile) {
        // node densities, then the enclosed charge at every node, segment by
        // segment in closed form (the same expression as the field kernel at
        // dd = h)
        const int64_t K = m->ion_profile_len - 1;
        const double h = (m->r_out - 1.0) / (double)K;
        ion_tab.assign(2 * (size_t)(K + 1), 0.0);
        for (int64_t j = 0; j <= K; ++j) ion_tab[j] = m->ion_profile[j];
        double q = 0.0;
        for (int64_t j = 0; j < K; ++j) {
            ion_tab[K + 1 + j] = q;
            const double rj = 1.0 + (double)j * h, dd = h, d2 = dd * dd;
            const double nj = m->ion_profile[j], beta = (m->ion_profile[j + 1] - nj) / h;
            const double seg = nj * (rj * rj * dd + rj * d2 + d2 * dd / 3.0) +
                               beta * (rj * rj * d2 / 2.0 + 2.0 * rj * d2 * dd / 3.0 + d2 * d2 / 4.0);
            q += 4.0 * kPi * m->ntilde * seg;
        }
        ion_tab[2 * K + 1] = q;
        sg.ion_tab = reinterpret_cast<double *>(md + 2 * align_unit(8 * ns));
        sg.ion_k = (int32_t)K;
        sg.ion_h = h;
        sg.ion_inv_h = (double)K / (m->r_out - 1.0);
    }

    if (hipStreamSynchronize(h->stream) != hipSuccess) {
        h->failed = true;
        return undo(fail(SIM_EDEVICE, "stream synchronisation failed"));
    }
    std::vector<PRec> recs((size_t)n);
    for (int64_t i = 0; i < n; ++i) {
        PRec &r = recs[i];
        r.x = m->pos[3 * i];
        r.y = m->pos[3 * i + 1];
        r.z = m->pos[3 * i + 2];
        r.vx = m->vel[3 * i];
        r.vy = m->vel[3 * i + 1];
        r.vz = m->vel[3 * i + 2];
        r.uid = uid[i];
        r.pad[0] = r.pad[1] = r.pad[2] = 0u;
    }
    Ctl ctl{};
    ctl.next_step = ctl.step = m->start_step;
    ctl.records = (uint32_t)n;
    ctl.n_live = (uint32_t)n;
    ctl.n_dead = 0;
    ctl.q_surface = m->q_surface0;
    std::vector<double> zeros(ns, 0.0);
    std::vector<uint32_t> tm(sh.nt, (uint32_t)slot), cm(sh.nc, (uint32_t)slot);
    if (hipMemcpy(h->A + sg.p0, recs.data(), sizeof(PRec) * n, hipMemcpyHostToDevice) ||
        hipMemset(h->dead + sg.p0, 0, sg.cap) ||
        hipMemcpy(q_dev, zeros.data(), 8 * ns, hipMemcpyHostToDevice) ||
        (m->n_steps > 0 && hipMemcpy(u_dev, m->u_asy, 8 * m->n_steps, hipMemcpyHostToDevice)) ||
        (!ion_tab.empty() && hipMemcpy((void *)sg.ion_tab, ion_tab.data(), 8 * ion_tab.size(),
                                       hipMemcpyHostToDevice)) ||
        hipMemcpy(h->ctl + slot, &ctl, sizeof(Ctl), hipMemcpyHostToDevice) ||
        hipMemcpy(h->tile_member + t0, tm.data(), 4 * tm.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->chunk_member + c0, cm.data(), 4 * cm.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->seg + slot, &sg, sizeof(Seg), hipMemcpyHostToDevice)) {
        h->failed = true;
        return undo(fail(SIM_EDEVICE, "member upload failed"));
    }
    h->members[slot] = std::move(mb);
    h->keys_needed = true;
    *index = slot;
    return SIM_OK;
}

int engine_remove(sim *h, int32_t index)
{
    int rc = check_member_index(h, index);
    if (rc) return rc;
    if (hipStreamSynchronize(h->stream) != hipSuccess) {
        h->failed = true;
        return fail(SIM_EDEVICE, "stream synchronisation failed");
    }
    Member &mb = h->members[index];
    Seg off{};   // used = 0
    std::vector<uint32_t> tm(mb.seg.nt, kNone), cm(mb.seg.nc, kNone);
    // the member's last push may have counted its particles into its buckets
    // for a next step; the buckets go back to the pool cleared
    if (hipMemcpy(h->seg + index, &off, sizeof(Seg), hipMemcpyHostToDevice) ||
        hipMemset(h->hist + mb.seg.b0, 0, sizeof(uint32_t) * mb.seg.nb) ||
        hipMemcpy(h->tile_member + mb.seg.t0, tm.data(), 4 * tm.size(), hipMemcpyHostToDevice) ||
        hipMemcpy(h->chunk_member + mb.seg.c0, cm.data(), 4 * cm.size(), hipMemcpyHostToDevice)) {
        h->failed = true;
        return fail(SIM_EDEVICE, "member table update failed");
    }
    free_member_arrays(h, mb);
    h->groups.give(mb.seg.g0, mb.seg.ng);
    h->chunks.give(mb.seg.c0, mb.seg.nc);
    h->buckets.give(mb.seg.b0, mb.seg.nb);
    mb = Member();
    return SIM_OK;
}

int enqueue_steps(sim *h, int64_t k)
{
    if (k > 0 && keys_in_push(h) && h->keys_needed) {
        launch_keys(h, h->stream, step_params(h, false));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            h->failed = true;
            return fail(SIM_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(e));
        }
        h->keys_needed = false;
    }
    for (int64_t i = 0; i < k; ++i) {
        hipError_t e = hipGraphLaunch(h->exec, h->stream);
        if (e != hipSuccess) {
            h->failed = true;
            return fail(SIM_EDEVICE, std::string("hipGraphLaunch: ") + hipGetErrorString(e));
        }
    }
    for (Member &m : h->members)
        if (m.used) m.step_host = std::min(m.step_host + k, m.seg.n_steps);
    return SIM_OK;
}

sim_member member_from_params(const sim_params *p, int64_t n, const double *pos, const double *vel,
                              const uint32_t *ids, const double *u_asy, int64_t n_steps,
                              int64_t start_step)
{
    sim_member m;
    std::memset(&m, 0, sizeof(m));
    m.struct_size = sizeof(sim_member);
    m.n = n;
    m.pos = pos;
    m.vel = vel;
    m.ids = ids;
    m.u_asy = u_asy;
    m.n_steps = n_steps;
    m.start_step = start_step;
    m.ntilde = p->ntilde;
    m.ion_density = p->ion_density;
    m.q_surface0 = p->q_surface0;
    m.r_out = p->r_out;
    m.dt = p->dt;
    m.seed = p->seed;
    m.probe_bc = p->probe_bc;
    m.wall_bc = p->wall_bc;
    return m;
}

int64_t slots_for(int64_t n) { return (int64_t)groups_for(n) * kGroupSlots; }

// ---------------------------------------------------------------------------
// Field evaluation without allocation: every working array in a static
// device buffer
// ---------------------------------------------------------------------------

// One buffer per GPU the library runs on, held until the process ends.
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;

}  // namespace

static __device__ __align__(256) char scratch[kScratchBytes];

namespace {

// Device address of this device's scratch (looked up once per device; the
// array's name in host code is a host-side stand-in, not this address).
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_address(void **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(SIM_EDEVICE, "device index out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(SIM_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") +
                                         hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SIM_OK;
}

// The tables and control words a one-member handle would hold before its
// first step, written by a kernel (the buffer keeps the previous call's
// contents): the member's description, its control block, the tile and chunk
// maps and the bucket histogram cleared, and the drive value of the evaluated
// step.
__global__ __launch_bounds__(kBlock) void k_static_setup(Seg sg, Ctl ct, Seg *seg, Ctl *ctl,
                                                         uint32_t *tile_member,
                                                         uint32_t *chunk_member, uint32_t *hist,
                                                         double *u_dev, double u_asy, int n_tiles,
                                                         int n_chunks, int nb)
{
    const int stride = gridDim.x * blockDim.x;
    const int i0 = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = i0; i < n_tiles; i += stride) tile_member[i] = 0;
    for (int i = i0; i < n_chunks; i += stride) chunk_member[i] = 0;
    for (int i = i0; i <= nb; i += stride) hist[i] = 0;
    if (i0 == 0) {
        seg[0] = sg;
        ctl[0] = ct;
        u_dev[0] = u_asy;
    }
}

// Particle records and sort keys from positions [3n] (particle-major), id =
// index; the blocks past the particles fill the constant tables beside them.
__global__ __launch_bounds__(kBlock) void k_static_pack(const double *pos, uint32_t n, PRec *A,
                                                        KeyRec *krec, uint32_t *hist,
                                                        double inv_vol, uint32_t nb, TableDst t)
{
    const uint32_t blocks = (n + kBlock - 1) / kBlock;
    if (blockIdx.x >= blocks) {
        fill_tables(t, (int)((blockIdx.x - blocks) * kBlock + threadIdx.x),
                    (int)(kTableBlocks * kBlock));
        return;
    }
    __shared__ uint32_t cnt[kWavesPerBlock][kSlotWindow];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = i < n;
    PRec r;
    KeyRec k{0ull, i, kNone};
    uint32_t b = 0;
    if (on) {
        r.x = pos[3 * (size_t)i];
        r.y = pos[3 * (size_t)i + 1];
        r.z = pos[3 * (size_t)i + 2];
        r.vx = r.vy = r.vz = 0.0;
        r.uid = i;
        r.pad[0] = r.pad[1] = r.pad[2] = 0u;
        A[i] = r;
        const double r2 = key_r2(r.x, r.y, r.z);
        k.key = (uint64_t)__double_as_longlong(r2);
        b = bucket_of(r2, inv_vol, 0, nb);
    }
    k.sub = take_slot(threadIdx.x & 63, on, b, hist, cnt[threadIdx.x >> 6]);
    if (on) krec[i] = k;
}

}  // namespace

extern "C" {

void sim_params_default(sim_params *p)
{
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->struct_size = sizeof(sim_params);
    p->d = 0.25;
    p->eps_r = 4.0;
    p->r_out = 5.0;
    p->dt = 0.05;
    p->ntilde = 1.0;
    p->ion_density = 1.0;
    p->q_surface0 = 0.0;
    p->l_max = 8;
    p->m_mode = SIM_M_FULL;
    p->probe_bc = SIM_BC_ABSORB;
    p->wall_bc = SIM_BC_SPECULAR;
    p->precision = SIM_FP64;
    p->tile = 0;
    p->seed = 0;
    p->mem_limit_bytes = 0;
}

void sim_member_default(sim_member *m)
{
    if (!m) return;
    sim_params p;
    sim_params_default(&p);
    *m = member_from_params(&p, 0, nullptr, nullptr, nullptr, nullptr, 0, 0);
}

}  // extern "C"

namespace {

int64_t footprint(const sim_params *common, int64_t slots, int32_t max_members, int64_t chunks,
                  size_t pool_bytes)
{
    Layout lo;
    std::string why;
    if (!make_layout(common, slots, max_members, chunks, &lo, &why)) return fail(SIM_EINVAL, why);
    sim tmp;
    tmp.lo = lo;
    Alloc al;
    plan_alloc(&tmp, al, pool_bytes);
    return (int64_t)al.total();
}

}  // namespace

extern "C" {

int64_t sim_member_data_bytes(int64_t n_steps, int64_t ion_profile_len)
{
    if (n_steps < 0 || ion_profile_len < 0) return fail(SIM_EINVAL, "negative size");
    return (int64_t)member_bytes(n_steps, ion_profile_len);
}

int64_t sim_batch_footprint_bytes(const sim_params *common, int64_t slot_capacity,
                                  int32_t max_members, int64_t member_data_bytes)
{
    if (member_data_bytes < 0) return fail(SIM_EINVAL, "member_data_bytes < 0");
    return footprint(common, slot_capacity, max_members, -1, align_unit((size_t)member_data_bytes));
}

int64_t sim_footprint_bytes(const sim_params *p, int64_t n, int64_t n_steps)
{
    std::string why;
    if (!check_common(p, &why)) return fail(SIM_EINVAL, why);
    sim_member m = member_from_params(p, n, nullptr, nullptr, nullptr, nullptr, n_steps, 0);
    if (!check_member_scalars(&m, &why)) return fail(SIM_EINVAL, why);
    return footprint(p, slots_for(n), 1, member_shape(n, tuning_of(p)).nc,
                     member_bytes(n_steps, 0));
}

int sim_batch_create(const sim_params *common, int64_t slot_capacity, int32_t max_members,
                     int64_t member_data_bytes, int32_t n_members, const sim_member *members,
                     void *hip_stream, const sim_allocator *alloc, sim_t **out)
{
    if (!out) return fail(SIM_EINVAL, "out is NULL");
    *out = nullptr;
    if (n_members < 0 || (n_members > 0 && !members)) return fail(SIM_EINVAL, "bad member list");
    if (member_data_bytes < 0) return fail(SIM_EINVAL, "member_data_bytes < 0");
    std::string why;
    if (!check_common(common, &why)) return fail(SIM_EINVAL, why);
    int64_t need = 0, chunks = 0;
    size_t pool_need = 0;
    std::vector<Prepared> prep((size_t)n_members);
    for (int32_t i = 0; i < n_members; ++i) {
        if (prepare_member(&members[i], &prep[i]))
            return fail(SIM_EINVAL, "member " + std::to_string(i) + ": " + g_last_error);
        need += slots_for(members[i].n);
        chunks += member_shape(members[i].n, tuning_of(common)).nc;
        pool_need += member_bytes(members[i].n_steps,
                                  members[i].ion_profile ? members[i].ion_profile_len : 0);
    }
    const size_t pool_bytes =
        member_data_bytes == 0 ? pool_need : align_unit((size_t)member_data_bytes);
    if (pool_bytes < pool_need)
        return fail(SIM_ENOMEM, "members need more member data bytes than member_data_bytes");
    // exactly the initial members, or room for any later mix
    const bool exact = slot_capacity == 0 && (max_members == 0 || max_members == n_members);
    if (max_members == 0) max_members = n_members;
    if (max_members < n_members) return fail(SIM_EINVAL, "max_members < n_members");
    if (slot_capacity == 0) slot_capacity = need;
    if (slot_capacity < need) return fail(SIM_ENOMEM, "members need more slots than slot_capacity");
    Layout lo;
    if (!make_layout(common, slot_capacity, max_members, exact ? chunks : -1, &lo, &why))
        return fail(SIM_EINVAL, why);
    sim *h = new (std::nothrow) sim();
    if (!h) return fail(SIM_ENOMEM, "host allocation failed");
    auto bail = [&](int code) {
        release(h);
        delete h;
        return code;
    };
    int rc = engine_init(h, common, lo, hip_stream, alloc, pool_bytes);
    if (rc) return bail(rc);
    for (int32_t i = 0; i < n_members; ++i) {
        int32_t idx = -1;
        rc = engine_add(h, &members[i], prep[i], &idx);
        if (rc) {
            const std::string msg = "member " + std::to_string(i) + ": " + g_last_error;
            bail(rc);
            return fail(rc, msg);
        }
    }
    rc = update_graph(h);
    if (rc) return bail(rc);
    *out = h;
    return SIM_OK;
}

int sim_create(const sim_params *p, int64_t n, const double *pos, const double *vel,
               const uint32_t *ids, const double *u_asy, int64_t n_steps, int64_t start_step,
               void *hip_stream, const sim_allocator *alloc, sim_t **out)
{
    if (!out) return fail(SIM_EINVAL, "out is NULL");
    *out = nullptr;
    std::string why;
    if (!check_common(p, &why)) return fail(SIM_EINVAL, why);
    sim_member m = member_from_params(p, n, pos, vel, ids, u_asy, n_steps, start_step);
    if (!check_member_scalars(&m, &why)) return fail(SIM_EINVAL, why);
    if (p->mem_limit_bytes) {
        const int64_t fp = sim_footprint_bytes(p, n, n_steps);
        if (fp > (int64_t)p->mem_limit_bytes)
            return fail(SIM_ENOMEM, "footprint " + std::to_string(fp) + " B exceeds mem_limit_bytes");
    }
    return sim_batch_create(p, 0, 1, 0, 1, &m, hip_stream, alloc, out);
}

int sim_batch_add(sim_t *h, const sim_member *m, int32_t *index)
{
    int rc = check_handle(h);
    if (rc) return rc;
    if (!index) return fail(SIM_EINVAL, "index is NULL");
    Prepared pr;
    rc = prepare_member(m, &pr);
    if (rc) return rc;
    rc = engine_add(h, m, pr, index);
    if (rc) return rc;
    return update_graph(h);
}

int sim_batch_remove(sim_t *h, int32_t index)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = engine_remove(h, index);
    if (rc) return rc;
    return update_graph(h);
}

int sim_step(sim_t *h, int64_t k)
{
    int rc = check_handle(h);
    if (rc) return rc;
    if (k < 0) return fail(SIM_EINVAL, "k < 0");
    for (const Member &m : h->members)
        if (m.used && m.step_host + k > m.seg.n_steps) return fail(SIM_ERANGE, "steps beyond n_steps");
    return enqueue_steps(h, k);
}

int sim_batch_step(sim_t *h, int64_t k)
{
    int rc = check_handle(h);
    if (rc) return rc;
    if (k < 0) return fail(SIM_EINVAL, "k < 0");
    int64_t left = 0;
    for (const Member &m : h->members)
        if (m.used) left = std::max(left, m.seg.n_steps - m.step_host);
    return enqueue_steps(h, std::min(k, left));
}

int sim_sync(sim_t *h)
{
    int rc = check_handle(h);
    if (rc) return rc;
    hipError_t e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        h->failed = true;
        return fail(SIM_EDEVICE, std::string("hipStreamSynchronize: ") + hipGetErrorString(e));
    }
    return SIM_OK;
}

int sim_query(sim_t *h)
{
    int rc = check_handle(h);
    if (rc) return rc;
    const hipError_t e = hipStreamQuery(h->stream);
    if (e == hipSuccess) return SIM_OK;
    if (e == hipErrorNotReady) return SIM_BUSY;
    h->failed = true;
    return fail(SIM_EDEVICE, std::string("hipStreamQuery: ") + hipGetErrorString(e));
}

int sim_member_info(sim_t *h, int32_t index, int64_t *n, int64_t *step, int64_t *n_steps)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = check_member_index(h, index);
    if (rc) return rc;
    const Member &m = h->members[index];
    if (n) *n = m.n;
    if (step) *step = m.step_host;
    if (n_steps) *n_steps = m.seg.n_steps;
    return SIM_OK;
}

int sim_member_read_response(sim_t *h, int32_t index, int64_t first, int64_t count, double *q_diff)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = check_member_index(h, index);
    if (rc) return rc;
    const Member &m = h->members[index];
    if (count == 0) return SIM_OK;
    if (!q_diff || count < 0 || first < m.start_step || first + count > m.step_host)
        return fail(SIM_ERANGE, "response range not computed");
    rc = sim_sync(h);
    if (rc) return rc;
    hipError_t e = hipMemcpy(q_diff, m.seg.qdiff + first, sizeof(double) * count, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return mark_failed(h, fail(SIM_EDEVICE, "copy of Q_diff failed"));
    return SIM_OK;
}

int sim_read_response(sim_t *h, int64_t first, int64_t count, double *q_diff)
{
    return sim_member_read_response(h, 0, first, count, q_diff);
}

int sim_member_read_state(sim_t *h, int32_t index, double *pos, double *vel, uint8_t *alive,
                          double *q_surface, int64_t *step)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = check_member_index(h, index);
    if (rc) return rc;
    rc = sim_sync(h);
    if (rc) return rc;
    const Member &mb = h->members[index];
    Ctl ctl;
    rc = read_ctl(h, index, &ctl);
    if (rc) return rc;
    const int64_t n = mb.n;
    const size_t p0 = mb.seg.p0;
    const size_t na = ctl.records & ~kKeyed, ng = ctl.n_dead;
    if (q_surface)
        *q_surface = (mb.q_surface0 + kQ * (double)(ctl.n_dead - ctl.n_dead_ion)) +
                     (double)ctl.n_dead_ion;
    if (step) *step = ctl.next_step;
    if (!pos && !vel && !alive) return SIM_OK;
    if (mb.ids_are_indices) {
        // Put in order on the device and copied once (a search per particle on
        // the host took 10 of the 11 ms that 100,117 particles needed: now 0.41
        // ms).  The sorted copy of the state, rewritten by the next step, is the
        // room: its three columns of all slots, one array, hold the member's [3n]
        // at 3 p0.
        const unsigned count = (unsigned)std::max(na, ng);
        double *dp = h->B.x + 3 * p0, *dv = h->B.vx + 3 * p0;
        uint8_t *da = reinterpret_cast<uint8_t *>(h->Eid + p0);
        hipStream_t st = h->stream;
        if (count)
            k_export_state<<<(count + kBlock - 1) / kBlock, kBlock, 0, st>>>(
                h->A, h->dead, (uint32_t)na, h->G, (uint32_t)p0, (uint32_t)ng, dp, dv, da);
        if (hipGetLastError() != hipSuccess ||
            (pos && hipMemcpyAsync(pos, dp, 24 * n, hipMemcpyDeviceToHost, st)) ||
            (vel && hipMemcpyAsync(vel, dv, 24 * n, hipMemcpyDeviceToHost, st)) ||
            (alive && hipMemcpyAsync(alive, da, n, hipMemcpyDeviceToHost, st)) ||
            hipStreamSynchronize(st) != hipSuccess)
            return mark_failed(h, fail(SIM_EDEVICE, "state copy failed"));
        return SIM_OK;
    }
    std::vector<double> a[6], g[6];
    std::vector<uint32_t> au(na), gu(ng);
    std::vector<uint8_t> ad(na);
    std::vector<PRec> ar(na);
    double *srcG[6] = {h->G.x, h->G.y, h->G.z, h->G.vx, h->G.vy, h->G.vz};
    for (int j = 0; j < 6; ++j) {
        g[j].resize(ng);
        if (ng && hipMemcpy(g[j].data(), srcG[j] + p0, 8 * ng, hipMemcpyDeviceToHost))
            return mark_failed(h, fail(SIM_EDEVICE, "state copy failed"));
    }
    if ((na && (hipMemcpy(ar.data(), h->A + p0, sizeof(PRec) * na, hipMemcpyDeviceToHost) ||
                hipMemcpy(ad.data(), h->dead + p0, na, hipMemcpyDeviceToHost))) ||
        (ng && hipMemcpy(gu.data(), h->G.uid + p0, 4 * ng, hipMemcpyDeviceToHost)))
        return mark_failed(h, fail(SIM_EDEVICE, "state copy failed"));
    for (int j = 0; j < 6; ++j) a[j].resize(na);
    for (size_t i = 0; i < na; ++i) {
        const PRec &r = ar[i];
        a[0][i] = r.x; a[1][i] = r.y; a[2][i] = r.z;
        a[3][i] = r.vx; a[4][i] = r.vy; a[5][i] = r.vz;
        au[i] = r.uid;
    }
    auto find = [&](uint32_t u) -> int64_t {
        auto it = std::lower_bound(mb.id_index.begin(), mb.id_index.end(),
                                   std::make_pair(u, (int64_t)-1));
        if (it == mb.id_index.end() || it->first != u) return -1;
        return it->second;
    };
    if (alive) std::memset(alive, 0, (size_t)n);
    auto put = [&](int64_t k, std::vector<double> *src, size_t i) {
        if (pos) for (int j = 0; j < 3; ++j) pos[3 * k + j] = src[j][i];
        if (vel) for (int j = 0; j < 3; ++j) vel[3 * k + j] = src[3 + j][i];
    };
    for (size_t i = 0; i < ng; ++i) {
        int64_t k = find(gu[i]);
        if (k < 0) return fail(SIM_EDEVICE, "unknown id in graveyard");
        put(k, g, i);
    }
    for (size_t i = 0; i < na; ++i) {
        if (ad[i]) continue;
        int64_t k = find(au[i]);
        if (k < 0) return fail(SIM_EDEVICE, "unknown id in state");
        put(k, a, i);
        if (alive) alive[k] = 1;
    }
    return SIM_OK;
}

int sim_member_counts(sim_t *h, int32_t index, int64_t *alive, int64_t *absorbed, int64_t *step)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = check_member_index(h, index);
    if (rc) return rc;
    rc = sim_sync(h);
    if (rc) return rc;
    Ctl ctl;
    rc = read_ctl(h, index, &ctl);
    if (rc) return rc;
    if (alive) *alive = h->members[index].n - (int64_t)ctl.n_dead;
    if (absorbed) *absorbed = (int64_t)ctl.n_dead;
    if (step) *step = ctl.next_step;
    return SIM_OK;
}

int sim_read_state(sim_t *h, double *pos, double *vel, uint8_t *alive, double *q_surface,
                   int64_t *step)
{
    return sim_member_read_state(h, 0, pos, vel, alive, q_surface, step);
}

int sim_member_eval_field(sim_t *h, int32_t index, double *E)
{
    int rc = check_handle(h);
    if (rc) return rc;
    rc = check_member_index(h, index);
    if (rc) return rc;
    if (!E) return fail(SIM_EINVAL, "E is NULL");
    h->keys_needed = true;   // the evaluation uses up the keys of the next step
    rc = launch_step(h, h->stream, true, true, nullptr);
    if (rc) return mark_failed(h, rc);
    rc = sim_sync(h);
    if (rc) return rc;
    const Member &mb = h->members[index];
    Ctl ctl;
    rc = read_ctl(h, index, &ctl);
    if (rc) return rc;
    const size_t nl = ctl.n_live, p0 = mb.seg.p0;
    std::vector<double> e(3 * nl);
    std::vector<uint32_t> u(nl);
    if (nl && (hipMemcpy(e.data(), h->Eout + 3 * p0, 8 * 3 * nl, hipMemcpyDeviceToHost) ||
               hipMemcpy(u.data(), h->Eid + p0, 4 * nl, hipMemcpyDeviceToHost)))
        return mark_failed(h, fail(SIM_EDEVICE, "field copy failed"));
    std::memset(E, 0, sizeof(double) * 3 * (size_t)mb.n);
    for (size_t i = 0; i < nl; ++i) {
        auto it = std::lower_bound(mb.id_index.begin(), mb.id_index.end(),
                                   std::make_pair(u[i], (int64_t)-1));
        if (it == mb.id_index.end() || it->first != u[i]) return fail(SIM_EDEVICE, "unknown id");
        for (int j = 0; j < 3; ++j) E[3 * it->second + j] = e[3 * i + j];
    }
    return SIM_OK;
}

int sim_eval_field(sim_t *h, double *E) { return sim_member_eval_field(h, 0, E); }

int64_t sim_eval_field_static_bytes(const sim_params *p, int64_t n)
{
    std::string why;
    if (!check_common(p, &why)) return fail(SIM_EINVAL, why);
    if (n <= 0 || n > 0x7fffffffLL) return fail(SIM_EINVAL, "n must be in [1, 2^31)");
    return footprint(p, slots_for(n), 1, member_shape(n, tuning_of(p)).nc, member_bytes(1, 0));
}

int sim_eval_field_static(const sim_params *p, int64_t n, const double *pos, double q_surface,
                          double u_asy, double *E, void *hip_stream)
{
    std::string why;
    if (!check_common(p, &why)) return fail(SIM_EINVAL, why);
    if (n <= 0 || n > 0x7fffffffLL) return fail(SIM_EINVAL, "n must be in [1, 2^31)");
    if (!pos || !E) return fail(SIM_EINVAL, "pos and E are required");
    if (!std::isfinite(q_surface) || !std::isfinite(u_asy))
        return fail(SIM_EINVAL, "q_surface and u_asy must be finite");
    sim_member m = member_from_params(p, n, nullptr, nullptr, nullptr, nullptr, 1, 0);
    if (!check_member_scalars(&m, &why)) return fail(SIM_EINVAL, why);
    const MemberShape sh = member_shape(n, tuning_of(p));
    // the same layout as sim_create's for these particles
    sim h;
    if (!make_layout(p, slots_for(n), 1, sh.nc, &h.lo, &why)) return fail(SIM_EINVAL, why);
    h.prm = *p;
    Alloc al;
    plan_alloc(&h, al, member_bytes(1, 0));
    if (al.total() > kScratchBytes)
        return fail(SIM_ENOMEM, "evaluation needs " + std::to_string(al.total()) +
                                    " B of working memory, more than the static buffer's " +
                                    std::to_string(kScratchBytes) + " B");
    void *base = nullptr;
    if (int rc = scratch_address(&base)) return rc;
    carve(&h, al, base);
    bind_device_tables(&h);
    h.ext.n_tiles = (int)sh.nt;
    h.ext.n_chunks = (int)sh.nc;
    h.ext.nb = (int)sh.nb;
    h.ext.nb_blocks = ((int)sh.nb + kScanPerBlock - 1) / kScanPerBlock;
    h.ext.n_members = 1;
    Seg sg{};
    sg.p0 = 0;
    sg.cap = sh.ng * kGroupSlots;
    sg.t0 = 0;
    sg.nt = sh.nt;
    sg.g0 = 0;
    sg.ng = sh.ng;
    sg.c0 = 0;
    sg.nc = sh.nc;
    sg.cl = sh.cl;
    sg.b0 = 0;
    sg.nb = sh.nb;
    sg.inv_vol = 1.0 / (p->r_out * p->r_out * p->r_out - 1.0);
    sg.ntilde = p->ntilde;
    sg.inv_ntilde = 1.0 / p->ntilde;
    sg.ion_density = p->ion_density;
    sg.q_surface0 = q_surface;
    sg.dt = p->dt;
    sg.r_out = p->r_out;
    sg.seed = p->seed;
    sg.probe_bc = p->probe_bc;
    sg.wall_bc = p->wall_bc;
    sg.n_steps = 1;
    sg.u_asy = reinterpret_cast<double *>(h.mdata);
    sg.qdiff = reinterpret_cast<double *>(h.mdata + kPoolUnit);
    sg.near_w = near_width(h.lo.tu, h.lo.fp32, h.lo.L, n);
    sg.one_carry = takes_one_carry(h.lo.tu, sh.ng) ? 1 : 0;
    (sg.one_carry ? h.ext.one_carry : h.ext.chunked) = true;
    sg.used = 1;
    Ctl ct{};
    ct.next_step = ct.step = 0;
    ct.records = (uint32_t)n;
    ct.n_live = (uint32_t)n;
    ct.q_surface = q_surface;
    hipStream_t s = (hipStream_t)hip_stream;
    const unsigned gSet = 16;
    const unsigned gN = (unsigned)((n + kBlock - 1) / kBlock);
    k_static_setup<<<gSet, kBlock, 0, s>>>(sg, ct, h.seg, h.ctl, h.tile_member, h.chunk_member, h.hist,
                                           const_cast<double *>(sg.u_asy), u_asy, (int)sh.nt,
                                           (int)sh.nc, h.lo.nb);
    k_static_pack<<<gN + kTableBlocks, kBlock, 0, s>>>(pos, (uint32_t)n, h.A, h.krec, h.hist,
                                                       sg.inv_vol, sg.nb, table_dst(&h, *p));
    // the field goes straight to the caller's array, by id
    h.Eout = E;
    h.Eid = nullptr;
    if (int rc = launch_step(&h, s, true, false, nullptr)) return rc;
    HIP_TRY(hipStreamSynchronize(s));
    return SIM_OK;
}

int sim_profile(sim_t *h, int64_t k, double *kernel_ms, int32_t n_kernels)
{
    int rc = check_handle(h);
    if (rc) return rc;
    if (k <= 0 || !kernel_ms) return fail(SIM_EINVAL, "k must be > 0 and kernel_ms non-NULL");
    for (const Member &m : h->members)
        if (m.used && m.step_host + k > m.seg.n_steps) return fail(SIM_ERANGE, "steps beyond n_steps");
    Marks marks;
    hipEvent_t *ev = marks.ev;
    for (int i = 0; i <= KN_COUNT; ++i)
        if (hipEventCreate(&ev[i]) != hipSuccess) return fail(SIM_EDEVICE, "hipEventCreate failed");
    std::vector<double> acc(KN_COUNT, 0.0);
    for (int64_t s = 0; s < k && rc == SIM_OK; ++s) {
        rc = launch_step(h, h->stream, false, !keys_in_push(h) || h->keys_needed, &marks);
        h->keys_needed = false;
        if (rc == SIM_OK && hipEventSynchronize(ev[KN_COUNT]) != hipSuccess)
            rc = fail(SIM_EDEVICE, "event sync failed");
        for (int i = 0; i < KN_COUNT && rc == SIM_OK; ++i) {
            float ms = 0.f;
            if (marks.ran[i] && hipEventElapsedTime(&ms, ev[i], ev[i + 1]) == hipSuccess) acc[i] += ms;
        }
        if (rc == SIM_OK)
            for (Member &m : h->members)
                if (m.used) m.step_host += 1;
    }
    for (int i = 0; i <= KN_COUNT; ++i) (void)hipEventDestroy(ev[i]);
    if (rc) return mark_failed(h, rc);
    for (int i = 0; i < KN_COUNT && i < n_kernels; ++i) kernel_ms[i] = acc[i] / (double)k;
    return SIM_OK;
}

int32_t sim_num_kernels(void) { return KN_COUNT; }

const char *sim_kernel_name(int32_t i)
{
    if (i < 0 || i >= KN_COUNT) return "";
    return kKernelNames[i];
}

int sim_info(sim_t *h, int64_t *n, int32_t *tile, int32_t *channels)
{
    int rc = check_handle(h);
    if (rc) return rc;
    if (n) *n = h->members.empty() || !h->members[0].used ? 0 : h->members[0].n;
    if (tile) *tile = kWave;
    if (channels) *channels = h->lo.C;
    return SIM_OK;
}

void sim_destroy(sim_t *h)
{
    if (!h) return;
    release(h);
    delete h;
}

const char *sim_strerror(int status)
{
    switch (status) {
    case SIM_OK: return "ok";
    case SIM_EINVAL: return "invalid argument";
    case SIM_ENOMEM: return "out of memory or over the memory limit";
    case SIM_ERANGE: return "index out of range";
    case SIM_ESTATE: return "invalid or failed handle";
    case SIM_EDEVICE: return "HIP runtime error";
    case SIM_BUSY: return "work still running";
    default: return "unknown status";
    }
}

const char *sim_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
